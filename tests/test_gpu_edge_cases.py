"""Calls at the edge of what the entry points take: staging areas that are just large enough, settings of extreme size, values that
are not finite, and what a call costs its own thread."""
import ctypes as C
import time

import numpy as np
import pytest
import torch

import synth_inputs as si

pytestmark = pytest.mark.gpu


def _ctx(cfg):
    from paper_2511_15618_amd import FlashMesh
    from paper_2511_15618_amd.binding import config_struct
    w = si.make_weights(cfg, 0)
    fm = FlashMesh(config_struct(cfg))
    fm.load_weights(si.pack_blob(cfg, w))
    return fm


@pytest.mark.parametrize("d,heads,mem,dtype", [(256, 4, 5461, "f32"), (64, 1, 26214, "bf16"), (192, 2, 7281, "f32")])
def test_static_prefill_takes_all_that_its_area_holds(d, heads, mem, dtype):
    """mem_len * d_model * (element size + 8) bytes, the largest memory below 16 MiB: the padding to whole key blocks does not count.
    The keys and values are those of the allocating call, bit for bit; one row more is refused."""
    esz = 4 if dtype == "f32" else 2
    assert mem * d * (esz + 8) <= 16 << 20 < (mem + 1) * d * (esz + 8)
    print("case static area", d, mem, dtype, flush=True)
    cfg = si.Config("static", d, heads, 32, 1, 1, 1, 1, 1, mem, dtype, 2, 2, 2, 0, 0)
    fm = _ctx(cfg)
    x = torch.from_numpy(si.make_memory(cfg, 0)).cuda()
    fm.prefill_condition(0, x)
    fm.prefill_condition_static(1, x)
    for block in range(cfg.n_layers):
        for a, b in zip(fm.debug_mem_kv(0, block), fm.debug_mem_kv(1, block)):
            assert np.array_equal(a, b) and np.abs(a).max() > 0, block
    more = cfg.replace(mem_len=mem + 1)
    fm = _ctx(more)
    y = torch.from_numpy(si.make_memory(more, 0)).cuda()
    assert fm.lib.fm_prefill_condition_static(fm.h, 0, C.c_void_p(y.data_ptr())) == -1


@pytest.mark.parametrize("d,heads,mem,dtype", [(64, 1, 1, "bf16"), (192, 2, 33, "f32"), (192, 3, 31, "bf16")])
def test_condition_memory_at_any_address(d, heads, mem, dtype):
    """A memory that is aligned to its elements alone, of 1 row or around a key block, 2 and 6 column tiles (no multiple of a workgroup's four)."""
    print("case memory address", d, mem, dtype, flush=True)
    cfg = si.Config("address", d, heads, 32, 1, 1, 1, 1, 1, mem, dtype, 2, 2, 2, 0, 0)
    fm = _ctx(cfg)
    x = torch.from_numpy(si.make_memory(cfg, 0)).cuda()
    y = torch.empty(x.numel() + 1, device="cuda")[1:].view(x.shape).copy_(x)
    assert x.data_ptr() % 16 == 0 and y.data_ptr() % 16 == 4
    fm.prefill_condition(0, x)
    fm.prefill_condition(1, y)
    for block in range(cfg.n_layers):
        for a, b in zip(fm.debug_mem_kv(0, block), fm.debug_mem_kv(1, block)):
            assert np.array_equal(a, b) and np.abs(a).max() > 0, block


@pytest.mark.parametrize("dtype,batch,temperature", [("f32", 1, 0.0), ("bf16", 1, 0.0), ("bf16", 2, 0.0), ("bf16", 1, 0.5)])
def test_steps_of_generate_are_those_of_the_calls(dtype, batch, temperature):
    """fm_generate writes no block for a step without drafts and commits one greedy sequence in the launch that chooses: the tokens and counts
    are those of separate calls, with drafts and without, over more steps than those that it times phase by phase."""
    cfg = si.Config("steps", 128, 2, 32, 1, 1, 1, 1, 1, 40, dtype, batch, 5, 2, 9, 9)
    for speculative in (False, True):
        print("case steps of generate", dtype, batch, temperature, speculative, flush=True)
        got = []
        for calls in (False, True):
            fm = _ctx(cfg)
            if temperature:
                fm.set_sampling(temperature, 7)
            for s in range(batch):
                fm.prefill_condition(s, torch.from_numpy(si.make_memory(cfg, s)).cuda())
            if calls:
                fm.set_budget(cfg.faces)
                tok, ln = fm.new_block()
                lg, acc = torch.zeros(batch, fm.block_max, fm.vocab, device="cuda"), torch.zeros_like(ln)
                lens = [[] for _ in range(batch)]
                for _ in range(9 * cfg.faces):
                    fm.draft(tok, ln)
                    if not speculative:
                        ln.clamp_(max=1)
                    fm.verify_block(tok, ln, lg, acc)
                    fm.commit(acc)
                    for s, a in enumerate(acc.tolist()):
                        if a:
                            lens[s].append(a)
                state = fm.read_state()
            out, n, st = fm.generate(cfg.faces, speculative)
            if not calls:
                hist = np.array([list(h) for h in st.acc_hist]).sum(0)
                state = fm.read_state()
                assert st.steps == st.tokens == 9 * cfg.faces if not speculative and batch == 1 else st.steps <= st.tokens
            else:
                hist = np.bincount([a for l in lens for a in l], minlength=32)
            got.append((out.cpu().numpy(), n.cpu().numpy(), hist, state[:, :5]))      # length, rows per level, main token, finished
        for a, b in zip(*got):
            assert np.array_equal(a, b)
        assert got[0][1].tolist() == [9 * cfg.faces] * batch


def test_a_step_without_drafts_forgets_the_sampled_ones():
    """fm_generate for one token, no drafts, behind an fm_draft: tokens of that draft in a block of the caller's are proposals with all their mass, as in a
    context that never drafted (the generator is keyed by position)."""
    cfg = si.Config("forget", 128, 2, 32, 1, 1, 1, 1, 1, 40, "bf16", 8, 5, 2, 9, 9)
    block, got = None, []
    for drafts in (True, False):
        print("case forgotten drafts", drafts, flush=True)
        fm = _ctx(cfg)
        fm.set_sampling(1.0, 7)
        for s in range(cfg.batch):
            fm.prefill_condition(s, torch.from_numpy(si.make_memory(cfg, s)).cuda())
        fm.set_budget(5)
        tok, ln = fm.new_block()
        lg, acc = torch.zeros(cfg.batch, fm.block_max, fm.vocab, device="cuda"), torch.zeros_like(ln)
        for _ in range(17):
            tok[:, 0] = torch.from_numpy(fm.read_state()[:, 3].astype(np.int32)).cuda()
            fm.verify_block(tok, ln.fill_(1), lg, acc)
            fm.commit(acc)
        if drafts:
            fm.draft(tok, ln)
            assert ln.min() > 2
            block = tok.clone()
        _, _, st = fm.generate(2, False)
        assert st.steps == 1
        fm.set_budget(5)
        block[:, 0] = torch.from_numpy(fm.read_state()[:, 3].astype(np.int32)).cuda()
        fm.verify_block(block, ln.fill_(3), lg, acc)
        got.append((acc.tolist(), lg[:, :3].cpu().numpy(), fm.read_state()[:, :3]))
    for a, b in zip(*got):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("hist", [1 << 30, (1 << 31) - 1])
def test_correct_stage_with_the_longest_histories(hist):
    """Steps recorded with the correct stage off are not replayed for it, however many historical vertices it looks at."""
    cfg = si.TEST_CONFIGS["t_f32_99"]
    print("case history", hist, flush=True)

    def labels(before):
        fm = _ctx(cfg)
        mems = [torch.from_numpy(si.make_memory(cfg, s)).cuda() for s in range(cfg.batch)]
        for n in before:
            for s, m in enumerate(mems):
                fm.prefill_condition(s, m)
            fm.set_correct(n)
            out, _, st = fm.generate(cfg.faces, True)
        return out.cpu(), st.hist(), fm.debug_draft(1), fm.debug_draft(2)

    got, want = labels([0, 0, hist]), labels([hist])
    assert np.allclose(want[2].sum(-1), 1, atol=1e-5)              # the label rows of a stage that is on
    assert torch.equal(got[0], want[0]) and got[1] == want[1]
    assert np.array_equal(got[2], want[2]) and np.array_equal(got[3], want[3])


def _small(name, d, heads, mem, dtype, batch):
    return si.Config(name, d, heads, 32, 1, 1, 1, 1, 2, mem, dtype, batch, 6, 2, 9, 9)


# keys of a memory in one split and in several, both verify paths, both storage types, two head widths
@pytest.mark.parametrize("bad", [float("nan"), float("inf")], ids=["nan", "inf"])
@pytest.mark.parametrize("cfg", [_small("f32", 128, 2, 24, "f32", 2), _small("f32_splits", 192, 2, 290, "f32", 2),
                                 _small("half", 128, 2, 40, "bf16", 3), _small("half_splits", 128, 2, 1001, "bf16", 2),
                                 _small("one_launch", 128, 2, 40, "bf16", 1), _small("one_launch_splits", 128, 2, 1001, "bf16", 1)],
                         ids=lambda c: c.name)
def test_memory_that_is_not_finite(cfg, bad):
    """A condition memory with one value that is not finite: the logits of its sequence show it and its rows are counted, the other
    sequences do not see it, and neither does the next mesh of the sequence, over caches that still hold the first one's rows."""
    print("case memory", cfg.name, bad, flush=True)
    mems = [torch.from_numpy(si.make_memory(cfg, s)).cuda() for s in range(cfg.batch)]
    broken = mems[0].clone()
    broken[cfg.mem_len // 2, 3] = bad

    def first_pass(fm, mem0):
        for s, m in enumerate([mem0] + mems[1:]):
            fm.prefill_condition(s, m)
        tok, ln = fm.new_block()
        tok[:] = torch.arange(fm.block_max, device="cuda", dtype=torch.int32)
        tok[:, 0] = cfg.bos
        ln[:] = fm.block_max
        acc = torch.zeros(cfg.batch, dtype=torch.int32, device="cuda")
        logits = torch.zeros(cfg.batch, fm.block_max, cfg.vocab, device="cuda")
        fm.verify_block(tok, ln, logits, acc)
        return logits.cpu()

    def mesh(fm, mem0):
        for s, m in enumerate([mem0] + mems[1:]):
            fm.prefill_condition(s, m)
        out, n, st = fm.generate(cfg.faces, True)
        assert n.tolist() == [9 * cfg.faces] * cfg.batch
        return out.cpu(), int(st.nonfinite_rows)

    fm = _ctx(cfg)
    want, (want_tok, healthy) = first_pass(fm, mems[0]), mesh(fm, mems[0])
    assert healthy == 0 and torch.isfinite(want).all()
    fm = _ctx(cfg)
    got, (tok, counted) = first_pass(fm, broken), mesh(fm, broken)
    assert not torch.isfinite(got[0]).any() and counted > 0
    assert torch.equal(got[1:], want[1:]) and torch.equal(tok[1:], want_tok[1:])
    assert torch.equal(first_pass(fm, mems[0]), want)
    tok, counted = mesh(fm, mems[0])
    assert counted == 0 and torch.equal(tok, want_tok)


@pytest.mark.parametrize("ban", [1, 0], ids=["to_the_budget", "to_eos"])
def test_generate_leaves_its_core_to_others(ban):
    """The thread that calls fm_generate sleeps while the device works: its CPU time stays below half of the call's time, where a thread
    that looks all the time has all of it (enqueueing the 30 launches of a step takes about 0.1 ms of its 0.8)."""
    cfg = si.Config("core", 512, 8, 64, 2, 2, 4, 4, 8, 1024, "bf16", 1, 60, 2, 9, 9, ban_specials=ban)
    print("case core", ban, flush=True)
    fm = _ctx(cfg)
    mem = torch.from_numpy(si.make_memory(cfg, 0)).cuda()
    shares = []
    for _ in range(3):
        fm.prefill_condition(0, mem)
        torch.cuda.synchronize()
        wall, cpu = time.perf_counter(), time.thread_time()
        _, _, st = fm.generate(cfg.faces, True)
        wall, cpu = time.perf_counter() - wall, time.thread_time() - cpu
        print(f"steps {st.steps}, {wall * 1e3:.1f} ms, {cpu * 1e3:.1f} ms of CPU time", flush=True)
        shares.append(cpu / wall)
    assert st.steps >= 20 and min(shares) < 0.5

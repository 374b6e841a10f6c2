"""The decode kernels (skinny GEMM, block attention, choice and merge, attention of the single-launch kernel) and the edge instance of the prefill kernel, at the sizes
where their tilings and launch rules change, against the CPU oracle."""
import numpy as np
import pytest
import torch

import synth_inputs as si

pytestmark = pytest.mark.gpu

# the bars of the lock-step tests (see parity_harness for how they carry over to probabilities)
TOL = {"f32": 1e-4, "bf16": 2e-2}


def _cfg(name, d, heads, mem, dtype, batch, faces, dc, m, n, bins=32, **kw):
    return si.Config(name, d, heads, bins, 1, 1, 1, 1, 2, mem, dtype, batch, faces, dc, m, n, **kw)


CASES = [
    # more than seven row tiles (13 x 9 rows): the tall tile, with a last row tile of 5 rows; memory one row past a tile
    _cfg("tall_rows", 192, 2, 257, "bf16", 13, 4, 2, 9, 9),
    # hidden rows of more than 64 and more than 128 K fragments, few and many workgroups (24 sets of heads, two row tiles)
    _cfg("long_k", 192, 3, 72, "bf16", 9, 6, 2, 9, 27, ffn_mult=12, hf_ffn_mult=12),
    _cfg("longest_k", 192, 2, 40, "bf16", 9, 6, 2, 9, 27, ffn_mult=22, hf_ffn_mult=22),
    # K between 32 and 64 fragments with many workgroups; a width that is no multiple of 128
    _cfg("mid_k", 384, 6, 300, "bf16", 3, 6, 2, 9, 27),
    _cfg("odd_width", 320, 5, 31, "bf16", 2, 4, 2, 9, 9, bins=45),
    # several splits of the memory's keys with one and two query tiles, every head width (last block partly filled)
    _cfg("splits_hd64", 128, 2, 1001, "bf16", 2, 6, 2, 9, 9),
    _cfg("splits_hd64_two", 128, 2, 1001, "bf16", 2, 6, 2, 15, 18),
    _cfg("splits_hd96", 192, 2, 700, "bf16", 2, 6, 2, 15, 18),
    _cfg("splits_hd128", 256, 2, 289, "bf16", 2, 6, 2, 15, 18),
    # the single-launch kernel: one split per group of four key blocks, the last group partly filled; two query tiles
    _cfg("one_launch_splits", 128, 2, 1001, "bf16", 1, 6, 2, 9, 9),
    _cfg("one_launch_two_tiles", 256, 4, 545, "bf16", 1, 6, 2, 15, 18),
    # its instances: the widths known to the compiler, and the general one (other widths, another hidden width), one and two row groups
    _cfg("one_launch_w512", 512, 8, 70, "bf16", 1, 3, 2, 9, 9, bins=45),
    _cfg("one_launch_w768", 768, 12, 33, "bf16", 1, 3, 2, 9, 9),
    _cfg("one_launch_w1024_two_tiles", 1024, 16, 40, "bf16", 1, 4, 17, 0, 0),
    _cfg("one_launch_w640_two_tiles", 640, 10, 70, "bf16", 1, 4, 2, 15, 18),
    _cfg("one_launch_w896", 896, 14, 40, "bf16", 1, 3, 2, 9, 9),
    _cfg("one_launch_hidden", 256, 4, 40, "bf16", 1, 4, 2, 9, 9, ffn_mult=8),
    _cfg("one_launch_widest_hidden", 128, 2, 40, "bf16", 1, 4, 2, 9, 9, ffn_mult=32),
    _cfg("one_launch_w256", 256, 4, 40, "bf16", 1, 4, 2, 9, 9),
    _cfg("one_launch_w512_two_tiles", 512, 8, 70, "bf16", 1, 4, 2, 15, 18),
    _cfg("one_launch_w1024", 1024, 16, 33, "bf16", 1, 3, 2, 9, 9),
    _cfg("one_launch_w768_two_tiles", 768, 12, 33, "bf16", 1, 4, 2, 9, 27),
    _cfg("one_launch_w128_two_tiles", 128, 2, 70, "bf16", 1, 4, 2, 15, 18),
    _cfg("one_launch_w384", 384, 6, 33, "bf16", 1, 3, 2, 9, 9),
    _cfg("one_launch_w384_two_tiles", 384, 6, 70, "bf16", 1, 4, 2, 9, 27),
    # a hidden width past what the single-launch kernel holds: the per-operator path
    _cfg("past_the_hidden", 256, 4, 40, "bf16", 1, 4, 2, 9, 9, ffn_mult=18),
    # more than 32 draft rows per sequence: two row sets of one attention launch
    _cfg("two_sets", 128, 2, 40, "bf16", 2, 8, 2, 27, 27),
    # fp32: tall tiles in the condition GEMM, K past one trip, splits, head widths
    _cfg("f32_tall", 128, 2, 131, "f32", 2, 6, 2, 9, 9),
    _cfg("f32_long_k", 320, 5, 33, "f32", 2, 4, 2, 9, 9, ffn_mult=5, hf_ffn_mult=5),
    _cfg("f32_splits_hd96", 192, 2, 290, "f32", 2, 6, 2, 15, 18),
    _cfg("f32_splits_hd128", 256, 2, 513, "f32", 1, 6, 2, 15, 18),
    # vocabulary past the registers of the draft softmax (2048 entries)
    _cfg("wide_vocab", 128, 2, 40, "bf16", 2, 4, 2, 9, 9, bins=2100),
]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_lockstep_where_tilings_change(cfg):
    from parity_harness import lockstep
    print("case", cfg.name, flush=True)
    rep, streams, fm = lockstep(cfg, cfg.faces, TOL[cfg.dtype], max_steps=12)
    print(rep, flush=True)
    assert rep.steps > 0 and fm.verify_path() == (cfg.name.startswith("one_launch"))


@pytest.mark.parametrize("name", ["t_f32_1815", "wide"])
def test_sampled_choice_over_wide_rows(name):
    """Draws from rows that are no whole number of waves, and past the registers of the draft softmax."""
    from parity_harness import lockstep
    cfg = CASES[-1].replace(name=name) if name == "wide" else si.TEST_CONFIGS[name].replace(n_bins=67)
    print("case", name, flush=True)
    rep, _, _ = lockstep(cfg, cfg.faces, TOL[cfg.dtype], max_steps=10, sampling=(0.8, 5))
    print(rep, flush=True)


@pytest.mark.parametrize("bins", [1280, 1281])
def test_sampled_choice_at_the_limit_of_the_kept_weights(bins):
    """Draws whose weights just fit a wave's registers (20 a lane), and one more."""
    from parity_harness import lockstep
    cfg = CASES[-1].replace(name="bins%d" % bins, n_bins=bins)
    print("case", cfg.name, flush=True)
    rep, _, _ = lockstep(cfg, cfg.faces, TOL[cfg.dtype], max_steps=8, sampling=(0.8, 5))
    print(rep, flush=True)


@pytest.mark.parametrize("hist", [64, 65, 100])
def test_correct_stage_over_more_vertices_than_a_wave(hist):
    """Historical vertices in one round of the wave, and in a second one; the longest blocks (9 points)."""
    from parity_harness import lockstep
    cfg = _cfg("hist%d" % hist, 128, 2, 24, "f32", 1, 36, 2, 9, 27, bins=64)
    print("case", cfg.name, flush=True)
    rep, streams, _ = lockstep(cfg, cfg.faces, TOL[cfg.dtype], correct_hist=hist)
    print(rep, flush=True)
    assert len(streams[0]) == 9 * cfg.faces and rep.corrected_blocks > 0


@pytest.mark.parametrize("d,heads,mem", [(128, 2, 1), (128, 2, 33), (192, 2, 255), (320, 5, 257), (384, 3, 511), (640, 5, 769)])
def test_condition_kv_at_tile_edges(d, heads, mem):
    """Memories and widths that are no whole 256-row tiles, every element against float64.  The bound: the memory rounded to half
    (2^-11 relative, the weights are exact), d products summed in fp32, one more rounding to half."""
    from oracle.hourglass import Model
    from paper_2511_15618_amd import FlashMesh
    from paper_2511_15618_amd.binding import config_struct
    cfg = _cfg("edges", d, heads, mem, "bf16", 2, 2, 2, 0, 0)
    print("case", d, heads, mem, flush=True)
    w = si.make_weights(cfg, 0)
    model, fm = Model(cfg, w), FlashMesh(config_struct(cfg))
    fm.load_weights(si.pack_blob(cfg, w))
    mems = [si.make_memory(cfg, s) for s in range(2)]
    for s in range(2):
        fm.prefill_condition(s, torch.from_numpy(mems[s]).cuda())
    blocks = [f"{st}.{i}." for st in si.STACKS for i in range(model.layers[st])]
    for s in range(2):
        for b, pfx in enumerate(blocks):
            for ref, dev, wn in zip(model.mem_kv(pfx, mems[s]), fm.debug_mem_kv(s, b), ("ck", "cv")):
                ref = ref.reshape(mem, d)
                mag = np.abs(np.asarray(mems[s], np.float64)) @ np.abs(model.w[pfx + wn]).T
                bound = 1.05 * ((2.0 ** -11 + (d + 2) * 2.0 ** -24) * mag + 2.0 ** -11 * np.abs(ref)) + 1e-30
                assert (np.abs(dev - ref) <= bound).all(), (s, pfx, wn)


@pytest.mark.parametrize("name", ["t_f32_99", "t_bf16_99"])
def test_recorded_steps_follow_buffers_and_settings(name):
    """Steps are replayed as recorded launches: more block buffers than a context keeps recordings for, settings that change
    between steps and whole-mesh calls of several lengths give what the first, unrecorded pass over the same mesh gave."""
    from paper_2511_15618_amd import FlashMesh
    from paper_2511_15618_amd.binding import config_struct
    cfg = si.TEST_CONFIGS[name]
    fm = FlashMesh(config_struct(cfg))
    fm.load_weights(si.pack_blob(cfg, si.make_weights(cfg, 0)))
    mems = [torch.from_numpy(si.make_memory(cfg, s)).cuda() for s in range(cfg.batch)]

    def begin():
        for s, mem in enumerate(mems):
            fm.prefill_condition(s, mem)

    def mesh(faces):
        begin()
        tok, n, _ = fm.generate(faces, True)
        return [tok[s, :int(n[s])].tolist() for s in range(cfg.batch)]

    def stepped(faces, buffers):
        begin()
        fm.set_budget(faces)
        acc = torch.zeros(cfg.batch, dtype=torch.int32, device="cuda")
        out = [[] for _ in range(cfg.batch)]
        for i in range(9 * faces):
            tok, ln = buffers[i % len(buffers)]
            fm.draft(tok, ln)
            fm.verify_block(tok, ln, None, acc)
            blocks, took = tok.tolist(), acc.tolist()
            fm.commit(acc)
            state = fm.read_state()
            for s in range(cfg.batch):
                if took[s]:
                    out[s] += blocks[s][1:took[s]] + [int(state[s, 3])]
            if state[:, 4].all():
                break
        return out

    whole = mesh(cfg.faces)
    assert [len(x) for x in whole] == [9 * cfg.faces] * cfg.batch
    many = [fm.new_block() for _ in range(11)]
    for buffers in (many[:1], many, many[:2]):
        assert stepped(cfg.faces, buffers) == whole
    for faces in (1, 2, cfg.faces):
        assert mesh(faces) == [x[:9 * faces] for x in whole]
    fm.set_sampling(0.9, 4)
    drawn = mesh(cfg.faces)
    assert stepped(cfg.faces, many[:2]) == drawn and drawn != whole
    fm.set_sampling(0.0, 0)
    assert mesh(cfg.faces) == whole and stepped(cfg.faces, many[:2]) == whole


@pytest.mark.parametrize("drafts", ["native", "none"])
@pytest.mark.parametrize("m,n", [(9, 9), (15, 18)])
def test_single_launch_past_the_first_group_of_keys(m, n, drafts):
    """The single-launch kernel from a context that one split holds (128 keys, no merge) to one that two do, one and two row groups, blocks and
    token by token (passes whose vertex and face levels have no row)."""
    from parity_harness import lockstep
    cfg = _cfg("one_launch_parts%d%s" % (n, drafts), 128, 2, 60, "bf16", 1, 17, 2, m, n)
    print("case", cfg.name, flush=True)
    rep, streams, fm = lockstep(cfg, cfg.faces, TOL[cfg.dtype], drafts=drafts)
    print(rep, flush=True)
    assert len(streams[0]) == 9 * cfg.faces > 128 + 18 and fm.verify_path() == 1


@pytest.mark.parametrize("dtype,batch", [("f32", 1), ("bf16", 2)])
def test_passes_whose_levels_have_no_row(dtype, batch):
    """One launch per operator, token by token: two passes in three begin no vertex, eight in nine no face."""
    from parity_harness import lockstep
    cfg = _cfg("no_rows_%s%d" % (dtype, batch), 128, 2, 60, dtype, batch, 4, 2, 9, 9)
    print("case", cfg.name, flush=True)
    rep, streams, fm = lockstep(cfg, cfg.faces, TOL[dtype], drafts="none")
    print(rep, flush=True)
    assert rep.steps == 9 * cfg.faces and fm.verify_path() == 0


@pytest.mark.parametrize("d,heads,dtype,batch", [(1152, 18, "bf16", 2), (2112, 33, "bf16", 1), (1088, 17, "f32", 1), (128, 2, "bf16", 17)])
def test_draft_rows_normed_by_their_gemms(d, heads, dtype, batch):
    """The norms of the draft heads inside their GEMMs with eight waves, past the widths that take them (half 2048, fp32 1024), and for more than one
    row tile per head (the output head's rows then are too many)."""
    from parity_harness import lockstep
    cfg = _cfg("draft_rows%d%s" % (d, dtype), d, heads, 24, dtype, batch, 2, 2, 9, 9)
    print("case", cfg.name, flush=True)
    rep, streams, fm = lockstep(cfg, cfg.faces, TOL[dtype], max_steps=6)
    print(rep, flush=True)
    assert rep.dist_rows > 0


@pytest.mark.parametrize("d,heads,dtype,batch", [(128, 2, "bf16", 1), (1152, 18, "bf16", 1), (128, 2, "bf16", 17), (128, 2, "f32", 1)])
def test_draft_rows_past_the_range_of_half(d, heads, dtype, batch):
    """The linear layers of the SP heads 2^16 times as large: their outputs, which the HF blocks and the output head norm, have elements past 65504 while the
    weights stay below it.  What a norm hands on is of order 1 whatever the row, so the bars on the draft distributions are the usual ones, for
    norms inside the GEMMs (four and eight waves) and, at 17 sequences, outside."""
    from parity_harness import lockstep, make_pair
    cfg = _cfg("large_rows%d%s" % (d, dtype), d, heads, 2, dtype, batch, 2, 2, 9, 9)
    print("case", cfg.name, batch, flush=True)

    def enlarge(w):
        for name in w:
            if name.startswith("sp.") and name.endswith(".lin"):
                w[name] = w[name] * np.float32(65536)
                assert np.abs(w[name]).max() < 65504
    pair = make_pair(cfg, edit_weights=enlarge)
    rep, streams, fm = lockstep(cfg, cfg.faces, TOL[dtype], max_steps=6, pair=pair)
    print(rep, flush=True)
    assert rep.dist_rows > 0


@pytest.mark.parametrize("mem,batch", [(512, 2), (513, 2), (500, 16), (500, 17)])
def test_fp32_attention_waves(mem, batch):
    """Two heads over the memory: two waves a workgroup for 16 key blocks, four for one block more and where two would give more than 256 workgroups."""
    from parity_harness import lockstep
    cfg = _cfg("f32_waves%d_%d" % (mem, batch), 128, 2, mem, "f32", batch, 2, 2, 9, 9)
    print("case", cfg.name, flush=True)
    rep, streams, fm = lockstep(cfg, cfg.faces, TOL["f32"], max_steps=4)
    print(rep, flush=True)
    assert rep.steps > 0 and fm.verify_path() == 0


@pytest.mark.parametrize("d,heads,mem,batch,blocks,dc,m,n", [(768, 8, 770, 3, 1, 2, 9, 9), (768, 12, 770, 3, 1, 17, 0, 0), (1024, 8, 860, 2, 1, 17, 0, 0)])
def test_memory_past_the_caches(d, heads, mem, batch, blocks, dc, m, n):
    """Keys and values as non-temporal loads, just past the line of 7 MB a block: heads of 96, 64 and 128, one and two query tiles."""
    from parity_harness import lockstep
    assert 7e6 <= 4 * batch * mem * d < 7.2e6
    cfg = _cfg("once%d_%d" % (d, heads), d, heads, mem, "bf16", batch, 2, dc, m, n).replace(l_face=blocks)
    print("case", cfg.name, flush=True)
    rep, streams, fm = lockstep(cfg, cfg.faces, TOL[cfg.dtype], max_steps=3)
    print(rep, flush=True)
    assert rep.steps == 3 and fm.verify_path() == 0


@pytest.mark.parametrize("faces,m,n", [(53, 9, 9), (54, 9, 9), (54, 15, 18)])
def test_caches_on_both_sides_of_the_line(faces, m, n):
    """13 sequences with caches of 4.8 and 5.1 MB at the coordinate level, a third of it at the vertex level, 0.6 MB of memory a block: coordinate blocks on
    both sides of the line of 5 MB, SP heads (all levels) past it, vertex blocks and memory below; one and two query tiles."""
    from parity_harness import lockstep
    cfg = _cfg("line%d_%d" % (faces, n), 192, 3, 40, "bf16", 13, faces, 2, m, n)
    assert (4 * 13 * -(-cfg.max_tokens // 32) * 32 * 192 >= 5e6) == (faces == 54)
    print("case", cfg.name, flush=True)
    rep, streams, fm = lockstep(cfg, cfg.faces, TOL[cfg.dtype], max_steps=4)
    print(rep, flush=True)
    assert rep.steps == 4 and fm.verify_path() == 0


@pytest.mark.parametrize("d,heads,mem", [(768, 8, 16384), (1024, 8, 12288), (1024, 16, 12288)])
def test_condition_kv_past_the_caches(d, heads, mem):
    """Five blocks of 50 MB lie below the line from which the prefill stores its results past the caches, six above: the leading blocks are the same bits."""
    from paper_2511_15618_amd import FlashMesh
    from paper_2511_15618_amd.binding import config_struct
    got = []
    for blocks in (1, 2):
        cfg = _cfg("past", d, heads, mem, "bf16", 1, 1, 2, 0, 0).replace(l_face=blocks)
        print("case prefill past the caches", d, heads, 4 + blocks, flush=True)
        assert ((4 + blocks) * 4 * mem * d > 256e6) == (blocks == 2)
        fm = FlashMesh(config_struct(cfg))
        fm.load_weights(si.pack_blob(cfg, si.make_weights(cfg, 0)))
        fm.prefill_condition(0, torch.from_numpy(si.make_memory(cfg, 0)).cuda())
        got.append([fm.debug_mem_kv(0, b) for b in range(3)])
        del fm
    for few, many in zip(*got):
        for a, b in zip(few, many):
            assert np.array_equal(a, b) and np.abs(a).max() > 0

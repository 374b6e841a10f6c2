"""The arithmetic of the verify pass to the last bit: rows of logits against those on record (tests/golden/logit_rows.txt).

A kernel that is only arranged differently gives the same bits; one that rounds elsewhere (another GELU, another reciprocal root, sums in another order) does not,
and shows here instead of as a few parts in 10^4 that every tolerance lets pass.  Whoever changes the arithmetic on purpose measures its error against float64
and writes the record anew (`record()`), in the commit that says why."""
import os
import zlib

import numpy as np
import pytest
import torch

import synth_inputs as si

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "logit_rows.txt")


def _cfg(name, d, heads, mem, dtype, batch, dc, m, n):
    return si.Config(name, d, heads, 32, 1, 1, 1, 1, 2, mem, dtype, batch, 12, dc, m, n)


CASES = [
    _cfg("one_launch", 256, 4, 100, "bf16", 1, 2, 9, 9),
    _cfg("one_launch_any_width", 128, 2, 40, "bf16", 1, 2, 9, 9),
    _cfg("one_launch_two_groups", 256, 4, 100, "bf16", 1, 2, 15, 18),
    _cfg("per_operator_hd96", 192, 2, 300, "bf16", 3, 2, 9, 9),
    _cfg("per_operator_hd128", 256, 2, 70, "bf16", 1, 2, 15, 18),
    _cfg("per_operator_f32", 128, 2, 60, "f32", 2, 3, 0, 0),
]


def rows(cfg):
    """'case pass sequence row crc32' of three passes over given tokens."""
    from paper_2511_15618_amd import FlashMesh
    from paper_2511_15618_amd.binding import config_struct
    fm = FlashMesh(config_struct(cfg))
    fm.load_weights(si.pack_blob(cfg, si.make_weights(cfg, 0, gain_jitter=0.25)))
    for s in range(cfg.batch):
        fm.prefill_condition(s, torch.from_numpy(si.make_memory(cfg, s)).cuda())
    fm.set_budget(cfg.faces)
    B = fm.block_max
    given = np.random.default_rng(7).integers(0, cfg.n_bins, (3, cfg.batch, B), dtype=np.int32)
    given[0, :, 0] = cfg.bos
    tok, ln = fm.new_block()
    lg, acc = torch.zeros(cfg.batch, B, cfg.vocab, device="cuda"), torch.zeros_like(ln)
    out = []
    for i in range(3):
        tok.copy_(torch.from_numpy(given[i]))
        ln.fill_(B)
        fm.verify_block(tok, ln, lg, acc)
        fm.commit(ln)
        h = lg.cpu().numpy()
        assert np.isfinite(h).all() and np.abs(h).max() > 0.1
        out += ["%s %d %d %d %08x" % (cfg.name, i, s, r, zlib.crc32(h[s, r].tobytes())) for s in range(cfg.batch) for r in range(B)]
    return out


def record():
    with open(GOLDEN, "w") as f:
        for cfg in CASES:
            f.write("\n".join(rows(cfg)) + "\n")


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_logits_keep_their_bits(cfg):
    print("case", cfg.name, flush=True)
    want = [l for l in open(GOLDEN).read().splitlines() if l.split()[0] == cfg.name]
    got = rows(cfg)
    assert len(want) == 3 * cfg.batch * cfg.block_max
    assert got == want, "%d of %d rows differ" % (sum(a != b for a, b in zip(got, want)), len(want))

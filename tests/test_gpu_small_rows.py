"""Rows of few units and batches of many rows: the kernels that pack several
rows into a workgroup or wavefront, against the oracle, at the edges of their
tiles and dispatch rules."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import dev, host, read_col, tree_consistent
from paper_2609_24456_amd import conduit as cd

pytestmark = pytest.mark.gpu

MEAN, STD = (0.485, 0.456, 0.406, 0.5), (0.229, 0.224, 0.225, 0.7)
XF_OUT = {cd.XF_NONE: torch.uint8, cd.XF_U8_F32: torch.float32, cd.XF_U8_BF16_NORM: torch.int16}


# (planes, 4-byte units per plane, transform, rows, source offset in bytes): one
# unit and one row; rows on and off 16 bytes; one, two and four units per lane
# with remainders; the largest bf16 frame of the flat kernel and the next one;
# several tiles per workgroup with the bf16 table
@pytest.mark.parametrize("planes,units,kind,n,offset", [
    (1, 1, cd.XF_NONE, 1, 0), (1, 3, cd.XF_NONE, 257, 0), (1, 12, cd.XF_NONE, 4097, 0), (1, 12, cd.XF_NONE, 85, 4),
    (1, 130, cd.XF_NONE, 4500, 0), (1, 301, cd.XF_NONE, 4001, 0), (1, 512, cd.XF_U8_F32, 2049, 4),
    (1, 513, cd.XF_NONE, 33, 0), (3, 1764, cd.XF_U8_F32, 5, 0), (1, 2048, cd.XF_NONE, 1111, 8),
    (1, 1024, cd.XF_U8_BF16_NORM, 4500, 0), (1, 1025, cd.XF_U8_BF16_NORM, 70, 0), (4, 3, cd.XF_U8_BF16_NORM, 3000, 4)])
def test_minibatch_flat_rows(planes, units, kind, n, offset):
    print(f"flat rows planes={planes} units={units} kind={kind} n={n} offset={offset}", flush=True)
    rng = np.random.default_rng(units * 7 + n)
    row, n_src = planes * units * 4, n + 13
    src = rng.integers(0, 256, (n_src, row), dtype=np.uint8)
    buf = torch.empty(n_src * row + offset, dtype=torch.uint8, device="cuda")
    buf[offset:].copy_(torch.from_numpy(src.reshape(-1)))
    cols = [rng.standard_normal(n_src).astype(np.float32) for _ in range(3)]
    perm = rng.permutation(n_src)[:n]
    xf = cd.transform(kind, MEAN[:planes], STD[:planes]) if kind == cd.XF_U8_BF16_NORM else cd.transform(kind)
    want = oracle.rows(src.reshape(n_src, planes, units * 4), perm, kind, MEAN[:planes], STD[:planes])
    bad = perm.copy()
    bad[::50], bad[n // 2] = n_src, -1
    for idx, ok in ((perm, np.ones(n, bool)), (bad, (bad >= 0) & (bad < n_src))):
        out = torch.full((n, row), 9, dtype=XF_OUT[kind], device="cuda")
        cols_out = [torch.full((n,), np.nan, device="cuda") for _ in cols]
        cd.conduit_minibatch_gather(buf[offset:], row, n_src, dev(idx), xf, out, [dev(c) for c in cols], cols_out)
        assert cd.conduit_sync_check() == (cd.OK if ok.all() else cd.ESTATE)
        cd.conduit_clear_error()
        got = host(out).reshape(n, -1).view(np.uint8)
        w = np.ascontiguousarray(want.reshape(n, -1)).view(np.uint8)
        assert np.array_equal(got[ok], w[ok]) and not got[~ok].any()
        for c, o in zip(cols, cols_out):
            assert np.array_equal(host(o)[ok], c[idx[ok]]) and not host(o)[~ok].any()


# update lists around the split (2,048), with the last pass partial and whole
# (4 and 8 entries per lane), several passes, repeats throughout, indices out of
# range, and lists whose slots all fall to one of the 64 workgroups (more than
# its lanes take at once), alone and with an ingest that evicts some of them
@pytest.mark.parametrize("n,skew,m", [(2047, False, 0), (2048, False, 5), (4096, True, 0), (4097, False, 300),
                                      (8191, True, 300), (8192, False, 0), (20000, True, 64), (20000, False, 300)])
def test_long_update_lists(n, skew, m):
    print(f"long update list n={n} skew={skew} ingest={m}", flush=True)
    rng = np.random.default_rng(n + m)
    cap = 70_000
    prio = synth.quantise_priority(rng.lognormal(0, 1, cap + 700))
    buf = cd.ReplayBuffer(cap, (1,), torch.float32, action_bytes=0)
    orc = oracle.Replay(cap, (1,), np.float32, act_bytes=0)
    for a, b in ((0, cap), (cap, cap + 700)):
        obs = np.zeros((b - a, 1), np.float32)
        buf.ingest(dev(obs), prio=dev(prio[a:b]))
        orc.ingest(b - a, obs=obs, prio=prio[a:b])
    slots = np.arange(cap)
    if skew:
        slots = slots[((slots ^ (slots >> 6) ^ (slots >> 12)) & 63) == 0]
    for it in range(2):
        idx = rng.choice(slots, n)
        idx[n // 3::3] = rng.choice(idx[:50], len(idx[n // 3::3]))  # repeats
        new = synth.quantise_priority(rng.lognormal(0, 2, n))
        new[::97] = 0
        bad = it == 1
        sent = idx.copy()
        if bad:
            sent[5], sent[-1] = cap, -1
        keep = (sent >= 0) & (sent < cap)
        if m:
            rows = np.zeros((m, 1), np.float32)
            buf.update_ingest(dev(sent), dev(new), dev(rows))
        else:
            buf.update(dev(sent), dev(new))
        assert buf.sync_check() == (cd.ESTATE if bad else cd.OK), cd.last_error()
        buf.clear_error()
        orc.update(idx[keep], new[keep])
        if m:
            orc.ingest(m, obs=rows)
        assert np.array_equal(read_col(buf, cd.COL_LEAVES, cap * 4, np.uint32), orc.leaf), it
        assert read_col(buf, cd.COL_MAX_PRIO, 4, np.uint32)[0] == orc.max_prio
        tree_consistent(buf, cap)
    buf.close()

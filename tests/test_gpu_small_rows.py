"""Rows of few units and batches of many rows: the kernels that pack several
rows into a workgroup or wavefront, against the oracle, at the edges of their
tiles and dispatch rules."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import assert_gae_close, assert_weights_close, dev, host, read_col, tree_consistent
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


# frames to fp32 out of sources around the size from which they take the item
# kernels (256 MiB), filling their items (1,764 of 1,792 units) and not (1,300)
@pytest.mark.parametrize("units,n", [(1764, 33), (1764, 1500), (1300, 70)])
@pytest.mark.parametrize("beyond", [False, True])
def test_minibatch_source_sizes(units, n, beyond):
    print(f"source sizes units={units} n={n} beyond={beyond}", flush=True)
    n_src = (256 << 20) // (units * 4) + (1 if beyond else 0)
    g = torch.Generator(device="cuda")
    g.manual_seed(units + n)
    src = torch.randint(-2 ** 31, 2 ** 31, (n_src, units), generator=g, device="cuda", dtype=torch.int32).view(torch.uint8)
    perm = torch.randint(0, n_src, (n,), generator=g, device="cuda")
    perm[0], perm[-1] = n_src - 1, 0
    out = torch.full((n, units * 4), 9.0, device="cuda")
    cd.conduit_minibatch_gather(src, units * 4, n_src, perm, cd.transform(cd.XF_U8_F32), out)
    assert cd.conduit_sync_check() == cd.OK, cd.last_error()
    assert np.array_equal(host(out), host(src[perm]).astype(np.float32) / np.float32(255))


# rows of 4-byte units around half an item (896 units), into outputs around 128 MiB
@pytest.mark.parametrize("units", [895, 897])
@pytest.mark.parametrize("beyond", [False, True])
def test_minibatch_wide_vectors(units, beyond):
    print(f"wide vectors units={units} beyond={beyond}", flush=True)
    n = (128 << 20) // (units * 4) + (1 if beyond else 0)
    g = torch.Generator(device="cuda")
    g.manual_seed(units)
    src = torch.randint(-2 ** 31, 2 ** 31, (n + 7, units), generator=g, device="cuda", dtype=torch.int32)
    perm = torch.randperm(n + 7, generator=g, device="cuda")[:n]
    out = torch.zeros((n, units), dtype=torch.int32, device="cuda")
    cd.conduit_minibatch_gather(src, units * 4, n + 7, perm, cd.transform(cd.XF_NONE), out)
    assert cd.conduit_sync_check() == cd.OK, cd.last_error()
    assert torch.equal(out, src[perm])


# columns alone: rows of 0 bytes, with and without an output pointer, under every transform
@pytest.mark.parametrize("kind", [cd.XF_NONE, cd.XF_U8_F32, cd.XF_U8_BF16_NORM])
@pytest.mark.parametrize("pointer", [False, True])
def test_minibatch_columns_alone(kind, pointer):
    print(f"columns alone kind={kind} pointer={pointer}", flush=True)
    rng = np.random.default_rng(kind)
    cols = [rng.standard_normal(40).astype(np.float32) for _ in range(2)]
    perm = rng.permutation(40)[:33]
    xf = cd.transform(kind, MEAN[:3], STD[:3]) if kind == cd.XF_U8_BF16_NORM else cd.transform(kind)
    rows = torch.full((16,), 9, dtype=torch.uint8, device="cuda") if pointer else None
    cols_out = [torch.full((33,), np.nan, device="cuda") for _ in cols]
    cd.conduit_minibatch_gather(rows, 0, 40, dev(perm), xf, rows, [dev(c) for c in cols], cols_out)
    assert cd.conduit_sync_check() == cd.OK, cd.last_error()
    for c, o in zip(cols, cols_out):
        assert np.array_equal(host(o), c[perm])
    assert rows is None or (host(rows) == 9).all()


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


# rows of few units through sample + gather: one unit; the largest row a
# wavefront takes (256 units) and the next one; stacks; every transform; batches
# around the ticket's limit (1,024), the one-workgroup weights' (2,048) and a
# partial last workgroup; n-step targets with them; both weight normalisations
@pytest.mark.parametrize("shape,K,kind,B,norm", [
    ((1, 4), 1, cd.XF_NONE, 1, 0), ((1, 1020), 1, cd.XF_NONE, 1024, 0), ((1, 1024), 1, cd.XF_U8_F32, 1025, 0),
    ((1, 1028), 1, cd.XF_NONE, 1025, 0), ((1, 48), 3, cd.XF_NONE, 2048, 1), ((1, 256), 4, cd.XF_U8_F32, 2049, 0),
    ((3, 80), 4, cd.XF_U8_BF16_NORM, 300, 1), ((2, 128), 4, cd.XF_U8_BF16_NORM, 2503, 1),
    ((1, 4096), 1, cd.XF_NONE, 1024, 1), ((1, 4112), 1, cd.XF_NONE, 1100, 0),
    # larger rows of small batches: one, two and four workgroups per sample, around the last batch of each
    ((1, 7056), 4, cd.XF_U8_F32, 60, 0), ((1, 10000), 4, cd.XF_U8_BF16_NORM, 40, 1), ((1, 7056), 4, cd.XF_NONE, 256, 0),
    ((1, 10000), 4, cd.XF_U8_F32, 64, 0), ((1, 10000), 4, cd.XF_U8_F32, 65, 1), ((1, 7056), 4, cd.XF_U8_F32, 128, 0),
    ((1, 7056), 4, cd.XF_U8_F32, 129, 0), ((1, 7056), 4, cd.XF_U8_BF16_NORM, 64, 0), ((3, 3920), 1, cd.XF_U8_BF16_NORM, 33, 0),
    # single frames that fill their items, of a batch beyond the one-launch kernels
    ((1, 7056), 1, cd.XF_U8_F32, 1100, 1), ((3, 20000), 1, cd.XF_U8_F32, 40, 0)])
def test_sample_gather_small_rows(shape, K, kind, B, norm):
    print(f"small rows shape={shape} K={K} kind={kind} B={B} norm={norm}", flush=True)
    rng = np.random.default_rng(B + K)
    cap, n, act = 900, 1300, 70  # the ring wraps; more scalar units than a wavefront has lanes
    row = int(np.prod(shape))
    done = (rng.random(n) < 0.1).astype(np.uint8)
    episode, step = synth.episodes_from_done(done)
    obs = rng.integers(0, 256, (n, row), dtype=np.uint8)
    reward = rng.standard_normal(n).astype(np.float32)
    action = rng.integers(0, 256, (n, act), dtype=np.uint8)
    prio = synth.quantise_priority(rng.lognormal(0, 1, n))
    buf = cd.ReplayBuffer(cap, shape, torch.uint8, frame_stack=K, action_bytes=act, weight_norm=norm)
    store = np.zeros((cap, row), np.uint8)
    orc = oracle.Replay(cap, shape, np.uint8, act_bytes=act, frame_stack=K, obs_storage=store)
    for a, b in ((0, 700), (700, n)):
        buf.ingest(dev(obs[a:b].reshape((b - a,) + shape)), action=dev(action[a:b]), reward=dev(reward[a:b]),
                   done=dev(done[a:b]), episode_id=dev(episode[a:b]), step=dev(step[a:b]), prio=dev(prio[a:b]))
        orc.ingest(b - a, obs=obs[a:b], action=action[a:b], reward=reward[a:b], done=done[a:b], episode=episode[a:b],
                   step=step[a:b], prio=prio[a:b])
    planes = shape[0]
    xf = cd.transform(kind, MEAN[:planes], STD[:planes]) if kind == cd.XF_U8_BF16_NORM else cd.transform(kind)
    new = lambda: torch.full((B, K) + shape, 7, dtype=XF_OUT[kind], device="cuda")  # noqa: E731
    bits = lambda x: np.ascontiguousarray(x).reshape(-1).view(np.uint8)  # noqa: E731
    for nstep in (0, 3, 0):
        u = synth.uniforms(rng, B)
        out, nxt = new(), new()
        o_act = torch.zeros((B, act), dtype=torch.uint8, device="cuda")
        o_rew, o_done = torch.zeros(B, device="cuda"), torch.zeros(B, dtype=torch.uint8, device="cuda")
        o_idx, o_w = orc.sample(u, buffer_norm=bool(norm))
        if nstep:
            idx, w, ni, ret, disc, valid = buf.sample_gather_nstep(dev(u), xf, nstep, 0.9, next_obs=nxt, obs=out,
                                                                   action=o_act, reward=o_rew, done=o_done)
            want = orc.nstep(o_idx, nstep, 0.9)
            assert np.array_equal(host(ni), want[0])
            assert np.allclose(host(ret), want[1], rtol=2.0 ** -23, atol=0)  # fp64 sums rounded to fp32 once
            assert np.array_equal(host(valid), want[3])
            has = np.flatnonzero(want[0] >= 0)
            stacks = orc.gather(want[0][has], kind, MEAN[:planes], STD[:planes])[0]
            assert np.array_equal(bits(host(nxt)[has]), bits(stacks))
            assert not host(nxt)[want[0] < 0].any()
        else:
            idx, w = buf.sample_gather(dev(u), xf, obs=out, action=o_act, reward=o_rew, done=o_done)
        assert np.array_equal(host(idx), o_idx)
        assert_weights_close(host(w), o_w)
        w_obs, w_act, w_rew, w_done = orc.gather(o_idx, kind, MEAN[:planes], STD[:planes])
        assert np.array_equal(bits(host(out)), bits(w_obs))
        assert np.array_equal(host(o_act).reshape(w_act.shape), w_act)
        assert np.array_equal(host(o_rew), w_rew) and np.array_equal(host(o_done), w_done)
        idx2, w2 = buf.sample(dev(u))
        assert np.array_equal(host(idx2), o_idx)
        assert_weights_close(host(w2), o_w)
    assert buf.sync_check() == cd.OK, cd.last_error()
    buf.close()


# the one-launch update + ingest of variable-length rows against the two calls
# (which other tests hold against the oracle): evicted slots among the updates, a
# wrap, rows of 0 to 5 elements and of a whole slot, too long and at bad offsets,
# short and long update lists, with and without log-probabilities and priorities
@pytest.mark.parametrize("max_len,n_update,aux,given", [(8, 40, True, False), (8, 2300, False, True),
                                                        (5000, 300, True, True), (4100, 2048, True, False)])
def test_update_ingest_ragged_rows(max_len, n_update, aux, given):
    print(f"ragged update_ingest max_len={max_len} n_update={n_update}", flush=True)
    rng = np.random.default_rng(max_len + n_update)
    cap, n = 300, 130
    bufs = [cd.ReplayBuffer(cap, (max_len,), torch.int32, ragged=True, aux_elem_bytes=4 if aux else 0) for _ in range(2)]
    for it in range(4):
        length = rng.integers(0, max_len + 1, n)
        length[:8] = [0, 1, 2, 3, 4, 5, max_len, max_len]
        bad = it == 3
        if bad:
            length[20] = max_len + 3  # stored truncated
        offsets = np.concatenate([[0], np.cumsum(length)])
        total = int(offsets[-1])
        if bad:  # beyond the source's end and before its start: both rows beside each are stored empty
            offsets[40], offsets[60] = total + 9, -1
            length[[39, 40, 59, 60]] = 0
        tok = rng.integers(0, 1 << 30, total).astype(np.int32)
        rows = dict(offsets=dev(offsets), action=dev(rng.integers(0, 256, (n, 4), dtype=np.uint8)),
                    reward=dev(rng.standard_normal(n).astype(np.float32)))
        if aux:
            rows["aux"] = dev(rng.standard_normal(total).astype(np.float32))
        if given:
            rows["prio"] = dev(synth.quantise_priority(rng.lognormal(0, 1, n)))
        size = min(cap, it * n)
        idx = dev(rng.integers(0, max(size, 1), n_update))
        prio = dev(synth.quantise_priority(rng.lognormal(0, 2, n_update)))
        if size:
            bufs[0].update_ingest(idx, prio, dev(tok), **rows)
            bufs[1].update(idx, prio)
        else:
            bufs[0].ingest(dev(tok), **rows)
        bufs[1].ingest(dev(tok), **rows)
        assert [b.sync_check() for b in bufs] == [cd.ESTATE if bad else cd.OK] * 2
        for b in bufs:
            b.clear_error()
        info = bufs[0].info()
        cols = [(cd.COL_LENGTH, cap * 4), (cd.COL_ACTION, cap * 4), (cd.COL_REWARD, cap * 4), (cd.COL_LEAVES, cap * 4),
                (cd.COL_MAX_PRIO, 4)]
        a, b = ([read_col(x, c, k, np.uint8) for c, k in cols] for x in bufs)
        lens = a[0].view(np.int32)[:min(cap, (it + 1) * n)]
        live = np.arange(max_len)[None, :] < lens[:, None]
        for x, y in zip(a, b):
            assert np.array_equal(x[:len(lens) * (len(x) // cap) or len(x)], y[:len(lens) * (len(y) // cap) or len(y)])
        for c in (cd.COL_OBS, cd.COL_AUX) if aux else (cd.COL_OBS,):
            x, y = (read_col(z, c, cap * max_len * 4, np.int32).reshape(cap, max_len)[:len(lens)] for z in bufs)
            assert np.array_equal(x[live], y[live])
        got = read_col(bufs[0], cd.COL_OBS, cap * max_len * 4, np.int32).reshape(cap, max_len)
        for j in range(n):  # this ingest's rows, as given
            k = min(int(length[j]), max_len)
            assert np.array_equal(got[(it * n + j) % cap, :k], tok[offsets[j]:offsets[j] + k])
        tree_consistent(bufs[0], cap)
        assert info.size == min(cap, (it + 1) * n)
    for b in bufs:
        b.close()


# variable-length rows around the most that take one launch, against the two calls
@pytest.mark.parametrize("n", [1024, 1025])
def test_update_ingest_ragged_limit(n):
    print(f"ragged update_ingest rows n={n}", flush=True)
    rng = np.random.default_rng(n)
    cap, max_len = 1500, 12
    length = rng.integers(0, max_len + 1, n)
    offsets = np.concatenate([[0], np.cumsum(length)])
    tok = dev(rng.integers(0, 1 << 30, int(offsets[-1])).astype(np.int32))
    rows = dict(offsets=dev(offsets), reward=dev(rng.standard_normal(n).astype(np.float32)))
    idx, prio = dev(rng.integers(0, n, 200)), dev(synth.quantise_priority(rng.lognormal(0, 2, 200)))
    got = []
    for one in (True, False):
        buf = cd.ReplayBuffer(cap, (max_len,), torch.int32, ragged=True)
        buf.ingest(tok, **rows)
        if one:
            buf.update_ingest(idx, prio, tok, **rows)
        else:
            buf.update(idx, prio)
            buf.ingest(tok, **rows)
        assert buf.sync_check() == cd.OK, cd.last_error()
        tree_consistent(buf, cap)
        lens = read_col(buf, cd.COL_LENGTH, cap * 4, np.int32)
        seq = read_col(buf, cd.COL_OBS, cap * max_len * 4, np.int32).reshape(cap, max_len)
        got.append((lens, np.where(np.arange(max_len) < lens[:, None], seq, -1), read_col(buf, cd.COL_REWARD, cap * 4, np.uint32),
                    read_col(buf, cd.COL_LEAVES, cap * 4, np.uint32)))
        buf.close()
    assert all(np.array_equal(x, y) for x, y in zip(*got))


# token delivery with advantages at each width it is dispatched on (256, 512 and
# 1,024 lanes), against the two calls it stands for
@pytest.mark.parametrize("max_len,B", [(4, 3), (1024, 130), (1028, 70), (4096, 33), (4100, 40)])
@pytest.mark.parametrize("values", [False, True])
def test_sample_pack_gae_widths(max_len, B, values):
    print(f"pack + gae max_len={max_len} B={B} values={values}", flush=True)
    rng = np.random.default_rng(max_len + B)
    cap = 150
    length = rng.integers(0, max_len + 1, cap)
    length[:3] = [0, 1, max_len]
    total = int(length.sum())
    buf = cd.ReplayBuffer(cap, (max_len,), torch.int32, ragged=True, aux_elem_bytes=4)
    buf.ingest(dev(rng.integers(0, 1 << 30, total).astype(np.int32)), aux=dev(rng.standard_normal(total).astype(np.float32)),
               offsets=dev(np.concatenate([[0], np.cumsum(length)])), reward=dev(rng.standard_normal(cap).astype(np.float32)),
               prio=dev(synth.quantise_priority(rng.lognormal(0, 1, cap))))
    u = dev(synth.uniforms(rng, B))
    v = dev(rng.standard_normal((B, max_len)).astype(np.float32)) if values else None
    xf = cd.transform(cd.XF_TOKENS_PAD, pad_id=7)
    outs = []
    for fused in (True, False):
        f = lambda *s: torch.full(s, np.nan, device="cuda")  # noqa: E731
        o = dict(obs=torch.zeros((B, max_len), dtype=torch.int32, device="cuda"), aux=f(B, max_len), reward=f(B),
                 mask=torch.zeros((B, max_len), dtype=torch.uint8, device="cuda"),
                 length=torch.zeros(B, dtype=torch.int32, device="cuda"))
        adv, ret = f(B, max_len), f(B, max_len)
        if fused:
            idx, w = buf.sample_pack_gae(u, xf, 0.99, 0.95, adv, ret, values=v, **o)
        else:
            idx, w = buf.sample_gather(u, xf, **o)
            cd.conduit_gae_packed(o["reward"], o["length"], v, max_len, 0.99, 0.95, adv, ret)
        assert buf.sync_check() == cd.OK and cd.conduit_sync_check() == cd.OK
        outs.append((idx, w, adv, ret, *o.values()))
    for x, y in zip(*outs):
        if x.dtype == torch.float32:
            assert_gae_close(host(x), host(y))
        else:
            assert torch.equal(x, y)
    buf.close()


# batches whose weights take two launches of their own: captured, replayed with new
# uniforms and priorities and eager calls between; then a tree of zeros
@pytest.mark.parametrize("norm", [0, 1])
def test_large_batch_weights_captured(norm):
    print(f"captured weights norm={norm}", flush=True)
    rng = np.random.default_rng(norm)
    cap, B = 3000, 2049
    obs = rng.standard_normal((cap, 8)).astype(np.float32)
    prio = synth.quantise_priority(rng.lognormal(0, 1, cap))
    buf = cd.ReplayBuffer(cap, (8,), torch.float32, action_bytes=0, weight_norm=norm)
    orc = oracle.Replay(cap, (8,), np.float32, act_bytes=0)
    buf.ingest(dev(obs), prio=dev(prio))
    orc.ingest(cap, obs=obs, prio=prio)
    u, p = dev(synth.uniforms(rng, B)), dev(prio[:B].copy())
    idx, w = torch.empty(B, dtype=torch.int64, device="cuda"), torch.empty(B, device="cuda")
    idx2, w2, out = torch.empty_like(idx), torch.empty_like(w), torch.empty((B, 1, 8), device="cuda")
    xf = cd.transform(cd.XF_NONE)

    def step():
        buf.sample_gather(u, xf, idx_out=idx, w_out=w, obs=out)
        buf.sample(u, idx2, w2)
        buf.update(idx, p)

    def check(uniforms, new):
        o_idx, o_w = orc.sample(uniforms, buffer_norm=bool(norm))
        assert np.array_equal(host(idx), o_idx) and np.array_equal(host(idx2), o_idx)
        assert_weights_close(host(w), o_w)
        assert torch.equal(w, w2) and np.array_equal(host(out)[:, 0], obs[o_idx])
        orc.update(o_idx, new)

    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        step()
    torch.cuda.current_stream().wait_stream(s)
    torch.cuda.synchronize()
    check(host(u, np.uint64), host(p, np.uint32))
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step()
    for _ in range(4):
        uniforms, new = synth.uniforms(rng, B), synth.quantise_priority(rng.lognormal(0, 2, B))
        u.copy_(dev(uniforms))
        p.copy_(dev(new))
        g.replay()
        torch.cuda.synchronize()
        check(uniforms, new)
        few = rng.integers(0, cap, 5)
        buf.update(dev(few), dev(np.full(5, 77, np.uint32)))
        orc.update(few, np.full(5, 77, np.uint32))
    assert buf.sync_check() == cd.OK, cd.last_error()
    buf.update(torch.arange(cap, device="cuda"), torch.zeros(cap, dtype=torch.int32, device="cuda"))
    for call in (lambda: buf.sample_gather(u, xf, idx_out=idx, w_out=w, obs=out), lambda: buf.sample(u, idx, w)):
        call()
        assert buf.sync_check() == cd.ESTATE
        buf.clear_error()
        assert (host(idx) == -1).all() and not host(w).any() and not host(out).any()
    buf.close()


# n-step delivery out of a ring beyond the last-level cache (256 MiB) and just below
# it, against the two calls it stands for
@pytest.mark.parametrize("cap", [38000, 38100])
def test_nstep_of_a_large_ring(cap):
    print(f"n-step large ring cap={cap}", flush=True)
    rng = np.random.default_rng(cap)
    done = (rng.random(cap) < 0.02).astype(np.uint8)
    episode, step = synth.episodes_from_done(done)
    g = torch.Generator(device="cuda")
    g.manual_seed(cap)
    obs = torch.randint(-2 ** 31, 2 ** 31, (cap, 1764), generator=g, device="cuda", dtype=torch.int32).view(torch.uint8)
    buf = cd.ReplayBuffer(cap, (84, 84), torch.uint8, frame_stack=2)
    buf.ingest(obs.view(cap, 84, 84), reward=dev(rng.standard_normal(cap).astype(np.float32)), done=dev(done),
               episode_id=dev(episode), step=dev(step), prio=dev(synth.quantise_priority(rng.lognormal(0, 1, cap))))
    B, n, xf = 300, 3, cd.transform(cd.XF_U8_F32)
    u = dev(synth.uniforms(rng, B))
    new = lambda: torch.full((B, 2, 84, 84), 7.0, device="cuda")  # noqa: E731
    one, nxt = new(), new()
    idx, w, ni, ret, disc, valid = buf.sample_gather_nstep(u, xf, n, 0.9, next_obs=nxt, obs=one)
    two, nxt2 = new(), new()
    idx2, w2 = buf.sample_gather(u, xf, obs=two)
    ni2, ret2, disc2, valid2 = (torch.empty_like(x) for x in (ni, ret, disc, valid))
    cd.conduit_nstep(buf.handle, idx2, n, 0.9, ni2, ret2, disc2, valid2, xf, nxt2)
    assert buf.sync_check() == cd.OK, cd.last_error()
    for x, y in ((idx, idx2), (w, w2), (one, two), (nxt, nxt2), (ni, ni2), (ret, ret2), (disc, disc2), (valid, valid2)):
        assert torch.equal(x, y)
    buf.close()

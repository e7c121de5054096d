"""GAE of rollouts that one tile holds (k_gae_tile), against the oracle, at the
edges of its tiles: the last step of a wavefront's and of a workgroup's tile and
the next one, partial quads, wavefronts and groups of environments, rows on and
off a 16-byte boundary, and outputs above the size from which they stream."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import assert_gae_close, dev, host
from paper_2609_24456_amd import conduit as cd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,shift,path,chunk", [
    (1, 1, 0, "short", 2), (16, 132, 0, "short", 2), (16, 127, 0, "short", 2), (17, 68, 0, "short", 2),
    (32, 63, 0, "short", 2), (32, 64, 1, "short", 2), (33, 36, 0, "short", 2), (64, 4100, 1, "short", 2),
    (65, 31, 0, "look", 2), (65, 32, 0, "short", 4), (128, 36, 0, "short", 4), (128, 8195, 0, "short", 4),
    (127, 4096, 1, "short", 4), (129, 4064, 0, "look", 2), (129, 4068, 0, "short", 8), (256, 4071, 0, "short", 8),
    (256, 33000, 0, "short", 8), (257, 4100, 0, "look", 8), (32, 262144, 0, "short", 2)])
@pytest.mark.parametrize("truncated", [False, True])
def test_gae_one_tile(T, E, shift, path, chunk, truncated):
    print(f"gae tile T={T} E={E} shift={shift} truncated={truncated}", flush=True)
    assert cd.gae_plan(T, E, shift == 0) == (path, chunk)
    rng = np.random.default_rng(T * 31 + E)
    f = lambda *s: rng.standard_normal(s).astype(np.float32)  # noqa: E731
    r, v, fv, boot = f(T, E), f(T, E), f(T, E), f(E)
    d, u = ((rng.random((T, E)) < p).astype(np.uint8) for p in (0.05, 0.05))

    def at(a):  # the array `shift` elements off a 16-byte boundary
        flat = torch.empty(a.size + shift, dtype=dev(a[:0]).dtype, device="cuda")
        flat[shift:].copy_(torch.from_numpy(a.reshape(-1)))
        return flat[shift:].view(a.shape)

    for gamma, lam in ((0.99, 0.95), (1.0, 1.0)):
        adv, ret = at(np.full((T, E), np.nan, np.float32)), at(np.full((T, E), np.nan, np.float32))
        if truncated:
            cd.conduit_gae_truncated(at(r), at(v), at(d), at(u), at(fv), at(boot), gamma, lam, adv, ret)
            oa, orr = oracle.gae(r, v, d, boot, gamma, lam, truncated=u, final_value=fv)
        else:
            cd.conduit_gae(at(r), at(v), at(d), at(boot), gamma, lam, adv, ret)
            oa, orr = oracle.gae(r, v, d, boot, gamma, lam)
        assert cd.conduit_sync_check() == cd.OK, cd.last_error()
        assert_gae_close(host(adv), oa)
        assert_gae_close(host(ret), orr)


# packed rows around each width the kernel is dispatched on, rows off 16 bytes,
# lengths at the edges of a wavefront's blocks and spans and of a pass (padding
# only, one live element, the whole row), and padding that must not be used
@pytest.mark.parametrize("Lmax,gamma,lam", [
    (1, 0.9, 0.8), (255, 1.0, 0.95), (1024, 1.0, 0.95), (1025, 0.99, 1.0), (2048, 1.0, 0.95), (2050, 1.0, 0.5),
    (4096, 0.0, 0.95), (4100, 1.0, 0.95), (8192, 1.0, 0.999), (8193, 0.99, 0.95), (16387, 1.0, 0.99)])
def test_gae_packed_widths(Lmax, gamma, lam):
    print(f"packed Lmax={Lmax}", flush=True)
    rng = np.random.default_rng(Lmax)
    edges = [0, 1, 2, 4, 5, 255, 256, 257, 260, 511, 512, 1023, 1024, 1025, 1028, 2047, 2049, 4095, 4096, 4097, 8192, 8193,
             Lmax - 1, Lmax]
    length = np.array([x for x in edges if 0 <= x <= Lmax], np.int32)
    B = len(length)
    R = rng.standard_normal(B).astype(np.float32)
    v = rng.standard_normal((B, Lmax)).astype(np.float32)
    oa, orr = oracle.gae_packed(R, length, v, Lmax, gamma, lam)
    pad = np.arange(Lmax)[None, :] >= length[:, None]
    v[pad] = np.nan  # never used
    adv = torch.full((B, Lmax), np.nan, dtype=torch.float32, device="cuda")
    ret = torch.full((B, Lmax), np.nan, dtype=torch.float32, device="cuda")
    cd.conduit_gae_packed(dev(R), dev(length), dev(v), Lmax, gamma, lam, adv, ret)
    assert cd.conduit_sync_check() == cd.OK, cd.last_error()
    assert_gae_close(host(adv), oa)
    assert_gae_close(host(ret), orr)
    assert not host(adv)[pad].any() and not host(ret)[pad].any()


# advantages or returns in the values' place, one pass a row and several
@pytest.mark.parametrize("Lmax", [700, 4096, 8192, 8193, 16384, 40001])
@pytest.mark.parametrize("place", ["adv", "ret"])
def test_gae_packed_in_place(Lmax, place):
    print(f"packed in place Lmax={Lmax} {place}", flush=True)
    rng = np.random.default_rng(Lmax)
    length = np.concatenate([rng.integers(0, Lmax + 1, 300), [0, 1, Lmax - 1, Lmax]]).astype(np.int32)
    B = len(length)
    R, v = dev(rng.standard_normal(B).astype(np.float32)), dev(rng.standard_normal((B, Lmax)).astype(np.float32))
    adv, ret, other = (torch.empty((B, Lmax), device="cuda") for _ in range(3))
    cd.conduit_gae_packed(R, dev(length), v, Lmax, 0.99, 0.95, adv, ret)
    outs = (v, other) if place == "adv" else (other, v)
    cd.conduit_gae_packed(R, dev(length), v, Lmax, 0.99, 0.95, *outs)
    assert cd.conduit_sync_check() == cd.OK, cd.last_error()
    assert torch.equal(outs[0], adv) and torch.equal(outs[1], ret)

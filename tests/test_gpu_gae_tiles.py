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

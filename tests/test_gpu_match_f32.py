"""f32 caches: every live row is decided in f64, its retained list whole (up to 256 keys) or shared by up to eight workgroups."""
import numpy as np
import pytest
import torch

from tests import gpu_util as U

pytestmark = pytest.mark.gpu


def _reference(K, keep, evict, n_ev, T):
    out = np.full(evict.shape, -7, np.int64)              # rows at or beyond n_evict are not written
    for j in range(n_ev):
        e = K[evict[j]]
        with np.errstate(all="ignore"):
            u = (K[keep] @ e) / np.sqrt(e @ e) / np.sqrt((K[keep] ** 2).sum(-1))
        u[~np.isfinite(u)] = -np.inf
        out[j] = int(np.argmax(u)) if u.max() > T else -1
    return out


# (heads, evictable, budget): one workgroup a row; two, four and eight; rows enough for one although the list is long
@pytest.mark.parametrize("heads,n_evict,budget", [(4, 32, 52), (4, 16, 256), (4, 16, 257), (2, 16, 1025), (1, 16, 2049), (8, 64, 600)])
@pytest.mark.parametrize("D", [64, 128])
def test_match(heads, n_evict, budget, D):
    kk = U.kk()
    lay = kk.Layout(1, heads, heads, D, kk.F32, D ** -0.5)
    g = np.random.default_rng(budget + D)
    cap = budget + n_evict
    c = kk.Cache(lay, cap)
    K = g.standard_normal((heads, cap, D)).astype(np.float32)
    K[:, 1] = 0.0                                         # a key without a direction
    K[:, budget // 2] = K[:, 3] * 2.0                     # parallel keys: the first of them wins
    slots = np.stack([g.permutation(cap) for _ in range(heads)])
    keep, evict = np.sort(slots[:, :budget], 1), np.sort(slots[:, budget:], 1)
    for h in range(heads):                                # some rows with a partner
        K[h, evict[h, ::3]] = 0.5 * K[h, g.choice(keep[h], len(evict[h, ::3]))]
    n_ev = np.array([n_evict - 3 * (h % 3) if h % 4 != 3 else 0 for h in range(heads)], np.int32)
    c.k.copy_(torch.from_numpy(K)[None])
    c.len.fill_(cap)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.int32)).cuda()[None]
    match = torch.full((1, heads, n_evict), -7, dtype=torch.int32, device="cuda")
    ws = kk.new_workspace(lay, cap, budget)
    for T in (0.8, -2.0):
        match.fill_(-7)
        for _ in range(2):                                # the tickets return to zero
            kk.match(lay, c, budget, dev(keep), dev(evict), dev(n_ev), T, match, None, ws)
        got = match.cpu().numpy()[0]
        assert not ws[:64 * 1024 + 256].any()
        for h in range(heads):
            want = _reference(K[h].astype(np.float64), keep[h], evict[h], int(n_ev[h]), T)
            same = got[h] == want
            # a numpy sum may round the other way where two keys are parallel: equal to the first one's
            for j in np.flatnonzero(~same):
                a, b = K[h, keep[h, got[h, j]]].astype(np.float64), K[h, keep[h, want[j]]].astype(np.float64)
                assert got[h, j] >= 0 and want[j] >= 0 and abs(a @ b) >= (1 - 1e-12) * np.sqrt((a @ a) * (b @ b)), (h, j)

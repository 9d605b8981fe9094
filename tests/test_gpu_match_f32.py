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


# (heads, most live rows of a head, budget, slots of the cache beyond them).  Workgroups a row: a list is shared by two from 257 keys on, by four
# from 513, by eight from 1025, if the live rows are at most 128, 64 and 32.  300 heads: two to a thread where the live rows are counted, 16384,
# the most there can be: 64.
@pytest.mark.parametrize("heads,n_evict,budget,beyond", [(4, 32, 52, 0), (4, 16, 256, 0), (4, 16, 257, 0), (2, 16, 1025, 0), (1, 16, 2049, 0), (8, 64, 600, 0),
                                                         (1, 16, 512, 0), (1, 16, 513, 7), (1, 16, 1024, 0), (1, 16, 1025, 3000), (2, 9, 52, 5000),
                                                         (300, 4, 40, 0), (300, 4, 40, 90), (16384, 3, 5, 0)])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("ragged", [True, False])
def test_match(heads, n_evict, budget, beyond, D, ragged):
    kk = U.kk()
    lay = kk.Layout(1, heads, heads, D, kk.F32, D ** -0.5)
    g = np.random.default_rng(budget + D)
    cap = budget + n_evict
    c = kk.Cache(lay, cap + beyond)
    K = g.standard_normal((heads, cap, D)).astype(np.float32)
    K[:, 1] = 0.0                                         # a key without a direction
    K[:, budget // 2] = K[:, 3] * 2.0                     # parallel keys: the first of them wins
    slots = np.stack([g.permutation(cap) for _ in range(heads)])
    keep, evict = np.sort(slots[:, :budget], 1), np.sort(slots[:, budget:], 1)
    for h in range(heads):                                # some rows with a partner
        K[h, evict[h, ::3]] = 0.5 * K[h, g.choice(keep[h], len(evict[h, ::3]))]
    n_ev = np.array([max(0, n_evict - 3 * (h % 3)) if h % 4 != 3 else 0 for h in range(heads)] if ragged else [n_evict] * heads, np.int32)
    c.k[:, :, :cap] = torch.from_numpy(K)[None]
    c.k[:, :, cap:] = float("nan")                        # (never read)
    c.len.fill_(cap)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.int32)).cuda()[None]
    evict_dev = torch.zeros(1, heads, n_evict + beyond, dtype=torch.int32, device="cuda")
    evict_dev[..., :n_evict] = dev(evict)
    match = torch.full((1, heads, n_evict + beyond), -7, dtype=torch.int32, device="cuda")
    ws = kk.new_workspace(lay, cap + beyond, budget)
    for T in (0.8, -2.0):
        match.fill_(-7)
        for _ in range(2):                                # the tickets return to zero
            kk.match(lay, c, budget, dev(keep), evict_dev, dev(n_ev), T, match, None, ws)
        got = match.cpu().numpy()[0]
        assert (got[:, n_evict:] == -7).all()
        got = got[:, :n_evict]
        assert not ws[:64 * 1024 + 256].any()
        for h in range(heads):
            want = _reference(K[h].astype(np.float64), keep[h], evict[h], int(n_ev[h]), T)
            same = got[h] == want
            # a numpy sum may round the other way where two keys are parallel: equal to the first one's
            for j in np.flatnonzero(~same):
                a, b = K[h, keep[h, got[h, j]]].astype(np.float64), K[h, keep[h, want[j]]].astype(np.float64)
                assert got[h, j] >= 0 and want[j] >= 0 and abs(a @ b) >= (1 - 1e-12) * np.sqrt((a @ a) * (b @ b)), (h, j)


@pytest.mark.parametrize("heads,cap,lens", [(4, 1500, (700, 1, 0, 333)), (4, 257, (257, 257, 257, 257)), (3, 3000, (9, 9, 9)), (300, 12, None)])
@pytest.mark.parametrize("D", [64, 128])
def test_prefill_match(heads, cap, lens, D):
    kk = U.kk()
    lay = kk.Layout(1, heads, heads, D, kk.F32, D ** -0.5)
    g = np.random.default_rng(cap + D)
    lens = np.array([h % 12 for h in range(heads)] if lens is None else lens, np.int32)
    K = g.standard_normal((heads, cap, D)).astype(np.float32)
    for h, n in enumerate(lens):
        K[h, n // 2:n:3] = 0.5 * K[h, g.integers(0, max(1, n // 2), len(K[h, n // 2:n:3]))]
        K[h, n:] = np.nan                                 # (never read)
    c = kk.Cache(lay, cap)
    c.k.copy_(torch.from_numpy(K)[None])
    c.len.copy_(torch.from_numpy(lens)[None])
    near = torch.full((1, heads, cap), -7, dtype=torch.int32, device="cuda")
    ws = kk.new_workspace(lay, cap, 1)
    for _ in range(2):
        kk.prefill_match(lay, c, 0.8, near, None, ws)
    got = near.cpu().numpy()[0]
    assert not ws[:64 * 1024 + 256].any()
    for h, n in enumerate(lens):
        k = K[h, :n].astype(np.float64)
        u = k @ k.T / np.sqrt((k ** 2).sum(-1))[:, None] / np.sqrt((k ** 2).sum(-1))[None]
        for j in range(n):
            want = int(np.argmax(u[j, :j])) if j and u[j, :j].max() > 0.8 else -1
            # (copies of one key are parallel: of equal similarities the first wins, and numpy's sum may round the other way)
            assert got[h, j] == want or (got[h, j] >= 0 and want >= 0 and abs(u[j, got[h, j]] - u[j, want]) < 1e-12), (h, j)
        assert (got[h, n:] == -7).all()

"""keepkv_merge on match lists built to reach every edge of its grouping and summing: list lengths around the lane
group (8, 16 or 32 lanes), the wavefront and the longest list that is ordered by counting (256); targets at the ends
of the ranges that workgroups share; heads without a match; few heads (several workgroups per head, one position per
wavefront) and many (one workgroup, full wavefronts)."""
import numpy as np
import pytest
import torch

from oracle import keepkv_oracle as O
from paper_2504_09936_amd import workloads as W
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

SIZES = [1, 6, 7, 8, 14, 15, 16, 30, 31, 32, 62, 63, 64, 65, 127, 128, 129, 255, 256, 257, 300, 700]


@pytest.mark.parametrize("dtype,head_dim,batch", [("bf16", 128, 1), ("bf16", 64, 1), ("f32", 128, 1), ("f32", 64, 1), ("bf16", 128, 40),
                                                  ("bf16", 64, 33)])
def test_merge_of_given_lists(dtype, head_dim, batch):
    kk = U.kk()
    H, budget, n_ev = 8, 101, sum(SIZES) + 400
    cap = budget + n_ev
    w = W.CONFIGS["llama3_8b"].scaled(batch=batch, head_dim=head_dim, dtype=dtype, context=cap, ratio=(budget - 0.5) / cap)
    g = np.random.default_rng(head_dim + batch)
    K, V = (W.round_storage(g.standard_normal((batch, H, cap, head_dim)), dtype) for _ in range(2))
    lay, c = U.new_cache(w, capacity=cap, K=K, V=V, votes=g.integers(1, 9, size=(batch, H, cap)))
    c.log_s[:] = torch.from_numpy((g.standard_normal((batch, H, cap)) - 6).astype(np.float32)).cuda()
    U.set_n_obs(c, g.integers(0, 60, size=(batch, H, cap)).astype(np.int32))     # some slots never observed
    keep, evict = np.empty((batch, H, budget), np.int32), np.empty((batch, H, n_ev), np.int32)
    match = np.full((batch, H, n_ev), -1, np.int32)
    # at the ends of the eight target ranges, then in between
    ends = sorted({e for s in range(9) for e in (budget * s // 8 - 1, budget * s // 8) if 0 <= e < budget})
    targets = (ends + [t for t in range(budget) if t not in ends])[:len(SIZES)]
    for b in range(batch):
        for h in range(H):
            kept = np.zeros(cap, bool)
            kept[g.choice(cap, budget, replace=False)] = True
            keep[b, h], evict[b, h] = np.flatnonzero(kept), np.flatnonzero(~kept)
            if (b, h) == (0, 3):
                continue                                                          # nothing matches in this head
            at = g.permutation(n_ev)
            for t, m in zip(targets, g.permutation(SIZES)):
                match[b, h, at[:m]], at = t, at[m:]
    up = lambda a: torch.from_numpy(a).cuda()                                     # noqa: E731
    n_evict = torch.full((batch, H), n_ev, dtype=torch.int32, device="cuda")
    dropped = torch.full((batch, H), 5, dtype=torch.int64, device="cuda")         # accumulated into
    ws = U.workspace(lay, cap, budget)
    alpha = U.f32(0.9)
    runs = []
    for _ in range(2):
        _, d = U.new_cache(w, capacity=budget + 3)
        kk.merge(lay, c, d, budget, up(keep), up(evict), n_evict, up(match), alpha, dropped, ws)
        torch.cuda.synchronize()
        runs.append(d)
    for f in d.FIELDS:                                                            # the same bits every time
        assert torch.equal(getattr(runs[0], f), getattr(runs[1], f)), f
    oc, dk, dv = U.download(c), U.to_host(d.k), U.to_host(d.v)
    for b, h in [(0, h) for h in range(H)] + [(batch - 1, 7)]:
        ref = O.merge(oc.k[b, h], oc.v[b, h], oc.votes[b, h], oc.log_S[b, h], oc.n_obs[b, h], keep[b, h], evict[b, h],
                      match[b, h], alpha)
        np.testing.assert_array_equal(d.votes[b, h, :budget].cpu().numpy(), ref.votes)
        np.testing.assert_array_equal(U.n_obs(d)[b, h, :budget].cpu().numpy(), ref.n_obs)
        assert dropped[b, h].item() == 5 + 2 * ref.dropped
        np.testing.assert_allclose(d.log_s[b, h, :budget].cpu().numpy(), ref.log_S, rtol=2e-6, atol=2e-6)
        # rows: up to 701 f32 products summed, 701 * 2^-24 relative to the sum of magnitudes in the worst case, and the
        # storage rounding; keys whose scale denominator is near the guard are ill-conditioned
        well = ~(np.abs(ref.ell_bar) < 4 * O.ELL_GUARD)
        assert U.storage_err_rows(dv[b, h, :budget], ref.v, dtype).max() <= 2e-3
        assert U.storage_err_rows(dk[b, h, :budget], ref.k, dtype)[well].max() <= 2e-3


# eight, sixteen and 32 workgroups a head; 8 entries a thread up to 8192 of them, 32 beyond
@pytest.mark.parametrize("n_ev", [300, 2100, 4096, 8191, 8192, 8193, 9217])
def test_merge_of_every_entry(n_ev):
    """Every entry reaches its target, whatever the number of entries a thread holds and of workgroups that share a head."""
    kk = U.kk()
    H, D, budget = 2, 64, 90
    cap = budget + n_ev
    w = W.CONFIGS["llama3_8b"].scaled(batch=1, n_q_heads=H, n_kv_heads=H, head_dim=D, context=cap, ratio=(budget - 0.5) / cap)
    g = np.random.default_rng(n_ev)
    K, V = (W.round_storage(g.standard_normal((1, H, cap, D)), "bf16") for _ in range(2))
    votes = g.integers(1, 9, size=(1, H, cap)).astype(np.int32)
    lay, c = U.new_cache(w, capacity=cap, K=K, V=V, votes=votes)
    c.log_s[:] = torch.from_numpy((g.standard_normal((1, H, cap)) - 6).astype(np.float32)).cuda()
    slots = np.stack([g.permutation(cap) for _ in range(H)]).astype(np.int32)
    keep, evict = np.sort(slots[:, :budget], 1)[None], np.sort(slots[:, budget:], 1)[None]
    live = np.array([[n_ev, n_ev - 5]], np.int32)
    match = g.integers(-1, budget, size=(1, H, n_ev)).astype(np.int32)
    up = lambda a: torch.from_numpy(a).cuda()                                     # noqa: E731
    dropped = torch.zeros(1, H, dtype=torch.int64, device="cuda")
    _, d = U.new_cache(w, capacity=budget)
    kk.merge(lay, c, d, budget, up(keep), up(evict), up(live), up(match), U.f32(0.9), dropped, U.workspace(lay, cap, budget))
    oc = U.download(c)
    for h in range(H):
        n = live[0, h]
        m, pv = match[0, h, :n], votes[0, h, evict[0, h, :n]].astype(np.int64)
        want = votes[0, h, keep[0, h]] + np.bincount(m[m >= 0], weights=pv[m >= 0], minlength=budget).astype(np.int64)
        np.testing.assert_array_equal(d.votes[0, h].cpu().numpy(), want)
        assert dropped[0, h].item() == pv[m < 0].sum()
        ref = O.merge(oc.k[0, h], oc.v[0, h], oc.votes[0, h], oc.log_S[0, h], oc.n_obs[0, h], keep[0, h], evict[0, h, :n], m, U.f32(0.9))
        assert U.storage_err_rows(U.to_host(d.v)[0, h], ref.v, "bf16").max() <= 2e-3

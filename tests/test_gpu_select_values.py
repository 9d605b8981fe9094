"""keepkv_select decides most slots in f32 and the few near the threshold in f64.  Ranking values that only f64 can
tell apart (few and many of them), exact ties across the threshold, values of very different magnitudes, unobserved
heads, counts and votes beyond the tables, at capacities around the instances of the kernel: index lists equal the
oracle's."""
import numpy as np
import pytest
import torch

from oracle import keepkv_oracle as O
from paper_2504_09936_amd import workloads as W
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("alpha", [0.9, 0.9999])
@pytest.mark.parametrize("cap", [65, 1023, 1024, 1025, 4096, 4097, 8192, 8193, 16384, 16385, 32768, 32769])
def test_select_at_the_threshold(cap, alpha):
    kk = U.kk()
    alpha = U.f32(alpha)
    g = np.random.default_rng(cap)
    B, H, budget, n_sink = 1, 8, max(20, cap // 9), 4
    n_recent = budget // 2
    w = W.CONFIGS["llama3_8b"].scaled(batch=B, n_q_heads=H, n_kv_heads=H, context=cap)
    lay, c = U.new_cache(w, capacity=cap)
    ws = U.workspace(lay, cap, budget)
    log_s = (g.standard_normal((H, cap)) * 3 - 5).astype(np.float32)
    votes = g.integers(1, 4, size=(H, cap)).astype(np.int32)
    n_obs = g.integers(1, 40, size=(H, cap)).astype(np.int32)
    near = g.choice(cap, min(cap // 2, 120), replace=False)     # close to each other, the rest far away: f64 decides
    log_s[1, near] = np.float32(2.0) + g.integers(-3, 4, len(near)).astype(np.float32) * np.float32(2.0 ** -22)
    log_s[2] = np.float32(-1.0) + g.integers(0, 5, cap).astype(np.float32) * np.float32(2.0 ** -24)   # all of them
    n_obs[2] = g.integers(300, 340, cap)
    log_s[3], votes[3], n_obs[3] = -2.5, 2, 17                  # all equal
    log_s[4] *= np.float32(10.0) ** g.integers(-20, 20, cap).astype(np.float32)
    log_s[5], n_obs[5] = -np.inf, 0                             # nothing observed
    n_obs[6, ::3] = 0
    log_s[6, ::3] = -np.inf
    votes[7, ::7] = g.integers(200, 100000, len(votes[7, ::7]))
    n_obs[7] = g.integers(1, 5000, cap)
    c.log_s[:] = torch.from_numpy(log_s[None]).cuda()
    c.votes[:] = torch.from_numpy(votes[None]).cuda()
    U.set_n_obs(c, n_obs[None])
    for lens in (np.full((1, H), cap), g.integers(budget + 1, cap + 1, size=(1, H))):
        c.len[:] = torch.from_numpy(lens.astype(np.int32)).cuda()
        keep = torch.full((B, H, budget), -7, dtype=torch.int32, device="cuda")
        evict = torch.full((B, H, cap - budget), -7, dtype=torch.int32, device="cuda")
        n_ev = torch.full((B, H), -7, dtype=torch.int32, device="cuda")
        kk.select(lay, c, budget, n_sink, n_recent, alpha, keep, evict, n_ev, ws)
        torch.cuda.synchronize()
        for h in range(H):
            n = int(lens[0, h])
            rk, re = O.select(log_s[h].astype(np.float64), n_obs[h], votes[h], n, budget, n_sink, n_recent, alpha)
            assert n_ev[0, h].item() == len(re)
            np.testing.assert_array_equal(keep[0, h].cpu().numpy(), rk, err_msg=f"head {h}")
            np.testing.assert_array_equal(evict[0, h, :len(re)].cpu().numpy(), re, err_msg=f"head {h}")
            assert (evict[0, h, len(re):] == -7).all()


@pytest.mark.parametrize("cap", [100, 1025, 8192, 20000, 32769])
def test_nan_scores_rank_by_their_sign(cap):
    """A NaN score ranks by its f64 image, above +inf or below -inf by its sign, whichever kernel decides: with one
    vote and alpha^n below half an ulp the ranking value is the score itself."""
    kk = U.kk()
    g = np.random.default_rng(cap)
    H, budget, n_sink, n_recent = 4, cap // 4, 3, cap // 9
    w = W.CONFIGS["llama3_8b"].scaled(batch=1, n_q_heads=H, n_kv_heads=H, context=cap)
    lay, c = U.new_cache(w, capacity=cap)
    ws = U.workspace(lay, cap, budget)
    log_s = (g.standard_normal((H, cap)) * 3).astype(np.float32)
    n_high = budget - n_sink - n_recent
    for h, (pos, neg) in enumerate([(5, 0), (0, 5), (n_high // 2, n_high // 2), (n_high + 7, cap // 8)]):
        at = g.choice(np.arange(n_sink, cap - n_recent), pos + neg + 4, replace=False)
        log_s[h, at[:pos]] = np.array([0x7FC00000], np.uint32).view(np.float32)
        log_s[h, at[pos:pos + neg]] = np.array([0xFFC00000], np.uint32).view(np.float32)
        log_s[h, at[-4:-2]], log_s[h, at[-2:]] = np.inf, -np.inf
    c.log_s[:] = torch.from_numpy(log_s[None]).cuda()
    c.votes[:] = 1
    U.set_n_obs(c, np.full((1, H, cap), 500))
    c.len[:] = cap
    keep = torch.full((1, H, budget), -7, dtype=torch.int32, device="cuda")
    evict = torch.full((1, H, cap - budget), -7, dtype=torch.int32, device="cuda")
    n_ev = torch.full((1, H), -7, dtype=torch.int32, device="cuda")
    kk.select(lay, c, budget, n_sink, n_recent, U.f32(0.9), keep, evict, n_ev, ws)
    torch.cuda.synchronize()
    bits = log_s.astype(np.float64).view(np.uint64)
    image = np.where(bits >> np.uint64(63) != 0, ~bits, bits | np.uint64(1 << 63))        # ascending with the value
    for h in range(H):
        mid = np.arange(n_sink, cap - n_recent)
        heavy = mid[np.lexsort((mid, ~image[h, mid]))][:n_high]
        rk = np.sort(np.concatenate([np.arange(n_sink), heavy, np.arange(cap - n_recent, cap)]))
        np.testing.assert_array_equal(keep[0, h].cpu().numpy(), rk, err_msg=f"head {h}")
        np.testing.assert_array_equal(evict[0, h].cpu().numpy(), np.setdiff1d(np.arange(cap), rk))


def _distributions(cap, g):
    """Twelve ranking arrays [12, cap]: outliers beyond and within what the histogram's range leaves out, heavy tails, long runs of
    equal values across the threshold, mixed with others and filling the head, hundreds of values a few ulps apart, infinities."""
    x = g.standard_normal((12, cap)).astype(np.float32)
    far = g.choice(cap, 12, replace=False)
    x[0, far[:3]] = [3e3, 8e2, 5e2]
    x[1, far] = -1e4                                            # in all four classes
    x[2] = np.exp(5 * x[2])
    # (none so small that ln p + ln S - ln(1 - alpha^n) would absorb it: the oracle adds the three in another order)
    x[3] *= np.float32(10.0) ** g.integers(-3, 30, cap).astype(np.float32)
    x[4] = 1.5
    x[5, g.random(cap) < 0.5] = 0.3
    x[6] = np.where(g.random(cap) < 0.95, 0.0, g.random(cap))
    x[7] = np.where(g.random(cap) < 0.9, -np.inf, x[7])
    x[8] = g.integers(0, 5, cap)
    x[9] = 2.0 + g.integers(-40, 40, cap).astype(np.float32) * np.float32(2.0 ** -22)
    x[10, g.random(cap) < 0.6] = np.inf
    x[11, g.random(cap) < 0.4] = np.float32(0.25) + np.float32(2.0 ** -25)
    return x


@pytest.mark.parametrize("varied", [False, True])
@pytest.mark.parametrize("cap,budget,n_sink,n_recent", [
    (300, 60, 2, 10), (884, 820, 4, 652), (1025, 103, 4, 82), (2048, 300, 0, 0), (5003, 501, 4, 397), (8192, 820, 4, 652),
    (9001, 4090, 4, 6), (20000, 1000, 4, 200), (32768, 3277, 4, 2618)])
def test_distributions(cap, budget, n_sink, n_recent, varied):
    """Lists of keepkv_select (votes and counts the same in all slots, or varied) and keepkv_select_by_key on skewed, spread,
    equal and nearly equal values, full and ragged heads: those of the oracle."""
    kk = U.kk()
    alpha = U.f32(0.9)
    g = np.random.default_rng(cap + varied)
    x = _distributions(cap, g)
    H = len(x)
    w = W.CONFIGS["llama3_8b"].scaled(batch=1, n_q_heads=H, n_kv_heads=H, context=cap)
    lay, c = U.new_cache(w, capacity=cap)
    ws = U.workspace(lay, cap, budget)
    votes = g.integers(1, 4, (H, cap)) if varied else np.full((H, cap), 2)
    n_obs = g.integers(1, 60, (H, cap)) if varied else np.full((H, cap), 21)
    c.log_s[:] = torch.from_numpy(x[None]).cuda()
    c.votes[:] = torch.from_numpy(votes[None].astype(np.int32)).cuda()
    U.set_n_obs(c, n_obs[None])
    rank = torch.from_numpy(x[None]).cuda()
    for lens in (np.full((1, H), cap), g.integers(budget + 1, cap + 1, size=(1, H))):
        c.len[:] = torch.from_numpy(lens.astype(np.int32)).cuda()
        for by_key in (False, True):
            keep = torch.full((1, H, budget), -7, dtype=torch.int32, device="cuda")
            evict = torch.full((1, H, cap - budget), -7, dtype=torch.int32, device="cuda")
            n_ev = torch.full((1, H), -7, dtype=torch.int32, device="cuda")
            if by_key:
                kk.select_by_key(lay, c, rank, budget, n_sink, n_recent, keep, evict, n_ev, ws)
            else:
                kk.select(lay, c, budget, n_sink, n_recent, alpha, keep, evict, n_ev, ws)
            torch.cuda.synchronize()
            for h in range(H):
                n = int(lens[0, h])
                if by_key:
                    rk, re = O.select_by_key(x[h], n, budget, n_sink, n_recent)
                else:
                    rk, re = O.select(x[h].astype(np.float64), n_obs[h], votes[h], n, budget, n_sink, n_recent, alpha)
                assert n_ev[0, h].item() == len(re)
                np.testing.assert_array_equal(keep[0, h].cpu().numpy(), rk, err_msg=f"head {h} by_key {by_key}")
                np.testing.assert_array_equal(evict[0, h, :len(re)].cpu().numpy(), re, err_msg=f"head {h} by_key {by_key}")

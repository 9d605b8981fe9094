"""The f64 re-check of undecided rows looks only at the column classes that can hold the best value (columns of equal
number modulo 32).  Rows whose two best columns are equal, or one bf16 step apart, and lie in the same class, in the
same block, in the two halves of a lane pair, in the first and the last column; all-zero rows and keys; rows whose
best value is negative: targets and similarities equal the oracle's."""
import numpy as np
import pytest
import torch

from oracle import keepkv_oracle as O
from paper_2504_09936_amd import workloads as W
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


def _nudge(row, g):
    """`row` with one element moved by one bf16 step."""
    out = row.copy()
    i = int(g.integers(0, len(row)))
    out[i] = W.from_bf16_bits((W.to_bf16_bits(row[i:i + 1]) + np.uint16(1)))[0]
    return out


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("budget,n_ev", [(40, 300), (128, 513), (129, 1100), (820, 600)])
@pytest.mark.parametrize("threshold", [-2.0, 0.8])
def test_ties_and_near_ties(head_dim, budget, n_ev, threshold):
    kk = U.kk()
    g = np.random.default_rng(budget + n_ev + head_dim)
    cap = budget + n_ev
    w = W.CONFIGS["llama3_8b"].scaled(batch=1, n_q_heads=8, n_kv_heads=2, head_dim=head_dim, context=cap)
    K = W.round_bf16(g.standard_normal((1, 2, cap, head_dim)))
    gaps = [1, 3, 4, 8, 31, 32, 33, 36, 64, 96, 128, budget - 1]
    for h in range(2):
        at = budget
        for gap in gaps:
            for c in (0, 5, int(g.integers(0, budget))):
                if c + gap >= budget or at + 4 > cap:
                    continue
                near = h == 1
                K[0, h, c + gap] = _nudge(K[0, h, c], g) if near else K[0, h, c]
                K[0, h, at] = K[0, h, c]                       # evicted rows: copies, scaled copies
                K[0, h, at + 1] = K[0, h, c] * 2
                K[0, h, at + 2] = _nudge(K[0, h, c], g)
                K[0, h, at + 3] = -K[0, h, c]
                at += 4
    K[0, 0, budget // 2] = 0                                   # a zero retained key, a zero evicted row
    K[0, 0, cap - 1] = 0
    K[0, 1, cap - 3:] = -np.abs(K[0, 1, cap - 3:])             # rows against which everything scores low
    lay, c = U.new_cache(w, capacity=cap, K=K, V=K)
    ws = U.workspace(lay, cap, budget)
    keep = torch.arange(budget, dtype=torch.int32, device="cuda").repeat(1, 2, 1).contiguous()
    evict = torch.arange(budget, cap, dtype=torch.int32, device="cuda").repeat(1, 2, 1).contiguous()
    n_evict = torch.full((1, 2), n_ev, dtype=torch.int32, device="cuda")
    T = U.f32(threshold)
    for want_sim in (True, False):
        match = torch.full((1, 2, n_ev), -9, dtype=torch.int32, device="cuda")
        sim = torch.zeros(1, 2, n_ev, device="cuda") if want_sim else None
        kk.match(lay, c, budget, keep, evict, n_evict, T, match, sim, ws)
        torch.cuda.synchronize()
        for h in range(2):
            tgt, s = O.match(K[0, h].astype(np.float64), np.arange(budget), np.arange(budget, cap), T, exact_any_order=True)
            np.testing.assert_array_equal(match[0, h].cpu().numpy(), tgt)
            if want_sim:                                       # f32 sums of at most 128 exact products, two f32 norms
                np.testing.assert_allclose(sim[0, h].cpu().numpy(), s, rtol=0, atol=2e-5)
    # the causal search of the prefill pass on the same keys
    near = torch.full((1, 2, cap), -9, dtype=torch.int32, device="cuda")
    kk.prefill_match(lay, c, T, near, None, ws)
    torch.cuda.synchronize()
    for h in range(2):
        ref, _ = O.prefill_nearest_earlier(K[0, h].astype(np.float64), cap, T, exact_any_order=True)
        np.testing.assert_array_equal(near[0, h].cpu().numpy(), ref)


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("batch,lengths", [
    (2, [1, 2, 31, 32, 33, 64, 65, 127, 128, 129, 191, 192, 255, 256, 257, 300]),            # blocks of 256 rows
    (2, [511, 512, 513, 640, 641, 767, 768, 769, 900, 1000, 1023, 1024, 1025, 1111, 1152, 1153]),
    (64, [1, 2, 33, 64, 127, 128, 129, 255, 256, 257, 383, 384, 385, 511, 512, 513])])       # blocks of 512 rows
def test_causal_search_at_block_edges(head_dim, batch, lengths):
    """Lengths around the tiles, stages and row blocks of the causal search, in a cache whose slots behind the length
    hold NaN, with the capacity at the longest head: links equal the oracle's, twice."""
    kk = U.kk()
    g = np.random.default_rng(head_dim + batch)
    cap = max(lengths)
    w = W.CONFIGS["llama3_8b"].scaled(batch=batch, n_q_heads=8, n_kv_heads=8, head_dim=head_dim, context=cap)
    assert (batch * 8 * ((cap + 511) // 512) >= 512) == (batch == 64)
    K = W.round_bf16(g.standard_normal((batch, 8, cap, head_dim)))
    K[:, :, cap // 2:] = W.round_bf16(K[:, :, :cap - cap // 2] * 0.5 + 0.2 * K[:, :, cap // 2:])      # many links
    lens = np.array([lengths[i % len(lengths)] for i in range(batch * 8)], dtype=np.int32).reshape(batch, 8)
    ref = {}
    for i in list(range(16)) + [batch * 8 - 1]:
        b, h = divmod(i, 8)
        ref[b, h], _ = O.prefill_nearest_earlier(K[b, h].astype(np.float64), int(lens[b, h]), U.f32(0.8), exact_any_order=True)
    for b in range(batch):
        for h in range(8):
            K[b, h, lens[b, h]:] = np.nan
    lay, c = U.new_cache(w, capacity=cap, K=K, V=np.zeros_like(K), lens=lens)
    ws = U.workspace(lay, cap, 10)
    runs = []
    for _ in range(2):
        near = torch.full((batch, 8, cap), -9, dtype=torch.int32, device="cuda")
        kk.prefill_match(lay, c, U.f32(0.8), near, None, ws)
        torch.cuda.synchronize()
        runs.append(near)
    assert torch.equal(*runs)
    got = near.cpu().numpy()
    for (b, h), r in ref.items():
        np.testing.assert_array_equal(got[b, h, :lens[b, h]], r)
        assert (got[b, h, lens[b, h]:] == -9).all()


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("budget,n_ev", [(820, 700), (129, 300), (820, 130), (100, 50)])     # first events, steady states
@pytest.mark.parametrize("scaled", ["rows", "rows, large", "a column", "a column, large", "the best columns", "not finite"])
def test_norms_beyond_f32(head_dim, budget, n_ev, scaled):
    """Keys whose |k|^2 is below or above the f32 range (elements near 2^-80 or 2^70) beside a dozen near-duplicate
    columns in different classes: the f32 values decide nothing there, targets are those of an f64 evaluation.  So they are
    beside keys that hold an infinity or a NaN."""
    kk = U.kk()
    g = np.random.default_rng(budget + head_dim + len(scaled))
    cap = budget + n_ev
    w = W.CONFIGS["llama3_8b"].scaled(batch=1, n_q_heads=8, n_kv_heads=2, head_dim=head_dim, context=cap)
    K = W.round_bf16(g.standard_normal((1, 2, cap, head_dim)))
    for h in range(2):
        for at, c in enumerate(g.choice(budget, 12, replace=False)):      # one centre, one bf16 step here and there
            K[0, h, c] = _nudge(K[0, h, 0], g) if at else K[0, h, 0]
        for j in range(budget, cap, 2):
            K[0, h, j] = W.round_bf16(K[0, h, 0] + 0.1 * g.standard_normal(head_dim))
        scale = 2.0 ** 70 if "large" in scaled else 2.0 ** -80
        if scaled.startswith("rows"):
            K[0, h, budget:] *= scale
        elif scaled.startswith("a column"):
            K[0, h, budget // 3] = K[0, h, 0] * scale
        elif scaled == "not finite":                                       # match nothing, and hide no other column
            K[0, h, budget // 4, 1], K[0, h, budget // 2, 0], K[0, h, cap - 1, 2] = np.inf, np.nan, np.inf
            K[0, h, budget // 4 + 1, 1], K[0, h, cap - 2, 2] = -np.inf, np.nan
        else:
            K[0, h, [5, budget - 1]] = W.round_bf16(K[0, h, 0] * 3.0) * np.array([[2.0 ** -80], [2.0 ** 70]])
    lay, c = U.new_cache(w, capacity=cap, K=K, V=np.zeros_like(K))
    np.testing.assert_array_equal(U.to_host(c.k).astype(np.float64), K)   # powers of two: representable as they are
    ws = U.workspace(lay, cap, budget)
    keep = torch.arange(budget, dtype=torch.int32, device="cuda").repeat(1, 2, 1).contiguous()
    evict = torch.arange(budget, cap, dtype=torch.int32, device="cuda").repeat(1, 2, 1).contiguous()
    n_evict = torch.full((1, 2), n_ev, dtype=torch.int32, device="cuda")
    T = U.f32(0.3)
    for want_sim in (True, False):
        match = torch.full((1, 2, n_ev), -9, dtype=torch.int32, device="cuda")
        kk.match(lay, c, budget, keep, evict, n_evict, T, match, torch.zeros(1, 2, n_ev, device="cuda") if want_sim else None, ws)
        torch.cuda.synchronize()
        for h in range(2):
            tgt, _ = O.match(K[0, h].astype(np.float64), np.arange(budget), np.arange(budget, cap), T, exact_any_order=True)
            np.testing.assert_array_equal(match[0, h].cpu().numpy(), tgt)
    near = torch.full((1, 2, cap), -9, dtype=torch.int32, device="cuda")
    kk.prefill_match(lay, c, T, near, None, ws)
    torch.cuda.synchronize()
    for h in range(2):
        ref, _ = O.prefill_nearest_earlier(K[0, h].astype(np.float64), cap, T, exact_any_order=True)
        np.testing.assert_array_equal(near[0, h].cpu().numpy(), ref)

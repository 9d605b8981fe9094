"""The matrix-core decode kernel for every group size: how its lanes share the slots of a tile.

16 / G lanes of a head share the 32 slots of a tile (G / 2 of every 8 per lane, one for G = 1 and 2), so every G and head dim
lays out its products differently.  Each is compared with the oracle (Eq. 6, Eq. 8; tolerances of the other decode tests)
as a single tile and as two tiles per wavefront, as a tile loop whose running maximum keeps rising (every tile rescales), and with
infinities among the values.
"""
import numpy as np
import pytest
import torch

from oracle import keepkv_oracle as O
from paper_2504_09936_amd import workloads as W
from tests import gpu_util as U
from tests import test_gpu_decode_instances as I

pytestmark = pytest.mark.gpu
CAP = 613                                            # 19 tiles and 5 slots


def _workload(G, D):
    return W.CONFIGS["llama3_8b"].scaled(batch=2, n_q_heads=3 * G, n_kv_heads=3, head_dim=D, context=CAP)


@pytest.mark.parametrize("waves,per", [(4, 128), (8, 256), (4, 224), (8, 320), (4, 640)])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_step(G, D, waves, per):
    w = _workload(G, D)
    g = np.random.default_rng(G * 100 + D)
    lens, _ = I._ragged_lens(g, w.batch, w.n_kv_heads, CAP, per, -(-CAP // per))
    lay, c = I._steady_state(w, CAP, 19, lens)
    c.plan_wavefronts, c.plan_slots_per_split = waves, per
    ws = I._workspace_for(lay, CAP, per)
    I._check_steps(w, lay, c, ws, list(range(w.batch * w.n_kv_heads)), 2, 19, hint=waves == 8, tag=(G, D, waves, per))


def _attend(w, lay, c, q, waves, per):
    kk = U.kk()
    c.plan_wavefronts, c.plan_slots_per_split = waves, per
    out = torch.zeros(w.batch, w.n_q_heads, w.head_dim, dtype=lay.torch_dtype, device="cuda")
    kk.decode_attn(lay, c, U.to_device(q, w.dtype), out, None, None, I._workspace_for(lay, CAP, per))
    torch.cuda.synchronize()
    return U.to_host(out)


@pytest.mark.parametrize("waves,cap", [(4, 120), (8, 250), (4, 250), (8, 500)])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_unsplit(G, D, waves, cap):
    """Heads that are not split, in one and in two tiles a wavefront: a kernel without combination."""
    kk = U.kk()
    w = _workload(G, D).scaled(context=cap)
    g = np.random.default_rng(G * 100 + D + cap)
    lens, _ = I._ragged_lens(g, w.batch, w.n_kv_heads, cap, cap, 1)
    lay, c = I._steady_state(w, cap, 29, lens)
    c.plan_wavefronts, c.plan_slots_per_split = waves, (cap + 31) // 32 * 32
    q = W.make_query(w, 29, 7)
    out = torch.zeros(w.batch, w.n_q_heads, D, dtype=lay.torch_dtype, device="cuda")
    lse = torch.zeros(w.batch, w.n_q_heads, device="cuda")
    kk.decode_attn(lay, c, U.to_device(q, w.dtype), out, None, lse, None)
    o_ref, lse_ref, _ = O.attend(U.download(c), q.astype(np.float64), w.scale)
    assert U.storage_err_rows(U.to_host(out), o_ref, w.dtype).max() <= I.TOL
    live = np.repeat(lens > 0, G, axis=1)
    np.testing.assert_allclose(lse.cpu().numpy()[live], lse_ref[live], rtol=1e-4, atol=2e-3)
    I._check_steps(w, lay, c, None, list(range(w.batch * w.n_kv_heads)), 2, 29, hint=waves == 8, tag=(G, D, waves, cap))


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_rising_maximum(G, D):
    """Keys that point ever more along the head's first query: every tile of the loop raises the maximum."""
    w = _workload(G, D)
    lens = np.full((w.batch, w.n_kv_heads), CAP, np.int32)
    lay, c = I._steady_state(w, CAP, 23, lens)
    q = W.make_query(w, 23, 0)
    along = torch.from_numpy(q.reshape(w.batch, w.n_kv_heads, G, D)[:, :, 0].astype(np.float32)).cuda()
    ramp = torch.linspace(-1.0, 1.0, CAP, device="cuda").view(1, 1, CAP, 1)
    c.k.copy_(c.k.float() * 0.3 + ramp * along.unsqueeze(2))
    oc = U.download(c)
    o_ref, _, _ = O.attend(oc, q.astype(np.float64), w.scale)
    for waves, per in ((4, 640), (8, 640)):
        err = U.storage_err_rows(_attend(w, lay, c, q, waves, per), o_ref, w.dtype)
        assert err.max() <= I.TOL, (G, D, waves, float(err.max()))


@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_infinite_value_stays_infinite(G):
    """One infinite element in V, at a slot whose weight is neither zero nor the largest: the head's channel is infinite and
    nothing else changes."""
    w = _workload(G, 128)
    lens = np.full((w.batch, w.n_kv_heads), CAP, np.int32)
    lay, c = I._steady_state(w, CAP, 29, lens)
    q = 0.05 * W.make_query(w, 29, 0)                # flat weights: none vanishes
    q = W.round_storage(q, w.dtype)
    c.k[:, :, 77] = 0                                # (the largest weight of a tile is exactly 1: its low bf16 part is zero)
    c.votes[:, :, 77] = 1
    before = _attend(w, lay, c, q, 8, 256)
    c.v[:, :, 77, 5] = float("inf")
    for waves, per in ((8, 256), (4, 640)):
        got = _attend(w, lay, c, q, waves, per)
        assert np.isposinf(got[:, :, 5]).all(), (G, waves, per)
        keep = np.arange(128) != 5
        np.testing.assert_allclose(got[:, :, keep], before[:, :, keep], rtol=2 ** -7, atol=1e-6)

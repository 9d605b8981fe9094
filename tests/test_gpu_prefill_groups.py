"""keepkv_prefill_merge on given links: which slots stay, what each absorbs (votes) and in which order they are listed.

The expected grouping follows the definition slot by slot: a slot is absorbed by the slot it links to unless that one is
itself absorbed.  Links from none at all to one chain through every slot (the pointer jumping then needs all its rounds),
sizes around a 64-slot chunk, around the 1024 threads of a workgroup and beyond the LDS limit.
"""
import numpy as np
import pytest
import torch

from tests import gpu_util as U

pytestmark = pytest.mark.gpu


def _links(kind, n, g):
    near = np.full(n, -1, np.int32)
    if kind == "chain":
        near[1:] = np.arange(n - 1)
    elif kind == "sparse":
        i = np.flatnonzero(g.random(n) < 0.05)
        i = i[i > 0]
        near[i] = (g.random(i.size) * i).astype(np.int32)
    elif kind == "forest":
        near[1:] = np.where(g.random(n - 1) < 0.7, np.arange(1, n) - 1 - (g.random(n - 1) * np.minimum(np.arange(1, n), 40)).astype(int), -1)
    elif kind == "star":
        near[1:] = 0
    return near


@pytest.mark.parametrize("kind", ["none", "sparse", "forest", "star", "chain"])
@pytest.mark.parametrize("cap", [63, 65, 1000, 1025, 8191, 16384, 20000])
def test_groups(cap, kind):
    kk = U.kk()
    B, H, D = 1, 3, 64
    lay = kk.Layout(B, H, H, D, kk.BF16, 0.125)
    g = np.random.default_rng(cap)
    lens = np.array([[cap, max(1, cap - 37), cap // 2 + 1]], np.int32)
    src, dst = kk.Cache(lay, cap), kk.Cache(lay, cap)
    src.k.copy_(torch.arange(cap, device="cuda").view(1, 1, cap, 1).expand_as(src.k) % 128)     # (exact in bf16)
    src.v.copy_(src.k)
    src.votes.fill_(1)
    src.log_s.zero_()
    src.t_obs.fill_(32)
    src.len.copy_(torch.from_numpy(lens))
    near = np.stack([_links(kind, cap, g) for _ in range(H)])[None]
    ws = kk.new_workspace(lay, cap, max(1, cap // 10))
    kk.prefill_merge(lay, src, dst, torch.from_numpy(near).cuda(), 0.9, ws)
    torch.cuda.synchronize()
    for h in range(H):
        n = int(lens[0, h])
        absorbed, votes = np.zeros(n, bool), np.ones(n, np.int64)
        for i in range(n):
            t = near[0, h, i]
            if t >= 0 and not absorbed[t]:
                absorbed[i] = True
                votes[t] += 1
        stay = np.flatnonzero(~absorbed)
        assert int(dst.len[0, h]) == stay.size, (cap, kind, h)
        np.testing.assert_array_equal(dst.votes[0, h, : stay.size].cpu().numpy(), votes[stay])
        alone = votes[stay] == 1                       # copied bit for bit: the row names its slot
        np.testing.assert_array_equal(dst.v[0, h, : stay.size, 0].float().cpu().numpy()[alone], (stay % 128)[alone])

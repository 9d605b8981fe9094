"""Heads whose splits are combined within one XCD: the same bits as through memory (a workspace of the documented least
size leaves no room for the former), whatever the workgroups find when they look where the others run."""
import pytest
import torch

from tests import gpu_util as U

pytestmark = pytest.mark.gpu
HEAD = 64 * 1024 + 256       # control words at the head of a workspace (keepkv.h)
ARRIVALS = 32 * 1024         # of which: one 64-bit word per head, from here on


def _state(kk, lay, cap, n):
    gen = torch.Generator(device="cuda").manual_seed(7)
    c = kk.Cache(lay, cap)
    for t in (c.k, c.v):
        t.normal_(generator=gen)
    c.votes.random_(1, 6, generator=gen)
    c.log_s.normal_(generator=gen)
    c.len.copy_(torch.randint(n // 2, n + 1, c.len.shape, generator=gen, device="cuda"))
    c.len[0, 0] = cap                       # a full head: attended without its new token
    c.len[0, 1] = 1
    return c


# heads a multiple of 8, one tile a wavefront or (the last three and where the chip is full) two; 256 heads: more workgroups than the chip
# holds, so that the first ones of a head may be done before its last ones start; 1200 slots: a short last split, which looks early
@pytest.mark.parametrize("G,D,heads,cap,per,waves", [(4, 128, 64, 884, 0, 0), (4, 128, 8, 884, 128, 8), (8, 64, 16, 300, 64, 4),
                                                     (1, 128, 8, 700, 96, 4), (2, 64, 8, 2000, 512, 8), (8, 128, 64, 600, 256, 4),
                                                     (4, 128, 16, 1000, 64, 8), (4, 64, 256, 700, 64, 4), (4, 128, 8, 1200, 224, 8),
                                                     (2, 128, 8, 1000, 64, 8), (8, 128, 8, 1700, 128, 8),
                                                     (4, 128, 64, 1500, 0, 0), (1, 64, 96, 700, 0, 0), (2, 128, 64, 700, 256, 4), (4, 128, 128, 836, 0, 0)])
def test_same_bits_as_through_memory(G, D, heads, cap, per, waves):
    kk = U.kk()
    lay = kk.Layout(heads // 8, 8 * G, 8, D, kk.BF16, D ** -0.5)
    gen = torch.Generator(device="cuda").manual_seed(3)
    q = torch.randn(heads // 8, 8 * G, D, generator=gen, device="cuda").bfloat16()
    k_t, v_t = (torch.randn(heads // 8, 8, D, generator=gen, device="cuda").bfloat16() for _ in range(2))
    ns = kk.decode_plan(lay, cap)[0] if per == 0 else -(-cap // per)
    assert ns > 1
    least = HEAD + heads * G * ns * (D + 2) * 4
    results = []
    elsewhere = torch.tensor([1 << 8 * ((u + 1) % 8) for u in range(heads)], device="cuda")   # (workgroups come to the XCDs in turn)
    marked = torch.full((heads,), -1 << 63, device="cuda")
    for size, found in ((least, None), (2 * least + 65536, None), (2 * least + 65536, marked), (2 * least + 65536, elsewhere)):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        c = _state(kk, lay, cap, cap - 5)
        c.plan_slots_per_split, c.plan_wavefronts = per, waves
        out = torch.zeros_like(q)
        kk.workspace_init(ws)
        for _ in range(3):
            if found is not None:               # as if a workgroup had found its head incomplete / ran on another XCD
                ws[ARRIVALS:ARRIVALS + 8 * heads].view(torch.int64).copy_(found)
            kk.decode_step(lay, c, q, k_t, v_t, out, None, 0.9, None, ws)
            assert not ws[:HEAD].any()
        results.append((out.clone(), c.log_s.clone(), c.len.clone(), c.k.clone(), c.v.clone(), c.votes.clone()))
    assert results[0][0].float().abs().sum() > 0
    for r in results[1:]:
        for a, b in zip(results[0], r):
            assert torch.equal(a, b)


# one tile a wavefront; two, in four and in two splits
@pytest.mark.parametrize("G,D,heads,cap", [(4, 128, 64, 884), (8, 64, 8, 500), (4, 128, 64, 1500), (1, 64, 96, 700), (4, 128, 128, 836)])
def test_the_route_is_taken(G, D, heads, cap):
    """Tickets of the route through memory that can never complete (far below zero; nothing waits for them): a head that meets within
    its XCD leaves its own alone and has its result, any other has added to it.  Workgroups come to the XCDs in turn, so that most
    heads should be of the first kind; one is asked for, so that the test above does not compare the other route with itself."""
    kk = U.kk()
    lay = kk.Layout(heads // 8, 8 * G, 8, D, kk.BF16, D ** -0.5)
    gen = torch.Generator(device="cuda").manual_seed(5)
    q = torch.randn(heads // 8, 8 * G, D, generator=gen, device="cuda").bfloat16()
    k_t, v_t = (torch.randn(heads // 8, 8, D, generator=gen, device="cuda").bfloat16() for _ in range(2))
    ns = kk.decode_plan(lay, cap)[0]
    assert ns > 1
    ws = kk.new_workspace(lay, cap, cap // 2)
    results = []
    for planted in (0, -1 << 20):
        c = _state(kk, lay, cap, cap - 5)
        out = torch.full_like(q, 3.0)
        tickets = ws[:4 * heads].view(torch.int32)
        tickets.fill_(planted)
        kk.decode_step(lay, c, q, k_t, v_t, out, None, 0.9, None, ws)
        results.append((out.view(heads, -1), c.len.flatten()))
        left = tickets.clone()
        kk.workspace_init(ws)
    within = left == planted
    assert ((left == planted) | (left == planted + ns)).all()
    assert within.any(), "every head went through memory"
    print(int(within.sum()), "of", heads, "heads within an XCD")
    for a, b in zip(*results):
        assert torch.equal(a[within], b[within])

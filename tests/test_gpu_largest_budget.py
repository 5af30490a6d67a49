"""Block-wise steps at the largest budget, 2^24 slots: a unit's keys of bf16 / 128 are 4 GiB, more than 32-bit offsets reach."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

B, D = 1 << 24, 128


def _attention(q, K, V, n, hide=None):
    """One query row in fp32 over slots [0, n) but `hide`, without a copy of the cache in fp32."""
    t = torch.cat([K[i:i + (1 << 21)].float() @ q for i in range(0, n, 1 << 21)])[:n] / math.sqrt(D)
    if hide is not None:
        t[hide] = float("-inf")
    p = torch.softmax(t, dim=0)
    out = torch.zeros(D, device="cuda")
    for i in range(0, n, 1 << 21):
        out += p[i:i + (1 << 21)] @ V[i:min(n, i + (1 << 21))].float()
    return out, p


@pytest.mark.parametrize("block,used", [(1, B - 1), (1, B), (2, B)])
def test_steps_of_the_largest_cache(block, used):
    import paper_2402_06262_amd as roco
    g = torch.Generator(device="cuda").manual_seed(block + used)
    p = roco.RocoParams(1, D, B, 40, roco.ROCO_BF16)
    c = roco.alloc_cache(p)
    for plane in (c.K, c.V):
        plane.normal_(generator=g)
    q, k, v = (torch.randn((1, block, D), generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    q[0] = q[0, 0]  # one direction for the block's queries, so that planted keys stand out for all of them
    places = [0, 33, (1 << 22) - 1, 1 << 22, (1 << 23) - 1, 1 << 23, (1 << 23) + 31, (1 << 24) - 65, (1 << 24) - 3]
    for i, slot in enumerate(places):
        c.K[0, slot] = q[0, 0] * (3.0 + 0.01 * i)
    c.stats[:, 0].uniform_(1.0, 2.0, generator=g)  # positive scores, variance the larger the later the slot: slots 0 .. are in scope
    c.stats[:, 2] = 4.0
    c.stats[:, 1] = c.stats[:, 0].square() / 4.0 + torch.linspace(1.0, 2.0, B, device="cuda")
    first = [70, 71]  # the lowest mean scores, in the scope
    c.stats[0, 0, first] = torch.tensor([0.25, 0.5], device="cuda")
    c.stats[0, 1, first] = 0.0
    c.pos.copy_(torch.arange(B, dtype=torch.int32, device="cuda"))
    c.n_used.fill_(used)
    taken = (1 << 23) + 5 if used == B else B - 1  # of a single token
    c.next_slot.fill_(taken if used == B else -1)
    slots = [taken] if block == 1 else first
    before = c.stats[0].clone()
    out = torch.empty((1, block, D), dtype=torch.bfloat16, device="cuda")
    es, ep = (torch.empty((1, block), dtype=torch.int32, device="cuda") for _ in range(2))
    ws = torch.empty(roco.block_workspace_bytes(p, block), dtype=torch.uint8, device="cuda")
    qpos = torch.full((1,), B, dtype=torch.int32, device="cuda")
    roco.roco_encode_block(p, block, q, k, v, qpos, c.K, c.V, c.stats, c.pos, c.n_used, c.next_slot, out, es, ep, ws)
    torch.cuda.synchronize()
    assert es[0].tolist() == (slots if used == B else [-1]) and ep[0].tolist() == (slots if used == B else [-1])
    assert torch.equal(c.K[0, slots], k[0]) and torch.equal(c.V[0, slots], v[0]) and c.n_used.item() == B
    acc = before[0]
    acc[slots] = 0.0
    for i in range(block):
        want, prob = _attention(q[0, i].float(), c.K[0], c.V[0], B, hide=slots[i + 1:])
        # bf16 rounds the probabilities and the output (2^-9 each); the planted keys carry nearly all of the weight
        assert torch.allclose(out[0, i].float(), want, rtol=2 ** -7, atol=2 ** -7 * want.abs().max().item())
        acc += prob
    assert torch.allclose(c.stats[0, 0], acc, rtol=1e-5, atol=1e-6)

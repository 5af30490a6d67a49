"""Block and grouped steps of bf16 on values that show what a probability is multiplied as: infinities, differences far below the
precision of a bf16 number, and queries of NaN."""
import pytest
import torch

pytestmark = pytest.mark.gpu

PATHS = {"8": "eight-waves", "4": "four-waves", "2": "halves", "0": "three-kernels"}


@pytest.fixture(params=list(PATHS), ids=list(PATHS.values()))
def kernels(request, monkeypatch):
    monkeypatch.setenv("ROCO_BLOCK_FUSED", request.param)
    return request.param


def _step(d, K, V, q, k_new, v_new, importance, scope_kind):
    """One step of full caches whose positions are those of their slots: the oldest tokens go.  (out, cache)"""
    import paper_2402_06262_amd as roco
    units, B, _ = K.shape
    block, group = q.shape[1:3]
    p = roco.RocoParams(units, d, B, 1, roco.ROCO_BF16, importance=importance, scope_kind=scope_kind)
    c = roco.alloc_cache(p)
    c.K.copy_(K)
    c.V.copy_(V)
    c.pos.copy_(torch.arange(B, device="cuda", dtype=torch.int32).expand(units, B))
    c.n_used.fill_(B)
    c.stats[:, 0], c.stats[:, 1], c.stats[:, 2] = 1.0, 1.0, 8.0
    c.next_slot.zero_()
    ws = torch.empty(roco.block_workspace_bytes(p, block), dtype=torch.uint8, device="cuda")
    out = torch.zeros((units, block, group, d), dtype=torch.bfloat16, device="cuda")
    qpos = torch.full((units,), B, dtype=torch.int32, device="cuda")
    roco.roco_encode_block_gqa(p, block, group, q, k_new, v_new, qpos, c.K, c.V, c.stats, c.pos, c.n_used, c.next_slot, out, None, None, ws)
    torch.cuda.synchronize()
    return out.float(), c


def _reference(c, q, block):
    """Outputs in 64 bits from the rows that the step has left in the cache: query i sees the block's tokens 0..i."""
    units, B, d = c.K.shape
    x = torch.einsum("utgd,ubd->utgb", q.double().cpu(), c.K.double().cpu()) / d ** 0.5
    tok = (c.pos.cpu() - B)[:, None, None, :]  # of the block's tokens; negative: an older one
    seen = tok <= torch.arange(block)[None, :, None, None]
    return torch.softmax(x.masked_fill(~seen, float("-inf")), dim=-1), seen


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("B,block,group", [(192, 1, 4), (1024, 5, 3), (2048, 16, 1), (2048, 1, 8), (512, 32, 1), (1100, 27, 1), (1536, 16, 4)])
def test_infinite_values_stay_infinite(B, block, group, d, kernels):
    """An infinite value of a token that a query attends makes that component of its output the same infinity, whatever the token's
    probability (2^-100 of the largest included); two of opposite signs make it NaN, and the other components stay finite."""
    units = 17
    g = torch.Generator(device="cuda").manual_seed(B + block)
    rnd = lambda *shape: torch.randn(shape, generator=g, device="cuda").bfloat16()
    K, V = rnd(units, B, d), rnd(units, B, d)
    q, k_new, v_new = rnd(units, block, group, d), rnd(units, block, d), rnd(units, block, d)
    inf = float("inf")
    infinite = torch.zeros((units, d), device="cuda")
    q[..., 0] = 8.0
    K[..., 0] = k_new[..., 0] = 0.0
    for u in range(units - 1):
        slots = torch.randperm(B - 64, generator=g, device="cuda")[:d - 8] + 64  # (the oldest tokens, which go, lie below)
        for i in range(0, d - 8, 3):
            V[u, slots[i], i] = infinite[u, i] = inf if i % 2 else -inf
        K[u, slots[3], 0] = -60.0 * d ** 0.5 / 8.0  # 2^-87 of the others
        if u % 2:
            V[u, slots[4], 6] = inf
            infinite[u, 6] = float("nan")
    v_new[:, 0, d - 1] = infinite[:, d - 1] = inf  # the first token of the block is seen by all of its queries
    out, c = _step(d, K, V, q, k_new, v_new, 2, 2)
    held = torch.isinf(c.V.float()).sum((1, 2))
    assert (held >= torch.isinf(infinite).sum(1)).all()  # no infinite value has been evicted
    want = infinite[:, None, None].expand_as(out)
    same = torch.where(want == 0, torch.isfinite(out), (out == want) | (torch.isnan(out) & torch.isnan(want)))
    bad = (~same).nonzero()
    assert bad.numel() == 0, (bad[:8].tolist(), out[tuple(bad[0].tolist())].item(), len(bad))


@pytest.mark.parametrize("B,block,group", [(256, 16, 1), (1024, 1, 5), (2048, 4, 4), (256, 30, 1), (1536, 13, 4)])
def test_probabilities_of_head_dim_64_keep_their_bits(B, block, group, kernels):
    """Neighbouring slots differ by 2^-12 in their logits and have values of 1 and -1: an output is the difference of two
    probabilities, 2^-12 of them.  Logits of up to 8 round by 2^-22.5 of a probability, exponentials by 2^-23, each twice: 2^-8.8 of
    the difference, and bf16 rounds it by 2^-9; held to the double of the sum.  (16 bits of the probabilities: 0.06, 8 bits: 30.)"""
    units, d = 17, 64
    g = torch.Generator(device="cuda").manual_seed(B + block)
    rnd = lambda *shape: torch.randn(shape, generator=g, device="cuda").bfloat16()
    K, V = rnd(units, B, d), torch.zeros((units, B, d), device="cuda").bfloat16()
    q, k_new, v_new = rnd(units, block, group, d), rnd(units, block, d), torch.zeros((units, block, d), device="cuda").bfloat16()
    q[..., 0] = 0.25
    K[:, 1::2] = K[:, 0::2]
    K[:, 0::2, 0], K[:, 1::2, 0] = 1.0, 1.0 + 2.0 ** -7
    for i in range(d):
        V[:, 64 + 2 * i, i], V[:, 65 + 2 * i, i] = 1.0, -1.0
    out, c = _step(d, K, V, q, k_new, v_new, 2, 2)
    prob, _ = _reference(c, q, block)
    want = torch.einsum("utgb,ubd->utgd", prob, c.V.double().cpu())
    worst = ((out.double().cpu() - want).abs() / want.abs()).max().item()
    assert worst <= 2.0 ** -7, worst


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("B,block,group", [(256, 16, 1), (1024, 5, 3), (2048, 16, 1), (2048, 27, 1), (1024, 16, 4), (2048, 40, 1)])
def test_a_query_of_nan_leaves_later_tokens_alone(B, block, group, d, kernels):
    """The statistics of a block's tokens behind a query of NaN, which does not see them, come from the queries that do."""
    units, at = 17, block // 2
    g = torch.Generator(device="cuda").manual_seed(B + block)
    rnd = lambda *shape: torch.randn(shape, generator=g, device="cuda").bfloat16()
    K, V, q = rnd(units, B, d), rnd(units, B, d), rnd(units, block, group, d)
    q[:, at] = float("nan")
    out, c = _step(d, K, V, q, rnd(units, block, d), rnd(units, block, d), 2, 2)
    tok = c.pos - B
    later = tok > at
    assert (later.sum(1) == block - 1 - at).all()
    prob, seen = _reference(c, q, block)
    mean = torch.where(seen, prob, 0.0).mean(2)  # [units, block, B] of the heads
    for plane, want in ((0, mean), (1, mean ** 2)):
        want = torch.where(tok.cpu()[:, None] <= torch.arange(block)[None, :, None], want, 0.0).sum(1)
        got = c.stats[:, plane].double().cpu()
        rel = ((got - want).abs() / want.abs().clamp_min(1e-6))[later.cpu()]
        assert torch.isfinite(got[later.cpu()]).all(), plane
        assert rel.max().item() <= 1e-4
    assert torch.isnan(c.stats[:, 0][~later & (tok < at)]).all() and torch.isnan(out[:, at]).all() and torch.isfinite(out[:, :at]).all()

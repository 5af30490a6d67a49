"""Steps of bf16 in one kernel (two above 32 query rows) and in three: the same step, at the edges of the tiles, of the waves' shares
and of the logits that registers and LDS hold."""
import pytest
import torch

import test_gpu_gqa as TG

pytestmark = pytest.mark.gpu


@pytest.fixture(params=["8", "4", "2", "0"], ids=["eight-waves", "four-waves", "halves", "three-kernels"])
def kernels(request, monkeypatch):
    monkeypatch.setenv("ROCO_BLOCK_FUSED", request.param)
    return request.param


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("B", [4, 28, 32, 36, 124, 128, 132, 256, 260, 1028])
def test_caches_that_end_at_the_edges_of_the_tiles(B, d, kernels):
    """From the first token on, in lock-step with the oracle: 1 to 16 rows; up to 32; up to 64.  Nine units where some of them evict
    behind the scores and stream V before the statistics (every other eight units of more than four tiles a wave).  Halves of 1 to 32
    rows are those of head_dim 128 from 17 on; above 32 rows halves are what eight and four waves mean too."""
    s = max(1, B // 8)
    units = 9 if B > 512 else 2
    fill = [16] * (B // 16) + [7, 1, 16, 9, 1] if B >= 16 else [3, 4, 1, 2, 1]
    if kernels != "2":
        TG.drive(units, B, s, 1, [min(b, B) for b in fill], seed=900 + B, recency=B % 128 == 4, tag=f"edge-{B}-{d}", d=d)
    if B >= 16 and (kernels != "2" or d == 128):
        TG.drive(units, B, s, 4, [8] * min(B // 8, 20) + [8, 1, 4, 1], seed=950 + B, tag=f"edge-{B}-{d}-g4", d=d)
    if B >= 16 and kernels in "20":
        TG.drive(9, B, s, 4, [min(16, B)] * min(B // 16, 6) + [13, 9, 1], seed=970 + B, recency=B % 64 == 0, tag=f"edge-{B}-{d}-halves", d=d)


POLICIES = [(0, 0, 0), (1, 2, 0), (0, 1, 0), (2, 2, 4), (3, 2, 0), (4, 1, 0)]  # importance, scope kind, sinks


def _seed(B, block, group):
    return B + 64 * block + group


def _paths(B, block, group, d):
    """The values of ROCO_BLOCK_FUSED that take the step to kernels of their own: eight waves, four, halves."""
    squares = POLICIES[_seed(B, block, group) % len(POLICIES)][0] < 3
    rows, half, split = block * group, (block + 1) // 2 * group, block > 1 and squares
    if rows > 32:
        return ["8"] if split and half <= 32 and B <= 2048 else []
    if rows > 16:
        return ["8"] * (B <= 2048) + ["4"] * (B <= 1024) + ["2"] * (split and half <= 16 and d == 128 and B <= 2048)
    return ["8"] * (B <= 4096) + ["4"] * (B <= 2048)


@pytest.mark.parametrize("B,block,group,d", [
    (B, block, group, d) for d in (128, 64) for B in (508, 512, 516, 1020, 1024, 1028, 2044, 2048, 2052, 4096)
    for block, group in [(1, 1), (1, 4), (1, 16), (16, 1), (3, 5), (2, 8), (1, 17), (32, 1), (5, 6), (6, 5), (33, 1), (64, 1), (16, 4), (3, 16), (9, 7), (17, 3)]
    if _paths(B, block, group, d)])
def test_one_kernel_and_three_take_the_same_step(B, block, group, d, monkeypatch):
    """Caches from full to nearly empty, with a recency bias and without, under every kind of policy, in units of both orders of phases:
    the same slots and positions bit for bit, and the next victim that the statistics left by the step have.  Tolerances: bf16 outputs
    differ by a rounding or two (2^-7 of the row's largest); the statistics by fp32 sums in another order (a logit of up to 2^7 in
    powers of two has an error of 2^-16, which is that of the probability)."""
    import paper_2402_06262_amd as roco
    units, seed = 20, _seed(B, block, group)
    g = torch.Generator(device="cuda").manual_seed(seed)
    rnd = lambda *shape: torch.randn(shape, generator=g, device="cuda")
    imp, kind, sinks = POLICIES[seed % len(POLICIES)]
    window = 64 if (B // 4 + block + group) % 3 == 0 else 0
    p = roco.RocoParams(units, d, B, max(1, B // 8), roco.ROCO_BF16, 0.0, window, 0.5 if window else 0.0, imp, kind, sinks)
    fills = torch.tensor([B, B - 1, B // 2 + 1, max(0, B - block), 0] * (units // 5), dtype=torch.int32, device="cuda")
    live = torch.arange(B, device="cuda")[None] < fills[:, None]
    K, V = rnd(units, B, d).bfloat16(), rnd(units, B, d).bfloat16()
    count = (1.0 + torch.randint(0, 100, (units, B), generator=g, device="cuda")).float()
    acc = torch.rand((units, B), generator=g, device="cuda") * count * 0.01
    stats = torch.stack([acc, acc * acc / count * (1.0 + torch.rand((units, B), generator=g, device="cuda")), count], 1)
    pos = torch.where(live, torch.arange(B, device="cuda", dtype=torch.int32)[None], -1).int()
    q = rnd(units, block, group, d).bfloat16()
    k_new, v_new = rnd(units, block, d).bfloat16(), rnd(units, block, d).bfloat16()
    wd = torch.empty(roco.decode_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    got = {}
    for path in ["0", *_paths(B, block, group, d)]:
        monkeypatch.setenv("ROCO_BLOCK_FUSED", path)
        c = roco.alloc_cache(p)
        c.K.copy_(K); c.V.copy_(V); c.stats.copy_(stats * live[:, None]); c.pos.copy_(pos); c.n_used.copy_(fills)
        ws = torch.full((roco.block_workspace_bytes(p, block),), 0xFF, dtype=torch.uint8, device="cuda")
        roco.roco_select_victims(p, c.stats, c.pos, c.n_used, c.next_slot, wd)
        out = torch.zeros((units, block, group, d), dtype=torch.bfloat16, device="cuda")
        es, ep = (torch.full((units, block), -7, dtype=torch.int32, device="cuda") for _ in range(2))
        finishing = _count(10, lambda: roco.roco_encode_block_gqa(p, block, group, q, k_new, v_new, fills.clone(), c.K, c.V, c.stats, c.pos,
                                                                  c.n_used, c.next_slot, out, es, ep, ws))
        assert finishing == (path == "0"), path
        chosen = torch.full_like(c.next_slot, -9)
        roco.roco_select_victims(p, c.stats, c.pos, c.n_used, chosen, wd)
        torch.cuda.synchronize()
        got[path] = dict(K=c.K, V=c.V, pos=c.pos, n_used=c.n_used, es=es, ep=ep, out=out.float(), stats=c.stats)
        assert torch.equal(c.next_slot, chosen), (path, "next victim")
    a = got.pop("0")
    for path, b in got.items():
        for name in ("K", "V", "pos", "n_used", "es", "ep"):
            same = torch.equal(a[name], b[name])
            assert same, (path, name)
        bad = ((a["out"] - b["out"]).abs().amax(-1) > 2.0 ** -7 * a["out"].abs().amax(-1)).any().item()
        assert not bad, (path, "out")
        held = torch.arange(B, device="cuda")[None] < b["n_used"][:, None]
        for i in range(3):
            x, y = a["stats"][:, i][held], b["stats"][:, i][held]
            if i == 1 and imp == 4:  # counts of probabilities above average: one within 1e-4 of it may fall on either side
                assert ((x - y).abs() > 0).float().mean().item() < 0.002 and ((x - y).abs().max().item() <= 1.0)
            else:
                rel = ((x - y).abs() / x.abs().clamp_min(1e-6)).max().item() if x.numel() else 0.0
                assert rel <= (0.0 if i == 2 else 1e-4), (path, i, rel)


def _count(kernel, run):
    """How often `run` launches a kernel, by the profiling aid."""
    import paper_2402_06262_amd as roco
    roco.roco_profile_kernel(kernel)
    try:
        run()
        return roco.roco_profile_read()[1]
    finally:
        roco.roco_profile_kernel(-1)


def _launches(run):
    """How often `run` launches the preparing, the attention and the finishing kernel of a block step."""
    return [_count(kernel, run) for kernel in (8, 9, 10)]  # ROCO_PROF_BLOCK_PREPARE, _ATTEND, _FINISH


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("block,group,default,prepared,split", [(1, 4, [0, 1, 0], [1, 1, 1], [0, 1, 1]), (1, 1, [0, 1, 0], [1, 1, 1], [0, 1, 1]),
                                                                (5, 3, [0, 1, 0], [0, 1, 0], [1, 1, 1]), (12, 4, [0, 1, 0], [0, 1, 0], [1, 1, 1])])
def test_switches_choose_the_kernels(block, group, default, prepared, split, d, monkeypatch):
    """As include/roco.h says: no preparing kernel left out of a single token that asks for it, splits in the kernels that have them, and
    none asked for by 0."""
    import paper_2402_06262_amd as roco
    units, B = 3, 256
    p = roco.RocoParams(units, d, B, 16, roco.ROCO_BF16)
    c = roco.alloc_cache(p)
    ws = torch.empty(roco.block_workspace_bytes(p, block), dtype=torch.uint8, device="cuda")
    q = torch.randn((units, block, group, d), device="cuda").bfloat16()
    k = torch.randn((units, block, d), device="cuda").bfloat16()
    at = torch.zeros(units, dtype=torch.int32, device="cuda")

    def run():
        roco.roco_encode_block_gqa(p, block, group, q, k, k, at, c.K, c.V, c.stats, c.pos, c.n_used, c.next_slot, torch.empty_like(q), None,
                                   None, ws)

    for env, want in (({}, default), ({"ROCO_BLOCK_SPLITS": "0"}, default), ({"ROCO_BLOCK_SPLITS": ""}, default),
                      ({"ROCO_BLOCK_SINGLE": "0"}, prepared), ({"ROCO_BLOCK_SINGLE": "1"}, default), ({"ROCO_BLOCK_SPLITS": "2"}, split),
                      ({"ROCO_BLOCK_FUSED": "0"}, split), ({"ROCO_BLOCK_FUSED": "8", "ROCO_BLOCK_SPLITS": "2"}, default)):
        with monkeypatch.context() as m:
            for name, value in env.items():
                m.setenv(name, value)
            got = _launches(run)
        assert got == want, (env, got)

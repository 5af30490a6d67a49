"""The k-smallest search behind every eviction, through calls whose statistics the test chooses: keys that share digits, ties
across the boundary, more candidates than are searched directly, and prompts whose ranking keys leave LDS one by one."""
import numpy as np
import pytest
import torch

from oracle import roco_oracle as orc

pytestmark = pytest.mark.gpu


def _keys(kind, n, rng):
    if kind == "equal":
        return np.full(n, 0.25, np.float32)
    if kind == "low_bits":  # one value but for the lowest three bits: all three digits are counted, ties in each
        return (np.float32(1.5).view(np.uint32) + rng.integers(0, 8, n).astype(np.uint32)).view(np.float32)
    if kind == "middle_bits":
        return (np.float32(1.5).view(np.uint32) + (rng.integers(0, 700, n).astype(np.uint32) << 9)).view(np.float32)
    if kind == "two_values":
        return np.where(rng.random(n) < 0.5, np.float32(0.0), np.float32(3e38)).astype(np.float32)
    return np.exp(rng.uniform(-60, 60, n)).astype(np.float32)


@pytest.mark.parametrize("kind", ["equal", "low_bits", "middle_bits", "two_values", "wide"])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 128, 129, 1024, 2047, 4100, 16384, 16400])
def test_lowest_keys_go_first_and_ties_by_slot(kind, n):
    import paper_2402_06262_amd as roco
    rng = np.random.default_rng([n, len(kind)])
    units = 3
    p = roco.RocoParams(units, 64, n, 1, roco.ROCO_F32, importance=roco.ROCO_IMPORTANCE_AAS, scope_kind=roco.ROCO_SCOPE_ALL)
    acc = np.stack([_keys(kind, n, rng) for _ in range(units)])
    stats = torch.from_numpy(np.stack([acc, acc, np.ones_like(acc)], axis=1)).cuda()
    n_used = torch.full((units,), n, dtype=torch.int32, device="cuda")
    mask = torch.empty((units, n), dtype=torch.int32, device="cuda")
    ws = torch.empty(roco.decode_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    order = np.argsort(acc, axis=1, kind="stable")
    for keep in sorted({n - 1, n // 2, n // 3, max(0, n - 129), min(n, 1), 0}):
        roco.roco_select_retained(p, keep, stats, None, n_used, mask, ws)
        want = np.ones((units, n), np.int32)
        for u in range(units):
            want[u, order[u, :n - keep]] = 0
        assert np.array_equal(mask.cpu().numpy(), want), (kind, n, keep)
    victim = torch.empty((units,), dtype=torch.int32, device="cuda")
    roco.roco_select_victims(p, stats, None, n_used, victim, ws)
    assert np.array_equal(victim.cpu().numpy(), order[:, 0])


@pytest.mark.parametrize("scope", [1, 5, 64, 500])
def test_victim_is_the_least_important_token_of_the_scope(scope):
    import paper_2402_06262_amd as roco
    rng = np.random.default_rng(scope)
    units, n = 4, 512
    acc = rng.uniform(0.1, 2.0, (units, n)).astype(np.float32)
    cnt = rng.integers(1, 400, (units, n)).astype(np.float32)
    mas = acc / cnt
    acc2 = (cnt * (mas * mas * rng.uniform(1.25, 4.0, (units, n)).astype(np.float32))).astype(np.float32)
    acc[:, 100:140] = acc[:, 99:100]  # ties in both keys
    cnt[:, 100:140], acc2[:, 100:140] = cnt[:, 99:100], acc2[:, 99:100]
    mas = acc / cnt
    var = np.maximum(acc2 / cnt - mas * mas, np.float32(0.0))
    p = roco.RocoParams(units, 64, n, scope, roco.ROCO_F32)
    stats = torch.from_numpy(np.stack([acc, acc2, cnt], axis=1)).cuda()
    n_used = torch.full((units,), n, dtype=torch.int32, device="cuda")
    victim = torch.empty((units,), dtype=torch.int32, device="cuda")
    ws = torch.empty(roco.decode_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    roco.roco_select_victims(p, stats, None, n_used, victim, ws)
    for u in range(units):
        inside = np.sort(np.argsort(var[u], kind="stable")[:scope])
        assert int(victim[u]) == inside[np.argmin(mas[u][inside])]


@pytest.mark.parametrize("L", [300, 16384, 16385, 32768, 32769])
def test_prompts_on_both_sides_of_what_lds_holds(L):
    """Recency with sinks: what stays is known without the statistics -- the sinks and the last tokens, in order; the first
    decode step evicts the oldest token that is no sink."""
    import paper_2402_06262_amd as roco
    units, B, sinks = 2, 200, 3
    lens = [L, max(B, L - 77)]
    p = roco.RocoParams(units, 64, B, 1, roco.ROCO_BF16, importance=roco.ROCO_IMPORTANCE_OLDEST,
                        scope_kind=roco.ROCO_SCOPE_ALL, sinks=sinks)
    g = torch.Generator(device="cuda").manual_seed(L)
    Q, K, V = (torch.randn((units, L, 64), generator=g, device="cuda").bfloat16() for _ in range(3))
    c = roco.alloc_cache(p)
    ws = torch.empty(roco.prefill_workspace_bytes(p, L), dtype=torch.uint8, device="cuda")
    roco.roco_prefill_compress(p, Q, K, V, torch.tensor(lens, dtype=torch.int32, device="cuda"), L, c.K, c.V, c.stats,
                               c.pos, c.n_used, c.next_slot, None, ws)
    for u, n in enumerate(lens):
        want = torch.tensor(list(range(sinks)) + list(range(n - B + sinks, n)))
        assert torch.equal(c.pos[u].cpu().long(), want)
        assert torch.equal(c.stats[u, 2].cpu(), (n - want).float())
        assert torch.equal(c.K[u].cpu(), K[u].cpu()[want])
        total = float(c.stats[u, 0].double().sum())
        assert 0.0 < total < n
        assert int(c.next_slot[u]) == sinks


@pytest.mark.parametrize("dtype,d,B", [("bf16", 128, 384), ("bf16", 128, 385), ("f32", 64, 384), ("f32", 64, 385),
                                       ("f32", 128, 192), ("f32", 128, 193), ("bf16", 64, 768), ("bf16", 64, 769)])
def test_decode_steps_on_both_sides_of_the_one_kernel_rule(dtype, d, B):
    """Units of up to 192 KiB of keys and values take one kernel per step whatever their number."""
    import paper_2402_06262_amd as roco
    import test_gpu_parity as TP
    row = d * (2 if dtype == "bf16" else 4)
    p = roco.RocoParams(3, d, B, 9, roco.ROCO_BF16 if dtype == "bf16" else roco.ROCO_F32)
    assert roco.decode_step_launches(p) == (1 if 2 * B * row <= 192 * 1024 else 2)
    TP.run_workload(dtype, d, 3, [B + 5, B, B - 2], B + 5, B, 9, 4, seed=B, want_out=False, tag=f"one-kernel-{dtype}-{d}-{B}")


# Window and variance scopes with no more than `sinks` tokens beyond the victims: the last victim is a sink, whose key is next
# to the mark of the tokens outside the scope, of which there are up to 4 thousand.
SINKS = [(300, 200, 1, 4), (4096, 1024, 4, 4), (8192, 4096, 1, 4), (16400, 8200, 1, 4), (700, 500, 150, 200)]


def _sink_policy(kind):
    import paper_2402_06262_amd as roco
    return roco.ROCO_SCOPE_WINDOW if kind == "window" else roco.ROCO_SCOPE_STD


@pytest.mark.parametrize("kind", ["window", "std"])
@pytest.mark.parametrize("n,keep,scope,sinks", SINKS)
def test_sinks_are_evicted_only_when_nothing_else_is_in_the_scope(kind, n, keep, scope, sinks):
    import paper_2402_06262_amd as roco
    units = 3
    p = roco.RocoParams(units, 64, n, scope, roco.ROCO_F32, importance=roco.ROCO_IMPORTANCE_OLDEST,
                        scope_kind=_sink_policy(kind), sinks=sinks)
    pos = np.broadcast_to(np.arange(n, dtype=np.int32), (units, n)).copy()
    pos[1] = pos[1][::-1]  # the sinks in the last slots
    # one query seen by every token: acc2 - acc^2 is the variance, exact in fp32 and growing with the position
    var = pos.astype(np.float32)
    stats = torch.from_numpy(np.stack([np.zeros_like(var), var, np.ones_like(var)], axis=1)).cuda()
    n_used = torch.full((units,), n, dtype=torch.int32, device="cuda")
    mask = torch.empty((units, n), dtype=torch.int32, device="cuda")
    ws = torch.empty(roco.decode_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    roco.roco_select_retained(p, keep, stats, torch.from_numpy(pos).cuda(), n_used, mask, ws)
    got = mask.cpu().numpy()
    for u in range(units):
        imp = np.where(pos[u] < sinks, np.inf, pos[u].astype(np.float64))
        want = np.ones(n, np.int32)
        want[orc.select_evictions(imp, pos[u].astype(np.float64), scope, n - keep)] = 0
        assert (imp[want == 0] == np.inf).any()  # a sink is among the victims
        assert np.array_equal(got[u], want), u


@pytest.mark.parametrize("n,keep,scope,sinks", SINKS)
def test_prompt_that_evicts_a_sink(n, keep, scope, sinks):
    import paper_2402_06262_amd as roco
    units = 2
    p = roco.RocoParams(units, 64, keep, scope, roco.ROCO_BF16, importance=roco.ROCO_IMPORTANCE_OLDEST,
                        scope_kind=roco.ROCO_SCOPE_WINDOW, sinks=sinks)
    g = torch.Generator(device="cuda").manual_seed(n)
    Q, K, V = (torch.randn((units, n, 64), generator=g, device="cuda").bfloat16() for _ in range(3))
    c = roco.alloc_cache(p)
    ws = torch.empty(roco.prefill_workspace_bytes(p, n), dtype=torch.uint8, device="cuda")
    roco.roco_prefill_compress(p, Q, K, V, torch.full((units,), n, dtype=torch.int32, device="cuda"), n, c.K, c.V, c.stats,
                               c.pos, c.n_used, c.next_slot, None, ws)
    pos = np.arange(n)
    imp = np.where(pos < sinks, np.inf, pos.astype(np.float64))
    kept = np.setdiff1d(pos, orc.select_evictions(imp, pos.astype(np.float64), scope, n - keep))
    assert kept[0] > 0 and len(kept) == keep  # the first sink is gone
    first = int(orc.select_victim(imp[kept], kept.astype(np.float64), scope))
    for u in range(units):
        assert np.array_equal(c.pos[u].cpu().numpy(), kept)
        assert torch.equal(c.K[u].cpu(), K[u].cpu()[torch.from_numpy(kept)])
        assert int(c.next_slot[u]) == first


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("n,scope", [(256, 2), (4096, 4)])
def test_block_that_evicts_a_sink(dtype, d, n, scope):
    import parity as P
    import paper_2402_06262_amd as roco
    units, block, sinks = 2, 16, 4
    rng = np.random.default_rng(n)
    sess = P.make_session(units, d, n, scope, dtype, policy=orc.Policy("oldest", "window", sinks))
    K, V = (rng.standard_normal((units, n, d)).astype(np.float32) for _ in range(2))
    P.gpu_prefill(sess, K, K, V, [n] * units, False)
    new = [rng.standard_normal((units, block, d)).astype(np.float32) for _ in range(3)]
    ws = torch.empty(roco.block_workspace_bytes(sess.params, block), dtype=torch.uint8, device="cuda")
    _, slots, evicted = P.gpu_encode_block(sess, block, *new, [n] * units, ws)
    pos = np.arange(n)
    imp = np.where(pos < sinks, np.inf, pos.astype(np.float64))
    want = orc.select_evictions(imp, pos.astype(np.float64), scope, block)
    assert want[0] == 0
    for u in range(units):
        assert np.array_equal(np.sort(slots[u]), want) and np.array_equal(np.sort(evicted[u]), want)


@pytest.mark.parametrize("B", [4100, 16384])
@pytest.mark.parametrize("scope", [1, 900])
def test_victims_of_more_units_than_compute_units_with_large_budgets(B, scope):
    """The decode step whose search packs two bins into a word: its victims are those of the search of roco_select_victims on
    the statistics that the step leaves, most of them equal (one value per unit but for the slots of a few others)."""
    import paper_2402_06262_amd as roco
    units, d = 257, 64
    p = roco.RocoParams(units, d, B, scope, roco.ROCO_BF16)
    c = roco.alloc_cache(p)
    g = torch.Generator(device="cuda").manual_seed(B + scope)
    c.K.zero_()  # every slot receives the same probability
    c.V.normal_(generator=g)
    c.pos.copy_(torch.arange(B, device="cuda", dtype=torch.int32).expand(units, B))
    c.n_used.fill_(B)
    c.stats[:, 0], c.stats[:, 1], c.stats[:, 2] = 1.0, 0.5, 64.0
    some = torch.randint(0, B, (units, 700), generator=g, device="cuda")
    c.stats[:, 1].scatter_(1, some, torch.rand((units, 700), generator=g, device="cuda") + 0.05)
    c.stats[:, 0].scatter_(1, some, torch.rand((units, 700), generator=g, device="cuda") + 0.5)
    c.next_slot.copy_(some[:, 0])
    ws = torch.empty(roco.decode_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    q, k, v = (torch.randn((units, d), generator=g, device="cuda").bfloat16() for _ in range(3))
    qpos = torch.full((units,), B, dtype=torch.int32, device="cuda")
    roco.roco_decode_step(p, q, torch.zeros_like(k), v, qpos, c.K, c.V, c.stats, c.pos, c.n_used, c.next_slot,
                          torch.empty_like(q), None, None, ws)
    got = c.next_slot.clone()
    fresh = torch.full_like(got, -9)
    roco.roco_select_victims(p, c.stats, c.pos, c.n_used, fresh, ws)
    assert torch.equal(got, fresh)
    stats = c.stats.cpu().numpy()
    for u in (0, 100, 256):
        acc, acc2, cnt = stats[u]
        mas = acc / cnt
        # one fused multiply-add on the device: float64 holds the product of two fp32 numbers exactly
        var = np.maximum(np.float32(0.0), ((acc2 / cnt).astype(np.float64) - mas.astype(np.float64) ** 2).astype(np.float32))
        assert int(got[u]) == orc.select_victim(mas, var, scope)


@pytest.mark.parametrize("n,top", [(5, 5), (64, 64), (700, 700), (130, 2048), (2048, 4097), (300, 1 << 22), (5000, 2 ** 31 - 1),
                                   (16400, 2 ** 30)])
def test_window_scopes_over_positions_of_every_size(n, top):
    """The search over positions starts at the highest bit that any of them has: the lowest positions are in the scope, the
    token of lowest score among them goes (equal scores: by slot)."""
    import paper_2402_06262_amd as roco
    units = 3
    rng = np.random.default_rng([n, top % 1000])
    pos = np.stack([rng.permutation(top)[:n] if top < 10000 else rng.permutation(np.unique(rng.integers(0, top, 2 * n)))[:n]
                    for _ in range(units)]).astype(np.int32)
    acc = rng.integers(1, 9, (units, n)).astype(np.float32)
    stats = torch.from_numpy(np.stack([acc, acc, np.ones_like(acc)], axis=1)).cuda()
    n_used = torch.full((units,), n, dtype=torch.int32, device="cuda")
    for scope in sorted({1, 2, n // 2, n - 1, n}):
        p = roco.RocoParams(units, 64, n, scope, roco.ROCO_F32, importance=roco.ROCO_IMPORTANCE_AAS,
                            scope_kind=roco.ROCO_SCOPE_WINDOW)
        ws = torch.empty(roco.decode_workspace_bytes(p), dtype=torch.uint8, device="cuda")
        victim = torch.empty((units,), dtype=torch.int32, device="cuda")
        mask = torch.empty((units, n), dtype=torch.int32, device="cuda")
        dpos = torch.from_numpy(pos).cuda()
        roco.roco_select_victims(p, stats, dpos, n_used, victim, ws)
        keep = n // 3
        roco.roco_select_retained(p, keep, stats, dpos, n_used, mask, ws)
        for u in range(units):
            assert int(victim[u]) == orc.select_victim(acc[u].astype(np.float64), pos[u].astype(np.float64), scope)
            want = np.ones(n, np.int32)
            want[orc.select_evictions(acc[u].astype(np.float64), pos[u].astype(np.float64), scope, n - keep)] = 0
            assert np.array_equal(mask[u].cpu().numpy(), want)


@pytest.mark.parametrize("kind", ["equal", "low_bits", "middle_bits", "two_values", "wide"])
@pytest.mark.parametrize("n", [65, 127, 130, 192, 255, 256, 257])
def test_few_keys(kind, n):
    test_lowest_keys_go_first_and_ties_by_slot(kind, n)


@pytest.mark.parametrize("kind", ["equal", "low_bits", "two_values", "wide"])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 128, 129])
def test_few_keys_are_counted(kind, n):
    """Up to 128 keys are counted instead of searched, in blocks of 64: every number of victims, so that the boundary falls between
    equal keys of one block and of both."""
    import paper_2402_06262_amd as roco
    units = 2
    rng = np.random.default_rng([n, len(kind), 7])
    p = roco.RocoParams(units, 64, n, 1, roco.ROCO_F32, importance=roco.ROCO_IMPORTANCE_AAS, scope_kind=roco.ROCO_SCOPE_ALL)
    acc = np.stack([_keys(kind, n, rng) for _ in range(units)])
    stats = torch.from_numpy(np.stack([acc, acc, np.ones_like(acc)], axis=1)).cuda()
    n_used = torch.full((units,), n, dtype=torch.int32, device="cuda")
    masks = torch.empty((n, units, n), dtype=torch.int32, device="cuda")
    ws = torch.empty(roco.decode_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    for keep in range(n):
        mask = torch.empty((units, n), dtype=torch.int32, device="cuda")
        roco.roco_select_retained(p, keep, stats, None, n_used, mask, ws)
        masks[keep] = mask
    rank = np.argsort(np.argsort(acc, axis=1, kind="stable"), axis=1)
    want = (rank[None] >= n - np.arange(n)[:, None, None]).astype(np.int32)
    assert np.array_equal(masks.cpu().numpy(), want)


@pytest.mark.parametrize("kind", ["equal", "low_bits", "middle_bits", "two_values", "wide", "bin_of_128", "bin_of_129", "ends"])
@pytest.mark.parametrize("n", [129, 257, 1000, 2048, 5000])
def test_last_of_the_scope(kind, n):
    """The victim is the last token of the scope: importance falls as the scope's key grows.  Keys that share one bin of the search of
    up to eight waves or fill it to the last candidate, and keys at and beyond the ends of its bins (2^-52 and 2^12)."""
    import paper_2402_06262_amd as roco
    rng = np.random.default_rng([n, len(kind), 9])
    units = 3
    var = np.stack([_keys(kind, n, rng) if kind in ("equal", "low_bits", "middle_bits", "two_values", "wide") else
                    rng.uniform(2.0, 4.0, n).astype(np.float32) for _ in range(units)])
    if kind.startswith("bin_of"):
        m = int(kind[-3:])
        for u in range(units):  # m keys inside one bin of 2^18 bit patterns, the others above and below
            at = rng.choice(n, min(m, n), replace=False)
            var[u] = np.where(rng.random(n) < 0.5, var[u], var[u] / 64)
            var[u, at] = (np.float32(0.5).view(np.uint32) + rng.choice(1 << 18, at.size, replace=False).astype(np.uint32)).view(np.float32)
    if kind == "ends":
        e = rng.choice(np.array([0.0, 2.0 ** -60, 2.0 ** -52, 1.01 * 2.0 ** -52, 2.0 ** -51, 4000.0, 4095.9, 4096.0, 5000.0]), (units, n))
        var = (e * rng.choice([1.0, 1.0 + 2.0 ** -20], (units, n))).astype(np.float32)
    order = np.argsort(var, axis=1, kind="stable")
    rank = np.argsort(order, axis=1)
    # acc / count is far below the resolution of acc2 / count; the importance is the oldest position
    pos = (n - 1 - rank).astype(np.int32)
    stats = np.zeros((units, 3, n), np.float32)
    stats[:, 1], stats[:, 2] = var, 1.0
    dpos, dstats = torch.from_numpy(pos).cuda(), torch.from_numpy(stats).cuda()
    n_used = torch.full((units,), n, dtype=torch.int32, device="cuda")
    for scope in sorted({1, 2, n // 32 + 1, n // 3, n // 2, n - 1, 64, 65, 128, 129} & set(range(1, n + 1))):
        p = roco.RocoParams(units, 64, n, scope, roco.ROCO_F32, importance=roco.ROCO_IMPORTANCE_OLDEST)
        victim = torch.empty((units,), dtype=torch.int32, device="cuda")
        ws = torch.empty(roco.decode_workspace_bytes(p), dtype=torch.uint8, device="cuda")
        roco.roco_select_victims(p, dstats, dpos, n_used, victim, ws)
        assert np.array_equal(victim.cpu().numpy(), order[:, scope - 1]), (kind, n, scope)

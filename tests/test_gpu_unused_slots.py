"""Block-wise and grouped steps on caches whose unused slots hold any bytes: K, V and statistics of every slot that no token has
taken, and those of a unit's worth of memory behind the last unit, are 0xFF (NaN in fp32 and in bf16) before each step, from the
first token until the budget is reached and evictions begin."""
import math

import numpy as np
import pytest
import torch

import test_gpu_gqa as TG
import test_gpu_parity as TP
from inputs import round_to_bf16

pytestmark = pytest.mark.gpu

FORMS = [("f32", 64), ("bf16", 64), ("f32", 128), ("bf16", 128)]


def _steps(dtype, d, B, group, blocks, seed):
    import paper_2402_06262_amd as roco
    P = TP._parity()
    units, s, T = 2, 9, sum(blocks)
    sc = 1.0 / math.sqrt(d)
    rng = np.random.default_rng(seed)
    Q = rng.standard_normal((units, T, group, d)).astype(np.float32) + 0.25
    K, V = (rng.standard_normal((units, T, d)).astype(np.float32) for _ in range(2))
    if dtype == "bf16":
        Q, K, V = round_to_bf16(Q), round_to_bf16(K), round_to_bf16(V)
    sess = P.make_session(units, d, B, s, dtype)
    behind = [torch.zeros((units + 1, B, d), dtype=P.torch_dtype(dtype), device="cuda") for _ in range(2)]
    for x in behind:
        x[units].view(torch.uint8).fill_(0xFF)
    sess.cache.K, sess.cache.V = (x[:units] for x in behind)
    states, ties, t = TG.empty_states(units, B, d), P.TieCount(), 0
    for b in blocks:
        TP._poison_unused(sess.cache, [min(t, B)] * units)
        ws = torch.full((roco.block_workspace_bytes(sess.params, b),), 0xFF, dtype=torch.uint8, device="cuda")
        now = slice(t, t + b)
        if b == 1 and t % 2 == 0:
            o, es, ep = (x[:, None] for x in P.gpu_decode_step_gqa(sess, group, Q[:, t], K[:, t], V[:, t], [t] * units, ws))
        elif group == 1:
            o, es, ep = P.gpu_encode_block(sess, b, Q[:, now, 0], K[:, now], V[:, now], [t] * units, ws)
            o = o[:, :, None]
        else:
            o, es, ep = P.gpu_encode_block_gqa(sess, b, group, Q[:, now], K[:, now], V[:, now], [t] * units, ws)
        finite = bool(np.isfinite(o).all())
        assert finite, f"block of {b} at {t}: bytes of an unused slot reached the output"
        for u in range(units):
            ties += P.lockstep_block_gqa_unit(states[u], u, o, es, ep, Q[u, now], K[u, now], V[u, now], t, s, sc, dtype,
                                              what=f"block of {b} at {t}")
        t += b
    host = P.cache_to_host(sess)
    for u in range(units):
        P.check_cache_unit(host, u, states[u], what="at the end")
    P.assert_few_ties(ties, f"unused-{dtype}-{d}-g{group}")
    return sess


@pytest.mark.parametrize("dtype,d", FORMS)
@pytest.mark.parametrize("group", [1, 3])
@pytest.mark.parametrize("blocks", [[1] * 150, [5, 1, 20, 1, 9, 1, 1, 21, 13, 1, 1, 20, 9, 1, 21, 20, 1, 7, 1]], ids=["tokens", "blocks"])
def test_bytes_of_unused_slots_reach_nothing(dtype, d, group, blocks):
    """Fills that end everywhere inside a tile of 32 and of 64 slots."""
    _steps(dtype, d, 132, group, blocks, seed=700 + d + group)


@pytest.mark.parametrize("dtype,d", FORMS)
@pytest.mark.parametrize("B", [68, 100])
def test_the_row_that_a_token_overwrites_is_gone(dtype, d, B):
    """The last slot of a cache that ends inside a tile is overwritten: its infinite value reaches nothing."""
    P = TP._parity()
    sess = _steps(dtype, d, B, 2, [1] * B, seed=800 + d + B)
    import paper_2402_06262_amd as roco
    sess.cache.V[:, B - 1] = math.inf
    sess.cache.next_slot.fill_(B - 1)
    ws = torch.empty(roco.block_workspace_bytes(sess.params, 1), dtype=torch.uint8, device="cuda")
    one = np.ones((2, 2, d), np.float32)
    out, slot, _ = P.gpu_decode_step_gqa(sess, 2, one, one[:, 0], one[:, 0], [B] * 2, ws)
    finite = bool(np.isfinite(out).all())
    assert finite and (slot == B - 1).all()

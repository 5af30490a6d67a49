"""Prompts of few units: the workgroups of the units that do not fill all dies evenly are dealt to the dies one by one, the waves
of a workgroup share its rows and several workgroups share a block's tiles.  Every form and both passes, with and without
output, against the vector-ALU passes (one wave per query, per key) on the same inputs."""
import math

import numpy as np
import pytest
import torch

import test_gpu_parity as TP
from inputs import round_to_bf16

pytestmark = pytest.mark.gpu

FORMS = [("f32", 64), ("bf16", 64), ("f32", 128), ("bf16", 128)]


def _inputs(rng, dtype, units, group, L, d):
    Q = rng.standard_normal((units, group, L, d)).astype(np.float32)
    K, V = (rng.standard_normal((units, L, d)).astype(np.float32) for _ in range(2))
    return tuple(round_to_bf16(x) for x in (Q, K, V)) if dtype == "bf16" else (Q, K, V)


def _both_paths(monkeypatch, dtype, d, units, group, L, lens, window=0, want_out=False):
    """Nothing is evicted (B = L), so the statistics of the two paths can be compared position by position."""
    P = TP._parity()
    Q, K, V = _inputs(np.random.default_rng(units * 1000 + L), dtype, units, group, L, d)
    res = []
    for simple in ("1", "0"):
        monkeypatch.setenv("ROCO_PREFILL_SIMPLE", simple)
        sess = P.make_session(units, d, L, 9, dtype, 0.0, window, 0.5 if window else 0.0)
        res.append(P.gpu_prefill_gqa(sess, group, Q, K, V, lens, want_out=want_out))
    want, got = res
    # fp32 sums of up to a few thousand probabilities in another order: a few 1e-7 of the largest, and the logits' own rounding
    np.testing.assert_allclose(got["stats"][:, :2], want["stats"][:, :2], rtol=2e-5, atol=1e-7)
    assert np.array_equal(got["stats"][:, 2], want["stats"][:, 2])
    if want_out:
        # bf16 / 128 rounds its probabilities to bf16 (2^-9 each, averaged) and every bf16 output is rounded (2^-9)
        tol = 2e-2 if dtype == "bf16" else 2e-5
        rms = np.sqrt(np.mean(np.square(want["O"], dtype=np.float64)))
        assert np.max(np.abs(got["O"].astype(np.float64) - want["O"])) <= tol * max(rms, np.max(np.abs(want["O"])))


@pytest.mark.parametrize("dtype,d", FORMS)
@pytest.mark.parametrize("units,group,L", [(1, 1, 700), (7, 1, 290), (9, 3, 270), (3, 4, 530), (15, 1, 129), (6, 2, 270),
                                           (13, 1, 300), (22, 1, 140)])
def test_units_left_over_by_the_dies(monkeypatch, dtype, d, units, group, L):
    lens = [L - (7 * u) % (L // 3) for u in range(units)]
    for want_out in (False, True):
        _both_paths(monkeypatch, dtype, d, units, group, L, lens, window=24 if units == 7 else 0, want_out=want_out)


@pytest.mark.parametrize("dtype,d", FORMS)
@pytest.mark.parametrize("units,group,L", [(1, 1, 2100), (2, 8, 600), (1, 3, 1300), (3, 5, 400), (2, 6, 500), (1, 7, 700),
                                           (1, 9, 300), (40, 2, 257), (70, 3, 200)])
def test_shared_blocks_and_every_group(monkeypatch, dtype, d, units, group, L):
    """Two to sixteen shares of a block's tiles, two or four waves per 32 owned rows, and the heads of a group (those that do not
    divide 16 leave registers of a result tile unused) summed inside a tile; 9 heads: the general kernel."""
    lens = [L - (11 * u) % (L // 2) for u in range(units)]
    _both_paths(monkeypatch, dtype, d, units, group, L, lens, window=24 if group == 3 else 0)


@pytest.mark.parametrize("dtype,d", FORMS)
@pytest.mark.parametrize("units,group,L", [(9, 1, 140), (34, 1, 1207), (66, 2, 334), (37, 2, 237), (122, 2, 140), (25, 3, 431)])
def test_schedules_of_two_shares(monkeypatch, dtype, d, units, group, L):
    """Numbers of units at which one form or another is estimated quicker with two shares at most than with what fills the chip."""
    _both_paths(monkeypatch, dtype, d, units, group, L, [L - (11 * u) % (L // 2) for u in range(units)])


@pytest.mark.parametrize("units,group,L", [(130, 1, 768), (130, 1, 769), (130, 2, 512), (130, 3, 513), (40, 8, 769), (70, 5, 1023)])
def test_owned_rows_of_a_column_block(monkeypatch, units, group, L):
    """128 or 256, with and without shares."""
    lens = [L - (13 * u) % (L // 2) for u in range(units)]
    _both_paths(monkeypatch, "bf16", 128, units, group, L, lens)


@pytest.mark.parametrize("qsplit", ["1", "2", "8"])
@pytest.mark.parametrize("group,L", [(1, 700), (3, 500), (5, 400), (6, 300), (7, 290), (8, 300)])
def test_shares_of_the_wide_kernels(monkeypatch, qsplit, group, L):
    monkeypatch.setenv("ROCO_PREFILL_QSPLIT", qsplit)
    _both_paths(monkeypatch, "bf16", 128, 3, group, L, [L, L - 70, L // 2])


@pytest.mark.parametrize("dtype,d", FORMS)
def test_a_smaller_workspace_takes_fewer_shares(dtype, d):
    """What the query asked for before it knew of more than two shares is still enough; less is refused."""
    import paper_2402_06262_amd as roco
    units, group, L, B = 1, 2, 3000, 3000
    P = TP._parity()
    Q, K, V = _inputs(np.random.default_rng(5), dtype, units, group, L, d)
    sess = P.make_session(units, d, B, 9, dtype)
    want = P.gpu_prefill_gqa(sess, group, Q, K, V, [L])["stats"]
    up = lambda n: (n + 255) // 256 * 256
    least = 4 * up(4 * units * L) + up(4 * units * group * L)
    assert least < sess.prefill_ws.nbytes
    q, k, v = (P.to_dev(x, dtype) for x in (Q, K, V))
    lens = torch.tensor([L], dtype=torch.int32, device="cuda")
    c = sess.cache
    for nbytes in (least, 2 * least, least - 1):
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        c.stats.zero_()
        call = lambda: roco.roco_prefill_compress_gqa(sess.params, group, q, k, v, lens, L, c.K, c.V, c.stats, c.pos, c.n_used,
                                                      c.next_slot, None, ws)
        if nbytes < least:
            with pytest.raises(roco.RocoError):
                call()
            continue
        call()
        torch.cuda.synchronize()
        np.testing.assert_allclose(c.stats.cpu().numpy()[:, :2], want[:, :2], rtol=2e-5, atol=1e-7)


@pytest.mark.parametrize("importance", ["MAS", "LAST", "COUNT"])
def test_shares_of_a_prompt_whose_keys_do_not_fit_the_lds(importance):
    """Above 16384 tokens a kernel of its own adds the shares; the last-token score needs them added before it writes its row.
    Two shares (the smallest workspace) against all that the query asks for, at the positions that both keep."""
    import paper_2402_06262_amd as roco
    L, B, d = 17000, 300, 128
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    Q, K, V = (torch.randn((1, L, d), generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    p = roco.RocoParams(1, d, B, 60, roco.ROCO_BF16, importance=getattr(roco, "ROCO_IMPORTANCE_" + importance),
                        scope_kind=roco.ROCO_SCOPE_STD if importance == "MAS" else roco.ROCO_SCOPE_ALL)
    least = 5 * 4 * L + 5 * 256
    assert roco.prefill_workspace_bytes(p, L) > least + 2 * 4 * L  # more than two shares
    stats = []
    for nbytes in (least, roco.prefill_workspace_bytes(p, L)):
        c = roco.alloc_cache(p)
        ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda")
        roco.roco_prefill_compress(p, Q, K, V, torch.tensor([L], dtype=torch.int32, device="cuda"), L, c.K, c.V, c.stats, c.pos,
                                   c.n_used, c.next_slot, None, ws)
        torch.cuda.synchronize()
        stats.append(dict(zip(c.pos[0].tolist(), c.stats[0].t().cpu().numpy())))
    a, b = stats
    both = sorted(a.keys() & b.keys())
    assert len(both) >= 0.98 * B  # ranking keys that agree within rounding may go either way
    x, y = (np.stack([s[i] for i in both]) for s in stats)
    np.testing.assert_allclose(x[:, 0], y[:, 0], rtol=2e-5, atol=1e-7)
    assert np.array_equal(x[:, 2], y[:, 2])
    if importance == "COUNT":  # a probability within rounding of 1 / (i + 1) may be counted or not: about one in 10^6
        assert np.max(np.abs(x[:, 1] - y[:, 1])) <= 2
    else:
        np.testing.assert_allclose(x[:, 1], y[:, 1], rtol=2e-5, atol=1e-7)


@pytest.mark.parametrize("dtype,d", FORMS)
@pytest.mark.parametrize("importance", ["ltas", "aqas"])
@pytest.mark.parametrize("units,group,L", [(1, 1, 2100), (2, 3, 600), (1, 5, 500), (2, 6, 400), (1, 7, 700), (2, 9, 300), (3, 8, 300)])
def test_scores_in_the_second_plane(monkeypatch, dtype, d, importance, units, group, L):
    """The last query's attention and the counted queries, over shared blocks and every group: against the vector-ALU passes."""
    from oracle.roco_oracle import Policy
    P = TP._parity()
    Q, K, V = _inputs(np.random.default_rng(units * 1000 + L + group), dtype, units, group, L, d)
    lens = [L - (11 * u) % (L // 2) for u in range(units)]
    res = []
    for simple in ("1", "0"):
        monkeypatch.setenv("ROCO_PREFILL_SIMPLE", simple)
        sess = P.make_session(units, d, L, 9, dtype, policy=Policy(importance, "all"))
        res.append(P.gpu_prefill_gqa(sess, group, Q, K, V, lens)["stats"])
    want, got = res
    np.testing.assert_allclose(got[:, 0], want[:, 0], rtol=2e-5, atol=1e-7)
    if importance == "aqas":  # see above; a few hundred thousand probabilities
        off = np.abs(got[:, 1] - want[:, 1])
        assert off.max() <= 1 and off.sum() <= 5
    else:
        np.testing.assert_allclose(got[:, 1], want[:, 1], rtol=2e-5, atol=1e-7)


@pytest.mark.parametrize("dtype,d,B", [("f32", 128, 256), ("f32", 128, 257), ("bf16", 64, 1024), ("bf16", 64, 1025), ("f32", 64, 1),
                                       ("bf16", 128, 63)])
def test_rows_copied_by_the_selection(dtype, d, B):
    """Up to 256 KiB of kept rows per unit the selection copies them itself: at the limit and beyond it, one row, an odd number,
    prompts shorter than the budget (nothing is ranked), one token."""
    L = max(300, B + 90)
    TP.run_workload(dtype, d, 5, [L, B, max(1, B - 1), 1, min(L, B + 1)], L, B, max(1, B // 3), 2, seed=B, tag=f"copy-{dtype}-{d}-{B}")


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 64)])
@pytest.mark.parametrize("waves", ["1", "4"])
def test_waves_that_share_a_row(dtype, d, waves, monkeypatch):
    """Prompts that end before, at and behind the blocks of keys that the four waves of a row take in turn."""
    monkeypatch.setenv("ROCO_PREFILL_SIMPLE", "1")
    monkeypatch.setenv("ROCO_PREFILL_WAVES_PER_ROW", waves)
    P, rng = TP._parity(), np.random.default_rng(d + int(waves))
    lens = [1, 15, 16, 17, 31, 33, 63, 64, 65, 96, 127, 128, 129, 161]
    L, B, s, sc = max(lens), 20, 5, 1.0 / math.sqrt(d)
    Q, K, V = (rng.standard_normal((len(lens), L, d)).astype(np.float32) for _ in range(3))
    if dtype == "bf16":
        Q, K, V = round_to_bf16(Q), round_to_bf16(K), round_to_bf16(V)
    for window in (0, 24):
        sess = P.make_session(len(lens), d, B, s, dtype, 0.0, window, 0.5 if window else 0.0)
        g = P.gpu_prefill(sess, Q, K, V, lens, True)
        for u in range(len(lens)):
            P.check_prefill_unit(g, u, Q[u], K[u], V[u], lens[u], B, s, sc, dtype, window, 0.5 if window else 0.0)


@pytest.mark.parametrize("threads", ["512", "1024"])
@pytest.mark.parametrize("dtype,d,B", [("f32", 64, 40), ("bf16", 64, 512), ("bf16", 128, 513), ("f32", 128, 600)])
def test_threads_of_the_selection(dtype, d, B, threads, monkeypatch):
    """Prompts that end before, at and behind the rounds of 512 and 1024 positions; rows copied by the selection and behind it."""
    monkeypatch.setenv("ROCO_SELECT_THREADS", threads)
    P, rng = TP._parity(), np.random.default_rng(d + B)
    lens = [1, 64, 511, 512, 513, 1023, 1024, 1025, 1030]
    L, s, sc = max(lens), max(1, B // 8), 1.0 / math.sqrt(d)
    Q, K, V = (rng.standard_normal((len(lens), L, d)).astype(np.float32) for _ in range(3))
    if dtype == "bf16":
        Q, K, V = round_to_bf16(Q), round_to_bf16(K), round_to_bf16(V)
    sess = P.make_session(len(lens), d, B, s, dtype, 0.0, 0, 0.0)
    g = P.gpu_prefill(sess, Q, K, V, lens, True)
    for u in range(len(lens)):
        P.check_prefill_unit(g, u, Q[u], K[u], V[u], lens[u], B, s, sc, dtype, 0, 0.0)

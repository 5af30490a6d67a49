"""The matrix-core prefill of fp32 storage and of head_dim 64: edges of its tiles (32 streamed rows, 64 / 128 rows per tile,
blocks of 64 / 128 owned rows), both ways of sharing a block between waves and workgroups, every way of summing the heads of
a group, and inputs that are not finite or near the ends of fp32's range."""
import math

import numpy as np
import pytest
import torch

import test_gpu_gqa as TG
import test_gpu_parity as TP
from inputs import round_to_bf16
from oracle import roco_oracle as orc

pytestmark = pytest.mark.gpu

FORMS = [("f32", 64), ("bf16", 64), ("f32", 128)]


@pytest.mark.parametrize("dtype,d", FORMS)
@pytest.mark.parametrize("L,lens", [(65, [65, 1, 64, 33, 32]), (130, [130, 129, 128, 127, 63]), (300, [300, 257, 256, 191, 2])])
@pytest.mark.parametrize("want_out", [False, True])
def test_edges_of_tiles_and_blocks(dtype, d, L, lens, want_out):
    B = max(16, L // 3)
    TP.run_workload(dtype, d, 5, lens, L, B, 7, 2, seed=71 + L, want_out=want_out, tag=f"planes-{dtype}-{d}-{L}")


@pytest.mark.parametrize("dtype,d", FORMS)
@pytest.mark.parametrize("units,L", [(1, 1030), (140, 200), (300, 260)])
def test_every_schedule(dtype, d, units, L):
    """Few units (shared blocks, halves of the streamed tiles), some, and enough for pairs of blocks per workgroup."""
    rng = np.random.default_rng(units)
    lens = [L] + [int(x) for x in rng.integers(L // 2, L + 1, size=units - 1)]
    P = TP._parity()
    B, s, sc = L // 2, 9, 1.0 / math.sqrt(d)
    Q, K, V = (rng.standard_normal((units, L, d)).astype(np.float32) for _ in range(3))
    if dtype == "bf16":
        Q, K, V = round_to_bf16(Q), round_to_bf16(K), round_to_bf16(V)
    sess = P.make_session(units, d, B, s, dtype, 0.0, 24, 0.5)
    for want_out in (False, True):
        g = P.gpu_prefill(sess, Q, K, V, lens, want_out)
        for u in (0, units // 2, units - 1):
            P.check_prefill_unit(g, u, Q[u], K[u], V[u], lens[u], B, s, sc, dtype, 24, 0.5, want_out)


@pytest.mark.parametrize("dtype,d", FORMS)
@pytest.mark.parametrize("group", [2, 3, 4, 8, 16])
def test_heads_of_a_group(dtype, d, group):
    for want_out in (False, True):
        TG.run_grouped_prefill(dtype, d, group, [150, 97], 150, 48, 6, seed=90 + group, steps=2, recency=group == 8,
                               tag=f"planes-group-{group}", want_out=want_out)


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 64), ("f32", 128)])
def test_thresholded_count(dtype, d):
    TP.run_workload(dtype, d, 3, [200, 131, 64], 200, 60, 60, 2, seed=77, policy=orc.Policy("aqas", "all"), tag="planes-count")


@pytest.mark.parametrize("dtype,d", FORMS)
@pytest.mark.parametrize("group", [3, 4])
def test_thresholded_count_of_a_group(dtype, d, group, monkeypatch):
    """Against the vector-ALU passes: a count may differ by the queries whose probability is within rounding of the mean."""
    P = TP._parity()
    rng = np.random.default_rng(8)
    units, L, B = 2, 190, 190
    Q = rng.standard_normal((units, group, L, d)).astype(np.float32) + 0.25
    K, V = (rng.standard_normal((units, L, d)).astype(np.float32) for _ in range(2))
    if dtype == "bf16":
        Q, K, V = round_to_bf16(Q), round_to_bf16(K), round_to_bf16(V)
    res = []
    for simple in ("1", "0"):
        monkeypatch.setenv("ROCO_PREFILL_SIMPLE", simple)
        sess = P.make_session(units, d, B, B, dtype, policy=orc.Policy("aqas", "all"))
        res.append(P.gpu_prefill_gqa(sess, group, Q, K, V, [L, L - 33])["stats"])
    np.testing.assert_allclose(res[1][:, 0], res[0][:, 0], rtol=1e-5, atol=1e-7)
    assert np.max(np.abs(res[1][:, 1] - res[0][:, 1])) <= 1.0
    assert np.mean(res[1][:, 1] != res[0][:, 1]) < 0.01


def _both_paths(monkeypatch, dtype, d, Q, K, V, lens, B=96, s=16):
    P = TP._parity()
    units, L = K.shape[0], K.shape[1]
    out = []
    for simple in ("1", "0"):
        monkeypatch.setenv("ROCO_PREFILL_SIMPLE", simple)
        sess = P.make_session(units, d, B, s, dtype)
        out.append(P.gpu_prefill(sess, Q, K, V, lens, True))
    return out


@pytest.mark.parametrize("dtype,d", FORMS)
def test_infinities_and_nan_go_where_a_plain_product_sends_them(dtype, d, monkeypatch):
    """An element that is not finite reaches the rows that see it and no others, on the matrix cores as on the vector ALUs.
    B > L: nothing is evicted, so positions can be compared one to one."""
    rng = np.random.default_rng(5)
    units, L, B = 6, 1100, 1200  # (large enough for the matrix-core row pass with output)
    Q, K, V = (rng.standard_normal((units, L, d)).astype(np.float32) for _ in range(3))
    if dtype == "bf16":
        Q, K, V = round_to_bf16(Q), round_to_bf16(K), round_to_bf16(V)
    Q[:, :, 3] = 1.0
    K[0, 40, 3] = -np.inf       # a key no query attends (query 40 included)
    K[1, 700, 3] = np.inf       # rows from 700 on are NaN
    V[2, 555, 7] = np.inf       # dimension 7 of the rows from 555 on
    V[2, 600, 8] = -np.inf
    V[3, 65, d - 1] = np.nan
    Q[4, 300] = np.nan          # one row, and the statistics of the keys up to it
    K[5, 10, 5] = np.nan
    want, got = _both_paths(monkeypatch, dtype, d, Q, K, V, [L] * 5 + [L - 3], B=B)
    tol = 2e-2 if dtype == "bf16" else 1e-5
    for key in ("O", "stats"):
        a, b = np.asarray(want[key], np.float64), np.asarray(got[key], np.float64)
        assert np.array_equal(np.isnan(a), np.isnan(b)), key
        assert np.array_equal(np.isinf(a), np.isinf(b)), key
        fine = np.isfinite(a)
        assert np.array_equal(a[np.isinf(a)], b[np.isinf(b)]), key
        np.testing.assert_allclose(b[fine], a[fine], rtol=tol, atol=tol * 0.1, err_msg=key)


@pytest.mark.parametrize("dtype,d", FORMS)
def test_an_infinite_value_of_a_far_lower_logit_stays_in_the_output(dtype, d, monkeypatch):
    """Every other 32 keys lie 260 powers of two below the rest, so what one half of a workgroup's waves summed has a weight
    that underflows: an infinity among its values is not finite in the rows that see it (0 x inf), as on the vector ALUs."""
    rng = np.random.default_rng(4)
    units, L = 3, 1100
    Q = np.full((units, L, d), 4.0 * math.sqrt(128.0 / d), np.float32)
    K, V = Q.copy(), rng.standard_normal((units, L, d)).astype(np.float32)
    if dtype == "bf16":
        Q, K, V = round_to_bf16(Q), round_to_bf16(K), round_to_bf16(V)
    K[0, np.arange(L) // 32 % 2 == 1] *= -1.0
    K[1, np.arange(L) // 32 % 2 == 0] *= -1.0
    V[0, 40, 7] = np.inf
    V[1, 70, 7] = np.inf
    want, got = _both_paths(monkeypatch, dtype, d, Q, K, V, [L] * units, B=L)
    for u, key in ((0, 40), (1, 70)):
        for O in (want["O"], got["O"]):
            assert not np.isfinite(O[u, key + 64:, 7]).any()
            assert np.isfinite(O[u, :key, 7]).all() and np.isfinite(np.delete(O[u], 7, axis=1)).all()
    assert np.isfinite(got["O"][2]).all()


@pytest.mark.parametrize("d", [64, 128])
def test_ends_of_the_fp32_range(d, monkeypatch):
    """Key elements up to the largest fp32 value (whose first plane may not round up to infinity) against the smallest
    normal one, keys and queries scaled against each other, large and small values: results are of ordinary relative size."""
    rng = np.random.default_rng(6)
    units, L, B = 4, 1024, 1024
    Q, K, V = (rng.standard_normal((units, L, d)).astype(np.float32) for _ in range(3))
    K[0, :, 3] = rng.uniform(1e38, 3.4028e38, L).astype(np.float32) * np.sign(K[0, :, 3])
    Q[0, :, 3] = np.float32(2.0 ** -126)
    K[1] *= np.float32(2.0 ** -60)
    Q[1] *= np.float32(2.0 ** 60)
    V[2] *= np.float32(1e30)
    V[3] *= np.float32(1e-30)
    want, got = _both_paths(monkeypatch, "f32", d, Q, K, V, [L] * units, B=B)
    for key in ("O", "stats"):
        a, b = np.asarray(want[key], np.float64), np.asarray(got[key], np.float64)
        assert np.array_equal(np.isfinite(a), np.isfinite(b)), key
        fine = np.isfinite(a)
        # 1e-5 relative to the row's largest: sums of up to 1024 fp32 terms, sqrt(1024) * 2^-24 and a margin of five
        scale = np.max(np.abs(np.where(fine, a, 0.0)), axis=-1, keepdims=True)
        assert np.all(np.abs(np.where(fine, b - a, 0.0)) <= 1e-5 * np.maximum(scale, 1e-30)), key


def test_tiny_prompts_take_the_vector_passes_and_agree(monkeypatch):
    """Both sides of the size rules: 64 tokens (both passes, fp32), 2^19 = units x heads x L^2 (fp32 with output), 2^18 (bf16
    with output), 2^17 and 128 or 192 tokens (fp32 / 128 and fp32 / 64 without)."""
    for units, L in ((2, 64), (2, 65), (8, 256), (9, 256)):
        TP.run_workload("f32", 64, units, [L] * units, L, L // 2, 5, 1, seed=units + L, tag="planes-tiny")
    for units, L in ((8, 128), (9, 128), (2, 128), (2, 129)):
        TP.run_workload("f32", 128, units, [L] * units, L, L // 2, 5, 1, seed=units + L, want_out=False, tag="planes-tiny")
    for units, L in ((8, 128), (9, 128), (2, 144), (2, 145), (3, 192), (3, 193), (4, 192)):
        TP.run_workload("f32", 64, units, [L] * units, L, L // 2, 5, 1, seed=units + L, want_out=False, tag="planes-tiny")
    for units, L in ((8, 128), (9, 128), (2, 129), (16, 128), (17, 128), (4, 256), (1, 513)):
        TP.run_workload("bf16", 64, units, [L] * units, L, L // 2, 5, 1, seed=units + L, tag="planes-tiny")


@pytest.mark.parametrize("L,lens", [(90, [90, 65]), (450, [450, 333]), (1500, [1500, 1027])])
def test_bf16_output_is_rounded_once(L, lens):
    """head_dim 64: the probabilities are fp32 numbers whatever kernel a prompt's size selects, so an output is the float64
    result rounded to bf16 but where that lies within fp32's error of a rounding boundary.  Bound: errors of 1e-5 of the row's
    rms (fp32 sums, as for fp32 storage) against boundaries 2^-8 of a value apart reach one in 0.5 % of the values of that
    size, more of the smaller ones: 2 % in all.  Probabilities rounded to bf16 before the product miss a third of them."""
    P = TP._parity()
    rng = np.random.default_rng(L)
    units, d = len(lens), 64
    Q, K, V = (round_to_bf16(rng.standard_normal((units, L, d)).astype(np.float32)) for _ in range(3))
    sess = P.make_session(units, d, L, 5, "bf16")
    O = P.gpu_prefill(sess, Q, K, V, lens, True)["O"]
    for u, n in enumerate(lens):
        want = orc.prefill_statistics(Q[u], K[u], V[u], n, 1.0 / math.sqrt(d), want_out=True).out
        exact = torch.from_numpy(want).bfloat16().float().numpy()
        assert np.mean(O[u, :n] != exact) < 0.02


def _wild(kind, units, group, L, d, dtype, seed):
    """Inputs of the kinds that bf16 planes do not hold, in the first units; the others are ordinary."""
    rng = np.random.default_rng(seed)
    Q = rng.standard_normal((units, group, L, d)).astype(np.float32)
    K, V = (rng.standard_normal((units, L, d)).astype(np.float32) for _ in range(2))
    if kind == "not finite":
        Q[..., 3] = 1.0
        K[0, 40, 3] = -np.inf                 # a key no query attends
        K[1, L - 60, 3] = np.inf              # rows from there on are NaN
        Q[2, group - 1, L // 2] = np.nan      # one row, and the statistics of the keys up to it
        K[3, 10, 5] = np.nan
    elif kind == "small keys":
        K[:4] *= np.float32(1e-34)
        Q[:4] *= np.float32(1e34)
    elif kind == "small queries":
        Q[:4] *= np.float32(1e-36)
        K[:4] *= np.float32(1e36)
    elif kind == "one small element":
        Q[0, 0, 37, 11] = np.float32(1.2345e-36)
        K[0, :, 11] *= np.float32(1e36)
        Q[0, :, :37, 11] = Q[0, :, 38:, 11] = 0.0
        if group > 1:
            Q[0, 1:, 37, 11] = 0.0
    else:
        assert kind == "largest"
        K[0, 5, 3] = np.finfo(np.float32).max
        Q[0, :, :, 3] = np.float32(2.0 ** -127)
    if dtype == "bf16":
        Q, K, V = round_to_bf16(Q), round_to_bf16(K), round_to_bf16(V)
    return Q, K, V


@pytest.mark.parametrize("dtype,d", FORMS)
@pytest.mark.parametrize("units,L,group", [(6, 1100, 1), (140, 300, 1), (600, 300, 1), (6, 200, 3), (6, 333, 4)])
@pytest.mark.parametrize("kind", ["not finite", "small keys", "small queries", "one small element", "largest"])
def test_wild_inputs_without_output(dtype, d, units, L, group, kind, monkeypatch):
    """Statistics of every schedule and grouping against the vector-ALU passes: what is not finite is the same, the rest within
    1e-5 (fp32 sums of up to 1100 probabilities; 2e-5 of the logits' rounding at their size of up to ten)."""
    P = TP._parity()
    Q, K, V = _wild(kind, units, group, L, d, dtype, 11)
    lens = [L - u % 3 for u in range(units)]
    res = []
    for simple in ("1", "0"):
        monkeypatch.setenv("ROCO_PREFILL_SIMPLE", simple)
        sess = P.make_session(units, d, L, 16, dtype)
        if group == 1:
            res.append(P.gpu_prefill(sess, Q[:, 0], K, V, lens, False)["stats"])
        else:
            res.append(P.gpu_prefill_gqa(sess, group, Q, K, V, lens, False)["stats"])
    a, b = (np.asarray(r, np.float64) for r in res)
    assert np.array_equal(np.isnan(a), np.isnan(b))
    assert np.array_equal(np.isinf(a), np.isinf(b))
    fine = np.isfinite(a)
    np.testing.assert_allclose(b[fine], a[fine], rtol=1e-5, atol=1e-6)


@pytest.mark.parametrize("d", [64, 128])
def test_outputs_of_small_values_keep_fp32_precision(d):
    """V down to fp32's subnormal range, queries and keys scaled against each other: an output is within 1e-5 of its row's
    largest, and a few times 2^-149 where that is the unit of fp32 itself."""
    P = TP._parity()
    rng = np.random.default_rng(16)
    units, L = 5, 700
    Q, K, V = (rng.standard_normal((units, L, d)).astype(np.float32) for _ in range(3))
    V[0] *= np.float32(1e-34)
    V[1] *= np.float32(2.0 ** -136)
    V[2, 1::2] *= np.float32(1e-35)
    K[3], Q[3] = K[3] * np.float32(1e-35), Q[3] * np.float32(1e35)
    sess = P.make_session(units, d, L, 5, "f32")
    O = P.gpu_prefill(sess, Q, K, V, [L] * units, True)["O"].astype(np.float64)
    for u in range(units):
        want = orc.prefill_statistics(Q[u], K[u], V[u], L, 1.0 / math.sqrt(d), want_out=True).out
        scale = np.max(np.abs(want), axis=1, keepdims=True)
        # subnormal sums lose up to half a unit per addition, of random sign: 700 of them, sqrt(700) / 2
        assert np.all(np.abs(O[u] - want) <= 1e-5 * scale + 16 * 2.0 ** -149), u


@pytest.mark.parametrize("dtype,d", FORMS)
def test_large_values_under_rising_scores(dtype, d):
    """V of 1e34 to 1e37 and logits that rise by 15 powers of two along the prompt: sums against an early reference would be
    2^15 times larger than the outputs and overflow."""
    P = TP._parity()
    rng = np.random.default_rng(17)
    units, L = 3, 900
    Q, K, V = (rng.standard_normal((units, L, d)).astype(np.float32) for _ in range(3))
    Q[..., 0] = 8.0
    K[..., 0] = np.linspace(0.0, 15.0 * math.log(2.0) * math.sqrt(d) / 8.0, L, dtype=np.float32)
    V *= np.array([1e34, 1e37, 1e20], np.float32)[:, None, None]
    V[2, 400:405] *= np.float32(1e17)
    if dtype == "bf16":
        Q, K, V = round_to_bf16(Q), round_to_bf16(K), round_to_bf16(V)
    sess = P.make_session(units, d, L, 5, dtype)
    O = P.gpu_prefill(sess, Q, K, V, [L] * units, True)["O"].astype(np.float64)
    # fp32: as for ordinary values (1e-5 of the row's largest); bf16: its rounding
    tol = 1e-5 if dtype == "f32" else 2.0 ** -8
    for u in range(units):
        want = orc.prefill_statistics(Q[u], K[u], V[u], L, 1.0 / math.sqrt(d), want_out=True).out
        assert np.all(np.abs(O[u] - want) <= tol * np.max(np.abs(want), axis=1, keepdims=True)), u

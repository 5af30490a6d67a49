"""Prompts of few units: the workgroups of the units that do not fill all dies evenly are dealt to the dies one by one.  Every
form and both passes, with and without output, against the vector-ALU passes (one wave per query, per key) on the same inputs."""
import numpy as np
import pytest

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
@pytest.mark.parametrize("units,group,L", [(1, 1, 700), (7, 1, 290), (9, 3, 270), (3, 4, 530), (15, 1, 129)])
def test_units_left_over_by_the_dies(monkeypatch, dtype, d, units, group, L):
    lens = [L - (7 * u) % (L // 3) for u in range(units)]
    for want_out in (False, True):
        _both_paths(monkeypatch, dtype, d, units, group, L, lens, window=24 if units == 7 else 0, want_out=want_out)

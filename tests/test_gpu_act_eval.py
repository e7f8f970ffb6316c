"""GPU parity of the evaluator's one-launch activation layers (dash_act_eval.hip) around the edges of their blocks: 2 or 1 values
per block (tiny form), 16 (shallow form), 64 (deep form), both label-length rules, the four digit sets, in place and not."""
import numpy as np
import pytest

import workloads
from test_gpu_layers import run_activation

pytestmark = pytest.mark.gpu


BIG = "1000000000"


def force(monkeypatch, form):
    monkeypatch.setenv("DASH_ACT_SHALLOW_MIN_ELEMS", BIG if form == "tiny" else "0")
    monkeypatch.setenv("DASH_ACT_DEEP_MIN_ELEMS", "0" if form == "deep" else BIG)


@pytest.mark.parametrize("form", ["tiny", "shallow", "deep"])
@pytest.mark.parametrize("k,rule", [(7, 0), (8, 0), (9, 0), (12, 0), (7, 1), (8, 1), (9, 1), (12, 1)])
def test_one_launch_activation_layers(monkeypatch, k, rule, form):
    force(monkeypatch, form)
    P = int(np.prod(workloads.PRIMES[:k]))
    g = np.random.default_rng(1000 + k + rule)
    for n in ((1, 63, 65) if form == "deep" else (1, 9, 16, 17)):
        X = np.concatenate([[P // 2], g.integers(0, P, n - 1)])
        run_activation(k, "relu", X, rule=rule, elem_base=2 ** 32 - 5, in_place=n == 9)
        run_activation(k, "scale", X, repeat=3, rule=rule, elem_base=11, in_place=n in (9, 65))


@pytest.mark.parametrize("form", ["tiny", "shallow", "deep"])
def test_one_launch_activation_layers_short_digit_set(monkeypatch, form):
    force(monkeypatch, form)
    X = np.random.default_rng(5).integers(0, int(np.prod(workloads.PRIMES[:8])), 70)
    run_activation(8, "relu", X, digits=workloads.DIGITS_REDUCED[8], exact=False)
    run_activation(8, "scale", X, repeat=6, digits=workloads.DIGITS_REDUCED[8], exact=False)


@pytest.mark.parametrize("k,n_digits", [(8, 14), (7, 16), (12, 16)])
def test_deep_layers_of_long_digit_sets(monkeypatch, k, n_digits):
    """digit sums that go on behind the span of the deep form's tables (72, 85 and 81 dwords; 64 fit)"""
    force(monkeypatch, "deep")
    digits = workloads.DIGITS[k][:2] + workloads.DIGITS[k][1:2] * (n_digits - 2)
    X = np.random.default_rng(k).integers(0, int(np.prod(workloads.PRIMES[:k])), 65)
    run_activation(k, "relu", X, digits=digits)
    run_activation(k, "scale", X, repeat=2, digits=digits)

"""The selection at the ends of its parameters' and inputs' ranges: eps whose square is
the smallest or largest the gains' quotient is formed from (and beyond either: the plain
division), eps whose square is infinite, and Gram matrices that hold nothing but NaN."""
import dataclasses

import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import check_lists_valid, compare_select, gpu_select, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps", [1e-160, 1e-120, 1e-100, 0.9e-100, 1.0, 1e100, 1.1e100, 1e150, 8e153, 1.3e154])
def test_eps_range(eps):
    """From an eps that is its square's end of the normal range to the other: V so large that the objective stays a
    normal number (float64 drift of about 2^200 eps^-2)."""
    scale = 2.0 ** 100 if eps > 1e10 else 1.0
    L = synth.make_layer(3, 800, 5, H=3, block=64, sparsity=0.6, seed=61, name=f"eps {eps:g}")
    v = synth.bf16_bits_to_f32(L.v) * np.float32(scale)
    L = dataclasses.replace(L, v=synth.f32_to_bf16_bits(v.astype(np.float32)))
    say(f"[eps] {eps:g} H={L.H} N={L.N} n_kb={L.n_kb}")
    gpu, _ = gpu_select(L, eps=eps)
    ref = oracle.select(L.q, L.k, L.v, L.gram, L.budgets, N=L.N, bq=L.bq, bk=L.bk, n_special=L.n_special_tail,
                        rounds=5, eps=eps)
    st = compare_select(L, gpu, ref, label=f"eps {eps:g}")
    assert st["checked"] > 0.9 * st["rows"]


@pytest.mark.parametrize("eps", [2e154, 1e200])
def test_eps_with_infinite_square(eps):
    """Every objective and every gain is 0: no round improves on the initial lists, the drifts are 0."""
    L = synth.make_layer(3, 800, 5, H=3, block=64, sparsity=0.6, seed=61, name=f"eps {eps:g}")
    gpu, _ = gpu_select(L, eps=eps)
    first, _ = gpu_select(L, rounds=0, eps=eps)
    assert np.array_equal(gpu["kept_idx"], first["kept_idx"]) and not gpu["drift"].any()


@pytest.mark.parametrize("bits", [0x7FC00000, 0xFFC00000, 0x7FFFFFFF, 0xFFFFFFFF])
@pytest.mark.parametrize("criterion", [0, 3])
def test_nan_gram_keeps_the_budget(bits, criterion):
    """No score is a number, so no choice is better than another, but every row still keeps its budget."""
    L = synth.make_layer(3, 800, 5, H=2, block=64, sparsity=0.6, seed=62, name="nan gram")
    L = dataclasses.replace(L, gram=np.full(L.gram.shape, bits, np.uint32).view(np.float32))
    gpu, _ = gpu_select(L, criterion=criterion, want_debug=False)
    check_lists_valid(L, gpu["kept_count"].reshape(-1), gpu["kept_idx"].reshape(-1, L.n_kb), L.budgets,
                      np.arange(L.H * L.n_qb))

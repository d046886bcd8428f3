"""GPU parity of the JS distance where a row's sweeps are shared by two or
four thread groups (calls of few rows over at least 16 sweeps of a row), and
where a block shares one token (calls of few tokens): both
sides of every line of that choice, ragged last sweeps, groups whose elements
are all masked, and values on both sides of the bf16 exp table, against the
CPU oracle with the bars of tests/test_gpu_js.py.
"""

import numpy as np
import pytest

from synth import logits as slog
from tests.test_gpu_js import _check, _run

pytestmark = pytest.mark.gpu

SWEEP = {"f32": 256 * 4, "bf16": 256 * 8}  # elements of one sweep


@pytest.fixture(scope="module")
def env():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_2606_22768_amd as fgd

    return fgd, torch


def _case(M, U, sweeps, over, dtype, seed):
    """Logits whose rows take `sweeps` sweeps and `over` elements."""
    K = sweeps * SWEEP[dtype] + over
    ldk = (K + 7) // 8 * 8
    A, W = slog.numpy_logits(M, U, K, ldk, dtype, seed=seed)
    return K, A, W


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("sweeps,over", [(15, 0), (15, 1), (16, 0), (16, 1), (17, 5), (18, -1), (19, 100), (33, 3)])
def test_sweeps_across_the_groups(env, sweeps, over, dtype):
    fgd, torch = env
    for M, U, k in ((1, 1, 1), (3, 2, 100), (2, 2, 400), (9, 1, 600)):
        print(f"[js split] {dtype} sweeps {sweeps} over {over} M {M} U {U} k {k}", flush=True)
        K, A, W = _case(M, U, sweeps, over, dtype, seed=sweeps + M)
        _check(fgd, torch, A, W, dtype, K, k)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_rows_at_the_lines(env, dtype):
    """Calls one row short of, at and past one and three rows per CU: the same
    tokens' results, whichever kernel streams their rows (equal token sets, d
    within a few units of float64 rounding of the largest distance)."""
    fgd, torch = env
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    K, A, W = _case(1, 3 * cus // 2 + 2, 16, 3, dtype, seed=5)
    full = None
    for U in (3 * cus // 2 + 2, 3 * cus // 2, cus // 2 + 1, cus // 2, 3):
        print(f"[js split] {dtype} U {U}", flush=True)
        d, _, tops = _run(fgd, torch, A[:U], np.ascontiguousarray(W[:, :U]), dtype, K, 100)
        if full is None:
            full = d, tops
        assert np.array_equal(tops, full[1][:U])
        # JS is a sum of 100 terms of at most 1, each a few roundings of log-probabilities below 32.
        assert np.abs(d ** 2 - full[0][:, :U] ** 2).max() <= 128 * 32 * 2.0 ** -52
    K2, A2, W2 = K, A[:3], np.ascontiguousarray(W[:, :3])
    _check(fgd, torch, A2, W2, dtype, K2, 100)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("dead", [(0, 1), (1, 2), (3, 4), (0, 3), (1, 4), (2, 4)])
def test_masked_groups(env, dead, dtype):
    """Quarters of the row masked (-inf): groups without a finite value; and
    a group's worth of values far outside the bf16 table."""
    fgd, torch = env
    K, A, W = _case(3, 2, 16, -7, dtype, seed=31)
    q = 4 * SWEEP[dtype]
    low = np.float32(-np.inf) if dtype == "f32" else np.uint16(0xFF80)
    big = np.float32(-300.0) if dtype == "f32" else np.uint16(0xC396)
    for fill in (low, big):
        a, w = A.copy(), W.copy()
        a[:, dead[0] * q:dead[1] * q] = fill
        w[..., dead[0] * q:dead[1] * q] = fill
        w[0] = a  # a worker equal to the averaged model: exactly 0
        d = _check(fgd, torch, a, w, dtype, K, 100)
        assert (d[0] == 0).all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("k,per_cu", [(100, 2), (256, 2), (257, 3), (512, 3)])
def test_tokens_at_the_lines(env, k, per_cu, dtype):
    """Tokens at and past the count up to which a block shares one token's
    terms, and worker counts that leave its waves without a worker or need
    more than one turn."""
    fgd, torch = env
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    K = 600
    for M, U in ((1, 3), (2, 3), (4, 3), (5, 3), (9, 3), (17, 2), (3, per_cu * cus), (3, per_cu * cus + 1)):
        print(f"[js share] {dtype} k {k} M {M} U {U}", flush=True)
        A, W = slog.numpy_logits(M, U, K, K, dtype, seed=k + M)
        _check(fgd, torch, A, W, dtype, K, k)

"""GPU parity of the JS distance where a row's sweeps are shared by four
thread groups (calls of at most one row per CU over at least 16 sweeps of a
row) or two (up to three rows per CU), and where a block shares one token
(calls of few tokens and more than 8 candidates) or a wave takes it: both
sides of every line of that choice, ragged last sweeps, groups whose elements
are all masked, and values on both sides of the bf16 exp table, against the
CPU oracle with the bars of tests/test_gpu_js.py.
"""

import numpy as np
import pytest

from oracle import js as ojs
from synth import logits as slog
from tests.test_gpu_js import _assert_d_close, _check, _js_bar, _run, _values

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


def _check_some(fgd, torch, A, W, dtype, K, k, n=6):
    """_check on n tokens of the call, its first and last among them; returns
    the distances of all."""
    d, mean, tops = _run(fgd, torch, A, W, dtype, K, k)
    at = np.unique(np.linspace(0, A.shape[0] - 1, n).astype(int))
    za, zw = _values(A[at], dtype)[:, :K], _values(W[:, at], dtype)[:, :, :K]
    rd, _, rtops = ojs.js_distances(zw, za, k)
    assert np.array_equal(tops[at], rtops), "top-k token sets differ"
    _assert_d_close(d[:, at], rd, _js_bar(zw, za, K, k, rd))
    assert np.all(np.abs(mean - d.mean(axis=1)) <= 1e-13 * mean + 1e-15)
    return d


def _tokens_of_two_groups(torch, M):
    """Tokens whose rows number a few more than one per CU (two groups a row)."""
    return torch.cuda.get_device_properties(0).multi_processor_count // (M + 1) + 2


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("sweeps,over", [(15, 0), (15, 1), (16, 0), (16, 1), (17, 5), (18, -1), (19, 100), (33, 3)])
def test_sweeps_across_the_groups(env, sweeps, over, dtype):
    fgd, torch = env
    for M, U, k in ((1, 1, 1), (3, 2, 100), (2, 2, 400), (9, 1, 600)):
        print(f"[js split] {dtype} sweeps {sweeps} over {over} M {M} U {U} k {k}", flush=True)
        K, A, W = _case(M, U, sweeps, over, dtype, seed=sweeps + M)
        _check(fgd, torch, A, W, dtype, K, k)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("sweeps,over,k", [(16, 0, 100), (17, 5, 400), (18, -1, 1), (33, 3, 300)])
def test_sweeps_across_two_groups(env, sweeps, over, k, dtype):
    fgd, torch = env
    for M in (2, 5):
        U = _tokens_of_two_groups(torch, M)
        print(f"[js split] two groups: {dtype} sweeps {sweeps} over {over} M {M} U {U} k {k}", flush=True)
        K, A, W = _case(M, U, sweeps, over, dtype, seed=sweeps + M)
        _check_some(fgd, torch, A, W, dtype, K, k)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_rows_past_the_lines(env, dtype):
    """More rows than the chip's blocks take at once, of 16 sweeps and of 17:
    a row per group again (js_rows_kernel), against the oracle."""
    fgd, torch = env
    U = torch.cuda.get_device_properties(0).multi_processor_count + 4  # 3 rows a token
    for sweeps, over, k in ((16, 0, 100), (17, 3, 300)):
        print(f"[js split] {dtype} sweeps {sweeps} over {over} M 2 U {U}", flush=True)
        K, A, W = _case(2, U, sweeps, over, dtype, seed=sweeps)
        _check_some(fgd, torch, A, W, dtype, K, k, n=12)


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
@pytest.mark.parametrize("dead", [(0, 2), (2, 4), (1, 4)])
def test_masked_groups_of_two(env, dead, dtype):
    """The same for rows of two groups: one group, or all but a quarter of the
    row, without a finite value; or far outside the bf16 table."""
    fgd, torch = env
    M = 3
    K, A, W = _case(M, _tokens_of_two_groups(torch, M), 16, -7, dtype, seed=32)
    q = 4 * SWEEP[dtype]
    low = np.float32(-np.inf) if dtype == "f32" else np.uint16(0xFF80)
    big = np.float32(-300.0) if dtype == "f32" else np.uint16(0xC396)
    for fill in (low, big):
        a, w = A.copy(), W.copy()
        a[:, dead[0] * q:dead[1] * q] = fill
        w[..., dead[0] * q:dead[1] * q] = fill
        w[0] = a  # a worker equal to the averaged model: exactly 0
        d = _check_some(fgd, torch, a, w, dtype, K, 100)
        assert (d[0] == 0).all()


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


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("k,K,per_cu", [(100, 600, 2), (300, 1100, 3)])
def test_tokens_of_one_wave(env, k, K, per_cu, dtype):
    """One token past the count of a block per token: every number of lanes
    per worker, worker counts of more than one turn, and among the tokens rows
    of equal logits (more candidates than a wave holds: the radix kernel)."""
    fgd, torch = env
    U = per_cu * torch.cuda.get_device_properties(0).multi_processor_count + 1
    for M in (1, 2, 3, 5, 9, 17):
        print(f"[js wave] {dtype} k {k} M {M} U {U}", flush=True)
        A, W = slog.numpy_logits(M, U, K, (K + 7) // 8 * 8, dtype, seed=k + M)
        A[5::97, :K] = A[0, 0]
        d = _check_some(fgd, torch, A, W, dtype, K, k, n=40)
        assert np.isfinite(d).all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("k", [7, 8, 9, 16, 17])
def test_few_candidates(env, k, dtype):
    """At most 8 candidates take a wave per token and 8 lanes per worker, but
    a block per token with two workers at most or from a third of a token per
    CU on up to one; more candidates a block per token."""
    fgd, torch = env
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for M, U in ((1, 3), (2, 3), (3, 3), (4, 3), (5, 3), (9, 3), (17, 3), (3, cus // 3), (9, cus // 3 + 1),
                 (5, cus), (2, cus), (2, cus + 1), (3, cus + 1)):
        print(f"[js few] {dtype} k {k} M {M} U {U}", flush=True)
        A, W = slog.numpy_logits(M, U, 600, 600, dtype, seed=k + M)
        _check(fgd, torch, A, W, dtype, 600, k)

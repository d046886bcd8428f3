"""Times of one call against another of the same build, in one process and in
turn, where a dispatch or a schedule went wrong once: a call that does less of
the same work, or the same work on rows that lie otherwise, takes no longer
than the bound, which lies between the ratio with the fault and without it
(both stated).  Absolute times are the benchmark's.
"""

import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_2606_22768_amd as fgd

    return fgd, torch


def _times(torch, *calls, rounds=9, n=6):
    """The least time per call (us) of each, over rounds in turn."""
    for call in calls:
        for _ in range(3):
            call()
    best = [float("inf")] * len(calls)
    for r in range(rounds):
        for i, call in enumerate(calls) if r % 2 == 0 else reversed(list(enumerate(calls))):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(n):
                call()
            b.record()
            b.synchronize()
            best[i] = min(best[i], a.elapsed_time(b) * 1e3 / n)
    return best


def _ring(M):
    from synth import configs

    return configs.topology(("ring", "metropolis", 0.0), M, 1, 0)


def _engine(fgd, M, P, dtype, mix1, mix2, ld=None, with_x=False):
    """An engine and its arrays, all zero, one after another."""
    eng = fgd.Engine(M, P, (P + 7) // 8 * 8 if ld is None else ld, dtype)
    for slot, kind in (("mix1", mix1), ("mix2", mix2)):
        if kind == "ring":
            eng.set_topology_dict(slot, _ring(M))
        else:
            eng.set_topology(slot, kind)
    mem = eng.alloc_state(spread=False, with_x=with_x)
    for k in ("theta_prev", "theta_local", "momentum") + (("x",) if with_x else ()):
        mem[k].zero_()
    return eng, mem


@pytest.mark.parametrize("mix1,mix2", [("global", "identity"), ("identity", "global")])
def test_three_workers_take_no_longer_than_four(env, mix1, mix2):
    """bf16 steps whose kinds are read at run time.  Three workers took 1.80
    times as long as four with one row load in flight at a time, 1.08 with
    all of them (322 and 193 us; four workers 179)."""
    fgd, torch = env
    P = 16_000_000
    runs, keep = [], []
    for M in (3, 4):
        eng, mem = _engine(fgd, M, P, "bf16", mix1, mix2)
        cd = torch.zeros((eng.num_cd_rows(), M), dtype=torch.float64, device="cuda")
        runs.append(lambda e=eng, m=mem, c=cd: e.outer_step(m["theta_prev"], m["theta_local"], m["momentum"], c))
        keep.append(eng)
    three, four = _times(torch, *runs)
    print(f"[times] step {mix1} {mix2}: three workers {three:.0f} us, four {four:.0f} us", flush=True)
    for eng in keep:
        eng.close()
    assert three <= 1.4 * four


def test_rows_off_the_cache_lines(env):
    """float32 rows that start inside a 128-byte line against rows that do
    not: with a block's waves apart, so that each fetches the lines they
    share, the blocking half took 1.26 times as long, together 1.12."""
    fgd, torch = env
    M, P = 28, 9_123_457
    runs, keep = [], []
    for ld in ((P + 7) // 8 * 8, (P + 31) // 32 * 32):
        eng, mem = _engine(fgd, M, P, "f32", "global", "ring", ld=ld, with_x=True)
        runs.append(lambda e=eng, m=mem: e.outer_step_blocking(m["x"], m["theta_prev"], m["theta_local"],
                                                               m["momentum"]))
        keep.append(eng)
    off, on = _times(torch, *runs)
    print(f"[times] blocking half: rows off the lines {off:.0f} us, on them {on:.0f} us", flush=True)
    for eng in keep:
        eng.close()
    assert off <= 1.22 * on  # nearer the fault: the two engines' arrays lie in different places


@pytest.mark.parametrize("M", [17, 20])
def test_mix1_half_takes_its_best_grid(env, M):
    """The Mix1 half's own grid against two blocks per CU: 1.12 times its
    time with as many blocks as fit, 1.00 now (the same grid)."""
    fgd, torch = env
    eng, mem = _engine(fgd, M, 4_000_000, "f32", "global", "ring", with_x=True)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    own, two = _times(torch, lambda: eng.mix1(mem["theta_prev"], mem["x"]),
                      lambda: eng.mix1(mem["theta_prev"], mem["x"], num_blocks=2 * cus))
    print(f"[times] Mix1 half, {M} workers: {own:.0f} us, with two blocks per CU {two:.0f} us", flush=True)
    eng.close()
    assert own <= 1.06 * two


@pytest.mark.parametrize("M", [64, 200])
def test_js_of_fewer_candidates(env, M):
    """One token's distances over its top 4 take no longer than over its top
    24: 1.10 times as long where a block shared the 4, now 0.92."""
    fgd, torch = env
    gen = torch.Generator(device="cuda").manual_seed(1)
    A = torch.randn((1, 600), device="cuda", generator=gen)
    W = torch.randn((M, 1, 600), device="cuda", generator=gen)
    ws = torch.empty(fgd.fgd_js_workspace_size("f32", M, 1), dtype=torch.uint8, device="cuda")
    few, more = _times(torch, *[lambda k=k: fgd.js_distance(A, W, top_k=k, workspace=ws) for k in (4, 24)], n=40)
    print(f"[times] JS, {M} workers: top 4 {few:.1f} us, top 24 {more:.1f} us", flush=True)
    assert few <= 1.02 * more

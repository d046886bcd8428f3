"""GPU parity of the worker classes: every worker count that is no power of
two runs on kernels built for the top of its class, whose rows past M read 0
and write nothing.  Both ends of every class (the fewest and the most rows
that do not exist) on a few tiles, and four classes on rows so long that
blocks take several tiles, against the CPU oracle with the bars of
tests/_parity.py; and the memory around the arrays unchanged.
"""

import pytest

from tests import _parity as pa

pytestmark = pytest.mark.gpu

G, ID = ("global",), ("identity",)
ENDS = [3, 5, 6, 7, 9, 10, 11, 12, 13, 14, 15, 17, 20, 21, 24, 25, 28, 29, 31, 33, 40, 41, 48, 49, 56, 57, 63]

# (mix1, K1, mix2, K2, state mixed, subset)
MIXES = [
    (G, 1, ("ring", "metropolis", 0.1), 1, False, None),
    (("er_mh", 0.3, 0.2), 1, ("er_mh", 0.5, 0.2), 2, False, None),
    (G, 1, ("ring_self", 0.3), 2, True, None),
    (ID, 0, ("ring_self", 0.3), 1, False, [(3, 700), (2040, 2051)]),
]


@pytest.fixture(scope="module")
def env():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_2606_22768_amd as fgd

    return fgd, torch


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M", ENDS)
def test_class_ends(env, M, dtype):
    fgd, torch = env
    for i, (s1, k1, s2, k2, state, subset) in enumerate(MIXES):
        print(f"[classes] M={M} {dtype} mix {i}", flush=True)
        pa.run_case(fgd, torch, M, 2051, dtype, s1, k1, s2, k2, seed=61 + i, mom_std=1e-3, mix1_state=state,
                    subset=subset)


# Rows longer than every resident block takes at once: 256 blocks of 1024
# parameters up to 16 workers, 768 of 512 (three blocks fit a CU beside their
# LDS rows) up to 32, 768 of 256 beyond.
LONG = [(6, 300_003), (11, 300_003), (12, 300_003), (23, 450_003), (24, 450_003), (48, 300_003), (49, 300_003)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,P", LONG)
def test_blocks_of_several_tiles(env, M, P, dtype):
    """Consensus sums carried from tile to tile, the rounds' LDS columns used
    again, a subset whose segments begin and end tiles apart."""
    fgd, torch = env
    for i, (s1, k1, s2, k2, state, subset) in enumerate(MIXES):
        if subset:
            subset = [(3, 700), (5_000, 140_001), (262_150, P - 1)]
        print(f"[classes] M={M} P={P} {dtype} mix {i}", flush=True)
        pa.run_case(fgd, torch, M, P, dtype, s1, k1, s2, k2, seed=71 + i, mom_std=1e-3, mix1_state=state,
                    subset=subset)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,P", LONG)
def test_split_halves_of_several_tiles(env, M, P, dtype):
    """The same through both halves of a split round: Mix1 blocks that take
    several chunks, the blocking half's tile loop with and without a subset."""
    from tests.test_gpu_split import _split_case

    _split_case(env, (M, P, dtype, G, 1, ("ring", "metropolis", 0.1), 1, False, None), True)
    _split_case(env, (M, P, dtype, ("er_mh", 0.4, 0.2), 2, ("ring_self", 0.3), 1, True,
                      [(3, 700), (5_000, 140_001), (262_150, P - 1)]), False)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,P", [(M, P) for M in (3, 6, 11, 24, 49) for P in (2051, 2112)] + LONG[::2])
def test_steps_without_tables(env, M, P, dtype):
    """No round gathers through LDS; rows that start inside a 128-byte line
    and (P = 2112) rows that are whole lines, which decides whether a block's
    waves meet at its tiles.  Both halves too."""
    from tests.test_gpu_split import _split_case

    fgd, torch = env
    for i, (s1, k1, s2, k2, state) in enumerate([(G, 1, ID, 0, False), (ID, 0, G, 1, False), (G, 1, ID, 0, True)]):
        print(f"[classes] M={M} P={P} {dtype} mix {i}", flush=True)
        pa.run_case(fgd, torch, M, P, dtype, s1, k1, s2, k2, seed=81 + i, mom_std=1e-3, mix1_state=state)
    _split_case(env, (M, P, dtype, G, 1, ID, 0, False, None), True)
    _split_case(env, (M, P, dtype, ID, 0, ("ring", "metropolis", 0.1), 1, False, None), False)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,P", [(6, 600_003), (12, 600_003), (17, 600_003), (24, 1_100_003), (31, 1_100_003),
                                 (48, 600_003)])
def test_consensus_of_several_tiles(env, M, P, dtype):
    """The standalone consensus kernel, up to eight blocks per CU."""
    import numpy as np

    import oracle
    from synth import tensors

    fgd, torch = env
    ld = pa.aligned_ld(P)
    x, _, _ = tensors.numpy_inputs(M, ld, dtype=dtype, seed=M)
    ref = oracle.consensus(x, P=P)
    eng = fgd.Engine(M, P, ld, dtype)
    g = torch.from_numpy(x if dtype == "f32" else x.view(np.int16)).cuda()
    out = torch.full((M,), float("nan"), dtype=torch.float64, device="cuda")
    eng.consensus_distance(g if dtype == "f32" else g.view(torch.bfloat16), out)
    torch.cuda.synchronize()
    pa.compare_cd(out.cpu().numpy()[None, :], ref[None, :])
    eng.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M", [3, 9, 17, 33, 57])
def test_memory_past_the_last_row(env, M, dtype):
    """Eight rows of NaN follow each array's last row (and the rows' padding
    is NaN): no output depends on them and none is written, by the fused
    step, both split halves and the consensus kernel."""
    from synth import configs

    fgd, torch = env
    P, ld = 2051, 2056
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    t1 = configs.topology(G, M, 1, 0)
    t2 = configs.topology(("ring", "metropolis", 0.1), M, 1, 0, step=1)

    def run(fill):
        gen = torch.Generator(device="cuda").manual_seed(3)
        buf = {}
        for name, d, std in (("prev", dt, 0.02), ("local", dt, 0.02), ("mom", torch.float32, 1e-3), ("x", dt, 0.02)):
            buf[name] = torch.full((M + 8, ld), fill, dtype=d, device="cuda")
            buf[name][:M, :P] = (torch.randn((M, P), generator=gen, device="cuda") * std).to(d)
        row = {k: v[:M] for k, v in buf.items()}
        eng = fgd.Engine(M, P, ld, dtype)
        eng.set_topology_dict("mix1", t1)
        eng.set_topology_dict("mix2", t2)
        r1, r2 = eng.num_cd_rows_split()
        cd = [torch.zeros((r, M), dtype=torch.float64, device="cuda") for r in (eng.num_cd_rows(), r1, r2, 1)]
        eng.outer_step(row["prev"], row["local"], row["mom"], cd[0])
        eng.mix1(row["prev"], row["x"], row["mom"], cd[1])
        eng.outer_step_blocking(row["x"], row["prev"], row["local"], row["mom"], cd[2], write_local=True)
        eng.consensus_distance(row["x"], cd[3])
        torch.cuda.synchronize()
        for v in buf.values():
            for rest in (v[M:], v[:, P:]):
                assert bool((rest.isnan() if fill != fill else rest == fill).all())
        eng.close()
        return [v[:M, :P].clone() for v in buf.values()] + cd

    for a, b in zip(run(0.0), run(float("nan"))):
        assert torch.equal(a, b)

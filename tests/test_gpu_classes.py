"""GPU parity of the worker classes: every worker count that is no power of
two runs on kernels built for the top of its class, whose rows past M read 0
and write nothing.  Both ends of every class (the fewest and the most rows
that do not exist), against the CPU oracle with the bars of tests/_parity.py,
and the memory around the arrays unchanged.
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

"""What runs under a plan's name at sizes where a form runs on other kernels:
the autotuner times every set of kernels once, the timed brackets hold the
whole readout, and the 16-atom readout tiles at the largest system that keeps
them agree with the streamed kernels bit for bit."""
import ctypes as C
import dataclasses

import pytest
import torch

from workloads import make_workload
from workloads.configs import make_params
from gpu_helpers import gpu, need_gpu

pytestmark = gpu


def _setup(g, n, width):
    batch, _, spec = make_workload("liquid", n=n)
    params = make_params(dataclasses.replace(spec.model, hidden=(width, width), n_heads=1), 5)
    system = g.System.from_batch(batch, "cuda")
    return system, g.build_neighbors(system, spec.model.r_cut, 0.0), g.Model.from_params(params, "cuda")


@pytest.mark.parametrize("precision,n,fused8,tile", [("fp32", 2048, True, True), ("fp32", 2056, False, True),
                                                     ("bf16", 2056, True, True), ("fp32", 8200, False, False),
                                                     ("bf16", 8200, True, False)])
def test_autotune_times_each_set_of_kernels_once(precision, n, fused8, tile):
    g = need_gpu()
    from paper_2505_22168_amd import autotune
    print(f"autotuned kernels {precision} N={n}", flush=True)
    system, nl, model = _setup(g, n, 64)
    plan, table = autotune.run_autotune(g.EnergyForces(model, system, nl, precision=precision, stress=True), reps=2)
    forms = {(p["schedule"], p["tile_atoms"], p["readout"]) for p, _, _ in table}
    assert forms == {(1, 16, 1), (2, 0, 2)} | ({(1, 8, 1)} if fused8 else set()) | ({(2, 0, 1)} if tile else set())
    assert (plan["schedule"], plan["tile_atoms"], plan["readout"]) in forms


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("n,width", [(4096, 512), (8192, 256)])
def test_largest_readout_tiles_equal_streamed_bitwise(precision, n, width):
    g = need_gpu()
    print(f"readout tiles {precision} N={n} width={width}", flush=True)
    system, nl, model = _setup(g, n, width)
    a, b = (g.EnergyForces(model, system, nl, precision=precision, stress=True, plan=(2, 16, r))(sync=True)
            for r in (1, 2))
    assert torch.equal(a.atomic_energy, b.atomic_energy) and torch.equal(a.energy, b.energy)
    assert torch.equal(a.forces, b.forces) and torch.equal(a.stress, b.stress)


def test_bench_stages_hold_the_whole_readout():
    """A TILE plan on the streamed kernels: its readout stage is the three kernels' sum, so it
    holds at least their network (the largest of them at 2x512)."""
    g = need_gpu()
    import bench
    from paper_2505_22168_amd import _capi as A
    print("bench stages of a TILE plan on the streamed kernels", flush=True)
    system, nl, model = _setup(g, 6000, 512)
    events = bench.HipEvents()
    tile, stream = (bench.run_path(g, A, model, system, nl, "fp32", 10, 3, events, plan=(2, 16, r))[1] for r in (1, 2))
    assert tile["readout_tile"] > 0.8 * stream["readout_network"]

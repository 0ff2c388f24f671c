"""The one-atom-per-lane invariant backward at the edges of its 64-atom runs
(one short run, exactly one, a run and one atom, a short last run) behind
both readouts, against the FP64 oracle at the FP32 bounds."""
import numpy as np
import pytest

from oracle import brute_force_neighbors, evaluate
from workloads import make_workload
from gpu_helpers import gpu, need_gpu

pytestmark = gpu


@pytest.mark.parametrize("n", [3, 63, 64, 65, 130])
@pytest.mark.parametrize("readout", [1, 2])
def test_run_edges_match_oracle(n, readout):
    g = need_gpu()
    batch, params, spec = make_workload("liquid", n=n)
    print(f"contract lanes N={n} readout={readout}", flush=True)
    system = g.System.from_batch(batch, "cuda")
    nl = g.build_neighbors(system, spec.model.r_cut, 0.0)
    model = g.Model.from_params(params, "cuda")
    ref = evaluate(batch, params, brute_force_neighbors(batch, spec.model.r_cut))
    out = g.EnergyForces(model, system, nl, precision="fp32", stress=True, plan=(2, 16, readout))(sync=True)
    assert np.abs(out.energy.cpu().numpy() - ref.energy).max() / n < 1e-5
    assert np.abs(out.forces.cpu().numpy()[:n] - ref.forces).max() < 1e-4
    assert np.abs(out.stress.cpu().numpy() - ref.stress).max() < 1e-6

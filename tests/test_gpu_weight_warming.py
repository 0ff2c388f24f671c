"""Fused tiles beside the blocks that only read the weights (FP32 2x256, BF16
2x512): a structure evaluated alone, where those blocks run, and as the first of
two, where the tiles leave them no room, gives the same energies and forces bit
for bit; one tile, some, and the most there is room for."""
import dataclasses

import numpy as np
import pytest
import torch

from workloads import make_workload
from workloads.configs import make_params
from gpu_helpers import gpu, need_gpu

pytestmark = gpu


@pytest.mark.parametrize("n,other", [(8, 1600), (1000, 1000), (8 * 192, 512)])
@pytest.mark.parametrize("precision,width", [("fp32", 256), ("bf16", 512)])
def test_alone_and_beside_another(n, other, precision, width):
    g = need_gpu()
    a, _, spec = make_workload("liquid", n=n)
    b, _, _ = make_workload("liquid", n=other)
    params = make_params(dataclasses.replace(spec.model, hidden=(width, width), n_heads=1), 7)
    print(f"weight warming N={n} {precision} width={width}", flush=True)
    model = g.Model.from_params(params, "cuda")
    both = g.System(np.concatenate([a.pos, b.pos]), np.concatenate([a.species, b.species]),
                    np.concatenate([a.cell, b.cell]), np.concatenate([a.pbc, b.pbc]), [0, n, n + other])
    out = []
    for system in (g.System.from_batch(a), both):
        nl = g.build_neighbors(system, spec.model.r_cut, 0.0)
        o = g.EnergyForces(model, system, nl, precision=precision, plan=(1, 64, 0, 8))(sync=True)
        out.append((o.atomic_energy[:n].clone(), o.forces[:n].clone()))
    assert torch.isfinite(out[0][1]).all()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])

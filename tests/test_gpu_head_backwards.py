"""One backward per head (force variance, per-head forces) at the edges of the
streamed head kernels and the matrix pair backward: atoms that end inside a
16-row block and a 64-atom run, head counts that end inside a block of four
heads, and a list too short to lend its gradients' memory (the readout tile
runs the heads then), against the FP64 oracle at the FP32 bounds; and few heads
of a system past the tile's first round against the tile."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import brute_force_neighbors, evaluate
from workloads import make_workload
from workloads.configs import make_params
from gpu_helpers import gpu, need_gpu
from paper_2505_22168_amd import _capi as A

pytestmark = gpu


@pytest.mark.parametrize("n,width,heads", [(3, 64, 2), (16, 128, 16), (65, 64, 9), (65, 256, 8), (130, 256, 13), (37, 128, 6),
                                           (64, 64, 7)])
@pytest.mark.parametrize("room", [False, True])
def test_heads_match_oracle(n, width, heads, room):
    g = need_gpu()
    batch, _, spec = make_workload("liquid", n=n)
    params = make_params(dataclasses.replace(spec.model, hidden=(width, width), n_heads=heads), 7)
    onl = brute_force_neighbors(batch, spec.model.r_cut)
    n_pairs = int(onl.n_pairs)
    print(f"heads N={n} width={width} M={heads} room={room} pairs={n_pairs}", flush=True)
    # swish' of both layers, [2][N][width], has to fit 3 * capacity * heads words
    capacity = max(n_pairs, 2 * n * width) if room else n_pairs
    system = g.System.from_batch(batch, "cuda")
    nl = g.build_neighbors(system, spec.model.r_cut, 0.0, capacity=capacity)
    model = g.Model.from_params(params, "cuda")
    ref = evaluate(batch, params, onl, want_force_var=True)
    out = g.EnergyForces(model, system, nl, precision="fp32", stress=True, force_var=True)(sync=True)
    assert np.abs(out.energy.cpu().numpy() - ref.energy).max() / n < 1e-5
    assert np.abs(out.forces.cpu().numpy()[:n] - ref.forces).max() < 1e-4
    fh = out.forces_heads.cpu().numpy()[:, :n]
    assert np.abs(fh.mean(0) - ref.forces).max() < 1e-4
    assert np.allclose(((fh - fh.mean(0)) ** 2).sum(-1).mean(0), ref.force_var, rtol=1e-3, atol=1e-5)
    assert np.allclose(out.force_var.cpu().numpy()[:n], ref.force_var, rtol=1e-3, atol=1e-5)


@pytest.mark.parametrize("heads", [4, 6])
def test_few_heads_past_one_round_match_the_tile(heads):
    g = need_gpu()
    n = 4200
    batch, _, spec = make_workload("liquid", n=n)
    params = make_params(dataclasses.replace(spec.model, hidden=(64, 64), n_heads=heads), 7)
    print(f"heads N={n} M={heads}", flush=True)
    system = g.System.from_batch(batch, "cuda")
    nl = g.build_neighbors(system, spec.model.r_cut, 0.0)
    model = g.Model.from_params(params, "cuda")
    got = []
    for flags in (0, A.GMNN_HEADS_TILE):
        ev = g.EnergyForces(model, system, nl, precision="fp32", stress=True, force_var=True)
        ev.flags |= flags
        got.append(ev(sync=True))
    a, b = got
    assert torch.equal(a.energy, b.energy)  # the forward's sums are the same
    assert (a.forces_heads - b.forces_heads)[:, :n].abs().max().item() < 1e-4
    assert torch.allclose(a.force_var[:n], b.force_var[:n], rtol=1e-3, atol=1e-5)
    assert (a.stress - b.stress).abs().max().item() < 1e-6

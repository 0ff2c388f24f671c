"""One backward per head on the lists that reach its other branches, against the
FP64 oracle: lists with a skin (records of pairs beyond the cutoff, whole
quads of heads and not), with and without the uncertainty bias's head weights;
lists too short to lend the streamed kernels their memory, where the readout
tile runs the heads before the matrix pair backward; and the streamed kernels
in BF16 at head counts and widths that end inside a block of four heads."""
import dataclasses

import numpy as np
import pytest

from oracle import brute_force_neighbors, evaluate
from oracle.gmnn import evaluate_udd
from workloads import make_batch, make_workload
from workloads.configs import make_params
from gpu_helpers import gpu, need_gpu

pytestmark = gpu

A, B = 1.0, 1.2


def _case(n, width, heads, stretch=1.0):
    batch, _, spec = make_workload("liquid", n=n)
    if stretch != 1.0:
        batch = make_batch([(batch.pos * np.float32(stretch), batch.species, batch.cell[0] * stretch, batch.pbc[0])])
    return batch, spec, make_params(dataclasses.replace(spec.model, hidden=(width, width), n_heads=heads), 11)


def _run(g, batch, spec, params, skin=0.0, capacity=None, precision="fp32", udd=None):
    system = g.System.from_batch(batch, "cuda")
    nl = g.build_neighbors(system, spec.model.r_cut, skin, capacity=capacity)
    model = g.Model.from_params(params, "cuda")
    return g.EnergyForces(model, system, nl, precision=precision, stress=True, force_var=True, udd=udd)(sync=True)


def _check(out, ref, batch):
    n = batch.n_atoms
    assert np.abs(out.energy.cpu().numpy() - ref.energy).max() / n < 1e-5
    assert np.abs(out.forces.cpu().numpy()[:n] - ref.forces).max() < 1e-4
    assert np.abs(out.stress.cpu().numpy() - ref.stress).max() < 1e-6
    fh = out.forces_heads.cpu().numpy()[:, :n]
    assert np.allclose(((fh - fh.mean(0)) ** 2).sum(-1).mean(0), ref.force_var, rtol=1e-3, atol=1e-5)
    assert np.allclose(out.force_var.cpu().numpy()[:n], ref.force_var, rtol=1e-3, atol=1e-5)


@pytest.mark.parametrize("n,heads", [(41, 8), (41, 11), (767, 6), (768, 6), (820, 7), (820, 8)])
def test_skin_list(n, heads):
    g = need_gpu()
    batch, spec, params = _case(n, 64, heads)
    print(f"heads on a skin list N={n} M={heads}", flush=True)
    ref = evaluate(batch, params, brute_force_neighbors(batch, spec.model.r_cut), want_force_var=True)
    _check(_run(g, batch, spec, params, skin=1.0), ref, batch)


@pytest.mark.parametrize("skin", [0.0, 1.0])
@pytest.mark.parametrize("heads", [8, 10])
def test_bias_weights(heads, skin):
    g = need_gpu()
    batch, spec, params = _case(130, 64, heads)
    print(f"heads with bias weights M={heads} skin={skin}", flush=True)
    out = _run(g, batch, spec, params, skin=skin, udd=(A, B))
    onl = brute_force_neighbors(batch, spec.model.r_cut)
    ref = evaluate_udd(batch, params, onl, A, B)
    n = batch.n_atoms
    assert np.abs(ref.bias_energy).min() > 1e-4  # the bias acts
    assert np.abs(out.bias_energy.cpu().numpy() - ref.bias_energy).max() < 1e-5
    assert np.abs(out.forces.cpu().numpy()[:n] - ref.forces).max() < 1e-4
    assert np.abs(out.stress.cpu().numpy() - ref.stress).max() < 1e-6
    plain = evaluate(batch, params, onl, want_force_var=True)
    assert np.allclose(out.force_var.cpu().numpy()[:n], plain.force_var, rtol=1e-3, atol=1e-5)


@pytest.mark.parametrize("n,heads", [(70, 8), (820, 9)])
@pytest.mark.parametrize("room", [False, True])
def test_short_list(n, heads, room):
    g = need_gpu()
    width = 256
    batch, spec, params = _case(n, width, heads, stretch=1.7)
    onl = brute_force_neighbors(batch, spec.model.r_cut)
    # swish' of both layers, 8 width bytes an atom, against 12 bytes a pair and head
    assert 8 * width * n > 12 * onl.n_pairs * heads
    print(f"heads of a short list N={n} M={heads} room={room} pairs={onl.n_pairs}", flush=True)
    ref = evaluate(batch, params, onl, want_force_var=True)
    _check(_run(g, batch, spec, params, capacity=n * width if room else onl.n_pairs), ref, batch)


@pytest.mark.parametrize("n,width,heads", [(65, 64, 9), (130, 256, 13), (40, 512, 11), (40, 512, 9), (200, 128, 8)])
def test_streamed_heads_bf16(n, width, heads):
    g = need_gpu()
    batch, spec, params = _case(n, width, heads)
    print(f"streamed heads BF16 N={n} width={width} M={heads}", flush=True)
    out = _run(g, batch, spec, params, precision="bf16", capacity=2 * n * width)
    ref = evaluate(batch, params, brute_force_neighbors(batch, spec.model.r_cut), bf16=True, want_force_var=True)
    assert np.abs(out.energy.cpu().numpy() - ref.energy).max() / n < 1e-5
    # the bounds of BF16 per-head forces: rounding flips of backward operands, 2^-8 of one operand each
    rms = np.sqrt(((ref.forces ** 2).sum(1) + ref.force_var).mean() / 3)
    assert np.sqrt(((out.forces.cpu().numpy()[:n] - ref.forces) ** 2).mean()) < 2e-3 * rms
    v = out.force_var.cpu().numpy()[:n]
    assert np.sqrt(((v - ref.force_var) ** 2).mean()) < 1e-2 * np.sqrt((ref.force_var ** 2).mean())

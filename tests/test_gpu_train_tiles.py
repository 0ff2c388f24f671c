"""The training kernels at the edges of their tiles (16- and 32-atom network
tiles, 6-atom invariant blocks, 64-atom backward runs)."""
import numpy as np
import pytest
import torch

from oracle import brute_force_neighbors, loss_and_param_grads
from oracle.gmnn import PARAM_NAMES
from workloads import make_batch, make_workload
from workloads.configs import ModelSpec, make_params
from workloads.structures import random_box
from gpu_helpers import gpu, need_gpu

pytestmark = gpu


@pytest.mark.parametrize("n", [1, 6, 7, 16, 17, 64, 65])
def test_tile_edges_match_oracle(n):
    g = need_gpu()
    rng = np.random.default_rng(n)
    L = max(6.0, (n / 0.1) ** (1.0 / 3.0))
    pos, sp = random_box(rng, n, L, (15, 8, 2, 1, 4), min_sep=0.9)
    batch = make_batch([(pos, sp, np.eye(3) * L, (1, 1, 1))])
    params = make_params(ModelSpec(n_species=5, hidden=(64, 64)), 7)
    print(f"training tiles N={n}", flush=True)
    _, gref, dE, dF = loss_and_param_grads(batch, params, brute_force_neighbors(batch, 5.0), np.zeros(1),
                                           rng.normal(size=(n, 3)))
    system = g.System.from_batch(batch, "cuda")
    nl = g.build_neighbors(system, 5.0)
    grads = g.param_grads(g.Model.from_params(params, "cuda"), system, nl, dE, dF)
    for k in PARAM_NAMES:
        got = grads[k].cpu().numpy().astype(np.float64).reshape(np.shape(gref[k]))
        err = np.linalg.norm(got - gref[k]) / max(np.linalg.norm(gref[k]), 1e-30)
        assert err < 1e-4, (k, err)


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_wide_tiles_add_up(precision):
    """Above 4096 atoms the 2x256 network runs 32-atom tiles: the gradients of
    a batch are the sums of its halves' (16-atom tiles).  Each side's FP32
    sums are good to about 1e-6, and the per-atom arithmetic is the same."""
    g = need_gpu()
    parts = [make_workload("train", n_structs=8, n_lo=250 + k, n_hi=290)[0] for k in range(2)]
    params = make_params(ModelSpec(n_species=5, hidden=(256, 256)), 7)
    model = g.Model.from_params(params, "cuda")
    rng = np.random.default_rng(3)
    total, whole_E, whole_F = None, [], []
    for b in parts:
        system = g.System.from_batch(b, "cuda")
        nl = g.build_neighbors(system, 5.0)
        dE, dF = rng.normal(size=b.n_structs), rng.normal(size=(b.n_atoms, 3)).astype(np.float32)
        gr = g.param_grads(model, system, nl, dE, dF, precision=precision)
        total = {k: v.double() + (0 if total is None else total[k]) for k, v in gr.items()}
        whole_E.append(dE)
        whole_F.append(dF)
    batch = make_batch([(b.pos[b.atom_ptr[s]:b.atom_ptr[s + 1]], b.species[b.atom_ptr[s]:b.atom_ptr[s + 1]], b.cell[s],
                         b.pbc[s]) for b in parts for s in range(b.n_structs)])
    assert batch.n_atoms > 4096 and max(b.n_atoms for b in parts) <= 4096
    print(f"training wide tiles {precision} N={batch.n_atoms}", flush=True)
    system = g.System.from_batch(batch, "cuda")
    nl = g.build_neighbors(system, 5.0)
    got = g.param_grads(model, system, nl, np.concatenate(whole_E), np.concatenate(whole_F), precision=precision)
    for k in PARAM_NAMES:
        err = float((got[k].double() - total[k]).norm() / total[k].norm())
        assert err < 1e-5, (k, err)


@pytest.mark.parametrize("n", [1, 7, 8, 9, 63, 65])
def test_bf16_per_head_invariant_backward_at_group_edges(n):
    """With one head the BF16 per-head double backward differs from the
    head-mean one in the invariant backward's form alone (differences of the
    exact polynomial over 8-atom groups against dual numbers): everything but
    beta is bitwise equal, and beta agrees to the differences' rounding, a few
    ulp of terms of the moments' size (1e-6), with a factor of ten to spare."""
    g = need_gpu()
    rng = np.random.default_rng(n)
    L = max(6.0, (n / 0.1) ** (1.0 / 3.0))
    pos, sp = random_box(rng, n, L, (15, 8, 2, 1, 4), min_sep=0.9)
    batch = make_batch([(pos, sp, np.eye(3) * L, (1, 1, 1))])
    model = g.Model.from_params(make_params(ModelSpec(n_species=5, hidden=(64, 64)), 7), "cuda")
    print(f"per-head backward N={n}", flush=True)
    system = g.System.from_batch(batch, "cuda")
    nl = g.build_neighbors(system, 5.0)
    dE, dF = rng.normal(size=(1, 1)), rng.normal(size=(1, n, 3)).astype(np.float32)
    a = g.param_grads(model, system, nl, dE, dF, precision="bf16", per_head=True)
    b = g.param_grads(model, system, nl, dE[:, 0], dF[0], precision="bf16")
    for k in PARAM_NAMES:
        if k != "beta":
            assert torch.equal(a[k], b[k]), k
    assert float((a["beta"] - b["beta"]).norm()) <= 1e-5 * float(b["beta"].norm())

"""FP32 wide branches whose activations overflow: the products run over three
bf16 planes per operand (csrc/branchgemm.h), and an infinity has to act as it
does in FP32 arithmetic.  One hidden unit of the first of two 256-wide layers
passes FP32's largest value on some atoms; its weights in the second layer are
positive and have one plane only (2^-10: their mid and lo planes are 0), so the
energy of a structure with such an atom is +inf.  Every other structure's
energy, from the same tiles, matches the oracle, and its forces are finite."""
import numpy as np
import pytest
import torch

import synth
from helpers import TOL, check_energies
from oracle.painn import batch_energies
from test_gpu_branch import batch, rt  # noqa: F401

pytestmark = pytest.mark.gpu

UNIT, SCALE, BIAS = 5, 0.5e38, 3.0e38         # positive on every atom
FLT_MAX = float(np.finfo(np.float32).max)


@pytest.mark.parametrize("atoms", [700, 8300])       # tiles of 32 and of 128 rows
def test_infinite_activation(rt, atoms):  # noqa: F811
    print(f"branch, overflowing activations, {atoms} atoms", flush=True)
    hp = synth.HyperParams(F=64, K=6, L=1, n_species=6, cutoff=3.0, n_heads=1, shared_dims=[],
                           branch_dims=[256, 256, 1])
    W = synth.make_weights(hp, 78)
    W["head0.0.w"][UNIT] = 0.0
    W["head0.0.w"][UNIT, 0] = SCALE
    W["head0.0.b"][UNIT] = BIAS
    W["head0.1.w"][:, UNIT] = 2.0 ** -10
    W["head0.2.w"] = np.abs(W["head0.2.w"]) * 1e-30
    m = rt.load_model(synth.weight_file_bytes(hp, W))
    b = batch(atoms, 2)
    b.dataset_id[:] = 0
    g = rt.build_graph(rt.upload_batch(b), hp.cutoff)
    s, _ = rt.features(m, g, 0, "fp32")
    z = BIAS + SCALE * s[:, 0].cpu().numpy()
    assert np.all(np.abs(z / FLT_MAX - 1) > 1e-6)     # no atom next to the edge
    over = np.add.reduceat((z > FLT_MAX).astype(int), b.struct_ptr[:-1]) > 0
    assert over.sum() >= 2 and (~over).sum() >= 5     # both kinds are there
    E = rt.forward(m, g, "fp32").cpu().numpy()
    assert np.all(np.isposinf(E[over]))
    idx = np.nonzero(~over)[0][:6].tolist()
    Er, Ar = batch_energies(b, hp, W, idx)
    check_energies(E[idx], Er, Ar, TOL["fp32"], f"overflow {atoms}")
    assert np.all(np.isfinite(E[~over]))
    E2, F = rt.forces(m, g, "fp32")
    assert np.array_equal(E2.cpu().numpy(), E)
    atom_over = np.repeat(over, np.diff(b.struct_ptr))
    assert torch.isfinite(F[torch.as_tensor(~atom_over, device=F.device)]).all()
    g.free()
    m.free()


def test_infinite_weight(rt):  # noqa: F811
    """A weight past FP32's range is an infinity there: the atoms' energies
    take the sign of the activation it meets (silu of a large positive
    pre-activation), as in FP32 arithmetic."""
    print("branch, a weight past FP32's range", flush=True)
    hp = synth.HyperParams(F=64, K=6, L=1, n_species=6, cutoff=3.0, n_heads=1, shared_dims=[],
                           branch_dims=[256, 256, 1])
    W = synth.make_weights(hp, 79)
    W["head0.0.b"][UNIT] = 50.0                       # silu(z) > 0 on every atom
    W["head0.1.w"][7, UNIT] = 1e39
    W["head0.2.w"][0, 7] = 0.25
    m = rt.load_model(synth.weight_file_bytes(hp, W))
    b = batch(40, 2)
    b.dataset_id[:] = 0
    g = rt.build_graph(rt.upload_batch(b), hp.cutoff)
    E = rt.forward(m, g, "fp32").cpu().numpy()
    assert np.all(np.isposinf(E)), E
    g.free()
    m.free()

"""Dataset ids outside [0, n_heads) with wide branches: the forces' route
differs from the narrow branches' (tests/test_gpu_forces.py), dE/dY of those
atoms is NaN and goes through the shared layers."""
import numpy as np
import pytest
import torch

import synth
from helpers import TOL, check_energies, check_forces
from oracle.forces import structure_forces
from oracle.painn import batch_energies
from test_gpu_branch import batch, rt  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shared", [[], [50], [40, 320]])
def test_invalid_ids_forces(rt, precision, shared):  # noqa: F811
    """A dataset id outside [0, n_heads): NaN energy and forces of that
    structure alone, also right after a batch of valid ids (whose dE/dY the
    workspace still holds), with and without shared layers."""
    print(f"wide branches, invalid ids, {precision}, shared {shared}", flush=True)
    hp = synth.HyperParams(F=64, K=6, L=2, n_species=6, cutoff=3.0, n_heads=4, shared_dims=shared,
                           branch_dims=[256, 1])
    W = synth.make_weights(hp, 81)
    m = rt.load_model(synth.weight_file_bytes(hp, W))
    b = batch(200, hp.n_heads)
    g = rt.build_graph(rt.upload_batch(b), hp.cutoff)
    n = b.n_struct
    assert n >= 7
    valid = np.asarray(b.dataset_id, dtype=np.int32)
    ds = torch.as_tensor(valid, device=rt.device)
    _, F0 = rt.forces(m, g, precision, dataset_id=ds)
    assert torch.isfinite(F0).all()
    bad = {0: -1, n // 2: hp.n_heads, n - 1: 1 << 30}
    ids = valid.copy()
    for k, d in bad.items():
        ids[k] = d
    E, F = rt.forces(m, g, precision, dataset_id=torch.as_tensor(ids, device=rt.device))
    E, F = E.cpu().numpy(), F.cpu().numpy()
    good = [k for k in range(n) if k not in bad]
    for k in bad:
        assert np.isnan(E[k]) and np.all(np.isnan(F[b.struct_ptr[k]:b.struct_ptr[k + 1]])), k
    ref = [structure_forces(*b.structure(k), hp, W)["F"] for k in good]
    check_forces(F, b, ref, good, {"fp64": 1e-10, "fp32": 2e-5}[precision], f"valid ones, {precision}")
    Er, Ar = batch_energies(b, hp, W, good)
    check_energies(E[good], Er, Ar, TOL[precision], f"valid ones, {precision}")
    g.free()
    m.free()

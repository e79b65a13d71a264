"""Wide branches where their rows take more space than the buffers whose place
they share: a last shared layer much wider than F, and many heads blended with
forces.  Atoms then go through in ranges."""
import pytest
import torch

import synth
from helpers import TOL, check_energies, check_forces
from oracle.forces import structure_forces, structure_forces_blend
from oracle.painn import batch_energies
from test_gpu_branch import batch, rt  # noqa: F401

pytestmark = pytest.mark.gpu


def wide_shared(rt, n_heads):  # noqa: F811
    hp = synth.HyperParams(F=64, K=6, L=1, n_species=6, cutoff=3.0, n_heads=n_heads, shared_dims=[1024],
                           branch_dims=[256, 1], blend_dims=[32])
    W = synth.make_weights(hp, 80)
    return hp, W, rt.load_model(synth.weight_file_bytes(hp, W))


@pytest.mark.parametrize("atoms", [9000, 13000])
def test_fixed_scratch_wide_shared(rt, atoms):  # noqa: F811
    """The 64 MiB entry point takes the batches that fit without the rows of
    all atoms (13,000 x 6 KiB alone exceed it), bit for bit as the allocating
    one."""
    from paper_2604_15380_amd import binding as B
    print(f"fixed scratch, 1,024-wide shared layer, {atoms} atoms", flush=True)
    hp, W, m = wide_shared(rt, 5)
    b = batch(atoms, hp.n_heads)
    g = rt.build_graph(rt.upload_batch(b), hp.cutoff)
    for ds in (None, torch.as_tensor(b.dataset_id, dtype=torch.int32, device=rt.device)):
        want = rt.forward(m, g, "fp32", dataset_id=ds)
        got = torch.full_like(want, float("nan"))
        B.painn_forward_noalloc(rt.ctx, m.handle, g.handle, ds.data_ptr() if ds is not None else None,
                                B.PRECISIONS["fp32"], got.data_ptr())
        torch.cuda.synchronize()
        assert torch.equal(got, want)
    idx = [0, b.n_struct // 2, b.n_struct - 1]
    Er, Ar = batch_energies(b, hp, W, idx)
    check_energies(want.cpu().numpy()[idx], Er, Ar, TOL["fp32"], f"wide shared {atoms}")
    g.free()
    m.free()


def test_forces_wide_shared(rt):  # noqa: F811
    """dE/dY wider than the gradients whose space it takes (1,024 against
    7 F = 448 columns), dataset heads and blended, FP32."""
    print("forces, 1,024-wide shared layer", flush=True)
    hp, W, m = wide_shared(rt, 5)
    b = batch(301, hp.n_heads)
    g = rt.build_graph(rt.upload_batch(b), hp.cutoff)
    ds = torch.as_tensor(b.dataset_id, dtype=torch.int32, device=rt.device)
    idx = list(range(b.n_struct))
    E, F = rt.forces(m, g, "fp32", dataset_id=ds)
    assert torch.equal(E, rt.forward(m, g, "fp32", dataset_id=ds))
    ref = [structure_forces(*b.structure(k), hp, W)["F"] for k in idx]
    check_forces(F.cpu().numpy(), b, ref, idx, 2e-5, "wide shared, dataset heads")
    E, F = rt.forces_blend(m, g, "fp32", skip=0.0)
    assert torch.equal(E, rt.forward_blend(m, g, "fp32", skip=0.0))
    ref = [structure_forces_blend(*b.structure(k)[:4], hp, W, skip=0.0)["F"] for k in idx]
    check_forces(F.cpu().numpy(), b, ref, idx, 2e-5, "wide shared, blended")
    g.free()
    m.free()


def test_blended_forces_in_ranges(rt):  # noqa: F811
    """64 heads over a 1,024-wide shared layer: 6,000 atoms' dE_h/dY is 1.6 GB,
    more than a range is given."""
    print("blended forces in ranges, 64 heads, 1,024-wide shared layer", flush=True)
    hp, W, m = wide_shared(rt, 64)
    b = batch(6000, hp.n_heads)
    g = rt.build_graph(rt.upload_batch(b), hp.cutoff)
    E, F = rt.forces_blend(m, g, "fp32", skip=0.0)
    Eb = rt.forward_blend(m, g, "fp32", skip=0.0)
    assert torch.equal(E, Eb)
    assert torch.isfinite(F).all()
    n = b.n_struct
    idx = [0, n // 2 - 1, n // 2, n // 2 + 1, n - 1]
    ref = [structure_forces_blend(*b.structure(k)[:4], hp, W, skip=0.0) for k in idx]
    check_forces(F.cpu().numpy(), b, [o["F"] for o in ref], idx, 2e-5, "blended in ranges")
    # alone the same structure is one range
    one = b.subset([n // 2])
    g1 = rt.build_graph(rt.upload_batch(one), hp.cutoff)
    _, F1 = rt.forces_blend(m, g1, "fp32", skip=0.0)
    check_forces(F1.cpu().numpy(), one, [ref[2]["F"]], [0], 2e-5, "the same alone")
    g1.free()
    g.free()
    m.free()

"""Wide branch layers (tiles of 32 and 128 rows, csrc/branch.hip) vs the
oracle: energies, forces and blended forces of models whose hidden branch
layers are at least 256 wide, at the edges of the dispatch: one to three
hidden layers, widths that pad to 128- and 160-feature workgroups, with and
without shared layers, batches on both sides of 4,096 atoms, heads
without atoms and tiles with one row.  Tolerances as in the other forward and
forces tests (the FP32 products run over three exact bf16 planes per operand,
so their error is that of FP32 sums).  The entry point with fixed scratch runs
the same tiles in more chunks: bit for bit the same energies."""
import sys

import numpy as np
import pytest
import torch

import synth
from helpers import TOL, check_blend, check_energies, check_forces, stored_weights
from oracle.forces import structure_forces, structure_forces_blend
from oracle.painn import batch_energies, structure_forward_blend

pytestmark = pytest.mark.gpu

F_TOL = {"fp64": 1e-10, "fp32": 2e-5}
CONFIGS = {
    "one_hidden_no_shared": dict(shared_dims=[], branch_dims=[256, 1], n_heads=3),
    "one_hidden": dict(shared_dims=[50], branch_dims=[300, 1], n_heads=5),
    "lead": dict(shared_dims=[50, 50], branch_dims=[776, 776, 1], n_heads=16),
    "three_hidden": dict(shared_dims=[40], branch_dims=[288, 256, 320, 1], n_heads=4),
}


@pytest.fixture(scope="module")
def rt():
    from paper_2604_15380_amd import Runtime
    r = Runtime(0)
    yield r
    r.close()


def model(rt, name, K=6):
    hp = synth.HyperParams(F=64, K=K, L=1, n_species=6, cutoff=3.0, blend_dims=[32], **CONFIGS[name])
    W = synth.make_weights(hp, 77)
    return hp, W, rt.load_model(synth.weight_file_bytes(hp, W))


def batch(atoms, n_heads, skip_head=1):
    """Molecules of 3-40 atoms up to `atoms` in total; no structure on head
    `skip_head`, one single structure on head 0."""
    rng = np.random.default_rng(atoms)
    out, left = [], atoms
    while left > 0:
        n = min(left, int(rng.integers(3, 41)))
        left -= n
        grid = np.stack(np.meshgrid(*[np.arange(4)] * 3), -1).reshape(-1, 3)[:n] * 1.4
        pos = grid + rng.uniform(-0.2, 0.2, (n, 3))
        ds = 0 if not out else int(rng.choice([h for h in range(1, n_heads) if h != skip_head or n_heads == 2]))
        out.append((pos, rng.integers(0, 6, n), np.zeros((3, 3)), np.zeros(3), ds))
    return synth.concat(out)


@pytest.mark.parametrize("atoms", [1, 33, 129, 4095, 4099])
@pytest.mark.parametrize("name", list(CONFIGS))
@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16"])
def test_branch_tiles(rt, precision, name, atoms):
    print(f"branch {name} {precision} {atoms} atoms", flush=True)
    sys.stdout.flush()
    hp, W, m = model(rt, name)
    b = batch(atoms, hp.n_heads)
    g = rt.build_graph(rt.upload_batch(b), hp.cutoff)
    ds = torch.as_tensor(b.dataset_id, dtype=torch.int32, device=rt.device)
    idx = sorted({0, b.n_struct - 1} | set(np.random.default_rng(5).choice(b.n_struct, min(5, b.n_struct)).tolist()))
    Ws = stored_weights(W, precision)
    Er, Ar = batch_energies(b, hp, Ws, idx)
    label = f"{name} {precision} {atoms}"
    E = rt.forward(m, g, precision, dataset_id=ds).cpu().numpy()
    check_energies(E[idx], Er, Ar, TOL[precision], label)
    if precision == "bf16":
        # (blended BF16 energies also carry the router's BF16 rounding, which
        # tests/test_gpu_blend.py bounds on the workloads)
        g.free()
        m.free()
        return
    w = torch.empty((b.n_struct, hp.n_heads), dtype=torch.float64, device=rt.device)
    Eb = rt.forward_blend(m, g, precision, skip=0.02, weights=w).cpu().numpy()
    refs = [structure_forward_blend(*b.structure(k)[:4], hp, Ws, skip=0.02) for k in idx]
    check_blend(Eb, w.cpu().numpy(), refs, idx, 0.02, precision, label)
    E2, F = rt.forces(m, g, precision, dataset_id=ds)
    assert np.array_equal(E2.cpu().numpy(), E)
    ref = [structure_forces(*b.structure(k), hp, W)["F"] for k in idx]
    check_forces(F.cpu().numpy(), b, ref, idx, F_TOL[precision], label)
    E3, F3 = rt.forces_blend(m, g, precision, skip=0.0)
    ref = [structure_forces_blend(*b.structure(k)[:4], hp, W, skip=0.0)["F"] for k in idx]
    check_forces(F3.cpu().numpy(), b, ref, idx, F_TOL[precision], label + " blended")
    g.free()
    m.free()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_head_zero_and_chunks(rt, precision):
    """No dataset ids (head 0, tiles of consecutive atoms), and the fixed
    64 MiB scratch, whose chunks of tiles are smaller."""
    from paper_2604_15380_amd import binding as B
    print(f"branch chunks {precision}", flush=True)
    hp, W, m = model(rt, "three_hidden")
    b = batch(6000, hp.n_heads)
    g = rt.build_graph(rt.upload_batch(b), hp.cutoff)
    idx = [0, b.n_struct // 2, b.n_struct - 1]
    E = rt.forward(m, g, precision)
    b0 = b.subset(idx)
    b0.dataset_id[:] = 0
    Er, Ar = batch_energies(b0, hp, W)
    check_energies(E.cpu().numpy()[idx], Er, Ar, TOL[precision], f"head 0 {precision}")
    for ds in (None, torch.as_tensor(b.dataset_id, dtype=torch.int32, device=rt.device)):
        want = rt.forward(m, g, precision, dataset_id=ds)
        got = torch.full_like(want, float("nan"))
        B.painn_forward_noalloc(rt.ctx, m.handle, g.handle, ds.data_ptr() if ds is not None else None,
                                B.PRECISIONS[precision], got.data_ptr())
        torch.cuda.synchronize()
        assert torch.equal(got, want)
    g.free()
    m.free()

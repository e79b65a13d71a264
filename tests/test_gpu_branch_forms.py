"""Which tiles, and in BF16 which kernels, run wide branches (csrc/internal.h:
branch_small, branch_products): calls next to each line against the oracle, in
every precision, with dataset heads and blended.  Blended energies are compared
with the oracle's head energies under the GPU's own head weights, so that the
router's rounding (bounded in tests/test_gpu_blend.py) plays no part; the
tolerances are those of the energies."""
import numpy as np
import pytest
import torch

from helpers import TOL, check_energies, stored_weights
from oracle.painn import batch_energies, structure_forward_blend
from test_gpu_branch import batch, model, rt  # noqa: F401

pytestmark = pytest.mark.gpu


def some(b):
    return sorted({0, b.n_struct - 1} | set(np.random.default_rng(5).choice(b.n_struct, min(4, b.n_struct)).tolist()))


# rows = atoms: 128-row tiles from 8,192 rows on (FP64: 32,768), one kernel per
# tile of atoms from 4,096 on (BF16)
@pytest.mark.parametrize("precision,atoms", [("fp32", 8191), ("fp32", 8192), ("bf16", 4095), ("bf16", 4096),
                                             ("fp64", 8192), ("fp64", 32767), ("fp64", 32768)])
def test_dataset_heads(rt, precision, atoms):  # noqa: F811
    print(f"branch forms, dataset heads, {precision} {atoms} atoms", flush=True)
    hp, W, m = model(rt, "lead")
    b = batch(atoms, hp.n_heads)
    g = rt.build_graph(rt.upload_batch(b), hp.cutoff)
    ds = torch.as_tensor(b.dataset_id, dtype=torch.int32, device=rt.device)
    E = rt.forward(m, g, precision, dataset_id=ds).cpu().numpy()
    idx = some(b)
    Er, Ar = batch_energies(b, hp, stored_weights(W, precision), idx)
    check_energies(E[idx], Er, Ar, TOL[precision], f"{precision} {atoms}")
    assert np.all(np.isfinite(E))
    g.free()
    m.free()


# rows = atoms x heads, a quarter of the heads with a threshold; BF16: one
# kernel per tile below 16,384
@pytest.mark.parametrize("precision,atoms,skip", [
    ("fp32", 511, 0.0), ("fp32", 512, 0.0), ("fp32", 2047, 0.02), ("fp32", 2048, 0.02),
    ("fp64", 2047, 0.0), ("fp64", 2048, 0.0), ("bf16", 511, 0.0), ("bf16", 512, 0.0), ("bf16", 1023, 0.0),
    ("bf16", 1024, 0.0), ("bf16", 4095, 0.02), ("bf16", 4096, 0.02)])
def test_blended_heads(rt, precision, atoms, skip):  # noqa: F811
    print(f"branch forms, blended, {precision} {atoms} atoms, skip {skip}", flush=True)
    hp, W, m = model(rt, "lead")
    b = batch(atoms, hp.n_heads)
    g = rt.build_graph(rt.upload_batch(b), hp.cutoff)
    w = torch.empty((b.n_struct, hp.n_heads), dtype=torch.float64, device=rt.device)
    E = rt.forward_blend(m, g, precision, skip=skip, weights=w).cpu().numpy()
    w = w.cpu().numpy()
    kept = np.where(w >= (np.float32(skip) if precision != "fp64" else skip), w, 0.0)
    assert np.all(np.isfinite(E))
    idx = some(b)
    Ws = stored_weights(W, precision)
    Er, Ar = [], []
    for k in idx:
        o = structure_forward_blend(*b.structure(k)[:4], hp, Ws, skip=0.0)
        Er.append(float(kept[k] @ o["E_heads"]))
        Ar.append(float(np.abs(o["e"]).sum()))
    check_energies(E[idx], np.array(Er), np.array(Ar), TOL[precision], f"blended {precision} {atoms}")
    g.free()
    m.free()

"""The per-atom layers' forms by batch size, energies and forces against the
oracle on both sides of every line between them: one launch per dense layer
(small batches), the fused kernels, and in FP64 from F = 256 on the reverse
kernels in F-wide chunks; ragged 16-row tiles, and an atom without neighbours
(|V| = 0 in the first layer).  Tolerances as in the other forces and forward
tests."""
import sys

import numpy as np
import pytest

import synth
from helpers import TOL, assert_same_energies, check_energies, check_forces
from oracle.forces import structure_forces
from oracle.painn import batch_energies

pytestmark = pytest.mark.gpu

F_TOL = {"fp64": 1e-10, "fp32": 2e-5}


@pytest.fixture(scope="module")
def rt():
    from paper_2604_15380_amd import Runtime
    r = Runtime(0)
    yield r
    r.close()


def batch(atoms):
    """Structures of at most 33 atoms; the last atom of each is alone."""
    rng = np.random.default_rng(atoms)
    out, left = [], atoms
    while left > 0:
        n = min(33, left)
        left -= n
        grid = np.stack(np.meshgrid(*[np.arange(4)] * 3), -1).reshape(-1, 3)[:n] * 1.4
        pos = grid + rng.uniform(-0.2, 0.2, (n, 3))
        pos[-1] += 50.0                     # beyond every cutoff
        out.append((pos, rng.integers(0, 4, n), np.zeros((3, 3)), np.zeros(3), 0))
    return synth.concat(out)


CASES = [(p, F, n) for p, F in [("fp64", 128), ("fp64", 256), ("fp64", 337), ("fp32", 256), ("fp32", 337)]
         for n in (1, 16, 17, 240, 241, 384, 385)]
CASES += [("fp64", 64, 1152), ("fp64", 64, 1153), ("fp64", 128, 768), ("fp64", 128, 769), ("fp64", 256, 1153),
          ("fp32", 64, 768), ("fp32", 64, 769), ("fp32", 128, 1536), ("fp32", 128, 1537), ("fp32", 256, 1536)]


@pytest.mark.parametrize("precision,F,atoms", CASES)
def test_rows_and_tiles(rt, precision, F, atoms):
    print(f"rows and tiles {precision} F={F} atoms={atoms}", flush=True)
    sys.stdout.flush()
    hp = synth.HyperParams(F=F, K=5, L=2, n_species=4, n_heads=1, cutoff=3.0, branch_dims=[20, 1])
    W = synth.make_weights(hp, 31)
    b = batch(atoms)
    m = rt.load_model(synth.weight_file_bytes(hp, W))
    g = rt.build_graph(rt.upload_batch(b), hp.cutoff)
    E0 = rt.forward(m, g, precision).cpu().numpy()
    E, Fg = rt.forces(m, g, precision)
    assert_same_energies(E.cpu().numpy(), E0, precision)
    idx = sorted({0, b.n_struct // 2, b.n_struct - 1})
    Er, Ar = batch_energies(b, hp, W, idx)
    check_energies(E0[idx], Er, Ar, TOL[precision], f"{precision} F={F} {atoms}")
    ref = [structure_forces(*b.structure(k), hp, W)["F"] for k in idx]
    check_forces(Fg.cpu().numpy(), b, ref, idx, F_TOL[precision], f"{precision} F={F} {atoms}")
    g.free()
    m.free()

"""The training step's matrix tiles at their edges vs the training oracle:
widths one past a tile (65 = 64 + 1, 33 = 32 + 1), weight gradients cut into
row chunks (one head, more than 256 atoms) and grouped over heads (one head
without atoms, one with a single structure), energies and gradients checked
as in tests/test_gpu_train.py (loss 1e-12, gradient 1e-9 of each array's
largest)."""
import numpy as np
import pytest

import synth
from test_gpu_train import CFG, check_step, gpu_step, refs_for, rt, say  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_heads,n_mol", [(1, 15), (4, 15), (4, 1)])
def test_train_tile_edges(rt, n_heads, n_mol):  # noqa: F811
    from paper_2604_15380_amd import binding as B
    say(f"training tiles, {n_heads} heads, {n_mol} molecules")
    hp = synth.HyperParams(F=65, K=5, L=1, n_species=5, n_heads=n_heads, cutoff=2.5, shared_dims=[33],
                           branch_dims=[64, 65, 1])
    W = synth.make_weights(hp, 5100)
    rng = np.random.default_rng(n_heads + n_mol)
    structs = []
    for k in range(n_mol):
        n = 27 if k else 20
        grid = np.stack(np.meshgrid(*[np.arange(3)] * 3), -1).reshape(-1, 3)[:n] * 1.5
        head = 0 if n_heads == 1 else 3 if k == 0 else 1 + k % 2      # head 0 of several: no atoms
        structs.append((grid + rng.uniform(-0.2, 0.2, (n, 3)), rng.integers(0, 5, n), np.zeros((3, 3)),
                        np.zeros(3, np.uint8), head))
    b = synth.concat(structs)
    m = rt.load_model(synth.weight_file_bytes(hp, W))
    tr = B.painn_trainer_create(rt.ctx, m.handle, CFG)
    try:
        E_ref, F_ref = refs_for(b, 9)
        loss, th, gr = gpu_step(rt, tr, hp, b, E_ref, F_ref)
        check_step(f"{n_heads} heads, {b.n_atoms} atoms", hp, W, b, E_ref, F_ref, loss, th, gr, {})
    finally:
        B.painn_trainer_free(tr)
        m.free()

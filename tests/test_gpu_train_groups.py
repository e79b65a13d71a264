"""The training step's grouping of atoms by head and the grouped weight
gradients on batches of many structures and of many rows per head: against
the training oracle as in tests/test_gpu_train.py (loss 1e-12, gradient 1e-9
of each array's largest), and that a step's time grows with the batch no
faster than the batch, and with a second head hardly at all."""
import numpy as np
import pytest
import torch

import synth
from test_gpu_train import CFG, check_step, gpu_step, refs_for, rt, say  # noqa: F401

pytestmark = pytest.mark.gpu


def small_structures(n_heads, per_head, empty):
    """`per_head` structures of 1 or 3 atoms on every head but the last (of
    several) and `empty` without atoms, in random order.  per_head is odd: a
    bias gradient is a sum of +- atoms / structures, which an odd number of odd
    terms keeps from zero (a sum that cancels to exactly 0 in one order and to
    an ulp of its terms in another has no scale to compare with)."""
    assert per_head % 2
    rng = np.random.default_rng(per_head + empty)
    heads = np.repeat(np.arange(max(1, n_heads - 1)), per_head)
    atoms = np.concatenate([rng.choice([1, 3], len(heads)), np.zeros(empty, int)])
    heads = np.concatenate([heads, rng.integers(0, n_heads, empty)])
    out = []
    for k in rng.permutation(len(heads)):
        n = int(atoms[k])
        pos = np.arange(n)[:, None] * np.array([1.3, 0.0, 0.0]) + rng.uniform(-0.2, 0.2, (n, 3))
        out.append((pos, rng.integers(0, 4, n), np.zeros((3, 3)), np.zeros(3, np.uint8), int(heads[k])))
    return synth.concat(out)


def step(rt, hp, batch, label):  # noqa: F811
    from paper_2604_15380_amd import binding as B
    W = synth.make_weights(hp, 5200)
    m = rt.load_model(synth.weight_file_bytes(hp, W))
    tr = B.painn_trainer_create(rt.ctx, m.handle, CFG)
    try:
        E_ref, F_ref = refs_for(batch, 9)
        loss, th, gr = gpu_step(rt, tr, hp, batch, E_ref, F_ref)
        check_step(label, hp, W, batch, E_ref, F_ref, loss, th, gr, {})
    finally:
        B.painn_trainer_free(tr)
        m.free()


# the grouping takes 256 structures at a time: 255, 256, 257, 600 structures
@pytest.mark.parametrize("n_heads,per_head,empty", [(5, 63, 3), (1, 255, 1), (5, 63, 5), (64, 9, 33)])
def test_train_many_structures(rt, n_heads, per_head, empty):  # noqa: F811
    batch = small_structures(n_heads, per_head, empty)
    say(f"training grouping, {batch.n_struct} structures, {n_heads} heads")
    hp = synth.HyperParams(F=8, K=4, L=1, n_species=4, n_heads=n_heads, cutoff=2.5, shared_dims=[6],
                           branch_dims=[5, 1])
    step(rt, hp, batch, f"{batch.n_struct} structures, {n_heads} heads")


# grouped weight gradients cut each head's rows into chunks of whole 64s: the
# rows on one head, next to the edges of the chunks, and a head with one row
@pytest.mark.parametrize("n_mol,per", [(41, 25), (64, 16), (65, 16), (513, 2)])
def test_train_few_heads_many_rows(rt, n_mol, per):  # noqa: F811
    say(f"grouped weight gradients, {n_mol} molecules of {per} atoms on two heads")
    hp = synth.HyperParams(F=8, K=4, L=1, n_species=4, n_heads=2, cutoff=2.0, branch_dims=[33, 1])
    rng = np.random.default_rng(per)
    structs = []
    for k in range(n_mol):
        n = 1 if k == 3 else per
        grid = np.stack(np.meshgrid(*[np.arange(3)] * 3), -1).reshape(-1, 3)[:n] * 1.6
        structs.append((grid + rng.uniform(-0.2, 0.2, (n, 3)), rng.integers(0, 4, n), np.zeros((3, 3)),
                        np.zeros(3, np.uint8), 1 if k == 3 else 0))
    step(rt, hp, synth.concat(structs), f"{n_mol} x {per} atoms, two heads")


def step_ms(rt, n_struct, n_heads, atoms):  # noqa: F811
    from paper_2604_15380_amd import binding as B
    hp = synth.HyperParams(F=8, K=4, L=1, n_species=4, n_heads=n_heads, cutoff=2.0, branch_dims=[64, 1])
    m = rt.load_model(synth.weight_file_bytes(hp, synth.make_weights(hp, 5201)))
    tr = B.painn_trainer_create(rt.ctx, m.handle, CFG)
    rng = np.random.default_rng(n_struct)
    N = n_struct * atoms
    pos = np.zeros((N, 3))
    pos[:, 0] = np.tile(np.arange(atoms) * 1.5, n_struct)
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a)).to(rt.device)  # noqa: E731
    ds = t(rng.integers(0, n_heads, n_struct).astype(np.int32))
    inp = dict(n_struct=n_struct, n_atoms=N, any_pbc=False, cell=None, pbc=None, pos=t(pos), dataset_id=ds,
               struct_ptr=t((np.arange(n_struct + 1) * atoms).astype(np.int32)),
               species=t(rng.integers(0, 4, N).astype(np.int32)))
    er, fr = t(rng.standard_normal(n_struct)), t(rng.standard_normal((N, 3)))
    g = rt.build_graph(inp, hp.cutoff)
    loss = torch.zeros(3, dtype=torch.float64, device=rt.device)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    times = []
    try:
        for _ in range(6):
            a.record()
            B.painn_trainer_step(rt.ctx, tr, g.handle, ds.data_ptr(), er.data_ptr(), fr.data_ptr(), loss.data_ptr())
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
    finally:
        g.free()
        B.painn_trainer_free(tr)
        m.free()
    say(f"{n_struct} structures of {atoms} atoms, {n_heads} heads: {min(times[1:]):.3f} ms")
    return min(times[1:])


def test_train_step_time_linear_in_structures(rt):  # noqa: F811
    """Eight times the structures: at most about eight times the time (a count
    over every pair of structures took 40 times as long here)."""
    few, many = step_ms(rt, 2048, 4, 2), step_ms(rt, 16384, 4, 2)
    assert many <= 12 * few, (few, many)


def test_train_second_head_is_cheap(rt):  # noqa: F811
    """The same rows on two heads instead of one (with each head's rows in one
    workgroup per tile: 1.5 times as long)."""
    one, two = step_ms(rt, 20000, 1, 8), step_ms(rt, 20000, 2, 8)
    assert two <= 1.25 * one, (one, two)

"""FP64 forces with more than 35 radial functions against the oracle: the
reverse message kernel then runs 12 or 17 filter k-blocks with one feature
tile per wave, its filter fragments read from global memory and 16 rows in the
per-edge reduction (csrc/backward.hip); 35 is the largest basis of the other
form.  Two layers, so that both the first layer's kernel and the general one
run; clusters whose senders have 1, 14 to 18 and 33 edges (chunks of 16 with
every remainder at the edges) and atom counts that no sender block divides."""
import numpy as np
import pytest

import synth
from helpers import check_forces
from oracle.forces import structure_forces
from test_gpu_branch import rt  # noqa: F401

pytestmark = pytest.mark.gpu


def clusters(sizes, seed):
    """One molecule per size, all its atoms within the cutoff of each other (a
    sender has size - 1 edges)."""
    rng = np.random.default_rng(seed)
    out = []
    for n in sizes:
        grid = np.stack(np.meshgrid(*[np.arange(4)] * 3), -1).reshape(-1, 3)[:n] * 1.1
        out.append((grid + rng.uniform(-0.15, 0.15, (n, 3)), rng.integers(0, 4, n), np.zeros((3, 3)),
                    np.zeros(3, np.uint8), 0))
    return synth.concat(out)


@pytest.mark.parametrize("K", [35, 36, 40, 64])
@pytest.mark.parametrize("F", [64, 100, 256, 337])
def test_forces_wide_basis(rt, F, K):  # noqa: F811
    print(f"FP64 forces, F {F}, K {K}", flush=True)
    hp = synth.HyperParams(F=F, K=K, L=2, n_species=4, n_heads=1, cutoff=7.0, branch_dims=[16, 1])
    W = synth.make_weights(hp, 5300 + K)
    m = rt.load_model(synth.weight_file_bytes(hp, W))
    b = clusters([2, 1, 15, 16, 17, 18, 19, 34, 3], K)
    assert b.n_atoms % 4
    g = rt.build_graph(rt.upload_batch(b), hp.cutoff)
    assert g.n_edges == sum(n * (n - 1) for n in np.diff(b.struct_ptr))
    _, Fg = rt.forces(m, g, "fp64")
    idx = list(range(b.n_struct))
    ref = [structure_forces(*b.structure(k)[:4], 0, hp, W)["F"] for k in idx]
    check_forces(Fg.cpu().numpy(), b, ref, idx, 1e-10, f"F {F} K {K}")
    g.free()
    m.free()

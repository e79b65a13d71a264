"""The forward's workspace under HIP graph capture: a call whose batch fits what
an earlier call left there allocates nothing, also where the wide branches
would run best with more.  Every replay gives the eager energies, with other
batches run on the context in between."""
import pytest
import torch

import synth
from test_gpu_branch import batch, model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_capture_in_small_workspace(precision):
    from paper_2604_15380_amd import Runtime
    print(f"capture, blended wide branches, {precision}", flush=True)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        rt = Runtime(0)
        try:
            # a narrow model's batch leaves room for the wide model's need alone
            hp = synth.HyperParams(F=64, K=6, L=1, n_species=6, cutoff=3.0, n_heads=1, branch_dims=[32, 1])
            narrow = rt.load_model(synth.weight_file_bytes(hp, synth.make_weights(hp, 3)))
            gn = rt.build_graph(rt.upload_batch(batch(5000, 2)), hp.cutoff)
            rt.forward(narrow, gn, precision)
            hp, _, wide = model(rt, "lead")
            tiny = rt.build_graph(rt.upload_batch(batch(5, hp.n_heads)), hp.cutoff)
            rt.forward_blend(wide, tiny, precision)
            b = batch(3000, hp.n_heads)
            g = rt.build_graph(rt.upload_batch(b), hp.cutoff)
            E = torch.full((b.n_struct,), float("nan"), dtype=torch.float64, device=rt.device)
            side.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=side):
                rt.forward_blend(wide, g, precision, skip=0.0, out=E)
            got = []
            for _ in range(3):
                E.fill_(float("nan"))
                graph.replay()
                got.append(E.clone())
                rt.forward(narrow, gn, precision)
                side.synchronize()
            del graph
            want = rt.forward_blend(wide, g, precision, skip=0.0)     # may grow the workspace now
            assert torch.isfinite(want).all()
            for e in got:
                assert torch.equal(e, want)
            for x in (gn, tiny, g):
                x.free()
            narrow.free()
            wide.free()
        finally:
            rt.close()

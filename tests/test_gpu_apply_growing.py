"""An apply of a few columns between pushes: its workspaces are made once for the handle's
capacity, so a call with more pairs than the last one allocates nothing.  Shown by capturing it
(an allocation would end the capture with an error) and by replaying the graph three times with
eager work and a synchronization between, against the eager result, bit for bit."""
import pytest
import torch

from workloads import quadratic as wq
from tests.helpers import gpu_input, make_pairs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("cols", [1, 2, 4])
def test_capture_after_more_pushes(storage, cols):
    import paper_2009_12663_amd as P
    prob, S, Y, h0 = make_pairs("secant", 47, 43, 40, seed=cols, precond=True)
    stream = torch.cuda.Stream()
    print(f"\n[growing {storage}] n={prob.n} cols={cols}", flush=True)
    with torch.cuda.stream(stream):
        H = P.Bfgs(prob.n, 45, gpu_input(h0, storage), storage, stream=stream)
        V = H._block(gpu_input(wq.normal_block(prob.n, cols, seed=2), storage))
        out = torch.empty(V.shape, dtype=H.rdt, device="cuda")
        for i in range(40):
            H.push_pair(gpu_input(S[i], storage), gpu_input(Y[i], storage))
            if i in (1, 7):
                H.apply_Hinv(V, out)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream, capture_error_mode="global"):
            H.apply_Hinv(V, out)
        want = H.apply_Hinv(V)
        for _ in range(3):
            out.fill_(float("nan"))
            graph.replay()
            stream.synchronize()
            assert torch.equal(out, want)
            assert torch.equal(H.apply_Hinv(V), want)
        assert H.get_status() == 0
        H.close()

"""GPU tests of captured calls at the token counts from which on their groups are smaller than those of other calls."""
import pytest
import torch

from tests.test_gpu_eigen_routes import Call, _params, _reference, _rows, _tc

pytestmark = pytest.mark.gpu


# Up to 768 tokens the same groups and so the same bits; above, both are held to the reference (sigma: the float32 output and a few eps ||G||
# on its square; C: reflectors and vectors in float32, about sqrt(N) 2^-24 a row of U).
@pytest.mark.parametrize("n,batch", [(129, 2), (448, 3), (768, 1), (769, 1), (1000, 2), (1152, 1), (1499, 2), (1728, 1)])
def test_a_captured_call_gives_what_another_gives(n, batch):
    tc = _tc()
    O = _rows(batch, n, 512, 5 * n).cuda()
    eager = Call(tc, _params(tc, batch, n, 4), O)
    eager()
    torch.cuda.synchronize()
    want = eager.outputs()
    call = Call(tc, _params(tc, batch, n, 4), O.clone())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        call(stream=torch.cuda.current_stream().cuda_stream)
    reference = [_reference(o) for o in O.cpu()]
    for _ in range(3):
        call.C.zero_()
        graph.replay()
        torch.cuda.synchronize()
        got = call.outputs()
        eager()   # between the replays
        torch.cuda.synchronize()
        assert got[3].cpu().tolist() == [1] * batch
        if n <= 768:
            assert all(torch.equal(x, y) for x, y in zip(want, got))
        for out in (want, got):
            for b, (s, c) in enumerate(reference):
                assert float((out[2][b].double().cpu() - s).abs().max() / s.max()) < 1e-6
                assert float((out[1][b].double().cpu() - c).abs().max() / c.abs().max()) < 2e-5

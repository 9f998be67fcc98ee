"""GPU tests of the reduction by groups that hold whole columns, and of the last columns by one workgroup: token counts at the edges of
their frames (128, 320, 384, 448, 576, 768, 1152, 1536, 1920, 2112), images that need more than one round over the device."""
import pytest
import torch

from tests.test_gpu_eigen_routes import Call, _params, _reference, _rows, _tc

pytestmark = pytest.mark.gpu


# sigma: the float32 output and a few eps ||G|| on its square; C: reflectors and vectors are held in float32, a row of U is off by
# about sqrt(N) 2^-24 (3e-6 at 2113 tokens), and so is its weighted sum
@pytest.mark.parametrize("n,batch", [(15, 2), (16, 1), (127, 3), (128, 1), (129, 2), (144, 1), (145, 1), (200, 16), (320, 64),
                                     (321, 65), (384, 33), (385, 2), (448, 17), (449, 40), (560, 1), (768, 9), (769, 1), (1153, 4), (1536, 1), (1537, 2), (1921, 1), (2112, 1), (2113, 1)])
def test_singular_values_and_scores_at_the_edges_of_the_column_frames(n, batch):
    tc = _tc()
    O = _rows(batch, n, 512, 3 * n + batch)
    call = Call(tc, _params(tc, batch, n, 4), O.cuda())
    call()
    torch.cuda.synchronize()
    assert call.info.cpu().tolist() == [1] * batch
    for b in {0, batch - 1}:
        s, c = _reference(O[b])
        assert float((call.sigma[b].double().cpu() - s).abs().max() / s.max()) < 1e-6
        assert float((call.C[b].double().cpu() - c).abs().max() / c.abs().max()) < 2e-5, b


def test_small_calls_side_by_side_give_what_they_give_alone():
    # calls of one to three images take turns on the XCDs
    tc = _tc()
    shapes = [(576, 1), (300, 2), (576, 3), (576, 1), (400, 1), (768, 1), (576, 1), (200, 1)]
    calls = [Call(tc, _params(tc, b, n, 4), _rows(b, n, 512, i).cuda()) for i, (n, b) in enumerate(shapes)]
    alone = []
    for c in calls:
        c()
        torch.cuda.synchronize()
        alone.append(c.outputs())
    streams = [torch.cuda.Stream() for _ in calls]
    torch.cuda.synchronize()
    for _ in range(5):
        for c, s in zip(calls, streams):
            c(stream=s.cuda_stream)
    torch.cuda.synchronize()
    for c, want in zip(calls, alone):
        for x, y in zip(want, c.outputs()):
            assert torch.equal(x, y)

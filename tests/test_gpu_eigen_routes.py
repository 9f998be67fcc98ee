"""GPU tests of the contribution score on attention outputs in hand: the triangular frames of the reduction to tridiagonal form
(256, 576 and multiples of 576 tokens), the split contraction of the Gram matrix, captured graphs and concurrent calls."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu


def _tc():
    from paper_2503_10501_amd import binding as tc
    tc.load_library()
    assert torch.cuda.is_available()
    return tc


def _params(tc, batch, n, heads, head_dim=128, **kw):
    return tc.make_params(batch=batch, seq_len=n, vis_start=0, n_vis=n, n_heads=heads, head_dim=head_dim,
                          hidden_dim=heads * head_dim, dtype=tc.TC_BF16, k_prune=max(1, n // 2), k_final=max(1, n // 2), lam=1.0,
                          norm_mode=0, **kw)


def _rows(batch, n, d, seed):
    """bf16 rows whose singular values fall from 1 to about 1e-2."""
    g = torch.Generator().manual_seed(seed)
    o = torch.randn(batch, n, d, generator=g) * torch.logspace(0, -2, d)
    return o.to(torch.bfloat16)


class Call:
    """Outputs and workspace of a tc_ipgs_score call."""

    def __init__(self, tc, p, O):
        B, N = p.batch, p.n_vis
        self.tc, self.p, self.O, self.ws = tc, p, O, tc.new_workspace(p)
        self.S = torch.zeros(B, N, device="cuda")
        self.E, self.C, self.sigma = (torch.empty(B, N, device="cuda") for _ in range(3))
        self.info = torch.empty(B, dtype=torch.int32, device="cuda")

    def __call__(self, **kw):
        self.tc.tc_ipgs_score(self.p, self.O, self.S, self.E, self.C, self.sigma, self.info, self.ws, **kw)

    def outputs(self):
        return [x.clone() for x in (self.E, self.C, self.sigma, self.info)]


def _reference(O):
    """sigma (descending) and C of one image in float64."""
    u, s, _ = torch.linalg.svd(O.double(), full_matrices=False)
    return torch.nn.functional.pad(s, (0, O.shape[0] - s.numel())), u.abs() @ s


# (tokens, batch, heads of 128).  Edges of the frames (256, 576, 1152, 1728, 2304, 2880; above 3456 the Jacobi iteration), a group
# of eight images and a ragged one of four-workgroup groups; the Gram matrix of few tiles is contracted by 8 (257 x 1), 4
# (577 x 3 with eight chunks each, 100 x 9), 2 (256 x 33) and 1 (576 x 18) workgroups per tile.
@pytest.mark.parametrize("n,batch,heads", [(1, 1, 2), (2, 3, 2), (17, 1, 4), (100, 9, 16), (255, 2, 8), (256, 33, 4), (257, 1, 32),
                                           (575, 8, 8), (576, 18, 8), (577, 3, 16), (1152, 1, 16), (1153, 2, 16), (1728, 1, 16),
                                           (1729, 1, 16), (2305, 1, 8), (2881, 1, 8), (3457, 1, 4)])
def test_singular_values_and_scores_at_the_edges_of_the_frames(n, batch, heads):
    # sigma: the float32 output and a few eps ||G|| on its square; C: reflectors and vectors are held in float32, a row of U is off
    # by about sqrt(N) 2^-24, and so is its weighted sum (4e-6 at 3456 tokens; 1e-4 where the method iterates)
    tc = _tc()
    O = _rows(batch, n, heads * 128, 7 * n + batch)
    call = Call(tc, _params(tc, batch, n, heads), O.cuda())
    call()
    torch.cuda.synchronize()
    assert int(call.info.min()) > 0
    for b in {0, batch // 2, batch - 1}:
        s, c = _reference(O[b])
        assert float((call.sigma[b].double().cpu() - s).abs().max() / s.max()) < 1e-6
        assert float((call.C[b].double().cpu() - c).abs().max() / c.abs().max()) < (2e-5 if n <= 3456 else 1e-4), b


@pytest.mark.parametrize("n,batch", [(300, 2), (576, 1), (700, 2), (1800, 1)])
def test_a_captured_call_replays_to_the_eager_result(n, batch):
    # 1800 tokens: groups of 64 workgroups, which two replays at once could not be kept apart: a captured call iterates instead
    tc = _tc()
    O = _rows(batch, n, 512, n).cuda()
    eager = Call(tc, _params(tc, batch, n, 4, **({"eig_method": 1} if n > 1728 else {})), O)
    eager()
    torch.cuda.synchronize()
    want = eager.outputs()
    call = Call(tc, _params(tc, batch, n, 4), O.clone())
    st = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        call(stream=torch.cuda.current_stream().cuda_stream)
    for rep in range(3):
        call.O.copy_(O * (1 if rep != 1 else 2))
        graph.replay()
        torch.cuda.synchronize()
        got = call.outputs()
        if rep == 1:   # other inputs in the same buffers: twice the rows, twice the scores
            assert float((got[1] / 2 - want[1]).abs().max() / want[1].abs().max()) < 1e-5
        else:
            for x, y in zip(want, got):
                assert torch.equal(x, y)


def test_captured_calls_replay_on_two_streams_at_once():
    # groups of 32 and of 16, spread over the XCDs, that nothing keeps apart: 320 and 160 workgroups each.  An image whose group gave up
    # differs by rounding
    tc = _tc()
    calls, graphs, want = [], [], []
    for i in range(2):
        c = Call(tc, _params(tc, 10, 701, 4), _rows(10, 701, 512, i).cuda())
        c()
        torch.cuda.synchronize()
        want.append(c.outputs())
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
            c(stream=torch.cuda.current_stream().cuda_stream)
        calls.append(c)
        graphs.append(graph)
    streams = [torch.cuda.Stream() for _ in graphs]
    torch.cuda.synchronize()
    for _ in range(3):
        for graph, s in zip(graphs, streams):
            with torch.cuda.stream(s):
                graph.replay()
        torch.cuda.synchronize()
        for c, w in zip(calls, want):
            got = c.outputs()
            assert torch.equal(got[3], w[3])
            for x, y in zip(got[1:3], w[1:3]):   # (the score is zero: lambda is 1 and the attention scores are)
                assert float((x - y).abs().max() / y.abs().max()) < 2e-5


@pytest.mark.parametrize("n,rows", [(833, 832), (3457, 3456)])
def test_the_rank_of_some_rows_fits_the_workspace_of_all(n, rows):
    # the plan for the rows has more workgroups per Gram tile, or another eigensolver, than that for all tokens
    tc = _tc()
    p = _params(tc, 1, n, 8)
    O = _rows(1, n, 1024, n)
    rank = torch.empty(1, dtype=torch.int32, device="cuda")
    sigma = torch.empty(1, rows, device="cuda")
    tc.tc_info_rank(p, O.cuda(), rank, tc.new_workspace(p), rows=torch.arange(rows, dtype=torch.int32, device="cuda")[None].contiguous(),
                    rtol=1e-3, sigma=sigma)
    torch.cuda.synchronize()
    s = torch.linalg.svdvals(O[0, :rows].double())
    s = torch.nn.functional.pad(s, (0, rows - s.numel()))
    assert float((sigma[0].double().cpu() - s).abs().max() / s.max()) < 1e-6
    assert abs(int(rank) - int((s > 1e-3 * s.max()).sum())) <= 1   # a value at the threshold


# (calls, tokens, images): workgroups of the widest groups, all calls together: 480 of 160 (one image a call); 640 of 32, then 320 of 16; 180
# of 36 beside 512 and 160 of 128 and 160; 576 of 64 (the triangle); 704 of 16 beside 128 of 16 (the triangle)
@pytest.mark.parametrize("shapes", [[(1729, 1)] * 3, [(701, 10)] * 2, [(1400, 5), (1153, 4), (1729, 1)], [(2200, 3)] * 3,
                                    [(576, 22), (576, 22), (900, 8)]])
def test_calls_on_several_streams_at_once(shapes):
    tc = _tc()
    calls = [Call(tc, _params(tc, b, n, 4), _rows(b, n, 512, i).cuda()) for i, (n, b) in enumerate(shapes)]
    alone = []
    for c in calls:
        c()
        torch.cuda.synchronize()
        alone.append(c.outputs())
    streams = [torch.cuda.Stream() for _ in calls]
    torch.cuda.synchronize()
    for _ in range(3):
        for c, s in zip(calls, streams):
            c(stream=s.cuda_stream)
    torch.cuda.synchronize()
    for c, want in zip(calls, alone):
        for x, y in zip(want, c.outputs()):
            assert torch.equal(x, y)


@pytest.mark.parametrize("n,batch", [(200, 300), (600, 66)])
def test_groups_of_images_give_what_one_group_gives(n, batch):
    tc = _tc()
    O = _rows(batch, n, 256, n).cuda()
    out = []
    for groups in (1, 0, 3):
        call = Call(tc, _params(tc, batch, n, 2, stream_groups=groups), O)
        call()
        torch.cuda.synchronize()
        out.append(call.outputs())
    for other in out[1:]:
        for x, y in zip(out[0], other):
            assert torch.equal(x, y)


@pytest.mark.parametrize("n,batch,phase", [(257, 1, 0), (300, 9, 0), (576, 2, 0), (577, 2, 0), (577, 2, 1), (1000, 1, 1), (1153, 2, 0),
                                           (1153, 2, 1), (1729, 1, 2), (576, 64, 1), (576, 64, 3), (901, 8, 1), (1729, 3, 1)])
def test_images_whose_groups_are_not_resident_at_once(n, batch, phase):
    # the groups give up from this phase on: one workgroup per image does the rest.  (The last four: columns behind a triangle)
    tc = _tc()
    patience = ctypes.c_int.in_dll(tc.load_library(), "tc_group_patience")
    O = _rows(batch, n, 512, 7 * n)
    call = Call(tc, _params(tc, batch, n, 4), O.cuda())
    usual = patience.value
    patience.value = -1 - phase
    try:
        call()
        torch.cuda.synchronize()
    finally:
        patience.value = usual
    assert call.info.cpu().tolist() == [1] * batch
    for b in {0, batch - 1}:
        s, c = _reference(O[b])
        assert float((call.sigma[b].double().cpu() - s).abs().max() / s.max()) < 1e-6
        assert float((call.C[b].double().cpu() - c).abs().max() / c.abs().max()) < 2e-5, b


@pytest.mark.parametrize("n", [64, 257, 576, 577, 1153])
def test_an_all_zero_image_scores_zero(n):
    # the exchanged values are zeros too
    tc = _tc()
    O = _rows(3, n, 512, n)
    O[1] = 0
    call = Call(tc, _params(tc, 3, n, 4), O.cuda())
    call()
    torch.cuda.synchronize()
    assert call.info.cpu().tolist() == [1, 1, 1]
    assert not call.C[1].any() and not call.sigma[1].any()
    for b in (0, 2):
        s, c = _reference(O[b])
        assert float((call.C[b].double().cpu() - c).abs().max() / c.abs().max()) < 2e-5, b

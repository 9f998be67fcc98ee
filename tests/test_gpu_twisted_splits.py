"""GPU test of the eigenvectors where the tridiagonal matrix is split: rows in groups that share no columns, with group ends at, before
and behind the segments of sixteen rows of the walks, and groups of one row."""
import pytest
import torch

from tests.test_gpu_eigen_routes import _reference, _tc

pytestmark = pytest.mark.gpu


# reflectors and vectors are held in float32: a row of U is off by about sqrt(group) 2^-24, the weighted sum by as much
@pytest.mark.parametrize("sizes", [[16, 16, 16], [15, 1, 17, 16], [1] * 33, [31, 2, 64, 1, 1, 30], [100, 16, 12], [17, 300, 1, 200]])
def test_scores_of_rows_in_groups_that_share_no_columns(sizes):
    tc = _tc()
    n, wide = sum(sizes), [s + 8 for s in sizes]
    D = -(-sum(wide) // 64) * 64
    g = torch.Generator().manual_seed(n)
    O = torch.zeros(2, n, D)
    r = c = 0
    for s, w in zip(sizes, wide):
        O[:, r:r + s, c:c + w] = torch.randn(2, s, w, generator=g) * torch.logspace(0, -2, w)
        r, c = r + s, c + w
    p = tc.make_params(batch=2, seq_len=n, vis_start=0, n_vis=n, n_heads=D // 64, head_dim=64, hidden_dim=D, dtype=tc.TC_F32, k_prune=1,
                       k_final=1, lam=1.0, norm_mode=0)
    E, C, sigma = (torch.empty(2, n, device="cuda") for _ in range(3))
    info = torch.empty(2, dtype=torch.int32, device="cuda")
    tc.tc_ipgs_score(p, O.cuda(), torch.zeros(2, n, device="cuda"), E, C, sigma, info, tc.new_workspace(p))
    torch.cuda.synchronize()
    assert info.cpu().tolist() == [1, 1]
    for b in range(2):
        s, want = _reference(O[b])
        assert float((sigma[b].double().cpu() - s).abs().max() / s.max()) < 1e-6
        assert float((C[b].double().cpu() - want).abs().max() / want.max()) < max(sizes) ** 0.5 * 2.0 ** -22

"""GPU test of the eigenvectors where the tridiagonal matrix is split: rows in groups that share no columns, with group ends at, before
and behind the segments of sixteen rows of the walks, and groups of one row; vectors that the walks do not find, next to other groups."""
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


# Rows of length 1 whose neighbours have scalar products of a few eps: T is their Gram matrix, an even number of equal diagonals with couplings
# just above those that count as zero.  An eigenvalue then has no float64 but the diagonal itself, every row has a minor of zero before or behind
# it, no row is taken and the vector is made anew: it must stay inside its group.  The others are shorter rows at right angles to all.
@pytest.mark.parametrize("n", [2, 4, 6, 8, 30])
@pytest.mark.parametrize("coupling", [1.02, 1.5, 2.0, 2.6])
@pytest.mark.parametrize("before,behind", [(0, 20), (20, 0), (17, 40)])
def test_a_vector_that_is_made_anew_stays_inside_its_group(n, coupling, before, behind):
    tc = _tc()
    rows, D = before + n + behind, 128
    length = torch.ones(rows, dtype=torch.float64)
    length[:before] = torch.linspace(0.3, 0.8, before, dtype=torch.float64)
    length[before + n:] = torch.linspace(0.7, 0.2, behind, dtype=torch.float64)
    O = torch.diag(length).to(torch.float32)
    for i in range(before, before + n - 1):
        O[i + 1, i] = coupling * 2.0 ** -52
    O = torch.nn.functional.pad(O, (0, D - rows))[None]
    p = tc.make_params(batch=1, seq_len=rows, vis_start=0, n_vis=rows, n_heads=D // 64, head_dim=64, hidden_dim=D, dtype=tc.TC_F32, k_prune=1,
                       k_final=1, lam=1.0, norm_mode=0)
    E, C, sigma = (torch.empty(1, rows, device="cuda") for _ in range(3))
    info = torch.empty(1, dtype=torch.int32, device="cuda")
    tc.tc_ipgs_score(p, O.cuda(), torch.zeros(1, rows, device="cuda"), E, C, sigma, info, tc.new_workspace(p))
    torch.cuda.synchronize()
    assert info.tolist() == [1]
    assert float((sigma[0].double().cpu() - O[0].double().norm(dim=1).sort(descending=True).values).abs().max()) < 1e-6
    c = C[0].double().cpu()
    own = torch.ones(rows, dtype=torch.bool)
    own[before:before + n] = False
    assert bool(c.isfinite().all())
    assert float((c - length)[own].abs().max()) < 2.0 ** -22
    # any orthonormal vectors are right inside the group (to eps, its values are all 1): a row of an orthogonal matrix, absolute values
    # added, is between 1 and sqrt(n)
    assert float(c[~own].min()) > 1 - n ** 0.5 * 2.0 ** -22 and float(c[~own].max()) < n ** 0.5 * (1 + 2.0 ** -22)

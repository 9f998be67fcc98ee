"""GPU tests of the attention over float32 storage: query and key counts around its tiles of sixteen, both head sizes, odd strides of the
statistics, and values that are not finite behind the causal line."""
import math

import pytest
import torch

from tests.test_gpu_eigen_routes import _tc

pytestmark = pytest.mark.gpu


def _attention(tc, B, n, n_sys, n_prompt, heads, dh, causal, prompt_queries, Q, K, V):
    p = tc.make_params(batch=B, seq_len=n_sys + n + n_prompt, vis_start=n_sys, n_vis=n, n_heads=heads, head_dim=dh, hidden_dim=heads * dh,
                       dtype=tc.TC_F32, k_prune=n, k_final=n, causal=causal, n_prompt_queries=prompt_queries)
    O = torch.empty(B, n, heads * dh, device="cuda")
    S = torch.empty(B, n, device="cuda")
    tc.tc_attn_output(p, Q, K, V, O, S, tc.new_workspace(p))
    torch.cuda.synchronize()
    return O.double().cpu(), S.double().cpu()


def _reference(n, n_sys, causal, prompt_queries, Q, K, V):
    B, heads, L, dh = Q.shape
    q = Q.double()[:, :, n_sys:n_sys + n + prompt_queries]
    s = q @ K.double().transpose(2, 3) / math.sqrt(dh)
    if causal:
        s.masked_fill_(torch.arange(L)[None, :] > n_sys + torch.arange(q.shape[2])[:, None], -math.inf)
    A = s.softmax(3)
    O = torch.where(A[..., None] == 0, 0.0, A[..., None] * V.double()[:, :, None]).sum(3) if not V.isfinite().all() else A @ V.double()
    return O[:, :, :n].transpose(1, 2).reshape(B, n, heads * dh), A[:, :, :, n_sys:n_sys + n].mean(dim=(1, 2))


def _inputs(B, n, n_sys, n_prompt, heads, dh, seed):
    g = torch.Generator().manual_seed(seed)
    return [torch.randn(B, heads, n_sys + n + n_prompt, dh, generator=g) for _ in range(3)]


# A score is a sum of dh products with terms of up to about 4 (sums of dh numbers of size 1 over sqrt(dh)): its error is below
# dh 2^-24 * 4 at worst, the probability's relative error the same, and O and S are means of order 1 and 1 / L under it.
@pytest.mark.parametrize("B,n,n_sys,n_prompt,heads,dh,causal,prompt_queries", [
    (1, 1, 0, 0, 1, 64, 1, 0), (2, 15, 0, 0, 1, 128, 1, 0), (1, 16, 3, 1, 2, 64, 0, 0), (3, 17, 0, 5, 1, 64, 1, 5),
    (2, 33, 31, 0, 3, 128, 1, 0), (1, 64, 1, 30, 2, 128, 0, 30), (2, 301, 5, 2, 1, 64, 1, 2), (1, 129, 36, 28, 5, 64, 1, 1)])
def test_outputs_and_scores_around_the_tiles(B, n, n_sys, n_prompt, heads, dh, causal, prompt_queries):
    Q, K, V = _inputs(B, n, n_sys, n_prompt, heads, dh, 7 * n + dh)
    O, S = _attention(_tc(), B, n, n_sys, n_prompt, heads, dh, causal, prompt_queries, Q.cuda(), K.cuda(), V.cuda())
    o, s = _reference(n, n_sys, causal, prompt_queries, Q, K, V)
    tol = 4 * dh * 2.0 ** -24
    assert float((O - o).abs().max() / o.abs().max()) < tol
    assert float((S - s).abs().max() / s.abs().max()) < tol


@pytest.mark.parametrize("dh", [64, 128])
def test_what_is_not_finite_reaches_only_the_queries_that_have_the_key(dh):
    n, n_sys = 40, 3
    Q, K, V = _inputs(1, n, n_sys, 2, 2, dh, dh)
    V[0, 0, n_sys + 21, 5] = math.inf
    V[0, 0, n_sys + 25, dh - 1] = -math.inf
    V[0, 1, n_sys + 30, 9] = math.nan
    O, S = _attention(_tc(), 1, n, n_sys, 2, 2, dh, 1, 0, Q.cuda(), K.cuda(), V.cuda())
    o, s = _reference(n, n_sys, 1, 0, Q, K, V)
    assert torch.equal(O.isnan(), o.isnan()) and torch.equal(O.isinf(), o.isinf())
    assert torch.equal(O[O.isinf()], o[o.isinf()])
    fin = o.isfinite()
    assert float((O - o)[fin].abs().max() / o[fin].abs().max()) < 4 * dh * 2.0 ** -24
    assert float((S - s).abs().max() / s.abs().max()) < 4 * dh * 2.0 ** -24

"""GPU tests of the attention over float32 storage: query and key counts around its tiles of sixteen, both head sizes, odd strides of the
statistics, values that are not finite behind the causal line, and values near the ends of the float32 range."""
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


# An output is a mean of values, so it has their range: sums of the products before the division must not leave it.  (L 2^-24: a sum of L
# terms; below 2^-126 the storage has steps of 2^-149, of which every product and the result lose half, and their sum is within L halves.)
@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("n,causal", [(40, 1), (300, 0)])
@pytest.mark.parametrize("size", [3.0e38, 1.0e30, 1.0e-30, 1.0e-37])
def test_values_of_any_size(dh, n, causal, size):
    Q, K, V = _inputs(1, n, 3, 2, 2, dh, dh + n)
    L = n + 5
    V = ((0.75 + 0.25 * V.tanh()) * size).float()
    O, S = _attention(_tc(), 1, n, 3, 2, 2, dh, causal, 0, Q.cuda(), K.cuda(), V.cuda())
    o, s = _reference(n, 3, causal, 0, Q, K, V)
    assert bool(O.isfinite().all())
    assert float((O - o).abs().max()) < (4 * dh + L) * 2.0 ** -24 * size + L * 2.0 ** -149
    assert float((S - s).abs().max() / s.abs().max()) < 4 * dh * 2.0 ** -24


# One key that all queries have, at a score far below the others', with the only value that is not zero: the output is that value times a
# probability near the ends of what float32 holds.  (exp of a score of size m is off by m 2^-24 and what the score is off by, 4 m 2^-24; the
# probability has steps of 2^-149 below 2^-126.)
@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("n", [20, 400])
@pytest.mark.parametrize("below", [40, 80, 86, 90])
def test_a_small_probability_of_a_large_value(dh, n, below):
    L, key = n + 4, 2
    Q, K, V = torch.zeros(1, 1, L, dh), torch.zeros(1, 1, L, dh), torch.zeros(1, 1, L, dh)
    Q[..., 0] = math.sqrt(dh)
    K[0, 0, key, 0] = -below
    V[0, 0, key] = torch.linspace(-1e38, 1e38, dh)
    O, S = _attention(_tc(), 1, n, 3, 1, 1, dh, 0, 0, Q.cuda(), K.cuda(), V.cuda())
    o, s = _reference(n, 3, 0, 0, Q, K, V)
    assert float((O - o).abs().max()) < 5 * below * 2.0 ** -24 * float(o.abs().max()) + 2.0 ** -149 * 1e38

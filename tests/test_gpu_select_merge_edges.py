"""GPU tests of the selection and the merge at the edges of their tiles, against plain torch in float64."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _tc():
    from paper_2503_10501_amd import binding as tc
    tc.load_library()
    assert torch.cuda.is_available()
    return tc


def _params(tc, batch, n, kp, kf, head_dim, heads, dtype):
    return tc.make_params(batch=batch, seq_len=n, vis_start=0, n_vis=n, n_heads=heads, head_dim=head_dim,
                          hidden_dim=heads * head_dim, dtype=dtype, k_prune=kp, k_final=kf)


@pytest.mark.parametrize("n,batch", [(1, 1), (7, 2), (63, 1), (64, 3), (65, 1), (577, 2), (2880, 1), (4096, 2)])
def test_order_with_ties_infinities_and_nan(n, batch):
    tc = _tc()
    p = _params(tc, batch, n, n, n, 64, 1, tc.TC_BF16)
    e = torch.randn(batch, n, generator=torch.Generator().manual_seed(n))
    e[:, ::3] = (e[:, ::3] * 2).round() / 2          # many equal scores, zeros of both signs among them
    if n > 6:
        e[:, 1], e[:, 2], e[:, 4], e[:, 5] = float("inf"), -float("inf"), float("nan"), -0.0
    order = torch.empty(batch, n, dtype=torch.int32, device="cuda")
    tc.tc_select_topk(p, e.cuda(), order, tc.new_workspace(p))
    key = torch.where(e.isnan(), torch.full_like(e, -float("inf")), e)
    want = torch.sort(key, dim=1, descending=True, stable=True).indices
    assert torch.equal(order.cpu().long(), want)


# (k_prune, k_final, batch): one SetA row (2, 3), tiles of 32 in few and tiles of 64 in many workgroups with remainders on
# both sides (192 of the latter is where the rule turns), everything merged and nothing merged
@pytest.mark.parametrize("kp,kf,batch", [(1, 1, 1), (2, 1, 3), (3, 2, 1), (63, 40, 1), (64, 32, 2), (66, 40, 1), (131, 90, 5), (300, 200, 1),
                                         (129, 70, 64), (127, 127, 192), (127, 64, 191), (900, 500, 4)])
@pytest.mark.parametrize("dtype,head_dim,heads", [("bf16", 64, 1), ("bf16", 128, 9), ("f16", 64, 3), ("f32", 64, 1)])
def test_merge_at_the_edges_of_the_tiles(kp, kf, batch, dtype, head_dim, heads):
    tc = _tc()
    n, d = kp + 5, heads * head_dim
    p = _params(tc, batch, n, kp, kf, head_dim, heads, {"bf16": tc.TC_BF16, "f16": tc.TC_F16, "f32": tc.TC_F32}[dtype])
    sd = tc.storage_dtype(p)
    g = torch.Generator().manual_seed(kp * 7 + batch)
    Z = torch.randn(batch, n, d, generator=g).to(sd)
    order = torch.stack([torch.randperm(n, generator=g)[:kp] for _ in range(batch)])
    nA = kp // 2
    if nA > 40:   # rows of SetA that are the same, in one tile and in two: the lower index has to win
        Z[:, :][torch.arange(batch), order[:, 3]] = Z[torch.arange(batch), order[:, 1]]
        Z[:, :][torch.arange(batch), order[:, nA - 1]] = Z[torch.arange(batch), order[:, 1]]
    X = torch.randn(batch, n, d, generator=g).to(sd)
    X_out = torch.empty(batch, kf, d, dtype=sd, device="cuda")
    kept, dst = torch.empty(batch, kf, dtype=torch.int32, device="cuda"), torch.empty(batch, n, dtype=torch.int32, device="cuda")
    tc.tc_merge(p, X.cuda(), Z.cuda(), order.to(torch.int32).cuda(), X_out, kept, dst, tc.new_workspace(p))
    X_out, kept, dst = X_out.cpu(), kept.cpu().long(), dst.cpu().long()
    for b in sorted({0, batch // 2, batch - 1}):
        zn = torch.nn.functional.normalize(Z[b].double(), dim=1)
        A, Bs = order[b, :nA], order[b, nA:]
        merged = [int(x) for x in Bs if int(dst[b, x]) != int(x)]
        assert len(merged) == kp - kf
        assert all(int(dst[b, x]) == int(x) for x in A)
        assert int((dst[b] >= 0).sum()) == kp
        if nA:
            sim = zn[Bs] @ zn[A].T
            best = sim.max(dim=1).values
            # products of 16-bit values are exact, sums of up to 1152 of them carry less than 1e-5 in float32
            for j, x in enumerate(Bs.tolist()):
                if x in merged:
                    t = int(dst[b, x])
                    i = (A == t).nonzero()
                    assert i.numel() == 1 and float(sim[j, i]) >= float(best[j]) - 1e-5
                    same = A[(zn[A] == zn[t]).all(dim=1)]
                    assert t == int(same.min())
            if merged and len(merged) < len(Bs):
                is_m = torch.tensor([x in merged for x in Bs.tolist()])
                assert float(best[is_m].min()) >= float(best[~is_m].max()) - 1e-5
        rows = sorted(int(x) for x in order[b] if int(x) not in merged)
        assert kept[b].tolist() == rows
        groups = [[x] + [y for y in merged if int(dst[b, y]) == x] for x in rows]
        want = torch.stack([X[b, q].double().mean(dim=0) for q in groups])
        eps = {"bf16": 2.0 ** -8, "f16": 2.0 ** -11, "f32": 2.0 ** -22}[dtype]
        assert float(((X_out[b].double() - want).abs() / want.abs().clamp_min(0.05)).max()) <= 1.01 * eps + 2e-6 * len(merged)

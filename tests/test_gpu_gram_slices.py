"""The Gram matrix of 16-bit rows in whole numbers: tile edges, number of columns, scales, rows that are no whole numbers."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _batch(n, D):
    """So many images that the call takes this way: 128 tiles of 64, and 200 000 columns of theirs."""
    nt = (n + 63) // 64
    tiles = nt * (nt + 1) // 2
    return max(-(-128 // tiles), -(-200000 // (tiles * D)))


def _sigma(O, heads, head_dim, **kw):
    from paper_2503_10501_amd import binding as tc
    B, n, _ = O.shape
    p = tc.make_params(batch=B, seq_len=n, vis_start=0, n_vis=n, n_heads=heads, head_dim=head_dim, hidden_dim=heads * head_dim,
                       dtype=tc.TC_BF16 if O.dtype == torch.bfloat16 else tc.TC_F16, k_prune=1, k_final=1, **kw)
    rank = torch.empty(B, dtype=torch.int32, device="cuda")
    info = torch.empty(B, dtype=torch.int32, device="cuda")
    sigma = torch.empty(B, n, device="cuda")
    tc.tc_info_rank(p, O.cuda().contiguous(), rank, tc.new_workspace(p), sigma=sigma, info=info)
    torch.cuda.synchronize()
    return sigma.double().cpu(), info.cpu()


def _rows(B, n, D, dtype, seed):
    """Every row twice: half of the singular values are zero, so that an error of 2^-31 in the products shows as 1e-5."""
    g = torch.Generator().manual_seed(seed)
    half = torch.randn(B, (n + 1) // 2, D, generator=g).to(dtype)
    return torch.cat([half, half], 1)[:, :n].clone()


def _check(O, sigma):
    n = O.shape[0]
    s = torch.linalg.svdvals(O.double())
    s = torch.nn.functional.pad(s, (0, max(0, n - s.numel())))[:n]
    # an eigenvalue of the float64 matrix is off by a few n roundings of the largest at most; its root by the root of that
    assert float((sigma - s).abs().max() / s.max()) < (16 * n * 2.0 ** -53) ** 0.5 + 2.0 ** -22


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("n,heads,head_dim", [(65, 1, 64), (96, 3, 64), (128, 1, 128), (191, 2, 128), (300, 33, 128), (70, 65, 128),
                                              (70, 128, 128)])
def test_sizes(dtype, n, heads, head_dim):
    B = _batch(n, heads * head_dim)
    O = _rows(B, n, heads * head_dim, dtype, n)
    sigma, _ = _sigma(O, heads, head_dim)
    for b in {0, B // 2, B - 1}:
        _check(O[b], sigma[b])


@pytest.mark.parametrize("power", [-60, 0, 55])
def test_scales_and_the_largest_numbers(power):
    # rows of one magnitude: every digit at its largest; and rows of very different scales, one of them zero
    O = torch.full((_batch(96, 256), 96, 256), 1.9921875 * 2.0 ** power)
    g = torch.Generator().manual_seed(1)
    O *= torch.randint(0, 2, O.shape, generator=g) * 2 - 1
    O[1] *= 2.0 ** torch.randint(-6, 1, (96, 1), generator=g)
    O[1, 5] = 0
    O = O.to(torch.bfloat16)
    sigma, _ = _sigma(O, 2, 128)
    for b in range(2):
        _check(O[b], sigma[b])


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("bad", [1, 8, 9, 130])   # 130 rows: up to eight one by one, above the image as a whole
@pytest.mark.parametrize("left", [1, 8, 9])       # values of such a row: up to eight added apart, above the row formed again
@pytest.mark.parametrize("eig", [0, 1])           # matrix in float64, in float32
def test_rows_that_are_not_whole_numbers(dtype, bad, left, eig):
    from paper_2503_10501_amd import binding as tc
    O = _rows(_batch(130, 256), 130, 256, dtype, bad)
    tiny = 2.0 ** -100 if dtype == torch.bfloat16 else 2.0 ** -24   # the smallest half; the row's largest is 2^14
    O[1, 130 - bad:] *= 1 if dtype == torch.bfloat16 else 4096
    for k in range(left):
        O[1, 130 - bad:, (17 + 31 * k) % 256] = tiny
    sigma, _ = _sigma(O, 2, 128, eig_dtype=(tc.TC_EIG_F64, tc.TC_EIG_F32)[eig])
    for b in range(3):
        if eig == 0:
            _check(O[b], sigma[b])
        else:   # the float32 iteration: its own accuracy, on the eigenvalues
            s = torch.linalg.svdvals(O[b].double())
            assert float((sigma[b] ** 2 - s ** 2).abs().max() / s.max() ** 2) < 1e-4


def _gram_ms(V, **kw):
    """Time of the Gram matrix of rows V in one image after another: keys of length far above their products make O = V."""
    from paper_2503_10501_amd import binding as tc
    B, n, D = V.shape
    g = torch.Generator(device="cuda").manual_seed(0)
    K = torch.randn(B, D // 128, n, 128, device="cuda", generator=g).bfloat16()
    p = tc.make_params(batch=B, seq_len=n, vis_start=0, n_vis=n, n_heads=D // 128, head_dim=128, hidden_dim=D, dtype=tc.TC_BF16,
                       k_prune=8, k_final=8, jacobi_max_sweeps=1, **kw)
    Vh = V.view(B, n, D // 128, 128).transpose(1, 2).contiguous()
    X_out = torch.empty(B, 8, D, dtype=V.dtype, device="cuda")
    kept, dst = torch.empty(B, 8, dtype=torch.int32, device="cuda"), torch.empty(B, n, dtype=torch.int32, device="cuda")
    info, ws = torch.empty(B, dtype=torch.int32, device="cuda"), tc.new_workspace(p)
    return lambda: tc.tc_profile_compress(p, 8 * K, K, Vh, V, X_out, kept, dst, info, ws)[0]["gram"][0]


@pytest.mark.parametrize("left", [0, 1, 4, 8, 12])   # per row; above eight the row is formed anew
def test_rows_of_many_scales_cost_little_more_than_float64(left):
    # The same rows through the float64 products alone (a float32 matrix takes no digits).  An image that leaves much is found before
    # its products are begun, so a call pays for reading its rows once; with the products, and the values
    # added one by one, it was 1.2 (four values) to 2.1 (eight).
    from paper_2503_10501_amd import binding as tc
    g = torch.Generator(device="cuda").manual_seed(left)
    V = torch.randn(32, 576, 4096, device="cuda", generator=g)
    V.scatter_(2, torch.randint(0, 4096, (32, 576, left), device="cuda", generator=g), 2.0 ** -100)
    V = V.bfloat16()
    digits, plain = _gram_ms(V), _gram_ms(V, eig_dtype=tc.TC_EIG_F32)
    t = torch.tensor([[f() for f in (digits, plain)] for _ in range(12)])
    assert float(t[:, 0].min() / t[:, 1].min()) < (0.75 if left == 0 else 1.2)


def test_a_float32_matrix_is_rounded_once():
    # A call of one image forms all products in one sum of float64, and so does a call of many: the same float32 matrix, the same
    # iteration, the same bits.  (Added to digits that were float32 already, six small values of a row would round a second time.)
    from paper_2503_10501_amd import binding as tc
    g = torch.Generator().manual_seed(3)
    O = torch.randn(_batch(130, 256), 130, 256, generator=g) * 4096
    O[:, :, 0] = 20000
    small = (1 + (2 * torch.randint(0, 512, (O.shape[0], 65, 6), generator=g) + 1) / 1024) * 2.0 ** -7   # odd, a quarter of the unit
    O[:, :65].scatter_(2, torch.rand(O.shape[0], 65, 255, generator=g).argsort(2)[:, :, :6] + 1, small)
    O = O.to(torch.float16)
    many, _ = _sigma(O, 2, 128, eig_dtype=tc.TC_EIG_F32)
    for b in (0, 1, O.shape[0] - 1):
        one, _ = _sigma(O[b:b + 1], 2, 128, eig_dtype=tc.TC_EIG_F32)
        assert torch.equal(many[b], one[0])


def test_a_row_with_an_infinity_leaves_the_other_images_alone():
    O = _rows(_batch(130, 256), 130, 256, torch.bfloat16, 5)
    want, _ = _sigma(O, 2, 128)
    O[1, 7, 3] = float("inf")
    sigma, _ = _sigma(O, 2, 128)
    assert torch.equal(sigma[0], want[0]) and torch.equal(sigma[2], want[2])

"""The Gram matrix of 16-bit rows in whole numbers, entry by entry against an exact product: tile edges, number of columns, scales, rows
that are no whole numbers; turns, stream groups, overlapping and captured calls."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _tc():
    from paper_2503_10501_amd import binding as tc
    tc.load_library()
    return tc


def _params(O, heads, head_dim, **kw):
    tc = _tc()
    B, n, _ = O.shape
    return tc.make_params(batch=B, seq_len=n, vis_start=0, n_vis=n, n_heads=heads, head_dim=head_dim, hidden_dim=heads * head_dim,
                          dtype={torch.bfloat16: tc.TC_BF16, torch.float16: tc.TC_F16}[O.dtype], k_prune=1, k_final=1, **kw)


def _digits(p):
    """Whether a call takes the digits."""
    yes = ctypes.c_int(-1)
    assert _tc().load_library().tc_gram_matrix(ctypes.byref(p), None, None, None, ctypes.c_size_t(0), None, ctypes.byref(yes)) == 0
    return yes.value == 1


def _batch(n, D):
    """So many images that the call takes this way: 128 tiles of 64, and 200 000 columns of theirs."""
    nt = (n + 63) // 64
    tiles = nt * (nt + 1) // 2
    return max(-(-128 // tiles), -(-200000 // (tiles * D)))


def _gram(O, heads, head_dim, **kw):
    """G of the call, on the GPU."""
    tc = _tc()
    p = _params(O, heads, head_dim, **kw)
    assert _digits(p)
    Np = (p.n_vis + 63) // 64 * 64
    G = torch.full((p.batch, Np, Np), float("nan"), dtype=torch.float64, device="cuda")
    ws, yes, O = tc.new_workspace(p), ctypes.c_int(), O.cuda().contiguous()
    ws.fill_(0x5a)
    assert tc.load_library().tc_gram_matrix(ctypes.byref(p), ctypes.c_void_p(O.data_ptr()), ctypes.c_void_p(G.data_ptr()),
                                            ctypes.c_void_p(ws.data_ptr()), ctypes.c_size_t(ws.numel()),
                                            ctypes.c_void_p(torch.cuda.current_stream().cuda_stream), ctypes.byref(yes)) == 0
    torch.cuda.synchronize()
    return G


def _sigma(O, heads, head_dim, **kw):
    tc = _tc()
    p = _params(O, heads, head_dim, **kw)
    B, n, _ = O.shape
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


def _slice(x):
    """The rule of the digits for rows x (float64): exponent of each row's scale, the whole numbers, what is left."""
    big = np.abs(x).max(1)
    mant, ex = np.frexp(big)
    s = np.where(big == 0, 0, np.where(np.floor(np.ldexp(mant, 31)) > 0x7f7f7f7f, 30, 31) - ex)
    v = np.ldexp(x, s[:, None])
    left = (np.trunc(v) != v) | ((np.trunc(v) == 0) & (x != 0))
    return s, np.where(left, 0.0, v), left


def _over(left):
    """Whether an image is left to the float64 kernel."""
    n, D = left.shape
    per_row = left.sum(1)
    return per_row[per_row <= 8].sum() + (per_row > 8).sum() * D / 128 > max(n * (D - 768) / 1280, n / 8)


def _check_gram(O, G, over=None):
    """An image's G against the exact products.  The digits' sums are whole numbers rounded once to float64, what is left is added with
    a second rounding: an entry is within one unit of its last place, 2^-52 of it, and the rounding of the part added.  Entries of
    rows formed anew, and images with much left, are float64 sums of D products: D 2^-53 of the sum of their magnitudes."""
    x = O.double().numpy()
    n, D = x.shape
    s, m, left = _slice(x)
    hi = np.floor(m / 65536)
    lo = m - hi * 65536
    cross = hi @ lo.T   # (each sum below 2^53: exact)
    digits = (hi @ hi.T).astype(np.longdouble) * 2.0 ** 32 + (cross + cross.T).astype(np.longdouble) * 65536 + lo @ lo.T
    e = np.where(left, np.ldexp(x, s[:, None]), 0.0)
    mixed = e @ m.T
    add = (mixed + mixed.T + e @ e.T).astype(np.longdouble)
    scale = -(s[:, None] + s[None, :])
    want = digits + add
    got = np.ldexp(G[:n, :n].cpu().numpy().astype(np.longdouble), -scale)
    assert torch.equal(G, G.T)
    assert not G[n:].any()
    size = np.abs(np.ldexp(x, s[:, None]))
    loose = D * 2.0 ** -53 * (size @ size.T)
    tight = 2.0 ** -53 * (np.abs(digits) + np.abs(want)) + 20 * 2.0 ** -53 * (np.abs(e) @ size.T + size @ np.abs(e).T)
    anew = left.sum(1) > 8
    bound = np.where(anew[:, None] | anew[None, :], loose, tight)
    error = np.abs(got - want)
    if _over(left):
        assert (error <= loose).all()
    else:
        assert (error <= bound).all()
        for r in np.flatnonzero((left.sum(1) > 0) & ~anew):   # a row's values that were not added, or wrongly, would show
            assert (np.abs(add[r]) > 4 * bound[r]).any()
    if over is not None:
        assert _over(left) == over


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("n,heads,head_dim", [(65, 1, 64), (96, 3, 64), (128, 1, 128), (191, 2, 128), (300, 33, 128), (70, 65, 128),
                                              (70, 128, 128)])
def test_sizes(dtype, n, heads, head_dim):
    B = _batch(n, heads * head_dim)
    O = _rows(B, n, heads * head_dim, dtype, n)
    sigma, _ = _sigma(O, heads, head_dim)
    G = _gram(O, heads, head_dim)
    for b in {0, B // 2, B - 1}:
        _check(O[b], sigma[b])
        _check_gram(O[b], G[b])


@pytest.mark.parametrize("power", [-124, -60, 0, 55, 115])   # (-124: some values are subnormal)
def test_scales_and_the_largest_numbers(power):
    # rows of one magnitude: every digit at its largest; and rows of very different scales, one of them zero
    O = torch.full((_batch(96, 256), 96, 256), 1.9921875 * 2.0 ** power)
    g = torch.Generator().manual_seed(1)
    O *= torch.randint(0, 2, O.shape, generator=g) * 2 - 1
    O[1] *= 2.0 ** torch.randint(-6, 1, (96, 1), generator=g)
    O[1, 5] = 0
    O = O.to(torch.bfloat16)
    sigma, _ = _sigma(O, 2, 128)
    G = _gram(O, 2, 128)
    for b in range(2):
        _check(O[b], sigma[b])
        _check_gram(O[b], G[b])


def test_digit_sums_at_their_largest():
    # bf16 numbers whose digits are -128 (the carry makes the one above odd), over as many columns as the digits are used for
    bits = torch.tensor([0x80, 0x8080, 0x808000, 0x80800000 >> 1, 0x7f0000, -0x80, -0x8000, -0x7f800000 >> 1], dtype=torch.float64)
    g = torch.Generator().manual_seed(0)
    O = bits[torch.randint(0, 8, (_batch(65, 16384), 65, 16384), generator=g)].to(torch.bfloat16)
    O[:, :, 0] = 2.0 ** 30
    O[:, 1] = O[:, 0]
    G = _gram(O, 128, 128)
    _check_gram(O[0], G[0])


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("bad", [1, 8, 9, 130])   # with the values below, the rows' work is on both sides of the line for an image
@pytest.mark.parametrize("left", [1, 8, 9])       # values of such a row: up to eight added apart, above the row formed anew
@pytest.mark.parametrize("eig", [0, 1])           # matrix in float64, in float32
def test_rows_that_are_not_whole_numbers(dtype, bad, left, eig):
    tc = _tc()   # (sigma; what these values are in G is seen in the next test)
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


def _plant(O, row, cols):
    """Values just below the last bit of the row's scale in the columns `cols` (bf16: the largest is in [1, 2); half: in [2^14, 2^15))."""
    g = torch.Generator().manual_seed(row * 1000 + len(cols))
    bits, top = (7, 2.0 ** -24) if O.dtype == torch.bfloat16 else (10, 2.0 ** -7)
    odd = 2 * torch.randint(0, 1 << (bits - 1), (len(cols),), generator=g) + 1
    sign = torch.randint(0, 2, (len(cols),), generator=g) * 2 - 1
    O[row, cols] = (sign * (1 + odd / 2.0 ** bits) * top).to(O.dtype)


# per image: rows with values left (how many values each, 0: one to eight at random; which columns), rows with nine or more, and
# whether the float64 kernel takes the image.  130 rows of 4096: the line is at 338 values, a row formed anew counts 32
MIXES = [((0, 0, "own"), 0, False), ((1, 1, "own"), 0, False), ((20, 0, "own"), 0, False), ((20, 8, "same"), 0, False),
         ((30, 5, "near"), 0, False), ((129, 2, "own"), 0, False), ((130, 2, "near"), 0, False), ((0, 0, "own"), 1, False),
         ((0, 0, "own"), 2, False), ((0, 0, "own"), 5, False), ((0, 0, "own"), 10, False), ((18, 1, "own"), 10, False),
         ((19, 1, "own"), 10, True), ((25, 6, "near"), 3, False), ((42, 8, "own"), 0, False), ((113, 3, "own"), 0, True),
         ((0, 0, "own"), 11, True), ((0, 0, "own"), 130, True), ((130, 8, "own"), 0, True), ((120, 0, "near"), 9, True)]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_what_the_digits_leave_out(dtype):
    n, D = 130, 4096
    g = torch.Generator().manual_seed(11)
    O = torch.randn(max(_batch(n, D), len(MIXES)), n, D, generator=g).clamp(-1.9, 1.9)
    O += O.sign() * 0.02
    O = (O * (1 if dtype == torch.bfloat16 else 16000)).to(dtype)
    for b, ((few, values, which), anew, _) in enumerate(MIXES):
        rows = torch.randperm(n, generator=g)
        for i in range(few + anew):
            k = int(torch.randint(9, 400, (1,), generator=g)) if i >= few else values or int(torch.randint(1, 9, (1,), generator=g))
            if i == few:
                k = 9   # the fewest
            pool = D if which == "own" or i >= few else k if which == "same" else 24   # "near": lists that overlap in part
            _plant(O[b], int(rows[i]), torch.randperm(pool, generator=g)[:k])
    G = _gram(O, 32, 128)
    for b, mix in enumerate(MIXES):
        _check_gram(O[b], G[b], over=mix[2])


def _gram_ms(V, **kw):
    """Time of the Gram matrix of rows V in one image after another: keys of length far above their products make O = V."""
    tc = _tc()
    B, n, D = V.shape
    g = torch.Generator(device="cuda").manual_seed(0)
    K = torch.randn(B, D // 128, n, 128, device="cuda", generator=g).bfloat16()
    p = tc.make_params(batch=B, seq_len=n, vis_start=0, n_vis=n, n_heads=D // 128, head_dim=128, hidden_dim=D, dtype=tc.TC_BF16,
                       k_prune=8, k_final=8, jacobi_max_sweeps=1, **kw)
    assert _digits(p) == (not kw)
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
    tc = _tc()
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
    tc = _tc()
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


def test_rows_with_infinities_and_nan():
    # they are formed in float64, which says what a product of float64 says; the other images do not notice
    O = _rows(_batch(130, 4096), 130, 4096, torch.bfloat16, 5)
    inf = float("inf")
    want, plain = _sigma(O, 32, 128)[0], _gram(O, 32, 128)
    O[1, 7, 3] = inf
    O[2, 7, 3], O[2, 90, 3], O[2, 91, 5] = inf, -inf, 0
    O[3, 129] = float("nan")
    O[4, :, 9] = inf      # every row: the float64 kernel
    O[4, 6, 9] = 0
    sigma, info = _sigma(O, 32, 128)
    G = _gram(O, 32, 128)
    for b in range(O.shape[0]):
        if 1 <= b <= 4:
            x = O[b].double().numpy()
            with np.errstate(invalid="ignore"):
                ref = np.stack([(x[i] * x).sum(1) for i in range(130)])
            got = G[b, :130, :130].cpu().numpy()
            fine = np.isfinite(ref)
            assert np.array_equal(fine, np.isfinite(got)) and np.array_equal(np.isnan(ref), np.isnan(got))
            assert np.array_equal(ref[np.isinf(ref)], got[np.isinf(got)])
            size = np.where(np.isfinite(x), np.abs(x), 0.0)
            assert (np.abs(got[fine] - ref[fine]) <= (2 * 4096 * 2.0 ** -53 * (size @ size.T))[fine]).all()
            one, one_info = _sigma(O[b:b + 1], 32, 128)
            assert torch.equal(torch.isnan(sigma[b]), torch.isnan(one[0])) and int(info[b]) == int(one_info[0])
        else:
            assert torch.equal(sigma[b], want[b]) and torch.equal(G[b], plain[b])


def test_images_in_turns():
    # digits for more than 1 GiB: 60 images of 576 x 8192 in two turns, against calls of half of them
    g = torch.Generator(device="cuda").manual_seed(2)
    O = torch.randn(60, 576, 8192, device="cuda", generator=g).bfloat16()
    O[:, 5, 100] = (1 + 2.0 ** -7) * 2.0 ** -23    # (one value that is added, and rows formed anew)
    O[::7, 9, :50] = 2.0 ** -60
    G = _gram(O, 64, 128)
    for first in (0, 30):
        assert torch.equal(G[first:first + 30], _gram(O[first:first + 30], 64, 128))
    _check_gram(O[35].cpu(), G[35])


class _Score:
    """A tc_ipgs_score call on 12 images of 576 x 512, some values left."""

    def __init__(self, seed, **kw):
        tc, B, n, D = _tc(), 12, 576, 512
        g = torch.Generator().manual_seed(seed)
        self.O = torch.randn(B, n, D, generator=g).bfloat16()
        self.O[:, ::100, 7 + seed] = 2.0 ** -60
        self.p = _params(self.O, 4, 128, lam=1.0, norm_mode=0, **kw)
        assert _digits(self.p)
        self.O, self.ws, self.S = self.O.cuda(), tc.new_workspace(self.p), torch.zeros(B, n, device="cuda")
        self.out = [torch.empty(B, n, device="cuda") for _ in range(3)] + [torch.empty(B, dtype=torch.int32, device="cuda")]

    def __call__(self, **kw):
        _tc().tc_ipgs_score(self.p, self.O, self.S, *self.out, self.ws, **kw)

    def result(self):
        torch.cuda.synchronize()
        return [x.clone() for x in self.out]


@pytest.mark.parametrize("method", [0, 1])   # automatic (the reduction), the iteration
def test_stream_groups_and_overlapping_calls(method):
    alone = []
    for seed in (0, 1):
        call = _Score(seed, eig_method=method, stream_groups=1)
        call()
        alone.append(call.result())
    calls = [_Score(i % 2, eig_method=method, stream_groups=g) for i, g in enumerate((2, 3, 4, 0))]
    for call in calls:   # the groups' digits share one place
        call()
    for i, call in enumerate(calls):
        assert all(torch.equal(x, y) for x, y in zip(call.result(), alone[i % 2]))
    streams = [torch.cuda.Stream() for _ in calls]
    torch.cuda.synchronize()
    for _ in range(3):
        for call, st in zip(calls, streams):
            call(stream=st.cuda_stream)
    for i, call in enumerate(calls):
        assert all(torch.equal(x, y) for x, y in zip(call.result(), alone[i % 2]))


@pytest.mark.parametrize("groups", [1, 3])
def test_a_captured_call(groups):
    call = _Score(3, stream_groups=groups)
    call()
    want, O = call.result(), call.O.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        call(stream=torch.cuda.current_stream().cuda_stream)
    for rep in range(3):
        call.O.copy_(O if rep != 1 else O.flip(0))   # other images in the same buffers
        call.ws.fill_(0x5a)
        for x in call.out:
            x.fill_(0)
        graph.replay()
        for x, y in zip(call.result(), want):
            assert torch.equal(x, y if rep != 1 else y.flip(0))

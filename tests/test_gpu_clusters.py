"""GPU tests of the contribution score where singular values repeat, or nearly so: Eq. 3-6 is then not unique, but the
vectors of a repeated value are still an orthonormal basis of its subspace."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _circulant(p, m, seed):
    """First row of a p x p circulant matrix of integers below 2^24 (p prime) and the sizes of its discrete Fourier transform.
    The row is constant on the cosets of the group of order m (even, so that it holds -1) of the multiplicative group of
    residues and sums to zero: all singular values but a zero come m times, with harmonics for vectors."""
    rng = np.random.default_rng(seed)
    g = next(g for g in range(2, p) if len({pow(g, k, p) for k in range(p - 1)}) == p - 1)
    n = (p - 1) // m
    while True:   # until the largest value is apart from the next
        half = rng.integers(-2 ** 23, 2 ** 23, n // 2)
        values = rng.permutation(np.concatenate([half, -half, np.zeros(n % 2, dtype=np.int64)]))
        row = np.zeros(p, dtype=np.int64)
        for k in range(p - 1):
            row[pow(g, k, p)] = values[k % n]
        size = np.abs(np.fft.fft(row))
        top = np.sort(size)[::-1]
        if top[m] < 0.99 * top[0]:
            return row, size


def _basis_behind(c, P, rng):
    """The matrix M, least squares over many starts, with c = sum_i |(P M)_i| (c: the terms of Eq. 3-6 of one subspace over
    its singular value, P: an orthonormal basis of it), and the largest deviation.  For given signs the right side is linear in M."""
    m = P.shape[1]
    best = (np.inf, None)
    for _ in range(400):
        M = np.linalg.qr(rng.standard_normal((m, m)))[0]
        sign = None
        for _ in range(60):
            new = np.sign(P @ M)
            if sign is not None and np.array_equal(new, sign):
                break
            sign = new
            A = (sign[:, :, None] * P[:, None, :]).reshape(len(c), m * m)
            M = np.linalg.lstsq(A, c, rcond=None)[0].reshape(m, m).T
        dev = np.abs(np.abs(P @ M).sum(1) - c).max()
        if dev < best[0]:
            best = (dev, M)
        if dev < 1e-5 * np.abs(c).max():
            break
    return best


# Values that come 2, 4 or 6 times, equal to the last bit (bumps = 0) or, with some entries of the matrix off by one, parted by
# 1e-10 ... 1e-12 of their square (which moves their subspace by less than 1e-8).  sv_rtol keeps the largest value only.
# Vectors and reflectors are held in float32: a row of U is off by about sqrt(N) 2^-24.  Vectors whose eigenvalues lie just over 1e-10
# of the norm apart are orthogonal to eps / 1e-10 = 2.2e-6 without help.
@pytest.mark.parametrize("p,m,bumps,seed", [(61, 4, 0, 1), (577, 2, 0, 1), (577, 4, 0, 1), (577, 4, 1, 1), (577, 4, 4, 232),
                                            (577, 6, 1, 1), (1153, 4, 0, 1), (1153, 4, 4, 122), (1153, 4, 4, 344), (1753, 4, 0, 1),
                                            (1753, 4, 8, 55), (3169, 4, 1, 1), (3169, 4, 8, 206)])
def test_vectors_of_close_singular_values_are_orthonormal(p, m, bumps, seed):
    from paper_2503_10501_amd import binding as tc
    D, batch = (p + 63) // 64 * 64, 2
    shift = (np.arange(p)[None, :] - np.arange(p)[:, None]) % p
    O = torch.zeros(batch, p, D)
    sizes = []
    for b in range(batch):
        rng = np.random.default_rng(seed + b)
        row, size = _circulant(p, m, seed + b)
        full = row[shift]
        for _ in range(bumps):
            full[rng.integers(p), rng.integers(p)] += 1
        O[b, :, :p] = torch.from_numpy(full)   # exact in float32
        sizes.append(size)
    par = tc.make_params(batch=batch, seq_len=p, vis_start=0, n_vis=p, n_heads=D // 64, head_dim=64, hidden_dim=D, dtype=tc.TC_F32,
                         k_prune=2, k_final=2, lam=0.0, norm_mode=0, sv_rtol=0.995)
    E, C, sigma = (torch.empty(batch, p, device="cuda") for _ in range(3))
    info = torch.empty(batch, dtype=torch.int32, device="cuda")
    tc.tc_ipgs_score(par, O.cuda(), None, E, C, sigma, info, tc.new_workspace(par))
    torch.cuda.synchronize()
    found = []
    for b in range(batch):
        want = np.sort(sizes[b])[::-1]
        assert np.abs(sigma[b].double().cpu().numpy() - want).max() < 1e-6 * want[0]
        freq = [k for k in range(1, (p + 1) // 2) if sizes[b][k] > 0.995 * want[0]]
        x = 2 * np.pi * np.outer(np.arange(p), freq) / p
        P = np.concatenate([np.cos(x), np.sin(x)], 1) * np.sqrt(2.0 / p)
        assert P.shape[1] == m
        c = C[b].double().cpu().numpy() / want[0]
        dev, M = _basis_behind(c, P, rng)
        found.append((float(dev / np.abs(c).max()), float(np.abs(M.T @ M - np.eye(m)).max())))
    print("deviation, M^T M - I:", found)
    assert info.cpu().tolist() == [1] * batch
    for dev, off in found:
        assert dev < 8 * (np.sqrt(p) * 2.0 ** -24 + 5e-7)
        assert off < 2 * 2.2e-6 + np.sqrt(p) * 2.0 ** -24

"""Numpy replicas of kernels' algebra and index arithmetic, against dense float64
references: the DST of rows of 2^m - 1 by the odd extension's FFT, the DST as two
products, the general matrices' two recurrences over chunks, and the tile
layouts of the line solves."""
import numpy as np
import pytest

EPS = 2.0 ** -52


def sine(n):
    j = np.arange(1, n + 1)
    return np.sqrt(2.0 / (n + 1)) * np.sin(np.pi * (np.outer(j, j) % (2 * (n + 1))) / (n + 1))


@pytest.mark.parametrize("N", [32, 64, 128, 512, 1024])
def test_odd_extension(N):
    n, M, rng = N - 1, N // 4, np.random.default_rng(N)
    a, b = rng.standard_normal((2, n))
    x = np.zeros(N + 1, complex)
    x[1:N] = a + 1j * b
    w = np.full((5, M), np.nan + 0j)
    for j in list(range(M // 2)) + [M // 2]:
        z = np.array([x[j + r * M] for r in range(4)] + [-x[N - j - r * M] for r in range(4)])
        X = np.fft.fft(z)
        for p in range(5):
            t = np.exp(-1j * np.pi * j * p / N)
            w[p, j] = X[p] * t
            if 0 < j < M // 2:
                w[p, M - j] = -X[(8 - p) % 8] * np.conj(t)
    assert np.isfinite(w).all()     # every entry is written
    Z = np.fft.fft(w, axis=1)
    out = np.empty(n, complex)
    for i in range(n):
        p, q = (i + 1) & 7, (i + 1) >> 3
        out[i] = -Z[8 - p, M - 1 - q] if p > 4 else Z[p, q]
    out *= 0.5 * np.sqrt(2.0 / N)
    S = sine(n)
    tol = EPS * (np.sqrt(n) + 4 * np.log2(2 * N)) * max(np.linalg.norm(a), np.linalg.norm(b))
    assert np.abs(-out.imag - S @ a).max() < tol and np.abs(out.real - S @ b).max() < tol
    # pairs per block, threads and butterflies of the launch
    C = 512 // M
    T = (5 * C * M // 8 + 63) // 64 * 64
    assert C * M // 2 + C <= T <= 320 and 5 * C * M // 8 <= T


@pytest.mark.parametrize("n", [16, 17, 32, 33, 100, 161, 256, 300, 439, 440])
def test_product(n):
    rng = np.random.default_rng(n)
    x, N = rng.standard_normal(n), n + 1
    kv = (n + 1) // 2
    ki, ko = (kv + 7) // 8 * 8, (kv + 15) // 16 * 16
    u, v = np.zeros(ki), np.zeros(ki)
    for j in range(1, ki + 1):
        if 2 * j < N:
            v[j - 1], u[j - 1] = x[j - 1] + x[N - j - 1], x[j - 1] - x[N - j - 1]
        elif 2 * j == N:
            v[j - 1] = x[j - 1]
    q = np.sin(np.pi * np.arange(2 * N) / N) * np.sqrt(2.0 / N)
    out = np.full(2 * ko, np.nan)
    for m in range(1, ko + 1):
        for part, k in ((v, 2 * m - 1), (u, 2 * m)):
            row = [q[j * k % (2 * N)] if k <= n and (2 * j <= N if part is v else 2 * j < N) else 0.0
                   for j in range(1, ki + 1)]
            out[k - 1] = np.dot(row, part)
    assert np.abs(out[:n] - sine(n) @ x).max() < EPS * n * np.linalg.norm(x)
    # the stride: 2 x odd, so that 16 rows' pairs of inputs fall on distinct banks
    stride = ki + 2
    assert stride % 4 == 2 and len({2 * r * stride % 64 for r in range(16)}) == 16
    tiles = ko // 16
    rounds = -(-tiles // 10)
    waves = max(-(-tiles // rounds), 8)
    assert waves <= 10 and waves * rounds >= tiles and 4 * waves >= 32
    assert 64 * stride * 8 <= 160 * 1024 and -(-ki // 64) <= 4


def chunk_solve(a, b, c, d, P, MR=8):
    """x of the tridiagonal system by the two recurrences: chunks of MR rows from
    a zero start with the product of their multipliers, then the chunk maps."""
    n = len(b)
    rows = P * MR
    A, B, C, D = (np.zeros(rows, complex) for _ in range(4))
    A[:n], B[:n], C[:n], D[:n] = a, b, c, d
    A[0] = 0
    C[n - 1] = 0
    B[n:] = 1.0
    piv = np.empty(rows, complex)
    for i in range(rows):
        piv[i] = B[i] - (A[i] * C[i - 1] / piv[i - 1] if i else 0.0)
    v, f, u = (np.empty(rows, complex) for _ in range(3))
    for t in range(P):
        z, p = 0.0, 1.0
        for i in range(t * MR, t * MR + MR):
            nl = -A[i] / piv[i - 1] if i else 0.0
            z, p = D[i] + nl * z, nl * p
            v[i], f[i], u[i] = z / piv[i], p / piv[i], -C[i] / piv[i]
    V = 0.0
    for t in range(P):
        s = slice(t * MR, t * MR + MR)
        last = t * MR + MR - 1
        nxt = (v[last] + f[last] * V) * piv[last]
        v[s] = v[s] + f[s] * V
        V = nxt
    x, W = np.empty(rows, complex), 0.0
    for t in range(P - 1, -1, -1):
        for i in range(t * MR + MR - 1, t * MR - 1, -1):
            W = v[i] + u[i] * W
            x[i] = W
    return x[:n], piv[:n]


@pytest.mark.parametrize("n,P", [(257, 64), (511, 64), (512, 64), (513, 128), (1000, 128)])
def test_general_recurrences(n, P):
    rng = np.random.default_rng(n)
    h = np.diff(np.linspace(0, 1, n + 2) ** 1.5) * rng.uniform(0.7, 1.3, n + 1)
    lam, tau = 0.3 + 0.9j, 0.02
    a = lam * h[:-1] / 6 - tau / h[:-1]
    c = lam * h[1:] / 6 - tau / h[1:]
    b = lam * (h[:-1] + h[1:]) / 3 + tau * (1 / h[:-1] + 1 / h[1:])
    d = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    x, piv = chunk_solve(a, b, c, d, P)
    r = b * x - d
    r[1:] += a[1:] * x[:-1]
    r[:-1] += c[:-1] * x[1:]
    scale = np.abs(b) * np.abs(x)
    scale[1:] += np.abs(a[1:]) * np.abs(x[:-1])
    scale[:-1] += np.abs(c[:-1]) * np.abs(x[1:])
    assert np.abs(r).max() < 24 * 8 * EPS * scale.max()
    assert (np.abs(piv) >= np.abs(b) / 16).all()     # the rule that admits the form


@pytest.mark.parametrize("n", list(range(2, 513, 7)) + [64, 65, 113, 127, 128, 255, 256, 511, 512])
def test_line_tiles(n):
    """Every row of every line has its own entry inside the tile, and the
    threads' shares cover it."""
    MR = 4 if n <= 64 else 8
    P = 1
    while P * MR < n:
        P *= 2
    S = 1
    while P * S * 2 <= 512:
        S *= 2
    while S > n:
        S //= 2
    entry = lambda i: i + (i >> 3)
    e = entry(n - 1)
    stride = (e + 16) // 16 * 16 + 16 // S if S < 16 else (e + 1) | 1
    assert P <= 64 and e < stride
    idx = np.array([[g * stride + entry(i) for i in range(n)] for g in range(S)])
    assert len(np.unique(idx)) == S * n and idx.max() < S * stride
    assert 2 * S * stride >= S * n                   # the sums' staging, as doubles
    assert P * MR >= n                               # rows y0 + u P, u < MR
    if MR == 8:
        assert P % 8 == 0
        y = np.arange(P)[:, None] + P * np.arange(MR)
        assert (entry(y) == entry(np.arange(P))[:, None] + np.arange(MR) * (P + P // 8)).all()
    entries = 9 + MR
    assert S * entries <= P * S * (2 if MR == 8 else entries)
    assert S * (stride + entries) * 16 <= 160 * 1024

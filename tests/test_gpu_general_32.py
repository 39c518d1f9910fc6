"""The fp64 kernels for 32-bit words where they are still the ones that run: moduli above
the matrix-core kernels' limit, here 16515073 = 63 * 2^18 + 1 (lengths up to 2^18), and
batches of 2^15 and 2^16 that fill the chip.  The launch counts tell that they ran.  Exact
results: the oracle's sums on sampled entries and bins, closed forms for constants, and
equality between the forms."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import host

pytestmark = pytest.mark.gpu

M, M_MATRIX = 16515073, 13631489
MATRIX = ("matrix_short", "matrix_one", "matrix_three", "matrix_transform")


@pytest.fixture(scope="module")
def nt():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_1005_1497_amd as nt
    return nt


class ran:
    """The block's launches were of this class (or of several), none on the matrix cores."""

    def __init__(self, nt, **want):
        self.nt, self.want = nt, want

    def __enter__(self):
        self.before = self.nt.launch_counts()

    def __exit__(self, *e):
        if e[0] is None:
            after = self.nt.launch_counts()
            d = {k: after[k] - self.before[k] for k in after}
            assert all(d[k] == v for k, v in self.want.items()) and not any(d[k] for k in MATRIX), d


def words(seed, *shape):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return torch.randint(-(1 << 31), 1 << 31, shape, generator=gen, dtype=torch.int64, device="cuda").to(torch.int32)


def reduced(x, m):
    return ((x.to(torch.int64) & 0xFFFFFFFF) % m).to(torch.int32)


def batch(nt, f, g, logs, offs, m=M, flags=0, out=None):
    order = nt.max_log2n(m)
    return nt.conv_batched(f, g, nt.BatchDesc(logs, offs), m, root=nt.euler_root(m, order), root_log2order=order,
                           flags=nt.FLAG_EULER | flags, out=out)


def rows(nt, f, g, m=M, flags=0):
    count, N = f.shape
    return batch(nt, f.view(-1), g.view(-1), np.full(count, N.bit_length() - 1), np.arange(count, dtype=np.int64) * N,
                 m, flags).view(f.shape)


def check(h, f, g, m, items, seed=3):
    N, rng = f.shape[1], np.random.default_rng(seed)
    for i in items:
        idx = np.concatenate([[0, 1, N // 2, N - 1], rng.integers(0, N, 12)]).astype(np.uint64)
        ref = oracle.conv_entries(host(f[i]) % np.uint32(m), host(g[i]) % np.uint32(m), m, idx)
        assert np.array_equal(host(h[i])[idx.astype(np.int64)], ref.astype(np.uint32)), i
    s = [(t.to(torch.int64) & 0xFFFFFFFF).sum(1) % m for t in (f, g, h)]
    assert torch.equal(s[2], s[0] * s[1] % m)
    assert int(h.max()) < m and int(h.min()) >= 0


# few items in the four-step form with workgroups of 512 and its row loops; enough for the
# persistent kernel
@pytest.mark.parametrize("n,few,many", [(13, 150, 700), (14, 100, 530), (15, 100, 350), (16, 100, 350), (17, 100, 180),
                                        (18, 96, 180)])
def test_batches(nt, n, few, many):
    for count, kind in ((few, "fourstep"), (many, "fused")):
        f, g = words(n + count, count, 1 << n), words(2 * n + count, count, 1 << n)
        with ran(nt, **{kind: 1}):
            h = rows(nt, f, g)
        check(h, f, g, M, (0, count // 2, count - 1))
        with ran(nt, fourstep=count):                  # each by itself: workgroups of 256
            assert torch.equal(h, rows(nt, f, g, flags=nt.FLAG_PER_ITEM))
        for a, b in ((M - 1, M - 1), (0xFFFFFFFF, 0x80000000), ((M - 1) // 2, (M + 1) // 2)):
            F, G = (torch.full(f.shape, c - (c >> 31 << 32), dtype=torch.int32, device="cuda") for c in (a, b))
            assert bool((rows(nt, F, G) == (1 << n) * a * b % M).all()), (hex(a), hex(b))


@pytest.mark.parametrize("n", range(4, 19))
def test_single(nt, n):
    N = 1 << n
    f, g = words(n, 1, N), words(n + 100, 1, N)
    with ran(nt, **{"small" if n <= 12 else "fourstep": 1}):
        h = nt.conv_circular(f[0], g[0], M, flags=nt.FLAG_EULER)
    check(h[None], f, g, M, (0,))
    out = torch.full_like(h, -1)
    with ran(nt, **{"small" if n <= 12 else "fourstep": 1}):
        nt.conv_circular_noalloc(f[0], g[0], M, nt.euler_root(M, n), out, flags=nt.FLAG_EULER)
    assert torch.equal(out, h)
    # tones at the highest bin: alternating signs
    t = torch.where(torch.arange(N, device="cuda") % 2 == 0, 1, M - 1).to(torch.int32)
    want = torch.where(torch.arange(N, device="cuda") % 2 == 0, N, M - N).to(torch.int32)
    assert torch.equal(nt.conv_circular(t, t, M, flags=nt.FLAG_EULER), want)


@pytest.mark.parametrize("n", range(4, 19))
def test_transforms(nt, n):
    N, w = 1 << n, nt.euler_root(M, n)
    kw = dict(flags=nt.FLAG_EULER)
    for count in (1, 3, 64):
        x = words(10 * n + count, count, N)
        with ran(nt, transform=2):
            X, Y = nt.ntt_forward(x, M, w, **kw), nt.ntt_inverse(x, M, w, **kw)
        canon = reduced(x, M)
        with ran(nt, transform=2):
            assert torch.equal(nt.ntt_inverse(X, M, w, **kw), canon)
            assert torch.equal(nt.ntt_forward(Y, M, w, **kw), canon)
        some = sorted({0, count // 2, count - 1})
        bins = np.concatenate([np.tile(np.array([0, 1, N // 2, N - 1], np.uint64), (len(some), 1)),
                               np.random.default_rng(n).integers(0, N, (len(some), 12)).astype(np.uint64)], axis=1)
        at, xs = bins.astype(np.int64), np.stack([host(canon[r]) for r in some])
        got = np.take_along_axis(np.stack([host(X[r]) for r in some]), at, axis=1)
        assert np.array_equal(got, oracle.ntt_bins_rows(xs, M, w, bins).astype(np.uint32))
        inv = oracle.ntt_bins_rows(xs, M, pow(w, M - 2, M), bins).astype(np.uint64)
        got = np.take_along_axis(np.stack([host(Y[r]) for r in some]), at, axis=1)
        assert np.array_equal(got, (inv * np.uint64(pow(N, M - 2, M)) % np.uint64(M)).astype(np.uint32))


@pytest.mark.parametrize("lo,hi,count", [(4, 18, 60), (13, 18, 300), (8, 15, 900)])
def test_uneven(nt, lo, hi, count):
    """Several lengths, scattered: the single launch against one launch per length and
    one per item, and nothing between the items."""
    rng = np.random.default_rng(lo + hi + count)
    logs = rng.integers(lo, hi + 1, count)
    sizes = (1 << logs) + 16
    offs = np.concatenate([[0], np.cumsum(sizes)[:-1]]).astype(np.int64)
    f, g = words(1, int(sizes.sum())), words(2, int(sizes.sum()))
    outs = []
    for flags, want in ((0, {"multi": 1}), (nt.FLAG_PER_CLASS, {"multi": 0}), (nt.FLAG_PER_ITEM, {"multi": 0})):
        out = torch.full_like(f, -7)
        with ran(nt, **want):
            batch(nt, f, g, logs, offs, flags=flags, out=out)
        outs.append(out)
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    o = host(outs[0]).view(np.int32)
    for n, at in zip(logs, offs):
        assert np.all(o[at + (1 << n):at + (1 << n) + 16] == -7)
    for i in rng.integers(0, count, 6):
        a, N = int(offs[i]), 1 << int(logs[i])
        check(outs[0][None, a:a + N], f[None, a:a + N], g[None, a:a + N], M, (0,))


def quotients(nt, n, count, m, kind):
    N, w = 1 << n, nt.euler_root(m, n)
    kw = dict(flags=nt.FLAG_EULER)
    F = reduced(words(3 * n + count, count, N), m - 1) + 1
    F[0] = m - 1
    g = reduced(words(4 * n + count, count, N), m)
    f = nt.ntt_inverse(F, m, w, **kw)
    h = nt.ntt_inverse((nt.ntt_forward(g, m, w, **kw).to(torch.int64) * F % m).to(torch.int32), m, w, **kw)
    with ran(nt, **{kind: 1}):
        assert torch.equal(nt.deconvolve(f, h, m, w, **kw), g)
    F[count - 1, N - 1] = 0
    f = nt.ntt_inverse(F, m, w, **kw)
    with ran(nt, **{kind: 1}), pytest.raises(nt.NttError) as e:
        nt.deconvolve(f, h, m, w, **kw)
    assert e.value.name == "NTT_E_SINGULAR"


@pytest.mark.parametrize("n", [5, 9, 12, 13, 14, 15, 16, 17, 18])
def test_quotients(nt, n):
    for count in (1, 2, max(3, 5000 >> n)):
        quotients(nt, n, count, M, "small" if n <= 12 else "fused")


@pytest.mark.parametrize("n,count", [(15, 513), (15, 700), (16, 257), (16, 400), (17, 200)])
def test_quotients_that_fill_the_chip(nt, n, count):
    """The persistent quotient kernel, which the matrix-core modulus takes as well with
    every compute unit busy and more than 2^24 elements."""
    quotients(nt, n, count, M_MATRIX, "fused")


@pytest.mark.parametrize("n,count", [(15, 1100), (16, 350)])
def test_batches_that_fill_the_chip(nt, n, count):
    """The persistent kernel at the matrix-core modulus against the items one by one,
    which run on the matrix cores."""
    f, g = words(n, count, 1 << n), words(n + 50, count, 1 << n)
    with ran(nt, fused=1):
        h = rows(nt, f, g, M_MATRIX)
    assert torch.equal(h, rows(nt, f, g, M_MATRIX, nt.FLAG_PER_ITEM))
    check(h, f, g, M_MATRIX, (0, count // 2, count - 1))


def test_two_dimensions(nt):
    R, C = 64, 256
    f, g = words(5, R, C), words(6, R, C)
    with ran(nt, transform=3, small=1):
        h = host(nt.conv2d(f, g, M, flags=nt.FLAG_EULER)).astype(object)
    a, b = (host(reduced(t, M)).astype(object) for t in (f, g))
    for i, j in ((0, 0), (1, 255), (63, 17), (40, 200)):
        want = sum(a[k, l] * b[(i - k) % R, (j - l) % C] for k in range(R) for l in range(C)) % M
        assert h[i, j] == want

"""The matrix-core kernels (32-bit words) on both sides of the sizes and moduli where their
launches change: several passes of a workgroup (2^5 .. 2^8), 32 columns to a workgroup
instead of 16 and two passes of the row kernels (2^13 and longer), more rows than one chunk
of scratch holds, and moduli below 2^21 at every length that one has.  Results are exact:
equality with the oracle's sums for sampled rows and entries, with the same rows run by
themselves, and of round trips for every word."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import dev, host

pytestmark = pytest.mark.gpu

M = 13631489
# the longest length that each small prime has: 2^15, 2^16, 2^16, 2^17, 2^18
SMALL = {163841: 15, 65537: 16, 1376257: 16, 1179649: 17, 786433: 18}
WIDE_BLOCKS = 1536   # of 4096 elements: from here on 32 columns to a workgroup


@pytest.fixture(scope="module")
def nt():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256   # the counts below are for as many
    import paper_1005_1497_amd as nt
    return nt


def words(seed, *shape):
    """Random 32-bit words, all of them (operands need not be reduced)."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return torch.randint(-(1 << 31), 1 << 31, shape, generator=gen, dtype=torch.int64, device="cuda").to(torch.int32)


def reduced(x, m):
    return ((x.to(torch.int64) & 0xFFFFFFFF) % m).to(torch.int32)


def batch(nt, f, g, n, m, offs=None, flags=0):
    order = nt.max_log2n(m)
    count = f.numel() >> n
    offs = np.arange(count, dtype=np.int64) << n if offs is None else offs
    out = nt.conv_batched(f.view(-1), g.view(-1), nt.BatchDesc(np.full(count, n), offs), m,
                          root=nt.euler_root(m, order), root_log2order=order, flags=nt.FLAG_EULER | flags)
    return out.view(f.shape)


def check_convolutions(h, f, g, m, items):
    n, rng = f.shape[1].bit_length() - 1, np.random.default_rng(7)
    N = 1 << n
    for i in items:
        a, b, c = host(f[i]) % np.uint32(m), host(g[i]) % np.uint32(m), host(h[i])
        idx = np.arange(N, dtype=np.uint64) if n <= 9 else \
            np.concatenate([[0, 1, 255, 256, N // 2, N - 1], rng.integers(0, N, 12)]).astype(np.uint64)
        assert np.array_equal(c[idx.astype(np.int64)], oracle.conv_entries(a, b, m, idx).astype(np.uint32)), i
    # every output at once, item by item: their sum is the product of the operands' sums
    s = [(t.to(torch.int64) & 0xFFFFFFFF).sum(1) % m for t in (f, g, h)]
    assert torch.equal(s[2], s[0] * s[1] % m)
    assert int(h.max()) < m and int(h.min()) >= 0


# ---------------------------------------------------------------- several passes
# words of the batch per pass of all workgroups: 3 * 256 * 4096
@pytest.mark.parametrize("n", [5, 7, 8])
@pytest.mark.parametrize("passes,extra", [(2, 3), (3, 4099), (4, 100003)])
def test_several_passes(nt, n, passes, extra):
    """Convolutions, quotients and integers of 2^5 .. 2^8 whose workgroups take several
    passes, the last one a part of one, against the same items in shares of one pass."""
    share = (3 * 256 * 4096 >> n) - 5
    count = (passes * 3 * 256 * 4096 >> n) + extra
    if passes == 4:
        count = max(count, 100003)
    f, g = words(10 * n + passes, count, 1 << n), words(20 * n + passes, count, 1 << n)

    def pieces(fn):
        return torch.cat([fn(f[i:i + share].contiguous(), g[i:i + share].contiguous()) for i in range(0, count, share)])

    items = (0, 1, 4096 >> n, count // 2, count - 2, count - 1)
    h = batch(nt, f, g, n, M)
    assert torch.equal(h, pieces(lambda a, b: batch(nt, a, b, n, M)))
    check_convolutions(h, f, g, M, items)
    a = f.clone()                                       # over f
    order = nt.modulus_order(M)
    nt.conv_batched(a.view(-1), g.view(-1), nt.BatchDesc(np.full(count, n), np.arange(count, dtype=np.int64) << n), M,
                    root=nt.euler_root(M, order), root_log2order=order, out=a.view(-1), flags=nt.FLAG_EULER)
    assert torch.equal(a, h)
    # integers: 15-bit operands, whose sums stay below 2^38
    f, g = f & 0x7FFF, g & 0x7FFF
    c = nt.conv_crt(f, g)
    assert torch.equal(c, pieces(nt.conv_crt))
    assert torch.equal(c.sum(1), f.to(torch.int64).sum(1) * g.to(torch.int64).sum(1))
    for i in items:
        assert np.array_equal(host(c[i]), oracle.conv_integer(host(f[i]), host(g[i])))
    # quotients: the g of f * g, from divisors whose spectra have no zero
    F = reduced(f, M - 1) + 1
    f, g = nt.ntt_inverse(F, M), reduced(g, M)
    h = batch(nt, f, g, n, M)
    assert torch.equal(nt.deconvolve(f, h, M), g)
    F[count - 1, (1 << n) - 1] = 0
    with pytest.raises(nt.NttError) as e:
        nt.deconvolve(nt.ntt_inverse(F, M), h, M)
    assert e.value.name == "NTT_E_SINGULAR"


# ---------------------------------------------------------------- long transforms
def transforms(nt, n, rows, m):
    N, w = 1 << n, nt.euler_root(m, n)
    x = words(100 * n + rows, rows, N)
    before = nt.launch_counts()["matrix_transform"]
    X, Y = nt.ntt_forward(x, m, w, flags=nt.FLAG_EULER), nt.ntt_inverse(x, m, w, flags=nt.FLAG_EULER)
    assert nt.launch_counts()["matrix_transform"] == before + 2
    canon = reduced(x, m)
    assert torch.equal(nt.ntt_inverse(X, m, w, flags=nt.FLAG_EULER), canon)
    assert torch.equal(nt.ntt_forward(Y, m, w, flags=nt.FLAG_EULER), canon)
    rng = np.random.default_rng(n)
    some = sorted({0, rows // 2, rows - 1, int(rng.integers(0, rows))})
    bins = np.concatenate([np.tile(np.array([0, 1, 15, 16, 255, 256, N // 2, N - 1], np.uint64), (len(some), 1)),
                           rng.integers(0, N, (len(some), 16)).astype(np.uint64)], axis=1)
    at, xs = bins.astype(np.int64), np.stack([host(canon[r]) for r in some])
    got = np.take_along_axis(np.stack([host(X[r]) for r in some]), at, axis=1)
    assert np.array_equal(got, oracle.ntt_bins_rows(xs, m, w, bins).astype(np.uint32))
    got = np.take_along_axis(np.stack([host(Y[r]) for r in some]), at, axis=1)
    inv = oracle.ntt_bins_rows(xs, m, pow(w, m - 2, m), bins).astype(np.uint64)
    assert np.array_equal(got, (inv * np.uint64(pow(N, m - 2, m)) % np.uint64(m)).astype(np.uint32))
    for r in some:                                      # one row takes 16 columns to a workgroup
        one = x[r:r + 1].contiguous()
        assert torch.equal(nt.ntt_forward(one, m, w, flags=nt.FLAG_EULER)[0], X[r])
        assert torch.equal(nt.ntt_inverse(one, m, w, flags=nt.FLAG_EULER)[0], Y[r])
    z = x.clone()                                       # in place
    nt.ntt_forward(z, m, w, out=z, flags=nt.FLAG_EULER)
    assert torch.equal(z, X)


@pytest.mark.parametrize("n", range(13, 20))
@pytest.mark.parametrize("which", ["below", "at", "two chunks"])
def test_long_transforms_by_rows(nt, n, which):
    """One row less than 32 columns to a workgroup ask for, as many, and one more than
    128 MiB of scratch hold."""
    at = WIDE_BLOCKS >> (n - 12)
    transforms(nt, n, {"below": at - 1, "at": at, "two chunks": ((1 << 25) >> n) + 1}[which], M)


@pytest.mark.parametrize("m", sorted(SMALL))
@pytest.mark.parametrize("n", range(13, 19))
def test_long_transforms_small_moduli(nt, n, m):
    if n > SMALL[m]:
        pytest.skip("no transform of this length modulo m")
    for rows in (1, 3, (WIDE_BLOCKS >> (n - 12)) + 1):
        transforms(nt, n, rows, m)


# ---------------------------------------------------------------- three launches
THREE = [(n, m) for m in sorted(SMALL) for n in range(14, SMALL[m] + 1)] + [(n, M) for n in (14, 15, 16, 17, 19)]


def three_counts(n):
    """Few items; just past the switch to 32 columns in the last launch (2^14 has no such
    count: 128 items and more go one to a workgroup)."""
    return (3, 127) if n == 14 else (3, (WIDE_BLOCKS >> (n - 12)) + 1)


@pytest.mark.parametrize("n,m", THREE)
def test_three_launches_by_count(nt, n, m):
    N = 1 << n
    for count in three_counts(n):
        f, g = words(300 * n + count, count, N), words(400 * n + count, count, N)
        before = nt.launch_counts()["matrix_three"]
        h = batch(nt, f, g, n, m)
        assert nt.launch_counts()["matrix_three"] == before + 1
        check_convolutions(h, f, g, m, (0, count // 2, count - 1))
        assert torch.equal(h, batch(nt, f, g, n, m, flags=nt.FLAG_PER_ITEM))
        # the items in another order: through their offsets
        assert torch.equal(h, batch(nt, f, g, n, m, offs=np.arange(count, dtype=np.int64)[::-1] << n))
        for a, b in ((0x7F7F7F7F, 0x80808080), (0xFFFFFFFF, 0xFFFFFFFF), (m - 1, m - 1)):
            F, G = (torch.full((count, N), c - (c >> 31 << 32), dtype=torch.int32, device="cuda") for c in (a, b))
            assert bool((batch(nt, F, G, n, m) == N * a * b % m).all()), (hex(a), hex(b))


@pytest.mark.parametrize("n,m", THREE)
def test_quotients_by_rows(nt, n, m):
    N, w = 1 << n, nt.euler_root(m, n)
    kw = dict(flags=nt.FLAG_EULER)
    for rows in three_counts(n):
        F = reduced(words(500 * n + rows, rows, N), m - 1) + 1
        F[0] = m - 1
        g = reduced(words(600 * n + rows, rows, N), m)
        g[-1] = m - 1
        f = nt.ntt_inverse(F, m, w, **kw)
        G = nt.ntt_forward(g, m, w, **kw)
        h = nt.ntt_inverse((G.to(torch.int64) * F % m).to(torch.int32), m, w, **kw)
        before = nt.launch_counts()["matrix_three"]
        assert torch.equal(nt.deconvolve(f, h, m, w, **kw), g), rows
        assert nt.launch_counts()["matrix_three"] == before + 1
        for r, u in ((0, 0), (rows - 1, N - 1)):
            Z = F.clone()
            Z[r, u] = 0
            with pytest.raises(nt.NttError) as e:
                nt.deconvolve(nt.ntt_inverse(Z, m, w, **kw), h, m, w, **kw)
            assert e.value.name == "NTT_E_SINGULAR", (rows, r)

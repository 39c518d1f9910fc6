"""GPU parity of the matrix-core convolutions (32-bit words, lengths 2^5 .. 2^12).

The kernels carry residues as four signed bytes and take quotients from 32-bit
floats, so the inputs sit where that arithmetic is tightest: words whose bytes
are all at the ends of the signed range, residues at the ends of the centred
range, and moduli at the ends of the range that the kernels take (primes
k 2^13 + 1 either side of their limit of 14,600,000, above which the general
kernels run, and either side of 2^21, below which a residue takes one more
reduction, and tiny ones).  Item counts leave a part of the last chunk empty.
The results are exact integers: equality (tolerance 0) with the oracle's direct
sum for the first and the last item, and with the closed form h = N a b mod m
for every item of constant operands."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import dev, host

pytestmark = pytest.mark.gpu

MODULI = [(13631489, 20), (14499841, 13), (14663681, 13), (2056193, 13), (2236417, 13), (12289, 12), (641, 7)]


@pytest.fixture(scope="module")
def nt():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_1005_1497_amd as nt
    return nt


def batch(nt, f, g, n, count, m):
    order = nt.max_log2n(m)
    desc = nt.BatchDesc(np.full(count, n), np.arange(count, dtype=np.int64) << n)
    return host(nt.conv_batched(dev(f), dev(g), desc, m, root=nt.euler_root(m, order), root_log2order=order,
                                flags=nt.FLAG_EULER))


@pytest.mark.parametrize("m,top", MODULI)
@pytest.mark.parametrize("n", range(5, 13))
def test_lengths_and_moduli(nt, m, top, n):
    if n > min(top, nt.max_log2n(m)):
        pytest.skip("no transform of this length modulo m")
    N = 1 << n
    # one item; a chunk of 4096 elements and a part of the next
    for count in (1, 4096 // N + 1):
        rng = np.random.default_rng(1000 * n + count)
        f = rng.integers(0, 1 << 32, size=count * N, dtype=np.uint64).astype(np.uint32)
        g = rng.integers(0, 1 << 32, size=count * N, dtype=np.uint64).astype(np.uint32)
        h = batch(nt, f, g, n, count, m)
        for i in {0, count - 1}:
            ref = oracle.conv_direct(f[i * N:(i + 1) * N] % m, g[i * N:(i + 1) * N] % m, m).astype(np.uint32)
            assert np.array_equal(h[i * N:(i + 1) * N], ref), (count, i)
        if count == 1:   # one convolution by itself
            one = host(nt.conv_circular(dev(f), dev(g), m, flags=nt.FLAG_EULER))
            assert np.array_equal(one, h)
        for a, b in ((0x7F7F7F7F, 0x80808080), (0xFFFFFFFF, 0xFFFFFFFF), (m - 1, m - 1), ((m - 1) // 2, (m + 1) // 2)):
            h = batch(nt, np.full(count * N, a, np.uint32), np.full(count * N, b, np.uint32), n, count, m)
            assert np.all(h == N * a * b % m), (count, hex(a), hex(b))


def test_capture_on_a_fresh_stream(nt):
    """A batch of a short length is capturable on a stream that the library has
    not seen, once the plan exists; replays follow the operands' new values."""
    m, n, count = 13631489, 10, 9
    rng = np.random.default_rng(7)
    ops = [rng.integers(0, m, size=count << n).astype(np.uint32) for _ in range(4)]
    want = [batch(nt, ops[0], ops[1], n, count, m), batch(nt, ops[2], ops[3], n, count, m)]
    f, g = dev(ops[0]), dev(ops[1])
    out = torch.empty_like(f)
    order = nt.max_log2n(m)
    desc = nt.BatchDesc(np.full(count, n), np.arange(count, dtype=np.int64) << n)
    root = nt.euler_root(m, order)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        nt.conv_batched(f, g, desc, m, root=root, root_log2order=order, flags=nt.FLAG_EULER, out=out)
    for k in (0, 1, 0):
        f.copy_(dev(ops[2 * k]))
        g.copy_(dev(ops[2 * k + 1]))
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(host(out), want[k])


# primes either side of the kernels' thresholds: 2^21, 2,200,000 N / 4096, the limit
WIDE_MODULI = [(13, m) for m in (13631489, 2056193, 2236417, 4366337, 4423681, 14499841, 14663681)] + \
              [(14, m) for m in (13631489, 1785857, 2277377, 8716289, 8814593, 14499841, 14663681)]


@pytest.mark.parametrize("n,m", WIDE_MODULI)
def test_one_workgroup_lengths(nt, n, m):
    """Lengths 2^13 and 2^14, an item per workgroup: the smallest batches that
    take these kernels; more items than start at once (2^14: a workgroup's second
    item), out of order and with gaps between them."""
    N = 1 << n
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for count, gaps in (((cus + 1) // 2 if n == 14 else (2 * cus + 2) // 3, False), (cus + 1, True)):
        rng = np.random.default_rng(1000 * n + count)
        slots = rng.permutation(count + 2)[:count] if gaps else np.arange(count)
        total = (count + 2 if gaps else count) * N
        order = nt.max_log2n(m)
        desc = nt.BatchDesc(np.full(count, n), slots.astype(np.int64) << n)

        def run(f, g):
            return host(nt.conv_batched(dev(f), dev(g), desc, m, root=nt.euler_root(m, order), root_log2order=order,
                                        flags=nt.FLAG_EULER, out=dev(np.zeros(total, np.uint32))))

        f = rng.integers(0, 1 << 32, size=total, dtype=np.uint64).astype(np.uint32)
        g = rng.integers(0, 1 << 32, size=total, dtype=np.uint64).astype(np.uint32)
        h = run(f, g)
        for i in {0, count // 2, count - 1}:
            at = slice(int(slots[i]) * N, (int(slots[i]) + 1) * N)
            idx = np.concatenate([[0, 1, N // 2, N - 1], rng.integers(0, N, size=60)]).astype(np.uint64)
            ref = oracle.conv_entries(f[at] % m, g[at] % m, m, idx)
            assert np.array_equal(h[at][idx.astype(np.int64)], ref.astype(np.uint32)), (count, i)
            # every output at once: the outputs' sum is the product of the operands' sums
            assert int(h[at].astype(np.uint64).sum()) % m == \
                int(f[at].astype(np.uint64).sum()) % m * (int(g[at].astype(np.uint64).sum()) % m) % m
            assert int(h[at].max()) < m
        for a, b in ((0x7F7F7F7F, 0x80808080), (0xFFFFFFFF, 0xFFFFFFFF), (m - 1, m - 1), ((m - 1) // 2, (m + 1) // 2)):
            h = run(np.full(total, a, np.uint32), np.full(total, b, np.uint32)).reshape(-1, N)
            assert np.all(h[slots] == N * a * b % m), (count, hex(a), hex(b))
            if gaps:
                assert not np.delete(h, slots, axis=0).any()   # nothing between the items


@pytest.mark.parametrize("m,top", MODULI)
@pytest.mark.parametrize("n", range(5, 13))
def test_transforms(nt, m, top, n):
    """Forward and inverse transforms, natural order: one row; a chunk of 4096
    elements and a part of the next.  Every bin against the oracle's sum (the
    inverse through its definition: N^-1 times the transform by w^-1), constants
    and their spectra in closed form."""
    if n > min(top, nt.max_log2n(m)):
        pytest.skip("no transform of this length modulo m")
    N = 1 << n
    w = nt.euler_root(m, n)
    bins = np.arange(N, dtype=np.uint64)
    for rows in (1, 4096 // N + 1):
        rng = np.random.default_rng(2000 * n + rows)
        x = rng.integers(0, 1 << 32, size=(rows, N), dtype=np.uint64).astype(np.uint32)
        X = host(nt.ntt_forward(dev(x), m, w, flags=nt.FLAG_EULER))
        Y = host(nt.ntt_inverse(dev(x), m, w, flags=nt.FLAG_EULER))
        some = sorted({0, rows - 1})
        idx = np.tile(bins, (len(some), 1))
        assert np.array_equal(X[some], oracle.ntt_bins_rows(x[some] % m, m, w, idx).astype(np.uint32))
        inv = oracle.ntt_bins_rows(x[some] % m, m, pow(w, m - 2, m), idx).astype(np.uint64)
        assert np.array_equal(Y[some], (inv * np.uint64(pow(N, m - 2, m)) % np.uint64(m)).astype(np.uint32))
        assert np.array_equal(host(nt.ntt_inverse(dev(X), m, w, flags=nt.FLAG_EULER)), x % m)
        for a in (0x7F7F7F7F, 0x80808080, 0xFFFFFFFF, m - 1, (m + 1) // 2):
            for back in (False, True):
                fn = nt.ntt_inverse if back else nt.ntt_forward
                got = host(fn(dev(np.full((rows, N), a, np.uint32)), m, w, flags=nt.FLAG_EULER))
                want = np.zeros((rows, N), np.uint32)
                want[:, 0] = a % m if back else N * a % m
                assert np.array_equal(got, want), (rows, hex(a), back)


@pytest.mark.parametrize("m", [13631489, 1785857, 2277377, 14499841, 14663681, 7340033])
@pytest.mark.parametrize("n", range(13, 20))
def test_long_transforms(nt, n, m):
    """Forward and inverse transforms of 2^13 .. 2^19, natural order: one row and
    three (a last group of neighbouring workgroups that is not whole).  Chosen
    bins against the oracle's sums, the inverse by its definition and by the round
    trip of every word, constants and their spectra in closed form."""
    if n > nt.max_log2n(m):
        pytest.skip("no transform of this length modulo m")
    N = 1 << n
    w = nt.euler_root(m, n)
    for rows in (1, 3):
        rng = np.random.default_rng(3000 * n + rows)
        x = rng.integers(0, 1 << 32, size=(rows, N), dtype=np.uint64).astype(np.uint32)
        X = host(nt.ntt_forward(dev(x), m, w, flags=nt.FLAG_EULER))
        Y = host(nt.ntt_inverse(dev(x), m, w, flags=nt.FLAG_EULER))
        bins = np.concatenate([np.tile(np.array([0, 1, 255, 256, N // 2, N - 1], np.uint64), (rows, 1)),
                               rng.integers(0, N, (rows, 24)).astype(np.uint64)], axis=1)
        at = bins.astype(np.int64)
        assert np.array_equal(np.take_along_axis(X, at, axis=1),
                              oracle.ntt_bins_rows(x % m, m, w, bins).astype(np.uint32))
        inv = oracle.ntt_bins_rows(x % m, m, pow(w, m - 2, m), bins).astype(np.uint64)
        assert np.array_equal(np.take_along_axis(Y, at, axis=1),
                              (inv * np.uint64(pow(N, m - 2, m)) % np.uint64(m)).astype(np.uint32))
        assert np.array_equal(host(nt.ntt_inverse(dev(X), m, w, flags=nt.FLAG_EULER)), x % m)
        assert np.array_equal(host(nt.ntt_forward(dev(Y), m, w, flags=nt.FLAG_EULER)), x % m)
        for a in (0x7F7F7F7F, 0x80808080, 0xFFFFFFFF, m - 1, (m + 1) // 2):
            for back in (False, True):
                fn = nt.ntt_inverse if back else nt.ntt_forward
                got = host(fn(dev(np.full((rows, N), a, np.uint32)), m, w, flags=nt.FLAG_EULER))
                want = np.zeros((rows, N), np.uint32)
                want[:, 0] = a % m if back else N * a % m
                assert np.array_equal(got, want), (rows, hex(a), back)


@pytest.mark.parametrize("m", [13631489, 1785857, 2277377, 14499841, 14663681, 7340033])
@pytest.mark.parametrize("n", range(13, 20))
def test_three_launch_lengths(nt, n, m):
    """Convolutions of 2^13 .. 2^19 in three launches: one item and a small batch (a last
    group of neighbouring workgroups that is not whole), each also over f.  Chosen
    outputs against the oracle's sums, all of them through their sum, constants in
    closed form."""
    if n > nt.max_log2n(m):
        pytest.skip("no transform of this length modulo m")
    N = 1 << n
    order = nt.max_log2n(m)
    root = nt.euler_root(m, order)
    for count in (1, 3):
        rng = np.random.default_rng(4000 * n + count)
        desc = nt.BatchDesc(np.full(count, n), np.arange(count, dtype=np.int64) << n)

        def run(f, g, over=False):
            if count == 1:
                return host(nt.conv_circular(dev(f), dev(g), m, flags=nt.FLAG_EULER))
            a = dev(f)
            return host(nt.conv_batched(a, dev(g), desc, m, root=root, root_log2order=order, flags=nt.FLAG_EULER,
                                        out=a if over else None))

        f = rng.integers(0, 1 << 32, size=count * N, dtype=np.uint64).astype(np.uint32)
        g = rng.integers(0, 1 << 32, size=count * N, dtype=np.uint64).astype(np.uint32)
        before = nt.launch_counts()["fourstep"]
        h = run(f, g)
        assert nt.launch_counts()["fourstep"] == before + 1
        assert np.array_equal(run(f, g, over=True), h)
        for i in range(count):
            at = slice(i * N, (i + 1) * N)
            idx = np.concatenate([[0, 1, 255, 256, N // 2, N - 1], rng.integers(0, N, size=20)]).astype(np.uint64)
            ref = oracle.conv_entries(f[at] % m, g[at] % m, m, idx)
            assert np.array_equal(h[at][idx.astype(np.int64)], ref.astype(np.uint32)), (count, i)
            assert int(h[at].astype(np.uint64).sum()) % m == \
                int(f[at].astype(np.uint64).sum()) % m * (int(g[at].astype(np.uint64).sum()) % m) % m
            assert int(h[at].max()) < m
        for a, b in ((0x7F7F7F7F, 0x80808080), (0xFFFFFFFF, 0xFFFFFFFF), (m - 1, m - 1), ((m - 1) // 2, (m + 1) // 2)):
            assert np.all(run(np.full(count * N, a, np.uint32), np.full(count * N, b, np.uint32)) == N * a * b % m)


@pytest.mark.parametrize("m", [13631489, 2056193, 2236417, 14499841, 14663681, 12289])
@pytest.mark.parametrize("n", range(5, 18))
def test_quotients(nt, n, m):
    """Deconvolutions through each of the matrix-core forms: one row, a part of a chunk,
    and as many rows as the one-workgroup kernels take.  g from f and f * g exactly,
    with divisors whose spectra (one of them all ones but one) have no zero; a zero
    coefficient in the last row alone is reported."""
    if n > min(nt.max_log2n(m), 20):
        pytest.skip("no transform of this length modulo m")
    N = 1 << n
    w = nt.euler_root(m, n)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for rows in {1, max(3, 4096 // N + 1), cus if n in (13, 14) else 2}:
        rng = np.random.default_rng(5000 * n + rows)
        F = rng.integers(1, m, size=(rows, N)).astype(np.uint32)
        F[0] = 1
        F[0, N - 1] = m - 1
        f = nt.ntt_inverse(dev(F), m, w, flags=nt.FLAG_EULER)
        g = rng.integers(0, m, size=(rows, N)).astype(np.uint32)
        g[-1] = m - 1
        G = host(nt.ntt_forward(dev(g), m, w, flags=nt.FLAG_EULER)).astype(np.uint64)
        h = nt.ntt_inverse(dev((G * F % np.uint64(m)).astype(np.uint32)), m, w, flags=nt.FLAG_EULER)
        assert np.array_equal(host(nt.deconvolve(f, h, m, w, flags=nt.FLAG_EULER)), g), rows
        F[-1, N // 2] = 0
        f0 = nt.ntt_inverse(dev(F), m, w, flags=nt.FLAG_EULER)
        with pytest.raises(nt.NttError) as e:
            nt.deconvolve(f0, h, m, w, flags=nt.FLAG_EULER)
        assert e.value.name == "NTT_E_SINGULAR"


@pytest.mark.parametrize("n", [13, 14, 15, 16, 17])
def test_crt_either_side_of_the_persistent_kernel(nt, n):
    """Integer convolutions at the counts where the form changes: the batch that the
    persistent kernel takes and the one with an item less agree item by item, and
    with the oracle's integer sums (2^13 and 2^17: one form at every count)."""
    N = 1 << n
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    rows = {13: 3, 14: 1025, 15: 1025, 16: (4 * cus + 2) // 3, 17: 3}[n]
    b = (46 - n) // 2
    rng = np.random.default_rng(6000 + n)
    f = rng.integers(0, 1 << b, (rows, N), dtype=np.uint32)
    g = rng.integers(0, 1 << b, (rows, N), dtype=np.uint32)
    df, dg = dev(f), dev(g)
    h = host(nt.conv_crt(df, dg)).reshape(rows, N)
    less = host(nt.conv_crt(df[:-1].contiguous(), dg[:-1].contiguous())).reshape(rows - 1, N)
    assert np.array_equal(h[:-1], less)
    for r in (0, rows - 1):
        idx = np.unique(np.r_[0, N - 1, rng.integers(0, N, 10)]).astype(np.uint64)
        assert np.array_equal(h[r][idx.astype(int)], oracle.conv_integer_entries(f[r], g[r], idx))


@pytest.mark.parametrize("m", [13631489, 2277377, 14499841])
@pytest.mark.parametrize("lo,hi,count", [(6, 19, 40), (13, 17, 24), (8, 16, 700)])
def test_uneven_lengths_apart(nt, m, lo, hi, count):
    """Batches of several lengths, scattered, whose long ones leave the single persistent
    launch (all from 2^15 on with few items, from 2^17 on with many), against the
    convolutions one by one, bit for bit, and untouched words between the items."""
    hi = min(hi, nt.max_log2n(m))
    rng = np.random.default_rng(7000 + hi + count)
    logs = rng.integers(lo, hi + 1, size=count)
    logs[:2] = hi
    rng.shuffle(logs)
    sizes = (1 << logs) + 64                                  # a gap after each item
    offs = np.concatenate([[0], np.cumsum(sizes)[:-1]]).astype(np.int64)
    total = int(sizes.sum())
    f = rng.integers(0, 1 << 32, size=total, dtype=np.uint64).astype(np.uint32)
    g = rng.integers(0, 1 << 32, size=total, dtype=np.uint64).astype(np.uint32)
    order = nt.max_log2n(m)
    kw = dict(root=nt.euler_root(m, order), root_log2order=order)
    desc = nt.BatchDesc(logs, offs)
    df, dg = dev(f), dev(g)
    outs = []
    for flags in (nt.FLAG_EULER, nt.FLAG_EULER | nt.FLAG_PER_ITEM):
        before = nt.launch_counts()["multi"]
        out = dev(np.full(total, 0xABCDEF01, np.uint32))
        nt.conv_batched(df, dg, desc, m, out=out, flags=flags, **kw)
        outs.append(host(out))
        assert nt.launch_counts()["multi"] == before + (flags == nt.FLAG_EULER)
    assert np.array_equal(*outs)
    for n, o in zip(logs, offs):
        N, o = 1 << int(n), int(o)
        assert np.all(outs[0][o + N:o + N + 64] == 0xABCDEF01)
    for i in rng.integers(0, count, 6):
        N, o = 1 << int(logs[i]), int(offs[i])
        idx = np.unique(np.r_[0, N - 1, rng.integers(0, N, 10)]).astype(np.uint64)
        ref = oracle.conv_entries(f[o:o + N] % m, g[o:o + N] % m, m, idx)
        assert np.array_equal(outs[0][o:o + N][idx.astype(int)], ref.astype(np.uint32))


@pytest.mark.parametrize("n", range(5, 14))
def test_crt_short_lengths(nt, n):
    """Integer convolutions whose combining store is that of the short kernels: one
    item, and a chunk of 4096 elements with a part of the next; operands at the top of the
    exact range in the last item."""
    N = 1 << n
    b = (46 - n) // 2
    for rows in (1, max(2, 4096 // N + 1)):
        rng = np.random.default_rng(8000 + 10 * n + rows)
        f = rng.integers(0, 1 << b, (rows, N), dtype=np.uint32)
        g = rng.integers(0, 1 << b, (rows, N), dtype=np.uint32)
        f[-1] = g[-1] = (1 << b) - 1
        h = host(nt.conv_crt(dev(f), dev(g))).reshape(rows, N)
        assert np.all(h[-1] == N * ((1 << b) - 1) ** 2)
        for r in {0, rows // 2}:
            assert np.array_equal(h[r], oracle.conv_integer(f[r], g[r])), (rows, r)


@pytest.mark.parametrize("n", [9, 12])
def test_transforms_beyond_the_cache(nt, n):
    """The first and the last row of a transform of more than 2^24 elements (another
    number of waves per SIMD) against the same rows by themselves."""
    m, N = 13631489, 1 << n
    rows = ((1 << 24) >> n) + 1
    x = torch.randint(0, m, (rows, N), dtype=torch.int32, device="cuda")
    for fn in (nt.ntt_forward, nt.ntt_inverse):
        X = fn(x, m)
        for r in (0, rows - 1):
            assert torch.equal(X[r], fn(x[r:r + 1].contiguous(), m)[0])

"""Plans by word width: the tables of the matrix-core kernels, which 64-bit words never
use, are laid out by the first call with 32-bit words, and a plan that a 64-bit call built
serves 32-bit calls that may not lay out anything (under capture, without allocation)."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import dev, host

pytestmark = pytest.mark.gpu

M = 13631489


@pytest.fixture(scope="module")
def nt():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_1005_1497_amd as nt
    return nt


def operands(n, bits):
    rng = np.random.default_rng(n + bits)
    dt = np.uint32 if bits == 32 else np.uint64
    return [dev(rng.integers(0, M, 1 << n, dtype=dt)) for _ in range(2)]


def check(h, f, g):
    idx = np.unique(np.r_[0, 1, f.numel() - 1, np.random.default_rng(1).integers(0, f.numel(), 10)]).astype(np.uint64)
    ref = oracle.conv_entries(host(f), host(g), M, idx)
    assert np.array_equal(host(h)[idx.astype(np.int64)].astype(np.uint64), ref)


def test_64_bit_words_lay_out_no_matrix_tables(nt):
    n = 19
    f64, g64 = operands(n, 64)
    f, g = operands(n, 32)
    h64, h = torch.empty_like(f64), torch.empty_like(f)
    for _ in range(2):                                  # (the second time with every code object in place)
        nt.release_caches()
        torch.cuda.synchronize()
        nt.conv_circular(f64, g64, M, out=h64)
        torch.cuda.synchronize()
        after64 = torch.cuda.mem_get_info()[0]
        nt.conv_circular(f, g, M, out=h)
        torch.cuda.synchronize()
        after32 = torch.cuda.mem_get_info()[0]
    # three tables of a word per element, 2 MiB each
    assert after64 - after32 >= 3 * 4 << n
    check(h64, f64, g64)
    check(h, f, g)


@pytest.mark.parametrize("n", [6, 10, 13, 16])
def test_plan_of_the_other_width(nt, n):
    matrix = ("matrix_short", "matrix_one", "matrix_three")

    def took_matrix(call):
        before = nt.launch_counts()
        call()
        torch.cuda.synchronize()
        after = nt.launch_counts()
        return any(after[k] != before[k] for k in matrix)

    f64, g64 = operands(n, 64)
    f, g = operands(n, 32)
    h, root, s = torch.empty_like(f), nt.default_root(M, n), torch.cuda.Stream()
    nt.release_caches()
    h64 = nt.conv_circular(f64, g64, M)
    assert not took_matrix(lambda: nt.conv_circular_noalloc(f, g, M, root, h))
    check(h, f, g)
    if n <= 12:                                         # (longer ones need the stream's workspace first)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            nt.conv_circular(f, g, M, out=h)
        for _ in range(3):
            h.fill_(-1)
            graph.replay()
            torch.cuda.synchronize()
            check(h, f, g)
    h.fill_(-1)
    assert took_matrix(lambda: nt.conv_circular(f, g, M, out=h))
    check(h, f, g)
    h.fill_(-1)
    assert took_matrix(lambda: nt.conv_circular_noalloc(f, g, M, root, h))
    check(h, f, g)
    # and the other way round, with the fp64 tables shared
    nt.release_caches()
    nt.conv_circular(f, g, M, out=h)
    out = torch.empty_like(f64)
    nt.conv_circular_noalloc(f64, g64, M, root, out)
    assert torch.equal(out, h64)
    assert torch.equal(nt.conv_circular(f64, g64, M), h64)
    check(h, f, g)
    nt.release_caches()                                 # each table is freed once
    check(nt.conv_circular(f, g, M), f, g)


@pytest.mark.parametrize("n", [8, 12])
def test_integers_captured_with_plans_of_the_other_width(nt, n):
    """Integer convolutions need both moduli's plans; under capture those of 64-bit calls
    serve, with the combination in a pass of its own."""
    s = torch.cuda.Stream()
    f, g = (torch.randint(0, 1 << 15, (3, 1 << n), dtype=torch.int32, device="cuda") for _ in range(2))
    want = nt.conv_crt(f, g)
    for r in (0, 2):
        assert np.array_equal(host(want[r]), oracle.conv_integer(host(f[r]), host(g[r])))
    nt.release_caches()
    for m in (13631489, 7340033):
        x = torch.ones(1 << n, dtype=torch.int64, device="cuda")
        root = nt.default_root(m, n) if m == 13631489 else None
        nt.conv_circular(x, x, m, root=root, flags=nt.FLAG_EULER)
    # the buffer (two sets of residues of 3 rows of 2^12)
    nt.conv_crt(*(torch.ones(3, 1 << 13, dtype=torch.int32, device="cuda") for _ in range(2)), stream=s)
    out = torch.empty_like(want)
    torch.cuda.synchronize()
    before = nt.launch_counts()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        nt.conv_crt(f, g, out=out)
    assert nt.launch_counts()["matrix_short"] == before["matrix_short"]
    for _ in range(3):
        out.fill_(-1)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
    nt.conv_crt(f, g, out=out)
    assert torch.equal(out, want) and nt.launch_counts()["matrix_short"] == before["matrix_short"] + 2

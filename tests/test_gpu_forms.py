"""Which kernels a call takes, told by the launch counts: the class of the work (as many
items, as long as they are) and, apart from it, whether the matrix-core kernels ran it.
One call of each form and the forms' neighbours in number of items; 16515073 =
63 * 2^18 + 1 lies above the matrix-core kernels' largest modulus."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

M, M_GENERAL = 13631489, 16515073
CLASSES = ("small", "fourstep", "fused", "multi", "transform", "matrix_short", "matrix_one", "matrix_three",
           "matrix_transform")


@pytest.fixture(scope="module")
def nt():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_1005_1497_amd as nt
    return nt


def taken(nt, call):
    before = nt.launch_counts()
    call()
    torch.cuda.synchronize()
    after = nt.launch_counts()
    return {k: after[k] - before[k] for k in CLASSES if after[k] != before[k]}


def words(*shape):
    return torch.randint(1, 1 << 20, shape, dtype=torch.int32, device="cuda")


def batch(nt, m, logs, scattered=False):
    """conv_batched over items of these lengths, back to back or with gaps."""
    logs = np.asarray(logs)
    sizes = (1 << logs) + (8 if scattered else 0)
    offs = np.concatenate([[0], np.cumsum(sizes)[:-1]]).astype(np.int64)
    f = words(int(sizes.sum()))
    order = nt.max_log2n(m)
    return taken(nt, lambda: nt.conv_batched(f, f, nt.BatchDesc(logs, offs), m, root=nt.euler_root(m, order),
                                             root_log2order=order, flags=nt.FLAG_EULER))


@pytest.mark.parametrize("n,count,matrix,general", [
    (8, 3, {"small": 1, "matrix_short": 1}, {"small": 1}),
    (12, 3, {"small": 1, "matrix_short": 1}, {"small": 1}),
    (13, 1, {"fourstep": 1, "matrix_one": 1}, {"fourstep": 1}),
    (13, 700, {"fused": 1, "matrix_one": 1}, {"fused": 1}),
    (14, 100, {"fourstep": 1, "matrix_three": 1}, {"fourstep": 1}),
    (14, 256, {"fourstep": 1, "matrix_one": 1}, {"fourstep": 1}),
    (14, 530, {"fused": 1, "matrix_one": 1, "matrix_three": 1}, {"fused": 1}),
    (15, 1024, {"fused": 1, "matrix_three": 1}, {"fused": 1}),
    (15, 1025, {"fused": 1}, {"fused": 1}),
    (16, 256, {"fourstep": 1, "matrix_three": 1}, {"fourstep": 1}),
    (16, 342, {"fused": 1}, {"fused": 1}),
    (17, 300, {"fused": 1, "matrix_three": 1}, {"fused": 1}),
    (18, 20, {"fourstep": 1, "matrix_three": 1}, {"fourstep": 1}),
])
def test_batches_of_one_length(nt, n, count, matrix, general):
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256
    assert batch(nt, M, [n] * count) == matrix
    assert batch(nt, M_GENERAL, [n] * count) == general


def test_batches_of_several_lengths(nt):
    rng = np.random.default_rng(1)
    few = [15, 8, 15, 9, 15, 17, 17, 6]
    many = list(rng.integers(6, 17, 900)) + [17, 18, 18]
    short = list(rng.integers(6, 14, 2000))
    # scattered: 2^15 and 2^17 of a few items, 2^17 and 2^18 of many leave the one launch
    assert batch(nt, M, few, scattered=True) == {"multi": 1, "matrix_three": 2}
    assert batch(nt, M, many, scattered=True) == {"multi": 1, "matrix_three": 2}
    assert batch(nt, M, short, scattered=True) == {"multi": 1}
    for logs in (few, many, short):
        assert batch(nt, M_GENERAL, logs, scattered=True) == {"multi": 1}


def test_single_calls(nt):
    for m, matrix in ((M, True), (M_GENERAL, False)):
        for n, kind, form in ((10, "small", "matrix_short"), (13, "fourstep", "matrix_one"), (14, "fourstep", "matrix_three"),
                              (18, "fourstep", "matrix_three")):
            x = words(1 << n)
            want = {kind: 1, form: 1} if matrix else {kind: 1}
            assert taken(nt, lambda: nt.conv_circular(x, x, m, flags=nt.FLAG_EULER)) == want
            for fn in (nt.ntt_forward, nt.ntt_inverse):
                want = {"transform": 1, "matrix_transform": 1} if matrix else {"transform": 1}
                assert taken(nt, lambda: fn(x, m, flags=nt.FLAG_EULER)) == want
        # without a workspace of its own 2^13 goes through the static one
        x, out = words(1 << 13), words(1 << 13)
        want = {"fourstep": 1, "matrix_three": 1} if matrix else {"fourstep": 1}
        assert taken(nt, lambda: nt.conv_circular_noalloc(x, x, m, nt.euler_root(m, 13), out,
                                                          flags=nt.FLAG_EULER)) == want


@pytest.mark.parametrize("n,rows,form", [(10, 5, "matrix_short"), (13, 5, "matrix_one"), (14, 5, "matrix_three"),
                                         (14, 128, "matrix_one"), (15, 600, None), (16, 256, "matrix_three"),
                                         (16, 300, None), (18, 3, "matrix_three")])
def test_quotients(nt, n, rows, form):
    f = torch.zeros(rows, 1 << n, dtype=torch.int32, device="cuda")
    f[:, 0] = 2                                     # its spectrum is 2 everywhere
    h = words(rows, 1 << n)
    kind = "small" if n <= 12 else "fused"
    assert taken(nt, lambda: nt.deconvolve(f, h, M)) == ({kind: 1, form: 1} if form else {kind: 1})
    assert taken(nt, lambda: nt.deconvolve(f, h, M_GENERAL, flags=nt.FLAG_EULER)) == {kind: 1}


@pytest.mark.parametrize("n,rows,want", [
    (10, 5, {"small": 2, "matrix_short": 2}),
    (13, 5, {"fourstep": 1, "fused": 1, "matrix_one": 2}),
    (14, 5, {"fourstep": 1, "fused": 1, "matrix_three": 2}),
    (15, 1025, {"fused": 2}),
    (17, 2, {"fourstep": 1, "fused": 1, "matrix_three": 2}),
])
def test_integers(nt, n, rows, want):
    f = words(rows, 1 << n)
    assert taken(nt, lambda: nt.conv_crt(f, f)) == want


def test_two_dimensions(nt):
    f = words(1 << 6, 1 << 7)
    assert taken(nt, lambda: nt.conv2d(f, f, M)) == {"transform": 3, "matrix_transform": 3, "small": 1, "matrix_short": 1}
    assert taken(nt, lambda: nt.conv2d(f, f, M_GENERAL, flags=nt.FLAG_EULER)) == {"transform": 3, "small": 1}

"""The short matrix-core kernels (32-bit words, lengths 2^5 .. 2^12) write their batch and
nothing else: the output is a part of a larger buffer whose other words are checked
afterwards, 4096 before it and 16384 after it (four chunks), for one item and for a chunk
of 4096 elements with a part of the next.  The results are those of constant operands in
closed form, next to inputs whose words beyond the batch are not those constants."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

M = 13631489
BEFORE, AFTER, MARK = 4096, 16384, 0x5A5A5A5A


@pytest.fixture(scope="module")
def nt():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_1005_1497_amd as nt
    return nt


def inside(shape, dtype, value):
    """A tensor of `value` in the middle of a buffer of MARK, and the buffer."""
    count = int(np.prod(shape))
    whole = torch.full((BEFORE + count + AFTER,), MARK, dtype=dtype, device="cuda")
    part = whole[BEFORE:BEFORE + count].view(shape)
    part.fill_(value)
    return part, whole


def untouched(whole):
    return bool((whole[:BEFORE] == MARK).all()) and bool((whole[-AFTER:] == MARK).all())


@pytest.mark.parametrize("n", range(5, 13))
@pytest.mark.parametrize("what", ["convolution", "forward", "inverse", "quotient", "integers"])
def test_nothing_beyond_the_batch(nt, what, n):
    N = 1 << n
    for rows in (1, 4096 // N + 1):
        shape, a, b = (rows, N), 1234567, M - 3
        f, _ = inside(shape, torch.int32, a)
        g, _ = inside(shape, torch.int32, b)
        out, whole = inside(shape, torch.int64 if what == "integers" else torch.int32, 7)
        want = np.zeros((rows, N), np.int64)
        if what == "convolution":
            desc = nt.BatchDesc(np.full(rows, n), np.arange(rows, dtype=np.int64) << n)
            nt.conv_batched(f.view(-1), g.view(-1), desc, M, out=out.view(-1))
            want[:] = N * a * b % M
        elif what == "forward":
            nt.ntt_forward(f, M, out=out)
            want[:, 0] = N * a % M
        elif what == "inverse":
            nt.ntt_inverse(f, M, out=out)
            want[:, 0] = a
        elif what == "quotient":
            # the divisor 2 at t = 0: its spectrum is 2 everywhere
            f.zero_()
            f[:, 0] = 2
            nt.deconvolve(f, g, M, out=out)
            want[:] = b * pow(2, M - 2, M) % M
        else:
            f.fill_(3)
            g.fill_(5)
            nt.conv_crt(f, g, out=out)
            want[:] = 15 * N
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), want), (what, rows)
        assert untouched(whole), (what, rows)

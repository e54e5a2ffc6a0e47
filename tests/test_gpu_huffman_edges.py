"""The Huffman kernels at their edges (bit for bit against the oracle): symbols per lane, per block and
per decoder chunk, streams that do not start on 16 bytes, code tables at the sizes where they move
between LDS and memory, and codes that end a decoder's staged stretch."""

import numpy as np
import pytest

from oracle import huffman as HF
from paper_2601_01596_amd import ffcz as F
from tests.test_gpu_huffman import _check, _parse

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.uint8, np.int32])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 255, 256, 257, 4095, 4096, 4097, 16383, 16384, 16385, 64 * 256 + 1])
def test_stream_lengths(n, dtype):
    g = np.random.default_rng(n)
    _check(np.minimum(g.geometric(0.3, n), 40) + (0 if dtype == np.uint8 else -17), dtype)


@pytest.mark.parametrize("nalpha", [2, 3, 2047, 2048, 2049, 8191, 8192, 8193, 32767, 32768, 32769, 65537])
def test_alphabet_sizes(nalpha):
    # every symbol occurs, most of them once: the longest code tables of each size
    g = np.random.default_rng(nalpha)
    sym = np.concatenate([np.arange(nalpha), g.integers(0, max(2, nalpha // 64), 50000)])
    g.shuffle(sym)
    _check(sym, np.int32)


@pytest.mark.parametrize("dtype,skip", [(np.uint8, 1), (np.uint8, 7), (np.uint8, 15), (np.int32, 1), (np.int32, 3)])
def test_streams_off_the_16_byte_grid(dtype, skip):
    import torch
    g = np.random.default_rng(9)
    sym = np.minimum(g.geometric(0.2, 20000), 60).astype(dtype)
    t = torch.from_numpy(sym).cuda()[skip:]
    stream, sizes = F.huffman_compress(t)
    ref = HF.encode(sym[skip:].astype(np.int64))
    got = _parse(stream, sym.itemsize)
    np.testing.assert_array_equal(got["words"], ref.words)
    np.testing.assert_array_equal(got["chunks"], ref.chunk_bits)
    back = F.huffman_decompress(stream, sym.size - skip, t.dtype, int(sizes.nalpha))
    np.testing.assert_array_equal(back.cpu().numpy()[: sym.size - skip], sym[skip:])


def test_chunks_of_long_and_of_short_codes():
    # chunks of 256 rare symbols (long codes, far apart) beside chunks of the commonest one
    fib = [1, 1]
    while len(fib) < 24:
        fib.append(fib[-1] + fib[-2])
    body = np.repeat(np.arange(24), fib)
    rare = np.arange(256) % 6
    _check(np.concatenate([rare, body, rare, body[-700:], rare]), np.int32)

"""Initial weights of a guess network for a seed stay bit for bit: He-normal weights from
std::normal_distribution<double> (libstdc++) on std::mt19937_64, drawn layer by layer, biases zero.  The checksums are those of
a program that draws them so."""

import zlib

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("widths,seed,count,first,crc", [
    ((16, 32, 64, 64), None, 111442, 0.28623873, 3882591860),
    ((32, 16, 32, 32), 7, 56706, 0.205696225, 2547839869),
    ((16, 16, 16, 16), 123456789012345, 21458, 0.151792124, 3162094573)])
def test_initial_weights(widths, seed, count, first, crc):
    from paper_2103_17081_amd.binding import GuessNet
    print("case: initial weights", widths, seed, flush=True)
    net = GuessNet(widths, tile=32, max_batch=1, seed=seed)
    w = net.get_params()
    net.close()
    assert w.size == count and w[0] == np.float32(first)
    assert zlib.crc32(w.tobytes()) == crc

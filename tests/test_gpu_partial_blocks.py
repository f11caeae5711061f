"""One-product path: a segment's tokens are cut into blocks of up to 32 token tiles, its last one or all of them partial; a block
of up to 4, 8, 12 or 16 tiles has its k blocks shared by two wavefronts per column, one of more has eight columns of three or
four.  Every number of tiles, with the contraction split over workgroups (few rows) and not, 7 and 8 row tiles per workgroup,
one launch and two."""
import pytest

from inputs import synth
from test_gpu_parity import run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_in,d_out,k,bits", [(520, 72, 8, 2), (264, 2064, 5, 3), (136, 4096, 0, 1), (1032, 200, 33, 4)])
@pytest.mark.parametrize("lengths", [[193], [256], [257], [320, 321], [449, 512, 384, 300], [192, 5, 448, 513], [255] * 3 + [258] * 3 + [200] * 3])
def test_partial_token_blocks(d_in, d_out, k, bits, lengths):
    off = [0]
    for n in lengths:
        off.append(off[-1] + n)
    run_case(synth.small_case(d_in, d_out, off, k, bits, seed=len(lengths)))


@pytest.mark.parametrize("d_in,d_out,k,bits", [(1480, 360, 64, 4), (520, 1928, 0, 2), (2056, 72, 33, 1), (896, 1032, 8, 3)])
@pytest.mark.parametrize("lengths", [[193], [270, 345], [200, 331, 449]])
def test_small_token_blocks(d_in, d_out, k, bits, lengths):
    """Launches that leave most of the chip idle are cut into blocks of up to 4 or 8 token tiles, also with the contraction split."""
    off = [0]
    for n in lengths:
        off.append(off[-1] + n)
    run_case(synth.small_case(d_in, d_out, off, k, bits, seed=3 + len(lengths)))

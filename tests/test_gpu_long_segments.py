"""Long segments on the one-product path: calls of more token blocks than a launch lists one by one."""
import pytest

from inputs import synth
from test_gpu_parity import run_case

pytestmark = pytest.mark.gpu


def offsets(lengths):
    off = [0]
    for n in lengths:
        off.append(off[-1] + n)
    return off


@pytest.mark.parametrize("d_in,d_out,k,bits,lengths", [
    (264, 136, 8, 2, [23000, 200, 45800]),   # 32-tile blocks, the last ones as halves, three partial ones
    (136, 72, 0, 3, [70000]),                # one row group: 24-tile blocks
    (72, 40, 5, 4, [9000] * 7 + [5, 9000]),  # eight long segments and a streamed one
])
def test_more_blocks_than_the_list_holds(d_in, d_out, k, bits, lengths):
    run_case(synth.small_case(d_in, d_out, offsets(lengths), k, bits, seed=len(lengths)))

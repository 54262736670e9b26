"""The convolution layer's im2col state on layers whose product has few tiles: 128-tiles shared by sixteen workgroups (up to 96
tiles of 64) and whole 64-tiles, against the oracle."""
import pytest

from paper_2605_28213_amd import gemm
from paper_2605_28213_amd import inputs as gen
from tests.test_conv_gpu import reference, run_state
from tests.util import TOL, norm_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [gen.F16, gen.BF16])
@pytest.mark.parametrize("n,hw,C,F,tile", [(1, 9, 3, 8, 128), (2, 31, 24, 70, 128), (3, 31, 3, 129, 64), (2, 56, 24, 66, 64)])
def test_im2col_of_few_tiles(dtype, n, hw, C, F, tile):
    cfg = gen.ConvConfig("few", n, hw, hw, C, F, 3, 3, dtype, dtype, biased=F % 2 == 0)
    inp = gen.make_conv_inputs(cfg, F)
    rc, y, q, dy = run_state(1, inp)
    assert rc == gemm.GEMM_OK and q.bm == tile and q.threads == 256, q
    y_ref, d = reference(inp)
    assert norm_err(y, y_ref, d) <= TOL[dtype]

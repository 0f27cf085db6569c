"""The coarse residual's backward kernels at the block counts where their tiles of 16 (above 1088 blocks: 4) rows end, and with
a block of one token, against the fp64 oracle's gradient."""
import pytest

import workloads as W
from test_gpu_backward import test_backward_on_oracle_lists as backward_matches_the_oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def I():
    import paper_2605_04569_amd as isa
    isa.lib()
    return isa


@pytest.mark.parametrize("src,ctx", [(1, 1), (9, 7), (10, 7), (20, 12), (21, 12), (24, 1064), (24, 1065), (24, 1077)])
def test_block_counts(I, src, ctx):
    # context blocks are not kept and no query block is exact: the residual is most of the gradient, and the oracle stays cheap
    wl = W.CONFIGS["cfg1"].with_(name="coarse_backward", H=1 if ctx > 100 else 3, src_grid=(1, 1, 128 * (src - 1) + 1),
                                 ctx_grids=(((1, 1, 128 * (ctx - 1) + 77),),), keep_ratio=0.0, full_frac=0.0, gamma=2.0,
                                 seed=900 + src + ctx)
    backward_matches_the_oracle(I, wl)

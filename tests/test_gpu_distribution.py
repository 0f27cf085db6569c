"""Work distribution of the pipelined kernels over the XCDs: every item of every (batch, head) runs exactly once whatever the
number of heads, and items that a launch of less than a round cuts into key ranges (forward) or parts of the streamed side
(backward, both phases) add up."""
import pytest

import workloads as W
from test_gpu_backward import test_backward_on_oracle_lists as backward_matches_the_oracle
from test_gpu_parity import check_end_to_end, gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def I():
    import paper_2605_04569_amd as isa
    isa.lib()
    return isa


def _wl(H, src, ctx, **kw):
    return W.CONFIGS["cfg1"].with_(name="distribution", H=H, src_grid=src, ctx_grids=ctx, **kw)


# fewer heads than XCDs, one more than a multiple of 8, heads x pairs that 8 does not divide, exactly 8 and 16
@pytest.mark.parametrize("H", [1, 2, 3, 5, 7, 8, 9, 12, 16, 20])
def test_forward(I, H):
    wl = _wl(H, (2, 10, 40), (((1, 10, 33), (1, 2, 50)),), keep_ratio=0.6, full_frac=0.4, seed=800 + H)
    check_end_to_end(I, wl, *gen(wl))


# key lists of 2 to 7 blocks: too short to be cut, two ranges, three ranges of unequal length
@pytest.mark.parametrize("blocks", [2, 3, 4, 5, 6, 7])
def test_forward_short_key_lists(I, blocks):
    wl = _wl(3, (1, 1, 128 * (blocks - 1) + 7), (((1, 1, 200),),), keep_ratio=0.0, full_frac=0.7, seed=830 + blocks)
    assert I.isa_get_counts(I.Problem(H=3, D=128, dtype="bf16", block=128, seg_len=[wl.seg_len(0)], keep_ratio=0.0, full_frac=0.7))["T_new"] == blocks
    check_end_to_end(I, wl, *gen(wl))


@pytest.mark.parametrize("exact_frac", [0.0, 0.3])
@pytest.mark.parametrize("H", [1, 5, 9, 12])
def test_backward(I, H, exact_frac):
    wl = _wl(H, (2, 10, 40), (((1, 10, 33),),), keep_ratio=0.6, full_frac=0.4, exact_frac=exact_frac, gamma=0.5 if H == 5 else 0.0,
             seed=850 + H)
    backward_matches_the_oracle(I, wl)


# one streamed entry only (not to be cut), two, and a ragged batch whose shorter item has fewer entries than parts
@pytest.mark.parametrize("full_frac", [0.05, 0.25])
def test_backward_few_streamed_entries(I, full_frac):
    wl = _wl(3, (1, 10, 60), (((1, 10, 33),), ((1, 1, 40),)), B=2, keep_ratio=1.0, full_frac=full_frac, exact_frac=0.3, seed=870)
    backward_matches_the_oracle(I, wl)

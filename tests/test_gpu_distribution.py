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


# dQ of both branches and the mean rows in one launch: 48 heads of 3 + 2 blocks are the most that fit one round of the chip (items cut for
# one round), 49 are the first that do not; one head has room for the most parts
@pytest.mark.parametrize("exact_frac", [0.0, 0.3])
@pytest.mark.parametrize("H", [1, 48, 49])
def test_backward_one_launch(I, H, exact_frac):
    wl = _wl(H, (1, 6, 64), (((1, 3, 70),),), keep_ratio=0.5, full_frac=0.6, exact_frac=exact_frac, seed=865 + H)
    c = I.isa_get_counts(I.Problem(H=H, D=128, dtype="bf16", block=128, seg_len=[wl.seg_len(0)], keep_ratio=0.5, full_frac=0.6), 0)
    assert (c["n_full"], c["n_flat"]) == (3, 2)
    assert (-(-2 * H // 8) + 3 * -(-H // 8) <= 32) == (H <= 48)      # items of an XCD: two pairs, one pair, one group of means twice
    backward_matches_the_oracle(I, wl)


# the three kinds of items fit one round as they are, their parts do not (6 pairs of an XCD in up to 5 parts each, 15 Taylor pairs, 3 groups of
# means twice in up to 4)
@pytest.mark.parametrize("exact_frac", [0.0, 0.2])
def test_backward_parts_past_a_round(I, exact_frac):
    wl = _wl(24, (1, 9, 100), (((1, 5, 127),),), keep_ratio=0.5, full_frac=0.3, exact_frac=exact_frac, seed=868)
    c = I.isa_get_counts(I.Problem(H=24, D=128, dtype="bf16", block=128, seg_len=[wl.seg_len(0)], keep_ratio=0.5, full_frac=0.3), 0)
    assert (c["n_full"], c["n_flat"], c["T_new"]) == (4, 9, 10)
    backward_matches_the_oracle(I, wl)


# one streamed entry only (not to be cut), two, and a ragged batch whose shorter item has fewer entries than parts
@pytest.mark.parametrize("full_frac", [0.05, 0.25])
def test_backward_few_streamed_entries(I, full_frac):
    wl = _wl(3, (1, 10, 60), (((1, 10, 33),), ((1, 1, 40),)), B=2, keep_ratio=1.0, full_frac=full_frac, exact_frac=0.3, seed=870)
    backward_matches_the_oracle(I, wl)


# launches of nothing but long items, 8 rounds or more: items from a counter, the last 64 as four key ranges each (the last heads);
# 16 key blocks is the shortest list that may be cut so, 17 makes the ranges unequal
@pytest.mark.parametrize("blocks", [16, 17])
def test_counted_items_dense(I, blocks):
    import numpy as np
    import torch
    from oracle import isa_oracle as O
    from test_gpu_parity import TOL
    from util import err_stats, f64, problem_of
    H = 300
    wl = _wl(H, (1, 1, 128 * (blocks - 1) + 5), ((),), seed=880 + blocks)
    assert H * ((blocks + 1) // 2) // 8 >= 8 * 32                                       # the premise: 8 rounds of an XCD's 32 units
    Q, K, V, q, k, v = gen(wl)
    pr = problem_of(wl)
    out = torch.full_like(q, float("nan"))
    I.isa_dense_attention(pr, q, k, v, out, I.new_workspace(pr))
    torch.cuda.synchronize()
    assert torch.isfinite(out.float()).all()
    for h in (0, 100, 290, 292, 295, 299):
        emax, emean = err_stats(f64(out[0, h]), O.dense_attention(f64(Q[0, h]), f64(K[0, h]), f64(V[0, h])))
        assert emax <= TOL["bf16"][0] and emean <= TOL["bf16"][1], (h, emax, emean)


def test_counted_items_beside_exact_sets(I):
    wl = _wl(200, (1, 1, 128 * 17 + 5), (((1, 1, 500),), ((1, 1, 70),)), B=2, keep_ratio=0.5, full_frac=0.6, exact_frac=0.2, gamma=0.5,
             seed=890)
    check_end_to_end(I, wl, *gen(wl), heads=[0, 77, 192, 199])


def test_counted_items_backward(I):
    """Backward of 8 rounds or more: the last 32 items of the dQ and of the dK / dV launch run in 8 parts each (the last heads).
    Everything kept and exact: the gradient of dense attention, whatever the scores."""
    import numpy as np
    import torch
    from oracle import isa_oracle_bwd as OB
    from test_gpu_backward import TOL_MAX_REL, TOL_MEAN_REL, _inputs
    from util import f64, problem_of
    H = 240
    wl = _wl(H, (1, 1, 128 * 9 + 5), (((1, 1, 128 * 7 + 60),),), keep_ratio=1.0, full_frac=1.0, seed=895)
    pr = problem_of(wl)
    c = I.isa_get_counts(pr, 0)
    assert c["n_full"] >= 16 and H * ((c["n_full"] + 1) // 2) // 8 >= 8 * 32 and c["n_flat"] == 0          # the premise
    Q, K, V, dO = _inputs(wl)
    q, k, v, g = (t.cuda() for t in (Q, K, V, dO))
    ws = I.new_workspace(pr)
    out = torch.empty_like(q)
    grads = [torch.full_like(q, float("nan")) for _ in range(3)]
    I.isa_attention(pr, q, k, v, out, ws)
    I.isa_attention_backward(pr, q, k, v, out, g, *grads, ws)
    torch.cuda.synchronize()
    assert all(torch.isfinite(x.float()).all() for x in grads)
    for h in (0, 120, 236, 237, 238, 239):
        for got, want in zip(grads, OB.dense_attention_bwd(*(f64(t[0, h]) for t in (Q, K, V, dO)))):
            d = np.abs(f64(got[0, h]) - want) / np.abs(want).max()
            assert d.max() <= TOL_MAX_REL and d.mean() <= TOL_MEAN_REL, (h, d.max(), d.mean())


def test_counted_items_whole(I):
    """64 rounds of long items beside a batch item too short to be cut: whole items from the counter, those of the short item among them."""
    import torch
    from oracle import isa_oracle as O
    from test_gpu_parity import TOL
    from util import err_stats, f64
    H, lens = 256, (128 * 63 + 5, 100)
    assert 2 * H * 32 // 8 >= 64 * 32                                                   # the premise
    g = torch.Generator(device="cuda").manual_seed(897)
    q, k, v = (torch.randn((2, H, lens[0], 128), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    pr = I.Problem(H=H, D=128, dtype="bf16", block=128, seg_len=[[n] for n in lens], keep_ratio=1.0, full_frac=1.0)
    out = torch.full_like(q, float("nan"))
    I.isa_dense_attention(pr, q, k, v, out, I.new_workspace(pr))
    torch.cuda.synchronize()
    for b, n in enumerate(lens):
        assert torch.isfinite(out[b, :, :n]).all() and torch.isnan(out[b, :, n:]).all()
        for h in (0, 1, 130, H - 1):
            rows = slice(0, n, 97 if b == 0 else 1)
            emax, emean = err_stats(f64(out[b, h, :n][rows]), O.dense_attention(f64(q[b, h, :n][rows]), f64(k[b, h, :n]), f64(v[b, h, :n])))
            assert emax <= TOL["bf16"][0] and emean <= TOL["bf16"][1], (b, h, emax, emean)


def test_counted_items_backward_taylor(I):
    """dQ of Taylor blocks over 1000 kept blocks (16 tiles of means): items from the counter, the last 32 in 8 parts along the means."""
    import numpy as np
    import torch
    from oracle import isa_oracle as O
    from oracle import isa_oracle_bwd as OB
    from test_gpu_backward import TOL_MAX_REL, TOL_MEAN_REL
    from util import f64
    H, T, S = 5, 1000, 128 * 999 + 77
    pr = I.Problem(H=H, D=128, dtype="bf16", block=128, seg_len=[[S]], keep_ratio=0.0, full_frac=0.0)
    c = I.isa_get_counts(pr, 0)
    assert c["n_flat"] == c["T_new"] == T > 960 and H * (T // 2) // 8 >= 8 * 32                     # the premise
    g = torch.Generator(device="cuda").manual_seed(898)
    rand = lambda n: torch.randn((1, H, n, 128), generator=g, device="cuda")
    blocks = lambda: rand(T).repeat_interleave(128, 2)[:, :, :S]                                # the means differ from block to block
    q, k, v, d_out = (x.bfloat16() for x in (rand(S), blocks() + 0.3 * rand(S), blocks() + 0.3 * rand(S), rand(S)))
    ws = I.new_workspace(pr)
    out = torch.empty_like(q)
    grads = [torch.full_like(q, float("nan")) for _ in range(3)]
    I.isa_attention(pr, q, k, v, out, ws)
    I.isa_attention_backward(pr, q, k, v, out, d_out, *grads, ws)
    torch.cuda.synchronize()
    assert all(torch.isfinite(x).all() for x in grads)
    for h in (0, 3, 4):
        x = [f64(t[0, h]) for t in (q, k, v, d_out)]
        plan = O.isa_plan(*x[:3], [S], 128, 0.0, 0.0)
        some = sorted({0, 1, 500, 934, 935, 936, 937, 980, 997, 998, 999})                     # 936 on: the last 32 pairs of head 4
        want = OB.isa_attention_bwd(*x, plan, query_blocks=some)[0]
        for i in some:
            rows = slice(128 * i, min(S, 128 * i + 128))
            d = np.abs(f64(grads[0][0, h, rows]) - want[rows]) / np.abs(want).max()
            assert d.max() <= TOL_MAX_REL and d.mean() <= TOL_MEAN_REL, (h, i, d.max(), d.mean())


def test_counted_items_backward_with_exact_sets(I):
    """dK and dV of 8 rounds or more beside exact sets: the parts of the last 32 items share the exact branch's list and that of the
    Taylor blocks linked to the item's block."""
    import numpy as np
    import torch
    from oracle import isa_oracle as O
    from oracle import isa_oracle_bwd as OB
    from test_gpu_backward import TOL_MAX_REL, TOL_MEAN_REL, _inputs
    from util import f64, problem_of
    wl = _wl(200, (1, 1, 128 * 17 + 5), (((1, 1, 500),),), keep_ratio=0.5, full_frac=0.75, exact_frac=0.3, seed=899)
    pr = problem_of(wl)
    c = I.isa_get_counts(pr, 0)
    assert wl.H * c["T_new"] // 8 >= 8 * 32 and c["n_full"] >= 16 and c["n_flat"] >= 5 and c["k_exact"] >= 5       # the premise
    Q, K, V, dO = _inputs(wl)
    q, k, v, d_out = (t.cuda() for t in (Q, K, V, dO))
    ws = I.new_workspace(pr)
    out = torch.empty_like(q)
    grads = [torch.full_like(q, float("nan")) for _ in range(3)]
    I.isa_attention(pr, q, k, v, out, ws)
    lay = I.isa_workspace_layout(pr)
    T_max, lists = c["T_max"], (1, wl.H, c["T_max"])
    kv_g, full_g, flat_g = (I.workspace_array(ws, lay[n], lists, torch.int32).cpu().numpy() for n in ("kv_list", "full_list", "flat_list"))
    mask_g = I.workspace_array(ws, lay["exact_mask"], lists + ((T_max + 31) // 32,), torch.int32).cpu().numpy().view(np.uint32)
    I.isa_attention_backward(pr, q, k, v, out, d_out, *grads, ws)
    torch.cuda.synchronize()
    assert all(torch.isfinite(x.float()).all() for x in grads)
    for h in (0, 100, 197, 198, 199):
        x = [f64(t[0, h]) for t in (Q, K, V, dO)]
        plan = O.isa_plan(*x[:3], wl.seg_len(0), 128, 0.5, 0.75, 0.3)
        # the comparison needs the lists and sets of the call: with these inputs fp32 and fp64 scores rank the blocks alike
        kv = plan["kv_list"].tolist()
        assert kv == kv_g[0, h, :c["T_new"]].tolist() and plan["full_list"].tolist() == full_g[0, h, :c["n_full"]].tolist()
        for r, i in enumerate(flat_g[0, h, :c["n_flat"]]):
            ex = [kv[t] for t in range(c["T_new"]) if (mask_g[0, h, r, t >> 5] >> (t & 31)) & 1]
            assert ex == list(OB.exact_blocks_of(plan, int(i)))
        for name, got, want in zip(("dQ", "dK", "dV"), grads, OB.isa_attention_bwd(*x, plan)):
            d = np.abs(f64(got[0, h]) - want) / np.abs(want).max()
            assert d.max() <= TOL_MAX_REL and d.mean() <= TOL_MEAN_REL, (h, name, d.max(), d.mean())


# more than one round of long items and few key blocks: whole items and cut ones, with Taylor groups behind them and without
@pytest.mark.parametrize("H,src,ctx,full_frac", [(176, 500, 500, 0.6), (100, 2000, 300, 0.3), (44, 2000, 1000, 0.5), (100, 500, 100, 1.0), (70, 500, 500, 1.0)],
                         ids=["taylor_short", "taylor_13", "taylor_one_item", "long_only_5", "long_only_8"])
def test_last_round_of_short_lists(I, H, src, ctx, full_frac):
    from util import problem_of
    wl = _wl(H, (1, 1, src), (((1, 1, ctx),),), keep_ratio=1.0 if full_frac == 1.0 else 0.5, full_frac=full_frac, seed=905 + H)
    c = I.isa_get_counts(problem_of(wl), 0)
    n_long = -(-H * ((c["n_full"] + 1) // 2) // 8)
    assert n_long > 32 and 0 < n_long % 32 <= 16                                         # the premise
    check_end_to_end(I, wl, *gen(wl), heads=[0, H // 2, H - 2, H - 1])


# ragged batches: an equal range of every batch item's own pairs per XCD, the longest lists first, whatever the order of the items; heads
# that 8 does not divide, an item without long items, cut items of both lengths, more than a round
@pytest.mark.parametrize("lens", [(2000, 100, 1000), (100, 1000, 2000), (600, 900, 900)], ids=["longest_first", "longest_last", "two_alike"])
@pytest.mark.parametrize("H,full_frac", [(1, 0.4), (3, 0.0), (5, 1.0), (12, 0.3), (30, 0.6)])
def test_ragged_batches(I, lens, H, full_frac):
    src = (1, 1, 300)
    wl = _wl(H, src, tuple(((1, 1, n),) for n in lens), B=3, keep_ratio=0.7, full_frac=full_frac, exact_frac=0.2 if H == 12 else 0.0, seed=930 + H)
    check_end_to_end(I, wl, *gen(wl), heads=[0, H // 2, H - 1])


@pytest.mark.parametrize("lens", [(3000, 100, 1620), (100, 1620, 3000)], ids=["longest_first", "longest_last"])
@pytest.mark.parametrize("H", [1, 9, 14])
def test_ragged_dense(I, lens, H):
    import torch
    from oracle import isa_oracle as O
    from test_gpu_parity import TOL
    from util import err_stats, f64
    g = torch.Generator(device="cuda").manual_seed(940 + H)
    q, k, v = (torch.randn((3, H, 3000, 128), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    pr = I.Problem(H=H, D=128, dtype="bf16", block=128, seg_len=[[n] for n in lens], keep_ratio=1.0, full_frac=1.0)
    out = torch.full_like(q, float("nan"))
    I.isa_dense_attention(pr, q, k, v, out, I.new_workspace(pr))
    torch.cuda.synchronize()
    for b, n in enumerate(lens):
        assert torch.isfinite(out[b, :, :n]).all() and torch.isnan(out[b, :, n:]).all()
        for h in {0, H // 2, H - 1}:
            rows = slice(0, n, 7)
            emax, emean = err_stats(f64(out[b, h, :n][rows]), O.dense_attention(f64(q[b, h, :n][rows]), f64(k[b, h, :n]), f64(v[b, h, :n])))
            assert emax <= TOL["bf16"][0] and emean <= TOL["bf16"][1], (b, h, emax, emean)

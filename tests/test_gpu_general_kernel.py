"""The general matrix-core kernel (csrc/attn_gen.hip: fp32, D = 64, blocks of 64, and the pipelined kernels' shape when
they are switched off) at the sizes where its tiles, pairs and splits can go wrong, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import isa_oracle as O
from util import err_stats, f64, problem_of
from test_gpu_parity import TOL, check_end_to_end, gen

pytestmark = pytest.mark.gpu

SHAPES = [("bf16", 64, 64), ("bf16", 64, 128), ("bf16", 128, 64), ("f32", 64, 64), ("f32", 128, 128), ("f32", 64, 128)]
SHAPE_IDS = ["%s_d%d_b%d" % s for s in SHAPES]


@pytest.fixture(scope="module")
def I():
    import paper_2605_04569_amd as isa
    isa.lib()
    return isa


def _wl(shape, H, src, ctx, **kw):
    dtype, D, block = shape
    return W.CONFIGS["cfg1"].with_(name="general", H=H, D=D, dtype=dtype, block=block, src_grid=src, ctx_grids=ctx, **kw)


def _align(n):
    return (n + 255) // 256 * 256


def _bytes_without_parts(I, pr):
    """The workspace up to the end of its last array before the partial results: exact_mask, o_coarse or flat_list."""
    lay, T = I.isa_workspace_layout(pr), I.isa_get_counts(pr, 0)["T_max"]
    rows = pr.B * pr.H * T
    if pr.exact_frac > 0:
        return lay["exact_mask"] + _align(rows * ((T + 31) // 32) * 4)
    if pr.gamma != 0:
        return lay["o_coarse"] + _align(rows * pr.D * 4)
    return lay["flat_list"] + _align(rows * 4)


def _is_cut(I, pr, q, k, v):
    """Whether isa_attention runs long items in parts: without room for partial results they stay whole, and some sum then ends otherwise."""
    ws, outs = I.new_workspace(pr), [torch.zeros_like(q) for _ in range(2)]
    I.isa_attention(pr, q, k, v, outs[0], ws)
    I.isa_attention(pr, q, k, v, outs[1], ws[:_bytes_without_parts(I, pr)])
    torch.cuda.synchronize()
    return not torch.equal(*outs)


# tails of 1, 31, 32, 33, 63, 64 and 65 tokens: a tile's half, both halves, one past
@pytest.mark.parametrize("tail", [1, 31, 32, 33, 63, 64, 65])
@pytest.mark.parametrize("shape", SHAPES, ids=SHAPE_IDS)
def test_tails(I, shape, tail):
    wl = _wl(shape, 2, (1, 1, 256 + tail), (((1, 1, 128 + tail), (1, 1, tail)),), keep_ratio=0.7, full_frac=0.4,
             exact_frac=0.3 if tail % 2 else 0.0, gamma=0.5 if tail == 33 else 0.0, seed=700 + tail)
    check_end_to_end(I, wl, *gen(wl))


# enough heads for 128-row workgroups: odd lists (a pair with one block), exact sets of both blocks of a pair, a ragged batch
@pytest.mark.parametrize("exact_frac", [0.0, 0.25])
@pytest.mark.parametrize("shape", [s for s in SHAPES if s[0] == "bf16"], ids=[i for i in SHAPE_IDS if i[:4] == "bf16"])
def test_wide_workgroups(I, shape, exact_frac):
    dtype, D, block = shape
    src, ctx = (1, 1, 5 * block + 40), (((1, 1, 5 * block),), ((1, 1, 2 * block + 9),))
    wl = _wl(shape, 300, src, ctx, B=2, keep_ratio=0.6, full_frac=0.6, exact_frac=exact_frac, seed=731)
    n_full = [I.isa_get_counts(problem_of(wl), b)["n_full"] for b in range(2)]
    assert max(n_full) % 2 == 1 and 600 * (max(n_full) + 1) // 2 >= 448            # the premise: odd list, enough items
    check_end_to_end(I, wl, *gen(wl), heads=[0, 7, 150, 299])


# no long items at all: 128-row workgroups of Taylor blocks (64-row ones with exact sets at D = 64), the same odd lists
@pytest.mark.parametrize("exact_frac", [0.0, 0.25])
@pytest.mark.parametrize("shape", [s for s in SHAPES if s[0] == "bf16"], ids=[i for i in SHAPE_IDS if i[:4] == "bf16"])
def test_wide_workgroups_of_taylor_blocks(I, shape, exact_frac):
    dtype, D, block = shape
    wl = _wl(shape, 300, (1, 1, 5 * block + 40), (((1, 1, 4 * block + 9),), ((1, 1, 2 * block),)), B=2, keep_ratio=0.6, full_frac=0.0,
             exact_frac=exact_frac, seed=733)
    c = [I.isa_get_counts(problem_of(wl), b) for b in range(2)]
    assert c[0]["n_flat"] % 2 == 1 and c[0]["n_full"] == c[1]["n_full"] == 0 and 600 * (c[0]["n_flat"] // 2) >= 448       # the premise
    check_end_to_end(I, wl, *gen(wl), heads=[0, 7, 150, 299])


# 1, 2 and 3 tiles (fp32: 32 tokens each), token tiles followed by tiles of means
@pytest.mark.parametrize("tokens", [32, 33, 64, 65, 96])
@pytest.mark.parametrize("shape", SHAPES, ids=SHAPE_IDS)
def test_few_tiles(I, shape, tokens):
    wl = _wl(shape, 2, (1, 1, tokens), (((1, 1, 40),),), keep_ratio=1.0, full_frac=0.5, exact_frac=0.5, seed=740 + tokens)
    check_end_to_end(I, wl, *gen(wl))


# a long list with few long items (in parts) and with many: the same answers
@pytest.mark.parametrize("H", [2, 60])
@pytest.mark.parametrize("shape", SHAPES, ids=SHAPE_IDS)
def test_few_and_many_long_items(I, shape, H):
    wl = _wl(shape, H, (1, 1, 1500), (((1, 1, 900),),), keep_ratio=0.5, full_frac=0.5, exact_frac=0.2, gamma=0.5, seed=745 + H)
    check_end_to_end(I, wl, *gen(wl), heads=[0, H // 2, H - 1])


# few heads: long items in parts over key lists of 2 blocks (of 128 in fp32: one each), of 9 (unequal parts) and of 40; odd lists of blocks, a
# batch item with fewer of them, the residual added where the parts are
@pytest.mark.parametrize("blocks", [2, 9, 40])
@pytest.mark.parametrize("shape", SHAPES, ids=SHAPE_IDS)
def test_items_in_parts(I, shape, blocks):
    block = shape[2]
    wl = _wl(shape, 3, (1, 1, block * (blocks - 1) + 9), (((1, 1, 3 * block),), ((1, 1, block + 1),)), B=2, keep_ratio=0.0, full_frac=0.4,
             exact_frac=0.2 if blocks == 9 else 0.0, gamma=0.5, seed=752 + blocks)
    assert I.isa_get_counts(problem_of(wl), 0)["T_new"] == blocks
    inputs = gen(wl)
    check_end_to_end(I, wl, *inputs)
    whole = shape[0] == "bf16" and blocks == 2 or (shape, blocks) in ((SHAPES[0], 9), (SHAPES[3], 2))       # lists too short for parts to pay
    assert _is_cut(I, problem_of(wl), *inputs[3:]) == (not whole)


# about an item of 64 rows per compute unit, bf16: workgroups of two groups of waves; rows of the second pass in some; exact sets of Taylor
# blocks beside long items
@pytest.mark.parametrize("exact_frac,gamma", [(0.0, 0.0), (0.2, 0.5)])
@pytest.mark.parametrize("shape", [s for s in SHAPES if s[0] == "bf16"], ids=[i for i in SHAPE_IDS if i[:4] == "bf16"])
def test_two_groups(I, shape, exact_frac, gamma):
    wl = _wl(shape, 8, (1, 10, 99), (((1, 9, 110),),), keep_ratio=1.0, full_frac=1.0 if exact_frac == 0 else 0.9, exact_frac=exact_frac, gamma=gamma, seed=767)
    Q, K, V, q, k, v = gen(wl)
    check_end_to_end(I, wl, Q, K, V, q, k, v, heads=[0, 3, 7])
    if exact_frac == 0:
        # the premise: whole items, whose sums do not end as with one group of waves (enough heads to fill the chip with those)
        assert not _is_cut(I, problem_of(wl), q, k, v)
        many = [t[:, :1].expand(1, 70, -1, -1).contiguous() for t in (q, k, v)]
        outs = [torch.empty_like(q), torch.empty_like(many[0])]
        for x, out in zip(((q, k, v), many), outs):
            pr = problem_of(wl, H=x[0].shape[1])
            I.isa_attention(pr, *x, out, I.new_workspace(pr))
        torch.cuda.synchronize()
        assert not torch.equal(outs[0][:, 0], outs[1][:, 0]) and torch.equal(outs[1][:, 0], outs[1][:, 69])
    for t in (Q, q):                                    # scores beyond 2^24 in every 50th row: its workgroup starts again
        t[:, :, ::50] *= 2.0 ** 24
    out = torch.empty_like(q)
    pr = problem_of(wl)
    I.isa_dense_attention(pr, q, k, v, out, I.new_workspace(pr))
    torch.cuda.synchronize()
    rest = np.arange(wl.tokens(0)) % 50 != 0            # (in the others the largest of the bf16 scores decides, which rounding may change)
    for h in (0, 7):
        emax, emean = err_stats(f64(out[0, h])[rest], O.dense_attention(f64(Q[0, h]), f64(K[0, h]), f64(V[0, h]))[rest])
        assert emax <= TOL[wl.dtype][0] and emean <= TOL[wl.dtype][1], (h, emax, emean)
    assert torch.isfinite(out.float()).all()


# batch items with key lists of different length, the longest neither first nor last: parts of about one length, so that the longest list has
# the most and the shortest one part, whose item is stored whole; 8 batch items; a launch of whole items over the same XCDs' shares
@pytest.mark.parametrize("H,blocks,cut", [(3, (3, 30, 1, 12), True), (1, (9, 0, 4, 30, 2, 30, 17, 1), True), (70, (3, 12, 1), False)],
                         ids=["4_items", "8_items", "whole"])
@pytest.mark.parametrize("shape", SHAPES, ids=SHAPE_IDS)
def test_ragged_batches(I, shape, H, blocks, cut):
    block = shape[2]
    ctx = tuple(((1, 1, n * block + 7),) if n else () for n in blocks)
    wl = _wl(shape, H, (1, 1, 2 * block + 9), ctx, B=len(blocks), keep_ratio=0.8, full_frac=0.4, exact_frac=0.1 if H == 3 else 0.0,
             gamma=0.5 if H == 3 else 0.0, seed=763)
    assert len({I.isa_get_counts(problem_of(wl), b)["T_new"] for b in range(wl.B)}) > 2
    inputs = gen(wl)
    check_end_to_end(I, wl, *inputs, heads=sorted({0, H // 2, H - 1}))
    if cut:
        assert _is_cut(I, problem_of(wl), *inputs[3:])


@pytest.mark.parametrize("shape", SHAPES, ids=SHAPE_IDS)
def test_no_room_for_parts(I, shape):
    """A workspace that holds everything but the partial results (a slice of one that does) is accepted: the items stay whole."""
    wl = _wl(shape, 2, (1, 1, 1000), (((1, 1, 500),),), keep_ratio=0.5, full_frac=0.5, seed=757)
    Q, K, V, q, k, v = gen(wl)
    pr = problem_of(wl)
    ws = I.new_workspace(pr)
    least = _bytes_without_parts(I, pr)
    outs = [torch.empty_like(q) for _ in range(2)]
    for out, w in zip(outs, (ws, ws[:least])):
        I.isa_dense_attention(pr, q, k, v, out, w)
    with pytest.raises(I.IsaError):
        I.isa_dense_attention(pr, q, k, v, outs[0], ws[:least - 256])
    torch.cuda.synchronize()
    assert not torch.equal(*outs)                       # the first call did cut them: its sums end otherwise
    want = np.stack([O.dense_attention(f64(Q[0, h]), f64(K[0, h]), f64(V[0, h])) for h in range(2)])
    for out in outs:
        emax, emean = err_stats(f64(out[0]), want)
        assert emax <= TOL[wl.dtype][0] and emean <= TOL[wl.dtype][1], (emax, emean)


@pytest.mark.parametrize("exponent", [12, 25])
@pytest.mark.parametrize("shape", SHAPES, ids=SHAPE_IDS)
def test_parts_of_both_passes(I, shape, exponent):
    """Scores of up to 1e8 and 7e11 against the keys of one block and of 0 elsewhere: the part that holds the block goes through the second
    pass, the others do not, and their maxima meet in the sum.  Channel 0 only, every score exact in fp32: weights of 0 and 1."""
    block, n = shape[2], 12 * shape[2] + 5
    wl = _wl(shape, 2, (1, 1, n), ((),), seed=759)
    g = torch.Generator().manual_seed(wl.seed + exponent)
    Q, K = (torch.zeros((1, 2, n, wl.D), dtype=W.torch_dtype(wl.dtype)) for _ in range(2))
    V = torch.randn((1, 2, n, wl.D), generator=g).to(Q.dtype)
    assert _is_cut(I, problem_of(wl, keep_ratio=1.0, full_frac=1.0), *(V.cuda(),) * 3)
    Q[..., 0] = ((128 + torch.arange(n) % 128) * 2.0 ** exponent).to(Q.dtype)
    Q[:, :, ::3] *= -1
    Q[:, :, ::7] = 0                                    # these rows see all keys alike
    at = slice(5 * block + 3, 6 * block)
    K[:, :, at, 0] = torch.randint(-127, 128, (1, 2, block - 3), generator=g).to(K.dtype)
    out = torch.empty_like(Q, device="cuda")
    pr = problem_of(wl)
    I.isa_dense_attention(pr, Q.cuda(), K.cuda(), V.cuda(), out, I.new_workspace(pr))
    torch.cuda.synchronize()
    for h in range(2):
        emax, emean = err_stats(f64(out[0, h]), O.dense_attention(f64(Q[0, h]), f64(K[0, h]), f64(V[0, h])))
        assert emax <= TOL[wl.dtype][0] and emean <= TOL[wl.dtype][1], (h, emax, emean)


@pytest.mark.parametrize("shape", [s for s in SHAPES if s[0] == "bf16"], ids=[i for i in SHAPE_IDS if i[:4] == "bf16"])
def test_maxima_of_both_passes_on_one_scale(I, shape):
    """All scores of a row are 2^26 and a little (exact in fp32, 2^23 in the log2 domain): the keys of one block share the weight evenly with all others, and
    other rows of the workgroup send the part that holds the block through the second pass, whose maximum has another unit.  Values 1 and -1:
    with the two units off by 1e-8 from each other the result is off by a few per cent."""
    block, D = shape[2], shape[1]
    n = 24 * block
    wl = _wl(shape, 2, (1, 1, n), ((),), seed=765)
    g = torch.Generator().manual_seed(wl.seed)
    Q, K, V = (torch.zeros((1, 2, n, D), dtype=torch.bfloat16) for _ in range(3))
    at = slice(5 * block, 6 * block)
    K[..., 0] = 2.0 ** 13
    K[..., 1] = (8 * torch.randint(0, 4, (1, 2, n), generator=g)).bfloat16()
    K[:, :, at, 1] += 8 * round(np.log(23.0) * D ** 0.5 / 8)
    K[:, :, at, 2] = 2.0 ** 14
    Q[..., 0], Q[..., 1] = 2.0 ** 13, 1.0
    Q[:, :, 7::16] = 0
    Q[:, :, 7::16, 2] = 2.0 ** 14                       # 2^28 against the block, 0 against the others
    V[...], V[:, :, at] = -1.0, 1.0
    q, k, v = Q.cuda(), K.cuda(), V.cuda()
    pr = problem_of(wl)
    out = torch.empty_like(q)
    I.isa_dense_attention(pr, q, k, v, out, I.new_workspace(pr))
    torch.cuda.synchronize()
    for h in range(2):
        want = O.dense_attention(f64(Q[0, h]), f64(K[0, h]), f64(V[0, h]))
        assert np.abs(want[0]).max() < 0.5              # the premise: neither side has all the weight
        emax, _ = err_stats(f64(out[0, h]), want)       # the rounding of the result, 2^-9, and as much for the weights
        assert emax <= 2.0 ** -8, (h, emax)


@pytest.mark.parametrize("H", [1, 3, 5, 9, 20])
def test_head_counts_over_the_xcds(I, H):
    wl = _wl(("bf16", 64, 64), H, (2, 10, 33), (((1, 10, 33),),), keep_ratio=0.5, full_frac=0.4, seed=750 + H)
    check_end_to_end(I, wl, *gen(wl))


@pytest.mark.parametrize("shape", SHAPES, ids=SHAPE_IDS)
def test_no_further_from_64_bits_than_the_storage_type(I, shape):
    # fp32: a softmax average of unit values in fp32 sums of 500 terms, scores up to about 30: 30 * 2^-24 per weight; bf16: the
    # rounding of the result alone, uniform in half a step: 2^-9 / sqrt(3) of the value in the 2-norm, times 1.5
    wl = _wl(shape, 2, (1, 10, 33), (((1, 5, 33),),), seed=761)
    Q, K, V, q, k, v = gen(wl)
    pr = problem_of(wl)
    out = torch.empty_like(q)
    I.isa_dense_attention(pr, q, k, v, out, I.new_workspace(pr))
    torch.cuda.synchronize()
    want = np.stack([O.dense_attention(f64(Q[0, h]), f64(K[0, h]), f64(V[0, h])) for h in range(2)])
    rel = np.linalg.norm(f64(out[0]) - want) / np.linalg.norm(want)
    assert rel <= (30 * 2.0 ** -24 if shape[0] == "f32" else 1.5 * 2.0 ** -9 / 3 ** 0.5), rel


@pytest.mark.parametrize("shape", SHAPES, ids=SHAPE_IDS)
@pytest.mark.parametrize("H", [2, 520], ids=["narrow", "wide"])
def test_infinities_pass_as_in_plain_arithmetic(I, shape, H):
    wl = _wl(shape, H, (1, 1, 4 * shape[2] + 17), (((1, 1, shape[2]),),), keep_ratio=1.0, full_frac=0.5, seed=771)
    Q, K, V, q, k, v = gen(wl)
    n = wl.tokens(0)
    # moderate scores, so that no weight underflows; one +inf value in the last token of a short block (whose row the tile loads
    # repeat past the block's end), and one key that no query may see: channel 0 of every query is positive
    q, k = q * 0.25, k * 0.25
    q[..., 0] = q[..., 0].abs() + 0.125
    v[:, :, 4 * shape[2] + 16, 3] = float("inf")
    k[:, :, 5, 0] = float("-inf")
    pr = problem_of(wl)
    ws = I.new_workspace(pr)
    out = torch.empty_like(q)
    I.isa_dense_attention(pr, q, k, v, out, ws)
    torch.cuda.synchronize()
    tol_max, tol_mean = TOL[wl.dtype]
    for h in sorted({0, H - 1}):
        got, kk, vv = f64(out[0, h, :n]), f64(k[0, h, :n]), f64(v[0, h, :n])
        assert np.isposinf(got[:, 3]).all()
        seen = np.arange(n) != 5
        vv[:, 3] = 0.0
        want = O.dense_attention(f64(q[0, h, :n]), kk[seen], vv[seen])
        got[:, 3] = want[:, 3]
        emax, emean = err_stats(got, want)
        assert emax <= tol_max and emean <= tol_mean, (h, emax, emean)


# scores far outside the range in which a softmax weight is usually formed: around +-2e10 and 7e11 (a rounded maximum is off by
# more there than exp2 can express), and rows whose scores are all below -1e31.  Only channel 0 is used, with values that make every
# score exact in fp32; the weights are then 0 or 1 (shared evenly between keys that tie).
@pytest.mark.parametrize("exponent,negative", [(12, False), (20, False), (25, False), (90, True)], ids=["1e8", "2e10", "7e11", "below_-1e31"])
@pytest.mark.parametrize("H", [2, 520], ids=["narrow", "wide"])
@pytest.mark.parametrize("shape", SHAPES, ids=SHAPE_IDS)
def test_range_of_the_scores(I, shape, H, exponent, negative):
    block = shape[2]
    for exact_frac in (0.0, 0.4):
        wl = _wl(shape, H, (1, 1, 4 * block + 17), (((1, 1, block),),), keep_ratio=1.0, full_frac=0.0, exact_frac=exact_frac, seed=781)
        n = wl.tokens(0)
        g = torch.Generator().manual_seed(wl.seed + exponent)
        Q, K = (torch.zeros((1, H, n, wl.D), dtype=W.torch_dtype(wl.dtype)) for _ in range(2))
        V = torch.randn((1, H, n, wl.D), generator=g).to(Q.dtype)
        Q[..., 0] = ((128 + torch.arange(n) % 128) * 2.0 ** exponent).to(Q.dtype)
        K[..., 0] = (-torch.randint(64, 128, (1, H, n), generator=g) if negative else torch.randint(-127, 128, (1, H, n), generator=g)).to(K.dtype)
        if not negative:
            Q[:, :, ::3] *= -1
        q, k, v = Q.cuda(), K.cuda(), V.cuda()
        pr = problem_of(wl)
        ws = I.new_workspace(pr)
        out, dense = torch.empty_like(q), torch.empty_like(q)
        I.isa_attention(pr, q, k, v, out, ws)
        I.isa_dense_attention(pr, q, k, v, dense, ws)
        torch.cuda.synchronize()
        for h in sorted({0, H - 1}):
            Qh, Kh, Vh = f64(Q[0, h]), f64(K[0, h]), f64(V[0, h])
            want, _ = O.isa_attention(Qh, Kh, Vh, wl.seg_len(0), wl.block, 1.0, 0.0, exact_frac)
            for name, x, y in (("taylor", out, want), ("dense", dense, O.dense_attention(Qh, Kh, Vh))):
                emax, emean = err_stats(f64(x[0, h]), y)
                assert emax <= TOL[wl.dtype][0] and emean <= TOL[wl.dtype][1], (name, exact_frac, h, emax, emean)


@pytest.mark.parametrize("shape", SHAPES, ids=SHAPE_IDS)
def test_values_near_the_largest_number(I, shape):
    """Scores that rise slowly along the keys (by 7.5 powers of two in all, so that a maximum raised only in steps falls behind) beside
    values of 2^120: the sums of at most 20 such values of weight 1 are numbers, whatever weights the kernel forms."""
    n, D = 200, shape[1]
    wl = _wl(shape, 2, (1, 1, n), ((),), seed=791)
    Q, K = (torch.zeros((1, 2, n, D), dtype=W.torch_dtype(wl.dtype)) for _ in range(2))
    V = torch.randn((1, 2, n, D), generator=torch.Generator().manual_seed(wl.seed)).clamp(-4, 4).to(Q.dtype)
    Q[..., 0] = 1.0
    K[..., 0] = (7.5 * np.log(2.0) * D ** 0.5 * torch.arange(n) / n).to(K.dtype)
    q, k, v = Q.cuda(), K.cuda(), (V.double() * 2.0 ** 120).to(V.dtype).cuda()
    out = torch.empty_like(q)
    pr = problem_of(wl)
    I.isa_dense_attention(pr, q, k, v, out, I.new_workspace(pr))
    torch.cuda.synchronize()
    for h in range(2):
        emax, emean = err_stats(f64(out[0, h]) / 2.0 ** 120, O.dense_attention(f64(Q[0, h]), f64(K[0, h]), f64(V[0, h])))
        assert emax <= TOL[wl.dtype][0] and emean <= TOL[wl.dtype][1], (h, emax, emean)


@pytest.mark.parametrize("shape", [x for x in SHAPES if x[0] == "f32"], ids=[i for i in SHAPE_IDS if i[:3] == "f32"])
def test_values_near_the_smallest_normal_number(I, shape):
    """Values of 2^-126: the products with weights of at most 1 are multiples of 2^-149, and 300 of them are off by sqrt(300 / 12) such
    steps, 2^-18 of results of 2^-129.  Weights that carried a factor of 2^-8 would lose eight bits more."""
    n, D = 300, shape[1]
    g = torch.Generator().manual_seed(793)
    q, k, v = (torch.randn((1, 2, n, D), generator=g) for _ in range(3))
    v = (v.double() * 2.0 ** -126).float()
    pr = I.Problem(H=2, D=D, dtype="f32", block=shape[2], seg_len=[[n]], keep_ratio=1.0, full_frac=1.0)
    out = torch.empty((1, 2, n, D), device="cuda")
    I.isa_dense_attention(pr, q.cuda(), k.cuda(), v.cuda(), out, I.new_workspace(pr))
    torch.cuda.synchronize()
    want = np.stack([O.dense_attention(f64(q[0, h]), f64(k[0, h]), f64(v[0, h])) for h in range(2)])
    rel = np.linalg.norm(f64(out[0]) - want) / np.linalg.norm(want)
    assert rel <= 2.0 ** -18, rel


@pytest.mark.parametrize("D,bound", [(64, 1.14e-6), (128, 1.06e-6)])
def test_fp32_scores_no_further_off_than_in_scalar_arithmetic(I, D, bound):
    """Queries of norm up to 4 sqrt(D): the distance from 64 bits is that of the scores' sums.  The bounds are what a kernel with
    four partial sums per score, in scalar arithmetic, showed on the same inputs."""
    H, S = 8, 1000
    g = torch.Generator().manual_seed(797)
    q, k, v = (torch.randn((1, H, S, D), generator=g) for _ in range(3))
    q = q * (0.5 * 8.0 ** torch.rand((1, H, S, 1), generator=g))
    pr = I.Problem(H=H, D=D, dtype="f32", block=D, seg_len=[[S]], keep_ratio=1.0, full_frac=1.0)
    out = torch.empty((1, H, S, D), device="cuda")
    I.isa_dense_attention(pr, q.cuda(), k.cuda(), v.cuda(), out, I.new_workspace(pr))
    torch.cuda.synchronize()
    want = np.stack([O.dense_attention(f64(q[0, h]), f64(k[0, h]), f64(v[0, h])) for h in range(H)])
    rel = np.linalg.norm(f64(out[0]) - want) / np.linalg.norm(want)
    assert rel <= bound, rel


F32 = [x for x in SHAPES if x[0] == "f32"]
F32_IDS = [i for i in SHAPE_IDS if i[:3] == "f32"]


# Numbers whose 24 bits leave much behind the first 8: 1 + 2^-7 - r 2^-23
@pytest.mark.parametrize("H", [2, 300], ids=["narrow", "wide"])
@pytest.mark.parametrize("shape", F32, ids=F32_IDS)
def test_fp32_scores_of_one_channel(I, shape, H):
    """Every other key has such a number in one channel, the others 1 in it and the rest in a second, so that all scores of a row are alike (63 to
    127 in the log2 domain) and values of 1 and -1 cancel.  A score's sum is rounded once, by at most 2^-18, and the left-out terms are at most
    2^-24 of a power of two of up to 64: three times 2^-18 between the two kinds of key, ln 2 / 2 of that in the result."""
    D, n = shape[1], 300
    g = torch.Generator().manual_seed(803)
    q, k, v = (torch.zeros((1, H, n, D)) for _ in range(3))
    odd = torch.arange(n) % 2 == 1
    q[..., 0] = 44 * D ** 0.5 * (1 + 0.99 * torch.rand((1, H, n), generator=g))
    q[..., 1] = q[..., 0]
    r = torch.randint(1, 4096, (1, H, n // 2), generator=g) * 2.0 ** -23
    k[:, :, odd, 0], k[:, :, ~odd, 0] = 1 + 2.0 ** -7 - r, 1.0
    k[:, :, ~odd, 1] = 2.0 ** -7 - r
    v[:, :, odd], v[:, :, ~odd] = 1.0, -1.0
    pr = I.Problem(H=H, D=D, dtype="f32", block=shape[2], seg_len=[[n]], keep_ratio=1.0, full_frac=1.0)
    out = torch.empty((1, H, n, D), device="cuda")
    I.isa_dense_attention(pr, q.cuda(), k.cuda(), v.cuda(), out, I.new_workspace(pr))
    torch.cuda.synchronize()
    assert out.abs().max().item() <= 3 * 2.0 ** -18 * np.log(2.0) / 2


@pytest.mark.parametrize("H", [2, 300], ids=["narrow", "wide"])
@pytest.mark.parametrize("shape", F32, ids=F32_IDS)
def test_fp32_weighted_values_of_one_key(I, shape, H):
    """One key alone has values, 1 in channel 0 and such a number in channel 1: whatever its weights, the results have this ratio.  Off by the
    roundings of the sum and of both results and by the left-out terms, at most 2^-24 each; on average by nothing."""
    D, n = shape[1], 300
    g = torch.Generator().manual_seed(805)
    q, k = (torch.randn((1, H, n, D), generator=g) for _ in range(2))
    v = torch.zeros((1, H, n, D))
    v[:, :, 77, 0], v[:, :, 77, 1] = 1.0, 1 + 2.0 ** -7 - 2.0 ** -23
    pr = I.Problem(H=H, D=D, dtype="f32", block=shape[2], seg_len=[[n]], keep_ratio=1.0, full_frac=1.0)
    out = torch.empty((1, H, n, D), device="cuda")
    I.isa_dense_attention(pr, q.cuda(), k.cuda(), v.cuda(), out, I.new_workspace(pr))
    torch.cuda.synchronize()
    o = f64(out)
    off = o[..., 1] / o[..., 0] / v[0, 0, 77, 1].double().item() - 1
    assert abs(off.mean()) <= 2.0 ** -24, off.mean()
    assert np.abs(off).max() <= 4 * 2.0 ** -24, np.abs(off).max()


# fp32, enough heads for 128-row workgroups: odd lists of blocks (a pair with one), short blocks, exact sets of both blocks of a pair, a ragged
# batch; with full_frac 0 Taylor blocks alone
@pytest.mark.parametrize("full_frac,exact_frac", [(0.6, 0.0), (0.6, 0.25), (0.0, 0.0), (0.0, 0.25)])
@pytest.mark.parametrize("shape", F32, ids=F32_IDS)
def test_fp32_wide_workgroups(I, shape, full_frac, exact_frac):
    block = shape[2]
    wl = _wl(shape, 300, (1, 1, 5 * block + 40), (((1, 1, 4 * block + 9),), ((1, 1, 2 * block),)), B=2, keep_ratio=0.6, full_frac=full_frac,
             exact_frac=exact_frac, seed=801)
    check_end_to_end(I, wl, *gen(wl), heads=[0, 7, 150, 299])


@pytest.mark.parametrize("H", [2, 300], ids=["narrow", "wide"])
@pytest.mark.parametrize("shape", F32, ids=F32_IDS)
def test_fp32_largest_number(I, shape, H):
    """The largest number rounds to infinity in 8 bits: as a value, and as a key in a channel that no query has, it counts as in plain arithmetic."""
    D, n = shape[1], 200
    g = torch.Generator().manual_seed(810)
    q, k, v = (torch.randn((1, H, n, D), generator=g) for _ in range(3))
    top = torch.finfo(torch.float32).max
    q[..., 9], k[:, :, 70:, 9] = 0, -top
    v[:, :, 33, 3], v[:, :, 133, 4] = top, -top
    pr = I.Problem(H=H, D=D, dtype="f32", block=shape[2], seg_len=[[n]], keep_ratio=1.0, full_frac=1.0)
    out = torch.empty((1, H, n, D), device="cuda")
    I.isa_dense_attention(pr, q.cuda(), k.cuda(), v.cuda(), out, I.new_workspace(pr))
    torch.cuda.synchronize()
    for h in (0, H - 1):
        got, want = f64(out[0, h]), O.dense_attention(f64(q[0, h]), f64(k[0, h]), f64(v[0, h]))
        for at in ([3, 4], [c for c in range(D) if c not in (3, 4)]):      # (norms of numbers of 2^120 are numbers in 64 bits)
            rel = np.linalg.norm(got[:, at] - want[:, at]) / np.linalg.norm(want[:, at])
            assert rel <= 30 * 2.0 ** -24, (h, rel)


@pytest.mark.parametrize("full_frac", [1.0, 0.0], ids=["exact", "taylor"])
@pytest.mark.parametrize("tiny", ["k", "v"])
@pytest.mark.parametrize("H", [2, 300], ids=["narrow", "wide"])
@pytest.mark.parametrize("shape", F32, ids=F32_IDS)
def test_fp32_tiny_numbers_beside_ordinary_ones(I, shape, H, tiny, full_frac):
    """Numbers of 2^-120 whose terms lose bits where that cannot show: keys in a channel that no query has, single values in one channel.  The item
    is not run again on fp32 instructions, whose sums end otherwise: (the other channels of) the result have the bits they have beside zeros."""
    wl = _wl(shape, H, (1, 10, 33), (((1, 5, 33),),), keep_ratio=1.0, full_frac=full_frac, seed=808)
    n, g = wl.tokens(0), torch.Generator().manual_seed(809)
    q, k, v = (torch.randn((1, H, n, wl.D), generator=g).cuda() for _ in range(3))
    q[..., 5] = 0
    at = (slice(None), slice(None), slice(None), 5) if tiny == "k" else (slice(None), slice(None), slice(3, None, 64), 7)
    pr, outs = problem_of(wl), []
    for zero in (False, True):
        x = k if tiny == "k" else v
        x[at] = 0 if zero else torch.ldexp(1 + torch.rand(x[at].shape, generator=g), torch.tensor(-120)).cuda()
        outs.append(torch.empty_like(q))
        I.isa_attention(pr, q, k, v, outs[-1], I.new_workspace(pr))
    torch.cuda.synchronize()
    others = [c for c in range(wl.D) if tiny == "k" or c != 7]
    assert torch.equal(outs[0][..., others], outs[1][..., others])
    assert (outs[0] - outs[1]).abs().max().item() <= 2.0 ** -22


@pytest.mark.parametrize("full_frac", [1.0, 0.0], ids=["exact", "taylor"])
@pytest.mark.parametrize("small", ["q", "k", "v", "channel_of_v"])
@pytest.mark.parametrize("H", [2, 300], ids=["narrow", "wide"])
@pytest.mark.parametrize("shape", F32, ids=F32_IDS)
def test_fp32_numbers_whose_terms_lose_bits(I, shape, H, small, full_frac):
    """One tensor, or one channel of the values, of about 2^-120 (queries and keys beside the other at 2^120): the third bf16 term of such a number would
    end below 2^-133, the smallest bf16 number, so it has lost bits and the item has to be run without terms (in terms the results would be off by
    2e-5 to 4e-4).  Bound: as for numbers of about 1."""
    wl = _wl(shape, H, (1, 10, 33), (((1, 5, 33),),), keep_ratio=1.0, full_frac=full_frac, seed=807)
    g = torch.Generator().manual_seed(wl.seed)
    x = {n: torch.randn((1, H, wl.tokens(0), wl.D), generator=g) for n in "qkv"}
    scale = {"q": {"q": -120, "k": 120}, "k": {"q": 120, "k": -120}, "v": {"v": -120}, "channel_of_v": {}}[small]
    for n, e in scale.items():
        x[n] = torch.ldexp(x[n], torch.tensor(e))
    if small == "channel_of_v":
        x["v"][..., 7] = torch.ldexp(x["v"][..., 7], torch.tensor(-120))
    pr = problem_of(wl)
    q, k, v = (x[n].cuda() for n in "qkv")
    out = torch.empty_like(q)
    I.isa_attention(pr, q, k, v, out, I.new_workspace(pr))
    torch.cuda.synchronize()
    for h in sorted({0, H - 1}):
        got, want = f64(out[0, h]), O.isa_attention(f64(x["q"][0, h]), f64(x["k"][0, h]), f64(x["v"][0, h]), wl.seg_len(0), wl.block, 1.0, full_frac)[0]
        for at in (slice(None), slice(7, 8)):
            rel = np.linalg.norm(got[:, at] - want[:, at]) / np.linalg.norm(want[:, at])
            assert rel <= 30 * 2.0 ** -24, (h, rel)


@pytest.mark.parametrize("shape", F32, ids=F32_IDS)
def test_fp32_infinities_in_wide_workgroups(I, shape):
    """An infinite value in the last token of a short block makes its channel infinite and leaves the others as they are without it."""
    wl = _wl(shape, 300, (1, 1, 4 * shape[2] + 17), ((),), seed=811)
    g = torch.Generator().manual_seed(wl.seed)
    q, k, v = (torch.randn((1, 300, wl.tokens(0), wl.D), generator=g).cuda() for _ in range(3))
    pr = problem_of(wl)
    ws, outs = I.new_workspace(pr), [torch.empty_like(q) for _ in range(2)]
    for out in outs:
        I.isa_dense_attention(pr, q, k, v, out, ws)
        v[:, :, -1, 3] = float("inf")
    torch.cuda.synchronize()
    assert torch.isposinf(outs[1][..., 3]).all()
    others = [c for c in range(wl.D) if c != 3]
    diff = (outs[1][..., others] - outs[0][..., others]).norm() / outs[0][..., others].norm()
    assert diff <= 30 * 2.0 ** -24, diff


# bf16: a tile of 64 keys is weighed at once, its last keys masked (tails around its 32-key halves in every block), and fetched row by row where it is not
# full or where rows are 2^22 elements apart or more (a view of one head of many)
@pytest.mark.parametrize("tail", [1, 33, 47, 48, 63])
@pytest.mark.parametrize("shape", [s for s in SHAPES if s[2] == 64], ids=[i for i in SHAPE_IDS if i[-3:] == "b64"])
def test_full_and_ragged_tiles_of_one_list(I, shape, tail):
    wl = _wl(shape, 2, (1, 1, 192 + tail), (((1, 1, 64 + tail), (1, 1, 128), (1, 1, tail)),), keep_ratio=1.0, full_frac=0.5, seed=817 + tail)
    check_end_to_end(I, wl, *gen(wl))


# q, k, v and the result as a projection leaves them, [B, S, H, D]: a head's rows lie H D apart; 64- and 128-row workgroups, full and short tiles,
# exact sets, the residual, batch items that differ, dense
@pytest.mark.parametrize("H", [3, 150], ids=["narrow", "wide"])
@pytest.mark.parametrize("shape", SHAPES, ids=SHAPE_IDS)
def test_token_layout(I, shape, H):
    block = shape[2]
    wl = _wl(shape, H, (1, 1, 5 * block + 40), (((1, 1, 4 * block + 9),), ((1, 1, 2 * block),)), B=2, keep_ratio=0.6, full_frac=0.6, exact_frac=0.25,
             gamma=0.5, seed=821)
    x = gen(wl)[3:]
    xt = [t.transpose(1, 2).contiguous().transpose(1, 2) for t in x]
    assert xt[0].stride(2) == H * wl.D
    for f, pr in ((I.isa_attention, problem_of(wl)), (I.isa_attention, problem_of(wl, full_frac=0.0)), (I.isa_dense_attention, problem_of(wl))):
        out, out_t = torch.zeros_like(x[0]), torch.zeros_like(xt[0])
        f(pr, *x, out, I.new_workspace(pr))
        f(pr, *xt, out_t, I.new_workspace(pr))
        torch.cuda.synchronize()
        assert torch.equal(out, out_t) and out.abs().max() > 0


@pytest.mark.parametrize("stride", [2 ** 22 - 64, 2 ** 22])
@pytest.mark.parametrize("shape", SHAPES, ids=SHAPE_IDS)
def test_rows_far_apart(I, shape, stride):
    D, n = shape[1], 140
    wl = _wl(shape, 1, (1, 1, n), ((),), seed=823)
    g = torch.Generator().manual_seed(wl.seed)
    x = [torch.randn((1, 1, n, D), generator=g).to(W.torch_dtype(wl.dtype)) for _ in range(3)]
    far = torch.zeros((4, D + (n - 1) * stride), dtype=x[0].dtype, device="cuda").as_strided((4, 1, 1, n, D), (D + (n - 1) * stride, 8, 8, stride, 1))
    for i, t in enumerate(x):
        far[i].copy_(t)
    near = torch.empty((1, 1, n, D), dtype=x[0].dtype, device="cuda")
    kw = dict(H=1, D=D, dtype=shape[0], block=shape[2], seg_len=[[n]], keep_ratio=1.0, full_frac=1.0)
    pr = I.Problem(**kw)
    I.isa_dense_attention(pr, *(t.cuda() for t in x), near, I.new_workspace(pr))
    pr = I.Problem(**kw)
    I.isa_dense_attention(pr, far[0], far[1], far[2], far[3], I.new_workspace(pr))
    torch.cuda.synchronize()
    assert torch.equal(far[3], near)

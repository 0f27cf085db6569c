"""isa_select at the list lengths where the selection kernels change their shape (entries a lane holds, rounds of the rank
count), with ties, both zeros, infinities and NaN among the scores, against counting in numpy."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def I():
    import paper_2605_04569_amd as isa
    isa.lib()
    return isa


def _chosen(s, k):
    """Entries that fewer than k others beat (larger, or equal at a lower index): a NaN beats nothing and is beaten by nothing."""
    order = np.lexsort((np.arange(len(s)), -np.where(np.isnan(s), -np.inf, s)))
    order = order[~np.isnan(s[order])]
    out = np.isnan(s) if k > 0 else np.zeros(len(s), bool)
    out[order[:k]] = True
    return out


@pytest.mark.parametrize("T_src,T_ctx,keep,exact", [
    (1, 1, 1.0, 1.0), (63, 1, 1.0, 0.5), (100, 156, 1.0, 0.25), (128, 129, 0.5, 0.3), (256, 256, 0.125, 0.0625),
    (300, 213, 1.0, 0.1), (512, 512, 0.5, 0.0625), (600, 425, 1.0, 0.9), (1024, 1024, 0.75, 0.02), (1025, 1024, 1.0, 0.001),
    (2048, 2048, 1.0, 0.0625)])
def test_select_edges(I, T_src, T_ctx, keep, exact):
    H, T = 2, T_src + T_ctx
    pr = I.Problem(H=H, D=64, dtype="bf16", block=64, seg_len=[[64 * T_src, 64 * T_ctx]], keep_ratio=keep, full_frac=0.3, exact_frac=exact)
    c = I.isa_get_counts(pr, 0)
    assert c["T_max"] == T
    rng = np.random.default_rng(T)
    s_ctx = np.round(rng.random((1, H, T)) * 40).astype(np.float32)                     # many ties
    sharp = rng.random((1, H, T)).astype(np.float32)
    z = np.round(rng.standard_normal((1, H, T, T)) * 8).astype(np.float32)
    z[..., 0, :] = 0.0
    z[..., 0, ::2] = -0.0                                                               # one row of zeros of both signs: all tie
    z[..., 1 % T, :] = -np.inf
    z[0, 0, :, T // 2] = np.nan
    z[0, 1, :, T // 3] = np.inf
    dev = lambda x: torch.from_numpy(x).cuda()
    lists = [torch.full((1, H, T), -7, device="cuda", dtype=torch.int32) for _ in range(3)]
    words = (T + 31) // 32
    mask = torch.full((1, H, T, words), -1, device="cuda", dtype=torch.int32)
    I.isa_select(pr, dev(s_ctx), dev(sharp), dev(z), *lists, mask, I.new_workspace(pr))
    torch.cuda.synchronize()
    kv_g, full_g, flat_g = (x.cpu().numpy() for x in lists)
    mask_g = mask.cpu().numpy().view(np.uint32)
    for h in range(H):
        kv = np.concatenate([np.arange(T_src), T_src + np.flatnonzero(_chosen(s_ctx[0, h, :T_ctx], c["k_keep"]))])
        full = np.flatnonzero(_chosen(sharp[0, h], c["n_full"]))
        flat = np.setdiff1d(np.arange(T), full)
        for got, want in ((kv_g, kv), (full_g, full), (flat_g, flat)):
            assert (got[0, h, :len(want)] == want).all() and (got[0, h, len(want):] == -1).all()
        for r, i in enumerate(flat):
            bits = np.zeros(32 * words, bool)
            bits[:len(kv)] = _chosen(z[0, h, i, kv], c["k_exact"])
            want = np.packbits(bits, bitorder="little").view(np.uint32)
            assert (mask_g[0, h, r] == want).all(), (h, r, i)


# at most 64 blocks with exact sets, 44 without: pooled scores, lists, exact sets and gathered means in one launch, one block more: in separate ones; against the staged entry points
# (the general kernels) on the call's own block means, bit by bit.  Repeated blocks tie; one block of infinite keys and a ragged batch item.
@pytest.mark.parametrize("shape", [("bf16", 128, 128), ("bf16", 64, 64), ("f32", 128, 128)], ids=["bf16_d128_b128", "bf16_d64_b64", "f32_d128_b128"])
@pytest.mark.parametrize("T_src,T_ctx,keep,full,exact", [
    (1, 0, 1.0, 1.0, 0.0), (1, 1, 1.0, 0.5, 1.0), (15, 1, 1.0, 0.0, 0.5), (9, 8, 0.5, 0.3, 0.3), (1, 62, 0.5, 0.2, 0.1), (33, 31, 0.75, 0.25, 0.0625),
    (62, 2, 0.5, 0.4, 0.2), (33, 32, 0.5, 0.3, 0.1), (30, 14, 0.5, 0.3, 0.0), (30, 15, 0.5, 0.3, 0.0), (30, 19, 0.5, 0.3, 0.0)])
def test_one_launch_plan(I, shape, T_src, T_ctx, keep, full, exact):
    dtype, D, block = shape
    H, T = 3, T_src + T_ctx
    short = max(1, T_src // 2) * block - block // 3
    pr = I.Problem(H=H, D=D, dtype=dtype, block=block, seg_len=[[T_src * block - 5, T_ctx * block], [short]], keep_ratio=keep, full_frac=full, exact_frac=exact)
    c = [I.isa_get_counts(pr, b) for b in range(2)]
    assert c[0]["T"] == T
    S = T * block - 5
    g = torch.Generator(device="cuda").manual_seed(T)
    q, k, v = (torch.randn((2, H, S, D), generator=g, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32) for _ in range(3))
    if T_src > 4:                                       # blocks 1 and 3 alike (their scores tie), and infinite keys in one head's block 2
        for x in (q, k):
            x[:, :, 3 * block:4 * block] = x[:, :, block:2 * block]
        k[0, 1, 2 * block:3 * block, 0] = float("inf")
    ws = I.new_workspace(pr)
    out = torch.zeros_like(q)
    I.isa_attention(pr, q, k, v, out, ws)
    torch.cuda.synchronize()
    lay = I.isa_workspace_layout(pr)
    at = lambda name, dt, *more: I.workspace_array(ws, lay[name], (2, H, T) + more, dt).clone()
    qc, kc, vc = (at(n, torch.float32, D) for n in ("qc", "kc", "vc"))
    words = (T + 31) // 32
    names = ["s_ctx", "sharp", "kv_list", "full_list", "flat_list"]
    got = {n: at(n, torch.float32 if i < 2 else torch.int32) for i, n in enumerate(names)}
    if exact > 0:
        got["exact_mask"] = at("exact_mask", torch.int32, words)
    ws2 = I.new_workspace(pr)
    s_ctx, sharp = (torch.zeros((2, H, T), device="cuda") for _ in range(2))
    z = torch.zeros((2, H, T, T), device="cuda")
    lists = [torch.zeros((2, H, T), device="cuda", dtype=torch.int32) for _ in range(3)]
    mask = torch.zeros((2, H, T, words), device="cuda", dtype=torch.int32)
    I.isa_coarse_scores(pr, qc, kc, s_ctx, sharp, z, ws2)
    I.isa_select(pr, s_ctx, sharp, z, *lists, mask, ws2)
    torch.cuda.synchronize()
    want = dict(zip(names, [s_ctx, sharp, *lists]), exact_mask=mask)
    rows = {"s_ctx": "T_ctx", "sharp": "T", "exact_mask": "n_flat"}
    for n, x in got.items():
        for b in range(2):
            m = c[b][rows[n]] if n in rows else T
            a, w = x[b, :, :m], want[n][b, :, :m]
            assert torch.equal(torch.nan_to_num(a, nan=-7.0) if a.is_floating_point() else a, torch.nan_to_num(w, nan=-7.0) if w.is_floating_point() else w), (n, b)
    # the gathered means are seen in what the attention makes of them (with exact sets or not, whole Taylor rows of NaN among them)
    out2 = torch.zeros_like(q)
    I.isa_attend(pr, q, k, v, kc, vc, *lists, mask if exact > 0 else None, out2, ws2)
    torch.cuda.synchronize()
    assert torch.equal(torch.nan_to_num(out.float(), nan=-7.0), torch.nan_to_num(out2.float(), nan=-7.0))

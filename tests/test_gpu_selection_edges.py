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

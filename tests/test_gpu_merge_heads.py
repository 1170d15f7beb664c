"""The merge with a block per query head: slot counts around its rounds of 64 loads and 512 slots, empty sequences, windows
with and without a folded projection, at 1 to 8 query heads per KV head."""
import numpy as np
import pytest
import torch

from oracle import int2kv_oracle as O
from paper_2608_02691_amd import int2kv as K
from paper_2608_02691_amd import workloads as W

from _helpers import assert_rows_close, dev, gpu_cache

pytestmark = pytest.mark.gpu


def _random_cache(w, rng, G):
    """A cache of quantized N(0, 1) rows, packed by the library's own (bit-exact) packer."""
    n = w.num_blocks * 16
    rows = lambda: torch.from_numpy(rng.standard_normal((n, w.num_kv_heads, 128)).astype(np.float32)).cuda()
    cache = gpu_cache(O.new_pool(w.num_blocks, w.num_kv_heads, G))
    K.int2kv_quantize_pack_rotated(cache, rows(), rows(), torch.arange(n, dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    return cache, cache.pool.cpu().numpy()


# (lengths, query heads, KV heads): 64 pages per slot round at four pages a slot, 512 slots at one KV head
@pytest.mark.parametrize("case", [([16 * 4 * 64], 2, 1), ([16 * 4 * 65 + 3], 8, 1), ([34000], 1, 1), ([0, 40000, 5], 3, 1),
                                  ([0], 4, 2), ([700, 0, 90], 40, 5)], ids=str)
@pytest.mark.parametrize("window", [0, 96, 500])
@pytest.mark.parametrize("wo", ["none", "plain", "folded"])
def test_merge_per_query_head(case, window, wo):
    lens, Hq, H = case
    dm = 0 if wo == "none" else 64
    w = W.make_workload(1, batch=len(lens), ctx_lens=np.array(lens), num_q_heads=Hq, num_kv_heads=H, d_model=dm or None)
    rng = np.random.default_rng([len(lens), Hq, window])
    cache, pool = _random_cache(w, rng, 32) if w.num_blocks else (gpu_cache(O.new_pool(1, H)), O.new_pool(1, H))
    q, table, ctx, Rk, Rv = dev(w.q), dev(w.block_table), dev(w.ctx_lens), dev(w.R_k), dev(w.R_v)
    W_o, fmt = None, K.INT2KV_WO_PLAIN
    if wo == "plain":
        W_o = dev(w.W_o)
    elif wo == "folded":
        W_o, fmt = K.int2kv_prepare_wo(dev(w.W_o), Rv, Hq), K.INT2KV_WO_PREPARED_FOLDED
    kw = dict(W_o=W_o, wo_format=fmt, d_model=dm)
    ref_wo = w.W_o if dm else None
    if window:
        B = len(lens)
        wk, wv = (W.f32_to_bf16_bits(rng.standard_normal((B, window, H, 128)).astype(np.float32)) for _ in range(2))
        wl = rng.integers(0, window + 1, B).astype(np.int32)
        wl[0] = window
        out = K.int2kv_decode_window(cache, q, table, ctx, max(lens), Rk, Rv, dev(wk.reshape(-1, H, 128)),
                                     dev(wv.reshape(-1, H, 128)), dev(wl), window, **kw)
        ref = O.decode_window(pool, w.q, w.block_table, w.ctx_lens, w.R_k, w.R_v, wk, wv, wl, ref_wo)
    else:
        out = K.int2kv_decode(cache, q, table, ctx, max(lens), Rk, Rv, **kw)
        ref = O.decode(pool, w.q, w.block_table, w.ctx_lens, w.R_k, w.R_v, ref_wo)
    torch.cuda.synchronize()
    assert_rows_close(out.cpu().numpy(), ref, what=f"{case} {window} {wo}")


# (sequences, query heads, KV heads) on both sides of two and of one and a half blocks per CU at 256 CUs, at under and
# over 32 sequences (eight and four slots); one query head per KV head at any size
@pytest.mark.parametrize("B,Hq,H", [(128, 4, 1), (129, 4, 1), (16, 32, 8), (17, 32, 8), (12, 32, 4), (13, 32, 4), (31, 24, 3),
                                    (600, 1, 1), (70, 9, 9)])
@pytest.mark.parametrize("window", [0, 100])
@pytest.mark.parametrize("wo", ["none", "folded"])
def test_merge_block_counts(B, Hq, H, window, wo):
    rng = np.random.default_rng([B, Hq, window])
    lens = rng.integers(0, 60, B)
    lens[:2] = 0, 700
    dm = 0 if wo == "none" else 32
    w = W.make_workload(1, batch=B, ctx_lens=lens, num_q_heads=Hq, num_kv_heads=H, d_model=dm or None)
    cache, pool = _random_cache(w, rng, 128)
    args = (dev(w.q), dev(w.block_table), dev(w.ctx_lens), int(lens.max()), dev(w.R_k), dev(w.R_v))
    kw = {}
    if dm:
        kw = dict(W_o=K.int2kv_prepare_wo(dev(w.W_o), dev(w.R_v), Hq), wo_format=K.INT2KV_WO_PREPARED_FOLDED, d_model=dm)
    ref_wo = w.W_o if dm else None
    if window:
        wk, wv = (W.f32_to_bf16_bits(rng.standard_normal((B, window, H, 128)).astype(np.float32)) for _ in range(2))
        wl = rng.integers(0, window + 1, B).astype(np.int32)
        out = K.int2kv_decode_window(cache, *args, dev(wk.reshape(-1, H, 128)), dev(wv.reshape(-1, H, 128)), dev(wl),
                                     window, **kw)
        ref = O.decode_window(pool, w.q, w.block_table, w.ctx_lens, w.R_k, w.R_v, wk, wv, wl, ref_wo)
    else:
        out = K.int2kv_decode(cache, *args, **kw)
        ref = O.decode(pool, w.q, w.block_table, w.ctx_lens, w.R_k, w.R_v, ref_wo)
    torch.cuda.synchronize()
    assert_rows_close(out.cpu().numpy(), ref, what=f"{B} {Hq}/{H} {window} {wo}")


@pytest.mark.parametrize("B,Hq,H", [(3, 8, 4), (40, 32, 8)])  # a block per query head, per KV head
@pytest.mark.parametrize("window", [0, 40])
@pytest.mark.parametrize("what", ["v_zero_nan", "v_scale_inf", "q_nan", "q_inf"])
def test_merge_keeps_non_finite_values_to_their_heads(B, Hq, H, window, what):
    """A NaN or an infinity in one head's cached values reaches that head's outputs and no other's bits; one in a query
    changes no other query's output (beyond the rounding of the heads scanned together with it)."""
    rng = np.random.default_rng([B, window])
    w = W.make_workload(1, batch=B, ctx_lens=np.full(B, 300), num_q_heads=Hq, num_kv_heads=H, d_model=None)
    cache, _ = _random_cache(w, rng, 32)
    q = dev(w.q)
    win = [dev(W.f32_to_bf16_bits(rng.standard_normal((B * window, H, 128)).astype(np.float32))) for _ in range(2)]
    wl = torch.full((B,), window, dtype=torch.int32, device="cuda")

    def run():
        args = (cache, q, dev(w.block_table), dev(w.ctx_lens), 300, dev(w.R_k), dev(w.R_v))
        out = K.int2kv_decode_window(*args, *win, wl, window) if window else K.int2kv_decode(*args)
        return out.cpu().numpy().reshape(B, H, Hq // H, 128)

    clean = run()
    halves = cache.pool.view(torch.int16)[int(w.block_table[1, 2]), 0]  # KV head 0 of sequence 1, token 0 of a page
    if what == "v_zero_nan":
        halves[1408 // 2] = 0x7E00
    elif what == "v_scale_inf":
        halves[1280 // 2] = 0x7C00
    else:
        q.view(torch.bfloat16)[1, 0, 5] = float("nan" if what == "q_nan" else "inf")
    got = run()
    assert np.isfinite(clean).all()
    others = np.ones((B, H), bool)
    others[1, 0] = False
    assert np.array_equal(got[others], clean[others])
    if what[0] == "v":
        assert not np.isfinite(got[1, 0]).all(axis=-1).any()
    else:
        assert_rows_close(got[1, 0, 1:], clean[1, 0, 1:], what="the other queries of the KV head")

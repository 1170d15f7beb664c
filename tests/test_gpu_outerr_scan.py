"""The output-error scan's scores and statistics against the CPU oracle at fp32 precision: query heads that fill and part-fill the
quads of the score tiles, queries far from unit scale (the scan rescales them by powers of two) and one of zeros,
page and chunk edges."""
import numpy as np
import pytest
import torch

from oracle import int2kv_oracle as O
from paper_2608_02691_amd import int2kv as K
from paper_2608_02691_amd import workloads as W

from _helpers import dev, gpu_cache, oracle_pool
from test_gpu_outerr import _rows

pytestmark = pytest.mark.gpu

# A logit is an fp32 sum of 128 products: its error is a few 2^-24 of |q| |k| / sqrt(128), about 4e-7 for queries of unit
# scale and in proportion to it above. o is an average under the softmax and its error no larger than that of
# p, 1e-6 of ||o|| with the fp32 sums; dy is a difference of two of them, 10% of ||o|| or more for INT2. Factor 2 for
# the norm over W_O's rows.
ROW_RTOL = 2e-5
# A statistic is a square or product of two rows, summed: its error is that of the rows along each other, and over many
# (sequence, head) pairs it is typical and not worst: 2^-24 of |q| |k| / sqrt(128) a logit, 1e-6 of dy, once for each row.
# Scores with subnormal fp16 operands, whose products lose their leading zeros, give 2e-5.
STATS_RMS = 2e-6


# heads of one KV head, KV heads, context lengths, group, scale of the queries
@pytest.mark.parametrize("gq,H,lens,G,scale", [
    (1, 3, [17, 515], 32, 1.0), (2, 2, [16, 129], 128, 2.0 ** -6), (3, 2, [300, 511], 32, 1.0), (4, 2, [1025, 64], 128, 4.0),
    (6, 1, [513, 15], 32, 2.0 ** -6), (8, 1, [255, 700], 128, 1.0), (12, 1, [128, 1], 32, 1.0), (16, 1, [530, 31], 32, 4.0),
    # more chunks than the merge holds in flight, and more sequences than one 16-row tile of the projection
    (2, 1, [4700, 2100, 513], 32, 1.0), (1, 1, [40, 7, 520, 16, 33, 90, 1, 64, 17], 128, 1.0),
])
def test_output_error_scores_hold_fp32(gq, H, lens, G, scale):
    print(f"\n[output_error scores] gq={gq} H={H} lens={lens} G={G} scale={scale}", flush=True)
    lens = np.array(lens)
    w = W.make_workload(1, batch=len(lens), ctx_lens=lens, num_q_heads=gq * H, num_kv_heads=H, d_model=96)
    q = (torch.from_numpy(w.q.astype(np.int32)) << 16).view(torch.float32) * scale  # bf16 bits; powers of two
    q[0, 0] = 0.0
    q = (q.view(torch.int32) >> 16).numpy().astype(np.uint16)
    row_cap = int(lens.max())
    pool = oracle_pool(w, group=G)
    kr, vr, ks, vs = _rows(w, row_cap)
    dyK, dyV, ref_stats = O.output_error(pool, ks, vs, q, lens, w.block_table, w.R_k, w.R_v, w.mu, w.W_o)
    stats, dy = K.int2kv_output_error(gpu_cache(pool), dev(q), dev(w.block_table), dev(lens.astype(np.int32)), row_cap,
                                  dev(w.R_k), dev(w.R_v), dev(kr), dev(vr), row_cap, dev(w.W_o), want_dy=True)
    dy = dy.cpu().numpy().astype(np.float64)
    # against the larger of the two: a key error of nearly equal keys can vanish, its rounding does not
    norm = np.maximum(np.linalg.norm(dyK, axis=-1), np.linalg.norm(dyV, axis=-1))
    worst = max(float((np.linalg.norm(dy[:, :, i] - ref, axis=-1) / norm).max()) for i, ref in enumerate((dyK, dyV)))
    print(f"worst row error {worst:.2e}", flush=True)
    assert worst <= ROW_RTOL * max(1.0, scale)
    rel = np.abs(stats.cpu().numpy() - ref_stats) / (norm ** 2)[..., None]
    rms = float(np.sqrt((rel ** 2).mean()))
    print(f"statistics: rms error {rms:.2e}", flush=True)
    assert rms <= STATS_RMS * max(1.0, scale)


@pytest.mark.parametrize("gq,H", [(2, 2), (6, 2), (12, 1)])
@pytest.mark.parametrize("what", ["k_nan", "v_nan", "v_inf", "q_nan"])
def test_non_finite_rows_stay_with_their_heads(gq, H, what):
    """A NaN or an infinity in one sequence's rows of a KV head, or in a query, changes no other sequence's, KV head's or
    query's statistics; in the values it reaches every statistic of its own."""
    w = W.make_workload(1, batch=3, ctx_lens=np.array([300, 200, 40]), num_q_heads=gq * H, num_kv_heads=H, d_model=64)
    kr, vr, _, _ = _rows(w, 300)
    q, kr, vr = dev(w.q), dev(kr), dev(vr)
    cache = gpu_cache(oracle_pool(w))

    def run():
        stats, dy = K.int2kv_output_error(cache, q, dev(w.block_table), dev(w.ctx_lens), 300, dev(w.R_k), dev(w.R_v), kr,
                                          vr, 300, dev(w.W_o), want_dy=True)
        return stats.cpu().numpy().reshape(3, H, gq, 4), dy.cpu().numpy().reshape(3, H, gq, -1)

    clean = run()
    bad = float("inf" if what == "v_inf" else "nan")
    if what == "q_nan":
        q.view(torch.bfloat16)[1, 0, 5] = bad
    else:
        (kr if what == "k_nan" else vr).view(torch.bfloat16).reshape(3, 300, H, 128)[1, 77, 0, 5] = bad
    others = np.ones((3, H, gq), bool)
    others[1, 0, 0 if what == "q_nan" else slice(None)] = False
    for x, y in zip(run(), clean):
        assert np.isfinite(y).all() and np.array_equal(x[others], y[others])
        if what[0] == "v":
            assert not np.isfinite(x[1, 0]).all(axis=-1).any()

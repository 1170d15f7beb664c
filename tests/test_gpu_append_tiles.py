"""The cache write around the sizes where its arrangement changes: parts of a 32-token tile, one tile more than the
blocks of a head, the first size of the wide arrangement and a ragged one above it; skipped and shuffled slots; with
and without the reconstruction error, and RoPE at position 0 (the identity) against the same oracle rows."""
import numpy as np
import pytest
import torch

from oracle import int2kv_oracle as O
from paper_2608_02691_amd import int2kv as K
from paper_2608_02691_amd import workloads as W

from _helpers import compare_cache_writes, dev, gpu_cache

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G", [32, 128])
@pytest.mark.parametrize("n,H", [(1, 1), (31, 2), (32, 2), (33, 8), (65, 3), (1029, 8), (4096, 8), (4133, 8), (8229, 4)])
def test_append_sizes_match_oracle(n, H, G):
    print(f"\n[append tiles] n={n} H={H} G={G}", flush=True)
    w = W.make_workload(1, batch=1, ctx_lens=np.array([n]), num_q_heads=H, num_kv_heads=H, d_model=None)
    k, v = w.kv(0)
    rng = np.random.default_rng(n)
    slots = rng.permutation(w.num_blocks * 16)[:n].astype(np.int32)
    if n > 40:
        slots[rng.choice(n, n // 20, replace=False)] = -1
    clip = (0.96, 0.92) if G == 128 else (1.0, 1.0)
    keep = slots >= 0
    ref = O.new_pool(w.num_blocks, H, G)
    k_rot, v_rot, _ = O.quantize_append(ref, k[keep], v[keep], slots[keep], w.R_k, w.R_v, w.mu, *clip)
    mu_rk = K.int2kv_prepare_mu_rot(dev(w.R_k), dev(w.mu))
    pools = []
    for form in ("plain", "error", "rope"):
        cache = gpu_cache(O.new_pool(w.num_blocks, H, G))
        args = (cache, dev(k), dev(v), dev(slots))
        if form == "plain":
            K.int2kv_quantize_append(*args, dev(w.R_k), dev(w.R_v), mu_rk, *clip)
        elif form == "error":
            K.int2kv_quantize_append_error(*args, dev(w.R_k), dev(w.R_v), mu_rk, *clip)
        else:
            cs = torch.cat([torch.ones(1, 64), torch.zeros(1, 64)], 1).cuda()
            K.int2kv_quantize_append_rope(*args, torch.zeros(n, dtype=torch.int32, device="cuda"), cs, dev(w.R_k),
                                          dev(w.R_v), mu_rk, *clip)
        torch.cuda.synchronize()
        pool = cache.pool.cpu().numpy()
        print(form, compare_cache_writes(pool, ref, slots[keep], k_rot, v_rot)["fraction"], flush=True)
        untouched = np.setdiff1d(np.arange(w.num_blocks * 16), slots[keep])
        codes = pool[:, :, :512].reshape(w.num_blocks, H, 16, 32).transpose(0, 2, 1, 3).reshape(-1, H, 32)
        assert not codes[untouched].any(), "rows no slot names stay as they were"
        pools.append(pool)
    assert np.array_equal(pools[0], pools[1]), "the error-reporting write stores the same bytes"

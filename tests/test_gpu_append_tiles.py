"""The cache write around the sizes where its arrangement changes: parts of a 32-token tile, one tile more than the
blocks of a head, the first size of the wide arrangement and a ragged one above it, few and many heads; skipped and
shuffled slots; with and without the reconstruction error, RoPE at position 0 (the identity) against the same oracle
rows, the Hadamard rotation of keys, values or both, and RoPE at differing positions over several tiles a block."""
import numpy as np
import pytest
import torch

from oracle import int2kv_oracle as O
from paper_2608_02691_amd import int2kv as K
from paper_2608_02691_amd import workloads as W

from _helpers import compare_cache_writes, dev, gpu_cache, slot_bytes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G", [32, 128])
@pytest.mark.parametrize("n,H", [(1, 1), (31, 2), (32, 2), (33, 8), (65, 3), (1029, 8), (4096, 8), (4133, 8), (8229, 4),
                                 (513, 8), (2049, 8), (3105, 8), (1313, 16), (300, 24), (257, 32), (513, 32), (770, 32), (120, 64),
                                 (40, 128)])
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
        assert not slot_bytes(pool)[untouched].any(), "rows no slot names stay as they were"
        pools.append(pool)
    assert np.array_equal(pools[0], pools[1]), "the error-reporting write stores the same bytes"


def _write(n, H, G, rng, had, rope):
    """One write of n shuffled slots (some skipped) against the oracle's, with the Hadamard rotation where `had` says."""
    w = W.make_workload(1, batch=1, ctx_lens=np.array([n]), num_q_heads=H, num_kv_heads=H, d_model=None)
    k, v = w.kv(0)
    mu = w.mu
    if rope:
        # The workload's key offsets (up to 30) would stay in the keys, since mu cannot follow them through RoPE: then a
        # group's least value can be of 1e-4, where the fp32 sum's error (2^-24 of 128 products of size 30 / sqrt(128), 1e-6
        # and more) is several fp16 ulps (1e-7). The least of 32 N(0, 1) values is about -2: an ulp of 1e-3.
        k = W.f32_to_bf16_bits(rng.standard_normal((n, H, 128)).astype(np.float32))
        mu = (0.1 * rng.standard_normal((H, 128))).astype(np.float32)
    slots = rng.permutation(w.num_blocks * 16)[:n].astype(np.int32)
    slots[rng.choice(n, n // 20, replace=False)] = -1
    Hd, Hn = K.hadamard_rotation(H), np.broadcast_to(O.hadamard(128), (H, 128, 128)).copy()
    R_k, R_v = (Hn if had & 1 else w.R_k), (Hn if had & 2 else w.R_v)
    mu_rk = K.int2kv_prepare_mu_rot(Hd if had & 1 else dev(w.R_k), dev(mu))
    keep, pos, cs, out, ref_k = slots >= 0, None, None, None, k
    if rope:
        cs = W.rope_cos_sin(5000)
        pos = rng.integers(0, 5000, n).astype(np.int32)
        pos[rng.choice(n, n // 20, replace=False)] = rng.choice([-1, 5000, 2**31 - 1], n // 20)
        inside = (pos >= 0) & (pos < 5000)
        keep &= inside
        ref_k = O.rope(k, np.where(inside, pos, 0), cs)
        out = torch.full((n, H, 128), 0x1234, dtype=torch.int16, device="cuda")
    ref = O.new_pool(w.num_blocks, H, G)
    k_rot, v_rot, _ = O.quantize_append(ref, ref_k[keep], v[keep], slots[keep], R_k, R_v, mu)
    cache = gpu_cache(O.new_pool(w.num_blocks, H, G))
    K.int2kv_quantize_append_rope(cache, dev(k), dev(v), dev(slots), dev(pos) if rope else None, dev(cs) if rope else None,
                                  None if had & 1 else dev(w.R_k), None if had & 2 else dev(w.R_v), mu_rk, flags=had,
                                  k_rope_out=out)
    pool = cache.pool.cpu().numpy()
    print(compare_cache_writes(pool, ref, slots[keep], k_rot, v_rot)["fraction"], flush=True)
    untouched = np.setdiff1d(np.arange(w.num_blocks * 16), slots[keep])
    assert not slot_bytes(pool)[untouched].any(), "rows no slot names stay as they were"
    if rope:
        got = out.cpu().numpy().view(np.uint16)
        assert np.array_equal(got[inside], ref_k[inside]), "post-RoPE keys must be bit-exact"
        assert np.all(got[~inside] == 0x1234), "skipped tokens leave k_rope_out untouched"


@pytest.mark.parametrize("G", [32, 128])
@pytest.mark.parametrize("had", [1, 2, 3])
@pytest.mark.parametrize("n,H", [(1029, 8), (4133, 8), (8229, 4)])
def test_hadamard_sizes_match_oracle(n, H, had, G):
    print(f"\n[append tiles] hadamard={had} n={n} H={H} G={G}", flush=True)
    _write(n, H, G, np.random.default_rng([n, had, G]), had, rope=False)


# 97, 194 and 22 tiles on 32, 64 and 8 blocks a head: three and four tiles in turn
@pytest.mark.parametrize("G", [32, 128])
@pytest.mark.parametrize("had", [0, 3])
@pytest.mark.parametrize("n,H", [(3100, 8), (6200, 4), (700, 32)])
def test_rope_positions_over_many_tiles(n, H, had, G):
    print(f"\n[append tiles] rope hadamard={had} n={n} H={H} G={G}", flush=True)
    _write(n, H, G, np.random.default_rng([n, had, G, 1]), had, rope=True)

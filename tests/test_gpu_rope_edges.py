"""Post-RoPE keys bit for bit where fp32 bounds on a result cannot settle its rounding to bf16: exact ties and values a
hair beside them, cancellation of the two products, signed zeros, subnormal and very small results, huge and infinite
ones. Table entries are free fp32 values here (not cosines), to reach those cases."""
import numpy as np
import pytest
import torch

from oracle import int2kv_oracle as O
from paper_2608_02691_amd import int2kv as K
from paper_2608_02691_amd import workloads as W

from _helpers import dev, slot_bytes

pytestmark = pytest.mark.gpu


def _table(kind, rng, rows):
    c, s = rng.standard_normal((2, rows, 64)).astype(np.float32)
    if kind == "ties":  # x c lands on, just below and just above the midpoint of two bf16 values
        ulp = np.float32(2.0 ** -23)
        c = (1.0 + 2.0 ** -8 * (2 * rng.integers(0, 64, c.shape) + 1)).astype(np.float32)
        c += ulp * rng.integers(-2, 3, c.shape).astype(np.float32)
        s = np.where(rng.random(s.shape) < 0.5, 0.0, s * 2.0 ** -30).astype(np.float32)
    elif kind == "cancel":
        s = (c * (1 + rng.integers(-3, 4, c.shape) * 2.0 ** -23)).astype(np.float32)
    elif kind == "tiny":
        c, s = c * np.float32(2.0 ** -100), s * np.float32(2.0 ** -110)
    elif kind == "huge":
        c, s = c * np.float32(2.0 ** 120), s * np.float32(2.0 ** 121)
    return np.concatenate([c, s], axis=1).astype(np.float32)


@pytest.mark.parametrize("kind", ["plain", "ties", "cancel", "tiny", "huge"])
@pytest.mark.parametrize("n", [1, 40, 300])
def test_rope_rounding_edges(kind, n):
    H = 2
    rng = np.random.default_rng([n, len(kind)])
    x = rng.standard_normal((n, H, 128)).astype(np.float32)
    if kind in ("ties", "cancel"):
        x = np.sign(x) * np.exp2(rng.integers(-3, 4, x.shape)).astype(np.float32)  # powers of two keep c's bits
    if kind == "cancel":
        x[..., 64:] = x[..., :64]
    if kind == "tiny":
        x *= np.exp2(rng.integers(-28, 0, x.shape)).astype(np.float32)
    x[rng.random(x.shape) < 0.02] = 0.0
    x[rng.random(x.shape) < 0.01] = -0.0
    k = W.f32_to_bf16_bits(x)
    v = W.f32_to_bf16_bits(rng.standard_normal((n, H, 128)).astype(np.float32))
    cs = _table(kind, rng, 64)
    pos = rng.integers(0, 64, n).astype(np.int32)
    cache = K.Int2KVCache((n + 15) // 16, H)
    R = K.hadamard_rotation(H)
    mu_rk = torch.zeros((H, 128), dtype=torch.float32, device="cuda")
    out = torch.zeros((n, H, 128), dtype=torch.int16, device="cuda")
    K.int2kv_quantize_append_rope(cache, dev(k), dev(v), dev(np.arange(n, dtype=np.int32)), dev(pos), dev(cs), R, R,
                                  mu_rk, k_rope_out=out)
    got = out.cpu().numpy().view(np.uint16)
    with np.errstate(over="ignore"):
        ref = O.rope(k, pos, cs)
    assert np.array_equal(got, ref), (kind, np.argwhere(got != ref)[:3])


# 40 tokens: one tile and a part; 3,100 at 8 heads: several tiles of 32 per work-group on any count of CUs up to 384
@pytest.mark.parametrize("G", [32, 128])
@pytest.mark.parametrize("had", [0, 1, 2, 3])
@pytest.mark.parametrize("n,H", [(40, 2), (3100, 8)])
def test_skipped_positions_leave_their_rows(n, H, had, G):
    """A token whose position lies outside the table writes nothing, key or value: the call stores what it would store
    with that token's slot at -1, over a cache that held other bytes."""
    print(f"\n[rope skip] n={n} H={H} hadamard={had} G={G}", flush=True)
    rng = np.random.default_rng([n, had, G])
    bits = lambda *s: W.f32_to_bf16_bits(rng.standard_normal(s).astype(np.float32))
    k, v, P = bits(n, H, 128), bits(n, H, 128), 512
    blocks = (n + 15) // 16 + 1
    slots = rng.permutation(blocks * 16)[:n].astype(np.int32)
    pos = rng.integers(0, P, n).astype(np.int32)
    bad = rng.random(n) < 0.2
    bad[[0, n - 1]] = True
    pos[bad] = rng.choice([-1, -2**31, P, P + 7, 2**31 - 1], int(bad.sum()))
    R = K.hadamard_rotation(H)
    mu_rk = torch.zeros((H, 128), dtype=torch.float32, device="cuda")
    before = rng.integers(0, 256, (blocks, H, K.RECORD_BYTES_BY_GROUP[G]), dtype=np.uint8)
    pools = []
    for sl, ps in ((slots, pos), (np.where(bad, -1, slots).astype(np.int32), np.where(bad, 0, pos).astype(np.int32))):
        cache = K.Int2KVCache(blocks, H, pool=torch.from_numpy(before.copy()).cuda(), group_size=G)
        K.int2kv_quantize_append_rope(cache, dev(k), dev(v), dev(sl), dev(ps), dev(W.rope_cos_sin(P)), R, R, mu_rk,
                                      flags=had)
        pools.append(cache.pool.cpu().numpy())
    same = slot_bytes(pools[0]) == slot_bytes(before)
    unnamed = np.ones(blocks * 16, bool)
    unnamed[slots[~bad]] = False
    assert same[unnamed].all(), "rows of skipped tokens and of no token stay as they were"
    assert not same[~unnamed].all(axis=-1).any(), "every other row is written"
    assert np.array_equal(pools[0], pools[1])

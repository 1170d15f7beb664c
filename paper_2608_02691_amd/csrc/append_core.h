// Append on the matrix cores (shared by the append kernel and the decode's preparation kernel).
#pragma once
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace int2kv {

// The cache write of one (KV head, K or V): x R (x bf16 [n, H, 128], R fp32 [128, 128]) as bf16 MFMA with R
// split into three bf16 terms by truncation (R = t0 + t1 + t2 exactly: t0 and t1 take the leading 8 significant
// bits of R and of R - t0, the remainder has at most 8 left; every product is exact in fp32), an fp32
// accumulation starting from - mu R_K for keys, smallest term first; then the group quantizer and the packed
// stores.
//
// A work-group has four waves and takes 32-token tiles. Wave g owns the 32 output channels of group g: its
// share of R^T, 32 channels x 128 x 3 terms, stays in registers (96 per lane) as the A operand of
// 32 x 32 x 16 products, so a work-group starts in a few microseconds (no R^T to stage) and the LDS traffic of a
// tile is its 8 KiB of tokens, read once by each wave. D^T[row][token]: lane (token t = l % 32, hf = l / 32)
// holds rows 8 a + 4 hf + b in register 4 a + b. R^T's rows are permuted so that row 8 a + 4 hf + b is
// channel 16 (a / 2) + 8 hf + 4 (a % 2) + b of the group: a lane's 16 values are then both 2-bit codes
// (positions 2 g, 2 g + 1) of the packed halves 8 hf .. 8 hf + 7, one 32-bit word of nibbles, and a group's
// extremes need one exchange with lane l ^ 32. The four waves' nibble words meet in LDS and a later step
// interleaves and stores them (32 contiguous bytes of key codes per token).
//
// Step i: packed stores of tile i - 2, loads of a later tile, products of tile i beside the quantizer of
// tile i - 1, one barrier. Tiles come by LDS-DMA, kApStages - 1 ahead; with RoPE through registers, since thread
// (token, channels 8 j .. 8 j + 7 and 64 + 8 j ..) holds whole rotate-half pairs and contiguous pieces of the row, of
// the table and of the post-RoPE output. Matrix cores and vector ALU (about 220 instructions per tile and
// wave, 80 of them the quantizer's) add up rather than overlap, also when alternated in one wave; long dense
// prompts therefore use the arrangement of append_wide.h.
//
// Us a call at 8 KV heads, against sixteen 16-token tiles per eight-wave work-group with R^T in LDS: RoPE,
// 32,768 tokens 91 -> 75; RoPE and Hadamard, 16,384 tokens 44.4 -> 33; RoPE, G = 128, 2,011 tokens 11.3 ->
// 10.6; one decode step (32/8 heads, 1,011 tokens), whose first launch carries the write, 30.5 -> 28.8.
typedef __bf16 ap_bf16x8_t __attribute__((ext_vector_type(8)));
typedef float ap_f16_t __attribute__((ext_vector_type(16)));
typedef uint32_t ap_u4_t __attribute__((ext_vector_type(4)));

constexpr int kApTok = 32;       // tokens per tile
constexpr int kApThreads = 256;  // four waves, one per 32-channel group
#ifndef INT2KV_AP_DEPTH
#define INT2KV_AP_DEPTH 2
#endif
constexpr int kApDepth = INT2KV_AP_DEPTH;  // tiles in flight in registers

// LDS of one append work-group
#ifndef INT2KV_AP_STAGES
#define INT2KV_AP_STAGES 4
#endif
constexpr int kApStages = INT2KV_AP_STAGES;  // tiles staged by LDS-DMA
struct ApLds {
  __attribute__((aligned(16))) uint8_t x[kApStages][kApTok * 256];  // tile rows, 16-byte piece q at q ^ (token % 16)
  __attribute__((aligned(16))) int slot[kApStages][kApThreads];     // each thread's slot (token tid / 8)
  __attribute__((aligned(16))) uint32_t words[2][kApTok][2][4];  // nibble words [token][hf][group]
  __attribute__((aligned(16))) uint32_t meta[2][kApTok][4];      // scale | zero << 16 per group
  float err[2][kApTok][4];                                       // squared reconstruction errors
  float ext[kApTok][4][2];                                       // extremes per 32 channels (one group per token)
  __attribute__((aligned(16))) float sub[kHeadDim];              // - mu R_K (keys), 0 (values)
  float recip[1024];                                             // RN(1 / (1 + m / 1024))
};
constexpr int kApPos = kApStages * kApThreads;  // ints of the staged positions, laid out as ApLds::slot
constexpr int kAppendLdsBytes = sizeof(ApLds);

// x / 3 correctly rounded, as a product with RN(1/3) and one FMA correction: checked against the
// correctly rounded quotient for every fp32 significand (so for every x whose intermediate values
// stay normal: x == 0 or x >= 2^-100).
__device__ __forceinline__ float div3_rn(float x) {
#pragma clang fp contract(off)
  const float c = 0x1.555556p-2f;  // RN(1/3)
  const float q0 = x * c;
  const float r = __builtin_fmaf(-q0, 3.0f, x);
  return __builtin_fmaf(r, c, q0);
}

// The quantizer's group parameters (bit-identical to int2_group_params), without branches: s = fp16((mx - mn) / 3)
// with the division above (below 2^-100 its value does not matter: fp16 rounds it to zero), and 1/s from a
// table of the correctly rounded reciprocals of 1 + m / 1024: s has at most 11 significant bits, so its fp32
// form (normalized, also for subnormal s) is (1 + m / 1024) 2^e and the scaling by 2^-e is exact. Zero,
// infinite and NaN scales have no reciprocal (0: 1/inf, and by definition for s = 0).
__device__ __forceinline__ void int2_group_params_fast(float mn, float mx, float clip, const float* recip_tab,
                                                       uint32_t& s_bits, uint32_t& z_bits, float& zf, float& inv) {
#pragma clang fp contract(off)
  mn = clip != 1.0f ? clip * mn : mn;
  mx = clip != 1.0f ? clip * mx : mx;
  const __half s = __float2half_rn(div3_rn(mx - mn));
  const __half z = __float2half_rn(mn);
  s_bits = __half_as_ushort(s);
  z_bits = __half_as_ushort(z);
  zf = __half2float(z);
  const float sf = __half2float(s);
  const uint32_t u = __float_as_uint(sf);
  const float r = __builtin_ldexpf(recip_tab[(u >> 13) & 1023u], 127 - (int)(u >> 23));
  inv = sf > 0.0f && sf < INFINITY ? r : 0.0f;
}

// Cross-lane exchanges of the group reductions on the vector ALU (no LDS round trip).
// lane_swap32(a, b): lanes 32-63 of a trade places with lanes 0-31 of b, so afterwards lane l < 32
// holds (a[l], a[l + 32]) and lane l >= 32 holds (b[l - 32], b[l]).
struct LanePair {
  float a, b;
};
__device__ __forceinline__ LanePair lane_swap32(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return LanePair{__uint_as_float(r[0]), __uint_as_float(r[1])};
}
// Quantizer parameters and codes of one tile: v[4 a + b] as above; returns the nibble word and the packed
// (scale, zero) of the lane's group, e = the token's squared error over the group (both lanes).
struct ApOut {
  uint32_t word, meta;
  float err;
};
template <bool ERR>
__device__ __forceinline__ ApOut quantize_group(const ap_f16_t& v, float mn, float mx, float clip,
                                                const float* recip_tab) {
  uint32_t s_bits, z_bits;
  float zf, inv;
  int2_group_params_fast(mn, mx, clip, recip_tab, s_bits, z_bits, zf, inv);
  const float sf = __half2float(__ushort_as_half((unsigned short)s_bits));
  // v_cvt_pk_u8_f32 rounds to nearest even into a byte: value (a, b), bits 8 (2 (a % 2) + b / 2) + 4 (b % 2) +
  // 2 (a / 2) of the word, goes to that byte of d[2 (b % 2) + a / 2], and the four words are shifted together
  uint32_t d[4] = {0u, 0u, 0u, 0u};
  float e = 0.0f;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
#pragma clang fp contract(off)
      const float x = v[4 * a + b];
      const float t = __builtin_amdgcn_fmed3f((x - zf) * inv, 0.0f, 3.0f);
      uint32_t& w = d[2 * (b & 1) + (a >> 1)];
      w = __builtin_amdgcn_cvt_pk_u8_f32(t, 2 * (a & 1) + (b >> 1), w);
      if constexpr (ERR) {
        const float r = x - __builtin_fmaf(__builtin_rintf(t), sf, zf);
        e = __builtin_fmaf(r, r, e);
      }
    }
  if constexpr (ERR) {
    const LanePair p = lane_swap32(e, e);
    e = p.a + p.b;
  }
  return ApOut{(d[0] | (d[1] << 2)) | ((d[2] | (d[3] << 2)) << 4), s_bits | (z_bits << 16), e};
}

// extremes of a lane's 16 values and its partner's (lane ^ 32), NaN-propagating as the oracle's
__device__ __forceinline__ void ap_extremes(const ap_f16_t& v, float& mn, float& mx) {
  mn = mx = v[0];
#pragma unroll
  for (int r = 1; r < 16; ++r) {
    mn = __builtin_elementwise_minimum(mn, v[r]);
    mx = __builtin_elementwise_maximum(mx, v[r]);
  }
  const LanePair n = lane_swap32(mn, mn), x = lane_swap32(mx, mx);
  mn = __builtin_elementwise_minimum(n.a, n.b);
  mx = __builtin_elementwise_maximum(x.a, x.b);
}

// Optional stages of the cache write. RoPE (with ROPE): the keys arrive pre-RoPE and each token is
// turned at its position into its post-RoPE bf16 row first (rotate-half pairs (i, i + 64); each
// output evaluated in fp64, where both products are exact, and rounded once to bf16), optionally
// stored to k_out. Hadamard (bit 0 of had for keys, bit 1 for values): the rotation is
// H_128 / sqrt(128) instead of R; its +-1 entries are exact bf16 operands, so one matrix-core pass
// replaces the three-term split, and the fp32 sum is scaled by RN(2^-3.5) afterwards.
struct ApOpts {
  const int32_t* pos = nullptr;    // token positions (ROPE)
  const float* cos_sin = nullptr;  // fp32 [max_pos, 128]: cos of the 64 angles, then their sines
  int max_pos = 0;
  uint16_t* k_out = nullptr;       // post-RoPE keys, bf16 [n, H, 128], or null
  int had = 0;
};

constexpr float kHadScale = 0x1.6a09e6p-4f;  // RN(1 / sqrt(128))

// fp64 to bf16, nearest even, in two steps that cannot double-round: to fp32 by rounding to odd
// (round toward zero, then set the last bit when inexact; Boldo and Melquiond's rounding to odd),
// then to bf16 by nearest even, which is exact rounding because fp32 keeps 16 more bits.
__device__ __forceinline__ uint32_t f64_to_bf16_rne(double d) {
  float r = (float)d;
  if ((double)r != d) {
    uint32_t b = __float_as_uint(r);
    if (fabs((double)r) > fabs(d)) b -= 1u;  // rounded away from zero: one ulp back toward it
    r = __uint_as_float(b | 1u);
  }
  return f32_to_bf16_rne(r);
}

// Two RoPE pairs in fp32 with proof of their rounding: words a, b hold x_i, x_{i+1} and x_{i+64}, x_{i+65}. With
// p = RN(x2 s) and y = RN(x1 c - p) (an FMA), |y - (x1 c - x2 s)| <= 2^-24 (|y| + |p|) for normal values, so with
// E a little above that bound (and above 2^-120, which covers underflow) the exact value lies in [y - E, y + E];
// when both ends round to the same bf16 value, so does the exact value (and its fp64 rounding, which lies between
// them too). Otherwise, and for infinities and NaN (E is not below 2^100 then), `unsure` is set and the caller
// takes fp64. On N(0, 1) keys one word in 3,000 is unsure, so a wave takes fp64 for 2 % of its words; words of zeros
// always are (an interval around zero has two signs: 16,384 tokens of zero keys 39 us against 33 to 35 of N(0, 1)
// keys, and 39.7 with fp64 throughout). Per pair 20 vector instructions instead of about 50, with fp64 at half
// rate; the write is bound by the rows and the table it moves (without the output rows 44 -> 30 us), so this shows
// only once those move well.
struct RopeWord {
  uint32_t a, b;
  bool unsure;
};
__device__ __forceinline__ RopeWord rope_word(uint32_t a, uint32_t b, float c0, float c1, float s0, float s1) {
#pragma clang fp contract(off)
  typedef float f2 __attribute__((ext_vector_type(2)));
  typedef __bf16 b2 __attribute__((ext_vector_type(2)));
  constexpr float k = 0x1.2p-24f;
  const float x1[2] = {__uint_as_float(a << 16), __uint_as_float(a & 0xFFFF0000u)};
  const float x2[2] = {__uint_as_float(b << 16), __uint_as_float(b & 0xFFFF0000u)};
  const float cc[2] = {c0, c1}, ss[2] = {s0, s1};
  f2 lo1, hi1, lo2, hi2;
  float emax = 0.0f;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const float p1 = x2[i] * ss[i], y1 = __builtin_fmaf(x1[i], cc[i], -p1);
    const float p2 = x1[i] * ss[i], y2 = __builtin_fmaf(x2[i], cc[i], p2);
    const float e1 = __builtin_fmaf(fabsf(p1), k, __builtin_fmaf(fabsf(y1), k, 0x1p-120f));
    const float e2 = __builtin_fmaf(fabsf(p2), k, __builtin_fmaf(fabsf(y2), k, 0x1p-120f));
    lo1[i] = y1 - e1;
    hi1[i] = y1 + e1;
    lo2[i] = y2 - e2;
    hi2[i] = y2 + e2;
    emax += e1 + e2;
  }
  const uint32_t l1 = __builtin_bit_cast(uint32_t, __builtin_convertvector(lo1, b2));
  const uint32_t h1 = __builtin_bit_cast(uint32_t, __builtin_convertvector(hi1, b2));
  const uint32_t l2 = __builtin_bit_cast(uint32_t, __builtin_convertvector(lo2, b2));
  const uint32_t h2 = __builtin_bit_cast(uint32_t, __builtin_convertvector(hi2, b2));
  return RopeWord{l1, l2, ((l1 ^ h1) | (l2 ^ h2)) != 0u || !(emax < 0x1p100f)};
}

// RoPE of eight pairs in place: x0 holds channels 8 j .. 8 j + 7 of a token, x1 channels 64 + 8 j .., cs the eight
// cosines then the eight sines.
__device__ __forceinline__ void rope_pairs(ap_u4_t& x0, ap_u4_t& x1, const float (&cs)[16]) {
#pragma clang fp contract(off)
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t a = x0[q], b = x1[q];
    const RopeWord r = rope_word(a, b, cs[2 * q], cs[2 * q + 1], cs[8 + 2 * q], cs[9 + 2 * q]);
    uint32_t oa = r.a, ob = r.b;
    if (__any(r.unsure)) {
      // a wave whose bounds did not settle a rounding takes the word in fp64
      oa = ob = 0u;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const double u1 = (double)__uint_as_float((a >> (16 * i)) << 16), u2 = (double)__uint_as_float((b >> (16 * i)) << 16);
        const double cc = (double)cs[2 * q + i], ss = (double)cs[8 + 2 * q + i];
        const double y1 = u1 * cc - u2 * ss;  // exact products, one rounding
        const double y2 = u2 * cc + u1 * ss;
        oa |= f64_to_bf16_rne(y1) << (16 * i);
        ob |= f64_to_bf16_rne(y2) << (16 * i);
      }
    }
    x0[q] = oa;
    x1[q] = ob;
  }
}

// LDS-DMA: lane i's bytes land at lds + 16 i (4 i). Issued through inline asm, so that the compiler's waits do
// not count them (it would wait for all of them before any LDS read); vmcnt counts the wave's memory
// operations in issue order.
__device__ __forceinline__ void ap_dma16(const void* p, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(p) : "memory", "m0");
}
__device__ __forceinline__ void ap_dma4(const void* p, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(lds), "v"(p) : "memory", "m0");
}

// One append work-group (kApThreads threads): KV head h, K (kv = 0) or V (kv = 1), block bx of nbx striding over
// the 32-token tiles. Every thread of the block must call it (it synchronizes). TERMS: 3 (dense R) or 1
// (Hadamard). With ERR, err[(token * H + h) * 2 + kv] receives each token's squared reconstruction error. With
// ROPE (keys), opt carries the positions and table; with POS (values of such a write) the positions only, so that a
// token skipped for its position keeps both halves of its row: pos_lds then
// holds kApPos ints.
template <int NG, bool ERR, bool ROPE, bool POS, int TERMS>
__device__ __forceinline__ void append_tiles(const CacheView& cv, const uint16_t* __restrict__ X,
                                             const int32_t* __restrict__ slots, int n, const float* __restrict__ R,
                                             const float* __restrict__ mu_rk, float clip, int bx, int nbx, int h, int kv,
                                             ApLds& L, int* pos_lds, float* __restrict__ err, const ApOpts& opt) {
  using Lay = Rec<NG>;
  const int H = cv.num_kv_heads, tid = threadIdx.x, l = tid & 63;
  const int g = __builtin_amdgcn_readfirstlane(tid >> 6);  // the wave's group
  const int tl = l & 31, hf = l >> 5;                      // its token and half in the products
  const int tt = tid >> 3, j = tid & 7;                    // the thread's token and piece in loads and stores
  const int tiles = (n + kApTok - 1) / kApTok, cnt = (tiles - bx + nbx - 1) / nbx;

  // ---- loads of tile i (of this block) into register set p; past the end: the last token, slot -1
  struct Pre {
    ap_u4_t x0, x1;
    int slot;
    float cs[16];
    bool pos_ok;
  };
  Pre pre[kApDepth];
  int pos_next = 0;
  auto token = [&](int i) { return (bx + i * nbx) * kApTok + tt; };
  // pointers of the next tile to load; past the end they stay on a row already read
  const int hop = nbx * kApTok;
  int tok_ld = token(0);
  const uint16_t* row_ld = X + ((size_t)min(tok_ld, n - 1) * H + h) * kHeadDim + 8 * j;
  const int32_t* slot_ld = slots + min(tok_ld, n - 1);
  const int32_t* pos_ld = ROPE || POS ? opt.pos + min(tok_ld, n - 1) : nullptr;
  auto load = [&](Pre& p) {
    const bool more = tok_ld + hop < n;
    if constexpr (ROPE) {
      // the position was fetched a step ago; the next one goes first, so that it is the oldest of this step's loads
      const int pos = pos_next;
      pos_ld += more ? hop : 0;
      pos_next = *pos_ld;
      p.pos_ok = pos >= 0 && pos < opt.max_pos;
      const float4* c = reinterpret_cast<const float4*>(opt.cos_sin + (size_t)(p.pos_ok ? pos : 0) * kHeadDim + 8 * j);
      const float4 c0 = c[0], c1 = c[1], s0 = c[16], s1 = c[17];
      p.cs[0] = c0.x, p.cs[1] = c0.y, p.cs[2] = c0.z, p.cs[3] = c0.w;
      p.cs[4] = c1.x, p.cs[5] = c1.y, p.cs[6] = c1.z, p.cs[7] = c1.w;
      p.cs[8] = s0.x, p.cs[9] = s0.y, p.cs[10] = s0.z, p.cs[11] = s0.w;
      p.cs[12] = s1.x, p.cs[13] = s1.y, p.cs[14] = s1.z, p.cs[15] = s1.w;
    }
    p.x0 = *reinterpret_cast<const ap_u4_t*>(row_ld);
    p.x1 = *reinterpret_cast<const ap_u4_t*>(row_ld + 64);
    p.slot = *slot_ld;
    row_ld += more ? (size_t)hop * H * kHeadDim : 0;
    slot_ld += more ? hop : 0;
    tok_ld += hop;
  };
  // register set p (tile i) into LDS buffer i % 2; returns the thread's slot (-1: not stored)
  auto consume = [&](int i, Pre& p) {
    const int tok = token(i);
    int slot = tok < n ? p.slot : -1;
    if constexpr (ROPE) {
      rope_pairs(p.x0, p.x1, p.cs);
      if (!p.pos_ok) slot = -1;
      if (opt.k_out && p.pos_ok && tok < n) {
        uint16_t* o = opt.k_out + ((size_t)tok * H + h) * kHeadDim + 8 * j;
        *reinterpret_cast<ap_u4_t*>(o) = p.x0;
        *reinterpret_cast<ap_u4_t*>(o + 64) = p.x1;
      }
    }
    uint8_t* x = L.x[i & 1] + 256 * tt;
    *reinterpret_cast<ap_u4_t*>(x + 16 * (j ^ (tt & 15))) = p.x0;
    *reinterpret_cast<ap_u4_t*>(x + 16 * ((j + 8) ^ (tt & 15))) = p.x1;
    return slot;
  };
  const int nslots = cv.num_blocks * kBlock;
  // packed stores of the tile in exchange buffer i % 2: thread (token tt, halves 2 j and 2 j + 1)
  auto finish = [&](int i, int slot) {
    const int s_hf = j >> 2, q = j & 3, buf = i & 1;
    const uint4 w = *reinterpret_cast<const uint4*>(&L.words[buf][tt][s_hf][0]);
    const uint32_t m = L.meta[buf][tt][NG == 4 ? q : 0];
    // byte q of the four groups' words, group g in byte g
    const uint32_t sel = 0x0C0C0400u + 0x0101u * q;
    const uint32_t lo = __builtin_amdgcn_perm(w.y, w.x, sel), hi = __builtin_amdgcn_perm(w.w, w.z, sel);
    const uint32_t b4 = lo | (hi << 16);
    uint32_t e = b4 & 0x0F0F0F0Fu, o = (b4 >> 4) & 0x0F0F0F0Fu;  // halves 2 j, 2 j + 1: nibble g in byte g
    e = (e | (e >> 4)) & 0x00FF00FFu;
    o = (o | (o >> 4)) & 0x00FF00FFu;
    e = (e | (e >> 8)) & 0xFFFFu;
    o = (o | (o >> 8)) & 0xFFFFu;
    float es = 0.0f;
    if constexpr (ERR) es = (L.err[buf][tt][0] + L.err[buf][tt][1]) + (L.err[buf][tt][2] + L.err[buf][tt][3]);
    if (slot >= 0 && slot < nslots) {
      const int t = slot & 15;
      uint8_t* rec = cv.pool + ((size_t)(slot >> 4) * H + h) * Lay::kBytes;
      if (kv == 0) {
        *reinterpret_cast<uint32_t*>(rec + kOffKCodes + 32 * t + 4 * j) = e | (o << 16);
        if (j < NG) *reinterpret_cast<uint32_t*>(rec + Lay::kOffKMeta + 4 * NG * t + 4 * j) = m;
      } else {
        uint8_t* vc = rec + kOffVCodes + 64 * j + 2 * t;
        *reinterpret_cast<uint16_t*>(vc) = (uint16_t)e;
        *reinterpret_cast<uint16_t*>(vc + 32) = (uint16_t)o;
        if (q < NG)
          *reinterpret_cast<uint16_t*>(rec + (s_hf ? Lay::kOffVZero : Lay::kOffVScale) + 32 * q + 2 * t) =
              (uint16_t)(s_hf ? m >> 16 : m);
      }
    }
    if constexpr (ERR) {
      const int tok = token(i);
      if (j == 0 && tok < n) err[((size_t)tok * H + h) * 2 + kv] = es;
    }
  };

  // without RoPE the tiles go straight to LDS: wave g fetches tokens 8 g .. + 7 (two operations) and its threads' slots
  const int t_dma = 8 * g + (l >> 4);
  const uint16_t* row_dma[2];
  int tok_dma[2];
  if constexpr (!ROPE) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int t = t_dma + 4 * u;
      tok_dma[u] = bx * kApTok + t;
      row_dma[u] = X + ((size_t)min(tok_dma[u], n - 1) * H + h) * kHeadDim + 8 * ((l & 15) ^ (t & 15));
    }
  }
  const uint32_t x_lds = (uint32_t)(uintptr_t)&L.x[0][0] + 2048 * g, slot_lds = (uint32_t)(uintptr_t)&L.slot[0][0] + 256 * g;
  const uint32_t pos_dst = POS ? (uint32_t)(uintptr_t)pos_lds + 256 * g : 0u;
  constexpr int kDma = POS ? 4 : 3;  // operations per tile and wave
  auto dma = [&](int stage) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      ap_dma16(row_dma[u], x_lds + (uint32_t)(stage * kApTok * 256 + 1024 * u));
      row_dma[u] += tok_dma[u] + hop < n ? (size_t)hop * H * kHeadDim : 0;
      tok_dma[u] += hop;
    }
    ap_dma4(slot_ld, slot_lds + (uint32_t)(stage * kApThreads * 4));
    if constexpr (POS) {
      ap_dma4(pos_ld, pos_dst + (uint32_t)(stage * kApThreads * 4));
      pos_ld += tok_ld + hop < n ? hop : 0;
    }
    slot_ld += tok_ld + hop < n ? hop : 0;
    tok_ld += hop;
  };
  if constexpr (ROPE) {
    pos_next = *pos_ld;
#pragma unroll
    for (int d = 0; d < kApDepth; ++d) load(pre[d]);
  } else {
#pragma unroll
    for (int s = 0; s < kApStages - 1; ++s) dma(s);
  }

  // ---- the wave's rows of R^T: lane (row l % 32, 8 hf ..) of k step ks holds R[16 ks + 8 hf + e][channel]
  ap_bf16x8_t A[TERMS][8];
  {
    const int a = tl >> 3, ch = 32 * g + 16 * (a >> 1) + 8 * ((tl >> 2) & 1) + 4 * (a & 1) + (tl & 3);
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      uint32_t t16[TERMS][8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int k = 16 * ks + 8 * hf + e;
        if constexpr (TERMS == 1) {
          t16[0][e] = (__builtin_popcount(k & ch) & 1) ? 0xBF80u : 0x3F80u;
        } else {
          const float r = R[k * kHeadDim + ch];
          const uint32_t b0 = __float_as_uint(r) & 0xFFFF0000u;
          const float r1 = r - __uint_as_float(b0);
          const uint32_t b1 = __float_as_uint(r1) & 0xFFFF0000u;
          t16[0][e] = b0 >> 16;
          t16[1][e] = b1 >> 16;
          t16[2][e] = __float_as_uint(r1 - __uint_as_float(b1)) >> 16;
        }
      }
#pragma unroll
      for (int t = 0; t < TERMS; ++t)
        A[t][ks] = __builtin_bit_cast(ap_bf16x8_t, ap_u4_t{t16[t][0] | (t16[t][1] << 16), t16[t][2] | (t16[t][3] << 16),
                                                           t16[t][4] | (t16[t][5] << 16), t16[t][6] | (t16[t][7] << 16)});
    }
  }
  for (int m = tid; m < 1024; m += kApThreads) L.recip[m] = 1.0f / (1.0f + (float)m * 0x1p-10f);
  if (tid < kHeadDim) L.sub[tid] = kv == 0 ? -mu_rk[(size_t)h * kHeadDim + tid] : 0.0f;
  auto barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
  int slot = -1, slot_prev = -1, slot_done = -1;  // of tiles i, i - 1 and i - 2
  if constexpr (ROPE) slot = consume(0, pre[0]);
  barrier();

  // ---- step i with its registers pre[i % kApDepth]: the products of tile i beside the quantizer of tile i - 1
  // (prev: its rotated values), which depend on nothing in common; both in one block without branches, so that
  // the schedule below can alternate them
  ap_f16_t acc[2];
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[1][r] = 0.0f;
  auto quantize = [&](int i, const ap_f16_t& prev) {
    float mn, mx;
    ap_extremes(prev, mn, mx);
    if constexpr (NG == 1) {
      if (hf == 0) *reinterpret_cast<float2*>(L.ext[tl][g]) = make_float2(mn, mx);
      barrier();
      const float4 e0 = *reinterpret_cast<const float4*>(L.ext[tl][0]), e1 = *reinterpret_cast<const float4*>(L.ext[tl][2]);
      mn = __builtin_elementwise_minimum(__builtin_elementwise_minimum(e0.x, e0.z), __builtin_elementwise_minimum(e1.x, e1.z));
      mx = __builtin_elementwise_maximum(__builtin_elementwise_maximum(e0.y, e0.w), __builtin_elementwise_maximum(e1.y, e1.w));
    }
    const ApOut o = quantize_group<ERR>(prev, mn, mx, clip, L.recip);
    L.words[i & 1][tl][hf][g] = o.word;
    L.meta[i & 1][tl][g] = o.meta;  // both halves hold the same
    if constexpr (ERR) L.err[i & 1][tl][g] = o.err;
  };
  auto product = [&](const uint8_t* tile, ap_f16_t& acc) {
    const uint8_t* x = tile + 256 * tl;
    auto sub = [&](int r4) {  // the lane's channels: 16 (a / 2) + 8 hf + 4 (a % 2) + b of group g
      return *reinterpret_cast<const float4*>(&L.sub[32 * g + 16 * (r4 >> 1) + 8 * hf + 4 * (r4 & 1)]);
    };
    ap_bf16x8_t B[8];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
      B[ks] = *reinterpret_cast<const ap_bf16x8_t*>(x + 16 * ((2 * ks + hf) ^ (tl & 15)));
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const float4 s = TERMS == 1 ? make_float4(0.f, 0.f, 0.f, 0.f) : sub(a);
      acc[4 * a] = s.x, acc[4 * a + 1] = s.y, acc[4 * a + 2] = s.z, acc[4 * a + 3] = s.w;
    }
#pragma unroll
    for (int t = TERMS - 1; t >= 0; --t)  // smallest term first
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[t][ks], B[ks], acc, 0, 0, 0);
    if constexpr (TERMS == 1) {
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const float4 s = sub(a);
        acc[4 * a] = __builtin_fmaf(acc[4 * a], kHadScale, s.x);
        acc[4 * a + 1] = __builtin_fmaf(acc[4 * a + 1], kHadScale, s.y);
        acc[4 * a + 2] = __builtin_fmaf(acc[4 * a + 2], kHadScale, s.z);
        acc[4 * a + 3] = __builtin_fmaf(acc[4 * a + 3], kHadScale, s.w);
      }
    }
  };
  auto schedule = [] {
#pragma unroll
    for (int m = 0; m < 8 * TERMS; ++m) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                    // one product
      __builtin_amdgcn_sched_group_barrier(0x002, TERMS == 1 ? 18 : 6, 0);  // vector instructions beside it
    }
  };
  if constexpr (ROPE) {
    // cur: where tile i's values go; prv: tile i - 1's; p: the registers of tile i (consumed), refilled with
    // tile i + kApDepth; pn: those of tile i + 1
    auto step = [&](int i, Pre& p, Pre& pn, ap_f16_t& cur, const ap_f16_t& prv) {
      if (i > 1) finish(i - 2, slot_done);
      load(p);
      product(L.x[i & 1], cur);
      quantize(i - 1, prv);  // of zeros in the first step, into a buffer that is rewritten before it is read
      schedule();
      slot_done = slot_prev;
      slot_prev = slot;
      slot = consume(i + 1, pn);
      barrier();
    };
    static_assert(kApDepth % 2 == 0, "the register sets and the accumulators repeat together");
    for (int i0 = 0; i0 < cnt; i0 += kApDepth) {
#pragma unroll
      for (int d = 0; d < kApDepth; ++d)
        if (i0 + d < cnt) step(i0 + d, pre[d], pre[(d + 1) % kApDepth], acc[d & 1], acc[1 - (d & 1)]);
    }
  } else {
    int stage = 0;  // of tile i
    auto step = [&](int i, ap_f16_t& cur, const ap_f16_t& prv) {
      // this wave's operations of tile i are done when at most those of the kApStages - 2 tiles after it are
      // outstanding (stores among them only make the wait longer); the barrier extends that to every
      // wave's, and says that tile i - 1's stage and the exchange buffers of tile i - 3 are free
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(kDma * (kApStages - 2)) : "memory");
      slot_done = slot_prev;
      slot_prev = slot;
      const int sl = L.slot[stage][tid];
      slot = token(i) < n ? sl : -1;
      if constexpr (POS) {
        const int pos = pos_lds[stage * kApThreads + tid];
        if (pos < 0 || pos >= opt.max_pos) slot = -1;
      }
      if (i > 1) finish(i - 2, slot_done);
      dma(stage == 0 ? kApStages - 1 : stage - 1);
      product(L.x[stage], cur);
      quantize(i - 1, prv);
      schedule();
      stage = stage + 1 == kApStages ? 0 : stage + 1;
    };
    for (int i0 = 0; i0 < cnt; i0 += 2) {
      step(i0, acc[0], acc[1]);
      if (i0 + 1 < cnt) step(i0 + 1, acc[1], acc[0]);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the tiles fetched past the end
    slot_done = slot_prev;
    slot_prev = slot;
    barrier();
  }
  if (cnt > 1) finish(cnt - 2, slot_done);
  if (cnt & 1)
    quantize(cnt - 1, acc[0]);
  else
    quantize(cnt - 1, acc[1]);
  barrier();
  finish(cnt - 1, slot_prev);
}

// One append work-group with the rotation its options ask for.
template <int NG, bool ERR = false, bool ROPE = false>
__device__ __forceinline__ void append_block(const CacheView& cv, const uint16_t* __restrict__ k,
                                             const uint16_t* __restrict__ v, const int32_t* __restrict__ slots,
                                             int n, const float* __restrict__ R_k, const float* __restrict__ R_v,
                                             const float* __restrict__ mu_rk, float clip_k, float clip_v, int bx,
                                             int nbx, int h, int kv, ApLds& L, int* pos_lds = nullptr,
                                             float* __restrict__ err = nullptr, const ApOpts& opt = ApOpts{}) {
  const uint16_t* X = kv == 0 ? k : v;
  const float clip = kv == 0 ? clip_k : clip_v;
  const bool had = ((opt.had >> kv) & 1) != 0;
  const float* R = had ? nullptr : (kv == 0 ? R_k : R_v) + (size_t)h * kHeadDim * kHeadDim;
  if (ROPE && kv == 0) {
    if (had)
      append_tiles<NG, ERR, ROPE, false, 1>(cv, X, slots, n, R, mu_rk, clip, bx, nbx, h, kv, L, pos_lds, err, opt);
    else
      append_tiles<NG, ERR, ROPE, false, 3>(cv, X, slots, n, R, mu_rk, clip, bx, nbx, h, kv, L, pos_lds, err, opt);
  } else if (had) {
    append_tiles<NG, ERR, false, ROPE, 1>(cv, X, slots, n, R, mu_rk, clip, bx, nbx, h, kv, L, pos_lds, err, opt);
  } else {
    append_tiles<NG, ERR, false, ROPE, 3>(cv, X, slots, n, R, mu_rk, clip, bx, nbx, h, kv, L, pos_lds, err, opt);
  }
}

}  // namespace int2kv

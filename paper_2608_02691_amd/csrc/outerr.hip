// Output-error diagnostics of the INT2 cache (Sec. 3.2; appendix output-space error metrics).
//
// For every sequence b and query head j, against the full-precision keys and values the cache was
// written from:
//   o1 = p^T V         full-precision keys and values (p = softmax of q.k / sqrt(d)),
//   o2 = p~^T V        INT2 keys (p~ = softmax of q.k~ / sqrt(d)), full-precision values,
//   o3 = p~^T V~       INT2 keys and values (the INT2 decode),
// then dy_K = (o2 - o1) W_{O,j}^T and dy_V = (o3 - o2) W_{O,j}^T (so y~ - y = dy_K + dy_V), and the
// four statistics (||dy_K + dy_V||^2, ||dy_K||^2, ||dy_V||^2, <dy_K, dy_V>).
//
// Kernels: a split-context scan (block = context chunk x KV head x sequence, four waves, a page of
// 16 tokens per wave step) that runs both softmaxes over the chunk and accumulates the three value
// sums; a merge of the chunk partials that also undoes the value rotation of o3 (o3 = o3' R_V^T);
// the per-head projection by W_{O,j} (block = query head x 128 rows of W_O, all sequences) with
// partial statistics per row tile; and the sum of those partials. The INT2 scores use the rotated
// query (q R_K) . k^, the full-precision ones q . k with the raw keys: both softmaxes are invariant
// to the key offset mu, which the effective keys k~ = k^ R_K^T + mu carry.
#include "common.h"
#include "kernels.h"

namespace int2kv {

namespace {

constexpr float kOeLogit2 = 1.4426950408889634f * 0.08838834764831845f;  // log2(e)/sqrt(128)
constexpr int kOeWaves = 4;

__device__ __forceinline__ int oe_seq_len(const OutErrArgs& e, int b) {
  int L = e.a.ctx_lens[b];
  L = min(L, e.a.max_ctx);
  L = min(L, e.a.max_blocks * kBlock);
  L = min(L, e.row_cap);
  return max(L, 0);
}

typedef _Float16 oe_f16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 oe_bf8_t __attribute__((ext_vector_type(8)));
typedef float oe_f4_t __attribute__((ext_vector_type(4)));
typedef uint32_t oe_u4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void oe_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace

// Block (chunk, KV head h, sequence b). Scores on the matrix cores, with fp32's precision: lane (token lo = l % 16,
// hi = l / 16) ends with the scores of token lo for query head 4 Q + hi of each quad Q of heads.
//  * full precision: q . k as bf16 products (exact), fp32 sums; query head j of the quad in row 4 j;
//  * INT2: a code's two bits, shifted to the bottom of a 16-bit half, are the fp16 number code 2^-24; times 2^15 it is
//    a normal number (the matrix cores align a product by its exponents, so that subnormal factors cost the sum
//    their leading zeros: statistics to 2e-5 of fp64's instead of 1e-6). q' = q R_K, scaled by a power of two, enters
//    as three fp16 terms, whose sum it is to 2^-38 of the row's largest value, in rows 4 j .. 4 j + 2: one product per
//    32-channel group gives sum_{c in g} q'_c code_c in the lane's first three registers.
// Softmaxes run on one (token, head) per lane, with maxima and sums over the 16 lanes of a DPP row. For the
// values lane l owns channels 2 l, 2 l + 1 on the vector ALU. Near the rows' stream: 16 x 4,096 tokens, 32/8 heads
// 121 us with the scores on the vector ALU (their products and LDS broadcasts of q) -> 83 us for 318 MB. Statistics
// differ from fp64's by 3e-7 to 8e-7 (on the vector ALU 4e-7 to 9e-7).
template <int MAXG, int NG>
__global__ __launch_bounds__(256, MAXG <= 4 ? 4 : 1) void outerr_scan_kernel(OutErrArgs e) {
  using Lay = Rec<NG>;
  constexpr int kQuads = (MAXG + 3) / 4;
  const DecodeArgs& a = e.a;
  __shared__ float pb[kOeWaves][2][kBlock][4 * kQuads];  // p of both softmaxes for the page (token-major)
  __shared__ float wst[kOeWaves][4 * kQuads][4];
  __shared__ float wout[kOeWaves][3][MAXG][kHeadDim];

  const int chunk = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  const int L = oe_seq_len(e, b);
  const int t0 = chunk * a.chunk_tokens;
  const int gq = a.gq, tid = threadIdx.x, w = tid >> 6, l = tid & 63, lo = l & 15, hi = l >> 4;
  if (t0 >= L) {
    // a chunk past the context: an empty partial (m = -inf) that the merge drops
    for (int i = tid; i < gq; i += blockDim.x) {
      float* dst = e.part + (((size_t)b * a.n_chunks + chunk) * a.Hq + h * gq + i) * kOePartStride;
      dst[0] = -INFINITY;
      dst[2] = -INFINITY;
    }
    return;
  }
  const int t1 = min(L, t0 + a.chunk_tokens);

  // query operands of each quad, the group sums of q' of head hi and the factor back to base-2 logits
  __shared__ oe_bf8_t A1[kQuads][4][64];  // in LDS: 16 vector registers less a quad, which would spill
  oe_f16x8_t A2[kQuads][4];
  float qsum[kQuads][kGroups], unscale[kQuads];
#pragma unroll
  for (int Q = 0; Q < kQuads; ++Q) {
    // row lo = 4 j + term of head j: the lane's channels of group g are 32 g + 4 hi + 0..3, 32 g + 16 + 4 hi + 0..3
    const int jr = 4 * Q + (lo >> 2), term = lo & 3;
    const size_t qrow = ((size_t)b * a.Hq + h * gq + min(jr, gq - 1)) * kHeadDim;
    const bool on = jr < gq;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const oe_u4_t x = *reinterpret_cast<const oe_u4_t*>(a.q + qrow + 32 * ks + 8 * hi);
      const uint32_t keep = on && term == 0 ? ~0u : 0u;
      const oe_bf8_t y = __builtin_bit_cast(oe_bf8_t, x & oe_u4_t{keep, keep, keep, keep});
      if (ks == w) A1[Q][ks][l] = y;
    }
    float x[4][8], mx = 0.0f;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 u = *reinterpret_cast<const float4*>(a.qrot + qrow + 32 * g + 4 * hi);
      const float4 v = *reinterpret_cast<const float4*>(a.qrot + qrow + 32 * g + 16 + 4 * hi);
      const float y[8] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        x[g][i] = on ? y[i] : 0.0f;
        mx = fmaxf(mx, fabsf(x[g][i]));
      }
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    int ex = 0;
    frexpf(mx, &ex);
    ex = mx > 0.0f && mx < INFINITY ? max(-80, ex) : 14;  // |q'| 2^(14 - ex) < 2^14
    const float sg = ldexpf(1.0f, 14 - ex);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      float s = 0.0f;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        s += x[g][i];
        const float y = x[g][i] * sg;
        const _Float16 f0 = (_Float16)y, f1 = (_Float16)(y - (float)f0);
        const _Float16 f2 = (_Float16)((y - (float)f0) - (float)f1);
        A2[Q][g][i] = term == 0 ? f0 : term == 1 ? f1 : term == 2 ? f2 : (_Float16)0.0f;
      }
      s += __shfl_xor(s, 16);
      s += __shfl_xor(s, 32);
      qsum[Q][g] = __shfl(s, 4 * hi) * kOeLogit2;  // lane 4 hi holds row 4 hi: head hi of the quad
    }
    unscale[Q] = ldexpf(kOeLogit2, 24 - 15 - 14 + __shfl(ex, 4 * hi));
  }

  __syncthreads();

  // running states: (m, l) of both softmaxes for head hi of each quad; the three value sums of channels 2l, 2l + 1
  float m1[kQuads], l1[kQuads], m2[kQuads], l2[kQuads], o[3][MAXG][2];
#pragma unroll
  for (int Q = 0; Q < kQuads; ++Q) {
    m1[Q] = m2[Q] = -INFINITY;
    l1[Q] = l2[Q] = 0.0f;
  }
#pragma unroll
  for (int j = 0; j < MAXG; ++j)
#pragma unroll
    for (int r = 0; r < 3; ++r) o[r][j][0] = o[r][j][1] = 0.0f;
  const int c0 = 2 * l, m0 = c0 & 15, pv = c0 >> 4, gv = c0 >> 5;
  const size_t row_stride = (size_t)a.H * kHeadDim;
  const uint16_t* krow0 = e.k_rows + ((size_t)b * e.row_cap * a.H + h) * kHeadDim;
  const uint16_t* vrow0 = e.v_rows + ((size_t)b * e.row_cap * a.H + h) * kHeadDim;

  const int pg0 = t0 / kBlock, pg1 = (t1 + kBlock - 1) / kBlock;
  for (int pg = pg0 + w; pg < pg1; pg += kOeWaves) {
    const int blk = a.block_table[(size_t)b * a.max_blocks + pg];
    if (blk < 0 || blk >= a.num_blocks) continue;  // uniform per wave
    const uint8_t* rec = a.pool + ((size_t)blk * a.H + h) * Lay::kBytes;
    const int pos = pg * kBlock + lo;
    const bool valid = pos >= t0 && pos < t1;
    const int posc = min(max(pos, t0), t1 - 1);  // a row inside the caller's store

    // ---- operands of token lo: its codes (halves 4 hi .. + 3), metadata and raw key channels 32 ks + 8 hi ..
    const uint2 kc = *reinterpret_cast<const uint2*>(rec + kOffKCodes + 32 * lo + 8 * hi);
    uint32_t km[NG];
    if constexpr (NG == 4) {
      const uint4 x = *reinterpret_cast<const uint4*>(rec + Lay::kOffKMeta + 16 * lo);
      km[0] = x.x, km[1] = x.y, km[2] = x.z, km[3] = x.w;
    } else {
      km[0] = *reinterpret_cast<const uint32_t*>(rec + Lay::kOffKMeta + 4 * lo);
    }
    oe_bf8_t kr[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
      kr[ks] = *reinterpret_cast<const oe_bf8_t*>(krow0 + (size_t)posc * row_stride + 32 * ks + 8 * hi);
    oe_f16x8_t kq[4];
#pragma unroll
    for (int g = 0; g < 4; ++g)
      kq[g] = __builtin_bit_cast(oe_f16x8_t, oe_u4_t{(kc.x >> (4 * g)) & 0x00030003u, (kc.y >> (4 * g)) & 0x00030003u,
                                                     (kc.x >> (4 * g + 2)) & 0x00030003u,
                                                     (kc.y >> (4 * g + 2)) & 0x00030003u}) *
              (_Float16)32768.0f;
    bool moved = false;
    float al1[kQuads], al2[kQuads];
#pragma unroll
    for (int Q = 0; Q < kQuads; ++Q) {
      oe_f4_t d1 = {0.f, 0.f, 0.f, 0.f}, d2[NG];
#pragma unroll
      for (int g = 0; g < NG; ++g) d2[g] = oe_f4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        d1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A1[Q][g][l], kr[g], d1, 0, 0, 0);
        d2[g % NG] = __builtin_amdgcn_mfma_f32_16x16x32_f16(A2[Q][g], kq[g], d2[g % NG], 0, 0, 0);
      }
      float s1 = d1[0] * kOeLogit2, s2 = 0.0f;
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        const float qs = NG == 4 ? qsum[Q][g] : (qsum[Q][0] + qsum[Q][1]) + (qsum[Q][2] + qsum[Q][3]);
        const float dot = ((d2[g][2] + d2[g][1]) + d2[g][0]) * unscale[Q];
        s2 += f16_bits_to_f32(km[g] & 0xFFFF) * dot + f16_bits_to_f32(km[g] >> 16) * qs;
      }
      s1 = valid ? s1 : -INFINITY;
      s2 = valid ? s2 : -INFINITY;
      const float n1 = fmaxf(m1[Q], row_max16(s1)), n2 = fmaxf(m2[Q], row_max16(s2));
      al1[Q] = n1 == -INFINITY ? 1.0f : exp2f(m1[Q] - n1);
      al2[Q] = n2 == -INFINITY ? 1.0f : exp2f(m2[Q] - n2);
      moved |= n1 != m1[Q] || n2 != m2[Q];
      const float p1 = valid ? exp2f(s1 - n1) : 0.0f, p2 = valid ? exp2f(s2 - n2) : 0.0f;
      l1[Q] = l1[Q] * al1[Q] + row_sum16(p1);
      l2[Q] = l2[Q] * al2[Q] + row_sum16(p2);
      m1[Q] = n1;
      m2[Q] = n2;
      pb[w][0][lo][4 * Q + hi] = p1;
      pb[w][1][lo][4 * Q + hi] = p2;
    }
    oe_wave_sync();
    if (__any(moved)) {
#pragma unroll
      for (int j = 0; j < MAXG; ++j) {
        const float f1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, al1[j >> 2]), 16 * (j & 3)));
        const float f2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, al2[j >> 2]), 16 * (j & 3)));
#pragma unroll
        for (int cc = 0; cc < 2; ++cc) {
          o[0][j][cc] *= f1;
          o[1][j][cc] *= f2;
          o[2][j][cc] *= f2;
        }
      }
    }

    // ---- values of channels c0, c0 + 1: INT2 (R_V basis) and full precision (model basis), in two
    // halves of eight tokens (the loads of a half, then its arithmetic)
    const uint4* vc = reinterpret_cast<const uint4*>(rec + kOffVCodes + 32 * m0);  // halves m0, m0 + 1
    const uint4* vsp = reinterpret_cast<const uint4*>(rec + Lay::kOffVScale + 32 * (NG == 4 ? gv : 0));
    const uint4* vzp = reinterpret_cast<const uint4*>(rec + Lay::kOffVZero + 32 * (NG == 4 ? gv : 0));
#pragma unroll
    for (int H = 0; H < 2; ++H) {
      const uint4 ca = vc[H], cb = vc[2 + H], s4 = vsp[H], z4 = vzp[H];  // tokens 8 H .. 8 H + 7
      const uint32_t hv0[4] = {ca.x, ca.y, ca.z, ca.w}, hv1[4] = {cb.x, cb.y, cb.z, cb.w};
      const uint32_t sw[4] = {s4.x, s4.y, s4.z, s4.w}, zw[4] = {z4.x, z4.y, z4.z, z4.w};
      uint32_t vf[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int pt = min(max(pg * kBlock + 8 * H + i, t0), t1 - 1);
        vf[i] = *reinterpret_cast<const uint32_t*>(vrow0 + (size_t)pt * row_stride + c0);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int t = 8 * H + i, sh = 16 * (i & 1);
        const float vs = f16_bits_to_f32((sw[i >> 1] >> sh) & 0xFFFF);
        const float vz = f16_bits_to_f32((zw[i >> 1] >> sh) & 0xFFFF);
        const float x0 = fmaf(static_cast<float>((hv0[i >> 1] >> (sh + 2 * pv)) & 3), vs, vz);
        const float x1 = fmaf(static_cast<float>((hv1[i >> 1] >> (sh + 2 * pv)) & 3), vs, vz);
        const float r0 = __uint_as_float(vf[i] << 16), r1 = __uint_as_float(vf[i] & 0xFFFF0000u);
#pragma unroll
        for (int j = 0; j < MAXG; ++j) {
          if (j < gq) {
            const float p1 = pb[w][0][t][j], p2 = pb[w][1][t][j];
            o[0][j][0] = fmaf(p1, r0, o[0][j][0]);
            o[0][j][1] = fmaf(p1, r1, o[0][j][1]);
            o[1][j][0] = fmaf(p2, r0, o[1][j][0]);
            o[1][j][1] = fmaf(p2, r1, o[1][j][1]);
            o[2][j][0] = fmaf(p2, x0, o[2][j][0]);
            o[2][j][1] = fmaf(p2, x1, o[2][j][1]);
          }
        }
      }
    }
    oe_wave_sync();
  }

  // ---- merge the four wave states into the chunk's partial
  if (lo == 0)
#pragma unroll
    for (int Q = 0; Q < kQuads; ++Q) {
      const int j = 4 * Q + hi;
      wst[w][j][0] = m1[Q];
      wst[w][j][1] = l1[Q];
      wst[w][j][2] = m2[Q];
      wst[w][j][3] = l2[Q];
    }
#pragma unroll
  for (int j = 0; j < MAXG; ++j) {
    if (j < gq) {
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        wout[w][r][j][c0] = o[r][j][0];
        wout[w][r][j][c0 + 1] = o[r][j][1];
      }
    }
  }
  __syncthreads();
  for (int i = tid; i < gq * kHeadDim; i += blockDim.x) {
    const int j = i / kHeadDim, c = i % kHeadDim;
    float M1 = -INFINITY, M2 = -INFINITY;
#pragma unroll
    for (int ww = 0; ww < kOeWaves; ++ww) {
      M1 = fmaxf(M1, wst[ww][j][0]);
      M2 = fmaxf(M2, wst[ww][j][2]);
    }
    float L1 = 0.0f, L2 = 0.0f, A[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int ww = 0; ww < kOeWaves; ++ww) {
      const float f1 = wst[ww][j][0] == -INFINITY ? 0.0f : exp2f(wst[ww][j][0] - M1);
      const float f2 = wst[ww][j][2] == -INFINITY ? 0.0f : exp2f(wst[ww][j][2] - M2);
      L1 = fmaf(f1, wst[ww][j][1], L1);
      L2 = fmaf(f2, wst[ww][j][3], L2);
      A[0] = fmaf(f1, wout[ww][0][j][c], A[0]);
      A[1] = fmaf(f2, wout[ww][1][j][c], A[1]);
      A[2] = fmaf(f2, wout[ww][2][j][c], A[2]);
    }
    float* dst = e.part + (((size_t)b * a.n_chunks + chunk) * a.Hq + h * gq + j) * kOePartStride;
    if (c == 0) {
      dst[0] = M1;
      dst[1] = L1;
      dst[2] = M2;
      dst[3] = L2;
    }
#pragma unroll
    for (int r = 0; r < 3; ++r) dst[4 + r * kHeadDim + c] = A[r];
  }
}

// Block (sequence b, query head j), thread (channel c, slot sl): the chunk partials of the head merged into o1, o2
// (model basis) and o3' (R_V basis), o3 = o3' R_V^T, then do = (o2 - o1, o3 - o2). Slot sl takes every fourth
// chunk, two in flight; R_V comes into LDS by LDS-DMA beside them (16-byte piece q of row r at q ^ (r % 32):
// conflict-free by rows). Latency-bound: 16 x 4,096 tokens, 32/8 heads 10.6 -> 6.6 us (the call 114.1 -> 110.3) against 128
// threads per block with R_V read by rows at the end.
constexpr int kOeSlots = 4;
__global__ __launch_bounds__(kHeadDim * kOeSlots) void outerr_merge_kernel(OutErrArgs e) {
  const DecodeArgs& a = e.a;
  __shared__ __attribute__((aligned(16))) float rl[kHeadDim * kHeadDim];
  __shared__ float ml[kOeSlots][4];              // m1, l1, m2, l2 of a slot
  __shared__ float as[kOeSlots][3][kHeadDim];    // its value sums, then the parts of o3
  __shared__ __attribute__((aligned(16))) float os[kHeadDim];
  const int b = blockIdx.x, j = blockIdx.y, tid = threadIdx.x, c = tid & 127, sl = tid >> 7, h = j / a.gq;
  {
    const float* Rv = a.R_v + (size_t)h * kHeadDim * kHeadDim;
    constexpr int kDma = kHeadDim * kHeadDim * 4 / (kHeadDim * kOeSlots * 16);  // 16-byte pieces per thread
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
    const uint32_t base = (uint32_t)(uintptr_t)&rl[0] + 1024 * kDma * w;
#pragma unroll
    for (int k = 0; k < kDma; ++k) {
      const int piece = 64 * (kDma * w + k) + l, row = piece >> 5, q = (piece & 31) ^ (row & 31);
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(base + 1024 * k),
                   "v"(Rv + row * kHeadDim + 4 * q)
                   : "memory", "m0");
    }
  }
  const int L = oe_seq_len(e, b);
  const int nch = (L + a.chunk_tokens - 1) / a.chunk_tokens;
  const float* part = e.part + ((size_t)b * a.n_chunks * a.Hq + j) * kOePartStride;
  const size_t stride = (size_t)a.Hq * kOePartStride;
  float M1 = -INFINITY, M2 = -INFINITY, L1 = 0.0f, L2 = 0.0f, A[3] = {0.0f, 0.0f, 0.0f};
  auto add = [&](float m1, float l1, float m2, float l2, const float (&x)[3]) {
    const float n1 = fmaxf(M1, m1), n2 = fmaxf(M2, m2);
    const float f1 = M1 == -INFINITY ? 0.0f : exp2f(M1 - n1), f2 = M2 == -INFINITY ? 0.0f : exp2f(M2 - n2);
    const float g1 = m1 == -INFINITY ? 0.0f : exp2f(m1 - n1), g2 = m2 == -INFINITY ? 0.0f : exp2f(m2 - n2);
    L1 = fmaf(g1, l1, f1 * L1);
    L2 = fmaf(g2, l2, f2 * L2);
    A[0] = fmaf(g1, x[0], f1 * A[0]);
    A[1] = fmaf(g2, x[1], f2 * A[1]);
    A[2] = fmaf(g2, x[2], f2 * A[2]);
    M1 = n1;
    M2 = n2;
  };
  for (int i = sl; i < nch; i += 2 * kOeSlots) {
    const bool two = i + kOeSlots < nch;
    const float *p = part + i * stride, *p2 = part + (two ? i + kOeSlots : i) * stride;
    const float s1[4] = {p[0], p[1], p[2], p[3]}, s2[4] = {p2[0], p2[1], p2[2], p2[3]};
    const float x1[3] = {p[4 + c], p[4 + kHeadDim + c], p[4 + 2 * kHeadDim + c]};
    const float x2[3] = {p2[4 + c], p2[4 + kHeadDim + c], p2[4 + 2 * kHeadDim + c]};
    add(s1[0], s1[1], s1[2], s1[3], x1);
    if (two) add(s2[0], s2[1], s2[2], s2[3], x2);
  }
  if (c == 0) {
    ml[sl][0] = M1;
    ml[sl][1] = L1;
    ml[sl][2] = M2;
    ml[sl][3] = L2;
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) as[sl][k][c] = A[k];
  __syncthreads();
  // every slot combines the four (in slot order), so that each thread has the head's o1 and o2
  M1 = M2 = -INFINITY;
#pragma unroll
  for (int t = 0; t < kOeSlots; ++t) {
    M1 = fmaxf(M1, ml[t][0]);
    M2 = fmaxf(M2, ml[t][2]);
  }
  L1 = L2 = A[0] = A[1] = A[2] = 0.0f;
#pragma unroll
  for (int t = 0; t < kOeSlots; ++t) {
    const float f1 = ml[t][0] == -INFINITY ? 0.0f : exp2f(ml[t][0] - M1);
    const float f2 = ml[t][2] == -INFINITY ? 0.0f : exp2f(ml[t][2] - M2);
    L1 = fmaf(f1, ml[t][1], L1);
    L2 = fmaf(f2, ml[t][3], L2);
    A[0] = fmaf(f1, as[t][0][c], A[0]);
    A[1] = fmaf(f2, as[t][1][c], A[1]);
    A[2] = fmaf(f2, as[t][2][c], A[2]);
  }
  const float o1 = L1 > 0.0f ? A[0] / L1 : 0.0f;
  const float o2 = L2 > 0.0f ? A[1] / L2 : 0.0f;
  if (sl == 0) os[c] = L2 > 0.0f ? A[2] / L2 : 0.0f;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's share of R_V
  __syncthreads();
  float o3 = 0.0f;
#pragma unroll
  for (int q = 8 * sl; q < 8 * sl + 8; ++q) {
    const float4 x = *reinterpret_cast<const float4*>(&os[4 * q]);
    const float4 r = *reinterpret_cast<const float4*>(&rl[kHeadDim * c + 4 * (q ^ (c & 31))]);
    o3 = fmaf(x.x, r.x, o3);
    o3 = fmaf(x.y, r.y, o3);
    o3 = fmaf(x.z, r.z, o3);
    o3 = fmaf(x.w, r.w, o3);
  }
  as[sl][0][c] = o3;  // read before the last barrier
  __syncthreads();
  if (sl != 0) return;
  o3 = ((as[0][0][c] + as[1][0][c]) + as[2][0][c]) + as[3][0][c];
  // do as three bf16 terms (the projection's matrix-core operands): truncation leaves each remainder
  // exact, and the third takes the last 8 significant bits, so t0 + t1 + t2 = do exactly
  const size_t plane = (size_t)a.B * a.Hq * 2 * kHeadDim;
  uint16_t* d = e.dov + ((size_t)b * a.Hq + j) * 2 * kHeadDim;
  const float dv[2] = {o2 - o1, o3 - o2};
#pragma unroll
  for (int kv = 0; kv < 2; ++kv) {
    const uint32_t b0 = __float_as_uint(dv[kv]) & 0xFFFF0000u;
    const float r1 = dv[kv] - __uint_as_float(b0);
    const uint32_t b1 = __float_as_uint(r1) & 0xFFFF0000u;
    const float r2 = r1 - __uint_as_float(b1);
    d[kv * kHeadDim + c] = (uint16_t)(b0 >> 16);
    d[plane + kv * kHeadDim + c] = (uint16_t)(b1 >> 16);
    d[2 * plane + kv * kHeadDim + c] = (uint16_t)(__float_as_uint(r2) >> 16);
  }
}

// Block (query head j, tile of kOeRowTile rows of W_O), four waves: dy[b][j][{K, V}][row] =
// do[b][j][{K, V}] . W_O[row][j * 128 ..] for every sequence, and the tile's partial statistics, on
// the bf16 matrix cores with do as three exact bf16 terms (fp32 products and accumulation, as an
// fp32 product would give): 16 x 16 x 32 steps, lane l holds A[l % 16][8 (l / 16) ..] and
// B[8 (l / 16) ..][l % 16], D[4 (l / 16) + v][l % 16] is element v of its accumulator. M: the 2B rows
// m = 2 b + {0: K, 1: V} of do, 16 at a time; N: wave w's two 16-row tiles of the block's rows; K:
// the head's 128 channels in four blocks of 32 (lane: channels 32 i + 8 (l / 16) .. + 7 of its do
// and W_O rows).
constexpr int kOeNT = kOeRowTile / 64;  // 16-row N tiles per wave
__global__ __launch_bounds__(256) void outerr_proj_kernel(OutErrArgs e, const uint16_t* __restrict__ W_o,
                                                          int d_model, float* __restrict__ dy,
                                                          float* __restrict__ spart, int ntiles) {
  const DecodeArgs& a = e.a;
  __shared__ float red[2][4][8][4];  // [M tile % 2][wave][sequence of the M tile][statistic]
  const int j = blockIdx.x, tile = blockIdx.y, tid = threadIdx.x;
  const int w = tid >> 6, l = tid & 63, li = l & 15, lk = l >> 4;
  int n[kOeNT];
  bool have[kOeNT];
  oe_bf8_t wb[kOeNT][4];
#pragma unroll
  for (int nt = 0; nt < kOeNT; ++nt) {
    n[nt] = tile * kOeRowTile + 16 * (kOeNT * w + nt) + li;  // this lane's W_O row of N tile nt
    have[nt] = n[nt] < d_model;
    const uint4* wp = reinterpret_cast<const uint4*>(W_o + (size_t)(have[nt] ? n[nt] : 0) * a.Hq * kHeadDim +
                                                     (size_t)j * kHeadDim + 8 * lk);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      wb[nt][i] = __builtin_bit_cast(oe_bf8_t, have[nt] ? wp[4 * i] : make_uint4(0, 0, 0, 0));
  }
  const int M = 2 * a.B;
  const size_t plane = (size_t)a.B * a.Hq * 2 * kHeadDim;
  // the M tile's rows of do, fetched a tile ahead, the first ones beside the weights (a call of 16 x 4,096 tokens
  // 110.3 -> 109.9 us with one barrier a tile instead of two)
  oe_bf8_t da[3][4], dn[3][4];
  auto fetch = [&](oe_bf8_t(&d)[3][4], int m0) {
    const int m = m0 + li, mc = min(m, M - 1);
    const uint32_t keep = m < M ? ~0u : 0u;
    const uint16_t* dp = e.dov + (((size_t)(mc >> 1) * a.Hq + j) * 2 + (mc & 1)) * kHeadDim + 8 * lk;
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        d[t][i] = __builtin_bit_cast(oe_bf8_t, *reinterpret_cast<const oe_u4_t*>(dp + t * plane + 32 * i) &
                                                   oe_u4_t{keep, keep, keep, keep});
  };
  fetch(dn, 0);
  for (int m0 = 0; m0 < M; m0 += 16) {
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) da[t][i] = dn[t][i];
    if (m0 + 16 < M) fetch(dn, m0 + 16);
    oe_f4_t acc[kOeNT];
#pragma unroll
    for (int nt = 0; nt < kOeNT; ++nt) acc[nt] = oe_f4_t{0.f, 0.f, 0.f, 0.f};
    // smallest term first
#pragma unroll
    for (int t = 2; t >= 0; --t)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int nt = 0; nt < kOeNT; ++nt)
          acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(da[t][i], wb[nt][i], acc[nt], 0, 0, 0);
    // acc[nt][v]: do row m0 + 4 lk + v, i.e. sequence m0 / 2 + 2 lk + v / 2, K (v even) or V (v odd)
#pragma unroll
    for (int hb = 0; hb < 2; ++hb) {
      const int b = m0 / 2 + 2 * lk + hb;
      float st[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int nt = 0; nt < kOeNT; ++nt) {
        const float yk = acc[nt][2 * hb], yv = acc[nt][2 * hb + 1];  // 0 past d_model or past the batch
        if (dy && have[nt] && b < a.B) {
          float* o = dy + ((size_t)b * a.Hq + j) * 2 * d_model;
          o[n[nt]] = yk;
          o[d_model + n[nt]] = yv;
        }
        st[0] += (yk + yv) * (yk + yv);
        st[1] += yk * yk;
        st[2] += yv * yv;
        st[3] += yk * yv;
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) st[k] = row_sum16(st[k]);
      if (li == 0)
#pragma unroll
        for (int k = 0; k < 4; ++k) red[m0 / 16 & 1][w][2 * lk + hb][k] = st[k];
    }
    __syncthreads();  // the other buffer's readers are past it too
    if (tid < 32) {
      const float(&rd)[4][8][4] = red[m0 / 16 & 1];
      const int bb = tid >> 2, k = tid & 3, b = m0 / 2 + bb;
      if (b < a.B)
        spart[(((size_t)b * a.Hq + j) * ntiles + tile) * 4 + k] =
            ((rd[0][bb][k] + rd[1][bb][k]) + rd[2][bb][k]) + rd[3][bb][k];
    }
  }
}

// Wave per (b, j): lane t sums the row tiles t, t + 64, ... in order, then a fixed butterfly over
// the lanes (deterministic).
__global__ __launch_bounds__(256) void outerr_stats_kernel(const float* __restrict__ spart, float* __restrict__ stats,
                                                           int n, int ntiles) {
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6), l = threadIdx.x & 63;
  if (i >= n) return;  // uniform over the wave
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int t = l; t < ntiles; t += 64) {
    const float4 x = *reinterpret_cast<const float4*>(spart + ((size_t)i * ntiles + t) * 4);
    s.x += x.x;
    s.y += x.y;
    s.z += x.z;
    s.w += x.w;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    s.x += __shfl_xor(s.x, off);
    s.y += __shfl_xor(s.y, off);
    s.z += __shfl_xor(s.z, off);
    s.w += __shfl_xor(s.w, off);
  }
  if (l == 0) {  // the caller's stats need only 4-byte alignment
    stats[(size_t)i * 4] = s.x;
    stats[(size_t)i * 4 + 1] = s.y;
    stats[(size_t)i * 4 + 2] = s.z;
    stats[(size_t)i * 4 + 3] = s.w;
  }
}

template <int NG>
static void launch_oe_scan(const OutErrArgs& e, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  const DecodeArgs& a = e.a;
  dim3 grid(a.n_chunks, a.H, a.B);
  if (a.gq <= 1)
    hipExtLaunchKernelGGL((outerr_scan_kernel<1, NG>), grid, dim3(256), 0, s, ev0, ev1, 0, e);
  else if (a.gq <= 2)
    hipExtLaunchKernelGGL((outerr_scan_kernel<2, NG>), grid, dim3(256), 0, s, ev0, ev1, 0, e);
  else if (a.gq <= 4)
    hipExtLaunchKernelGGL((outerr_scan_kernel<4, NG>), grid, dim3(256), 0, s, ev0, ev1, 0, e);
  else if (a.gq <= 8)
    hipExtLaunchKernelGGL((outerr_scan_kernel<8, NG>), grid, dim3(256), 0, s, ev0, ev1, 0, e);
  else
    hipExtLaunchKernelGGL((outerr_scan_kernel<16, NG>), grid, dim3(256), 0, s, ev0, ev1, 0, e);
}

hipError_t launch_output_error(const OutErrArgs& e, const uint16_t* W_o, int d_model, float* stats, float* dy,
                               hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  const DecodeArgs& a = e.a;
  hipError_t err = launch_qrot(a, s);
  if (err != hipSuccess) return err;
  if (a.groups == 1)
    launch_oe_scan<1>(e, s, ev0, ev1);
  else
    launch_oe_scan<4>(e, s, ev0, ev1);
  hipLaunchKernelGGL(outerr_merge_kernel, dim3(a.B, a.Hq), dim3(kHeadDim * kOeSlots), 0, s, e);
  const int ntiles = (d_model + kOeRowTile - 1) / kOeRowTile;
  hipLaunchKernelGGL(outerr_proj_kernel, dim3(a.Hq, ntiles), dim3(256), 0, s, e, W_o, d_model, dy, e.spart,
                     ntiles);
  const int n = a.B * a.Hq;
  hipLaunchKernelGGL(outerr_stats_kernel, dim3((n + 3) / 4), dim3(256), 0, s, e.spart, stats, n, ntiles);
  return hipGetLastError();
}

}  // namespace int2kv

// OptR offline calibration on the GPU (Sec. 4.2 - 4.5; Algorithm 1 of the appendix), in fp64.
//
// Per KV head h, with R = R^0 exp(A - A^T):
//   rows:        x_s = k_s - mu (keys) or v_s (values), bf16 inputs, exact in fp64
//   rotation:    z_s = x_s R, rounded to fp32 and quantized by the cache's quantizer (codes, fp16
//                scale and zero); zhat_s = code * s + z (exact); mask = element inside its group's
//                clipped range [c mn, c mx] (the straight-through estimator of eq:OptR_ste)
//   effective:   xeff_s = zhat_s R^T
//   key loss:    rows (t, j) over the final n_last positions; logits over s <= t with xeff for
//                tokens read from INT2 (sink <= s <= t - recent) and x otherwise;
//                KL(p || p^K) + lambda ||(p^K - p)^T V W_{O,j}^T||^2 / d_model, averaged over rows,
//                the output term as dO^T M_j dO with the Gram matrix M_j = W_{O,j}^T W_{O,j}
//   value loss:  ||p^Khat^T (Veff - V) W_{O,j}^T||^2 / d_model under fixed key probabilities
// Gradients by hand: dL/dlogit, then dL/dxeff (per token, summed over its rows), dL/dzhat =
// G R masked, dL/dR = X^T (mask . G R) + G^T Zhat, dL/dE = R0^T dL/dR for E = exp(S), dL/dS as the
// Frechet derivative of exp at S^T applied to dL/dE (the upper-right block of the exponential of
// [[S^T, dL/dE], [0, S^T]]), and dL/dA = dL/dS - dL/dS^T.
// exp: a Taylor polynomial of S 2^-j by column blocks, the last of the j doublings as squarings (see the matrix functions
// below).
#include <vector>

#include "common.h"
#include "kernels.h"

namespace int2kv {

namespace {

constexpr int kD = kHeadDim;
constexpr int kMat = kD * kD;

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

// fp64 matrix-core step D += A B for 16 x 4 by 4 x 16 operands: lane l holds A[l % 16][l / 16] and
// B[l / 16][l % 16]; D[l / 16 + 4 v][l % 16] is element v of its accumulator.
__device__ __forceinline__ f64x4 mfma64(double a, double b, f64x4 d) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, d, 0, 0, 0);
}
constexpr double kInvSqrtD = 0.08838834764831845;  // 1 / sqrt(128)

__device__ __forceinline__ double bf16d(uint16_t b) { return (double)__uint_as_float((uint32_t)b << 16); }

__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
  return x;
}

// block-wide reductions over blockDim.x threads (a multiple of 64, at most 1024); red: 16 doubles
__device__ double block_sum(double x, double* red) {
  x = wave_sum(x);
  const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = x;
  __syncthreads();
  double t = 0.0;
  for (int i = 0; i < nw; ++i) t += red[i];  // fixed order: deterministic
  return t;
}

// Offset of token s, KV head h in the per-head rows of the workspace ([H, T, 128]: each head's
// rows contiguous), as against the traces' [T, H, 128].
__device__ __forceinline__ size_t hrow(const CalSet& S, int s, int h) { return ((size_t)h * S.T + s) * kD; }

__device__ __forceinline__ bool int2_token(int s, int t, int sink, int recent) {
  return s >= sink && s <= t - recent;
}

__device__ __forceinline__ void bf16x8_to_f64(uint4 u, double (&d)[8]) {
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    d[2 * i] = (double)__uint_as_float(w[i] << 16);
    d[2 * i + 1] = (double)__uint_as_float(w[i] & 0xFFFF0000u);
  }
}

// 16 bytes of an input that has no alignment beyond its type's (q, R^0, A and W_O; one 16-byte load all the same).
template <class V, class T>
__device__ __forceinline__ V load16(const T* p) {
  static_assert(sizeof(V) == 16, "one 16-byte piece");
  V v;
  __builtin_memcpy(&v, p, sizeof(v));
  return v;
}

// ---------------------------------------------------------------------------------------------
// Rows times a 128 x 128 matrix on the fp64 matrix cores, as out^T = Bm^T y^T: M = the 128 output
// channels (eight 16-row tiles), N = the wave's 16 rows y (lane l holds row l % 16), K = the 128
// input channels. The lane's B operand at step s is ya[s] = y[row][k(s)], k(4 q + d) = 32 (l / 16) +
// 4 q + d (KMAP 0: each lane reads 32 contiguous channels of its row) or 16 q + 4 d + l / 16 (KMAP 1:
// the channels this layout leaves in a lane, see below); Bm goes through Bs (LDS, kBsRows rows x
// kBsStride) kBsRows rows at a time. Result element v of acc[ct]: channel 16 ct + l / 16 + 4 v of row
// l % 16. Contains block barriers: every thread of the block calls it.
// The next kBsRows rows of Bm are fetched into registers while the matrix cores run on the staged ones.
constexpr int kBsStride = 132;  // doubles per staged row
constexpr int kBsRows = 32;     // rows staged at a time: 64 matrix-core steps per wave hide the next fetch
constexpr int kMatThreads = 256;
template <int KMAP>
__device__ __forceinline__ void mat_t_rows(const double (&ya)[32], const double* __restrict__ Bm, double* Bs,
                                           f64x4 (&acc)[8]) {
  const int tid = threadIdx.x, l = tid & 63, li = l & 15, lk = l >> 4;
  constexpr int kPer = kBsRows * kD / (2 * kMatThreads);  // 16-byte pieces per thread
  f64x2 next[kPer];
  auto fetch = [&](int q) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int e = tid + kMatThreads * u, rr = e / (kD / 2), col = 2 * (e % (kD / 2));
      const int krow = KMAP == 0 ? 32 * (rr >> 3) + 8 * q + (rr & 7) : kBsRows * q + rr;
      next[u] = *reinterpret_cast<const f64x2*>(Bm + krow * kD + col);
    }
  };
  fetch(0);
#pragma unroll
  for (int q = 0; q < kD / kBsRows; ++q) {  // unrolled: ya is indexed by q
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int e = tid + kMatThreads * u;
      *reinterpret_cast<f64x2*>(Bs + (e / (kD / 2)) * kBsStride + 2 * (e % (kD / 2))) = next[u];
    }
    __syncthreads();
    if (q + 1 < kD / kBsRows) fetch(q + 1);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const double b = ya[8 * q + e];
      const double* br = Bs + (KMAP == 0 ? 8 * lk + e : 16 * (e >> 2) + 4 * (e & 3) + lk) * kBsStride + li;
#pragma unroll
      for (int ct = 0; ct < 8; ++ct) acc[ct] = mfma64(br[16 * ct], b, acc[ct]);
    }
  }
}

// y's 32 channels 32 (l / 16) .. + 31 of a row of fp64 storage (zero when !ok).
__device__ __forceinline__ void row_operand_f64(const double* row, bool ok, double (&ya)[32]) {
  const double2* r2 = reinterpret_cast<const double2*>(row + 32 * ((threadIdx.x & 63) >> 4));
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const double2 x = ok ? r2[i] : make_double2(0.0, 0.0);
    ya[2 * i] = x.x;
    ya[2 * i + 1] = x.y;
  }
}

// Rotation and quantization: zhat (the dequantized codes of (x - mu) R, fp64), the in-range mask, and
// the effective rows zhat R^T, of the tokens some query reads from INT2 (S.units; the rest of those
// buffers is never read into a result: with the paper's windows about two thirds of the tokens).
// Block (four units, KV head), wave w: unit 4 bx + w (one token per lane l % 16), every lane group
// l / 16 a quarter of the channels. A token's quantization group is spread over its four lane
// groups: min / max through two cross-group exchanges. 77 -> 35 us (every token, 16 staged rows before).
__global__ __launch_bounds__(kMatThreads) void cal_rotq_kernel(CalSet S, CalCfg c, int value) {
  __shared__ __align__(16) double Bs[kBsRows * kBsStride];
  const int h = blockIdx.y, tid = threadIdx.x, w = tid >> 6, l = tid & 63, li = l & 15, lk = l >> 4;
  const int4 unit = 4 * (int)blockIdx.x + w < S.nunits ? S.units[4 * blockIdx.x + w] : make_int4(0, 0, 0, 0);
  const int tok = unit.x + li;
  const bool ok = li < unit.y;
  const size_t xo = ((size_t)(ok ? tok : 0) * c.H + h) * kD, rowo = hrow(S, ok ? tok : 0, h);
  const uint16_t* X = value ? S.v : S.k;
  double ya[32];
  {
    const uint4* xr = reinterpret_cast<const uint4*>(X + xo + 32 * lk);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      double d[8];
      bf16x8_to_f64(ok ? xr[g] : make_uint4(0, 0, 0, 0), d);
#pragma unroll
      for (int i = 0; i < 8; ++i)
        ya[8 * g + i] = ok ? d[i] - (value ? 0.0 : (double)c.mu[h * kD + 32 * lk + 8 * g + i]) : 0.0;
    }
  }
  f64x4 acc[8];
#pragma unroll
  for (int ct = 0; ct < 8; ++ct) acc[ct] = f64x4{0.0, 0.0, 0.0, 0.0};
  mat_t_rows<0>(ya, c.R + (size_t)h * kMat, Bs, acc);  // z = (x - mu) R: channel 16 ct + lk + 4 v
  const float clip = value ? c.clip_v : c.clip_k;
  // groups: 32 channels (tiles 2 g, 2 g + 1) or all 128 (one group)
  const int ng = c.ng, tpg = 8 / ng;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    if (g >= ng) break;
    float mn = INFINITY, mx = -INFINITY;
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) {
      if (ct / tpg != g) continue;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float x = (float)acc[ct][v];
        mn = fminf(mn, x);
        mx = fmaxf(mx, x);
      }
    }
    mn = fminf(mn, __shfl_xor(mn, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mn = fminf(mn, __shfl_xor(mn, 32));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    uint32_t s_bits, z_bits;
    float zf, inv;
    int2_group_params(mn, mx, clip, s_bits, z_bits, zf, inv);
    const double sd = (double)__half2float(__ushort_as_half((unsigned short)s_bits));
    float lo = mn, hi = mx;
    if (clip != 1.0f) {
#pragma clang fp contract(off)
      lo = clip * mn;
      hi = clip * mx;
    }
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) {
      if (ct / tpg != g) continue;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float x = (float)acc[ct][v];
        const double zh = (double)int2_code(x, zf, inv) * sd + (double)zf;
        ya[4 * ct + v] = zh;  // the B operand of the second product (KMAP 1)
        if (ok) {
          const size_t o = rowo + 16 * ct + lk + 4 * v;
          S.zhat[o] = zh;
          S.mask[o] = (x >= lo && x <= hi) ? 1 : 0;
        }
      }
    }
  }
#pragma unroll
  for (int ct = 0; ct < 8; ++ct) acc[ct] = f64x4{0.0, 0.0, 0.0, 0.0};
  mat_t_rows<1>(ya, c.Rt + (size_t)h * kMat, Bs, acc);  // effective rows zhat R^T
  if (ok)
#pragma unroll
    for (int ct = 0; ct < 8; ++ct)
#pragma unroll
      for (int v = 0; v < 4; ++v) S.xeff[rowo + 16 * ct + lk + 4 * v] = acc[ct][v];
}

// ---------------------------------------------------------------------------------------------
// The objectives over row tiles.

// The tile kernels take a tile of up to kTileRows rows: 16 / G_q consecutive query positions of
// one sequence with all their query heads (tiles[i] = (sequence, first row, rows, position of the
// first row)), so each key and value row is loaded once for the whole tile. Row r of a tile is
// position t_first + r / G_q, query head h G_q + r % G_q. The row x token and row x channel
// products run on the fp64 matrix cores with the tile's 16 rows as the M dimension.
constexpr int kTileRows = 16;
constexpr int kTileThreads = 256;  // four waves; one token per thread in the softmax passes
constexpr int kDlStride = 18;      // doubles per token of the staged row weights (16-byte rows)


// Row operand of a tile in matrix-core form: lane (li, lk) holds x[row li][32 lk + m], m = 0..31, for
// the contraction over 128 channels taken as 32 steps m whose 4-deep slices are channels 32 k + m
// (k = 0..3); rows li >= nr are zero. From bf16 (queries) or fp64 (row vectors) storage.
__device__ __forceinline__ void rows_operand_bf16(const uint16_t* row, bool ok, int lk, double (&x)[32]) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    double d[8];
    bf16x8_to_f64(ok ? load16<uint4>(row + 32 * lk + 8 * g) : make_uint4(0, 0, 0, 0), d);
#pragma unroll
    for (int i = 0; i < 8; ++i) x[8 * g + i] = d[i];
  }
}

// Logits of 16 rows against the 16 tokens of a tile (token li of this lane's B operand): acc +=
// x . y_token with y the token's bf16 row; the same slice convention as rows_operand_*.
__device__ __forceinline__ f64x4 dot_tokens_bf16(const double (&x)[32], const uint16_t* yrow, bool ok, int lk) {
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    double d[8];
    bf16x8_to_f64(ok ? *reinterpret_cast<const uint4*>(yrow + 32 * lk + 8 * g) : make_uint4(0, 0, 0, 0), d);
#pragma unroll
    for (int i = 0; i < 8; ++i) acc = mfma64(x[8 * g + i], d[i], acc);
  }
  return acc;
}
__device__ __forceinline__ f64x4 dot_tokens_f64(const double (&x)[32], const double* yrow, bool ok, int lk) {
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  const double2* y2 = reinterpret_cast<const double2*>(yrow + 32 * lk);
#pragma unroll
  for (int g = 0; g < 16; ++g) {
    const double2 y = ok ? y2[g] : make_double2(0.0, 0.0);
    acc = mfma64(x[2 * g], y.x, acc);
    acc = mfma64(x[2 * g + 1], y.y, acc);
  }
  return acc;
}

// Row x channel accumulation: acc[t] (t = 0..7) += A B with A[row li][token lk] = a and
// B[token lk][column li] = y[t], the token's channel 8 li + t. Result element v of acc[t]: row
// lk + 4 v, channel 8 li + t.
__device__ __forceinline__ void acc_channels(f64x4 (&acc)[8], double a, const double (&y)[8]) {
#pragma unroll
  for (int t = 0; t < 8; ++t) acc[t] = mfma64(a, y[t], acc[t]);
}

// Sums the four waves' channel accumulators in the fixed order (w0 + w2) + (w1 + w3) through buf
// (32 KiB of LDS, free on entry) and stores rows r < nr at out + r 128 (row lk + 4 v, channel 8 li + t),
// plus add_w[r] times row r of add when add is given (add_w visible to wave 0 at entry).
__device__ __forceinline__ void sum_waves_store(f64x4 (&acc)[8], double* buf, double* out, int nr,
                                                const double* add = nullptr, const double* add_w = nullptr) {
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, li = l & 15, lk = l >> 4;
  __syncthreads();
  if (w >= 2)
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) buf[((w - 2) * 32 + 4 * t + v) * 64 + l] = acc[t][v];
  __syncthreads();
  if (w < 2)
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[t][v] += buf[(w * 32 + 4 * t + v) * 64 + l];
  __syncthreads();
  if (w == 1)
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) buf[(4 * t + v) * 64 + l] = acc[t][v];
  __syncthreads();
  if (w == 0)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = lk + 4 * v;
      double o[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) o[t] = acc[t][v] + buf[(4 * t + v) * 64 + l];
      if (r < nr && add)
#pragma unroll
        for (int t = 0; t < 8; ++t) o[t] = fma(add_w[r], add[(size_t)r * kD + 8 * li + t], o[t]);
      if (r < nr) {
        double2* dst = reinterpret_cast<double2*>(out + (size_t)r * kD + 8 * li);
#pragma unroll
        for (int i = 0; i < 4; ++i) dst[i] = make_double2(o[2 * i], o[2 * i + 1]);
      }
    }
}

// Row maxima from the matrix-core layout (m4[v]: this lane's value for row lk + 4 v): over the 16
// lanes of each lk group, then over the four waves through red4 ([4][16] doubles). Returns the
// maxima of rows 4 w .. 4 w + 3, the rows wave w owns in the softmax passes.
__device__ __forceinline__ void rows_max(const double (&m4)[4], double* red4, double (&m)[4]) {
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, li = l & 15, lk = l >> 4;
  double x[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    x[v] = m4[v];
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) x[v] = fmax(x[v], __shfl_xor(x[v], off));
  }
  __syncthreads();
  if (li == 0)
#pragma unroll
    for (int v = 0; v < 4; ++v) red4[w * 16 + lk + 4 * v] = x[v];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = 4 * w + i;
    m[i] = fmax(fmax(red4[r], red4[16 + r]), fmax(red4[32 + r], red4[48 + r]));
  }
}

// The tile's 4-token steps of a 256-token chunk for wave w: tokens 64 w + k4 + lk, k4 = 0, 4, ..., 60,
// those below end.

// The rotation-independent part of the key objective, once per set: for every row the full-precision
// logits f_s = q.(k_s - mu)/sqrt(d) over its tokens s <= t_r (fc; q.(k - mu) = q.k - q.mu with q.mu once
// per row), p = softmax(f) (pc), lse_f and LW = log-sum-exp of f over the row's tokens held in BF16
// windows (-inf when none) (rc), and W~ = sum over those tokens of exp(f_s - LW) v_s (wt). A window
// token keeps g_s = f_s under every rotation, so the key forward needs only these sums for them.
// Block (tile, KV head), the layout of the key forward.
__global__ __launch_bounds__(kTileThreads) void cal_const_kernel(CalSet S, CalCfg c) {
  constexpr int R = kTileRows;
  __shared__ double qmu[R];
  __shared__ double red4[4 * R];
  __shared__ __align__(16) double dl[kTileThreads * kDlStride];
  const int h = blockIdx.y, tid = threadIdx.x, gq = c.gq;
  const int w = tid >> 6, l = tid & 63, li = l & 15, lk = l >> 4;
  const int4 tile = S.tiles[blockIdx.x];
  const CalSeq sq = S.seqs[tile.x];
  const int row0 = tile.y, nr = tile.z, tf = tile.w, a0 = sq.start, L = sq.len;
  const int tmax = tf + (nr - 1) / gq;
  const size_t pb = (size_t)h * S.pelems + sq.p0 + (size_t)(row0 - sq.row0) * L;  // row r at + r L
  double *fcb = S.fc + pb, *pcb = S.pc + pb;
  double qa[32];
  rows_operand_bf16(S.q + ((size_t)(a0 + tf + li / gq) * c.Hq + h * gq + li % gq) * kD, li < nr, lk, qa);
  {
    double t = 0.0;
#pragma unroll
    for (int m = 0; m < 32; ++m) t = fma(qa[m], (double)c.mu[h * kD + 32 * lk + m], t);
    t += __shfl_xor(t, 16);
    t += __shfl_xor(t, 32);
    if (w == 0 && lk == 0) qmu[li] = t;
  }
  __syncthreads();
  double m4f[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) m4f[v] = -INFINITY;
  for (int tt = w; 16 * tt <= tmax; tt += 4) {
    const int s = 16 * tt + li;
    const bool ok = s <= tmax;
    const f64x4 af = dot_tokens_bf16(qa, S.k + ((size_t)(a0 + s) * c.H + h) * kD, ok, lk);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = lk + 4 * v, tr = tf + r / gq;
      if (r < nr && s <= tr) {
        const double f = (af[v] - qmu[r]) * kInvSqrtD;
        fcb[(size_t)r * L + s] = f;
        m4f[v] = fmax(m4f[v], f);
      }
    }
  }
  const int rb = 4 * w;
  double mf[4];
  rows_max(m4f, red4, mf);  // its barriers also make the logits visible to the whole block
  int tr4[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) tr4[i] = rb + i < nr ? tf + (rb + i) / gq : -1;
  double zf[4], zw[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) zf[i] = zw[i] = 0.0;
  for (int s = l; s <= tmax; s += 64)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (s > tr4[i]) continue;
      const double e = exp(fcb[(size_t)(rb + i) * L + s] - mf[i]);
      zf[i] += e;
      if (!int2_token(s, tr4[i], c.sink, c.recent)) zw[i] += e;
    }
  double lse[4], lw[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    zf[i] = wave_sum(zf[i]);
    zw[i] = wave_sum(zw[i]);
    lse[i] = mf[i] + log(zf[i]);
    lw[i] = zw[i] > 0.0 ? mf[i] + log(zw[i]) : -INFINITY;
  }
  // p, and W~ from the window tokens' weights exp(f - LW) staged in LDS by 256-token chunk
  f64x4 acc[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
  for (int base = 0; base <= tmax; base += kTileThreads) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int j = 64 * q + l, s = base + j;
      double d[4] = {0.0, 0.0, 0.0, 0.0};
      if (s <= tmax) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (s > tr4[i]) continue;
          const size_t o = (size_t)(rb + i) * L + s;
          const double f = fcb[o];
          pcb[o] = exp(f - lse[i]);
          if (!int2_token(s, tr4[i], c.sink, c.recent)) d[i] = exp(f - lw[i]);  // lw finite: a window token
        }
      }
      double2* dj = reinterpret_cast<double2*>(dl + j * kDlStride + rb);
      dj[0] = make_double2(d[0], d[1]);
      dj[1] = make_double2(d[2], d[3]);
    }
    __syncthreads();
    const int end = min(kTileThreads, tmax + 1 - base);
    for (int k4 = 0; k4 < 64 && 64 * w + k4 < end; k4 += 4) {
      const int j = 64 * w + k4 + lk;
      const bool ok = j < end;
      double y[8];
      bf16x8_to_f64(ok ? *reinterpret_cast<const uint4*>(S.v + ((size_t)(a0 + base + j) * c.H + h) * kD + 8 * li)
                       : make_uint4(0, 0, 0, 0),
                    y);
      acc_channels(acc, ok ? dl[j * kDlStride + li] : 0.0, y);
    }
    __syncthreads();
  }
  sum_waves_store(acc, dl, S.wt + ((size_t)h * S.nrows + row0) * kD, nr);
  if (l == 0)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (rb + i < nr) {
        S.rc[((size_t)h * S.nrows + row0 + rb + i) * 2] = lse[i];
        S.rc[((size_t)h * S.nrows + row0 + rb + i) * 2 + 1] = lw[i];
      }
}

// Forward of the key objective on a tile, with the rotation-independent part from cal_const_kernel.
// Logits g = q.x~/sqrt(d) on the tokens read from INT2 (elsewhere g = f); the softmax p^K over all
// tokens, the window tokens entering as one term exp(LW - mk); KL(p || p^K) = sum_INT2 p (f - g) +
// lse_k - lse_f into lrow (p sums to one); p^K on the INT2 tokens into pd (the rest of pd stays zero);
// dO = sum_INT2 (p^K - p) v + (exp(LW - lse_k) - exp(LW - lse_f)) W~ into wrow and exp(LW - lse_k)
// into erow. With probs_only: pd only. Block (tile, KV head); every pass covers only the tokens
// s_lo .. s_hi some row of the tile reads from INT2.
__global__ __launch_bounds__(kTileThreads) void cal_pos_fwd_kernel(CalSet S, CalCfg c, int probs_only) {
  constexpr int R = kTileRows;
  __shared__ double red4[4 * R];
  __shared__ double dw[R];  // exp(LW - lse_k) - exp(LW - lse_f) per row
  __shared__ __align__(16) double dl[kTileThreads * kDlStride];
  const int h = blockIdx.y, tid = threadIdx.x, gq = c.gq;
  const int w = tid >> 6, l = tid & 63, li = l & 15, lk = l >> 4;
  const int4 tile = S.tiles[blockIdx.x];
  const CalSeq sq = S.seqs[tile.x];
  const int row0 = tile.y, nr = tile.z, tf = tile.w, a0 = sq.start, L = sq.len;
  const int tmax = tf + (nr - 1) / gq;
  const int s_lo = c.sink, s_hi = tmax - c.recent;
  const size_t pb = (size_t)h * S.pelems + sq.p0 + (size_t)(row0 - sq.row0) * L;  // row r at + r L
  double* pdb = S.pd + pb;
  const double *fcb = S.fc + pb, *pcb = S.pc + pb;
  double qa[32];
  rows_operand_bf16(S.q + ((size_t)(a0 + tf + li / gq) * c.Hq + h * gq + li % gq) * kD, li < nr, lk, qa);
  // logits on the INT2 tokens: wave w takes the 16-token tiles w, w + 4, ... that meet s_lo .. s_hi;
  // lane (li, lk) ends with rows lk + 4 v of token 16 tt + li
  double m4k[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) m4k[v] = -INFINITY;
  for (int tt = w; 16 * tt <= s_hi; tt += 4) {
    if (16 * tt + 15 < s_lo) continue;  // uniform over the wave
    const int s = 16 * tt + li;
    const bool ok = s <= tmax;
    const f64x4 ak = dot_tokens_f64(qa, S.xeff + hrow(S, ok ? a0 + s : a0, h), ok, lk);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = lk + 4 * v, tr = tf + r / gq;
      if (r < nr && int2_token(s, tr, c.sink, c.recent)) {
        const double g = ak[v] * kInvSqrtD;
        pdb[(size_t)r * L + s] = g;
        m4k[v] = fmax(m4k[v], g);
      }
    }
  }
  // softmax passes: wave w owns rows rb .. rb + 3 (rb = 4 w), lane l the tokens s_lo + l, + 64, ...
  const int rb = 4 * w;
  double mk[4];
  rows_max(m4k, red4, mk);  // its barriers also make the logits visible to the whole block
  int tr4[4];
  double lsf[4], lw[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const bool ok = rb + i < nr;
    tr4[i] = ok ? tf + (rb + i) / gq : -1;
    const size_t ro = ((size_t)h * S.nrows + row0 + (ok ? rb + i : 0)) * 2;
    lsf[i] = S.rc[ro];
    lw[i] = S.rc[ro + 1];
    mk[i] = fmax(mk[i], lw[i]);  // finite: a row has INT2 or window tokens
  }
  // e = exp(g - mk) in place of the logits, the row sums and sum_INT2 p (f - g)
  double zk[4], klp[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) zk[i] = klp[i] = 0.0;
  for (int s = s_lo + l; s <= s_hi; s += 64)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (tr4[i] < 0 || !int2_token(s, tr4[i], c.sink, c.recent)) continue;
      const size_t o = (size_t)(rb + i) * L + s;
      const double g = pdb[o], e = exp(g - mk[i]);
      pdb[o] = e;  // this lane's own elements
      zk[i] += e;
      klp[i] = fma(pcb[o], fcb[o] - g, klp[i]);
    }
  double kl[4], er[4], rden[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    zk[i] = wave_sum(zk[i]);
    klp[i] = wave_sum(klp[i]);
    const bool win = lw[i] != -INFINITY;
    const double den = zk[i] + (win ? exp(lw[i] - mk[i]) : 0.0);
    const double lsk = mk[i] + log(den);
    kl[i] = klp[i] + (lsk - lsf[i]);
    er[i] = win ? exp(lw[i] - lsk) : 0.0;
    if (l == 0 && rb + i < nr) dw[rb + i] = er[i] - (win ? exp(lw[i] - lsf[i]) : 0.0);
    rden[i] = 1.0 / den;
  }
  // p^K = e / den on the INT2 tokens by 256-token chunk (four tokens per lane); dO over them from the
  // differences p^K - p staged in LDS
  f64x4 acc[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
  for (int base = s_lo; base <= s_hi; base += kTileThreads) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int j = 64 * q + l, s = base + j;
      double d[4] = {0.0, 0.0, 0.0, 0.0};
      if (s <= s_hi) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (tr4[i] < 0 || !int2_token(s, tr4[i], c.sink, c.recent)) continue;
          const size_t o = (size_t)(rb + i) * L + s;
          const double pk = pdb[o] * rden[i];
          pdb[o] = pk;
          d[i] = pk - pcb[o];
        }
      }
      if (!probs_only) {
        double2* dj = reinterpret_cast<double2*>(dl + j * kDlStride + rb);
        dj[0] = make_double2(d[0], d[1]);
        dj[1] = make_double2(d[2], d[3]);
      }
    }
    if (probs_only) continue;  // uniform
    __syncthreads();
    const int end = min(kTileThreads, s_hi + 1 - base);
    for (int k4 = 0; k4 < 64 && 64 * w + k4 < end; k4 += 4) {
      const int j = 64 * w + k4 + lk;
      const bool ok = j < end;
      double y[8];
      bf16x8_to_f64(ok ? *reinterpret_cast<const uint4*>(S.v + ((size_t)(a0 + base + j) * c.H + h) * kD + 8 * li)
                       : make_uint4(0, 0, 0, 0),
                    y);
      acc_channels(acc, ok ? dl[j * kDlStride + li] : 0.0, y);
    }
    __syncthreads();
  }
  if (probs_only) return;  // uniform
  sum_waves_store(acc, dl, S.wrow + ((size_t)h * S.nrows + row0) * kD, nr, S.wt + ((size_t)h * S.nrows + row0) * kD,
                  dw);  // + dw W~ per row
  if (l == 0)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (rb + i < nr) {
        S.lrow[(size_t)h * S.nrows + row0 + rb + i] = kl[i];
        S.erow[(size_t)h * S.nrows + row0 + rb + i] = er[i];
      }
}

// Value objective on a tile: dO_V = sum_s p^K-hat_s (v~_s - v_s) into wrow (pd holds p^K-hat on the
// tokens read from INT2, 0 elsewhere). Block (tile, KV head); pd is staged through LDS by token chunk
// over the tokens s_lo .. s_hi some row of the tile reads from INT2.
__global__ __launch_bounds__(kTileThreads) void cal_pos_val_kernel(CalSet S, CalCfg c) {
  constexpr int R = kTileRows;
  __shared__ __align__(16) double dl[kTileThreads * kDlStride];
  const int h = blockIdx.y, tid = threadIdx.x, gq = c.gq;
  const int w = tid >> 6, l = tid & 63, li = l & 15, lk = l >> 4;
  const int4 tile = S.tiles[blockIdx.x];
  const CalSeq sq = S.seqs[tile.x];
  const int row0 = tile.y, nr = tile.z, tf = tile.w, a0 = sq.start, L = sq.len;
  const int tmax = tf + (nr - 1) / gq;
  const int s_lo = c.sink, s_hi = tmax - c.recent;
  const double* pdb = S.pd + (size_t)h * S.pelems + sq.p0 + (size_t)(row0 - sq.row0) * L;
  f64x4 acc[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
  for (int base = s_lo; base <= s_hi; base += kTileThreads) {
    const int end = min(kTileThreads, s_hi + 1 - base);
    for (int e = tid; e < R * kTileThreads; e += kTileThreads) {
      const int r = e / kTileThreads, j = e % kTileThreads;
      dl[j * kDlStride + r] = r < nr && j < end ? pdb[(size_t)r * L + base + j] : 0.0;
    }
    __syncthreads();
    for (int k4 = 0; k4 < 64 && 64 * w + k4 < end; k4 += 4) {
      const int j = 64 * w + k4 + lk;
      const bool ok = j < end;
      const size_t o = ((size_t)(a0 + base + j) * c.H + h) * kD + 8 * li;
      double y[8];
      bf16x8_to_f64(ok ? *reinterpret_cast<const uint4*>(S.v + o) : make_uint4(0, 0, 0, 0), y);
      const double2* x2 = reinterpret_cast<const double2*>(S.xeff + hrow(S, ok ? a0 + base + j : a0, h) + 8 * li);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const double2 x = ok ? x2[i] : make_double2(0.0, 0.0);
        y[2 * i] = x.x - y[2 * i];
        y[2 * i + 1] = x.y - y[2 * i + 1];
      }
      acc_channels(acc, ok ? dl[j * kDlStride + li] : 0.0, y);
    }
    __syncthreads();
  }
  sum_waves_store(acc, dl, S.wrow + ((size_t)h * S.nrows + row0) * kD, nr);
}

// u = M_j dO for the rows of query head j (M_j = W_{O,j}^T W_{O,j}, symmetric), E = dO . u / d_model.
// Keys: urow = u, lrow += lambda E. Values: wrow = 2 u / (d_model rows), lrow = E. Block (query head j,
// 64 positions), the layout of the rotation kernel with positions as rows (a row's four lane groups
// are in one wave, each reads dO at its own output channels before writing them).
constexpr int kUTile = 64;
__global__ __launch_bounds__(kMatThreads) void cal_u_kernel(CalSet S, CalCfg c, int value) {
  __shared__ __align__(16) double Bs[kBsRows * kBsStride];
  const int j = blockIdx.x, h = j / c.gq, jj = j % c.gq, tid = threadIdx.x;
  const int w = tid >> 6, l = tid & 63, li = l & 15, lk = l >> 4;
  const int npos = S.nrows / c.gq, pp = blockIdx.y * kUTile + 16 * w + li;
  const bool ok = pp < npos;
  const size_t row = (size_t)h * S.nrows + (size_t)(ok ? pp : 0) * c.gq + jj;
  double ya[32];
  row_operand_f64(S.wrow + row * kD, ok, ya);
  f64x4 acc[8];
#pragma unroll
  for (int ct = 0; ct < 8; ++ct) acc[ct] = f64x4{0.0, 0.0, 0.0, 0.0};
  mat_t_rows<0>(ya, c.gram + (size_t)j * kMat, Bs, acc);
  double e = 0.0;
  if (ok)
#pragma unroll
    for (int ct = 0; ct < 8; ++ct)
#pragma unroll
      for (int v = 0; v < 4; ++v) e = fma(S.wrow[row * kD + 16 * ct + lk + 4 * v], acc[ct][v], e);
  e += __shfl_xor(e, 16);
  e += __shfl_xor(e, 32);
  if (!ok) return;
  const double dm = (double)c.dm;
#pragma unroll
  for (int ct = 0; ct < 8; ++ct)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const size_t o = row * kD + 16 * ct + lk + 4 * v;
      if (value)
        S.wrow[o] = 2.0 * acc[ct][v] / (dm * (double)S.nrows);
      else
        S.urow[o] = acc[ct][v];
    }
  if (lk == 0) {
    if (value)
      S.lrow[row] = e / dm;
    else
      S.lrow[row] += c.lam * e / dm;
  }
}

// Logit gradients of the key objective on a tile: G_s = 2 u . v_s / d_model, gbar = sum over all tokens of
// p^K_s G_s (the window tokens as exp(LW - lse_k) 2 u . W~ / d_model), and on the tokens read from INT2
// pd = ((p^K - p) + lambda p^K (G - gbar)) / rows (zero elsewhere, untouched). Block (tile, KV head);
// u . v_s on the fp64 matrix cores (16-token tiles per wave) over the INT2 span s_lo .. s_hi only.
__global__ __launch_bounds__(kTileThreads) void cal_pos_grad_kernel(CalSet S, CalCfg c) {
  constexpr int R = kTileRows;
  __shared__ double red[16 * R];
  __shared__ double gbw[R];  // window part of gbar per row
  const int h = blockIdx.y, tid = threadIdx.x, gq = c.gq;
  const int w = tid >> 6, l = tid & 63, li = l & 15, lk = l >> 4;
  const int4 tile = S.tiles[blockIdx.x];
  const CalSeq sq = S.seqs[tile.x];
  const int row0 = tile.y, nr = tile.z, tf = tile.w, a0 = sq.start, L = sq.len;
  const int tmax = tf + (nr - 1) / gq;
  const int s_lo = c.sink, s_hi = tmax - c.recent;
  const size_t pb = (size_t)h * S.pelems + sq.p0 + (size_t)(row0 - sq.row0) * L;
  double* pdb = S.pd + pb;
  double* pfb = S.pf + pb;
  const double* pcb = S.pc + pb;
  const double* urw = S.urow + ((size_t)h * S.nrows + row0) * kD;
  const double two_dm = 2.0 / (double)c.dm;
  {
    // u . W~ for row tid / 16, eight channels per lane, reduced over the row's 16 lanes
    const int r = tid >> 4, c8 = 8 * (tid & 15);
    double d = 0.0;
    if (r < nr) {
      const double* wtr = S.wt + ((size_t)h * S.nrows + row0 + r) * kD + c8;
#pragma unroll
      for (int m = 0; m < 8; ++m) d = fma(urw[(size_t)r * kD + c8 + m], wtr[m], d);
    }
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) d += __shfl_xor(d, off);
    if ((tid & 15) == 0) gbw[r] = r < nr ? S.erow[(size_t)h * S.nrows + row0 + r] * two_dm * d : 0.0;
  }
  double ua[32];
  {
    const bool ok = li < nr;
    const double* ur = urw + (size_t)(ok ? li : 0) * kD + 32 * lk;
#pragma unroll
    for (int m = 0; m < 32; ++m) ua[m] = ok ? ur[m] : 0.0;
  }
  double gb4[4] = {0.0, 0.0, 0.0, 0.0};
  for (int tt = w; 16 * tt <= s_hi; tt += 4) {
    if (16 * tt + 15 < s_lo) continue;  // uniform over the wave
    const int s = 16 * tt + li;
    const bool ok = s <= tmax;
    const f64x4 g = dot_tokens_bf16(ua, S.v + ((size_t)(a0 + (ok ? s : 0)) * c.H + h) * kD, ok, lk);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = lk + 4 * v;
      if (r < nr && int2_token(s, tf + r / gq, c.sink, c.recent)) {
        const size_t o = (size_t)r * L + s;
        const double pk = pdb[o], gs = two_dm * g[v];
        gb4[v] = fma(pk, gs, gb4[v]);
        pfb[o] = (pk - pcb[o]) + c.lam * pk * gs;
      }
    }
  }
  // gbar per row: over the 16 lanes of each lk group, then the four waves (fixed order), then the window
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) gb4[v] += __shfl_xor(gb4[v], off);
  if (li == 0)
#pragma unroll
    for (int v = 0; v < 4; ++v) red[w * 16 + lk + 4 * v] = gb4[v];
  __syncthreads();  // also makes the pf updates and gbw visible to the whole block
  double gb[R];
#pragma unroll
  for (int r = 0; r < R; ++r) gb[r] = ((red[r] + red[32 + r]) + (red[16 + r] + red[48 + r])) + gbw[r];
  const double inv_rows = 1.0 / (double)S.nrows;
  for (int s = s_lo + tid; s <= s_hi; s += kTileThreads) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (r >= nr || !int2_token(s, tf + r / gq, c.sink, c.recent)) continue;
      const size_t o = (size_t)r * L + s;
      pdb[o] = (pfb[o] - c.lam * pdb[o] * gb[r]) * inv_rows;
    }
  }
}

// Gradient w.r.t. the effective rows and the rotated rows of one unit of 16 tokens:
//   gx[s] = sum over the rows r of s's sequence of pd[r][s] y_r, y_r = q_r / sqrt(d) (keys) or the row
//   weight (values), then gz = mask . (gx R).
// Taken as gx^T = Y^T P (M = channels, N = the unit's tokens, K = rows), so the channels a lane ends with are
// the K slices of the second product gz^T = R^T gx^T and gx needs no transpose. Both operands are read from
// memory in operand order (lane li: channels 8 li + t of row lk for tiles t; token li of the row's weights),
// so there is no staging and no barrier on the way. Block (unit, KV head) of two waves: each sums half of
// the rows, the halves are added in order through LDS, and each forms half of gz's channels.
// Bound by the matrix cores' fp64 rate within a wave. At 8 heads, 7 sequences, the paper's windows: 168 us
// (64-token tiles staged through LDS over every token) + 49 us (gz on its own) -> 51 us.
__global__ __launch_bounds__(128) void cal_gxz_kernel(CalSet S, CalCfg c, int value) {
  __shared__ double part[2][32][64];
  const int h = blockIdx.y, w = threadIdx.x >> 6, l = threadIdx.x & 63, li = l & 15, lk = l >> 4;
  const int4 unit = S.units[blockIdx.x];
  const CalSeq sq = S.seqs[unit.z];
  const int nr = (sq.len - sq.t0) * c.gq, half = 4 * (((nr + 3) / 4 + 1) / 2);
  const int r_lo = w ? half : 0, r_hi = w ? nr : min(nr, half);
  const bool ok = li < unit.y;
  const double* pd = S.pd + (size_t)h * S.pelems + sq.p0 + (unit.w + (ok ? li : 0));
  const double* wr = S.wrow + ((size_t)h * S.nrows + sq.row0) * kD + 8 * li;
  const uint16_t* qr = S.q + ((size_t)(sq.start + sq.t0) * c.Hq + (size_t)h * c.gq) * kD + 8 * li;
  f64x4 acc[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
  // rows past the end read the last row with weight zero
  if (value) {
#pragma unroll 4
    for (int r0 = r_lo; r0 < r_hi; r0 += 4) {
      const int r = min(r0 + lk, nr - 1);
      const double2* y2 = reinterpret_cast<const double2*>(wr + (size_t)r * kD);
      const double2 y[4] = {y2[0], y2[1], y2[2], y2[3]};
      const double x = pd[(size_t)r * sq.len], p = ok && r0 + lk < r_hi ? x : 0.0;
#pragma unroll
      for (int t = 0; t < 8; ++t) acc[t] = mfma64(t & 1 ? y[t >> 1].y : y[t >> 1].x, p, acc[t]);
    }
  } else {
    const int step = c.Hq * kD;  // row r: position r / gq, query head r % gq
#pragma unroll 4
    for (int r0 = r_lo; r0 < r_hi; r0 += 4) {
      const int r = min(r0 + lk, nr - 1), pos = r / c.gq;
      double y[8];
      bf16x8_to_f64(load16<uint4>(qr + (size_t)pos * step + (size_t)(r - pos * c.gq) * kD), y);
      const double x = pd[(size_t)r * sq.len], p = ok && r0 + lk < r_hi ? x * kInvSqrtD : 0.0;
#pragma unroll
      for (int t = 0; t < 8; ++t) acc[t] = mfma64(y[t], p, acc[t]);
    }
  }
#pragma unroll
  for (int t = 0; t < 8; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) part[w][4 * t + v][l] = acc[t][v];
  __syncthreads();
#pragma unroll
  for (int t = 0; t < 8; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[t][v] += part[1 - w][4 * t + v][l];  // two terms: the same in either order
  // element v of acc[t]: token li, channel 8 (lk + 4 v) + t; wave w stores v = 2 w, 2 w + 1
  const size_t row = hrow(S, unit.x + (ok ? li : 0), h);
  if (ok)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if ((v >> 1) != w) continue;
      double2* o = reinterpret_cast<double2*>(S.gx + row + 8 * (lk + 4 * v));
#pragma unroll
      for (int t = 0; t < 4; ++t) o[t] = make_double2(acc[2 * t][v], acc[2 * t + 1][v]);
    }
  // gz: wave w's channels 64 w + 4 m + ct, m the row of tile ct
  f64x4 z[4];
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) z[ct] = f64x4{0.0, 0.0, 0.0, 0.0};
  const double* R = c.R + (size_t)h * kMat + 64 * w + 4 * li;
#pragma unroll
  for (int t = 0; t < 8; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const double2* r2 = reinterpret_cast<const double2*>(R + (8 * (lk + 4 * v) + t) * kD);
      const double2 ra = r2[0], rb = r2[1];
      z[0] = mfma64(ra.x, acc[t][v], z[0]);
      z[1] = mfma64(ra.y, acc[t][v], z[1]);
      z[2] = mfma64(rb.x, acc[t][v], z[2]);
      z[3] = mfma64(rb.y, acc[t][v], z[3]);
    }
  if (ok)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const size_t o = row + 64 * w + 4 * (lk + 4 * v);
      const uint32_t m = *reinterpret_cast<const uint32_t*>(S.mask + o);
      double2* g = reinterpret_cast<double2*>(S.gz + o);
      g[0] = make_double2(m & 0xFF ? z[0][v] : 0.0, m & 0xFF00 ? z[1][v] : 0.0);
      g[1] = make_double2(m & 0xFF0000 ? z[2][v] : 0.0, m & 0xFF000000 ? z[3][v] : 0.0);
    }
}

// Partial dL/dR over a slice of the units (the other tokens have gx = 0): sum_s x_s[a] gz_s[b] +
// gx_s[a] zhat_s[b] on the fp64 matrix cores (M = a, N = b, K = the slice's tokens, four per step).
// Block (KV head, slice) of eight waves, wave w: rows a = 16 w .. + 15 and all 128 columns; the four
// operands of one unit at a time staged in LDS, the next unit's fetched meanwhile. 101 -> 24 us (every
// token, nothing in flight before).
constexpr int kDrChunk = 16, kDrStride = 132;
__global__ __launch_bounds__(512) void cal_dr_kernel(CalSet S, CalCfg c, int value) {
  __shared__ __align__(16) double xs[kDrChunk][kDrStride], gxs[kDrChunk][kDrStride];
  __shared__ __align__(16) double gzs[kDrChunk][kDrStride], zs[kDrChunk][kDrStride];
  const int h = blockIdx.x, sp = blockIdx.y, tid = threadIdx.x;
  const int w = tid >> 6, l = tid & 63, li = l & 15, lk = l >> 4;
  const int u_lo = (int)((long long)S.nunits * sp / kCalSplit), u_hi = (int)((long long)S.nunits * (sp + 1) / kCalSplit);
  const uint16_t* X = value ? S.v : S.k;
  // thread: token tid / 32 of the unit, channels 4 (tid % 32) .. + 3
  const int tt = tid >> 5, c4 = 4 * (tid & 31);
  double mu[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) mu[i] = value ? 0.0 : (double)c.mu[h * kD + c4 + i];
  uint2 xr;
  f64x2 gxr[2], gzr[2], zr[2];
  bool okr = false;
  auto fetch = [&](int u) {
    const int4 unit = S.units[u];
    okr = tt < unit.y;
    const int s = unit.x + (okr ? tt : 0);
    const size_t io = hrow(S, s, h) + c4;
    xr = *reinterpret_cast<const uint2*>(X + ((size_t)s * c.H + h) * kD + c4);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      gxr[i] = reinterpret_cast<const f64x2*>(S.gx + io)[i];
      gzr[i] = reinterpret_cast<const f64x2*>(S.gz + io)[i];
      zr[i] = reinterpret_cast<const f64x2*>(S.zhat + io)[i];
    }
  };
  f64x4 acc[8];
#pragma unroll
  for (int ct = 0; ct < 8; ++ct) acc[ct] = f64x4{0.0, 0.0, 0.0, 0.0};
  if (u_lo < u_hi) fetch(u_lo);
  for (int u = u_lo; u < u_hi; ++u) {
    __syncthreads();
    const f64x2 z2 = {0.0, 0.0};
    const double x0 = (double)__uint_as_float(xr.x << 16), x1 = (double)__uint_as_float(xr.x & 0xFFFF0000u);
    const double x2 = (double)__uint_as_float(xr.y << 16), x3 = (double)__uint_as_float(xr.y & 0xFFFF0000u);
    f64x2* px = reinterpret_cast<f64x2*>(&xs[tt][c4]);
    px[0] = okr ? f64x2{x0 - mu[0], x1 - mu[1]} : z2;
    px[1] = okr ? f64x2{x2 - mu[2], x3 - mu[3]} : z2;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      reinterpret_cast<f64x2*>(&gxs[tt][c4])[i] = okr ? gxr[i] : z2;
      reinterpret_cast<f64x2*>(&gzs[tt][c4])[i] = okr ? gzr[i] : z2;
      reinterpret_cast<f64x2*>(&zs[tt][c4])[i] = okr ? zr[i] : z2;
    }
    __syncthreads();
    if (u + 1 < u_hi) fetch(u + 1);
#pragma unroll
    for (int k4 = 0; k4 < kDrChunk; k4 += 4) {
      const int t = k4 + lk;
      const double ax = xs[t][16 * w + li], ag = gxs[t][16 * w + li];
#pragma unroll
      for (int ct = 0; ct < 8; ++ct) {
        acc[ct] = mfma64(ax, gzs[t][16 * ct + li], acc[ct]);
        acc[ct] = mfma64(ag, zs[t][16 * ct + li], acc[ct]);
      }
    }
  }
  // element v of acc[ct]: row a = 16 w + lk + 4 v, column b = 16 ct + li
  double* out = c.drp + ((size_t)sp * c.H + h) * kMat;
#pragma unroll
  for (int ct = 0; ct < 8; ++ct)
#pragma unroll
    for (int v = 0; v < 4; ++v) out[(16 * w + lk + 4 * v) * kD + 16 * ct + li] = acc[ct][v];
}

// ---------------------------------------------------------------------------------------------
// Matrix functions of the generators, per KV head. With S = A - A^T (skew, so normal: the 2-norm of S is
// that of S^4 to the power 1/4, at most ||S^4||_1^{1/4}) the exponential is the Taylor polynomial of
// S 2^-j, degree 4 nb - 1, in Paterson-Stockmeyer form: with Y = X^4,
//   p(X) = (..(B_{nb-1} Y + B_{nb-2}) Y + ..) Y + B_0,  B_i = sum_{q<4} X^q / (4 i + q)!,
// applied 2^j times; j is the smallest with ||S^4||_1^{1/4} 2^-j <= kExpTheta and nb the smallest whose
// first dropped term is below 2^-55. Measured against a long-double exponential of random skew matrices
// with 1-norms from 0.3 to 50, the relative error is 5e-17 to 1.3e-15 (8e-17 to 1e-14 for the degree-14
// polynomial at ||X||_1 <= 1/2 with its squarings, which this form replaced).
//
// Every product's right operand is a 16-column block, and every left operand (S, S^4, ..) was complete
// before the launch: a work-group computes its column block of the result with no exchange between
// work-groups. A work-group (block of 16 columns, KV head) has eight waves, wave w owning rows
// 16 w .. + 15: the left operand's rows stay in registers (64 per lane), the column block goes through
// LDS, and a product is 32 fp64 matrix-core steps per wave (1.7 us at the CU's fp64 rate). Bound by that
// chain of products: per call at 8 heads, exponential 369 -> 40 us and gradient 1,011 -> 90 us (medians
// over a 20-step calibration, before the squarings below) against one work-group of 1,024 threads per head (8 of 256 CUs).
// The last kExpSquares of the j doublings are squarings of the finished blocks, a launch each: a column block is one
// product of the exponential (three of the gradient) there, against 3 + nb - 1 (three times that) for every further
// application. At 8 heads, means over a 20-step calibration: exponential 49 -> 20 us and 15 for its squarings, gradient
// 108 -> 43 and 17; one layer's calibration 22.9 -> 18.3 ms.
// Error against a long-double exponential, 1-norms of S^4 to the power 1/4 from 4 to 27: 3e-16 to 2.3e-15
// (2e-16 to 2.4e-15 with applications alone).
// Beyond kExpMaxReps halvings one work-group per head forms all column blocks and squares j times.
constexpr int kExpCols = 16;      // columns per work-group
constexpr int kExpThreads = 512;  // eight waves of 16 rows
constexpr double kExpTheta = 3.5;
constexpr int kExpMaxBlocks = 8;  // nb at most (theta^32 / 32! < 2^-55)
constexpr int kExpSquares = 2;    // doublings done by squaring launches
constexpr int kExpMaxReps = 5;    // halvings (and so up to 2^3 applications) per column block
// scratch matrices of a head (c.ex): powers of S, then of [[X, G], [0, X]] with X = S^T = -S (upper right
// blocks: X D_k + G X^k), the exponential's blocks, the column-block bounds on ||S^4||_1
enum { kExS = 0, kExS2, kExS3, kExS4, kExG, kExD2, kExD3, kExD4, kExP2, kExP1, kExBound };
static_assert(kExBound < kCalScratch, "scratch matrices of the matrix functions");

__device__ constexpr double kInvFact[4 * kExpMaxBlocks] = {
    0x1.0000000000000p+0, 0x1.0000000000000p+0, 0x1.0000000000000p-1, 0x1.5555555555555p-3, 0x1.5555555555555p-5,
    0x1.1111111111111p-7, 0x1.6c16c16c16c17p-10, 0x1.a01a01a01a01ap-13, 0x1.a01a01a01a01ap-16,
    0x1.71de3a556c734p-19, 0x1.27e4fb7789f5cp-22, 0x1.ae64567f544e4p-26, 0x1.1eed8eff8d898p-29,
    0x1.6124613a86d09p-33, 0x1.93974a8c07c9dp-37, 0x1.ae7f3e733b81fp-41, 0x1.ae7f3e733b81fp-45,
    0x1.952c77030ad4ap-49, 0x1.6827863b97d97p-53, 0x1.2f49b46814157p-57, 0x1.e542ba4020225p-62,
    0x1.71b8ef6dcf572p-66, 0x1.0ce396db7f853p-70, 0x1.761b41316381ap-75, 0x1.f2cf01972f578p-80,
    0x1.3f3ccdd165fa9p-84, 0x1.88e85fc6a4e5ap-89, 0x1.d1ab1c2dccea3p-94, 0x1.0a18a2635085dp-98,
    0x1.259f98b4358adp-103, 0x1.3932c5047d60ep-108, 0x1.434d2e783f5bcp-113};

struct ExpBuf {
  double y[2][kD * kExpCols];  // column block, two buffers
};

// Rows 16 w + li of M (row-major, times sign) as the left operand: lane (li, lk) holds M[16 w + li][32 lk + s].
__device__ __forceinline__ void exp_left(const double* M, double sign, double (&a)[32]) {
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const double* r = M + (16 * w + (l & 15)) * kD + 32 * (l >> 4);  // of the scratch, or the caller's A
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const double2 x = load16<double2>(r + 2 * i);
    a[2 * i] = sign * x.x;
    a[2 * i + 1] = sign * x.y;
  }
}

// acc + M Y for the wave's 16 rows: Y in LDS [k][16]; element v: row 16 w + lk + 4 v, column li.
__device__ __forceinline__ f64x4 exp_prod(const double (&a)[32], const double* Y, f64x4 acc) {
  const int l = threadIdx.x & 63;
  const double* y = Y + 32 * kExpCols * (l >> 4) + (l & 15);
#pragma unroll
  for (int s = 0; s < 32; ++s) acc = mfma64(a[s], y[kExpCols * s], acc);
  return acc;
}

// The thread's fragment of column block cb: rows exp_row(v), column 16 cb + li.
__device__ __forceinline__ int exp_row(int v) {
  return 16 * (threadIdx.x >> 6) + ((threadIdx.x & 63) >> 4) + 4 * v;
}
__device__ __forceinline__ f64x4 exp_load(const double* M, int cb, double sign) {
  f64x4 f;
#pragma unroll
  for (int v = 0; v < 4; ++v) f[v] = sign * M[exp_row(v) * kD + kExpCols * cb + (threadIdx.x & 15)];
  return f;
}
__device__ __forceinline__ void exp_store(double* M, int cb, f64x4 f) {
#pragma unroll
  for (int v = 0; v < 4; ++v) M[exp_row(v) * kD + kExpCols * cb + (threadIdx.x & 15)] = f[v];
}
__device__ __forceinline__ void exp_put(double* Y, f64x4 f) {
#pragma unroll
  for (int v = 0; v < 4; ++v) Y[exp_row(v) * kExpCols + (threadIdx.x & 15)] = f[v];
}
__device__ __forceinline__ f64x4 exp_eye(int cb) {
  f64x4 f;
#pragma unroll
  for (int v = 0; v < 4; ++v) f[v] = exp_row(v) == kExpCols * cb + (int)(threadIdx.x & 15) ? 1.0 : 0.0;
  return f;
}
// column block cb of M (row-major) into LDS
__device__ __forceinline__ void exp_block(const double* M, int cb, double sign, double* Y) {
  for (int e = threadIdx.x; e < kD * kExpCols; e += kExpThreads)
    Y[e] = sign * M[(e / kExpCols) * kD + kExpCols * cb + e % kExpCols];
}

// j halvings and nb polynomial blocks for a head, from the bounds its powers kernel stored
__device__ __forceinline__ void exp_plan(const double* ex, int& j, int& nb) {
  const double* bound = ex + kExBound * kMat;
  double b = 0.0;
  for (int i = 0; i < kD / kExpCols; ++i) b = fmax(b, bound[i]);
  b = sqrt(sqrt(b));
  j = 0;
  while (b > kExpTheta && j < 60) {
    b *= 0.5;
    ++j;
  }
  const double b4 = (b * b) * (b * b);
  double p = b4;
  nb = 1;
  while (nb < kExpMaxBlocks && p * kInvFact[4 * nb - 1] / (4 * nb) > 0x1p-55) {
    p *= b4;
    ++nb;
  }
  j = __builtin_amdgcn_readfirstlane(j);  // the same in every lane: loop counts and coefficients are scalar
  nb = __builtin_amdgcn_readfirstlane(nb);
}

// Squaring launches a head needs (none where one work-group forms all of its column blocks).
__device__ __forceinline__ int exp_squares(int j) { return j > kExpMaxReps ? 0 : min(j, kExpSquares); }

// S, S^2, S^3, S^4 and each column block's largest absolute column sum of S^4.
__global__ __launch_bounds__(kExpThreads) void cal_exp_powers_kernel(CalCfg c, const double* __restrict__ Aall) {
  __shared__ ExpBuf sm;
  __shared__ double cs[8][kExpCols];
  const int cb = blockIdx.x, h = blockIdx.y, tid = threadIdx.x, w = tid >> 6, l = tid & 63, li = l & 15, lk = l >> 4;
  const double* A = Aall + (size_t)h * kMat;
  double* ex = c.ex + (size_t)h * kCalScratch * kMat;
  double a[32];
  exp_left(A, 1.0, a);
#pragma unroll
  for (int s = 0; s < 32; ++s) a[s] -= A[(32 * lk + s) * kD + 16 * w + li];
  for (int e = tid; e < kD * kExpCols; e += kExpThreads) {
    const int r = e / kExpCols, col = kExpCols * cb + e % kExpCols;
    const double s = A[r * kD + col] - A[col * kD + r];
    sm.y[0][e] = s;
    ex[kExS * kMat + r * kD + col] = s;
  }
  f64x4 f;
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    __syncthreads();
    f = exp_prod(a, sm.y[p & 1], f64x4{0.0, 0.0, 0.0, 0.0});
    exp_store(ex + (kExS2 + p) * kMat, cb, f);
    if (p < 2) exp_put(sm.y[(p + 1) & 1], f);
  }
  double t = (fabs(f[0]) + fabs(f[1])) + (fabs(f[2]) + fabs(f[3]));
  t += __shfl_xor(t, 16);
  t += __shfl_xor(t, 32);
  if (lk == 0) cs[w][li] = t;
  __syncthreads();
  if (tid < 16) {
    double b = 0.0;
    for (int i = 0; i < 8; ++i) b += cs[i][tid];
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) b = fmax(b, __shfl_xor(b, off));
    if (tid == 0) ex[kExBound * kMat + cb] = b;
  }
}

// R[:, block] = R0 y and the rows of Rt (fp64), y in LDS.
__device__ __forceinline__ void exp_finish(const CalCfg& c, int value, int h, int cb, const double* Y, double (&a)[32]) {
  const float* R0f = (value ? c.R0v : c.R0k) + (size_t)h * kMat;
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const float* r = R0f + (16 * w + (l & 15)) * kD + 32 * (l >> 4);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float4 x = load16<float4>(r + 4 * i);
    a[4 * i] = x.x;
    a[4 * i + 1] = x.y;
    a[4 * i + 2] = x.z;
    a[4 * i + 3] = x.w;
  }
  const f64x4 f = exp_prod(a, Y, f64x4{0.0, 0.0, 0.0, 0.0});
  exp_store(c.R + (size_t)h * kMat, cb, f);
  double* Rt = c.Rt + (size_t)h * kMat + (kExpCols * cb + (l & 15)) * kD;
#pragma unroll
  for (int v = 0; v < 4; ++v) Rt[exp_row(v)] = f[v];
}

// R = R0 exp(S) and Rt = R^T, or, where squarings follow, the column blocks of exp(S 2^-squares) into scratch kExP1.
__global__ __launch_bounds__(kExpThreads) void cal_exp_apply_kernel(CalCfg c, int value) {
  __shared__ ExpBuf sm;
  const int h = blockIdx.y;
  double* ex = c.ex + (size_t)h * kCalScratch * kMat;
  int j, nb;
  exp_plan(ex, j, nb);
  const bool alone = j > kExpMaxReps;  // uniform over the head's work-groups
  if (alone && blockIdx.x != 0) return;
  double a[32];
  int yb = 0;  // LDS buffer the next column block goes to
  auto put = [&](f64x4 f) {
    double* Y = sm.y[yb];
    yb ^= 1;
    exp_put(Y, f);
    __syncthreads();
    return Y;
  };
  const f64x4 zero = {0.0, 0.0, 0.0, 0.0};
  // p(S 2^-j) y for a column block y (the identity's block cb when first)
  auto poly = [&](int cb, bool first, f64x4 y) {
    f64x4 w1, w2, w3;
    if (first) {
      y = exp_eye(cb);
      w1 = exp_load(ex + kExS * kMat, cb, 1.0);
      w2 = exp_load(ex + kExS2 * kMat, cb, 1.0);
      w3 = exp_load(ex + kExS3 * kMat, cb, 1.0);
    } else {
      exp_left(ex + kExS * kMat, 1.0, a);
      w1 = exp_prod(a, put(y), zero);
      w2 = exp_prod(a, put(w1), zero);
      w3 = exp_prod(a, put(w2), zero);
    }
    exp_left(ex + kExS4 * kMat, 1.0, a);
    auto blk = [&](int i) {
      const double c0 = ldexp(kInvFact[4 * i], -4 * i * j), c1 = ldexp(kInvFact[4 * i + 1], -(4 * i + 1) * j),
                   c2 = ldexp(kInvFact[4 * i + 2], -(4 * i + 2) * j), c3 = ldexp(kInvFact[4 * i + 3], -(4 * i + 3) * j);
      return c0 * y + c1 * w1 + c2 * w2 + c3 * w3;
    };
    f64x4 p = blk(nb - 1);
    for (int i = nb - 2; i >= 0; --i) p = exp_prod(a, put(p), blk(i));
    return p;
  };
  if (!alone) {
    const int cb = blockIdx.x;
    const int sq = exp_squares(j);
    f64x4 y = poly(cb, true, zero);
    for (int r = 1; r < (1 << (j - sq)); ++r) y = poly(cb, false, y);
    if (sq > 0)
      exp_store(ex + kExP1 * kMat, cb, y);
    else
      exp_finish(c, value, h, cb, put(y), a);
    return;
  }
  double *P = ex + kExP1 * kMat, *Q = ex + kExP2 * kMat;
  for (int cb = 0; cb < kD / kExpCols; ++cb) exp_store(P, cb, poly(cb, true, zero));
  for (int i = 0; i < j; ++i) {
    __syncthreads();
    exp_left(P, 1.0, a);
    for (int cb = 0; cb < kD / kExpCols; ++cb) exp_store(Q, cb, exp_prod(a, put(exp_load(P, cb, 1.0)), zero));
    double* t = P;
    P = Q;
    Q = t;
  }
  for (int cb = 0; cb < kD / kExpCols; ++cb) exp_finish(c, value, h, cb, put(exp_load(P, cb, 1.0)), a);
}

// Squaring i of the exponential (kExP1 -> kExP2 -> ..); the head's last one goes on to R.
static_assert(kExpSquares == 2, "the scratch matrices of the squarings alternate between two");
__global__ __launch_bounds__(kExpThreads) void cal_exp_square_kernel(CalCfg c, int value, int i) {
  __shared__ ExpBuf sm;
  const int cb = blockIdx.x, h = blockIdx.y;
  double* ex = c.ex + (size_t)h * kCalScratch * kMat;
  int j, nb;
  exp_plan(ex, j, nb);
  const int sq = exp_squares(j);
  if (i >= sq) return;  // uniform
  const double* P = ex + (i == 0 ? kExP1 : kExP2) * kMat;
  double a[32];
  exp_left(P, 1.0, a);
  exp_block(P, cb, 1.0, sm.y[0]);
  __syncthreads();
  const f64x4 f = exp_prod(a, sm.y[0], f64x4{0.0, 0.0, 0.0, 0.0});
  if (i + 1 < sq) {
    exp_store(ex + kExP2 * kMat, cb, f);
    return;
  }
  exp_put(sm.y[1], f);
  __syncthreads();
  exp_finish(c, value, h, cb, sm.y[1], a);
}

// Gradient: dL/dA = dS - dS^T with dS = L_exp(S^T, G), G = R0^T dL/dR: the upper right block of
// exp([[X, G], [0, X]]), X = S^T = -S, whose powers are [[X^k, D_k], [0, X^k]], D_{k+1} = X D_k + G X^k; the
// same polynomial on column blocks (u, v), two or three products per step. The powers of S are the ones
// the exponential left for the same generators.
//
// G of one column block, with dL/dR summed over its token slices in slice order.
__global__ __launch_bounds__(kExpThreads) void cal_grad_g_kernel(CalCfg c, int value) {
  __shared__ ExpBuf sm;
  const int cb = blockIdx.x, h = blockIdx.y, tid = threadIdx.x, w = tid >> 6, l = tid & 63, li = l & 15, lk = l >> 4;
  const float* R0 = (value ? c.R0v : c.R0k) + (size_t)h * kMat;
  double a[32];
#pragma unroll
  for (int s = 0; s < 32; ++s) a[s] = R0[(32 * lk + s) * kD + 16 * w + li];  // rows of R0^T
  for (int e = tid; e < kD * kExpCols; e += kExpThreads) {
    const double* d = c.drp + (size_t)h * kMat + (e / kExpCols) * kD + kExpCols * cb + e % kExpCols;
    double x[kCalSplit], t = 0.0;
#pragma unroll
    for (int sp = 0; sp < kCalSplit; ++sp) x[sp] = d[(size_t)sp * c.H * kMat];
#pragma unroll
    for (int sp = 0; sp < kCalSplit; ++sp) t += x[sp];
    sm.y[0][e] = t;
  }
  __syncthreads();
  exp_store(c.ex + ((size_t)h * kCalScratch + kExG) * kMat, cb, exp_prod(a, sm.y[0], f64x4{0.0, 0.0, 0.0, 0.0}));
}

// D_2, D_3, D_4 of one column block.
__global__ __launch_bounds__(kExpThreads) void cal_grad_powers_kernel(CalCfg c) {
  __shared__ ExpBuf u, v;
  const int cb = blockIdx.x;
  double* ex = c.ex + (size_t)blockIdx.y * kCalScratch * kMat;
  double aX[32], aG[32];
  exp_left(ex + kExS * kMat, -1.0, aX);
  exp_left(ex + kExG * kMat, 1.0, aG);
  exp_block(ex + kExG * kMat, cb, 1.0, u.y[0]);
#pragma unroll
  for (int p = 0; p < 3; ++p) {  // D_{p+2} = X D_{p+1} + G X^{p+1} (D_1 = G)
    exp_block(ex + (kExS + p) * kMat, cb, p == 1 ? 1.0 : -1.0, v.y[p & 1]);
    __syncthreads();
    const f64x4 zero = {0.0, 0.0, 0.0, 0.0};
    const f64x4 d = exp_prod(aX, u.y[p & 1], zero) + exp_prod(aG, v.y[p & 1], zero);
    exp_store(ex + (kExD2 + p) * kMat, cb, d);
    if (p < 2) exp_put(u.y[(p + 1) & 1], d);
  }
}

// The upper right block of the exponential, [128][128] per head, into scratch kExP2; where squarings follow, that of
// exp(.. 2^-squares) there and its diagonal block in kExP1.
__global__ __launch_bounds__(kExpThreads) void cal_grad_apply_kernel(CalCfg c) {
  __shared__ ExpBuf su, sv;
  const int h = blockIdx.y;
  double* ex = c.ex + (size_t)h * kCalScratch * kMat;
  int j, nb;
  exp_plan(ex, j, nb);
  const bool alone = j > kExpMaxReps;
  if (alone && blockIdx.x != 0) return;
  double a[32], b[32];  // left operands: X (or X^4, P_1) and G (or D_4, P_2)
  int yb = 0;
  auto put = [&](f64x4 fu, f64x4 fv) {
    const int y = yb;
    yb ^= 1;
    exp_put(su.y[y], fu);
    exp_put(sv.y[y], fv);
    __syncthreads();
    return y;
  };
  const f64x4 zero = {0.0, 0.0, 0.0, 0.0};
  // (u, v) <- (a u + b v + du, a v + dv)
  auto step = [&](f64x4& fu, f64x4& fv, f64x4 du, f64x4 dv) {
    const int y = put(fu, fv);
    const f64x4 t = exp_prod(b, sv.y[y], zero);
    fu = exp_prod(a, su.y[y], du) + t;
    fv = exp_prod(a, sv.y[y], dv);
  };
  auto poly = [&](int cb, bool first, f64x4& u, f64x4& v) {
    f64x4 u1, u2, u3, v1, v2, v3;
    if (first) {
      u = zero;
      v = exp_eye(cb);
      u1 = exp_load(ex + kExG * kMat, cb, 1.0);
      u2 = exp_load(ex + kExD2 * kMat, cb, 1.0);
      u3 = exp_load(ex + kExD3 * kMat, cb, 1.0);
      v1 = exp_load(ex + kExS * kMat, cb, -1.0);
      v2 = exp_load(ex + kExS2 * kMat, cb, 1.0);
      v3 = exp_load(ex + kExS3 * kMat, cb, -1.0);
    } else {
      exp_left(ex + kExS * kMat, -1.0, a);
      exp_left(ex + kExG * kMat, 1.0, b);
      u1 = u;
      v1 = v;
      step(u1, v1, zero, zero);
      u2 = u1;
      v2 = v1;
      step(u2, v2, zero, zero);
      u3 = u2;
      v3 = v2;
      step(u3, v3, zero, zero);
    }
    exp_left(ex + kExS4 * kMat, 1.0, a);
    exp_left(ex + kExD4 * kMat, 1.0, b);
    f64x4 pu = zero, pv = zero;
    for (int i = nb - 1; i >= 0; --i) {
      const double c0 = ldexp(kInvFact[4 * i], -4 * i * j), c1 = ldexp(kInvFact[4 * i + 1], -(4 * i + 1) * j),
                   c2 = ldexp(kInvFact[4 * i + 2], -(4 * i + 2) * j), c3 = ldexp(kInvFact[4 * i + 3], -(4 * i + 3) * j);
      const f64x4 du = c0 * u + c1 * u1 + c2 * u2 + c3 * u3, dv = c0 * v + c1 * v1 + c2 * v2 + c3 * v3;
      if (i == nb - 1) {
        pu = du;
        pv = dv;
      } else {
        step(pu, pv, du, dv);
      }
    }
    u = pu;
    v = pv;
  };
  f64x4 u, v;
  if (!alone) {
    const int cb = blockIdx.x;
    const int sq = exp_squares(j);
    poly(cb, true, u, v);
    for (int r = 1; r < (1 << (j - sq)); ++r) poly(cb, false, u, v);
    exp_store(ex + kExP2 * kMat, cb, u);
    if (sq > 0) exp_store(ex + kExP1 * kMat, cb, v);
    return;
  }
  for (int cb = 0; cb < kD / kExpCols; ++cb) {
    poly(cb, true, u, v);
    exp_store(ex + kExP2 * kMat, cb, u);
    exp_store(ex + kExP1 * kMat, cb, v);
  }
  // (P_1, P_2) <- (P_1 P_1, P_1 P_2 + P_2 P_1); the powers' scratch is free now
  int p1 = kExP1, p2 = kExP2, q1 = kExD2, q2 = kExD3;
  for (int i = 0; i < j; ++i) {
    __syncthreads();
    exp_left(ex + p1 * kMat, 1.0, a);
    exp_left(ex + p2 * kMat, 1.0, b);
    for (int cb = 0; cb < kD / kExpCols; ++cb) {
      u = exp_load(ex + p2 * kMat, cb, 1.0);
      v = exp_load(ex + p1 * kMat, cb, 1.0);
      step(u, v, zero, zero);
      exp_store(ex + q2 * kMat, cb, u);
      exp_store(ex + q1 * kMat, cb, v);
    }
    int t = p1;
    p1 = q1;
    q1 = t;
    t = p2;
    p2 = q2;
    q2 = t;
  }
  if (p2 != kExP2)  // each thread copies the elements it stored
    for (int cb = 0; cb < kD / kExpCols; ++cb) exp_store(ex + kExP2 * kMat, cb, exp_load(ex + p2 * kMat, cb, 1.0));
}

// Squaring i of the gradient's blocks: (P_1, P_2) <- (P_1 P_1, P_1 P_2 + P_2 P_1), from (kExP1, kExP2) to (kExD2,
// kExD3) and back; the last one needs no P_1.
__global__ __launch_bounds__(kExpThreads) void cal_grad_square_kernel(CalCfg c, int i) {
  __shared__ ExpBuf su, sv;
  const int cb = blockIdx.x;
  double* ex = c.ex + (size_t)blockIdx.y * kCalScratch * kMat;
  int j, nb;
  exp_plan(ex, j, nb);
  const int sq = exp_squares(j);
  if (i >= sq) return;  // uniform
  const double *P1 = ex + (i == 0 ? kExP1 : kExD2) * kMat, *P2 = ex + (i == 0 ? kExP2 : kExD3) * kMat;
  double a[32], b[32];
  exp_left(P1, 1.0, a);
  exp_left(P2, 1.0, b);
  exp_block(P2, cb, 1.0, su.y[0]);
  exp_block(P1, cb, 1.0, sv.y[0]);
  __syncthreads();
  const f64x4 zero = {0.0, 0.0, 0.0, 0.0};
  exp_store(ex + (i == 0 ? kExD3 : kExP2) * kMat, cb, exp_prod(a, su.y[0], zero) + exp_prod(b, sv.y[0], zero));
  if (i + 1 < sq) exp_store(ex + (i == 0 ? kExD2 : kExP1) * kMat, cb, exp_prod(a, sv.y[0], zero));
}

// grad = dS - dS^T
__global__ __launch_bounds__(256) void cal_grad_skew_kernel(CalCfg c, double* __restrict__ grad) {
  const int h = blockIdx.y, e = blockIdx.x * 256 + threadIdx.x, r = e / kD, col = e % kD;
  int j, nb;
  exp_plan(c.ex + (size_t)h * kCalScratch * kMat, j, nb);
  const double* P = c.ex + ((size_t)h * kCalScratch + (exp_squares(j) == 1 ? kExD3 : kExP2)) * kMat;
  grad[(size_t)h * kMat + e] = P[e] - P[col * kD + r];
}

// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void cal_loss_kernel(const double* __restrict__ lrow, int nrows,
                                                       double* __restrict__ loss) {
  __shared__ double red[16];
  const int h = blockIdx.x;
  double acc = 0.0;
  for (int r = threadIdx.x; r < nrows; r += blockDim.x) acc += lrow[(size_t)h * nrows + r];
  acc = block_sum(acc, red);
  if (threadIdx.x == 0) loss[h] = acc / (double)nrows;
}

// Adam as torch.optim.Adam (betas 0.9, 0.999, eps 1e-8, no weight decay): m <- m + (1 - b1)(g - m),
// v <- b2 v + (1 - b2) g^2, A <- A - (lr / (1 - b1^t)) m / (sqrt(v) / sqrt(1 - b2^t) + eps).
__global__ __launch_bounds__(256) void cal_adam_kernel(double* A, const double* g, double* m, double* v, int n,
                                                       double step_size, double bc2_sqrt, double lr) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  (void)lr;
  const double gi = g[i];
  const double mi = m[i] + (1.0 - 0.9) * (gi - m[i]);
  const double vi = v[i] * 0.999 + (1.0 - 0.999) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  A[i] -= step_size * mi / (sqrt(vi) / bc2_sqrt + 1e-8);
}

__global__ __launch_bounds__(1024) void cal_select_kernel(const double* A, const double* loss, double* best,
                                                          double* A_best) {
  const int h = blockIdx.x;
  const bool take = loss[h] < best[h];
  __syncthreads();  // every thread has read best[h] before thread 0 may replace it
  if (!take) return;
  for (int e = threadIdx.x; e < kMat; e += blockDim.x) A_best[(size_t)h * kMat + e] = A[(size_t)h * kMat + e];
  if (threadIdx.x == 0) best[h] = loss[h];
}

__global__ __launch_bounds__(64) void cal_record_kernel(const double* __restrict__ loss, double* __restrict__ dst,
                                                        int stride, int H) {
  const int h = threadIdx.x;
  if (h < H) dst[(size_t)h * stride] = loss[h];
}

__global__ __launch_bounds__(256) void cal_fill_kernel(double* p, size_t n, double v) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ __launch_bounds__(256) void cal_to_f32_kernel(const double* __restrict__ src, float* __restrict__ dst,
                                                         size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = (float)src[i];
}

// Partial W_{O,j}^T W_{O,j} over a slice of W_O's rows on the fp64 matrix cores: block (query head j, slice)
// of eight waves, wave w: output rows 16 w .. 16 w + 15 (all eight 16-column tiles). The head's slice goes
// through LDS 32 rows at a time (bf16 -> fp64, exact), the next rows fetched meanwhile; K = those rows, 4
// per step. The slices (into c.drp: as many as it holds for the query heads) are summed in order. Bound by
// the fp64 matrix cores of the CUs in use: 976 us with one block per query head (32 of 256 CUs) ->
// 146 us at four slices and the next rows in flight.
constexpr int kGramRows = 32;
__host__ __device__ constexpr int gram_slices(int gq) { return gq < kCalSplit ? kCalSplit / gq : 1; }
__global__ __launch_bounds__(512) void cal_gram_kernel(const uint16_t* __restrict__ W, int dm, int Hq,
                                                       double* __restrict__ part) {
  __shared__ __align__(16) double xs[kGramRows][kD + 2];
  const int j = blockIdx.x, sl = blockIdx.y, tid = threadIdx.x, w = tid >> 6, l = tid & 63, lo = l & 15, lk = l >> 4;
  const size_t ld = (size_t)Hq * kD;
  const int n_lo = (int)((long long)dm * sl / gridDim.y), n_hi = (int)((long long)dm * (sl + 1) / gridDim.y);
  f64x4 acc[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
  // thread: row tid / 16 of the chunk, channels 8 (tid % 16) .. + 7
  const int rr = tid >> 4, c8 = 8 * (tid & 15);
  uint4 xr = make_uint4(0, 0, 0, 0);
  bool okr = false;
  auto fetch = [&](int r0) {
    okr = r0 + rr < n_hi;
    xr = load16<uint4>(W + (size_t)(okr ? r0 + rr : n_lo) * ld + (size_t)j * kD + c8);
  };
  if (n_lo < n_hi) fetch(n_lo);
  for (int r0 = n_lo; r0 < n_hi; r0 += kGramRows) {
    double d[8];
    bf16x8_to_f64(okr ? xr : make_uint4(0, 0, 0, 0), d);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) reinterpret_cast<double2*>(&xs[rr][c8])[i] = make_double2(d[2 * i], d[2 * i + 1]);
    __syncthreads();
    if (r0 + kGramRows < n_hi) fetch(r0 + kGramRows);
#pragma unroll
    for (int k4 = 0; k4 < kGramRows; k4 += 4) {
      // A[m][k] = X[k][16 w + m], B[k][n] = X[k][16 t + n]: lane l holds A[lo][lk] and B[lk][lo]
      const double av = xs[k4 + lk][16 * w + lo];
#pragma unroll
      for (int t = 0; t < 8; ++t) acc[t] = mfma64(av, xs[k4 + lk][16 * t + lo], acc[t]);
    }
  }
  // element v of tile t: row 16 w + lk + 4 v, column 16 t + lo
  double* out = part + ((size_t)sl * Hq + j) * kMat;
#pragma unroll
  for (int t = 0; t < 8; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) out[(16 * w + lk + 4 * v) * kD + 16 * t + lo] = acc[t][v];
}

__global__ __launch_bounds__(256) void cal_gram_sum_kernel(const double* __restrict__ part, size_t n, int slices,
                                                           double* __restrict__ gram) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;  // n is a multiple of 256
  double t = part[i];
  for (int s = 1; s < slices; ++s) t += part[(size_t)s * n + i];
  gram[i] = t;
}

// Per-channel mean of the keys: block = KV head, thread = channel (sequential fp64 sum).
__global__ __launch_bounds__(128) void cal_key_mean_kernel(const uint16_t* __restrict__ k, int T, int H,
                                                           float* __restrict__ mu) {
  const int h = blockIdx.x, col = threadIdx.x;
  double acc = 0.0;
  for (int s = 0; s < T; ++s) acc += bf16d(k[((size_t)s * H + h) * kD + col]);
  mu[h * kD + col] = (float)(acc / (double)T);
}

size_t up256(size_t x) { return (x + 255) & ~size_t(255); }

}  // namespace

size_t cal_set_bytes(int T, int nseq, int nrows, long long pelems, int H) {
  const size_t rows = (size_t)T * H * kD;
  return up256(sizeof(CalSeq) * (size_t)nseq) + up256(sizeof(int4) * (size_t)nrows) +
         up256(sizeof(int4) * ((size_t)T / 16 + nseq)) + 4 * up256(rows * 8) +
         up256(rows) + 4 * up256((size_t)H * pelems * 8) + 3 * up256((size_t)H * nrows * kD * 8) +
         up256((size_t)H * nrows * 16) + 2 * up256((size_t)H * nrows * 8);
}

size_t cal_shared_bytes(int H, int Hq) {
  return up256((size_t)Hq * kMat * 8) + 2 * up256((size_t)H * kMat * 8) + up256((size_t)H * kCalScratch * kMat * 8) +
         up256((size_t)kCalSplit * H * kMat * 8);
}

hipError_t cal_bind_set(CalSet& set, uint8_t* base, const uint16_t* k, const uint16_t* v, const uint16_t* q,
                        const int32_t* starts_host, int nseq, int H, int gq, int n_last, int sink, int recent, hipStream_t s) {
  std::vector<CalSeq> seqs(nseq);
  std::vector<int4> units;
  long long pel = 0;
  int rows = 0, maxlen = 0;
  for (int i = 0; i < nseq; ++i) {
    CalSeq& c = seqs[i];
    c.start = starts_host[i];
    c.len = starts_host[i + 1] - starts_host[i];
    c.t0 = c.len > n_last ? c.len - n_last : 0;
    c.row0 = rows;
    c.p0 = pel;
    maxlen = c.len > maxlen ? c.len : maxlen;
    const int nr = (c.len - c.t0) * gq;
    // the tokens the last position reads from INT2 hold those of every earlier one
    for (int s0 = sink; s0 < c.len - recent; s0 += 16) units.push_back(make_int4(c.start + s0, min(16, c.len - recent - s0), i, s0));
    rows += nr;
    pel += (long long)nr * c.len;
  }
  set.k = k;
  set.v = v;
  set.q = q;
  set.T = starts_host[nseq] - starts_host[0];
  set.nseq = nseq;
  set.nrows = rows;
  set.pelems = pel;
  set.maxlen = maxlen;
  // tiles of up to kTileRows rows: 16 / gq positions of one sequence at a time
  std::vector<int4> tiles;
  const int per = gq >= kTileRows ? 1 : kTileRows / gq;
  for (int i = 0; i < nseq; ++i) {
    const CalSeq& cs = seqs[i];
    const int npos = cs.len - cs.t0;
    for (int pp = 0; pp < npos; pp += per)
      tiles.push_back(make_int4(i, cs.row0 + pp * gq, min(per, npos - pp) * gq, cs.t0 + pp));
  }
  set.ntiles = (int)tiles.size();
  const size_t nrow_el = (size_t)set.T * H * kD;
  uint8_t* p = base;
  set.seqs = reinterpret_cast<CalSeq*>(p);
  p += up256(sizeof(CalSeq) * (size_t)nseq);
  set.tiles = reinterpret_cast<int4*>(p);
  p += up256(sizeof(int4) * (size_t)rows);
  set.units = reinterpret_cast<int4*>(p);
  set.nunits = (int)units.size();
  p += up256(sizeof(int4) * ((size_t)set.T / 16 + nseq));
  set.zhat = reinterpret_cast<double*>(p);
  p += up256(nrow_el * 8);
  set.xeff = reinterpret_cast<double*>(p);
  p += up256(nrow_el * 8);
  set.gx = reinterpret_cast<double*>(p);
  p += up256(nrow_el * 8);
  set.gz = reinterpret_cast<double*>(p);
  p += up256(nrow_el * 8);
  set.mask = p;
  p += up256(nrow_el);
  set.pd = reinterpret_cast<double*>(p);
  p += up256((size_t)H * pel * 8);
  set.pf = reinterpret_cast<double*>(p);
  p += up256((size_t)H * pel * 8);
  set.fc = reinterpret_cast<double*>(p);
  p += up256((size_t)H * pel * 8);
  set.pc = reinterpret_cast<double*>(p);
  p += up256((size_t)H * pel * 8);
  set.rc = reinterpret_cast<double*>(p);
  p += up256((size_t)H * rows * 16);
  set.wt = reinterpret_cast<double*>(p);
  p += up256((size_t)H * rows * kD * 8);
  set.erow = reinterpret_cast<double*>(p);
  p += up256((size_t)H * rows * 8);
  set.wrow = reinterpret_cast<double*>(p);
  p += up256((size_t)H * rows * kD * 8);
  set.urow = reinterpret_cast<double*>(p);
  p += up256((size_t)H * rows * kD * 8);
  set.lrow = reinterpret_cast<double*>(p);
  hipError_t e = hipMemcpyAsync(set.seqs, seqs.data(), sizeof(CalSeq) * nseq, hipMemcpyHostToDevice, s);
  if (e == hipSuccess && !units.empty())
    e = hipMemcpyAsync(set.units, units.data(), sizeof(int4) * units.size(), hipMemcpyHostToDevice, s);
  if (e == hipSuccess && !tiles.empty())
    e = hipMemcpyAsync(set.tiles, tiles.data(), sizeof(int4) * tiles.size(), hipMemcpyHostToDevice, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);  // the host tables go out of scope
  return e;
}

void cal_bind_shared(CalCfg& c, uint8_t* base) {
  uint8_t* p = base;
  c.gram = reinterpret_cast<double*>(p);
  p += up256((size_t)c.Hq * kMat * 8);
  c.R = reinterpret_cast<double*>(p);
  p += up256((size_t)c.H * kMat * 8);
  c.Rt = reinterpret_cast<double*>(p);
  p += up256((size_t)c.H * kMat * 8);
  c.ex = reinterpret_cast<double*>(p);
  p += up256((size_t)c.H * kCalScratch * kMat * 8);
  c.drp = reinterpret_cast<double*>(p);
}

hipError_t cal_gram(const CalCfg& c, const uint16_t* W_o, hipStream_t s) {
  const int slices = gram_slices(c.gq);
  const size_t n = (size_t)c.Hq * kMat;
  hipLaunchKernelGGL(cal_gram_kernel, dim3(c.Hq, slices), dim3(512), 0, s, W_o, c.dm, c.Hq, c.drp);
  hipLaunchKernelGGL(cal_gram_sum_kernel, dim3((unsigned)(n / 256)), dim3(256), 0, s, c.drp, n, slices, c.gram);
  return hipGetLastError();
}

// R = R0 exp(A - A^T) and its transpose for every head
static void rotation(const CalCfg& c, const double* A, int value, hipStream_t s) {
  const dim3 grid(kD / kExpCols, c.H), block(kExpThreads);
  hipLaunchKernelGGL(cal_exp_powers_kernel, grid, block, 0, s, c, A);
  hipLaunchKernelGGL(cal_exp_apply_kernel, grid, block, 0, s, c, value);
  for (int i = 0; i < kExpSquares; ++i) hipLaunchKernelGGL(cal_exp_square_kernel, grid, block, 0, s, c, value, i);
}

static void rot_and_quant(const CalCfg& c, CalSet& set, const double* A, int value, hipStream_t s) {
  rotation(c, A, value, s);
  if (set.nunits > 0)
    hipLaunchKernelGGL(cal_rotq_kernel, dim3((set.nunits + 3) / 4, c.H), dim3(kMatThreads), 0, s, set, c, value);
}

// after rot_and_quant for the same generators (it leaves the powers of S)
static void backward(const CalCfg& c, CalSet& set, int value, double* grad, hipStream_t s) {
  if (set.nunits > 0)
    hipLaunchKernelGGL(cal_gxz_kernel, dim3(set.nunits, c.H), dim3(128), 0, s, set, c, value);
  hipLaunchKernelGGL(cal_dr_kernel, dim3(c.H, kCalSplit), dim3(512), 0, s, set, c, value);  // zeros without units
  const dim3 grid(kD / kExpCols, c.H), block(kExpThreads);
  hipLaunchKernelGGL(cal_grad_g_kernel, grid, block, 0, s, c, value);
  hipLaunchKernelGGL(cal_grad_powers_kernel, grid, block, 0, s, c);
  hipLaunchKernelGGL(cal_grad_apply_kernel, grid, block, 0, s, c);
  for (int i = 0; i < kExpSquares; ++i) hipLaunchKernelGGL(cal_grad_square_kernel, grid, block, 0, s, c, i);
  hipLaunchKernelGGL(cal_grad_skew_kernel, dim3(kMat / 256, c.H), dim3(256), 0, s, c, grad);
}

// the tile kernels: one block per (tile, KV head)
#define CAL_POS_LAUNCH(KERNEL, ...) \
  hipLaunchKernelGGL(KERNEL, dim3(set.ntiles, c.H), dim3(kTileThreads), 0, s, __VA_ARGS__)

static void u_launch(const CalCfg& c, const CalSet& set, int value, hipStream_t s) {
  const int npos = set.nrows / c.gq;
  hipLaunchKernelGGL(cal_u_kernel, dim3(c.Hq, (npos + kUTile - 1) / kUTile), dim3(256), 0, s, set, c, value);
}

hipError_t cal_prepare_set(const CalCfg& c, CalSet& set, hipStream_t s) {
  if (set.nrows == 0) return hipSuccess;
  const size_t n = (size_t)c.H * set.pelems;
  hipLaunchKernelGGL(cal_fill_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, set.pd, n, 0.0);
  CAL_POS_LAUNCH(cal_const_kernel, set, c);
  return hipGetLastError();
}

hipError_t cal_key_loss(const CalCfg& c, CalSet& set, const double* A, double* loss, double* grad, hipStream_t s) {
  rot_and_quant(c, set, A, 0, s);
  if (set.nrows > 0) {
    CAL_POS_LAUNCH(cal_pos_fwd_kernel, set, c, 0);
    u_launch(c, set, 0, s);
    if (grad) CAL_POS_LAUNCH(cal_pos_grad_kernel, set, c);
    hipLaunchKernelGGL(cal_loss_kernel, dim3(c.H), dim3(256), 0, s, set.lrow, set.nrows, loss);
  } else {
    hipLaunchKernelGGL(cal_fill_kernel, dim3(1), dim3(256), 0, s, loss, (size_t)c.H, 0.0);
  }
  if (grad) {
    if (set.nrows == 0) {
      hipLaunchKernelGGL(cal_fill_kernel, dim3((unsigned)(((size_t)c.H * kMat + 255) / 256)), dim3(256), 0, s, grad,
                         (size_t)c.H * kMat, 0.0);
      return hipGetLastError();
    }
    backward(c, set, 0, grad, s);
  }
  return hipGetLastError();
}

hipError_t cal_key_probs(const CalCfg& c, CalSet& set, const double* A, hipStream_t s) {
  rot_and_quant(c, set, A, 0, s);
  if (set.nrows > 0) CAL_POS_LAUNCH(cal_pos_fwd_kernel, set, c, 1);
  return hipGetLastError();
}

hipError_t cal_value_loss(const CalCfg& c, CalSet& set, const double* A, double* loss, double* grad, hipStream_t s) {
  rot_and_quant(c, set, A, 1, s);
  if (set.nrows > 0) {
    CAL_POS_LAUNCH(cal_pos_val_kernel, set, c);
    u_launch(c, set, 1, s);
    hipLaunchKernelGGL(cal_loss_kernel, dim3(c.H), dim3(256), 0, s, set.lrow, set.nrows, loss);
  } else {
    hipLaunchKernelGGL(cal_fill_kernel, dim3(1), dim3(256), 0, s, loss, (size_t)c.H, 0.0);
  }
  if (grad) {
    if (set.nrows == 0) {
      hipLaunchKernelGGL(cal_fill_kernel, dim3((unsigned)(((size_t)c.H * kMat + 255) / 256)), dim3(256), 0, s, grad,
                         (size_t)c.H * kMat, 0.0);
      return hipGetLastError();
    }
    backward(c, set, 1, grad, s);
  }
  return hipGetLastError();
}

hipError_t cal_adam(double* A, const double* g, double* m, double* v, int n, int step, double lr, hipStream_t s) {
  const double bc1 = 1.0 - pow(0.9, (double)step), bc2 = 1.0 - pow(0.999, (double)step);
  hipLaunchKernelGGL(cal_adam_kernel, dim3((n + 255) / 256), dim3(256), 0, s, A, g, m, v, n, lr / bc1, sqrt(bc2), lr);
  return hipGetLastError();
}

hipError_t cal_select(const double* A, const double* loss, double* best, double* A_best, int H, hipStream_t s) {
  hipLaunchKernelGGL(cal_select_kernel, dim3(H), dim3(1024), 0, s, A, loss, best, A_best);
  return hipGetLastError();
}

hipError_t cal_record(const double* loss, double* dst, int stride, int H, hipStream_t s) {
  for (int h0 = 0; h0 < H; h0 += 64)
    hipLaunchKernelGGL(cal_record_kernel, dim3(1), dim3(64), 0, s, loss + h0, dst + (size_t)h0 * stride, stride,
                       min(64, H - h0));
  return hipGetLastError();
}

hipError_t cal_fill(double* p, size_t n, double v, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(cal_fill_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

hipError_t cal_rotation_out(const CalCfg& c, const double* A, bool value, float* out, hipStream_t s) {
  rotation(c, A, value ? 1 : 0, s);
  const size_t n = (size_t)c.H * kMat;
  hipLaunchKernelGGL(cal_to_f32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, c.R, out, n);
  return hipGetLastError();
}

hipError_t cal_key_mean(const uint16_t* k, int T, int H, float* mu, hipStream_t s) {
  hipLaunchKernelGGL(cal_key_mean_kernel, dim3(H), dim3(kD), 0, s, k, T, H, mu);
  return hipGetLastError();
}

}  // namespace int2kv

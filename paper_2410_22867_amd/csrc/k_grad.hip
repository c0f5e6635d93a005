// Parameter gradients of an energy loss, sum_f dL/dE_f dE_f/dtheta, from the
// state of the last FP64 compute (energy-loss training of the model; the
// paper's model is trained this way, its Background section cites the
// training papers).  Everything downstream of E_f is linear in the seed, so
// each centre-atom column is weighted by w_col = dL/dE of its frame and the
// unit-seed deltas stored by the force backward are reused where they exist.
//
// Fitting weights:   dW_l = sum_col X_l[col]^T w_col dz_l[col]  (column
//   reduction; MFMA with columns along K, split over column chunks whose
//   partial sums are written to a workspace and summed in chunk order).
// Embedding weights: the backward of each neighbour row is recomputed (as in
//   the force path, with g_T scaled by w_col; the last layer's tanh is read
//   from the activation store when that was kept); per 16-row tile the
//   activations and deltas are transposed through LDS so that the reduction
//   over rows is an MFMA product, accumulated in registers (w = 25) or in
//   per-work-group LDS sums (w = 32) that are written to the workspace and
//   summed in work-group order.
//   No global atomics.  The fitting gradients are bitwise deterministic; in
//   the embedding gradients a wave adds the columns it happened to take (and
//   with w = 32 the LDS sums take the waves' contributions in arrival order),
//   so they can differ in the last bits from run to run.
#include "dp_internal.h"
#include "dp_device.h"
#include "dp_embed.h"

namespace dpse {

// ------------------------------------------------------------ column weights
__global__ void k_col_weights(const int32_t* __restrict__ atom_at, const int32_t* __restrict__ frame_of,
                              const double* __restrict__ dLdE, double* __restrict__ w, int ncols) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= ncols) return;
  const int i = atom_at[c];
  w[c] = i >= 0 ? dLdE[frame_of[i]] : 0.0;
}

// ------------------------------------------------------------ fitting grads
// dW_l[m][n] = sum_col X_l[col][m] w[col] dz_l[col][n] and db_l[n] = sum_col
// w[col] dz_l[col][n], all three layers in one launch.  The columns of all
// types are cut into nchunks chunks of nearly equal length (chunk_range), so
// that every work-group has the same work and one round of two per CU takes
// them all: with chunks per type and layer some CUs held two work-groups and
// most one, which doubled the launch.  X and dz are read in the type the
// compute left them in (kinds 0 f64, 1 f32, 2 bf16, 3 f16).  train batch of
// 26,000 atoms: products, bias sums and their sums over chunks 1,280 -> 515 us.
struct WGradLayer {
  const void* X;
  const void* Y;
  int ldx, ldy, M, first;  // first: the layer's first m-group in the grid
  int64_t off;             // its [M + 1][N] block (bias row last) in a chunk's record
};
struct WGradArgs {
  WGradLayer l[3];
  const double* w;
  const int32_t* meta;
  int N, ntypes, nchunks;
  int64_t rec;      // doubles of a chunk's record
  double* part;     // [chunk][rec] partial sums
};

// Chunk k of nchunks (at least one per type, the others in proportion to the
// types' columns): type t and columns [c0, c1) of its segment.  For given t,
// [lo, hi) are the type's chunks.
__device__ __forceinline__ void chunk_span(const int32_t* meta, int ntypes, int nchunks, int t, int* lo, int* hi) {
  int64_t total = 0, before = 0;
  for (int q = 0; q < ntypes; ++q) {
    total += meta[2 * q];
    if (q < t) before += meta[2 * q];
  }
  const int64_t spare = nchunks - ntypes;
  *lo = (int)(t + (total > 0 ? spare * before / total : 0));
  *hi = (int)(t + 1 + (total > 0 ? spare * (before + meta[2 * t]) / total : 0));
}
__device__ __forceinline__ int chunk_range(const int32_t* meta, int ntypes, int nchunks, int k, int* c0, int* c1) {
  for (int t = 0; t < ntypes; ++t) {
    int lo, hi;
    chunk_span(meta, ntypes, nchunks, t, &lo, &hi);
    if (k >= lo && k < hi) {
      const int64_t n = meta[2 * t];
      *c0 = (int)(n * (k - lo) / (hi - lo));
      *c1 = (int)(n * (k - lo + 1) / (hi - lo));
      return t;
    }
  }
  return -1;
}

template <int K>
__device__ __forceinline__ double load_f64(const void* p, int64_t i) {
  if constexpr (K == 0) return static_cast<const double*>(p)[i];
  if constexpr (K == 1) return (double)static_cast<const float*>(p)[i];
  if constexpr (K == 2) return (double)PrecBF16::tof(static_cast<const uint16_t*>(p)[i]);
  if constexpr (K == 3) return (double)PrecF16::tof(static_cast<const uint16_t*>(p)[i]);
}

// Work-group mg owns MT m-tiles of out; its wave w owns n-tiles
// NT w ... NT w + NT - 1 (slots past the last tile repeat it and are not
// stored), so the four waves read the same X values (served once from L1)
// and different Y.  Per k-step of 4 columns a lane loads one value of X per
// m-tile and one of Y (scaled by w) per n-tile; the next step's operands are
// requested before the current products issue (two register buffers used
// alternately).  m-group 0 also sums the scaled Y (the bias row).
template <int XK, int YK, int MT, int NT>
__device__ __forceinline__ void wgrad_tiles(const WGradLayer& L, int N, const double* w, int cb, int c0, int c1, int mg,
                                            double* out) {
  const int lane = threadIdx.x & 63, ng = threadIdx.x >> 6;
  const int r16 = lane & 15, g = lane >> 4;
  const int mtiles = L.M / 16, ntiles = N / 16;
  if (ng * NT >= ntiles) return;
  int mt[MT], nt[NT];
#pragma unroll
  for (int j = 0; j < MT; ++j) mt[j] = min(mg * MT + j, mtiles - 1);
#pragma unroll
  for (int i = 0; i < NT; ++i) nt[i] = min(ng * NT + i, ntiles - 1);
  d4 acc[MT][NT];
  double bs[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i) bs[i] = 0.0;
#pragma unroll
  for (int j = 0; j < MT; ++j)
#pragma unroll
    for (int i = 0; i < NT; ++i) acc[j][i] = d4{0.0, 0.0, 0.0, 0.0};
  // raw operands and the column weight are buffered and the weight is
  // applied when the step consumes them; columns past the chunk load the
  // chunk's last column (no branch around a load, so nothing forces an
  // early wait) and get weight 0
  double xA[MT], yA[NT], xB[MT], yB[NT], wA, wB;
  auto load = [&](int c, double* xv, double* yv, double& wv_) {
    const int64_t col = cb + min(c + g, c1 - 1);
    wv_ = w[col];
#pragma unroll
    for (int j = 0; j < MT; ++j) xv[j] = load_f64<XK>(L.X, col * L.ldx + mt[j] * 16 + r16);
#pragma unroll
    for (int i = 0; i < NT; ++i) yv[i] = load_f64<YK>(L.Y, col * L.ldy + nt[i] * 16 + r16);
  };
  auto step = [&](int c, const double* xv, const double* yv, double wl) {
    const double wc = c + g < c1 ? wl : 0.0;
    double ys[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) ys[i] = yv[i] * wc;
    if (mg == 0) {
#pragma unroll
      for (int i = 0; i < NT; ++i) bs[i] += ys[i];
    }
#pragma unroll
    for (int j = 0; j < MT; ++j)
#pragma unroll
      for (int i = 0; i < NT; ++i) acc[j][i] = mfma_f64(xv[j], ys[i], acc[j][i]);
  };
  if (c0 < c1) {
    load(c0, xA, yA, wA);
    int c = c0;
    for (; c + 4 < c1; c += 8) {
      load(c + 4, xB, yB, wB);
      __builtin_amdgcn_sched_barrier(0);
      step(c, xA, yA, wA);
      __builtin_amdgcn_sched_barrier(0);
      load(c + 8, xA, yA, wA);  // past c1: weight 0
      __builtin_amdgcn_sched_barrier(0);
      step(c + 4, xB, yB, wB);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (c < c1) step(c, xA, yA, wA);
  }
#pragma unroll
  for (int j = 0; j < MT; ++j) {
    if (mg * MT + j >= mtiles) continue;
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      if (ng * NT + i >= ntiles) continue;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = mt[j] * 16 + 4 * v + g;
        const int n = nt[i] * 16 + r16;
        out[(int64_t)m * N + n] = acc[j][i][v];
      }
    }
  }
  if (mg == 0) {
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      bs[i] += shfl_xor_d(bs[i], 16);
      bs[i] += shfl_xor_d(bs[i], 32);
      if (g == 0 && ng * NT + i < ntiles) out[(int64_t)L.M * N + nt[i] * 16 + r16] = bs[i];
    }
  }
}

constexpr int kWgMT = 4, kWgNT = 4;

template <int X1, int Y1, int X23, int Y23>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_wgrad_cols(WGradArgs a) {
  int c0 = 0, c1 = 0;
  const int t = chunk_range(a.meta, a.ntypes, a.nchunks, blockIdx.x, &c0, &c1);
  if (t < 0) return;
  const int cb = a.meta[2 * t + 1];
  const int y = blockIdx.y;
  double* out = a.part + (int64_t)blockIdx.x * a.rec;
  if (y < a.l[1].first) {
    wgrad_tiles<X1, Y1, kWgMT, kWgNT>(a.l[0], a.N, a.w, cb, c0, c1, y, out + a.l[0].off);
  } else {
    const WGradLayer& L = y < a.l[2].first ? a.l[1] : a.l[2];
    wgrad_tiles<X23, Y23, kWgMT, kWgNT>(L, a.N, a.w, cb, c0, c1, y - L.first, out + L.off);
  }
}

// grad of element e of a record (blocks [M + 1][N] of the layers) = the sum
// over the type's chunks, in chunk order
struct WSumArgs {
  const double* part;
  const int32_t* meta;
  int ntypes, nchunks;
  int64_t rec, off[3], wdst[3], bdst[3], wlen[3], type_stride;
  double* grad;
};
__global__ void k_wgrad_sum(WSumArgs a) {
  const int t = blockIdx.y;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= a.rec) return;
  int lo, hi;
  chunk_span(a.meta, a.ntypes, a.nchunks, t, &lo, &hi);
  const double* p = a.part + e;
  double acc = 0.0;
  for (int c = lo; c < hi; ++c) acc += p[(int64_t)c * a.rec];
  const int l = e < a.off[1] ? 0 : e < a.off[2] ? 1 : 2;
  const int64_t k = e - a.off[l];
  a.grad[t * a.type_stride + (k < a.wlen[l] ? a.wdst[l] + k : a.bdst[l] + (k - a.wlen[l]))] = acc;
}

// Output layer: part[t][chunk][n] = sum over the chunk's 64 columns of w h3[n]
// (n < N) and of w (n = N)
constexpr int kWoChunk = 64;
template <int K>
__global__ __launch_bounds__(320) void k_wout_cols(const void* __restrict__ h3, int ld, const double* __restrict__ w,
                                                   const int32_t* __restrict__ meta, int N, int nchunks,
                                                   double* __restrict__ part) {
  const int t = blockIdx.y, n = threadIdx.x;
  const int n_t = meta[2 * t], cb = meta[2 * t + 1];
  const int c0 = blockIdx.x * kWoChunk;
  if (c0 >= n_t || n > N) return;
  const int c1 = min(n_t, c0 + kWoChunk);
  double acc = 0.0;
#pragma unroll 8
  for (int c = c0; c < c1; ++c) {
    const int64_t col = cb + c;
    acc = fma(w[col], n < N ? load_f64<K>(h3, col * ld + n) : 1.0, acc);
  }
  part[((int64_t)t * nchunks + blockIdx.x) * (N + 1) + n] = acc;
}
// 16 outputs per work-group, their chunks in 16 interleaved sums added in a
// fixed order; output N goes to b_out and to e_bias
__global__ __launch_bounds__(256) void k_wout_sum(const double* __restrict__ part, const int32_t* __restrict__ meta, int N,
                                                  int nchunks, double* __restrict__ grad, int64_t type_stride,
                                                  int64_t w_off, int64_t b_off, int64_t e_off) {
  __shared__ double red[16][16];
  const int t = blockIdx.y, l = threadIdx.x & 15, q = threadIdx.x >> 4, n = blockIdx.x * 16 + l;
  const int used = (meta[2 * t] + kWoChunk - 1) / kWoChunk;
  double acc = 0.0;
  if (n <= N)
    for (int c = q; c < used; c += 16) acc += part[((int64_t)t * nchunks + c) * (N + 1) + n];
  red[q][l] = acc;
  __syncthreads();
  if (q != 0 || n > N) return;
  acc = 0.0;
#pragma unroll
  for (int k = 0; k < 16; ++k) acc += red[k][l];
  if (n < N) {
    grad[t * type_stride + w_off + n] = acc;
  } else {
    grad[t * type_stride + b_off] = acc;
    grad[e_off + t] = acc;
  }
}

// ------------------------------------------------------------ embedding grads
struct EGradArgs {
  const int32_t* atom_at;
  const int32_t* meta;
  const double* R;
  const int32_t* nnei;
  const double* frag64;
  const double* vec64;
  int64_t vec_per_net;
  EmbFragOffsets fo;
  const void* gT;   // FP64, or FP32 when gt32
  int gt32;
  const double* wcol;
  double* grad;
  double* part;     // [net][slot][kEgRec] partial records
  int nslots;
  int64_t offW[kMaxT * kMaxT][3], offB[kMaxT * kMaxT][3];
  int ntypes, nm;
  int ngroups;      // work-groups per net (contiguous column ranges)
  int32_t* ctr;     // [nets][ngroups][32] per-work-group column counters
  int sec[kMaxT + 1];
  double inv_nm;
  // last embedding layer's tanh per 16-row tile of the forward pass
  // ([N, tpa, m1, 16]) when it was stored, else null (recomputed)
  const double* act;
  int tpa;
  int toff[kMaxT + 1];
  const double* tanh_lut;
};

// g_T row (four values) k of the columns' [m1] rows
__device__ __forceinline__ d4 g_T_of(const EGradArgs& A, int64_t k) {
  if (A.gt32) {
    const f4 x = static_cast<const f4*>(A.gT)[k];
    return d4{(double)x[0], (double)x[1], (double)x[2], (double)x[3]};
  }
  return static_cast<const d4*>(A.gT)[k];
}

template <int W>
__device__ __forceinline__ int e_feat1(int p) { return p < W ? p : -1; }
template <int W>
__device__ __forceinline__ int e_feat2(int p) { return (p & 31) < W ? (p >> 5) * W + (p & 31) : -1; }
template <int W>
__device__ __forceinline__ int e_feat3(int p) {
  const int f = e_feat2<W>(p & 63);
  return f < 0 ? -1 : (p >> 6) * 2 * W + f;
}

// waves per work-group of the w = 32 embedding-gradient kernel: one
// work-group per CU holds the slot-indexed accumulators (82 KB) and per-wave
// buffers (20.5 KB)
constexpr int kEgWaves = 3;
// partial record of one work-group (slot-indexed): W3 | W2 | b3 | b2 | b1 | W1
constexpr int kEgW3 = 0, kEgW2 = 64 * 128, kEgB3 = kEgW2 + 32 * 64, kEgB2 = kEgB3 + 128, kEgB1 = kEgB2 + 64,
              kEgW1 = kEgB1 + 32, kEgRec = kEgW1 + 32;

template <int W, bool ST>
__global__ __launch_bounds__(256) void k_embed_grad_f64(EGradArgs A) {
  constexpr int M1 = 4 * W, GW = kEgWaves;
  // per-block accumulators (slot-indexed)
  __shared__ double aW3[64 * 128];
  __shared__ double aW2[32 * 64];
  __shared__ double aW1[32], aB1[32], aB2[64], aB3[128];
  // per-wave transposition buffers [row][slot]: h2 | one half of dz3, then
  // h1 | dz2 | dz1 | s
  __shared__ double tb[GW][16][129];
  __shared__ d4 gts[GW][M1];  // feature-indexed
  const int net = blockIdx.y;
  const int ti = net / A.ntypes, tj = net - ti * A.ntypes;
  const int n_t = A.meta[2 * ti], cb = A.meta[2 * ti + 1];
  // contiguous column range of this work-group; its waves take the columns
  // from a counter that only this work-group uses (next one requested ahead)
  const int c_lo = (int)((int64_t)n_t * blockIdx.x / gridDim.x);
  const int c_hi = (int)((int64_t)n_t * (blockIdx.x + 1) / gridDim.x);
  double* pr = A.part + ((int64_t)net * A.nslots + blockIdx.x) * kEgRec;
  if (c_lo >= c_hi) {
    for (int k = threadIdx.x; k < kEgRec; k += 64 * GW) pr[k] = 0.0;
    return;
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int r16 = lane & 15, g = lane >> 4;
  int* const next_col = A.ctr + (net * gridDim.x + blockIdx.x) * 32;
  if (threadIdx.x == 0) atomicExch(next_col, c_lo);
  auto take = [&]() {
    int k = 0;
    if (lane == 0) k = atomicAdd(next_col, 1);
    return k;
  };
  for (int k = threadIdx.x; k < 64 * 128; k += 64 * GW) aW3[k] = 0.0;
  for (int k = threadIdx.x; k < 32 * 64; k += 64 * GW) aW2[k] = 0.0;
  for (int k = threadIdx.x; k < 128; k += 64 * GW) {
    aB3[k] = 0.0;
    if (k < 64) aB2[k] = 0.0;
    if (k < 32) { aB1[k] = 0.0; aW1[k] = 0.0; }
  }
  __syncthreads();
  const double* base = A.frag64 + net * A.fo.per_net;
  const double* vec = A.vec64 + net * A.vec_per_net;
  double w1s[2][4], b1s[2][4];
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      w1s[mt][v] = vec[16 * mt + 4 * v + g];
      b1s[mt][v] = vec[32 + 16 * mt + 4 * v + g];
    }
  double (*T)[129] = tb[wv];
  for (int c_next = take();;) {
    const int c = __builtin_amdgcn_readfirstlane(c_next);
    if (c >= c_hi) break;
    c_next = take();
    const int col = cb + c;
    const int i = A.atom_at[col];
    const double wc = A.wcol[col];
    {
      wave_lds_sync();
      for (int a = lane; a < M1; a += 64) gts[wv][a] = g_T_of(A, (int64_t)col * M1 + a) * (A.inv_nm * wc);
      wave_lds_sync();
    }
    const int nn = A.nnei[i * kMaxT + tj];
    const double* Rs = A.R + ((int64_t)i * A.nm + A.sec[tj]) * 4;
    const env_rsrc_t Rb = env_rsrc(Rs, nn);
    d4 R_next = env_row(Rb, r16);  // row of the next tile is always in flight
    for (int r0 = 0; r0 < nn; r0 += 16) {
      const double* F2 = opaque(base + A.fo.F2);
      const double* F3 = opaque(base + A.fo.F3t);
      const double* B3 = opaque(base + A.fo.B3);
      const double* B2 = opaque(base + A.fo.B2);
      const int row = r0 + r16;
      const d4 Rrow = R_next;  // zero past the section's real rows
      R_next = env_row(Rb, row + 16);
      const double s = Rrow[0];
      double t1[2][4];
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int v = 0; v < 4; ++v) t1[mt][v] = tanh_d(fma(s, w1s[mt][v], b1s[mt][v]));
      double t2[4][4], h2[4][4];
      // weight fragments are requested one group ahead of their products
      // (one wave per SIMD: nothing else hides their latency)
      double f2[2][8];
      auto ld_f2 = [&](int ot, double* f) {
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            f[mt * 4 + v] = F2[((ot * 2 + mt) * 4 + v) * 64 + lane];
      };
      ld_f2(0, f2[0]);
#pragma unroll
      for (int ot = 0; ot < 4; ++ot) {
        if (ot + 1 < 4) ld_f2(ot + 1, f2[(ot + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
        d4 z = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            z = mfma_f64(f2[ot & 1][mt * 4 + v], t1[mt][v], z);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          t2[ot][v] = tanh_d(z[v] + vec[64 + 16 * ot + 4 * v + g]);
          h2[ot][v] = t1[ot & 1][v] + t2[ot][v];
        }
      }
      wave_lds_sync();
      // h2 -> T[row][0..64)
#pragma unroll
      for (int ot = 0; ot < 4; ++ot)
#pragma unroll
        for (int v = 0; v < 4; ++v) T[r16][16 * ot + 4 * v + g] = h2[ot][v];
      double skip2[4][4];
      d4 dh2a[4];
#pragma unroll
      for (int ot = 0; ot < 4; ++ot) {
        dh2a[ot] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int v = 0; v < 4; ++v) skip2[ot][v] = 0.0;
      }
      // stored t3 of the tile: slot p = 64 oo + 16 o4 + 4 v + g holds feature
      // 2W oo + W (o4 / 2) + 16 (o4 % 2) + 4 v + g when 16 (o4 % 2) + 4 v + g
      // < W; a padding slot may read past its record (one record of slack at
      // the end of the store) and its value is not used
      const double* rec =
          ST ? A.act + ((int64_t)i * A.tpa + A.toff[tj] + (r0 >> 4)) * (M1 * 16) + g * 16 + r16 : nullptr;
#pragma unroll 1
      for (int oo = 0; oo < 2; ++oo) {
        const double* F3o = opaque(F3 + oo * 4 * 16 * 64);
        const double* B3o = opaque(B3 + oo * 4 * 4 * 64);
        double t3v[16];
        if constexpr (ST) {
#pragma unroll
          for (int o4 = 0; o4 < 4; ++o4)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const int lo = 16 * (o4 & 1) + 4 * v;
              t3v[o4 * 4 + v] = (lo < W) ? rec[(oo * 2 * W + (o4 >> 1) * W + lo) * 16] : 0.0;
            }
        }
        double fb[2][16];
        auto ld_b3 = [&](int o4, double* f) {
#pragma unroll
          for (int i2 = 0; i2 < 4; ++i2)
#pragma unroll
            for (int v = 0; v < 4; ++v)
              f[i2 * 4 + v] = B3o[((i2 * 8 + o4) * 4 + v) * 64 + lane];
        };
        ld_b3(0, fb[0]);
#pragma unroll
        for (int o4 = 0; o4 < 4; ++o4) {
          if (o4 + 1 < 4) ld_b3(o4 + 1, fb[(o4 + 1) & 1]);
          __builtin_amdgcn_sched_barrier(0);
          d4 z = {0.0, 0.0, 0.0, 0.0};
          if constexpr (!ST) {
            const double* b3 = vec + 128 + 16 * (4 * oo + o4) + g;
            z = d4{b3[0], b3[4], b3[8], b3[12]};
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
#pragma unroll
              for (int v = 0; v < 4; ++v) z = mfma_f64(F3o[((o4 * 4 + mt) * 4 + v) * 64 + lane], h2[mt][v], z);
          }
          double dz3[4];
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int a = e_feat3<W>(16 * (4 * oo + o4) + 4 * v + g);
            const double t3 = ST ? t3v[o4 * 4 + v] : tanh_d(z[v]);
            double dG = 0.0;
            if (a >= 0) {
              const d4 gt = gts[wv][a];
              dG = gt[0] * Rrow[0] + gt[1] * Rrow[1] + gt[2] * Rrow[2] + gt[3] * Rrow[3];
            }
            dz3[v] = a >= 0 ? dG * (1.0 - t3 * t3) : 0.0;
            skip2[o4][v] += dG;
            T[r16][64 + 16 * o4 + 4 * v + g] = dz3[v];
          }
#pragma unroll
          for (int i2 = 0; i2 < 4; ++i2)
#pragma unroll
            for (int v = 0; v < 4; ++v)
              dh2a[i2] = mfma_f64(fb[o4 & 1][i2 * 4 + v], dz3[v], dh2a[i2]);
        }
        wave_lds_sync();
        // dW3[p][q] += sum_row h2[row][p] dz3[row][q];  db3[q] += sum_row dz3[row][q]  (q in this half)
        const double one = 1.0;
        // the h2 operands are the same for every q tile: read once
        double hA[4][4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
          for (int pt = 0; pt < 4; ++pt) hA[ks][pt] = T[4 * ks + g][16 * pt + r16];
#pragma unroll 1
        for (int qh = 0; qh < 4; ++qh) {
          const int qt = 4 * oo + qh;
          d4 acc[4] = {{0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}};
          d4 bacc = {0, 0, 0, 0};
          double bqv[4];
#pragma unroll
          for (int ks = 0; ks < 4; ++ks) bqv[ks] = T[4 * ks + g][64 + 16 * qh + r16];
#pragma unroll
          for (int ks = 0; ks < 4; ++ks) {
            const double bq = bqv[ks];
#pragma unroll
            for (int pt = 0; pt < 4; ++pt) acc[pt] = mfma_f64(hA[ks][pt], bq, acc[pt]);
            bacc = mfma_f64(one, bq, bacc);
          }
#pragma unroll
          for (int pt = 0; pt < 4; ++pt)
#pragma unroll
            for (int v = 0; v < 4; ++v) atomicAdd(&aW3[(16 * pt + 4 * v + g) * 128 + 16 * qt + r16], acc[pt][v]);
          if (g == 0) atomicAdd(&aB3[16 * qt + r16], bacc[0]);
        }
        wave_lds_sync();  // the next half overwrites dz3
      }
      // dz2 = (dh2 + skip)(1 - t2^2); dh1 = W2 dz2 + skip; dz1 = dh1 (1 - t1^2)
      double dz2[4][4], skip1[2][4];
      double fb2[2][16];
      auto ld_b2 = [&](int i2, double* f) {
#pragma unroll
        for (int o = 0; o < 4; ++o)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            f[o * 4 + v] = B2[((i2 * 4 + o) * 4 + v) * 64 + lane];
      };
      ld_b2(0, fb2[0]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i2 = 0; i2 < 2; ++i2)
#pragma unroll
        for (int v = 0; v < 4; ++v) skip1[i2][v] = 0.0;
#pragma unroll
      for (int i2 = 0; i2 < 4; ++i2)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const double dh2 = dh2a[i2][v] + skip2[i2][v];
          dz2[i2][v] = dh2 * (1.0 - t2[i2][v] * t2[i2][v]);
          skip1[i2 & 1][v] += dh2;
        }
      double dz1[2][4];
#pragma unroll
      for (int i2 = 0; i2 < 2; ++i2) {
        if (i2 == 0) ld_b2(1, fb2[1]);
        __builtin_amdgcn_sched_barrier(0);
        d4 z = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int o = 0; o < 4; ++o)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            z = mfma_f64(fb2[i2][o * 4 + v], dz2[o][v], z);
#pragma unroll
        for (int v = 0; v < 4; ++v) dz1[i2][v] = (z[v] + skip1[i2][v]) * (1.0 - t1[i2][v] * t1[i2][v]);
      }
      wave_lds_sync();
      // buffer: h1 [0,32), dz2 [32,96), dz1 [96,128), s at 128
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          T[r16][16 * mt + 4 * v + g] = t1[mt][v];
          T[r16][96 + 16 * mt + 4 * v + g] = dz1[mt][v];
        }
#pragma unroll
      for (int ot = 0; ot < 4; ++ot)
#pragma unroll
        for (int v = 0; v < 4; ++v) T[r16][32 + 16 * ot + 4 * v + g] = dz2[ot][v];
      if (g == 0) T[r16][128] = row < nn ? s : 0.0;
      wave_lds_sync();
      {
        const double one = 1.0;
        double h1A[4][2];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
          for (int pt = 0; pt < 2; ++pt) h1A[ks][pt] = T[4 * ks + g][16 * pt + r16];
#pragma unroll 1
        for (int qt = 0; qt < 4; ++qt) {
          d4 acc[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
          d4 bacc = {0, 0, 0, 0};
          double bqv[4];
#pragma unroll
          for (int ks = 0; ks < 4; ++ks) bqv[ks] = T[4 * ks + g][32 + 16 * qt + r16];
#pragma unroll
          for (int ks = 0; ks < 4; ++ks) {
            const double bq = bqv[ks];
#pragma unroll
            for (int pt = 0; pt < 2; ++pt) acc[pt] = mfma_f64(h1A[ks][pt], bq, acc[pt]);
            bacc = mfma_f64(one, bq, bacc);
          }
#pragma unroll
          for (int pt = 0; pt < 2; ++pt)
#pragma unroll
            for (int v = 0; v < 4; ++v) atomicAdd(&aW2[(16 * pt + 4 * v + g) * 64 + 16 * qt + r16], acc[pt][v]);
          if (g == 0) atomicAdd(&aB2[16 * qt + r16], bacc[0]);
        }
        // dW1[q] = sum_row s dz1[q] and db1[q] = sum_row dz1[q] as rows 0
        // and 1 of one product (A row 0: s, row 1: 1)
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) {
          d4 wacc = {0, 0, 0, 0};
#pragma unroll
          for (int ks = 0; ks < 4; ++ks) {
            const int rr = 4 * ks + g;
            const double bq = T[rr][96 + 16 * qt + r16];
            const double sr = T[rr][128];  // read by every lane, then selected
            wacc = mfma_f64(r16 == 0 ? sr : (r16 == 1 ? one : 0.0), bq, wacc);
          }
          if (g == 0) atomicAdd(&aW1[16 * qt + r16], wacc[0]);
          if (g == 1) atomicAdd(&aB1[16 * qt + r16], wacc[0]);
        }
      }
    }
  }
  __syncthreads();
  // slot-indexed block sums -> this work-group's partial record
  for (int k = threadIdx.x; k < 64 * 128; k += 64 * GW) pr[kEgW3 + k] = aW3[k];
  for (int k = threadIdx.x; k < 32 * 64; k += 64 * GW) pr[kEgW2 + k] = aW2[k];
  for (int k = threadIdx.x; k < 128; k += 64 * GW) {
    pr[kEgB3 + k] = aB3[k];
    if (k < 64) pr[kEgB2 + k] = aB2[k];
    if (k < 32) {
      pr[kEgB1 + k] = aB1[k];
      pr[kEgW1 + k] = aW1[k];
    }
  }
}

// sums the partial records of the work-groups that held columns, in
// work-group order, and maps slots to the flat parameter layout
template <int W>
__global__ void k_egrad_reduce(EGradArgs A) {
  const int net = blockIdx.y;
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= kEgRec) return;
  const int used = A.ngroups;
  int dst = -1;
  if (k < kEgW2) {
    const int fi = e_feat2<W>(k >> 7), fo = e_feat3<W>(k & 127);
    if (fi >= 0 && fo >= 0) dst = (int)A.offW[net][2] + fi * 4 * W + fo;
  } else if (k < kEgB3) {
    const int kk = k - kEgW2, fi = e_feat1<W>(kk >> 6), fo = e_feat2<W>(kk & 63);
    if (fi >= 0 && fo >= 0) dst = (int)A.offW[net][1] + fi * 2 * W + fo;
  } else if (k < kEgB2) {
    const int f3 = e_feat3<W>(k - kEgB3);
    if (f3 >= 0) dst = (int)A.offB[net][2] + f3;
  } else if (k < kEgB1) {
    const int f2 = e_feat2<W>(k - kEgB2);
    if (f2 >= 0) dst = (int)A.offB[net][1] + f2;
  } else if (k < kEgW1) {
    if (k - kEgB1 < W) dst = (int)A.offB[net][0] + (k - kEgB1);
  } else {
    if (k - kEgW1 < W) dst = (int)A.offW[net][0] + (k - kEgW1);
  }
  if (dst < 0) return;
  const double* p = A.part + (int64_t)net * A.nslots * kEgRec + k;
  double acc = 0.0;
  for (int c = 0; c < used; ++c) acc += p[(int64_t)c * kEgRec];
  A.grad[dst] = acc;
}

// ------------------------------------------------------------ w = 25
// The same gradients with the denser layout of the force kernels (13 + 25
// element groups of four slots instead of 14 + 28) and every sum over rows in
// registers.  A wave keeps dW3 (52 x 100: 82 FP64 accumulators per lane) and
// dW2 (28 x 52: 23) as matrix-core accumulators over all its columns and dW1,
// db1 as 14 vector ones, so one wave per SIMD runs and nothing is added
// through LDS; the weights (one copy of W2 and W3, read in both directions),
// the tanh table and the transposition buffers fill the 160 KB.  The
// bias gradients are rows of dW2 and dW3: slots of h1 and h2 that hold copies
// (no outgoing weights) carry 1.0 in the transposed buffers.
//   ACT 0 recomputes the last layer, 1 reads its tanh from the store, 2
// recomputes and writes the store.
// Training batch of 16 frames (26,000 atoms): 2,780 -> 1,700 us with the store
// (5,120 -> 2,220 us recomputing; 2,330 us recomputing and storing, where the
// mixed forms ran the FP64 forward for 1,080 us first); the matrix cores are
// busy half of the time, operands requested an element ahead (1,766 us without).
typedef EmbLay<25> L25;
constexpr int kG3 = 52, kG3N = 100, kG2 = 28;         // h2, dz3, h1 columns
constexpr int kGr2 = kG3 * kG3N, kGr1 = kGr2 + kG2 * kG3;  // record: dW3 | dW2 | b1 | W1
constexpr int kGrRec = kGr1 + 2 * kG2;
constexpr int kTS = 113;  // row stride of the transposition buffers (17 mod 32: no bank conflicts)

template <int ACT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void k_embed_grad25(EGradArgs A) {
  constexpr int W = 25, M1 = 100, GW = 4;
  constexpr int n1 = L25::n1, n2 = L25::n2, n3 = L25::n3;
  constexpr int FT = 66;  // doubles per k element of a full tile: read transposed with two-way conflicts only
  // W3 as the B3 operand (m = layer-2 element, k = layer-3 element) and W2 as
  // the B2 operand (m = layer-1 element, k = layer-2 element): full tiles
  // [tile][k][66], single elements [m][k][16]
  constexpr int o3s = 2 * n3 * FT - 8 * n3 * 16, N3W = 2 * n3 * FT + (n2 - 8) * n3 * 16;
  constexpr int o2s = n2 * FT - 4 * n2 * 16, N2W = n2 * FT + (n1 - 4) * n2 * 16;
  __shared__ double w3[N3W], w2[N2W], vec_s[kVecPerNet], lut[kTanhLutEntries];
  __shared__ double tb[GW][16 * kTS];
  __shared__ d4 gts[GW][M1];
  int grp = 0, ngrp = 1;
  const int net = net_of_group(A.meta, A.ntypes, gridDim.x, blockIdx.x, &grp, &ngrp, 0);
  double* pr = A.part + (int64_t)blockIdx.x * kGrRec;
  if (net < 0) return;
  const int ti = net / A.ntypes, tj = net - ti * A.ntypes;
  const int n_t = A.meta[2 * ti], cb = A.meta[2 * ti + 1];
  const int c_lo = part_start(n_t, grp, ngrp), c_hi = part_start(n_t, grp + 1, ngrp);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int r16 = lane & 15, g = lane >> 4;
  int* const next_col = A.ctr + blockIdx.x * 32;
  if (threadIdx.x == 0) atomicExch(next_col, c_lo);
  auto take = [&]() {
    int k = 0;
    if (lane == 0) k = atomicAdd(next_col, 1);
    return k;
  };
  {
    const double* src = A.frag64 + net * A.fo.per_net;
    for (int e = threadIdx.x; e < 2 * n3 * 64; e += 256) w3[(e >> 6) * FT + (e & 63)] = src[A.fo.B3 + e];
    for (int e = threadIdx.x; e < (n2 - 8) * n3 * 16; e += 256) w3[2 * n3 * FT + e] = src[A.fo.B3 + 2 * n3 * 64 + e];
    for (int e = threadIdx.x; e < n2 * 64; e += 256) w2[(e >> 6) * FT + (e & 63)] = src[A.fo.B2 + e];
    for (int e = threadIdx.x; e < (n1 - 4) * n2 * 16; e += 256) w2[n2 * FT + e] = src[A.fo.B2 + n2 * 64 + e];
    for (int e = threadIdx.x; e < kVecPerNet; e += 256) vec_s[e] = A.vec64[net * A.vec_per_net + e];
    for (int e = threadIdx.x; e < kTanhLutEntries; e += 256) lut[e] = A.tanh_lut[e];
  }
  __syncthreads();
  const int lo4 = (lane & 3) + 4 * (lane >> 4);
  // transposed reads: A[m][k] = W[k][m], m four elements e..e+3 (lane bits
  // 2-3: the element) or one
  const int tF = ((lane >> 2) & 3) * FT + 16 * (lane & 3) + g, tS = ((lane >> 2) & 3) * 16 + 4 * (lane & 3) + g;
  const int uF = 16 * (lane & 3) + g, uS = 4 * (lane & 3) + g;
  // Operands of a product's k element, one value per tile or single element
  // (wt: the weights, ns: offset of the single elements, whose index counts
  // on from the full tiles'; nk: the out elements); they are requested one
  // element ahead of the products that use them.
  // transposed: in element ei against out tiles with (first element, count)
  auto ld_fwd = [&](const double* wt, int ns, int nk, int full, int ei, int eo, int nv, double* f) {
    const double* p = ei < full ? wt + ((ei >> 2) * nk + eo) * FT + 4 * (ei & 3) : wt + ns + (ei * nk + eo) * 16;
    if (nv == 4) {
      f[0] = p[ei < full ? tF : tS];
    } else {
#pragma unroll
      for (int e = 0; e < nv; ++e) f[e] = p[(ei < full ? e * FT : e * 16) + (ei < full ? uF : uS)];
    }
  };
  // as the force backward reads them: m tile at element em, out element k
  auto ld_bwd = [&](const double* wt, int ns, int nk, int full, int em, int k, int nv, double* f) {
    if (em < full) {
      f[0] = wt[((em >> 2) * nk + k) * FT + lane];
    } else {
#pragma unroll
      for (int e = 0; e < nv; ++e) f[e] = wt[ns + ((em + e) * nk + k) * 16 + lo4];
    }
  };
  auto mma = [&](int nv, const double* f, double b, d4 z) {
    if (nv == 4) return mfma_f64(f[0], b, z);
#pragma unroll
    for (int e = 0; e < nv; ++e) z[e] = mfma4_f64(f[e], b, z[e]);
    return z;
  };
#define DPSE_FENCE __builtin_amdgcn_sched_barrier(0)
  d4 a3[6][3];       // dW3: dz3 columns 16 j.., h2 columns 16 p..
  double a3s[6];     // h2 columns 48..51
  double a3r[4];     // dz3 columns 96..99 against h2 columns 16 p..
  d4 a2[3];          // dW2: dz2 columns 16 j.., h1 columns 0..15
  double a2s[3][3];  // h1 columns 16 + 4 e..
  double a2r[2];     // dz2 columns 48..51 against h1 columns 16 p..
  double ab1[n1], aw1[n1];
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    a3s[j] = 0.0;
#pragma unroll
    for (int p = 0; p < 3; ++p) a3[j][p] = d4{0.0, 0.0, 0.0, 0.0};
  }
#pragma unroll
  for (int p = 0; p < 4; ++p) a3r[p] = 0.0;
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    a2[j] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int e = 0; e < 3; ++e) a2s[j][e] = 0.0;
  }
  a2r[0] = a2r[1] = 0.0;
#pragma unroll
  for (int e = 0; e < n1; ++e) ab1[e] = aw1[e] = 0.0;
  double* const T = tb[wv];
  double* const Tw = T + r16 * kTS + g;       // this lane's row, column g
  const double* const Tm = T + g * kTS + r16;  // row g, column r16 (operand reads: + 4 ks rows)
  const double* const Ts = T + g * kTS + (lane & 3);

  for (int c_next = c_lo < c_hi ? take() : c_hi;;) {
    const int c = __builtin_amdgcn_readfirstlane(c_next);
    if (c >= c_hi) break;
    c_next = take();
    const int col = cb + c;
    const int i = A.atom_at[col];
    const double wc = A.wcol[col];
    {
      wave_lds_sync();
      for (int p = lane; p < kP3; p += 64) {
        const int a = feat3d_of_slot<W>(p), cp = L25::col3(p);
        if (cp >= 0) gts[wv][cp] = g_T_of(A, (int64_t)col * M1 + a) * (A.inv_nm * wc);
      }
      wave_lds_sync();
    }
    const int nn = A.nnei[i * kMaxT + tj];
    const double* Rs = A.R + ((int64_t)i * A.nm + A.sec[tj]) * 4;
    const env_rsrc_t Rb = env_rsrc(Rs, nn);
    d4 R_next = env_row(Rb, r16);  // row of the next tile is always in flight
    for (int r0 = 0; r0 < nn; r0 += 16) {
      const int z0 = opaque_zero();
      const double* vec = vec_s + z0;
      const double* W3 = w3 + z0;
      const double* W2 = w2 + z0;
      const int row = r0 + r16;
      const d4 Rrow = R_next;  // zero past the section's real rows
      R_next = env_row(Rb, row + 16);
      const double s = Rrow[0];
      double* const rec =
          ACT ? const_cast<double*>(A.act) + ((int64_t)i * A.tpa + A.toff[tj] + (r0 >> 4)) * (M1 * 16) + r16 : nullptr;
      // stored t3, requested before layers 1-2 (addresses as in the force
      // backward: feature of slot 64 oo + 16 o4 + 4 v + g)
      double t3v[2][4][4];
      auto rec_at = [&](int oo, int o4, int v) {
        if (oo == 0 && o4 == 1 && v == 2) return (W - 1 + W * g) * 16;  // features 24, 49, 74, 99
        return (oo * 2 * W + (o4 >> 1) * W + 16 * (o4 & 1) + 4 * v + g) * 16;
      };
      if constexpr (ACT == 1) {
#pragma unroll
        for (int oo = 0; oo < 2; ++oo)
#pragma unroll
          for (int o4 = 0; o4 < 4; ++o4)
#pragma unroll
            for (int v = 0; v < nv3<W>(oo, o4); ++v) t3v[oo][o4][v] = rec[rec_at(oo, o4, v)];
      }
      double t1[2][4];
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int v = 0; v < nv1<W>(mt); ++v)
          t1[mt][v] = tanh_lut<7>(fma(s, vec[kV_W1 + 16 * mt + 4 * v + g], vec[kV_B1 + 16 * mt + 4 * v + g]), lut);
      double t2[4][4], h2[4][4];
      d4 z2[4];
#pragma unroll
      for (int ot = 0; ot < 4; ++ot) {
        const double* b2 = vec + kV_B2 + 16 * ot + g;
        z2[ot] = d4{b2[0], b2[4], b2[8], b2[12]};
      }
      {
        double f[2][4][4];
        auto ld = [&](int k, double (*q)[4]) {
#pragma unroll
          for (int ot = 0; ot < 4; ++ot) ld_fwd(W2, o2s, n2, 4, k, L25::e2(ot), nv2<W>(ot), q[ot]);
        };
        ld(0, f[0]);
#pragma unroll
        for (int k = 0; k < n1; ++k) {
          if (k + 1 < n1) ld(k + 1, f[(k + 1) & 1]);
          DPSE_FENCE;
#pragma unroll
          for (int ot = 0; ot < 4; ++ot) z2[ot] = mma(nv2<W>(ot), f[k & 1][ot], t1[k >> 2][k & 3], z2[ot]);
        }
      }
#pragma unroll
      for (int ot = 0; ot < 4; ++ot)
#pragma unroll
        for (int v = 0; v < nv2<W>(ot); ++v) {
          t2[ot][v] = tanh_lut<7>(z2[ot][v], lut);
          h2[ot][v] = t1[ot & 1][v] + t2[ot][v];
        }
      wave_lds_sync();
      // h2 -> columns [0, 52) (slot 26, a copy: 1.0 for the bias gradient)
#pragma unroll
      for (int ot = 0; ot < 4; ++ot)
#pragma unroll
        for (int v = 0; v < nv2<W>(ot); ++v)
          Tw[4 * (L25::e2(ot) + v)] = (ot == 1 && v == 2 && g == 2) ? 1.0 : h2[ot][v];
      // layer 3: dz3 per element, dh2 = W3 dz3
      double dz3[n3], skip2[4][4];
      d4 dh2a[4];
#pragma unroll
      for (int ot = 0; ot < 4; ++ot) {
        dh2a[ot] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int v = 0; v < 4; ++v) skip2[ot][v] = 0.0;
      }
      d4 z3[8];
      if constexpr (ACT != 1) {
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const double* b3 = vec + kV_B3S + 16 * t + g;
          z3[t] = d4{b3[0], b3[4], b3[8], b3[12]};
        }
        // tiles of a half at a time
#pragma unroll
        for (int oo = 0; oo < 2; ++oo) {
          double f[2][4][4];
          auto ld = [&](int k, double (*q)[4]) {
#pragma unroll
            for (int t = 0; t < 4; ++t) ld_fwd(W3, o3s, n3, 8, k, L25::e3(4 * oo + t), nv3<W>(oo, t), q[t]);
          };
          ld(0, f[0]);
#pragma unroll
          for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int v = 0; v < nv2<W>(mt); ++v) {
              const int seq = (mt > 0) * 4 + (mt > 1) * 3 + (mt > 2) * 4 + v;  // layer-2 elements in slot order
              const int nx = seq + 1, nmt = nx < 4 ? 0 : nx < 7 ? 1 : nx < 11 ? 2 : 3;
              const int nv_ = nx - (nmt > 0) * 4 - (nmt > 1) * 3 - (nmt > 2) * 4;
              if (nx < n2) ld(L25::e2(nmt) + nv_, f[nx & 1]);
              DPSE_FENCE;
#pragma unroll
              for (int t = 0; t < 4; ++t)
                z3[4 * oo + t] = mma(nv3<W>(oo, t), f[seq & 1][t], h2[mt][v], z3[4 * oo + t]);
            }
        }
      }
#pragma unroll
      for (int oo = 0; oo < 2; ++oo)
#pragma unroll
        for (int o4 = 0; o4 < 4; ++o4) {
          const int e0 = L25::e3(4 * oo + o4);
#pragma unroll
          for (int v = 0; v < nv3<W>(oo, o4); ++v) {
            const bool real = (o4 == 1 && v == 2) || 16 * (o4 & 1) + 4 * v + g < W;
            double t3;
            if constexpr (ACT == 1) {
              t3 = real ? t3v[oo][o4][v] : 0.0;
            } else {
              t3 = tanh_lut<7>(z3[4 * oo + o4][v], lut);
              if constexpr (ACT == 2)
                if (real) rec[rec_at(oo, o4, v)] = t3;
            }
            const d4 gt = gts[wv][4 * (e0 + v) + g];
            const double dG = gt[0] * Rrow[0] + gt[1] * Rrow[1] + gt[2] * Rrow[2] + gt[3] * Rrow[3];
            dz3[e0 + v] = dG * (1.0 - t3 * t3);
            skip2[o4][v] += dG;
          }
        }
      // dh2 and dW3; the dz3 columns pass through the buffer in two batches
#pragma unroll
      for (int bt = 0; bt < 2; ++bt) {
        constexpr int kB0 = 12;  // elements of the first batch (three 16-column tiles)
        const int eb = bt ? kB0 : 0, ee = bt ? n3 : kB0;
        if (bt) wave_lds_sync();
#pragma unroll
        for (int e = eb; e < ee; ++e) Tw[kG3 + 4 * (e - eb)] = dz3[e];
        double f[2][4][4], x[2][8];
        auto ldb = [&](int e, double (*q)[4]) {
#pragma unroll
          for (int i2 = 0; i2 < 4; ++i2) ld_bwd(W3, o3s, n3, 8, L25::e2(i2), e, nv2<W>(i2), q[i2]);
        };
        auto ldw = [&](int ks, double* q) {
#pragma unroll
          for (int p = 0; p < 3; ++p) q[p] = Tm[4 * ks * kTS + 16 * p];
          q[3] = Ts[4 * ks * kTS + 48];
#pragma unroll
          for (int j = 0; j < 3; ++j) q[4 + j] = Tm[4 * ks * kTS + kG3 + 16 * j];
          if (bt) q[7] = Ts[4 * ks * kTS + kG3 + 48];
        };
        ldb(eb, f[eb & 1]);
        wave_lds_sync();
#pragma unroll
        for (int e = eb; e < ee; ++e) {
          if (e + 1 < ee) ldb(e + 1, f[(e + 1) & 1]);
          else ldw(0, x[0]);
          DPSE_FENCE;
#pragma unroll
          for (int i2 = 0; i2 < 4; ++i2) dh2a[i2] = mma(nv2<W>(i2), f[e & 1][i2], dz3[e], dh2a[i2]);
        }
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          if (ks < 3) ldw(ks + 1, x[(ks + 1) & 1]);
          DPSE_FENCE;
          const double* q = x[ks & 1];
#pragma unroll
          for (int j = 0; j < 3; ++j) {
#pragma unroll
            for (int p = 0; p < 3; ++p) a3[3 * bt + j][p] = mfma_f64(q[p], q[4 + j], a3[3 * bt + j][p]);
            a3s[3 * bt + j] = mfma4_f64(q[3], q[4 + j], a3s[3 * bt + j]);
          }
          if (bt) {
#pragma unroll
            for (int p = 0; p < 4; ++p) a3r[p] = mfma4_f64(q[7], q[p], a3r[p]);
          }
        }
      }
      // dz2 = (dh2 + skip)(1 - t2^2); dh1 = W2 dz2 + skip; dz1 = dh1 (1 - t1^2)
      double dz2[4][4];
      d4 z1[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll
      for (int i2 = 0; i2 < 4; ++i2)
#pragma unroll
        for (int v = 0; v < nv2<W>(i2); ++v) {
          const double dh2 = dh2a[i2][v] + skip2[i2][v];
          dz2[i2][v] = dh2 * (1.0 - t2[i2][v] * t2[i2][v]);
          z1[i2 & 1][v] += dh2;
        }
      wave_lds_sync();
      // buffer: h1 [0, 28) (slot 25, a copy: 1.0), dz2 [28, 80)
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int v = 0; v < nv1<W>(mt); ++v) Tw[4 * (4 * mt + v)] = (mt == 1 && v == 2 && g == 1) ? 1.0 : t1[mt][v];
#pragma unroll
      for (int ot = 0; ot < 4; ++ot)
#pragma unroll
        for (int v = 0; v < nv2<W>(ot); ++v) Tw[kG2 + 4 * (L25::e2(ot) + v)] = dz2[ot][v];
      wave_lds_sync();
      {
        double f[2][2][4], x[2][9];
        auto ldb = [&](int k, double (*q)[4]) {
          ld_bwd(W2, o2s, n2, 4, 0, k, 4, q[0]);
          ld_bwd(W2, o2s, n2, 4, 4, k, n1 - 4, q[1]);
        };
        auto ldw = [&](int ks, double* q) {
          q[0] = Tm[4 * ks * kTS];
#pragma unroll
          for (int e = 0; e < 3; ++e) q[1 + e] = Ts[4 * ks * kTS + 16 + 4 * e];
#pragma unroll
          for (int j = 0; j < 3; ++j) q[4 + j] = Tm[4 * ks * kTS + kG2 + 16 * j];
          q[7] = Ts[4 * ks * kTS + kG2 + 48];
          q[8] = Tm[4 * ks * kTS + 16];  // columns past 27 are dz2: not read out
        };
        ldb(0, f[0]);
#pragma unroll
        for (int o = 0; o < 4; ++o)
#pragma unroll
          for (int v = 0; v < nv2<W>(o); ++v) {
            const int seq = (o > 0) * 4 + (o > 1) * 3 + (o > 2) * 4 + v;
            const int nx = seq + 1, no = nx < 4 ? 0 : nx < 7 ? 1 : nx < 11 ? 2 : 3;
            const int nv_ = nx - (no > 0) * 4 - (no > 1) * 3 - (no > 2) * 4;
            if (nx < n2) ldb(L25::e2(no) + nv_, f[nx & 1]);
            else ldw(0, x[0]);
            DPSE_FENCE;
            z1[0] = mma(4, f[seq & 1][0], dz2[o][v], z1[0]);
            z1[1] = mma(n1 - 4, f[seq & 1][1], dz2[o][v], z1[1]);
          }
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          if (ks < 3) ldw(ks + 1, x[(ks + 1) & 1]);
          DPSE_FENCE;
          const double* q = x[ks & 1];
#pragma unroll
          for (int j = 0; j < 3; ++j) {
            a2[j] = mfma_f64(q[0], q[4 + j], a2[j]);
#pragma unroll
            for (int e = 0; e < 3; ++e) a2s[j][e] = mfma4_f64(q[1 + e], q[4 + j], a2s[j][e]);
          }
          a2r[0] = mfma4_f64(q[7], q[0], a2r[0]);
          a2r[1] = mfma4_f64(q[7], q[8], a2r[1]);
        }
      }
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int v = 0; v < nv1<W>(mt); ++v) {
          const double dz1 = z1[mt][v] * (1.0 - t1[mt][v] * t1[mt][v]);
          ab1[4 * mt + v] += dz1;
          aw1[4 * mt + v] = fma(s, dz1, aw1[4 * mt + v]);
        }
    }
  }
#undef DPSE_FENCE
  // dW1, db1: sum over the 16 rows held by a lane group
#pragma unroll
  for (int e = 0; e < n1; ++e)
#pragma unroll
    for (int m = 1; m < 16; m <<= 1) {
      ab1[e] += shfl_xor_d(ab1[e], m);
      aw1[e] += shfl_xor_d(aw1[e], m);
    }
  // the waves' sums in wave order, through LDS (tb and the weights are free)
  __syncthreads();
  constexpr int kBuf = GW * 16 * kTS;  // tb
  static_assert(kGrRec <= kBuf, "the record fits the transposition buffers");
  double* const buf = &tb[0][0];
  for (int w = 0; w < GW; ++w) {
    if (w == wv) {
      auto put = [&](int at, double x) { buf[at] = w ? buf[at] + x : x; };
#pragma unroll
      for (int j = 0; j < 6; ++j) {
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
          for (int v = 0; v < 4; ++v) put((16 * p + 4 * v + g) * kG3N + 16 * j + r16, a3[j][p][v]);
        put((48 + g) * kG3N + 16 * j + r16, a3s[j]);
      }
#pragma unroll
      for (int p = 0; p < 4; ++p)
        if (p < 3 || r16 < 4) put((16 * p + r16) * kG3N + 96 + g, a3r[p]);
#pragma unroll
      for (int j = 0; j < 3; ++j) {
#pragma unroll
        for (int v = 0; v < 4; ++v) put(kGr2 + (4 * v + g) * kG3 + 16 * j + r16, a2[j][v]);
#pragma unroll
        for (int e = 0; e < 3; ++e) put(kGr2 + (16 + 4 * e + g) * kG3 + 16 * j + r16, a2s[j][e]);
      }
      put(kGr2 + r16 * kG3 + 48 + g, a2r[0]);
      if (r16 < 12) put(kGr2 + (16 + r16) * kG3 + 48 + g, a2r[1]);
      if (r16 == 0) {
#pragma unroll
        for (int e = 0; e < n1; ++e) {
          put(kGr1 + 4 * e + g, ab1[e]);
          put(kGr1 + kG2 + 4 * e + g, aw1[e]);
        }
      }
    }
    __syncthreads();
  }
  for (int e = threadIdx.x; e < kGrRec; e += 256) pr[e] = buf[e];
}

// Sums a net's records in work-group order (four interleaved quarters, added
// in a fixed order) for 64 parameters per work-group.  A unit that the denser
// layout holds twice has its gradient in both slots.
__global__ __launch_bounds__(256) void k_egrad25_reduce(EGradArgs A, int G) {
  constexpr int W = 25;
  __shared__ double red[4][64];
  const int net = blockIdx.y, k = blockIdx.x * 64 + (threadIdx.x & 63), q4 = threadIdx.x >> 6;
  const NetShares* S = net_shares(A.meta);
  int lo = 0, hi = 0;
  for (int r = 0; r < A.ntypes * A.ntypes; ++r)
    if (S->net[0][r] == net) {
      lo = share_start(S, 0, A.ntypes * A.ntypes, G, r);
      hi = share_start(S, 0, A.ntypes * A.ntypes, G, r + 1);
    }
  constexpr int nW3 = 50 * 100, nW2 = 25 * 50, total = nW3 + 100 + nW2 + 50 + 2 * W;
  auto c2 = [](int f) { return L25::col2(slot2d_of_feat<W>(f)); };
  int64_t dst = -1;
  int src[4] = {0, 0, 0, 0}, ns = 1;
  if (k < nW3 + 100) {  // dW3 rows, then db3 (the row of slot 26)
    const int f2 = k / 100, f3 = k - 100 * f2;
    const int z = f3 >= 50, f = f3 - 50 * z;
    // slot of layer-3 feature f3: the last features of each quarter share slots 24..27 of the first half
    const int slot = f == 24 ? 24 + 2 * z : f == 49 ? 25 + 2 * z : 64 * z + slot2d_of_feat<W>(f);
    src[0] = (k < nW3 ? c2(f2) : L25::col2(26)) * kG3N + L25::col3(slot);
    dst = k < nW3 ? A.offW[net][2] + f2 * 100 + f3 : A.offB[net][2] + f3;
  } else if (k < nW3 + 100 + nW2 + 50) {  // dW2 rows, then db2 (the row of slot 25)
    const int kk = k - nW3 - 100, f1 = kk / 50, f2 = kk - 50 * f1;
    const int row = kGr2 + (kk < nW2 ? f1 : 25) * kG3;
    src[0] = row + c2(f2);
    if (f2 == W - 1 || f2 == 2 * W - 1) {
      src[1] = row + L25::col2(f2 == W - 1 ? 26 : 27);
      ns = 2;
    }
    dst = kk < nW2 ? A.offW[net][1] + f1 * 50 + f2 : A.offB[net][1] + f2;
  } else if (k < total) {
    const int kk = k - nW3 - 100 - nW2 - 50, f = kk % W;
    ns = f == W - 1 ? 4 : 1;
    for (int e = 0; e < 4; ++e) src[e] = kGr1 + (kk < W ? 0 : kG2) + f + (f == W - 1 ? e : 0);
    dst = kk < W ? A.offB[net][0] + f : A.offW[net][0] + f;
  }
  double acc = 0.0;
  if (dst >= 0)
    for (int r = lo + q4; r < hi; r += 4) {
      const double* p = A.part + (int64_t)r * kGrRec;
      double x = p[src[0]];
      for (int e = 1; e < ns; ++e) x += p[src[e]];
      acc += x;
    }
  red[q4][threadIdx.x & 63] = acc;
  __syncthreads();
  if (q4 == 0 && dst >= 0) {
    const int l = threadIdx.x;
    A.grad[dst] = (red[0][l] + red[1][l]) + (red[2][l] + red[3][l]);
  }
}

// ------------------------------------------------------------ launcher
void launch_param_grads(dp_ctx* c, const ParamGradInputs& in, const double* dLdE, double* grad, bool fill_act,
                        hipStream_t s) {
  const dp_model* m = c->model;
  const int n = (int)c->natoms_last;
  const int nt = m->desc.ntypes;
  const int ncols = (int)(c->natoms_last + nt * kColPad);
  if (n <= 0) {
    launch_fill_f64(grad, 0.0, m->n_params, s);
    return;
  }
  // (every parameter is written below: types and nets without atoms get their
  // empty sums)
  hipLaunchKernelGGL(k_col_weights, dim3((ncols + 255) / 256), dim3(256), 0, s, c->atom_at, c->frame_of, dLdE,
                     c->gE_col, ncols);
  // ---- fitting: per layer dW = X^T diag(w) dz, db = sum w dz; w_out, b_out, e_bias
  // Partial sums go to the workspace, which the next kernel sums in chunk
  // order; launches on one stream reuse it in turn.
  const int fw = m->fw, nd = m->nd;
  const int Kin[3] = {nd, fw, fw};
  WGradArgs a = {};
  WSumArgs q = {};
  int groups = 0;
  int64_t rec = 0;
  for (int l = 0; l < 3; ++l) {
    a.l[l] = WGradLayer{in.X[l], in.dz[l], in.ldx[l], in.ldz, Kin[l], groups, rec};
    q.off[l] = rec;
    q.wlen[l] = (int64_t)Kin[l] * fw;
    q.wdst[l] = m->fit_param_off[l];
    q.bdst[l] = m->fit_param_off[3 + l];
    groups += (Kin[l] / 16 + kWgMT - 1) / kWgMT;
    rec += (int64_t)(Kin[l] + 1) * fw;
  }
  // one round of two work-groups per CU, chunks of 64 columns at least
  int nch = (int)((2LL * c->ncu) / groups);
  const int most = (n + 63) / 64;
  if (nch > most) nch = most;
  if (nch > c->grad_chunks) nch = c->grad_chunks;
  if (nch < nt) nch = nt;
  a.w = c->gE_col;
  a.meta = q.meta = c->type_meta;
  a.N = fw;
  a.ntypes = q.ntypes = nt;
  a.nchunks = q.nchunks = nch;
  a.rec = q.rec = rec;
  a.part = c->gpart;
  q.part = c->gpart;
  q.type_stride = m->fit_param_stride;
  q.grad = grad;
  const dim3 wgrid(nch, groups), wblock(256);
  switch (in.kind[0] * 100 + in.kind[1] * 10 + in.kind[2]) {  // X1 and dz1 | X2, X3, h3 | dz2, dz3
    case 0: hipLaunchKernelGGL((k_wgrad_cols<0, 0, 0, 0>), wgrid, wblock, 0, s, a); break;
    case 111: hipLaunchKernelGGL((k_wgrad_cols<1, 1, 1, 1>), wgrid, wblock, 0, s, a); break;
    case 212: hipLaunchKernelGGL((k_wgrad_cols<2, 2, 1, 2>), wgrid, wblock, 0, s, a); break;
    case 313: hipLaunchKernelGGL((k_wgrad_cols<3, 3, 1, 3>), wgrid, wblock, 0, s, a); break;
    default: hipLaunchKernelGGL((k_wgrad_cols<3, 3, 1, 1>), wgrid, wblock, 0, s, a); break;  // 311
  }
  hipLaunchKernelGGL(k_wgrad_sum, dim3((unsigned)((rec + 255) / 256), nt), dim3(256), 0, s, q);
  const int ochunks = (n + kWoChunk - 1) / kWoChunk;
  const dim3 ogrid(ochunks, nt), oblock(320);
  if (in.kind[1] == 0)
    hipLaunchKernelGGL(k_wout_cols<0>, ogrid, oblock, 0, s, in.h3, in.ldx[2], c->gE_col, c->type_meta, fw, ochunks, c->gpart);
  else
    hipLaunchKernelGGL(k_wout_cols<1>, ogrid, oblock, 0, s, in.h3, in.ldx[2], c->gE_col, c->type_meta, fw, ochunks, c->gpart);
  hipLaunchKernelGGL(k_wout_sum, dim3((fw + 16) / 16, nt), dim3(256), 0, s, c->gpart, c->type_meta, fw, ochunks, grad,
                     m->fit_param_stride, m->fit_param_off[6], m->fit_param_off[7], m->ebias_off);
  // ---- embedding nets
  EGradArgs A = {};
  A.atom_at = c->atom_at;
  A.meta = c->type_meta;
  A.R = c->R;
  A.nnei = c->nnei;
  A.frag64 = m->emb_frag64;
  A.vec64 = m->emb_vec64;
  A.vec_per_net = m->emb_vec_per_net;
  A.fo = m->efo;
  A.gT = in.gT;
  A.gt32 = in.gt32;
  A.wcol = c->gE_col;
  A.grad = grad;
  A.part = c->gpart;
  A.nslots = c->grad_slots;
  for (int k = 0; k < nt * nt; ++k)
    for (int l = 0; l < 3; ++l) {
      A.offW[k][l] = m->emb_param_off[k][2 * l];
      A.offB[k][l] = m->emb_param_off[k][2 * l + 1];
    }
  A.ntypes = nt;
  A.nm = m->nm;
  // one work-group per CU and net (at most nslots records per net)
  int ng = c->ncu < A.nslots ? c->ncu : A.nslots;
  if ((int64_t)ng * kEgWaves > n) ng = (n + kEgWaves - 1) / kEgWaves;
  A.ngroups = ng < 1 ? 1 : ng;
  A.ctr = c->emb_ctr;
  for (int t = 0; t <= kMaxT; ++t) A.sec[t] = t <= nt ? m->sec[t] : m->nm;
  A.inv_nm = 1.0 / (double)m->nm;
  dim3 grid(A.ngroups, nt * nt);
  dim3 rgrid((kEgRec + 255) / 256, nt * nt);
  // the forward's stored last-layer activations (FP64 computes that fit the
  // workspace) replace the recomputation of the last embedding layer
  A.act = c->act_used_last || c->grad_act ? (const double*)c->act : nullptr;
  A.tpa = m->tpa;
  for (int t = 0; t <= kMaxT; ++t) A.toff[t] = t <= nt ? m->toff[t] : m->tpa;
  if (m->w1 == 25) {
    A.frag64 = m->emb_frag64d;
    A.vec64 = m->emb_vec64d;
    A.fo = m->efd;
    A.tanh_lut = m->tanh_lut;
    const int64_t need = ((int64_t)n * nt + 3) / 4;
    int G = (int)(need < c->ncu ? need : c->ncu);
    if (G > c->grad_slots) G = c->grad_slots;
    if (G < nt * nt) G = nt * nt;
    if (fill_act) {
      A.act = (const double*)c->act;
      hipLaunchKernelGGL(k_embed_grad25<2>, dim3(G), dim3(256), 0, s, A);
    } else if (A.act) {
      hipLaunchKernelGGL(k_embed_grad25<1>, dim3(G), dim3(256), 0, s, A);
    } else {
      hipLaunchKernelGGL(k_embed_grad25<0>, dim3(G), dim3(256), 0, s, A);
    }
    constexpr int total = 50 * 100 + 100 + 25 * 50 + 50 + 50;
    hipLaunchKernelGGL(k_egrad25_reduce, dim3((total + 63) / 64, nt * nt), dim3(256), 0, s, A, G);
  } else {
    if (A.act) hipLaunchKernelGGL((k_embed_grad_f64<32, true>), grid, dim3(64 * kEgWaves), 0, s, A);
    else hipLaunchKernelGGL((k_embed_grad_f64<32, false>), grid, dim3(64 * kEgWaves), 0, s, A);
    hipLaunchKernelGGL(k_egrad_reduce<32>, rgrid, dim3(256), 0, s, A);
  }
}

}  // namespace dpse

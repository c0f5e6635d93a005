// DP-compress: the embedding nets as tables of piecewise quintics (the
// compression of the embedding net that the Background section cites), built
// on the device from the model's parameters and evaluated, fused with the
// G^T R contraction, in the FP64 force path.
//
// Grid (shared with the documentation of dp_model_compress): a fine stride
// h on [0, X1) with n1 intervals (X1 = n1 h) and a coarse stride H = 10 h on
// [X1, X2) with n2 intervals.  Node n is at n h for n <= n1 and at
// X1 + (n - n1) H beyond.  On interval k the quintic in t = x - x_k matches
// G, dG/dx and d2G/dx2 at both ends.  Table layout [net][k][p][a]: for a
// power p the m1 features are contiguous, so 16 lanes that evaluate 16
// consecutive features of one row read 128 contiguous bytes.
//
// Inputs x >= X2 take G(X2) with zero slope and raise DP_FLAG_TABLE_RANGE.
#include "dp_internal.h"
#include "dp_device.h"

namespace dpse {

// ------------------------------------------------------------ table build
// Node values: one work-group per (net, node), one thread per feature.
// Forward-mode derivatives through the layers: z = h W + b, z' = h' W,
// z'' = h'' W, tau = tanh z, tau' = (1 - tau^2) z',
// tau'' = (1 - tau^2)(z'' - 2 tau z'^2); the identity skips carry h, h', h''.
__global__ __launch_bounds__(128) void k_tab_nodes(const double* __restrict__ P, TabGrid g, int ntypes, int w1,
                                                   TabNetOffsets off, double* __restrict__ nodes) {
  const int net = blockIdx.y, node = blockIdx.x;
  const int m1 = 4 * w1;
  __shared__ double hv[3][128];  // value, slope, curvature of the layer's outputs
  const double x = node <= g.n1 ? (double)node * g.h : fma((double)(node - g.n1), g.H, g.X1);
  const int q = threadIdx.x;
  const double* W[3] = {P + off.W[net][0], P + off.W[net][1], P + off.W[net][2]};
  const double* B[3] = {P + off.b[net][0], P + off.b[net][1], P + off.b[net][2]};
  // layer 1: input x with x' = 1, x'' = 0 (width w1, no skip)
  double v = 0.0, v1 = 0.0, v2 = 0.0;
  if (q < w1) {
    const double z = fma(x, W[0][q], B[0][q]), z1 = W[0][q];
    const double tt = tanh_d(z), gg = 1.0 - tt * tt;
    v = tt;
    v1 = gg * z1;
    v2 = gg * (-2.0 * tt * z1 * z1);
  }
  int wp = w1;
  for (int l = 1; l < 3; ++l) {
    __syncthreads();
    if (q < wp) {
      hv[0][q] = v;
      hv[1][q] = v1;
      hv[2][q] = v2;
    }
    __syncthreads();
    const int w = 2 * wp;
    if (q < w) {
      double z = B[l][q], z1 = 0.0, z2 = 0.0;
      for (int p = 0; p < wp; ++p) {
        const double wt = W[l][(int64_t)p * w + q];
        z = fma(hv[0][p], wt, z);
        z1 = fma(hv[1][p], wt, z1);
        z2 = fma(hv[2][p], wt, z2);
      }
      const double tt = tanh_d(z), gg = 1.0 - tt * tt;
      const int s = q % wp;  // [h, h] skip of a doubled width
      v = hv[0][s] + tt;
      v1 = hv[1][s] + gg * z1;
      v2 = hv[2][s] + gg * (z2 - 2.0 * tt * z1 * z1);
    }
    wp = w;
  }
  if (q < m1) {
    double* o = nodes + ((int64_t)net * (g.nint + 1) + node) * 3 * m1;
    o[q] = v;
    o[m1 + q] = v1;
    o[2 * m1 + q] = v2;
  }
}

// Coefficients: one thread per (net, interval, feature).  With
// A = y1 - y0 - d0 L - s0 L^2/2, B = d1 - d0 - s0 L, C = s1 - s0:
// c0 = y0, c1 = d0, c2 = s0/2, c3 = (20A - 8BL + CL^2)/(2L^3),
// c4 = (-30A + 14BL - 2CL^2)/(2L^4), c5 = (12A - 6BL + CL^2)/(2L^5).
__global__ void k_tab_coef(const double* __restrict__ nodes, TabGrid g, int m1, int nnets, double* __restrict__ table) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = (int64_t)nnets * g.nint * m1;
  if (id >= total) return;
  const int a = (int)(id % m1);
  const int64_t nk = id / m1;
  const int k = (int)(nk % g.nint), net = (int)(nk / g.nint);
  const double L = k < g.n1 ? g.h : g.H;
  const double* n0 = nodes + ((int64_t)net * (g.nint + 1) + k) * 3 * m1;
  const double* n1 = n0 + 3 * m1;
  const double y0 = n0[a], d0 = n0[m1 + a], s0 = n0[2 * m1 + a];
  const double y1 = n1[a], d1 = n1[m1 + a], s1 = n1[2 * m1 + a];
  const double A = y1 - y0 - d0 * L - 0.5 * s0 * L * L;
  const double B = d1 - d0 - s0 * L;
  const double C = s1 - s0;
  const double L2 = L * L, L3 = L2 * L;
  double* c = table + ((int64_t)net * g.nint + k) * 6 * m1 + a;
  c[0] = y0;
  c[m1] = d0;
  c[2 * m1] = 0.5 * s0;
  c[3 * m1] = (20.0 * A - 8.0 * B * L + C * L2) / (2.0 * L3);
  c[4 * m1] = (-30.0 * A + 14.0 * B * L - 2.0 * C * L2) / (2.0 * L3 * L);
  c[5 * m1] = (12.0 * A - 6.0 * B * L + C * L2) / (2.0 * L3 * L2);
}

void launch_tab_build(const dp_model* m, hipStream_t s) {
  const TabGrid& g = m->tab_grid;
  const int nnets = m->desc.ntypes * m->desc.ntypes;
  hipLaunchKernelGGL(k_tab_nodes, dim3((unsigned)(g.nint + 1), (unsigned)nnets), dim3(128), 0, s,
                     (const double*)m->params, g, m->desc.ntypes, m->w1, m->tab_off, m->tab_nodes);
  const int64_t total = (int64_t)nnets * g.nint * m->m1;
  hipLaunchKernelGGL(k_tab_coef, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, (const double*)m->tab_nodes,
                     g, m->m1, nnets, m->table);
}

// ------------------------------------------------------------ evaluation
// Interval and offset of input x (the same operations as the checking
// implementation: IEEE division and floor pick the interval, one fused
// multiply-add gives t).
__device__ __forceinline__ int tab_interval(const TabGrid& g, double x, double& t, bool& clip) {
  clip = false;
  if (x < g.X1) {
    int k = (int)floor(x / g.h);
    k = k >= g.n1 ? g.n1 - 1 : (k < 0 ? 0 : k);
    t = fma(-(double)k, g.h, x);
    return k;
  }
  if (x < g.X2) {
    int m = (int)floor((x - g.X1) / g.H);
    m = m >= g.n2 ? g.n2 - 1 : m;
    t = fma(-(double)m, g.H, x - g.X1);
    return g.n1 + m;
  }
  clip = true;
  t = g.n2 > 0 ? g.H : g.h;
  return g.nint - 1;
}

struct TabArgs {
  const int32_t* atom_at;
  const int32_t* meta;
  const double* R;
  const int32_t* nnei;
  const double* table;
  TabGrid g;
  double* Tpart;          // forward: [ntypes][cols][m1][4]
  int64_t tpart_stride;
  const double* gT;       // backward: [cols][m1][4]
  double* netd;
  int ntypes, nm;
  int sec[kMaxT + 1];
  double inv_nm;
  int32_t* ctr;
  int32_t* flags;
};

// Work layout: one wavefront per centre atom and neighbour section (columns
// of the net taken from a per-work-group counter as in the MLP kernels).
//
// Window.  48 bytes of coefficients per row and feature (5 GB at water12k)
// made the table's trip from L2 the bound of both kernels.  Most rows lie at
// small x (s(r) falls to 0 at the cut-off: 9 of 10 water rows at x < 3, 30 of
// the 1,475 intervals), so a work-group of WPB = 16 waves, one per CU, keeps
// the first nk intervals of its net in LDS, [interval][feature][power] with
// the interval stride an odd number of 16-byte units: lanes that read
// neighbouring intervals, or neighbouring features, fall in different banks.
// Rows past the window read L2.  Frames of few columns take 4-wave
// work-groups and no window (launch_embed_tab).  water12k: forward 395 ->
// 86 us, backward 418 -> 176 us; copper of 23,328 atoms 2,175 -> 346 and
// 1,746 -> 596 us.  The backward is now bound by LDS reads (4.8 KB per window
// row of 64 lanes at 128 bytes per cycle: ~100 us), the forward by issue.  The
// window holds intervals, so a finer table has fewer rows in it; the whole
// compute with it and with every row from L2 as before, 12,288 water atoms:
// h = 0.1 835 / 1,440 us, 0.02 973 / 1,443, 0.01 1,051 / 1,451, 0.005 1,138 /
// 1,465; 4,000 copper atoms: 459 / 1,094, 554 / 1,225, 593 / 1,282, 660 / 1,336.
template <int M1>
struct TabWin {
  static constexpr int stride = 6 * M1 + 2;                   // doubles per interval
  static constexpr int most = (148 * 1024) / (8 * stride);    // intervals that fit: 31 (m1 = 100), 24 (128)
};

typedef double d2 __attribute__((ext_vector_type(2)));

// Copies the window's nk intervals of a net's table [k][p][a] to LDS
// [k][a][p]: two features per thread and read, every read requested before
// the first is used.
template <int M1, int NT>
__device__ __forceinline__ void tab_stage(const double* __restrict__ tabnet, int nk, double* __restrict__ tw) {
  constexpr int NL = (TabWin<M1>::most * 3 * M1 + NT - 1) / NT;
  const int total = nk * 3 * M1;
  d2 x[NL];
#pragma unroll
  for (int l = 0; l < NL; ++l) x[l] = *reinterpret_cast<const d2*>(tabnet + 2 * min((int)threadIdx.x + l * NT, total - 1));
#pragma unroll
  for (int l = 0; l < NL; ++l) {
    const int e = threadIdx.x + l * NT;
    if (e >= total) break;
    const int k = e / (3 * M1), pa = e - k * 3 * M1, p = pa / (M1 / 2), a = 2 * (pa - p * (M1 / 2));
    double* w = tw + k * TabWin<M1>::stride + a * 6 + p;
    w[0] = x[l][0];
    w[6] = x[l][1];
  }
}

#define DPSE_TAB_PROLOGUE                                                  \
  int grp = 0, ngrp = 1;                                                  \
  const int net = net_of_group(A.meta, A.ntypes, gridDim.x, blockIdx.x, &grp, &ngrp, 0); \
  if (net < 0) return;                                                    \
  const int ti = net / A.ntypes, tj = net - ti * A.ntypes;                \
  const int n_t = A.meta[2 * ti], cb = A.meta[2 * ti + 1];                \
  const int c_lo = part_start(n_t, grp, ngrp);                            \
  const int c_hi = part_start(n_t, grp + 1, ngrp);                        \
  if (c_lo >= c_hi) return;                                               \
  const int lane = threadIdx.x & 63;                                      \
  int* const next_col = A.ctr + blockIdx.x * 32;                          \
  if (threadIdx.x == 0) atomicExch(next_col, c_lo);                       \
  const double* tabnet = A.table + (int64_t)net * A.g.nint * 6 * M1;      \
  constexpr bool WIN = WPB == 16;                                         \
  constexpr int TS = TabWin<M1>::stride;                                  \
  __shared__ __attribute__((aligned(16))) double tw[WIN ? TabWin<M1>::most * TS : 2]; \
  const int nk = WIN ? min(TabWin<M1>::most, A.g.nint) : 0;               \
  if constexpr (WIN) tab_stage<M1, 64 * WPB>(tabnet, nk, tw);             \
  __syncthreads();                                                        \
  auto take = [&]() {                                                     \
    int k = 0;                                                            \
    if (lane == 0) k = atomicAdd(next_col, 1);                            \
    return k;                                                             \
  };

// Reads through the constant address space: a wave-uniform address then
// becomes one scalar load for the wave (the buffers read so are written by
// earlier kernels only).
typedef const __attribute__((address_space(4))) double* cdouble_p;
__device__ __forceinline__ cdouble_p uniform_ptr(const double* p) {
  const unsigned long long a = reinterpret_cast<unsigned long long>(p);
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
  return (cdouble_p)(((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ double readlane_d(double x, int l) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
  const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)b, l);
  const unsigned hi = __builtin_amdgcn_readlane((int)(unsigned)(b >> 32), l);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// Forward: lanes are features (two per lane: l and l + M1/2), rows are taken
// one after another with their input wave-uniform.  A section is sorted by
// distance, so rows of one interval follow each other and its coefficients
// stay in registers from row to row; no sum crosses lanes.  Correct for any
// order of the rows.
template <int M1, int WPB>
__global__ __launch_bounds__(64 * WPB) void k_embed_fwd_tab(TabArgs A) {
  constexpr int MH = M1 / 2;  // features l and l + MH of lane l < MH
  static_assert(MH <= 64 && M1 % 2 == 0, "two features per lane");
  DPSE_TAB_PROLOGUE
  const int fl = lane < MH ? lane : MH - 1;  // the lanes past MH repeat the last and store nothing
  bool clipped = false;
  for (int c_next = take();;) {
    const int c = __builtin_amdgcn_readfirstlane(c_next);
    if (c >= c_hi) break;
    c_next = take();
    const int col = cb + c;
    const int i = __builtin_amdgcn_readfirstlane(A.atom_at[col]);
    const int nn = __builtin_amdgcn_readfirstlane(A.nnei[i * kMaxT + tj]);
    const double* Rs = A.R + ((int64_t)i * A.nm + A.sec[tj]) * 4;
    const cdouble_p Ru = uniform_ptr(Rs);
    double acc[2][4];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[u][q] = 0.0;
    double cf[2][6];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int p = 0; p < 6; ++p) cf[u][p] = 0.0;
    int kcur = -1;
    for (int r0 = 0; r0 < nn; r0 += 64) {
      // interval and offset of 64 rows, one per lane
      const int row = r0 + lane;
      double t;
      bool cl;
      const int kl = tab_interval(A.g, row < nn ? Rs[(int64_t)row * 4] : 0.0, t, cl);
      clipped |= cl && row < nn;
      const int nr = min(64, nn - r0);
      for (int r = 0; r < nr; ++r) {
        const int k = __builtin_amdgcn_readlane(kl, r);
        const double tr = readlane_d(t, r);
        const double R0 = Ru[(r0 + r) * 4], R1 = Ru[(r0 + r) * 4 + 1], R2 = Ru[(r0 + r) * 4 + 2],
                     R3 = Ru[(r0 + r) * 4 + 3];
        if (k != kcur) {
          kcur = k;
          if (k < nk) {
            const double* cw = tw + k * TS + fl * 6;
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
              for (int p = 0; p < 6; p += 2) {
                const d2 x = *reinterpret_cast<const d2*>(cw + u * MH * 6 + p);
                cf[u][p] = x[0];
                cf[u][p + 1] = x[1];
              }
          } else {
            const double* cg = tabnet + (int64_t)k * 6 * M1 + fl;
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
              for (int p = 0; p < 6; ++p) cf[u][p] = cg[p * M1 + u * MH];
          }
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          double G = cf[u][5];
#pragma unroll
          for (int p = 4; p >= 0; --p) G = fma(G, tr, cf[u][p]);
          acc[u][0] = fma(G, R0, acc[u][0]);
          acc[u][1] = fma(G, R1, acc[u][1]);
          acc[u][2] = fma(G, R2, acc[u][2]);
          acc[u][3] = fma(G, R3, acc[u][3]);
        }
      }
    }
    double* T = A.Tpart + tj * A.tpart_stride + (int64_t)col * M1 * 4;
    if (lane < MH) {
#pragma unroll
      for (int u = 0; u < 2; ++u)
        *reinterpret_cast<d4*>(T + (lane + u * MH) * 4) =
            d4{acc[u][0] * A.inv_nm, acc[u][1] * A.inv_nm, acc[u][2] * A.inv_nm, acc[u][3] * A.inv_nm};
    }
  }
  if (__ballot(clipped) && lane == 0) set_flag(A.flags, DP_FLAG_TABLE_RANGE);
}

// Backward: per row, dE/dG_a = g_T[a] . R~ / nm, the direct term
// dE/dR~ = sum_a g_T[a] G_a / nm and dE/dx = sum_a dE/dG_a dG_a/dx.
// Rows of the window: lanes are rows, the features are taken one after
// another with g_T wave-uniform, so no sum crosses lanes (three 16-byte LDS
// reads and 18 multiply-adds per row and feature).  The others (and every row
// without a window), one at a time: lanes are features as in the forward,
// coefficients from L2 kept while the interval stays, four sums over the wave.
template <int M1, int WPB>
__global__ __launch_bounds__(64 * WPB) void k_embed_bwd_tab(TabArgs A) {
  constexpr int MH = M1 / 2;
  DPSE_TAB_PROLOGUE
  const int fl = lane < MH ? lane : MH - 1;
  for (int c_next = take();;) {
    const int c = __builtin_amdgcn_readfirstlane(c_next);
    if (c >= c_hi) break;
    c_next = take();
    const int col = cb + c;
    const int i = __builtin_amdgcn_readfirstlane(A.atom_at[col]);
    const int nn = __builtin_amdgcn_readfirstlane(A.nnei[i * kMaxT + tj]);
    const int64_t rbase = (int64_t)i * A.nm + A.sec[tj];
    const env_rsrc_t Rb = env_rsrc(A.R + rbase * 4, nn);
    const double* gcol = A.gT + (int64_t)col * M1 * 4;
    const cdouble_p gu = uniform_ptr(gcol);
    const cdouble_p Ru = uniform_ptr(A.R + rbase * 4);
    // g_T of the lane's two features, zero in the lanes past MH
    d4 gt[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      gt[u] = *reinterpret_cast<const d4*>(gcol + (fl + u * MH) * 4);
      if (lane >= MH) gt[u] = d4{0.0, 0.0, 0.0, 0.0};
    }
    for (int r0 = 0; r0 < nn; r0 += 64) {
      const int row = r0 + lane;
      const d4 Rv = env_row(Rb, row);  // zero past the section's real rows
      double t;
      bool cl;
      const int k = tab_interval(A.g, Rv[0], t, cl);
      const bool win = k < nk;
      if constexpr (WIN) {
        const double* cw = tw + (win ? k : 0) * TS;
        double ds = 0.0, dr[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
        for (int a = 0; a < M1; ++a) {
          const double g0 = gu[4 * a], g1 = gu[4 * a + 1], g2 = gu[4 * a + 2], g3 = gu[4 * a + 3];
          const d2 c01 = *reinterpret_cast<const d2*>(cw + a * 6);
          const d2 c23 = *reinterpret_cast<const d2*>(cw + a * 6 + 2);
          const d2 c45 = *reinterpret_cast<const d2*>(cw + a * 6 + 4);
          // value and slope by Horner's rule in one sweep
          double G = fma(c45[1], t, c45[0]);
          double Gp = fma(c45[1], t, G);
          G = fma(G, t, c23[1]);
          Gp = fma(Gp, t, G);
          G = fma(G, t, c23[0]);
          Gp = fma(Gp, t, G);
          G = fma(G, t, c01[1]);
          Gp = fma(Gp, t, G);
          G = fma(G, t, c01[0]);
          const double dG = fma(g0, Rv[0], fma(g1, Rv[1], fma(g2, Rv[2], g3 * Rv[3])));
          ds = fma(dG, Gp, ds);
          dr[0] = fma(g0, G, dr[0]);
          dr[1] = fma(g1, G, dr[1]);
          dr[2] = fma(g2, G, dr[2]);
          dr[3] = fma(g3, G, dr[3]);
        }
        if (cl) ds = 0.0;
        if (win && row < nn)
          *reinterpret_cast<d4*>(A.netd + (rbase + row) * 4) =
              d4{(dr[0] + ds) * A.inv_nm, dr[1] * A.inv_nm, dr[2] * A.inv_nm, dr[3] * A.inv_nm};
      }
      int kcur = -1;
      double cf[2][6];
      const unsigned long long clips = __ballot(cl);
      for (unsigned long long todo = __ballot(!win && row < nn); todo; todo &= todo - 1) {
        const int r = __builtin_ctzll(todo);
        const int kr = __builtin_amdgcn_readlane(k, r);
        const double tr = readlane_d(t, r);
        const double R0 = Ru[(r0 + r) * 4], R1 = Ru[(r0 + r) * 4 + 1], R2 = Ru[(r0 + r) * 4 + 2],
                     R3 = Ru[(r0 + r) * 4 + 3];
        if (kr != kcur) {
          kcur = kr;
          const double* cg = tabnet + (int64_t)kr * 6 * M1 + fl;
#pragma unroll
          for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int p = 0; p < 6; ++p) cf[u][p] = cg[p * M1 + u * MH];
        }
        double dr[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          double G = fma(cf[u][5], tr, cf[u][4]);
          double Gp = fma(cf[u][5], tr, G);
          G = fma(G, tr, cf[u][3]);
          Gp = fma(Gp, tr, G);
          G = fma(G, tr, cf[u][2]);
          Gp = fma(Gp, tr, G);
          G = fma(G, tr, cf[u][1]);
          Gp = fma(Gp, tr, G);
          G = fma(G, tr, cf[u][0]);
          if ((clips >> r) & 1) Gp = 0.0;
          const double dG = fma(gt[u][0], R0, fma(gt[u][1], R1, fma(gt[u][2], R2, gt[u][3] * R3)));
          dr[0] = fma(gt[u][0], G, fma(dG, Gp, dr[0]));
          dr[1] = fma(gt[u][1], G, dr[1]);
          dr[2] = fma(gt[u][2], G, dr[2]);
          dr[3] = fma(gt[u][3], G, dr[3]);
        }
        const double v = wave_sum4(dr[0], dr[1], dr[2], dr[3]);
        if ((lane & 15) == 0) A.netd[(rbase + r0 + r) * 4 + (lane >> 4)] = v * A.inv_nm;
      }
    }
  }
}

template <int M1>
static void launch_tab(bool bwd, int wpb, dim3 grid, const TabArgs& A, hipStream_t s) {
  if (wpb == 16) {
    if (bwd) hipLaunchKernelGGL((k_embed_bwd_tab<M1, 16>), grid, dim3(1024), 0, s, A);
    else hipLaunchKernelGGL((k_embed_fwd_tab<M1, 16>), grid, dim3(1024), 0, s, A);
  } else {
    if (bwd) hipLaunchKernelGGL((k_embed_bwd_tab<M1, 4>), grid, dim3(256), 0, s, A);
    else hipLaunchKernelGGL((k_embed_fwd_tab<M1, 4>), grid, dim3(256), 0, s, A);
  }
}

void launch_embed_tab(dp_ctx* c, bool bwd, hipStream_t s) {
  const dp_model* m = c->model;
  if (c->natoms_last <= 0) return;
  TabArgs A;
  A.atom_at = c->atom_at;
  A.meta = c->type_meta;
  A.R = c->R;
  A.nnei = c->nnei;
  A.table = m->table;
  A.g = m->tab_grid;
  A.Tpart = (double*)c->Tpart;
  A.tpart_stride = c->max_cols * m->m1 * 4;
  A.gT = (const double*)c->gT;
  A.netd = c->netd;
  A.ntypes = m->desc.ntypes;
  A.nm = m->nm;
  for (int t = 0; t <= kMaxT; ++t) A.sec[t] = t <= m->desc.ntypes ? m->sec[t] : m->nm;
  A.inv_nm = 1.0 / (double)m->nm;
  A.ctr = c->emb_ctr;
  A.flags = c->flags_dev;
  // one grid row shared out among the nets by their work (net_of_group), all
  // work-groups resident at once.  The window pays from about ten columns
  // per CU (below, its staging and the one work-group per CU cost more than
  // the L2 reads): forward / backward with and without it at water's 2,400
  // columns 36 / 47 against 37 / 49 us, copper's 1,372 72 / 104 against
  // 55 / 88 us, copper's 4,000 80 / 122 against 116 / 214 us
  const int nnets = A.ntypes * A.ntypes;
  const int64_t columns = c->natoms_last * A.ntypes;
  const int wpb = columns >= (int64_t)c->ncu * 10 ? 16 : 4;
  const int64_t need = (columns + wpb - 1) / wpb, res = (int64_t)c->ncu * (wpb == 16 ? 1 : 3);
  static_assert(kEmbPerCu >= 3, "a column counter per work-group");
  const int64_t groups = need < res ? need : res;
  dim3 grid((unsigned)(groups > nnets ? groups : nnets), 1);
  if (m->m1 == 100) launch_tab<100>(bwd, wpb, grid, A, s);
  else launch_tab<128>(bwd, wpb, grid, A, s);
}

}  // namespace dpse

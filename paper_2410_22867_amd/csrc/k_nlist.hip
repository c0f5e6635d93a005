// Neighbour list (Background section, Fig. 1(a); Evaluation section:
// per-type neighbour counts sel): cell binning + 27-cell stencil search +
// per-type sorted, truncated, -1-padded sections.
//
// Work layout: binning is one thread per atom (counting sort by cell with
// global atomics); the search is one wavefront per centre atom: lanes walk
// the atoms of each stencil cell 64 at a time, survivors of r^2 < rc^2 are
// appended to a wave-private LDS candidate list with ballot/prefix counts,
// then every candidate's rank within its type section is counted against all
// candidates (a deterministic total order on (r^2, packed)), so the written
// list does not depend on the nondeterministic order of binning.
#include "dp_internal.h"
#include "dp_device.h"

// Every floating-point operation of this file is rounded on its own (no fused
// multiply-add): the cut-off test and the sort key must reproduce the plain
// expression bit for bit.
#pragma clang fp contract(off)

namespace dpse {

// r^2 = (dx*dx + dy*dy) + dz*dz, each operation rounded separately.
__device__ __forceinline__ double r2_nofma(double dx, double dy, double dz) {
  return (dx * dx + dy * dy) + dz * dz;
}

__device__ __forceinline__ int cell_coord(double x, double L, int nc) {
  int k = (int)floor(x / L * (double)nc);
  return k < 0 ? 0 : (k >= nc ? nc - 1 : k);
}

// With xw != NULL (a Verlet build) the positions are first wrapped into
// [0, L) in place by whole box lengths, the lengths moved being added to the
// image counters (when non-NULL).  gate: see launch_nl_skin_update.
__global__ void k_nl_bin(const double* __restrict__ x, const FrameInfo* __restrict__ fr, int nframes, int ntot,
                         int32_t* __restrict__ cell_of, int32_t* __restrict__ cell_count, int32_t* flags,
                         double* xw, int32_t* images, const int32_t* gate) {
  if (gate && *gate == 0) return;
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= ntot) return;
  int f = find_frame(fr, nframes, i);
  const FrameInfo F = fr[f];
  int c[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    double xa = x[3 * i + a];
    if (xw && !(xa >= 0.0 && xa < F.L[a])) {
      const double L = F.L[a];
      const double k = floor(xa / L);
      xa -= k * L;
      if (xa >= L) xa -= L;  // rounding of x - k L
      if (xa < 0.0) xa += L;
      if (xa >= L) xa = 0.0;
      xw[3 * i + a] = xa;
      if (images) images[3 * i + a] += (int32_t)k;
    }
    if (!(xa >= 0.0 && xa < F.L[a])) set_flag(flags, DP_FLAG_NOT_WRAPPED);
    c[a] = cell_coord(xa, F.L[a], F.ncell[a]);
  }
  int cid = F.cell_off + c[0] + F.ncell[0] * (c[1] + F.ncell[1] * c[2]);
  cell_of[i] = cid;
  atomicAdd(&cell_count[cid], 1);
}

// Exclusive scan of cell counts with one work-group (cells number in the
// thousands); also clears the fill counters, and the counts once read, so
// that the next binning starts from zero.
__global__ __launch_bounds__(1024) void k_nl_scan(int32_t* __restrict__ count, int32_t* __restrict__ start,
                                                  int32_t* __restrict__ fill, int ncells, const int32_t* gate) {
  if (gate && *gate == 0) return;
  __shared__ int32_t part[1024];
  __shared__ int32_t carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int base = 0; base < ncells; base += 1024) {
    int k = base + threadIdx.x;
    int v = k < ncells ? count[k] : 0;
    if (k < ncells) count[k] = 0;
    part[threadIdx.x] = v;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
      int t = threadIdx.x >= off ? part[threadIdx.x - off] : 0;
      __syncthreads();
      part[threadIdx.x] += t;
      __syncthreads();
    }
    if (k < ncells) {
      start[k] = carry + part[threadIdx.x] - v;
      fill[k] = 0;
    }
    __syncthreads();
    if (threadIdx.x == 1023) carry += part[1023];
    __syncthreads();
  }
  if (threadIdx.x == 0) start[ncells] = carry;
}

__global__ void k_nl_scatter(const int32_t* __restrict__ cell_of, const int32_t* __restrict__ start,
                             int32_t* __restrict__ fill, int32_t* __restrict__ cell_atoms, int ntot,
                             const int32_t* gate) {
  if (gate && *gate == 0) return;
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= ntot) return;
  int c = cell_of[i];
  int p = atomicAdd(&fill[c], 1);
  cell_atoms[start[c] + p] = i;
}

struct SearchArgs {
  const double* x;
  const int32_t* types;
  const FrameInfo* fr;
  const int32_t* cell_start;
  const int32_t* cell_atoms;
  int32_t* nlist;
  int32_t* overflow;
  int32_t* flags;
  int nframes, ntot, ntypes, nm;
  int sel[kMaxT];
  int sec[kMaxT + 1];
  double rc2;
};

constexpr int kSearchWaves = 4;

// Wave-private candidate buffers in LDS: one 16-byte record per candidate.
struct CandRec {
  double r2;
  int32_t pk;
  int16_t k;  // position in the Verlet candidate list (format only)
  int8_t t;
  int8_t pad;
};
// CAP records per wave: kCandCap for the Verlet build (every pair within
// r_c + skin); for the search and the format, which keep pairs within r_c
// only, 256 when the sections hold at most 256 neighbours (half the LDS,
// twice the resident work-groups), kCandCap otherwise.  More kept pairs
// than CAP raise DP_FLAG_CAND_CAPACITY.
constexpr int kKeepCapSmall = 256;
// While cells are walked, also per wave: the non-empty stencil cells (position of flat index 0 among
// the binned atoms, image code, shift) and one bit per flat index, set where a
// cell ends.
struct CellRec {
  double sh[3];
  int32_t off, code;
};
constexpr int kMarkWords = 64;  // 2,048 flat indices at a time
template <int CAP>
struct CandLds {
  CandRec r[kSearchWaves][CAP];
};
struct CellLds {
  CellRec cell[kSearchWaves][28];
  uint32_t mark[kSearchWaves][kMarkWords];
};

// Walks the 27 stencil cells of atom i (one wavefront) and appends every
// (j, s) with r^2 < rad2 to the LDS buffers of wave w, in a fixed order.
// Returns the candidate count (capped at CAP; *capacity set beyond).
template <int CAP>
__device__ __forceinline__ int gather_cells(const SearchArgs& A, CandLds<CAP>& L, CellLds& C, int w, int lane, int i, const FrameInfo& F, double rad2,
                            bool* capacity) {
  const double xi = A.x[3 * i], yi = A.x[3 * i + 1], zi = A.x[3 * i + 2];
  const int ci[3] = {cell_coord(xi, F.L[0], F.ncell[0]), cell_coord(yi, F.L[1], F.ncell[1]),
                     cell_coord(zi, F.L[2], F.ncell[2])};
  int ncand = 0;
  // Lane c < 27 describes stencil cell c (dx, dy, dz in {-1,0,1}): first
  // atom, atom count and image code; a wave prefix sum over the counts turns
  // the 27 cell loops into one flat loop over all candidates.
  int c_start = 0, c_cnt = 0, c_code = 13;
  if (lane < 27) {
    const int dx = lane % 3 - 1, dy = (lane / 3) % 3 - 1, dz = lane / 9 - 1;
    int cc[3] = {ci[0] + dx, ci[1] + dy, ci[2] + dz};
    int sh[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      sh[a] = 0;
      if (cc[a] < 0) { cc[a] += F.ncell[a]; sh[a] = -1; }
      else if (cc[a] >= F.ncell[a]) { cc[a] -= F.ncell[a]; sh[a] = 1; }
    }
    const int cid = F.cell_off + cc[0] + F.ncell[0] * (cc[1] + F.ncell[1] * cc[2]);
    c_start = A.cell_start[cid];
    c_cnt = A.cell_start[cid + 1] - c_start;
    c_code = (sh[0] + 1) + 3 * (sh[1] + 1) + 9 * (sh[2] + 1);
  }
  int c_end = c_cnt;  // inclusive prefix sum
#pragma unroll
  for (int off = 1; off < 32; off <<= 1) {
    const int y = __shfl_up(c_end, off, 64);
    if (lane >= off) c_end += y;
  }
  const int total = __shfl(c_end, 26, 64);
  const uint64_t full = __ballot(lane < 27 && c_cnt > 0);
  if (lane < 27 && c_cnt > 0) {
    CellRec rec;
    rec.sh[0] = (double)(c_code % 3 - 1) * F.L[0];
    rec.sh[1] = (double)((c_code / 3) % 3 - 1) * F.L[1];
    rec.sh[2] = (double)(c_code / 9 - 1) * F.L[2];
    rec.off = c_start - (c_end - c_cnt);
    rec.code = c_code;
    C.cell[w][__builtin_amdgcn_mbcnt_lo((uint32_t)full, 0)] = rec;
  }
  // Flat index t lies in cell number (ends before t): the marks below it,
  // counted for a whole batch of 64 by one read and two bit counts (a search
  // over the 27 ends by lane exchanges was most of this kernel's instructions).
  // Four batches at a time: atom numbers, then positions and types of all four
  // are requested before the first is used.  The search of 3,333 water atoms
  // 28.8 -> 26.0 us, 12,288 46 -> 42, 4,000 copper atoms 49 -> 41, 19,652
  // 195 -> 161.
  int cell0 = 0;  // cells that end before the batch
  constexpr int U = 4;
  for (int t0 = 0; t0 < total; t0 += 64 * U) {
    if ((t0 & (32 * kMarkWords - 1)) == 0) {
      wave_lds_sync();
      C.mark[w][lane] = 0;
      wave_lds_sync();
      const int e = c_end - 1 - t0;
      if (lane < 27 && c_cnt > 0 && e >= 0 && e < 32 * kMarkWords) atomicOr(&C.mark[w][e >> 5], 1u << (e & 31));
      wave_lds_sync();
    }
    int c[U], j[U], tj[U];
    double x[U][3];
#pragma unroll
    for (int m = 0; m < U; ++m) {
      const int t = t0 + 64 * m + lane, k = ((t0 >> 5) + 2 * m) & (kMarkWords - 1);
      const uint32_t m0 = __builtin_amdgcn_readfirstlane(C.mark[w][k]);
      const uint32_t m1 = __builtin_amdgcn_readfirstlane(C.mark[w][k + 1]);
      c[m] = cell0 + __builtin_amdgcn_mbcnt_hi(m1, __builtin_amdgcn_mbcnt_lo(m0, 0));
      cell0 += __popc(m0) + __popc(m1);
      j[m] = t < total ? A.cell_atoms[C.cell[w][c[m]].off + t] : i;
    }
#pragma unroll
    for (int m = 0; m < U; ++m) {
      if (t0 + 64 * m >= total) break;
#pragma unroll
      for (int a = 0; a < 3; ++a) x[m][a] = A.x[3 * j[m] + a];
      tj[m] = A.types[j[m]];
    }
#pragma unroll
    for (int m = 0; m < U; ++m) {
      if (t0 + 64 * m >= total) break;
      const CellRec cr = C.cell[w][t0 + 64 * m + lane < total ? c[m] : 0];
      const double r2 = r2_nofma((x[m][0] - xi) + cr.sh[0], (x[m][1] - yi) + cr.sh[1], (x[m][2] - zi) + cr.sh[2]);
      const bool keep = t0 + 64 * m + lane < total && !(cr.code == 13 && j[m] == i) && r2 < rad2;
      const uint64_t mask = __ballot(keep);
      const int before = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
      const int slot = ncand + before;
      if (keep && slot < CAP) {
        CandRec rec;
        rec.r2 = r2;
        rec.pk = 27 * j[m] + cr.code;
        rec.k = 0;
        rec.t = (int8_t)valid_type(tj[m], A.ntypes, A.flags);
        rec.pad = 0;
        L.r[w][slot] = rec;
      }
      ncand += __popcll(mask);
    }
  }
  if (ncand > CAP) {
    *capacity = true;
    ncand = CAP;
  }
  return ncand;
}

// Ranks the ncand LDS candidates of wave w inside their type sections by
// (r^2, packed) -- a total order, so the result does not depend on the order
// of the buffer -- writes the first sel[t] of each section to row i of the
// list, pads with -1 and counts what was dropped.  The buffer is first
// regrouped by type (through registers), so each candidate is compared only
// with its own section.  With cof != NULL (Verlet format) it also records,
// per written slot, the candidate it came from and, per kept candidate, its
// slot (-1 when truncated).
template <int CAP>
__device__ __forceinline__ void rank_and_write(const SearchArgs& A, CandLds<CAP>& L, int w, int lane, int i, int ncand, bool capacity,
                               int32_t* cof, int32_t* slot_of) {
  constexpr int kPer = CAP / 64;
  // records move as 16-byte vectors (r^2 bits | packed | k, type)
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  u32x4* R = reinterpret_cast<u32x4*>(&L.r[w][0]);
  u32x4 mine[kPer];
  int pos[kPer], mt[kPer];
  int cnt[kMaxT] = {0, 0, 0, 0};
#pragma clang loop unroll(full)
  for (int m = 0; m < kPer; ++m) {
    pos[m] = -1;
    mt[m] = -1;
    if (m * 64 < ncand) {
      const int c = m * 64 + lane;
      if (c < ncand) {
        mine[m] = R[c];
        mt[m] = (int)((mine[m][3] >> 16) & 0xff);
      }
#pragma unroll
      for (int u = 0; u < kMaxT; ++u) {
        if (u < A.ntypes) {
          const uint64_t bal = __ballot(mt[m] == u);
          const int before = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                       __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0));
          if (mt[m] == u) pos[m] = cnt[u] + before;
          cnt[u] += __popcll(bal);
        }
      }
    }
  }
  int off[kMaxT];
  {
    int acc = 0;
#pragma unroll
    for (int u = 0; u < kMaxT; ++u) {
      off[u] = acc;
      acc += cnt[u];
    }
  }
  wave_lds_sync();
#pragma clang loop unroll(full)
  for (int m = 0; m < kPer; ++m)
    if (pos[m] >= 0) {
      int base = 0;  // off[t] without a dynamically indexed register array
#pragma unroll
      for (int u = 1; u < kMaxT; ++u) base = mt[m] == u ? off[u] : base;
      R[base + pos[m]] = mine[m];
    }
  wave_lds_sync();
  int32_t* row = A.nlist + (int64_t)i * A.nm;
  int ovf = 0;
#pragma unroll
  for (int u = 0; u < kMaxT; ++u) {
    if (u >= A.ntypes) break;
    const CandRec* sec = &L.r[w][off[u]];
    const int n_u = cnt[u];
    const int sel = A.sel[u];
    // Rank of each candidate in its section on (r^2, packed).  Exact ties in
    // r^2 are rare, so each candidate first counts the candidates whose r^2
    // is <= its own (one compare per pair).  Without ties these counts are
    // a permutation of 1..n_u; with T pairs of equal r^2 they sum to
    // n_u (n_u + 1) / 2 + T, so one wave sum tells whether the section
    // needs the full comparison with the packed-index tie-break.
    int rk[kPer];
    int sum = 0;
#pragma clang loop unroll(full)
    for (int m = 0; m < kPer; ++m) {
      rk[m] = 0;
      if (64 * m < n_u) {
        const int c = 64 * m + lane;
        if (c < n_u) {
          const double r2 = sec[c].r2;
          int le = 0;
#pragma unroll 4
          for (int o = 0; o < n_u; ++o) le += sec[o].r2 <= r2;
          rk[m] = le;
          sum += le;
        }
      }
    }
#pragma unroll
    for (int x = 32; x >= 1; x >>= 1) sum += __shfl_xor(sum, x, 64);
    const bool ties = sum != n_u * (n_u + 1) / 2;
#pragma clang loop unroll(full)
    for (int m = 0; m < kPer; ++m) {
      if (64 * m >= n_u) break;
      const int c = 64 * m + lane;
      if (c >= n_u) continue;
      const CandRec me = sec[c];
      int rank = rk[m] - 1;
      if (ties) {
        rank = 0;
        for (int o = 0; o < n_u; ++o) {
          const CandRec ot = sec[o];
          rank += (ot.r2 < me.r2 || (ot.r2 == me.r2 && ot.pk < me.pk));
        }
      }
      const bool kept = rank < sel;
      if (kept) row[A.sec[u] + rank] = me.pk;
      if (cof) {
        if (kept) cof[(int64_t)i * A.nm + A.sec[u] + rank] = me.k;
        slot_of[(int64_t)i * kCandCap + me.k] = kept ? i * A.nm + A.sec[u] + rank : -1;
      }
    }
    const int kept = n_u < sel ? n_u : sel;
    for (int q = kept + lane; q < sel; q += 64) row[A.sec[u] + q] = -1;
    ovf += n_u - kept;
  }
  if (lane == 0) {
    if (ovf) {
      atomicAdd(A.overflow, ovf);
      set_flag(A.flags, DP_FLAG_SEL_OVERFLOW);
    }
    if (capacity) set_flag(A.flags, DP_FLAG_CAND_CAPACITY);
  }
}

template <int CAP>
__global__ __launch_bounds__(256) void k_nl_search(SearchArgs A) {
  __shared__ CandLds<CAP> L;
  __shared__ CellLds C;
  const int lane = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
  const int i = blockIdx.x * kSearchWaves + w;
  if (i >= A.ntot) return;
  const FrameInfo F = A.fr[find_frame(A.fr, A.nframes, i)];
  bool capacity = false;
  const int ncand = gather_cells(A, L, C, w, lane, i, F, A.rc2, &capacity);
  wave_lds_sync();
  rank_and_write(A, L, w, lane, i, ncand, capacity, nullptr, nullptr);
}

// ------------------------------------------------------------ Verlet list
// Build: every (j, s) with r^2 < (r_c + skin)^2 on the wrapped positions,
// stored per atom sorted by packed value (so a pair's reverse entry is found
// by binary search), with the positions of the build.
struct SkinArgs {
  int32_t* cand;    // [n, kCandCap]
  int32_t* ncand;   // [n]
  int32_t* crev;    // [n, kCandCap]
  int32_t* slot_of; // [n, kCandCap]
  int32_t* cof;     // [n, nm]
  double* xref;     // [n, 3]
  double L[3];
  double half_skin2;
  // rebuild decided on the device (launch_nl_skin_update): gate[0] != 0
  // when the kernels of a build run, gate[1] counts formats since the last
  // build; NULL for a build the host asked for
  int32_t* gate;
  int32_t* rebuilds;  // incremented by every gated build (nullable)
};

// One wavefront per atom, atoms taken in a grid-stride loop (the grid is
// sized to the resident capacity, so a gated launch that does nothing is
// cheap).
__global__ __launch_bounds__(256) void k_nl_skin_build(SearchArgs A, SkinArgs S, double rl2) {
  if (S.gate && S.gate[0] == 0) return;
  __shared__ CandLds<kCandCap> L;
  __shared__ CellLds C;
  const int lane = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
  if (S.gate && blockIdx.x == 0 && threadIdx.x == 0) {
    S.gate[1] = 0;
    if (S.rebuilds) *S.rebuilds += 1;
  }
  for (int i = blockIdx.x * kSearchWaves + w; i < A.ntot; i += gridDim.x * kSearchWaves) {
    const FrameInfo F = A.fr[find_frame(A.fr, A.nframes, i)];
    bool capacity = false;
    const int ncand = gather_cells(A, L, C, w, lane, i, F, rl2, &capacity);
    wave_lds_sync();
    // rank of each candidate by its packed key (keys are distinct): one pass
    // over the list serves all of a lane's candidates, each record read once
    constexpr int M = kCandCap / 64;
    const int mmax = (ncand + 63) / 64;  // wave-uniform
    int pkm[M], rank[M];
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const int c = 64 * m + lane;
      pkm[m] = c < ncand ? L.r[w][c].pk : 0x7fffffff;
      rank[m] = 0;
    }
    for (int o = 0; o < ncand; ++o) {
      const int v = L.r[w][o].pk;
#pragma unroll
      for (int m = 0; m < M; ++m)
        if (m < mmax) rank[m] += v < pkm[m];
    }
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const int c = 64 * m + lane;
      if (c < ncand) S.cand[(int64_t)i * kCandCap + rank[m]] = pkm[m];
    }
    if (lane < 3) S.xref[3 * i + lane] = A.x[3 * i + lane];
    if (lane == 0) {
      S.ncand[i] = ncand;
      if (capacity) set_flag(A.flags, DP_FLAG_CAND_CAPACITY);
    }
    wave_lds_sync();  // the wave's LDS records are rewritten by its next atom
  }
}

// Position of each of atom i's candidates' reverse pair (i, -s) in j's
// candidate list, by one wave: lane l takes candidates l, l + 64, ... of i's
// list, four at a time, and runs their binary searches in j's sorted candidate
// list in lockstep (a fixed ten halvings cover the 512-entry capacity), so
// that four dependent-load chains are in flight per lane instead of one.
__device__ __forceinline__ void crev_row(const SkinArgs& S, int i, int lane) {
  const int nc = S.ncand[i];
  const int32_t* ci = S.cand + (int64_t)i * kCandCap;
  constexpr int M = kCandCap / 64, U = 4;
  static_assert(kCandCap <= 1024, "ten halvings cover the list");
#pragma unroll 1
  for (int m0 = 0; m0 < M && 64 * m0 < nc; m0 += U) {
    int lo[U], hi[U], nj[U], tgt[U];
    const int32_t* cj[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = 64 * (m0 + u) + lane;
      lo[u] = 0;
      hi[u] = 0;
      nj[u] = 0;
      tgt[u] = 0;
      cj[u] = ci;
      if (m0 + u < M && k < nc) {
        const int e = ci[k];
        const int j = e / 27;
        tgt[u] = 27 * i + (26 - (e - 27 * j));
        cj[u] = S.cand + (int64_t)j * kCandCap;
        nj[u] = S.ncand[j];
        hi[u] = nj[u];
      }
    }
#pragma unroll 1
    for (int it = 0; it < 10; ++it)
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (lo[u] < hi[u]) {
          const int mid = (lo[u] + hi[u]) >> 1;
          if (cj[u][mid] < tgt[u]) lo[u] = mid + 1;
          else hi[u] = mid;
        }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = 64 * (m0 + u) + lane;
      if (m0 + u < M && k < nc) S.crev[(int64_t)i * kCandCap + k] = (lo[u] < nj[u] && cj[u][lo[u]] == tgt[u]) ? lo[u] : -1;
    }
  }
}

// The reverse positions after a build the host asked for (a gated build's
// are found by the next format, one launch less in every update).
__global__ __launch_bounds__(256) void k_nl_skin_crev(SkinArgs S, int ntot) {
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i < ntot) crev_row(S, i, threadIdx.x & 63);
}

// After a build the host asked for: no rebuild pending, no format since.
__global__ void k_fill_gate(int32_t* gate) {
  if (threadIdx.x < 2) gate[threadIdx.x] = 0;
}

// Rebuild decision of a Verlet update: gate[0] is set when an atom has moved
// more than skin/2 since the build (the format's exactness condition) or
// when `every` > 0 updates have passed since it.  gate[0] was cleared by the
// previous format's second pass.
__device__ __forceinline__ bool skin_moved(const double* x, const double* xref, int ntot, double half_skin2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= ntot) return false;
  const double ex = x[3 * i] - xref[3 * i], ey = x[3 * i + 1] - xref[3 * i + 1], ez = x[3 * i + 2] - xref[3 * i + 2];
  return !((ex * ex + ey * ey) + ez * ez <= half_skin2);
}
__device__ __forceinline__ bool skin_due(int every, int32_t* gate) {  // one thread of the grid
  const int k = gate[1] + 1;
  gate[1] = k;
  return every > 0 && k >= every;
}

__global__ __launch_bounds__(256) void k_nl_skin_check(const double* __restrict__ x, const double* __restrict__ xref,
                                                       int ntot, double half_skin2, int every, int32_t* gate) {
  const bool moved = skin_moved(x, xref, ntot, half_skin2);
  if (__ballot(moved) && (threadIdx.x & 63) == 0) atomicOr(gate, 1);
  if (blockIdx.x == 0 && threadIdx.x == 0 && skin_due(every, gate)) atomicOr(gate, 1);
}

// Exclusive scan of a work-group's LDS cell counts (1,024 threads): thread t
// sums its run of cells, a scan of the 1,024 sums, then the run's starts, to
// LDS and memory; the counts are cleared for the scatter.
constexpr int kPrepSmallCells = 4096;
__device__ __forceinline__ void scan_cells(int32_t* cnt, int32_t* st, int32_t* part, int32_t* __restrict__ start, int ncells) {
  constexpr int kRun = kPrepSmallCells / 1024;
  const int tid = threadIdx.x, c0 = tid * kRun;
  int run = 0;
#pragma unroll
  for (int q = 0; q < kRun; ++q) run += c0 + q < ncells ? cnt[c0 + q] : 0;
  part[tid] = run;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    const int t = tid >= off ? part[tid - off] : 0;
    __syncthreads();
    part[tid] += t;
    __syncthreads();
  }
  int acc = part[tid] - run;
#pragma unroll
  for (int q = 0; q < kRun; ++q)
    if (c0 + q < ncells) {
      st[c0 + q] = acc;
      start[c0 + q] = acc;
      acc += cnt[c0 + q];
      cnt[c0 + q] = 0;
    }
  if (tid == 1023) start[ncells] = part[1023];
}

// Frames of up to 131,072 atoms and 4,096 cells: the check and the cell
// binning of a gated Verlet build (wrap in place, cell counts, their scan, the
// scatter) in one launch instead of four.  Every work-group checks 1,024
// atoms; the one that ends last, when all have read their positions, sees the
// decision and does the binning alone if there is one (counts and fill
// counters stay in LDS; the global ones, which the multi-work-group binning
// uses, stay zero).  A launch that finds nothing to do costs 4.6 us in a
// stream of kernels, whatever its size (check, empty binning and
// empty reverse search at 12,288 atoms: 13.9 us before, 4.6 and 0.9 in the
// format now).
constexpr int kPrepSmallAtoms = 1 << 17;
__global__ __launch_bounds__(1024) void k_nl_check_bin(double* __restrict__ x, const double* __restrict__ xref,
                                                      const FrameInfo* __restrict__ fr, int ntot, double half_skin2,
                                                      int every, int ncells, int32_t* gate, int32_t* done,
                                                      int32_t* __restrict__ cell_of, int32_t* __restrict__ cell_start,
                                                      int32_t* __restrict__ cell_atoms, int32_t* flags,
                                                      int32_t* images) {
  __shared__ int32_t go;
  const bool due = blockIdx.x == 0 && threadIdx.x == 0 && skin_due(every, gate);
  const int any = __syncthreads_or(skin_moved(x, xref, ntot, half_skin2) || due);
  if (threadIdx.x == 0) {
    // (a decision has reached memory before this work-group counts itself done:
    // the atomic's result is waited for; nothing else is handed over)
    if (any) {
      const int old = atomicOr(gate, 1);
      asm volatile("" ::"v"(old) : "memory");
    }
    go = 0;
    if (gridDim.x == 1) {
      go = any;
    } else if (atomicAdd(done, 1) == (int)gridDim.x - 1) {
      atomicExch(done, 0);
      go = atomicOr(gate, 0);
    }
  }
  __syncthreads();
  if (go == 0) return;
  __shared__ int32_t cnt[kPrepSmallCells];  // counts, then fill counters
  __shared__ int32_t st[kPrepSmallCells];   // cell starts
  __shared__ int32_t part[1024];
  const int tid = threadIdx.x;
  for (int c = tid; c < ncells; c += 1024) cnt[c] = 0;
  __syncthreads();
  const FrameInfo F = fr[0];
  for (int i = tid; i < ntot; i += 1024) {
    int cc[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      double xa = x[3 * i + a];
      if (!(xa >= 0.0 && xa < F.L[a])) {
        const double L = F.L[a];
        const double k = floor(xa / L);
        xa -= k * L;
        if (xa >= L) xa -= L;  // rounding of x - k L
        if (xa < 0.0) xa += L;
        if (xa >= L) xa = 0.0;
        x[3 * i + a] = xa;
        if (images) images[3 * i + a] += (int32_t)k;
      }
      if (!(xa >= 0.0 && xa < F.L[a])) set_flag(flags, DP_FLAG_NOT_WRAPPED);
      cc[a] = cell_coord(xa, F.L[a], F.ncell[a]);
    }
    const int cid = cc[0] + F.ncell[0] * (cc[1] + F.ncell[1] * cc[2]);
    cell_of[i] = F.cell_off + cid;
    atomicAdd(&cnt[cid], 1);
  }
  __syncthreads();
  scan_cells(cnt, st, part, cell_start + F.cell_off, ncells);
  __syncthreads();
  for (int i = tid; i < ntot; i += 1024) {
    const int cid = cell_of[i] - F.cell_off;
    const int p = atomicAdd(&cnt[cid], 1);
    cell_atoms[st[cid] + p] = i;
  }
}

// Calls of up to 8,192 atoms and 4,096 cells: everything a list build does
// before its search, and the type sort, in one launch of two work-groups
// instead of eight launches (each 4.5 to 17 us in a stream of kernels: 3,333
// water atoms 39 -> 9 us, 8,190 43 -> 16, 4,000 copper atoms 61 -> 10).  Work-group 0 bins
// (overflow count cleared, cell counts and fill counters in LDS, the scan, the
// scatter); work-group 1 sorts the types, as k_type_count, k_type_scan and
// k_type_assign do.  A thread's eight atoms are loaded before any is used.
// The launches' time hardly grows with the atoms, this kernel's in proportion:
// beyond the registers of eight atoms a thread there is little to win, and the
// multi-work-group kernels are taken.
constexpr int kPrepAtoms = 8192, kPrepPer = kPrepAtoms / 1024;
struct PrepArgs {
  const double* x;
  const int32_t* types;
  const FrameInfo* fr;
  int nframes, ntot, ncells, ntypes, ncols;
  int32_t *overflow, *flags;
  int32_t *cell_of, *cell_start, *cell_atoms;
  int32_t *meta, *col_of, *atom_at, *frame_of;
  Sections q;
};

__global__ __launch_bounds__(1024) void k_nl_prep(PrepArgs A) {
  __shared__ int32_t lds[2 * kPrepSmallCells + 1024];
  const int tid = threadIdx.x;
  if (blockIdx.x == 0) {
    int32_t *cnt = lds, *st = lds + kPrepSmallCells, *part = lds + 2 * kPrepSmallCells;
    if (tid == 0) *A.overflow = 0;
    for (int c = tid; c < A.ncells; c += 1024) cnt[c] = 0;
    double x[kPrepPer][3];
    int cid[kPrepPer];
#pragma unroll
    for (int m = 0; m < kPrepPer; ++m)
#pragma unroll
      for (int a = 0; a < 3; ++a) x[m][a] = 1024 * m + tid < A.ntot ? A.x[3 * (1024 * m + tid) + a] : 0.0;
    __syncthreads();
#pragma unroll
    for (int m = 0; m < kPrepPer; ++m) {
      const int i = 1024 * m + tid;
      if (i < A.ntot) {
        const FrameInfo& F = A.fr[find_frame(A.fr, A.nframes, i)];
        int c[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          if (!(x[m][a] >= 0.0 && x[m][a] < F.L[a])) set_flag(A.flags, DP_FLAG_NOT_WRAPPED);
          c[a] = cell_coord(x[m][a], F.L[a], F.ncell[a]);
        }
        cid[m] = F.cell_off + c[0] + F.ncell[0] * (c[1] + F.ncell[1] * c[2]);
        A.cell_of[i] = cid[m];
        atomicAdd(&cnt[cid[m]], 1);
      }
    }
    __syncthreads();
    scan_cells(cnt, st, part, A.cell_start, A.ncells);
    __syncthreads();
#pragma unroll
    for (int m = 0; m < kPrepPer; ++m)
      if (1024 * m + tid < A.ntot) A.cell_atoms[st[cid[m]] + atomicAdd(&cnt[cid[m]], 1)] = 1024 * m + tid;
    return;
  }
  // [type][chunk of 1,024 atoms][wave]: atoms of the type in the wave, then before it
  constexpr int kW = kPrepPer * 16;
  int32_t *wc = lds, *tot = lds + kMaxT * kW;
  const int lane = tid & 63, w = tid >> 6;
  int ty[kPrepPer], before[kPrepPer];
#pragma unroll
  for (int m = 0; m < kPrepPer; ++m) ty[m] = 1024 * m + tid < A.ntot ? A.types[1024 * m + tid] : -1;
  for (int c = tid; c < A.ncols; c += 1024) A.atom_at[c] = -1;
#pragma unroll
  for (int m = 0; m < kPrepPer; ++m) {
    if (1024 * m + tid < A.ntot) ty[m] = valid_type(ty[m], A.ntypes, A.flags);
    before[m] = 0;
#pragma unroll
    for (int u = 0; u < kMaxT; ++u) {
      const uint64_t b = __ballot(ty[m] == u);
      if (ty[m] == u)
        before[m] = __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0));
      if (lane == 0) wc[u * kW + m * 16 + w] = __popcll(b);
    }
  }
  __syncthreads();
  if (w < kMaxT) {  // wave u: exclusive prefix over the kW waves of type u
    int run = 0;
#pragma unroll
    for (int c = 0; c < kW; c += 64) {
      const int v = wc[w * kW + c + lane];
      int inc = v;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(inc, off, 64);
        if (lane >= off) inc += y;
      }
      wc[w * kW + c + lane] = run + inc - v;
      run += __shfl(inc, 63, 64);
    }
    if (lane == 0) tot[w] = run;
  }
  __syncthreads();
  if (tid < 64) write_type_meta(tot, A.ntypes, A.q, A.meta, tid);
  int base[kMaxT], acc = 0;
#pragma unroll
  for (int u = 0; u < kMaxT; ++u) {
    base[u] = acc;
    acc += (tot[u] + kColPad - 1) / kColPad * kColPad;
  }
#pragma unroll
  for (int m = 0; m < kPrepPer; ++m) {
    const int i = 1024 * m + tid;
    if (i < A.ntot) {
      int b = base[0];
#pragma unroll
      for (int u = 1; u < kMaxT; ++u) b = ty[m] == u ? base[u] : b;
      const int col = b + wc[ty[m] * kW + m * 16 + w] + before[m];
      A.col_of[i] = col;
      A.atom_at[col] = i;
      A.frame_of[i] = find_frame(A.fr, A.nframes, i);
    }
  }
}

// Format: the sorted, truncated list on the current positions from the
// candidates of the last build (same test and order as the cell search).
template <int CAP>
__global__ __launch_bounds__(256) void k_nl_skin_format(SearchArgs A, SkinArgs S) {
  __shared__ CandLds<CAP> L;
  const int lane = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
  const int i = blockIdx.x * kSearchWaves + w;
  if (i >= A.ntot) return;
  const int rebuilt = S.gate[0];
  const double xi = A.x[3 * i], yi = A.x[3 * i + 1], zi = A.x[3 * i + 2];
  if (lane == 0) {
    const double ex = xi - S.xref[3 * i], ey = yi - S.xref[3 * i + 1], ez = zi - S.xref[3 * i + 2];
    if (!((ex * ex + ey * ey) + ez * ez <= S.half_skin2)) set_flag(A.flags, DP_FLAG_SKIN_EXCEEDED);
  }
  const int nc = S.ncand[i];
  const int32_t* ci = S.cand + (int64_t)i * kCandCap;
  // all loads of a lane's candidates are issued before any is used
  constexpr int kPer = kCandCap / 64;
  int e[kPer], tj[kPer];
  double r2[kPer];
#pragma unroll
  for (int m = 0; m < kPer; ++m) e[m] = (64 * m < nc && 64 * m + lane < nc) ? ci[64 * m + lane] : -1;
#pragma unroll
  for (int m = 0; m < kPer; ++m) {
    r2[m] = 0.0;
    tj[m] = 0;
    if (e[m] >= 0) {
      const int j = e[m] / 27, sc = e[m] - 27 * j;
      const double ddx = (A.x[3 * j] - xi) + (double)(sc % 3 - 1) * S.L[0];
      const double ddy = (A.x[3 * j + 1] - yi) + (double)((sc / 3) % 3 - 1) * S.L[1];
      const double ddz = (A.x[3 * j + 2] - zi) + (double)(sc / 9 - 1) * S.L[2];
      r2[m] = r2_nofma(ddx, ddy, ddz);
      tj[m] = A.types[j];
    }
  }
  int ncand = 0;
#pragma unroll
  for (int m = 0; m < kPer; ++m) {
    if (64 * m >= nc) break;
    const int k = 64 * m + lane;
    const bool keep = e[m] >= 0 && r2[m] < A.rc2;
    if (e[m] >= 0 && !keep) S.slot_of[(int64_t)i * kCandCap + k] = -1;
    const uint64_t mask = __ballot(keep);
    const int before = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                 __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
    if (keep && ncand + before >= CAP) S.slot_of[(int64_t)i * kCandCap + k] = -1;  // beyond capacity (flagged)
    if (keep && ncand + before < CAP) {
      int t = tj[m];
      if (t < 0 || t >= A.ntypes) {
        set_flag(A.flags, DP_FLAG_BAD_INPUT);
        t = t < 0 ? 0 : A.ntypes - 1;
      }
      CandRec rec;
      rec.r2 = r2[m];
      rec.pk = e[m];
      rec.k = (int16_t)k;
      rec.t = (int8_t)t;
      rec.pad = 0;
      L.r[w][ncand + before] = rec;
    }
    ncand += __popcll(mask);
  }
  const bool capacity = ncand > CAP;
  if (capacity) ncand = CAP;
  wave_lds_sync();
  rank_and_write(A, L, w, lane, i, ncand, capacity, S.cof, S.slot_of);
  if (rebuilt) crev_row(S, i, lane);  // the update's build has just run
}

// Reverse index from the candidate bookkeeping of the format (same meaning
// as the index built by binary search below).  Its first thread also moves
// the format's truncation count to the caller's buffer and clears the
// internal counter for the next format (stream order: every format block
// has finished, and the next format has not started).
__global__ void k_nl_skin_revmap(const int32_t* __restrict__ nlist, SkinArgs S, int32_t* __restrict__ rev, int ntot,
                                 int nm, int32_t* __restrict__ ovf_ctr, int32_t* __restrict__ overflow,
                                 int32_t* __restrict__ gate) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q == 0) {
    *overflow = *ovf_ctr;
    *ovf_ctr = 0;
    gate[0] = 0;  // the next update decides again
  }
  if (q >= (int64_t)ntot * nm) return;
  const int e = nlist[q];
  int out = -1;
  if (e >= 0) {
    const int i = (int)(q / nm);
    const int kr = S.crev[(int64_t)i * kCandCap + S.cof[q]];
    if (kr >= 0) out = S.slot_of[(int64_t)(e / 27) * kCandCap + kr];
  }
  rev[q] = out;
}

// Reverse index of a symmetric list: for entry q' of atom i pointing to
// (j, s), the slot q of j's list holding (i, -s), stored as j*nm + q
// (-1 when j's section was truncated before i).  The packed entry is looked
// for itself, so a pair missing from j's list is never matched to a wrong
// slot, and no distance is computed.  Sections are sorted by distance and the
// pair's distance is the same from both ends, so the search begins at the rank
// the entry has in its own list, scaled by the sections' sizes: sixteen
// entries there, then eight on either side at a time until the section's ends.
// Against a binary search on the distance (two dependent gathers a halving):
// 3,333 water atoms 20 -> 8.4 us, 12,288 66 -> 20, 4,000 copper atoms 49 -> 15,
// 19,652 243 -> 53.
struct RevArgs {
  const int32_t* types;
  const int32_t* nlist;
  int32_t* rev;
  int ntot, nm, ntypes;
  int sel[kMaxT];
  int sec[kMaxT + 1];
};

typedef int32_t i4u __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ int match4(i4u v, int at, int target, int found) {
#pragma unroll
  for (int k = 0; k < 4; ++k) found = v[k] == target ? at + k : found;
  return found;
}

__global__ __launch_bounds__(256) void k_nl_reverse(RevArgs A) {
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (i >= A.ntot) return;
  int ti = A.types[i];
  ti = ti < 0 ? 0 : (ti >= A.ntypes ? A.ntypes - 1 : ti);
  const int n = A.sel[ti], first = A.sec[ti];
  constexpr int U = 2;  // slots of a lane whose first windows are read together
  for (int q0 = 0; q0 < A.nm; q0 += 64 * U) {
    int j[U], target[U], at[U], found[U];
    i4u v[U][4];
#pragma unroll
    for (int m = 0; m < U; ++m) {
      const int q = q0 + 64 * m + lane;
      const int e = q < A.nm ? A.nlist[(int64_t)i * A.nm + q] : -1;
      const bool on = e >= 0 && e / 27 < A.ntot;
      j[m] = on ? e / 27 : -1;
      target[m] = on ? 27 * i + (26 - (e - 27 * j[m])) : -1;
      found[m] = -1;
      int base = 0, width = A.sel[0];
#pragma unroll
      for (int t = 1; t < kMaxT; ++t)
        if (t < A.ntypes && q >= A.sec[t]) {
          base = A.sec[t];
          width = A.sel[t];
        }
      at[m] = max(0, min((int)((float)(q - base) * ((float)n / (float)max(width, 1))) - 8, n - 16));
    }
    if (n >= 16) {
#pragma unroll
      for (int m = 0; m < U; ++m)
        if (j[m] >= 0) {
          const int32_t* row = A.nlist + (int64_t)j[m] * A.nm + first;
#pragma unroll
          for (int k = 0; k < 4; ++k) v[m][k] = *reinterpret_cast<const i4u*>(row + at[m] + 4 * k);
        }
#pragma unroll
      for (int m = 0; m < U; ++m) {
        if (j[m] < 0) continue;
        const int32_t* row = A.nlist + (int64_t)j[m] * A.nm + first;
#pragma unroll
        for (int k = 0; k < 4; ++k) found[m] = match4(v[m][k], at[m] + 4 * k, target[m], found[m]);
        for (int lo = at[m], hi = at[m] + 16; found[m] < 0 && (lo > 0 || hi < n); lo -= 8, hi += 8) {
          const int l = max(lo - 8, 0), h = min(hi, n - 8);
          const i4u a = *reinterpret_cast<const i4u*>(row + l), b = *reinterpret_cast<const i4u*>(row + l + 4);
          const i4u c = *reinterpret_cast<const i4u*>(row + h), d = *reinterpret_cast<const i4u*>(row + h + 4);
          found[m] = match4(a, l, target[m], match4(b, l + 4, target[m], match4(c, h, target[m], match4(d, h + 4, target[m], -1))));
        }
      }
    } else {
#pragma unroll
      for (int m = 0; m < U; ++m)
        if (j[m] >= 0)
          for (int k = 0; k < n && found[m] < 0; ++k)
            if (A.nlist[(int64_t)j[m] * A.nm + first + k] == target[m]) found[m] = k;
    }
#pragma unroll
    for (int m = 0; m < U; ++m)
      if (q0 + 64 * m + lane < A.nm)
        A.rev[(int64_t)i * A.nm + q0 + 64 * m + lane] = found[m] < 0 ? -1 : j[m] * A.nm + first + found[m];
  }
}

void launch_nl_reverse(dp_ctx* c, const int32_t* types, const int32_t* nlist, int32_t ntot,
                       hipStream_t s) {
  if (ntot <= 0) return;
  const dp_model* m = c->model;
  RevArgs A;
  A.types = types;
  A.nlist = nlist;
  A.rev = c->rev;
  A.ntot = ntot;
  A.nm = m->nm;
  A.ntypes = m->desc.ntypes;
  for (int t = 0; t < kMaxT; ++t) A.sel[t] = t < m->desc.ntypes ? m->desc.sel[t] : 0;
  for (int t = 0; t <= kMaxT; ++t) A.sec[t] = t <= m->desc.ntypes ? m->sec[t] : m->nm;
  hipLaunchKernelGGL(k_nl_reverse, dim3((ntot + 3) / 4), dim3(256), 0, s, A);
}

void launch_nl_bin(dp_ctx* c, const double* x, int32_t ntot, int32_t nframes, hipStream_t s) {
  if (ntot <= 0) return;
  hipLaunchKernelGGL(k_nl_bin, dim3((ntot + 255) / 256), dim3(256), 0, s, x, c->frames_dev, nframes, ntot,
                     c->cell_of, c->cell_count, c->flags_dev, (double*)nullptr, (int32_t*)nullptr,
                     (const int32_t*)nullptr);
}

void launch_nl_scan(dp_ctx* c, int32_t ncells, hipStream_t s) {
  hipLaunchKernelGGL(k_nl_scan, dim3(1), dim3(1024), 0, s, c->cell_count, c->cell_start, c->cell_fill, ncells,
                     (const int32_t*)nullptr);
}

void launch_nl_scatter(dp_ctx* c, int32_t ntot, hipStream_t s) {
  if (ntot <= 0) return;
  hipLaunchKernelGGL(k_nl_scatter, dim3((ntot + 255) / 256), dim3(256), 0, s, c->cell_of, c->cell_start,
                     c->cell_fill, c->cell_atoms, ntot, (const int32_t*)nullptr);
}

static SearchArgs search_args(dp_ctx* c, const double* x, const int32_t* types, int32_t ntot, int32_t nframes,
                              int32_t* nlist, int32_t* overflow) {
  const dp_model* m = c->model;
  SearchArgs A;
  A.x = x;
  A.types = types;
  A.fr = c->frames_dev;
  A.cell_start = c->cell_start;
  A.cell_atoms = c->cell_atoms;
  A.nlist = nlist;
  A.overflow = overflow;
  A.flags = c->flags_dev;
  A.nframes = nframes;
  A.ntot = ntot;
  A.ntypes = m->desc.ntypes;
  A.nm = m->nm;
  for (int t = 0; t < kMaxT; ++t) A.sel[t] = t < m->desc.ntypes ? m->desc.sel[t] : 0;
  for (int t = 0; t <= kMaxT; ++t) A.sec[t] = t <= m->desc.ntypes ? m->sec[t] : m->nm;
  A.rc2 = m->desc.rcut * m->desc.rcut;
  return A;
}

bool launch_nl_prep(dp_ctx* c, const double* x, const int32_t* types, int32_t ntot, int32_t nframes, int64_t ncells,
                    int32_t* overflow, hipStream_t s) {
  if (ntot <= 0 || ntot > kPrepAtoms || ncells > kPrepSmallCells) return false;
  const dp_model* m = c->model;
  PrepArgs A;
  A.x = x;
  A.types = types;
  A.fr = c->frames_dev;
  A.nframes = nframes;
  A.ntot = ntot;
  A.ncells = (int)ncells;
  A.ntypes = m->desc.ntypes;
  A.ncols = ntot + A.ntypes * kColPad;  // more than the padded segments
  A.overflow = overflow;
  A.flags = c->flags_dev;
  A.cell_of = c->cell_of;
  A.cell_start = c->cell_start;
  A.cell_atoms = c->cell_atoms;
  A.meta = c->type_meta;
  A.col_of = c->col_of;
  A.atom_at = c->atom_at;
  A.frame_of = c->frame_of;
  for (int t = 0; t <= kMaxT; ++t) A.q.sec[t] = m->sec[t < A.ntypes ? t : A.ntypes];
  hipLaunchKernelGGL(k_nl_prep, dim3(2), dim3(1024), 0, s, A);
  return true;
}

static SkinArgs skin_args(dp_ctx* c) {
  SkinArgs S;
  S.cand = c->skin_cand;
  S.ncand = c->skin_ncand;
  S.crev = c->skin_crev;
  S.slot_of = c->skin_slot;
  S.cof = c->skin_cof;
  S.xref = c->skin_xref;
  for (int a = 0; a < 3; ++a) S.L[a] = c->skin_L[a];
  S.half_skin2 = 0.25 * c->skin * c->skin;
  S.gate = nullptr;
  S.rebuilds = nullptr;
  return S;
}

void launch_nl_search(dp_ctx* c, const double* x, const int32_t* types, int32_t ntot, int32_t nframes,
                      int32_t* nlist, int32_t* overflow, hipStream_t s) {
  if (ntot <= 0) return;
  SearchArgs A = search_args(c, x, types, ntot, nframes, nlist, overflow);
  const dim3 grid((ntot + kSearchWaves - 1) / kSearchWaves), block(64 * kSearchWaves);
  if (A.nm <= kKeepCapSmall) hipLaunchKernelGGL(k_nl_search<kKeepCapSmall>, grid, block, 0, s, A);
  else hipLaunchKernelGGL(k_nl_search<kCandCap>, grid, block, 0, s, A);
}

// Verlet build from the binned wrapped positions.  The frame (box, cell
// grid of edge >= r_c + skin) is the context's copy made at the last
// dp_nlist_skin_build: dp_compute replaces the general frame table.
static void skin_build_kernels(dp_ctx* c, const double* x, const int32_t* types, int32_t ntot, int32_t* gate,
                               int32_t* rebuilds, hipStream_t s) {
  SearchArgs A = search_args(c, x, types, ntot, 1, nullptr, nullptr);
  A.fr = c->skin_frame;
  SkinArgs S = skin_args(c);
  S.gate = gate;
  S.rebuilds = rebuilds;
  const double rl = c->model->desc.rcut + c->skin;
  // 4-wave work-groups with 36 KB of LDS: 4 resident per CU
  const int64_t gb = (ntot + kSearchWaves - 1) / kSearchWaves, gbmax = 4LL * c->ncu;
  hipLaunchKernelGGL(k_nl_skin_build, dim3((unsigned)(gb < gbmax ? gb : gbmax)), dim3(64 * kSearchWaves), 0, s, A, S,
                     rl * rl);
  if (!gate) hipLaunchKernelGGL(k_nl_skin_crev, dim3((ntot + 3) / 4), dim3(256), 0, s, S, ntot);
}

void launch_nl_skin_build(dp_ctx* c, double* x, const int32_t* types, int32_t ntot, int32_t ncells, int32_t* images,
                          hipStream_t s) {
  if (ntot <= 0) return;
  hipLaunchKernelGGL(k_nl_bin, dim3((ntot + 255) / 256), dim3(256), 0, s, (const double*)x, c->skin_frame, 1, ntot,
                     c->cell_of, c->cell_count, c->flags_dev, x, images, (const int32_t*)nullptr);
  launch_nl_scan(c, ncells, s);
  launch_nl_scatter(c, ntot, s);
  skin_build_kernels(c, x, types, ntot, nullptr, nullptr, s);
  hipLaunchKernelGGL(k_fill_gate, dim3(1), dim3(64), 0, s, c->skin_gate);
}

void launch_nl_skin_update(dp_ctx* c, double* x, const int32_t* types, int32_t ntot, int32_t every, int32_t* images,
                           int32_t* rebuilds, hipStream_t s) {
  if (ntot <= 0) return;
  int32_t* gate = c->skin_gate;
  const double half_skin2 = 0.25 * c->skin * c->skin;
  if (ntot <= kPrepSmallAtoms && c->skin_ncells <= kPrepSmallCells) {
    hipLaunchKernelGGL(k_nl_check_bin, dim3((ntot + 1023) / 1024), dim3(1024), 0, s, x, (const double*)c->skin_xref,
                       c->skin_frame, ntot, half_skin2, every, c->skin_ncells, gate, c->ovf_ctr + 16, c->cell_of,
                       c->cell_start, c->cell_atoms, c->flags_dev, images);
  } else {
    hipLaunchKernelGGL(k_nl_skin_check, dim3((ntot + 255) / 256), dim3(256), 0, s, (const double*)x,
                       (const double*)c->skin_xref, ntot, half_skin2, every, gate);
    hipLaunchKernelGGL(k_nl_bin, dim3((ntot + 255) / 256), dim3(256), 0, s, (const double*)x, c->skin_frame, 1, ntot,
                       c->cell_of, c->cell_count, c->flags_dev, x, images, (const int32_t*)gate);
    hipLaunchKernelGGL(k_nl_scan, dim3(1), dim3(1024), 0, s, c->cell_count, c->cell_start, c->cell_fill,
                       c->skin_ncells, (const int32_t*)gate);
    hipLaunchKernelGGL(k_nl_scatter, dim3((ntot + 255) / 256), dim3(256), 0, s, c->cell_of, c->cell_start,
                       c->cell_fill, c->cell_atoms, ntot, (const int32_t*)gate);
  }
  skin_build_kernels(c, x, types, ntot, gate, rebuilds, s);
}

void launch_nl_skin_format(dp_ctx* c, const double* x, const int32_t* types, int32_t ntot, int32_t* nlist,
                           int32_t* overflow, hipStream_t s) {
  if (ntot <= 0) return;
  SearchArgs A = search_args(c, x, types, ntot, 1, nlist, c->ovf_ctr);
  SkinArgs S = skin_args(c);
  S.gate = c->skin_gate;
  const dim3 grid((ntot + kSearchWaves - 1) / kSearchWaves), block(64 * kSearchWaves);
  if (A.nm <= kKeepCapSmall) hipLaunchKernelGGL(k_nl_skin_format<kKeepCapSmall>, grid, block, 0, s, A, S);
  else hipLaunchKernelGGL(k_nl_skin_format<kCandCap>, grid, block, 0, s, A, S);
  const int64_t q = (int64_t)ntot * A.nm;
  hipLaunchKernelGGL(k_nl_skin_revmap, dim3((unsigned)((q + 255) / 256)), dim3(256), 0, s, nlist, S, c->rev, ntot,
                     A.nm, c->ovf_ctr, overflow, c->skin_gate);
}

}  // namespace dpse

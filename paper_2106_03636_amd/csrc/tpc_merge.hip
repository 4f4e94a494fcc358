// Merging of track segments across sector boundaries: the segments the
// tracker found in neighbouring sectors (or split inside one) joined where
// one continues the other.  The paper's synchronous processing needs full
// tracking (§2.1) and does not describe this step; the operation is stated
// with tpc_merge_tracks in include/tpc_track.h.
//
// Launches on the caller's stream:
//   k_mg_init   status, counters, per-track outputs and best-match keys;
//   k_mg_rows   per track: first and last hit row; per (unit, z' cell)
//               counts of the refitted segments that start after row 0
//               (only those can continue another); cells are at least
//               dz_max wide, so a z' window meets at most three;
//   k_mg_scan   one block: bin offsets;
//   k_mg_fill   those segments filed by (unit, z' cell);
//   k_mg_sort   one wave per cell: its segments sorted by first row (bitonic
//               in LDS up to SORT_MAX; larger cells by one lane), with their
//               inner z', y, x and first row written in that order as one
//               16-byte record each;
//   k_mg_pairs  a wave takes 8 to 64 consecutive segments a (scan_unit): a
//               lane each, their outer states are turned into the frame of
//               every unit on their side within max_dalpha (parameters, FP64)
//               and the segments starting 1 .. max_gap rows after a's last
//               row are found in the cells a's z' window meets; then, one
//               segment after the other, the wave reads its candidates'
//               records 64 at a time and passes over those that fail the z'
//               or the y window by more than FP32 can err; what is left gets
//               the exact test, z' window and y carried along the helix in
//               FP64, a lane each; pairs that pass are buffered in LDS, and
//               one atomic per block reserves their list ranges;
//   k_mg_chi2   one lane per pair: the turn with its Jacobian, the helix
//               transport with its Jacobian, both covariances summed, chi2
//               by Cholesky (FP64); candidates take the least chi2 per
//               segment both ways (64-bit atomic minima on the chi2's bits:
//               non-negative doubles order like their bit patterns);
//   k_mg_pick   per candidate at its segment's least chi2: the least index;
//   k_mg_link   per segment: linked when its best outward match takes it as
//               its best inward match.
// FP64 with contraction off, so the decisions follow the exact arithmetic to
// about 1e-15 relative.

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "tpc_track.h"

namespace {

constexpr int TPB = 256;
constexpr int SCAN_T = 1024;
constexpr int SORT_MAX = 1024;  // bins sorted in LDS up to this size
constexpr int MAX_BLOCKS = 4096;
constexpr double KAPPA = 0.00299792458;
constexpr double TWO_PI = 6.283185307179586476925286766559;
constexpr unsigned long long NONE64 = ~0ull;

// a filed segment as the scan reads it
struct __align__(16) Filed {
  float z, y, x;  // inner z', y and x
  int32_t fr;     // first row
};
// and as the chi2 of a pair reads it: its inner state, unit and track index
struct __align__(16) Inner {
  float p[5], x;
  int32_t unit, b;
  float c[15], pad;
};
static_assert(sizeof(Inner) == 96, "six 16-byte loads");

struct MgArgs {
  // clusters, geometry
  const uint16_t *row;
  int64_t n_clusters;
  int32_t n_rows;
  // tracks
  const int32_t *trk_status, *n_hits, *first_hit, *hits, *unit;
  const int64_t *trk_counts;
  int64_t cap_tracks, cap_hits;
  // refit
  const float *p_in, *c_in, *x_in, *p_out, *c_out, *x_out;
  const uint8_t *ok;
  const int32_t *rf_status;
  // units
  const float *alpha;
  const int32_t *side;
  int32_t n_units;
  // parameters
  double k, smx, max_dalpha, dz_max, dy_max, chi2_max;
  int32_t max_gap;
  int32_t nzc;       // z' cells per unit
  double zlo, cw;    // first cell's lower edge, cell width
  int64_t cap_pairs;
  // outputs
  int32_t *next, *prev;
  double *link_chi2;
  int32_t *status;
  // workspace
  int32_t *bin;  // [nbins + 1] counts, then offsets
  int32_t *rank;  // place of each filed segment in its cell
  int32_t *idx;
  Filed *filed;   // the filed segments, in scan order
  Inner *inner;   // their inner states, in the same order
  int32_t *frs;    // their first rows, in filing order (the sort's key), then in scan order
  int32_t *rows;  // first row | last row << 16
  unsigned long long *ob_chi, *ib_chi;
  int32_t *ob_idx, *ib_idx;
  int2 *pairs;
  double *pair_chi;
  unsigned long long *ctr;  // pairs, candidates, links (the output counts)
};

__device__ __forceinline__ int64_t n_tracks(const MgArgs &A) {
  const int64_t T = A.trk_counts[0];
  return T < A.cap_tracks ? T : A.cap_tracks;
}
__device__ __forceinline__ int64_t n_track_hits(const MgArgs &A) {
  const int64_t H = A.trk_counts[1];
  return H < A.cap_hits ? H : A.cap_hits;
}

// ---- FP64 track model --------------------------------------------------------

// asin(u)/u and (d/du asin(u)/u) / u, by their series below u = 1e-3
__device__ double asin_over(double u) {
#pragma clang fp contract(off)
  return u < 1e-3 ? 1.0 + u * u / 6.0 : asin(u) / u;
}
__device__ double asin_over_d(double u) {
#pragma clang fp contract(off)
  return u < 1e-3 ? 1.0 / 3.0 + 0.3 * u * u : (u / sqrt(1.0 - u * u) - asin(u)) / (u * u * u);
}

// The state (y, z, sin(phi), tan(lambda), q/pT) at plane x turned by d into
// another sector's frame: the point turns, so does the direction; the new
// state lives at the turned point's x.  J (optional): the Jacobian of the
// new state at the new plane against the old one (a shift of the track along
// the old y, taken back to the new plane along the track; a turn of the
// direction).  False when the direction reaches |sin| >= smx or cos <= 0.
// cd, sd: cosine and sine of the turn.
__device__ __forceinline__ bool turn(const double p[5], double x, double cd, double sd, double k, double smx, double q[5],
                                     double &xq, double *J) {
#pragma clang fp contract(off)
  const double s = p[2];
  if (!(fabs(s) < 1.0)) return false;
  const double c = sqrt(1.0 - s * s);
  const double s2 = s * cd - c * sd, c2 = c * cd + s * sd;
  if (!(c2 > 0.0) || !(fabs(s2) < smx)) return false;
  xq = x * cd + p[0] * sd;
  q[0] = -x * sd + p[0] * cd;
  q[1] = p[1];
  q[2] = s2;
  q[3] = p[3];
  q[4] = p[4];
  if (J) {
#pragma unroll
    for (int i = 0; i < 25; ++i) J[i] = (i % 6 == 0) ? 1.0 : 0.0;
    J[0] = c / c2;
    J[5] = -sd * p[3] / c2;
    J[10] = -k * p[4] * sd;
    J[12] = c2 / c;
  }
  return true;
}

// Helix transport of the parameters from x1 to x2: sin(phi) grows by C dx,
// y by dx (sin1 + sin2) / (cos1 + cos2), z by tan(lambda) times the arc
// length sign(dx) L asin(u)/u (L the chord, u = |C| L / 2).  F (optional):
// its Jacobian.  False when |sin(phi)| reaches smx at either end or u >= 1.
__device__ __forceinline__ bool carry(const double p[5], double x1, double x2, double k, double smx, double q[5], double *F) {
#pragma clang fp contract(off)
  const double dx = x2 - x1;
  const double C = k * p[4];
  const double s1 = p[2], s2 = s1 + C * dx;
  if (!(fabs(s1) < smx) || !(fabs(s2) < smx)) return false;
  const double c1 = sqrt(1.0 - s1 * s1), c2 = sqrt(1.0 - s2 * s2);
  const double D = c1 + c2, N = s1 + s2;
  const double dy = dx * N / D;
  const double L = sqrt(dx * dx + dy * dy);
  const double u = fabs(C) * L * 0.5;
  if (!(u < 1.0)) return false;
  const double sg = dx < 0 ? -1.0 : 1.0;
  const double fu = asin_over(u);
  const double sT = sg * L * fu;
  q[0] = p[0] + dy;
  q[1] = p[1] + p[3] * sT;
  q[2] = s2;
  q[3] = p[3];
  q[4] = p[4];
  if (F) {
#pragma unroll
    for (int i = 0; i < 25; ++i) F[i] = (i % 6 == 0) ? 1.0 : 0.0;
    const double a = dx * ((2.0 * D + N * (s1 / c1 + s2 / c2)) / (D * D));
    const double b = dx * (k * dx * (D + N * s2 / c2) / (D * D));
    const double g = asin_over_d(u);
    const double dsdy = L > 0 ? sg * (dy / L) * (fu + u * u * g) : 0.0;
    const double dsdC = sg * C * L * L * L * g * 0.25;
    F[2] = a;
    F[4] = b;
    F[7] = p[3] * dsdy * a;
    F[8] = sT;
    F[9] = p[3] * (dsdy * b + dsdC * k);
    F[14] = k * dx;
  }
  return true;
}

// y of the parameters carried from x1 to x2 along the helix (the transport
// above without the arc length); false where the transport fails.
__device__ bool carry_y(const double p[5], double x1, double x2, double k, double smx, double &y) {
#pragma clang fp contract(off)
  const double dx = x2 - x1;
  const double C = k * p[4];
  const double s1 = p[2], s2 = s1 + C * dx;
  if (!(fabs(s1) < smx) || !(fabs(s2) < smx)) return false;
  const double c1 = sqrt(1.0 - s1 * s1), c2 = sqrt(1.0 - s2 * s2);
  const double dy = dx * (s1 + s2) / (c1 + c2);
  const double L = sqrt(dx * dx + dy * dy);
  if (!(fabs(C) * L * 0.5 < 1.0)) return false;
  y = p[0] + dy;
  return true;
}

// C <- M C M^T (5x5, full products)
__device__ __forceinline__ void sandwich(const double M[25], double C[25]) {
#pragma clang fp contract(off)
  double T[25];
#pragma unroll
  for (int i = 0; i < 5; ++i)
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      double s = 0.0;
#pragma unroll
      for (int l = 0; l < 5; ++l) s += M[i * 5 + l] * C[l * 5 + j];
      T[i * 5 + j] = s;
    }
#pragma unroll
  for (int i = 0; i < 5; ++i)
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      double s = 0.0;
#pragma unroll
      for (int l = 0; l < 5; ++l) s += T[i * 5 + l] * M[j * 5 + l];
      C[i * 5 + j] = s;
    }
}

__device__ __forceinline__ void load_cov(const float *c15, double C[25]) {
  int m = 0;
#pragma unroll
  for (int i = 0; i < 5; ++i)
#pragma unroll
    for (int j = 0; j <= i; ++j) C[i * 5 + j] = C[j * 5 + i] = double(c15[m++]);
}

// r^T S^-1 r by Cholesky; -1 when S is not positive definite
__device__ __forceinline__ double chi2_solve(const double S[25], const double r[5]) {
#pragma clang fp contract(off)
  double L[25];
#pragma unroll
  for (int i = 0; i < 25; ++i) L[i] = 0.0;
#pragma unroll
  for (int i = 0; i < 5; ++i)
#pragma unroll
    for (int j = 0; j <= i; ++j) {
      double v = S[i * 5 + j];
#pragma unroll
      for (int m = 0; m < j; ++m) v -= L[i * 5 + m] * L[j * 5 + m];
      if (i == j) {
        if (!(v > 0.0)) return -1.0;
        L[i * 5 + i] = sqrt(v);
      } else {
        L[i * 5 + j] = v / L[j * 5 + j];
      }
    }
  double w[5], q = 0.0;
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    double v = r[i];
#pragma unroll
    for (int m = 0; m < i; ++m) v -= L[i * 5 + m] * w[m];
    w[i] = v / L[i * 5 + i];
    q += w[i] * w[i];
  }
  return q;
}

__device__ __forceinline__ int zcell(const MgArgs &A, double z) {
  const double c = floor((z - A.zlo) / A.cw);
  return c < 0.0 ? 0 : (c >= double(A.nzc) ? A.nzc - 1 : int(c));
}

__device__ __forceinline__ double turn_angle(const MgArgs &A, int ua, int w) {
  return remainder(double(A.alpha[w]) - double(A.alpha[ua]), TWO_PI);
}

// ---- kernels -------------------------------------------------------------------

__global__ void __launch_bounds__(TPB) k_mg_init(MgArgs A) {
  const int64_t T = n_tracks(A);
  const int64_t nb = int64_t(A.n_units) * A.nzc + 1;
  const int64_t i0 = int64_t(blockIdx.x) * TPB + threadIdx.x, st = int64_t(gridDim.x) * TPB;
  if (i0 == 0) {
    *A.status = *A.trk_status != TPC_OK ? *A.trk_status : *A.rf_status;
    A.ctr[0] = A.ctr[1] = A.ctr[2] = 0ull;
  }
  for (int64_t i = i0; i < nb; i += st) A.bin[i] = 0;
  for (int64_t t = i0; t < T; t += st) {
    A.next[t] = A.prev[t] = -1;
    A.link_chi2[t] = 0.0;
    A.ob_chi[t] = A.ib_chi[t] = NONE64;
    A.ob_idx[t] = A.ib_idx[t] = INT32_MAX;
  }
}

__global__ void __launch_bounds__(TPB) k_mg_rows(MgArgs A) {
  if (*A.status != TPC_OK) return;
  const int64_t T = n_tracks(A), H = n_track_hits(A);
  bool bad = false;
  for (int64_t t = int64_t(blockIdx.x) * TPB + threadIdx.x; t < T; t += int64_t(gridDim.x) * TPB) {
    const int n = A.n_hits[t], f = A.first_hit[t], u = A.unit[t];
    if (n < 0 || f < 0 || int64_t(f) + n > H) {  // the track's hits lie outside the hit list
      bad = true;
      continue;
    }
    int fr = 0, lr = 0;
    if (n > 0) {
      const int32_t h0 = A.hits[f], h1 = A.hits[f + n - 1];
      if (h0 < 0 || h0 >= A.n_clusters || h1 < 0 || h1 >= A.n_clusters) {
        bad = true;
        continue;
      }
      fr = A.row[h0];
      lr = A.row[h1];
    }
    if (u < 0 || u >= A.n_units || (A.side[u] != 1 && A.side[u] != -1) || fr >= A.n_rows || lr >= A.n_rows) {
      bad = true;
      continue;
    }
    A.rows[t] = fr | (lr << 16);
    // the rank in the cell is the segment's place there: k_mg_fill needs no second counter
    // (6 us against 32 with an atomic there too)
    if (A.ok[t] && fr > 0) A.rank[t] = atomicAdd(&A.bin[u * A.nzc + zcell(A, double(A.p_in[t * 5 + 1]))], 1);
  }
  if (bad) *A.status = TPC_E_INVALID;
}

// exclusive scan of the bin counts (one block): each thread takes PER
// consecutive counts, so one block scan covers 1024 * PER of them (9.3 k
// counts: 7 us; with one count a thread and turn 20)
__global__ void __launch_bounds__(SCAN_T) k_mg_scan(MgArgs A) {
  constexpr int PER = 12;
  __shared__ int32_t wsum[2][SCAN_T / 64];
  if (*A.status != TPC_OK) return;
  const int64_t nb = int64_t(A.n_units) * A.nzc;
  const int lane = __lane_id(), wave = threadIdx.x >> 6;
  int32_t carry = 0;
  int flip = 0;
  for (int64_t b0 = 0; b0 <= nb; b0 += SCAN_T * PER, flip ^= 1) {
    const int64_t i0 = b0 + int64_t(threadIdx.x) * PER;
    int32_t v[PER], sum = 0;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      v[e] = i0 + e < nb ? A.bin[i0 + e] : 0;
      sum += v[e];
    }
    int32_t inc = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int32_t x = __shfl_up(inc, o, 64);
      if (lane >= o) inc += x;
    }
    if (lane == 63) wsum[flip][wave] = inc;
    __syncthreads();
    int32_t ex = carry + inc - sum;
#pragma unroll
    for (int w = 0; w < SCAN_T / 64; ++w) {
      const int32_t t = wsum[flip][w];
      ex += w < wave ? t : 0;
      carry += t;
    }
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      if (i0 + e <= nb) A.bin[i0 + e] = ex;
      ex += v[e];
    }
  }
}

__global__ void __launch_bounds__(TPB) k_mg_fill(MgArgs A) {
  if (*A.status != TPC_OK) return;
  const int64_t T = n_tracks(A);
  for (int64_t t = int64_t(blockIdx.x) * TPB + threadIdx.x; t < T; t += int64_t(gridDim.x) * TPB) {
    const int fr = A.rows[t] & 0xFFFF;
    if (!A.ok[t] || fr == 0) continue;
    const int pos = A.bin[A.unit[t] * A.nzc + zcell(A, double(A.p_in[t * 5 + 1]))] + A.rank[t];
    A.idx[pos] = int32_t(t);
    A.frs[pos] = fr;
  }
}

// Adds the block's total of the threads' v to a counter with one atomic per
// block (the counter is shared by the whole grid: an atomic per wave on the
// one address serialized thousands of them).  Called by every thread of the
// block, after its loop.
__device__ __forceinline__ void block_count(unsigned long long &counter, unsigned v) {
  __shared__ unsigned s;
  if (threadIdx.x == 0) s = 0u;
  __syncthreads();
  if (v) atomicAdd(&s, v);
  __syncthreads();
  if (threadIdx.x == 0 && s) atomicAdd(&counter, (unsigned long long)s);
}

__device__ __forceinline__ void file_entry(const MgArgs &A, int32_t s, int32_t b, int32_t fr) {
  A.idx[s] = b;
  Filed f;
  f.z = A.p_in[int64_t(b) * 5 + 1];
  f.y = A.p_in[int64_t(b) * 5];
  f.x = A.x_in[b];
  f.fr = fr;
  A.filed[s] = f;
  Inner r;
  for (int j = 0; j < 5; ++j) r.p[j] = A.p_in[int64_t(b) * 5 + j];
  r.x = f.x;
  r.unit = A.unit[b];
  r.b = b;
  for (int j = 0; j < 15; ++j) r.c[j] = A.c_in[int64_t(b) * 15 + j];
  r.pad = 0.f;
  A.inner[s] = r;
}

__global__ void __launch_bounds__(64) k_mg_sort(MgArgs A) {
  __shared__ unsigned long long key[SORT_MAX];
  if (*A.status != TPC_OK) return;
  const int64_t nb = int64_t(A.n_units) * A.nzc;
  for (int64_t c = blockIdx.x; c < nb; c += gridDim.x) {  // block-uniform
    const int32_t s0 = A.bin[c], n = A.bin[c + 1] - s0;
    if (n == 0) continue;
    if (n > SORT_MAX) {  // rare: one lane, insertion sort by (first row, index) in place
      if (threadIdx.x == 0) {
        for (int32_t i = 1; i < n; ++i) {
          const int32_t b = A.idx[s0 + i], fr = A.frs[s0 + i];
          int32_t j = i - 1;
          for (; j >= 0 && (A.frs[s0 + j] > fr || (A.frs[s0 + j] == fr && A.idx[s0 + j] > b)); --j) {
            A.idx[s0 + j + 1] = A.idx[s0 + j];
            A.frs[s0 + j + 1] = A.frs[s0 + j];
          }
          A.idx[s0 + j + 1] = b;
          A.frs[s0 + j + 1] = fr;
        }
        for (int32_t i = 0; i < n; ++i) file_entry(A, s0 + i, A.idx[s0 + i], A.frs[s0 + i]);
      }
      continue;
    }
    int np = 1;
    while (np < n) np <<= 1;
    for (int i = threadIdx.x; i < np; i += 64)
      key[i] = i < n ? (uint64_t(uint32_t(A.frs[s0 + i])) << 32) | uint32_t(A.idx[s0 + i]) : ~0ull;
    __syncthreads();
    for (int k = 2; k <= np; k <<= 1)
      for (int j = k >> 1; j > 0; j >>= 1) {
        for (int i = threadIdx.x; i < np; i += 64) {
          const int l = i ^ j;
          if (l > i) {
            const unsigned long long x = key[i], y = key[l];
            if ((x > y) == ((i & k) == 0)) {
              key[i] = y;
              key[l] = x;
            }
          }
        }
        __syncthreads();
      }
    for (int i = threadIdx.x; i < n; i += 64) {
      file_entry(A, s0 + i, int32_t(uint32_t(key[i])), int32_t(key[i] >> 32));
      A.frs[s0 + i] = int32_t(key[i] >> 32);
    }
    __syncthreads();
  }
}

constexpr int WAVES = TPB / 64;
constexpr int CELLS = 3;       // z' cells a window meets at most (cells are at least dz_max wide)
constexpr int NEAR_BUF = 128;  // candidates a wave keeps for the exact test, which takes 64 at a time
constexpr int PAIR_BUF = 512;  // pairs a wave keeps before it reserves list space
constexpr int SEGS_MIN = 8, SEGS_MAX = 64;  // segments a wave of the scan takes

// a wave's part of the scan's LDS
struct WaveScan {
  double y[64], x[64], s[64], q[64];  // its segments' outer states in the unit at hand, for the exact test
  float z[64];
  int32_t near[NEAR_BUF], pair[PAIR_BUF];            // filed slots ...
  uint8_t near_seg[NEAR_BUF], pair_seg[PAIR_BUF];  // ... and the segments (lanes) they are candidates of
};

// what one lane wrote to its wave's LDS is there for the others
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
__device__ __forceinline__ int lanes_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0));
}
__device__ __forceinline__ int32_t lane_int(int32_t v, int lane) { return __builtin_amdgcn_readlane(v, lane); }
__device__ __forceinline__ float lane_float(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
__device__ __forceinline__ double lane_double(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane(int(b), lane), hi = __builtin_amdgcn_readlane(int(b >> 32), lane);
  return __longlong_as_double((long long)((unsigned long long)unsigned(hi) << 32 | unsigned(lo)));
}

// n buffered pairs of the wave whose first segment is a0, written to the list
// from base on (past cap_pairs they are only counted)
__device__ __forceinline__ void write_pairs(const MgArgs &A, const WaveScan &L, int64_t a0, int n, unsigned long long base) {
  for (int i = __lane_id(); i < n; i += 64)
    if (base + i < (unsigned long long)A.cap_pairs) A.pairs[base + i] = make_int2(int32_t(a0) + L.pair_seg[i], L.pair[i]);
}

// A segment's outer state in one unit's frame, rounded for the first look at
// its candidates.
struct Reach {
  float z, y, x, s, c, C;
  int32_t plain;  // the first look's bound holds (|sin(phi)| well below 1)

  // Whether the record cannot pass the z' and y windows: their test in FP32,
  // with margins above its error.  The state's x and y, up to 8192 cm, round by
  // 5e-4 cm, z' differences by as much; for |C| < 0.05 / cm that puts sin(phi) off by less
  // than 3e-5 and, where it is below 0.96 at both ends (tan < 3.5), the
  // carried y by less than 3e-3 cm and 6e-4 dx.  Anything else, NaN too, is
  // left to the exact test.  (Most segments of low-pT particles end where
  // they turn back: the transport fails for most of their candidates.)
  __device__ __forceinline__ bool misses(const Filed &f, float dz, float dy, float smx) const {
    const float dx = f.x - x, s2 = s + C * dx;
    const float c2 = __builtin_amdgcn_sqrtf(fmaxf(0.f, 1.f - s2 * s2));
    const float off = f.y - y - dx * (s + s2) * __builtin_amdgcn_rcpf(c + c2);
    return fabsf(f.z - z) > dz ||
           (plain && (fabsf(s2) > smx || (fabsf(s2) < 0.96f && fabsf(off) > dy + 1e-3f * fabsf(dx))));
  }
};

// The exact test of the wave's kept candidates first .. first + 63 (those
// below n), a lane each; those that pass go to the wave's pairs.
__device__ __forceinline__ void settle(const MgArgs &A, WaveScan &L, int64_t a0, int first, int n, int &n_pair) {
  const int lane = __lane_id();
  wave_sync();
  int32_t s = 0;
  int seg = 0;
  bool pass = false;
  if (first + lane < n) {
    s = L.near[first + lane];
    seg = L.near_seg[first + lane];
    const Filed f = A.filed[s];
    const double p[5] = {L.y[seg], 0.0, L.s[seg], 0.0, L.q[seg]};
    double y;
    pass = fabs(double(f.z) - double(L.z[seg])) <= A.dz_max && carry_y(p, L.x[seg], double(f.x), A.k, A.smx, y) &&
           fabs(double(f.y) - y) <= A.dy_max;
  }
  const uint64_t m = __ballot(pass);
  const int more = __popcll(m);
  if (n_pair + more > PAIR_BUF) {
    unsigned long long base = 0;
    if (lane == 0) base = atomicAdd(&A.ctr[0], (unsigned long long)n_pair);
    write_pairs(A, L, a0, n_pair, __shfl(base, 0, 64));
    wave_sync();
    n_pair = 0;
  }
  if (pass) {
    const int i = n_pair + lanes_below(m);
    L.pair[i] = s;  // the filed slot; k_mg_chi2 puts the track index in its place
    L.pair_seg[i] = uint8_t(seg);
  }
  n_pair += more;
  wave_sync();
}

// The candidates, in unit w, of the segments of the lanes with `mine` (a0 is
// lane 0's): each such lane turns its outer state (pa, xa) into the unit's
// frame by an angle of cosine cd and sine sd (same: it is its own unit) and
// finds the ranges of the records to check; then the wave takes the segments
// one after the other, 64 records at a time.
__device__ __forceinline__ void scan_unit(const MgArgs &A, WaveScan &L, int64_t a0, bool mine, int lr, const double pa[5],
                                          double xa, int w, bool same, double cd, double sd, int &n_pair) {
  const int lane = __lane_id();
  const int r1 = min(lr + A.max_gap, A.n_rows - 1);
  const double za = pa[1];
  Reach r = {};
  if (mine) {
    double q[5], xq = xa;
    if (same) {
      for (int i = 0; i < 5; ++i) q[i] = pa[i];
    } else {
      mine = turn(pa, xa, cd, sd, A.k, A.smx, q, xq, nullptr);
    }
    if (mine) {
      L.y[lane] = q[0];
      L.x[lane] = xq;
      L.s[lane] = q[2];
      L.q[lane] = q[4];
      L.z[lane] = float(za);  // exact: it came as a float
      r.z = float(za);
      r.y = float(q[0]);
      r.x = float(xq);
      r.s = float(q[2]);
      r.C = float(A.k * q[4]);
      r.c = __builtin_amdgcn_sqrtf(fmaxf(0.f, 1.f - r.s * r.s));
      // |x|, |y| and |C| within their limits, by one comparison
      r.plain = fabsf(r.s) < 0.96f && fmaxf(fmaxf(fabsf(r.x), fabsf(r.y)), fabsf(r.C) * (8192.f / 0.05f)) < 8192.f;
    }
  }
  const float dz = float(A.dz_max) * 1.000001f + 2e-3f, dy = float(A.dy_max) * 1.000001f + 6e-3f, smx = float(A.smx) + 1e-4f;
  const int c0 = zcell(A, za - A.dz_max), c1 = zcell(A, za + A.dz_max);
  int n_near = 0;
  for (int cb = c0; __ballot(mine && cb <= c1); cb += CELLS) {  // once, but for a rounded cell width
    // Each cell is sorted by first row.  The bounds of the segments starting in
    // rows lr+1 .. r1 are searched for in all of them together (six searches,
    // one load each per step).
    int32_t lo[CELLS], hi[CELLS], le[CELLS], he[CELLS], span = 0;
#pragma unroll
    for (int c = 0; c < CELLS; ++c) {
      const bool on = mine && cb + c <= c1;
      const int64_t cell = int64_t(w) * A.nzc + (on ? cb + c : 0);
      const int32_t s0 = A.bin[cell], s1 = on ? A.bin[cell + 1] : s0;
      lo[c] = hi[c] = s0;  // [lo, le): the first row above lr is sought in it; [hi, he): the first above r1
      le[c] = he[c] = s1;
      span = max(span, s1 - s0);
    }
    for (; span > 0; span >>= 1) {
#pragma unroll
      for (int c = 0; c < CELLS; ++c) {
        const int32_t m = (lo[c] + le[c]) >> 1, n = (hi[c] + he[c]) >> 1;
        const bool vm = lo[c] < le[c], vn = hi[c] < he[c];
        const int32_t fm = vm ? A.frs[m] : 0, fn = vn ? A.frs[n] : 0;
        if (vm) {
          if (fm <= lr) lo[c] = m + 1; else le[c] = m;
        }
        if (vn) {
          if (fn <= r1) hi[c] = n + 1; else he[c] = n;
        }
      }
    }
    // their records as one list: record t is filed in slot t + a0_, a1 or a2
    const int32_t e0 = hi[0] - lo[0], e1 = e0 + hi[1] - lo[1], tot = e1 + hi[2] - lo[2];
    const int32_t b0 = lo[0], b1 = lo[1] - e0, b2 = lo[2] - e1;
    for (uint64_t todo = __ballot(tot > 0); todo; todo &= todo - 1) {
      const int i = __ffsll((unsigned long long)todo) - 1;
      const Reach u = {lane_float(r.z, i), lane_float(r.y, i), lane_float(r.x, i), lane_float(r.s, i),
                       lane_float(r.c, i), lane_float(r.C, i), lane_int(r.plain, i)};
      const int32_t n = lane_int(tot, i), n0 = lane_int(e0, i), n1 = lane_int(e1, i);
      const int32_t s0 = lane_int(b0, i), s1 = lane_int(b1, i), s2 = lane_int(b2, i);
      for (int32_t t0 = 0; t0 < n; t0 += 64) {
        const int32_t t = min(t0 + lane, n - 1), s = t + (t < n0 ? s0 : t < n1 ? s1 : s2);
        const bool keep = !u.misses(A.filed[s], dz, dy, smx) && t0 + lane < n;
        const uint64_t m = __ballot(keep);
        if (keep) {
          const int k = n_near + lanes_below(m);
          L.near[k] = s;
          L.near_seg[k] = uint8_t(i);
        }
        n_near += __popcll(m);
        if (n_near >= 64) {
          n_near -= 64;
          settle(A, L, a0, n_near, n_near + 64, n_pair);
        }
      }
    }
  }
  if (n_near) settle(A, L, a0, 0, n_near, n_pair);
}

// The candidates of a wave's segments (a lane each; on: those that look for
// any).  The units that one of the lanes' units may continue in are found by
// the wave's lanes together, a unit each with its angle, cosine and sine: the
// FP64 remainder and the sincos are then paid once for a wave whose segments
// share their unit, and nearly all waves do.
__device__ __forceinline__ void scan_wave(const MgArgs &A, WaveScan &L, int64_t a0, bool on, int lr, int &n_pair) {
  const int lane = __lane_id();
  double pa[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, xa = 0.0;
  int ua = -1;
  if (on) {
    ua = A.unit[a0 + lane];
    for (int i = 0; i < 5; ++i) pa[i] = double(A.p_out[(a0 + lane) * 5 + i]);
    xa = double(A.x_out[a0 + lane]);
  }
  uint64_t todo = __ballot(on);
  while (todo) {
    const int u = lane_int(ua, __ffsll((unsigned long long)todo) - 1);
    const bool mine = on && ua == u;
    todo &= ~__ballot(mine);
    const int side = A.side[u];
    for (int w0 = 0; w0 < A.n_units; w0 += 64) {
      const int w = w0 + lane;
      double cd = 1.0, sd = 0.0;
      bool reach = false;
      if (w < A.n_units && A.side[w] == side) {
        const double d = turn_angle(A, u, w);
        reach = fabs(d) <= A.max_dalpha;
        if (reach) {
          cd = cos(d);
          sd = sin(d);
        }
      }
      for (uint64_t m = __ballot(reach); m; m &= m - 1) {
        const int k = __ffsll((unsigned long long)m) - 1;
        scan_unit(A, L, a0, mine, lr, pa, xa, w0 + k, w0 + k == u, lane_double(cd, k), lane_double(sd, k), n_pair);
      }
    }
  }
}

// What bounds it: FP32 issue (95 M wave instructions for 237 k segments that
// look on and 56 M records: 0.6 of the time) and the records' latency, which
// six waves a SIMD cover most of.  265 us; 667 with a lane per segment that
// tested each of its candidates in FP64: 64 lanes then read 64 far records
// with every load.
__global__ void __launch_bounds__(TPB, 6) k_mg_pairs(MgArgs A) {
  __shared__ WaveScan scans[WAVES];
  __shared__ int32_t n_wave[WAVES];
  __shared__ unsigned long long base;
  if (*A.status != TPC_OK) return;
  const int64_t T = n_tracks(A);
  const int lane = __lane_id(), wave = threadIdx.x >> 6;
  WaveScan &L = scans[wave];
  int64_t segs = SEGS_MIN;  // small batches are spread over the chip's waves
  while (segs < SEGS_MAX && segs * WAVES * gridDim.x < T) segs *= 2;
  for (int64_t b0 = blockIdx.x * segs * WAVES; b0 < T; b0 += gridDim.x * segs * WAVES) {  // block-uniform
    const int64_t a0 = b0 + wave * segs, a = a0 + lane;
    const bool in = lane < segs && a < T;
    const int lr = in ? A.rows[a] >> 16 : 0;
    int n_pair = 0;
    scan_wave(A, L, a0, in && A.ok[a] && lr + 1 < A.n_rows, lr, n_pair);
    // the block's buffered pairs: one atomic reserves all their ranges (an
    // atomic per wave on the one counter would serialize them)
    if (lane == 0) n_wave[wave] = n_pair;
    __syncthreads();
    int32_t before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      before += w < wave ? n_wave[w] : 0;
      total += n_wave[w];
    }
    if (threadIdx.x == 0 && total) base = atomicAdd(&A.ctr[0], (unsigned long long)total);
    __syncthreads();
    if (total) write_pairs(A, L, a0, n_pair, base + (unsigned long long)before);
    __syncthreads();
  }
}

__global__ void __launch_bounds__(TPB) k_mg_chi2(MgArgs A) {
  if (*A.status != TPC_OK) return;
  const unsigned long long np = A.ctr[0];
  if (np > (unsigned long long)A.cap_pairs) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *A.status = TPC_E_CAPACITY;
    return;
  }
  unsigned n_cand = 0;
  for (int64_t i = int64_t(blockIdx.x) * TPB + threadIdx.x; i < int64_t(np); i += int64_t(gridDim.x) * TPB) {
    const int2 pr = A.pairs[i];
    const int a = pr.x;
    const Inner bi = A.inner[pr.y];  // b's inner state, filed next to the other candidates of a's cells
    const int b = bi.b, ub = bi.unit;
    A.pairs[i].y = b;                // k_mg_pick reads track indices
    const int ua = A.unit[a];
    double pa[5], C[25], q[5], c[5];
    for (int j = 0; j < 5; ++j) pa[j] = double(A.p_out[a * 5 + j]);
    load_cov(A.c_out + int64_t(a) * 15, C);
    double xq = double(A.x_out[a]);
    double chi = -1.0;
    bool ok = true;
    if (ua != ub) {
      const double d = turn_angle(A, ua, ub);
      double J[25];
      ok = turn(pa, double(A.x_out[a]), cos(d), sin(d), A.k, A.smx, q, xq, J);
      if (ok) sandwich(J, C);
    } else {
      for (int j = 0; j < 5; ++j) q[j] = pa[j];
    }
    double F[25];
    if (ok) ok = carry(q, xq, double(bi.x), A.k, A.smx, c, F);
    if (ok) {
#pragma clang fp contract(off)
      sandwich(F, C);
      double Cb[25], r[5];
      load_cov(bi.c, Cb);
      for (int j = 0; j < 25; ++j) C[j] += Cb[j];
      for (int j = 0; j < 5; ++j) r[j] = double(bi.p[j]) - c[j];
      chi = chi2_solve(C, r);
    }
    A.pair_chi[i] = chi;
    const bool cand = chi >= 0.0 && chi <= A.chi2_max;
    if (cand) {
      const unsigned long long bits = (unsigned long long)__double_as_longlong(chi);
      atomicMin(&A.ob_chi[a], bits);
      atomicMin(&A.ib_chi[b], bits);
    }
    n_cand += cand;
  }
  block_count(A.ctr[1], n_cand);
}

__global__ void __launch_bounds__(TPB) k_mg_pick(MgArgs A) {
  if (*A.status != TPC_OK) return;
  const int64_t np = int64_t(A.ctr[0]);
  for (int64_t i = int64_t(blockIdx.x) * TPB + threadIdx.x; i < np; i += int64_t(gridDim.x) * TPB) {
    const double chi = A.pair_chi[i];
    if (!(chi >= 0.0 && chi <= A.chi2_max)) continue;
    const unsigned long long bits = (unsigned long long)__double_as_longlong(chi);
    const int2 pr = A.pairs[i];
    if (A.ob_chi[pr.x] == bits) atomicMin(&A.ob_idx[pr.x], pr.y);
    if (A.ib_chi[pr.y] == bits) atomicMin(&A.ib_idx[pr.y], pr.x);
  }
}

__global__ void __launch_bounds__(TPB) k_mg_link(MgArgs A) {
  if (*A.status != TPC_OK) return;
  const int64_t T = n_tracks(A);
  unsigned n_link = 0;
  for (int64_t a = int64_t(blockIdx.x) * TPB + threadIdx.x; a < T; a += int64_t(gridDim.x) * TPB) {
    const int32_t b = A.ob_idx[a];
    const bool link = b != INT32_MAX && A.ib_idx[b] == int32_t(a);
    if (link) {
      A.next[a] = b;
      A.prev[b] = int32_t(a);
      A.link_chi2[a] = __longlong_as_double((long long)A.ob_chi[a]);
    }
    n_link += link;
  }
  block_count(A.ctr[2], n_link);
}

size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

struct Layout {
  size_t bin, idx, filed, inner, frs, rows, ob_chi, ib_chi, ob_idx, ib_idx, pairs, pair_chi, total;
};

Layout layout(int64_t nbins, int64_t cap_tracks, int64_t cap_pairs) {
  Layout L;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    const size_t at = o;
    o += align256(bytes);
    return at;
  };
  L.bin = take(size_t(nbins + 1) * 4);
  L.idx = take(size_t(cap_tracks) * 4);
  L.filed = take(size_t(cap_tracks) * sizeof(Filed));
  L.inner = take(size_t(cap_tracks) * sizeof(Inner));
  L.frs = take(size_t(cap_tracks) * 4);
  L.rows = take(size_t(cap_tracks) * 4);
  L.ob_chi = take(size_t(cap_tracks) * 8);
  L.ib_chi = take(size_t(cap_tracks) * 8);
  L.ob_idx = take(size_t(cap_tracks) * 4);
  L.ib_idx = take(size_t(cap_tracks) * 4);
  L.pairs = take(size_t(cap_pairs) * 8);
  L.pair_chi = take(size_t(cap_pairs) * 8);
  L.total = o;
  return L;
}

// z' cells of the candidate filing: at least dz_max wide where that keeps
// the bins below 2^18 (a window then meets at most three cells), over
// [-8256, 8256) cm (inputs lie within |z'| <= 8192; the rest is clamped).
struct Cells {
  int32_t nzc;
  double zlo, cw;
};
Cells cells(const tpc_merge_params_t *p, int32_t n_units) {
  constexpr double SPAN = 16512.0;
  const int64_t most = (int64_t(1) << 18) / (n_units > 0 ? n_units : 1);
  int64_t nz = p->dz_max > 0.f ? int64_t(SPAN / double(p->dz_max)) : most;
  if (nz > most) nz = most;
  if (nz > 65536) nz = 65536;
  if (nz < 1) nz = 1;
  Cells c;
  c.nzc = int32_t(nz);
  c.zlo = -SPAN / 2;
  c.cw = SPAN / double(nz);
  return c;
}

}  // namespace

extern "C" size_t tpc_merge_workspace_size(int32_t n_units, int32_t n_rows, int64_t cap_tracks,
                                           const tpc_merge_params_t *params) {
  if (!params || n_units < 1 || n_rows < 3 || n_rows > 255 || cap_tracks < 0 || cap_tracks >= (int64_t(1) << 31) ||
      params->cap_pairs < 0 || params->cap_pairs >= (int64_t(1) << 31) || n_units > (1 << 18))
    return 0;
  return layout(int64_t(n_units) * cells(params, n_units).nzc, cap_tracks, params->cap_pairs).total;
}

extern "C" int tpc_merge_tracks(const tpc_clusters_t *clusters, const tpc_geometry_t *geometry,
                                const tpc_field_t *field, const tpc_tracks_t *tracks, const tpc_refit_t *refit,
                                const float *unit_alpha, const int32_t *unit_side, int32_t n_units,
                                const tpc_merge_params_t *params, tpc_merged_t *out, void *workspace,
                                size_t workspace_bytes, void *stream) {
  if (!clusters || !geometry || !field || !tracks || !refit || !params || !out || !unit_alpha || !unit_side)
    return TPC_E_INVALID;
  if (clusters->n < 0 || (clusters->n > 0 && !clusters->row) || !geometry->row_x) return TPC_E_INVALID;
  if (!tracks->n_hits || !tracks->first_hit || !tracks->hits || !tracks->unit || !tracks->counts ||
      !tracks->status || tracks->cap_tracks < 0 || tracks->cap_hits < 0)
    return TPC_E_INVALID;
  if (!refit->params || !refit->cov || !refit->x_ref || !refit->params_out || !refit->cov_out ||
      !refit->x_out || !refit->ok || !refit->status)
    return TPC_E_INVALID;
  if (!out->next || !out->prev || !out->link_chi2 || !out->counts || !out->status) return TPC_E_INVALID;
  if (!(params->max_dalpha >= 0.f) || params->max_gap < 1 || params->max_gap > 255 || !(params->dz_max >= 0.f) ||
      !(params->dy_max >= 0.f) || !(params->chi2_max > 0.f) || !(params->sinphi_max > 0.f) ||
      !(params->sinphi_max < 1.f) || !isfinite(field->bz_tesla))
    return TPC_E_INVALID;
  const size_t need = tpc_merge_workspace_size(n_units, geometry->n_rows, tracks->cap_tracks, params);
  if (need == 0) return TPC_E_INVALID;
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255)) return TPC_E_INVALID;
  if (workspace_bytes < need) return TPC_E_NOMEM;
  MgArgs A;
  A.row = clusters->row;
  A.n_clusters = clusters->n;
  A.n_rows = geometry->n_rows;
  A.trk_status = tracks->status;
  A.n_hits = tracks->n_hits;
  A.first_hit = tracks->first_hit;
  A.hits = tracks->hits;
  A.unit = tracks->unit;
  A.trk_counts = tracks->counts;
  A.cap_tracks = tracks->cap_tracks;
  A.cap_hits = tracks->cap_hits;
  A.p_in = refit->params;
  A.c_in = refit->cov;
  A.x_in = refit->x_ref;
  A.p_out = refit->params_out;
  A.c_out = refit->cov_out;
  A.x_out = refit->x_out;
  A.ok = refit->ok;
  A.rf_status = refit->status;
  A.alpha = unit_alpha;
  A.side = unit_side;
  A.n_units = n_units;
  A.k = double(-float(KAPPA) * field->bz_tesla);  // the tracker's curvature constant, as its fit used it
  A.smx = params->sinphi_max;
  A.max_dalpha = params->max_dalpha;
  A.dz_max = params->dz_max;
  A.dy_max = params->dy_max;
  A.chi2_max = params->chi2_max;
  A.max_gap = params->max_gap;
  A.cap_pairs = params->cap_pairs;
  A.next = out->next;
  A.prev = out->prev;
  A.link_chi2 = out->link_chi2;
  A.status = out->status;
  const Cells cz = cells(params, n_units);
  A.nzc = cz.nzc;
  A.zlo = cz.zlo;
  A.cw = cz.cw;
  const int64_t nb = int64_t(n_units) * cz.nzc;
  const Layout L = layout(nb, tracks->cap_tracks, params->cap_pairs);
  char *w = static_cast<char *>(workspace);
  A.bin = reinterpret_cast<int32_t *>(w + L.bin);
  A.rank = reinterpret_cast<int32_t *>(w + L.inner);  // read by k_mg_fill, before k_mg_sort writes the records
  A.idx = reinterpret_cast<int32_t *>(w + L.idx);
  A.filed = reinterpret_cast<Filed *>(w + L.filed);
  A.inner = reinterpret_cast<Inner *>(w + L.inner);
  A.frs = reinterpret_cast<int32_t *>(w + L.frs);
  A.rows = reinterpret_cast<int32_t *>(w + L.rows);
  A.ob_chi = reinterpret_cast<unsigned long long *>(w + L.ob_chi);
  A.ib_chi = reinterpret_cast<unsigned long long *>(w + L.ib_chi);
  A.ob_idx = reinterpret_cast<int32_t *>(w + L.ob_idx);
  A.ib_idx = reinterpret_cast<int32_t *>(w + L.ib_idx);
  A.pairs = reinterpret_cast<int2 *>(w + L.pairs);
  A.pair_chi = reinterpret_cast<double *>(w + L.pair_chi);
  A.ctr = reinterpret_cast<unsigned long long *>(out->counts);
  hipStream_t st = static_cast<hipStream_t>(stream);
  auto blocks = [](int64_t n) { return unsigned(n < TPB ? 1 : ((n + TPB - 1) / TPB > MAX_BLOCKS ? MAX_BLOCKS : (n + TPB - 1) / TPB)); };
  const int64_t T = tracks->cap_tracks;
  hipLaunchKernelGGL(k_mg_init, dim3(blocks(T > nb + 1 ? T : nb + 1)), dim3(TPB), 0, st, A);
  hipLaunchKernelGGL(k_mg_rows, dim3(blocks(T)), dim3(TPB), 0, st, A);
  hipLaunchKernelGGL(k_mg_scan, dim3(1), dim3(SCAN_T), 0, st, A);
  hipLaunchKernelGGL(k_mg_fill, dim3(blocks(T)), dim3(TPB), 0, st, A);
  hipLaunchKernelGGL(k_mg_sort, dim3(unsigned(nb < MAX_BLOCKS ? nb : MAX_BLOCKS)), dim3(64), 0, st, A);
  const int64_t scan_blocks = (T + SEGS_MIN * WAVES - 1) / (SEGS_MIN * WAVES);
  hipLaunchKernelGGL(k_mg_pairs, dim3(unsigned(scan_blocks < 1 ? 1 : scan_blocks < MAX_BLOCKS ? scan_blocks : MAX_BLOCKS)), dim3(TPB), 0, st, A);
  hipLaunchKernelGGL(k_mg_chi2, dim3(blocks(params->cap_pairs)), dim3(TPB), 0, st, A);
  hipLaunchKernelGGL(k_mg_pick, dim3(blocks(params->cap_pairs)), dim3(TPB), 0, st, A);
  hipLaunchKernelGGL(k_mg_link, dim3(blocks(T)), dim3(TPB), 0, st, A);
  return hipGetLastError() == hipSuccess ? TPC_OK : TPC_E_HIP;
}

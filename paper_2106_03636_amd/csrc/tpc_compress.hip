// Hit removal and track-model compression, the consumer of the tracks (paper
// §2.1: hits of tracks not used for physics are removed, the remaining hits
// go through entropy-reduction steps such as the track model compression).
// The operation is stated with tpc_compress in include/tpc_track.h.
//
// Two launches on the caller's stream:
//   k_cmp_init   clear the histograms and counts, take over the tracking
//                call's status;
//   k_cmp_codes  per cluster (grid-stride, four consecutive ones a thread):
//                its class and codes; each block counts its classes and builds
//                its residual histograms in LDS, then adds the non-zero bins
//                to the global ones.
// One cluster reads its position and row (10 bytes), its track index (4)
// and, when attached, its track's state (24 bytes); it writes its class and
// codes (9 bytes).
// What bounds it: neighbouring clusters lie on different tracks, so the states
// are gathers, and their requests to the L2 set the time (88 M of them, over
// half of what it can take, when each of a state's six floats was loaded by
// itself and the rest of its line had left the L1 in between).  The parameters
// are therefore one 16-byte and one 4-byte load, and four clusters' states are
// on their way together: 24 M clusters 363 us instead of 540 (one cluster a
// thread with the wide load: 392; four with the narrow ones: 516 - 784), and
// with each XCD on a contiguous range 310.
// Each block adds its residuals to the same few hundred histogram bins, one
// after the other: 512 blocks.  1024 cost more (374 against 363; with 1 M
// clusters 50 us against 42), 256 leave too few loads in flight.

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "tpc_track.h"

namespace {

constexpr int TPB = 256;
constexpr int MAX_HIST_HALF = 2048;
constexpr int CMP_BLOCKS = 512;
constexpr float KAPPA = 0.00299792458f;

struct CmpArgs {
  const float *y, *z;
  const uint16_t *row;
  int64_t n;
  const float *row_x;
  int32_t n_rows;
  const int32_t *cluster_track, *trk_status;
  const int64_t *trk_counts;
  const float *par, *xref;
  double k, step, inv_step, pt_remove, sinphi_max;  // inv_step: 1 / step where that is exact (a power of two), else 0
  int32_t hh;  // hist_half
  uint8_t *cls;
  int32_t *code_y, *code_z;
  unsigned long long *hist, *counts;
  int32_t *status;
};

__global__ void __launch_bounds__(TPB) k_cmp_init(CmpArgs A) {
  const int64_t i = int64_t(blockIdx.x) * TPB + threadIdx.x;
  if (i == 0) *A.status = *A.trk_status;  // no codes for a failed tracking call
  if (i < 4 * int64_t(A.hh)) A.hist[i] = 0ull;
  if (i < 6) A.counts[i] = 0ull;
}

// The track's state (y, z, sin(phi), tan(lambda), q/pT at x1) carried along
// its helix to the plane x2 in FP64: sin(phi) changes by C dx (C = k q/pT),
// y by dx (sin1 + sin2) / (cos1 + cos2), z by tan(lambda) times the
// transverse arc length, 2 asin(C L / 2) / C over the chord L.  False when
// |sin(phi)| reaches sinphi_max or the chord is longer than a diameter.
__device__ __forceinline__ bool carry(const float *p, double x1, double x2, double k, double smax, double &yo,
                                      double &zo) {
#pragma clang fp contract(off)
  const double dx = x2 - x1;
  const double C = k * double(p[4]);
  const double s1 = p[2];
  const double s2 = s1 + C * dx;
  if (!(fabs(s1) < smax) || !(fabs(s2) < smax)) return false;
  const double c1 = sqrt(1.0 - s1 * s1), c2 = sqrt(1.0 - s2 * s2);
  const double dy = dx * (s1 + s2) / (c1 + c2);
  const double L = sqrt(dx * dx + dy * dy);
  const double u = fabs(C) * L * 0.5;
  if (!(u < 1.0)) return false;
  const double f = u < 1e-3 ? 1.0 + u * u / 6.0 : asin(u) / u;  // asin(u) / u
  const double sT = (dx < 0 ? -1.0 : 1.0) * L * f;
  yo = double(p[0]) + dy;
  zo = double(p[1]) + double(p[3]) * sT;
  return true;
}

// four of a track's five parameters (rows of 20 bytes) at once
typedef float F4 __attribute__((ext_vector_type(4), aligned(4)));

// The clusters c0 .. c0 + PER - 1 of the arrays as one access each; PER = 4
// wants the arrays aligned (whole quads).
template <int PER>
struct Quad {
  int32_t t[PER], r[PER];
  float y[PER], z[PER];
  __device__ __forceinline__ void load(const CmpArgs &A, int64_t c0) {
    if (PER == 4) {
      const int4 a = *reinterpret_cast<const int4 *>(A.cluster_track + c0);
      const float4 b = *reinterpret_cast<const float4 *>(A.y + c0), d = *reinterpret_cast<const float4 *>(A.z + c0);
      const ushort4 e = *reinterpret_cast<const ushort4 *>(A.row + c0);
      t[0] = a.x, t[1 % PER] = a.y, t[2 % PER] = a.z, t[3 % PER] = a.w;
      y[0] = b.x, y[1 % PER] = b.y, y[2 % PER] = b.z, y[3 % PER] = b.w;
      z[0] = d.x, z[1 % PER] = d.y, z[2 % PER] = d.z, z[3 % PER] = d.w;
      r[0] = e.x, r[1 % PER] = e.y, r[2 % PER] = e.z, r[3 % PER] = e.w;
    } else {
      t[0] = A.cluster_track[c0];
      y[0] = A.y[c0];
      z[0] = A.z[c0];
      r[0] = A.row[c0];
    }
  }
};

template <int PER>
__device__ __forceinline__ void codes(const CmpArgs &A, int64_t c0, int64_t T, const float *row_x, int32_t *hy, int32_t *hz,
                                      int32_t (&n)[6]) {
  Quad<PER> q;
  q.load(A, c0);
  float p[PER][5], x[PER];
  bool att[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) {  // the tracks' states, all on their way before the first is used
    att[e] = q.t[e] >= 0 && q.t[e] < T && q.r[e] < A.n_rows;
    const int64_t t = q.t[e];
    if (att[e]) {
      const F4 f = *reinterpret_cast<const F4 *>(A.par + t * 5);
      p[e][0] = f.x, p[e][1] = f.y, p[e][2] = f.z, p[e][3] = f.w;
      p[e][4] = A.par[t * 5 + 4];
      x[e] = A.xref[t];
    }
  }
  int32_t cy[PER], cz[PER], cls[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    double vy = double(q.y[e]), vz = double(q.z[e]);
    int cl = 0;
    if (att[e]) {
      double yp, zp;
      if (fabs(double(p[e][4])) * A.pt_remove > 1.0) {
        cl = 2;
      } else if (carry(p[e], double(x[e]), double(row_x[q.r[e]]), A.k, A.sinphi_max, yp, zp)) {
        cl = 1;
        vy -= yp;
        vz -= zp;
      } else {
        cl = 3;
      }
    }
    // the quotient by the step; a power of two's is a product, as exact
    vy = A.inv_step != 0.0 ? vy * A.inv_step : vy / A.step;
    vz = A.inv_step != 0.0 ? vz * A.inv_step : vz / A.step;
    cls[e] = cl;
    cy[e] = cl != 2 ? int32_t(rint(vy)) : 0;
    cz[e] = cl != 2 ? int32_t(rint(vz)) : 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) n[i] += cl == i;
    if (cl == 1) {
      if (cy[e] >= -A.hh && cy[e] < A.hh) atomicAdd(&hy[cy[e] + A.hh], 1); else ++n[4];
      if (cz[e] >= -A.hh && cz[e] < A.hh) atomicAdd(&hz[cz[e] + A.hh], 1); else ++n[5];
    }
  }
  if (PER == 4) {
    *reinterpret_cast<uchar4 *>(A.cls + c0) = make_uchar4(cls[0], cls[1 % PER], cls[2 % PER], cls[3 % PER]);
    *reinterpret_cast<int4 *>(A.code_y + c0) = make_int4(cy[0], cy[1 % PER], cy[2 % PER], cy[3 % PER]);
    *reinterpret_cast<int4 *>(A.code_z + c0) = make_int4(cz[0], cz[1 % PER], cz[2 % PER], cz[3 % PER]);
  } else {
    A.cls[c0] = uint8_t(cls[0]);
    A.code_y[c0] = cy[0];
    A.code_z[c0] = cz[0];
  }
}

// PER: clusters a thread takes at a time (4 where the arrays are aligned for
// it; the last few then one by one)
template <int PER>
__global__ void __launch_bounds__(TPB) k_cmp_codes(CmpArgs A) {
  extern __shared__ int32_t hist[];  // y codes, then z codes, then the rows' positions
  __shared__ int32_t cnt[6];
  if (*A.status != TPC_OK) return;
  const int32_t nb = 2 * A.hh;
  int32_t *hy = hist, *hz = hist + nb;
  float *row_x = reinterpret_cast<float *>(hist + 2 * nb);
  for (int32_t b = threadIdx.x; b < 2 * nb; b += TPB) hist[b] = 0;
  for (int32_t r = threadIdx.x; r < A.n_rows; r += TPB) row_x[r] = A.row_x[r];
  if (threadIdx.x < 6) cnt[threadIdx.x] = 0;
  __syncthreads();
  const int64_t T = A.trk_counts[0];
  int32_t n[6] = {0, 0, 0, 0, 0, 0};
  const int64_t quads = A.n / PER;
  // a unit's clusters share its tracks' states, so each XCD (blocks go to the
  // eight in turn) takes one contiguous range
  const int64_t turns = (quads + TPB - 1) / TPB, n8 = (turns + 7) & ~int64_t(7);
  for (int64_t k = blockIdx.x; k < n8; k += gridDim.x) {
    const int64_t i = ((k & 7) * (n8 >> 3) + (k >> 3)) * TPB + threadIdx.x;
    if (i < quads) codes<PER>(A, i * PER, T, row_x, hy, hz, n);
  }
  if (PER > 1 && blockIdx.x == 0 && quads * PER + threadIdx.x < A.n)
    codes<1>(A, quads * PER + threadIdx.x, T, row_x, hy, hz, n);
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    int32_t v = n[k];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if (__lane_id() == 0 && v) atomicAdd(&cnt[k], v);
  }
  __syncthreads();
  for (int32_t b = threadIdx.x; b < 2 * nb; b += TPB)
    if (hist[b]) atomicAdd(&A.hist[b], (unsigned long long)hist[b]);
  if (threadIdx.x < 6 && cnt[threadIdx.x]) atomicAdd(&A.counts[threadIdx.x], (unsigned long long)cnt[threadIdx.x]);
}

}  // namespace

extern "C" int tpc_compress(const tpc_clusters_t *clusters, const tpc_geometry_t *geometry,
                            const tpc_field_t *field, const tpc_tracks_t *tracks,
                            const tpc_compress_params_t *params, tpc_compressed_t *out, void *stream) {
  if (!clusters || !geometry || !field || !tracks || !params || !out) return TPC_E_INVALID;
  if (clusters->n < 0 || (clusters->n > 0 && (!clusters->y || !clusters->z || !clusters->row))) return TPC_E_INVALID;
  if (geometry->n_rows < 1 || geometry->n_rows > 255 || !geometry->row_x) return TPC_E_INVALID;
  if (!tracks->cluster_track || !tracks->params || !tracks->x_ref || !tracks->counts || !tracks->status)
    return TPC_E_INVALID;
  if (!(params->step > 0.0f) || !(params->pt_remove >= 0.0f) || !(params->sinphi_max > 0.0f) ||
      !(params->sinphi_max < 1.0f) || params->hist_half < 1 || params->hist_half > MAX_HIST_HALF ||
      !isfinite(field->bz_tesla))
    return TPC_E_INVALID;
  if (!out->cls || !out->code_y || !out->code_z || !out->hist || !out->counts || !out->status) return TPC_E_INVALID;
  CmpArgs A;
  A.y = clusters->y;
  A.z = clusters->z;
  A.row = clusters->row;
  A.n = clusters->n;
  A.row_x = geometry->row_x;
  A.n_rows = geometry->n_rows;
  A.cluster_track = tracks->cluster_track;
  A.trk_status = tracks->status;
  A.trk_counts = tracks->counts;
  A.par = tracks->params;
  A.xref = tracks->x_ref;
  A.k = double(-KAPPA * field->bz_tesla);  // the tracker's curvature constant, as its fit used it
  A.step = params->step;
  int exponent;
  A.inv_step = frexp(A.step, &exponent) == 0.5 ? 1.0 / A.step : 0.0;
  A.pt_remove = params->pt_remove;
  A.sinphi_max = params->sinphi_max;
  A.hh = params->hist_half;
  A.cls = out->cls;
  A.code_y = out->code_y;
  A.code_z = out->code_z;
  A.hist = reinterpret_cast<unsigned long long *>(out->hist);
  A.counts = reinterpret_cast<unsigned long long *>(out->counts);
  A.status = out->status;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int64_t ib = (4 * int64_t(A.hh) + TPB - 1) / TPB;
  const uintptr_t quad = reinterpret_cast<uintptr_t>(A.cluster_track) | reinterpret_cast<uintptr_t>(A.y) |
                         reinterpret_cast<uintptr_t>(A.z) | reinterpret_cast<uintptr_t>(A.code_y) |
                         reinterpret_cast<uintptr_t>(A.code_z);
  const bool aligned = (quad & 15) == 0 && (reinterpret_cast<uintptr_t>(A.row) & 7) == 0 &&
                       (reinterpret_cast<uintptr_t>(A.cls) & 3) == 0;
  const int64_t per = aligned ? 4 : 1, cb = (A.n / per + TPB - 1) / TPB;
  const unsigned blocks = (unsigned(cb < 1 ? 1 : (cb > CMP_BLOCKS ? CMP_BLOCKS : cb)) + 7u) & ~7u;
  const unsigned lds = unsigned(sizeof(int32_t)) * (4 * unsigned(A.hh) + unsigned(A.n_rows));
  hipLaunchKernelGGL(k_cmp_init, dim3(unsigned(ib)), dim3(TPB), 0, st, A);
  if (aligned)
    hipLaunchKernelGGL(k_cmp_codes<4>, dim3(blocks), dim3(TPB), lds, st, A);
  else
    hipLaunchKernelGGL(k_cmp_codes<1>, dim3(blocks), dim3(TPB), lds, st, A);
  return hipGetLastError() == hipSuccess ? TPC_OK : TPC_E_HIP;
}

// Track refit: every output track of a tracking call fitted again over
// exactly the hits it kept (the paper's synchronous processing needs full
// tracking, §2.1, at a resolution that matches offline reconstruction, §2.3).
// The operation is stated with tpc_refit_tracks in include/tpc_track.h.
//
// Seven launches on the caller's stream:
//   k_rf_init    clear the length histogram, take over the tracking status;
//   k_rf_pack    per cluster (coalesced): its row and its y, z in quanta,
//                packed into one 64-bit record;
//   k_rf_hist    histogram of the tracks' hit counts (LDS per block);
//   k_rf_scan    one block: bucket offsets, longest tracks first;
//   k_rf_order   each track's slot in the length order (one global atomic
//                per block and bucket, the slots inside a block from LDS);
//   k_rf_gather  per track hit: its cluster's record, in the order of the
//                track's hit list (one random 8-byte read per hit);
//   k_rf_fit     one lane per track, in length order (so the lanes of a wave
//                run loops of about the same length): seed, pass 1 forward,
//                pass 2 backward; state and covariance stay in registers.
// Clusters are in no particular order, so a track's hits are scattered over
// the cluster arrays: the pack turns three random reads per hit (y, z, row,
// each a cache line for 2 or 4 bytes) into one.
// What bounds them, on 20 M hits of 412 k tracks: the gather, its random reads:
// each XCD takes one contiguous range of the hit list, so that it works on one
// unit's clusters (5 MB of records) at a time and its L2 serves most of them
// (404 to 340 us; 60 G random reads/s).  The fit, FP32 issue, once its
// records come through LDS (below): 478 to 312 us, 35 TFLOP/s.

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "tpc_kalman.h"
#include "tpc_track.h"

namespace {

using namespace tpc_kf;

constexpr int TPB = 256;
constexpr int FTB = 128;  // threads per block of the fit
constexpr int NB = 256;   // length buckets (hit counts >= 255 share the last)
constexpr int ORDER_PER = 8;   // tracks per thread of the length order: one global atomic per bucket and 2048 tracks
constexpr int GATHER_BLOCKS = 4096;
constexpr int FIT_BLOCKS = 4096;
constexpr float KAPPA = 0.00299792458f;
constexpr int QBIAS = 1 << 23;  // record fields hold Y + 2^23 and Z + 2^23 (24 bits each)

struct RfArgs {
  const float *y, *z;
  const uint16_t *row;
  int64_t n_clusters;
  const float *row_x;
  int32_t n_rows;
  const int32_t *trk_status, *n_hits, *first_hit, *hits;
  const int64_t *trk_counts;
  int64_t cap_tracks, cap_hits;
  float k, smx, sy2, sz2;
  float cov0[5];
  // outputs
  float *par, *cov, *xref, *chi2, *par_out, *cov_out, *xout;
  uint8_t *ok;
  int32_t *status;
  // workspace
  int32_t *bucket;   // [NB] histogram, then running offsets
  int32_t *order;    // [cap_tracks] slot -> track
  uint64_t *cl;      // [n_clusters] packed (row, Y, Z) per cluster, NO_REC when out of range
  uint64_t *rec;     // [cap_hits] packed (row, Y, Z) per track hit
  int32_t *bad;      // [1] a track hit names no cluster or one out of range, or a track's hits lie outside the list
};

constexpr uint64_t NO_REC = ~uint64_t(0);  // row field 0xFFFF: never a valid row

__device__ __forceinline__ int bucket_of(int n) {  // longest first
  return NB - 1 - (n < 0 ? 0 : n < NB - 1 ? n : NB - 1);
}
// tracks and track hits of the tracking call, within the output capacities
__device__ __forceinline__ int64_t n_tracks(const RfArgs &A) {
  const int64_t T = A.trk_counts[0];
  return T < A.cap_tracks ? T : A.cap_tracks;
}
__device__ __forceinline__ int64_t n_track_hits(const RfArgs &A) {
  const int64_t H = A.trk_counts[1];
  return H < A.cap_hits ? H : A.cap_hits;
}

__global__ void __launch_bounds__(TPB) k_rf_init(RfArgs A) {
  const int i = threadIdx.x;
  if (i == 0) {
    *A.status = *A.trk_status;
    *A.bad = 0;
  }
  if (i < NB) A.bucket[i] = 0;
}

__global__ void __launch_bounds__(TPB) k_rf_hist(RfArgs A) {
  __shared__ int32_t h[NB];
  if (*A.status != TPC_OK) return;
  h[threadIdx.x] = 0;
  __syncthreads();
  const int64_t T = n_tracks(A), H = n_track_hits(A);
  bool bad = false;
  for (int64_t t = int64_t(blockIdx.x) * TPB + threadIdx.x; t < T; t += int64_t(gridDim.x) * TPB) {
    const int n = A.n_hits[t];
    const int64_t f = A.first_hit[t];
    if (n < 0 || f < 0 || f + n > H) bad = true;  // the track's hits lie outside the hit list
    atomicAdd(&h[bucket_of(n)], 1);
  }
  __syncthreads();
  if (h[threadIdx.x]) atomicAdd(&A.bucket[threadIdx.x], h[threadIdx.x]);
  if (bad) atomicOr(A.bad, 1);  // k_rf_fit reports it
}

// exclusive scan of the NB bucket counts (one block of NB threads)
__global__ void __launch_bounds__(NB) k_rf_scan(RfArgs A) {
  __shared__ int32_t s[NB];
  if (*A.status != TPC_OK) return;
  const int i = threadIdx.x;
  const int v = A.bucket[i];
  s[i] = v;
  __syncthreads();
  for (int d = 1; d < NB; d <<= 1) {
    const int a = i >= d ? s[i - d] : 0;
    __syncthreads();
    s[i] += a;
    __syncthreads();
  }
  A.bucket[i] = s[i] - v;
}

__global__ void __launch_bounds__(TPB) k_rf_pack(RfArgs A) {
  if (*A.status != TPC_OK) return;
  for (int64_t c = int64_t(blockIdx.x) * TPB + threadIdx.x; c < A.n_clusters; c += int64_t(gridDim.x) * TPB) {
    const int r = A.row[c];
    const float y = A.y[c], z = A.z[c];
    uint64_t v = NO_REC;
    if (r < A.n_rows && fabsf(y) <= 8192.f && fabsf(z) <= 8192.f) {  // |Y|, |Z| <= 2^21 fit the 24-bit fields
      const int Y = __float2int_rn(y * 256.0f), Z = __float2int_rn(z * 256.0f);
      v = (uint64_t(r) << 48) | (uint64_t(uint32_t(Y + QBIAS)) << 24) | uint64_t(uint32_t(Z + QBIAS));
    }
    A.cl[c] = v;
  }
}

// Slots of the length order: per chunk of tracks, those of each bucket count
// themselves in LDS, one thread per bucket reserves the chunk's range with one
// global atomic, and each track takes the range's start + its LDS rank.
template <class F>  // bucket of track t, -1 none
__device__ __forceinline__ void order_slots(int64_t T, int32_t *bucket, int32_t *order, F bucket_at) {
  static_assert(TPB == NB, "one thread per bucket");
  __shared__ int32_t cnt[NB];
  for (int64_t t0 = int64_t(blockIdx.x) * TPB * ORDER_PER; t0 < T; t0 += int64_t(gridDim.x) * TPB * ORDER_PER) {
    cnt[threadIdx.x] = 0;
    __syncthreads();
    int b[ORDER_PER], rank[ORDER_PER];
#pragma unroll
    for (int e = 0; e < ORDER_PER; ++e) {
      const int64_t t = t0 + e * TPB + threadIdx.x;
      b[e] = t < T ? bucket_at(t) : -1;
      rank[e] = b[e] >= 0 ? atomicAdd(&cnt[b[e]], 1) : 0;
    }
    __syncthreads();
    const int32_t c = cnt[threadIdx.x];
    if (c) cnt[threadIdx.x] = atomicAdd(&bucket[threadIdx.x], c);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < ORDER_PER; ++e)
      if (b[e] >= 0) order[cnt[b[e]] + rank[e]] = int32_t(t0 + e * TPB + threadIdx.x);
    __syncthreads();  // cnt is reused by the next chunk
  }
}

__global__ void __launch_bounds__(TPB) k_rf_order(RfArgs A) {
  if (*A.status != TPC_OK) return;
  order_slots(n_tracks(A), A.bucket, A.order, [&](int64_t t) { return bucket_of(A.n_hits[t]); });
}

// Blocks are dealt to the 8 XCDs in turn: XCD x takes the x-th eighth of the
// chunks, in order.  Calls f(chunk) for the chunks of this block (the grid is
// a multiple of 8).
template <class F>
__device__ __forceinline__ void xcd_chunks(int64_t n_chunks, F f) {
  const int64_t per = (n_chunks + 7) >> 3, step = gridDim.x >> 3;
  const int64_t lo = int64_t(blockIdx.x & 7) * per, hi = min(lo + per, n_chunks);
  for (int64_t c = lo + (blockIdx.x >> 3); c < hi; c += step) f(c);
}

constexpr int GATHER_PER = 4;  // records a thread has on their way
__global__ void __launch_bounds__(TPB) k_rf_gather(RfArgs A) {
  if (*A.status != TPC_OK) return;
  const int64_t H = n_track_hits(A);
  xcd_chunks((H + TPB * GATHER_PER - 1) / (TPB * GATHER_PER), [&](int64_t c) {
    const int64_t i0 = c * TPB * GATHER_PER + threadIdx.x;
    uint64_t r[GATHER_PER];
#pragma unroll
    for (int e = 0; e < GATHER_PER; ++e) {
      const int64_t i = i0 + e * TPB;
      const int32_t h = i < H ? A.hits[i] : -1;
      r[e] = h >= 0 && h < A.n_clusters ? A.cl[h] : NO_REC;
    }
#pragma unroll
    for (int e = 0; e < GATHER_PER; ++e) {
      const int64_t i = i0 + e * TPB;
      if (i < H && r[e] == NO_REC) {
        atomicOr(A.bad, 1);
        r[e] = 0;
      }
      if (i < H) A.rec[i] = r[e];
    }
  });
}

struct Hit {
  int row, Y, Z;
};
__device__ __forceinline__ Hit unpack(uint64_t r) {
  Hit h;
  h.row = int(r >> 48) & 0xFF;
  h.Y = int((r >> 24) & 0xFFFFFFu) - QBIAS;
  h.Z = int(r & 0xFFFFFFu) - QBIAS;
  return h;
}

// The state in absolute coordinates (the filter runs relative to the first
// hit's quanta Yr, Zr), its covariance and x; zeros for a track not fitted.
__device__ __forceinline__ void store(KStateR &s, bool ok, int Yr, int Zr, float *p, float *c, float *x) {
  p[0] = ok ? s.p[0] + float(Yr) * (1.f / 256.f) : 0.f;
  p[1] = ok ? s.p[1] + float(Zr) * (1.f / 256.f) : 0.f;
#pragma unroll
  for (int q = 2; q < 5; ++q) p[q] = ok ? s.p[q] : 0.f;
#pragma unroll
  for (int q = 0; q < 15; ++q) c[q] = ok ? cv(s, q) : 0.f;
  *x = ok ? s.x : 0.f;
}

// The records of a wave's 64 runs (a lane each) on their way to the filter, 8
// records of every run at a time, in two buffers of LDS: the loads of the next
// 8 go straight to LDS while the filter takes these, so that no step of the
// filter waits for memory, and each line is read once per pass (the lanes'
// runs are far apart; read a record per lane and step, a line is fetched
// again for nearly each of its 16 records).  Four lanes load the 64 bytes of
// a run, and the 16-byte pieces of run t are turned by (t >> 2) & 3, which
// puts the 64 records of one step on distinct banks.
constexpr int CHUNK = 8;
struct Runs {
  uint64_t *buf;  // [2][64 * CHUNK] of the wave, 16-byte aligned
  const uint64_t *rec;
  int64_t src[4];
  int n[4];

  __device__ __forceinline__ void init(uint64_t *lds, const uint64_t *records, int64_t first, int len) {
    const int lane = __lane_id();
    buf = lds;
    rec = records;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int t = 16 * i + (lane >> 2), piece = (lane & 3) ^ ((t >> 2) & 3);
      src[i] = __shfl((long long)first, t, 64) + 2 * piece;
      n[i] = __shfl(len, t, 64) - 2 * piece;  // records of the run from this lane's piece on
    }
  }
  // loads records [CHUNK c, CHUNK c + CHUNK) of every run; the last piece of a
  // run may read one record past it (see Layout)
  __device__ __forceinline__ void load(int c) const {
    uint64_t *to = buf + (c & 1) * (64 * CHUNK);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (CHUNK * c < n[i])
        __builtin_amdgcn_global_load_lds(
            (const __attribute__((address_space(1))) void *)(rec + src[i] + CHUNK * c),
            (__attribute__((address_space(3))) void *)(to + i * 128), 16, 0, 0);
  }
  static __device__ __forceinline__ void arrived() {  // every load so far is in LDS
    __builtin_amdgcn_s_waitcnt(0x0F70);               // vmcnt(0)
    __builtin_amdgcn_wave_barrier();
  }
  // record j of the lane's run, loaded with its chunk
  __device__ __forceinline__ uint64_t at(int j) const {
    const int lane = __lane_id();
    const uint64_t *from = buf + ((j / CHUNK) & 1) * (64 * CHUNK);
    return from[lane * CHUNK + ((((j >> 1) & 3) ^ ((lane >> 2) & 3)) << 1) + (j & 1)];
  }
};

// Maximum over the wave, in a scalar register.
__device__ __forceinline__ int wave_max(int v) {
  for (int d = 32; d >= 1; d >>= 1) v = max(v, __shfl_xor(v, d));
  return __builtin_amdgcn_readfirstlane(v);
}

__global__ void __launch_bounds__(FTB) k_rf_fit(RfArgs A) {
  __shared__ __align__(16) uint64_t stage[FTB / 64][2 * 64 * CHUNK];
  __shared__ float row_x[256];
  if (*A.status != TPC_OK) return;
  if (*A.bad) {  // every block sees the same flag; one writes the status
    if (blockIdx.x == 0 && threadIdx.x == 0) *A.status = TPC_E_INVALID;
    return;
  }
  for (int r = threadIdx.x; r < A.n_rows; r += FTB) row_x[r] = A.row_x[r];
  __syncthreads();
  const int64_t T = n_tracks(A);
  KStateR s;  // the covariance in registers: no LDS round trip in the update chain
  const float k = A.k, smx = A.smx, sy2 = A.sy2, sz2 = A.sz2;
  for (int64_t i0 = int64_t(blockIdx.x) * FTB; i0 < T; i0 += int64_t(gridDim.x) * FTB) {
    const int64_t i = i0 + threadIdx.x;
    if ((i & ~int64_t(63)) >= T) break;  // whole wave past the tracks (wave-uniform)
    const bool valid = i < T;
    const int32_t t = valid ? A.order[i] : 0;
    const int n = valid ? A.n_hits[t] : 0;
    const int64_t first = valid ? A.first_hit[t] : 0;
    const uint64_t *R = A.rec + first;
    bool ok = valid && n >= 3;
    int Yr = 0, Zr = 0;
    Runs runs;
    runs.init(stage[threadIdx.x >> 6], A.rec, first, ok ? n : 0);
    runs.load(0);
    uint64_t last = 0;
    if (ok) {
      last = R[n - 1];
      const Hit a = unpack(R[0]), m = unpack(R[n / 2]), b = unpack(last);
      Yr = a.Y;
      Zr = a.Z;
      ok = seed3<true>(s, row_x[a.row], row_x[m.row], row_x[b.row], float(m.Y - Yr) * (1.f / 256.f),
                 float(b.Y - Yr) * (1.f / 256.f), float(b.Z - Zr) * (1.f / 256.f), k, smx, A.cov0);
    }
    if (ok) kf_update(s, 0.f - s.p[0], 0.f - s.p[1], sy2, sz2);  // the first hit is the reference
    auto step = [&](int j) {
      const Hit h = unpack(runs.at(j));
      const float xr = row_x[h.row];
      Step st;
      if (!step_prepare(s, xr, k, smx, st)) {
        ok = false;
        return;
      }
      step_apply(s, st, xr, k);
      upd_hit(s, make_int2(h.Y, h.Z), Yr, Zr, sy2, sz2);
    };
    // pass 1: hits 1 .. n-1
    const int nmax = wave_max(ok ? n : 0);
    for (int c = 0; c * CHUNK < nmax; ++c) {
      Runs::arrived();
      runs.load(c + 1);
      for (int j = max(c * CHUNK, 1), je = min(c * CHUNK + CHUNK, nmax); j < je; ++j)
        if (ok && j < n) step(j);
    }
    // outer state: the end of pass 1
    if (valid) store(s, ok, Yr, Zr, A.par_out + int64_t(t) * 5, A.cov_out + int64_t(t) * 15, A.xout + t);
    // pass 2: hits n-2 .. 0, the covariance reset
    if (ok) {
      cov_reset(s, A.cov0);
      s.chi2 = 0.f;
      const Hit h = unpack(last);
      upd_hit(s, make_int2(h.Y, h.Z), Yr, Zr, sy2, sz2);
    }
    const int c1 = nmax >= 2 ? (nmax - 2) / CHUNK : -1;
    Runs::arrived();
    if (c1 >= 0) runs.load(c1);
    for (int c = c1; c >= 0; --c) {
      Runs::arrived();
      if (c > 0) runs.load(c - 1);
      for (int j = min(c * CHUNK + CHUNK - 1, nmax - 2); j >= c * CHUNK; --j)
        if (ok && j <= n - 2) step(j);
    }
    if (valid && !ok) store(s, false, 0, 0, A.par_out + int64_t(t) * 5, A.cov_out + int64_t(t) * 15, A.xout + t);
    if (valid) {
      A.ok[t] = ok ? 1 : 0;
      store(s, ok, Yr, Zr, A.par + int64_t(t) * 5, A.cov + int64_t(t) * 15, A.xref + t);
      A.chi2[t] = ok ? s.chi2 : 0.f;
    }
  }
}

size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

// The workspace of a refit or a chain fit.  The 16-byte loads of the hit
// records may touch one record past the last: the order follows them, which is
// never empty where there are records to load.
struct Layout {
  size_t cl, rec, order, total;
};
Layout layout(int64_t n_clusters, int64_t cap_tracks, int64_t cap_hits) {
  Layout L;
  L.cl = align256(NB * 4 + 256);  // after the length buckets and the flags
  L.rec = L.cl + align256(size_t(n_clusters) * 8);
  L.order = L.rec + align256(size_t(cap_hits) * 8);
  L.total = L.order + align256(size_t(cap_tracks) * 4);
  return L;
}
bool layout_ok(int64_t n_clusters, int64_t cap_tracks, int64_t cap_hits) {
  return n_clusters >= 0 && n_clusters < (int64_t(1) << 30) && cap_tracks >= 0 && cap_hits >= 0 &&
         cap_tracks <= (int64_t(1) << 31) && cap_hits <= (int64_t(1) << 31);
}

}  // namespace

extern "C" size_t tpc_refit_workspace_size(int64_t n_clusters, int64_t cap_tracks, int64_t cap_hits) {
  return layout_ok(n_clusters, cap_tracks, cap_hits) ? layout(n_clusters, cap_tracks, cap_hits).total : 0;
}

extern "C" int tpc_refit_tracks(const tpc_clusters_t *clusters, const tpc_geometry_t *geometry,
                                const tpc_field_t *field, const tpc_params_t *params, const tpc_tracks_t *tracks,
                                tpc_refit_t *out, void *workspace, size_t workspace_bytes, void *stream) {
  if (!clusters || !geometry || !field || !params || !tracks || !out) return TPC_E_INVALID;
  if (clusters->n < 0 || clusters->n >= (int64_t(1) << 30) ||
      (clusters->n > 0 && (!clusters->y || !clusters->z || !clusters->row)))
    return TPC_E_INVALID;
  if (geometry->n_rows < 3 || geometry->n_rows > 255 || !geometry->row_x) return TPC_E_INVALID;
  if (!tracks->n_hits || !tracks->first_hit || !tracks->hits || !tracks->counts || !tracks->status ||
      tracks->cap_tracks < 0 || tracks->cap_hits < 0)
    return TPC_E_INVALID;
  if (!isfinite(field->bz_tesla) || !(params->sinphi_max > 0.f) || !(params->sinphi_max < 1.f) ||
      !(params->sigma_y > 0.f) || !(params->sigma_z > 0.f))
    return TPC_E_INVALID;
  for (int q = 0; q < 5; ++q)
    if (!(params->cov0[q] > 0.f) || !isfinite(params->cov0[q])) return TPC_E_INVALID;
  if (!out->params || !out->cov || !out->x_ref || !out->chi2 || !out->params_out || !out->cov_out ||
      !out->x_out || !out->ok || !out->status)
    return TPC_E_INVALID;
  if (!layout_ok(clusters->n, tracks->cap_tracks, tracks->cap_hits)) return TPC_E_INVALID;
  const Layout L = layout(clusters->n, tracks->cap_tracks, tracks->cap_hits);
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255)) return TPC_E_INVALID;
  if (workspace_bytes < L.total) return TPC_E_NOMEM;
  RfArgs A;
  A.y = clusters->y;
  A.z = clusters->z;
  A.row = clusters->row;
  A.n_clusters = clusters->n;
  A.row_x = geometry->row_x;
  A.n_rows = geometry->n_rows;
  A.trk_status = tracks->status;
  A.n_hits = tracks->n_hits;
  A.first_hit = tracks->first_hit;
  A.hits = tracks->hits;
  A.trk_counts = tracks->counts;
  A.cap_tracks = tracks->cap_tracks;
  A.cap_hits = tracks->cap_hits;
  A.k = -KAPPA * field->bz_tesla;  // the tracker's curvature constant
  A.smx = params->sinphi_max;
  A.sy2 = params->sigma_y * params->sigma_y;
  A.sz2 = params->sigma_z * params->sigma_z;
  for (int q = 0; q < 5; ++q) A.cov0[q] = params->cov0[q];
  A.par = out->params;
  A.cov = out->cov;
  A.xref = out->x_ref;
  A.chi2 = out->chi2;
  A.par_out = out->params_out;
  A.cov_out = out->cov_out;
  A.xout = out->x_out;
  A.ok = out->ok;
  A.status = out->status;
  char *w = static_cast<char *>(workspace);
  A.bucket = reinterpret_cast<int32_t *>(w);
  A.bad = A.bucket + NB;
  A.cl = reinterpret_cast<uint64_t *>(w + L.cl);
  A.rec = reinterpret_cast<uint64_t *>(w + L.rec);
  A.order = reinterpret_cast<int32_t *>(w + L.order);
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int64_t tb = (tracks->cap_tracks + TPB - 1) / TPB;
  const int64_t hb = (tracks->cap_hits + TPB * GATHER_PER - 1) / (TPB * GATHER_PER);
  const int64_t cb = (clusters->n + TPB - 1) / TPB;
  const int64_t fb = (tracks->cap_tracks + FTB - 1) / FTB;
  auto clamp = [](int64_t b, int64_t hi) { return unsigned(b < 1 ? 1 : (b > hi ? hi : b)); };
  hipLaunchKernelGGL(k_rf_init, dim3(1), dim3(TPB), 0, st, A);
  hipLaunchKernelGGL(k_rf_pack, dim3(clamp(cb, GATHER_BLOCKS)), dim3(TPB), 0, st, A);
  hipLaunchKernelGGL(k_rf_hist, dim3(clamp((tb + ORDER_PER - 1) / ORDER_PER, 1024)), dim3(TPB), 0, st, A);
  hipLaunchKernelGGL(k_rf_scan, dim3(1), dim3(NB), 0, st, A);
  hipLaunchKernelGGL(k_rf_order, dim3(clamp((tb + ORDER_PER - 1) / ORDER_PER, 1024)), dim3(TPB), 0, st, A);
  hipLaunchKernelGGL(k_rf_gather, dim3((clamp(hb, GATHER_BLOCKS) + 7) & ~7u), dim3(TPB), 0, st, A);
  hipLaunchKernelGGL(k_rf_fit, dim3(clamp(fb, FIT_BLOCKS)), dim3(FTB), 0, st, A);
  return hipGetLastError() == hipSuccess ? TPC_OK : TPC_E_HIP;
}

// ---------------------------------------------------------------------------
// Fit of merged chains: the hits of linked segments (a tpc_merge_tracks
// output) in chain order, across their sectors' frames.  Launches: status;
// the refit's k_rf_pack; k_ch_len (each head's chain length, a length
// histogram, a place for its records, the turns between its segments' frames,
// and zeros for the tracks that head no chain); k_rf_scan; k_ch_order (heads
// in length order); k_ch_gather (a wave per track: the records of the
// chains' hits, each chain's one after the other); k_ch_fit (one lane per
// head in length order, so the lanes of a wave walk chains of about one
// length; their records come through LDS as the refit's do): before a hit of
// another frame the state and its covariance are turned into that frame (the
// turn's Jacobian), then carried and updated as in the refit.  The state
// stays relative to the current frame's reference quanta (z: the chain's
// first hit; y: the first hit seen in the frame), re-based at each turn.  The
// operation is stated with tpc_fit_chains in include/tpc_track.h.
// What bounds the fit: the latency of the longest chains' 2 x 152 steps (all
// waves are resident at once).  With the records, the row positions and the
// turns out of a step's way: 732 to 478 us for 118 k chains, the call 1280 to 920 us.

namespace {

constexpr int MAX_CHAIN = 64;  // segments a chain may hold
constexpr double CH_TWO_PI = 6.283185307179586476925286766559;

struct ChArgs {
  const float *y, *z;
  const uint16_t *row;
  int64_t n_clusters;
  const float *row_x;
  int32_t n_rows;
  const int32_t *trk_status, *n_hits, *first_hit, *hits, *unit;
  const int64_t *trk_counts;
  int64_t cap_tracks, cap_hits;
  const int32_t *next, *prev, *mg_status;
  const float *alpha;
  int32_t n_units;
  float k, smx, sy2, sz2;
  float cov0[5];
  float *par, *cov, *xref, *chi2;
  int32_t *n_chain;
  uint8_t *ok;
  int32_t *status;
  // workspace (the refit's layout)
  const uint64_t *cl;   // [n_clusters] packed (row, Y, Z) per cluster
  uint64_t *rec;        // [cap_hits] the same per chain hit, a segment's first one marked
  int32_t *order;       // [cap_tracks] slot -> chain head
  int32_t *bucket;      // [NB] length histogram, then offsets
  int32_t *bad;         // [0] a hit out of range (the gather's flag), [1] number of heads,
                        // [2] the tracks' hit lists do not follow one another from 0 to the end
  unsigned long long *given;  // [1] records given out to the chains
};
// A neighbour of a chain segment, and the cosine and sine of the turn into its
// frame: one read when a walk enters the segment.
struct Side {
  float c, s;
  int32_t q;
};
// What the fit has to know of a track is kept in the track's own output rows
// until its results are known: the place of a chain segment's first record in
// x_ref (-1: the track is in no chain), its neighbours in cov.
__device__ __forceinline__ int32_t *place(const ChArgs &A, int64_t t) { return reinterpret_cast<int32_t *>(A.xref + t); }
__device__ __forceinline__ Side *sides(const ChArgs &A, int64_t t) {  // the next segment, the one before
  return reinterpret_cast<Side *>(A.cov + t * 15);
}
constexpr int SIDES = 2 * sizeof(Side) / 4;        // floats of the row that they take
constexpr float SAME_FRAME = 2.f;                  // in place of the cosine: the segments share their unit
constexpr uint64_t FIRST = uint64_t(1) << 56;      // mark of a segment's first record

// the unit of the chain's hit j: its segment found by walking the links from the head
__device__ __forceinline__ int unit_at(const ChArgs &A, int32_t head, int j) {
  int32_t s = head;
  for (int g = 0; g < MAX_CHAIN && j >= A.n_hits[s]; ++g) {
    j -= A.n_hits[s];
    s = A.next[s];
  }
  return A.unit[s];
}

__device__ __forceinline__ float frame_turn(const ChArgs &A, int from, int to) {
  return float(remainder(double(A.alpha[to]) - double(A.alpha[from]), CH_TWO_PI));
}

// Turn the state by d (cosine cd, sine sd) into another frame: the point (x, ya) and the
// direction turn, the state moves to the turned point's x; the covariance by
// the turn's Jacobian (rows y, z, sin(phi) change: dy'/dy = cos phi / cos
// phi', dz'/dy = -sin d tan(lambda) / cos phi', dsin'/dy = -C sin d,
// dsin'/dsin = cos phi' / cos phi).  ya: absolute y in, turned y out.
__device__ __forceinline__ bool turn32(KStateR &s, float cd, float sd, float &ya, float k, float smx) {
  const float sp = s.p[2];
  if (!(fabsf(sp) < 1.f)) return false;
  const float c = sqrtf(1.f - sp * sp);
  const float s2 = sp * cd - c * sd, c2 = c * cd + sp * sd;
  if (!(c2 > 0.f) || !(fabsf(s2) < smx)) return false;
  const float x2 = s.x * cd + ya * sd;
  const float y2 = -s.x * sd + ya * cd;
  const float j00 = c / c2, j10 = -sd * s.p[3] / c2, j20 = -k * s.p[4] * sd, j22 = c2 / c;
  float C[5][5];
  int m = 0;
#pragma unroll
  for (int i = 0; i < 5; ++i)
#pragma unroll
    for (int j = 0; j <= i; ++j, ++m) C[i][j] = C[j][i] = s.c[m];
  // T = J C (rows 0..2 change), then C' = T J^T (columns 0..2 change)
  float T[5][5];
#pragma unroll
  for (int j = 0; j < 5; ++j) {
    T[0][j] = j00 * C[0][j];
    T[1][j] = C[1][j] + j10 * C[0][j];
    T[2][j] = j20 * C[0][j] + j22 * C[2][j];
    T[3][j] = C[3][j];
    T[4][j] = C[4][j];
  }
  m = 0;
#pragma unroll
  for (int i = 0; i < 5; ++i)
#pragma unroll
    for (int j = 0; j <= i; ++j, ++m) {
      const float v = j == 0 ? j00 * T[i][0]
                    : j == 1 ? T[i][1] + j10 * T[i][0]
                    : j == 2 ? j20 * T[i][0] + j22 * T[i][2]
                             : T[i][j];
      s.c[m] = v;
    }
  s.p[2] = s2;
  s.x = x2;
  ya = y2;
  return true;
}

__global__ void __launch_bounds__(TPB) k_ch_init(ChArgs A) {
  const int i = threadIdx.x;
  if (i == 0) {
    *A.status = *A.trk_status != TPC_OK ? *A.trk_status : *A.mg_status;
    A.bad[0] = A.bad[1] = A.bad[2] = 0;
    *A.given = 0ull;
  }
  if (i < NB) A.bucket[i] = 0;
}

__device__ __forceinline__ int64_t ch_tracks(const ChArgs &A) {
  const int64_t T = A.trk_counts[0];
  return T < A.cap_tracks ? T : A.cap_tracks;
}

// per track: the checks of the input (its hits inside the hit list; links
// that are mutual, name tracks of the call and, followed back, reach a head
// within MAX_CHAIN segments, so that no closed loop is left; a linked track's
// unit in range), and the length of the chain it heads (0 for other tracks,
// whose outputs are cleared); heads counted and histogrammed by length
// (longest first), and given a range of the records
__global__ void __launch_bounds__(TPB) k_ch_len(ChArgs A) {
  __shared__ int32_t h[NB];
  __shared__ int32_t heads;
  __shared__ unsigned long long given, base;
  if (*A.status != TPC_OK) return;
  h[threadIdx.x] = 0;
  if (threadIdx.x == 0) heads = 0;
  const int64_t T = ch_tracks(A);
  const int64_t H = A.trk_counts[1] < A.cap_hits ? A.trk_counts[1] : A.cap_hits;
  bool bad = false, apart = false;
  for (int64_t t0 = int64_t(blockIdx.x) * TPB; t0 < T; t0 += int64_t(gridDim.x) * TPB) {  // block-uniform
    const int64_t t = t0 + threadIdx.x;
    if (threadIdx.x == 0) given = 0;
    __syncthreads();
    int64_t n = 0;
    unsigned long long at = 0ull;
    if (t < T) {
      const int nt = A.n_hits[t];
      const int64_t ft = A.first_hit[t];
      const int32_t nx = A.next[t], pv = A.prev[t];
      if (nt < 0 || ft < 0 || ft + nt > H) bad = true;
      if ((t == 0 && ft != 0) || (t + 1 < T ? A.first_hit[t + 1] : H) != ft + nt) apart = true;
      if ((nx >= 0 && (nx >= T || A.prev[nx] != t)) || (pv >= 0 && (pv >= T || A.next[pv] != t))) bad = true;
      if ((nx >= 0 || pv >= 0) && (A.unit[t] < 0 || A.unit[t] >= A.n_units)) bad = true;
      if (pv >= 0 && !bad) {
        int32_t q = pv;
        for (int g = 1; q >= 0 && q < T && g < MAX_CHAIN; ++g) q = A.prev[q];
        if (q >= 0) bad = true;
      }
      if (pv < 0 && nx >= 0) {
        int nseg = 0;
        for (int32_t q = int32_t(t); q >= 0; q = A.next[q], ++nseg) {
          if (q >= T || nseg >= MAX_CHAIN || A.n_hits[q] < 1) {
            bad = true;
            n = 0;
            break;
          }
          n += A.n_hits[q];
        }
        if (n > INT32_MAX) {
          bad = true;
          n = 0;
        }
        if (n > 0) {
          atomicAdd(&h[bucket_of(int(n))], 1);
          atomicAdd(&heads, 1);
          at = atomicAdd(&given, (unsigned long long)n);
        }
      }
      A.n_chain[t] = int32_t(n);
      if (n == 0) {  // the outputs of a track that heads no chain
        const bool none = nx < 0 && pv < 0;
        A.ok[t] = 0;
#pragma unroll
        for (int q = 0; q < 5; ++q) A.par[t * 5 + q] = 0.f;
#pragma unroll
        for (int q = 0; q < 15; ++q)
          if (none || q >= SIDES) A.cov[t * 15 + q] = 0.f;
        A.chi2[t] = 0.f;
        if (none) *place(A, t) = -1;  // the rest of a chain segment's row is its head's until the fit has ended
      }
    }
    __syncthreads();
    if (threadIdx.x == 0 && given) base = atomicAdd(A.given, given);
    __syncthreads();
    if (n > 0) {  // the segments' places, and the turns into their frames
      unsigned long long to = base + at;
      int32_t from = 0, before = -1;
      int nseg = 0;
      for (int32_t q = int32_t(t); q >= 0 && q < T && nseg < MAX_CHAIN; q = A.next[q], ++nseg) {
        *place(A, q) = int32_t(to);
        to += A.n_hits[q];
        const int u = A.unit[q];
        float c = SAME_FRAME, sn = 0.f;
        // the segments' units may be out of range (their own threads report it): neither is then looked up
        if (before >= 0 && u != from && min(u, from) >= 0 && max(u, from) < A.n_units) {
          const float d = frame_turn(A, from, u);  // back again it is -d: remainder, sine and cosine are odd or even
          c = cosf(d);
          sn = sinf(d);
        }
        if (before >= 0) sides(A, before)[0] = Side{c, sn, q};
        sides(A, q)[1] = Side{c, -sn, before};
        from = u;
        before = q;
      }
    }
  }
  __syncthreads();
  if (h[threadIdx.x]) atomicAdd(&A.bucket[threadIdx.x], h[threadIdx.x]);
  if (threadIdx.x == 0 && heads) atomicAdd(&A.bad[1], heads);
  if (apart) atomicOr(&A.bad[2], 1);
  if (bad) *A.status = TPC_E_INVALID;
}

// slots of the heads in length order
__global__ void __launch_bounds__(TPB) k_ch_order(ChArgs A) {
  if (*A.status != TPC_OK) return;
  order_slots(ch_tracks(A), A.bucket, A.order, [&](int64_t t) {
    const int n = A.n_chain[t];
    return n > 0 ? bucket_of(n) : -1;
  });
}

// The record of hit h, 0 and the flag where it names no cluster or one out of range.
__device__ __forceinline__ uint64_t record_of(const ChArgs &A, int32_t h) {
  const uint64_t r = h >= 0 && h < A.n_clusters ? A.cl[h] : NO_REC;
  if (r != NO_REC) return r;
  atomicOr(A.bad, 1);
  return 0;
}

// Whether the chains' records have no room one after the other: hit lists
// that overlap may add up to more hits than the list holds.
__device__ __forceinline__ bool crowded(const ChArgs &A) { return *A.given > (unsigned long long)A.cap_hits; }

// The chain's record j then, from the hit lists.
__device__ uint64_t walk_to(const ChArgs &A, int32_t head, int j) {
  int32_t q = head;
  for (int g = 0; g < MAX_CHAIN && j >= A.n_hits[q]; ++g) {
    j -= A.n_hits[q];
    q = A.next[q];
  }
  const uint64_t r = A.cl[A.hits[A.first_hit[q] + j]];
  return j == 0 ? r | FIRST : r;
}

// The records of every track's hits, a wave per track (each XCD a contiguous
// range of the tracks, as in k_rf_gather): checked, and those of chain
// segments written at their places.  Hits that belong to no track are checked
// too, where the lists leave any: with no track at all, every hit.
__global__ void __launch_bounds__(TPB) k_ch_gather(ChArgs A) {
  constexpr int WAVES = TPB / 64;
  if (*A.status != TPC_OK) return;
  const int64_t T = ch_tracks(A);
  const int64_t H = A.trk_counts[1] < A.cap_hits ? A.trk_counts[1] : A.cap_hits;
  const int lane = __lane_id();
  const bool room = !crowded(A);
  if (A.bad[2] || T == 0)
    for (int64_t i = int64_t(blockIdx.x) * TPB + threadIdx.x; i < H; i += int64_t(gridDim.x) * TPB) record_of(A, A.hits[i]);
  xcd_chunks((T + WAVES - 1) / WAVES, [&](int64_t c) {
    const int64_t t = c * WAVES + (threadIdx.x >> 6);
    if (t >= T) return;
    const int n = A.n_hits[t];
    const int64_t f = A.first_hit[t];
    const int32_t d = *place(A, t);
    if (d < 0 && lane == 0) A.xref[t] = 0.f;
    for (int j = lane; j < n; j += 64) {
      const uint64_t r = record_of(A, A.hits[f + j]);
      if (room && d >= 0) A.rec[int64_t(d) + j] = j == 0 ? r | FIRST : r;
    }
  });
}

__global__ void __launch_bounds__(FTB) k_ch_fit(ChArgs A) {
  __shared__ __align__(16) uint64_t stage[FTB / 64][2 * 64 * CHUNK];
  __shared__ float row_x[256];
  if (*A.status != TPC_OK) return;
  if (A.bad[0]) {  // a track hit out of range (the gather's flag): every block sees it
    if (blockIdx.x == 0 && threadIdx.x == 0) *A.status = TPC_E_INVALID;
    return;
  }
  const int64_t H = A.bad[1];
  const bool room = !crowded(A);
  const float k = A.k, smx = A.smx, sy2 = A.sy2, sz2 = A.sz2;
  for (int r = threadIdx.x; r < A.n_rows; r += FTB) row_x[r] = A.row_x[r];
  __syncthreads();
  for (int64_t i0 = int64_t(blockIdx.x) * FTB; i0 < H; i0 += int64_t(gridDim.x) * FTB) {
    const int64_t i = i0 + threadIdx.x;
    if ((i & ~int64_t(63)) >= H) break;  // whole wave past the heads (wave-uniform)
    const bool valid = i < H;            // the other lanes stay for the shuffles below
    KStateR s;
    const int32_t t = valid ? A.order[i] : 0;
    const int n = valid ? A.n_chain[t] : 0;
    const int64_t first = valid && room ? *place(A, t) : 0;
    bool ok = valid && n >= 3;
    int Yr = 0, Zr = 0;
    uint64_t last = 0;
    Runs runs;
    runs.init(stage[threadIdx.x >> 6], A.rec, first, ok && room ? n : 0);
    runs.load(0);
    auto record = [&](int j) { return room ? A.rec[first + j] : walk_to(A, t, j); };
    // the segment the walk is in, and the one it comes to (loaded when the walk enters a segment)
    int32_t q = t;
    Side to{SAME_FRAME, 0.f, -1};
    if (ok) {  // seed in the first hit's frame
      last = record(n - 1);
      const Hit h0 = unpack(record(0)), hm = unpack(record(n / 2)), hl = unpack(last);
      to = sides(A, t)[0];
      const int cu = A.unit[t];
      Yr = h0.Y;
      Zr = h0.Z;
      const float y0 = float(Yr) * (1.f / 256.f);
      float xs[2], ys[2];
      const Hit hs[2] = {hm, hl};
      const int us[2] = {unit_at(A, t, n / 2), unit_at(A, t, n - 1)};
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const float d = frame_turn(A, us[e], cu), x = row_x[hs[e].row];
        const float cd = cosf(d), sd = sinf(d), yy = float(hs[e].Y) * (1.f / 256.f);
        xs[e] = us[e] == cu ? x : fmaf(yy, sd, x * cd);
        ys[e] = us[e] == cu ? float(hs[e].Y - Yr) * (1.f / 256.f) : fmaf(yy, cd, -(x * sd)) - y0;
      }
      ok = seed3(s, row_x[h0.row], xs[0], xs[1], ys[0], ys[1], float(hl.Z - Zr) * (1.f / 256.f), k, smx, A.cov0);
    }
    // one hit of the chain: into its unit's frame when it changes (turn: cosine
    // and sine; re-based on the hit), then the transport and the update
    auto step = [&](const Hit h, bool turned, float cd, float sd) {
      if (turned && cd != SAME_FRAME) {
        float ya = s.p[0] + float(Yr) * (1.f / 256.f);
        if (!turn32(s, cd, sd, ya, k, smx)) {
          ok = false;
          return;
        }
        Yr = h.Y;
        s.p[0] = ya - float(Yr) * (1.f / 256.f);
      }
      const float x = row_x[h.row];
      Step st;
      if (!step_prepare(s, x, k, smx, st)) {
        ok = false;
        return;
      }
      step_apply(s, st, x, k);
      upd_hit<true>(s, make_int2(h.Y, h.Z), Yr, Zr, sy2, sz2);
    };
    // pass 1: hits 1 .. n-1 in chain order
    const int nmax = wave_max(ok ? n : 0);
    if (ok) kf_update<true>(s, 0.f - s.p[0], 0.f - s.p[1], sy2, sz2);
    for (int c = 0; c * CHUNK < nmax; ++c) {
      Runs::arrived();
      runs.load(c + 1);
      for (int j = max(c * CHUNK, 1), je = min(c * CHUNK + CHUNK, nmax); j < je; ++j) {
        if (!ok || j >= n) continue;
        const uint64_t r = room ? runs.at(j) : walk_to(A, t, j);
        const bool enter = r & FIRST;
        step(unpack(r), enter, to.c, to.s);
        if (enter) {
          q = to.q;
          to = sides(A, q)[0];  // not read further in the last segment, where it is not written
        }
      }
    }
    // pass 2: from the last hit back, covariance reset, turning back at each change of frame
    bool leave = false;  // the hit before this one is another segment's
    if (ok) {
      cov_reset(s, A.cov0);
      s.chi2 = 0.f;
      const Hit hl = unpack(last);
      upd_hit<true>(s, make_int2(hl.Y, hl.Z), Yr, Zr, sy2, sz2);
      leave = last & FIRST;
      to = sides(A, q)[1];
    }
    const int c1 = nmax >= 2 ? (nmax - 2) / CHUNK : -1;
    Runs::arrived();
    if (c1 >= 0) runs.load(c1);
    for (int c = c1; c >= 0; --c) {
      Runs::arrived();
      if (c > 0) runs.load(c - 1);
      for (int j = min(c * CHUNK + CHUNK - 1, nmax - 2); j >= c * CHUNK; --j) {
        if (!ok || j > n - 2) continue;
        const uint64_t r = room ? runs.at(j) : walk_to(A, t, j);
        step(unpack(r), leave, to.c, to.s);
        if (leave) to = sides(A, to.q)[1];
        leave = r & FIRST;
      }
    }
    if (!valid) continue;
    A.ok[t] = ok ? 1 : 0;
    float *par = A.par + int64_t(t) * 5, *cov = A.cov + int64_t(t) * 15;
    par[0] = ok ? s.p[0] + float(Yr) * (1.f / 256.f) : 0.f;
    par[1] = ok ? s.p[1] + float(Zr) * (1.f / 256.f) : 0.f;
#pragma unroll
    for (int e = 2; e < 5; ++e) par[e] = ok ? s.p[e] : 0.f;
#pragma unroll
    for (int e = 0; e < 15; ++e) cov[e] = ok ? s.c[e] : 0.f;
    A.xref[t] = ok ? s.x : 0.f;
    A.chi2[t] = ok ? s.chi2 : 0.f;
    for (int32_t r = A.next[t]; r >= 0; r = A.next[r]) {  // the rows of the chain's other segments, which it used
#pragma unroll
      for (int e = 0; e < SIDES; ++e) A.cov[int64_t(r) * 15 + e] = 0.f;
      A.xref[r] = 0.f;
    }
  }
}

}  // namespace

extern "C" int tpc_fit_chains(const tpc_clusters_t *clusters, const tpc_geometry_t *geometry, const tpc_field_t *field,
                              const tpc_params_t *params, const tpc_tracks_t *tracks, const tpc_merged_t *merged,
                              const float *unit_alpha, int32_t n_units, tpc_chain_fit_t *out, void *workspace,
                              size_t workspace_bytes, void *stream) {
  if (!clusters || !geometry || !field || !params || !tracks || !merged || !unit_alpha || !out) return TPC_E_INVALID;
  if (clusters->n < 0 || clusters->n >= (int64_t(1) << 30) ||
      (clusters->n > 0 && (!clusters->y || !clusters->z || !clusters->row)))
    return TPC_E_INVALID;
  if (geometry->n_rows < 3 || geometry->n_rows > 255 || !geometry->row_x || n_units < 1) return TPC_E_INVALID;
  if (!tracks->n_hits || !tracks->first_hit || !tracks->hits || !tracks->unit || !tracks->counts ||
      !tracks->status || tracks->cap_tracks < 0 || tracks->cap_hits < 0)
    return TPC_E_INVALID;
  if (!merged->next || !merged->prev || !merged->status) return TPC_E_INVALID;
  if (!isfinite(field->bz_tesla) || !(params->sinphi_max > 0.f) || !(params->sinphi_max < 1.f) ||
      !(params->sigma_y > 0.f) || !(params->sigma_z > 0.f))
    return TPC_E_INVALID;
  for (int q = 0; q < 5; ++q)
    if (!(params->cov0[q] > 0.f) || !isfinite(params->cov0[q])) return TPC_E_INVALID;
  if (!out->params || !out->cov || !out->x_ref || !out->chi2 || !out->n_hits || !out->ok || !out->status)
    return TPC_E_INVALID;
  if (!layout_ok(clusters->n, tracks->cap_tracks, tracks->cap_hits)) return TPC_E_INVALID;
  const Layout L = layout(clusters->n, tracks->cap_tracks, tracks->cap_hits);
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255)) return TPC_E_INVALID;
  if (workspace_bytes < L.total) return TPC_E_NOMEM;
  // the refit's workspace layout; its pack and gather fill the hit records
  char *w = static_cast<char *>(workspace);
  RfArgs R{};
  R.y = clusters->y;
  R.z = clusters->z;
  R.row = clusters->row;
  R.n_clusters = clusters->n;
  R.row_x = geometry->row_x;
  R.n_rows = geometry->n_rows;
  R.trk_status = tracks->status;
  R.n_hits = tracks->n_hits;
  R.first_hit = tracks->first_hit;
  R.hits = tracks->hits;
  R.trk_counts = tracks->counts;
  R.cap_tracks = tracks->cap_tracks;
  R.cap_hits = tracks->cap_hits;
  R.status = out->status;
  R.bucket = reinterpret_cast<int32_t *>(w);
  R.bad = R.bucket + NB;
  R.cl = reinterpret_cast<uint64_t *>(w + L.cl);
  R.rec = reinterpret_cast<uint64_t *>(w + L.rec);
  R.order = reinterpret_cast<int32_t *>(w + L.order);
  ChArgs A;
  A.y = clusters->y;
  A.z = clusters->z;
  A.row = clusters->row;
  A.n_clusters = clusters->n;
  A.row_x = geometry->row_x;
  A.n_rows = geometry->n_rows;
  A.trk_status = tracks->status;
  A.n_hits = tracks->n_hits;
  A.first_hit = tracks->first_hit;
  A.hits = tracks->hits;
  A.unit = tracks->unit;
  A.trk_counts = tracks->counts;
  A.cap_tracks = tracks->cap_tracks;
  A.cap_hits = tracks->cap_hits;
  A.next = merged->next;
  A.prev = merged->prev;
  A.mg_status = merged->status;
  A.alpha = unit_alpha;
  A.n_units = n_units;
  A.k = -KAPPA * field->bz_tesla;
  A.smx = params->sinphi_max;
  A.sy2 = params->sigma_y * params->sigma_y;
  A.sz2 = params->sigma_z * params->sigma_z;
  for (int q = 0; q < 5; ++q) A.cov0[q] = params->cov0[q];
  A.par = out->params;
  A.cov = out->cov;
  A.xref = out->x_ref;
  A.chi2 = out->chi2;
  A.n_chain = out->n_hits;
  A.ok = out->ok;
  A.status = out->status;
  A.cl = R.cl;
  A.rec = R.rec;
  A.order = R.order;
  A.bucket = R.bucket;
  A.bad = R.bad;
  A.given = reinterpret_cast<unsigned long long *>(R.bad + 4);
  hipStream_t st = static_cast<hipStream_t>(stream);
  auto clamp = [](int64_t b, int64_t hi) { return unsigned(b < 1 ? 1 : (b > hi ? hi : b)); };
  const int64_t tb = (tracks->cap_tracks + TPB - 1) / TPB;
  const int64_t cb = (clusters->n + TPB - 1) / TPB;
  const int64_t fb = (tracks->cap_tracks + FTB - 1) / FTB;
  const int64_t wb = (tracks->cap_tracks + TPB / 64 - 1) / (TPB / 64);
  hipLaunchKernelGGL(k_ch_init, dim3(1), dim3(TPB), 0, st, A);
  hipLaunchKernelGGL(k_rf_pack, dim3(clamp(cb, GATHER_BLOCKS)), dim3(TPB), 0, st, R);
  hipLaunchKernelGGL(k_ch_len, dim3(clamp(tb, 1024)), dim3(TPB), 0, st, A);
  hipLaunchKernelGGL(k_rf_scan, dim3(1), dim3(NB), 0, st, R);
  hipLaunchKernelGGL(k_ch_order, dim3(clamp((tb + ORDER_PER - 1) / ORDER_PER, 1024)), dim3(TPB), 0, st, A);
  hipLaunchKernelGGL(k_ch_gather, dim3((clamp(wb, GATHER_BLOCKS) + 7) & ~7u), dim3(TPB), 0, st, A);
  hipLaunchKernelGGL(k_ch_fit, dim3(clamp(fb, FIT_BLOCKS)), dim3(FTB), 0, st, A);
  return hipGetLastError() == hipSuccess ? TPC_OK : TPC_E_HIP;
}

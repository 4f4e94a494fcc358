// Clusterizer: zero-suppressed raw ADC digits to clusters, the producer of
// the tracker's input (paper §2.1: a clusterizing algorithm turns the raw
// ADC values into hits; §3.2: it runs much faster on GPUs than on CPUs).
// The operation is stated with tpc_clusterize in include/tpc_track.h.
//
// Two launches on the caller's stream:
//   k_clu_init   status, count, the rows' first pads, and for each block the
//                row it works on, in its look-back word;
//   k_clu_find   a block per part of a row (taken by ticket): the digits of its
//                pads and of the pads either side go to LDS once; each wave
//                filters a contiguous share of them (only a digit of q_min or
//                more that its neighbours in time do not beat can be a peak:
//                about 3 in 10), tests the survivors against the pads either
//                side (a binary search over their time-ordered digits) and
//                keeps the peaks, the first in registers, the rest by their
//                places; the blocks' counts are added up by a decoupled
//                look-back, and the peaks are written at their places, so
//                clusters come in (unit, row, pad, time) order.  Digits are read
//                once (those of edge pads twice).
// A look-back waits for the slowest block before it, so the blocks have to cost
// alike, whatever rows, units or regions are dense: a row has as many parts as
// multiples of digits_per_part lie among its digits' numbers, and one more
// (first_block: known for every row by itself, without a scan), and its pads are
// cut at like many digits.  A part still holds more than a block stages where
// single pads are very dense, or a sparse row is long: it is taken a run of
// pads at a time, all counted before the first is written.  36 units of 1.75 M
// digits each, evenly: 811 us; the same digits ten times denser in a tenth of
// the pads: 857; 20 M digits with two rows of 152 a hundred times denser: 683;
// one unit of 5 M among 35 of 50 k: 232; one unit of 0.48 M evenly, and with
// two such rows: 31 and 67.  (With the same number of parts in every row, by
// pads: 863, 2030, 6768, 379, 32 and 814; with a wave per pad and two passes:
// 2272, 2645, 2322, 1443, 60 and 239.)
// Peaks and charge sums are integer; the centre and position are FP64
// expressions rounded once to FP32, so the result is exact.
//
// What bounds it: instruction issue (half of it the searches'), then the
// look-back and the tickets.  What k_clu_init found lies in another cache
// line than the ticket, which all blocks add to (in its line: 1.58 ms for
// 0.87).  Peaks kept in registers are not searched for a second time when they
// are written: 63 M digits 849 to 811 us.  A slice of 15 collisions, 63 M digits
// of 540 k pads: 532 us, 0.75 TB/s of the bytes it cannot do without; 0.48 M
// digits of 15 k pads: 22 us.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tpc_track.h"

namespace {

constexpr int TPB = 256;
constexpr int WAVES = TPB / 64;
constexpr int MAX_ROWS = 255;
constexpr int MAX_PADS = 124;        // pads of a block (with one either side and an end: two to a wave's lane)
constexpr int RUN_PADS = 60;         // pads of a run of a part that does not fit (one to a lane)
// digits a block holds in LDS, with the pads either side (60 M digits: 817, 651 and 605 us with 3072, 4096 and 6144, 682
// with 8192 and 512 threads; fewer blocks take fewer tickets, which one counter serves, but leave fewer waves)
constexpr int STAGE_DIGITS = 6144;
constexpr int SPIN_MAX = 1 << 26;

struct CluArgs {
  const int64_t *off;  // [n_units * pads_total + 1]
  const uint16_t *time, *q;
  int64_t n;
  int64_t n_pads;      // n_units * pads_total
  int32_t n_units, n_rows, pads_total, q_min;
  const int32_t *half;  // [n_rows]
  double pw, tb, zoff;
  int64_t cap;
  // outputs
  float *y, *z, *padf, *timef;
  uint16_t *row, *qmax;
  int32_t *qtot;
  int64_t *unit_offsets, *count;
  int32_t *status;
  uint32_t share;      // digits of a part (see first_block)
  int32_t init_blocks;
  int64_t n_blocks;
  bool wide;  // time and q allow loads of four digits (8-byte aligned)
  // workspace
  unsigned long long *ticket;
  int32_t *misordered; // [init_blocks] whether the block of k_clu_init met offsets out of order
  uint64_t *lookback;  // [n_blocks] flag (bits 62-63: 1 count, 2 inclusive sum), clusters; before (flag 0) unit << 8 | row
  int32_t *rbase;      // [n_rows] first pad of each row
};

__device__ __forceinline__ void fail(int32_t *status, int32_t code) { atomicCAS(status, TPC_OK, code); }

// A digit as the searches hold it: its time above its charge, so that digits of
// a pad compare like their times.
__device__ __forceinline__ uint32_t pack(uint16_t t, uint16_t q) { return (uint32_t(t) << 16) | q; }

// A pad's time-ordered digits, n of them: packed in LDS, or in the arrays.
// lower(key): the first digit not below key.  In LDS all lanes take the same
// steps (top: the largest power of two up to the longest list of the block).
struct Packed {
  const uint32_t *d;
  int32_t n, top;
  __device__ __forceinline__ uint32_t at(int32_t i) const { return d[i]; }
  static __device__ __forceinline__ void lower2(const Packed &x, const Packed &y, uint32_t key, int32_t &a, int32_t &b) {
    a = b = 0;
    const int32_t lx = max(x.n, 1), ly = max(y.n, 1);
    for (int32_t st = x.top; st > 0; st >>= 1) {  // both searches step together
      const int32_t i = a + st, j = b + st;
      const uint32_t u = x.d[min(i, lx) - 1], v = y.d[min(j, ly) - 1];
      if (i <= x.n && u < key) a = i;
      if (j <= y.n && v < key) b = j;
    }
  }
};
struct Arrays {
  const uint16_t *t, *q;
  int32_t n;
  __device__ __forceinline__ uint32_t at(int32_t i) const { return pack(t[i], q[i]); }
  __device__ __forceinline__ int32_t lower(uint32_t key) const {
    int32_t a = 0, b = n;
    while (a < b) {
      const int32_t m = (a + b) >> 1;
      if (at(m) < key) a = m + 1; else b = m;
    }
    return a;
  }
  static __device__ __forceinline__ void lower2(const Arrays &x, const Arrays &y, uint32_t key, int32_t &a, int32_t &b) {
    a = x.lower(key);
    b = y.lower(key);
  }
};

struct Peak {
  bool is;
  int32_t t, v, Q, Sp, St;
};

// One neighbour w of a peak candidate at (dp, dt): earlier in (pad, time) order
// it must be smaller, later at most equal.
__device__ __forceinline__ void neighbour(Peak &k, int32_t w, int dp, int32_t dt) {
  if (dp < 0 || (dp == 0 && dt < 0) ? !(w < k.v) : !(w <= k.v)) k.is = false;
  k.Q += w;
  k.Sp += dp * w;
  k.St += dt * w;
}

// The test against the digits of the same pad: the adjacent ones (times
// increase inside a pad), `before` and `after` where the pad has them.
__device__ __forceinline__ Peak own_pad(int32_t q_min, uint32_t d, bool has_before, uint32_t before, bool has_after,
                                        uint32_t after) {
  Peak k;
  k.t = int32_t(d >> 16);
  k.v = int32_t(d & 0xFFFFu);
  k.Q = k.v;
  k.Sp = 0;
  k.St = 0;
  k.is = k.v >= q_min;
  if (has_before && int32_t(before >> 16) == k.t - 1) neighbour(k, int32_t(before & 0xFFFFu), 0, -1);
  if (has_after && int32_t(after >> 16) == k.t + 1) neighbour(k, int32_t(after & 0xFFFFu), 0, 1);
  return k;
}

// The test against the pads below and above (empty at a row's edge): their
// digits of time t-1 .. t+1, from a binary search in each.
template <class L>
__device__ __forceinline__ void other_pads(Peak &k, const L &lo, const L &hi) {
  const uint32_t key = uint32_t(max(k.t - 1, 0)) << 16;  // the first digit of time >= t - 1
  int32_t a, c;
  L::lower2(lo, hi, key, a, c);
#pragma unroll
  for (int m = 0; m < 3; ++m) {
    if (a + m < lo.n) {
      const uint32_t w = lo.at(a + m);
      const int32_t dt = int32_t(w >> 16) - k.t;
      if (dt <= 1) neighbour(k, int32_t(w & 0xFFFFu), -1, dt);
    }
    if (c + m < hi.n) {
      const uint32_t w = hi.at(c + m);
      const int32_t dt = int32_t(w >> 16) - k.t;
      if (dt <= 1) neighbour(k, int32_t(w & 0xFFFFu), 1, dt);
    }
  }
}

// First pad of row r of unit u (the rows' own first pads in rbase), and of the row after it.
__device__ __forceinline__ int64_t row_start(const CluArgs &A, const int32_t *rbase, int u, int r) {
  return min(max(int64_t(u) * A.pads_total + rbase[r], int64_t(0)), A.n_pads);
}
__device__ __forceinline__ int64_t next_start(const CluArgs &A, const int32_t *rbase, int u, int r) {
  return r + 1 < A.n_rows ? row_start(A, rbase, u, r + 1) : row_start(A, rbase, u + 1, 0);
}
// First block of row j where the rows have parts by their digits, off the first
// of these: at least a block each, and one more for each multiple of `share`
// among its digits' numbers.  Known for every row by itself, and so is the sum.
__device__ __forceinline__ int64_t first_block(const CluArgs &A, int64_t j, int64_t off) {
  return int64_t(uint32_t(off) / A.share) + j;
}

__global__ void __launch_bounds__(TPB) k_clu_init(CluArgs A) {
  __shared__ int32_t wsum[WAVES], rbase[TPB];
  const int64_t i0 = int64_t(blockIdx.x) * TPB + threadIdx.x, stride = int64_t(gridDim.x) * TPB;
  const int lane = __lane_id(), wave = threadIdx.x >> 6;
  // exclusive sum of the rows' pads
  const int32_t v = int32_t(threadIdx.x) < A.n_rows ? 2 * A.half[threadIdx.x] : 0;
  int32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int32_t y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[wave] = x;
  __syncthreads();
  for (int w = 0; w < wave; ++w) x += wsum[w];
  rbase[threadIdx.x] = x - v;
  if (blockIdx.x == 0) {
    if (int32_t(threadIdx.x) < A.n_rows) A.rbase[threadIdx.x] = x - v;
    if (threadIdx.x == 0) {
      *A.status = TPC_OK;
      *A.count = 0;
      *A.ticket = 0ull;
    }
  }
  __syncthreads();
  // every row writes its number to its blocks' words
  const int64_t rows = int64_t(A.n_units) * A.n_rows;
  bool bad = false;
  for (int64_t jb = i0 - lane; jb < rows; jb += stride) {  // wave-uniform
    const int64_t j = jb + lane;
    int64_t lo = 0, hi = 0;
    uint64_t word = 0;
    if (j < rows) {
      const int u = int(uint32_t(j) / uint32_t(A.n_rows)), r = int(uint32_t(j) - uint32_t(u) * uint32_t(A.n_rows));
      const int64_t a = A.off[row_start(A, rbase, u, r)], b = j + 1 < rows ? A.off[next_start(A, rbase, u, r)] : A.n;
      word = uint64_t(u) << 8 | uint64_t(r);
      if (a < 0 || b < a || b > A.n || (j == 0 && a != 0)) {
        bad = true;
      } else {
        lo = first_block(A, j, a);
        hi = first_block(A, j + 1, b);
      }
    }
    for (int k = 0; k < 16 && lo < hi; ++k) A.lookback[lo++] = word;
    for (uint64_t m = __ballot(lo < hi); m; m &= m - 1) {  // long rows by the wave
      const int l = __ffsll((unsigned long long)m) - 1;
      const int64_t end = __shfl((long long)hi, l);
      const uint64_t x = __shfl((unsigned long long)word, l);
      for (int64_t k = __shfl((long long)lo, l) + lane; k < end; k += 64) A.lookback[k] = x;
    }
  }
  const int any = __syncthreads_or(bad);
  if (threadIdx.x == 0) A.misordered[blockIdx.x] = any;
}

// A block's run of pads: slot s holds pad first - 1 + s of the row, slots
// 1 .. np the block's own.
struct Run {
  int32_t a[MAX_PADS + 3];  // slot s: digits [a[s], a[s+1]), counted from digit g0 of the arrays
  int64_t g0;
  int32_t first, np;        // own pads of the row
  int32_t row, half;
  int32_t top;              // largest power of two up to the longest slot
  bool ok, fits;
};

// First slot whose end lies past digit e (own digits only).
__device__ __forceinline__ int slot_of(const Run &R, int32_t e) {
  int lo = 1, hi = R.np;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (R.a[mid + 1] <= e) lo = mid + 1; else hi = mid;
  }
  return lo;
}

// np pads of row r of unit u from pad `first` on: their offsets, checked.  SOME:
// as many of them as fit the block's LDS with the pads either side, and where
// not even one does, the pads up to the next that does, with fits = false.
// Run by one wave.
template <bool SOME>
__device__ __forceinline__ void load_run(const CluArgs &A, Run &R, const int32_t *rbase, const int32_t *half, int u, int r,
                                         int32_t first, int32_t np) {
  constexpr int E = SOME ? 1 : 2;  // offsets of a lane
  const int t = __lane_id();
  const int64_t j0 = int64_t(u) * A.pads_total + rbase[r] + first;
  // the offset at the start of pad j0 - 1 + t + 64 e (pads outside the arrays are empty)
  int64_t v[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int i = t + 64 * e;
    v[e] = i < np + 3 ? A.off[min(max(j0 - 1 + i, int64_t(0)), A.n_pads)] : 0;
  }
  bool good = true;
  int32_t len = 0;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int i = t + 64 * e;
    int64_t next = __shfl_down(v[e], 1);
    if (e + 1 < E) {
      const int64_t over = __shfl(v[E - 1], 0);
      if (t == 63) next = over;
    }
    good = good && (i >= np + 3 || (v[e] >= 0 && v[e] <= A.n && (i == np + 2 || v[e] <= next)));
    if (i < np + 2) len = max(len, int32_t(next - v[e]));
  }
  if (t == 0 && j0 == 0) good = good && A.off[0] == 0;
  if (t == 0 && j0 + np >= A.n_pads) good = good && A.off[A.n_pads] == A.n;
  const bool ok = __ballot(good) == ~uint64_t(0);
  const int64_t at = __shfl(v[0], 0) & ~int64_t(3);  // loads of four start at a multiple of four
  if (!ok) len = 0;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) len = max(len, __shfl_xor(len, o));
  const int64_t last = __shfl(E > 1 && np + 2 >= 64 ? v[E - 1] : v[0], (np + 2) & 63);
  int k = np;
  bool fits = ok && last - at <= STAGE_DIGITS;
  if (SOME && ok && !fits && np > 0) {
    // slots 0 .. k + 1 end with the offset of lane k + 2
    k = __popcll(__ballot(t < np + 3 && v[0] - at <= STAGE_DIGITS)) - 3;
    fits = k > 0;
    if (!fits) {  // pad first + t by itself, with its neighbours
      const bool one = __shfl_down(v[0], 3) - (v[0] & ~int64_t(3)) <= STAGE_DIGITS;
      k = min(np, __ffsll((unsigned long long)__ballot(one || t >= np)) - 1);
    }
  }
#pragma unroll
  for (int e = 0; e < E; ++e)
    if (t + 64 * e < np + 3) R.a[t + 64 * e] = ok ? int32_t(v[e] - at) : 0;
  if (t == 0) {
    if (!ok) fail(A.status, TPC_E_INVALID);
    R.g0 = at;
    R.first = first;
    R.np = k;
    R.row = r;
    R.half = half[r];
    R.top = len > 0 ? 1 << (31 - __clz(len)) : 0;
    R.ok = ok;
    R.fits = fits;
  }
}

// What a block does: np pads of row r of unit u from `first` on; lead: the
// row's first ones.
struct Part {
  int32_t u, r, first, np;
  bool lead;
};

// The part of block vb: of a row cut into parts of like many digits, a pad to
// the part that its first digit lies in.  Run by one wave.
__device__ __forceinline__ Part cut_part(const CluArgs &A, const int32_t *rbase, const int32_t *half, int64_t vb) {
  const int lane = __lane_id();
  const uint64_t word = A.lookback[vb];
  Part P;
  P.u = int32_t(word >> 8);
  P.r = int32_t(word & 0xFF);
  const int64_t j = int64_t(P.u) * A.n_rows + P.r, rows = int64_t(A.n_units) * A.n_rows;
  const int32_t pads = min(max(2 * half[P.r], 0), A.pads_total);
  const int64_t s = row_start(A, rbase, P.u, P.r), e = min(s + pads, A.n_pads);
  const int64_t a = A.off[s], b = j + 1 < rows ? A.off[next_start(A, rbase, P.u, P.r)] : A.n;
  int64_t v[2];  // most rows' pads, on their way with a and b
#pragma unroll
  for (int h = 0; h < 2; ++h) v[h] = s + 64 * h + lane < e ? A.off[s + 64 * h + lane] : INT64_MAX;
  const int64_t b0 = first_block(A, j, a), k = vb - b0;
  const uint32_t c = uint32_t(first_block(A, j + 1, b) - b0);
  const int64_t step = int64_t(uint32_t(b - a) / c) + 1, from = a + k * step, to = from + step;
  int32_t na = 0, nb = 0;
  for (int64_t i = s; i < e; i += 128) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (i > s) v[h] = i + 64 * h + lane < e ? A.off[i + 64 * h + lane] : INT64_MAX;
      na += __popcll(__ballot(v[h] < from));
      nb += __popcll(__ballot(v[h] < to));
    }
  }
  P.first = k == 0 ? 0 : na;
  P.np = (k + 1 == int64_t(c) ? pads : nb) - P.first;
  P.lead = k == 0;
  return P;
}

// Clusters of the blocks before this one: publishes the block's count, adds
// up its predecessors' (64 at a time) until it meets an inclusive sum, and
// publishes its own.  The count travels in the same 64-bit word as its flag,
// so relaxed device-scope atomics suffice.  Blocks are taken by ticket, so
// every predecessor has started, and none waits for a later one.
__device__ __forceinline__ int64_t look_back(const CluArgs &A, int64_t vb, int32_t count) {
  constexpr uint64_t CNT = uint64_t(1) << 62, INC = uint64_t(2) << 62, VAL = CNT - 1;
  const int lane = __lane_id();
  uint64_t *lb = A.lookback;
  int64_t before = 0;
  if (vb > 0) {
    if (lane == 0) __hip_atomic_store(&lb[vb], CNT | uint64_t(count), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int64_t top = vb - 1;  // lane k reads block top - k
    for (int spins = 0;;) {
      const int64_t j = top - lane;
      const uint64_t v = j >= 0 ? __hip_atomic_load(&lb[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : INC;
      const uint64_t inc = __ballot((v >> 62) == 2), empty = __ballot((v >> 62) == 0);
      const int first = inc ? __ffsll((unsigned long long)inc) - 1 : 64;
      const uint64_t need = first < 64 ? ((uint64_t(1) << first) << 1) - 1 : ~uint64_t(0);
      if (empty & need) {
        if (++spins > SPIN_MAX) {
          if (lane == 0) fail(A.status, TPC_E_HIP);
          break;
        }
        __builtin_amdgcn_s_sleep(1);
        continue;
      }
      int64_t x = lane <= first ? int64_t(v & VAL) : 0;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
      before += x;
      if (first < 64) break;
      top -= 64;
    }
  }
  if (lane == 0)
    __hip_atomic_store(&lb[vb], INC | uint64_t(before + count), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return before;
}

// Cluster c from peak k of slot s.
__device__ __forceinline__ void write_cluster(const CluArgs &A, const Run &R, int s, const Peak &k, int64_t c) {
  // the oracle's order of operations, each rounded (no fused multiply-add)
#pragma clang fp contract(off)
  if (c >= A.cap) return;  // the last block reports it
  const double padf = double(R.first + s - 1) + double(k.Sp) / double(k.Q);
  const double timef = double(k.t) + double(k.St) / double(k.Q);
  A.y[c] = float((padf + 0.5 - double(R.half)) * A.pw);
  A.z[c] = float((timef + 0.5) * A.tb - A.zoff);
  A.padf[c] = float(padf);
  A.timef[c] = float(timef);
  A.row[c] = uint16_t(R.row);
  A.qmax[c] = uint16_t(k.v);
  A.qtot[c] = k.Q;
}

// The lists of slot s (neighbours stay in the row).
template <class L, class F>
__device__ __forceinline__ void lists(const Run &R, int s, F list, L &lo, L &hi) {
  lo = list(s - 1);
  hi = list(s + 1);
  if (R.first + s - 1 == 0) lo.n = 0;
  if (R.first + s == 2 * R.half) hi.n = 0;
}

// Pads that do not fit in LDS even one by one: a wave per pad reads the arrays,
// once to count (EMIT false: into cnt) and once to write from place o0 on.
template <bool EMIT>
__device__ __forceinline__ void sweep(const CluArgs &A, const Run &R, int32_t *cnt, int64_t o0) {
  const int lane = __lane_id();
  auto list = [&](int s) {
    Arrays L;
    L.t = A.time + R.g0 + R.a[s];
    L.q = A.q + R.g0 + R.a[s];
    L.n = R.a[s + 1] - R.a[s];
    return L;
  };
  for (int p = threadIdx.x >> 6; p < R.np; p += WAVES) {
    const Arrays own = list(p + 1);
    Arrays lo, hi;
    lists(R, p + 1, list, lo, hi);
    int64_t o = o0;
    if (EMIT)
      for (int x = 0; x < p; ++x) o += cnt[x];
    int32_t n = 0;
    for (int32_t i0 = 0; i0 < own.n; i0 += 64) {
      const int32_t i = i0 + lane;
      Peak k;
      k.is = false;
      if (i < own.n) {
        const bool hb = i > 0, ha = i + 1 < own.n;
        const uint32_t d = own.at(i), b = hb ? own.at(i - 1) : 0, a = ha ? own.at(i + 1) : 0;
        if (hb && (d >> 16) <= (b >> 16)) fail(A.status, TPC_E_INVALID);  // times must increase
        k = own_pad(A.q_min, d, hb, b, ha, a);
        if (k.is) other_pads(k, lo, hi);
      }
      const uint64_t m = __ballot(k.is);
      if (EMIT && k.is) write_cluster(A, R, p + 1, k, o + n + __popcll(m & ((1ull << lane) - 1ull)));
      n += __popcll(m);
    }
    if (!EMIT && lane == 0) cnt[p] = n;
  }
}

__global__ void __launch_bounds__(TPB) k_clu_find(CluArgs A) {
  __shared__ __align__(16) uint32_t dig[STAGE_DIGITS + 4];
  __shared__ uint16_t found[STAGE_DIGITS];         // per wave, from its first digit's place: candidates, then peaks
  __shared__ uint32_t starts[STAGE_DIGITS / 32 + 2];  // bit e: digit e is the first of its pad
  __shared__ Run R;
  __shared__ Part part;
  __shared__ int32_t rbase[MAX_ROWS], half[MAX_ROWS];  // the rows' first pads and half pads
  __shared__ int32_t cnt[MAX_PADS];                // per pad (sweep)
  __shared__ int32_t wcnt[WAVES];
  __shared__ int64_t s_vb, s_before;
  const int lane = __lane_id(), wave = threadIdx.x >> 6;
  if (threadIdx.x == 0) s_vb = int64_t(atomicAdd(A.ticket, 1ull));
  for (int i = threadIdx.x; i < STAGE_DIGITS / 32 + 2; i += TPB) starts[i] = 0;
  if (int32_t(threadIdx.x) < A.n_rows) {
    rbase[threadIdx.x] = A.rbase[threadIdx.x];
    half[threadIdx.x] = A.half[threadIdx.x];
  }
  const bool bad = lane < A.init_blocks && A.misordered[lane] != 0;
  __syncthreads();
  const int64_t vb = s_vb;
  if (__ballot(bad)) {  // the words say nothing then: every block sees it
    if (threadIdx.x == 0) fail(A.status, TPC_E_INVALID);
    return;
  }
  if (wave == 0) {
    const Part P = cut_part(A, rbase, half, vb);
    load_run<false>(A, R, rbase, half, P.u, P.r, P.first, min(P.np, MAX_PADS));
    if (lane == 0) part = P;
  }
  __syncthreads();
  const int u = part.u, r = part.r;
  const int32_t first = part.first, np = part.np;
  const bool whole = np <= MAX_PADS && R.fits;

  auto slot_list = [&](int s) {
    Packed L;
    L.d = dig + R.a[s];
    L.n = R.a[s + 1] - R.a[s];
    L.top = R.top;
    return L;
  };
  auto peak = [&](int32_t e, int &s) {
    s = slot_of(R, e);
    const bool hb = e > R.a[s], ha = e + 1 < R.a[s + 1];
    Peak k = own_pad(A.q_min, dig[e], hb, dig[max(e - 1, 0)], ha, dig[e + 1]);
    Packed lo, hi;
    lists(R, s, slot_list, lo, hi);
    other_pads(k, lo, hi);
    return k;
  };
  uint16_t *list;
  constexpr int KEPT = 4;
  struct Kept {
    int32_t at, where, Q, Sp, St;  // place among the wave's peaks (-1: none), digit << 8 | slot
  } kept[KEPT];
  int32_t n_kept = 0;
  // The peaks of the run's digits in this wave's share, `mine` of them, the
  // first n_kept in kept and the rest in list; wcnt: those of each wave.
  auto find = [&](int32_t n) -> int32_t {
    int32_t mine = 0;
    const int32_t m = R.a[n + 2];
    if (A.wide) {
      for (int32_t e = int32_t(threadIdx.x) * 4; e < m; e += TPB * 4) {
        const int64_t g = R.g0 + e;
        uint4 v;
        if (g + 4 <= A.n) {
          const ushort4 t = *reinterpret_cast<const ushort4 *>(A.time + g), q = *reinterpret_cast<const ushort4 *>(A.q + g);
          v = make_uint4(pack(t.x, q.x), pack(t.y, q.y), pack(t.z, q.z), pack(t.w, q.w));
        } else {  // the arrays' last digits
          v.x = g < A.n ? pack(A.time[g], A.q[g]) : 0;
          v.y = g + 1 < A.n ? pack(A.time[g + 1], A.q[g + 1]) : 0;
          v.z = g + 2 < A.n ? pack(A.time[g + 2], A.q[g + 2]) : 0;
          v.w = 0;
        }
        *reinterpret_cast<uint4 *>(dig + e) = v;
      }
    } else {
      for (int32_t e = threadIdx.x; e < m; e += TPB) {
        const int64_t g = R.g0 + e;
        if (g < A.n) dig[e] = pack(A.time[g], A.q[g]);
      }
    }
    if (int(threadIdx.x) <= n) {
      const int32_t e = R.a[threadIdx.x + 1];
      atomicOr(&starts[e >> 5], 1u << (e & 31));
    }
    __syncthreads();
    // the wave's share of the own digits: whole groups of 64
    const int32_t e0 = R.a[1], e1 = R.a[n + 1];
    const int32_t groups = (e1 - e0 + 63) >> 6, per = (groups + WAVES - 1) / WAVES;
    const int32_t w0 = min(e1, e0 + wave * per * 64), w1 = min(e1, w0 + per * 64);
    list = found + (w0 - e0);
    int32_t n_cand = 0;
    for (int32_t eb = w0; eb < w1; eb += 64) {
      const int32_t e = eb + lane;
      bool c = false;
      if (e < w1) {
        const bool hb = !((starts[e >> 5] >> (e & 31)) & 1u), ha = !((starts[(e + 1) >> 5] >> ((e + 1) & 31)) & 1u);
        const uint32_t d = dig[e], b = dig[max(e - 1, 0)], a = dig[e + 1];
        if (hb && (d >> 16) <= (b >> 16)) fail(A.status, TPC_E_INVALID);  // times must increase
        c = own_pad(A.q_min, d, hb, b, ha, a).is;
      }
      const uint64_t k = __ballot(c);
      if (c) list[n_cand + __popcll(k & ((1ull << lane) - 1ull))] = uint16_t(e);
      n_cand += __popcll(k);
    }
    __builtin_amdgcn_wave_barrier();
    // the peaks among them: the first KEPT * 64 candidates' in registers, the rest in the list's front
#pragma unroll
    for (int x = 0; x < KEPT; ++x) {
      kept[x].at = -1;
      if (x * 64 >= n_cand) continue;
      const int32_t i = x * 64 + lane;
      int32_t e = 0;
      int s = 0;
      Peak k;
      k.is = false;
      if (i < n_cand) {
        e = list[i];
        k = peak(e, s);
      }
      const uint64_t m = __ballot(k.is);
      if (k.is) kept[x] = Kept{mine + int32_t(__popcll(m & ((1ull << lane) - 1ull))), e << 8 | s, k.Q, k.Sp, k.St};
      mine += __popcll(m);
    }
    n_kept = mine;
    __builtin_amdgcn_wave_barrier();
    for (int32_t i0 = KEPT * 64; i0 < n_cand; i0 += 64) {
      const int32_t i = i0 + lane;
      int32_t e = 0;
      bool is = false;
      if (i < n_cand) {
        e = list[i];
        int s;
        is = peak(e, s).is;
      }
      const uint64_t k = __ballot(is);
      if (is) list[mine + __popcll(k & ((1ull << lane) - 1ull))] = uint16_t(e);
      mine += __popcll(k);
      __builtin_amdgcn_wave_barrier();
    }
    if (lane == 0) wcnt[wave] = mine;
    __syncthreads();
    return mine;
  };
  // and their clusters, from place o of the output on
  auto write = [&](int32_t mine, int64_t o) {
    for (int w = 0; w < wave; ++w) o += wcnt[w];
#pragma unroll
    for (int x = 0; x < KEPT; ++x)
      if (kept[x].at >= 0) {
        const uint32_t d = dig[kept[x].where >> 8];
        const Peak k{true, int32_t(d >> 16), int32_t(d & 0xFFFFu), kept[x].Q, kept[x].Sp, kept[x].St};
        write_cluster(A, R, kept[x].where & 0xFF, k, o + kept[x].at);
      }
    for (int32_t i = n_kept + lane; i < mine; i += 64) {
      int s;
      const Peak k = peak(list[i], s);
      write_cluster(A, R, s, k, o + i);
    }
  };
  auto sum = [&]() {
    int32_t all = 0;
    for (int w = 0; w < WAVES; ++w) all += wcnt[w];
    return all;
  };
  auto place = [&](int32_t count) {  // of the block's first cluster, by wave 0
    const int64_t before = look_back(A, vb, count);
    if (lane == 0) s_before = before;
  };
  if (__builtin_expect(whole, 1)) {
    const int32_t mine = find(np);
    if (wave == 0) place(sum());
    __syncthreads();
    write(mine, s_before);
  } else {
    // Too many digits (single pads denser than a part is meant to be) or pads: a
    // run at a time, once to count and once to write.
    int32_t total = 0;
    const bool keep = np <= MAX_PADS;  // cnt holds all of the part's pads
    auto next_run = [&](int32_t p) {
      __syncthreads();
      if (wave == 0) load_run<true>(A, R, rbase, half, u, r, first + p, min(np - p, RUN_PADS));
      for (int i = threadIdx.x; i < STAGE_DIGITS / 32 + 2; i += TPB) starts[i] = 0;
      __syncthreads();
    };
    for (int32_t p = 0; p < np;) {
      next_run(p);
      const int32_t got = R.np;
      if (R.fits) {
        find(got);
        total += sum();
      } else if (R.ok) {
        int32_t *c = cnt + (keep ? p : 0);
        sweep<false>(A, R, c, 0);
        __syncthreads();
        for (int x = 0; x < got; ++x) total += c[x];
      }
      p += got;
    }
    if (wave == 0) place(total);
    __syncthreads();
    int64_t o = s_before;
    for (int32_t p = 0; p < np;) {
      next_run(p);
      const int32_t got = R.np;
      if (R.fits) {
        const int32_t mine = find(got);
        write(mine, o);
        o += sum();
      } else if (R.ok) {
        int32_t *c = cnt + (keep ? p : 0);
        if (!keep) sweep<false>(A, R, c, 0);
        __syncthreads();
        sweep<true>(A, R, c, o);
        for (int x = 0; x < got; ++x) o += c[x];
      }
      p += got;
    }
    __syncthreads();
    if (threadIdx.x < WAVES) wcnt[threadIdx.x] = threadIdx.x == 0 ? total : 0;
    __syncthreads();
  }
  if (r == 0 && part.lead && threadIdx.x == 0) A.unit_offsets[u] = s_before;
  if (vb == A.n_blocks - 1 && threadIdx.x == 0) {
    const int64_t all = s_before + sum();
    *A.count = all;
    A.unit_offsets[A.n_units] = all;
    if (all > A.cap) fail(A.status, TPC_E_CAPACITY);
  }
}

constexpr int INIT_BLOCKS = 32;  // their findings take the words after the line of the ticket

// Digits of a part.  Many blocks: 4096, which leaves room for a dense part's
// edge pads (63 M digits evenly: 889, 877, 877 and 865 us with 3600, 4096, 4608
// and 5120; 20 M mostly of one unit 464, 465, 514 and 540).  Up to four times the 1024
// blocks that run at a time: 3234, or the last ones are too few to fill the
// chip (one unit of 5 M: 103 us, with 4096 112, with 5632 127).  A few hundred
// blocks: by the mean row, whose pads are three parts (one unit of 1 M: 42 us, in two
// to three 46), or two to three where three would hold under 2048 digits and
// cost little but their fixed part (one unit of 0.48 M: 25.0 and 24.6 us).
// Never more blocks than the workspace has words.
uint32_t digits_per_part(int64_t n, int64_t n_pads, int64_t rows) {
  const int64_t few = STAGE_DIGITS * 10 / 19, many = 4096, blocks = n / few + rows, mean = n / rows;
  int64_t share = blocks > 4096 ? many : few;
  if (blocks <= 512) {
    const int64_t splits = n_pads / rows / 40 > 1 ? n_pads / rows / 40 : 1, low = mean * 2 / 3 < 2048 ? mean * 2 / 3 : 2048;
    share = (mean / splits > low ? mean / splits : low) + 1;
  }
  const int64_t room = n_pads / 2 - rows;
  if (room < 1) return uint32_t(1) << 31;  // a part a row: n is below it
  return uint32_t(share > n / room + 1 ? share : n / room + 1);
}

size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

}  // namespace

extern "C" size_t tpc_clusterize_workspace_size(int32_t n_units, const tpc_pad_geometry_t *g) {
  if (!g || n_units < 1 || g->n_rows < 1 || g->n_rows > MAX_ROWS || g->pads_total < 1) return 0;
  const int64_t n_pads = int64_t(n_units) * g->pads_total;
  const int64_t rows = int64_t(n_units) * g->n_rows;
  const int64_t blocks = n_pads / 2 > rows ? n_pads / 2 : rows;  // parts have at least two pads on average
  return 256 + align256(sizeof(int32_t) * MAX_ROWS) + align256(sizeof(uint64_t) * size_t(blocks));
}

extern "C" int tpc_clusterize(const tpc_digits_t *digits, const tpc_pad_geometry_t *g,
                              const tpc_clusterizer_params_t *params, tpc_cluster_out_t *out, void *workspace,
                              size_t workspace_bytes, void *stream) {
  if (!digits || !g || !params || !out) return TPC_E_INVALID;
  if (digits->n < 0 || digits->n >= (int64_t(1) << 31) || digits->n_units < 1 || !digits->pad_offsets ||
      (digits->n > 0 && (!digits->time || !digits->q)))
    return TPC_E_INVALID;
  if (g->n_rows < 1 || g->n_rows > MAX_ROWS || !g->half || g->pads_total < 1 || !(g->pad_width > 0.0f) ||
      !(g->time_bin > 0.0f))
    return TPC_E_INVALID;
  if (params->q_min < 1) return TPC_E_INVALID;
  if (out->cap < 0 || !out->unit_offsets || !out->count || !out->status) return TPC_E_INVALID;
  if (out->cap > 0 && (!out->y || !out->z || !out->row || !out->qtot || !out->qmax || !out->pad || !out->time))
    return TPC_E_INVALID;
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255)) return TPC_E_INVALID;
  if (workspace_bytes < tpc_clusterize_workspace_size(digits->n_units, g)) return TPC_E_NOMEM;

  CluArgs A;
  A.off = digits->pad_offsets;
  A.time = digits->time;
  A.q = digits->q;
  A.n = digits->n;
  A.n_units = digits->n_units;
  A.n_rows = g->n_rows;
  A.pads_total = g->pads_total;
  A.n_pads = int64_t(digits->n_units) * g->pads_total;
  A.q_min = params->q_min;
  A.half = g->half;
  A.pw = g->pad_width;
  A.tb = g->time_bin;
  A.zoff = g->z_offset;
  A.cap = out->cap;
  A.y = out->y;
  A.z = out->z;
  A.padf = out->pad;
  A.timef = out->time;
  A.row = out->row;
  A.qmax = out->qmax;
  A.qtot = out->qtot;
  A.unit_offsets = out->unit_offsets;
  A.count = out->count;
  A.status = out->status;
  char *ws = static_cast<char *>(workspace);
  A.ticket = reinterpret_cast<unsigned long long *>(ws);
  A.rbase = reinterpret_cast<int32_t *>(ws + 256);
  A.lookback = reinterpret_cast<uint64_t *>(ws + 256 + align256(sizeof(int32_t) * MAX_ROWS));
  A.misordered = reinterpret_cast<int32_t *>(ws + 128);  // not in the line of the ticket
  const int64_t rows = int64_t(A.n_units) * A.n_rows, rb = (rows + TPB - 1) / TPB;
  A.share = digits_per_part(A.n, A.n_pads, rows);
  A.n_blocks = A.n / A.share + rows;
  A.init_blocks = int32_t(rb > INIT_BLOCKS ? INIT_BLOCKS : rb);
  A.wide = ((reinterpret_cast<uintptr_t>(A.time) | reinterpret_cast<uintptr_t>(A.q)) & 7) == 0;

  hipStream_t st = static_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(k_clu_init, dim3(unsigned(A.init_blocks)), dim3(TPB), 0, st, A);
  hipLaunchKernelGGL(k_clu_find, dim3(unsigned(A.n_blocks)), dim3(TPB), 0, st, A);
  return hipGetLastError() == hipSuccess ? TPC_OK : TPC_E_HIP;
}

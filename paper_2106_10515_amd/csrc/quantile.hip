// Quantile bucketing of dense data (paper Algorithm 1): for each projection
// a_p, the objects are ranked by the QALSH value a_p . x_i (ties by id) and
// the ranks split evenly into t buckets, rank r going to bucket
// floor(r t / n); bucket b starts at rank ceil(b n / t).
//
//   values    exact float64 values of all tables (the attributes summed in
//             order, one rounding per addition, products exact), as order-
//             preserving 64-bit patterns (k_qv).
//   ranks     a sample sort, several tables at once: every 16th value of a
//             sorted sample splits the values into cells of about QF_MEAN
//             objects, one pass counts and one scatters (k_qs_*), and each
//             cell is ranked in LDS (k_qs_cell).  Cells that ties or chance
//             made hard go to an exact comparison sort in LDS
//             (k_qs_cell_exact); a table with a cell beyond even that (one
//             value shared by thousands of objects) is ranked by a stable
//             radix sort of its (value, id) pairs (k_qr_*), decided on the
//             device.
//   buckets   every bucket's ids in ascending order: by counting the smaller ids
//             of buckets of at most QT_MAX objects, ranked in LDS per bucket
//             when buckets hold at most QS_MAX objects, else by a stable sort
//             of the ids keyed by bucket (rank-derived).
#include <math.h>

#include <algorithm>

#include "common.hpp"
#include "radix.hpp"

namespace geek {

constexpr int QV_ROWS = 256;   // rows per block, one per thread
constexpr int QV_CHUNK = 8;    // attributes staged at a time
constexpr int QV_STR = QV_CHUNK + 4;
constexpr int QV_GRP = 8;      // projections per step
constexpr int QV_ATT = 2;      // attributes per step (with one: 5.5 instead of 4.4 ms)

// Projections widened to float64, attribute-major in groups of QV_GRP:
// Ad[p / QV_GRP][t][p % QV_GRP], zero past m and d (to a multiple of QV_CHUNK).
__global__ void k_qv_prep(const float* __restrict__ A, int m, int d, int dpad, double* __restrict__ Ad, int32_t* st) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  const int groups = (m + QV_GRP - 1) / QV_GRP;
  if (q >= groups * dpad * QV_GRP) return;
  const int u = q % QV_GRP, t = (q / QV_GRP) % dpad, p = q / (QV_GRP * dpad) * QV_GRP + u;
  const float v = p < m && t < d ? A[(int64_t)p * d + t] : 0.f;
  if (!isfinite(v)) set_status(st, GEEK_ERR_NONFINITE);
  Ad[q] = (double)v;
}

// Values of projections p0 .. p0 + NG * QV_GRP - 1: a thread owns a row and
// keeps one float64 chain per projection; rows pass through LDS a chunk of
// attributes at a time (coalesced loads, the next chunk's in flight during the
// current one's arithmetic), the projections come through scalar loads.  Each
// chain adds in attribute order, one rounding per addition (the product of
// two float32 values is exact in float64, so the fused form rounds once, as
// the addition does).  The value is written as an order-preserving pattern
// (negative values complemented, positive ones with the sign bit set; -0
// becomes +0 so that equal values compare equal).  A non-finite x makes every
// chain of its row non-finite (finite float32 products cannot).
// Bound: float64 issue, 2 d m flop per row (1.3 ms at n = 10^7, d = 128,
// m = 40), then the 8 m n bytes written; 4.4 ms there (17.4 with eight chains per
// thread and both operands converted from LDS at every use).
template <int NG>
__global__ __launch_bounds__(QV_ROWS) void k_qv(const float* __restrict__ X, int64_t ldx, int64_t n, int d, int dpad,
                                                const double* __restrict__ Ad, int p0, int m,
                                                uint64_t* __restrict__ kv, int32_t* st) {
  __shared__ __attribute__((aligned(16))) float xs[2][QV_ROWS * QV_STR];
  const int64_t i0 = (int64_t)blockIdx.x * QV_ROWS;
  constexpr int LD = QV_ROWS * QV_CHUNK / QV_ROWS;  // values staged per thread
  float pre[LD];
  const int lc = threadIdx.x % QV_CHUNK, lr = threadIdx.x / QV_CHUNK;
  // (past d the projections are zero, so the last attribute may stand there)
  const float* xrow[LD];
#pragma unroll
  for (int q = 0; q < LD; ++q) {
    const int64_t r = i0 + lr + q * (QV_ROWS / QV_CHUNK);
    xrow[q] = X + (r < n ? r : n - 1) * ldx;
  }
  auto fetch = [&](int c0) {
    const int c = c0 + lc < d ? c0 + lc : d - 1;
#pragma unroll
    for (int q = 0; q < LD; ++q) pre[q] = xrow[q][c];
  };
  auto stage = [&](float* to) {
#pragma unroll
    for (int q = 0; q < LD; ++q) to[(lr + q * (QV_ROWS / QV_CHUNK)) * QV_STR + lc] = pre[q];
  };
  double acc[NG * QV_GRP];
#pragma unroll
  for (int u = 0; u < NG * QV_GRP; ++u) acc[u] = 0.0;
  fetch(0);
  stage(xs[0]);
  __syncthreads();
  for (int c0 = 0, b = 0; c0 < dpad; c0 += QV_CHUNK, b ^= 1) {
    if (c0 + QV_CHUNK < dpad) fetch(c0 + QV_CHUNK);
    double x[QV_CHUNK];
    const float* xr = xs[b] + threadIdx.x * QV_STR;
#pragma unroll
    for (int t = 0; t < QV_CHUNK; t += 4) {
      const float4 v = *reinterpret_cast<const float4*>(xr + t);
      x[t] = (double)v.x;
      x[t + 1] = (double)v.y;
      x[t + 2] = (double)v.z;
      x[t + 3] = (double)v.w;
    }
    // QV_ATT attributes x QV_GRP projections per step, the next step's values
    // loading into scalar registers meanwhile (the empty asm ties the loads of
    // a step to the sums of the one before: left free, the compiler loads all
    // steps first and spills scalar registers)
    constexpr int PER = QV_CHUNK / QV_ATT, STEPS = NG * PER;
    double cur[QV_ATT * QV_GRP], nxt[QV_ATT * QV_GRP];
    auto load = [&](int z, double* w, double (&to)[QV_ATT * QV_GRP]) {
      int off = ((p0 / QV_GRP + z / PER) * dpad + c0 + z % PER * QV_ATT) * QV_GRP;
      asm volatile("" : "+v"(off), "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]), "+v"(w[4]), "+v"(w[5]), "+v"(w[6]),
                   "+v"(w[7]));
      const double* ag = Ad + __builtin_amdgcn_readfirstlane(off);
#pragma unroll
      for (int u = 0; u < QV_ATT * QV_GRP; ++u) to[u] = ag[u];
    };
    load(0, acc, cur);
#pragma unroll
    for (int z = 0; z < STEPS; ++z) {
      if (z + 1 < STEPS) load(z + 1, acc + z / PER * QV_GRP, nxt);
#pragma unroll
      for (int t = 0; t < QV_ATT; ++t)
#pragma unroll
        for (int u = 0; u < QV_GRP; ++u) {
          double& a = acc[z / PER * QV_GRP + u];
          a = __fma_rn(cur[t * QV_GRP + u], x[z % PER * QV_ATT + t], a);
        }
#pragma unroll
      for (int u = 0; u < QV_ATT * QV_GRP; ++u) cur[u] = nxt[u];
    }
    if (c0 + QV_CHUNK < dpad) stage(xs[b ^ 1]);
    __syncthreads();
  }
  const int64_t i = i0 + threadIdx.x;
  if (i >= n) return;
  bool finite = true;
#pragma unroll
  for (int u = 0; u < NG * QV_GRP; ++u) {
    finite = finite && isfinite(acc[u]);
    uint64_t uv = (uint64_t)__double_as_longlong(acc[u] + 0.0);  // -0 -> +0
    uv = (uv >> 63) ? ~uv : (uv | 0x8000000000000000ull);
    if (p0 + u < m) kv[(int64_t)(p0 + u) * n + i] = uv;
  }
  if (!finite) set_status(st, GEEK_ERR_NONFINITE);
}

// ---------------------------------------------------------------- sample sort
// n = 10^7, m = 40, t = 10^4, all tables: ranks 11 ms (sample 0.3, count 3.3,
// scatter 4.3, cells 3.2), buckets 4.3 ms; eight stable radix passes over 12-byte
// items took 53 ms and the buckets 9.9 ms.  The passes move 8 + 8, 8 + 8 and
// 8 + 4 bytes per (table, object), about 18 GB or 4 ms at the copy rate; the
// rest is the scatter's short runs and LDS latency.
constexpr int QF_MEAN = 3000;        // objects per cell aimed at (n / cells is at most this)
constexpr int QF_CELLS_MAX = 8192;   // cells per table (splitters and counts in LDS)
constexpr int QF_OVER = 16;          // sample values per cell: nearly all cells stay below 2.6 x the mean
constexpr int QF_CHUNK = 16384;      // sample values sorted by one block
constexpr int QF_BLK = 32768;        // objects counted and scattered by one block
constexpr int QF_STAGE = 8192;       // records staged at a time by the scatter
constexpr int QF_CAP = 4096;         // cell size ranked by k_qs_cell
constexpr int QF_CAP_EXACT = 8192;   // ... by k_qs_cell_exact
constexpr int QF_CROWD = 24;         // objects of one LDS slot before a cell counts as hard

// Cells of a table of n objects (a power of two), or 0: too many objects.
// Above QF_CELLS_MAX * QF_MEAN the radix sort carries keys and ids (it did so
// at every size before: 63 ms of passes at n = 10^7, m = 40).
static int q_cells(int64_t n) {
  int c = 1;
  while ((int64_t)c * QF_MEAN < n && c <= QF_CELLS_MAX) c *= 2;
  return c <= QF_CELLS_MAX ? c : 0;
}

// Bitonic sort of P (a power of two) LDS items, ascending.
template <class Less, class Swap>
GEEK_D void lds_bitonic(int P, Less less, Swap swap) {
  for (int kk = 2; kk <= P; kk <<= 1)
    for (int jj = kk >> 1; jj > 0; jj >>= 1) {
      for (int q = threadIdx.x; q < P / 2; q += blockDim.x) {
        const int lo = 2 * q - (q & (jj - 1)), hi = lo + jj;
        const bool up = (lo & kk) == 0;
        if (up ? less(hi, lo) : less(lo, hi)) swap(lo, hi);
      }
      __syncthreads();
    }
}

// One block sorts one chunk of a table's sample (value j of the sample is the
// value at a pseudo-random place of the j-th of S equal stretches).
__global__ __launch_bounds__(1024) void k_qs_sample(const uint64_t* __restrict__ kv, int64_t n, int S,
                                                    uint64_t* __restrict__ smp) {
  extern __shared__ __attribute__((aligned(16))) uint64_t qs_v[];
  const int len = S < QF_CHUNK ? S : QF_CHUNK;
  const uint64_t* src = kv + (int64_t)blockIdx.y * n;
  for (int q = threadIdx.x; q < len; q += blockDim.x) {
    const uint64_t j = (uint64_t)blockIdx.x * len + q;
    const uint64_t lo = j * (uint64_t)n / S, hi = (j + 1) * (uint64_t)n / S;
    qs_v[q] = src[lo + (hi > lo ? fmix32((uint32_t)j * 2654435761u + blockIdx.y) % (hi - lo) : 0)];
  }
  __syncthreads();
  lds_bitonic(
      len, [&](int a, int b) { return qs_v[a] < qs_v[b]; },
      [&](int a, int b) {
        const uint64_t t = qs_v[a];
        qs_v[a] = qs_v[b];
        qs_v[b] = t;
      });
  for (int q = threadIdx.x; q < len; q += blockDim.x) smp[(int64_t)blockIdx.y * S + (int64_t)blockIdx.x * len + q] = qs_v[q];
}

// Splitter r = the sample value of rank (r + 1) QF_OVER over all chunks
// (ties ranked by chunk, then position).
__global__ void k_qs_split(const uint64_t* __restrict__ smp, int S, int C, uint64_t* __restrict__ spl) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= S) return;
  const uint64_t* v = smp + (int64_t)blockIdx.y * S;
  const int len = S < QF_CHUNK ? S : QF_CHUNK, mine = q / len;
  const uint64_t x = v[q];
  int rank = q - mine * len;
  for (int ch = 0; ch < S / len; ++ch) {
    if (ch == mine) continue;
    int lo = 0, hi = len;  // values below x, and equal ones of earlier chunks
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      const uint64_t y = v[(int64_t)ch * len + mid];
      if (y < x || (y == x && ch < mine)) lo = mid + 1; else hi = mid;
    }
    rank += lo;
  }
  if (rank > 0 && rank % QF_OVER == 0) spl[(int64_t)blockIdx.y * C + rank / QF_OVER - 1] = x;
  if (q == 0) spl[(int64_t)blockIdx.y * C + C - 1] = ~0ull;  // no finite value's pattern
}

// Cell of every value (the number of splitters at or below it), its place
// within (block, cell), and its offset from the cell's lower splitter in at
// most 32 bits (the width's leading ones); counts per (block, cell).
__global__ __launch_bounds__(1024) void k_qs_count(const uint64_t* __restrict__ kv, int64_t n, int C,
                                                   const uint64_t* __restrict__ spl, uint2* __restrict__ tmp,
                                                   uint32_t* __restrict__ cnt) {
  extern __shared__ __attribute__((aligned(16))) uint64_t qs_v[];  // [C] splitters, [C] counts
  uint32_t* h = reinterpret_cast<uint32_t*>(qs_v + C);
  const int64_t tb = (int64_t)blockIdx.y;
  for (int q = threadIdx.x; q < C; q += 1024) {
    qs_v[q] = spl[tb * C + q];
    h[q] = 0u;
  }
  __syncthreads();
  const int64_t i0 = (int64_t)blockIdx.x * QF_BLK;
  constexpr int E = 8;  // searches of a thread that advance together
  for (int r = 0; r < QF_BLK / 1024; r += E) {
    uint64_t v[E];
    int pos[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int64_t i = i0 + (int64_t)(r + e) * 1024 + threadIdx.x;
      v[e] = i < n ? kv[tb * n + i] : 0ull;
      pos[e] = 0;
    }
    for (int step = C >> 1; step > 0; step >>= 1)
#pragma unroll
      for (int e = 0; e < E; ++e) pos[e] += qs_v[pos[e] + step - 1] <= v[e] ? step : 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int64_t i = i0 + (int64_t)(r + e) * 1024 + threadIdx.x;
      if (i < n) {
        const int c = pos[e];
        const uint64_t lo = c ? qs_v[c - 1] : 0ull, w = qs_v[c] - lo;
        const int bits = 64 - __clzll((long long)((w - 1ull) | 1ull)), sh = bits > 32 ? bits - 32 : 0;
        const uint32_t rk = atomicAdd(&h[c], 1u);
        tmp[tb * n + i] = make_uint2((uint32_t)((v[e] - lo) >> sh), ((uint32_t)c << 16) | rk);
      }
    }
  }
  __syncthreads();
  for (int q = threadIdx.x; q < C; q += 1024) cnt[(tb * gridDim.x + blockIdx.x) * C + q] = h[q];
}

// Counts to exclusive sums over the blocks, per (table, cell); cell totals.
__global__ __launch_bounds__(64) void k_qs_colscan(uint32_t* __restrict__ cnt, int nblk, int C, uint32_t* __restrict__ tot) {
  const int c = blockIdx.x * 64 + threadIdx.x;
  if (c >= C) return;
  uint32_t* p = cnt + (int64_t)blockIdx.y * nblk * C + c;
  uint32_t run = 0;
  int b = 0;
  for (; b + 16 <= nblk; b += 16) {
    uint32_t v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = p[(int64_t)(b + u) * C];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      p[(int64_t)(b + u) * C] = run;
      run += v[u];
    }
  }
  for (; b < nblk; ++b) {
    const uint32_t v = p[(int64_t)b * C];
    p[(int64_t)b * C] = run;
    run += v;
  }
  tot[(int64_t)blockIdx.y * C + c] = run;
}

// First rank of every cell and the buckets of its first and last rank; tables with a cell beyond QF_CAP_EXACT go on the
// radix list, whose digit counts start at zero.  state: [0] tables on that list, [1] cells on the exact list.
__global__ __launch_bounds__(1024) void k_qs_rowscan(const uint32_t* __restrict__ tot, int C, int64_t n, int t_buckets,
                                                     uint32_t* __restrict__ first, uint2* __restrict__ range,
                                                     uint32_t* __restrict__ bad, uint32_t* __restrict__ state,
                                                     uint32_t* __restrict__ badlist, uint32_t* __restrict__ digits) {
  __shared__ uint32_t wsum[16];
  __shared__ uint32_t over;
  for (int q = threadIdx.x; q < 8 * 256; q += 1024) digits[(int64_t)blockIdx.x * 8 * 256 + q] = 0u;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (threadIdx.x == 0) over = 0u;
  const uint32_t* t = tot + (int64_t)blockIdx.x * C;
  const int per = (C + 1023) / 1024, c0 = threadIdx.x * per;
  uint32_t sum = 0, big = 0;
  for (int c = c0; c < c0 + per && c < C; ++c) {
    sum += t[c];
    big |= t[c] > (uint32_t)QF_CAP_EXACT;
  }
  uint32_t incl = sum;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(incl, o);
    if (lane >= o) incl += y;
  }
  if (lane == 63) wsum[wv] = incl;
  __syncthreads();
  if (big) over = 1u;
  uint32_t run = incl - sum;
  for (int w = 0; w < wv; ++w) run += wsum[w];
  for (int c = c0; c < c0 + per && c < C; ++c) {
    first[(int64_t)blockIdx.x * C + c] = run;
    const uint64_t l = run + (t[c] ? t[c] - 1u : 0u);
    range[(int64_t)blockIdx.x * C + c] = make_uint2((uint32_t)((uint64_t)run * (uint64_t)t_buckets / (uint64_t)n),
                                                    (uint32_t)(l * (uint64_t)t_buckets / (uint64_t)n));
    run += t[c];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    bad[blockIdx.x] = over;
    if (over) badlist[atomicAdd(&state[0], 1u)] = blockIdx.x;
  }
}

// Records (offset, id) to their cells: a block lays its records out by cell in
// LDS, a window at a time, so that a cell's records leave as one run (8 of 64
// bytes at the mean; written record by record from registers the pass took
// 12.5 instead of 4.3 ms at n = 10^7, m = 40).
__global__ __launch_bounds__(1024) void k_qs_scatter(const uint2* __restrict__ tmp, int64_t n, int C, int nblk,
                                                     const uint32_t* __restrict__ cnt, const uint32_t* __restrict__ tot,
                                                     const uint32_t* __restrict__ first, const uint32_t* __restrict__ bad,
                                                     uint64_t* __restrict__ rec) {
  extern __shared__ __attribute__((aligned(16))) uint64_t qs_v[];  // [QF_STAGE] records, [C] + [C] words, cells
  uint32_t* lofs = reinterpret_cast<uint32_t*>(qs_v + QF_STAGE);   // first place of a cell within the block
  uint32_t* delta = lofs + C;                                      // place in the table minus place in the block
  uint16_t* scell = reinterpret_cast<uint16_t*>(delta + C);        // [QF_STAGE] cell of a staged record
  __shared__ uint32_t wsum[16];
  const int64_t tb = blockIdx.y;
  if (bad[tb]) return;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const uint32_t* cb = cnt + (tb * nblk + blockIdx.x) * C;
  const bool last = (int)blockIdx.x == nblk - 1;
  const int per = (C + 1023) / 1024, c0 = threadIdx.x * per;
  uint32_t sum = 0;
  for (int c = c0; c < c0 + per && c < C; ++c) sum += (last ? tot[tb * C + c] : cb[C + c]) - cb[c];
  uint32_t incl = sum;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(incl, o);
    if (lane >= o) incl += y;
  }
  if (lane == 63) wsum[wv] = incl;
  __syncthreads();
  uint32_t run = incl - sum;
  for (int w = 0; w < wv; ++w) run += wsum[w];
  for (int c = c0; c < c0 + per && c < C; ++c) {
    const uint32_t before = cb[c];
    lofs[c] = run;
    delta[c] = first[tb * C + c] + before - run;
    run += (last ? tot[tb * C + c] : cb[C + c]) - before;
  }
  __syncthreads();
  const int64_t i0 = (int64_t)blockIdx.x * QF_BLK;
  const int len = n - i0 < QF_BLK ? (int)(n - i0) : QF_BLK;
  for (int w0 = 0; w0 < len; w0 += QF_STAGE) {
    constexpr int E = 8;
    for (int r = 0; r < len; r += 1024 * E) {
      uint2 x[E];
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int q = r + e * 1024 + threadIdx.x;
        x[e] = q < len ? tmp[tb * n + i0 + q] : make_uint2(0u, 0u);
      }
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int q = r + e * 1024 + threadIdx.x;
        const uint32_t c = x[e].y >> 16, at = q < len ? lofs[c] + (x[e].y & 0xFFFFu) - w0 : 0xFFFFFFFFu;
        if (at < (uint32_t)QF_STAGE) {
          qs_v[at] = ((uint64_t)x[e].x << 32) | (uint32_t)(i0 + q);
          scell[at] = (uint16_t)c;
        }
      }
    }
    __syncthreads();
    for (int q = threadIdx.x; q < QF_STAGE && w0 + q < len; q += 1024)
      rec[tb * n + delta[scell[q]] + (uint32_t)(w0 + q)] = qs_v[q];
    __syncthreads();
  }
}

// Ranks of up to CAP items spread over the block (item tid + e NT in x[e], c in
// all): items are counted into pow2 >= c slots by their place between the
// smallest and largest position, laid out slot by slot, and each is compared
// with the others of its slot, about one for evenly spread positions.  False
// (for the whole block) if some slot holds more than QF_CROWD items.
template <int NT, int CAP, class T, class Pos, class Less>
GEEK_D bool block_rank(const T (&x)[CAP / NT], int c, T* buf, uint32_t* cnt, uint32_t* sh, Pos pos, Less less,
                       uint32_t (&rank)[CAP / NT]) {
  constexpr int E = CAP / NT, NW = NT / 64;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint32_t mn = 0xFFFFFFFFu, mx = 0u;
#pragma unroll
  for (int e = 0; e < E; ++e)
    if ((int)threadIdx.x + e * NT < c) {
      mn = min(mn, pos(x[e]));
      mx = max(mx, pos(x[e]));
    }
  for (int o = 32; o > 0; o >>= 1) {
    mn = min(mn, (uint32_t)__shfl_xor((int)mn, o));
    mx = max(mx, (uint32_t)__shfl_xor((int)mx, o));
  }
  if (lane == 0) {
    sh[wv] = mn;
    sh[NW + wv] = mx;
  }
  int P = 64;
  while (P < c) P <<= 1;
  for (int q = threadIdx.x; q <= P; q += NT) cnt[q] = 0u;
  if (threadIdx.x == 0) sh[2 * NW] = 0u;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    mn = min(mn, sh[w]);
    mx = max(mx, sh[NW + w]);
  }
  // slot = floor((pos - mn) scale / 2^32) < P; monotone in pos
  const uint64_t scale = ((uint64_t)P << 32) / ((uint64_t)(mx - mn) + 1ull);
  uint32_t slot[E], at[E];
  bool crowd = false;
#pragma unroll
  for (int e = 0; e < E; ++e)
    if ((int)threadIdx.x + e * NT < c) {
      slot[e] = (uint32_t)(((uint64_t)(pos(x[e]) - mn) * scale) >> 32);
      at[e] = atomicAdd(&cnt[slot[e]], 1u);
      crowd |= at[e] >= (uint32_t)QF_CROWD;
    }
  if (crowd) sh[2 * NW] = 1u;
  __syncthreads();
  if (sh[2 * NW]) return false;
  // exclusive scan of the slot counts, cnt[P] = c
  const int per = (P + NT - 1) / NT, q0 = threadIdx.x * per;
  uint32_t sum = 0;
  for (int q = q0; q < q0 + per && q < P; ++q) sum += cnt[q];
  uint32_t incl = sum;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(incl, o);
    if (lane >= o) incl += y;
  }
  if (lane == 63) sh[wv] = incl;
  __syncthreads();
  uint32_t run = incl - sum;
#pragma unroll
  for (int w = 0; w < NW; ++w)
    if (w < wv) run += sh[w];
  for (int q = q0; q < q0 + per && q < P; ++q) {
    const uint32_t v = cnt[q];
    cnt[q] = run;
    run += v;
  }
  if (threadIdx.x == 0) cnt[P] = (uint32_t)c;
  __syncthreads();
#pragma unroll
  for (int e = 0; e < E; ++e)
    if ((int)threadIdx.x + e * NT < c) buf[cnt[slot[e]] + at[e]] = x[e];
  __syncthreads();
#pragma unroll
  for (int e = 0; e < E; ++e)
    if ((int)threadIdx.x + e * NT < c) {
      const uint32_t s0 = cnt[slot[e]], s1 = cnt[slot[e] + 1];
      uint32_t r = s0;
      for (uint32_t q = s0; q < s1; ++q) r += less(buf[q], x[e]) ? 1u : 0u;
      rank[e] = r;
    }
  return true;
}

// Record order within a cell; v: the table's values.
GEEK_D bool rec_less(const uint64_t* v, uint64_t a, uint64_t b) {
  if ((uint32_t)(a >> 32) != (uint32_t)(b >> 32) || a == b) return a < b;
  const uint64_t va = v[(uint32_t)a], vb = v[(uint32_t)b];
  return va != vb ? va < vb : a < b;
}

// Ids of one cell in value order (ties by id) at the cell's ranks.  Equal
// offsets (a cell wider than 2^32 patterns drops low bits) are settled by the
// exact values.
__global__ __launch_bounds__(512) void k_qs_cell(const uint64_t* __restrict__ rec, const uint64_t* __restrict__ kv,
                                                 int64_t n, int C, const uint32_t* __restrict__ tot,
                                                 const uint32_t* __restrict__ first, const uint32_t* __restrict__ bad,
                                                 uint32_t* __restrict__ state, uint32_t* __restrict__ hard,
                                                 uint32_t* __restrict__ sid) {
  __shared__ __attribute__((aligned(16))) uint64_t buf[QF_CAP];
  __shared__ uint32_t cnt[QF_CAP + 1], sh[2 * 512 / 64 + 1];
  const int64_t tb = blockIdx.y, cell = tb * C + blockIdx.x;
  const int c = (int)tot[cell];
  if (c == 0 || bad[tb]) return;
  if (c <= QF_CAP) {
    const int64_t base = tb * n + first[cell];
    uint64_t x[QF_CAP / 512];
    uint32_t rank[QF_CAP / 512];
#pragma unroll
    for (int e = 0; e < QF_CAP / 512; ++e)
      x[e] = (int)threadIdx.x + e * 512 < c ? rec[base + threadIdx.x + e * 512] : 0ull;
    const uint64_t* v = kv + tb * n;
    const bool ok = block_rank<512, QF_CAP>(
        x, c, buf, cnt, sh, [](uint64_t y) { return (uint32_t)(y >> 32); },
        [&](uint64_t a, uint64_t b) { return rec_less(v, a, b); }, rank);
    if (ok) {
#pragma unroll
      for (int e = 0; e < QF_CAP / 512; ++e)
        if ((int)threadIdx.x + e * 512 < c) sid[base + rank[e]] = (uint32_t)x[e];
      return;
    }
  }
  if (threadIdx.x == 0) hard[atomicAdd(&state[1], 1u)] = (uint32_t)cell;
}

// The cells of the exact list: ranked as above if only their size put them
// there, else a comparison sort of (value, id) in LDS.
__global__ __launch_bounds__(1024) void k_qs_cell_exact(const uint64_t* __restrict__ rec, const uint64_t* __restrict__ kv,
                                                        int64_t n, int C, const uint32_t* __restrict__ tot,
                                                        const uint32_t* __restrict__ first,
                                                        const uint32_t* __restrict__ state,
                                                        const uint32_t* __restrict__ hard, uint32_t* __restrict__ sid) {
  extern __shared__ __attribute__((aligned(16))) uint64_t qs_v[];  // [QF_CAP_EXACT] values, [QF_CAP_EXACT + 1] ids
  uint32_t* ids = reinterpret_cast<uint32_t*>(qs_v + QF_CAP_EXACT);
  __shared__ uint32_t sh[2 * 1024 / 64 + 1];
  for (uint32_t z = blockIdx.x; z < state[1]; z += gridDim.x) {
    const uint32_t cell = hard[z];
    const int64_t tb = cell / (uint32_t)C, base = tb * n + first[cell];
    const int c = (int)tot[cell];
    const uint64_t* v = kv + tb * n;
    if (c > QF_CAP) {
      uint64_t x[QF_CAP_EXACT / 1024];
      uint32_t rank[QF_CAP_EXACT / 1024];
#pragma unroll
      for (int e = 0; e < QF_CAP_EXACT / 1024; ++e)
        x[e] = (int)threadIdx.x + e * 1024 < c ? rec[base + threadIdx.x + e * 1024] : 0ull;
      const bool ok = block_rank<1024, QF_CAP_EXACT>(
          x, c, qs_v, ids, sh, [](uint64_t y) { return (uint32_t)(y >> 32); },
          [&](uint64_t a, uint64_t b) { return rec_less(v, a, b); }, rank);
      if (ok) {
#pragma unroll
        for (int e = 0; e < QF_CAP_EXACT / 1024; ++e)
          if ((int)threadIdx.x + e * 1024 < c) sid[base + rank[e]] = (uint32_t)x[e];
        __syncthreads();
        continue;
      }
      __syncthreads();
    }
    int P = 1;
    while (P < c) P <<= 1;
    for (int q = threadIdx.x; q < P; q += 1024) {
      const uint32_t id = q < c ? (uint32_t)rec[base + q] : 0xFFFFFFFFu;
      ids[q] = id;
      qs_v[q] = q < c ? v[id] : ~0ull;
    }
    __syncthreads();
    lds_bitonic(
        P, [&](int a, int b) { return qs_v[a] != qs_v[b] ? qs_v[a] < qs_v[b] : ids[a] < ids[b]; },
        [&](int a, int b) {
          const uint64_t t = qs_v[a];
          qs_v[a] = qs_v[b];
          qs_v[b] = t;
          const uint32_t u = ids[a];
          ids[a] = ids[b];
          ids[b] = u;
        });
    for (int q = threadIdx.x; q < c; q += 1024) sid[base + q] = ids[q];
    __syncthreads();
  }
}

// ---- radix ranks of the listed tables: (value, id) sorted by the values'
// bytes, least significant first (stable, so ties keep id order).  Blocks loop
// over (table, tile) and end at once when no table is listed.  Values travel with
// the ids, in the tables' own buffers: gathered through the ids at every pass,
// with one block scanning a table's counts, eight tables of 10^7 x 16 rows with
// 1 % zero rows took 36.1 ms a call, 13.7 ms with the sort that this one replaced.
constexpr int QR_TILE = 4096, QR_THREADS = 256, QR_ITEMS = QR_TILE / QR_THREADS;

// Sum over a block of QR_THREADS (all threads), and the sum before each thread.
GEEK_D uint32_t qr_exscan(uint32_t v, uint32_t* total, uint32_t* sh) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint32_t incl = v;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(incl, o);
    if (lane >= o) incl += y;
  }
  __syncthreads();  // the last call's sums are read
  if (lane == 63) sh[wv] = incl;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < QR_THREADS / 64; ++w) {
    before += w < wv ? sh[w] : 0u;
    all += sh[w];
  }
  *total = all;
  return before + incl - v;
}

// Digit counts of every tile, and of the table (digits[table][pass][digit]).
__global__ __launch_bounds__(QR_THREADS) void k_qr_hist(const uint64_t* __restrict__ v, int64_t n, int pass, int ntile,
                                                        const uint32_t* __restrict__ state,
                                                        const uint32_t* __restrict__ badlist,
                                                        uint32_t* __restrict__ hist, uint32_t* __restrict__ digits) {
  __shared__ uint32_t h[256];
  const int64_t items = (int64_t)state[0] * ntile;
  for (int64_t z = blockIdx.x; z < items; z += gridDim.x) {
    const int64_t tb = badlist[z / ntile], tile = z % ntile, s = tile * QR_TILE;
    h[threadIdx.x] = 0u;
    __syncthreads();
    uint64_t x[QR_ITEMS];
#pragma unroll
    for (int r = 0; r < QR_ITEMS; ++r) {
      const int64_t q = s + r * QR_THREADS + threadIdx.x;
      x[r] = v[tb * n + (q < n ? q : n - 1)];
    }
#pragma unroll
    for (int r = 0; r < QR_ITEMS; ++r)
      if (s + r * QR_THREADS + threadIdx.x < n) atomicAdd(&h[(x[r] >> (8 * pass)) & 255u], 1u);
    __syncthreads();
    const uint32_t c = h[threadIdx.x];
    hist[(tb * 256 + threadIdx.x) * ntile + tile] = c;
    if (c) atomicAdd(&digits[(tb * 8 + pass) * 256 + threadIdx.x], c);
  }
}

// Counts to first places: one block per (digit, table).
__global__ __launch_bounds__(QR_THREADS) void k_qr_scan(uint32_t* __restrict__ hist, int pass, int ntile,
                                                        const uint32_t* __restrict__ state,
                                                        const uint32_t* __restrict__ badlist,
                                                        const uint32_t* __restrict__ digits) {
  __shared__ uint32_t sh[QR_THREADS / 64];
  for (uint32_t z = blockIdx.y; z < state[0]; z += gridDim.y) {
    const int64_t tb = badlist[z];
    uint32_t carry;  // items of smaller digits
    qr_exscan(threadIdx.x < blockIdx.x ? digits[(tb * 8 + pass) * 256 + threadIdx.x] : 0u, &carry, sh);
    uint32_t* h = hist + (tb * 256 + blockIdx.x) * ntile;
    constexpr int PER = 4;
    for (int q0 = 0; q0 < ntile; q0 += QR_THREADS * PER) {
      uint32_t c[PER], sum = 0, all;
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        const int q = q0 + (int)threadIdx.x * PER + u;
        c[u] = q < ntile ? h[q] : 0u;
        sum += c[u];
      }
      uint32_t run = carry + qr_exscan(sum, &all, sh);
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        const int q = q0 + (int)threadIdx.x * PER + u;
        if (q < ntile) h[q] = run;
        run += c[u];
      }
      carry += all;
    }
  }
}

// Items of a tile ranked in order (rounds in thread order, within a wave by
// matching the digit's bits), laid out by digit in LDS and written by consecutive
// threads, so that a digit's items of the tile leave as one run.  Pass 0: the ids
// are the places; the last pass writes no values.
__global__ __launch_bounds__(QR_THREADS) void k_qr_scatter(const uint64_t* __restrict__ v, const uint32_t* __restrict__ ids,
                                                           int64_t id_stride, int64_t n, int pass, int ntile,
                                                           const uint32_t* __restrict__ state,
                                                           const uint32_t* __restrict__ badlist,
                                                           const uint32_t* __restrict__ hist,
                                                           uint64_t* __restrict__ vdst, uint32_t* __restrict__ idst,
                                                           int64_t idst_stride) {
  __shared__ __attribute__((aligned(16))) uint64_t sv[QR_TILE];
  __shared__ uint32_t si[QR_TILE], first[256], place[256], run[256], wcnt[QR_THREADS / 64][256];
  __shared__ uint32_t sh[QR_THREADS / 64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t items = (int64_t)state[0] * ntile;
  for (int64_t z = blockIdx.x; z < items; z += gridDim.x) {
    const int64_t tb = badlist[z / ntile], tile = z % ntile, s = tile * QR_TILE;
    const int len = n - s < QR_TILE ? (int)(n - s) : QR_TILE;
    // the tile's counts: places are a running sum over (digit, tile)
    const int64_t at = (tb * 256 + threadIdx.x) * ntile + tile;
    const uint32_t g0 = hist[at];
    const uint32_t g1 = tile + 1 < ntile || threadIdx.x < 255 ? hist[at + 1] : (uint32_t)n;
    uint32_t all;
    const uint32_t l0 = qr_exscan(g1 - g0, &all, sh);  // (its barriers also end the last item's reads)
    first[threadIdx.x] = g0;
    place[threadIdx.x] = l0;
    run[threadIdx.x] = l0;
#pragma unroll
    for (int w = 0; w < QR_THREADS / 64; ++w) wcnt[w][threadIdx.x] = 0u;
    uint64_t x[QR_ITEMS];
    uint32_t id[QR_ITEMS];
#pragma unroll
    for (int r = 0; r < QR_ITEMS; ++r) {
      const int64_t q = s + r * QR_THREADS + threadIdx.x, c = q < n ? q : n - 1;
      x[r] = v[tb * n + c];
      id[r] = pass ? ids[tb * id_stride + c] : (uint32_t)c;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < QR_ITEMS; ++r) {
      const bool has = r * QR_THREADS + (int)threadIdx.x < len;
      const uint32_t dg = (uint32_t)(x[r] >> (8 * pass)) & 255u;
      uint64_t mask = __ballot(has);
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        const uint64_t bb = __ballot((dg >> b) & 1u);
        mask &= ((dg >> b) & 1u) ? bb : ~bb;
      }
      const uint32_t below = (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
      const bool leader = has && below == 0;
      if (leader) wcnt[wv][dg] = (uint32_t)__popcll(mask);
      __syncthreads();
      if (has) {
        uint32_t p = run[dg] + below;
        for (int w = 0; w < wv; ++w) p += wcnt[w][dg];
        sv[p] = x[r];
        si[p] = id[r];
      }
      __syncthreads();
      uint32_t sum = 0;
#pragma unroll
      for (int w = 0; w < QR_THREADS / 64; ++w) sum += wcnt[w][threadIdx.x];
      run[threadIdx.x] += sum;
      __syncthreads();
      if (leader) wcnt[wv][dg] = 0u;
      __syncthreads();
    }
    for (int q = threadIdx.x; q < len; q += QR_THREADS) {
      const uint32_t d = (uint32_t)(sv[q] >> (8 * pass)) & 255u;
      const uint32_t to = first[d] + (uint32_t)q - place[d];
      if (pass < 7) vdst[tb * n + to] = sv[q];
      idst[tb * idst_stride + to] = si[q];
    }
  }
}

// (value pattern words and ids of one table, for the radix sort that carries them)
__global__ void k_q_words(const uint64_t* __restrict__ kv, int64_t n, uint32_t* __restrict__ klo,
                          uint32_t* __restrict__ khi, uint32_t* __restrict__ ids) {
  const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (q >= n) return;
  klo[q] = (uint32_t)kv[q];
  khi[q] = (uint32_t)(kv[q] >> 32);
  ids[q] = (uint32_t)q;
}

// bucket of every object from its rank; the id-ordered bucket keys and ids
// feed the second sort
__global__ void k_q_rank(const uint32_t* __restrict__ sorted_ids, int64_t n, int t, uint32_t* __restrict__ bkey,
                         uint32_t* __restrict__ ids, uint32_t* __restrict__ bucket_of) {
  const int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (r >= n) return;
  const uint32_t i = sorted_ids[r];
  const uint32_t b = (uint32_t)((uint64_t)r * (uint64_t)t / (uint64_t)n);
  bkey[i] = b;
  ids[r] = (uint32_t)r;  // id order for the second sort (position r holds id r)
  if (bucket_of) bucket_of[i] = b;
}

__global__ void k_q_copy(const uint32_t* __restrict__ src, int64_t n, uint32_t* __restrict__ dst) {
  const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (q < n) dst[q] = src[q];
}

// The (offset, id) of the object at the first rank of every bucket.
__global__ void k_qs_bounds(const uint32_t* __restrict__ sid, const uint2* __restrict__ tmp, int64_t n, int t,
                            uint2* __restrict__ bound) {
  const int64_t b = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, tb = blockIdx.y;
  if (b >= t) return;
  const uint32_t id = sid[tb * n + (int64_t)(((uint64_t)b * (uint64_t)n + (uint64_t)t - 1) / (uint64_t)t)];
  bound[tb * t + b] = make_uint2(tmp[tb * n + id].x, id);
}

// bucket_of in id order: an object's bucket is the last one of its cell whose
// first object is not above it.  (Scattered from the rank order instead, the
// 4-byte stores took most of the bucket pass: 9.8 ms at n = 10^7, m = 40.)
// STAGED: the cells' bucket ranges and the bounds' offsets lie in LDS, where
// they fit in QB_LDS bytes (1.5 against 5.8 ms from global memory at t = 10^4).
constexpr size_t QB_LDS = 80 << 10;
constexpr int QB_BLK = 32768;  // objects per block
template <bool STAGED>
__global__ __launch_bounds__(1024) void k_qs_bucket_of(const uint2* __restrict__ tmp, const uint64_t* __restrict__ kv,
                                                       int64_t n, int t, int C, const uint2* __restrict__ range,
                                                       const uint32_t* __restrict__ bad,
                                                       const uint2* __restrict__ bound,
                                                       uint32_t* __restrict__ bucket_of) {
  extern __shared__ __attribute__((aligned(16))) uint64_t qs_v[];  // [C] ranges, [t] offsets
  const int64_t tb = blockIdx.y;
  if (bad[tb]) return;
  uint2* lr = reinterpret_cast<uint2*>(qs_v);
  uint32_t* lb = reinterpret_cast<uint32_t*>(qs_v + C);
  const uint64_t* v = kv + tb * n;
  const uint2* bt = bound + tb * t;
  if (STAGED) {
    for (int q = threadIdx.x; q < C; q += 1024) lr[q] = range[tb * C + q];
    for (int q = threadIdx.x; q < t; q += 1024) lb[q] = bt[q].x;
    __syncthreads();
  }
  const int64_t i0 = (int64_t)blockIdx.x * QB_BLK;
  constexpr int E = 8;
  for (int r = 0; r < QB_BLK; r += 1024 * E) {
    uint2 x[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int64_t i = i0 + r + e * 1024 + threadIdx.x;
      x[e] = i < n ? tmp[tb * n + i] : make_uint2(0u, 0u);
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int64_t i = i0 + r + e * 1024 + threadIdx.x;
      if (i >= n) continue;
      const uint2 rg = STAGED ? lr[x[e].y >> 16] : range[tb * C + (x[e].y >> 16)];
      uint32_t lo = rg.x, hi = rg.y;
      while (lo < hi) {  // bucket in [lo, hi]; buckets above the cell's first start within the cell
        const uint32_t mid = (lo + hi + 1u) >> 1, off = STAGED ? lb[mid] : bt[mid].x;
        bool above = off < x[e].x;
        if (off == x[e].x) {  // settled by the values, then the ids
          const uint32_t id = bt[mid].y;
          const uint64_t vy = v[id], vx = v[i];
          above = vy != vx ? vy < vx : id <= (uint32_t)i;
        }
        if (above) lo = mid; else hi = mid - 1u;
      }
      bucket_of[tb * n + i] = lo;
    }
  }
}

// Buckets of at most QS_MAX objects: bucket b's ids (ranks ceil(b n / t) ..
// ceil((b + 1) n / t) - 1 of the value order) are ranked in LDS (by their place
// between the bucket's smallest and largest id; where that crowds a slot, by
// a bitonic sort) and written as its members; bucket_of is scattered along
// (with bad: for the tables it marks).  One workgroup per (bucket, table).
constexpr int QS_MAX = 4096;
template <int CAP>  // buckets hold at most CAP objects
__global__ __launch_bounds__(256) void k_q_segsort(const uint32_t* __restrict__ sorted_ids, int64_t n, int t,
                                                   uint32_t* __restrict__ members, const uint32_t* __restrict__ bad,
                                                   uint32_t* __restrict__ bucket_of) {
  __shared__ uint32_t v[CAP], cnt[CAP + 1], sh[2 * 256 / 64 + 1];
  const int b = blockIdx.x;
  const int64_t tab = (int64_t)blockIdx.y * n;
  if (bad && !bad[blockIdx.y]) bucket_of = nullptr;
  const int64_t s0 = ((uint64_t)b * (uint64_t)n + (uint64_t)t - 1) / (uint64_t)t;
  const int64_t s1 = ((uint64_t)(b + 1) * (uint64_t)n + (uint64_t)t - 1) / (uint64_t)t;
  const int len = (int)(s1 - s0);
  uint32_t x[CAP / 256], rank[CAP / 256];
#pragma unroll
  for (int e = 0; e < CAP / 256; ++e)
    x[e] = (int)threadIdx.x + e * 256 < len ? sorted_ids[tab + s0 + threadIdx.x + e * 256] : 0u;
  if (block_rank<256, CAP>(
          x, len, v, cnt, sh, [](uint32_t y) { return y; }, [](uint32_t p, uint32_t q) { return p < q; }, rank)) {
#pragma unroll
    for (int e = 0; e < CAP / 256; ++e)
      if ((int)threadIdx.x + e * 256 < len) {
        members[tab + s0 + rank[e]] = x[e];
        if (bucket_of) bucket_of[tab + x[e]] = (uint32_t)b;
      }
    return;
  }
  int P = 1;
  while (P < len) P <<= 1;
  __syncthreads();
#pragma unroll
  for (int e = 0; e < CAP / 256; ++e)
    if ((int)threadIdx.x + e * 256 < P) v[threadIdx.x + e * 256] = (int)threadIdx.x + e * 256 < len ? x[e] : 0xFFFFFFFFu;
  __syncthreads();
  lds_bitonic(
      P, [&](int p, int q) { return v[p] < v[q]; },
      [&](int p, int q) {
        const uint32_t y = v[p];
        v[p] = v[q];
        v[q] = y;
      });
  for (int q = threadIdx.x; q < len; q += blockDim.x) {
    members[tab + s0 + q] = v[q];
    if (bucket_of) bucket_of[tab + v[q]] = (uint32_t)b;
  }
}

// Buckets of at most QT_MAX objects: a thread per rank counts the smaller ids of
// its bucket and writes bucket_of along.  A workgroup per bucket is mostly idle
// there: four tables of 10^6 rows, a call with one object per bucket 9.9 ms so (8.2
// with the bitonic sort before) against 0.44, 16 objects 1.17 against 0.44, 60
// objects 0.61 against 0.49; at 100 a workgroup per bucket takes 0.54.
constexpr int QT_MAX = 64;
__global__ __launch_bounds__(256) void k_q_tiny(const uint32_t* __restrict__ sorted_ids, int64_t n, int t,
                                                uint32_t* __restrict__ members, uint32_t* __restrict__ bucket_of) {
  const int64_t r = blockIdx.x * (int64_t)256 + threadIdx.x, tab = (int64_t)blockIdx.y * n;
  if (r >= n) return;
  const uint64_t b = (uint64_t)r * (uint64_t)t / (uint64_t)n;
  const int64_t s0 = (b * (uint64_t)n + (uint64_t)t - 1) / (uint64_t)t;
  const int64_t s1 = ((b + 1) * (uint64_t)n + (uint64_t)t - 1) / (uint64_t)t;
  const uint32_t x = sorted_ids[tab + r];
  int64_t p = s0;
  for (int64_t q = s0; q < s1; ++q) p += sorted_ids[tab + q] < x ? 1 : 0;
  members[tab + p] = x;
  if (bucket_of) bucket_of[tab + x] = (uint32_t)b;
}

// bucket b starts at rank ceil(b n / t)
__global__ void k_q_offsets(int64_t n, int t, uint32_t* __restrict__ off) {
  const int64_t b = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (b > t) return;
  off[(int64_t)blockIdx.y * (t + 1) + b] = (uint32_t)(((uint64_t)b * (uint64_t)n + (uint64_t)t - 1) / (uint64_t)t);
}

struct QWs {
  double* Ad;
  uint64_t* kv;  // [m][n] value patterns of every table
  // sample sort, G tables at a time
  int C, S, nblk, G, ntile;
  uint64_t *smp, *spl, *rec;
  uint2 *tmp, *bound, *range;
  uint32_t *sid, *cnt, *tot, *first, *bad, *badlist, *hard, *state, *hist, *digits;
  // radix sort with keys and ids, one table at a time
  uint32_t *klo, *khi, *ids, *klo2, *khi2, *ids2, *rtmp;
};

constexpr int64_t QF_GROUP_BYTES = 2ll << 30;  // records of the tables ranked together

static size_t carve_q(const geek_quantile_job& J, void* base, QWs& W) {
  Carver c(base);
  const int64_t n = J.n;
  const int dpad = (J.d + QV_CHUNK - 1) / QV_CHUNK * QV_CHUNK;
  W.Ad = c.take<double>((size_t)((J.m + QV_GRP - 1) / QV_GRP) * QV_GRP * dpad);
  W.kv = c.take<uint64_t>((size_t)J.m * n);
  W.C = q_cells(n);
  const bool second = (n + J.t - 1) / J.t > QS_MAX;  // the ids are sorted again by bucket
  if (W.C) {
    W.S = W.C * QF_OVER;
    W.nblk = ceil_div(n, QF_BLK);
    W.ntile = ceil_div(n, QR_TILE);
    const int64_t most = std::max<int64_t>(1, std::min<int64_t>(1024, QF_GROUP_BYTES / (20 * n)));
    const int64_t groups = (J.m + most - 1) / most;
    W.G = (int)((J.m + groups - 1) / groups);
    const size_t g = W.G;
    W.smp = c.take<uint64_t>((size_t)J.m * W.S);
    W.spl = c.take<uint64_t>((size_t)J.m * W.C);
    W.tmp = c.take<uint2>(g * n);
    W.sid = c.take<uint32_t>(g * n);
    W.bound = c.take<uint2>(J.bucket_of && !second ? g * (size_t)J.t : 0);
    W.rec = c.take<uint64_t>(g * n);
    W.cnt = c.take<uint32_t>(g * W.nblk * W.C);
    W.tot = c.take<uint32_t>(g * W.C);
    W.first = c.take<uint32_t>(g * W.C);
    W.range = c.take<uint2>(g * W.C);
    W.bad = c.take<uint32_t>(g);
    W.badlist = c.take<uint32_t>(g);
    W.hard = c.take<uint32_t>(g * W.C);
    W.state = c.take<uint32_t>(2);
    W.hist = c.take<uint32_t>(g * 256 * W.ntile);
    W.digits = c.take<uint32_t>(g * 8 * 256);
  }
  if (!W.C) {
    W.klo = c.take<uint32_t>(n);
    W.khi = c.take<uint32_t>(n);
    W.ids = c.take<uint32_t>(n);
    W.klo2 = c.take<uint32_t>(n);
    W.khi2 = c.take<uint32_t>(n);
    W.ids2 = c.take<uint32_t>(n);
  }
  if (!W.C || second) W.rtmp = c.take<uint32_t>(radix_tmp_words(n));
  return c.used + 256;
}

size_t quantile_ws(const geek_quantile_job& J) {
  QWs W;
  return carve_q(J, nullptr, W);
}

template <int NG>
static void launch_qv(const geek_quantile_job& J, const QWs& W, int dpad, int p0, int32_t* st, hipStream_t s) {
  hipLaunchKernelGGL(k_qv<NG>, dim3(ceil_div(J.n, QV_ROWS)), dim3(QV_ROWS), 0, s, J.X, J.ldx, J.n, J.d, dpad, W.Ad, p0,
                     J.m, W.kv, st);
}

__global__ void k_q_clear(uint32_t* p) { p[threadIdx.x] = 0u; }

// Ids of the tables p0 .. p0 + g - 1 in value order, at W.sid[table][n].
static void q_rank_group(const geek_quantile_job& J, const QWs& W, int p0, int g, hipStream_t s) {
  const int64_t n = J.n;
  uint64_t* kv = W.kv + (int64_t)p0 * n;
  const uint64_t* spl = W.spl + (size_t)p0 * W.C;
  hipLaunchKernelGGL(k_q_clear, dim3(1), dim3(2), 0, s, W.state);
  hipLaunchKernelGGL(k_qs_count, dim3(W.nblk, g), dim3(1024), (sizeof(uint64_t) + sizeof(uint32_t)) * W.C, s, kv, n, W.C,
                     spl, W.tmp, W.cnt);
  hipLaunchKernelGGL(k_qs_colscan, dim3(ceil_div(W.C, 64), g), dim3(64), 0, s, W.cnt, W.nblk, W.C, W.tot);
  hipLaunchKernelGGL(k_qs_rowscan, dim3(g), dim3(1024), 0, s, W.tot, W.C, n, J.t, W.first,
                     W.range, W.bad, W.state, W.badlist, W.digits);
  hipLaunchKernelGGL(k_qs_scatter, dim3(W.nblk, g), dim3(1024),
                     (sizeof(uint64_t) + sizeof(uint16_t)) * QF_STAGE + 2 * sizeof(uint32_t) * W.C, s, W.tmp, n, W.C,
                     W.nblk, W.cnt, W.tot, W.first, W.bad, W.rec);
  hipLaunchKernelGGL(k_qs_cell, dim3(W.C, g), dim3(512), 0, s, W.rec, kv, n, W.C, W.tot, W.first, W.bad, W.state,
                     W.hard, W.sid);
  hipLaunchKernelGGL(k_qs_cell_exact, dim3(std::min(256, W.C * g)), dim3(1024),
                     (sizeof(uint64_t) + sizeof(uint32_t)) * QF_CAP_EXACT + 16, s, W.rec, kv, n, W.C, W.tot, W.first,
                     W.state, W.hard, W.sid);
  if (n <= QF_CAP_EXACT) return;  // no cell can be larger
  // the listed tables: eight passes between their values and sid on one side,
  // their (unused) records and offsets on the other
  uint32_t* other = reinterpret_cast<uint32_t*>(W.tmp);
  // (as many blocks as the chip holds: most calls list no table)
  const int grid = (int)std::min<int64_t>(512, (int64_t)g * W.ntile);
  for (int pass = 0; pass < 8; ++pass) {
    const bool odd = pass & 1;
    hipLaunchKernelGGL(k_qr_hist, dim3(grid), dim3(QR_THREADS), 0, s, odd ? W.rec : kv, n, pass, W.ntile, W.state,
                       W.badlist, W.hist, W.digits);
    hipLaunchKernelGGL(k_qr_scan, dim3(256, std::min(g, 2)), dim3(QR_THREADS), 0, s, W.hist, pass, W.ntile, W.state,
                       W.badlist, W.digits);
    hipLaunchKernelGGL(k_qr_scatter, dim3(grid), dim3(QR_THREADS), 0, s, odd ? W.rec : kv, odd ? other : W.sid,
                       odd ? 2 * n : n, n, pass, W.ntile, W.state, W.badlist, W.hist, odd ? kv : W.rec,
                       odd ? W.sid : other, odd ? n : 2 * n);
  }
}

// Members by a stable sort of the ids keyed by bucket.
static void q_sort_by_bucket(const geek_quantile_job& J, const QWs& W, const uint32_t* sorted_ids, uint32_t* members,
                             uint32_t* bof, uint32_t* bkey, uint32_t* bid, uint32_t* bkey2, uint32_t* bid2,
                             hipStream_t s) {
  const int grid = ceil_div(J.n, 256);
  hipLaunchKernelGGL(k_q_rank, dim3(grid), dim3(256), 0, s, sorted_ids, J.n, J.t, bkey, bid, bof);
  int w2[4], s2[4], np = 0;
  for (int sh = 0; sh < 32 && ((uint32_t)(J.t - 1) >> sh) != 0u; sh += 8) {
    w2[np] = 0;
    s2[np++] = sh;
  }
  RsView C{{bkey, nullptr, nullptr, nullptr}, bid}, D{{bkey2, nullptr, nullptr, nullptr}, bid2};
  const int alt2 = radix_sort(C, D, 1, J.n, w2, s2, np, W.rtmp, s);
  hipLaunchKernelGGL(k_q_copy, dim3(grid), dim3(256), 0, s, alt2 ? bid2 : bid, J.n, members);
}

int32_t quantile_run(const geek_quantile_job& J, void* ws, int32_t* st, hipStream_t s) {
  QWs W;
  carve_q(J, ws, W);
  const int64_t n = J.n;
  const int dpad = (J.d + QV_CHUNK - 1) / QV_CHUNK * QV_CHUNK, ngrp = (J.m + QV_GRP - 1) / QV_GRP;
  hipLaunchKernelGGL(k_qv_prep, dim3(ceil_div((int64_t)ngrp * QV_GRP * dpad, 256)), dim3(256), 0, s, J.A, J.m, J.d, dpad,
                     W.Ad, st);
  // up to five groups of projections per pass over X
  for (int g0 = 0; g0 < ngrp;) {
    const int passes = (ngrp - g0 + 4) / 5, ng = (ngrp - g0 + passes - 1) / passes;
    switch (ng) {
      case 1: launch_qv<1>(J, W, dpad, g0 * QV_GRP, st, s); break;
      case 2: launch_qv<2>(J, W, dpad, g0 * QV_GRP, st, s); break;
      case 3: launch_qv<3>(J, W, dpad, g0 * QV_GRP, st, s); break;
      case 4: launch_qv<4>(J, W, dpad, g0 * QV_GRP, st, s); break;
      default: launch_qv<5>(J, W, dpad, g0 * QV_GRP, st, s); break;
    }
    g0 += ng;
  }
  const int64_t most = (n + J.t - 1) / J.t;
  const bool small = most <= QS_MAX;  // every bucket fits one workgroup's LDS
  const bool tiny = most <= QT_MAX;
  auto emit = [&](const uint32_t* sorted_ids, int p0, int g, const uint32_t* bad) {
    uint32_t *mem = J.members + (int64_t)p0 * n, *bof = J.bucket_of ? J.bucket_of + (int64_t)p0 * n : nullptr;
    if (tiny) {  // (bucket_of of every table is written here)
      hipLaunchKernelGGL(k_q_tiny, dim3(ceil_div(n, 256), g), dim3(256), 0, s, sorted_ids, n, J.t, mem, bof);
      return;
    }
    const auto kern = most <= 512 ? k_q_segsort<512> : most <= 1024 ? k_q_segsort<1024>
                      : most <= 2048 ? k_q_segsort<2048> : k_q_segsort<QS_MAX>;
    hipLaunchKernelGGL(kern, dim3(J.t, g), dim3(256), 0, s, sorted_ids, n, J.t, mem, bad, bof);
  };
  if (W.C) {
    const int len = std::min(W.S, QF_CHUNK);
    for (int p0 = 0; p0 < J.m; p0 += 1024) {
      const int g = std::min(1024, J.m - p0);
      uint64_t* smp = W.smp + (size_t)p0 * W.S;
      hipLaunchKernelGGL(k_qs_sample, dim3(W.S / len, g), dim3(1024), sizeof(uint64_t) * len, s,
                         W.kv + (int64_t)p0 * n, n, W.S, smp);
      hipLaunchKernelGGL(k_qs_split, dim3(ceil_div(W.S, 256), g), dim3(256), 0, s, smp, W.S, W.C,
                         W.spl + (size_t)p0 * W.C);
    }
    for (int p0 = 0; p0 < J.m; p0 += W.G) {
      const int g = std::min(W.G, J.m - p0);
      q_rank_group(J, W, p0, g, s);
      if (small) {
        if (J.bucket_of && !tiny) {
          hipLaunchKernelGGL(k_qs_bounds, dim3(ceil_div(J.t, 256), g), dim3(256), 0, s, W.sid, W.tmp, n, J.t, W.bound);
          const size_t lds = sizeof(uint2) * W.C + sizeof(uint32_t) * (size_t)J.t;
          hipLaunchKernelGGL(lds <= QB_LDS ? k_qs_bucket_of<true> : k_qs_bucket_of<false>, dim3(ceil_div(n, QB_BLK), g),
                             dim3(1024), lds <= QB_LDS ? lds : 0, s, W.tmp, W.kv + (int64_t)p0 * n, n, J.t, W.C, W.range,
                             W.bad, W.bound, J.bucket_of + (int64_t)p0 * n);
        }
        emit(W.sid, p0, g, W.bad);
        continue;
      }
      // in the group's records, which the ranks no longer need
      uint32_t *a = reinterpret_cast<uint32_t*>(W.rec), *b = reinterpret_cast<uint32_t*>(W.tmp);
      for (int p = p0; p < p0 + g; ++p)
        q_sort_by_bucket(J, W, W.sid + (int64_t)(p - p0) * n, J.members + (int64_t)p * n,
                         J.bucket_of ? J.bucket_of + (int64_t)p * n : nullptr, a, a + n, b, b + n, s);
    }
  } else {
    for (int p = 0; p < J.m; ++p) {
      hipLaunchKernelGGL(k_q_words, dim3(ceil_div(n, 256)), dim3(256), 0, s, W.kv + (int64_t)p * n, n, W.klo, W.khi,
                         W.ids);
      // 64-bit value patterns, least significant byte first; ties keep id order
      const int words[8] = {0, 0, 0, 0, 1, 1, 1, 1}, shifts[8] = {0, 8, 16, 24, 0, 8, 16, 24};
      RsView A{{W.klo, W.khi, nullptr, nullptr}, W.ids}, B{{W.klo2, W.khi2, nullptr, nullptr}, W.ids2};
      const int alt = radix_sort(A, B, 2, n, words, shifts, 8, W.rtmp, s);
      const uint32_t* sorted_ids = alt ? W.ids2 : W.ids;
      if (small) {
        emit(sorted_ids, p, 1, nullptr);
        continue;
      }
      // in the buffers the first sort's result does not occupy
      q_sort_by_bucket(J, W, sorted_ids, J.members + (int64_t)p * n,
                       J.bucket_of ? J.bucket_of + (int64_t)p * n : nullptr, alt ? W.klo : W.klo2,
                       alt ? W.ids : W.ids2, alt ? W.khi : W.khi2, alt ? W.ids2 : W.ids, s);
    }
  }
  for (int p0 = 0; p0 < J.m; p0 += 1024)
    hipLaunchKernelGGL(k_q_offsets, dim3(ceil_div((int64_t)J.t + 1, 256), std::min(1024, J.m - p0)), dim3(256), 0, s, n,
                       J.t, J.offsets + (int64_t)p0 * (J.t + 1));
  GEEK_LAUNCH_CHECK();
  return GEEK_OK;
}

}  // namespace geek

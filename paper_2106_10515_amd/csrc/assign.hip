// One-pass data assignment (paper Section 3.3, Eq. (1)) on gfx950.
//
// Pipeline for Euclidean data (all stream-ordered, no host synchronization):
//   k_centroids   float64 centroids, one thread per (seed, dim), members summed
//                 in ascending order one rounding at a time (exact parity),
//                 their values loaded 32 at a time.
//   k_cprep       centroid copies for the matrix cores (three bf16 pieces, e4m3),
//                 |c|^2 and max |c| for the error bound.
//   k_scan<M,DP>  matrix-core tile |x|^2 - 2 x.c + |c|^2 over all centroids for
//                 a block of rows.  Float32: per row it keeps every centroid
//                 whose approximate distance lies within 2*eps_i of the
//                 running minimum (eps_i a rigorous bound of the approximation
//                 error), up to TCAND candidates (TCAND32 in the rescan of
//                 ambiguous rows).  The BF16 and FP8 (e4m3) first passes keep
//                 only the best and second-best values (branch-free); a row is
//                 settled when the runner-up lies beyond 2*eps_i, else it is
//                 rescanned: after FP8 in BF16 the same way, then in float32.
//   k_finalize    float64 distance (the reference formula, same operation
//                 order) for each candidate; lowest index wins exact ties.
//                 Rows whose candidate window overflowed are escalated.
//   k_fallback64  float64 distance to every centroid for the rows left
//                 (64 x 64 row-seed tiles, split over workgroups for few rows).
//   k_sse_*       SSE in fixed 4096-row blocks; radius per cluster.
//
// Heterogeneous rows (numeric attributes + categorical attributes) use the
// same pipeline with D = D_num + gamma * #mismatching attributes: the
// mismatch count is exact and added in the scan epilogue; the categorical
// central vector is the per-attribute mode (assign_sig.hip computes modes).
#include <math.h>

#include <algorithm>
#include <type_traits>
#include <vector>

#include "radix.hpp"
#include "scan.hpp"

namespace geek {

constexpr int SSE_BLOCK = 4096;

// ---------------------------------------------------------------- centroids
// The sum over a seed's members is one chain of float64 additions (the
// reference order), so a seed with many members is bound by memory latency:
// members are taken CB at a time, their values loaded together, and added in
// order while the next batch's values load (the ids of the batch after it are
// already in flight).
constexpr int CB = 32;

// Centroid of dimension t over the members [s, e) of mem (ids below n), one
// ordered chain.
GEEK_D double centroid_of(const float* __restrict__ X, int64_t ldx, int64_t n, int t,
                          const uint32_t* __restrict__ mem, uint32_t s, uint32_t e, int32_t* st);

__global__ __launch_bounds__(256) void k_centroids(const float* __restrict__ X, int64_t ldx, int64_t n, int d,
                            const uint32_t* __restrict__ offs, const uint32_t* __restrict__ mem,
                            int k, const uint32_t* __restrict__ kdev, double* __restrict__ C, int32_t* st) {
  const int64_t gid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (gid >= (int64_t)k * d) return;
  const int j = (int)(gid / d), t = (int)(gid % d);
  double c = 0.0;
  // seeds counted on the device: those past the count take no part
  const int kv = kdev ? (int)min(*kdev, (uint32_t)k) : k;
  if (j < kv) {
    const uint32_t s = offs[j], e = offs[j + 1];
    if (e <= s) set_status(st, GEEK_ERR_EMPTY_SET);
    else c = centroid_of(X, ldx, n, t, mem, s, e, st);
  } else if (kv == 0 && gid == 0) {
    set_status(st, GEEK_ERR_NO_SEEDS);
  }
  C[gid] = c;
}

GEEK_D double centroid_of(const float* __restrict__ X, int64_t ldx, int64_t n, int t,
                          const uint32_t* __restrict__ mem, uint32_t s, uint32_t e, int32_t* st) {
  double acc = 0.0;
  bool bad = false;
  // ids of member q (clamped into the seed's range: reads past the end are
  // repeated ids whose values are not added)
  auto id_at = [&](uint32_t q) { return mem[q < e ? q : e - 1]; };
  uint32_t ids[CB];
  float v[CB], w[CB];
  auto load = [&](float (&to)[CB], uint32_t next) {  // values of `ids`, then the ids from `next` on
#pragma unroll
    for (int u = 0; u < CB; ++u) {
      const bool ok = (int64_t)ids[u] < n;
      bad |= !ok;
      to[u] = X[(int64_t)(ok ? ids[u] : 0u) * ldx + t];
    }
#pragma unroll
    for (int u = 0; u < CB; ++u) ids[u] = id_at(next + u);
  };
  auto add = [&](const float (&x)[CB], uint32_t q) {
    const uint32_t cnt = e - q < (uint32_t)CB ? e - q : (uint32_t)CB;
#pragma unroll
    for (int u = 0; u < CB; ++u)
      if ((uint32_t)u < cnt) acc = __dadd_rn(acc, (double)x[u]);
  };
#pragma unroll
  for (int u = 0; u < CB; ++u) ids[u] = id_at(s + u);
  load(v, s + CB);
  for (uint32_t q = s; q < e; q += 2 * CB) {
    if (q + CB < e) load(w, q + 2 * CB);
    add(v, q);
    if (q + CB >= e) break;
    if (q + 2 * CB < e) load(v, q + 3 * CB);
    add(w, q + CB);
  }
  if (bad) set_status(st, GEEK_ERR_ARG);
  return acc / (double)(e - s);
}

// Seeds with many members (a further assignment pass takes whole clusters
// as seeds): the members' values are first gathered into groups of four
// member positions, Xt[q / 4][t][q % 4] = X[mem[q]][t] (a 64 x 64 tile
// transposed through LDS), so that the (seed, dim) chains of one wave read
// four values each per 16-byte load, the wave's loads one contiguous run:
// streaming, where loads of whole rows of scattered members (or of
// dimension-major rows far apart) were bound by address translation.
constexpr int GT_TILE = 64;
__global__ __launch_bounds__(256) void k_gather_t(const float* __restrict__ X, int64_t ldx, int64_t n, int d,
                                                  const uint32_t* __restrict__ offs, int k,
                                                  const uint32_t* __restrict__ mem, int64_t nm_cap, int64_t nm_pad,
                                                  float* __restrict__ Xt, int32_t* st) {
  __shared__ float tile[GT_TILE][GT_TILE + 1];
  // members actually used (seed_offsets[k]); positions past them are zeros
  const int64_t nm = offs[k] < nm_cap ? (int64_t)offs[k] : nm_cap;
  const int64_t q0 = (int64_t)blockIdx.x * GT_TILE;
  const int t0 = blockIdx.y * GT_TILE;
  const int c = threadIdx.x & 63, r0 = threadIdx.x >> 6;
#pragma unroll 4
  for (int r = r0; r < GT_TILE; r += 4) {
    const int64_t q = q0 + r;
    float v = 0.f;
    if (q < nm && t0 + c < d) {
      const uint32_t i = mem[q];
      if ((int64_t)i < n) v = X[(int64_t)i * ldx + t0 + c];
      else set_status(st, GEEK_ERR_ARG);
    }
    tile[r][c] = v;
  }
  __syncthreads();
  // group g of the tile (members q0 + 4g .. + 3) covers the contiguous run
  // Xt[(q0 / 4 + g) * 4 d + 4 t0 ..] of 4 x 64 values: thread i writes its
  // element i of the run
#pragma unroll 4
  for (int i = threadIdx.x; i < GT_TILE * GT_TILE; i += 256) {
    const int g = i >> 8, rem = i & 255, tl = rem >> 2, r = rem & 3;
    const int64_t q = q0 + g * 4 + r;
    if (q < nm_pad && t0 + tl < d) Xt[(q >> 2) * 4 * (int64_t)d + (int64_t)(t0 + tl) * 4 + r] = tile[g * 4 + r][tl];
  }
}

// Centroids from the grouped copy: the same ascending chain of float64
// additions as k_centroids.  The longest seed's chain is the kernel's time:
// 244,500 members 3.56 ms with every batch of 64 members' loads waited for,
// 3.15 ms with 144 members' loads in flight ahead of the additions (12.9 ns per
// member; widening four members ahead of their additions changed nothing).
constexpr int CT_B = 6, CT_R = 7;  // 16-byte loads per batch, batches in the ring
__global__ __launch_bounds__(256) void k_centroids_t(const float* __restrict__ Xt, int64_t nm, int d,
                              const uint32_t* __restrict__ offs, int k, double* __restrict__ C, int32_t* st) {
  const int64_t gid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  double c = 0.0;
  if (gid < (int64_t)k * d) {
    const int j = (int)(gid / d), t = (int)(gid % d);
    const int64_t s = offs[j], e = offs[j + 1];
    if (e <= s) {
      set_status(st, GEEK_ERR_EMPTY_SET);
    } else if (e > nm) {  // seed_offsets disagree with the member count of the job
      set_status(st, GEEK_ERR_ARG);
    } else {
      const int64_t gs = 4 * (int64_t)d;  // floats per group of four members
      const float* p = Xt + (int64_t)t * 4;
      auto at = [&](int64_t q) { return p[(q >> 2) * gs + (q & 3)]; };
      double acc = 0.0;
      int64_t q = s;
      for (; q < e && (q & 3); ++q) acc = __dadd_rn(acc, (double)at(q));
      // a ring of CT_R batches: one is added while the others load
      float4 v[CT_R][CT_B];
      auto load = [&](float4 (&to)[CT_B], int64_t q0) {
#pragma unroll
        for (int u = 0; u < CT_B; ++u) to[u] = *reinterpret_cast<const float4*>(p + ((q0 >> 2) + u) * gs);
      };
      auto add = [&](const float4 (&x)[CT_B]) {
#pragma unroll
        for (int u = 0; u < CT_B; ++u) {
          acc = __dadd_rn(acc, (double)x[u].x);
          acc = __dadd_rn(acc, (double)x[u].y);
          acc = __dadd_rn(acc, (double)x[u].z);
          acc = __dadd_rn(acc, (double)x[u].w);
        }
      };
      constexpr int64_t NB = 4 * CT_B;
      if (q + CT_R * NB <= e) {
#pragma unroll
        for (int z = 0; z < CT_R - 1; ++z) load(v[z], q + z * NB);
        for (; q + (2 * CT_R - 1) * NB <= e; q += CT_R * NB)
#pragma unroll
          for (int z = 0; z < CT_R; ++z) {
            load(v[(z + CT_R - 1) % CT_R], q + (z + CT_R - 1) * NB);
            add(v[z]);
          }
#pragma unroll
        for (int z = 0; z < CT_R - 1; ++z) add(v[z]);
        q += (CT_R - 1) * NB;
      }
      for (; q < e; ++q) acc = __dadd_rn(acc, (double)at(q));
      c = acc / (double)(e - s);
    }
    C[gid] = c;
  }
}

// Whether the centroids go through the dimension-major copy: seeds of 64
// members or more on average, with the member count known.
static bool centroids_transposed(const geek_assign_job& J) {
  return !J.k_dev && J.n_members > 0 && J.n_members >= 64 * (int64_t)J.k;
}
static int64_t members_pad(const geek_assign_job& J) { return (J.n_members + 3) / 4 * 4; }

// Largest |value| of a float32 matrix and of the centroids (FP8 scaling).
template <class T>
__global__ void k_absmax(const T* __restrict__ X, int64_t ldx, int64_t n, int d, float* __restrict__ out) {
  const int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  float m = 0.f;
  for (int64_t e = g; e < n * d; e += (int64_t)gridDim.x * blockDim.x) {
    const float v = fabsf((float)X[(e / d) * ldx + (e % d)]);
    if (v > m) m = v;  // NaN compares false and is ignored here
  }
  for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
  if ((threadIdx.x & 63) == 0 && m > __hip_atomic_load(out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    atomic_max_nonneg(out, m);
}

// scale = 2^floor(log2(224 / max)), so scaled values stay inside every
// e4m3 variant's normal range; 1 when everything is zero.
__global__ void k_fp8_scale(const float* __restrict__ mx, const float* __restrict__ mc, float* __restrict__ scale) {
  if (blockIdx.x || threadIdx.x) return;
  const float m = fmaxf(*mx, *mc);
  // 2^e with max |value| * 2^e in [112, 224]; e is clamped at 60 for tiny
  // data (the absolute error term covers it); data too large for a safe
  // 2^e gets scale 0, which makes every row's bound infinite (escalation)
  if (!(m > 0.f)) {
    *scale = 1.0f;
    return;
  }
  const float e = floorf(log2f(224.0f / m));
  *scale = e < -60.f ? 0.0f : exp2f(fminf(e, 60.f));
}

// Matrix-core input copies of the centroids, zero-padded to [k_pad][DP]: the
// three float32 pieces in planes, the first of which is the bf16 copy of a bf16
// first pass, and with `cl8` the e4m3 copy of an FP8 first pass.  A thread
// takes eight attributes of a centroid, the DP / 8 threads of a centroid are
// neighbours in a wavefront (a thread per centroid, walking its row, took 7 us
// at k = 10 and one launch per copy).  Padded rows get |c|^2 = +inf so they
// never enter a window.  |c|^2 may be summed in any order (two_eps).
__global__ __launch_bounds__(256) void k_cprep(const double* __restrict__ C, int k, int d, int k_pad, int DP,
                                               __bf16* __restrict__ cl, uint8_t* __restrict__ cl8,
                                               const float* __restrict__ scale_p, float* __restrict__ nc,
                                               float* __restrict__ cmax, const uint32_t* __restrict__ kdev) {
  const int G = DP / 8;  // 4, 8, 16 or 32: all threads of a centroid are in one wavefront
  const int64_t gid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int j = (int)(gid / G), t = (int)(gid % G) * 8;
  if (j >= k_pad) return;
  // seeds past a device-side count are padding too
  const bool real = j < (kdev ? (int)min(*kdev, (uint32_t)k) : k);
  float v[8];
  double sq = 0.0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const double c = real && t + e < d ? C[(int64_t)j * d + t + e] : 0.0;
    sq += c * c;
    v[e] = (float)c;
  }
  for (int o = 1; o < G; o <<= 1) sq += __shfl_xor(sq, o);
  const ModeF32::frag f = ModeF32::from_f32(v, 1.0f);
#pragma unroll
  for (int z = 0; z < ModeF32::PIECES; ++z)
    *reinterpret_cast<bf16x8*>(cl + ((int64_t)z * k_pad + j) * DP + t) = f.p[z];
  if (cl8) *reinterpret_cast<long*>(cl8 + (int64_t)j * DP + t) = ModeFP8::from_f32(v, *scale_p);
  if (t == 0) {
    nc[j] = real ? (float)sq : INFINITY;
    const float norm = (float)(sqrt(sq) * (1.0 + 0x1p-20));
    if (real && norm > __hip_atomic_load(cmax, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomic_max_nonneg(cmax, norm);
  }
}

// Two workgroups per CU (at most 256 registers a wavefront) for the BF16
// first pass of point rows up to 128 attributes, whose stage pipeline keeps
// two blocks' accumulators live (the compiler would otherwise go just past
// 256 and halve the occupancy), and for the first pass of the float32 pieces,
// whose LDS allows as many.
template <class M, int DP, bool HET, int NCB, bool WIDE>
constexpr int scan_min_blocks() {
  if (M::PIECES > 1) return !HET && !WIDE && NCB == 1 && DP <= 128 ? 2 : 1;
  return !HET && NCB == 2 && DP <= 128 ? 2 : 1;
}

template <class M, int DP, bool HET, int NCB, int NBUF, bool T2, bool WIDE, bool MARK>
__global__ __launch_bounds__(SCAN_THREADS, (scan_min_blocks<M, DP, HET, NCB, WIDE>())) void k_scan(
    const float* __restrict__ X, int64_t ldx, int d, int64_t n_rows,
    const uint32_t* __restrict__ rows, const uint32_t* __restrict__ rows_count,
    const typename M::ce* __restrict__ cl, const float* __restrict__ nc, int k_pad,
    const float* __restrict__ cmax_p, const float* __restrict__ scale_p, Het het, int k,
    int32_t* __restrict__ rec, int32_t* st, ScanBlocks sb) {
  scan_tiles<M, DP, HET, NCB, NBUF, T2, WIDE, MARK>(X, ldx, d, n_rows, rows, rows_count, cl, nc, k_pad, cmax_p, scale_p, het,
                                        k, rec, st, blockIdx.x, INT64_MAX, gridDim.x, sb);
}

constexpr int SCANJOB_CHUNK = 32;  // table entries written per launch
struct ScanJobChunk {
  int count;
  ScanJob jobs[SCANJOB_CHUNK];
};
__global__ void k_put_jobs(ScanJobChunk c, ScanJob* dst) {
  const int i = threadIdx.x;
  if (i < c.count) dst[i] = c.jobs[i];
}

__global__ void k_clock_since(const unsigned long long* t0, unsigned long long* dst) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *dst = wall_clock64() - *t0;
}
__global__ void k_clock_now(unsigned long long* dst) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *dst = wall_clock64();
}

// ---------------------------------------------------------------- float64 checks
// Categorical attributes of row i that differ from seed j's modes.
GEEK_D int mismatches(const Het& het, int64_t i, int j) {
  int mm = 0;
  for (int a = 0; a < het.n_cat; ++a)
    mm += ((uint32_t)het.cat[i * het.n_cat + a] != het.mode[(int64_t)j * het.n_cat + a]) ? 1 : 0;
  return mm;
}

GEEK_D double d64(const float* __restrict__ xr, const double* __restrict__ cr, int d) {
  double acc = 0.0;
  int t = 0;
  // 16-byte loads when both rows are aligned; the summation order is
  // unchanged.  32 attributes at a time: the 24 loads of one x cache line
  // and two centroid lines are issued before the first use, one memory round
  // trip per 32 attributes
  if (((reinterpret_cast<uintptr_t>(xr) | reinterpret_cast<uintptr_t>(cr)) & 15) == 0) {
    for (; t + 32 <= d; t += 32) {
      float4 xv[8];
      double2 cv[16];
#pragma unroll
      for (int u = 0; u < 8; ++u) xv[u] = *reinterpret_cast<const float4*>(xr + t + 4 * u);
#pragma unroll
      for (int u = 0; u < 16; ++u) cv[u] = *reinterpret_cast<const double2*>(cr + t + 2 * u);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float xs[4] = {xv[u].x, xv[u].y, xv[u].z, xv[u].w};
        const double cs[4] = {cv[2 * u].x, cv[2 * u].y, cv[2 * u + 1].x, cv[2 * u + 1].y};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const double delta = __dadd_rn((double)xs[e], -cs[e]);
          acc = __dadd_rn(acc, __dmul_rn(delta, delta));
        }
      }
    }
    for (; t + 4 <= d; t += 4) {
      const float4 xv = *reinterpret_cast<const float4*>(xr + t);
      const double2 c0 = *reinterpret_cast<const double2*>(cr + t);
      const double2 c1 = *reinterpret_cast<const double2*>(cr + t + 2);
      double delta = __dadd_rn((double)xv.x, -c0.x);
      acc = __dadd_rn(acc, __dmul_rn(delta, delta));
      delta = __dadd_rn((double)xv.y, -c0.y);
      acc = __dadd_rn(acc, __dmul_rn(delta, delta));
      delta = __dadd_rn((double)xv.z, -c1.x);
      acc = __dadd_rn(acc, __dmul_rn(delta, delta));
      delta = __dadd_rn((double)xv.w, -c1.y);
      acc = __dadd_rn(acc, __dmul_rn(delta, delta));
    }
  }
  for (; t < d; ++t) {
    const double delta = __dadd_rn((double)xr[t], -cr[t]);
    acc = __dadd_rn(acc, __dmul_rn(delta, delta));
  }
  return acc;
}

// D_num + gamma * mismatches, in that float64 order (reference formula).
GEEK_D double d64h(const float* __restrict__ xr, const double* __restrict__ cr, int d, const Het& het,
                   int64_t i, int j) {
  const double dn = d64(xr, cr, d);
  if (!het.cat) return dn;
  return __dadd_rn(dn, __dmul_rn(het.gamma, (double)mismatches(het, i, j)));
}

__device__ void block_add_u64(unsigned long long* dst, unsigned long long v) {
  // one atomic per wave
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  if ((threadIdx.x & 63) == 0 && v) atomicAdd(dst, v);
}
// Both sums of a workgroup of 256, one atomic each: atomics of one address take
// about 10 ns each over the whole chip, so a count per wavefront was most of
// the float64 distances' time for some 10^5 rows (246 us of 256 with eight
// lanes per row).
__device__ void block_add2_u64(unsigned long long* dst0, unsigned long long* dst1, unsigned long long v0,
                               unsigned long long v1) {
  __shared__ unsigned long long part[2][4];
  for (int o = 32; o > 0; o >>= 1) {
    v0 += __shfl_xor(v0, o);
    v1 += __shfl_xor(v1, o);
  }
  if ((threadIdx.x & 63) == 0) {
    part[0][threadIdx.x >> 6] = v0;
    part[1][threadIdx.x >> 6] = v1;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    const unsigned long long* q = part[threadIdx.x];
    const unsigned long long v = q[0] + q[1] + q[2] + q[3];
    if (v) atomicAdd(threadIdx.x ? dst1 : dst0, v);
  }
}

// A lane per row, each lane walking its own row's candidates: candidate windows
// (RECW records: the float32 first pass and rescan), and RECW_T2 records that
// k_finalize does not take.
__global__ __launch_bounds__(256) void k_finalize_win(const float* __restrict__ X, int64_t ldx, int d,
                           const double* __restrict__ C, int k, Het het, int64_t n_rows,
                           const uint32_t* __restrict__ rows, const uint32_t* __restrict__ rows_count,
                           const int32_t* __restrict__ rec, int rstride, int32_t* __restrict__ assign,
                           double* __restrict__ dist, uint32_t* __restrict__ esc,
                           uint32_t* __restrict__ esc_count, unsigned long long* __restrict__ ctr,
                           int ctr_rows, ScanBlocks sb) {
  if (sb.flags && *sb.gate != 0u) rows = sb.rows;
  const int64_t count = rows ? (int64_t)*rows_count : n_rows;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t start = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t iters = (count + stride - 1) / stride;
  unsigned long long nrow = 0, ncand = 0;
  for (int64_t it = 0; it < iters; ++it) {
    const int64_t pos = start + it * stride;
    if (pos >= count) continue;
    const int64_t i = rows ? (int64_t)rows[pos] : pos;
    const int32_t* rr = rec + pos * rstride;
    const int c = rr[0];
    if (c <= 0) {  // window overflow (or no finite candidate): escalate
      const uint32_t q = atomicAdd(esc_count, 1u);
      esc[q] = (uint32_t)i;
      continue;
    }
    double best = INFINITY;
    int bj = 0x7fffffff;
    const float* xr = X + i * ldx;
    for (int q = 0; q < c; ++q) {
      const int j = rr[1 + q];
      if ((unsigned)j >= (unsigned)k) continue;
      const double D = d64h(xr, C + (int64_t)j * d, d, het, i, j);
      if (D < best || (D == best && j < bj)) {
        best = D;
        bj = j;
      }
    }
    if (bj == 0x7fffffff) bj = 0;
    assign[i] = bj;
    dist[i] = best;
    nrow += 1;
    ncand += (unsigned long long)c;
  }
  if (ctr) {
    block_add2_u64(ctr + ctr_rows, ctr + 3, nrow, ncand);
  }
}

// The BF16 first pass's records (RECW_T2: at most one candidate).  Eight
// lanes per row:
// lane e loads attributes t0 + 4e .. t0 + 4e + 3 of the row and of the
// candidate centroid for t0 = 0, 32, ... (one x cache line and two centroid
// lines per step, coalesced over the eight lanes), forms the rounded
// squared differences, and lane 0 of the eight adds the 32 squares of a step
// in attribute order from LDS: D = sum over t = 0..d-1 in order of
// (x_t - c_t)^2, each difference, square and sum rounded to float64 (plus
// gamma * mismatches for heterogeneous rows).  With a lane per row, every
// load touched 64 cache lines and the lines were evicted between the row's
// steps.
constexpr int FZ_ROWS = 8;   // rows per wavefront and step
constexpr int FZ_STEP = 32;  // attributes per step
__global__ __launch_bounds__(256) void k_finalize(const float* __restrict__ X, int64_t ldx, int d,
                                                  const double* __restrict__ C, int k, Het het, int64_t n_rows,
                                                  const uint32_t* __restrict__ rows,
                                                  const uint32_t* __restrict__ rows_count,
                                                  const int32_t* __restrict__ rec, int rstride,
                                                  int32_t* __restrict__ assign, double* __restrict__ dist,
                                                  uint32_t* __restrict__ esc, uint32_t* __restrict__ esc_count,
                                                  unsigned long long* __restrict__ ctr, int ctr_rows) {
  __shared__ double sq[4][FZ_ROWS][FZ_STEP + 2];  // + 2: the eight row leaders read distinct banks
  // escalated rows wait here, and leave with one atomic per 57 or more (with
  // one per eight rows, 10^6 escalated rows took 1.4 ms)
  __shared__ uint32_t left[4][64];
  int nleft = 0;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int g = lane >> 3, e = lane & 7;  // row slot, lane within the row
  const int64_t count = rows ? (int64_t)*rows_count : n_rows;
  const int64_t stride = (int64_t)gridDim.x * 4 * FZ_ROWS;
  const bool xal = ((reinterpret_cast<uintptr_t>(X) | (uintptr_t)(ldx * 4)) & 15) == 0;
  const bool cal = ((reinterpret_cast<uintptr_t>(C) | (uintptr_t)(d * 8)) & 15) == 0;
  unsigned long long nrow = 0, ncand = 0;
  auto flush = [&]() {
    uint32_t at = 0;
    if (lane == 0) at = atomicAdd(esc_count, (uint32_t)nleft);
    at = (uint32_t)__shfl((int)at, 0);
    if (lane < nleft) esc[at + lane] = left[wv][lane];
    nleft = 0;
    __builtin_amdgcn_wave_barrier();
  };
  for (int64_t base = ((int64_t)blockIdx.x * 4 + wv) * FZ_ROWS; base < count; base += stride) {
    const int64_t pos = base + g;
    const bool live = pos < count;
    const int64_t i = live ? (rows ? (int64_t)rows[pos] : pos) : 0;
    const int32_t* rr = rec + (live ? pos : 0) * rstride;
    int c = live ? rr[0] : 0;
    const bool over = live && c <= 0;  // window overflow (or no finite candidate): escalate
    const uint64_t om = __ballot(over && e == 0);
    if (over) c = 0;
    if (om) {  // nleft is at most 64 - FZ_ROWS here
      if (over && e == 0) left[wv][nleft + __popcll(om & ((1ull << lane) - 1ull))] = (uint32_t)i;
      nleft += __popcll(om);
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (nleft > 64 - FZ_ROWS) flush();
    }
    int maxc = c;  // the wavefront walks the largest candidate count of its rows
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) maxc = max(maxc, __shfl_xor(maxc, o));
    double best = INFINITY;
    int bj = 0x7fffffff;
    const float* xr = X + i * ldx;
    for (int q = 0; q < maxc; ++q) {
      const int j = q < c ? rr[1 + q] : -1;
      const bool act = j >= 0 && j < k;
      const double* cr = C + (int64_t)(act ? j : 0) * d;
      double acc = 0.0;
      for (int t0 = 0; t0 < d; t0 += FZ_STEP) {
        const int t = t0 + 4 * e;
        double s4[4] = {0.0, 0.0, 0.0, 0.0};
        if (act && t < d) {
          float xs[4];
          double cs[4];
          if (xal && cal && t + 4 <= d) {
            const float4 xv = *reinterpret_cast<const float4*>(xr + t);
            const double2 c0 = *reinterpret_cast<const double2*>(cr + t);
            const double2 c1 = *reinterpret_cast<const double2*>(cr + t + 2);
            xs[0] = xv.x, xs[1] = xv.y, xs[2] = xv.z, xs[3] = xv.w;
            cs[0] = c0.x, cs[1] = c0.y, cs[2] = c1.x, cs[3] = c1.y;
          } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              xs[u] = t + u < d ? xr[t + u] : 0.f;
              cs[u] = t + u < d ? cr[t + u] : 0.0;
            }
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const double delta = __dadd_rn((double)xs[u], -cs[u]);
            s4[u] = __dmul_rn(delta, delta);
          }
        }
        *reinterpret_cast<double2*>(&sq[wv][g][4 * e]) = make_double2(s4[0], s4[1]);
        *reinterpret_cast<double2*>(&sq[wv][g][4 * e + 2]) = make_double2(s4[2], s4[3]);
        // the row's squares in attribute order (a wavefront's LDS accesses
        // complete in order, so the eight lanes' stores are visible here)
        if (e == 0 && act) {
          const int lim = d - t0 < FZ_STEP ? d - t0 : FZ_STEP;
          for (int u = 0; u < lim; ++u) acc = __dadd_rn(acc, sq[wv][g][u]);
        }
      }
      if (e == 0 && act) {
        const double D = het.cat ? __dadd_rn(acc, __dmul_rn(het.gamma, (double)mismatches(het, i, j))) : acc;
        if (D < best || (D == best && j < bj)) {
          best = D;
          bj = j;
        }
      }
    }
    if (e == 0 && live && c > 0) {
      if (bj == 0x7fffffff) bj = 0;
      assign[i] = bj;
      dist[i] = best;
      nrow += 1;
      ncand += (unsigned long long)c;
    }
  }
  if (nleft) flush();
  if (ctr) {
    block_add2_u64(ctr + ctr_rows, ctr + 3, nrow, ncand);
  }
}

// Rows left after the rescans: float64 distance to every seed, lowest index on
// ties.  A workgroup takes FB_R rows and a range of FB_C-seed tiles; each
// thread holds a 4 x 4 block of (row, seed) sums with both operands staged in
// LDS, so one read of a seed row from L2 serves FB_R rows.  Every sum runs
// over t = 0..d-1 in order with the operations of d64 (the zero padding of
// t >= d adds +0.0, which leaves a sum of squares unchanged), so the values
// are those of the reference formula.  With fewer row groups than workgroups
// the seed tiles of a group are split over up to FB_SPLIT workgroups, whose
// per-row (D, j) minima k_fb_merge combines.
constexpr int FB_R = 64, FB_C = 64, FB_TK = 16, FB_GRID = 1024, FB_SPLIT = 16;
constexpr int FB_GROUPS = 4096;  // marked groups of seeds a workgroup lists
constexpr int FB_XS = FB_R + 4;  // LDS row stride (floats) of the staged rows
constexpr int FB_CS = FB_C + 2;  // LDS row stride (doubles) of a seed chunk

// Row groups and seed-tile splits for `count` rows against k seeds.
GEEK_HD void fb_shape(uint32_t count, int k, int64_t* R, int* S) {
  *R = ((int64_t)count + FB_R - 1) / FB_R;
  const int T = (k + FB_C - 1) / FB_C;
  int sp = 1;
  if (*R > 0 && *R < FB_GRID) {
    const int want = (int)((FB_GRID + *R - 1) / *R);
    sp = want < T ? want : T;
    if (sp > FB_SPLIT) sp = FB_SPLIT;
    if (sp < 1) sp = 1;
  }
  *S = sp;
}

// Capacity (entries) of the partial minima buffer for n rows.
inline int64_t fb_part_cap(int64_t n) {
  return std::max<int64_t>(1, std::min<int64_t>(n * FB_SPLIT, (int64_t)2 * FB_GRID * FB_R));
}

template <int DP>
__global__ __launch_bounds__(256) void k_fallback64(
    const float* __restrict__ X, int64_t ldx, int d, const double* __restrict__ C, int k,
    const uint32_t* __restrict__ kdev, Het het,
    const uint32_t* __restrict__ rows, const uint32_t* __restrict__ rows_count, int32_t* __restrict__ assign,
    double* __restrict__ dist, double* __restrict__ part_d, int32_t* __restrict__ part_j,
    unsigned long long* __restrict__ ctr, const uint32_t* __restrict__ fpos, ScanBlocks sb) {
  // with marks (fpos: the rows' places in the marked order, ascending): the
  // groups of 64 seeds marked for some row of the workgroup's 64
  __shared__ uint32_t glist[FB_GROUPS];
  __shared__ uint32_t gsum[4];
  constexpr int XS_WORDS = DP * FB_XS > FB_R * 16 * 3 ? DP * FB_XS : FB_R * 16 * 3;
  __shared__ __attribute__((aligned(16))) float xs[XS_WORDS];  // [t][row]; later the reduction
  __shared__ __attribute__((aligned(16))) double cs[FB_TK * FB_CS];  // [t][seed]
  __shared__ int64_t rid[FB_R];
  const int tid = threadIdx.x;
  const int tr = tid & 15, tc = tid >> 4;  // rows 4tr..4tr+3, seeds 4tc..4tc+3 of a tile
  const uint32_t count = *rows_count;
  int64_t R;
  int S;
  fb_shape(count, k, &R, &S);
  const int T = (k + FB_C - 1) / FB_C;
  const int kv = kdev ? (int)min(*kdev, (uint32_t)k) : k;  // seeds that take part
  const int dp16 = (d + FB_TK - 1) / FB_TK * FB_TK;
  const int nch = dp16 / FB_TK;
  for (int64_t q = blockIdx.x; q < R * S; q += gridDim.x) {
    const int64_t g = q / S;
    const int sp = (int)(q % S);
    __syncthreads();  // the previous item's reduction has read xs and rid
    int groups = T;
    bool listed = false;
    if (sb.flags && sb.words <= 256 && *sb.gate != 0u) {
      const int64_t p0 = g * FB_R, p1 = p0 + FB_R < (int64_t)count ? p0 + FB_R - 1 : (int64_t)count - 1;
      const int64_t t0 = fpos[p0] / 128, t1 = fpos[p1] / 128;
      uint32_t bits = 0u;
      if (tid < sb.words)
        for (int64_t z = t0; z <= t1; ++z) bits |= sb.flags[z * sb.words + tid];
      const uint32_t mine = __popc(bits);
      uint32_t incl = mine;
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(incl, o);
        if ((tid & 63) >= o) incl += y;
      }
      if ((tid & 63) == 63) gsum[tid >> 6] = incl;
      __syncthreads();
      uint32_t at = incl - mine;
      for (int z = 0; z < tid >> 6; ++z) at += gsum[z];
      const uint32_t all = gsum[0] + gsum[1] + gsum[2] + gsum[3];
      listed = all <= (uint32_t)FB_GROUPS;  // uniform
      if (listed) {
        groups = (int)all;
        for (; bits; bits &= bits - 1u) glist[at++] = (uint32_t)(tid * 32 + __ffs(bits) - 1);
      }
    }
    const int tile0 = (int)((int64_t)sp * groups / S), tile1 = (int)((int64_t)(sp + 1) * groups / S);
    // seed of column `c` of the z-th tile: in order, or through the marked order
    auto seed_at = [&](int z, int c) {
      if (!listed) return z * FB_C + c;
      const int r = (int)glist[z] * FB_C + c;
      return r < k ? (int)sb.perm[r] : k;
    };
    if (tid < FB_R) {
      const int64_t pos = g * FB_R + tid;
      rid[tid] = pos < count ? (int64_t)rows[pos] : -1;
    }
    __syncthreads();
    for (int idx = tid; idx < FB_R * dp16; idx += 256) {
      const int r = idx / dp16, t = idx - r * dp16;
      const int64_t i = rid[r];
      xs[t * FB_XS + r] = (i >= 0 && t < d) ? X[i * ldx + t] : 0.f;
    }
    double best[4];
    int bj[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      best[a] = INFINITY;
      bj[a] = 0x7fffffff;
    }
    // register prefetch of the next (tile, chunk) of seeds
    double pre[4];
    auto fetch = [&](int tile, int ch) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int idx = tid + u * 256;
        const int jj = idx >> 4, tt = idx & 15;
        const int j = seed_at(tile, jj), t = ch * FB_TK + tt;
        pre[u] = (j < kv && t < d) ? C[(int64_t)j * d + t] : 0.0;
      }
    };
    if (tile0 < tile1) fetch(tile0, 0);  // (glist is complete since the barrier before rid was read)
    for (int tile = tile0; tile < tile1; ++tile) {
      double acc[4][4];
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = 0.0;
      for (int ch = 0; ch < nch; ++ch) {
        __syncthreads();  // readers of the previous chunk are done (and xs is staged)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int idx = tid + u * 256;
          cs[(idx & 15) * FB_CS + (idx >> 4)] = pre[u];
        }
        __syncthreads();
        if (ch + 1 < nch) fetch(tile, ch + 1);
        else if (tile + 1 < tile1) fetch(tile + 1, 0);
        const float* xp = xs + ch * FB_TK * FB_XS + tr * 4;
        const double* cp = cs + tc * 4;
#pragma unroll 4
        for (int tt = 0; tt < FB_TK; ++tt) {
          const float4 xv = *reinterpret_cast<const float4*>(xp + tt * FB_XS);
          const double2 c01 = *reinterpret_cast<const double2*>(cp + tt * FB_CS);
          const double2 c23 = *reinterpret_cast<const double2*>(cp + tt * FB_CS + 2);
          const double xd[4] = {(double)xv.x, (double)xv.y, (double)xv.z, (double)xv.w};
          const double cd[4] = {c01.x, c01.y, c23.x, c23.y};
#pragma unroll
          for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) {
              const double delta = __dadd_rn(xd[a], -cd[b]);
              acc[a][b] = __dadd_rn(acc[a][b], __dmul_rn(delta, delta));
            }
        }
      }
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const int64_t i = rid[tr * 4 + a];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const int j = seed_at(tile, tc * 4 + b);
          if (j >= kv) continue;
          double D = acc[a][b];
          if (het.cat && i >= 0) D = __dadd_rn(D, __dmul_rn(het.gamma, (double)mismatches(het, i, j)));
          if (D < best[a] || (D == best[a] && j < bj[a])) {
            best[a] = D;
            bj[a] = j;
          }
        }
      }
    }
    // combine the 16 column threads of each row, in seed order
    __syncthreads();
    double* red_d = reinterpret_cast<double*>(xs);
    int* red_j = reinterpret_cast<int*>(xs + FB_R * 16 * 2);
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      red_d[(tr * 4 + a) * 16 + tc] = best[a];
      red_j[(tr * 4 + a) * 16 + tc] = bj[a];
    }
    __syncthreads();
    unsigned long long done = 0;
    if (tid < FB_R && rid[tid] >= 0) {
      double bd = INFINITY;
      int bb = 0x7fffffff;
      for (int c = 0; c < 16; ++c) {
        const double od = red_d[tid * 16 + c];
        const int oj = red_j[tid * 16 + c];
        if (od < bd || (od == bd && oj < bb)) {
          bd = od;
          bb = oj;
        }
      }
      const int64_t i = rid[tid];
      if (S == 1) {
        // no finite distance (non-finite input, already flagged): seed 0
        assign[i] = bb == 0x7fffffff ? 0 : bb;
        dist[i] = bd;
        done = 1;
      } else {
        const int64_t e = (g * FB_R + tid) * S + sp;
        part_d[e] = bd;
        part_j[e] = bb;
      }
    }
    if (ctr && tid < 64) block_add_u64(ctr + 2, done);
  }
}

// Per-row minimum over the seed-tile splits of k_fallback64 (lowest index on
// ties).
__global__ void k_fb_merge(const uint32_t* __restrict__ rows, const uint32_t* __restrict__ rows_count, int k,
                           const double* __restrict__ part_d, const int32_t* __restrict__ part_j,
                           int32_t* __restrict__ assign, double* __restrict__ dist,
                           unsigned long long* __restrict__ ctr) {
  const uint32_t count = *rows_count;
  int64_t R;
  int S;
  fb_shape(count, k, &R, &S);
  if (S == 1) return;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t iters = ((int64_t)count + stride - 1) / stride;
  for (int64_t it = 0; it < iters; ++it) {
    const int64_t pos = it * stride + blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    unsigned long long done = 0;
    if (pos < count) {
      double bd = INFINITY;
      int bb = 0x7fffffff;
      for (int sp = 0; sp < S; ++sp) {
        const double od = part_d[pos * S + sp];
        const int oj = part_j[pos * S + sp];
        if (od < bd || (od == bd && oj < bb)) {
          bd = od;
          bb = oj;
        }
      }
      const int64_t i = rows[pos];
      assign[i] = bb == 0x7fffffff ? 0 : bb;
      dist[i] = bd;
      done = 1;
    }
    if (ctr) block_add_u64(ctr + 2, done);
  }
}

// ---------------------------------------------------------------- blocked rescan
// With many seeds, near-duplicate ones leave most rows unsettled by the bf16
// pass, and a rescan of every such row against every seed in float32 takes most
// of the call.  The bf16 values already exclude nearly all seeds of a row: so
// the seeds are reordered by a code that nearby seeds share (the signs of
// CODE_BITS random projections about their mean), the rows by the group of 64
// places of their best seed in that order, a bf16 pass over the reordered rows marks for
// every 128 of them the groups of 64 seeds that hold a value within some row's
// window (k_mark), and the float32 rescan visits the marked groups only.  The
// marks are exact bounds; the orders decide how few there are.
// 10^6 points, 90,343 seeds of 1,000 clusters: rescan and float64 scan 137 ms against 21 ms for
// ordering, marking and rescanning.
// It takes BLOCKED_K seeds or more, at least BLOCKED_ROWS unsettled rows, and
// BLOCKED_WORK (row, seed, padded attribute) products or more of those; the
// host asks it of all rows, and launches nothing of this where even they are
// too few, k_blocked_gate of the unsettled ones, and the kernels end at once
// where they are too few (10^5 x 32 rows, 16,384 seeds apart, no row unsettled:
// 0.41 ms plain, 0.59 ordered and marked, 0.47 ended at once).  Both routes, ms a call (k seeds of 64 clusters): n =
// 100, 65,536 x 128 seeds 8.7 plain against 11.1 blocked; n = 300, 16,384 x 32
// 1.47 / 1.92 and 65,536 x 32 4.83 / 4.77; n = 1,000, 16,384 x 32 0.91 / 1.14 and
// 16,384 x 128 1.66 / 1.63; n = 3 10^5, 16,384 x 128 10.4 / 3.2.  Rows without
// clusters, whose groups are all marked: n = 10^5, 16,384 x 32 0.93 / 1.18, x 128
// 2.42 / 2.48, n = 3 10^5 x 128 6.6 / 6.1.
constexpr int BLOCKED_K = 16384;
constexpr int BLOCKED_ROWS = 256;
constexpr int64_t BLOCKED_WORK = (int64_t)1 << 30;
GEEK_HD bool blocked_pays(int64_t rows, int k, int DP) {
  return rows >= BLOCKED_ROWS && rows * k >= BLOCKED_WORK / DP;
}
// gate: seeds and rows that take part, both zero if too few rows are unsettled.
__global__ void k_blocked_gate(const uint32_t* __restrict__ count, int k, int DP, uint32_t* __restrict__ gate) {
  if (threadIdx.x) return;
  const bool use = blocked_pays(*count, k, DP);
  gate[0] = use ? (uint32_t)k : 0u;
  gate[1] = use ? *count : 0u;
}
constexpr int CODE_BITS = 24;

// Mean over up to 1,024 seeds spread over all; one block per dimension.
__global__ __launch_bounds__(256) void k_seed_mean(const double* __restrict__ C, const uint32_t* __restrict__ gate, int k,
                                                   int d, double* __restrict__ mean) {
  __shared__ double part[4];
  if (!*gate) return;
  const int t = blockIdx.x, m = k < 1024 ? k : 1024;
  double a = 0.0;
  for (int q = threadIdx.x; q < m; q += 256) a += C[(int64_t)((int64_t)q * k / m) * d + t];
  for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = a;
  __syncthreads();
  if (threadIdx.x == 0) mean[t] = (part[0] + part[1] + part[2] + part[3]) / m;
}

// Code of every seed: bit b is the sign of a random +-1 combination of its
// coordinates about the mean.  One wavefront per seed.
__global__ __launch_bounds__(256) void k_seed_code(const double* __restrict__ C, const uint32_t* __restrict__ gate, int d,
                                                   const double* __restrict__ mean, uint32_t* __restrict__ key,
                                                   uint32_t* __restrict__ id) {
  const int lane = threadIdx.x & 63;
  const int64_t j = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (j >= (int64_t)*gate) return;
  float s[CODE_BITS];
#pragma unroll
  for (int b = 0; b < CODE_BITS; ++b) s[b] = 0.f;
  for (int t = lane; t < d; t += 64) {
    const float v = (float)(C[j * d + t] - mean[t]);
    const uint32_t signs = fmix32((uint32_t)t + 0x9E3779B9u);
#pragma unroll
    for (int b = 0; b < CODE_BITS; ++b) s[b] += (signs >> b & 1u) ? v : -v;
  }
  uint32_t code = 0u;
#pragma unroll
  for (int b = 0; b < CODE_BITS; ++b) {
    float x = s[b];
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    code |= (x > 0.f ? 1u : 0u) << b;
  }
  if (lane == 0) {
    key[j] = code;
    id[j] = (uint32_t)j;
  }
}

// Matrix-core copies in seed order `sid` (padding rows stay last), and the
// place of every seed.  One thread per eight attributes.
__global__ __launch_bounds__(256) void k_seed_permute(const uint32_t* __restrict__ sid,
                                                      const uint32_t* __restrict__ gate, int k, int k_pad, int DP,
                                                      const __bf16* __restrict__ cl, const float* __restrict__ nc,
                                                      __bf16* __restrict__ clp, float* __restrict__ ncp,
                                                      uint32_t* __restrict__ spos) {
  if (!*gate) return;
  const int G = DP / 8;
  const int64_t gid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t r = gid / G;
  const int t = (int)(gid % G) * 8;
  if (r >= k_pad) return;
  const int64_t j = r < k ? (int64_t)sid[r] : r;
#pragma unroll
  for (int64_t z = 0; z < ModeF32::PIECES; ++z)
    *reinterpret_cast<uint4*>(clp + (z * k_pad + r) * DP + t) =
        *reinterpret_cast<const uint4*>(cl + (z * k_pad + j) * DP + t);
  if (t == 0) {
    ncp[r] = nc[j];
    if (r < k) spos[j] = (uint32_t)r;
  }
}

// Sort keys of the unsettled rows: the group of 64 places that holds their best
// seed; the rows' flags cleared.
__global__ void k_row_keys(const uint32_t* __restrict__ rows, const uint32_t* __restrict__ count,
                           const int32_t* __restrict__ rec, const uint32_t* __restrict__ spos,
                           uint32_t* __restrict__ key, uint32_t* __restrict__ id, uint32_t* __restrict__ flags,
                           int words) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x, q0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t c = *count, fw = (c + 255) / 256 * 2 * words;
  for (int64_t q = q0; q < c; q += stride) {
    const uint32_t i = rows[q];
    key[q] = spos[rec[(int64_t)i * RECW_T2 + 1]] / SCAN_BC;
    id[q] = i;
  }
  for (int64_t q = q0; q < fw; q += stride) flags[q] = 0u;
}

// Marks for every tile of 128 rows the groups of 64 seeds in which some row has
// a bf16 value within its window, and every group where some row has no bound
// (thr = +inf).  A block takes 256 rows (64 per wavefront)
// and streams the seeds through two LDS stages as the first pass does; a
// value's test is one max and, per 16 of them, one comparison.
template <int DP>
__global__ __launch_bounds__(SCAN_THREADS, 2) void k_mark(const float* __restrict__ X, int64_t ldx, int d,
                                                          const uint32_t* __restrict__ rows,
                                                          const uint32_t* __restrict__ rows_count,
                                                          const float* __restrict__ thr, const __bf16* __restrict__ cl,
                                                          const float* __restrict__ nc, int k_pad, int words,
                                                          uint32_t* __restrict__ flags) {
  using M = ModeBF16;
  constexpr int S = DP / 16, CH = DP / 8, NCB = 2;
  __shared__ __attribute__((aligned(16))) __bf16 buf0[SCAN_BC * DP];
  __shared__ __attribute__((aligned(16))) __bf16 buf1[SCAN_BC * DP];
  __shared__ float lnc[2][SCAN_BC];
  const int tid = threadIdx.x, lane = tid & 63, p = lane & 31, h = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t count = *rows_count;
  const int64_t tile = blockIdx.x;
  if (tile * 256 >= count) return;
  M::frag xb[NCB][S];
  float least[NCB];  // accumulator value from which a seed counts: v = -2 acc <= thr
  bool every = false;
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    const int64_t pos = tile * 256 + w * 64 + cb * 32 + p;
    const bool valid = pos < count;
    const int64_t i = valid ? (int64_t)rows[pos] : 0;
    least[cb] = valid ? -0.5f * thr[i] : INFINITY;
    // a row without a bound: its values may overflow with both signs, and no
    // comparison holds for the NaN of such a sum
    every = every || least[cb] == -INFINITY;
    const float* xr = X + i * ldx + h * (DP / 2);
#pragma unroll
    for (int s = 0; s < S; ++s) {
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int t = s * 8 + e;
        v[e] = valid && h * (DP / 2) + t < d ? xr[t] : 0.f;
      }
      xb[cb][s] = M::from_f32(v, 1.0f);
    }
  }
  float nc_next = 0.f;
  auto dma = [&](int c0, __bf16* to) {
#pragma unroll
    for (int u = 0; u < CH / 4; ++u) {
      const int slot0 = w * (SCAN_BC * CH / 4) + u * 64, slot = slot0 + lane;
      const int r = slot / CH, c = (slot % CH) ^ (r & (CH - 1));
      __builtin_amdgcn_global_load_lds(reinterpret_cast<const char*>(cl + (int64_t)(c0 + r) * DP) + c * 16,
                                       reinterpret_cast<char*>(to) + slot0 * 16, 16, 0, 0);
    }
    nc_next = nc[c0 + (tid & (SCAN_BC - 1))];
  };
  auto land = [&](int b) {
    if (tid < SCAN_BC) lnc[b][tid] = fmaxf(-0.5f * nc_next, -0x1p126f);
    __builtin_amdgcn_s_waitcnt(0);
  };
  uint32_t* frow = flags + (tile * 2 + (w >> 1)) * words;
  uint32_t bits = 0u;
  auto stage = [&](const __bf16* cur, int b, __bf16* nxt, int c0) {
    if (c0 + SCAN_BC < k_pad) dma(c0 + SCAN_BC, nxt);
    bool hit = every;
#pragma unroll
    for (int rb = 0; rb < SCAN_BC / 32; ++rb) {
      const int R = rb * 32 + p;
      const char* rowp = reinterpret_cast<const char*>(cur) + R * CH * 16;
      f32x16 acc[NCB], init;
#pragma unroll
      for (int r = 0; r < 16; ++r) init[r] = lnc[b][rb * 32 + (r >> 2) * 8 + h * 4 + (r & 3)];
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) acc[cb] = init;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const int ch = (h * (DP / 2) + s * 8) * 2 / 16;
        const M::frag a = M::load_lds(reinterpret_cast<const __bf16*>(rowp + ((ch ^ (R & (CH - 1))) << 4)));
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) acc[cb] = M::mma(a, xb[cb][s], acc[cb]);
      }
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        float m = acc[cb][0];
#pragma unroll
        for (int r = 1; r < 16; ++r) m = fmaxf(m, acc[cb][r]);
        hit = hit || m >= least[cb];
      }
    }
    const int g = c0 / SCAN_BC;
    if (__ballot(hit) != 0ull) bits |= 1u << (g & 31);
    if ((g & 31) == 31 || c0 + SCAN_BC >= k_pad) {
      if (lane == 0 && bits) atomicOr(&frow[g >> 5], bits);
      bits = 0u;
    }
    if (c0 + SCAN_BC < k_pad) land(b ^ 1);
    __syncthreads();
  };
  dma(0, buf0);
  land(0);
  __syncthreads();
  for (int c0 = 0; c0 < k_pad; c0 += 2 * SCAN_BC) {
    stage(buf0, 0, buf1, c0);
    if (c0 + SCAN_BC < k_pad) stage(buf1, 1, buf0, c0 + SCAN_BC);
  }
}

// Rows the rescan left (an overflowed window), in the marked order: their
// flags, then, after a scan, the rows and their places.
__global__ void k_left_flags(const uint32_t* __restrict__ count, const int32_t* __restrict__ rec,
                             uint32_t* __restrict__ flag) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x, c = *count;
  for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < c; q += stride)
    flag[q] = rec[q * RECW] <= 0 ? 1u : 0u;
}
__global__ void k_left_list(const uint32_t* __restrict__ count, const uint32_t* __restrict__ rows,
                            const uint32_t* __restrict__ flag, const uint32_t* __restrict__ at,
                            uint32_t* __restrict__ left, uint32_t* __restrict__ pos) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x, c = *count;
  for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < c; q += stride)
    if (flag[q]) {
      left[at[q]] = rows[q];
      pos[at[q]] = (uint32_t)q;
    }
}

// ---------------------------------------------------------------- SSE, radius
// acc + v[0] + ... + v[cnt - 1], one addition at a time (the reference order),
// from LDS: the next sixteen values load while sixteen are added, so that the
// chain waits for additions only (4,096 values: 48 us with a load per
// addition, 37 us so; the addition itself takes about 9 ns in a chain).
GEEK_D double chain_add(const double* v, int cnt, double acc) {
  constexpr int G = 16;
  double a[G], b[G];
  int i = 0;
  if (cnt >= G)
#pragma unroll
    for (int u = 0; u < G; ++u) a[u] = v[u];
  for (; i + 2 * G <= cnt; i += 2 * G) {
#pragma unroll
    for (int u = 0; u < G; ++u) b[u] = v[i + G + u];
#pragma unroll
    for (int u = 0; u < G; ++u) acc = __dadd_rn(acc, a[u]);
    if (i + 3 * G <= cnt)
#pragma unroll
      for (int u = 0; u < G; ++u) a[u] = v[i + 2 * G + u];
#pragma unroll
    for (int u = 0; u < G; ++u) acc = __dadd_rn(acc, b[u]);
  }
  for (; i < cnt; ++i) acc = __dadd_rn(acc, v[i]);
  return acc;
}

// One workgroup per 4096-row block: a coalesced copy into LDS, then one lane
// adds the block's values in row order.
GEEK_D void sse_block(double* v, int64_t b, const double* __restrict__ dist, int64_t n, double* __restrict__ blk) {
  const int64_t s = b * SSE_BLOCK;
  const int cnt = (int)(n - s < SSE_BLOCK ? n - s : SSE_BLOCK);
  for (int i = threadIdx.x; i < cnt; i += 256) v[i] = dist[s + i];
  __syncthreads();
  if (threadIdx.x == 0) blk[b] = chain_add(v, cnt, 0.0);
}
__global__ __launch_bounds__(256) void k_sse_blocks(const double* __restrict__ dist, int64_t n,
                                                    double* __restrict__ blk) {
  __shared__ __attribute__((aligned(16))) double v[SSE_BLOCK];
  sse_block(v, blockIdx.x, dist, n, blk);
}

__global__ __launch_bounds__(256) void k_sse_total(const double* __restrict__ blk, int64_t nb, double* __restrict__ out) {
  __shared__ __attribute__((aligned(16))) double v[SSE_BLOCK];
  double acc = 0.0;
  for (int64_t s = 0; s < nb; s += SSE_BLOCK) {
    const int cnt = (int)(nb - s < SSE_BLOCK ? nb - s : SSE_BLOCK);
    __syncthreads();
    for (int i = threadIdx.x; i < cnt; i += 256) v[i] = blk[s + i];
    __syncthreads();
    if (threadIdx.x == 0) acc = chain_add(v, cnt, acc);
  }
  if (threadIdx.x == 0) *out = acc;
}

// Radii start at zero (k_fill_f64 or k_assign_init).  The square root is
// correctly rounded and monotone, so the largest root is the root of the
// largest distance.
GEEK_D double radius_of(double dist, int take_sqrt) { return take_sqrt ? sqrt(dist) : dist; }

__global__ void k_radius(const int32_t* __restrict__ assign, const double* __restrict__ dist,
                         int64_t n, int k, int take_sqrt, double* __restrict__ rad) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= n || (unsigned)assign[i] >= (unsigned)k) return;
  const double v = radius_of(dist[i], take_sqrt);
  double* slot = rad + assign[i];
  if (v > __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    atomic_max_nonneg(slot, v);
}

// Up to CAP clusters: per-workgroup maxima in LDS (bit patterns of
// non-negative doubles order like the values), then one global atomic per
// touched slot.
constexpr int RAD_LDS = 4096, RAD_LDS_BIG = 16384;
GEEK_D void radius_lds(unsigned long long* m, int64_t b, int64_t nb, const int32_t* __restrict__ assign,
                       const double* __restrict__ dist, int64_t n, int k, int take_sqrt, double* __restrict__ rad) {
  for (int j = threadIdx.x; j < k; j += 256) m[j] = 0ull;
  __syncthreads();
  for (int64_t i = b * 256 + threadIdx.x; i < n; i += nb * 256) {
    const int a = assign[i];
    if ((unsigned)a < (unsigned)k) atomicMax(&m[a], (unsigned long long)__double_as_longlong(dist[i]));
  }
  __syncthreads();
  for (int j = threadIdx.x; j < k; j += 256)
    if (m[j]) atomic_max_nonneg(rad + j, radius_of(__longlong_as_double((long long)m[j]), take_sqrt));
}
template <int CAP>
__global__ __launch_bounds__(256) void k_radius_lds(const int32_t* __restrict__ assign,
                                                    const double* __restrict__ dist, int64_t n, int k, int take_sqrt,
                                                    double* __restrict__ rad) {
  __shared__ unsigned long long m[CAP];
  radius_lds(m, blockIdx.x, gridDim.x, assign, dist, n, k, take_sqrt, rad);
}

// Up to RAD_LDS clusters: workgroups 0 .. nblk - 1 take one block of the SSE
// each, the others the radii, which are done while the SSE's chains (37 us
// each) run; two launches one after the other before.
static_assert(RAD_LDS == SSE_BLOCK, "one array serves both");
__global__ __launch_bounds__(256) void k_sse_radius(const double* __restrict__ dist, const int32_t* __restrict__ assign,
                                                    int64_t n, int k, int nblk, double* __restrict__ blk,
                                                    double* __restrict__ rad, int take_sqrt) {
  __shared__ __attribute__((aligned(16))) double v[SSE_BLOCK];
  if ((int)blockIdx.x < nblk)
    sse_block(v, blockIdx.x, dist, n, blk);
  else
    radius_lds(reinterpret_cast<unsigned long long*>(v), (int)blockIdx.x - nblk, (int)gridDim.x - nblk, assign, dist, n,
               k, take_sqrt, rad);
}

// Both for one block of rows and at most SMALL_K clusters.
constexpr int SMALL_K = 2048;
__global__ __launch_bounds__(256) void k_sse_radius_small(const double* __restrict__ dist,
                                                          const int32_t* __restrict__ assign, int n, int k,
                                                          double* __restrict__ sse, double* __restrict__ radius,
                                                          int take_sqrt) {
  __shared__ __attribute__((aligned(16))) double v[SSE_BLOCK];
  __shared__ unsigned long long m[SMALL_K];
  for (int j = threadIdx.x; j < k; j += 256) m[j] = 0ull;
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += 256) {
    const double x = dist[i];
    const int a = assign[i];
    v[i] = x;
    if ((unsigned)a < (unsigned)k) atomicMax(&m[a], (unsigned long long)__double_as_longlong(x));
  }
  __syncthreads();
  if (threadIdx.x == 0) *sse = 0.0 + chain_add(v, n, 0.0);
  if (radius)
    for (int j = threadIdx.x; j < k; j += 256) radius[j] = radius_of(__longlong_as_double((long long)m[j]), take_sqrt);
}

// Zeroes a job's counters, row counts, maxima and radii.
__global__ void k_assign_init(uint32_t* counts, unsigned long long* ctr, float* cmax, double* radius, int k) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < 4) {
    counts[i] = 0u;
    ctr[i] = 0ull;
    cmax[i] = 0.f;
  }
  if (radius && i < k) radius[i] = 0.0;
}

__global__ void k_pad_modes(const uint32_t* __restrict__ mode, int k, int n_cat, int k_pad,
                            uint32_t* __restrict__ out) {
  const int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (g >= (int64_t)k_pad * MAX_CAT) return;
  const int j = (int)(g / MAX_CAT), a = (int)(g % MAX_CAT);
  out[g] = (j < k && a < n_cat) ? mode[(int64_t)j * n_cat + a] : 0u;
}

__global__ void k_fill_f64(double* p, int64_t n, double v) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}
// ---------------------------------------------------------------- host side
// SSE over 4096-row blocks and the per-cluster radius (sqrt of the largest
// member distance when `take_sqrt`), shared by every metric.  `zeroed`: the
// radii are already zero.
void sse_and_radius(const double* dist, const int32_t* assign, int64_t n, int k, double* sse, double* radius,
                    int take_sqrt, double* sse_blk, bool zeroed, hipStream_t s) {
  if (n <= SSE_BLOCK && k <= SMALL_K) {  // one launch instead of three or four
    hipLaunchKernelGGL(k_sse_radius_small, dim3(1), dim3(256), 0, s, dist, assign, (int)n, k, sse, radius, take_sqrt);
    return;
  }
  const int64_t nblk = (n + SSE_BLOCK - 1) / SSE_BLOCK;
  if (radius && !zeroed) hipLaunchKernelGGL(k_fill_f64, dim3(ceil_div(k, 256)), dim3(256), 0, s, radius, k, 0.0);
  const bool both = radius && k <= RAD_LDS;
  if (both)
    hipLaunchKernelGGL(k_sse_radius, dim3((int)nblk + (int)std::min<int64_t>(ceil_div(n, 4096), 512)), dim3(256), 0, s,
                       dist, assign, n, k, (int)nblk, sse_blk, radius, take_sqrt);
  else
    hipLaunchKernelGGL(k_sse_blocks, dim3(nblk), dim3(256), 0, s, dist, n, sse_blk);
  hipLaunchKernelGGL(k_sse_total, dim3(1), dim3(256), 0, s, sse_blk, nblk, sse);
  if (radius && !both) {
    if (k <= RAD_LDS_BIG)  // 128 KB of LDS: one workgroup per CU, fewer of them
      hipLaunchKernelGGL(k_radius_lds<RAD_LDS_BIG>, dim3((int)std::min<int64_t>(ceil_div(n, 16384), 128)), dim3(256),
                         0, s, assign, dist, n, k, take_sqrt, radius);
    else
      hipLaunchKernelGGL(k_radius, dim3(ceil_div(n, 256)), dim3(256), 0, s, assign, dist, n, k, take_sqrt, radius);
  }
}

size_t sse_blk_words(int64_t n) { return (size_t)((n + SSE_BLOCK - 1) / SSE_BLOCK + 1); }

static int pick_dp(int d) { return d <= 32 ? 32 : d <= 64 ? 64 : d <= 128 ? 128 : d <= 256 ? 256 : 0; }

size_t modes_ws(int64_t n_members, int F, int k);
int32_t modes_compute(const uint32_t* V, int64_t ldv, int F, int64_t n, const uint32_t* so, const uint32_t* sm,
                      int k, int64_t NC, uint32_t* modes, void* ws, int32_t* st, hipStream_t s);

struct AssignWs {
  __bf16* cl;  // the centroids' pieces (ModeF32), the first also the bf16 first pass's copy
  float* nc;
  uint8_t* cl8;  // e4m3 copy for an FP8 first pass
  float* cmax;   // [0] max |c|, [1] max |x_t|, [2] max |c_t|, [3] scale (FP8)
  int32_t* rec;
  uint32_t* esc;
  uint32_t* fb;
  uint32_t* counts;  // rows after each pass: [0] of esc, [1] of fb, [2] of esc again (FP8)
  double* part_d;    // per-split minima of the float64 full scans
  int32_t* part_j;
  unsigned long long* ctr;
  double* dist;
  double* sse_blk;
  void* modes_ws;
  size_t modes_bytes;
  uint32_t* mode16;
  float* xt;  // dimension-major member values (centroids_transposed)
  // blocked rescan
  float *thr, *ncp;
  double* mean;
  uint32_t *skey, *sid, *skey2, *sid2, *spos;  // seeds by code
  uint32_t *rkey, *rid, *rkey2, *rid2;         // unsettled rows by their best seed's place
  __bf16* clp;  // the pieces in seed order
  uint32_t *gate, *flags, *rtmp;
  int fwords;
};



static bool blocked_rescan(const geek_assign_job& J) {
  return J.precision == GEEK_PREC_BF16 && J.metric == GEEK_METRIC_EUCLID && J.k >= BLOCKED_K && J.k < (1 << 26) &&
         blocked_pays(J.n, J.k, pick_dp(J.d));
}

static size_t carve_assign(const geek_assign_job& J, void* ws, AssignWs* out) {
  Carver c(ws);
  const int DP = pick_dp(J.d);
  const int64_t k_pad = ((int64_t)J.k + SCAN_BC - 1) / SCAN_BC * SCAN_BC;
  out->cl = c.take<__bf16>(ModeF32::PIECES * k_pad * DP);
  out->cl8 = c.take<uint8_t>(J.precision == GEEK_PREC_FP8 ? k_pad * DP : 16);
  out->nc = c.take<float>(k_pad);
  out->cmax = c.take<float>(4);
  out->rec = c.take<int32_t>(J.n * RECW);
  out->esc = c.take<uint32_t>(J.n);
  out->fb = c.take<uint32_t>(J.n);
  out->counts = c.take<uint32_t>(4);
  out->part_d = c.take<double>(fb_part_cap(J.n));
  out->part_j = c.take<int32_t>(fb_part_cap(J.n));
  out->ctr = c.take<unsigned long long>(4);
  out->dist = c.take<double>(J.dist ? 1 : J.n);
  out->sse_blk = c.take<double>((J.n + SSE_BLOCK - 1) / SSE_BLOCK + 1);
  out->modes_bytes = J.metric == GEEK_METRIC_HETERO ? modes_ws(J.n_members, J.n_cat, J.k) : 0;
  out->modes_ws = c.take<char>(out->modes_bytes + 16);
  out->mode16 = c.take<uint32_t>(J.metric == GEEK_METRIC_HETERO ? k_pad * MAX_CAT : 4);
  if (blocked_rescan(J)) {
    const int64_t n = J.n, k = J.k;
    out->fwords = (int)((k_pad / 64 + 31) / 32);
    out->thr = c.take<float>(n);
    out->ncp = c.take<float>(k_pad);
    out->mean = c.take<double>(DP);
    out->gate = c.take<uint32_t>(2);
    out->skey = c.take<uint32_t>(k);
    out->sid = c.take<uint32_t>(k);
    out->skey2 = c.take<uint32_t>(k);
    out->sid2 = c.take<uint32_t>(k);
    out->spos = c.take<uint32_t>(k);
    out->rkey = c.take<uint32_t>(n);
    out->rid = c.take<uint32_t>(n);
    out->rkey2 = c.take<uint32_t>(n);
    out->rid2 = c.take<uint32_t>(n);
    out->clp = c.take<__bf16>(ModeF32::PIECES * k_pad * DP);
    out->flags = c.take<uint32_t>((size_t)(ceil_div(n, 256) * 2) * out->fwords);
    out->rtmp = c.take<uint32_t>(radix_tmp_words(std::max(n, k)));
  }
  out->xt = c.take<float>(centroids_transposed(J) ? (size_t)members_pad(J) * J.d : 4);
  return c.used + 256;
}

size_t assign_euclid_ws(const geek_assign_job& J) {
  AssignWs W;
  return carve_assign(J, nullptr, &W);
}

// Column blocks per wave and LDS buffering per mode: the low-precision modes
// reuse every LDS fragment for two column blocks; float32's three pieces of two
// blocks would leave one wavefront per SIMD (500,009 x 100 rows, 3,001 seeds:
// whole call 2.20 ms with one block and two stages; 4.12 ms with float32 matrix
// instructions).
// The BF16 and FP8 passes keep the best two values per row (T2); the float32
// pass, which also rescans rows with several candidates, keeps the full
// candidate window.  (An FP8 pass with windows, whose rows e4m3's rounding
// leaves with a few candidates or many more, and float32 rescans of those: 2 10^6
// heterogeneous rows, k = 1,000, hash and buckets included, 23.9 ms, of them
// the pass 8.3 and the rescan 7.6; see assign_finish.)
// Heterogeneous rows carry their categorical values in registers: one
// column block.
template <class M, bool HET> struct ScanShape {
  static constexpr int NCB = HET ? 1 : 2, NBUF = 2;
  static constexpr bool T2 = true;
};
template <bool HET> struct ScanShape<ModeF32, HET> {
  static constexpr int NCB = 1, NBUF = 2;
  static constexpr bool T2 = false;
};

template <class M>
int scan_rows_per_tile(bool het_on) {
  return 128 * (het_on ? ScanShape<M, true>::NCB : ScanShape<M, false>::NCB);
}

template <class M, bool HET, bool WIDE, bool MARK>
static void launch_scan(int DP, int grid, hipStream_t s, const geek_assign_job& J, int64_t n_rows,
                        const uint32_t* rows, const uint32_t* rows_count, const void* cl, const AssignWs& W,
                        int k_pad, const Het& het, int32_t* st, const ScanBlocks& sb) {
  using CE = typename M::ce;
  constexpr int NCB = ScanShape<M, HET>::NCB;
  constexpr bool T2 = ScanShape<M, HET>::T2;
  // (two stages of 256 attributes in three pieces and wide windows exceed the LDS)
  constexpr int NBUF = ScanShape<M, HET>::NBUF, NBUF256 = M::PIECES > 1 && WIDE ? 1 : NBUF;
  switch (DP) {
#define GEEK_SCAN_CASE(DPV)                                                                            \
  case DPV:                                                                                            \
    hipLaunchKernelGGL((k_scan<M, DPV, HET, NCB, DPV == 256 ? NBUF256 : NBUF, T2, WIDE, MARK>), dim3(grid), dim3(SCAN_THREADS), 0, s, J.X,\
                       J.ldx, J.d, n_rows, rows, rows_count, static_cast<const CE*>(cl), W.nc, k_pad, \
                       W.cmax, W.cmax + 3, het, J.k, W.rec, st, sb);                                     \
    break;
    GEEK_SCAN_CASE(32)
    GEEK_SCAN_CASE(64)
    GEEK_SCAN_CASE(128)
    GEEK_SCAN_CASE(256)
#undef GEEK_SCAN_CASE
  }
}

template <class M, bool WIDE = false, bool MARK = false>
static void scan_any(bool het_on, int DP, int grid, hipStream_t s, const geek_assign_job& J, int64_t n_rows,
                     const uint32_t* rows, const uint32_t* rows_count, const void* cl, const AssignWs& W,
                     int k_pad, const Het& het, int32_t* st, const ScanBlocks& sb = {}) {
  if constexpr (!MARK) {
    if (het_on) {
      launch_scan<M, true, WIDE, false>(DP, grid, s, J, n_rows, rows, rows_count, cl, W, k_pad, het, st, sb);
      return;
    }
  }
  launch_scan<M, false, WIDE, MARK>(DP, grid, s, J, n_rows, rows, rows_count, cl, W, k_pad, het, st, sb);
}

// Per-job state between the three phases of an assignment.
struct AssignCtx {
  AssignWs W;
  int DP = 0;
  int k_pad = 0;
  double* dist = nullptr;
  bool het_on = false;
  bool marked = false;  // the first pass left what a blocked rescan needs (batched ones do not)
  Het het{nullptr, nullptr, nullptr, 0, 0.f, 0.0};
};

// Centroids (and modes), matrix-core copies, |c|^2, bounds and scale.
static int32_t assign_prep(const geek_assign_job& J, void* ws, AssignCtx& C, int32_t* st, hipStream_t s) {
  carve_assign(J, ws, &C.W);
  AssignWs& W = C.W;
  C.DP = pick_dp(J.d);
  C.k_pad = (J.k + SCAN_BC - 1) / SCAN_BC * SCAN_BC;
  C.dist = J.dist ? J.dist : W.dist;
  C.het_on = J.metric == GEEK_METRIC_HETERO;
  if (C.het_on) C.het = Het{J.cat, J.modes, W.mode16, J.n_cat, (float)J.gamma, J.gamma};
  const int DP = C.DP, k_pad = C.k_pad;
  if (J.counters) W.ctr = J.counters;  // counted in place
  hipLaunchKernelGGL(k_assign_init, dim3(J.radius ? ceil_div(J.k, 256) : 1), dim3(256), 0, s, W.counts, W.ctr, W.cmax,
                     J.radius, J.k);
  if (centroids_transposed(J)) {
    const int64_t nmp = members_pad(J);
    hipLaunchKernelGGL(k_gather_t, dim3(ceil_div(nmp, GT_TILE), ceil_div(J.d, GT_TILE)), dim3(256), 0, s, J.X,
                       J.ldx, J.n, J.d, J.seed_offsets, J.k, J.seed_members, J.n_members, nmp, W.xt, st);
    hipLaunchKernelGGL(k_centroids_t, dim3(ceil_div((int64_t)J.k * J.d, 256)), dim3(256), 0, s, W.xt,
                       J.n_members, J.d, J.seed_offsets, J.k, J.centroids, st);
  } else {
    hipLaunchKernelGGL(k_centroids, dim3(ceil_div((int64_t)J.k * J.d, 256)), dim3(256), 0, s, J.X,
                       J.ldx, J.n, J.d, J.seed_offsets, J.seed_members, J.k, J.k_dev, J.centroids, st);
  }
  if (C.het_on) {
    if (int32_t rc = modes_compute(reinterpret_cast<const uint32_t*>(J.cat), J.n_cat, J.n_cat, J.n,
                                   J.seed_offsets, J.seed_members, J.k, J.n_members, J.modes, W.modes_ws, st, s))
      return rc;
    hipLaunchKernelGGL(k_pad_modes, dim3(ceil_div((int64_t)k_pad * MAX_CAT, 256)), dim3(256), 0, s, J.modes, J.k,
                       J.n_cat, k_pad, W.mode16);
  }
  const bool fp8 = J.precision == GEEK_PREC_FP8;
  if (fp8) {
    hipLaunchKernelGGL(k_absmax<float>, dim3(1024), dim3(256), 0, s, J.X, J.ldx, J.n, J.d, W.cmax + 1);
    hipLaunchKernelGGL(k_absmax<double>, dim3(256), dim3(256), 0, s, J.centroids, (int64_t)J.d, (int64_t)J.k, J.d,
                       W.cmax + 2);
    hipLaunchKernelGGL(k_fp8_scale, dim3(1), dim3(1), 0, s, W.cmax + 1, W.cmax + 2, W.cmax + 3);
  }
  hipLaunchKernelGGL(k_cprep, dim3(ceil_div((int64_t)k_pad * (DP / 8), 256)), dim3(256), 0, s, J.centroids, J.k, J.d,
                     k_pad, DP, W.cl, fp8 ? W.cl8 : nullptr, W.cmax + 3, W.nc, W.cmax, J.k_dev);
  GEEK_LAUNCH_CHECK();
  return GEEK_OK;
}

// Workgroups of a persistent pass over a device-counted subset of n rows.
static int esc_grid(int64_t n, int rows_per_group) {
  return (int)std::max<int64_t>(1, std::min<int64_t>(1024, ceil_div(n, rows_per_group)));
}

// The first pass of one job: every row gets a candidate record.
static void assign_first_pass(const geek_assign_job& J, AssignCtx& C, int32_t* st, hipStream_t s) {
  if (J.precision == GEEK_PREC_BF16) {
    const int grid_all = ceil_div(J.n, scan_rows_per_tile<ModeBF16>(C.het_on));
    C.marked = blocked_rescan(J);
    if (C.marked)
      scan_any<ModeBF16, false, true>(false, C.DP, grid_all, s, J, J.n, nullptr, nullptr, C.W.cl, C.W, C.k_pad, C.het,
                                      st, ScanBlocks{nullptr, 0, nullptr, C.W.thr, nullptr, nullptr, nullptr, nullptr});
    else
      scan_any<ModeBF16>(C.het_on, C.DP, grid_all, s, J, J.n, nullptr, nullptr, C.W.cl, C.W, C.k_pad, C.het, st);
  } else if (J.precision == GEEK_PREC_FP8) {
    const int grid_all = ceil_div(J.n, scan_rows_per_tile<ModeFP8>(C.het_on));
    scan_any<ModeFP8>(C.het_on, C.DP, grid_all, s, J, J.n, nullptr, nullptr, C.W.cl8, C.W, C.k_pad, C.het, st);
  } else {
    const int grid_all = ceil_div(J.n, scan_rows_per_tile<ModeF32>(C.het_on));
    scan_any<ModeF32>(C.het_on, C.DP, grid_all, s, J, J.n, nullptr, nullptr, C.W.cl, C.W, C.k_pad, C.het, st);
  }
}

// Orders seeds and unsettled rows and marks the groups of seeds each 128 rows
// need.
static ScanBlocks blocked_marks(const geek_assign_job& J, const AssignCtx& C, hipStream_t s) {
  const AssignWs& W = C.W;
  const int k = J.k, k_pad = C.k_pad;
  hipLaunchKernelGGL(k_blocked_gate, dim3(1), dim3(64), 0, s, W.counts + 0, k, C.DP, W.gate);
  hipLaunchKernelGGL(k_seed_mean, dim3(J.d), dim3(256), 0, s, J.centroids, W.gate, k, J.d, W.mean);
  hipLaunchKernelGGL(k_seed_code, dim3(ceil_div(k, 4)), dim3(256), 0, s, J.centroids, W.gate, J.d, W.mean, W.skey, W.sid);
  const int zero[4] = {0, 0, 0, 0}, shifts[4] = {0, 8, 16, 24};
  RsView A{{W.skey, nullptr, nullptr, nullptr}, W.sid}, B{{W.skey2, nullptr, nullptr, nullptr}, W.sid2};
  const uint32_t* sid = radix_sort_dn(A, B, 1, k, W.gate, zero, shifts, CODE_BITS / 8, W.rtmp, s) ? W.sid2 : W.sid;
  hipLaunchKernelGGL(k_seed_permute, dim3(ceil_div((int64_t)k_pad * (C.DP / 8), 256)), dim3(256), 0, s, sid, W.gate, k, k_pad,
                     C.DP, W.cl, W.nc, W.clp, W.ncp, W.spos);
  hipLaunchKernelGGL(k_row_keys, dim3(1024), dim3(256), 0, s, W.esc, W.gate + 1, W.rec, W.spos, W.rkey, W.rid,
                     W.flags, W.fwords);
  int np = 1;
  while (np < 4 && (uint32_t)((k - 1) / SCAN_BC) >> (8 * np)) ++np;
  RsView R{{W.rkey, nullptr, nullptr, nullptr}, W.rid}, R2{{W.rkey2, nullptr, nullptr, nullptr}, W.rid2};
  const uint32_t* rows =
      radix_sort_dn(R, R2, 1, J.n, W.gate + 1, zero, shifts, np, W.rtmp, s) ? W.rid2 : W.rid;
  const int64_t tiles = ceil_div(J.n, 256);
  switch (C.DP) {
#define GEEK_MARK_CASE(DPV)                                                                                          \
  case DPV:                                                                                                          \
    hipLaunchKernelGGL(k_mark<DPV>, dim3(tiles), dim3(SCAN_THREADS), 0, s, J.X, J.ldx, J.d, rows, W.gate + 1, W.thr,   \
                       W.clp, W.ncp, k_pad, W.fwords, W.flags);                                                      \
    break;
    GEEK_MARK_CASE(32)
    GEEK_MARK_CASE(64)
    GEEK_MARK_CASE(128)
    GEEK_MARK_CASE(256)
#undef GEEK_MARK_CASE
  }
  return ScanBlocks{W.flags, W.fwords, sid, nullptr, W.gate, rows, W.clp, W.ncp};
}

// Float64 checks, rescans and fallbacks, SSE, radius, counters.
static void assign_finish(const geek_assign_job& J, AssignCtx& C, int32_t* st, hipStream_t s,
                          const unsigned long long* t0) {
  AssignWs& W = C.W;
  unsigned long long* ctr = W.ctr;
  const int fz_grid = (int)std::min<int64_t>(
      8192, std::max<int64_t>(ceil_div(J.n, 1024), std::min<int64_t>(ceil_div(J.n, 8 * FZ_ROWS), 2048)));
  const int rstride = J.precision == GEEK_PREC_FP32 ? RECW : RECW_T2;
  // Eight lanes per row for the BF16 records of many wide rows, whose lines do
  // not stay in the caches between a lane's steps (whole assignment, k = 500,
  // eight lanes against one: 10^6 x 256 1.20 / 1.26 ms, 1.5 10^6 x 128 0.82 /
  // 0.84, 5 10^5 x 128 0.33 / 0.33; but 2 10^5 x 128 0.213 / 0.206, 1.5 10^6 x
  // 64 0.48 / 0.47, x 20 0.28 / 0.23).
  if (rstride == RECW_T2 && J.d > 64 && J.n * J.d >= ((int64_t)1 << 26))
    hipLaunchKernelGGL(k_finalize, dim3(fz_grid), dim3(256), 0, s, J.X, J.ldx, J.d, J.centroids, J.k, C.het, J.n,
                       nullptr, nullptr, W.rec, rstride, J.assign, C.dist, W.esc, W.counts + 0, ctr, 0);
  else
    hipLaunchKernelGGL(k_finalize_win, dim3((int)std::min<int64_t>(ceil_div(J.n, 256), 1024)), dim3(256), 0, s, J.X, J.ldx, J.d, J.centroids, J.k,
                       C.het, J.n, nullptr, nullptr, W.rec, rstride, J.assign, C.dist, W.esc, W.counts + 0, ctr, 0, ScanBlocks{});
  // rows with several first-pass candidates (persistent grids, at most one row
  // tile / block per group)
  const uint32_t* esc = W.esc;
  uint32_t *esc_n = W.counts + 0, *left = W.fb, *left_n = W.counts + 1;
  if (J.precision == GEEK_PREC_FP8) {
    // e4m3's window (2^-3) leaves most rows of close clusters; bf16 settles
    // nearly all of those at a third of the float32 rescan's cost
    scan_any<ModeBF16>(C.het_on, C.DP, esc_grid(J.n, scan_rows_per_tile<ModeBF16>(C.het_on)), s, J, 0, esc, esc_n, W.cl,
                       W, C.k_pad, C.het, st);
    hipLaunchKernelGGL(k_finalize_win, dim3(esc_grid(J.n, 256)), dim3(256), 0, s, J.X, J.ldx, J.d, J.centroids, J.k,
                       C.het, (int64_t)0, esc, esc_n, W.rec, RECW_T2, J.assign, C.dist, left, left_n, ctr, 1,
                       ScanBlocks{});
    esc = W.fb, esc_n = W.counts + 1;
    left = W.esc, left_n = W.counts + 2;
  }
  // float32 rescan with a wider window
  ScanBlocks sb{};
  const bool blocked = C.marked;
  if (blocked) sb = blocked_marks(J, C, s);
  scan_any<ModeF32, true>(C.het_on, C.DP, esc_grid(J.n, 128), s, J, 0, esc, esc_n, W.cl, W, C.k_pad, C.het, st, sb);
  hipLaunchKernelGGL(k_finalize_win, dim3(esc_grid(J.n, 256)), dim3(256), 0, s, J.X, J.ldx, J.d, J.centroids,
                     J.k, C.het, (int64_t)0, esc, esc_n, W.rec, RECW, J.assign, C.dist, left, left_n,
                     ctr, 1, sb);
  const uint32_t* fpos = nullptr;
  if (blocked) {
    // the float64 scan visits marked groups too: its rows in the marked order
    // (k_finalize_win listed the same rows in any order)
    uint32_t *flag = W.rkey, *at = W.rkey2, *pos = sb.rows == W.rid ? W.rid2 : W.rid;
    hipLaunchKernelGGL(k_left_flags, dim3(1024), dim3(256), 0, s, W.gate + 1, W.rec, flag);
    exscan_u32_dn(flag, at, J.n, W.gate + 1, W.rtmp, nullptr, s);
    hipLaunchKernelGGL(k_left_list, dim3(1024), dim3(256), 0, s, W.gate + 1, sb.rows, flag, at, left, pos);
    fpos = pos;
  }
  const int fb_grid = (int)std::min<int64_t>(FB_GRID, ceil_div(J.n, FB_R) * FB_SPLIT);
  switch (C.DP) {
#define GEEK_FB_CASE(DPV)                                                                                  \
  case DPV:                                                                                                \
    hipLaunchKernelGGL(k_fallback64<DPV>, dim3(fb_grid), dim3(256), 0, s, J.X, J.ldx, J.d, J.centroids, J.k, \
                       J.k_dev, C.het, left, left_n, J.assign, C.dist, W.part_d, W.part_j, ctr, fpos, sb);\
    break;
    GEEK_FB_CASE(32)
    GEEK_FB_CASE(64)
    GEEK_FB_CASE(128)
    GEEK_FB_CASE(256)
#undef GEEK_FB_CASE
  }
  hipLaunchKernelGGL(k_fb_merge, dim3(esc_grid(J.n, 256)), dim3(256), 0, s, left, left_n, J.k, W.part_d,
                     W.part_j, J.assign, C.dist, ctr);
  sse_and_radius(C.dist, J.assign, J.n, J.k, J.sse, J.radius, C.het_on ? 0 : 1, W.sse_blk, true, s);
  if (J.t_done) {
    if (t0) hipLaunchKernelGGL(k_clock_since, dim3(1), dim3(64), 0, s, t0, J.t_done);
    else hipLaunchKernelGGL(k_clock_now, dim3(1), dim3(64), 0, s, J.t_done);
  }
}

int32_t assign_euclid(const geek_assign_job& J, void* ws, size_t ws_bytes, int32_t* st,
                      hipStream_t s) {
  AssignCtx C;
  if (ws_bytes < carve_assign(J, ws, &C.W)) return GEEK_ERR_WORKSPACE;
  prof_begin(GEEK_PROF_ASSIGN, s);
  if (int32_t rc = assign_prep(J, ws, C, st, s)) return rc;
  prof_begin(GEEK_PROF_ASSIGN_SCAN, s);
  assign_first_pass(J, C, st, s);
  prof_end(GEEK_PROF_ASSIGN_SCAN, s);
  assign_finish(J, C, st, s, nullptr);
  prof_end(GEEK_PROF_ASSIGN, s);
  GEEK_LAUNCH_CHECK();
  return GEEK_OK;
}

// ---------------------------------------------------------------- batches
// Jobs of one call that can share persistent first-pass launches: Euclidean,
// all in the same precision.  Each job gets its own workspace slice.
bool assign_batchable(const geek_assign_job* jobs, int njobs) {
  if (njobs < 2) return false;
  for (int j = 0; j < njobs; ++j)
    if (jobs[j].metric != GEEK_METRIC_EUCLID || jobs[j].precision != jobs[0].precision || jobs[j].k_dev)
      return false;
  return true;
}

static size_t slice_bytes(const geek_assign_job& J) {
  AssignWs W;
  return (carve_assign(J, nullptr, &W) + 255) / 256 * 256;
}

size_t assign_batch_ws(const geek_assign_job* jobs, int njobs) {
  size_t b = 0;
  for (int j = 0; j < njobs; ++j) b += slice_bytes(jobs[j]);
  return b + (size_t)njobs * sizeof(ScanJob) + 512;
}

int32_t assign_euclid_batch(const geek_assign_job* jobs, int njobs, void* ws, size_t ws_bytes, int32_t* st,
                            hipStream_t s) {
  if (ws_bytes < assign_batch_ws(jobs, njobs)) return GEEK_ERR_WORKSPACE;
  std::vector<AssignCtx> C(njobs);
  std::vector<char*> slice(njobs);
  char* base = static_cast<char*>(ws);
  size_t off = 0;
  for (int j = 0; j < njobs; ++j) {
    slice[j] = base + off;
    off += slice_bytes(jobs[j]);
  }
  ScanJob* table = reinterpret_cast<ScanJob*>(base + (off + 255) / 256 * 256);
  unsigned long long* t0 = reinterpret_cast<unsigned long long*>(table + njobs);
  const geek_assign_job& J0 = jobs[0];
  prof_begin(GEEK_PROF_ASSIGN, s);
  hipLaunchKernelGGL(k_clock_now, dim3(1), dim3(64), 0, s, t0);
  {  // jobs prepared concurrently on the fan-out lanes (independent slices)
    Fan fan(s, njobs);
    for (int j = 0; j < njobs; ++j)
      if (int32_t rc = assign_prep(jobs[j], slice[j], C[j], st, fan.lane(j))) return rc;
  }
  // one persistent launch per padded depth, jobs in call order, with the
  // tile shape set for that (precision, depth)
  prof_begin(GEEK_PROF_ASSIGN_SCAN, s);
  int tslot = 0;
  for (const int DP : {32, 64, 128, 256}) {
    const int rows_per_tile = 128 * scan_tiles_get(J0.precision, DP).ncb;
    std::vector<ScanJob> tab;
    int64_t total = 0;
    for (int j = 0; j < njobs; ++j) {
      if (C[j].DP != DP) continue;
      const geek_assign_job& J = jobs[j];
      const AssignWs& W = C[j].W;
      ScanJob e{};
      e.X = J.X;
      e.ldx = J.ldx;
      e.n = J.n;
      e.cl = J0.precision == GEEK_PREC_FP8 ? static_cast<const void*>(W.cl8) : W.cl;
      e.nc = W.nc;
      e.cmax = W.cmax;
      e.scale = W.cmax + 3;
      e.rec = W.rec;
      e.tile_begin = total;
      e.d = J.d;
      e.k = J.k;
      e.k_pad = C[j].k_pad;
      tab.push_back(e);
      total += ceil_div(J.n, rows_per_tile);
    }
    if (tab.empty()) continue;
    ScanJob* dst = table + tslot;
    for (size_t c0 = 0; c0 < tab.size(); c0 += SCANJOB_CHUNK) {
      ScanJobChunk ch{};
      ch.count = (int)std::min<size_t>(SCANJOB_CHUNK, tab.size() - c0);
      for (int i = 0; i < ch.count; ++i) ch.jobs[i] = tab[c0 + i];
      hipLaunchKernelGGL(k_put_jobs, dim3(1), dim3(SCANJOB_CHUNK), 0, s, ch, dst + c0);
    }
    launch_scan_batch(J0.precision, DP, dst, (int)tab.size(), total, st, s);
    tslot += (int)tab.size();
  }
  prof_end(GEEK_PROF_ASSIGN_SCAN, s);
  {
    Fan fan(s, njobs);
    for (int j = 0; j < njobs; ++j) assign_finish(jobs[j], C[j], st, fan.lane(j), t0);
  }
  prof_end(GEEK_PROF_ASSIGN, s);
  GEEK_LAUNCH_CHECK();
  return GEEK_OK;
}

}  // namespace geek

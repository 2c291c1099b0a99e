// Assignment of MinHash signatures to the modes of the seeds (paper Section
// 3.3: the central vector of sets is the mode; Section 2.1: Dist = 1 - Sim)
// on gfx950.
//
//   modes       a thread per (seed j, position f) counts the members' values
//               against each other in LDS; seeds of more than MODE_SMALL
//               members: items (seed, position, value) sorted by (j*F + f,
//               value), each (j, f) a known segment of the sorted array,
//               scanned by one thread for its longest run.  Smallest value on
//               ties.
//   index       an exact inverted index: (f, mode value) -> ascending list of
//               seeds j, as a hash table of run extents over the sorted
//               (f, value, j) triples.
//   bit planes  (k * F <= SIG_DENSE_MAX, k <= SIG_BITS_K) per (f, mode value) a
//               bit mask of its seeds; a row adds the masks of its F values
//               into bit-sliced counters of all seeds (k_sig_bits).
//   assign      otherwise one wavefront per row probes its F (f, sig[f]) pairs, gathers
//               the matching seeds in LDS, sorts them and takes the longest
//               run (lowest j on ties); a row whose matches overflow the LDS
//               list is compared against every mode instead.  Rows with no
//               match at all take seed 0 (every count is 0).
#include <algorithm>

#include "common.hpp"
#include "radix.hpp"

namespace geek {

void sse_and_radius(const double* dist, const int32_t* assign, int64_t n, int k, double* sse, double* radius,
                    int take_sqrt, double* sse_blk, bool zeroed, hipStream_t s);
size_t sse_blk_words(int64_t n);

constexpr int SG_CAP = 2048;  // matched seeds held in LDS per row
// k * F up to which every row is compared against every mode directly
constexpr int64_t SIG_DENSE_MAX = 1 << 20;
// ... by bit planes up to this k (masks of k * F rows of k bits)
constexpr int SIG_BITS_K = 4096;

// Members of seed j, or 0 and a status: none, or some past the job's member
// count NC, which the member ids and the sort's buffers are sized by.
GEEK_D uint32_t mode_members(const uint32_t* __restrict__ so, int64_t j, int64_t NC, int32_t* st) {
  const uint32_t s0 = so[j], s1 = so[j + 1];
  if (s1 > s0 && (int64_t)s1 <= NC) return s1 - s0;
  set_status(st, s1 > s0 ? GEEK_ERR_ARG : GEEK_ERR_EMPTY_SET);
  return 0u;
}

// Seeds of at most MODE_SMALL members: thread f of a workgroup copies its
// position's values of the seed's members (a row's positions are contiguous)
// into a column of LDS and compares them with each other.  64,000 members in
// 2,000 seeds, F = 256: 0.1 ms where sorting the 1.6 10^7 items took 2.0 ms.
// MODE_SMALL: the columns set the LDS and with it how many workgroups run.  Whole
// calls of 20,000 rows, ms, sorted / columns of 48 / of 96: F = 256, 2,000 seeds of
// 16 1.17 / 0.55 / 0.60, of 32 2.20 / 0.65 / 0.78, of 48 3.19 / 0.80 / 1.08, of 64
// 4.22 / - / 1.47; ten categorical attributes, 2,000 seeds of 32 0.54 / 0.46 /
// 0.59, of 48 0.551 / 0.548 / 0.82, of 64 0.59 / - / 1.16: at 48 the counting no
// longer gains where few positions share a workgroup, and columns for more cost
// the smaller seeds.
constexpr int MODE_SMALL = 48, MODE_THREADS = 256;
__global__ __launch_bounds__(MODE_THREADS) void k_mode_small(const uint32_t* __restrict__ V, int64_t ldv, int F,
                                                             int64_t n, const uint32_t* __restrict__ so,
                                                             const uint32_t* __restrict__ sm, int k, int64_t NC,
                                                             uint32_t* __restrict__ modes, int32_t* st) {
  __shared__ uint32_t v[MODE_SMALL][MODE_THREADS];  // a thread reads its own column only
  const int f = blockIdx.y * MODE_THREADS + threadIdx.x;
  for (int64_t j = blockIdx.x; j < k; j += gridDim.x) {
    const uint32_t s0 = so[j], sj = mode_members(so, j, NC, st);
    if (sj > (uint32_t)MODE_SMALL || f >= F) continue;
    if (sj == 0u) {
      modes[j * F + f] = 0u;
      continue;
    }
    for (uint32_t q0 = 0; q0 < sj; q0 += 8) {  // eight members' loads in flight
      uint32_t x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const uint32_t id = sm[s0 + (q0 + u < sj ? q0 + u : sj - 1u)];
        if ((int64_t)id >= n) {
          set_status(st, GEEK_ERR_ARG);
          x[u] = 0u;
        } else {
          x[u] = V[(int64_t)id * ldv + f];
        }
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (q0 + u < sj) v[q0 + u][threadIdx.x] = x[u];
    }
    uint32_t best = 0u, most = 0u;
    for (uint32_t q = 0; q < sj; ++q) {
      const uint32_t x = v[q][threadIdx.x];
      uint32_t c = 0u;
      for (uint32_t r = q; r < sj; ++r) c += v[r][threadIdx.x] == x ? 1u : 0u;  // full count at the first occurrence
      if (c > most || (c == most && x < best)) {
        most = c;
        best = x;
      }
    }
    modes[j * F + f] = best;
  }
}

// Members of the seeds the sort takes (0 for the others), and the items of
// positions f0 .. f0 + F - 1: (position's segment, value) at boff[j] F + f s_j + q.
__global__ void k_mode_sizes(const uint32_t* __restrict__ so, int k, int64_t NC, uint32_t* __restrict__ size) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= k) return;
  const uint32_t sj = mode_members(so, j, NC, nullptr);
  size[j] = sj > (uint32_t)MODE_SMALL ? sj : 0u;
}
__global__ void k_mode_total(const uint32_t* __restrict__ members, int F, int64_t NC, uint32_t* __restrict__ items) {
  if (threadIdx.x == 0) *items = (int64_t)*members <= NC ? *members * (uint32_t)F : 0u;
}
__global__ void k_mode_items(const uint32_t* __restrict__ V, int64_t ldv, int f0, int F, int64_t n,
                             const uint32_t* __restrict__ so, const uint32_t* __restrict__ sm, int k,
                             const uint32_t* __restrict__ boff, const uint32_t* __restrict__ items,
                             uint32_t* __restrict__ val, uint32_t* __restrict__ seg, int32_t* st) {
  const int64_t total = *items, stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; g < total; g += stride) {
    const uint32_t mpos = (uint32_t)(g / F);
    const int f = (int)(g % F);
    // the last seed that starts at or before mpos (seeds of no items share a
    // start with their successor)
    int lo = 0, hi = k;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (boff[mid] <= mpos) lo = mid; else hi = mid;
    }
    const int j = lo;
    const uint32_t sj = so[j + 1] - so[j], q = mpos - boff[j], id = sm[so[j] + q];
    const int64_t at = (int64_t)boff[j] * F + (int64_t)f * sj + q;
    const bool ok = (int64_t)id < n;
    if (!ok) set_status(st, GEEK_ERR_ARG);
    val[at] = ok ? V[(int64_t)id * ldv + f0 + f] : 0u;
    seg[at] = (uint32_t)j * (uint32_t)F + (uint32_t)f;
  }
}

__global__ void k_mode_pick(const uint32_t* __restrict__ val, const uint32_t* __restrict__ so,
                            const uint32_t* __restrict__ boff, int k, int f0, int F, int ldm, int64_t NC,
                            uint32_t* __restrict__ modes) {
  const int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (g >= (int64_t)k * F) return;
  const int j = (int)(g / F), f = (int)(g % F);
  const uint32_t sj = mode_members(so, j, NC, nullptr);
  if (sj <= (uint32_t)MODE_SMALL || (int64_t)boff[j] + sj > NC) return;
  const uint32_t* p = val + (int64_t)boff[j] * F + (int64_t)f * sj;
  uint32_t best = p[0], bcnt = 0, cur = p[0], ccnt = 0;
  for (uint32_t q = 0; q < sj; ++q) {
    if (p[q] == cur) {
      ++ccnt;
    } else {
      if (ccnt > bcnt) {
        bcnt = ccnt;
        best = cur;
      }
      cur = p[q];
      ccnt = 1;
    }
  }
  if (ccnt > bcnt) best = cur;
  modes[(int64_t)j * ldm + f0 + f] = best;
}

// (f, value, j) triples of the modes for the inverted index
__global__ void k_index_items(const uint32_t* __restrict__ modes, int k, int F, uint32_t* __restrict__ wj,
                              uint32_t* __restrict__ wv, uint32_t* __restrict__ wf) {
  const int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (g >= (int64_t)k * F) return;
  wj[g] = (uint32_t)(g / F);
  wf[g] = (uint32_t)(g % F);
  wv[g] = modes[g];
}

__device__ __forceinline__ uint64_t pack_fv(uint32_t f, uint32_t v) { return ((uint64_t)f << 32) | v; }
__device__ __forceinline__ uint32_t slot_of(uint64_t key, uint32_t mask) {
  return fmix32((uint32_t)key ^ fmix32((uint32_t)(key >> 32) + 0x9E3779B9u)) & mask;
}

__global__ void k_fill_u64(unsigned long long* p, int64_t n, unsigned long long v) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Insert every run head of the sorted (f, v) keys: value = start << 32 | len.
__global__ void k_index_insert(const uint32_t* __restrict__ sv, const uint32_t* __restrict__ sf, int64_t NI,
                               unsigned long long* __restrict__ hkey, unsigned long long* __restrict__ hval,
                               uint32_t mask) {
  const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (q >= NI) return;
  if (q > 0 && sv[q] == sv[q - 1] && sf[q] == sf[q - 1]) return;
  int64_t e = q + 1;
  while (e < NI && sv[e] == sv[q] && sf[e] == sf[q]) ++e;
  const uint64_t key = pack_fv(sf[q], sv[q]);
  uint32_t h = slot_of(key, mask);
  while (true) {
    const unsigned long long old = atomicCAS(&hkey[h], ~0ull, (unsigned long long)key);
    if (old == ~0ull || old == key) break;
    h = (h + 1) & mask;
  }
  hval[h] = ((unsigned long long)q << 32) | (unsigned long long)(e - q);
}

__device__ __forceinline__ bool index_find(const unsigned long long* __restrict__ hkey,
                                           const unsigned long long* __restrict__ hval, uint32_t mask,
                                           uint32_t f, uint32_t v, uint32_t& start, uint32_t& len) {
  const uint64_t key = pack_fv(f, v);
  uint32_t h = slot_of(key, mask);
  while (true) {
    const unsigned long long kk = hkey[h];
    if (kk == key) {
      const unsigned long long vv = hval[h];
      start = (uint32_t)(vv >> 32);
      len = (uint32_t)vv;
      return true;
    }
    if (kk == ~0ull) return false;
    h = (h + 1) & mask;
  }
}

// One wavefront (block of 64) per row.
__global__ __launch_bounds__(64) void k_sig_assign(const uint32_t* __restrict__ S, int64_t lds, int F, int64_t n,
                                                   const unsigned long long* __restrict__ hkey,
                                                   const unsigned long long* __restrict__ hval, uint32_t mask,
                                                   const uint32_t* __restrict__ jlist, int32_t* __restrict__ assign,
                                                   double* __restrict__ dist, uint32_t* __restrict__ dense,
                                                   uint32_t* __restrict__ dense_count,
                                                   unsigned long long* __restrict__ ctr) {
  __shared__ uint32_t lst[SG_CAP];
  __shared__ uint32_t cnt;
  unsigned long long my_rows = 0, my_matches = 0;
  for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
    if (threadIdx.x == 0) cnt = 0;
    __syncthreads();
    const uint32_t* row = S + i * lds;
    for (int f = threadIdx.x; f < F; f += 64) {
      uint32_t st, ln;
      if (index_find(hkey, hval, mask, (uint32_t)f, row[f], st, ln)) {
        const uint32_t at = atomicAdd(&cnt, ln);
        for (uint32_t e = 0; e < ln; ++e)
          if (at + e < SG_CAP) lst[at + e] = jlist[st + e];
      }
    }
    __syncthreads();
    const uint32_t c = cnt;
    if (c > SG_CAP) {
      if (threadIdx.x == 0) dense[atomicAdd(dense_count, 1u)] = (uint32_t)i;
      __syncthreads();
      continue;
    }
    int P2 = 1;
    while (P2 < (int)c) P2 <<= 1;
    for (int q = (int)c + threadIdx.x; q < P2; q += 64) lst[q] = 0xFFFFFFFFu;
    __syncthreads();
    for (int kk = 2; kk <= P2; kk <<= 1) {
      for (int jj = kk >> 1; jj > 0; jj >>= 1) {
        for (int q = threadIdx.x; q < P2; q += 64) {
          const int o = q ^ jj;
          if (o > q) {
            const uint32_t a = lst[q], b = lst[o];
            const bool up = (q & kk) == 0;
            if (up ? (b < a) : (a < b)) {
              lst[q] = b;
              lst[o] = a;
            }
          }
        }
        __syncthreads();
      }
    }
    if (threadIdx.x == 0) {
      uint32_t best = 0, bcnt = 0, cur = 0, ccnt = 0;
      for (uint32_t q = 0; q < c; ++q) {
        if (q > 0 && lst[q] == cur) {
          ++ccnt;
        } else {
          if (q > 0 && ccnt > bcnt) {
            bcnt = ccnt;
            best = cur;
          }
          cur = lst[q];
          ccnt = 1;
        }
      }
      if (c > 0 && ccnt > bcnt) {
        bcnt = ccnt;
        best = cur;
      }
      assign[i] = (int32_t)best;  // no match: every count is 0, seed 0 wins
      dist[i] = 1.0 - (double)bcnt / (double)F;
      ++my_rows;
      my_matches += c;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0 && ctr) {
    atomicAdd(ctr + 0, my_rows);
    atomicAdd(ctr + 3, my_matches);
  }
}

// Rows whose match lists overflowed: count against every mode, lowest j on
// ties.  One lane per row, 256 rows per workgroup; blocks of 32 seeds x 256
// signature positions are staged in LDS and read by every lane at the same
// address (broadcast); each lane keeps 16 of its row's words and 32 match
// counters in registers (a compare and an add-with-carry per comparison).
constexpr int SD_SEEDS = 32;   // seeds per register block
constexpr int SD_F = 16;       // signature words per register chunk
constexpr int SD_SEG = 256;    // signature positions per LDS segment
__global__ __launch_bounds__(256) void k_sig_dense(const uint32_t* __restrict__ S, int64_t lds, int F,
                                                   const uint32_t* __restrict__ modes, int k,
                                                   const uint32_t* __restrict__ rows,
                                                   const uint32_t* __restrict__ count, int64_t n_rows,
                                                   int32_t* __restrict__ assign, double* __restrict__ dist,
                                                   unsigned long long* __restrict__ ctr) {
  __shared__ __attribute__((aligned(16))) uint32_t lm[SD_SEEDS * SD_SEG];
  const int64_t nr = rows ? (int64_t)*count : n_rows;  // rows == nullptr: every row
  const int lane = threadIdx.x & 63;
  for (int64_t base = (int64_t)blockIdx.x * 256; base < nr; base += (int64_t)gridDim.x * 256) {
    const int64_t pos = base + threadIdx.x;
    const bool live = pos < nr;
    const int64_t i = !live ? 0 : rows ? (int64_t)rows[pos] : pos;
    const uint32_t* srow = S + i * lds;
    const bool row_vec = (lds & 3) == 0;
    uint32_t best = 0, bj = 0x7fffffffu;
    for (int jb = 0; jb < k; jb += SD_SEEDS) {
      uint32_t cnt[SD_SEEDS];
#pragma unroll
      for (int q = 0; q < SD_SEEDS; ++q) cnt[q] = 0u;
      for (int fs = 0; fs < F; fs += SD_SEG) {
        const int seg = F - fs < SD_SEG ? F - fs : SD_SEG;
        __syncthreads();  // previous segment consumed
        for (int t = threadIdx.x; t < SD_SEEDS * SD_SEG; t += 256) {
          const int q = t / SD_SEG, f = t % SD_SEG;
          lm[t] = (jb + q < k && f < seg) ? modes[(int64_t)(jb + q) * F + fs + f] : 0u;
        }
        __syncthreads();
        for (int f0 = 0; f0 < seg; f0 += SD_F) {
          if (row_vec && f0 + SD_F <= seg) {
            uint32_t x[SD_F];
#pragma unroll
            for (int e = 0; e < SD_F; e += 4) {
              const uint4 v = *reinterpret_cast<const uint4*>(srow + fs + f0 + e);
              x[e] = v.x;
              x[e + 1] = v.y;
              x[e + 2] = v.z;
              x[e + 3] = v.w;
            }
#pragma unroll
            for (int q = 0; q < SD_SEEDS; ++q) {
#pragma unroll
              for (int e = 0; e < SD_F; e += 4) {
                const uint4 m = *reinterpret_cast<const uint4*>(lm + q * SD_SEG + f0 + e);
                cnt[q] += (x[e] == m.x) ? 1u : 0u;
                cnt[q] += (x[e + 1] == m.y) ? 1u : 0u;
                cnt[q] += (x[e + 2] == m.z) ? 1u : 0u;
                cnt[q] += (x[e + 3] == m.w) ? 1u : 0u;
              }
            }
          } else {
            for (int f = f0; f < seg && f < f0 + SD_F; ++f) {
              const uint32_t xv = srow[fs + f];
#pragma unroll
              for (int q = 0; q < SD_SEEDS; ++q) cnt[q] += (xv == lm[q * SD_SEG + f]) ? 1u : 0u;
            }
          }
        }
      }
      // strict > with ascending j keeps the lowest index on ties
#pragma unroll
      for (int q = 0; q < SD_SEEDS; ++q) {
        const int j = jb + q;
        if (j < k && (cnt[q] > best || bj == 0x7fffffffu)) {
          best = cnt[q];
          bj = (uint32_t)j;
        }
      }
    }
    if (live) {
      assign[i] = (int32_t)bj;
      dist[i] = 1.0 - (double)best / (double)F;
    }
    if (ctr) {
      const unsigned long long nlive = __popcll(__ballot(live));
      if (lane == 0 && nlive) atomicAdd(ctr + 2, nlive);
    }
  }
}


// ---- match counts as bit planes
//
// Every distinct (position f, mode value v) gets a bit mask over the seeds
// that hold v at f; a row's counts against all seeds are then the sum of the
// masks of its F (f, value) pairs.  GL lanes own a row, each with four mask
// words (128 seeds), and add the masks into NP bit planes (plane b holds bit
// b of every seed's count) with carry-save adders: about 2.5 vector
// operations per mask word, 32 seeds each, where a comparison with every mode
// takes two per seed.  The largest count is read off the planes from the top
// (the seeds that still tie are a mask), the lowest seed of the tie wins.
//
// What bounds it: half the time is the table probes (one 16-byte load per
// position from a table of a few MB), half the mask reads (16 * GL bytes per
// position that any mode shares with the row, 193 of 256 on the sets workload:
// 49 GB per 10^6 rows at about 20 TB/s, mostly from L2).  Figures at
// sig_use_bits.
constexpr int SB_VW = 4;        // mask words per lane
constexpr int SB_THREADS = 128;
constexpr int SB_STEP = 8;      // masks added per step

constexpr int BI_THREADS = 512;
constexpr int BI_BUCKET = 4;    // entries of a bucket: one 16-byte load
constexpr int BI_BITS_MAX = 15; // buckets per position: at most 2^15
constexpr int BI_SEEDS = 6;     // hashes tried per bucket count

// A bijection of 32-bit words per seed, so (bucket, remaining bits) names a
// value exactly.
GEEK_D uint32_t bits_hash(uint32_t v, uint32_t seed) { return fmix32(v ^ (seed * 0x9E3779B9u)); }

// How position f's values are found: bucket = hash & bmask at table[first +
// bucket], mask rows from row0; bmask 0: no hash tried kept every bucket within
// BI_BUCKET entries, the value is searched in runs[].
struct BitsPos {
  uint32_t first, bmask, seed, row0;
};

// One workgroup per position f: the seeds sorted by (mode value, seed) in LDS
// and written to keys[f][0..k); the number of distinct values and a hash that
// puts at most BI_BUCKET of them into a bucket, with the fewest buckets of a
// mean load of at most 0.6 (one load then finds a value or its absence: with
// linear probing the longest probe of a wavefront's 1,024 set the time).
__global__ __launch_bounds__(BI_THREADS) void k_bits_sort(const uint32_t* __restrict__ modes, int k, int F, int P,
                                                          int bits_cap, unsigned long long* __restrict__ keys,
                                                          uint32_t* __restrict__ distinct, BitsPos* __restrict__ pos) {
  extern __shared__ __attribute__((aligned(16))) unsigned long long bi_key[];  // [P], P = pow2 >= k
  __shared__ uint32_t fill[(1 << BI_BITS_MAX) / 4];  // byte counts of the buckets
  __shared__ uint32_t total, over;
  const uint32_t f = blockIdx.x;
  if (threadIdx.x == 0) total = 0u;
  for (int q = threadIdx.x; q < P; q += BI_THREADS)
    bi_key[q] = q < k ? ((unsigned long long)modes[(int64_t)q * F + f] << 32) | (uint32_t)q : ~0ull;
  __syncthreads();
  for (int kk = 2; kk <= P; kk <<= 1)
    for (int jj = kk >> 1; jj > 0; jj >>= 1) {
      for (int q = threadIdx.x; q < P / 2; q += BI_THREADS) {
        const int lo = 2 * q - (q & (jj - 1)), hi = lo + jj;
        const unsigned long long x = bi_key[lo], y = bi_key[hi];
        if ((x > y) == ((lo & kk) == 0)) {
          bi_key[lo] = y;
          bi_key[hi] = x;
        }
      }
      __syncthreads();
    }
  uint32_t heads = 0;
  for (int q = threadIdx.x; q < k; q += BI_THREADS) {
    heads += q == 0 || (bi_key[q] >> 32) != (bi_key[q - 1] >> 32);
    keys[(size_t)f * k + q] = bi_key[q];
  }
  if (heads) atomicAdd(&total, heads);
  __syncthreads();
  const uint32_t D = total;
  int bits = 2;
  while (3u << bits < 5u * D || (1u << bits) <= D) ++bits;
  uint32_t bmask = 0u, seed = 0u;
  for (; bits <= bits_cap && bmask == 0u; ++bits)
    for (uint32_t sd = 0; sd < BI_SEEDS; ++sd) {
      const uint32_t bm = (1u << bits) - 1u;
      for (uint32_t q = threadIdx.x; q <= bm / 4u; q += BI_THREADS) fill[q] = 0u;
      if (threadIdx.x == 0) over = 0u;
      __syncthreads();
      for (int q = threadIdx.x; q < k; q += BI_THREADS)
        if (q == 0 || (bi_key[q] >> 32) != (bi_key[q - 1] >> 32)) {
          const uint32_t h = bits_hash((uint32_t)(bi_key[q] >> 32), sd) & bm, sh = 8u * (h & 3u);
          if ((atomicAdd(&fill[h >> 2], 1u << sh) >> sh & 255u) >= (uint32_t)BI_BUCKET) over = 1u;
        }
      __syncthreads();
      const bool ok = over == 0u;
      __syncthreads();
      if (ok) {
        bmask = bm;
        seed = sd;
        break;
      }
    }
  if (threadIdx.x == 0) {
    distinct[f] = D;
    pos[f] = BitsPos{0u, bmask, seed, 0u};
  }
}

// One workgroup per position f: the first bucket and mask row (tables and rows
// of all positions lie without gaps; row 0 is all zeros), the bucket entries,
// runs[f][r] = {value, mask row} of the r-th distinct value, and the masks.  An
// entry holds the hash above its bucket bits and, below them, 1 + r.
__global__ __launch_bounds__(BI_THREADS) void k_bits_fill(const unsigned long long* __restrict__ keys, int k,
                                                          const uint32_t* __restrict__ distinct,
                                                          const BitsPos* __restrict__ pos_in,
                                                          BitsPos* __restrict__ pos, uint32_t* __restrict__ table,
                                                          unsigned long long* __restrict__ runs,
                                                          uint32_t* __restrict__ masks, int row_words) {
  __shared__ uint32_t base[2];  // distinct values and buckets of the positions before f
  __shared__ uint32_t wsum[BI_THREADS / 64];
  const uint32_t f = blockIdx.x;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (threadIdx.x < 2) base[threadIdx.x] = 0u;
  __syncthreads();
  for (uint32_t p = threadIdx.x; p < f; p += BI_THREADS) {
    atomicAdd(&base[0], distinct[p]);
    atomicAdd(&base[1], pos_in[p].bmask + 1u);
  }
  if (f == 0)
    for (int q = threadIdx.x; q < row_words; q += BI_THREADS) masks[q] = 0u;
  const unsigned long long* kf = keys + (size_t)f * k;
  // rank of an item's value among the distinct ones: thread t owns the items
  // t per .. t per + per - 1
  const int per = (k + BI_THREADS - 1) / BI_THREADS, q0 = threadIdx.x * per;
  uint32_t heads = 0;
  for (int q = q0; q < q0 + per && q < k; ++q) heads += q == 0 || (kf[q] >> 32) != (kf[q - 1] >> 32);
  uint32_t incl = heads;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(incl, o);
    if (lane >= o) incl += y;
  }
  if (lane == 63) wsum[wv] = incl;
  __syncthreads();
  uint32_t rank = incl - heads;
  for (int w = 0; w < wv; ++w) rank += wsum[w];
  const BitsPos p = pos_in[f];
  const uint32_t D = distinct[f], row0 = base[0] + 1u;
  if (threadIdx.x == 0) pos[f] = BitsPos{base[1], p.bmask, p.seed, row0};
  uint32_t* tf = table + (size_t)base[1] * BI_BUCKET;
  uint32_t* mf = masks + (size_t)row0 * row_words;
  for (uint32_t q = threadIdx.x; q < (p.bmask + 1u) * BI_BUCKET; q += BI_THREADS) tf[q] = 0u;
  for (uint32_t q = threadIdx.x; q < D * (uint32_t)row_words; q += BI_THREADS) mf[q] = 0u;
  __syncthreads();  // the atomics below follow the workgroup's own stores
  for (int q = q0; q < q0 + per && q < k; ++q) {
    const uint32_t v = (uint32_t)(kf[q] >> 32), j = (uint32_t)kf[q];
    if (q == 0 || (uint32_t)(kf[q - 1] >> 32) != v) {
      if (p.bmask) {
        const uint32_t h = bits_hash(v, p.seed), e = (h & ~p.bmask) | (rank + 1u);
        uint32_t* b = tf + (size_t)(h & p.bmask) * BI_BUCKET;
        while (atomicCAS(b, 0u, e) != 0u) ++b;  // at most BI_BUCKET values per bucket (k_bits_sort)
      }
      runs[(size_t)f * k + rank] = ((unsigned long long)v << 32) | (row0 + rank);
      ++rank;
    }
    atomicOr(&mf[(size_t)(rank - 1u) * row_words + (j >> 5)], 1u << (j & 31));
  }
}

// Mask row of value v at a position without a hash: binary search, 0 if absent.
GEEK_D uint32_t bits_search(const unsigned long long* __restrict__ runs, uint32_t D, uint32_t v) {
  uint32_t lo = 0, hi = D;
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if ((uint32_t)(runs[mid] >> 32) < v) lo = mid + 1u; else hi = mid;
  }
  return lo < D && (uint32_t)(runs[lo] >> 32) == v ? (uint32_t)runs[lo] : 0u;
}

GEEK_D void csa(uint32_t& hi, uint32_t& lo, uint32_t a, uint32_t b, uint32_t c) {
  hi = (a & b) | (c & (a ^ b));
  lo = a ^ b ^ c;
}

template <int GL, int NP>
__global__ __launch_bounds__(SB_THREADS) void k_sig_bits(const uint32_t* __restrict__ S, int64_t lds, int F,
                                                         int64_t n, int k,
                                                         const uint4* __restrict__ table,
                                                         const BitsPos* __restrict__ tpos,
                                                         const unsigned long long* __restrict__ runs,
                                                         const uint32_t* __restrict__ distinct,
                                                         const uint32_t* __restrict__ masks,
                                                         int32_t* __restrict__ assign, double* __restrict__ dist,
                                                         unsigned long long* __restrict__ ctr) {
  constexpr int R = 64 / GL;  // rows per wavefront
  constexpr int U = R >= 8 ? 2 : 4;  // words of a row per lane and step
  extern __shared__ __attribute__((aligned(16))) uint32_t sb_list[];
  const int fpad = (F + SB_STEP - 1) / SB_STEP * SB_STEP + 2 * SB_STEP;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t* lst = sb_list + (size_t)wave * R * fpad;
  const int g = lane / GL, sub = lane % GL;
  const uint32_t row_bytes = GL * SB_VW * 4;
  const int64_t tiles = (n + R - 1) / R, waves = (int64_t)gridDim.x * (SB_THREADS / 64);
  for (int64_t t = (int64_t)blockIdx.x * (SB_THREADS / 64) + wave; t < tiles; t += waves) {
    const int64_t i0 = t * R;
    // mask rows of the positions that share a value with some mode: the words
    // of all R rows, then all their probes, are in flight together
    int cnt[R];
#pragma unroll
    for (int r = 0; r < R; ++r) cnt[r] = 0;
    for (int f0 = 0; f0 < F; f0 += 64 * U) {
      uint32_t v[R][U];
      uint4 e[R][U];
      BitsPos tp[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        tp[u] = f0 + u * 64 + lane < F ? tpos[f0 + u * 64 + lane] : BitsPos{0u, 1u, 0u, 0u};
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int f = f0 + u * 64 + lane;
          v[r][u] = f < F && i0 + r < n ? S[(i0 + r) * lds + f] : 0u;
        }
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int u = 0; u < U; ++u) {
          v[r][u] = bits_hash(v[r][u], tp[u].seed);
          e[r][u] = table[tp[u].first + (v[r][u] & tp[u].bmask)];
        }
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int f = f0 + u * 64 + lane;
          const uint32_t bm = tp[u].bmask, q = v[r][u] & ~bm;
          const uint32_t ex[4] = {e[r][u].x ^ q, e[r][u].y ^ q, e[r][u].z ^ q, e[r][u].w ^ q};
          uint32_t rk = 0u;  // 1 + the value's rank; the entry's other bits agree
#pragma unroll
          for (int z = 0; z < 4; ++z) rk = ex[z] - 1u < bm ? ex[z] : rk;
          uint32_t row = rk ? tp[u].row0 + rk - 1u : 0u;
          const bool live = f < F && i0 + r < n;
          if (live && bm == 0u) row = bits_search(runs + (size_t)f * k, distinct[f], S[(i0 + r) * lds + f]);
          const bool some = live && row != 0u;
          const uint64_t hit = __ballot(some);
          if (some) lst[r * fpad + cnt[r] + __popcll(hit & ((1ull << lane) - 1ull))] = row;
          cnt[r] += __popcll(hit);
        }
    }
    int most = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      // padded with the zero mask to whole steps
      if (lane < 2 * SB_STEP) lst[r * fpad + cnt[r] + lane] = 0u;
      if (g == r) most = cnt[r];
    }
    int steps = (most + SB_STEP - 1) / SB_STEP;  // per row
    int all = steps;
#pragma unroll
    for (int o = GL; o < 64; o <<= 1) all = max(all, __shfl_xor(all, o));
    uint32_t pl[NP][SB_VW];
#pragma unroll
    for (int b = 0; b < NP; ++b)
#pragma unroll
      for (int w = 0; w < SB_VW; ++w) pl[b][w] = 0u;
    const uint32_t* my = lst + g * fpad;
    const char* mbase = reinterpret_cast<const char*>(masks) + sub * (SB_VW * 4);
    __builtin_amdgcn_wave_barrier();
    uint4 x[SB_STEP];
    {
#pragma unroll
      for (int u = 0; u < SB_STEP; ++u)
        x[u] = *reinterpret_cast<const uint4*>(mbase + (uint64_t)(steps > 0 ? my[u] : 0u) * row_bytes);
    }
    for (int c = 0; c < all; ++c) {
      uint4 y[SB_STEP];
      const bool more = c + 1 < steps;
#pragma unroll
      for (int u = 0; u < SB_STEP; ++u)
        y[u] = *reinterpret_cast<const uint4*>(mbase + (uint64_t)(more ? my[(c + 1) * SB_STEP + u] : 0u) * row_bytes);
#pragma unroll
      for (int w = 0; w < SB_VW; ++w) {
        uint32_t m[SB_STEP];
#pragma unroll
        for (int u = 0; u < SB_STEP; ++u) m[u] = w == 0 ? x[u].x : w == 1 ? x[u].y : w == 2 ? x[u].z : x[u].w;
        uint32_t t2a, t2b, t2c, t2d, t4a, t4b, t8;
        csa(t2a, pl[0][w], pl[0][w], m[0], m[1]);
        csa(t2b, pl[0][w], pl[0][w], m[2], m[3]);
        csa(t4a, pl[1][w], pl[1][w], t2a, t2b);
        csa(t2c, pl[0][w], pl[0][w], m[4], m[5]);
        csa(t2d, pl[0][w], pl[0][w], m[6], m[7]);
        csa(t4b, pl[1][w], pl[1][w], t2c, t2d);
        csa(t8, pl[2][w], pl[2][w], t4a, t4b);
#pragma unroll
        for (int b = 3; b < NP; ++b) {
          const uint32_t c2 = pl[b][w] & t8;
          pl[b][w] ^= t8;
          t8 = c2;
        }
      }
#pragma unroll
      for (int u = 0; u < SB_STEP; ++u) x[u] = y[u];
    }
    // largest count: seeds that tie on the bits read so far
    uint32_t cand[SB_VW];
#pragma unroll
    for (int w = 0; w < SB_VW; ++w) {
      const int j0 = (sub * SB_VW + w) * 32;
      cand[w] = j0 + 32 <= k ? ~0u : j0 >= k ? 0u : (1u << (k - j0)) - 1u;
    }
    const uint64_t gmask = (GL == 64 ? ~0ull : ((1ull << (GL & 63)) - 1ull) << (g * GL));
    uint32_t best = 0;
#pragma unroll
    for (int b = NP - 1; b >= 0; --b) {
      uint32_t q[SB_VW], any = 0;
#pragma unroll
      for (int w = 0; w < SB_VW; ++w) {
        q[w] = cand[w] & pl[b][w];
        any |= q[w];
      }
      const bool some = (__ballot(any != 0u) & gmask) != 0ull;
      if (some) best |= 1u << b;
#pragma unroll
      for (int w = 0; w < SB_VW; ++w) cand[w] = some ? q[w] : cand[w];
    }
    const uint64_t holders = __ballot((cand[0] | cand[1] | cand[2] | cand[3]) != 0u) & gmask;
    if (holders != 0ull && lane == __ffsll((unsigned long long)holders) - 1 && i0 + g < n) {
      const int w = cand[0] ? 0 : cand[1] ? 1 : cand[2] ? 2 : 3;
      const uint32_t cw = cand[0] ? cand[0] : cand[1] ? cand[1] : cand[2] ? cand[2] : cand[3];
      assign[i0 + g] = (sub * SB_VW + w) * 32 + __ffs(cw) - 1;
      dist[i0 + g] = 1.0 - (double)best / (double)F;
    }
    __builtin_amdgcn_wave_barrier();
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) atomicAdd(ctr + 2, (unsigned long long)n);  // every row, counted once
}

__global__ void k_zero_words(uint32_t* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
}
__global__ void k_copy_ctr(const unsigned long long* a, unsigned long long* b) {
  if (threadIdx.x < 4) b[threadIdx.x] = a[threadIdx.x];
}

// ---------------------------------------------------------------- host side
// Lanes per row of the bit-plane counts (a power of two of at least 8 and
// k / 128; rows of more than 512 positions take at least 16, so that the
// match lists of a wavefront's rows fit in LDS).
static int sig_lanes(int F, int k) {
  int gl = F > 512 ? 16 : 8;
  while ((int64_t)gl * 32 * SB_VW < k) gl *= 2;
  return gl;
}

// Whether rows are counted by bit planes where every row meets every mode
// (k * F <= SIG_DENSE_MAX).  Measured per call against k_sig_dense's path, which
// also sorted an index it did not read (us, F = 256): n = 1,000, k = 16: 277
// against 517; n = 10^5, k = 16: 477 against 590, k = 1,000: 693 against 3,683;
// 10^6 sets, k = 2,000: the counting alone 4.35 ms against 33 ms.  The bit
// planes won at every size tried; above SIG_BITS_K seeds the masks outgrow
// half a gigabyte and the direct comparison stays.
static bool sig_use_bits(const geek_assign_job& J) {
  return (int64_t)J.k * J.F <= SIG_DENSE_MAX && J.k <= SIG_BITS_K;
}

struct SigWs {
  uint32_t *val, *seg, *val2, *seg2;
  uint32_t *boff, *bcount;  // modes by sorting: first member of each seed; members, items
  uint32_t *wj, *wv, *wf, *wj2, *wv2, *wf2;
  unsigned long long *hkey, *hval, *ctr;
  uint32_t *dense, *small, *rtmp;
  double *dist, *sse_blk;
  uint32_t hmask;
  // bit-plane counts (sig_use_bits): per-position slot tables and the masks
  unsigned long long *btab, *bkeys, *runs;
  BitsPos *bpos, *tpos;
  uint32_t *masks, *distinct;
  int row_words, bits_cap;
};

static uint64_t pow2_at_least(uint64_t v) {
  uint64_t p = 1;
  while (p < v && p < (1ull << 32)) p <<= 1;
  return p;
}

static int bits_of(uint64_t v) {
  int b = 0;
  while (b < 32 && (v >> b)) ++b;
  return b;
}

// Positions whose items are sorted together: as many as keep the sort's 32-bit
// item count (and segment number: k <= NC) below 2^31.
static int mode_slice(int64_t NC, int F) {
  return (int)std::max<int64_t>(1, std::min<int64_t>(F, ((int64_t)1 << 31) / std::max<int64_t>(NC, 1)));
}

static size_t carve_sig(const geek_assign_job& J, void* ws, SigWs& W) {
  Carver c(ws);
  const int64_t F = J.F;
  const int64_t NI = J.n_members * mode_slice(J.n_members, J.F);
  const int64_t KI = (int64_t)J.k * F;
  const int64_t NR = NI > KI ? NI : KI;
  W.val = c.take<uint32_t>(NR + 1);
  W.seg = c.take<uint32_t>(NR + 1);
  W.val2 = c.take<uint32_t>(NR + 1);
  W.seg2 = c.take<uint32_t>(NR + 1);
  W.boff = c.take<uint32_t>(J.k + 1);
  W.bcount = c.take<uint32_t>(2);
  W.wj = c.take<uint32_t>(KI + 1);
  W.wv = c.take<uint32_t>(KI + 1);
  W.wf = c.take<uint32_t>(KI + 1);
  W.wj2 = c.take<uint32_t>(KI + 1);
  W.wv2 = c.take<uint32_t>(KI + 1);
  W.wf2 = c.take<uint32_t>(KI + 1);
  // at most half full, or (KI < 2^32 from 2^31 on) with slots left empty: a
  // probe ends at one
  const uint64_t HS = pow2_at_least(2 * (uint64_t)KI + 2);
  W.hmask = (uint32_t)(HS - 1);
  const bool bits = sig_use_bits(J), index = KI > SIG_DENSE_MAX;
  W.hkey = c.take<unsigned long long>(index ? HS : 0);
  W.hval = c.take<unsigned long long>(index ? HS : 0);
  W.row_words = sig_lanes(J.F, J.k) * SB_VW;
  // at most 2^bits_cap buckets per position (mean load 1/8 or less)
  W.bits_cap = std::min(BI_BITS_MAX, bits_of((uint64_t)J.k) + 3);
  W.btab = c.take<unsigned long long>(bits ? ((size_t)F << W.bits_cap) * BI_BUCKET / 2 : 0);
  W.bkeys = c.take<unsigned long long>(bits ? KI : 0);
  W.runs = c.take<unsigned long long>(bits ? KI : 0);
  W.bpos = c.take<BitsPos>(bits ? F : 0);
  W.tpos = c.take<BitsPos>(bits ? F : 0);
  W.distinct = c.take<uint32_t>(bits ? F : 0);
  W.masks = c.take<uint32_t>(bits ? (size_t)(KI + 1) * W.row_words : 0);
  W.ctr = c.take<unsigned long long>(4);
  W.dense = c.take<uint32_t>(J.n + 1);
  W.small = c.take<uint32_t>(16);
  W.rtmp = c.take<uint32_t>(radix_tmp_words(NR));
  W.dist = c.take<double>(J.dist ? 1 : J.n);
  W.sse_blk = c.take<double>(sse_blk_words(J.n));
  return c.used + 256;
}

size_t assign_sig_ws(const geek_assign_job& J) {
  SigWs W;
  return carve_sig(J, nullptr, W);
}

int32_t modes_run(const uint32_t* V, int64_t ldv, int F, int64_t n, const uint32_t* so, const uint32_t* sm, int k,
                  int64_t NC, uint32_t* modes, SigWs& W, int32_t* st, hipStream_t s) {
  const int64_t NI = NC * F;
  if (NI <= 0) return GEEK_OK;
  // (a launch holds less than 2^32 threads per dimension)
  hipLaunchKernelGGL(k_mode_small, dim3(std::min(k, 1 << 22), ceil_div(F, MODE_THREADS)), dim3(MODE_THREADS), 0, s, V,
                     ldv, F, n, so, sm, k, NC, modes, st);
  if (NC <= MODE_SMALL) return GEEK_OK;  // no seed can be larger
  hipLaunchKernelGGL(k_mode_sizes, dim3(ceil_div(k, 256)), dim3(256), 0, s, so, k, NC, W.boff);
  exscan_u32(W.boff, W.boff, k, W.rtmp, W.bcount, s);
  const int slice = mode_slice(NC, F);
  for (int f0 = 0; f0 < F; f0 += slice) {
    const int Fs = std::min(slice, F - f0);
    hipLaunchKernelGGL(k_mode_total, dim3(1), dim3(64), 0, s, W.bcount, Fs, NC, W.bcount + 1);
    hipLaunchKernelGGL(k_mode_items, dim3((int)std::min<int64_t>(4096, ceil_div(NC * Fs, 256))), dim3(256), 0, s, V,
                       ldv, f0, Fs, n, so, sm, k, W.boff, W.bcount + 1, W.val, W.seg, st);
    int words[8], shifts[8], np = 0;
    for (int sh = 0; sh < 32; sh += 8) {
      words[np] = 0;
      shifts[np++] = sh;
    }
    const int sb = bits_of((uint64_t)k * Fs - 1);
    for (int sh = 0; sh < sb; sh += 8) {
      words[np] = 1;
      shifts[np++] = sh;
    }
    RsView A{{W.val, W.seg, nullptr, nullptr}, nullptr}, B{{W.val2, W.seg2, nullptr, nullptr}, nullptr};
    const int alt = radix_sort_dn(A, B, 2, NC * Fs, W.bcount + 1, words, shifts, np, W.rtmp, s);
    hipLaunchKernelGGL(k_mode_pick, dim3(ceil_div((int64_t)k * Fs, 256)), dim3(256), 0, s, alt ? W.val2 : W.val, so,
                       W.boff, k, f0, Fs, F, NC, modes);
  }
  return GEEK_OK;
}

// Standalone modes of an integer matrix (the categorical attributes of
// heterogeneous rows), with its own workspace.
size_t modes_ws(int64_t n_members, int F, int k) {
  Carver c(nullptr);
  const int64_t NI = n_members * mode_slice(n_members, F), KI = (int64_t)k * F;
  const int64_t NR = NI > KI ? NI : KI;
  for (int q = 0; q < 4; ++q) c.take<uint32_t>(NR + 1);
  c.take<uint32_t>(k + 1);
  c.take<uint32_t>(2);
  c.take<uint32_t>(radix_tmp_words(NR));
  return c.used + 256;
}

int32_t modes_compute(const uint32_t* V, int64_t ldv, int F, int64_t n, const uint32_t* so, const uint32_t* sm,
                      int k, int64_t NC, uint32_t* modes, void* ws, int32_t* st, hipStream_t s) {
  Carver c(ws);
  const int64_t NI = NC * mode_slice(NC, F), KI = (int64_t)k * F;
  const int64_t NR = NI > KI ? NI : KI;
  SigWs W{};
  W.val = c.take<uint32_t>(NR + 1);
  W.seg = c.take<uint32_t>(NR + 1);
  W.val2 = c.take<uint32_t>(NR + 1);
  W.seg2 = c.take<uint32_t>(NR + 1);
  W.boff = c.take<uint32_t>(k + 1);
  W.bcount = c.take<uint32_t>(2);
  W.rtmp = c.take<uint32_t>(radix_tmp_words(NR));
  return modes_run(V, ldv, F, n, so, sm, k, NC, modes, W, st, s);
}

int32_t assign_sig(const geek_assign_job& J, void* ws, size_t ws_bytes, int32_t* st, hipStream_t s) {
  SigWs W;
  if (ws_bytes < carve_sig(J, ws, W)) return GEEK_ERR_WORKSPACE;
  const int64_t NC = J.n_members;
  prof_begin(GEEK_PROF_ASSIGN, s);
  const int F = J.F, k = J.k;
  double* dist = J.dist ? J.dist : W.dist;
  hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, s, W.small, 16);
  hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, s, reinterpret_cast<uint32_t*>(W.ctr), 8);
  modes_run(J.sig, F, F, J.n, J.seed_offsets, J.seed_members, k, NC, J.modes, W, st, s);
  const int64_t KI = (int64_t)k * F;
  const bool bits = sig_use_bits(J), index = KI > SIG_DENSE_MAX;
  const uint32_t *sj = nullptr, *sv = nullptr, *sf = nullptr;
  if (index) {  // seeds by (f, mode value)
    hipLaunchKernelGGL(k_index_items, dim3(ceil_div(KI, 256)), dim3(256), 0, s, J.modes, k, F, W.wj, W.wv, W.wf);
    int words[12], shifts[12], np = 0;
    for (int sh = 0; sh < bits_of((uint64_t)k - 1); sh += 8) {
      words[np] = 0;
      shifts[np++] = sh;
    }
    for (int sh = 0; sh < 32; sh += 8) {
      words[np] = 1;
      shifts[np++] = sh;
    }
    for (int sh = 0; sh < bits_of((uint64_t)F - 1); sh += 8) {
      words[np] = 2;
      shifts[np++] = sh;
    }
    RsView A{{W.wj, W.wv, W.wf, nullptr}, nullptr}, B{{W.wj2, W.wv2, W.wf2, nullptr}, nullptr};
    const int alt = radix_sort(A, B, 3, KI, words, shifts, np, W.rtmp, s);
    sj = alt ? W.wj2 : W.wj;
    sv = alt ? W.wv2 : W.wv;
    sf = alt ? W.wf2 : W.wf;
  }
  const int dgrid = (int)std::max<int64_t>(1, std::min<int64_t>(2048, ceil_div(J.n, 256)));
  if (bits) {
    const int P = (int)pow2_at_least((uint64_t)k);
    hipLaunchKernelGGL(k_bits_sort, dim3(F), dim3(BI_THREADS), sizeof(unsigned long long) * P, s, J.modes, k, F, P,
                       W.bits_cap, W.bkeys, W.distinct, W.bpos);
    hipLaunchKernelGGL(k_bits_fill, dim3(F), dim3(BI_THREADS), 0, s, W.bkeys, k, W.distinct, W.bpos, W.tpos,
                       reinterpret_cast<uint32_t*>(W.btab), W.runs, W.masks, W.row_words);
    prof_begin(GEEK_PROF_ASSIGN_SCAN, s);
    const int gl = W.row_words / SB_VW, R = 64 / gl, per_block = R * (SB_THREADS / 64);
    const int fpad = (F + SB_STEP - 1) / SB_STEP * SB_STEP + 2 * SB_STEP;
    const size_t shm = sizeof(uint32_t) * (size_t)per_block * fpad;
    const dim3 grid((unsigned)std::min<int64_t>(8192, (J.n + per_block - 1) / per_block));
    const auto kern = F < 512 ? (gl == 8 ? k_sig_bits<8, 9> : gl == 16 ? k_sig_bits<16, 9> : k_sig_bits<32, 9>)
                              : (gl == 8 ? k_sig_bits<8, 11> : gl == 16 ? k_sig_bits<16, 11> : k_sig_bits<32, 11>);
    hipLaunchKernelGGL(kern, grid, dim3(SB_THREADS), shm, s, J.sig, (int64_t)F, F, J.n, k,
                       reinterpret_cast<const uint4*>(W.btab), W.tpos, W.runs, W.distinct, W.masks, J.assign, dist, W.ctr);
  } else if (!index) {
    prof_begin(GEEK_PROF_ASSIGN_SCAN, s);
    hipLaunchKernelGGL(k_sig_dense, dim3(dgrid), dim3(256), 0, s, J.sig, (int64_t)F, F, J.modes, k, nullptr,
                       nullptr, J.n, J.assign, dist, W.ctr);
  } else {
    hipLaunchKernelGGL(k_fill_u64, dim3(ceil_div((int64_t)W.hmask + 1, 256)), dim3(256), 0, s, W.hkey,
                       (int64_t)W.hmask + 1, ~0ull);
    hipLaunchKernelGGL(k_index_insert, dim3(ceil_div(KI, 256)), dim3(256), 0, s, sv, sf, KI, W.hkey, W.hval,
                       W.hmask);
    prof_begin(GEEK_PROF_ASSIGN_SCAN, s);
    const int grid = J.n < 65536 ? (int)J.n : 65536;
    hipLaunchKernelGGL(k_sig_assign, dim3(grid), dim3(64), 0, s, J.sig, (int64_t)F, F, J.n, W.hkey, W.hval,
                       W.hmask, sj, J.assign, dist, W.dense, W.small, W.ctr);
    hipLaunchKernelGGL(k_sig_dense, dim3(dgrid), dim3(256), 0, s, J.sig, (int64_t)F, F, J.modes, k, W.dense,
                       W.small, (int64_t)0, J.assign, dist, W.ctr);
  }
  prof_end(GEEK_PROF_ASSIGN_SCAN, s);
  sse_and_radius(dist, J.assign, J.n, k, J.sse, J.radius, 0, W.sse_blk, false, s);
  if (J.counters) hipLaunchKernelGGL(k_copy_ctr, dim3(1), dim3(64), 0, s, W.ctr, J.counters);
  prof_end(GEEK_PROF_ASSIGN, s);
  GEEK_LAUNCH_CHECK();
  return GEEK_OK;
}

}  // namespace geek

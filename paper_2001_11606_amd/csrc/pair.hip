// Pair form of the fine-level operator (see pair.h): its structure from the
// neighbour lists, and per assembly its values (Sec. 2.4: the V-scaled
// Brookshaw couplings), the diagonal and the ghost couplings.
//
// Structure, one block per tile of 256 rows:
//   1. k_pair_build reads the tile's interior neighbours twice.  The first
//      sweep collects the columns outside the tile as 64-bit masks of
//      64-column blocks in an LDS hash table and counts each row's neighbours
//      right of the diagonal; the blocks are sorted by rank.  The second sweep
//      writes each row's pairs with local columns.  A wave takes four rows at
//      a time, so four list reads are in flight; the second sweep is served
//      by the last-level cache.
//   2. k_pair_scan (one block) turns the tiles' external column counts into
//      offsets and collects what the host needs to know, read back once.
//   3. k_pair_lists writes the external columns and, into every later tile
//      they belong to, a segment; k_pair_sort puts a tile's segments in order
//      and k_pair_recv turns them into the rows' lists of incoming sums.
// Values, one pass over the pairs: the tile's particle records are staged in
// LDS once and every pair is evaluated once, where the CSR assembly evaluates
// it from both ends with records gathered from global memory.  The diagonal
// needs the sums of both ends: a product of the pair form with the vector of
// ones.
#include <algorithm>
#include <cstring>

#include "internal.h"
#include "kernels_sph.h"
#include "pair.h"
#include "prim.h"

namespace rt {
namespace {

constexpr int kPairSlots = 512;   // hash table of 64-column blocks
constexpr int kPairRows = 4;      // rows a wave reads at a time

struct PairStat {   // per tile; bad: 1 it does not fit, 2 nor would a tile of CSR rows
  int32_t ext, distinct, max_row, bad;
  int64_t nnz;
};
struct PairTotals {   // read back by the host
  int64_t ext, distinct, nnz;
  int32_t max_ext, max_row, bad, pad;
};

__device__ __forceinline__ int pair_slot(int32_t b) {
  return (int)(((uint32_t)b * 2654435761u) >> 23) & (kPairSlots - 1);
}

// Insert column c; returns false when the table is full.
__device__ __forceinline__ bool pair_insert(int32_t c, int* keys, unsigned long long* masks) {
  const int32_t b = c >> 6;
  int s = pair_slot(b);
  for (int step = 0; step < kPairSlots; ++step, s = (s + 1) & (kPairSlots - 1)) {
    int cur = ((volatile int*)keys)[s];
    if (cur == -1) {
      cur = atomicCAS(&keys[s], -1, b);
      if (cur == -1) cur = b;
    }
    if (cur == b) {
      const unsigned long long bit = 1ull << (c & 63);
      if (!(((volatile unsigned long long*)masks)[s] & bit)) atomicOr(&masks[s], bit);
      return true;
    }
  }
  return false;
}

// Exclusive prefix sum of one value per thread over the block; *total: the sum.
template <typename T>
__device__ __forceinline__ T block_prefix(T v, T* wsum, T* total) {
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  T incl = v;
  for (int o = 1; o < kWave; o <<= 1) {
    const T u = __shfl_up(incl, o);
    if (lane >= o) incl += u;
  }
  __syncthreads();
  if (lane == kWave - 1) wsum[w] = incl;
  __syncthreads();
  T base = 0, all = 0;
  for (int q = 0; q < (int)(blockDim.x / kWave); ++q) {
    if (q < w) base += wsum[q];
    all += wsum[q];
  }
  *total = all;
  return base + incl - v;
}

// Where group g of a tile's ng groups is stored: threads T < ng mod 256 walk
// ng / 256 + 1 consecutive groups, the others one less, and step k of thread T
// lies at 256 k + T.
struct GroupPlace {
  int steps, longer, split;   // short run, threads with one more, their groups
  float inv_short, inv_long;
  __device__ explicit GroupPlace(int ng)
      : steps(ng / kBlock), longer(ng % kBlock), split(longer * (steps + 1)),
        inv_short(steps ? 1.0f / steps : 0.0f), inv_long(1.0f / (steps + 1)) {}
  __device__ __forceinline__ int operator()(int g) const {
    const bool first = g < split;
    const int run = first ? steps + 1 : steps, q = first ? g : g - split;
    int T = (int)(q * (first ? inv_long : inv_short));   // q / run, put right below
    T -= T * run > q;
    T += (T + 1) * run <= q;
    return (q - T * run) * kBlock + T + (first ? 0 : longer);
  }
};

// First group of tile t: an upper bound on the groups of the rows before it
// (a row of m neighbours has at most m/4 + 3/4), so no scan is needed.
__device__ __forceinline__ int64_t first_group(int64_t ptr_r0, int64_t r0) {
  return (ptr_r0 >> 2) + r0;
}

__global__ void __launch_bounds__(kBlock)
k_pair_build(int64_t nin, const int64_t* __restrict__ ptr, const int32_t* __restrict__ nint,
             const int32_t* __restrict__ idx, int64_t* __restrict__ goff,
             int32_t* __restrict__ gcnt, uint16_t* __restrict__ hcol, uint8_t* __restrict__ hrow,
             int32_t* __restrict__ bid, uint64_t* __restrict__ bmask, int32_t* __restrict__ nblk,
             PairStat* __restrict__ stat) {
  __shared__ int keys[kPairSlots];
  __shared__ unsigned long long masks[kPairSlots];
  __shared__ int pre[kPairSlots];        // local column of a block's first set bit
  __shared__ uint16_t list[kPairSlots], sorted[kPairSlots];
  __shared__ int srp[kTileRows], slen[kTileRows], scnt[kTileRows], sgo[kTileRows];
  __shared__ int wsum[kBlock / kWave];
  __shared__ int nocc, bad, owned, longest;
  __shared__ int64_t sbase;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = RT_UNIFORM(tid / kWave);
  const int64_t t = blockIdx.x, r0 = t * kTileRows, i = r0 + tid;
  for (int s = tid; s < kPairSlots; s += kBlock) {
    keys[s] = -1;
    masks[s] = 0;
  }
  if (tid == 0) {
    nocc = bad = owned = longest = 0;
    sbase = ptr[r0];
  }
  __syncthreads();
  const int64_t base = sbase;
  srp[tid] = i < nin ? (int)(ptr[i] - base) : 0;
  slen[tid] = i < nin ? nint[i] : 0;
  scnt[tid] = 0;
  __syncthreads();
  const int32_t* __restrict__ in = idx + base;
  const int32_t lo = (int32_t)r0, hi = (int32_t)(r0 + kTileRows);
  // sweep 1: columns outside the tile, neighbours right of the diagonal
  int own_rows = 0;
  for (int b = wave; b < kTileRows; b += (kBlock / kWave) * kPairRows) {
    int32_t c[kPairRows];
#pragma unroll
    for (int u = 0; u < kPairRows; ++u) {
      const int r = b + u * (kBlock / kWave);
      c[u] = lane < slen[r] ? in[srp[r] + lane] : -1;
    }
#pragma unroll
    for (int u = 0; u < kPairRows; ++u) {
      const int r = b + u * (kBlock / kWave);
      const int len = RT_UNIFORM(slen[r]);
      const int32_t me = lo + r;
      int up = 0;
      unsigned long long own = 0;
      int32_t cc = c[u];
      for (int k = 0; k < len; k += kWave) {
        if (k > 0) cc = k + lane < len ? in[srp[r] + k + lane] : -1;
        up += __popcll(__ballot(cc > me));
        own |= __ballot(cc >= lo && cc < hi);
        if (cc >= 0 && (cc < lo || cc >= hi) && !pair_insert(cc, keys, masks))
          *(volatile int*)&bad = 1;
      }
      if (lane == 0) scnt[r] = up;
      own_rows += own != 0;
    }
  }
  if (lane == 0) atomicAdd(&owned, own_rows);
  __syncthreads();
  // groups of the rows, longest row, entries
  int groups = 0, nnz = 0, ext = 0, low = 0, blocks = 0, total_blocks = 0;
  const int go = block_prefix((scnt[tid] + 3) / 4, wsum, &groups);
  sgo[tid] = go;
  (void)block_prefix(slen[tid], wsum, &nnz);
  atomicMax(&longest, slen[tid]);
  // blocks in ascending order: the rank of a block is the number of smaller ones
  for (int s = tid; s < kPairSlots; s += kBlock)
    if (keys[s] != -1) list[atomicAdd(&nocc, 1)] = (uint16_t)s;
  __syncthreads();
  const int occ = nocc;
  for (int k = tid; k < occ; k += kBlock) {
    const int s = list[k], key = keys[s];
    int rank = 0;
    for (int j = 0; j < occ; ++j) rank += keys[list[j]] < key;
    sorted[rank] = (uint16_t)s;
  }
  __syncthreads();
  // local columns of the later blocks; how many columns and tiles lie before
  int e2[2] = {0, 0}, m2[2] = {0, 0}, b2[2] = {0, 0}, f2[2] = {0, 0};
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int k = 2 * tid + q;
    if (k < occ) {
      const int s = sorted[k], pc = __popcll(masks[s]);
      const bool later = (int64_t)keys[s] * 64 >= hi;
      (later ? e2[q] : m2[q]) = pc;
      b2[q] = later;
      f2[q] = !later && (k == 0 || (keys[sorted[k - 1]] >> 2) != (keys[s] >> 2));
    }
  }
  const int eo = block_prefix(e2[0] + e2[1], wsum, &ext);
  (void)block_prefix(m2[0] + m2[1], wsum, &low);
  const int bo = block_prefix(b2[0] + b2[1], wsum, &blocks);
  (void)block_prefix(f2[0] + f2[1], wsum, &total_blocks);
  const bool fits = !bad && ext <= kPairMaxExt && blocks <= kPairBlocks &&
                    total_blocks <= kPairSegs && ext + low + owned < kTileMaxCols;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int k = 2 * tid + q;
    if (k < occ && b2[q]) {
      const int s = sorted[k];
      pre[s] = kTileRows + eo + (q ? e2[0] : 0);
      if (fits) {
        const int64_t o = t * kPairBlocks + bo + (q ? b2[0] : 0);
        bid[o] = keys[s];
        bmask[o] = masks[s];
      }
    }
  }
  const int64_t g0 = first_group(base, r0);
  if (tid == 0) {
    nblk[t] = fits ? blocks : 0;
    goff[t] = g0;
    gcnt[t] = groups;
    // (a full table has missed columns, so that many at least)
    const int distinct = ext + low + owned;
    stat[t] = PairStat{ext, distinct, longest, fits ? 0 : distinct < kTileMaxCols ? 1 : 2,
                       (int64_t)nnz};
  }
  __syncthreads();
  if (!fits) return;   // uniform over the block
  // sweep 2: the pairs of every row
  uint16_t* __restrict__ oc = hcol + 4 * g0;
  uint8_t* __restrict__ orow = hrow + g0;
  const GroupPlace place(groups);
  for (int b = wave; b < kTileRows; b += (kBlock / kWave) * kPairRows) {
    int32_t c[kPairRows];
#pragma unroll
    for (int u = 0; u < kPairRows; ++u) {
      const int r = b + u * (kBlock / kWave);
      c[u] = lane < slen[r] ? in[srp[r] + lane] : -1;
    }
#pragma unroll
    for (int u = 0; u < kPairRows; ++u) {
      const int r = b + u * (kBlock / kWave);
      const int len = RT_UNIFORM(slen[r]);
      const int32_t me = lo + r;
      const int o = sgo[r];
      int done = 0;
      int32_t cc = c[u];
      for (int k = 0; k < len; k += kWave) {
        if (k > 0) cc = k + lane < len ? in[srp[r] + k + lane] : -1;
        const bool up = cc > me;
        const unsigned long long m = __ballot(up);
        int l = cc - lo;
        if (up && cc >= hi) {
          const int32_t key = cc >> 6;
          int s = pair_slot(key);
          while (keys[s] != key) s = (s + 1) & (kPairSlots - 1);
          l = pre[s] + __popcll(masks[s] & ((1ull << (cc & 63)) - 1));
        }
        if (up) {
          const int e = done + __popcll(m & ((1ull << lane) - 1));
          oc[4 * place(o + (e >> 2)) + (e & 3)] = (uint16_t)l;
        }
        done += __popcll(m);
      }
      const int ng = (done + 3) / 4;
      for (int q = lane; q < ng; q += kWave) {
        const int at = place(o + q);
        orow[at] = (uint8_t)r;
        if (q == ng - 1)   // the row's last group is filled up
          for (int e = done - 4 * q; e < 4; ++e) oc[4 * at + e] = (uint16_t)(kTileRows + ext);
      }
    }
  }
}

constexpr int kScanThreads = 1024;

// offsets of the tiles' external columns and the totals, one block
__global__ void __launch_bounds__(kScanThreads)
k_pair_scan(int64_t nt, const PairStat* __restrict__ stat, int64_t* __restrict__ xoff,
            PairTotals* __restrict__ out) {
  __shared__ int64_t wsum[kScanThreads / kWave];   // a sum past 32 bits ends the pair form
  __shared__ double red[kScanThreads / kWave];
  const int64_t per = (nt + kScanThreads - 1) / kScanThreads;
  const int64_t a = threadIdx.x * per, b = a + per < nt ? a + per : nt;
  int64_t ext = 0;
  double distinct = 0, nnz = 0, max_ext = 0, max_row = 0, bad = 0;   // whole numbers below 2^53
  for (int64_t k = a; k < b; ++k) {
    const PairStat s = stat[k];
    ext += s.bad ? 0 : s.ext;
    distinct += s.distinct;
    nnz += (double)s.nnz;
    max_ext = fmax(max_ext, (double)s.ext);
    max_row = fmax(max_row, (double)s.max_row);
    bad = fmax(bad, (double)s.bad);
  }
  int64_t total = 0;
  int64_t o = block_prefix(ext, wsum, &total);
  for (int64_t k = a; k < b; ++k) {
    xoff[k] = o;
    o += stat[k].bad ? 0 : stat[k].ext;
  }
  distinct = block_sum(distinct, red);
  nnz = block_sum(nnz, red);
  max_ext = block_max(max_ext, red);
  max_row = block_max(max_row, red);
  bad = block_max(bad, red);
  if (threadIdx.x == 0) {
    xoff[nt] = total;
    *out = PairTotals{total, (int64_t)distinct, (int64_t)nnz, (int32_t)max_ext, (int32_t)max_row,
                      (int32_t)bad, 0};
  }
}

__global__ void k_zero_i32(int64_t n, int32_t* __restrict__ p) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// external columns of a tile from its blocks, and a segment in every tile
// they belong to (four consecutive blocks are one tile)
__global__ void __launch_bounds__(kBlock)
k_pair_lists(const int32_t* __restrict__ nblk, const int32_t* __restrict__ bid,
             const uint64_t* __restrict__ bmask, const int64_t* __restrict__ xoff,
             int32_t* __restrict__ xcol, int32_t* __restrict__ nseg, PairSeg* __restrict__ seg) {
  __shared__ int32_t sid[kPairBlocks];
  __shared__ uint64_t sm[kPairBlocks];
  __shared__ int so[kPairBlocks];
  __shared__ int wsum[kBlock / kWave];
  static_assert(kPairBlocks == kBlock, "one block of columns per thread");
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int64_t t = blockIdx.x, o0 = xoff[t];
  const int nb = nblk[t];
  const int32_t id = tid < nb ? bid[t * kPairBlocks + tid] : -1;
  const uint64_t m = tid < nb ? bmask[t * kPairBlocks + tid] : 0;
  int total = 0;
  const int o = block_prefix((int)__popcll(m), wsum, &total);
  sid[tid] = id;
  sm[tid] = m;
  so[tid] = o;
  __syncthreads();
  for (int b = tid / kWave; b < nb; b += kBlock / kWave) {
    const uint64_t mk = sm[b];
    if ((mk >> lane) & 1)
      xcol[o0 + so[b] + __popcll(mk & (((uint64_t)1 << lane) - 1))] = sid[b] * kWave + lane;
  }
  if (tid < nb && (tid == 0 || (sid[tid - 1] >> 2) != (id >> 2))) {
    const int64_t target = id >> 2;
    PairSeg s;
    s.pos = o0 + o;
    for (int w = 0; w < 4; ++w) {
      s.off[w] = 0;
      s.mask[w] = 0;
    }
    for (int b = tid; b < nb && (sid[b] >> 2) == target; ++b) {
      s.off[sid[b] & 3] = (uint16_t)(so[b] - o);
      s.mask[sid[b] & 3] = sm[b];
    }
    const int q = atomicAdd(&nseg[target], 1);
    if (q < kPairSegs) seg[target * kPairSegs + q] = s;
  }
}

// a tile's segments in ascending order of their sums' places, and how many
// sums they hold; one wave
__global__ void __launch_bounds__(kWave)
k_pair_sort(const int32_t* __restrict__ nseg, PairSeg* __restrict__ seg,
            int32_t* __restrict__ recv) {
  const int64_t t = blockIdx.x;
  const int ns = nseg[t], l = threadIdx.x;
  PairSeg s;
  s.pos = INT64_MAX;
  int sums = 0;
  if (l < ns) {
    s = seg[t * kPairSegs + l];
    for (int w = 0; w < 4; ++w) sums += (int)__popcll(s.mask[w]);
  }
  int rank = 0;
  for (int q = 0; q < ns; ++q) rank += __shfl(s.pos, q) < s.pos;
  sums = group_sum<kWave>(sums);
  __syncthreads();   // every segment is read
  if (l < ns) seg[t * kPairSegs + rank] = s;
  if (l == 0) recv[t] = sums;
}

// exclusive prefix sums of v (nt values), in place, one block
__global__ void __launch_bounds__(kScanThreads)
k_pair_offsets(int64_t nt, int32_t* __restrict__ v) {
  __shared__ int wsum[kScanThreads / kWave];
  const int64_t per = (nt + kScanThreads - 1) / kScanThreads;
  const int64_t a = threadIdx.x * per, b = a + per < nt ? a + per : nt;
  int s = 0, total = 0;
  for (int64_t k = a; k < b; ++k) s += v[k];
  int o = block_prefix(s, wsum, &total);
  for (int64_t k = a; k < b; ++k) {
    const int x = v[k];
    v[k] = o;
    o += x;
  }
}

// the places of the sums left for each row, in segment order
__global__ void __launch_bounds__(kBlock)
k_pair_recv(int64_t n, int32_t total, const int32_t* __restrict__ recv,
            const int32_t* __restrict__ nseg, const PairSeg* __restrict__ seg,
            int32_t* __restrict__ in_ptr, int32_t* __restrict__ in_pos) {
  __shared__ PairSeg ss[kPairSegs];
  __shared__ int wsum[kBlock / kWave];
  const int64_t t = blockIdx.x, i = t * kTileRows + threadIdx.x;
  const int ns = nseg[t];
  if (threadIdx.x < ns) ss[threadIdx.x] = seg[t * kPairSegs + threadIdx.x];
  __syncthreads();
  const int w = threadIdx.x / kWave, l = threadIdx.x & (kWave - 1);
  int own = 0, all = 0;
  for (int q = 0; q < ns; ++q) own += (int)((ss[q].mask[w] >> l) & 1);
  int o = recv[t] + block_prefix(own, wsum, &all);
  if (i < n) in_ptr[i] = o;
  if (i == n - 1) in_ptr[n] = total;
  for (int q = 0; q < ns; ++q) {
    const uint64_t m = ss[q].mask[w];
    if ((m >> l) & 1)
      in_pos[o++] = (int32_t)(ss[q].pos + ss[q].off[w] + __popcll(m & (((uint64_t)1 << l) - 1)));
  }
}

// ---- values --------------------------------------------------------------------
struct PairRec {
  double x, y, z, h, V, D;
};

// Threads per block: eight waves share a tile's records, so that a CU holds
// 16 to 32 waves beside 34 KB (cubic spline) or 76 KB (Wendland) of records.
constexpr int kValBlock = 512;

template <int DIM>
__global__ void __launch_bounds__(kValBlock)
k_pair_values(int64_t n, int kernel, PairArgs A, const double* __restrict__ sp4,
              const double* __restrict__ VD, PeriodicBox box, double* __restrict__ val64,
              float* __restrict__ val32) {
  RT_DYNAMIC_LDS(dyn_lds);
  const int tid = threadIdx.x;
  const int64_t t = blockIdx.x, r0 = t * kTileRows;
  const int64_t x0 = A.xoff[t];
  const int ncol = kTileRows + (int)(A.xoff[t + 1] - x0);
  rt_f64x2_t* rec = reinterpret_cast<rt_f64x2_t*>(dyn_lds);   // (x, y), (z, h), (V, D) per column
  for (int k = tid; k < ncol; k += kValBlock) {
    int64_t j = r0 + k;
    if (k >= kTileRows) j = A.xcol[x0 + k - kTileRows];
    if (j < n) {
      rec[3 * k] = load_pair(sp4, 2 * j);
      rec[3 * k + 1] = load_pair(sp4, 2 * j + 1);
      rec[3 * k + 2] = load_pair(VD, j);
    }
  }
  __syncthreads();
  const int64_t g0 = A.goff[t];
  const int ng = A.gcnt[t];
  const rt_u16x4* __restrict__ ct = reinterpret_cast<const rt_u16x4*>(A.col + 4 * g0);
  rt_f64x2_t* __restrict__ o64 = reinterpret_cast<rt_f64x2_t*>(val64 + 4 * g0);
  rt_f32x4* __restrict__ o32 = val32 ? reinterpret_cast<rt_f32x4*>(val32 + 4 * g0) : nullptr;
  if (ng == 0) return;
  // the next group's columns and row are requested before this one is evaluated
  // (2.1M Wendland rows 1.46 -> 1.35 ms, 16.8M cubic-spline rows 2.04 -> 1.95)
  rt_u16x4 c = ct[min(tid, ng - 1)];
  int r = A.row[g0 + min(tid, ng - 1)];
  for (int g = tid; g < ng; g += kValBlock) {
    const int nx = min(g + kValBlock, ng - 1);
    const rt_u16x4 c_next = ct[nx];
    const int r_next = A.row[g0 + nx];
    const rt_f64x2_t pxy = rec[3 * r], pzh = rec[3 * r + 1], pvd = rec[3 * r + 2];
    double v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (c[q] >= ncol) {   // the filling of a row's last group
        v[q] = 0.0;
        continue;
      }
      const rt_f64x2_t qxy = rec[3 * c[q]], qzh = rec[3 * c[q] + 1], qvd = rec[3 * c[q] + 2];
      const double dx = periodic_disp(pxy[0] - qxy[0], box, 0);
      const double dy = periodic_disp(pxy[1] - qxy[1], box, 1);
      const double dz = DIM == 3 ? periodic_disp(pzh[0] - qzh[0], box, 2) : 0.0;
      const double dist = sqrt(dx * dx + dy * dy + dz * dz);
      // equal smoothing lengths give equal kernel derivatives: evaluate once
      const double wi = sph_dwdr<DIM>(dist, pzh[1], kernel);
      const double wj = qzh[1] == pzh[1] ? wi : sph_dwdr<DIM>(dist, qzh[1], kernel);
      const double F = -0.5 * (wi + wj) / dist;
      v[q] = -(pvd[0] * qvd[0]) * (pvd[1] + qvd[1]) * F;
    }
    o64[g] = rt_f64x2_t{v[0], v[1]};
    o64[ng + g] = rt_f64x2_t{v[2], v[3]};
    if (o32) o32[g] = rt_f32x4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
    c = c_next;
    r = r_next;
  }
}

struct DiagArgs {
  const int64_t* ptr;
  const int32_t *nint, *idx;
  const double *sp4, *VD, *sa, *f, *Eall;
  double *diag64, *dinv64, *sinv64, *g;
  float *diag32, *dinv32, *sinv32;
  PeriodicBox box;
};

// Diagonal, Jacobi and l1-Jacobi inverses and ghost couplings of the rows, one
// row per thread: diag64 holds the tile's own part of the row sums on entry;
// the row's ghost neighbours follow its interior ones in the lists.
template <int DIM>
__global__ void __launch_bounds__(kBlock)
k_pair_diag(int64_t nin, int kernel, double dt, double c, DiagArgs A, PairIn P,
            const double* __restrict__ xsum) {
  const int64_t i = blockIdx.x * (int64_t)kTileRows + threadIdx.x;
  if (i >= nin) return;
  const double in = pair_in<double>(P, i, xsum);
  const double absoff = -(A.diag64[i] + in);   // the couplings are negative
  const Rec4 p = load_rec4(A.sp4, i);
  const rt_f64x2_t vd = load_pair(A.VD, i);
  double suma = 0.0, gsum = 0.0;
  for (int64_t k = A.ptr[i] + A.nint[i]; k < A.ptr[i + 1]; ++k) {
    const int32_t j = A.idx[k];
    const Rec4 q = load_rec4(A.sp4, j);
    const rt_f64x2_t vj = load_pair(A.VD, j);
    const double dx = periodic_disp(p.x - q.x, A.box, 0);
    const double dy = periodic_disp(p.y - q.y, A.box, 1);
    const double dz = DIM == 3 ? periodic_disp(p.z - q.z, A.box, 2) : 0.0;
    const double r = sqrt(dx * dx + dy * dy + dz * dz);
    const double F = -0.5 * (sph_dwdr<DIM>(r, p.h, kernel) + sph_dwdr<DIM>(r, q.h, kernel)) / r;
    const double aij = vj[0] * (vd[1] + vj[1]) * F;
    suma += aij;
    gsum += aij * A.Eall[j];
  }
  const double d = vd[0] * (1.0 / dt + c * A.sa[i] * A.f[i]) + (absoff + vd[0] * suma);
  A.diag64[i] = d;
  A.dinv64[i] = 1.0 / d;
  A.sinv64[i] = 1.0 / (d + absoff);
  if (A.diag32) {
    A.diag32[i] = (float)d;
    A.dinv32[i] = (float)(1.0 / d);
    A.sinv32[i] = (float)(1.0 / (d + absoff));
  }
  A.g[i] = vd[0] * gsum;
}

// r = b - (r + the sums earlier tiles left) with the residual product's block
// partials and weights (see k_spmv)
__global__ void __launch_bounds__(kBlock)
k_pair_resid(int64_t n, PairIn P, const double* __restrict__ xsum, const double* __restrict__ x,
             const double* __restrict__ b, const double* __restrict__ diag,
             double* __restrict__ r, float* __restrict__ r32, float* __restrict__ w32,
             double* __restrict__ part, double* __restrict__ pmax,
             const int32_t* __restrict__ tprob, const int32_t* __restrict__ skip) {
  __shared__ double red[kBlock / kWave];
  if (skip && skip[tprob ? tprob[blockIdx.x] : 0]) return;   // a finished problem's tile
  const int64_t i = blockIdx.x * (int64_t)kTileRows + threadIdx.x;
  double rr = 0.0, cw = 0.0;
  if (i < n) {
    const double ri = b[i] - (r[i] + pair_in<double>(P, i, xsum));
    r[i] = ri;
    if (r32) r32[i] = (float)ri;
    rr = ri * ri;
    const double xi = x[i], di = diag[i];
    cw = cw_term(ri, di, xi);
    if (w32) w32[i] = cw_weight(di, xi);
  }
  rr = block_sum(rr, red);
  cw = block_max(cw, red);
  if (threadIdx.x == 0) {
    part[blockIdx.x] = rr;
    if (pmax) pmax[blockIdx.x] = cw;
  }
}

// ---- CSR rows from the pair form ------------------------------------------------
// For levels without neighbour lists (a batch) whose caller asks for a plain
// shape.  One block per tile; FILL: the entries of both rows of a pair at their
// rows' next free places (the rows are sorted afterwards), else their numbers.
// Made once per batch at most, so the rows' counters are global atomics.
template <bool FILL>
__global__ void __launch_bounds__(kBlock)
k_pair_rows(PairArgs A, const double* __restrict__ val, const int64_t* __restrict__ rp,
            int32_t* __restrict__ cnt, int32_t* __restrict__ col, double* __restrict__ out) {
  const int64_t t = blockIdx.x, r0 = t * kTileRows, x0 = A.xoff[t];
  const int ncol = kTileRows + (int)(A.xoff[t + 1] - x0);
  const int64_t g0 = A.goff[t];
  const int ng = A.gcnt[t];
  const double* v = val + 4 * g0;   // two planes: entries 0-1 of every group, entries 2-3
  for (int g = threadIdx.x; g < ng; g += kBlock) {
    const int64_t i = r0 + A.row[g0 + g];
    for (int q = 0; q < 4; ++q) {
      const int c = A.col[4 * (g0 + g) + q];
      if (c >= ncol) continue;   // the filling of a row's last group
      const int64_t j = c < kTileRows ? r0 + c : A.xcol[x0 + c - kTileRows];
      const int a = atomicAdd(&cnt[i], 1), b = atomicAdd(&cnt[j], 1);
      if (FILL) {
        const double w = v[2 * (q < 2 ? g : ng + g) + (q & 1)];
        col[rp[i] + a] = (int32_t)j;
        out[rp[i] + a] = w;
        col[rp[j] + b] = (int32_t)i;
        out[rp[j] + b] = w;
      }
    }
  }
}

__global__ void k_pair_to_f32(int64_t n, const double* __restrict__ a, float* __restrict__ b) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) b[i] = (float)a[i];
}

}  // namespace

int pair_rows(rt_ctx* ctx, Level& L, bool fp32) {
  hipStream_t st = ctx->stream;
  const int64_t n = L.n;
  DevBuf<int32_t> cnt;
  RT_CHECK(cnt.reserve(n + 1));
  RT_CHECK(L.rp.reserve(n + 1));
  RT_CHECK(L.col.reserve(std::max<int64_t>(L.nnz, 1)));
  RT_CHECK(L.val64.reserve(L.nnz + kSpmvPad));
  if (fp32) RT_CHECK(L.val32.reserve(L.nnz + kSpmvPad));
  const dim3 tiles((unsigned)L.pair.ntiles);
  for (int fill = 0; fill < 2; ++fill) {
    hipLaunchKernelGGL(k_zero_i32, dim3(grid_for(n + 1)), dim3(kBlock), 0, st, n + 1, cnt.p);
    if (fill)
      hipLaunchKernelGGL(k_pair_rows<true>, tiles, dim3(kBlock), 0, st, L.pair.args(),
                         L.pair.val64.p, L.rp.p, cnt.p, L.col.p, L.val64.p);
    else
      hipLaunchKernelGGL(k_pair_rows<false>, tiles, dim3(kBlock), 0, st, L.pair.args(),
                         L.pair.val64.p, nullptr, cnt.p, nullptr, nullptr);
    RT_LAUNCH_CHECK();
    if (!fill) RT_CHECK((scan<int32_t, int64_t>(ctx, cnt.p, L.rp.p, n + 1, false)));
  }
  RT_CHECK((row_sort<int32_t, double>(ctx, L.rp.p, L.col.p, L.val64.p, n)));
  if (fp32) {
    hipLaunchKernelGGL(k_pair_to_f32, dim3(grid_for(L.nnz)), dim3(kBlock), 0, st, L.nnz, L.val64.p,
                       L.val32.p);
    RT_LAUNCH_CHECK();
  }
  L.csr_rows = L.csr_vals = true;
  return RT_OK;
}

int build_pairs(rt_ctx* ctx, const rt_neighbors* nb, Level& L, bool* no_tiles) {
  hipStream_t st = ctx->stream;
  PairForm& P = L.pair;
  P.on = false;
  const int64_t n = nb->n_interior;
  const int64_t nt = (n + kTileRows - 1) / kTileRows;
  if (n == 0 || nt >= ((int64_t)1 << 24)) return RT_OK;
  const int64_t groups = (nb->npairs >> 2) + n + 1;   // an upper bound (first_group)
  for (auto* b : {&P.goff, &P.xoff}) RT_CHECK(b->reserve(nt + 1));
  RT_CHECK(P.gcnt.reserve(nt));
  RT_CHECK(P.col.reserve((size_t)4 * groups));
  RT_CHECK(P.row.reserve(groups));
  DevBuf<int32_t> bid, nblk, nseg, recv;
  DevBuf<PairSeg> seg;
  DevBuf<uint64_t> bmask;
  DevBuf<PairStat> stat;
  DevBuf<PairTotals> totals;
  RT_CHECK(bid.reserve((size_t)nt * kPairBlocks));
  RT_CHECK(bmask.reserve((size_t)nt * kPairBlocks));
  for (auto* b : {&nblk, &nseg, &recv}) RT_CHECK(b->reserve(nt));
  RT_CHECK(stat.reserve(nt));
  RT_CHECK(totals.reserve(1));
  hipLaunchKernelGGL(k_pair_build, dim3((unsigned)nt), dim3(kBlock), 0, st, n, nb->ptr.p,
                     nb->n_int_nbrs.p, nb->idx.p, P.goff.p, P.gcnt.p, P.col.p, P.row.p, bid.p, bmask.p,
                     nblk.p, stat.p);
  hipLaunchKernelGGL(k_pair_scan, dim3(1), dim3(kScanThreads), 0, st, nt, stat.p, P.xoff.p,
                     totals.p);
  hipLaunchKernelGGL(k_zero_i32, dim3(grid_for(nt)), dim3(kBlock), 0, st, nt, nseg.p);
  RT_LAUNCH_CHECK();
  RT_CHECK(ctx->sync_read(totals.p, sizeof(PairTotals)));
  PairTotals tot;
  std::memcpy(&tot, ctx->host, sizeof(tot));
  if (tot.bad || tot.ext >= INT32_MAX) {
    *no_tiles = tot.bad == 2;
    P = PairForm();   // the columns and offsets go back to the cache
    return RT_OK;
  }
  L.n = n;
  L.nnz = tot.nnz;
  L.max_row = tot.max_row;
  L.tile_cols_total = tot.distinct;
  P.ntiles = nt;
  P.ext_total = tot.ext;
  P.max_ext = tot.max_ext;
  RT_CHECK(P.xcol.reserve(tot.ext));
  RT_CHECK(P.in_ptr.reserve(n + 1));
  RT_CHECK(P.in_pos.reserve(tot.ext));
  RT_CHECK(seg.reserve((size_t)nt * kPairSegs));
  hipLaunchKernelGGL(k_pair_lists, dim3((unsigned)nt), dim3(kBlock), 0, st, nblk.p, bid.p, bmask.p,
                     P.xoff.p, P.xcol.p, nseg.p, seg.p);
  hipLaunchKernelGGL(k_pair_sort, dim3((unsigned)nt), dim3(kWave), 0, st, nseg.p, seg.p, recv.p);
  hipLaunchKernelGGL(k_pair_offsets, dim3(1), dim3(kScanThreads), 0, st, nt, recv.p);
  hipLaunchKernelGGL(k_pair_recv, dim3((unsigned)nt), dim3(kBlock), 0, st, n, (int32_t)tot.ext,
                     recv.p, nseg.p, seg.p, P.in_ptr.p, P.in_pos.p);
  RT_LAUNCH_CHECK();
  P.on = true;
  return RT_OK;
}

int assemble_pairs(rt_ctx* ctx, rt_matrix* A) {
  hipStream_t st = ctx->stream;
  const rt_neighbors* nb = A->nb;
  Level& L = A->levels[0];
  PairForm& P = L.pair;
  const int64_t n = L.n;
  const bool fp32 = A->amg.build_fp32 != 0;
  const int64_t values = 4 * ((nb->npairs >> 2) + n + 1);
  RT_CHECK(P.val64.reserve(values));
  RT_CHECK(P.sum64.reserve(P.ext_total));
  for (auto* b : {&L.diag64, &L.dinv64, &L.sinv64}) RT_CHECK(b->reserve(n));
  if (fp32) {
    RT_CHECK(P.val32.reserve(values));
    RT_CHECK(P.sum32.reserve(P.ext_total));
    for (auto* b : {&L.diag32, &L.dinv32, &L.sinv32}) RT_CHECK(b->reserve(n));
  }
  A->has_fp32 = fp32;   // the buffers exist
  L.csr_vals = false;
  const size_t lds = sizeof(PairRec) * (size_t)(kTileRows + P.max_ext);
  DiagArgs da{nb->ptr.p, nb->n_int_nbrs.p, nb->idx.p, nb->sp4.p, A->VD.p, A->sa.p, A->f.p,
              A->Eall.p, L.diag64.p, L.dinv64.p, L.sinv64.p, A->g.p, fp32 ? L.diag32.p : nullptr,
              fp32 ? L.dinv32.p : nullptr, fp32 ? L.sinv32.p : nullptr, nb->box};
#define RT_PAIR_VALUES(D_)                                                                       \
  hipLaunchKernelGGL((k_pair_values<D_>), dim3((unsigned)P.ntiles), dim3(kValBlock), lds, st, n,  \
                     nb->kernel, P.args(), nb->sp4.p, A->VD.p, nb->box, P.val64.p,                \
                     fp32 ? P.val32.p : nullptr)
#define RT_PAIR_DIAG(D_)                                                                          \
  hipLaunchKernelGGL((k_pair_diag<D_>), dim3((unsigned)P.ntiles), dim3(kBlock), 0, st, n,          \
                     nb->kernel, A->dt, A->c, da, P.in(), P.sum64.p)
  if (nb->dim == 3) RT_PAIR_VALUES(3);
  else RT_PAIR_VALUES(2);
  RT_LAUNCH_CHECK();
  RT_CHECK((launch_pair<double, PP_ONES>(st, L, nullptr, nullptr, L.diag64.p, nullptr, nullptr)));
  if (nb->dim == 3) RT_PAIR_DIAG(3);
  else RT_PAIR_DIAG(2);
#undef RT_PAIR_VALUES
#undef RT_PAIR_DIAG
  RT_LAUNCH_CHECK();
  return RT_OK;
}

int pair_resid(rt_ctx* ctx, const Level& L, const double* x, const double* b, double* r,
               float* r32, float* w32, double* part, double* pmax, int* nparts, int shape,
               const int32_t* tprob, const int32_t* skip) {
  RT_CHECK((launch_pair<double, PP_PLAIN>(ctx->stream, L, L.diag64.p, x, r, nullptr, nullptr,
                                          shape, tprob, skip)));
  hipLaunchKernelGGL(k_pair_resid, dim3((unsigned)L.pair.ntiles), dim3(kBlock), 0, ctx->stream,
                     L.n, L.pair.in(), L.pair.sum64.p, x, b, L.diag64.p, r, r32, w32, part, pmax, tprob,
                     skip);
  RT_LAUNCH_CHECK();
  *nparts = (int)L.pair.ntiles;
  return RT_OK;
}

}  // namespace rt

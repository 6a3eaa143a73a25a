// Reordering of particle sets whose order bears no relation to the wanted one:
// the first sort of freshly loaded particles, and the export to the original
// order.
//
// Moving a random permutation element by element writes every value into a
// cache line of its own: at 67M float32 particles the first sort took 34 ms
// and the export 33 ms for 3 and 9 GB.  Both go through an intermediate order
// in the other particle set, which is free between sorts.  A workgroup of the
// split pass groups its particles by bucket in LDS and writes one contiguous
// run per bucket and array (k_split): for the sort first by tile, then by cell
// inside each tile; for the export by runs of 2^shift original indices, whose
// values one workgroup then puts in place in LDS (k_bucket_export).
#include "particle_math.h"

#include <algorithm>
#include <type_traits>

namespace pic {

namespace {

constexpr int kSplitThreads = kSplitWidth;
// particles per thread when an array of the set has less than kSplitMany bytes:
// a set of 1M float32 particles then makes 512 workgroups instead of 128 (first
// sort 116 instead of 142 us); from 2M on the longer runs are worth more (167
// instead of 235 us)
constexpr int kSplitFew = 4;
constexpr int64_t kSplitMany = 1 << 23;

// the instance and local block of a flattened block, or instance `only` (a
// launch over that instance alone)
__device__ __forceinline__ const InstDesc& split_inst(const InstDesc* __restrict__ D, int ninst, int only, int b,
                                                      int& lb) {
  const int ii = only >= 0 ? only : find_inst(D, ninst, BK_SPLIT, b);
  lb = only >= 0 ? b : b - D[ii].blk[BK_SPLIT];
  return D[ii];
}

// bucket of a particle: by = -1: the tile group of its position; -2: its cell
// key; by >= 0: its original index >> by
template <typename T>
__device__ __forceinline__ int bucket_of(const InstDesc& d, const TileP& tp, int set, int64_t i, int by) {
  if (by >= 0) return gp((const int32_t*)d.ids[set])[i] >> by;
  const int c = cell_key(gp((const T*)d.set[set][0])[i], gp((const T*)d.set[set][1])[i], d.g, tp);
  return by == -2 ? c : c >> (2 * tp.log_ts + tp.log_group);
}

// particles per tile bucket (added to tb.bcount, zero between uses)
template <typename T, int NI>
__global__ void __launch_bounds__(kSplitThreads) k_bucket_count(const InstDesc* __restrict__ D, int ninst, int set) {
  __shared__ int hist[kMaxBuckets];
  int lb;
  const InstDesc& d = split_inst(D, ninst, -1, blockIdx.x, lb);
  const TileP tp = d.tp;
  for (int b = threadIdx.x; b < kMaxBuckets; b += kSplitThreads) hist[b] = 0;
  __syncthreads();
  const int64_t base = (int64_t)lb * NI * kSplitThreads;
#pragma unroll
  for (int k = 0; k < NI; ++k) {
    const int64_t i = base + k * kSplitThreads + threadIdx.x;
    if (i < d.n) atomicAdd(&hist[bucket_of<T>(d, tp, set, i, -1)], 1);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < kMaxBuckets; b += kSplitThreads)
    if (hist[b]) gadd(gp(d.tb.bcount) + b, hist[b]);
}

// exclusive scan of v over the workgroup's kMaxBuckets values (two per thread)
__device__ __forceinline__ void scan_buckets(int (&v)[2], int* wave_sums) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int own = v[0] + v[1];
  int inc = own;
  for (int off = 1; off < 64; off <<= 1) {
    const int u = __shfl_up(inc, off);
    if (lane >= off) inc += u;
  }
  if (lane == 63) wave_sums[wave] = inc;
  __syncthreads();
  int before = 0;
  for (int w = 0; w < kSplitThreads / 64; ++w) before += w < wave ? wave_sums[w] : 0;
  v[1] = before + inc - v[1];      // exclusive
  v[0] = before + inc - own;
}

// first slot of every bucket into tb.bcursor: from the counts (which return
// to zero), or b << by for buckets of original indices, which are all full
__global__ void __launch_bounds__(kSplitThreads) k_bucket_start(const InstDesc* __restrict__ D, int only, int by) {
  static_assert(kMaxBuckets == 2 * kSplitThreads, "two buckets per thread");
  __shared__ int wave_sums[kSplitThreads / 64];
  const InstDesc& d = D[only >= 0 ? only : blockIdx.x];
  const int b0 = 2 * threadIdx.x;
  int v[2] = {b0 << max(by, 0), (b0 + 1) << max(by, 0)};
  if (by < 0) {
    v[0] = d.tb.bcount[b0];
    v[1] = d.tb.bcount[b0 + 1];
    scan_buckets(v, wave_sums);
    d.tb.bcount[b0] = d.tb.bcount[b0 + 1] = 0;
  }
  d.tb.bcursor[b0] = v[0];
  d.tb.bcursor[b0 + 1] = v[1];
}

// cells a workgroup of the cell passes covers in LDS: from the first cell of
// its first particle's tile on
__device__ __forceinline__ int first_cell(int cell, const TileP& tp) { return cell >> (2 * tp.log_ts) << (2 * tp.log_ts); }

// Cell histogram of a set grouped by tile (tb.ccount), counted in LDS; a
// particle beyond the workgroup's LDS cells counts by itself.
template <typename T, int NI>
__global__ void __launch_bounds__(kSplitThreads) k_cell_count(const InstDesc* __restrict__ D, int ninst, int set) {
  __shared__ int hist[kMaxBuckets];
  int lb;
  const InstDesc& d = split_inst(D, ninst, -1, blockIdx.x, lb);
  const TileP tp = d.tp;
  const GridP g = d.g;
  const gptr<const T> px = gp((const T*)d.set[set][0]), py = gp((const T*)d.set[set][1]);
  const gptr<int32_t> ccount = gp(d.tb.ccount);
  const int64_t base = (int64_t)lb * NI * kSplitThreads;
  if (base >= d.n) return;  // whole workgroup
  const int c0 = first_cell(cell_key(px[base], py[base], g, tp), tp);
  for (int b = threadIdx.x; b < kMaxBuckets; b += kSplitThreads) hist[b] = 0;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NI; ++k) {
    const int64_t i = base + k * kSplitThreads + threadIdx.x;
    if (i < d.n) {
      const int c = cell_key(px[i], py[i], g, tp);
      if ((unsigned)(c - c0) < (unsigned)kMaxBuckets)
        atomicAdd(&hist[c - c0], 1);
      else
        gadd(ccount + c, 1);
    }
  }
  __syncthreads();
  for (int b = threadIdx.x; b < kMaxBuckets; b += kSplitThreads)
    if (hist[b]) gadd(ccount + c0 + b, hist[b]);
}

// tb.ccount back to zero (BK_TILES blocks, one wave per tile)
__global__ void __launch_bounds__(256) k_cell_zero(const InstDesc* __restrict__ D, int ninst) {
  const int ii = find_inst(D, ninst, BK_TILES, blockIdx.x);
  const InstDesc& d = D[ii];
  const int t = (blockIdx.x - d.blk[BK_TILES]) * 4 + (threadIdx.x >> 6);
  if (t >= d.tp.ntiles) return;
  const int cells = d.tp.ts * d.tp.ts;
  for (int j = threadIdx.x & 63; j < cells; j += 64) gp(d.tb.ccount)[(size_t)t * cells + j] = 0;
}

// Set src into set src ^ 1, grouped by bucket.  A workgroup ranks its particles
// by bucket with LDS counters, takes a run of slots per bucket, and passes each
// array through LDS so that neighbouring lanes write a run.  Memory-bound: 48
// bytes read and written per float32 particle; 67M particles in 1024 buckets
// (runs of eight) 3.0 ms.
// BY_TILE, BY_ID: slots from tb.bcursor.  BY_CELL: the source is grouped by
// tile and the destination is the sorted order (the cell scan's offsets plus
// tb.ccount as the running counter, to be zeroed again); a particle beyond the
// workgroup's LDS cells moves by itself.
enum { BY_TILE = 0, BY_ID = 1, BY_CELL = 2 };

template <typename T, int BY, int NI>
__global__ void __launch_bounds__(kSplitThreads) k_split(const InstDesc* __restrict__ D, int ninst, int only, int src,
                                                         int shift) {
  constexpr int NP = NI * kSplitThreads;
  __shared__ int hist[kMaxBuckets], offs[kMaxBuckets], first[kMaxBuckets];
  __shared__ int wave_sums[kSplitThreads / 64];
  __shared__ __align__(16) T stage[NP];
  int lb;
  const InstDesc& d = split_inst(D, ninst, only, blockIdx.x, lb);
  const TileP tp = d.tp;
  const int64_t base = (int64_t)lb * NP;
  if (base >= d.n) return;  // whole workgroup
  const int count = (int)min((int64_t)NP, d.n - base);
  const int tile_bits = 2 * tp.log_ts;
  const gptr<const int32_t> start = gp((const int32_t*)d.tb.start), ccursor = gp((const int32_t*)d.tb.ccursor);
  int c0 = 0;
  if (BY == BY_CELL) c0 = first_cell(bucket_of<T>(d, tp, src, base, -2), tp);
  for (int b = threadIdx.x; b < kMaxBuckets; b += kSplitThreads) hist[b] = 0;
  __syncthreads();
  // key: the bucket; BY_CELL: >= kMaxBuckets for a particle beyond the LDS cells
  int key[NI], slot[NI];
#pragma unroll
  for (int k = 0; k < NI; ++k) {
    const int j = k * kSplitThreads + threadIdx.x;
    key[k] = kMaxBuckets;
    slot[k] = -1;  // moves by itself, or past the end
    if (j < count) {
      key[k] = BY == BY_CELL ? bucket_of<T>(d, tp, src, base + j, -2) - c0
                             : bucket_of<T>(d, tp, src, base + j, BY == BY_ID ? shift : -1);
      if ((unsigned)key[k] < (unsigned)kMaxBuckets) slot[k] = atomicAdd(&hist[key[k]], 1);
    }
  }
  __syncthreads();
  {
    const int b0 = 2 * threadIdx.x;
    int v[2] = {hist[b0], hist[b0 + 1]};
    const int cnt[2] = {v[0], v[1]};
    scan_buckets(v, wave_sums);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      offs[b0 + u] = v[u];
      if (!cnt[u]) continue;
      const int c = c0 + b0 + u;
      const gptr<int32_t> ctr = gp(BY == BY_CELL ? d.tb.ccount + c : d.tb.bcursor + b0 + u);
      first[b0 + u] = __hip_atomic_fetch_add(ctr, cnt[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) +
                      (BY == BY_CELL ? start[c >> tile_bits] + ccursor[c] : 0);
    }
  }
  __syncthreads();
  // slot in the workgroup's bucket order, and through LDS the destination of
  // each slot this thread will write
  int32_t* st32 = reinterpret_cast<int32_t*>(stage);
  // slots of the LDS order in use: all of the workgroup's but those that move by themselves
  const int staged = offs[kMaxBuckets - 1] + hist[kMaxBuckets - 1];
#pragma unroll
  for (int k = 0; k < NI; ++k) {
    const int j = k * kSplitThreads + threadIdx.x;
    if (j >= count) continue;
    const int c = c0 + key[k];
    int o;
    if (slot[k] >= 0) {
      o = first[key[k]] + slot[k];
      slot[k] += offs[key[k]];
      st32[slot[k]] = o;
    } else {
      o = start[c >> tile_bits] + ccursor[c] +
          __hip_atomic_fetch_add(gp(d.tb.ccount) + c, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (BY == BY_CELL) {
      // a chunk's first and last particles record its span of cell rows, as in the sort's scatter
      const int tt = c >> tile_bits, t0 = start[tt], rel = o - t0;
      const int sz = gp((const int32_t*)d.tb.csize)[tt];
      const int jc = (int)((uint32_t)rel / (uint32_t)sz), in_chunk = rel - jc * sz;
      const bool fst = in_chunk == 0;
      const bool lst = in_chunk == sz - 1 || rel == start[tt + 1] - t0 - 1;
      if (fst || lst) {
        const int row = (c & ((1 << tile_bits) - 1)) >> tp.log_ts;
        const gptr<int> rows = gp(reinterpret_cast<int*>(d.tb.work + d.tb.cstart[tt] + jc) + 3);
        if (fst) __hip_atomic_fetch_or(rows, row, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (lst) __hip_atomic_fetch_or(rows, row << 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    key[k] = o;  // the destination of a particle that moves by itself
  }
  __syncthreads();
  int dst[NI];
#pragma unroll
  for (int k = 0; k < NI; ++k) dst[k] = st32[k * kSplitThreads + threadIdx.x];
  auto move = [&](auto* from, auto* to, auto* lds) {
    using V = std::remove_cv_t<std::remove_pointer_t<decltype(lds)>>;
    const gptr<const V> s = gp((const V*)from) + base;
    const gptr<V> o = gp((V*)to);
    V v[NI];
#pragma unroll
    for (int k = 0; k < NI; ++k) {
      const int j = k * kSplitThreads + threadIdx.x;
      if (j < count) v[k] = s[j];
    }
    __syncthreads();  // the previous array has left LDS
#pragma unroll
    for (int k = 0; k < NI; ++k) {
      if (k * kSplitThreads + (int)threadIdx.x >= count) continue;
      if (BY != BY_CELL || slot[k] >= 0)
        lds[slot[k]] = v[k];
      else
        o[key[k]] = v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NI; ++k) {
      const int j = k * kSplitThreads + threadIdx.x;
      if (j < staged) o[dst[k]] = lds[j];
    }
  };
  for (int a = 0; a < 11; ++a) move(d.set[src][a], d.set[src ^ 1][a], stage);
  move(d.ids[src], d.ids[src ^ 1], st32);
}

// out[a n + id] = array a of a set split by original index (float64, original
// order): one workgroup per array and window of 2^log_win original indices
// puts the window's values in place in LDS and writes them out in order.
// Reads 4 + 4 and writes 8 bytes per float32 value; bound by the reads in
// flight, so eight of each are issued before the first is used.
template <typename T>
__global__ void __launch_bounds__(1024) k_bucket_export(Parts<T> p, int64_t n, int shift, int log_win,
                                                        double* __restrict__ out) {
  constexpr int U = 8;
  extern __shared__ __align__(16) unsigned char smem[];
  T* win = reinterpret_cast<T*>(smem);
  const int bb = xcd_contiguous(blockIdx.x, gridDim.x);  // a bucket's windows and arrays on one XCD
  const int w = bb & ((1 << (shift - log_win)) - 1), rest = bb >> (shift - log_win);
  const int bucket = rest / 11, a = rest - bucket * 11;
  const T* src = a == 0 ? p.x : a == 1 ? p.y : a < 5 ? p.P[a - 2] : a < 8 ? p.v[a - 5] : p.w[a - 8];
  const int64_t b0 = (int64_t)bucket << shift, lo = b0 + ((int64_t)w << log_win);
  const int count = (int)min((int64_t)1 << shift, n - b0);
  const int len = (int)min((int64_t)1 << log_win, n - lo);  // <= 0: a window past the end
  const gptr<const T> s = gp(src) + b0;
  const gptr<const int32_t> id = gp((const int32_t*)p.id) + b0;
  for (int k0 = threadIdx.x; k0 < count; k0 += 1024 * U) {
    T v[U];
    int at[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = k0 + u * 1024;
      at[u] = -1;
      if (k < count) {
        at[u] = (int)(id[k] - lo);
        v[u] = s[k];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if ((unsigned)at[u] < (unsigned)max(len, 0)) win[at[u]] = v[u];
  }
  __syncthreads();
  const gptr<double> o = gp(out + (int64_t)a * n + lo);
  for (int k = threadIdx.x; k < len; k += 1024) o[k] = (double)win[k];
}

}  // namespace

template <typename T, int NI>
static hipError_t first_sort(const InstDesc* D, int ninst, int nb_split, int nb_tiles, int src, hipStream_t s) {
  const dim3 grid(nb_split), th(kSplitThreads);
  hipLaunchKernelGGL((k_bucket_count<T, NI>), grid, th, 0, s, D, ninst, src);
  hipLaunchKernelGGL(k_bucket_start, dim3(ninst), th, 0, s, D, -1, -1);
  hipLaunchKernelGGL((k_split<T, BY_TILE, NI>), grid, th, 0, s, D, ninst, -1, src, 0);
  hipLaunchKernelGGL((k_cell_count<T, NI>), grid, th, 0, s, D, ninst, src ^ 1);
  hipError_t e = launch_cell_scan(D, ninst, nb_tiles, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_split<T, BY_CELL, NI>), grid, th, 0, s, D, ninst, -1, src ^ 1, 0);
  hipLaunchKernelGGL(k_cell_zero, dim3(nb_tiles), dim3(256), 0, s, D, ninst);
  return hipGetLastError();
}

// the most particles per thread whose staging is 32 KB, or few enough that a
// smaller set still fills the chip
int split_items(int64_t n, int es) { return n * es < kSplitMany ? kSplitFew : 64 / es; }

hipError_t launch_first_sort(int dtype, const InstDesc* D, int ninst, int items, int nb_split, int nb_tiles, int src,
                             hipStream_t s) {
  auto* fn = dtype == PIC_F32 ? (items == kSplitFew ? first_sort<float, kSplitFew> : first_sort<float, 16>)
                              : (items == kSplitFew ? first_sort<double, kSplitFew> : first_sort<double, 8>);
  return fn(D, ninst, nb_split, nb_tiles, src, s);
}

template <typename T, int NI>
static hipError_t export_split(const InstDesc* D, int inst, int64_t n, int src, const Parts<T>& split, double* out,
                               hipStream_t s) {
  constexpr int np = NI * kSplitThreads;
  // windows of 64 KB while their buckets suffice, then 128 KB; buckets of more
  // than one window only when there would be too many
  int log_win = sizeof(T) == 4 ? 14 : 13;
  if ((n - 1) >> log_win >= kMaxBuckets) ++log_win;
  int shift = log_win;
  while ((n - 1) >> shift >= kMaxBuckets) ++shift;
  const int64_t nbuckets = ((n - 1) >> shift) + 1;
  const dim3 egrid((unsigned)(nbuckets * 11 << (shift - log_win)));
  const int lds = (int)sizeof(T) << log_win;
  (void)hipFuncSetAttribute((const void*)k_bucket_export<T>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  hipLaunchKernelGGL(k_bucket_start, dim3(1), dim3(kSplitThreads), 0, s, D, inst, shift);
  hipLaunchKernelGGL((k_split<T, BY_ID, NI>), dim3((unsigned)((n + np - 1) / np)), dim3(kSplitThreads), 0, s, D, 0,
                     inst, src, shift);
  hipLaunchKernelGGL(k_bucket_export<T>, egrid, dim3(1024), lds, s, split, n, shift, log_win, out);
  return hipGetLastError();
}

hipError_t launch_export(int dtype, const InstDesc* D, int inst, int64_t n, int src, const void* split_parts,
                         double* out, hipStream_t s) {
  const bool few = split_items(n, dtype == PIC_F32 ? 4 : 8) == kSplitFew;
  if (dtype == PIC_F32) {
    const Parts<float>& p = *(const Parts<float>*)split_parts;
    return few ? export_split<float, kSplitFew>(D, inst, n, src, p, out, s)
               : export_split<float, 16>(D, inst, n, src, p, out, s);
  }
  const Parts<double>& p = *(const Parts<double>*)split_parts;
  return few ? export_split<double, kSplitFew>(D, inst, n, src, p, out, s)
             : export_split<double, 8>(D, inst, n, src, p, out, s);
}

}  // namespace pic

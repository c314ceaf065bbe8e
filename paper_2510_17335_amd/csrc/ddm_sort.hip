// Binning of particles: exact integer cell keys from the stored positions, the
// stable sort by key, the state gather into sorted order, and the list of
// occupied tiles that the scatter kernels work on.  Two ways to the same
// order: a least-significant-digit radix sort (8-bit digits, wave64 ballot
// ranking), and a two-level counting sort (by tile with counters, inside a
// tile in LDS) in four or five launches, described below.
//
// Key of a live particle: inst * (n^D + 1) + tile * B^D + cell-in-tile, with
// tile and cell-in-tile lexicographic in (x, y[, z]) (last axis fastest) and
// B = kTile.  Padding slots get inst * (n^D + 1) + n^D, so every instance keeps
// its slot range and its padding stays at the end of it.
#include <hip/hip_runtime.h>

#include "ddm_kernels.hpp"

namespace ddm {

constexpr int kSortItems = 8;                       // keys per thread in a sort block
constexpr int kSortBlockKeys = kBlock * kSortItems; // 2048

// Base cell of one axis from a stored position (same rule as the stencil).
__device__ __forceinline__ bool cell_f32(uint32_t xr, const KCfg& c, int& base) {
  const uint64_t q = (uint64_t)xr << c.nlog2;
  if (q < 0x80000000ull) { base = 0; return false; }
  const uint64_t b = (q - 0x80000000ull) >> 32;
  if (b > (uint64_t)(c.n - 3)) { base = c.n - 3; return false; }
  base = (int)b;
  return true;
}
__device__ __forceinline__ bool cell_f64(double xr, const KCfg& c, int& base) {
  const double bf = floor(xr * c.inv_dx - 0.5);
  if (!(bf >= 0.0)) { base = 0; return false; }
  if (!(bf <= (double)(c.n - 3))) { base = c.n - 3; return false; }
  base = (int)bf;
  return true;
}

template <int PREC>
__global__ void k_keys(KCfg c, const int* blk_inst, const InstDev* inst, const void* state, uint32_t* keys,
                       uint32_t* vals, DevErr* err, const uint32_t* order) {
  const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const int64_t p = order ? (int64_t)order[j] : j;
  const int i = blk_inst[p / kBlock];
  const InstDev& I = inst[i];
  const uint32_t cells = (uint32_t)c.nodes;
  uint32_t key = (uint32_t)i * (cells + 1u) + cells;
  if (p - I.off < I.n) {
    const int nt = c.n / kTile;
    uint32_t t = 0, cl = 0;
    bool ok = true;
    for (int a = 0; a < c.dim; ++a) {
      int b;
      if (PREC == 0) ok &= cell_f32(static_cast<const uint32_t*>(state)[(int64_t)a * c.ntot + p], c, b);
      else ok &= cell_f64(static_cast<const double*>(state)[(int64_t)a * c.ntot + p], c, b);
      t = t * nt + b / kTile;
      cl = cl * kTile + b % kTile;
    }
    if (!ok) atomicOr(&err->flags, 2u);
    const uint32_t tcells = c.dim == 3 ? kTile * kTile * kTile : kTile * kTile;
    key = (uint32_t)i * (cells + 1u) + t * tcells + cl;
  }
  keys[j] = key;
  vals[j] = (uint32_t)p;
}

void launch_keys(int prec, const KCfg& c, const Bufs& b, int nblk, const void* state, uint32_t* keys, uint32_t* vals,
                 hipStream_t s, const uint32_t* order) {
  if (prec == 0) hipLaunchKernelGGL(k_keys<0>, dim3(nblk), dim3(kBlock), 0, s, c, b.blk_inst, b.inst, state, keys, vals, b.err, order);
  else hipLaunchKernelGGL(k_keys<1>, dim3(nblk), dim3(kBlock), 0, s, c, b.blk_inst, b.inst, state, keys, vals, b.err, order);
}

// Keys of the deterministic mode's first sort: the particle id (padding slots
// last), so that a stable sort by cell afterwards orders a cell's particles by id.
__global__ void k_pid_keys(const uint32_t* pid, uint32_t* keys, uint32_t* vals, int64_t ntot) {
  const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (p >= ntot) return;
  const uint32_t id = pid[p];
  keys[p] = id == 0xFFFFFFFFu ? (uint32_t)ntot : id;
  vals[p] = (uint32_t)p;
}

void launch_pid_keys(const uint32_t* pid, uint32_t* keys, uint32_t* vals, int64_t ntot, hipStream_t s) {
  hipLaunchKernelGGL(k_pid_keys, dim3((unsigned)((ntot + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, pid, keys, vals,
                     ntot);
}

// ---------------------------------------------------------------------------
// Radix sort pass: digit histogram per block, exclusive scan over
// hist[digit][block], stable scatter.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(kBlock) k_radix_hist(const uint32_t* keys, int64_t n, int shift, uint32_t* hist,
                                                       int nsb) {
  __shared__ uint32_t h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kSortBlockKeys;
  for (int k = 0; k < kSortItems; ++k) {
    const int64_t e = base + (int64_t)k * kBlock + threadIdx.x;
    if (e < n) atomicAdd(&h[(keys[e] >> shift) & 255u], 1u);
  }
  __syncthreads();
  hist[(int64_t)threadIdx.x * nsb + blockIdx.x] = h[threadIdx.x];
}

// Exclusive scan of a uint32 array in three launches (block scan, scan of
// block totals, add).  Block = 256 threads x 8 items.
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* total) {
  __shared__ uint32_t ws[kBlock / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) ws[wid] = x;
  __syncthreads();
  uint32_t off = 0, tot = 0;
  for (int w = 0; w < kBlock / 64; ++w) {
    if (w < wid) off += ws[w];
    tot += ws[w];
  }
  __syncthreads();
  *total = tot;
  return off + x - v;
}

__global__ void __launch_bounds__(kBlock) k_scan_local(uint32_t* a, int64_t n, uint32_t* sums) {
  const int64_t base = (int64_t)blockIdx.x * kSortBlockKeys + (int64_t)threadIdx.x * kSortItems;
  uint32_t v[kSortItems], s = 0;
  for (int k = 0; k < kSortItems; ++k) {
    v[k] = base + k < n ? a[base + k] : 0u;
    s += v[k];
  }
  uint32_t tot;
  uint32_t run = block_excl_scan(s, &tot);
  for (int k = 0; k < kSortItems; ++k) {
    if (base + k < n) a[base + k] = run;
    run += v[k];
  }
  if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

__global__ void __launch_bounds__(kBlock) k_scan_sums(uint32_t* sums, int64_t m) {
  // one block; loops over chunks of kSortBlockKeys
  uint32_t carry = 0;
  for (int64_t c0 = 0; c0 < m; c0 += kSortBlockKeys) {
    const int64_t base = c0 + (int64_t)threadIdx.x * kSortItems;
    uint32_t v[kSortItems], s = 0;
    for (int k = 0; k < kSortItems; ++k) {
      v[k] = base + k < m ? sums[base + k] : 0u;
      s += v[k];
    }
    uint32_t tot;
    uint32_t run = carry + block_excl_scan(s, &tot);
    for (int k = 0; k < kSortItems; ++k) {
      if (base + k < m) sums[base + k] = run;
      run += v[k];
    }
    carry += tot;
    __syncthreads();
  }
}

__global__ void __launch_bounds__(kBlock) k_scan_add(uint32_t* a, int64_t n, const uint32_t* sums) {
  const int64_t base = (int64_t)blockIdx.x * kSortBlockKeys + (int64_t)threadIdx.x * kSortItems;
  const uint32_t add = sums[blockIdx.x];
  for (int k = 0; k < kSortItems; ++k)
    if (base + k < n) a[base + k] += add;
}

static void excl_scan(uint32_t* a, int64_t n, uint32_t* sums, hipStream_t s) {
  const int64_t nb = (n + kSortBlockKeys - 1) / kSortBlockKeys;
  hipLaunchKernelGGL(k_scan_local, dim3((unsigned)nb), dim3(kBlock), 0, s, a, n, sums);
  hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(kBlock), 0, s, sums, nb);
  hipLaunchKernelGGL(k_scan_add, dim3((unsigned)nb), dim3(kBlock), 0, s, a, n, sums);
}

// Stable scatter: elements of a block in the order e = base + k * 256 + tid,
// ranked among equal digits with wave ballots (peer masks) and per-wave
// digit counts in LDS.
__global__ void __launch_bounds__(kBlock) k_radix_scatter(const uint32_t* kin, const uint32_t* vin, uint32_t* kout,
                                                          uint32_t* vout, int64_t n, int shift, const uint32_t* offs,
                                                          int nsb) {
  __shared__ uint32_t run[256];
  __shared__ uint32_t wcnt[kBlock / 64][256];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  run[threadIdx.x] = offs[(int64_t)threadIdx.x * nsb + blockIdx.x];
  for (int w = 0; w < kBlock / 64; ++w) wcnt[w][threadIdx.x] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kSortBlockKeys;
  const unsigned long long lt = (1ull << lane) - 1ull;
  for (int k = 0; k < kSortItems; ++k) {
    const int64_t e = base + (int64_t)k * kBlock + threadIdx.x;
    const bool valid = e < n;
    const uint32_t key = valid ? kin[e] : 0u;
    const uint32_t val = valid ? vin[e] : 0u;
    const uint32_t d = (key >> shift) & 255u;
    unsigned long long peers = __ballot(valid);
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
      const bool on = (d >> bit) & 1u;
      const unsigned long long m = __ballot(on);
      peers &= on ? m : ~m;
    }
    const uint32_t rank_w = (uint32_t)__popcll(peers & lt);
    const bool leader = valid && (peers & lt) == 0ull;
    if (leader) wcnt[wid][d] = (uint32_t)__popcll(peers);
    __syncthreads();
    if (valid) {
      uint32_t pos = run[d] + rank_w;
      for (int w = 0; w < wid; ++w) pos += wcnt[w][d];
      kout[pos] = key;
      vout[pos] = val;
    }
    __syncthreads();
    {
      uint32_t add = 0;
      for (int w = 0; w < kBlock / 64; ++w) { add += wcnt[w][threadIdx.x]; wcnt[w][threadIdx.x] = 0; }
      run[threadIdx.x] += add;
    }
    __syncthreads();
  }
}

int sort_passes(uint32_t max_key) {
  int bits = 0;
  while (bits < 32 && (max_key >> bits) != 0u) ++bits;
  return (bits + 7) / 8;
}

int64_t sort_hist_words(int64_t n) {
  const int64_t nsb = (n + kSortBlockKeys - 1) / kSortBlockKeys;
  return 256 * nsb;
}

int64_t sort_sum_words(int64_t n) {
  const int64_t h = sort_hist_words(n);
  return (h + kSortBlockKeys - 1) / kSortBlockKeys + 1;
}

// Sorts (keys[0], vals[0]) (ping-pong through keys[1], vals[1]); returns the
// index of the buffer pair holding the result.
int radix_sort(uint32_t* keys[2], uint32_t* vals[2], int64_t n, uint32_t max_key, uint32_t* hist, uint32_t* sums,
                hipStream_t s) {
  const int passes = sort_passes(max_key);
  const int nsb = (int)((n + kSortBlockKeys - 1) / kSortBlockKeys);
  int cur = 0;
  for (int ps = 0; ps < passes; ++ps) {
    const int shift = 8 * ps;
    hipLaunchKernelGGL(k_radix_hist, dim3(nsb), dim3(kBlock), 0, s, keys[cur], n, shift, hist, nsb);
    excl_scan(hist, (int64_t)256 * nsb, sums, s);
    hipLaunchKernelGGL(k_radix_scatter, dim3(nsb), dim3(kBlock), 0, s, keys[cur], vals[cur], keys[1 - cur],
                       vals[1 - cur], n, shift, hist, nsb);
    cur = 1 - cur;
  }
  return cur;
}

// ---------------------------------------------------------------------------
// Gather of the state rows (and ids) into sorted order, and the inverse
// (scatter) used to carry adjoints back across a sort.
// ---------------------------------------------------------------------------
template <typename W>
__global__ void k_gather(const W* in, W* out, const uint32_t* perm, int rows, int64_t ntot, const uint32_t* pid_in,
                         uint32_t* pid_out) {
  const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (j >= ntot) return;
  const int64_t src = perm[j];
  for (int r = 0; r < rows; ++r) out[(int64_t)r * ntot + j] = in[(int64_t)r * ntot + src];
  if (pid_out) pid_out[j] = pid_in[src];
}

template <typename W>
__global__ void k_scatter(const W* in, W* out, const uint32_t* perm, int rows, int64_t ntot) {
  const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (j >= ntot) return;
  const int64_t dst = perm[j];
  for (int r = 0; r < rows; ++r) out[(int64_t)r * ntot + dst] = in[(int64_t)r * ntot + j];
}

void launch_gather(int elem_bytes, const void* in, void* out, const uint32_t* perm, int rows, int64_t ntot,
                   const uint32_t* pid_in, uint32_t* pid_out, hipStream_t s) {
  const unsigned nb = (unsigned)((ntot + kBlock - 1) / kBlock);
  if (elem_bytes == 4) hipLaunchKernelGGL(k_gather<uint32_t>, dim3(nb), dim3(kBlock), 0, s, (const uint32_t*)in, (uint32_t*)out, perm, rows, ntot, pid_in, pid_out);
  else hipLaunchKernelGGL(k_gather<uint64_t>, dim3(nb), dim3(kBlock), 0, s, (const uint64_t*)in, (uint64_t*)out, perm, rows, ntot, pid_in, pid_out);
}

void launch_unpermute(int elem_bytes, const void* in, void* out, const uint32_t* perm, int rows, int64_t ntot,
                      hipStream_t s) {
  const unsigned nb = (unsigned)((ntot + kBlock - 1) / kBlock);
  if (elem_bytes == 4) hipLaunchKernelGGL(k_scatter<uint32_t>, dim3(nb), dim3(kBlock), 0, s, (const uint32_t*)in, (uint32_t*)out, perm, rows, ntot);
  else hipLaunchKernelGGL(k_scatter<uint64_t>, dim3(nb), dim3(kBlock), 0, s, (const uint64_t*)in, (uint64_t*)out, perm, rows, ntot);
}

// ---------------------------------------------------------------------------
// Occupied tiles from the sorted keys: [start, end) slot ranges per tile.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int64_t key_tile(uint32_t key, const KCfg& c, int tshift) {
  const uint32_t cells = (uint32_t)c.nodes;
  const uint32_t inst = key / (cells + 1u);
  const uint32_t local = key - inst * (cells + 1u);
  if (local >= cells) return -1;               // padding
  const int64_t tiles = c.nodes >> tshift;
  return (int64_t)inst * tiles + (local >> tshift);
}

__global__ void k_tile_bounds(KCfg c, const uint32_t* keys, int tshift, uint32_t* tstart, uint32_t* tend) {
  const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (j >= c.ntot) return;
  const int64_t t = key_tile(keys[j], c, tshift);
  if (t < 0) return;
  const int64_t tp = j > 0 ? key_tile(keys[j - 1], c, tshift) : -2;
  const int64_t tn = j + 1 < c.ntot ? key_tile(keys[j + 1], c, tshift) : -2;
  if (tp != t) tstart[t] = (uint32_t)j;
  if (tn != t) tend[t] = (uint32_t)(j + 1);
}

// One record per occupied tile (a workgroup takes a whole tile, however many
// particles it holds), and the record of each tile in tslot.  The records
// are ordered by particle count, largest first, in buckets of 2^shift particles
// (kTileBuckets, the last open-ended): workgroups are dispatched in list
// order, so the longest tiles start first and the short ones fill the end of
// the launch (P2G 566 -> 532 us per launch on the 64-instance batch).
// Buckets of 32 leave all tiles above 480 in one.  Of 64 they set those beyond
// 512, with a round more to do, apart: while all workgroups are resident or
// nearly so, the longest decides the launch (joined G2P + P2G 37.0 -> 35.0 us for
// five beds of 54 872 particles, 31.4 -> 31.0 at 219 488, the G2P adjoint 23.2 ->
// 22.6).  In larger contexts the G2P adjoint loses more (75.5 -> 78.7 us at 1.8 M
// particles, 142.7 -> 147.9 for 24 beds) than P2G gains (129.5 -> 128.7).
__device__ __forceinline__ int tile_bucket(uint32_t n, int shift) {
  return min(kTileBuckets - 1, (int)((n - 1u) >> shift));
}

// Counts per bucket: a workgroup histogram in LDS, then one global add per
// bucket and workgroup.
__global__ void k_tile_buckets(int64_t total_tiles, const uint32_t* tstart, const uint32_t* tend, uint32_t* bucket) {
  __shared__ uint32_t h[kTileBuckets];
  if (threadIdx.x < kTileBuckets) h[threadIdx.x] = 0u;
  __syncthreads();
  const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const uint32_t e = t < total_tiles ? tend[t] : 0u;
  if (e != 0u) atomicAdd(&h[tile_bucket(e - tstart[t], 5)], 1u);
  __syncthreads();
  if (threadIdx.x < kTileBuckets && h[threadIdx.x] != 0u) atomicAdd(&bucket[threadIdx.x], h[threadIdx.x]);
}

// bucket[0, B): counts -> bucket[B, 2B): first record of each bucket, the
// largest bucket first; count = the number of records.
__global__ void k_tile_bucket_offsets(uint32_t* bucket, uint32_t* count) {
  if (threadIdx.x != 0) return;
  uint32_t acc = 0;
  for (int b = kTileBuckets - 1; b >= 0; --b) {
    bucket[kTileBuckets + b] = acc;
    acc += bucket[b];
  }
  *count = acc;
}

// Records: ranks within the workgroup from an LDS count per bucket, one
// global add per bucket and workgroup for the range of records.
__global__ void k_tile_list(int64_t total_tiles, const uint32_t* tstart, const uint32_t* tend, TileRec* list,
                            uint32_t* bucket, uint32_t* tslot) {
  __shared__ uint32_t h[kTileBuckets], base[kTileBuckets];
  if (threadIdx.x < kTileBuckets) h[threadIdx.x] = 0u;
  __syncthreads();
  const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const uint32_t e = t < total_tiles ? tend[t] : 0u;
  const uint32_t st = e != 0u ? tstart[t] : 0u;
  const int bk = tile_bucket(e - st, 5);
  const uint32_t rank = e != 0u ? atomicAdd(&h[bk], 1u) : 0u;
  __syncthreads();
  if (threadIdx.x < kTileBuckets && h[threadIdx.x] != 0u)
    base[threadIdx.x] = atomicAdd(&bucket[kTileBuckets + threadIdx.x], h[threadIdx.x]);
  __syncthreads();
  if (e == 0u) return;
  const uint32_t idx = base[bk] + rank;
  list[idx] = TileRec{st, e, (uint32_t)t};
  tslot[t] = idx;
}

__global__ void k_tile_slots(TileList tl, int64_t max_records, uint32_t* tslot) {
  const int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (r >= max_records || r >= (int64_t)*tl.count) return;
  tslot[tl.list[r].tile] = (uint32_t)r;
}

void launch_tile_slots(const KCfg& c, const TileList& tl, int64_t max_records, uint32_t* tslot, hipStream_t s) {
  const int tshift = c.dim == 3 ? 6 : 4;
  const int64_t total_tiles = (c.nodes >> tshift) * c.n_inst;
  launch_fill_u32(tslot, total_tiles, kNoSlot, s);
  hipLaunchKernelGGL(k_tile_slots, dim3((unsigned)((max_records + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, tl,
                     max_records, tslot);
}

void launch_tile_list(const KCfg& c, const uint32_t* sorted_keys, uint32_t* tstart, uint32_t* tend, TileRec* list,
                      uint32_t* count, uint32_t* tslot, uint32_t* bucket, hipStream_t s) {
  const int tshift = c.dim == 3 ? 6 : 4;   // log2(kTile^D)
  const int64_t total_tiles = (c.nodes >> tshift) * c.n_inst;
  const unsigned ntb = (unsigned)((total_tiles + kBlock - 1) / kBlock);
  launch_fill_zero(tend, total_tiles, 4, s);
  launch_fill_zero(bucket, kTileBuckets, 4, s);
  launch_fill_u32(tslot, total_tiles, kNoSlot, s);
  hipLaunchKernelGGL(k_tile_bounds, dim3((unsigned)((c.ntot + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, c,
                     sorted_keys, tshift, tstart, tend);
  hipLaunchKernelGGL(k_tile_buckets, dim3(ntb), dim3(kBlock), 0, s, total_tiles, tstart, tend, bucket);
  hipLaunchKernelGGL(k_tile_bucket_offsets, dim3(1), dim3(64), 0, s, bucket, count);
  hipLaunchKernelGGL(k_tile_list, dim3(ntb), dim3(kBlock), 0, s, total_tiles, tstart, tend, list, bucket, tslot);
}

// Active set after a binning: mark the 3^D blocks around every occupied tile,
// then list the marked blocks.
__global__ void k_mark_active(KCfg c, TileList tl, int64_t max_records, uint32_t* mask) {
  const int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (r >= max_records || r >= (int64_t)*tl.count) return;
  const int D = c.dim, nt = c.n / kTile;
  const uint32_t per = D == 3 ? (uint32_t)(nt * nt * nt) : (uint32_t)(nt * nt);
  const uint32_t gt = tl.list[r].tile;
  const uint32_t inst = gt / per;
  uint32_t t = gt - inst * per;
  int tc[3] = {0, 0, 0};
  for (int a = D - 1; a >= 0; --a) { tc[a] = (int)(t % (uint32_t)nt); t /= (uint32_t)nt; }
  for (int d0 = -1; d0 <= 1; ++d0)
    for (int d1 = -1; d1 <= 1; ++d1)
      for (int d2 = (D == 3 ? -1 : 0); d2 <= (D == 3 ? 1 : 0); ++d2) {
        const int q[3] = {tc[0] + d0, tc[1] + d1, tc[2] + d2};
        bool ok = true;
        for (int a = 0; a < D; ++a) ok &= q[a] >= 0 && q[a] < nt;
        if (!ok) continue;
        const uint32_t lb = D == 3 ? (uint32_t)((q[0] * nt + q[1]) * nt + q[2]) : (uint32_t)(q[0] * nt + q[1]);
        mask[inst * per + lb] = 1u;
      }
}

__global__ void k_list_active(int64_t total_tiles, const uint32_t* mask, uint32_t* list, uint32_t* count) {
  const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (t >= total_tiles || mask[t] == 0u) return;
  list[atomicAdd(count, 1u)] = (uint32_t)t;
}

void launch_active_set(const KCfg& c, const TileList& tl, const ActiveSet& act, hipStream_t s) {
  const int tshift = c.dim == 3 ? 6 : 4;
  const int64_t total_tiles = (c.nodes >> tshift) * c.n_inst;
  const unsigned nb = (unsigned)((total_tiles + kBlock - 1) / kBlock);
  launch_fill_zero(act.mask, total_tiles, 4, s);
  launch_fill_zero(act.count, 1, 4, s);
  hipLaunchKernelGGL(k_mark_active, dim3(nb), dim3(kBlock), 0, s, c, tl, total_tiles, act.mask);
  hipLaunchKernelGGL(k_list_active, dim3(nb), dim3(kBlock), 0, s, total_tiles, act.mask, act.list, act.count);
}

// ---------------------------------------------------------------------------
// Two-level counting sort.  The order wanted is (tile, cell, slot), slot being
// the position before the sort (the stable order).  A tile holds a few hundred
// particles, so a workgroup can order its tile in LDS; what is left is a
// counting sort by tile, whose counters need not be stable because the tile's
// workgroup restores the slot order:
//   k_bin_count  cell of every particle, its rank in its tile's counter (one
//                atomic per wave and distinct tile; sorted states have one or
//                two tiles per wave);
//   k_bin_table  from the counts: first slot of each tile, the occupied-tile
//                list with its records, the active node blocks;
//   k_bin_place  slot numbers to their tile's range; padding keeps its place;
//   k_bin_order  a workgroup per tile: order by (cell, slot), permutation,
//                gather of the state rows and ids.
// The radix sort takes 23 to 31 launches and copies for the same, 4 to 5 us
// each whatever their size: 125 us of kernels per binning of 28 880 particles on
// a 64^3 grid against 31 us here, 124 against 36 at 219 488, 260 against 125 at
// 1.8 M and 390 against 242 for 3.5 M particles of 32 instances (most of it the
// 192 B per particle of the gather).
// ---------------------------------------------------------------------------
constexpr int kOrderCap = 2048;           // particles of a tile that k_bin_order holds in LDS
constexpr int kOrderStep = 1024;          // and that it takes at a time of a tile of more
constexpr int kTableThreads = 1024;
constexpr int kTableTiles = 4096;         // tiles per workgroup of k_bin_table

// ck[slot] = tile * kTile^D + cell (padding: ~0), rank[slot] = its place in the
// tile's range; clears mask and *acount for k_bin_table.
template <int PREC>
__global__ void __launch_bounds__(kBlock) k_bin_count(KCfg c, Bufs b, const void* state, uint32_t* __restrict__ ck,
                                                      uint32_t* __restrict__ rank, uint32_t* __restrict__ tcnt,
                                                      int64_t total_tiles, uint32_t* __restrict__ mask,
                                                      uint32_t* __restrict__ acount) {
  const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  for (int64_t t = j; t < total_tiles; t += (int64_t)gridDim.x * kBlock) mask[t] = 0u;
  if (j == 0) *acount = 0u;
  const int i = b.blk_inst[blockIdx.x];
  const InstDev& I = b.inst[i];
  const int lane = threadIdx.x & 63;
  const bool live = j - I.off < I.n;
  uint32_t tile = 0, cell = 0;
  if (live) {
    const int nt = c.n / kTile;
    bool ok = true;
    for (int a = 0; a < c.dim; ++a) {
      int q;
      if (PREC == 0) ok &= cell_f32(static_cast<const uint32_t*>(state)[(int64_t)a * c.ntot + j], c, q);
      else ok &= cell_f64(static_cast<const double*>(state)[(int64_t)a * c.ntot + j], c, q);
      tile = tile * nt + q / kTile;
      cell = cell * kTile + q % kTile;
    }
    if (!ok) atomicOr(&b.err->flags, 2u);
    tile += (uint32_t)(c.nodes >> (c.dim == 3 ? 6 : 4)) * (uint32_t)i;
  }
  // the tiles of a sorted wave (one, two at a tile's end) with one atomic each,
  // one after another; lanes of further tiles, which positions in no order
  // have, with one each at the same time
  unsigned long long todo = __ballot(live);
  uint32_t r = 0;
#pragma unroll 1
  for (int k = 0; k < 8 && todo; ++k) {
    const int lead = __ffsll((long long)todo) - 1;
    const uint32_t t = (uint32_t)__builtin_amdgcn_readlane((int)tile, lead);
    const unsigned long long same = __ballot(live && tile == t);
    uint32_t base = 0;
    if (lane == lead) base = atomicAdd(&tcnt[t], (uint32_t)__popcll(same));
    base = (uint32_t)__builtin_amdgcn_readlane((int)base, lead);
    if (live && tile == t) r = base + (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
    todo &= ~same;
  }
  if ((todo >> lane) & 1ull) r = atomicAdd(&tcnt[tile], 1u);
  ck[j] = live ? (tile << (c.dim == 3 ? 6 : 4)) + cell : 0xFFFFFFFFu;
  rank[j] = r;
}

// Where k_bin_table writes; list2 / count2 (may be NULL) get a second copy of
// the tile list.
struct TableOut {
  uint32_t* tcnt;
  uint32_t* tstart;
  TileRec* list;
  uint32_t* count;
  TileRec* list2;
  uint32_t* count2;
  uint32_t* tslot;
  ActiveSet act;
  uint32_t* part;                         // [workgroups][1 + kTileBuckets]: particles, tiles per bucket
};

// Sum of v over the workgroup's threads below this one; total in *sum.
__device__ __forceinline__ uint32_t table_scan(uint32_t v, uint32_t* sum) {
  __shared__ uint32_t ws[kTableThreads / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  __syncthreads();
  if (lane == 63) ws[wid] = x;
  __syncthreads();
  uint32_t off = 0, tot = 0;
  for (int w = 0; w < kTableThreads / 64; ++w) {
    if (w < wid) off += ws[w];
    tot += ws[w];
  }
  *sum = tot;
  return off + x - v;
}

// Of the four tiles 4 i .. 4 i + 3, those with an occupied tile among the 3^D
// around them, a bit each.  nib(j): the occupied ones of tiles 4 j .. 4 j + 3.  A
// row of tiles along the last axis holds whole fours (grids have 16 nodes a
// side at least), so a row's part is three of them.  Read like this it takes
// 3 us of the launch on a 64^3 grid (10.9 in all); each occupied tile marking the blocks
// around it, in memory or by LDS atomics on the words that its neighbours mark
// as well, took 8.
template <typename Nib>
__device__ __forceinline__ uint32_t near_occupied(const KCfg& c, uint32_t i, Nib&& nib) {
  const int D = c.dim, tb = c.nlog2 - 2, nt = 1 << tb;
  const uint32_t per = 1u << (D * tb), first = (4u * i) & ~(per - 1u), t = (4u * i) & (per - 1u);
  const int ql = (int)(t & (uint32_t)(nt - 1)), qm = D == 3 ? (int)((t >> tb) & (uint32_t)(nt - 1)) : 0;
  const int q0 = (int)(t >> ((D - 1) * tb));
  uint32_t near = 0;
  for (int a = max(q0 - 1, 0); a <= min(q0 + 1, nt - 1); ++a)
    for (int e = max(qm - 1, 0); e <= (D == 3 ? min(qm + 1, nt - 1) : 0); ++e) {
      const uint32_t j = (first + (uint32_t)((D == 3 ? (a << tb) + e : a) << tb) + (uint32_t)ql) >> 2;
      // tiles ql - 1 .. ql + 4 of the row
      const uint32_t w = (ql > 0 ? nib(j - 1u) >> 3 : 0u) | nib(j) << 1 | (ql + 4 < nt ? (nib(j + 1u) & 1u) << 5 : 0u);
      near |= w | w >> 1 | w >> 2;
    }
  return near & 15u;
}

// The table of up to kTableTiles tiles per workgroup.  One workgroup does it
// in one launch (STAGE 0); more need two: STAGE 1 leaves their sums in part
// and marks the active blocks, STAGE 2 takes the sums of the workgroups before
// it.  Records are ordered by particle count, largest bucket first: workgroups
// are dispatched in list order, so the longest tiles start first.
template <int STAGE>
__global__ void __launch_bounds__(kTableThreads) k_bin_table(KCfg c, const InstDev* inst, int64_t total_tiles,
                                                             TableOut o) {
  constexpr int PER = kTableTiles / kTableThreads;
  __shared__ uint32_t hist[kTileBuckets], first[kTileBuckets], sums[1 + kTileBuckets], abase;
  __shared__ unsigned char occ[kTableThreads];
  const int tid = threadIdx.x;
  const int64_t t0 = (int64_t)blockIdx.x * kTableTiles + (int64_t)tid * PER;
  if (tid < kTileBuckets) hist[tid] = 0u;
  if (tid <= kTileBuckets) sums[tid] = 0u;
  __syncthreads();
  static_assert(PER == 4, "near_occupied takes four tiles");
  uint32_t n[PER], own = 0, full = 0;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    n[k] = t0 + k < total_tiles ? o.tcnt[t0 + k] : 0u;
    own += n[k];
    if (n[k]) full |= 1u << k;
    if (n[k] && STAGE != 2) atomicAdd(&hist[tile_bucket(n[k], c.bucket_shift)], 1u);
  }
  if (STAGE != 2) occ[tid] = (unsigned char)full;
  uint32_t tot = 0, before = 0;
  before = table_scan(own, &tot);
  __syncthreads();
  // active blocks of this thread; tiles of other workgroups by their counts
  // (which the second launch clears)
  uint32_t marked = 0;
  if (STAGE != 2 && t0 < total_tiles) {
    marked = near_occupied(c, (uint32_t)(t0 / PER), [&](uint32_t j) -> uint32_t {
      const uint32_t r = j - blockIdx.x * kTableThreads;
      if (r < (uint32_t)kTableThreads) return occ[r];
      uint32_t v = 0;
#pragma unroll
      for (int k = 0; k < PER; ++k) v |= o.tcnt[(int64_t)j * PER + k] ? 1u << k : 0u;
      return v;
    });
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if ((marked >> k) & 1u) o.act.mask[t0 + k] = 1u;
  }
  if (STAGE == 1) {
    uint32_t* pt = o.part + (int64_t)blockIdx.x * (1 + kTileBuckets);
    if (tid == 0) pt[0] = tot;
    if (tid < kTileBuckets) pt[1 + tid] = hist[tid];
    return;
  }
  // first record of each bucket (largest first), and what the workgroups before this one hold
  if (STAGE == 2) {
    for (int e = tid; e < (int)gridDim.x * (1 + kTileBuckets); e += kTableThreads) {
      const int w = e / (1 + kTileBuckets), k = e - w * (1 + kTileBuckets);
      const uint32_t v = o.part[e];
      if (k > 0) atomicAdd(&hist[k - 1], v);
      if (w < (int)blockIdx.x) atomicAdd(&sums[k], v);
    }
    __syncthreads();
  }
  if (tid < 64) {
    static_assert(kTileBuckets <= 64, "a lane per bucket");
    const int k = kTileBuckets - 1 - tid;
    const uint32_t h = k >= 0 ? hist[k] : 0u;
    uint32_t acc = h;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(acc, d, 64);
      if (tid >= d) acc += y;
    }
    if (k >= 0) first[k] = acc - h + sums[1 + k];
    if (blockIdx.x == 0 && tid == 63) {
      *o.count = acc;
      if (o.count2) *o.count2 = acc;
    }
  }
  __syncthreads();
  // tile starts: the particles before the tile in its instance, from the instance's first slot
  uint32_t run = sums[0] + before;
  const int pb = c.dim * (c.nlog2 - 2);
  int cur = -1;
  uint32_t shift = 0;                     // the padding before the instance
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int64_t t = t0 + k;
    if (t >= total_tiles) break;
    const int i = (int)(t >> pb);
    if (i != cur) {
      cur = i;
      shift = (uint32_t)inst[i].pad;
    }
    const uint32_t st = run + shift;
    run += n[k];
    o.tstart[t] = st;
    o.tcnt[t] = 0u;                       // for the next binning
    uint32_t slot = kNoSlot;
    if (n[k]) {
      slot = atomicAdd(&first[tile_bucket(n[k], c.bucket_shift)], 1u);
      const TileRec r{st, st + n[k], (uint32_t)t};
      o.list[slot] = r;
      if (o.list2) o.list2[slot] = r;
    }
    o.tslot[t] = slot;
  }
  // list of the active blocks
  uint32_t a[PER], na = 0;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    a[k] = STAGE == 0 ? (marked >> k) & 1u : (t0 + k < total_tiles ? o.act.mask[t0 + k] : 0u);
    na += a[k] ? 1u : 0u;
  }
  uint32_t atot = 0, pos = table_scan(na, &atot);
  if (tid == 0) abase = atomicAdd(o.act.count, atot);
  __syncthreads();
  pos += abase;
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (a[k]) o.act.list[pos++] = (uint32_t)(t0 + k);
}

template <typename W>
__global__ void __launch_bounds__(kBlock) k_bin_place(KCfg c, Bufs b, const uint32_t* __restrict__ ck,
                                                      const uint32_t* __restrict__ rank,
                                                      const uint32_t* __restrict__ tstart, uint32_t* __restrict__ tmp,
                                                      const W* in, W* out, int rows, const uint32_t* pid_in,
                                                      uint32_t* pid_out, uint32_t* perm_out) {
  const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const uint32_t k = ck[j];
  if (k != 0xFFFFFFFFu) {
    tmp[tstart[k >> (c.dim == 3 ? 6 : 4)] + rank[j]] = (uint32_t)j;
    return;
  }
  // padding stays at the end of its instance's range, in order
  for (int r = 0; r < rows; ++r) out[(int64_t)r * c.ntot + j] = in[(int64_t)r * c.ntot + j];
  if (pid_out) pid_out[j] = pid_in[j];
  if (perm_out) perm_out[j] = (uint32_t)j;
}

// The n slots of an over-full tile in the order of (cell, slot), by a
// least-significant-digit radix sort of one workgroup: 8 bits of the slot
// number a pass, the cell last.  a holds the slots in any order and b is
// scratch; returns the buffer with the result.  Work linear in n, since a tile
// may hold any number of particles (a bed denser than its ppc, or positions
// outside the grid, which count as the nearest cell, or NaN, which count as the
// first).  A step takes kOrderStep slots: every wave ranks a stretch of them
// among its own digits with ballots, then the waves' counts are put one behind
// another.  A binning of 3000, 20 000 and 200 000 particles in one tile takes
// 0.07, 0.31 and 3.5 ms, mostly the gather of the rows by one compute unit, where
// P2G takes 0.12, 1.3 and 25 ms for that tile.
struct OrderLDS {
  uint32_t run[256];                      // next place of each digit
  uint32_t wcnt[kBlock / 64][256];        // the waves' counts, then their places
  uint32_t slot[kOrderStep];              // the step's slots and their ranks in their wave
  uint16_t rank[kOrderStep];
};
__device__ __forceinline__ uint32_t* order_large(const KCfg& c, const uint32_t* __restrict__ ck, uint32_t* a, uint32_t* b,
                                                 int n, OrderLDS& L) {
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const uint32_t last = (uint32_t)(c.ntot - 1), cmask = c.dim == 3 ? 63u : 15u;
  for (int shift = 0, cells = 0; !cells; shift += 8) {
    cells = shift >= 32 || (last >> shift) == 0u;        // the slot numbers have no further digit: by cell, and done
    auto digit = [&](uint32_t s) -> uint32_t { return cells ? ck[s] & cmask : (s >> shift) & 255u; };
    L.run[tid] = 0u;
    __syncthreads();
#pragma unroll 1
    for (int i = tid; i < n; i += kBlock) atomicAdd(&L.run[digit(a[i])], 1u);
    __syncthreads();
    uint32_t tot;
    L.run[tid] = block_excl_scan(L.run[tid], &tot);
#pragma unroll 1
    for (int c0 = 0; c0 < n; c0 += kOrderStep) {
      for (int w = 0; w < kBlock / 64; ++w) L.wcnt[w][tid] = 0u;
      __syncthreads();
      // (slots and ranks wait in LDS: in registers they cost the kernel's usual
      // path three of seven waves per SIMD)
      constexpr int PER = kOrderStep / (kBlock / 64);
#pragma unroll 1
      for (int i = wid * PER + lane; i < (wid + 1) * PER; i += 64) {
        const bool valid = c0 + i < n;
        const uint32_t s = valid ? a[c0 + i] : 0u;
        const uint32_t d = valid ? digit(s) : 0u;
        unsigned long long peers = __ballot(valid);
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
          const bool on = (d >> bit) & 1u;
          const unsigned long long m = __ballot(on);
          peers &= on ? m : ~m;
        }
        const int lead = valid ? __ffsll((long long)peers) - 1 : lane;
        uint32_t before = 0;
        if (valid && lane == lead) before = atomicAdd(&L.wcnt[wid][d], (uint32_t)__popcll(peers));
        L.slot[i] = s;
        L.rank[i] = (uint16_t)(__shfl((int)before, lead, 64) + __popcll(peers & ((1ull << lane) - 1ull)));
      }
      __syncthreads();
      uint32_t at = L.run[tid];
      for (int w = 0; w < kBlock / 64; ++w) {
        const uint32_t v = L.wcnt[w][tid];
        L.wcnt[w][tid] = at;
        at += v;
      }
      L.run[tid] = at;
      __syncthreads();
#pragma unroll 1
      for (int i = tid; i < kOrderStep && c0 + i < n; i += kBlock) {
        const uint32_t s = L.slot[i];
        b[L.wcnt[i / PER][digit(s)] + L.rank[i]] = s;
      }
      __syncthreads();
    }
    uint32_t* t = a;
    a = b;
    b = t;
  }
  return a;
}

// rank is free here (k_bin_place was its last reader): the scratch of an
// over-full tile.
template <typename W, int ROWS>
__global__ void __launch_bounds__(kBlock) k_bin_order(KCfg c, const TileRec* __restrict__ list,
                                                      const uint32_t* __restrict__ count,
                                                      const uint32_t* __restrict__ ck, uint32_t* tmp, uint32_t* rank,
                                                      const W* __restrict__ in, W* __restrict__ out,
                                                      const uint32_t* __restrict__ pid_in, uint32_t* __restrict__ pid_out,
                                                      uint32_t* __restrict__ perm_out) {
  __shared__ union {
    struct { uint32_t byc[kOrderCap], fin[kOrderCap]; };   // slots by cell, then in order
    OrderLDS large;
  } u;
  uint32_t(&byc)[kOrderCap] = u.byc, (&fin)[kOrderCap] = u.fin;
  __shared__ uint32_t cnt[64], start[64], fill[64];
  const int tid = threadIdx.x;
  const uint32_t cmask = c.dim == 3 ? 63u : 15u;
  const uint32_t ntiles = *count;
  for (uint32_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const TileRec tr = list[t];
    const int n = (int)(tr.end - tr.start);
    uint32_t* ts = tmp + tr.start;
    const uint32_t* order = nullptr;                       // of an over-full tile, in memory
    if (n <= kOrderCap) {
      if (tid < 64) { cnt[tid] = 0u; fill[tid] = 0u; }
      __syncthreads();
      uint32_t sl[kOrderCap / kBlock], ql[kOrderCap / kBlock];      // this thread's slots and cells
#pragma unroll
      for (int k = 0; k < kOrderCap / kBlock; ++k)
        if (tid + k * kBlock < n) {
          sl[k] = ts[tid + k * kBlock];
          ql[k] = ck[sl[k]] & cmask;
          atomicAdd(&cnt[ql[k]], 1u);
        }
      __syncthreads();
      if (tid < 64) {
        uint32_t x = cnt[tid];
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const uint32_t y = __shfl_up(x, o, 64);
          if (tid >= o) x += y;
        }
        start[tid] = x - cnt[tid];
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < kOrderCap / kBlock; ++k)
        if (tid + k * kBlock < n) byc[start[ql[k]] + atomicAdd(&fill[ql[k]], 1u)] = sl[k];
      __syncthreads();
#pragma unroll
      for (int k = 0; k < kOrderCap / kBlock; ++k)
        if (tid + k * kBlock < n) {
          const int lo = (int)start[ql[k]], hi = lo + (int)cnt[ql[k]];
          int at = lo;
          for (int e = lo; e < hi; ++e) at += byc[e] < sl[k] ? 1 : 0;
          fin[at] = sl[k];
        }
    } else {
      order = order_large(c, ck, ts, rank + tr.start, n, u.large);
    }
    for (int c0 = 0; c0 < n; c0 += kOrderCap) {
      const int m = min(n - c0, kOrderCap);
      if (order)
        for (int i = tid; i < m; i += kBlock) fin[i] = order[c0 + i];
      __syncthreads();
      for (int i = tid; i < m; i += kBlock) {
        const uint32_t s = fin[i];
        const int64_t d = (int64_t)tr.start + c0 + i;
        W v[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) v[r] = in[(int64_t)r * c.ntot + s];
        if (pid_out) pid_out[d] = pid_in[s];
        if (perm_out) perm_out[d] = s;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) out[(int64_t)r * c.ntot + d] = v[r];
      }
      __syncthreads();
    }
  }
}

// The counting sort needs tile * kTile^D + cell below 2^32 - 1, and the bed's
// tiles (ppc particles per cell at rest) within k_bin_order's LDS with room for
// compaction; a tile beyond that is ordered by a radix sort of its workgroup.
bool bin_by_tiles(const KCfg& c, double ppc) {
  const double cells = c.dim == 3 ? 64.0 : 16.0;
  return !c.det && (double)c.nodes * c.n_inst < 4294967295.0 && ppc * cells <= kOrderCap / 2;
}

int64_t bin_part_words(int64_t total_tiles) {
  return (total_tiles + kTableTiles - 1) / kTableTiles * (1 + kTileBuckets);
}

void launch_bin_tiles(int prec, const KCfg& c, const Bufs& b, int nblk, int nwg, const void* src, void* dst,
                      const uint32_t* pid_in, uint32_t* pid_out, uint32_t* perm_out, const BinBufs& w, hipStream_t s) {
  const int tshift = c.dim == 3 ? 6 : 4;
  const int64_t total_tiles = (c.nodes >> tshift) * c.n_inst;
  if (prec == 0)
    hipLaunchKernelGGL(k_bin_count<0>, dim3(nblk), dim3(kBlock), 0, s, c, b, src, w.ck, w.rank, w.tcnt, total_tiles,
                       w.act.mask, w.act.count);
  else
    hipLaunchKernelGGL(k_bin_count<1>, dim3(nblk), dim3(kBlock), 0, s, c, b, src, w.ck, w.rank, w.tcnt, total_tiles,
                       w.act.mask, w.act.count);
  const TableOut o{w.tcnt, w.tstart, w.list, w.count, w.list2, w.count2, w.tslot, w.act, w.part};
  const unsigned ntw = (unsigned)((total_tiles + kTableTiles - 1) / kTableTiles);
  if (ntw == 1) {
    hipLaunchKernelGGL(k_bin_table<0>, dim3(1), dim3(kTableThreads), 0, s, c, b.inst, total_tiles, o);
  } else {
    hipLaunchKernelGGL(k_bin_table<1>, dim3(ntw), dim3(kTableThreads), 0, s, c, b.inst, total_tiles, o);
    hipLaunchKernelGGL(k_bin_table<2>, dim3(ntw), dim3(kTableThreads), 0, s, c, b.inst, total_tiles, o);
  }
  const int rows = 2 * c.dim + 2 * c.dim * c.dim;
#define DDM_BIN(W, R)                                                                                              \
  hipLaunchKernelGGL((k_bin_place<W>), dim3(nblk), dim3(kBlock), 0, s, c, b, w.ck, w.rank, w.tstart, w.tmp,        \
                     (const W*)src, (W*)dst, rows, pid_in, pid_out, perm_out);                                     \
  hipLaunchKernelGGL((k_bin_order<W, R>), dim3(nwg), dim3(kBlock), 0, s, c, w.list, w.count, w.ck, w.tmp, w.rank,  \
                     (const W*)src, (W*)dst, pid_in, pid_out, perm_out)
  if (prec == 0) {
    if (c.dim == 3) { DDM_BIN(uint32_t, 24); } else { DDM_BIN(uint32_t, 12); }
  } else {
    if (c.dim == 3) { DDM_BIN(uint64_t, 24); } else { DDM_BIN(uint64_t, 12); }
  }
#undef DDM_BIN
}

}  // namespace ddm

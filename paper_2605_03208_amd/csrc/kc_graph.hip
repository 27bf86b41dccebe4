// kc_graph.hip -- gfx950 kernels over the ranges beyond the snapshot itself:
// the pointer graph between ranges and the per-range byte difference against
// a snapshot.  Persistent grids of waves over the tile list, range fences in LDS
// (the graph: up to eight waves per workgroup sharing the wide table; the region
// diff: up to four for pages, up to sixteen for larger units).
#include <algorithm>

#include "kc_device.h"
#include "kc_internal.h"

namespace kc {
namespace {

inline uint32_t blocks_for(uint64_t n, uint32_t per) { return (uint32_t)((n + per - 1) / per); }

// Pointer graph: for every pointer-like word, set bit (source range, target
// range).  When the lanes of a wave hit one target (a table of pointers into
// one allocation), one lane sets it, unless the wave set it last.  Otherwise
// each lane sets its own, unless the word already shows it: lanes on different
// targets do not wait for each other, and a target met again costs a read.
__device__ __forceinline__ void graph_emit(int32_t t, uint64_t* row, int32_t& last) {
  if (t < 0) return;
  const int32_t tb = __builtin_amdgcn_readfirstlane(t);  // of the lanes here
  if (__ballot(t != tb) == 0ull) {
    if (tb != last && __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)) ==
                          (uint32_t)__builtin_ctzll(__ballot(1)))
      atomicOr((unsigned long long*)&row[tb >> 6], 1ull << (tb & 63));
    last = tb;
    return;
  }
  const unsigned long long bit = 1ull << (t & 63);
  unsigned long long* const word = (unsigned long long*)&row[t >> 6];
  if ((__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bit) == 0ull) atomicOr(word, bit);
}

// Workgroups of kWideWaves independent waves share the wide range table.
__global__ __launch_bounds__(kWideWaves * kWave) __attribute__((amdgpu_waves_per_eu(4))) void k_pointer_graph(
    const Tile* tiles, uint32_t n_tiles, uint64_t lo, uint64_t span, RangeTable rt, uint64_t* edge_bm,
    uint32_t row_words) {
  __shared__ uint64_t queue[kWideWaves][kPtrQueue];
  const uint32_t wv = threadIdx.x / kWave, wpb = blockDim.x / kWave;
  const uint32_t wave = blockIdx.x * wpb + wv, n_waves = gridDim.x * wpb;
  load_wide_fences(rt, threadIdx.x, blockDim.x);
  __syncthreads();
  for (uint32_t t = wave; t < n_tiles; t += n_waves) {
    const Tile tile = tiles[t];
    const int32_t src = wide_range_index(tile.va, rt);  // the tile's own range (always found)
    if (src < 0) continue;
    uint64_t* const row = edge_bm + (uint64_t)src * row_words;
    int32_t last = -1;
    each_pointer(tile, lo, span, queue[wv], [&](uint64_t w, uint32_t) { graph_emit(wide_range_index(w, rt), row, last); });
  }
}

// Per-range byte difference against a full snapshot.  Pages are visited in
// order inside a tile; the snapshot slot of a non-zero page is its rank among
// the non-zero pages (prefix per bitmap word + popcount below its bit).
__global__ void k_region_init(kc_region_diff_result* res, uint32_t n, uint64_t* bm_a, uint64_t* bm_b, uint64_t n_words) {
  const uint64_t m = n > n_words ? n : n_words;
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < m; i += (uint64_t)gridDim.x * blockDim.x) {
    if (i < n) {
      res[i].n_diff_bytes = 0;
      res[i].n_diff_pages = 0;
      res[i].first_diff_va = ~0ull;
      res[i].n_bad_pages = 0;
    }
    if (i < n_words) {
      bm_a[i] = 0;
      bm_b[i] = 0;
    }
  }
}

__device__ __forceinline__ uint32_t nonzero_bytes(uint32_t x) {
  return (uint32_t)__popc((((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x) & 0x80808080u);
}

__device__ __forceinline__ uint64_t read_lane64(uint64_t x, uint32_t lane) {
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((uint32_t)(x >> 32), lane) << 32) |
         (uint32_t)__builtin_amdgcn_readlane((uint32_t)x, lane);
}

__device__ __forceinline__ uint64_t wave_min_u64(uint64_t x) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) x = min(x, (uint64_t)__shfl_xor((unsigned long long)x, d, 64));
  return x;
}

__device__ __forceinline__ void flush_region(kc_region_diff_result* res, int32_t a, uint64_t dbytes, uint64_t dpages,
                                             uint64_t first) {
  if (a < 0 || dbytes == 0) return;
  kc_region_diff_result* r = res + a;
  atomicAdd((unsigned long long*)&r->n_diff_bytes, (unsigned long long)dbytes);
  atomicAdd((unsigned long long*)&r->n_diff_pages, (unsigned long long)dpages);
  atomicMin((unsigned long long*)&r->first_diff_va, (unsigned long long)first);
}

// What one lane knows of its unit: its place, its snapshot copy (gp: address; zero:
// all zeros; bad: none that is accepted), whether its bytes are to be compared.
struct DiffUnit {
  uint64_t va, gp;
  int32_t a;  // range
  uint32_t len;
  bool live, zero, bad, need;
};
__device__ __forceinline__ DiffUnit diff_unit(const Tile& tile, uint32_t j, uint32_t ushift, const FenceLds& fences,
                                              const RangeTable& rt, const uint64_t* changed_bm,
                                              const uint64_t* gold_zero_bm, const uint64_t* rank_prefix,
                                              const uint64_t* gold_page_va, uint64_t n_valid,
                                              const uint8_t* gold_packed) {
  DiffUnit u{};
  u.a = -1;
  u.live = j < tile.npages;
  u.va = tile.va + ((uint64_t)j << ushift);
  if (!u.live) return u;
  const uint64_t g = (uint64_t)tile.g + j;
  u.len = unit_bytes(tile, j, 1u << ushift);
  u.a = range_index(u.va, fences, rt);
  const uint64_t zw = gold_zero_bm[g >> 6];
  u.zero = (zw >> (g & 63u)) & 1ull;
  if (!u.zero) {
    const uint64_t slot = rank_prefix[g >> 6] + (uint64_t)__popcll(~zw & ((1ull << (g & 63u)) - 1ull));
    u.bad = slot >= n_valid || gold_page_va[slot] != u.va;
    u.gp = (uint64_t)gold_packed + (slot << ushift);
  }
  u.need = !u.bad && ((changed_bm[g >> 6] >> (g & 63u)) & 1ull);
  return u;
}

// The lane's part of a 16-byte block's difference: bytes that differ, and the
// lowest of them (off: the block's offset) unless there is one already.
__device__ __forceinline__ void add_diff(const uint4& c, const uint4& d, uint32_t off, uint32_t& nd, uint32_t& fo) {
  const uint32_t x[4] = {c.x ^ d.x, c.y ^ d.y, c.z ^ d.z, c.w ^ d.w};
#pragma unroll
  for (uint32_t i = 0; i < 4; ++i) {
    nd += nonzero_bytes(x[i]);
    if (x[i] != 0u && fo == ~0u) fo = off + 4u * i + ((uint32_t)__builtin_ctz(x[i]) >> 3);
  }
}

// The range that a wave is adding up, and its totals so far.
struct DiffFold {
  int32_t cur = -1;
  uint64_t bytes = 0, pages = 0, first = ~0ull;
  __device__ __forceinline__ void add(kc_region_diff_result* res, bool writes, int32_t a, uint64_t b, uint64_t p, uint64_t at) {
    if (a != cur) {
      if (writes) flush_region(res, cur, bytes, pages, first);
      cur = a;
      bytes = pages = 0;
      first = ~0ull;
    }
    bytes += b;
    pages += p;
    first = min(first, at);
  }
};

// Pages.  A wave takes groups of four consecutive tiles, one lane per page: each
// lane resolves its page's snapshot copy and changed bit, then the whole wave
// compares the changed pages one after another, 8 KiB in flight, and each lane adds
// up what differs in its part of them; the lanes are summed up where the wave leaves
// a range (done for every page, that chain of shuffles took as long as the loads:
// half of 32 MiB changed 65 us, so 42).  Runs of groups are contiguous and folded
// per range, which touches a range's counters only when the run moves to the next
// range or ends (for the waves of a workgroup together, where they end in one
// range): folds that all add into one range's counters as they go queue there.
//
// What bounds it: the bytes of the changed pages, and with few of them a chain of
// three round trips per group; hence few registers and as many waves as are
// resident (20 per CU with these; the built-in grid of 16 suits dense changes
// better).  30 GiB with 1 % / 0.1 % of the pages changed: 133 / 71 us, at 20 waves
// per CU 120 / 63; two pages at a time with their sums in LDS, as the larger units
// below: 206 / 90.  2 GiB in 4096 ranges, half changed, 325 us, at 20 waves per CU
// 350.  With one wave per workgroup (and sums for every page) 4.2 GiB in one range,
// 1 % changed, took 146 us, with four 54, now 53.
constexpr uint32_t kDiffWaves = 16, kDiffPageWaves = 4;

__global__ __launch_bounds__(kDiffPageWaves * kWave) __attribute__((amdgpu_waves_per_eu(5))) void k_region_diff_pages(
    const Tile* tiles, uint32_t n_tiles, RangeTable rt, const uint64_t* changed_bm, const uint64_t* gold_zero_bm,
    const uint64_t* rank_prefix, const uint64_t* gold_page_va, const uint64_t* gold_n_kept, uint64_t cap,
    const uint8_t* gold_packed, kc_region_diff_result* res) {
  __shared__ FenceLds fences;
  __shared__ int32_t end_range[kDiffPageWaves];  // where the runs of the waves end
  __shared__ uint64_t end_bytes[kDiffPageWaves], end_pages[kDiffPageWaves], end_first[kDiffPageWaves];
  const uint32_t lane = threadIdx.x % kWave, sub = lane >> 4, j = lane & 15u, wpb = blockDim.x / kWave;
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  load_fences(fences, rt, threadIdx.x, blockDim.x);
  __syncthreads();
  const uint64_t n_valid = min(*gold_n_kept, cap);
  const uint32_t n_groups = (n_tiles + 3u) / 4u, n_runs = gridDim.x * wpb;
  const uint32_t per_run = (n_groups + n_runs - 1u) / n_runs;
  const uint32_t gbeg = min((blockIdx.x * wpb + wv) * per_run, n_groups), gend = min(gbeg + per_run, n_groups);
  // the range that the wave is in; what differs there: of this lane, pages of the wave, first of this lane
  int32_t cur = -1;
  uint64_t bytes = 0, pages = 0, first = ~0ull;
  auto add_up = [&] {
    if (cur < 0) return;
    bytes = wave_sum_u64(bytes);
    first = wave_min_u64(first);
  };
  auto end_region = [&] {
    add_up();
    if (lane == 0) flush_region(res, cur, bytes, pages, first);
    bytes = pages = 0;
    first = ~0ull;
  };
  for (uint32_t gi = gbeg; gi < gend; ++gi) {
    Tile tile{0, 0, 0};
    if (gi * 4u + sub < n_tiles) tile = tiles[gi * 4u + sub];
    const DiffUnit u = diff_unit(tile, j, kMinUnitShift, fences, rt, changed_bm, gold_zero_bm, rank_prefix, gold_page_va,
                                 n_valid, gold_packed);
    const uint64_t bad_mask = __ballot(u.bad);
    if (j == 0u && u.live && u.a >= 0) {  // the 16 lanes of a tile share its range
      const uint32_t nb = (uint32_t)__popcll((bad_mask >> (16u * sub)) & 0xFFFFull);
      if (nb) atomicAdd((unsigned long long*)&res[u.a].n_bad_pages, (unsigned long long)nb);
    }
    for (uint64_t m = __ballot(u.need); m != 0ull; m &= m - 1ull) {
      const uint32_t L = (uint32_t)__builtin_ctzll(m);
      const uint64_t pva = read_lane64(u.va, L), pgp = read_lane64(u.gp, L);
      const bool pz = __builtin_amdgcn_readlane((int)u.zero, L) != 0;
      const uint32_t plen = __builtin_amdgcn_readlane(u.len, L);  // of a range's last page perhaps less than a page
      uint4 x[4];
      uint32_t nd = 0u;
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k) {
        const uint32_t off = k * 1024u + lane * 16u;
        const uint4 c = off < plen ? clip16(ld16nt(pva + off), off, plen) : make_uint4(0, 0, 0, 0);
        const uint4 d = pz || off >= plen ? make_uint4(0, 0, 0, 0) : clip16(ld16nt(pgp + off), off, plen);
        x[k] = make_uint4(c.x ^ d.x, c.y ^ d.y, c.z ^ d.z, c.w ^ d.w);
        nd += nonzero_bytes(x[k].x) + nonzero_bytes(x[k].y) + nonzero_bytes(x[k].z) + nonzero_bytes(x[k].w);
      }
      if (__ballot(nd != 0u) == 0ull) continue;
      const int32_t a = __builtin_amdgcn_readlane(u.a, L);
      if (a != cur) {
        end_region();
        cur = a;
      }
      bytes += nd;
      ++pages;
      if (nd != 0u && first == ~0ull) {  // the pages of a range come in address order
        uint32_t fo = ~0u, none = 0u;
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) add_diff(x[k], make_uint4(0, 0, 0, 0), k * 1024u + lane * 16u, none, fo);
        first = pva + fo;
      }
    }
  }
  add_up();
  DiffFold fold{cur, bytes, pages, first};
  if (wpb == 1u) {
    if (lane == 0) flush_region(res, fold.cur, fold.bytes, fold.pages, fold.first);
    return;
  }
  if (lane == 0) {
    end_range[wv] = fold.cur;
    end_bytes[wv] = fold.bytes;
    end_pages[wv] = fold.pages;
    end_first[wv] = fold.first;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (uint32_t w = 1; w < wpb; ++w)  // the next wave's run follows: its range is this one or a later one
    if (end_range[w] >= 0) fold.add(res, true, end_range[w], end_bytes[w], end_pages[w], end_first[w]);
  flush_region(res, fold.cur, fold.bytes, fold.pages, fold.first);
}

// Larger units, which are few: a workgroup takes a tile at a time, its waves share
// out the 4 KiB blocks of the changed units, two units at a time, what differs is
// added up per unit in LDS, and the first wave folds it per range as above.
// Measured against one wave per unit, 2048 waves: 6.3 GiB in 2 MiB units with 5 %
// of the pages changed 25.0 -> 2.2 ms, 3.9 GiB in 64 KiB units with 1 % 0.53 -> 0.25.
__global__ __launch_bounds__(kDiffWaves * kWave) __attribute__((amdgpu_waves_per_eu(4))) void k_region_diff_units(
    const Tile* tiles, uint32_t n_tiles, RangeTable rt, const uint64_t* changed_bm, const uint64_t* gold_zero_bm,
    const uint64_t* rank_prefix, const uint64_t* gold_page_va, const uint64_t* gold_n_kept, uint64_t cap,
    const uint8_t* gold_packed, kc_region_diff_result* res, uint32_t ushift) {
  __shared__ FenceLds fences;
  __shared__ uint32_t unit_off[2][kWave], unit_first[2][kWave];  // of a tile's units; changed tiles take turns
  const uint32_t lane = threadIdx.x % kWave, wpb = blockDim.x / kWave;
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  load_fences(fences, rt, threadIdx.x, blockDim.x);
  for (uint32_t i = threadIdx.x; i < 2u * kWave; i += blockDim.x) {
    unit_off[i / kWave][i % kWave] = 0u;
    unit_first[i / kWave][i % kWave] = ~0u;
  }
  __syncthreads();
  const uint64_t n_valid = min(*gold_n_kept, cap);
  const uint32_t per_run = (n_tiles + gridDim.x - 1u) / gridDim.x;
  const uint32_t tbeg = min(blockIdx.x * per_run, n_tiles), tend = min(tbeg + per_run, n_tiles);
  DiffFold fold;  // of the first wave
  uint32_t row = 0u;
  for (uint32_t t = tbeg; t < tend; ++t) {
    Tile tile{0, 0, 0};
    if (lane < kTilePages) tile = tiles[t];
    const DiffUnit u = diff_unit(tile, lane, ushift, fences, rt, changed_bm, gold_zero_bm, rank_prefix, gold_page_va,
                                 n_valid, gold_packed);
    const uint32_t n_bad = (uint32_t)__popcll(__ballot(u.bad));
    if (wv == 0 && lane == 0u && u.a >= 0 && n_bad != 0u)  // the units of a tile share its range
      atomicAdd((unsigned long long*)&res[u.a].n_bad_pages, (unsigned long long)n_bad);
    const uint64_t need_mask = __ballot(u.need);  // the same in every wave
    if (need_mask == 0ull) continue;
    uint32_t* const s_off = unit_off[row];
    uint32_t* const s_first = unit_first[row];
    row ^= 1u;
    for (uint64_t m = need_mask; m != 0ull;) {  // two units at a time: 16 KiB in flight
      int32_t L[2];
      uint64_t pva[2], pgp[2];
      uint32_t plen[2], nd[2] = {0u, 0u}, fo[2] = {~0u, ~0u};  // bytes of the unit (a range's last may be partial)
      bool pz[2];
#pragma unroll
      for (uint32_t i = 0; i < 2; ++i) {
        L[i] = m ? __ffsll((long long)m) - 1 : 0;
        pva[i] = __shfl((unsigned long long)u.va, L[i], 64);
        pgp[i] = __shfl((unsigned long long)u.gp, L[i], 64);
        pz[i] = __shfl((int)u.zero, L[i], 64) != 0;
        plen[i] = m ? __shfl(u.len, L[i], 64) : 0u;
        m &= m - 1ull;
      }
      for (uint32_t o0 = wv * kPage; o0 < max(plen[0], plen[1]); o0 += wpb * kPage) {  // in address order
        uint4 c[8], d[8];
#pragma unroll
        for (uint32_t k = 0; k < 8; ++k) {
          const uint32_t i = k >> 2, off = o0 + (k & 3u) * 1024u + lane * 16u;
          c[k] = off < plen[i] ? clip16(ld16nt(pva[i] + off), off, plen[i]) : make_uint4(0, 0, 0, 0);
          d[k] = pz[i] || off >= plen[i] ? make_uint4(0, 0, 0, 0) : clip16(ld16nt(pgp[i] + off), off, plen[i]);
        }
#pragma unroll
        for (uint32_t k = 0; k < 8; ++k) add_diff(c[k], d[k], o0 + (k & 3u) * 1024u + lane * 16u, nd[k >> 2], fo[k >> 2]);
      }
#pragma unroll
      for (uint32_t i = 0; i < 2; ++i) {
        if (__ballot(nd[i] != 0u) == 0ull) continue;
        nd[i] = wave_sum_u32(nd[i]);
#pragma unroll
        for (int dd = 32; dd >= 1; dd >>= 1) fo[i] = min(fo[i], (uint32_t)__shfl_xor(fo[i], dd, 64));
        if (lane == 0) {
          atomicAdd(&s_off[L[i]], nd[i]);
          atomicMin(&s_first[L[i]], fo[i]);
        }
      }
    }
    __syncthreads();  // the one barrier per changed tile: sums two apart share a row
    if (wv != 0) continue;
    const uint32_t nd = s_off[lane], fo = s_first[lane];
    s_off[lane] = 0u;
    s_first[lane] = ~0u;
    const uint64_t diff = __ballot(nd != 0u);
    if (diff == 0ull) continue;
    const int32_t L = __ffsll((long long)diff) - 1;  // the lowest unit that differs: units ascend
    const uint64_t first = __shfl((unsigned long long)u.va, L, 64) + __shfl(fo, L, 64);
    fold.add(res, lane == 0, __shfl(u.a, L, 64), wave_sum_u32(nd), (uint64_t)__popcll(diff), first);  // 16 units of 2 MiB at most
  }
  if (threadIdx.x == 0) flush_region(res, fold.cur, fold.bytes, fold.pages, fold.first);
}

}  // namespace

hipError_t launch_pointer_graph(const Tile* tiles, uint32_t n_tiles, uint64_t lo, uint64_t span,
                                const RangeTable& rt, uint64_t* edge_bm, uint32_t row_words, uint32_t grid,
                                uint32_t n_cu, hipStream_t s) {
  if (n_tiles == 0) return hipSuccess;
  uint32_t blocks = 1, wpb = 1;
  wide_shape(std::min(grid, n_tiles), n_cu, &blocks, &wpb);  // grid counts waves
  hipLaunchKernelGGL(k_pointer_graph, dim3(blocks), dim3(wpb * kWave), wide_lds_bytes(rt), s, tiles, n_tiles, lo,
                     span, rt, edge_bm, row_words);
  return hipGetLastError();
}

hipError_t launch_region_init(kc_region_diff_result* res, uint32_t n, uint64_t* bm_a, uint64_t* bm_b, uint64_t n_words,
                              hipStream_t s) {
  const uint64_t m = std::max<uint64_t>(n, n_words);
  if (m == 0) return hipSuccess;
  const uint64_t nbk = blocks_for(m, 256);
  hipLaunchKernelGGL(k_region_init, dim3((uint32_t)(nbk < 4096 ? nbk : 4096)), dim3(256), 0, s, res, n, bm_a, bm_b,
                     n_words);
  return hipGetLastError();
}

hipError_t launch_region_diff(const Tile* tiles, uint32_t n_tiles, const RangeTable& rt, const uint64_t* changed_bm,
                              const uint64_t* gold_zero_bm, const uint64_t* rank_prefix, const uint64_t* gold_page_va,
                              const uint64_t* gold_n_kept, uint64_t cap, const uint8_t* gold_packed,
                              kc_region_diff_result* res, uint32_t ushift, uint32_t grid, uint32_t n_cu,
                              hipStream_t s) {
  if (n_tiles == 0) return hipSuccess;
  // grid counts waves.  Pages: a group of four tiles per wave at least, the waves of a workgroup few while there are few
  // of them.  Larger units: a wave for each 16 KiB of a unit, and two workgroups per CU at least.
  if (ushift == kMinUnitShift) {
    const uint32_t waves = std::max(1u, std::min(grid, blocks_for(n_tiles, 4u)));
    const uint32_t wpb = std::min(kDiffPageWaves, std::max(1u, waves / n_cu)), blocks = blocks_for(waves, wpb);
    hipLaunchKernelGGL(k_region_diff_pages, dim3(blocks), dim3(wpb * kWave), 0, s, tiles, n_tiles, rt, changed_bm,
                       gold_zero_bm, rank_prefix, gold_page_va, gold_n_kept, cap, gold_packed, res);
    return hipGetLastError();
  }
  const uint32_t wpb = std::max(1u, std::min(kDiffWaves, (1u << ushift) >> 14));
  const uint32_t blocks = std::max(1u, std::min(std::max(2u * n_cu, grid / wpb), n_tiles));
  hipLaunchKernelGGL(k_region_diff_units, dim3(blocks), dim3(wpb * kWave), 0, s, tiles, n_tiles, rt, changed_bm,
                     gold_zero_bm, rank_prefix, gold_page_va, gold_n_kept, cap, gold_packed, res, ushift);
  return hipGetLastError();
}

}  // namespace kc

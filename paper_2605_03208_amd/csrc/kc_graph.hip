// kc_graph.hip -- gfx950 kernels over the ranges beyond the snapshot itself:
// the pointer graph between ranges and the per-range byte difference against
// a snapshot.  Same execution model as the snapshot kernels: persistent grids
// of 64-lane waves over the 16-page tile list, range fences in LDS (the graph:
// up to eight waves per workgroup sharing the wide table; the region diff:
// one wave per workgroup).
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
  return (uint32_t)((x & 0xFFu) != 0u) + (uint32_t)((x & 0xFF00u) != 0u) + (uint32_t)((x & 0xFF0000u) != 0u) +
         (uint32_t)((x & 0xFF000000u) != 0u);
}

__device__ __forceinline__ void flush_region(kc_region_diff_result* res, int32_t a, uint64_t dbytes, uint64_t dpages,
                                             uint64_t first) {
  if (a < 0 || dbytes == 0) return;
  kc_region_diff_result* r = res + a;
  atomicAdd((unsigned long long*)&r->n_diff_bytes, (unsigned long long)dbytes);
  atomicAdd((unsigned long long*)&r->n_diff_pages, (unsigned long long)dpages);
  atomicMin((unsigned long long*)&r->first_diff_va, (unsigned long long)first);
}

// Groups of `tpg` consecutive tiles (four, one of units above 4 KiB) are taken
// one lane per unit: each lane resolves its unit's snapshot copy and changed bit,
// then the changed units are compared two at a time, and what differs is added up
// per unit in LDS.  SHARE (larger units): the waves of a workgroup share out the
// 4 KiB blocks of a unit.  Else each wave takes groups of its own.  Runs of
// groups are contiguous and folded per range, which touches a range's counters
// only when the run moves to the next range or ends (for the waves of a
// workgroup together, where they end in one range): folds that all add into one
// range's counters as they go queue on those addresses.  The bytes of the changed
// units bound it, and with few of them a chain of three round trips per group.
// Measured against one wave per unit, 2048 waves: 6.3 GiB in 2 MiB units with 5 %
// of the pages changed 25.0 -> 2.2 ms, 3.9 GiB in 64 KiB units with 1 % 0.53 ->
// 0.25 ms; pages: 2 GiB with 50 % changed 439 -> 394 us, 4.2 GiB in one range
// with 1 % 98 -> 65 us.
constexpr uint32_t kDiffWaves = 16, kDiffApart = 4;

template <bool SHARE>
__global__ __launch_bounds__((SHARE ? kDiffWaves : kDiffApart) * kWave) __attribute__((amdgpu_waves_per_eu(4))) void
k_region_diff(const Tile* tiles, uint32_t n_tiles, uint32_t tpg, RangeTable rt, const uint64_t* changed_bm,
              const uint64_t* gold_zero_bm, const uint64_t* rank_prefix, const uint64_t* gold_page_va,
              const uint64_t* gold_n_kept, uint64_t cap, const uint8_t* gold_packed, kc_region_diff_result* res,
              uint32_t ushift) {
  constexpr uint32_t kRows = SHARE ? 2u : kDiffApart;
  __shared__ FenceLds fences;
  __shared__ uint32_t unit_off[kRows][kWave], unit_first[kRows][kWave];  // of a group's units; SHARE: groups take turns
  __shared__ int32_t end_range[kDiffApart];  // where the runs of the waves end
  __shared__ uint64_t end_bytes[kDiffApart], end_pages[kDiffApart], end_first[kDiffApart];
  const uint32_t lane = threadIdx.x % kWave, sub = lane >> 4, j = lane & 15u, wpb = blockDim.x / kWave;
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t unit = 1u << ushift;
  load_fences(fences, rt, threadIdx.x, blockDim.x);
  if (wv < kRows) {
    unit_off[wv][lane] = 0u;
    unit_first[wv][lane] = ~0u;
  }
  if (SHARE && wpb == 1u) {
    unit_off[1][lane] = 0u;
    unit_first[1][lane] = ~0u;
  }
  __syncthreads();
  const uint64_t kept = *gold_n_kept;
  const uint64_t n_valid = kept < cap ? kept : cap;
  const uint32_t n_groups = (n_tiles + tpg - 1u) / tpg;
  const uint32_t n_runs = SHARE ? gridDim.x : gridDim.x * wpb, run = SHARE ? blockIdx.x : blockIdx.x * wpb + wv;
  const uint32_t per_run = (n_groups + n_runs - 1u) / n_runs;
  const uint32_t gbeg = min(run * per_run, n_groups), gend = min(gbeg + per_run, n_groups);
  int32_t cur = -1;  // the range being folded (SHARE: by the first wave), and its totals so far
  uint64_t dbytes = 0, dpages = 0, first = ~0ull;
  uint32_t row = SHARE ? 0u : wv;
  for (uint32_t gi = gbeg; gi < gend; ++gi) {
    const uint32_t t = gi * tpg + sub;
    Tile tile{0, 0, 0};
    if (sub < tpg && t < n_tiles) tile = tiles[t];
    const bool live = j < tile.npages;
    const uint64_t g = (uint64_t)tile.g + j, va = tile.va + ((uint64_t)j << ushift);
    bool zero = false, bad = false, need = false;
    uint64_t gp = 0;
    int32_t a = -1;
    const uint32_t len = live ? unit_bytes(tile, j, unit) : 0u;
    if (live) {
      a = range_index(va, fences, rt);
      const uint64_t zw = gold_zero_bm[g >> 6];
      zero = (zw >> (g & 63u)) & 1ull;
      if (!zero) {
        const uint64_t slot = rank_prefix[g >> 6] + (uint64_t)__popcll(~zw & ((1ull << (g & 63u)) - 1ull));
        bad = slot >= n_valid || gold_page_va[slot] != va;
        gp = (uint64_t)gold_packed + (slot << ushift);
      }
      need = !bad && ((changed_bm[g >> 6] >> (g & 63u)) & 1ull);
    }
    const uint64_t bad_mask = __ballot(bad);
    if ((!SHARE || wv == 0) && j == 0u && live && a >= 0) {  // the 16 lanes of a tile share its range
      const uint32_t nb = (uint32_t)__popcll((bad_mask >> (16u * sub)) & 0xFFFFull);
      if (nb) atomicAdd((unsigned long long*)&res[a].n_bad_pages, (unsigned long long)nb);
    }
    uint64_t need_mask = __ballot(need);  // SHARE: the same in every wave
    if (need_mask == 0ull) continue;
    uint32_t* const s_off = unit_off[row];
    uint32_t* const s_first = unit_first[row];
    if (SHARE) row ^= 1u;
    for (uint64_t m = need_mask; m != 0ull;) {  // two units at a time: 16 KiB in flight
      int32_t L[2];
      uint64_t pva[2], pgp[2];
      uint32_t plen[2], nd[2] = {0u, 0u}, fo[2] = {~0u, ~0u};  // bytes of the unit (a range's last may be partial)
      bool pz[2];
#pragma unroll
      for (uint32_t u = 0; u < 2; ++u) {
        L[u] = m ? __ffsll((long long)m) - 1 : 0;
        pva[u] = __shfl((unsigned long long)va, L[u], 64);
        pgp[u] = __shfl((unsigned long long)gp, L[u], 64);
        pz[u] = __shfl((int)zero, L[u], 64) != 0;
        plen[u] = m ? __shfl(len, L[u], 64) : 0u;
        m &= m - 1ull;
      }
      for (uint32_t o0 = SHARE ? wv * kPage : 0u; o0 < max(plen[0], plen[1]); o0 += SHARE ? wpb * kPage : kPage) {  // in address order
        uint4 c[8], d[8];
#pragma unroll
        for (uint32_t k = 0; k < 8; ++k) {
          const uint32_t u = k >> 2, off = o0 + (k & 3u) * 1024u + lane * 16u;
          c[k] = off < plen[u] ? clip16(ld16nt(pva[u] + off), off, plen[u]) : make_uint4(0, 0, 0, 0);
          d[k] = pz[u] || off >= plen[u] ? make_uint4(0, 0, 0, 0) : clip16(ld16nt(pgp[u] + off), off, plen[u]);
        }
#pragma unroll
        for (uint32_t k = 0; k < 8; ++k) {
          const uint32_t u = k >> 2, off = o0 + (k & 3u) * 1024u + lane * 16u;
          const uint32_t x[4] = {c[k].x ^ d[k].x, c[k].y ^ d[k].y, c[k].z ^ d[k].z, c[k].w ^ d[k].w};
#pragma unroll
          for (uint32_t i = 0; i < 4; ++i) {
            nd[u] += nonzero_bytes(x[i]);
            if (x[i] != 0u && fo[u] == ~0u) fo[u] = off + 4u * i + ((uint32_t)__builtin_ctz(x[i]) >> 3);
          }
        }
      }
#pragma unroll
      for (uint32_t u = 0; u < 2; ++u) {
        if (__ballot(nd[u] != 0u) == 0ull) continue;
        nd[u] = wave_sum_u32(nd[u]);
#pragma unroll
        for (int dd = 32; dd >= 1; dd >>= 1) {
          const uint32_t y = __shfl_xor(fo[u], dd, 64);
          fo[u] = y < fo[u] ? y : fo[u];
        }
        if (lane == 0) {
          atomicAdd(&s_off[L[u]], nd[u]);
          atomicMin(&s_first[L[u]], fo[u]);
        }
      }
    }
    if (SHARE) {
      __syncthreads();  // the one barrier per changed group: sums two apart share a row
      if (wv != 0) continue;
    }
    wave_lds_order();
    const uint32_t nd = s_off[lane], fo = s_first[lane];
    s_off[lane] = 0u;
    s_first[lane] = ~0u;
    for (uint64_t diff = __ballot(nd != 0u); diff != 0ull;) {
      const int32_t L = __ffsll((long long)diff) - 1;
      const int32_t pa = __shfl(a, L, 64);
      const uint64_t same = __ballot(nd != 0u && a == pa);
      if (pa != cur) {
        if (lane == 0) flush_region(res, cur, dbytes, dpages, first);
        cur = pa;
        dbytes = dpages = 0;
        first = ~0ull;
      }
      dbytes += wave_sum_u32(a == pa ? nd : 0u);  // 64 units of 2 MiB at most
      dpages += (uint64_t)__popcll(same);
      if (first == ~0ull) first = __shfl((unsigned long long)va, L, 64) + __shfl(fo, L, 64);  // units ascend
      diff &= ~same;
    }
  }
  if (SHARE) {
    if (threadIdx.x == 0) flush_region(res, cur, dbytes, dpages, first);
    return;
  }
  if (lane == 0) {
    end_range[wv] = cur;
    end_bytes[wv] = dbytes;
    end_pages[wv] = dpages;
    end_first[wv] = first;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (uint32_t w = 1; w < wpb; ++w) {  // the next wave's run follows: its range is this one or a later one
    if (end_range[w] < 0) continue;
    if (end_range[w] != cur) {
      flush_region(res, cur, dbytes, dpages, first);
      cur = end_range[w];
      dbytes = dpages = 0;
      first = ~0ull;
    }
    dbytes += end_bytes[w];
    dpages += end_pages[w];
    first = min(first, end_first[w]);
  }
  flush_region(res, cur, dbytes, dpages, first);
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
  // Pages: four waves per workgroup, each with runs of four tiles.  Larger units, which are few: a tile at a time, a
  // wave for each 16 KiB of a unit, eight waves per CU and two workgroups at least.  grid counts waves.
  if (ushift == kMinUnitShift) {
    const uint32_t blocks = std::max(1u, std::min(blocks_for(grid, kDiffApart), blocks_for(n_tiles, 4u * kDiffApart)));
    hipLaunchKernelGGL((k_region_diff<false>), dim3(blocks), dim3(kDiffApart * kWave), 0, s, tiles, n_tiles, 4u, rt,
                       changed_bm, gold_zero_bm, rank_prefix, gold_page_va, gold_n_kept, cap, gold_packed, res, ushift);
    return hipGetLastError();
  }
  const uint32_t wpb = std::max(1u, std::min(kDiffWaves, (1u << ushift) >> 14));
  const uint32_t blocks = std::max(1u, std::min(std::max(2u * n_cu, grid / wpb), n_tiles));
  hipLaunchKernelGGL((k_region_diff<true>), dim3(blocks), dim3(wpb * kWave), 0, s, tiles, n_tiles, 1u, rt, changed_bm,
                     gold_zero_bm, rank_prefix, gold_page_va, gold_n_kept, cap, gold_packed, res, ushift);
  return hipGetLastError();
}

}  // namespace kc

// kc_hash.hip -- the hashing pass: XXH64 of every hash unit (4 KiB pages, or
// units of 8 KiB to 2 MiB), with the zero / changed bits, the packed copy of a
// full snapshot and the closure scan riding on the same read of the data.
#include <algorithm>

#include "kc_device.h"
#include "kc_internal.h"
#include "kc_xxh64.h"

namespace kc {
namespace {

constexpr uint32_t kOutside = 0x80000000u;  // an offset beyond any resource made here (tiles are below 64 MiB)

constexpr uint32_t kRoundLoads = 16;        // 1 KiB runs a wave loads per round
constexpr uint32_t kHashWaves = 4;          // most waves per workgroup
constexpr uint32_t kLdsBytes = 160u << 10;  // of a CU
constexpr uint64_t kMaxThreads = (1ull << 32) - 1;  // of a launch

// marks = 2 * marks + (d <= span), in two instructions.
__device__ __forceinline__ void mark_high(uint32_t& marks, uint32_t d, uint32_t span) {
  asm("v_cmp_ge_u32_e32 vcc, %1, %2\n\tv_addc_co_u32_e32 %0, vcc, %0, %0, vcc"
      : "+v"(marks)
      : "s"(span), "v"(d)
      : "vcc");
}

// The same of words: marks = 2 * marks + (d < span).
__device__ __forceinline__ void mark_word(uint32_t& marks, uint64_t d, uint64_t span) {
  asm("v_cmp_gt_u64_e32 vcc, %1, %2\n\tv_addc_co_u32_e32 %0, vcc, %0, %0, vcc"
      : "+v"(marks)
      : "s"(span), "v"(d)
      : "vcc");
}

// Units kept (zero bit clear) among the first n, at most 64 * kInlineWords: all words loaded at once.
__device__ __forceinline__ uint32_t kept_before(const uint64_t* zero_bm, uint32_t n, uint32_t lane) {
  constexpr uint32_t kEach = kInlineWords / kWave;
  typedef unsigned int v2u __attribute__((ext_vector_type(2)));
  const __amdgpu_buffer_rsrc_t src = raw_rsrc((uint64_t)zero_bm, (n + 63u) / 64u * 8u);
  v2u w[kEach];
#pragma unroll
  for (uint32_t i = 0; i < kEach; ++i) w[i] = __builtin_amdgcn_raw_buffer_load_b64(src, (i * kWave + lane) * 8u, 0, 0);
  uint32_t kept = 0;
#pragma unroll
  for (uint32_t i = 0; i < kEach; ++i) {
    const uint32_t u = (i * kWave + lane) * 64u;  // the word's first unit
    const uint64_t mine = u >= n ? 0ull : n - u >= 64u ? ~0ull : (1ull << (n - u)) - 1ull;
    kept += (uint32_t)__popcll(~(((uint64_t)w[i][1] << 32) | w[i][0]) & mine);
  }
  return wave_sum_u32(kept);
}

// One wave hashes up to ROWS units of a tile: lane quad q takes unit (row) q,
// lane k of the quad runs XXH64 accumulator k over the words 8k + 32s of each
// stripe s (the four accumulators are serial over a unit, so a unit never takes
// more than four lanes).  A round takes one chunk of every row, 16 KiB in all:
// 16 loads, each one 1 KiB run of one row, go to the row of an LDS stage (and to
// the unit's packed slot), the loads of the next round are issued, and the quads
// hash their chunks from the stage.  With 16 rows (1 KiB chunks) every quad
// works.  With 8 or 4, the quads without a row repeat the last one's work, but
// there are twice or four times the waves, and a round takes 2 or 4 KiB of a
// row: which shape when, with figures, at hash_rows in kc_api.hip.
//
// What bounds it: memory, while there are waves enough (5.9 TB/s read and
// written, 6.5 read only); with few and long units, a wave's chain of rounds,
// each a wait for memory, a pass through LDS and a serial run of 64-bit
// multiplies.
//
// A load belongs to one row, so whether its unit is kept and where its packed
// slot lies are settled once per tile.  The loads and stores go through buffer
// resources bounded to the tile's bytes and to its kept units' packed slots, so
// no lane branches around a memory access (a branch that may skip one leaves the
// compiler unsure how many are in flight, and it then waits for all of them):
// zero units of a full snapshot and missing rows use an offset outside the
// resource.  A partial last unit needs no launch of its own: its last 16-byte
// block is read whole and cleared past the end when staged.
//
// The rows of a round lie a unit apart and are read in step, which costs nothing
// on this memory: a copy that reads 16 rows 64 KiB apart, 1 KiB of each in turn,
// ran at 5.6 TB/s, one that reads the same bytes in address order at 5.3; with
// rows kept some chunks behind each other 5.1, and idle quads at both ends.
//
// GATHER: zero bits come from the probe, zero units are not read (their hash
// is computed from zeros), kept units are also stored to their packed slots.
// SCAN (a closure scan rides on the pass), kScanHigh: words whose upper half lies
// in the window's are marked (three instructions a word); once a round is
// staged, the marked ones get the exact test, and pointer-like words go to the wave's queue (PtrQueue) with the
// 4 KiB-page scan tile they lie in, where out-of-range ones are counted.  kScanWord, for windows that reach below 4 GiB: every zero and every
// small integer has such an upper half, and the steps over those marks took more
// than the pass (2 GiB of zeros, window from 4096: 590 us, 370 with the words
// themselves marked).  For other windows that costs small snapshots (64 MiB: 50.9
// -> 52.5 us).
//
// The waves of a workgroup are independent; with the closure scan they share
// one range table.  LDS, all dynamic: the table, then per wave its stage,
// a partial unit's last bytes and the queue (hash_lds_per_wave).
constexpr uint32_t kHashQueue = 128;  // below 64 left over, and up to 64 of one push
__host__ __device__ constexpr uint32_t stage_stride(uint32_t rows) {
  return kRoundLoads / rows * 1024u + 32u;  // a chunk, padded: the quads' rows fall in distinct banks
}
__host__ __device__ constexpr uint32_t hash_lds_per_wave(uint32_t rows, bool scan) {
  return rows * (stage_stride(rows) + 32u) + (scan ? kHashQueue * 10u : 0u);
}

enum ScanKind : uint32_t { kNoScan = 0, kScanHigh = 1, kScanWord = 2 };

template <bool GATHER, bool PRIOR, uint32_t SCAN, uint32_t ROWS>
__global__ __launch_bounds__(kHashWaves * kWave) __attribute__((amdgpu_waves_per_eu(2))) void k_page_hash(
    HashParams p) {
  constexpr uint32_t kPer = kRoundLoads / ROWS;  // loads per row and round
  constexpr uint32_t kChunk = kPer * 1024u, kStripes = kChunk / 32u;
  constexpr uint32_t kStride = stage_stride(ROWS);
  const uint32_t lane = threadIdx.x % kWave, wpb = blockDim.x / kWave;
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t table = SCAN ? 16u * p.scan.rt.n_fence_w + 2u * kBuckets : 0u;
  uint8_t* const stage = reinterpret_cast<uint8_t*>(kc_wide_lds) + table + wv * hash_lds_per_wave(ROWS, SCAN != kNoScan);
  // a partial unit's bytes past its last whole stripe
  uint64_t(*const tail_lds)[4] = reinterpret_cast<uint64_t(*)[4]>(stage + ROWS * kStride);
  uint64_t* const queue_lds = reinterpret_cast<uint64_t*>(tail_lds + ROWS);
  const uint32_t k = lane & 3u, lane16 = lane * 16u;
  const uint32_t q = min(lane >> 2, ROWS - 1u);  // this lane's row
  const uint32_t ushift = p.ushift, unit = 1u << ushift;
  bool table_in = false;  // the same in every wave at the barrier: each gets there once, whether it has items or not
  auto load_table = [&] {
    load_wide_fences(p.scan.rt, threadIdx.x, blockDim.x);
    __syncthreads();  // the only workgroup barrier: the waves share nothing else
    table_in = true;
  };
  if (SCAN && !GATHER) load_table();
  uint32_t n_ptr = 0, n_in = 0;  // of this lane
  // the window's upper halves: a word whose upper half is not among them is not pointer-like
  const uint32_t win_hi = (uint32_t)(p.scan.lo >> 32);
  const uint32_t win_span = (uint32_t)((p.scan.lo + p.scan.span - 1ull) >> 32) - win_hi;
  const uint64_t n_items = (uint64_t)p.n_tiles << p.sub_shift;  // 1 << sub_shift parts of ROWS units per tile
  for (uint64_t it = (uint64_t)blockIdx.x * wpb + wv; it < n_items; it += (uint64_t)gridDim.x * wpb) {
    const uint32_t t = (uint32_t)(it >> p.sub_shift), first = ((uint32_t)it & ((1u << p.sub_shift) - 1u)) * ROWS;
    const Tile tile = const_load(p.tiles + t);
    if (first >= tile.npages) continue;
    const uint32_t np = min(tile.npages - first, ROWS);  // 1 .. ROWS units
    const uint32_t g0 = tile.g + first;
    const uint64_t va = tile.va + ((uint64_t)first << ushift);
    // only the tile's last unit can be partial
    const uint32_t last = np - 1u, last_len = first + np == tile.npages ? (uint32_t)tile.last_len : unit;
    const bool partial = last_len != unit;
    const uint32_t valid = (1u << np) - 1u;
    uint32_t keep = valid;
    __amdgpu_buffer_rsrc_t dst = raw_rsrc((uint64_t)p.packed, 0u);  // no slots: every store dropped
    if (GATHER) {
      uint64_t slot = 0;
      bool kept = false;
      if (lane < np) {
        const uint64_t g = (uint64_t)g0 + lane;
        const uint64_t zw = p.zero_bm[g >> 6];
        kept = ((zw >> (g & 63u)) & 1ull) == 0ull;
        if (p.word_prefix) slot = p.word_prefix[g >> 6] + (uint64_t)__popcll(~zw & ((1ull << (g & 63u)) - 1ull));
      }
      if (!p.word_prefix) {  // few words: their kept units are counted here
        slot = kept_before(p.zero_bm, g0, lane) + (uint32_t)__popcll(__ballot(kept) & ((1ull << lane) - 1ull));
      }
      keep = (uint32_t)__ballot(kept);
      if (kept && slot < p.cap_pages) p.page_va[slot] = va + ((uint64_t)lane << ushift);
      // the tile's kept units have consecutive slots from the first one's; those below the capacity are written
      const uint64_t slot0 = __shfl(slot, keep ? __builtin_ctz(keep) : 0, 64);
      const uint64_t n_kept = (uint64_t)__popc(keep);
      const uint64_t room = slot0 < p.cap_pages ? min(n_kept, p.cap_pages - slot0) : 0ull;
      dst = raw_rsrc((uint64_t)p.packed + (slot0 << ushift), (uint32_t)(room << ushift));
    }
    uint64_t prior_l = 0;  // lane i < np: unit i's prior hash
    if (PRIOR && lane < np) prior_l = p.prior[g0 + lane];
    // the tile's bytes, the last 16-byte block of a partial unit included
    const __amdgpu_buffer_rsrc_t src = raw_rsrc(va, ((last << ushift) + last_len + 15u) & ~15u);
    // each row's first byte in the tile and in the packed slots (kOutside: not read, not stored)
    uint32_t from[ROWS], to[ROWS];
#pragma unroll
    for (uint32_t r = 0; r < ROWS; ++r) {
      const bool on = ((keep >> r) & 1u) != 0u;
      from[r] = on ? r << ushift : kOutside;
      to[r] = on ? (uint32_t)__popc(keep & ((1u << r) - 1u)) << ushift : kOutside;
    }
    // rounds: to the end of the units; with nothing to store, only to the end of the bytes
    const uint32_t n_rounds = (!GATHER && np == 1u ? last_len + kChunk - 1u : unit) / kChunk;
    uint4 cur[kRoundLoads];
    auto load = [&](uint32_t c) {
#pragma unroll
      for (uint32_t i = 0; i < kRoundLoads; ++i) {
        const v4u x = __builtin_amdgcn_raw_buffer_load_b128(
            src, from[i / kPer] + c * kChunk + (i % kPer) * 1024u + lane16, 0, kNt);
        cur[i] = make_uint4(x[0], x[1], x[2], x[3]);
      }
    };
    // this lane's row: its bytes, whole stripes and the bytes past them
    const uint32_t qlen = q == last ? last_len : unit;
    const uint32_t lim = qlen / 32u, rem = qlen & 31u;
    uint32_t nonzero = 0;  // bit i: unit i holds a non-zero byte
    uint64_t acc = acc_init(p.seed, k);
    PtrQueue queue{queue_lds, reinterpret_cast<uint16_t*>(queue_lds + kHashQueue)};
    // the scan tile of these units' first byte: with 4 KiB units the tile itself
    uint32_t scan0 = p.tile0 + t;
    if (SCAN && p.scan0) scan0 = const_load32(p.scan0 + t) + ((first << ushift) >> 16);
    // Out-of-range words are added once per scan tile among the lanes (an atomic per word queued on the tile's address:
    // 2 GiB of nothing but such words 33 ms, so 1.6).
    auto search = [&](uint64_t w, uint32_t tag) {
      const bool out = wide_range_index(w, p.scan.rt) < 0;
      n_in += out ? 0u : 1u;
      for (uint64_t m = __ballot(out); m != 0ull;) {
        const uint32_t leader = (uint32_t)__builtin_ctzll(m), its = __builtin_amdgcn_readlane(tag, leader);
        const uint64_t same = __ballot(out && tag == its);
        if (lane == leader) atomicAdd(&p.scan.tile_oob[scan0 + its], (uint32_t)__popcll(same));
        m &= ~same;
      }
    };
    load(0u);
    // Snapshots load the table while the first loads are under way (8 GiB 2.78 ms, table first 2.85); for the others
    // it goes first (1.39 ms, else 1.42).
    if (SCAN && GATHER && !table_in) load_table();
#pragma unroll 1
    for (uint32_t c = 0; c < n_rounds; ++c) {
      uint32_t marks = 0;  // bit 31 - (2i + h): word h of this lane's 16 bytes of run i may be pointer-like
#pragma unroll
      for (uint32_t i = 0; i < kRoundLoads; ++i) {
        const uint32_t r = i / kPer, o = c * kChunk + (i % kPer) * 1024u;  // this run's place in its unit
        uint4 v = cur[i];  // zeros where the load was outside
        const bool part = partial && r == last;
        if (part) v = clip16(v, o + lane16, last_len);  // the partial unit's bytes past its end
        if (!GATHER && __ballot(nz16(v)) != 0ull) nonzero |= 1u << r;
        if (SCAN) {
          if (SCAN == kScanWord) {
            mark_word(marks, (((uint64_t)v.y << 32) | v.x) - p.scan.lo, p.scan.span);
            mark_word(marks, (((uint64_t)v.w << 32) | v.z) - p.scan.lo, p.scan.span);
          } else {
            mark_high(marks, v.y - win_hi, win_span);
            mark_high(marks, v.w - win_hi, win_span);
          }
        }
        if (GATHER) {  // a partial unit's slot: zeros after its bytes
          const v4u x = {v.x, v.y, v.z, v.w};
          __builtin_amdgcn_raw_buffer_store_b128(x, dst, to[r] + o + lane16, 0, kNt);
        }
        *reinterpret_cast<uint4*>(stage + r * kStride + (i % kPer) * 1024u + lane16) = v;
      }
      wave_lds_order();
      // All of the next round's loads at once, after all of this round's stores: issued one by one as each run's
      // registers fell free, between the stores, the pass over 30 GiB took 12.0 ms instead of 11.2.
      if (c + 1u < n_rounds) load(c + 1u);
      while (SCAN && __ballot(marks != 0u) != 0ull) {  // the marked words, read back from the stage
        const bool marked = marks != 0u;
        const uint32_t b = marked ? 31u - (uint32_t)__builtin_ctz(marks) : 0u;
        const uint32_t i = b >> 1, r = i / kPer, in_row = (i % kPer) * 1024u, o = c * kChunk + in_row;
        const uint64_t w = *reinterpret_cast<const uint64_t*>(stage + r * kStride + in_row + lane16 + (b & 1u) * 8u);
        // words wholly inside the range only
        const bool inside = !partial || r != last || o + lane16 + (b & 1u) * 8u + 8u <= last_len;
        const bool hit = marked && (w - p.scan.lo) < p.scan.span && inside;
        n_ptr += hit ? 1u : 0u;
        queue.push(hit, w, p.scan0 ? ((r << ushift) + o) >> 16 : 0u);
        if (queue.n >= kWave) queue.drain(false, search);
        marks &= marks - 1u;
      }
      const uint8_t* row = stage + q * kStride + k * 8u;
      // The words of the next kBatch stripes are read while these are hashed: left to itself the compiler reads
      // two at a time and waits for them, 200 cycles a stripe instead of 50.
      constexpr uint32_t kBatch = 16;
      uint64_t w[kBatch], nxt[kBatch];
      auto read = [&](uint64_t (&x)[kBatch], uint32_t s0) {
#pragma unroll
        for (uint32_t s = 0; s < kBatch; ++s) x[s] = *reinterpret_cast<const uint64_t*>(row + (s0 + s) * 32u);
      };
      auto each_batch = [&](auto hash) {
        read(w, 0u);
#pragma unroll 1
        for (uint32_t s0 = 0; s0 < kStripes; s0 += 2u * kBatch) {
          read(nxt, s0 + kBatch);
          wave_lds_order();
          hash(w, s0);
          if (s0 + 2u * kBatch < kStripes) read(w, s0 + 2u * kBatch);
          wave_lds_order();
          hash(nxt, s0 + kBatch);
        }
      };
      if (!partial || (c + 1u) * kStripes <= last_len / 32u) {  // every row holds a whole chunk
        each_batch([&](const uint64_t (&x)[kBatch], uint32_t) {
#pragma unroll
          for (uint32_t s = 0; s < kBatch; ++s) acc = xround(acc, x[s]);
        });
      } else {  // the partial unit's row ends in this chunk or has ended: its lanes keep their accumulators
        const uint32_t done = c * kStripes, s_end = lim > done ? min(lim - done, kStripes) : 0u;
        each_batch([&](const uint64_t (&x)[kBatch], uint32_t s0) {
#pragma unroll
          for (uint32_t s = 0; s < kBatch; ++s) {
            const uint64_t next = xround(acc, x[s]);
            acc = s0 + s < s_end ? next : acc;
          }
        });
        if (rem != 0u && c == lim / kStripes)  // a partial unit's last bytes are in this chunk
          tail_lds[q][k] = *reinterpret_cast<const uint64_t*>(row + (lim - done) * 32u);
      }
      wave_lds_order();
    }
    const uint64_t merged = xxh64_merge4(acc, k);  // every lane of the quad takes part
    uint64_t h = (lim > 0u ? merged : p.seed + kP5) + qlen;
    if (partial && rem != 0u) {
      const uint64_t tail[4] = {tail_lds[q][0], tail_lds[q][1], tail_lds[q][2], tail_lds[q][3]};
      h = xxh64_tail(h, tail, rem);
    }
    h = xxh64_avalanche(h);
    h = __shfl(h, (int)(min(lane, ROWS - 1u) * 4u), 64);  // unit i's hash to lane i
    if (SCAN) queue.drain(true, search);
    if (lane < np) p.hash[g0 + lane] = h;
    if (!GATHER) {
      const uint32_t zero = ~nonzero & valid;
      if (lane == 0) or_page_bits(p.zero_bm, g0, np, zero);
    }
    if (PRIOR) {
      const uint32_t ch = (uint32_t)__ballot(lane < np && h != prior_l);
      if (lane == 0) or_page_bits(p.changed_bm, g0, np, ch);
    }
  }
  if (GATHER && !p.word_prefix && blockIdx.x == 0 && wv == 0) {  // with the prefixes goes the total
    const uint32_t n = kept_before(p.zero_bm, (uint32_t)p.n_units, lane);
    if (lane == 0) *p.n_kept = n;
  }
  if (SCAN) {
    if (!table_in) load_table();
    const uint32_t a = wave_sum_u32(n_ptr), b = wave_sum_u32(n_in);
    if (lane == 0) add_scan_counts(p.scan.counts, blockIdx.x * wpb + wv, a, b);
  }
}

}  // namespace

hipError_t launch_page_hash(HashParams p, bool gather, bool prior, bool scan, uint32_t rows, uint32_t grid,
                            uint32_t n_cu, hipStream_t s) {
  const uint64_t n_items = (uint64_t)p.n_tiles << p.sub_shift;
  if (n_items == 0) return hipSuccess;
  // The table of up to 256 fences (6 KiB at most) serves the scan: what a larger one saves in searches, it costs in
  // waves per CU and in loading.  Hash only, 2 GiB in 4096 ranges, 1 % pointers 385 us, with 4096 fences 504; 2 GB in
  // 1422 ranges, 0.1 % pointers 331 / 377; snapshots of the first 745 / 858.
  RangeTable& rt = p.scan.rt;
  rt.bucket_w = rt.bucket;
  rt.stride_w = rt.stride;
  rt.n_fence_w = rt.n_fence;
  // Waves per workgroup: one while there are few, which spreads them over the SIMDs (1 GiB in 512 KiB units, 520 waves:
  // 0.73 ms, in pairs 0.92; with a scan 0.82 / 1.01), else four (30 GiB of 4 KiB pages, hash only: 4.69 ms; one by one
  // 4.82), which with a scan share the range table.
  const uint32_t per = hash_lds_per_wave(rows, scan), table = scan ? (uint32_t)wide_lds_bytes(rt) : 0u;
  uint64_t waves = grid == 0u ? n_items : std::min<uint64_t>(grid, n_items);  // 0: one item per wave
  uint32_t wpb = 4;
  if (waves <= (scan ? 4ull : 8ull) * n_cu) wpb = 1;
  const size_t lds = table + (size_t)wpb * per;
  // Hash only with a scan: the waves that fit on the chip stride over the tiles and load the table once (the 2 GiB
  // above: 385 us, one item per wave 474; 1 GiB in 100 ranges 200 / 206).  Snapshots stay in address order (1 GiB
  // 348 us, striding 401).
  if (grid == 0u && scan && !gather) waves = std::min(waves, (uint64_t)(kLdsBytes / lds) * wpb * n_cu);
  const uint32_t blocks = (uint32_t)std::min<uint64_t>((waves + wpb - 1) / wpb, kMaxThreads / (wpb * kWave));
  const uint32_t kind = !scan ? kNoScan : (p.scan.lo >> 32) != 0ull ? kScanHigh : kScanWord;
#define KC_HASH_CASE(G, P, S, N)                                                                     \
  if (gather == G && prior == P && kind == S && rows == N) {                                         \
    hipLaunchKernelGGL((k_page_hash<G, P, S, N>), dim3(blocks), dim3(wpb * kWave), lds, s, p);       \
    return hipGetLastError();                                                                        \
  }
#define KC_HASH_CASES(N)                  \
  KC_HASH_CASE(false, false, kNoScan, N)   \
  KC_HASH_CASE(false, false, kScanHigh, N) \
  KC_HASH_CASE(false, false, kScanWord, N) \
  KC_HASH_CASE(false, true, kNoScan, N)    \
  KC_HASH_CASE(false, true, kScanHigh, N)  \
  KC_HASH_CASE(false, true, kScanWord, N)  \
  KC_HASH_CASE(true, false, kNoScan, N)    \
  KC_HASH_CASE(true, false, kScanHigh, N)  \
  KC_HASH_CASE(true, false, kScanWord, N)
  KC_HASH_CASES(16u)
  KC_HASH_CASES(8u)
  KC_HASH_CASES(4u)
#undef KC_HASH_CASES
#undef KC_HASH_CASE
  return hipErrorInvalidValue;
}

}  // namespace kc

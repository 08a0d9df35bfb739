// ckv_score.hpp -- retrieval scoring of one tile of positions (MFMA path).
//
// The paper scores offloaded entries by the query's inner product with
// GPU-resident key summaries (Sec. 2.2, Sec. 4.1); with a summary per
// position the scan reads every key of the context once.  One KV head serves
// a group of G query heads, so the scores of a 16-key block form the dense
// product Q[16 x d] . K^T[d x 16] (heads padded to 16 rows), which is what a
// v_mfma_f32_16x16x32_bf16 computes in four steps over d = 128 channels.
//
// Operand placement (wave64): lane l holds key (l % 16) of the block as the B
// operand and query head (l % 16) as the A operand; lane group kg = l / 16
// supplies channels [32t + 8kg, 32t + 8kg + 8) of step t.  The accumulator of
// lane l then holds heads 4kg..4kg+3 of key (l % 16).
#pragma once

#include "ckv_device.hpp"

namespace ckv {

// Adds the workgroup's LDS histogram into the unit's global fine and coarse
// histograms (NT threads, kHistBins bins, kBinsPerThread each).
template <int NT = kScoreThreads>
__device__ __forceinline__ void flush_hist(const uint32_t* lds_hist,
                                           uint32_t* g_hist,
                                           uint32_t* g_coarse) {
  constexpr int kBinsPerThread = kHistBins / NT;
  constexpr int kThreadsPerCoarse = kHistBins / kCoarseBins / kBinsPerThread;
  const int t = threadIdx.x;
  uint32_t csum = 0;
#pragma unroll
  for (int i = 0; i < kBinsPerThread; ++i) {
    const uint32_t v = lds_hist[kBinsPerThread * t + i];
    if (v) {
      atomicAdd(&g_hist[kBinsPerThread * t + i], v);
      csum += v;
    }
  }
#pragma unroll
  for (int o = 1; o < kThreadsPerCoarse; o <<= 1) csum += __shfl_xor(csum, o);
  if ((t % kThreadsPerCoarse) == 0 && csum) atomicAdd(&g_coarse[t / kThreadsPerCoarse], csum);
}

// Stores the workgroup's LDS histogram as its slot (NT threads).
template <int NT = kScoreThreads>
__device__ __forceinline__ void store_hist(const uint32_t* lds_hist, uint32_t* slot) {
  constexpr int kPer = kHistBins / NT;
  static_assert(kPer % 4 == 0, "16-byte stores");
  const int t = threadIdx.x;
#pragma unroll
  for (int i = 0; i < kPer; i += 4)
    *reinterpret_cast<uint4*>(slot + kPer * t + i) =
        *reinterpret_cast<const uint4*>(lds_hist + kPer * t + i);
}

// The workgroup's LDS histogram as its slot, device-coherent, 8 bytes per lane
// with consecutive lanes on consecutive words (NT threads).
template <int NT>
__device__ __forceinline__ void store_hist_coherent(const uint32_t* lds_hist, uint32_t* slot) {
  constexpr int kPairs = kHistBins / NT / 2;
  const int t = threadIdx.x;
#pragma unroll
  for (int q = 0; q < kPairs; ++q) {
    const int i = 2 * (t + NT * q);
    const uint64_t w = (uint64_t)lds_hist[i] | ((uint64_t)lds_hist[i + 1] << 32);
    __hip_atomic_store(reinterpret_cast<uint64_t*>(slot + i), w, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Scores of one staged group (kStageRows keys of one unit starting at row
// jb) into out[0, kStageRows): the MFMA products with the G query rows, the
// maximum over the heads, the scale; rows at or past n get -inf and are not
// counted.  If HIST, counts the first radix digit of the others in lds_hist.
// TWO: rows [G, 2G) of the products are a second query's, whose scores go to
// out[stride2 ..] and are counted in the next kHistBins bins.
template <int G, bool HIST, bool TWO = false>
__device__ __forceinline__ void score_group(const uint32_t* stage, const bf16x8* qa, int jb,
                                            int n, float scale, uint32_t* lds_hist,
                                            float* out, int stride2 = 0) {
  const int lane = threadIdx.x & 63;
  const int r16 = lane & 15, kg = lane >> 4;
  // with two queries each lane's result is set `set`'s: both in the first 32
  // lanes, or with 2G = 16 rows, after one exchange, in lanes 0..15 and 32..47
  const int set = TWO ? (G == 8 ? lane >> 5 : (lane >> 4) & 1) : 0;
  const bool writer = TWO ? (G == 8 ? (lane & 16) == 0 : lane < 32) : lane < 16;
#pragma unroll
  for (int u = 0; u < kStageRows / 16; ++u) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f}, acc2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const uint4 kv = *reinterpret_cast<const uint4*>(
          stage + (16 * u + r16) * kStageRowDwords + 4 * (4 * t + kg));
      acc = mfma_16x16x32(qa[t], as_bf16x8(kv), acc);
      if (TWO && G == 16) acc2 = mfma_16x16x32(qa[4 + t], as_bf16x8(kv), acc2);
    }
    float sc = -INFINITY;
    if constexpr (TWO && G <= 2) {  // both queries' rows in lane group 0
      float s1 = -INFINITY;
#pragma unroll
      for (int i = 0; i < G; ++i) {
        sc = fmaxf(sc, acc[i]);
        s1 = fmaxf(s1, acc[G + i]);
      }
      s1 = __shfl(s1, r16);
      sc = set ? s1 : sc;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (4 * kg + i < (TWO && G < 16 ? 2 * G : G)) sc = fmaxf(sc, acc[i]);
      if (G > 4) sc = fmaxf(sc, __shfl_xor(sc, 16));
      if (G > 8) sc = fmaxf(sc, __shfl_xor(sc, 32));
      if constexpr (TWO && G == 16) {
        float s1 = fmaxf(fmaxf(acc2[0], acc2[1]), fmaxf(acc2[2], acc2[3]));
        s1 = fmaxf(s1, __shfl_xor(s1, 16));
        s1 = fmaxf(s1, __shfl_xor(s1, 32));
        sc = set ? s1 : sc;
      }
    }
    sc *= scale;
    const int j = jb + 16 * u + (TWO ? r16 : lane);
    if (writer) {
      if (j < n) {
        if (HIST)
          atomicAdd(&lds_hist[set * kHistBins + (order_key(sc) >> (32 - kHistBits))], 1u);
      } else {
        sc = -INFINITY;
      }
      out[set * stride2 + 16 * u + (TWO ? r16 : lane)] = sc;
    }
  }
}

// The G query rows of a unit as MFMA A operands (rows past G are zero); TWO:
// the second query's rows follow as rows [G, 2G), or, at G = 16, as a second
// operand (qa[4..7]).
template <int G, bool TWO = false>
__device__ __forceinline__ void load_query(const ScoreArgs& a, int unit, bf16x8* qa) {
  const int lane = threadIdx.x & 63;
  const int r16 = lane & 15, kg = lane >> 4;
  const int b = unit / a.Hkv, h = unit - b * a.Hkv;
  const int64_t row0 = (int64_t)b * a.Hq + (int64_t)h * G;
  constexpr int kRows = TWO && G < 16 ? 2 * G : G;
  const bool second = TWO && G < 16 && r16 >= G;
  const uint16_t* qrow = (second ? a.q2 : a.q) + (row0 + (second ? r16 - G : r16)) * kD + 8 * kg;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (r16 < kRows) v = ld16(qrow + 32 * t);
    qa[t] = as_bf16x8(v);
  }
  if constexpr (TWO && G == 16) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
      qa[4 + t] = as_bf16x8(ld16(a.q2 + (row0 + r16) * kD + 8 * kg + 32 * t));
  }
}

// Scores of the groups past the units' last valid ones: -inf, in equal shares
// of the stored groups (all threads of the workgroup; only score_keys, whose
// output has those rows, needs them).  Each lane looks at one group, so that a
// batch without such groups pays for little more than one look at the lengths;
// then eight lanes write each group found, one 128-byte line.
__device__ __forceinline__ void fill_tails(const ScoreArgs& a, int wg, int nwg) {
  static_assert(kStageRows == 32, "eight lanes of four rows per group");
  const int lane = threadIdx.x & 63;
  const uint32_t gu = groups_of(a.max_ctx);
  const uint32_t total = (uint32_t)a.units * gu;
  const uint32_t share = (total + (uint32_t)nwg - 1u) / (uint32_t)nwg;
  const uint32_t t0 = (uint32_t)wg * share, t1 = min(t0 + share, total);
  for (uint32_t tw = t0 + threadIdx.x - lane; tw < t1; tw += blockDim.x) {  // wave-uniform
    const uint32_t t = min(tw + lane, t1 - 1u), unit = t / gu;
    const int g = (int)(t - unit * gu);
    const int n = unit_len(a.ctx_lens[unit / (uint32_t)a.Hkv], a.max_ctx, a.chunk);
    const uint64_t tails = __ballot(tw + lane < t1 && g >= (int)groups_of(n));
    if (!tails) continue;
#pragma unroll
    for (int r = 0; r < 64; r += 8) {
      const int src = r + (lane >> 3);
      if (!((tails >> r) & 0xffu)) continue;  // uniform
      const int64_t row = (int64_t)__shfl((int)unit, src) * a.max_ctx;
      const int j = __shfl(g, src) * kStageRows + 4 * (lane & 7);
      if (!((tails >> src) & 1u)) continue;
      float* const at = a.scores + row + j;
      if ((a.max_ctx & 3) == 0) {
        if (j < a.max_ctx)
          *reinterpret_cast<float4*>(at) =
              make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (j + i < a.max_ctx) at[i] = -INFINITY;
      }
    }
  }
}

// Scores a balanced share of the whole batch: the positions below n_b of
// every unit are cut into groups of kStageRows keys, the groups of all units
// are numbered unit-major, and workgroup `wg` of `nwg` takes a contiguous range
// of R groups (range_groups).  A range spans few units; for each
// unit it touches the workgroup loads that unit's G query rows once and, if
// HIST, counts the first radix digit of its scores in LDS and, when it leaves
// the unit, adds the counts to the unit's histogram or stores them as its own
// slot (hist_part).  Rows of a unit's last group at or past n_b get -inf; later
// groups are not written (the selections read only below n_b; fill_tails
// writes them for score_keys).  Must be called by all
// 64 * NW threads of the workgroup; lds_stage holds NW * (kStageDwords +
// kFlushGroups * kStageRows) dwords.
//
// Memory path: the NW waves take the range's groups round-robin (wave w the
// groups w, w + NW, ...), so that the workgroup streams one region at a
// time: with a contiguous quarter per wave the scan ran 5 % slower (four
// times as many regions in flight over the device).  A wave reads each group
// with fully coalesced 16-byte loads (one instruction = 4 whole 256-byte
// rows), writes it to a private, padded LDS stage and reads it back in the
// MFMA operand placement while the loads of its next group are in flight.
// Loading the operand placement straight from HBM (16 rows x 64 bytes per
// instruction) costs about a tenth of the achievable bandwidth.
//
// Scores are collected in a per-wave LDS buffer and written out every
// kFlushGroups groups, one 128-byte line per group (for a Llama-8B-sized
// batch that is once, at the end of the range).  A global store pending in the loop
// would make every wait for the current group also wait for the prefetched
// one (loads and stores share one counter), and score writes interleaved
// with the key stream cost bandwidth even in large batches: about 10 % at
// every 16 groups against 2 % when written once.
//
// HALVES: a wave requests the next group in two halves, the second once the
// first has landed (after scoring the current group), so that it has 4 KiB
// rather than 8 KiB in flight.  That suits the scoring role of the one-launch
// attend-and-score kernels, which share the memory system with the
// attention's random row reads: 186-188 against 189-192 us per Llama-8B
// layer, alternated over two sessions.  The 8-wave histogram pass is slower with it (167-170 against
// 158-165 us), as it is with 16-row groups.
//
// FUSED (the scoring role of the one-launch same-step kernel, HIST with
// per-workgroup slots): the ranges are XCD-affine (hist_slots); the workgroup
// may have more than NW waves, the others only join its barriers; scores and
// slots are stored device-coherent, 8 bytes per lane over whole lines, and
// each finished (unit, slot) is handed over through fs (FusedSync).
//
// TWO: the pass scores two queries (a.q and a.q2) against each key it reads,
// into two score arrays and two histograms (lds_hist holds both); a wave's
// score buffer is shared by the two, so it is flushed twice as often.
template <int G, bool HIST, int NW = 4, bool HALVES = false, bool FUSED = false, bool TWO = false,
          bool PART = false>
__device__ __forceinline__ void score_range(const ScoreArgs& a, int wg, int nwg,
                                            uint32_t* lds_hist,
                                            uint32_t* lds_stage, FusedSync fs = FusedSync{}) {
  static_assert(!FUSED || (HIST && !HALVES), "the fused scoring role counts histograms");
  static_assert(!TWO || (HIST && !FUSED), "two queries: the pass with histograms");
  constexpr int kSets = TWO ? 2 : 1;
  constexpr int kFlush = kFlushGroups / kSets;      // groups of scores held per query
  constexpr int kSetStride = kFlush * kStageRows;
  constexpr int NT = 64 * NW;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int lrow = lane >> 4, lchunk = lane & 15;
  const bool active = !FUSED || wave < NW;  // uniform over the wave
  constexpr int kLoads = kStageRows / 4;  // 4 rows per load instruction
  // FUSED: XCD x = wg % 8 scores units x, x + 8, ... with its nwg / 8 workgroups
  const int xcd = FUSED ? (wg & 7) : 0;
  const int wr = FUSED ? (wg >> 3) : wg, nwr = FUSED ? (nwg >> 3) : nwg;
  const int items = FUSED ? (a.units >> 3) : a.units / a.Hkv;
  const uint32_t mult = FUSED ? 1u : (uint32_t)a.Hkv;
  auto valid = [&](int i) {
    return unit_len(a.ctx_lens[FUSED ? (8 * i + xcd) / a.Hkv : i], a.max_ctx, a.chunk);
  };
  auto part = [](int n) { return PART ? static_rows(n) : n; };
  // the fused role has too few requests for stored ranges
  const auto len = range_lens(items, !FUSED && a.stored ? part(a.max_ctx) : -1,
                              [&](int i) { return part(valid(i)); });
  GroupScan scan;
  const uint32_t total = mult * sum_groups(len, &scan);
  const uint32_t R = range_groups(total, nwr, a.min_range);
  const GroupRange range = range_of(wr, R, total);
  const uint32_t g0 = range.g0, g1 = range.g1;
  if (g0 >= g1) return;  // uniform over the workgroup
  GroupItem it = find_item(len, scan, mult, g0);
  uint32_t* stage = lds_stage + (active ? wave : 0) * kStageDwords;
  float* sbuf = reinterpret_cast<float*>(lds_stage + NW * kStageDwords) +
                (active ? wave : 0) * kFlushGroups * kStageRows;
  const int item0 = it.item;

  for (uint32_t seg = g0; seg < g1;) {
    while (seg >= it.base + mult * it.vg) {  // the next item that has groups
      it.base += mult * it.vg;
      ++it.item;
      it.n = len(it.item);
      it.vg = groups_of(it.n);
    }
    const uint32_t h = FUSED ? 0u : (seg - it.base) / it.vg;
    const int unit = FUSED ? 8 * it.item + xcd : it.item * a.Hkv + (int)h;
    const int64_t slot =
        FUSED ? (int64_t)xcd * (items + nwr) + it.item + wr : (int64_t)unit + wg;
    const uint32_t ubase = it.base + h * it.vg;
    uint32_t seg_end = min(g1, ubase + it.vg);
    int n = it.n;
    if (!FUSED && a.stored) {  // the groups of the range below n_b, if any
      n = min(n, (int)__builtin_amdgcn_readfirstlane(valid(it.item)));
      const uint32_t next = seg_end;
      seg_end = min(seg_end, ubase + groups_of(n));
      if (seg >= seg_end) {  // uniform over the workgroup
        seg = next;
        continue;
      }
    }
    if (HIST) {
      if (!FUSED || tid < NT)
        for (int i = tid; i < kSets * kHistBins; i += NT) lds_hist[i] = 0u;
      __syncthreads();
    }
    bf16x8 qa[TWO && G == 16 ? 8 : 4];
    load_query<G, TWO>(a, unit, qa);
    const uint16_t* kunit = a.keys + (int64_t)unit * a.max_ctx * a.key_stride;
    // Rows at or past n_b load row n_b - 1 instead (their scores are
    // replaced by -inf): lane-conditional loads would make the compiler
    // wait for every outstanding load at each use.
    // loads [i0, i1) of a group's kLoads
    auto load_part = [&](uint32_t gg, uint4* v, int i0, int i1) {
      const int jb = (int)(gg - ubase) * kStageRows;
#pragma unroll
      for (int i = i0; i < i1; ++i) {
        const int j = min(jb + 4 * i + lrow, n - 1);
        v[i] = ld16_nt(kunit + (int64_t)j * a.key_stride + 8 * lchunk);
      }
    };
    auto load_group = [&](uint32_t gg, uint4* v) { load_part(gg, v, 0, kLoads); };
    // writes the scores of `count` buffered positions of one query, the
    // wave's groups from position jb on: one contiguous run, 16 bytes per
    // lane when rows are 16-byte aligned
    auto flush_rows = [&](float* scores, const float* buf, int jb, int count) {
      float* const srow = scores + (int64_t)unit * a.max_ctx;
      if constexpr (FUSED) {
        // 8 bytes per lane, consecutive lanes on consecutive pairs: each
        // instruction covers whole 128-byte lines of four groups
        for (int c = 2 * lane; c < count; c += 128) {
          const int j = jb + (c / kStageRows) * NW * kStageRows + c % kStageRows;
          const float2 v = *reinterpret_cast<const float2*>(buf + c);
          if ((a.max_ctx & 1) == 0 && j + 1 < a.max_ctx) {
            const uint64_t w = (uint64_t)__float_as_uint(v.x) |
                               ((uint64_t)__float_as_uint(v.y) << 32);
            __hip_atomic_store(reinterpret_cast<uint64_t*>(srow + j), w, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
          } else {
            if (j < a.max_ctx)
              __hip_atomic_store(srow + j, v.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (j + 1 < a.max_ctx)
              __hip_atomic_store(srow + j + 1, v.y, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
          }
        }
      } else if ((a.max_ctx & 3) == 0) {
        for (int c = 4 * lane; c < count; c += 256) {
          const float4 v = *reinterpret_cast<const float4*>(buf + c);
          const int j = jb + (c / kStageRows) * NW * kStageRows + c % kStageRows;
          if (j + 3 < a.max_ctx) {
            *reinterpret_cast<float4*>(srow + j) = v;
          } else {
            if (j < a.max_ctx) srow[j] = v.x;
            if (j + 1 < a.max_ctx) srow[j + 1] = v.y;
            if (j + 2 < a.max_ctx) srow[j + 2] = v.z;
          }
        }
      } else {
        for (int c = lane; c < count; c += 64) {
          const int j = jb + (c / kStageRows) * NW * kStageRows + c % kStageRows;
          if (j < a.max_ctx) srow[j] = buf[c];
        }
      }
    };
    // the nb buffered groups from group `first` on
    auto flush = [&](uint32_t first, int nb) {
      __builtin_amdgcn_wave_barrier();
      const int jb = (int)(first - ubase) * kStageRows;
      flush_rows(a.scores, sbuf, jb, nb * kStageRows);
      if (TWO) flush_rows(a.scores2, sbuf + kSetStride, jb, nb * kStageRows);
      __builtin_amdgcn_wave_barrier();
    };
    // this wave's groups of the segment: every NW-th one (none for the waves
    // past NW of the fused role)
    const uint32_t w1 = seg_end, w0 = active ? seg + wave : w1;
    uint4 cur[kLoads], nxt[kLoads];
    uint32_t gg = w0;
    uint32_t first = gg;
    int nb = 0;
    if (gg < w1) load_group(gg, cur);
#pragma unroll 1
    for (; gg < w1; gg += NW) {
#pragma unroll
      for (int i = 0; i < kLoads; ++i)
        *reinterpret_cast<uint4*>(stage + (4 * i + lrow) * kStageRowDwords + 4 * lchunk) =
            cur[i];
      const bool more = gg + NW < w1;
      if (more) load_part(gg + NW, nxt, 0, HALVES ? kLoads / 2 : kLoads);
      __builtin_amdgcn_wave_barrier();
      score_group<G, HIST, TWO>(stage, qa, (int)(gg - ubase) * kStageRows, n, a.scale,
                                lds_hist, sbuf + nb * kStageRows, kSetStride);
      if (HALVES && more) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        load_part(gg + NW, nxt, kLoads / 2, kLoads);
      }
      if (++nb == kFlush) {
        flush(first, nb);
        first = gg + NW;
        nb = 0;
      }
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int i = 0; i < kLoads; ++i) cur[i] = nxt[i];
    }
    if (nb) flush(first, nb);
    if (HIST) {
      __syncthreads();
      if constexpr (FUSED) {
        if (tid < NT) store_hist_coherent<NT>(lds_hist, a.hist_part + slot * kHistBins);
      } else if (a.hist_part) {
        store_hist<NT>(lds_hist, a.hist_part + slot * kHistBins);
        if (TWO) store_hist<NT>(lds_hist + kHistBins, a.hist_part2 + slot * kHistBins);
      } else if (a.hist) {
        flush_hist<NT>(lds_hist, a.hist + (int64_t)unit * kHistBins,
                       a.coarse + (int64_t)unit * kCoarseBins);
        if (TWO)
          flush_hist<NT>(lds_hist + kHistBins, a.hist2 + (int64_t)unit * kHistBins,
                         a.coarse2 + (int64_t)unit * kCoarseBins);
      }
      __syncthreads();
    }
    seg = ubase + it.vg;
  }
  if constexpr (FUSED) {
    // every slot of the range handed over at its end, after one wait for all
    // its stores (a wait between units would stall the key stream): each
    // thread waits for its own, the barrier then covers the workgroup's, and
    // each slot's two flags take the launch's tag.  Units without positions
    // have no slot, and nobody would clear its flags.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    const int64_t slot0 = (int64_t)xcd * (items + nwr) + wr;
    for (int t = tid; t < 2 * (it.item - item0 + 1); t += blockDim.x) {
      const int i = item0 + (t >> 1);
      if (valid(i))
        __hip_atomic_store(fs.flags + 2 * (slot0 + i) + (t & 1), fs.tag, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// The dynamic part of that pass, for the added histograms of the pipelined
// attend-and-score launch (a.claim set, a.hist_part null).  The first
// kStaticEighths / 8 of each unit were scored as ranges (score_range, PART); the
// valid groups after them are cut into claims of kClaimGroups.
// Workgroups take claims in increasing order from the counter a.claim, so a
// workgroup on a CU slowed by other work (the zero-copy gather running beside
// the pass) takes fewer of them and the pass is not held up by its slowest
// CUs.  A claim costs a workgroup about 8 us whatever its size: all workgroups
// ask the one counter at about the same time, and their device-scope atomics
// queue.  So half the work needs no claim, and claims are large.  A million
// positions of 8 units: all claims 414 us, all static 352, half and half 357
// (claims of 32 groups 431, three quarters static 357); beside the gather of
// the million-token loop, per layer with the same selection: 662, -, 650 us
// (three quarters static 690).
//
// Thread 0 takes claims two ahead of the one being scored, at the start of
// each claim, and passes them through a two-entry LDS ring (one barrier per
// claim), so each wave knows the next claim while it scores the current one
// and prefetches that claim's first group across the boundary.  A
// workgroup thus holds up to two claims it has not started, which leaves
// workgroups idle at the end unless there are several claims per workgroup:
// the host uses claims from four of stored positions per workgroup, static ones
// included.  (Taking the next claim
// later, two rounds before the current claim's end, made the
// million-token loop's gather beside the pass slower.)  Each workgroup takes
// exactly one claim at or past the total; those take values total ..
// total + nwg - 1, and the workgroup that gets the last one resets the
// counter, so it is zero again when the launch ends.  A wave's scores stay
// in its LDS buffer for up to kFlushGroups / (kClaimGroups / 4) claims
// before one flush writes them, each claim's groups to its own unit's row.
// The LDS histogram counts one unit at a time and is added to that unit's
// histogram when the workgroup's claims move to another unit (claims
// increase, so once per unit) and at the end.  lds_claim: two words.  Must
// be called by all kScoreThreads threads.
template <int G>
__device__ __forceinline__ void score_claims(const ScoreArgs& a, int nwg, uint32_t* lds_hist,
                                             uint32_t* lds_stage, uint32_t* lds_claim) {
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int lrow = lane >> 4, lchunk = lane & 15;
  constexpr int kLoads = kStageRows / 4;
  constexpr int kPerWave = kClaimGroups / 4;       // a wave's groups of one claim
  constexpr int kRecs = kFlushGroups / kPerWave;   // claims per score flush
  constexpr int kClaimRows = kClaimGroups * kStageRows;
  static_assert(kClaimGroups % 4 == 0 && kFlushGroups % kPerWave == 0, "claim layout");
  const int items = a.units / a.Hkv;
  const uint32_t mult = (uint32_t)a.Hkv;
  auto full = [&](int i) { return unit_len(a.ctx_lens[i], a.max_ctx, a.chunk); };
  auto part = [](int n) { return n - static_rows(n); };
  const auto len = range_lens(items, a.stored ? part(a.max_ctx) : -1,
                              [&](int i) { return part(full(i)); });
  GroupScan scan;
  const uint32_t total = mult * sum_groups<kClaimRows>(len, &scan);
  uint32_t* stage = lds_stage + wave * kStageDwords;
  float* sbuf = reinterpret_cast<float*>(lds_stage + 4 * kStageDwords) +
                wave * kFlushGroups * kStageRows;

  // thread 0: the claim that makes the counter reach total + nwg is the last
  // of the launch, and whoever holds it resets the counter
  auto last_resets = [&](uint32_t c) {
    if (c == total + (uint32_t)nwg - 1u) atomicExch(a.claim, 0u);
  };
  // a claim's unit, valid length, and groups [g0, v1), none if it lies past n_b
  struct Geo {
    int unit, n, g0, v1;
  };
  auto geo = [&](uint32_t c) {
    const GroupItem it = find_item<kClaimRows>(len, scan, mult, c);
    const uint32_t h = (c - it.base) / it.vg;
    Geo r;
    r.unit = it.item * a.Hkv + (int)h;
    r.n = __builtin_amdgcn_readfirstlane(full(it.item));
    r.g0 = static_rows(a.stored ? a.max_ctx : r.n) / kStageRows +
           (int)(c - it.base - h * it.vg) * kClaimGroups;
    r.v1 = min(r.g0 + kClaimGroups, (int)groups_of(r.n));
    return r;
  };
  auto load_group = [&](const Geo& c, int g, uint4* v) {
    const uint16_t* kunit = a.keys + (int64_t)c.unit * a.max_ctx * a.key_stride;
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const int j = min(g * kStageRows + 4 * i + lrow, c.n - 1);
      v[i] = ld16_nt(kunit + (int64_t)j * a.key_stride + 8 * lchunk);
    }
  };

  // buffered claims of this wave: unit, first group, groups scored
  int rec_unit[kRecs], rec_g0[kRecs], rec_nr[kRecs];
  int nrec = 0;
  auto flush = [&]() {
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int q = 0; q < kRecs; ++q) {
      if (q < nrec) {
        float* srow = a.scores + (int64_t)rec_unit[q] * a.max_ctx;
        const float* src = sbuf + q * kPerWave * kStageRows;
        const int count = rec_nr[q] * kStageRows;
        if ((a.max_ctx & 3) == 0) {
          for (int c = 4 * lane; c < count; c += 256) {
            const float4 v = *reinterpret_cast<const float4*>(src + c);
            const int j = (rec_g0[q] + wave + 4 * (c / kStageRows)) * kStageRows + c % kStageRows;
            if (j + 3 < a.max_ctx) {
              *reinterpret_cast<float4*>(srow + j) = v;
            } else {
              if (j < a.max_ctx) srow[j] = v.x;
              if (j + 1 < a.max_ctx) srow[j + 1] = v.y;
              if (j + 2 < a.max_ctx) srow[j + 2] = v.z;
            }
          }
        } else {
          for (int c = lane; c < count; c += 64) {
            const int j = (rec_g0[q] + wave + 4 * (c / kStageRows)) * kStageRows + c % kStageRows;
            if (j < a.max_ctx) srow[j] = src[c];
          }
        }
      }
    }
    nrec = 0;
    __builtin_amdgcn_wave_barrier();
  };

  if (tid == 0) {  // claims 0 and 1
    const uint32_t c0 = atomicAdd(a.claim, 1u);
    const uint32_t c1 = c0 < total ? atomicAdd(a.claim, 1u) : c0;
    last_resets(max(c0, c1));  // claims increase
    lds_claim[0] = c0;
    lds_claim[1] = c1;
  }
  __syncthreads();
  uint32_t cur = lds_claim[0], nxt = lds_claim[1];
  int cur_unit = -1;
  bf16x8 qa[4];
  uint4 cbuf[kLoads], nbuf[kLoads];
  bool have = false;  // cbuf holds this wave's first group of the current claim
#pragma unroll 1
  for (int i = 0; cur < total; ++i) {  // cur is uniform over the workgroup
    const Geo c = geo(cur);
    uint32_t ahead = 0;  // claim i + 2 (none once a claim has failed)
    const bool takes = tid == 0 && nxt < total;
    if (takes) ahead = atomicAdd(a.claim, 1u);
    if (c.unit != cur_unit) {
      if (cur_unit >= 0) {
        __syncthreads();
        flush_hist(lds_hist, a.hist + (int64_t)cur_unit * kHistBins,
                   a.coarse + (int64_t)cur_unit * kCoarseBins);
        __syncthreads();
      }
      for (int t = tid; t < kHistBins; t += kScoreThreads) lds_hist[t] = 0u;
      __syncthreads();
      load_query<G>(a, c.unit, qa);
      cur_unit = c.unit;
    }
    const int w0 = c.g0 + wave;
    if (!have && w0 < c.v1) load_group(c, w0, cbuf);
    have = false;
    int r = 0;
#pragma unroll 1
    for (int g = w0; g < c.v1; g += 4, ++r) {
#pragma unroll
      for (int k = 0; k < kLoads; ++k)
        *reinterpret_cast<uint4*>(stage + (4 * k + lrow) * kStageRowDwords + 4 * lchunk) =
            cbuf[k];
      bool pf = false;
      if (g + 4 < c.v1) {
        load_group(c, g + 4, nbuf);
        pf = true;
      } else if (nxt < total) {  // the wave's last group: prefetch across the claim
        const Geo d = geo(nxt);
        if (d.g0 + wave < d.v1) {
          load_group(d, d.g0 + wave, nbuf);
          pf = true;
          have = true;
        }
      }
      __builtin_amdgcn_wave_barrier();
      score_group<G, true>(stage, qa, g * kStageRows, c.n, a.scale, lds_hist,
                           sbuf + (nrec * kPerWave + r) * kStageRows);
      __builtin_amdgcn_wave_barrier();
      if (pf) {
#pragma unroll
        for (int k = 0; k < kLoads; ++k) cbuf[k] = nbuf[k];
      }
    }
    if (r) {
#pragma unroll
      for (int q = 0; q < kRecs; ++q)
        if (q == nrec) {
          rec_unit[q] = c.unit;
          rec_g0[q] = c.g0;
          rec_nr[q] = r;
        }
      if (++nrec == kRecs) flush();
    }
    if (tid == 0) {
      if (takes) last_resets(ahead);
      lds_claim[i & 1] = takes ? ahead : nxt;
    }
    __syncthreads();  // publishes claim i + 2
    cur = nxt;
    nxt = lds_claim[i & 1];
  }
  if (nrec) flush();
  if (cur_unit >= 0) {
    __syncthreads();
    flush_hist(lds_hist, a.hist + (int64_t)cur_unit * kHistBins,
               a.coarse + (int64_t)cur_unit * kCoarseBins);
  }
}

}  // namespace ckv

// ERT remap with failure mask, per-slot counts, deterministic permutation and
// the activation gather (§4.2, §5.1, §5.3; per-expert batching, §2.2.1).
//
// Three passes over the routed pairs, all integer and free of ordering races:
//   1. remap_count: per pair, the first live candidate slot of its expert;
//      per chunk of pairs, an S-wide histogram and an unserved count
//      (integer LDS atomics: the totals do not depend on their order).
//      Pairs of tokens outside the batch (token_valid[t] == 0, the partial
//      batch of §5.2) get slot -2 and are not counted. In replay mode (§5.1)
//      a pair keeps its first-pass slot while that slot is alive and is
//      otherwise given its first live candidate now, to be recomputed;
//   2. scan: per-slot totals, exclusive slot offsets, and the position of
//      every (chunk, slot) within its slot in chunk order (the histograms
//      are slot-major, so one wave sums one slot's chunks). Each scatter block
//      does this for itself from the whole histogram;
//   3. scatter: each wave walks an equal share of a chunk in pair order and
//      ranks the pairs of each group of 64 by slot: one ballot per bit of
//      the slot index gives every lane the lanes that share its slot, so the
//      rank costs the same for any mix of slots, and rows follow
//      (slot, token, rank).
// Up to 4096 pairs, one block runs all three passes (the batch of a decode
// step fits, and a launch is saved; past that the two grids are
// faster, as each group of 1024 pairs costs the one block about 1.7 us).
// The gather then copies one activation row per routed pair with 16-byte
// loads and stores (rows are contiguous in source and destination, so the
// copy is fully coalesced without staging).
#include "tg_device.h"
#include "tg_launch.h"
#include "tg_shapes.h"

namespace tg {
namespace {

constexpr int kMaxS = 1024;
constexpr int kBlock = 256;
constexpr int kSmallHist = 1024;  // entries that a scatter block loads as they lie,
constexpr int kSmallChunks = 32;  // of at most so many chunks

// Slot of a pair of expert e: the first live ERT candidate of e.
// REPLAY: -1 also when the first pass's slot pr is still alive (its result
// stands). *unserved: the expert lists a local candidate, none alive.
template <bool REPLAY>
__device__ __forceinline__ int resolve_expert(int e, int pr, const int32_t* __restrict__ ert,
                                              int E, int R, const uint8_t* __restrict__ alive,
                                              int S, bool* unserved) {
  int slot = -1;
  bool listed = false;
  if (e >= 0 && e < E) {
    for (int r = 0; r < R; ++r) {
      const int c = ert[(size_t)e * R + r];
      if (c >= 0 && c < S) {
        listed = true;
        if (alive[c]) {
          slot = c;
          break;
        }
      }
    }
  }
  *unserved = slot < 0 && listed;
  if (REPLAY && pr >= 0 && pr < S && alive[pr]) slot = -1;  // first-pass result stands
  return slot;
}

// Slot that pair p is computed on: the first live ERT candidate of its
// expert; -2 for a token outside the batch. REPLAY: -1 also when the first
// pass's slot prior[p] is still alive (its result stands) or the token was
// outside the batch. *unserved: the expert lists a local candidate, none
// alive.
template <bool REPLAY>
__device__ __forceinline__ int resolve_pair(int p, const int32_t* __restrict__ ids, int k,
                                            const int32_t* __restrict__ ert, int E, int R,
                                            const uint8_t* __restrict__ alive, int S,
                                            const uint8_t* __restrict__ token_valid,
                                            const int32_t* __restrict__ prior, bool* unserved) {
  *unserved = false;
  int pr = 0;
  if (REPLAY) {
    pr = prior[p];
    if (pr == -2) return -1;
  } else if (token_valid && !token_valid[p / k]) {
    return -2;
  }
  return resolve_expert<REPLAY>(ids[p], pr, ert, E, R, alive, S, unserved);
}

// Lanes of the wave that hold a routed pair (s >= 0) on the same slot as
// this lane: start from the routed lanes and keep, for every bit of the slot
// index (sbits bits), the lanes that agree with this lane on that bit. The
// cost is the same for any mix of slots. 0 on lanes with s < 0.
__device__ __forceinline__ uint64_t same_slot_lanes(int s, int sbits) {
  uint64_t eq = __ballot(s >= 0);
  for (int b = 0; b < sbits; ++b) {
    const bool bit = (s >> b) & 1;
    const uint64_t mb = __ballot(bit);
    eq &= bit ? mb : ~mb;
  }
  return s >= 0 ? eq : 0;
}

// Plans both GEMMs of the call (wave 0 the gate/up GEMM, wave 1 the down
// GEMM; other waves have nothing to do here). count(s): rows of slot s.
// COUNTS false leaves the plan's row blocks to the caller.
template <bool COUNTS, typename Count>
__device__ __forceinline__ void plan_gemms(int which, int S, Count count, int32_t* sched,
                                           const GemmDims& g) {
  if (which > 1) return;
  const Census cs = census(S, count);
  const int shape = which == 0 ? choose_shape<true, false>(cs, g.grid, g.d, g.I)
                               : choose_shape<false, true>(cs, g.grid, g.I, g.d);
  int32_t* const plan = sched + 16 * which + kSchedPlan;
  const int lane = lane_id();
  if (lane == 0) plan[0] = shape;
  if (COUNTS && lane < 4)
    plan[1 + lane] = lane == 0 ? cs.b32 : lane == 1 ? cs.b64 : lane == 2 ? cs.b128 : cs.b256;
}

// The claim counters of both GEMMs start at zero.
__device__ __forceinline__ void zero_claims(int32_t* sched, int tid) {
  if (tid < 2 * kSchedPlan) sched[tid < kSchedPlan ? tid : tid - kSchedPlan + 16] = 0;
}

// REPLAY: `prior` holds the first pass's slot of every pair; out_slot gets
// the slot the pair is recomputed on, or -1 when its first-pass result still
// stands (slot alive), it is outside the batch (-2), or no candidate is live.
template <bool REPLAY>
__global__ __launch_bounds__(kBlock) void remap_count_kernel(
    const int32_t* __restrict__ ids, int npairs, int k, const int32_t* __restrict__ ert, int E,
    int R, const uint8_t* __restrict__ alive, int S, const uint8_t* __restrict__ token_valid,
    const int32_t* __restrict__ prior, int32_t* __restrict__ out_slot, int32_t* __restrict__ hist,
    int32_t* __restrict__ unserved_chunk, int chunk, int32_t* __restrict__ sched) {
  __shared__ int h[kMaxS];
  __shared__ int nu;
  for (int s = threadIdx.x; s < S; s += kBlock) h[s] = 0;
  if (threadIdx.x == 0) nu = 0;
  __syncthreads();
  const int base = blockIdx.x * chunk;
  for (int i = threadIdx.x; i < chunk; i += kBlock) {
    const int p = base + i;
    if (p >= npairs) break;
    bool unserved;
    const int slot =
        resolve_pair<REPLAY>(p, ids, k, ert, E, R, alive, S, token_valid, prior, &unserved);
    out_slot[p] = slot;
    if (unserved) atomicAdd(&nu, 1);
    if (slot >= 0) atomicAdd(&h[slot], 1);
  }
  __syncthreads();
  for (int s = threadIdx.x; s < S; s += kBlock) hist[(size_t)s * gridDim.x + blockIdx.x] = h[s];
  if (threadIdx.x == 0) unserved_chunk[blockIdx.x] = nu;
  if (sched && blockIdx.x == 0) zero_claims(sched, threadIdx.x);
}

__device__ __forceinline__ int wave_sum_int(int v) {
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// hist holds the per-chunk counts of remap_count (slot-major), and every block
// derives its chunk's position in each slot and the slot offsets itself, from
// all of it; block 0 also writes counts, offsets, the unserved count and the
// total. sbits: bits of the largest slot index. With a schedule area one block
// more than there are chunks is launched, which plans the GEMMs. CH: chunks
// per lane, nchunks <= 64 CH; 0 for at most kSmallHist entries, and at most
// kSmallChunks per slot.
template <int CH>
__global__ __launch_bounds__(kBlock) void scatter_kernel(
    const int32_t* __restrict__ pair_slot, int npairs, int S, int nchunks, int sbits,
    const int32_t* __restrict__ hist, const int32_t* __restrict__ unserved_chunk,
    int32_t* __restrict__ counts, int32_t* __restrict__ offsets,
    int32_t* __restrict__ n_unserved, int32_t* __restrict__ total_out,
    int32_t* __restrict__ perm, int32_t* __restrict__ pair_row, int chunk,
    int32_t* __restrict__ sched, GemmDims dims) {
  constexpr int kWaves = kBlock / kWave;
  __shared__ int cnt[kWaves][kMaxS];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int lane = lane_id();
  const bool planner = (int)blockIdx.x == nchunks;
  // The chunk's pairs are split evenly (in multiples of 64) over the waves.
  const int c0 = blockIdx.x * chunk;
  const int n_c = min(chunk, npairs - c0);
  const int span = ((n_c + kWaves * kWave - 1) / (kWaves * kWave)) * kWave;
  const int p0 = c0 + wave * span;
  const int p1 = min(c0 + n_c, p0 + span);
  __shared__ int base[kMaxS];  // first row of this chunk's pairs on each slot
  __shared__ int tot[kMaxS];
  __shared__ int wsum[kWaves];
  for (int s = lane; s < S; s += kWave) cnt[wave][s] = 0;
  // A small histogram is loaded as it lies, four entries per thread at once, and
  // summed by LDS atomics (integers: their order does not matter). Otherwise
  // wave w takes slots w, w + 4, ..., kGroup of them at a time so that their
  // loads are in flight together, 16 whatever CH is: lane l holds chunks l,
  // l + 64, ... of each; the sums over all chunks and over the chunks before
  // this one are DPP reductions. The chain of loads bounds it. Against a kernel
  // of one block between count and scatter (17 to 64 chunks; 128; 256), us for
  // the whole dispatch without the row copy: 40 slots 10 -> 8, 10 -> 9,
  // 12 -> 10; 200 slots 17 -> 15, 19 -> 17, 29 -> 20; 1024 slots 48 -> 43,
  // 62 -> 57, 110 -> 77. (With the loads of 256 chunks for any number of them,
  // four slots at a time, 200 slots of 17 to 64 chunks took 18 and 960 of 17
  // took 57.) For 24 to 60 slots of 17 chunks the atomics are 0.5 to 1.2 us
  // faster than the reductions, for 1 to 16 of up to 32 chunks 0.3; 16 slots of
  // 64 chunks, whose entries of a wave meet in one slot, are 0.8 slower.
  if (CH == 0) {
    constexpr int kPer = kSmallHist / kBlock;
    const int nh = S * nchunks;
    int v[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int j = threadIdx.x + q * kBlock;
      v[q] = j < nh ? hist[j] : 0;
    }
    for (int s = threadIdx.x; s < S; s += kBlock) {
      tot[s] = 0;
      base[s] = 0;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int j = threadIdx.x + q * kBlock;
      if (v[q]) {
        const int s = j / nchunks, c = j - s * nchunks;
        atomicAdd(&tot[s], v[q]);
        if (c < (int)blockIdx.x) atomicAdd(&base[s], v[q]);
      }
    }
  }
  constexpr int kLanes = CH ? CH : 1, kGroup = 16 / kLanes;
  for (int s0 = wave; CH && s0 < S; s0 += kGroup * kWaves) {
    int v[kGroup][kLanes];
#pragma unroll
    for (int g = 0; g < kGroup; ++g)
#pragma unroll
      for (int q = 0; q < kLanes; ++q) {
        const int s = s0 + g * kWaves, c = lane + q * kWave;
        v[g][q] = s < S && c < nchunks ? hist[(size_t)s * nchunks + c] : 0;
      }
#pragma unroll
    for (int g = 0; g < kGroup; ++g) {
      const int s = s0 + g * kWaves;
      if (s >= S) break;
      int all = 0, before = 0;
#pragma unroll
      for (int q = 0; q < kLanes; ++q) {
        all += v[g][q];
        before += lane + q * kWave < (int)blockIdx.x ? v[g][q] : 0;
      }
      all = wave_reduce<false>(all);
      before = wave_reduce<false>(before);
      if (lane == 0) {
        tot[s] = all;
        base[s] = before;
      }
    }
  }
  __syncthreads();
  if (planner) {
    plan_gemms<true>(wave, S, [&](int s) { return tot[s]; }, sched, dims);
    return;
  }
  // Exclusive scan of the slot totals: thread i holds slots 4i .. 4i+3.
  {
    int v[4], sum = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int s = 4 * threadIdx.x + j;
      v[j] = s < S ? tot[s] : 0;
      sum += v[j];
    }
    int incl = sum;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const int t = __shfl_up(incl, off);
      if (lane >= off) incl += t;
    }
    if (lane == kWave - 1) wsum[wave] = incl;
    __syncthreads();
    for (int w = 0; w < wave; ++w) incl += wsum[w];
    int run = incl - sum;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int s = 4 * threadIdx.x + j;
      if (s < S) {
        base[s] += run;
        if (blockIdx.x == 0) {
          counts[s] = v[j];
          offsets[s] = run;
        }
      }
      run += v[j];
    }
    if (blockIdx.x == 0) {
      if (threadIdx.x == kBlock - 1) {
        offsets[S] = run;  // the last thread's run is the grand total
        if (total_out) total_out[0] = run;
      }
      if (wave == 0) {
        int nu = 0;
        for (int c = lane; c < nchunks; c += kWave) nu += unserved_chunk[c];
        nu = wave_sum_int(nu);
        if (lane == 0) n_unserved[0] = nu;
      }
    }
  }
  for (int p = p0 + lane; p < p1; p += kWave) {
    const int s = pair_slot[p];
    if (s >= 0) atomicAdd(&cnt[wave][s], 1);
  }
  __syncthreads();
  for (int s = threadIdx.x; s < S; s += kBlock) {
    int run = base[s];
    for (int w = 0; w < kWaves; ++w) {
      const int v = cnt[w][s];
      cnt[w][s] = run;
      run += v;
    }
  }
  __syncthreads();
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  for (int g = p0; g < p1; g += kWave) {
    const int p = g + lane;
    int s = -1;
    if (p < p1) {
      s = pair_slot[p];
      if (s < 0) pair_row[p] = -1;
    }
    if (!__ballot(s >= 0)) continue;  // uniform
    const uint64_t eq = same_slot_lanes(s, sbits);
    if (s >= 0) {
      const int row = cnt[wave][s] + __builtin_popcountll(eq & lt);
      perm[row] = p;
      pair_row[p] = row;
      // The slot's lowest lane advances the slot's next row (every lane's
      // read above precedes this write in the wave's LDS order).
      if (!(eq & lt)) cnt[wave][s] = row + __builtin_popcountll(eq);
    }
  }
}

// All three passes in one block of 1024 threads, for at most kSmallPairs
// pairs; thread i takes pairs i, i + 1024, ... The ERT and the liveness mask
// are first copied to LDS while the pairs' expert ids load, so resolving a
// pair costs one memory latency. Each wave counts its pairs per slot with
// same_slot_lanes (one LDS add per distinct slot), a wave scan with one
// barrier gives the slot offsets, and the pairs are then ranked 1024 at a
// time in pair order (wave w holds pairs 64w .. 64w+63 of the group) exactly
// as scatter_kernel does, so rows follow (slot, token, rank). With a schedule
// area a second block counts the pairs too and chooses the GEMMs' tile shapes,
// beside the first one's ranking (chosen by two waves of the same block, the
// kernel took 1.5 us more). That block reads the liveness mask again, which may
// have been written meanwhile: its choice, right for any rows, is all that is
// taken from it, and the row blocks that the GEMMs walk are counted by the
// first block from the totals that become the offsets.
constexpr int kOneBlock = 1024;
constexpr int kSmallPairs = 4096;
constexpr int kSmallPer = kSmallPairs / kOneBlock;
constexpr int kMaxErt = 1024 * 16;  // E * R entries staged in LDS (E <= 1024, R <= 16)

template <bool REPLAY>
__global__ __launch_bounds__(kOneBlock) void dispatch_one_block_kernel(
    const int32_t* __restrict__ ids, int npairs, int k, const int32_t* __restrict__ ert, int E,
    int R, const uint8_t* __restrict__ alive, int S, int sbits,
    const uint8_t* __restrict__ token_valid, const int32_t* __restrict__ prior,
    int32_t* __restrict__ out_slot, int32_t* __restrict__ counts, int32_t* __restrict__ offsets,
    int32_t* __restrict__ perm, int32_t* __restrict__ pair_row, int32_t* __restrict__ n_unserved,
    int32_t* __restrict__ total_out, int32_t* __restrict__ sched, GemmDims dims) {
  constexpr int kWaves = kOneBlock / kWave;
  // cnt[w][s]: pairs of wave w on slot s in the current group of 1024, then
  // their first row; 0 wherever wave w has no pair on s.
  __shared__ int cnt[kWaves][kMaxS];
  __shared__ int run[kMaxS];
  __shared__ int ert_s[kMaxErt];
  __shared__ uint8_t alive_s[kMaxS];
  __shared__ int wsum[kWaves];
  __shared__ int blocks[4];  // row blocks at heights 32, 64, 128 and 256
  __shared__ int nu;
  const int tid = threadIdx.x;
  const int wave = tid / kWave, lane = lane_id();
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));

  // Loads that do not depend on one another: the pairs' ids (and first-pass
  // slots or batch flags), the ERT and the mask. Raw values only, so no load
  // waits for another.
  // Every lane loads (indices past the end read the last pair, and their
  // values are never used), so no load sits in a divergent branch.
  int e_of[kSmallPer], f_of[kSmallPer];
  if (npairs > 0) {
#pragma unroll
    for (int i = 0; i < kSmallPer; ++i) {
      const int p = min(tid + i * kOneBlock, npairs - 1);
      e_of[i] = ids[p];
      f_of[i] = REPLAY ? prior[p] : 1;
    }
    if (!REPLAY && token_valid) {
#pragma unroll
      for (int i = 0; i < kSmallPer; ++i)
        f_of[i] = token_valid[min(tid + i * kOneBlock, npairs - 1) / k];
    }
  }
  for (int j = tid; j < E * R; j += kOneBlock) ert_s[j] = ert[j];
  for (int j = tid; j < S; j += kOneBlock) {
    alive_s[j] = alive[j];
    run[j] = 0;
  }
  for (int j = tid; j < kWaves * S; j += kOneBlock) cnt[j / S][j % S] = 0;
  if (tid == 0) nu = 0;
  if (tid < 4) blocks[tid] = 0;
  __syncthreads();

  // Global stores wait until the end: on this chip a wait for a load also
  // waits for every earlier store, so stores issued here would stall the
  // passes below.
  int my_slot[kSmallPer];
  uint64_t my_eq[kSmallPer];
#pragma unroll
  for (int i = 0; i < kSmallPer; ++i) {
    my_slot[i] = -1;
    my_eq[i] = 0;
    if (i * kOneBlock >= npairs) continue;  // uniform
    const int p = tid + i * kOneBlock;
    bool unserved = false;
    int s = -1;
    if (p < npairs) {
      if (REPLAY ? f_of[i] != -2 : f_of[i] != 0)
        s = resolve_expert<REPLAY>(e_of[i], REPLAY ? f_of[i] : 0, ert_s, E, R, alive_s, S,
                                   &unserved);
      else
        s = REPLAY ? -1 : -2;
    }
    const int n_un = __builtin_popcountll(__ballot(unserved));
    if (lane == 0 && n_un) atomicAdd(&nu, n_un);
    const uint64_t eq = same_slot_lanes(s, sbits);
    if (s >= 0 && !(eq & lt)) atomicAdd(&run[s], __builtin_popcountll(eq));
    my_slot[i] = s;
    my_eq[i] = eq;
  }
  __syncthreads();

  if (blockIdx.x == 1) {  // the planner
    plan_gemms<false>(wave, S, [&](int s) { return run[s]; }, sched, dims);
    return;
  }

  // Exclusive scan of the slot totals: a wave scan per 64 slots, then the
  // totals of the waves before.
  const int total = (tid < S) ? run[tid] : 0;
  int incl = total;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int t = __shfl_up(incl, off);
    if (lane >= off) incl += t;
  }
  if (lane == kWave - 1) wsum[wave] = incl;
  if (sched && wave * kWave < S) {
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      const int n = wave_reduce<false>((total + (32 << h) - 1) / (32 << h));
      if (lane == 0) atomicAdd(&blocks[h], n);
    }
  }
  __syncthreads();
  for (int w = 0; w < wave; ++w) incl += wsum[w];
  if (tid < S) run[tid] = incl - total;  // next row of the slot

  int my_row[kSmallPer];
#pragma unroll
  for (int i = 0; i < kSmallPer; ++i) my_row[i] = -1;
#pragma unroll
  for (int i = 0; i < kSmallPer; ++i) {
    if (i * kOneBlock >= npairs) break;  // uniform
    const int s = my_slot[i];
    const uint64_t eq = my_eq[i];
    const bool lead = s >= 0 && !(eq & lt);
    if (lead) cnt[wave][s] = __builtin_popcountll(eq);
    __syncthreads();
    // Thread q turns slot q's per-wave counts into first rows (all reads
    // first, so they are in flight together; absent waves keep 0).
    if (tid < S) {
      int v[kWaves];
#pragma unroll
      for (int w = 0; w < kWaves; ++w) v[w] = cnt[w][tid];
      int r = run[tid];
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        cnt[w][tid] = v[w] ? r : 0;
        r += v[w];
      }
      run[tid] = r;
    }
    __syncthreads();
    if (s >= 0) my_row[i] = cnt[wave][s] + __builtin_popcountll(eq & lt);
    // Every lane's read above precedes this write in the wave's LDS order.
    if (lead) cnt[wave][s] = 0;
  }

  if (tid < S) {
    counts[tid] = total;
    offsets[tid] = incl - total;
  }
  if (tid == S - 1) {
    offsets[S] = incl;
    if (total_out) total_out[0] = incl;
  }
  if (tid == 0) n_unserved[0] = nu;
#pragma unroll
  for (int i = 0; i < kSmallPer; ++i) {
    const int p = tid + i * kOneBlock;
    if (p < npairs) {
      out_slot[p] = my_slot[i];
      pair_row[p] = my_row[i];
      if (my_row[i] >= 0) perm[my_row[i]] = p;
    }
  }
  if (sched) {
    zero_claims(sched, tid);
    if (tid < 8) sched[tid / 4 * 16 + kSchedPlan + 1 + tid % 4] = blocks[tid % 4];
  }
}

__global__ __launch_bounds__(kBlock) void gather_kernel(const uint4* __restrict__ x,
                                                        const int32_t* __restrict__ perm,
                                                        const int32_t* __restrict__ offsets, int S,
                                                        int k, int nch, uint4* __restrict__ x_perm) {
  const int P = offsets[S];
  const long total = (long)P * nch;
  for (long q = (long)blockIdx.x * kBlock + threadIdx.x; q < total; q += (long)gridDim.x * kBlock) {
    const int r = (int)(q / nch);
    const int c = (int)(q - (long)r * nch);
    const int t = perm[r] / k;
    x_perm[q] = x[(size_t)t * nch + c];
  }
}

}  // namespace

int dispatch_chunk(long npairs) {
  const long per = (npairs + kDispatchChunks - 1) / kDispatchChunks;
  const long c = (per + 255) / 256 * 256;
  return (int)(c < 256 ? 256 : c);
}

size_t dispatch_workspace_bytes(int T, int k, int S) {
  const size_t npairs = (size_t)T * k;
  const int chunk = dispatch_chunk((long)npairs);
  const size_t nchunks = (npairs + chunk - 1) / chunk;
  const size_t hist = nchunks * (size_t)S * sizeof(int32_t);
  return ((hist + 255) & ~(size_t)255) + ((nchunks * sizeof(int32_t) + 255) & ~(size_t)255) + 256;
}

namespace {

hipError_t remap_dispatch(bool replay, const int32_t* ids, int T, int k, const int32_t* ert, int E,
                          int R, const uint8_t* alive, int S, const uint8_t* token_valid,
                          const int32_t* prior, const uint16_t* x, int d, int32_t* pair_slot,
                          int32_t* counts, int32_t* offsets, int32_t* perm, int32_t* pair_row,
                          uint16_t* x_perm, int32_t* n_unserved, int32_t* total_out, void* ws,
                          hipStream_t stream, void* sched_area, const GemmDims& dims) {
  int32_t* const sched = static_cast<int32_t*>(sched_area);
  const int npairs = T * k;
  const int chunk = dispatch_chunk(npairs);
  const int nchunks = (npairs + chunk - 1) / chunk;
  const size_t hist_bytes = ((size_t)nchunks * S * sizeof(int32_t) + 255) & ~(size_t)255;
  int32_t* hist = static_cast<int32_t*>(ws);
  int32_t* unserved_chunk = reinterpret_cast<int32_t*>(static_cast<char*>(ws) + hist_bytes);
  const int sbits = (S > 1) ? 32 - __builtin_clz((unsigned)(S - 1)) : 0;
  if (npairs <= kSmallPairs) {
    if (replay)
      hipLaunchKernelGGL(dispatch_one_block_kernel<true>, dim3(sched ? 2 : 1), dim3(kOneBlock), 0,
                         stream, ids, npairs, k, ert, E, R, alive, S, sbits, nullptr, prior,
                         pair_slot, counts, offsets, perm, pair_row, n_unserved, total_out, sched,
                         dims);
    else
      hipLaunchKernelGGL(dispatch_one_block_kernel<false>, dim3(sched ? 2 : 1), dim3(kOneBlock), 0,
                         stream, ids, npairs, k, ert, E, R, alive, S, sbits, token_valid, nullptr,
                         pair_slot, counts, offsets, perm, pair_row, n_unserved, total_out, sched,
                         dims);
  } else {
    if (replay)
      hipLaunchKernelGGL(remap_count_kernel<true>, dim3(nchunks), dim3(kBlock), 0, stream, ids,
                         npairs, k, ert, E, R, alive, S, nullptr, prior, pair_slot, hist,
                         unserved_chunk, chunk, sched);
    else
      hipLaunchKernelGGL(remap_count_kernel<false>, dim3(nchunks), dim3(kBlock), 0, stream, ids,
                         npairs, k, ert, E, R, alive, S, token_valid, nullptr, pair_slot, hist,
                         unserved_chunk, chunk, sched);
    const dim3 grid(nchunks + (sched ? 1 : 0));
    // The fewest chunks per lane, so that more slots' loads are in flight.
#define TG_SCATTER(CH)                                                                          \
  hipLaunchKernelGGL(scatter_kernel<CH>, grid, dim3(kBlock), 0, stream, pair_slot, npairs, S,   \
                     nchunks, sbits, hist, unserved_chunk, counts, offsets, n_unserved, total_out, \
                     perm, pair_row, chunk, sched, dims)
    if (nchunks <= kSmallChunks && S * nchunks <= kSmallHist) TG_SCATTER(0);
    else if (nchunks <= kWave) TG_SCATTER(1);
    else if (nchunks <= 2 * kWave) TG_SCATTER(2);
    else TG_SCATTER(kDispatchChunks / kWave);
#undef TG_SCATTER
  }
  if (x_perm && npairs > 0) {
    const int nch = d / 8;
    const long maxq = (long)npairs * nch;
    const long blocks = (maxq + kBlock - 1) / kBlock;
    const int grid = (int)(blocks < 8192 ? blocks : 8192);
    hipLaunchKernelGGL(gather_kernel, dim3(grid), dim3(kBlock), 0, stream,
                       reinterpret_cast<const uint4*>(x), perm, offsets, S, k, nch,
                       reinterpret_cast<uint4*>(x_perm));
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_remap_dispatch(const int32_t* ids, int T, int k, const int32_t* ert, int E, int R,
                                 const uint8_t* alive, int S, const uint16_t* x, int d,
                                 int32_t* pair_slot, int32_t* counts, int32_t* offsets,
                                 int32_t* perm, int32_t* pair_row, uint16_t* x_perm,
                                 int32_t* n_unserved, void* ws, hipStream_t stream,
                                 const uint8_t* token_valid, void* sched_area, GemmDims dims) {
  return remap_dispatch(false, ids, T, k, ert, E, R, alive, S, token_valid, nullptr, x, d,
                        pair_slot, counts, offsets, perm, pair_row, x_perm, n_unserved, nullptr,
                        ws, stream, sched_area, dims);
}

hipError_t launch_replay_dispatch(const int32_t* ids, int T, int k, const int32_t* ert, int E,
                                  int R, const uint8_t* alive, int S, const int32_t* prior_slot,
                                  const uint16_t* x, int d, int32_t* replay_slot, int32_t* counts,
                                  int32_t* offsets, int32_t* perm, int32_t* replay_row,
                                  uint16_t* x_perm, int32_t* n_unserved, int32_t* n_replayed,
                                  void* ws, hipStream_t stream, void* sched_area, GemmDims dims) {
  return remap_dispatch(true, ids, T, k, ert, E, R, alive, S, nullptr, prior_slot, x, d,
                        replay_slot, counts, offsets, perm, replay_row, x_perm, n_unserved,
                        n_replayed, ws, stream, sched_area, dims);
}

}  // namespace tg

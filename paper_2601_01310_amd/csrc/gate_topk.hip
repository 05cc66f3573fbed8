// Gating (§2.1): gate logits, top-k selection and renormalised gate weights.
//
// In weight mode every logit that is returned, compared or turned into a gate
// weight is a float64 sum of the exact bf16 x bf16 products, rounded once to
// float32. Three kernels form them, chosen by launch_gate_topk from the sizes:
//   token   one token per block, the vector unit's float64 FMA (few tokens);
//   dense   all logits by float64 MFMA into memory, then the top-k over
//           them (logits wanted, or memory for them at hand);
//   screen  bf16 MFMA sums with an error bound tell which experts can be
//           among the k largest; only those get a float64 logit.
// All three add in one order, so that a token's ids and weights do not depend
// on the batch it is in: 64 partial sums, the l-th over the 8-element chunks
// l, l + 64, ... of the row, element by element; then neighbours are added
// pairwise up to sixteen partial sums, and the four sixteens in order.
//
// Top-k (larger float32 logit first, ties to the lower expert id) counts, for
// each of a few candidates, the ones that beat it, or, over more of them or
// all, takes k rounds of an arg-max over a wave or a 16-lane row of it (the
// cross-lane step in DPP row operations and lane reads). Lane j holds the j-th
// winner; the k exponentials are summed in rank order.
#include <type_traits>

#include "tg_device.h"
#include "tg_launch.h"

namespace tg {
namespace {

constexpr int kWaves = 4;  // waves per block of logits_topk_kernel

__device__ __forceinline__ bool better(float v, int id, float bv, int bid) {
  return v > bv || (v == bv && id < bid);
}

// Arg-max of (v, id) over the 16 lanes of each DPP row: xor 1, xor 2
// (quad permutes), then half-row and row mirrors; afterwards every lane of a
// row holds the row's best.
__device__ __forceinline__ void row_best(float& bv, int& bid) {
#define TG_DPP_STEP(ctrl)                                                                 \
  do {                                                                                    \
    const float ov = __int_as_float(                                                      \
        __builtin_amdgcn_update_dpp(0, __float_as_int(bv), ctrl, 0xF, 0xF, false));       \
    const int oid = __builtin_amdgcn_update_dpp(0, bid, ctrl, 0xF, 0xF, false);           \
    if (better(ov, oid, bv, bid)) {                                                       \
      bv = ov;                                                                            \
      bid = oid;                                                                          \
    }                                                                                     \
  } while (0)
  TG_DPP_STEP(0xB1);   // quad_perm [1,0,3,2]
  TG_DPP_STEP(0x4E);   // quad_perm [2,3,0,1]
  TG_DPP_STEP(0x141);  // row_half_mirror
  TG_DPP_STEP(0x140);  // row_mirror
#undef TG_DPP_STEP
}

// The same over the wave: the four rows are compared with lane reads.
__device__ __forceinline__ void wave_best(float& bv, int& bid) {
  row_best(bv, bid);
  float gv = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(bv), 0));
  int gid = __builtin_amdgcn_readlane(bid, 0);
#pragma unroll
  for (int r = 1; r < 4; ++r) {
    const float rv = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(bv), 16 * r));
    const int rid = __builtin_amdgcn_readlane(bid, 16 * r);
    if (better(rv, rid, gv, gid)) {
      gv = rv;
      gid = rid;
    }
  }
  bv = gv;
  bid = gid;
}

// Lane j < k holds the token's j-th choice: its id and its weight
// exp(l_j - l_0) / sum_{j'<k} exp(l_j' - l_0), the sum in rank order.
__device__ __forceinline__ void store_topk(float my_v, int my_id, int k, int t,
                                           int32_t* __restrict__ ids, float* __restrict__ w) {
  const int lane = lane_id();
  const float v0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_v), 0));
  const float ex = (lane < k) ? expf(my_v - v0) : 0.0f;
  float z = 0.0f;
  for (int j = 0; j < k; ++j) z += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ex), j));
  if (lane < k) {
    ids[(size_t)t * k + lane] = my_id;
    w[(size_t)t * k + lane] = ex / z;
  }
}

// Top-k over the logits held in `lg` (LDS, E <= 64 * NQ floats) by one
// wave; writes ids and weights of token t. Each round takes the best
// remaining candidate of every lane, reduces the rows with DPP and the four
// rows with lane reads, so no round goes through LDS.
template <int NQ>
__device__ void wave_topk(const float* lg, int E, int k, int t, int32_t* __restrict__ ids,
                          float* __restrict__ w) {
  const int lane = lane_id();
  float v[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int e = lane + q * kWave;
    v[q] = (e < E) ? lg[e] : 0.0f;
  }
  uint32_t taken = 0;
  float my_v = 0.0f;
  int my_id = 0;
  for (int j = 0; j < k; ++j) {
    float bv = -__builtin_inff();
    int bid = 0x7fffffff;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int e = lane + q * kWave;
      if (e < E && !(taken & (1u << q)) && better(v[q], e, bv, bid)) {
        bv = v[q];
        bid = e;
      }
    }
    wave_best(bv, bid);
    if ((bid & (kWave - 1)) == lane) taken |= 1u << (bid / kWave);
    if (lane == j) {
      my_v = bv;
      my_id = bid;
    }
  }
  store_topk(my_v, my_id, k, t, ids, w);
}

// Top-k over n <= 64 candidates, lane l < n holding candidate l (n >= k, ids
// distinct): a lane's rank is the number of candidates that beat its own. A
// NaN is never chosen; a choice that is left empty for it is what wave_topk
// leaves there.
__device__ void wave_topk_lanes(float v, int id, int n, int k, int t, int32_t* __restrict__ ids,
                                float* __restrict__ w) {
  const int lane = lane_id();
  int rank = 0;
  for (int i = 0; i < n; ++i) {
    const float ov = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), i));
    const int oid = __builtin_amdgcn_readlane(id, i);
    rank += better(ov, oid, v, id) ? 1 : 0;
  }
  // The others go behind the m that can be chosen, in lane order.
  const bool is = lane < n && v == v;
  const uint64_t m = __ballot(is), lt = (1ull << lane) - 1;
  if (!is) {
    rank = __builtin_popcountll(m) + __builtin_popcountll(~m & lt);
    v = -__builtin_inff();
    id = 0x7fffffff;
  }
  const int to = 4 * rank;
  const float my_v = __int_as_float(__builtin_amdgcn_ds_permute(to, __float_as_int(v)));
  const int my_id = __builtin_amdgcn_ds_permute(to, id);
  store_topk(my_v, my_id, k, t, ids, w);
}

// wave_topk for the smallest NQ that covers E.
__device__ __forceinline__ void wave_topk_any(const float* lg, int E, int k, int t,
                                              int32_t* __restrict__ ids, float* __restrict__ w) {
  if (E <= 64) wave_topk<1>(lg, E, k, t, ids, w);
  else if (E <= 128) wave_topk<2>(lg, E, k, t, ids, w);
  else if (E <= 256) wave_topk<4>(lg, E, k, t, ids, w);
  else if (E <= 512) wave_topk<8>(lg, E, k, t, ids, w);
  else wave_topk<16>(lg, E, k, t, ids, w);
}

// Sum over the wave of a float64 held per lane, the same on every lane, in
// a fixed order: DPP row steps (xor 1, xor 2, half-row mirror, row mirror)
// give each 16-lane row its sum, then the four row sums are added.
__device__ __forceinline__ double wave_sum_f64(double v) {
#define TG_DPP_ADD(ctrl)                                                                     \
  do {                                                                                       \
    const int lo = __builtin_amdgcn_update_dpp(0, (int)__double2loint(v), ctrl, 0xF, 0xF,     \
                                               false);                                       \
    const int hi = __builtin_amdgcn_update_dpp(0, (int)__double2hiint(v), ctrl, 0xF, 0xF,     \
                                               false);                                       \
    v += __hiloint2double(hi, lo);                                                           \
  } while (0)
  TG_DPP_ADD(0xB1);
  TG_DPP_ADD(0x4E);
  TG_DPP_ADD(0x141);
  TG_DPP_ADD(0x140);
#undef TG_DPP_ADD
  double total = 0.0;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int lo = __builtin_amdgcn_readlane((int)__double2loint(v), 16 * r);
    const int hi = __builtin_amdgcn_readlane((int)__double2hiint(v), 16 * r);
    total += __hiloint2double(hi, lo);
  }
  return total;
}

// float64 logits of one token for the NC experts e[0..NC-1] (wave-uniform).
// Lane l sums 8-element chunks l, l + 64, ... of the row, then the lanes are
// added. The vector unit bounds it: per product and wave an unpack, a
// widening (8 cycles, measured) and an FMA, 16 cycles; the next chunk's loads
// are in flight meanwhile.
template <int NC>
__device__ __forceinline__ void logits_of(const uint4* __restrict__ xr,
                                          const uint16_t* __restrict__ wg, int d, const int* e,
                                          float* out) {
  const int nchunk = d / 8;
  double acc[NC];
  uint4 xn, wn[NC];
  auto load = [&](int c) {
    xn = xr[c];
#pragma unroll
    for (int q = 0; q < NC; ++q) wn[q] = reinterpret_cast<const uint4*>(wg + (size_t)e[q] * d)[c];
  };
#pragma unroll
  for (int q = 0; q < NC; ++q) acc[q] = 0.0;
  load(min(lane_id(), nchunk - 1));
  for (int c = lane_id(); c < nchunk; c += kWave) {
    const uint32_t xs[4] = {xn.x, xn.y, xn.z, xn.w};
    uint4 wv[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) wv[q] = wn[q];
    load(min(c + kWave, nchunk - 1));  // one chunk ahead
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const double x0 = (double)__uint_as_float(xs[i] << 16);
      const double x1 = (double)__uint_as_float(xs[i] & 0xffff0000u);
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        const uint32_t ws[4] = {wv[q].x, wv[q].y, wv[q].z, wv[q].w};
        acc[q] = fma(x0, (double)__uint_as_float(ws[i] << 16), acc[q]);
        acc[q] = fma(x1, (double)__uint_as_float(ws[i] & 0xffff0000u), acc[q]);
      }
    }
  }
#pragma unroll
  for (int q = 0; q < NC; ++q) out[q] = (float)wave_sum_f64(acc[q]);
}

// logits_of for the first 8, 4, 2 or 1 of n experts: id(j) gives the j-th,
// out(j, logit) takes its logit on every lane. Returns how many.
template <typename Id, typename Out>
__device__ __forceinline__ int run_of_logits(const uint4* __restrict__ xr,
                                             const uint16_t* __restrict__ wg, int d, int n, Id id,
                                             Out out) {
  auto take = [&](auto nc) {
    constexpr int NC = decltype(nc)::value;
    int e[NC];
    float v[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) e[j] = id(j);
    logits_of<NC>(xr, wg, d, e, v);
#pragma unroll
    for (int j = 0; j < NC; ++j) out(j, v[j]);
    return NC;
  };
  if (n >= 8) return take(std::integral_constant<int, 8>{});
  if (n >= 4) return take(std::integral_constant<int, 4>{});
  if (n >= 2) return take(std::integral_constant<int, 2>{});
  return take(std::integral_constant<int, 1>{});
}

// Weight mode for many experts: a screen on the matrix cores, then float64
// logits only for the experts that can be among the k largest.
//
// Screen: 16 waves form s~[t,e], the float32 dot products of TT token rows
// with every gate row, by v_mfma_f32_16x16x32_bf16, and beside them
// a[t,e] = sum_i |x_i w_i| from the same fragments with the sign bits
// cleared. bf16 products are exact in float32, so |s~ - s| comes from the
// additions alone: an accumulator takes at most 256 products before it is
// added to the wave's float32 total and cleared, and each of those
// additions, however the unit orders or truncates them, loses at most
// 2^-23 of the running magnitude, which a bounds. With nadd additions on any
// product's way, |s~ - s| <= nadd * 2^-23 * a; the host passes twice that,
// and a term for products below the smallest float32 (`tiny`). (Denormal
// bf16 inputs and float32 results are kept by this instruction: checked on
// an MI355X, where the largest error found over adversarial operands was
// 3.8 * 2^-23 * a for an instruction's 32 products and 8.2 * 2^-23 * a for an
// accumulator's 256.) A bound that is not
// finite keeps its expert.
//
// Selection: tau, the k-th largest of the 64 lanes' largest s~ - B (lane l
// holds experts l, l + 64, ...), is reached by k experts and so at most the
// k-th largest exact logit: an expert with s~ + B < tau cannot be chosen, nor
// tie. The others get their float64 logits, one wave per token, and the top-k
// runs over those: ids and weights have the bits that all E float64 logits
// would give. For independent logits of more than 64 experts these are the
// sum of 64 / (64 - i) over i < k, as two of the largest may share a lane, and
// what the bounds leave open: 8.5 for k = 8, 18 for 16, 44 for 32.
//
// Both operands go global -> LDS with buffer loads that write LDS directly,
// 128 bytes of a row at a time, through a ring of NB stage buffers; 16-byte
// chunks sit XOR-swizzled in their row against bank conflicts. A stage holds
// 256 gate-matrix rows of 64 elements: for
// P = 1 rows of 256 experts, for P > 1 the rows of 256 / P experts at P
// consecutive 64-element pieces of the hidden dimension. A wave multiplies
// two tiles of 16 experts by one 32-deep half of their stage, so that a token
// fragment read from LDS serves two products (with one tile and both halves
// per wave the LDS reads, 64 KB a stage, set the pace); the 2 P parts' sums
// are added at the end.
constexpr int kScreenWaves = 16;  // waves, and tokens, per block

template <int P>
struct ScreenShape {
  static constexpr int TT = 16;                // tokens per block
  static constexpr int GE = 256 / P;           // experts at once
  static constexpr int NB = P == 4 ? 3 : 4;    // stage buffers
  static constexpr int W_ST = 256 * 64;        // elements per stage
  static constexpr int X_ST = P * TT * 64;
  static constexpr int LDS = NB * (W_ST + X_ST) * 2;
  static_assert(LDS <= 160 * 1024 && 2 * P * TT * GE * 8 <= LDS, "the sums take the ring's place");
};

typedef uint32_t u32x4g __attribute__((ext_vector_type(4)));

// XOR swizzle of the eight 16-byte chunks of a staged row.
__device__ __forceinline__ int screen_swz(int r) { return (r & 7) ^ ((r >> 3) & 1); }

__device__ __forceinline__ float wave_max_f32(float v) {
#define TG_DPP_FMAX(ctrl)                                                               \
  v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xF, 0xF, \
                                                          false)))
  TG_DPP_FMAX(0xB1);
  TG_DPP_FMAX(0x4E);
  TG_DPP_FMAX(0x141);
  TG_DPP_FMAX(0x140);
#undef TG_DPP_FMAX
  float m = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0));
#pragma unroll
  for (int r = 1; r < 4; ++r)
    m = fmaxf(m, __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16 * r)));
  return m;
}

// Top-k of one token by one wave: lane l holds the bounds lo and hi of the
// experts l, l + 64, ... `scratch`: LDS of the wave's own, 6 E bytes.
template <int NQ>
__device__ __forceinline__ void screened_topk(const float* lo, const float* hi, char* scratch,
                                              const uint4* __restrict__ xr,
                                              const uint16_t* __restrict__ wg, int d, int E, int k,
                                              int t, int32_t* __restrict__ ids,
                                              float* __restrict__ w) {
  const int lane = lane_id();
  // tau: the k-th largest of the lanes' largest lower bounds, or lower where
  // lanes are equal. k experts reach it, so it is at most the k-th largest of
  // all lower bounds (two of the k largest in one lane cost a candidate).
  float best = lo[0];
#pragma unroll
  for (int q = 1; q < NQ; ++q) best = fmaxf(best, lo[q]);
  float tau = 0.0f;
  for (int j = 0; j < k; ++j) {
    tau = wave_max_f32(best);
    best = best == tau ? -__builtin_inff() : best;
  }
  // The candidates in expert order, as a list in LDS.
  float* const lg = reinterpret_cast<float*>(scratch);
  uint16_t* const list = reinterpret_cast<uint16_t*>(lg + E);
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  int n = 0;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int e = lane + q * kWave;
    const bool on = e < E && !(hi[q] < tau);
    const uint64_t m = __ballot(on);
    if (on) list[n + __builtin_popcountll(m & lt)] = (uint16_t)e;
    if (e < E) lg[e] = -__builtin_inff();
    n += __builtin_popcountll(m);
  }
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  float my_v = -__builtin_inff();
  for (int i = 0; i < n;) {
    i += run_of_logits(xr, wg, d, n - i,
                       [&](int j) { return __builtin_amdgcn_readfirstlane((int)list[i + j]); },
                       [&](int j, float v) {
                         if (n <= kWave) my_v = (lane == i + j) ? v : my_v;
                         else if (lane == 0) lg[list[i + j]] = v;
                       });
  }
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  if (n > kWave) {
    wave_topk<NQ>(lg, E, k, t, ids, w);
  } else {  // lane l holds candidate l
    const int id = lane < n ? (int)list[lane] : 0x7fffffff;
    wave_topk_lanes(my_v, id, n, k, t, ids, w);
  }
}

template <int P, int NG>
__global__ __launch_bounds__(64 * kScreenWaves) void gate_screen_topk_kernel(
    const uint16_t* __restrict__ x, const uint16_t* __restrict__ wg, int T, int d, int E, int k,
    float bound, float tiny, int32_t* __restrict__ ids, float* __restrict__ w) {
  using Sh = ScreenShape<P>;
  constexpr int TT = Sh::TT, GE = Sh::GE, NB = Sh::NB, W_ST = Sh::W_ST, X_ST = Sh::X_ST;
  constexpr int kOut = (int)0x80000000u;  // an offset past any resource: reads zeros
  constexpr int XI = X_ST / 512;          // x load instructions per stage (512 elements each)
  __shared__ __attribute__((aligned(16))) uint16_t smem[Sh::LDS / 2];
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int t0 = blockIdx.x * TT;
  const int nstage = (d + 64 * P - 1) / (64 * P);
  lds_u16* const smem3 = (lds_u16*)smem;

  // Load instruction i of a stage fills 8 rows of 128 bytes; lane l writes
  // chunk position l % 8 of row l / 8 and fetches the chunk that the swizzle
  // puts there. Wave w loads rows 16 w .. 16 w + 15 of the gate matrix's
  // stage, the first XI waves 8 rows of x each. Experts past the last read
  // zeros, as do tokens past the last and pieces past d.
  const __amdgpu_buffer_rsrc_t x_rsrc =
      make_rsrc(x + (size_t)t0 * d, (uint32_t)min(TT, T - t0) * d * 2);
  const int wp = wave * 16 / GE;  // the wave's piece of the hidden dimension
  int w_off[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = wave * 16 + i * 8 + lane / 8;
    w_off[i] = ((r % GE) * d + wp * 64 + ((lane % 8) ^ screen_swz(r)) * 8) * 2;
  }
  const int xp = wave / 2;  // piece and rows of the wave's x load (wave < XI)
  const int xr = (wave % 2) * 8 + lane / 8;
  const int x_off = (xr * d + xp * 64 + ((lane % 8) ^ screen_swz(xr)) * 8) * 2;
  __amdgpu_buffer_rsrc_t w_rsrc;
  auto issue = [&](int st, int buf) {
    const int k0 = min(st, nstage - 1) * 64 * P;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      load_lds16(w_rsrc, smem3 + buf * W_ST + (wave * 16 + i * 8) * 64,
                 k0 + wp * 64 < d ? w_off[i] : kOut, k0 * 2);
    if (wave < XI)
      load_lds16(x_rsrc, smem3 + NB * W_ST + buf * X_ST + wave * 512,
                 k0 + xp * 64 < d ? x_off : kOut, k0 * 2);
  };
  // The wave multiplies rows 32 (w / 2) .. + 31 of a stage by its half w % 2.
  // Fragments: row l % 16 of a tile (or of x), chunk 4 half + l / 16.
  const int half = wave & 1, fr = (wave >> 1) * 32 + (lane & 15), fp = (wave >> 1) * 32 / GE;
  const int fchunk = 4 * half + lane / 16;
  const int woff[2] = {fr * 64 + ((fchunk ^ screen_swz(fr)) << 3),
                       (fr + 16) * 64 + ((fchunk ^ screen_swz(fr + 16)) << 3)};
  const int xoff = NB * W_ST + (fp * TT + (lane & 15)) * 64 + ((fchunk ^ screen_swz(lane & 15)) << 3);

  // Lane l: bounds of experts l, l + 64, ... for the wave's token, group by group.
  constexpr int GQ = GE / kWave, NQ = NG * GQ;
  float lo[NQ], hi[NQ];
  const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    const int ne = min(max(E - g * GE, 0), GE);  // experts of this group
    w_rsrc = make_rsrc(wg + (size_t)g * GE * d, (uint32_t)ne * d * 2);
    f32x4 tot[2] = {zero, zero}, tota[2] = {zero, zero}, acc[2] = {zero, zero},
          acca[2] = {zero, zero};
#pragma unroll
    for (int j = 0; j < NB - 1; ++j) issue(j, j);
    for (int st = 0; st < nstage; ++st) {
      // Stage st has landed for every wave, and every wave is done with stage
      // st - 1, whose buffer takes stage st + NB - 1.
      if (wave < XI) TG_WAIT_VM((NB - 2) * 3);
      else TG_WAIT_VM((NB - 2) * 2);
      __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
      block_barrier();
      issue(st + NB - 1, (st + NB - 1) % NB);
      const u32x4g xf = *reinterpret_cast<const u32x4g*>(smem + (st % NB) * X_ST + xoff);
      const u32x4g xa = xf & 0x7fff7fffu;
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const u32x4g wf = *reinterpret_cast<const u32x4g*>(smem + (st % NB) * W_ST + woff[b]);
        const u32x4g wa = wf & 0x7fff7fffu;
        acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            __builtin_bit_cast(bf16x8, xf), __builtin_bit_cast(bf16x8, wf), acc[b], 0, 0, 0);
        acca[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            __builtin_bit_cast(bf16x8, xa), __builtin_bit_cast(bf16x8, wa), acca[b], 0, 0, 0);
      }
      if ((st & 7) == 7 || st == nstage - 1) {  // 256 products
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          tot[b] += acc[b];
          tota[b] += acca[b];
          acc[b] = acca[b] = zero;
        }
      }
    }
    TG_WAIT_VM(0);
    __syncthreads();  // no load may land in the ring any more
    // Register r of lane l: token 4 (l / 16) + r, expert l % 16 of the tile.
    float2* const part = reinterpret_cast<float2*>(smem);  // [2 P][TT][GE]
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        part[((2 * fp + half) * TT + 4 * (lane / 16) + r) * GE + (fr + 16 * b) % GE] =
            make_float2(tot[b][r], tota[b][r]);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < GQ; ++q) {
      const int e = lane + q * kWave;
      float s = 0.0f, a = 0.0f;
#pragma unroll
      for (int p = 0; p < 2 * P; ++p) {
        const float2 v = part[(p * TT + wave) * GE + e];
        s += v.x;
        a += v.y;
      }
      const float bd = fmaf(a, bound, tiny);
      // Not finite: nothing is known of this logit.
      const bool known = bd < __builtin_inff();
      lo[g * GQ + q] = e < ne && known ? s - bd : -__builtin_inff();
      hi[g * GQ + q] = e < ne ? (known ? s + bd : __builtin_inff()) : -__builtin_inff();
    }
    __syncthreads();  // the sums have been read: the ring and the scratch take their place
  }
  const int t = t0 + wave;  // one token per wave
  if (t < T)
    screened_topk<NQ>(lo, hi, reinterpret_cast<char*>(smem) + (size_t)wave * 6 * NG * GE,
                      reinterpret_cast<const uint4*>(x + (size_t)t * d), wg, d, E, k, t, ids, w);
}

// Weight mode, few tokens: one token per block of NW waves, each taking an
// equal run of experts, up to eight at a time, straight from L2. (One token
// per wave would leave most of the chip idle.)
template <int NW>
__global__ __launch_bounds__(64 * NW) void gate_token_topk_kernel(
    const uint16_t* __restrict__ x, const uint16_t* __restrict__ wg, int d, int E, int k,
    float* __restrict__ logits_out, int32_t* __restrict__ ids, float* __restrict__ w) {
  __shared__ float lg[1024];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int t = blockIdx.x;
  const uint4* const xr = reinterpret_cast<const uint4*>(x + (size_t)t * d);
  const int per = (E + NW - 1) / NW, end = min(E, (wave + 1) * per);
  for (int e0 = wave * per; e0 < end;) {
    e0 += run_of_logits(xr, wg, d, end - e0, [&](int j) { return e0 + j; },
                        [&](int j, float v) {
                          if (lane_id() == 0) {
                            lg[e0 + j] = v;
                            if (logits_out) logits_out[(size_t)t * E + e0 + j] = v;
                          }
                        });
  }
  __syncthreads();
  if (wave == 0) wave_topk_any(lg, E, k, t, ids, w);
}

// Four chunks of 8 elements, one per 16-lane row of the wave (row q holds chunk
// q of its lane's token or expert), turned over: out[m] on row q gets elements
// q (low half) and 4 + q (high half) of chunk m.
__device__ __forceinline__ void turn_chunks(const uint4& v, uint32_t* out) {
  // Word j: elements j and 4 + j of the lane's own chunk. Then the 4 x 4 blocks
  // of (word, row) are transposed: rows 2, 3 of words 0, 1 against rows 0, 1 of
  // words 2, 3, then odd rows of even words against even rows of odd ones.
  const uint32_t w0 = __builtin_amdgcn_perm(v.z, v.x, 0x05040100);
  const uint32_t w1 = __builtin_amdgcn_perm(v.z, v.x, 0x07060302);
  const uint32_t w2 = __builtin_amdgcn_perm(v.w, v.y, 0x05040100);
  const uint32_t w3 = __builtin_amdgcn_perm(v.w, v.y, 0x07060302);
  const auto a = __builtin_amdgcn_permlane32_swap(w0, w2, false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(w1, w3, false, false);
  const auto lo = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
  out[0] = lo[0];
  out[1] = lo[1];
  out[2] = hi[0];
  out[3] = hi[1];
}

// All logits [T, E] in float64 on the matrix cores (v_mfma_f64_16x16x4: the
// rate of the vector unit's float64 FMA, but the operands are widened once
// per 16 tokens or experts instead of once per product, beside it). A block
// of 16 waves forms 16 tokens x 16 experts. The instruction adds its four
// products to the accumulator one after the other, each rounded as an FMA
// (checked on an MI355X: 2^20 sums, none different), so chains of it give the
// partial sums of logits_of bit for bit: wave w holds partial sums 4 w .. + 3 in
// four accumulators, takes the 32-element pieces w, w + 16, ... (four chunks)
// and feeds chunk m to accumulator m, elements 0-3 and then 4-7. Lane l loads
// chunk l / 16 of row l % 16 and gets element l / 16 of each half of all four
// chunks by turn_chunks. The waves' sums are added in LDS in the order of
// wave_sum_f64 and rounded once. 4096 x 256 x 7168: 310 us, 48 TFLOP/s of
// float64 (280 us with one accumulator per wave and no turning, in an order of
// its own; the float64 MFMA does not overlap the vector unit's work). Wider
// tiles with fewer waves measured 5 % faster there and half as fast at 128
// tokens.
// TOPK (E <= 16): the block holds all logits of its tokens and finishes them,
// one wave each; logits may then be null.
typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int kDenseWaves = 16;
template <bool TOPK>
__global__ __launch_bounds__(64 * kDenseWaves) void gate_logits_f64_kernel(
    const uint16_t* __restrict__ x, const uint16_t* __restrict__ wg, int T, int d, int E, int k,
    float* __restrict__ logits, int32_t* __restrict__ ids, float* __restrict__ w) {
  __shared__ float lg[TOPK ? 16 : 1][16];
  __shared__ f64x4 part[kDenseWaves][kWave];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int lane = lane_id();
  const int t0 = blockIdx.x * 16, e0 = blockIdx.y * 16;
  // Rows past the last token or expert repeat it; they are not stored.
  const uint16_t* const xr = x + (size_t)min(t0 + (lane & 15), T - 1) * d + 8 * (lane / 16);
  const uint16_t* const wr = wg + (size_t)min(e0 + (lane & 15), E - 1) * d + 8 * (lane / 16);
  const int np = d / 32;
  auto widen = [](uint32_t u, int half) {
    return (double)__uint_as_float(half ? u & 0xffff0000u : u << 16);
  };
  f64x4 acc[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) acc[m] = f64x4{0.0, 0.0, 0.0, 0.0};
  uint4 xn, wn;
  auto load = [&](int p) {
    p = min(p, np - 1);
    xn = *reinterpret_cast<const uint4*>(xr + p * 32);
    wn = *reinterpret_cast<const uint4*>(wr + p * 32);
  };
  load(wave);
  for (int p = wave; p < np; p += kDenseWaves) {
    uint32_t xv[4], wv[4];
    turn_chunks(xn, xv);
    turn_chunks(wn, wv);
    load(p + kDenseWaves);
#pragma unroll
    for (int half = 0; half < 2; ++half)
#pragma unroll
      for (int m = 0; m < 4; ++m)
        acc[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(widen(xv[m], half), widen(wv[m], half),
                                                      acc[m], 0, 0, 0);
  }
  part[wave][lane] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  __syncthreads();
  if (wave == 0) {
    f64x4 sum = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < kDenseWaves; q += 4)
      sum += (part[q][lane] + part[q + 1][lane]) + (part[q + 2][lane] + part[q + 3][lane]);
    // Register r of lane l: token 4 r + l / 16, expert l % 16.
    const int e = e0 + (lane & 15);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int t = t0 + 4 * r + lane / 16;
      if (TOPK) lg[4 * r + lane / 16][lane & 15] = (float)sum[r];
      if (t < T && e < E && (!TOPK || logits)) logits[(size_t)t * E + e] = (float)sum[r];
    }
  }
  if (TOPK) {
    __syncthreads();
    if (t0 + wave < T) wave_topk<1>(lg[wave], E, k, t0 + wave, ids, w);
  }
}

__global__ __launch_bounds__(256) void logits_topk_kernel(const float* __restrict__ logits, int T,
                                                          int E, int k, int32_t* __restrict__ ids,
                                                          float* __restrict__ w) {
  __shared__ float lg_s[kWaves][1024];
  const int wave = threadIdx.x / kWave;
  const int lane = lane_id();
  const int t = blockIdx.x * kWaves + wave;
  float* lg = lg_s[wave];
  if (t >= T) return;
  for (int e = lane; e < E; e += kWave) lg[e] = logits[(size_t)t * E + e];
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  wave_topk_any(lg, E, k, t, ids, w);
}

// Logits mode for E <= 256 and k <= 16: four tokens per wave, one 16-lane
// DPP row per token; lane l of a row holds the candidates l, l + 16, ... of its
// token in registers. A candidate's 64-bit key is the float32 logit in an
// order-preserving encoding (-0 taken as +0) above the complement of the
// expert id, so a larger key is a larger logit or, on equal logits, a lower
// id, and no two keys are equal. Two kernels, chosen by launch_logits_topk:
//   rounds  takes every lane's largest key below the previous winner's, k
//           times, reduced over the row with the four DPP row steps;
//   rows    counts larger keys among a few candidates instead.
// Both sum the k exponentials in rank order, the same sum as the
// one-token-per-wave kernel.
//
// skip_nan: a NaN logit is never chosen, as in wave_topk, and a choice left
// empty for it has id 0x7fffffff. Otherwise NaN logits are ordered by their
// bits (the positive ones above +inf, the negative ones below -inf).
constexpr int kRowTokens = 4;  // tokens per wave

__device__ __forceinline__ uint64_t topk_key(float v, int e) {
  uint32_t u = __float_as_uint(v == 0.0f ? 0.0f : v);
  u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return ((uint64_t)u << 32) | (0xffffffffu - (uint32_t)e);
}

__device__ __forceinline__ float key_value(uint64_t key) {
  const uint32_t u = (uint32_t)(key >> 32);
  return __uint_as_float((u & 0x80000000u) ? (u & 0x7fffffffu) : ~u);
}

__device__ __forceinline__ uint64_t row_max_key(uint64_t k) {
#define TG_DPP_MAX(ctrl)                                                                  \
  do {                                                                                    \
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)k, ctrl, 0xF, 0xF,   \
                                                    false);                               \
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(k >> 32), ctrl,     \
                                                    0xF, 0xF, false);                     \
    const uint64_t o = ((uint64_t)hi << 32) | lo;                                         \
    k = o > k ? o : k;                                                                    \
  } while (0)
  TG_DPP_MAX(0xB1);   // quad_perm [1,0,3,2]
  TG_DPP_MAX(0x4E);   // quad_perm [2,3,0,1]
  TG_DPP_MAX(0x141);  // row_half_mirror
  TG_DPP_MAX(0x140);  // row_mirror
#undef TG_DPP_MAX
  return k;
}

#define TG_ROW_MOV(v, ctrl) __builtin_amdgcn_update_dpp(0, v, ctrl, 0xF, 0xF, false)

// Largest value of the row, on every lane of it.
__device__ __forceinline__ float row_max_f32(float v) {
  v = fmaxf(v, __int_as_float(TG_ROW_MOV(__float_as_int(v), 0xB1)));
  v = fmaxf(v, __int_as_float(TG_ROW_MOV(__float_as_int(v), 0x4E)));
  v = fmaxf(v, __int_as_float(TG_ROW_MOV(__float_as_int(v), 0x141)));
  return fmaxf(v, __int_as_float(TG_ROW_MOV(__float_as_int(v), 0x140)));
}

// k rounds; the vector ALU bounds it, NQ + 4 64-bit maxima a round. (SKIP at run
// time cost 100000 tokens of 8 experts, k = 1, 6.7 us instead of 5.5.)
template <int NQ, bool SKIP>
__global__ __launch_bounds__(256) void logits_topk_rounds_kernel(const float* __restrict__ logits,
                                                                 int T, int E, int k,
                                                                 int32_t* __restrict__ ids,
                                                                 float* __restrict__ w) {
  const int lane = lane_id();
  const int l16 = lane & 15;
  const int t = (blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave) * kRowTokens + (lane >> 4);
  const bool on = t < T;
  uint64_t key[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int e = l16 + 16 * q;
    key[q] = 0;  // no candidate
    if (on && e < E) {
      const float v = logits[(size_t)t * E + e];
      key[q] = SKIP && v != v ? 0 : topk_key(v, e);
    }
  }
  // An empty choice: value -inf, id 0x7fffffff, a key below those of -inf logits.
  constexpr uint64_t empty = SKIP ? 0x007fffff80000000ull : 0;
  uint64_t thr = ~0ull;
  float my_v = 0.0f, v0 = 0.0f, z = 0.0f;
  int my_id = 0;
  for (int j = 0; j < k; ++j) {
    uint64_t best = empty;
#pragma unroll
    for (int q = 0; q < NQ; ++q) best = (key[q] < thr && key[q] > best) ? key[q] : best;
    best = row_max_key(best);  // every lane of the row: this round's winner
    thr = best;
    const float bv = key_value(best);
    if (j == 0) v0 = bv;
    const float ex = expf(bv - v0);
    z += ex;
    if (l16 == j) {
      my_v = ex;
      my_id = (int)(0xffffffffu - (uint32_t)best);
    }
  }
  if (on && l16 < k) {
    ids[(size_t)t * k + l16] = my_id;
    w[(size_t)t * k + l16] = my_v / z;
  }
}

// tau, the k-th largest of the row's (up to) 32 half maxima (each lane's
// candidates alternate between two halves, which are even for any E: with the
// lower and the upper half of NQ, 16384 tokens of 160 experts, k = 8, took 8.4 us
// instead of 6.2), or lower where some are equal, is reached by at least k
// candidates, so only candidates >= tau can be chosen: k and a few more. They
// are gathered into the row's lanes through LDS, a lane's rank is the number of
// larger keys among the row's 16, and the lanes take their candidates in rank
// order. With more than 16 candidates in one of the wave's rows (k near 16,
// many equal logits, or NaN among them) the wave finds the winners round by
// round after all, having formed tau for nothing: 10 to 30 % slower than the
// other kernel.
template <int NQ>
__global__ __launch_bounds__(256) void logits_topk_rows_kernel(const float* __restrict__ logits,
                                                               int T, int E, int k,
                                                               int32_t* __restrict__ ids,
                                                               float* __restrict__ w,
                                                               bool skip_nan) {
  __shared__ uint64_t list_s[4][kRowTokens][16];
  const int lane = lane_id();
  const int wave = threadIdx.x / kWave;
  const int l16 = lane & 15;
  const int t = (blockIdx.x * (blockDim.x / kWave) + wave) * kRowTokens + (lane >> 4);
  const bool on = t < T;
  float v[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int e = l16 + 16 * q;
    v[q] = (on && e < E) ? logits[(size_t)t * E + e] : -__builtin_inff();
  }
  float m0 = -__builtin_inff(), m1 = m0;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    if (q % 2 == 0) m0 = fmaxf(m0, v[q]);
    else m1 = fmaxf(m1, v[q]);
  }
  float tau = 0.0f;
  for (int j = 0; j < k; ++j) {
    tau = row_max_f32(fmaxf(m0, m1));
    m0 = m0 == tau ? -__builtin_inff() : m0;
    m1 = m1 == tau ? -__builtin_inff() : m1;
  }
  // A NaN is a candidate unless it is skipped.
  uint32_t mine = 0;
#pragma unroll
  for (int q = 0; q < NQ; ++q)
    mine |= (l16 + 16 * q < E && (skip_nan ? v[q] >= tau : !(v[q] < tau)) ? 1u : 0u) << q;
  const int cnt = __builtin_popcount(mine);
  int incl = cnt;  // over the row's lanes up to this one
  incl += TG_ROW_MOV(incl, 0x111);  // row_shr 1, 2, 4, 8
  incl += TG_ROW_MOV(incl, 0x112);
  incl += TG_ROW_MOV(incl, 0x114);
  incl += TG_ROW_MOV(incl, 0x118);
  const int n = TG_ROW_MOV(incl, 0x15F);  // row_newbcast 15: the row's total
  float my_v = 0.0f;
  int my_id = 0;
  if (!__ballot(on && n > 16)) {
    uint64_t* const list = list_s[wave][lane >> 4];
    int pos = incl - cnt;
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      if (on && (mine >> q & 1)) list[pos++] = topk_key(v[q], l16 + 16 * q);
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    const uint64_t key = on && l16 < n ? list[l16] : 0;
    int rank = 0;
#define TG_RANK(i)                                                                       \
  do {                                                                                   \
    const uint32_t lo = (uint32_t)TG_ROW_MOV((int)(uint32_t)key, 0x120 + i);             \
    const uint32_t hi = (uint32_t)TG_ROW_MOV((int)(uint32_t)(key >> 32), 0x120 + i);     \
    rank += ((uint64_t)hi << 32 | lo) > key ? 1 : 0;                                     \
  } while (0)
    TG_RANK(1); TG_RANK(2); TG_RANK(3); TG_RANK(4); TG_RANK(5); TG_RANK(6); TG_RANK(7);
    TG_RANK(8); TG_RANK(9); TG_RANK(10); TG_RANK(11); TG_RANK(12); TG_RANK(13); TG_RANK(14);
    TG_RANK(15);
#undef TG_RANK
    const int to = 4 * ((lane & 48) + (l16 < n ? rank : l16));
    const float kv = key ? key_value(key) : -__builtin_inff();
    const int kid = key ? (int)(0xffffffffu - (uint32_t)key) : 0x7fffffff;
    my_v = __int_as_float(__builtin_amdgcn_ds_permute(to, __float_as_int(kv)));
    my_id = __builtin_amdgcn_ds_permute(to, kid);
  } else {
    uint64_t key[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      key[q] = (mine >> q & 1) ? topk_key(v[q], l16 + 16 * q) : 0;  // 0: no candidate
    uint64_t thr = ~0ull;
    for (int j = 0; j < k; ++j) {
      uint64_t best = 0;
#pragma unroll
      for (int q = 0; q < NQ; ++q) best = (key[q] < thr && key[q] > best) ? key[q] : best;
      thr = row_max_key(best);  // every lane of the row: this round's winner
      if (l16 == j) {
        my_v = thr ? key_value(thr) : -__builtin_inff();
        my_id = thr ? (int)(0xffffffffu - (uint32_t)thr) : 0x7fffffff;
      }
    }
  }
  // Lane j of the row holds the j-th choice; row_newbcast j in rank order.
  const float v0 = __int_as_float(TG_ROW_MOV(__float_as_int(my_v), 0x150));
  const float ex = expf(my_v - v0);
  float z = 0.0f;
#define TG_SUM(j) \
  if (j < k) z += __int_as_float(TG_ROW_MOV(__float_as_int(ex), 0x150 + j))
  TG_SUM(0); TG_SUM(1); TG_SUM(2); TG_SUM(3); TG_SUM(4); TG_SUM(5); TG_SUM(6); TG_SUM(7);
  TG_SUM(8); TG_SUM(9); TG_SUM(10); TG_SUM(11); TG_SUM(12); TG_SUM(13); TG_SUM(14); TG_SUM(15);
#undef TG_SUM
#undef TG_ROW_MOV
  if (on && l16 < k) {
    ids[(size_t)t * k + l16] = my_id;
    w[(size_t)t * k + l16] = ex / z;
  }
}

// Additions on the way of any product of the screen: 256 within an
// accumulator, one per chunk, and the parts' sum; doubled.
template <int P, int NG>
void launch_screen(const uint16_t* x, const uint16_t* wg, int T, int d, int E, int k, int32_t* ids,
                   float* w, hipStream_t stream) {
  constexpr int TT = ScreenShape<P>::TT;
  const double nadd = 256.0 + (d / 64 + 7) / 8 + 2 * P;
  const float bound = (float)(2.0 * nadd * 0x1p-23), tiny = (float)(d * 0x1p-126);
  hipLaunchKernelGGL((gate_screen_topk_kernel<P, NG>), dim3((T + TT - 1) / TT),
                     dim3(64 * kScreenWaves), 0, stream, x, wg, T, d, E, k, bound,
                     tiny, ids, w);
}

void launch_logits_topk(const float* logits, int T, int E, int k, int32_t* ids, float* w,
                        bool skip_nan, hipStream_t stream) {
  // us at 2048 | 16384 | 100000 tokens: one token per wave, rounds, rows
  //   256 experts  k = 1    3.2  3.4  4.2 |  -  5.0  5.6 |  -   25   21
  //                k = 3    4.3  4.2  4.5 |  -  6.5  5.9 |  -   31   22
  //                k = 8    7.1  6.7  5.1 |  -   11  6.7 |  -   47   26
  //                k = 11   8.8  7.8  8.9 |  -   13   13 |  -   58   39
  //                k = 16    12  9.6   11 |  -   17   19 |  -   79   89
  //   8 experts    k = 2    3.0  2.6  2.9 |  -  3.0  3.8 |  -  7.6   11
  //                k = 4    3.7  3.0  3.0 |  -  3.8  4.1 |  -   12   13
  //                k = 8    5.3  3.7  3.3 |  -  5.6  4.7 |  -   22   16
  // Rounds cost in proportion to k and, beyond a few ten thousand tokens, where
  // the vector ALU is full, to E. Rows cost little until a wave's candidates
  // are too many: never with 32 experts, each a half's maximum, else from about
  // ten choices on, which delays all of a small batch but few waves of a large
  // one. A wave per token is the shortest chain for a few rounds over many
  // experts while there are waves to spare.
  const bool wave = T < 4096 && E > 64 && k <= (E > 128 ? 3 : 2);
  if (E <= 256 && k <= 16 && !wave) {
    // Few tokens: one wave per block, so that more CUs take part.
    const int waves = T >= 4096 ? 4 : 1;
    const int per_block = waves * kRowTokens;
    const dim3 grid((T + per_block - 1) / per_block), block(64 * waves);
    const int least = E <= 64 ? 5 : T > 32768 ? 1 : E <= 128 ? 4 : 3;
    const int most = E <= 32 ? 16 : T > 32768 ? 12 : T > 8192 ? 11 : E <= 64 ? 10 : 9;
    const bool rows = k >= least && k <= most;
#define TG_ROWS(NQ)                                                                      \
  hipLaunchKernelGGL(logits_topk_rows_kernel<NQ>, grid, block, 0, stream, logits, T, E, k, \
                     ids, w, skip_nan)
#define TG_ROUNDS(NQ, SKIP)                                                                   \
  hipLaunchKernelGGL((logits_topk_rounds_kernel<NQ, SKIP>), grid, block, 0, stream, logits, T, \
                     E, k, ids, w)
    if (rows) {
      if (E <= 64) TG_ROWS(4);
      else if (E <= 128) TG_ROWS(8);
      else TG_ROWS(16);
    } else if (skip_nan) {
      if (E <= 64) TG_ROUNDS(4, true);
      else if (E <= 128) TG_ROUNDS(8, true);
      else TG_ROUNDS(16, true);
    } else {
      if (E <= 64) TG_ROUNDS(4, false);
      else if (E <= 128) TG_ROUNDS(8, false);
      else TG_ROUNDS(16, false);
    }
#undef TG_ROWS
#undef TG_ROUNDS
  } else {
    hipLaunchKernelGGL(logits_topk_kernel, dim3((T + kWaves - 1) / kWaves), dim3(256), 0, stream,
                       logits, T, E, k, ids, w);
  }
}

// Which kernel forms the logits in weight mode. `stored`: there is memory for
// all T x E logits (the caller wants them, or has scratch to lend). Measured,
// us, calls of tg_gate_topk back to back (dense counts its second launch, the
// top-k, from E = 17 on; `before`: one token per wave, the gate matrix in LDS
// where it fits, else from L2):
//   d, E, k       T =            1    128    512   1024   2048   4096
//   7168, 256, 8  token         54     56      -      -      -      -
//                 dense         26     29     47     84    159    310
//                 screen        71     96     99    101    101    102
//                 before      1073   1177   1184   1212   1185   1334
//   4096, 64, 6   token         12     13      -      -      -      -
//                 dense         16     17     17     17     29     51
//                 screen        19     30     31     31     32     32
//                 before        94    116    111    178    176    187
//   7168, 16, 8   token          -      -     18     32      -      -
//                 dense          -      -     28     28     29     30
//                 before         -      -     51     79     79     88
//   4096, 8, 2    token        4.6    5.0    6.6    9.3      -      -
//                 dense          -      -     16     16     17     17
//                 screen        13     17     18     18     19     21
//                 before       9.8     17     17     18     18     19
enum GateKernel { kGateToken, kGateDense, kGateDenseTopk, kGateScreen };
GateKernel gate_kernel(int T, int d, int E, bool wanted, bool stored) {
  // One block per token: about one round of blocks over the chip, or, with
  // at most 16 experts (one per wave), a few. A token's E x d products at one
  // CU's rate are worth dense's second launch from about half a million on.
  const bool few = T <= (E <= 8 ? 1024 : E <= 16 ? 512 : 256);
  if (few && !(stored && (long long)E * d > 512 * 1024)) return kGateToken;
  if (E <= 16) return kGateDenseTopk;
  if (wanted) return kGateDense;
  // Dense costs T x E x d, the screen a pass over the gate matrix per 16
  // tokens of a CU: equal near 1300 tokens of 256 experts, 2100 of 64.
  const long long te = (long long)T * E;
  if (stored && te <= (E <= 128 ? 1 << 17 : 1 << 18)) return kGateDense;
  // The screen addresses 256 experts' rows at once with 31-bit byte offsets.
  if (512LL * d < (1LL << 31)) return kGateScreen;
  return stored ? kGateDense : kGateToken;
}

}  // namespace

hipError_t launch_gate_topk(const uint16_t* x, const uint16_t* wg, const float* logits_in, int T,
                            int d, int E, int k, float* logits_out, int32_t* ids, float* w,
                            hipStream_t stream, float* scratch) {
  if (T == 0) return hipSuccess;
  if (logits_in) {
    // From 4096 tokens on NaN logits are ordered, below and in the other
    // kernels skipped.
    launch_logits_topk(logits_in, T, E, k, ids, w, T < 4096, stream);
    return hipGetLastError();
  }
  float* const logits = logits_out ? logits_out : scratch;
  switch (gate_kernel(T, d, E, logits_out != nullptr, logits != nullptr)) {
    case kGateToken:
      // 8 waves, so that more blocks share a CU, where that is a wave per expert.
      if (E <= 8)
        hipLaunchKernelGGL(gate_token_topk_kernel<8>, dim3(T), dim3(64 * 8), 0, stream, x, wg, d, E,
                           k, logits_out, ids, w);
      else
        hipLaunchKernelGGL(gate_token_topk_kernel<16>, dim3(T), dim3(64 * 16), 0, stream, x, wg, d,
                           E, k, logits_out, ids, w);
      break;
    case kGateDense:
      hipLaunchKernelGGL(gate_logits_f64_kernel<false>, dim3((T + 15) / 16, (E + 15) / 16),
                         dim3(64 * kDenseWaves), 0, stream, x, wg, T, d, E, k, logits, ids, w);
      launch_logits_topk(logits, T, E, k, ids, w, true, stream);
      break;
    case kGateDenseTopk:
      hipLaunchKernelGGL(gate_logits_f64_kernel<true>, dim3((T + 15) / 16), dim3(64 * kDenseWaves),
                         0, stream, x, wg, T, d, E, k, logits_out, ids, w);
      break;
    case kGateScreen:
      if (E > 512) launch_screen<1, 4>(x, wg, T, d, E, k, ids, w, stream);
      else if (E > 256) launch_screen<1, 2>(x, wg, T, d, E, k, ids, w, stream);
      else if (E > 128) launch_screen<1, 1>(x, wg, T, d, E, k, ids, w, stream);
      else if (E > 64) launch_screen<2, 1>(x, wg, T, d, E, k, ids, w, stream);
      else launch_screen<4, 1>(x, wg, T, d, E, k, ids, w, stream);
      break;
  }
  return hipGetLastError();
}

}  // namespace tg

// Routing of many decode positions (gfx950): a LANE per token.
//
// The row-per-token routing (route_kernel) finds a token's best experts one after the other, and every
// round costs a row of 16 lanes some 60 instructions that yield one expert: with many positions in
// a launch the vector ALUs are the bound (about 3 500 instructions per position of 16 tokens), not
// the logits.  Here a lane holds all logits of one token in registers and keeps the best C of them as
// a sorted list; a logit enters it with one median-of-three per list place, all independent:
//     list[j] = med3(logit, list[j-1], list[j]),  list[0] = max(logit, list[0])
// so 64 tokens are ranked with C instructions per expert and no exchange between lanes.  The list
// holds values only.  Which experts they belong to follows from the last value that made it: the
// experts at or above it form a bit mask (two instructions per expert: difference, sign bit shifted
// in), and equal logits at the limit, the only case in which the mask has too many bits, are cut to
// the lowest ids on a path of its own.
//   Phase 1 of Algorithm 1   list of the k0 best -> mask -> OR over the position's tokens (LDS)
//   Phase 2 in closed form   everything but the union's other members masked, list of the k - k0 best -> mask
//   rank order               the experts of each mask, ascending, with their logits fetched again, are
//                            placed by counting who precedes whom (equal logits: lower id)
// A median drops logits that are not numbers.  A wavefront that meets one among its candidates ranks all its
// tokens again by the integer keys of the other routing kernels, so that results do not depend on which kernel
// a launch takes.
// 65 535 positions of B = 16, N = 128, k0 = 3: 160 us (4.0 TB/s) instead of 243 us.  A wavefront issues 3 051
// vector instructions for its four positions (13 950 before); computing alone (logits in the
// cache) takes 115 us, loading alone 125 us, and two wavefronts per SIMD overlap the two only in part.
#include "oea_internal.h"
#include "oea_route_dev.h"

#include <math.h>

namespace oea {
namespace {

constexpr int kLaneThreads = 64;   // one wavefront: nothing to wait for but its own memory operations
constexpr int kLaneChunk = 32;     // experts staged through LDS at a time
constexpr int kLanePitch = 36;     // words between token rows of a staged chunk: 16-byte aligned, no bank conflicts

// (the builtin is the bare instruction; fmaxf would quiet its operands first)
__device__ __forceinline__ float med3_raw(float a, float b, float c) { return __builtin_amdgcn_fmed3f(a, b, c); }
__device__ __forceinline__ float max_raw(float a, float b) { return __builtin_amdgcn_fmed3f(a, b, INFINITY); }

// The C largest logits, descending (minus infinity where there are fewer).
template <int C, int NE>
__device__ __forceinline__ void lane_best(const float (&v)[NE], float (&best)[C]) {
#pragma unroll
  for (int j = 0; j < C; ++j) best[j] = -INFINITY;
#pragma unroll
  for (int e = 0; e < NE; ++e) {
#pragma unroll
    for (int j = C - 1; j > 0; --j) best[j] = med3_raw(v[e], best[j - 1], best[j]);
    best[0] = max_raw(v[e], best[0]);
  }
}

// bit e of the words: v[e] >= limit.  The sign of the difference decides, except at infinite limits (two
// equal infinities differ by a NaN of either sign): everything reaches minus infinity, which is
// also the limit of a list with free places, and plus infinity is compared with (what is not a number counts
// as reaching it).
template <int NE>
__device__ __forceinline__ void lane_at_least(const float (&v)[NE], float limit, uint32_t (&m)[NE / 32]) {
#pragma unroll
  for (int w = 0; w < NE / 32; ++w) {
    uint32_t below = 0;
#pragma unroll
    for (int b = 31; b >= 0; --b)
      below = __builtin_amdgcn_alignbit(below, __float_as_uint(v[32 * w + b] - limit), 31);
    m[w] = limit == -INFINITY ? ~0u : ~below;
  }
  if (__any(limit == INFINITY)) {
#pragma unroll
    for (int w = 0; w < NE / 32; ++w) {
      uint32_t top = 0;
#pragma unroll
      for (int b = 31; b >= 0; --b) top = (top << 1) | (v[32 * w + b] < INFINITY ? 0u : 1u);
      m[w] = limit == INFINITY ? top : m[w];
    }
  }
}

template <int NW>
__device__ __forceinline__ int lane_count(const uint32_t (&m)[NW]) {
  int n = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) n += __popc(m[w]);
  return n;
}

// m holds the candidates at or above `limit`; if logits equal to the limit made them more than
// `want`, the ones with the highest ids go.  (Rare, so not in the way of the rest.)
template <int NE>
__device__ __forceinline__ void lane_cut_ties(const float (&v)[NE], float limit, int want, uint32_t (&m)[NE / 32]) {
  int extra = lane_count(m) - want;
#pragma unroll
  for (int w = NE / 32 - 1; w >= 0; --w) {
    uint32_t equal = 0;
#pragma unroll
    for (int b = 31; b >= 0; --b) equal = (equal << 1) | (v[32 * w + b] == limit ? 1u : 0u);
    equal &= m[w];
    while (extra > 0 && equal != 0) {  // at most 32 turns
      const uint32_t top = 0x80000000u >> __builtin_clz(equal);
      equal ^= top;
      m[w] ^= top;
      --extra;
    }
  }
}

// Whether one of the logits is not a number (by the bits: a comparison each would fill the scalar registers).
template <int NE>
__device__ __forceinline__ bool lane_any_nan(const float (&v)[NE]) {
  uint32_t most = 0;
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    const uint32_t u = __float_as_uint(v[e]) & 0x7fffffffu;
    most = u > most ? u : most;
  }
  return most > 0x7f800000u;
}

// value at a wave-uniform place of a list (by masks: a chain of selects is taken for an indexed load
// and puts the list into memory)
template <int C>
__device__ __forceinline__ float list_at(const float (&v)[C], int place) {
  uint32_t r = 0;
#pragma unroll
  for (int j = 0; j < C; ++j) r |= __float_as_uint(v[j]) & (j == place ? ~0u : 0u);
  return __uint_as_float(r);
}

// The experts of mask m, ascending: ids to id[FROM .. FROM + C), 0 for places past the last one.
template <int FROM, int C, int NW, int K>
__device__ __forceinline__ void lane_ids(const uint32_t (&m)[NW], int N, int (&id)[K]) {
  unsigned long long lo = m[0], hi = 0;
  if (NW > 1) lo |= (unsigned long long)m[NW > 1 ? 1 : 0] << 32;
  if (NW > 2) hi = m[NW > 2 ? 2 : 0] | (unsigned long long)m[NW > 3 ? 3 : 0] << 32;
#pragma unroll
  for (int i = FROM; i < FROM + C; ++i) {
    const bool low = NW <= 2 || lo != 0;
    const unsigned long long cur = low ? lo : hi;
    const int b = cur ? int(__builtin_ctzll(cur)) + (low ? 0 : 64) : 0;
    id[i] = b < N ? b : N - 1;
    const unsigned long long rest = cur & (cur - 1);
    lo = low ? rest : lo;
    hi = low ? hi : rest;
  }
}

// order-preserving key of a logit: a total order, so that places are a permutation also among values
// that are not numbers; -0.0 ranks equal to +0.0
__device__ __forceinline__ int lane_key(float v) {
  const int u = __float_as_int(v + 0.0f);
  return u ^ ((u >> 31) & 0x7fffffff);
}

// Rank order inside id[FROM .. FROM + C), ids ascending: place[i] is the expert's place among all.
template <int FROM, int C, int K>
__device__ __forceinline__ void lane_places(const int (&v)[K], int (&place)[K]) {
#pragma unroll
  for (int i = FROM; i < FROM + C; ++i) place[i] = i;
#pragma unroll
  for (int i = FROM; i < FROM + C; ++i)
#pragma unroll
    for (int j = i + 1; j < FROM + C; ++j) {
      const int later_first = v[j] > v[i] ? 1 : 0;  // equal: the lower id, i, stays in front
      place[i] += later_first;
      place[j] -= later_first;
    }
}

// The routing of a lane's token by the integer keys of the other kernels (make_key), straight from memory: its
// experts in rank order to ids with their keys, the position's union to U; returns how many experts it has.  `uni`
// is cleared.  Called by the whole wavefront.  Some k N dependent loads per token: only where a logit is
// not a number (a launch of NaNs alone is still served, slowly).
template <int NW>
__device__ __forceinline__ int lane_rank_by_key(const float* __restrict__ row, bool live, int N, int k, int k0,
                                                uint32_t* uni, uint32_t (&U)[NW], int* ids, uint32_t* keys) {
  unsigned long long taken[2] = {0, 0}, cand[2] = {~0ull, ~0ull};
  int n = 0;
  auto pick = [&]() __attribute__((always_inline)) {  // the best candidate that is not taken; false if there is none
    uint32_t top = 0;
    int id = 0;
    for (int e = 0; e < N; ++e) {
      const unsigned long long open = e < 64 ? cand[0] & ~taken[0] : cand[1] & ~taken[1];
      const uint32_t key = (open >> (e & 63)) & 1 ? make_key(row[e]) : 0;
      if (key > top) {
        top = key;
        id = e;
      }
    }
    if (top == 0) return false;
    taken[0] |= id < 64 ? 1ull << id : 0;
    taken[1] |= id < 64 ? 0 : 1ull << (id - 64);
    ids[n] = id;
    keys[n] = top;
    ++n;
    return true;
  };
  if (live) {
    while (n < k0 && pick()) {
    }
#pragma unroll
    for (int w = 0; w < NW; ++w) atomicOr(&uni[w], uint32_t(taken[w / 2] >> (32 * (w & 1))));
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NW; ++w) U[w] = uni[w];
  cand[0] = U[0] | (unsigned long long)U[1] << 32;
  cand[1] = NW > 2 ? U[NW > 2 ? 2 : 0] | (unsigned long long)U[NW > 3 ? 3 : 0] << 32 : 0;
  if (live) {
    while (n < k && pick()) {
    }
  }
  return n;
}

// NE: experts rounded up to 64 or 128.  K: most experts per token.  C1: list places of Phase 1.
// K == 8: C1 is k0 itself, and the list of Phase 2 has the other 8 - C1 places.  K == 16: k0 <= C1, and
// Phase 2 ranks the whole union.
// N a multiple of 4, logits 16-byte aligned; a workgroup (one wavefront) takes ppw = 64 / B
// consecutive positions.  Two wavefronts per SIMD for 128 experts: a third one costs spills (179 instead of 167 us).
template <int NE, int K, int C1>
__global__ __launch_bounds__(kLaneThreads) __attribute__((amdgpu_waves_per_eu(NE > 64 || K > 8 ? 2 : 4)))
void route_lanes_kernel(const float* __restrict__ logits, const uint8_t* __restrict__ token_mask, int L, int B, int N,
                        int k, int k0_, int ppw, RouteOut o) {
  constexpr int NW = NE / 32;
  constexpr bool EXACT = K == 8;
  constexpr int C2 = EXACT ? K - C1 : K;
  const int k0 = EXACT ? C1 : k0_;
  __shared__ __attribute__((aligned(16))) float s_stage[kLaneThreads * kLanePitch];
  __shared__ __attribute__((aligned(16))) uint32_t s_union[kLaneThreads][NW];
  const int lane = threadIdx.x;
  const int pos0 = blockIdx.x * ppw;
  const int npos = L - pos0 < ppw ? L - pos0 : ppw;
  const int nrows = npos * B;                // <= 64
  const size_t row0 = (size_t)pos0 * B;
  const int mine = lane < nrows ? lane : 0;  // lanes without a token repeat the first one and write nothing
  const int lpos = mine / B;
  const char* const base = reinterpret_cast<const char*>(logits + row0 * N);  // 64 rows of at most 512 bytes

  // ---- the logits: 8 lanes read 128 contiguous bytes of a row, all requests first
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  f32x4 in[NE / 4];
  const int sub = lane & 7;
  {
    uint32_t row_at[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = i * 8 + (lane >> 3);
      row_at[i] = uint32_t((r < nrows ? r : nrows - 1) * N) * 4u;
    }
#pragma unroll
    for (int c = 0; c < NE / kLaneChunk; ++c) {
      const int col = c * kLaneChunk + sub * 4;
      const uint32_t col_at = uint32_t(col < N ? col : N - 4) * 4u;
#pragma unroll
      for (int i = 0; i < 8; ++i) in[c * 8 + i] = *reinterpret_cast<const f32x4*>(base + (row_at[i] + col_at));
    }
  }
  const bool live = lane < nrows && !(token_mask && token_mask[row0 + mine] == 0);
#pragma unroll
  for (int w = 0; w < NW; ++w) s_union[lane][w] = 0;

  float v[NE];
#pragma unroll
  for (int c = 0; c < NE / kLaneChunk; ++c) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      *reinterpret_cast<f32x4*>(s_stage + (i * 8 + (lane >> 3)) * kLanePitch + sub * 4) = in[c * 8 + i];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kLaneChunk / 4; ++j) {
      const f32x4 q = *reinterpret_cast<const f32x4*>(s_stage + lane * kLanePitch + 4 * j);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[c * kLaneChunk + 4 * j + i] = q[i] + 0.0f;  // -0.0 ranks equal to +0.0
    }
    __syncthreads();
  }

  // experts that exist; the columns past them hold copies and are no candidates
  uint32_t exists[NW];
#pragma unroll
  for (int w = 0; w < NW; ++w) exists[w] = N >= 32 * w + 32 ? ~0u : (N > 32 * w ? (1u << (N - 32 * w)) - 1u : 0u);
  if (N < NE) {
#pragma unroll
    for (int e = 4; e < NE; ++e) v[e] = e < N ? v[e] : -INFINITY;
  }

  // ---- Phase 1: the k0 best of every token, united over the position
  float best[K];  // the chosen logits in rank order
  // A selected NaN shows in one of three ways: its sign bit clear, it counts as above the limit and makes the mask
  // too full; set, it is only reached by a limit of minus infinity, which makes the mask too full as well ...
  bool odd = false;
  uint32_t m1[NW], m2[NW];
  {
    float b1[C1];
    lane_best<C1, NE>(v, b1);
    const float limit = EXACT ? b1[C1 - 1] : list_at(b1, k0 - 1);
    lane_at_least<NE>(v, limit, m1);
#pragma unroll
    for (int w = 0; w < NW; ++w) m1[w] &= exists[w];
    if (__any(lane_count(m1) > k0)) {
      odd = live && lane_any_nan<NE>(v);
      lane_cut_ties<NE>(v, limit, k0, m1);
    }
    if (live) {
#pragma unroll
      for (int w = 0; w < NW; ++w) atomicOr(&s_union[lpos][w], m1[w]);
    }
    if (EXACT) {
#pragma unroll
      for (int j = 0; j < C1; ++j) best[j] = b1[j];
    }
  }
  __syncthreads();
  uint32_t U[NW];
  int T = 0, before[NW];  // members, and members in the words below
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    U[w] = s_union[lpos][w];
    before[w] = T;
    T += __popc(U[w]);
  }

  // ---- Phase 2: the best members of the union beyond the token's own k0, up to k in all
  int n = live ? (T < k ? T : k) : 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) m2[w] = EXACT ? U[w] & ~m1[w] : U[w];
  if constexpr (C2 > 0) {
    if (!EXACT || k > C1) {
      constexpr int kMinusInf = int(0xff800000u);
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        const int member = int(m2[e / 32] << (31 - e % 32)) >> 31;  // all ones or zero
        v[e] = __int_as_float((__float_as_int(v[e]) & member) | (kMinusInf & ~member));
      }
      float b2[C2];
      lane_best<C2, NE>(v, b2);
      const int taken = EXACT ? C1 : 0;
      const float limit = list_at(b2, k - taken - 1);
      uint32_t at[NW];
      lane_at_least<NE>(v, limit, at);
#pragma unroll
      for (int w = 0; w < NW; ++w) m2[w] &= at[w];
      if (__any(live && lane_count(m2) > n - taken)) {
        odd |= live && lane_any_nan<NE>(v);
        lane_cut_ties<NE>(v, limit, n - taken, m2);
      }
#pragma unroll
      for (int j = 0; j < C2; ++j) best[taken + j] = b2[j];
    } else {
#pragma unroll
      for (int j = 0; j < C2; ++j) best[(EXACT ? C1 : 0) + j] = -INFINITY;
    }
  }

  // ---- the chosen experts, each group ascending, with their logits (fetched again: registers have no
  // index), then in rank order through LDS (the places are a permutation of 0 .. K-1)
  constexpr int kPitch = K + 1;
  static_assert(2 * kPitch <= kLanePitch, "ids and keys fit the staging area");
  int* const s_ids = reinterpret_cast<int*>(s_stage) + lane * kPitch;
  {
    int id[K], place[K];
    float lv[K];
    int key[K];
    if constexpr (EXACT) lane_ids<0, C1>(m1, N, id);
    if constexpr (C2 > 0) lane_ids<EXACT ? C1 : 0, C2>(m2, N, id);
    const uint32_t row_at = uint32_t(mine * N) * 4u;
#pragma unroll
    for (int i = 0; i < K; ++i) lv[i] = *reinterpret_cast<const float*>(base + (row_at + uint32_t(id[i]) * 4u));
#pragma unroll
    for (int i = 0; i < K; ++i) odd |= i < n && lv[i] != lv[i];  // ... or there was no choice
#pragma unroll
    for (int i = 0; i < K; ++i) key[i] = i < n ? lane_key(lv[i]) : int(0x80000000u);  // unused places stay behind
    if constexpr (EXACT) lane_places<0, C1>(key, place);
    if constexpr (C2 > 0) lane_places<EXACT ? C1 : 0, C2>(key, place);
#pragma unroll
    for (int i = 0; i < K; ++i) s_ids[place[i]] = i < n ? id[i] : -1;
  }
  __syncthreads();
  if (__any(odd)) {  // rare
    uint32_t* const s_keys = reinterpret_cast<uint32_t*>(s_stage) + (kLaneThreads + lane) * kPitch;
#pragma unroll
    for (int w = 0; w < NW; ++w) s_union[lane][w] = 0;
    __syncthreads();
    n = lane_rank_by_key<NW>(logits + (row0 + mine) * N, live, N, k, k0, s_union[lpos], U, s_ids, s_keys);
    T = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      before[w] = T;
      T += __popc(U[w]);
    }
#pragma unroll
    for (int j = 0; j < K; ++j) {
      if (j >= n) s_ids[j] = -1;
      best[j] = j < n ? from_orderable(s_keys[j]) : -INFINITY;
    }
  }

  // ---- weights: softmax over the chosen logits (the sum in the order in which the row-per-token
  // kernels take it)
  float gate[K], part[K];
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const float w = j == 0 ? (best[0] - best[0]) + 1.f : expf(best[j] - best[0]);
    gate[j] = part[j] = j < n ? w : 0.f;
  }
#pragma unroll
  for (int s = 1; s < K; s *= 2)
#pragma unroll
    for (int j = 0; j < K; j += 2 * s) part[j] += part[j + s];
#pragma unroll
  for (int j = 0; j < K; ++j) gate[j] = j < n ? gate[j] / part[0] : 0.f;

  if (lane < nrows) {
    const size_t at = (row0 + lane) * k;
    int32_t* const ids = o.expert_idx + at;
    float* const gw = o.gate_w + at;
    if ((k & 3) == 0 && ((reinterpret_cast<uintptr_t>(o.expert_idx) | reinterpret_cast<uintptr_t>(o.gate_w)) & 15) == 0) {
#pragma unroll
      for (int j = 0; j < K; j += 4)
        if (j < k) {
          *reinterpret_cast<int4*>(ids + j) = make_int4(s_ids[j], s_ids[j + 1], s_ids[j + 2], s_ids[j + 3]);
          *reinterpret_cast<float4*>(gw + j) = make_float4(gate[j], gate[j + 1], gate[j + 2], gate[j + 3]);
        }
    } else {
#pragma unroll
      for (int j = 0; j < K; ++j)
        if (j < k) {
          ids[j] = s_ids[j];
          gw[j] = gate[j];
        }
    }
    o.n_sel[row0 + lane] = n;

    // ---- the union, ascending: the position's tokens take the experts in turn
    int32_t* const act = o.active_list + (size_t)(pos0 + lpos) * N;
    const int tok = lane - lpos * B;
    for (int e = tok; e < N; e += B) {
      const int w = e >> 5;
      uint32_t word = U[0];
      int rank = 0;
#pragma unroll
      for (int x = 1; x < NW; ++x) {
        word = x == w ? U[x] : word;
        rank = x == w ? before[x] : rank;
      }
      rank += __popc(word & ((1u << (e & 31)) - 1u));
      if ((word >> (e & 31)) & 1u) act[rank] = e;
      if (e >= T) act[e] = -1;
    }
    if (tok == 0) o.n_active[pos0 + lpos] = T;
  }
}

template <int NE>
hipError_t launch_route_lanes_one(const float* logits, const uint8_t* token_mask, int L, int B, int N, int k, int k0,
                                  RouteOut o, hipStream_t s) {
  const int ppw = kLaneThreads / B;
  const dim3 g((unsigned)((L + ppw - 1) / ppw)), b(kLaneThreads);
#define OEA_LANES(K, C1) \
  hipLaunchKernelGGL((route_lanes_kernel<NE, K, C1>), g, b, 0, s, logits, token_mask, L, B, N, k, k0, ppw, o)
  if (k > 8) {
    if (k0 <= 4)
      OEA_LANES(16, 4);
    else if (k0 <= 8)
      OEA_LANES(16, 8);
    else
      OEA_LANES(16, 16);
  } else {
    switch (k0) {
      case 1: OEA_LANES(8, 1); break;
      case 2: OEA_LANES(8, 2); break;
      case 3: OEA_LANES(8, 3); break;
      case 4: OEA_LANES(8, 4); break;
      case 5: OEA_LANES(8, 5); break;
      case 6: OEA_LANES(8, 6); break;
      case 7: OEA_LANES(8, 7); break;
      default: OEA_LANES(8, 8); break;
    }
  }
#undef OEA_LANES
  return hipGetLastError();
}

}  // namespace

// Many positions, a lane per token; hipErrorNotSupported where another kernel has to be, or is better, used.
//
// A wavefront works for 7 to 9 us on its up to 64 tokens (14 with lists of 16), a workgroup of the
// row-per-token kernel for less than 5 on one position; what the lanes save shows once the chip is
// full.  Measured (us, this kernel / route_kernel; N = 128, k = 8, k0 = 3):
//   B = 16: 1024 positions 8.9 / 7.6, 2048 10.3 / 11.7, 4096 13 / 20, 65535 164 / 277
//   B = 4:  4096 11.4 / 10.9, 8192 12.9 / 18.6;   B = 1: 8192 21.4 / 18.6, 16384 22.1 / 33.5
//   B = 64 (route_kernel with 1024 threads): 256 9.4 / 7.3, 512 9.8 / 13.6;   k = 12, B = 16: 2048 16.2 / 13.8, 4096 19.1 / 24.2
hipError_t try_launch_route_lanes(const float* logits, const uint8_t* token_mask, int L, int B, int N, int k, int k0,
                                  RouteOut o, hipStream_t s) {
  if (N > 128 || (N & 3) != 0 || k > 16 || B > kLaneThreads || o.grp_off) return hipErrorNotSupported;
  if ((reinterpret_cast<uintptr_t>(logits) & 15) != 0) return hipErrorNotSupported;
  int from = B > 16 ? 512 : 2048 + 8192 / B;
  if (k > 8) from += from / 2;
  if (L < from) return hipErrorNotSupported;
  return N <= 64 ? launch_route_lanes_one<64>(logits, token_mask, L, B, N, k, k0, o, s)
                 : launch_route_lanes_one<128>(logits, token_mask, L, B, N, k, k0, o, s);
}

}  // namespace oea

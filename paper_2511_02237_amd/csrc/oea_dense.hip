// Expert stages on the matrix cores, for batches in which an expert serves many tokens.
//
// The dot-product stages multiply every weight once per token of its expert on the vector ALUs:
// fine while an expert has a handful of tokens (the layer is then bound by the weight stream,
// Section 3.1, Eq. 2: the b T term), but with B*k/N of 16 and more the a B k term takes over and the
// vector ALUs, not HBM, set the latency.  Here a weight tile meets 16 tokens per instruction
// instead: v_mfma_f32_16x16x32_bf16 multiplies 16 weight rows x 32 columns with the same 32
// entries of 16 token vectors (bf16 products, fp32 accumulation).
//
// A workgroup takes an equal share of all active experts' rows, in granules of 16 rows of W_gate AND
// W_up (gate/up stage) or 32 rows of W_down (down stage), and works through it in jobs of up to eight
// granules of one expert against up to 128 of its tokens (an expert with more takes further passes over
// the same rows), walking the inner dimension in slabs of 64 columns.  Its twelve wavefronts have two roles:
//   * Four load: every operand goes from memory straight into LDS (global_load_lds, 16 bytes per lane, whole
//     128-byte row pieces per 8 lanes), two to five slabs ahead of their use, across jobs; the tokens and gate weights of
//     a job's pairs come with its last slab (down stage).  Loads are all that their memory counter counts, so waiting
//     for the oldest slab never waits for anything else.
//   * Eight multiply, a granule each, and load nothing.  Their results leave the registers directly at the end of a job:
//     silu(gate) * up rounded to the storage type into h, or gate-weighted atomic adds into out (Eq. 1).
// One workgroup barrier per slab orders the two: the slab has landed, the slab before it is used up.
//
// Bound by the weight stream: a loop of these requests alone reaches 7.0 TB/s with two slabs of 32 KB in flight per
// compute unit (128-byte pieces or whole rows, one barrier per slab or none; 6.2 without the non-temporal hint); the
// kernel without its results 6.3 to 6.5.  What is left are the results (kernel trace, with / without them: B=512, d=2048, I=768
// gate/up 148 / 139 us, down 81 / 67; B=1000, d=4096, I=1536 555 / 520 and 315 / 255), in the down stage the adds into `out`
// themselves: taking the multiplying wavefronts' own loads out, which had waited for them, gave 2 and 3 us.  In the form
// in which every wavefront loaded into registers, multiplied and wrote, the first slab of a job waited for the results of
// the one before (gate/up + down, us, that / this, in turn on one card: B=512, d=2048, I=768 139 + 83 / 136 + 83;
// B=1000, d=4096, I=1536 560 + 330 / 549 + 319; other cards and allocations have had 545 to 578 for that gate/up stage).
#include "oea_ffn_dev.h"

namespace oea {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef int32_t i32x4_t __attribute__((ext_vector_type(4)));

constexpr int kDenseGroups = 8;     // groups of 16 tokens per pass
constexpr int kDenseTokens = 16 * kDenseGroups;
constexpr int kDenseSlab = 64;      // columns per slab: two matrix-core steps of 32
constexpr int kMaxRing = 6;         // most slabs in LDS
constexpr int kMulWaves = 8;        // wavefronts that multiply; a job's most granules
constexpr int kLoadWaves = 4;       // wavefronts that load: two granules and 32 token rows each
constexpr int kDenseThreads = 64 * (kMulWaves + kLoadWaves);
constexpr int kRowBytes = kDenseSlab * 2;                  // of a slab in LDS
constexpr int kRows32 = 32 * kRowBytes;                    // a granule's rows (16 + 16 in the gate/up stage), or 32 token rows
constexpr int kRingBytes = 3 * (kMulWaves + kDenseTokens / 32) * kRows32;  // three of the largest slabs
constexpr int kPairBytes = kDenseTokens * 8;               // token and gate weight of a job's pairs, one copy per place of the ring
constexpr size_t kDenseLdsBytes = (size_t)kRingBytes + (size_t)kMaxRing * kPairBytes;

struct DenseParams {
  const uint16_t* wa;   // gate/up stage: W_gate; down stage: W_down   [N, rows, L]
  const uint16_t* wb;   // gate/up stage: W_up
  const uint16_t* vec;  // gate/up stage: x [B, L]; down stage: h [pairs, L] in grouped order
  uint16_t* h_out;      // gate/up stage: h [pairs, rows]
  float* out;           // down stage: out [B, rows] (or [pairs, rows], one row per pair)
  Grouping g;
  int rows, L, N, B, pairs_max;
  int deterministic;  // a row of `out` per pair (down stage), and every sum in one order (see the slabs' start)
  int divisors;  // bit c: an expert's granules are a multiple of c
};

// One job of a workgroup: granules of one expert against one pass of at most kDenseTokens pairs.
struct DenseJob {
  int u;      // first granule; granules are numbered expert-major over the active list
  int n;      // granules, 1..kMulWaves; 0: no further job
  int pass;
  int e;      // expert id
  int row0;   // first row of the job inside the expert
  int pair0;  // first pair of the pass (grouped order)
  int cnt;    // pairs in the pass, 1..kDenseTokens
};

// The routing's lists, read with scalar loads: in the loading wavefronts a vector load or an LDS read between the
// requests would wait for every request before it.
typedef const __attribute__((address_space(4))) int32_t* scalar_ints;
struct DenseLists {
  scalar_ints active, off, tok;
};

// The first job at or behind pass `pass` of granule u; u1: end of the workgroup's share.
template <int STAGE>
__device__ __forceinline__ DenseJob dense_job(const DenseLists& w, int u, int pass, int u1, int gpe, int N,
                                              int pairs_max) {
  constexpr int kRows = STAGE == 0 ? 16 : 32;
  DenseJob j{};
  while (u < u1) {
    const int a = u / gpe;
    int n = (a + 1) * gpe - u;
    n = n < u1 - u ? n : u1 - u;
    const int jobs = (n + kMulWaves - 1) / kMulWaves;
    n = (n + jobs - 1) / jobs;
    const int off = w.off[a], cnt = w.off[a + 1] - off;
    // experts without usable pairs never occur after a valid routing
    if (off >= 0 && cnt > 0 && off + cnt <= pairs_max && pass * kDenseTokens < cnt) {
      j.u = u;
      j.n = n;
      j.pass = pass;
      const int e = w.active[a];
      j.e = e < 0 ? 0 : (e >= N ? N - 1 : e);
      j.row0 = (u - a * gpe) * kRows;
      j.pair0 = off + pass * kDenseTokens;
      const int rem = cnt - pass * kDenseTokens;
      j.cnt = rem < kDenseTokens ? rem : kDenseTokens;
      return j;
    }
    u += n;
    pass = 0;
  }
  return j;
}
template <int STAGE>
__device__ __forceinline__ DenseJob dense_next(const DenseJob& j, const DenseLists& w, int u1, int gpe, int N, int pairs_max) {
  const bool again = (j.pass + 1) * kDenseTokens < w.off[j.u / gpe + 1] - w.off[j.u / gpe];
  return dense_job<STAGE>(w, again ? j.u : j.u + j.n, again ? j.pass + 1 : 0, u1, gpe, N, pairs_max);
}

// 16 bytes per lane from memory to LDS, lane l's at `lds` (wave-uniform) + 16 l; with WORD 4 bytes, at 4 l.
template <int AUX, bool WORD = false>
__device__ __forceinline__ void load_to_lds(const char* from, const char* lds) {
  const auto src = (const __attribute__((address_space(1))) void*)(from);
  const auto dst = (__attribute__((address_space(3))) void*)(__attribute__((address_space(3))) char*)(lds);
  if constexpr (WORD)
    __builtin_amdgcn_global_load_lds(src, dst, 4, 0, AUX);
  else
    __builtin_amdgcn_global_load_lds(src, dst, 16, 0, AUX);
}
constexpr int kAuxStream = 2;  // non-temporal: weights are read once

// Every wavefront passes the same barriers in the same order (the two roles in code of their own).
__device__ __forceinline__ void dense_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// ---- the loading wavefronts
// Wavefront l brings a slab's rows 64 l .. 64 l + 63 of the job's tiles (granules 2 l and 2 l + 1: eight requests, or
// none past the job's last granule) and token rows 32 l .. 32 l + 31 (four requests, or none).  In LDS a row's eight
// 16-byte pieces are swapped among themselves by its number (piece c lies at c ^ (row % 8)), which keeps the
// multiplying wavefronts' reads free of bank conflicts; the request does it by which piece a lane asks for.
// A workgroup's ring: room for the granules of its largest job and the token rows of its fullest pass, as many slabs
// as fit.
struct DenseRing {
  char* lds;
  int w32, t32;  // granules and blocks of 32 token rows per slab
  int slabs;
  __device__ __forceinline__ char* weights(int slot) const { return lds + slot * (w32 + t32) * kRows32; }
  __device__ __forceinline__ char* tokens(int slot) const { return weights(slot) + w32 * kRows32; }
  // down stage: the pairs of the job whose last slab is in this place, 32 tokens then 32 gate weights at a time
  __device__ __forceinline__ char* pairs(int slot) const { return lds + kRingBytes + slot * kPairBytes; }
  __device__ __forceinline__ int next(int slot) const { return slot + 1 == slabs ? 0 : slot + 1; }
};

// Waits until at most n of this wavefront's requests (a multiple of four) are outstanding.
__device__ __forceinline__ void wait_outstanding(int n) {
  switch (n >> 2) {
#define OEA_CASE(Q)                                              \
  case Q:                                                        \
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * Q) : "memory"); \
    break;
    OEA_CASE(1) OEA_CASE(2) OEA_CASE(3) OEA_CASE(4) OEA_CASE(5) OEA_CASE(6) OEA_CASE(7)
    OEA_CASE(8) OEA_CASE(9) OEA_CASE(10) OEA_CASE(11) OEA_CASE(12) OEA_CASE(13) OEA_CASE(14)
#undef OEA_CASE
    default:
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
}

template <int STAGE>
__device__ __forceinline__ void dense_load_wave(const DenseParams& p, const DenseLists& w, const DenseRing ring,
                                                DenseJob j, int u1, int gpe, int l, int lane) {
  constexpr int kRows = STAGE == 0 ? 16 : 32;
  const int slabs = p.L / kDenseSlab;
  const int lr = lane >> 3;                                  // row of a request's eight
  const uint32_t piece = uint32_t((lane & 7) ^ lr) * 16;     // byte inside its 128
  const uint32_t row_bytes = uint32_t(p.L) * 2;
  const uint32_t off_w = uint32_t(lr) * row_bytes + piece;
  const char *wa0 = nullptr, *wb0 = nullptr;  // first row of granule 2 l in W_gate and W_up, or in W_down
  uint32_t off_t[4];                          // this lane's pieces of its token rows
  bool first_half = false, second_half = false, some = false;  // granules 2 l and 2 l + 1 and any of the token rows are in the job
  auto open = [&]() __attribute__((always_inline)) {
    first_half = 2 * l < j.n;
    second_half = 2 * l + 1 < j.n;
    some = 32 * l < j.cnt;
    const size_t at = ((size_t)j.e * p.rows + (size_t)(j.row0 + 2 * l * kRows)) * row_bytes;
    wa0 = reinterpret_cast<const char*>(p.wa) + at;
    wb0 = reinterpret_cast<const char*>(p.wb) + at;
    if (!some) return;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      int mine = 0;
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const int n = 32 * l + 8 * i + r;
        const int pi = j.pair0 + (n < j.cnt ? n : j.cnt - 1);  // past the last token: the last again
        const int t = STAGE == 0 ? w.tok[pi] : pi;
        mine = lr == r ? t : mine;
      }
      const int lim = STAGE == 0 ? p.B : p.pairs_max;
      mine = mine < 0 ? 0 : (mine >= lim ? lim - 1 : mine);
      // below 2^32 by the entry points' limits on B, k, d and I
      off_t[i] = uint32_t(mine) * row_bytes + piece;
    }
  };
  // Requests of the next slab, into the next place of the ring.  Which slabs this wavefront had anything to request for
  // is kept as bits, the latest lowest: the number of requests behind a slab says whether it has landed.
  // The chip's eight XCDs walk the columns from eight different ones on: all workgroups at one column offset of rows that
  // lie a power of two apart crowd the same memory channels (gate/up, us, from column 0 / like this: d=4096, I=192, B=200
  // 88 / 67, B=1000 93 / 72; I=1536, B=160 543 / 510; d=2048, I=768, B=512 139 / 136, B=1000 161 / 153).  Not where the
  // token rows of the whole batch do not fit an XCD's L2 and an expert's many jobs read them: in step the XCDs find in the
  // memory-side cache what one of them has fetched (d=4096, I=1536: B=600 530 / 543, B=1000 549 / 578; at B=400, which
  // fits, still 498 / 506).  With fewer jobs the channels count for more (layers, d=4096, B=1000: I=1536 882 / 888, I=768 505 /
  // 491, I=384 341 / 310, I=192 244 / 233; d=8192, I=512, N=32, B=600 249 / 234; d=3072, I=1024, N=64 424 / 422).  And not in a
  // deterministic layer: which workgroup has a row depends on the batch, and a token's sums there add in one order
  // whatever the rest of the batch.
  const bool in_step = p.deterministic || (STAGE == 0 && (long long)p.B * p.L > (2 << 20) && p.rows > 1024);
  const int first_slab = in_step ? 0 : int(blockIdx.x % 8) * slabs / 8;
  int slab = first_slab, slot = 0, asked = 0;
  uint32_t had_first = 0, had_second = 0, had_some = 0;
  auto more = [&]() __attribute__((always_inline)) {
    if (j.n == 0) return;
    const int next_slab = slab + 1 == slabs ? 0 : slab + 1;
    if (STAGE == 1 && some && next_slab == first_slab) {
      // With the job's last slab come the tokens and gate weights of its pairs: that slab's barrier hands them over, and
      // their place is requested again only behind the next barrier, which the multiplying wavefronts reach with
      // their results written.  (Not counted below: a wait for a slab before this one then waits for one request too
      // many.)
      const int n = 32 * l + (lane & 31);
      const int pi = j.pair0 + (n < j.cnt ? n : j.cnt - 1);
      const char* const list = lane < 32 ? reinterpret_cast<const char*>(p.g.grp_tok) : reinterpret_cast<const char*>(p.g.grp_gw);
      load_to_lds<0, true>(list + (size_t)pi * 4, ring.pairs(slot) + l * 256);
    }
    const uint32_t col = uint32_t(slab) * kRowBytes;
    char* const to = ring.weights(slot) + l * 2 * kRows32;
#pragma unroll
    for (int half = 0; half < 2; ++half)
      if (half ? second_half : first_half) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const char* from = STAGE == 0 ? ((i & 2) ? wb0 : wa0) + (size_t)(half * 16 + (i & 1) * 8) * row_bytes
                                        : wa0 + (size_t)(half * 32 + i * 8) * row_bytes;
          load_to_lds<kAuxStream>(from + (off_w + col), to + (half * 4 + i) * 8 * kRowBytes);
        }
      }
    if (some) {
      char* const to_t = ring.tokens(slot) + l * kRows32;
      const char* const from = reinterpret_cast<const char*>(p.vec) + col;
#pragma unroll
      for (int i = 0; i < 4; ++i) load_to_lds<0>(from + off_t[i], to_t + i * 8 * kRowBytes);
    }
    had_first = had_first * 2 + (first_half ? 1 : 0);
    had_second = had_second * 2 + (second_half ? 1 : 0);
    had_some = had_some * 2 + (some ? 1 : 0);
    slot = ring.next(slot);
    ++asked;
    slab = next_slab;
    if (slab == first_slab) {
      j = dense_next<STAGE>(j, w, u1, gpe, p.N, p.pairs_max);
      open();
    }
  };
  open();
  // All but one of the ring's places are requested ahead; barrier g hands slab g over and frees slab g - 1's place.
  for (int i = 0; i + 1 < ring.slabs; ++i) more();
  for (int g = 0; g < asked; ++g) {
    // slab g has landed once nothing but the requests behind it is outstanding
    const uint32_t behind = (1u << (asked - g - 1)) - 1u;
    wait_outstanding(4 * (__popc(had_first & behind) + __popc(had_second & behind) + __popc(had_some & behind)));
    dense_barrier();
    more();
  }
}

// ---- the multiplying wavefronts: wavefront v takes granule v of every job
template <int STAGE>
__device__ __forceinline__ void dense_store(const DenseParams& p, const char* pairs, const DenseJob& j,
                                            const f32x4_t (&acc)[kDenseGroups][2], int v, int lane) {
  constexpr int kRows = STAGE == 0 ? 16 : 32;
  const int r = lane & 15, q = lane >> 4;
  const int rows = p.rows;
  if (STAGE == 0) {
    // the lane holds rows 4 q .. 4 q + 3 of the gate and the up tile for token r of each group
    const int row = j.row0 + v * kRows + 4 * q;
#pragma unroll
    for (int c = 0; c < kDenseGroups; ++c) {
      const int n = c * 16 + r;
      if (n < j.cnt) {
        uint16_t hv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float gsum = acc[c][0][i], usum = acc[c][1][i];
          hv[i] = f32_to_bf16_rne(gsum / (1.f + __expf(-gsum)) * usum);
        }
        uint2 packed;
        packed.x = uint32_t(hv[0]) | (uint32_t(hv[1]) << 16);
        packed.y = uint32_t(hv[2]) | (uint32_t(hv[3]) << 16);
        *reinterpret_cast<uint2*>(p.h_out + (size_t)(j.pair0 + n) * rows + row) = packed;
      }
    }
  } else {
    // the lane holds output coordinate r of both tiles for tokens 4 q .. 4 q + 3 of each group: an
    // atomic instruction adds 64 consecutive bytes to each of four rows of out
    const int row = j.row0 + v * kRows + r;
    int first = 4 * q;
    asm volatile("" : "+v"(first));  // worked out here, not ahead of all jobs: the registers are the accumulators'
    const int left = j.cnt - first;
    const char* const mine = pairs + first * 4;
#pragma unroll
    for (int c = 0; c < kDenseGroups; ++c) {
      // the four tokens' entries at once (those past the last pair are bytes of the place, unused)
      const char* const entry = mine + (c >> 1) * 256 + (c & 1) * 64;
      const i32x4_t tok = *reinterpret_cast<const i32x4_t*>(entry);
      const f32x4_t gws = *reinterpret_cast<const f32x4_t*>(entry + 128);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (c * 16 + i < left) {
          const int t = tok[i] < 0 ? 0 : (tok[i] >= p.B ? p.B - 1 : tok[i]);
          const int orow = p.deterministic ? j.pair0 + first + c * 16 + i : t;
          const float gw = gws[i];
          float* const o = p.out + (size_t)orow * rows + row;
          unsafeAtomicAdd(o, gw * acc[c][0][i]);
          unsafeAtomicAdd(o + 16, gw * acc[c][1][i]);
        }
      }
    }
  }
}

template <int STAGE>
__device__ __forceinline__ void dense_multiply_wave(const DenseParams& p, const DenseLists& w, const DenseRing ring,
                                                    DenseJob j, int u1, int gpe, int v, int lane) {
  const int r = lane & 15, q = lane >> 4;
  const int slabs = p.L / kDenseSlab;
  // a lane's piece of a row: columns 8 q .. 8 q + 7 of each of the slab's two steps (see the loading wavefronts)
  const int at0 = r * kRowBytes + ((q ^ (r & 7)) * 16), at1 = r * kRowBytes + (((4 + q) ^ (r & 7)) * 16);
  int slot = 0;
  while (j.n != 0) {
    const bool mine = v < j.n;
    const int ng = (j.cnt + 15) >> 4;
    f32x4_t acc[kDenseGroups][2];
#pragma unroll
    for (int c = 0; c < kDenseGroups; ++c) acc[c][0] = acc[c][1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const char* pairs = nullptr;
    DenseJob nxt{};
    for (int s = 0; s < slabs; ++s) {
      dense_barrier();
      if (s == slabs / 2) nxt = dense_next<STAGE>(j, w, u1, gpe, p.N, p.pairs_max);  // trips to memory, between results no more
      const char* const wv = ring.weights(slot) + (mine ? v : 0) * kRows32;
      const char* const tv = ring.tokens(slot);
      bf16x8_t a[2][2];
#pragma unroll
      for (int i2 = 0; i2 < 2; ++i2)
#pragma unroll
        for (int tile = 0; tile < 2; ++tile)
          a[i2][tile] = __builtin_bit_cast(
              bf16x8_t, *reinterpret_cast<const u32x4_t*>(wv + tile * 16 * kRowBytes + (i2 ? at1 : at0)));
      if (mine) {
#pragma unroll
        for (int c = 0; c < kDenseGroups; ++c) {
          if (c >= ng) break;
#pragma unroll
          for (int i2 = 0; i2 < 2; ++i2) {
            const bf16x8_t b = __builtin_bit_cast(
                bf16x8_t, *reinterpret_cast<const u32x4_t*>(tv + 16 * c * kRowBytes + (i2 ? at1 : at0)));
            if (STAGE == 0) {  // result tile [weight row][token]: a lane holds four rows of one token
              acc[c][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i2][0], b, acc[c][0], 0, 0, 0);
              acc[c][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i2][1], b, acc[c][1], 0, 0, 0);
            } else {  // [token][weight row]: 16 lanes hold 16 consecutive output coordinates of one token
              acc[c][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, a[i2][0], acc[c][0], 0, 0, 0);
              acc[c][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, a[i2][1], acc[c][1], 0, 0, 0);
            }
          }
        }
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the slab's token rows have been read
      pairs = ring.pairs(slot);
      slot = ring.next(slot);
    }
    if (mine) dense_store<STAGE>(p, pairs, j, acc, v, lane);
    j = nxt;
  }
}

template <int STAGE>
__global__ __launch_bounds__(kDenseThreads) void expert_dense_kernel(DenseParams p) {
  extern __shared__ uint4 lds4[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  const DenseLists w{(scalar_ints)p.g.active_list, (scalar_ints)p.g.grp_off, (scalar_ints)p.g.grp_tok};
  int T = *(scalar_ints)p.g.n_active;
  T = T < 0 ? 0 : (T > p.N ? p.N : T);
  constexpr int kRows = STAGE == 0 ? 16 : 32;
  const int gpe = p.rows / kRows;
  const long long U = (long long)T * gpe;
  // Consecutive shares go to workgroups of the same XCD (workgroups are dealt out to the eight in turn), so
  // the units of an expert find its token rows in one L2 instead of fetching them into all eight
  // (B=1000, d=4096, I=1536: gate/up 567 -> 558 us, down 336 -> 328 us; layers up to 2.4 GB of active weights 0 to 2 %).
  // Not with more than 3 GB of them and few tokens per expert, where the stream of weights suffers (layer, XCD order /
  // in turn, us: d=4096, N=128, I=1024 564 / 534 at B=200 and 577 / 557 at B=400, I=1536 813 / 803 at B=200, 818 / 817 at
  // B=400, 856 / 859 at B=640, 893 / 898 at B=800).
  const int G = int(gridDim.x), per_xcd = G / 8;
  const bool by_xcd = G % 8 == 0 && ((long long)T * p.rows * p.L <= 500000000ll || w.off[T] >= 40 * T);
  const int share = by_xcd ? int(blockIdx.x % 8) * per_xcd + int(blockIdx.x / 8) : int(blockIdx.x);
  // Equal shares of whole jobs of m granules, or (m = 1) shares that end anywhere, which makes a job more of most: a
  // job's slab costs its granules and about three granules' time of its own.  Gate/up and down, us, any / whole: d=2048,
  // I=768, B=200 142 + 76 / 132 + 72; d=4096, I=1536, B=160 down 272 / 265.
  int m = 1;
  {
    const float shares = float(G), most = ceilf(float(U) / shares);
    float best = most <= 1.f ? 4.f : most + 3.f * (ceilf(most / kMulWaves) + 1.f);
#pragma unroll
    for (int c = kMulWaves; c >= 2; --c) {
      const float cost = ceilf(float(U) * (1.f / c) / shares) * (c + 3.f);
      if ((p.divisors >> c & 1) && cost < best) {
        best = cost;
        m = c;
      }
    }
  }
  const int u0 = int(U / m * share / G) * m, u1 = int(U / m * (share + 1) / G) * m;
  const DenseJob first = dense_job<STAGE>(w, u0, 0, u1, gpe, p.N, p.pairs_max);
  if (first.n == 0) return;  // uniform over the workgroup
  DenseRing ring{reinterpret_cast<char*>(lds4), gpe < u1 - u0 ? gpe : u1 - u0, 1, 0};
  ring.w32 = ring.w32 < kMulWaves ? ring.w32 : kMulWaves;
  for (int a = u0 / gpe; a <= (u1 - 1) / gpe; ++a) {
    const int t32 = (w.off[a + 1] - w.off[a] + 31) / 32;
    ring.t32 = t32 > ring.t32 ? t32 : ring.t32;
  }
  ring.t32 = ring.t32 < kDenseTokens / 32 ? ring.t32 : kDenseTokens / 32;
  ring.slabs = kRingBytes / ((ring.w32 + ring.t32) * kRows32);
  ring.slabs = ring.slabs < kMaxRing ? ring.slabs : kMaxRing;
  if (wave < kMulWaves)
    dense_multiply_wave<STAGE>(p, w, ring, first, u1, gpe, wave, lane);
  else
    dense_load_wave<STAGE>(p, w, ring, first, u1, gpe, wave - kMulWaves, lane);
}

}  // namespace

// One expert stage (0 gate/up, 1 down) on the matrix cores; hipErrorNotSupported for storage types
// and shapes it is not built for (bf16; rows a multiple of a granule, inner dimension of a slab).
hipError_t try_launch_dense_stage(int stage, const void* vec, const void* wa, const void* wb, void* h_out, float* out,
                                  int B, int d, int N, int I, int k, oea_dtype dt, Grouping g, bool deterministic,
                                  hipStream_t s) {
  static_assert(kDenseSlab == 64, "dense_stage_fits");
  if (!dense_stage_fits(stage, d, N, I, dt)) return hipErrorNotSupported;
  const int rows = stage == 0 ? I : d, L = stage == 0 ? d : I;
  int dev = 0, grid = 0;
  if (!current_device(&dev, &grid)) return hipErrorUnknown;
  if (grid < 1) return hipErrorNotSupported;
  DenseParams p{};
  p.wa = static_cast<const uint16_t*>(wa);
  p.wb = static_cast<const uint16_t*>(wb);
  p.vec = static_cast<const uint16_t*>(vec);
  p.h_out = static_cast<uint16_t*>(h_out);
  p.out = out;
  p.g = g;
  p.rows = rows;
  p.L = L;
  p.N = N;
  p.B = B;
  p.pairs_max = B * k;
  p.deterministic = deterministic ? 1 : 0;
  for (int c = 2; c <= kMulWaves; ++c)
    if (rows / (stage == 0 ? 16 : 32) % c == 0) p.divisors |= 1 << c;
  static PerDevice attr0, attr1;
  const void* kern = stage == 0 ? reinterpret_cast<const void*>(expert_dense_kernel<0>)
                                : reinterpret_cast<const void*>(expert_dense_kernel<1>);
  hipError_t e = ensure_dynamic_lds(kern, (int)kDenseLdsBytes, stage == 0 ? attr0 : attr1);
  if (e != hipSuccess) return e;
  if (stage == 0)
    hipLaunchKernelGGL(expert_dense_kernel<0>, dim3(grid), dim3(kDenseThreads), kDenseLdsBytes, s, p);
  else
    hipLaunchKernelGGL(expert_dense_kernel<1>, dim3(grid), dim3(kDenseThreads), kDenseLdsBytes, s, p);
  return hipGetLastError();
}

}  // namespace oea

// Sparse decode attention over gathered records for gfx950 (the consumer of the resolve
// step's slot vector, Section 3.4 Phase 5; exactness per Section 3.1).
//
// For each unit and query head h:  out_h = sum_j softmax_j(scale * q_h . key_j) value_j,
// over the tokens of the k selected records, in the order of the slot vector.
//
// Structure (every attention kernel: one workgroup per (unit, token split, head block); each
// 32-token chunk is staged into LDS once with direct global->LDS loads and shared by the
// workgroup's head waves)
//   attn_partial_kernel  grouped-query records (d 128), and latent calls of up to 16 heads over at
//     most 128 tokens. Bound by HBM for large calls (64 units x 4 heads x 4096 tokens, 134 MB:
//     36.3 us with one partial result per wave, 29.7 now, merge included; the copy rate gives 26)
//     and by latency for small ones. A wave owns 16 query heads (the MFMA N dimension) and one
//     32-token chunk per iteration.
//       S^T[token][head] = K[token][:] . Q^T[:][head]     v_mfma_f32_16x16x32_bf16, K from LDS
//                                                        rows, Q resident in VGPRs
//       online softmax in fp32 (exp2, reference max per head), P rounded to bf16
//       O[head][dim]   += P[head][token] . V[token][dim]  v_mfma_f32_16x16x32_bf16, V by LDS
//                                                        transpose reads
//     A lane's S^T accumulator holds tokens {4g..4g+3, 16+4g..16+4g+3} (g = lane/16) of its
//     head, which is exactly one P operand when the PV contraction index runs over the tokens
//     in that order, so P never leaves the lane; the V operand is read in the same order.
//   attn_mla_kernel  latent records (d_qk 576, d_v 512 = the key's first 512 dims): 32 heads
//     per wave on v_mfma_f32_32x32x16_bf16, the output in accumulation registers.
//   A workgroup's token groups (waves on different chunks of its split) are merged through LDS, so
//     a split is one partial result; a unit that is one split is written out by the kernel.
//   attn_combine_kernel / attn_combine_mla_kernel  merge the per-split (max, sum, unnormalised
//     output) triples of each (unit, head) in ascending split order.
//   Either attention kernel can carry an exact-prefetch replay: extra workgroups after the
//   attention's copy records into other layers' caches and exit (replay_worker).
// The reduction order depends only on token positions in the sequence, never on the slot
// values, so any placement of the same records gives bit-identical outputs.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "fetch_device.h"

namespace hisparse {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kChunk = 32;            // tokens per wave per iteration
constexpr int kTargetWorkgroups = 256;
// A carried replay keeps to the CUs the attention leaves if there are this many at least. On fewer, a
// workgroup or two per unit would copy everything: 16 units of 16 heads x 1024 tokens that left
// none took 462 us for a share group of four layers, 222 with the replay's full grid behind the
// attention's (in the order of block indices it starts as CUs come free).
constexpr int kMinIdle = 64;
constexpr int kMaxSplitRecords = 2048;  // record indices of one split staged in LDS
// Rescale the running output only when a head's running max grows by more than this (log2
// units): exponentials are taken against a slightly stale max (values up to 2^8), which is
// exact softmax arithmetic with a different reference point and keeps fp32/bf16 far from
// overflow; the final normalisation uses the same reference.
constexpr float kRescaleSlack = 8.0f;

// 16-byte loads of padding tokens and padding slots read zeros from here.
__device__ __attribute__((aligned(16))) uint8_t g_zero_token[2048];

// A replay carried by a launch (attention or merge): the extra workgroups after the launch's
// own, per_pair of them for each (unit, target layer) of the plan.
struct CarriedReplay {
  FetchArgs pf;
  FastDiv pf_div;
  int32_t pf_per_pair, pf_wg, pf_u;  // pf_u: 16-byte loads each replay thread keeps in flight
};

struct AttnArgs {
  const uint8_t* pool;
  const uint16_t* q;
  const int32_t* idx;
  float* part_o;    // [units][n_parts][H][DV]
  float2* part_ml;  // [units][n_parts][H] (running max in log2 units, running sum)
  float* out;       // [units][H][DV]: the output, for the kernels that write it themselves
  int32_t direct;   // grouped-query kernels: write the output, not partials (one split per unit)
  int64_t rec_per_unit;
  int32_t R, token_bytes, tpr_shift, k, H, n_tok;
  int32_t split_tokens, n_wg_splits, hb, n_parts, n_wg;
  int32_t Hp;         // latent attention: heads rounded up to 32 (partial-output block layout)
  int32_t idx_units;  // unit u reads index row u % idx_units
  FastDiv div_hb, div_splits, div_idx;  // by hb, n_wg_splits, idx_units
  float scale_log2;
  // A prefetch replay carried by the launch: extra workgroups after the attention workgroups
  // copy that plan's records (pf_wg = 0: none).
  CarriedReplay rp;
};

// The arguments an attention workgroup needs before its first memory access, loaded together at
// the start: left to themselves the scalar loads go out one use at a time, each a round trip.
__device__ __forceinline__ void load_args(const AttnArgs& a) {
  asm volatile("" ::"s"(a.pool), "s"(a.q), "s"(a.idx), "s"(a.rec_per_unit), "s"(a.R),
               "s"(a.token_bytes), "s"(a.tpr_shift), "s"(a.k), "s"(a.H), "s"(a.n_tok));
  asm volatile("" ::"s"(a.split_tokens), "s"(a.n_wg_splits), "s"(a.hb), "s"(a.n_wg),
               "s"(a.idx_units), "s"(a.div_hb.magic), "s"(a.div_hb.shift),
               "s"(a.div_splits.magic), "s"(a.div_splits.shift), "s"(a.div_idx.magic),
               "s"(a.div_idx.shift), "s"(a.scale_log2));
}

// Extra workgroup e of a launch: its share of the carried replay. It shares no memory with the
// launch's own workgroups (other layers' caches), so it needs no synchronisation.
__device__ __forceinline__ void replay_worker(const CarriedReplay& r, int e) {
  const int pair = e / r.pf_per_pair, x = e - pair * r.pf_per_pair;
  const int unit = pair % r.pf.units, z = pair / r.pf.units;
  const uint32_t first = x * blockDim.x + threadIdx.x, stride = r.pf_per_pair * blockDim.x;
  if (r.pf_u >= 4) fetch_slice<4>(r.pf, r.pf_div, unit, z, first, stride);
  else if (r.pf_u == 2) fetch_slice<2>(r.pf, r.pf_div, unit, z, first, stride);
  else fetch_slice<1>(r.pf, r.pf_div, unit, z, first, stride);
}

// Latent-attention partial outputs are stored in the PV accumulators' own layout, so every
// lane writes 16 contiguous bytes: per part, 32-head block b, output tile n (dims 32n..32n+31),
// group q and lane L hold heads 32b + 8q + 4(L >> 5) + e, e = 0..3, of dim 32n + (L & 31).
__device__ __host__ inline int64_t mla_part_offset(int head, int dim) {
  const int hl = head & 31, q = hl >> 3, e = hl & 3, ln = ((hl >> 2) & 1) * 32 + (dim & 31);
  return (int64_t)(head >> 5) * 32 * 512 + ((((dim >> 5) * 4 + q) * 64 + ln) * 4 + e);
}

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// Two softmax weights 2^e0, 2^e1 rounded to bf16 (nearest even, one packed v_cvt_pk_bf16_f32), the
// first in the low half. The exponential is the hardware v_exp_f32: weights below 2^-126 flush to
// zero.
__device__ inline uint32_t weights_bf16x2(float e0, float e1) {
  const f32x2 e = {__builtin_amdgcn_exp2f(e0), __builtin_amdgcn_exp2f(e1)};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(e, bf16x2_t));
}
// s * scale - m with the product rounded first, as the products that references are taken from are:
// 0 for the score that m is.
__device__ inline float over_reference(float s, float scale, float m) {
#pragma clang fp contract(off)
  return s * scale - m;
}
// Up to this reference (powers of two) a weight comes from one fused multiply-add: against the
// rounded product m, the score that m is then weighs 2^0.5 at most, and so do its peers, which the
// softmax does not see. Beyond 2^31 such a weight would leave the float range; there the product is
// rounded first (for every score: 96 units of 128 heads x 2048 tokens 88.2 us, this way 87.5).
constexpr float kFusedReference = 16777216.f;
// The weights of N scores of one head against its reference m, two to a word.
template <int N>
__device__ __forceinline__ void softmax_weights(uint32_t (&pw)[N / 2], const float (&sc)[N],
                                                float scale, float m) {
#pragma unroll
  for (int j = 0; j < N; j += 2)
    pw[j >> 1] = weights_bf16x2(__builtin_fmaf(sc[j], scale, -m),
                                __builtin_fmaf(sc[j + 1], scale, -m));
  // some head of the wave has a larger reference, or none yet and weighs nothing
  if (__ballot(!(__builtin_fabsf(m) <= kFusedReference))) {
#pragma unroll
    for (int j = 0; j < N; j += 2) {
      const uint32_t rounded = weights_bf16x2(over_reference(sc[j], scale, m),
                                              over_reference(sc[j + 1], scale, m));
      pw[j >> 1] = m == -INFINITY ? 0u
                   : __builtin_fabsf(m) <= kFusedReference ? pw[j >> 1] : rounded;
    }
  }
}
// sum + both (rounded) weights of w.
__device__ inline float add_weights(uint32_t w, float sum) {
  const bf16x2_t ones = {(__bf16)1.0f, (__bf16)1.0f};
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w), ones, sum, false);
}
__device__ inline float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }


typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16 lds_v4i16;
typedef __attribute__((address_space(3))) void lds_void;

// LDS reads that the compiler does not see as memory accesses. In the latent-attention loop the
// next chunk's direct-to-LDS loads are in flight while the current chunk is read from another
// buffer; before a compiler-visible LDS read the compiler would wait for those loads (it cannot
// tell the buffers apart), which takes the load of chunk it+1 out from under the compute of
// chunk it. The caller waits for these reads itself, with s_waitcnt lgkmcnt(N), N = the number
// of its own reads issued after the one it needs: LDS reads complete in order, so any other
// LGKM operation in flight can only lengthen that wait.
__device__ inline uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(const lds_void*)p;
}
template <int OFF>
__device__ __forceinline__ u32x4 lds_read_b128(uint32_t addr) {
  static_assert(OFF >= 0 && OFF < 65536, "immediate offset");
  u32x4 v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
  return v;
}
template <int OFF>
__device__ __forceinline__ v4i16 lds_read_tr16_b64(uint32_t addr) {
  static_assert(OFF >= 0 && OFF < 65536, "immediate offset");
  v4i16 v;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
  return v;
}
// f(0), f(1), ..., f(N - 1) with the index as a compile-time constant (immediate offsets).
template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}
// Wait until at most N LGKM operations are outstanding; a and b are the registers of the reads
// waited for (tied, so that their users stay after the wait).
template <int N>
__device__ __forceinline__ void lgkm_wait2(v4i16& a, v4i16& b) {
  asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(a), "+v"(b) : "n"(N));
}
template <int N>
__device__ __forceinline__ void lgkm_wait2(u32x4& a, u32x4& b) {
  asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(a), "+v"(b) : "n"(N));
}
// S^T += K . Q^T for one k-step once the K rows' read (with at most N later LDS reads) is in;
// the first step of a chain (FIRST) starts from zero. The s_nop covers the wait states after a
// just-written operand that the compiler does not see through the assembly.
template <int N, bool FIRST>
__device__ __forceinline__ void mfma_qk(f32x16& acc, const u32x4& k, const bf16x8_t& q) {
  if constexpr (FIRST)
    asm volatile("s_waitcnt lgkmcnt(%3)\n\ts_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, 0"
                 : "=&v"(acc) : "v"(k), "v"(q), "n"(N));
  else
    asm volatile("s_waitcnt lgkmcnt(%3)\n\ts_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0"
                 : "+v"(acc) : "v"(k), "v"(q), "n"(N));
}

// Wait until at most N direct-to-LDS loads of this wave are outstanding and its LDS writes are
// done, then synchronise the workgroup. (A workgroup fence would also drain the younger
// prefetches, which is exactly what the pipeline must not do.)
template <int N>
__device__ inline void wait_loads_and_barrier() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// Every LDS write of this wave (and any LDS read) done, then the workgroup synchronised; loads
// stay in flight.
__device__ inline void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// LDS tile of 32 rows (a chunk's tokens, or 32 query rows) of P 16-byte pieces, P a multiple of
// 8: blocks of 8 rows x 8 pieces (128 bytes of each row), 1 KB each, block (row group, segment)
// at (rg * NSEG + seg) * 1024. One 64-lane direct global->LDS load fills one block, 8 lanes per
// row: each group of 8 lanes reads one 128-byte run of its row, and a lane needs one global
// address per row group, the segment being an immediate offset (an earlier layout of padded rows
// spent 18 vector instructions per load on finding each lane's row, and its loads straddled
// rows: 64 units of 16 heads took 81 us that way, 39 this way). Inside a block, piece p
// of row r sits in 16-byte slot p ^ tile_swizzle(r): any 16 consecutive rows then place the same
// piece in 16 different slots of the 256 bytes that all 64 banks serve (row parity picks the
// half). A transpose read's 16-lane group has rows of one parity, 4 apart, in the 128 bytes of one
// half; the latent kernel's two groups of 32 lanes share it and take each read's banks twice.
// Counted (SQ_LDS_BANK_CONFLICT per wave and chunk): latent 128 of 555 LDS cycles, two for each
// transpose read (padded rows: none of 401); grouped-query 32 of 156 (padded rows: 64 of 151).
template <int P>
struct Tile {
  static_assert(P % 8 == 0, "whole 128-byte segments");
  static constexpr int NSEG = P / 8;
  static constexpr int BYTES = kChunk * P * 16;
  __device__ static int row(int r) { return (r >> 3) * (NSEG * 1024) + (r & 7) * 128; }
};
__device__ inline int tile_swizzle(int r) { return (r >> 1) & 7; }

// Row order of a 16-token group inside the MFMA tiles: operand row m reads token
// tile_row(m) = 4 (m & 3) + (m >> 2). A lane's S^T accumulator then holds tokens tile_row(4g + j)
// (+16), and the four rows of a PV transpose read are 4 apart, which the swizzle spreads over
// four different 32-byte slot pairs.
__device__ inline int tile_row(int m) { return 4 * (m & 3) + (m >> 2); }

// Direct global->LDS load of one block, segment SEG of row group rg: `src` is this lane's row (row
// 8 rg + lane / 8) already advanced by the lane's 16-byte piece. The load's immediate offset
// moves both addresses.
template <int P, int SEG>
__device__ __forceinline__ void stage_block(uint8_t* tile, int rg, const uint8_t* src) {
  __builtin_amdgcn_global_load_lds(
      src, (lds_void*)(tile + (rg * Tile<P>::NSEG + SEG) * 1024 - SEG * 128), 16, SEG * 128, 0);
}
template <int P>
__device__ __forceinline__ void stage_rows(uint8_t* tile, int rg, const uint8_t* src) {
  static_for<Tile<P>::NSEG>([&](auto seg) { stage_block<P, seg>(tile, rg, src); });
}
// The same by way of registers, for rows at any address: a direct-to-LDS load has to be aligned.
template <int P>
__device__ __forceinline__ void copy_rows(uint8_t* tile, int rg, const uint8_t* src) {
  typedef u32x4 any_u32x4 __attribute__((aligned(2)));
  u32x4* dst = reinterpret_cast<u32x4*>(tile + rg * Tile<P>::NSEG * 1024) + (threadIdx.x & 63);
#pragma unroll
  for (int seg = 0; seg < Tile<P>::NSEG; ++seg)
    dst[seg * 64] = *reinterpret_cast<const any_u32x4*>(src + seg * 128);
}
// The 16-byte piece (times 16) that a lane fetches for its row of row group rg.
__device__ inline int stage_piece(int lane, int rg) {
  return ((lane & 7) ^ tile_swizzle(8 * rg + (lane >> 3))) << 4;
}

// The records of a split: where its tokens' indices are and how a token finds its bytes.
struct SplitRows {
  const int32_t* idx;     // the split's record indices in memory
  const uint8_t* pool;    // the unit's part of the pool
  int tok_end, rec_begin, tpr_shift, R, token_bytes;
  int64_t rec_per_unit;
  __device__ int32_t checked(int32_t r) const { return (r >= 0 && r < rec_per_unit) ? r : -1; }
  // index entry of token tk (entry 0 for a token past the split end)
  __device__ int entry(int tk) const { return tk < tok_end ? (tk >> tpr_shift) - rec_begin : 0; }
  // Token tk of record s. Padding slots (s < 0) and tokens past the split end read zeros: their
  // scores are masked to -inf, so they carry P = 0.
  __device__ const uint8_t* row(int tk, int32_t s) const {
    const uint32_t off = (uint32_t)(s * R + (tk & ((1 << tpr_shift) - 1)) * token_bytes);
    return (tk < tok_end && s >= 0) ? pool + off : g_zero_token;
  }
};

// Where each lane reads its row of row groups rg0 .. rg0 + N - 1 of the 32-token chunk starting at
// token cbase, by the checked indices in LDS.
template <int N>
__device__ __forceinline__ void chunk_rows(const uint8_t* (&src)[N], const int32_t* s_idx,
                                           const SplitRows& r, int cbase, int rg0) {
  // recompute the per-lane arithmetic here instead of keeping it live across the loop
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int tk = cbase + 8 * (rg0 + i) + (lane >> 3);
    src[i] = r.row(tk, s_idx[r.entry(tk)]) + stage_piece(lane, rg0 + i);
  }
}
// The same for a workgroup's first chunk, in two halves: its index entries straight from memory
// (the first loads of the kernel), and the rows once they are here. The chunk then leaves
// without waiting for the indices' way through LDS and a barrier.
template <int N>
__device__ __forceinline__ void first_entries(int32_t (&e)[N], const SplitRows& r, int cbase,
                                              int rg0) {
#pragma unroll
  for (int i = 0; i < N; ++i)
    e[i] = r.idx[r.entry(cbase + 8 * (rg0 + i) + (int)((threadIdx.x & 63) >> 3))];
}
template <int N>
__device__ __forceinline__ void first_rows(const uint8_t* (&src)[N], const int32_t (&e)[N],
                                           const SplitRows& r, int cbase, int rg0) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int i = 0; i < N; ++i)
    src[i] = r.row(cbase + 8 * (rg0 + i) + (lane >> 3), r.checked(e[i])) +
             stage_piece(lane, rg0 + i);
}

// The split's n_rec index entries on their way to LDS, NT threads: all loads first, the checked
// entries stored later.
template <int NT>
struct IndexCopy {
  static constexpr int N = kMaxSplitRecords / NT;
  int32_t v[N];
  __device__ __forceinline__ void load(const SplitRows& r, int n_rec) {
#pragma unroll
    for (int u = 0; u < N; ++u)
      if (u * NT < n_rec) v[u] = r.idx[min((int)threadIdx.x + u * NT, n_rec - 1)];  // uniform
  }
  __device__ __forceinline__ void store(int32_t* s_idx, const SplitRows& r, int n_rec) {
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int i = threadIdx.x + u * NT;
      if (u * NT < n_rec && i < n_rec) s_idx[i] = r.checked(v[u]);
    }
  }
};

// Validity words of tokens [tok_begin, tok_begin + span), span a multiple of 32, one 64-token
// group per wave and step: bit t of word c is token tok_begin + 32 c + t. Tokens past the split
// end have zero bits.
template <int NW>
__device__ __forceinline__ void valid_words(uint32_t* s_valid, const int32_t* s_idx,
                                            const SplitRows& r, int tok_begin, int span) {
  const int lane = threadIdx.x & 63;
  for (int base = (threadIdx.x >> 6) * 64; base < span; base += 64 * NW) {
    const int tk = tok_begin + base + lane;
    const uint64_t m = __ballot(tk < r.tok_end && s_idx[r.entry(tk)] >= 0);
    if (lane == 0) {
      s_valid[base >> 5] = (uint32_t)m;
      if (base + 32 < span) s_valid[(base >> 5) + 1] = (uint32_t)(m >> 32);
    }
  }
}

// The calling wave's loads of the current chunk are done once at most `younger` (at most
// NST - 2, none with one buffer) later chunks' loads, LPW each, are outstanding; then the
// workgroup synchronises. With one head wave per token group (HW = 1) the tiles are the wave's
// own and nobody waits for another wave: the waves drift apart and one's loads overlap another's
// arithmetic.
template <int N, bool BARRIER>
__device__ __forceinline__ void wait_loads() {
  if constexpr (BARRIER) wait_loads_and_barrier<N>();
  else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
}
template <int NST, int LPW, int HW>
__device__ __forceinline__ void wait_chunk(int younger) {
  if (NST > 3 && younger >= 2) wait_loads<(NST > 3 ? 2 : 0) * LPW, (HW > 1)>();
  else if (NST > 2 && younger >= 1) wait_loads<(NST > 2 ? 1 : 0) * LPW, (HW > 1)>();
  else wait_loads<0, (HW > 1)>();
}

template <int DQK, int DV, int VOFF, int HW, int TW, int NST>
__global__ __launch_bounds__(64 * HW * TW, (HW * TW >= 8) ? 2 : 1)
void attn_partial_kernel(AttnArgs a) {
  constexpr int TE = (DQK > VOFF + DV) ? DQK : VOFF + DV;  // bf16 per token used here
  using T = Tile<TE / 8>;
  constexpr int RGW = 4 / HW;              // row groups of a chunk that one head wave stages
  constexpr int LPW = RGW * T::NSEG;       // its loads per chunk
  constexpr int NKK = DQK / 32;
  constexpr int NOUT = DV / 16;
  static_assert(DQK % 32 == 0 && DV % 16 == 0 && VOFF % 8 == 0, "shape");
  static_assert(NST >= 1 && NST <= 4 && (NST - 2) * LPW < 64, "pipeline depth");
  static_assert(NST > 1 || HW == 1, "one round (NST = 1): a split of at most TW chunks");
  __shared__ __align__(1024) uint8_t s_kv[TW * NST * T::BYTES];
  __shared__ int32_t s_idx[kMaxSplitRecords];  // the split's record indices, -1 = skip
  __shared__ uint32_t s_valid[kMaxSplitTokens / 32];  // bit t of word c: token 32c+t attends

  load_args(a);
  // XCD-aware mapping: consecutive workgroup ids go round-robin over the 8 XCDs, so give each
  // XCD a contiguous range of work items; the head blocks of one (unit, split) then share the
  // staged records through the same L2.
  const int nwg_pad = (a.n_wg + 7) & ~7;
  if ((int)blockIdx.x >= nwg_pad) {  // wave-uniform: the whole workgroup replays
    replay_worker(a.rp, (int)blockIdx.x - nwg_pad);
    return;
  }
  const int w = (int)(blockIdx.x & 7) * (nwg_pad >> 3) + (int)(blockIdx.x >> 3);
  if (w >= a.n_wg) return;
  const int col_split = (int)fastdiv(w, a.div_hb), hb = w - col_split * a.hb;
  const int unit = (int)fastdiv(col_split, a.div_splits);
  const int split = col_split - unit * a.n_wg_splits;
  const int idx_row = unit - (int)fastdiv(unit, a.div_idx) * a.idx_units;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int hg = wave % HW, tg = wave / HW;
  const int g = lane >> 4;
  uint8_t* s_tiles = s_kv + tg * NST * T::BYTES;

  const int tok_begin = split * a.split_tokens;
  const int tok_end = min(a.n_tok, tok_begin + a.split_tokens);
  const int rec_begin = tok_begin >> a.tpr_shift;
  const int n_rec = ((tok_end - 1) >> a.tpr_shift) - rec_begin + 1;
  const SplitRows rows{a.idx + (int64_t)idx_row * a.k + rec_begin,
                       a.pool + (int64_t)unit * a.rec_per_unit * a.R,
                       tok_end, rec_begin, a.tpr_shift, a.R, a.token_bytes, a.rec_per_unit};
  // wave hg stages row groups [hg * RGW, (hg + 1) * RGW) of each chunk of its token group
  const int rg0 = __builtin_amdgcn_readfirstlane(hg) * RGW;
  const int chunk0 = tok_begin + __builtin_amdgcn_readfirstlane(tg) * kChunk;
  int32_t entry0[RGW];
  first_entries(entry0, rows, chunk0, rg0);
  IndexCopy<64 * HW * TW> ic;
  ic.load(rows, n_rec);

  const int head = hb * 16 * HW + hg * 16 + (lane & 15);
  const bool head_ok = head < a.H;
  // Q^T operand, loaded unconditionally (a head past H reads head 0's row: its scores are never
  // stored and, being head 0's, move no reference max that head 0 does not)
  bf16x8_t qreg[NKK];
  {
    const uint16_t* qrow = a.q + ((int64_t)unit * a.H + (head_ok ? head : 0)) * DQK + 8 * g;
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk)
      qreg[kk] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4*>(qrow + kk * 32));
  }
  const uint8_t* src[RGW];
  first_rows(src, entry0, rows, chunk0, rg0);
  // the query has arrived before the first chunk is issued: a wait for it inside the loop would
  // drain the chunks in flight
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk) asm volatile("" : "+v"(qreg[kk]));
  auto issue = [&](int buf) {
#pragma unroll
    for (int i = 0; i < RGW; ++i) stage_rows<TE / 8>(s_tiles + buf * T::BYTES, rg0 + i, src[i]);
  };
  auto next_rows = [&](int it) {
    chunk_rows(src, s_idx, rows, chunk0 + it * kChunk * TW, rg0);
  };
  issue(0);
  ic.store(s_idx, rows, n_rec);

  f32x4 o[NOUT];
#pragma unroll
  for (int n = 0; n < NOUT; ++n) o[n] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;
  const int n_it = (tok_end - tok_begin + kChunk * TW - 1) / (kChunk * TW);
  lds_barrier();  // s_idx is ready
  // every chunk the token groups iterate over gets its word, including chunks that lie wholly
  // past the split end
  valid_words<HW * TW>(s_valid, s_idx, rows, tok_begin, n_it * kChunk * TW);
  if constexpr (HW == 1) lds_barrier();  // the loop has no barrier to publish the words
#pragma unroll
  for (int st = 1; st < NST - 1; ++st)
    if (st < n_it) {
      next_rows(st);
      issue(st);
    }

  // Per chunk: scores (QK), softmax against the running reference max, then P.V. O is touched
  // only by MFMAs inside the loop; the rare move of a head's reference max (growth beyond the
  // slack) leaves the loop, rescales, finishes that chunk and re-enters.
  f32x4 s0, s1;
  float sc[8];
  float cmax = -INFINITY;
  int it = 0;

  // the head's largest score from its four lanes' largest
  auto head_max = [](float v) {
    v = fmaxf(v, __shfl_xor(v, 16, 64));
    return fmaxf(v, __shfl_xor(v, 32, 64));
  };
  auto finish_chunk = [&](const uint8_t* tile) {
    uint32_t pw[4];
    softmax_weights<8>(pw, sc, a.scale_log2, m_run);
#pragma unroll
    for (int j = 0; j < 4; ++j) l_run = add_weights(pw[j], l_run);
    const bf16x8_t pa = __builtin_bit_cast(bf16x8_t, u32x4{pw[0], pw[1], pw[2], pw[3]});
    // V operand by transpose reads: in each 16-lane group, lane 4s+q addresses
    // V[token][16n + 4q .. +3] of token tile_row(4g+s) (first read) or 16 further (second
    // read); lane t then holds V[those tokens][16n + t], i.e. B[k = 8g .. 8g+7][n = t], in the
    // token order of this lane's P values.
    const int vr = tile_row(4 * g + ((lane & 15) >> 2));  // row; the second read's is 16 further
    const uint32_t vrow = lds_addr(tile + T::row(vr) + 8 * (lane & 1));
    const int vp = (((lane & 3) >> 1) ^ tile_swizzle(vr)) << 4;
    // transpose reads VD output tiles ahead of their MFMAs (opaque LDS reads, see lds_read_b128)
    constexpr int VD = 3;
    static_assert(VD == 3 && NOUT > VD, "the waits below count a ring of 3 read pairs");
    static_assert(VOFF % 64 == 0 && DV % 64 == 0, "V starts on a segment");
    v4i16 vlo[VD], vhi[VD];
    uint32_t va[4];  // tiles n, n + 4, ...: dims 16n sit at piece 2n of segment VOFF / 64 + n / 4
#pragma unroll
    for (int n = 0; n < 4; ++n) va[n] = vrow + (vp ^ (32 * n));
    auto vread = [&](auto n) {
      constexpr int OFF = (VOFF / 64 + n / 4) * 1024;
      vlo[n % VD] = lds_read_tr16_b64<OFF>(va[n & 3]);
      vhi[n % VD] = lds_read_tr16_b64<OFF + 2 * T::NSEG * 1024>(va[n & 3]);
    };
    static_for<VD>(vread);
    static_for<NOUT>([&](auto n) {
      // the reads issued after tile n's pair: those of tiles n+1 .. min(n+VD-1, NOUT-1)
      constexpr int later = NOUT - 1 - n < VD - 1 ? NOUT - 1 - n : VD - 1;
      lgkm_wait2<2 * later>(vlo[n % VD], vhi[n % VD]);
      const bf16x8_t vb = __builtin_bit_cast(
          bf16x8_t, __builtin_shufflevector(vlo[n % VD], vhi[n % VD], 0, 1, 2, 3, 4, 5, 6, 7));
      o[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pa, vb, o[n], 0, 0, 0);
      if constexpr (n + VD < NOUT) vread(std::integral_constant<int, n + VD>{});
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  // the chunk's scores (sc, this lane's largest in cmax), and the head's reference max if it has
  // none yet
  auto scores = [&](const uint8_t* tile, uint32_t vmask) {
    // ---- scores: S^T tiles for tokens [0,16) and [16,32) of the chunk ----
    // K reads KD k-steps ahead (opaque LDS reads, see lds_read_b128), each k-step's MFMAs once
    // its pair is in
    s0 = f32x4{0.f, 0.f, 0.f, 0.f};
    s1 = f32x4{0.f, 0.f, 0.f, 0.f};
    const int kr = tile_row(lane & 15);
    const uint32_t krow = lds_addr(tile + T::row(kr));
    const int kp = (g ^ tile_swizzle(kr)) << 4;  // piece 4 kk + g: kk odd is 64 bytes apart
    const uint32_t ka_even = krow + kp, ka_odd = krow + (kp ^ 64);
    constexpr int KD = 4;  // read pairs in flight
    static_assert(KD <= NKK && 2 * KD <= 15, "lgkmcnt holds at most 15 outstanding reads");
    u32x4 ka[KD], kb[KD];
    auto kread = [&](auto kk) {
      const uint32_t ad = (kk & 1) ? ka_odd : ka_even;
      ka[kk % KD] = lds_read_b128<(kk / 2) * 1024>(ad);
      kb[kk % KD] = lds_read_b128<(kk / 2) * 1024 + 2 * T::NSEG * 1024>(ad);
    };
    static_for<KD>(kread);
    static_for<NKK>([&](auto kk) {
      // the pairs issued after pair kk: those of k-steps kk+1 .. min(kk+KD-1, NKK-1)
      constexpr int later = NKK - 1 - kk < KD - 1 ? NKK - 1 - kk : KD - 1;
      lgkm_wait2<2 * later>(ka[kk % KD], kb[kk % KD]);
      s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, ka[kk % KD]),
                                                  qreg[kk], s0, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, kb[kk % KD]),
                                                  qreg[kk], s1, 0, 0, 0);
      if constexpr (kk + KD < NKK) kread(std::integral_constant<int, kk + KD>{});
      __builtin_amdgcn_sched_barrier(0);
    });
#pragma unroll
    for (int j = 0; j < 8; ++j) sc[j] = j < 4 ? s0[j] : s1[j - 4];
    if (vmask != 0xFFFFFFFFu) {  // uniform: a chunk with padding
      int gq = g;
      asm volatile("" : "+v"(gq));
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int bit = j < 4 ? tile_row(4 * gq + j) : 16 + tile_row(4 * gq + (j - 4));
        sc[j] = ((vmask >> bit) & 1u) ? sc[j] : -INFINITY;
      }
    }
    cmax = sc[0];
#pragma unroll
    for (int j = 1; j < 8; ++j) cmax = fmaxf(cmax, sc[j]);
    cmax *= a.scale_log2;  // this lane's quarter of the head's scores
    // Validity is per token, so every head of the wave agrees on whether m_run is -inf.
    // While it is, O and l are exactly zero and the reference max can simply be set.
    if (__ballot(m_run == -INFINITY)) {
      const float all = head_max(cmax);
      if (m_run == -INFINITY) m_run = all;
    }
  };

  if constexpr (NST == 1) {  // one round: no later chunk to wait for or to outgrow the reference
    wait_chunk<NST, LPW, HW>(0);
    scores(s_tiles, __builtin_amdgcn_readfirstlane(s_valid[tg]));
    finish_chunk(s_tiles);
  } else {
    for (;;) {
      for (; it < n_it; ++it) {
        // chunks it+1 .. it+NST-2 were issued earlier and may still be in flight
        wait_chunk<NST, LPW, HW>(min(NST - 2, n_it - 1 - it));
        const uint8_t* tile = s_tiles + (it % NST) * T::BYTES;
        // the chunk's validity word, read before the next chunk's loads are issued
        const uint32_t vmask = __builtin_amdgcn_readfirstlane(s_valid[it * TW + tg]);
        __builtin_amdgcn_sched_barrier(0);
        // every wave is past its reads of buffer (it-1) % NST: refill it with chunk it+NST-1
        if (it + NST - 1 < n_it) {
          next_rows(it + NST - 1);
          issue((it + NST - 1) % NST);
        }
        scores(tile, vmask);
        if (__ballot(cmax > m_run + kRescaleSlack)) break;
        finish_chunk(tile);
      }
      if (it >= n_it) break;
      // rare path: move the reference max of the heads whose scores outgrew it
      const float m_new = fmaxf(m_run, head_max(cmax));
      const float alpha = m_run == -INFINITY ? 1.f : exp2f(m_run - m_new);  // -inf: l and O are 0
      l_run *= alpha;
      m_run = m_new;
      float al[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) al[j] = __shfl(alpha, 4 * g + j, 64);
#pragma unroll
      for (int n = 0; n < NOUT; ++n) {
#pragma unroll
        for (int j = 0; j < 4; ++j) o[n][j] *= al[j];
      }
      finish_chunk(s_tiles + (it % NST) * T::BYTES);
      ++it;
    }
  }

  l_run += __shfl_xor(l_run, 16, 64);  // each lane summed its quarter of the head's weights
  l_run += __shfl_xor(l_run, 32, 64);

  // ---- results of this split: the token groups' results merged per head through LDS, in group
  // order, each wave finishing NOUT / TW of its heads' output tiles. A split is then one partial
  // result instead of one per token group, and a unit that is one split is written out here,
  // as the merge of one part would (weight 1, one reciprocal). ----
  constexpr int NF = NOUT / TW;
  static_assert(NOUT % TW == 0 && TW * NST * T::BYTES >= TW * HW * (NOUT * 64 * 16 + 16 * 8),
                "the tiles hold every wave's results");
  f32x4* s_o = reinterpret_cast<f32x4*>(s_kv);  // [TW][HW][NOUT][64 lanes]
  float2* s_ml = reinterpret_cast<float2*>(s_o + TW * HW * NOUT * 64);  // [TW][HW][16 heads]
  lds_barrier();  // every wave is past its tiles
#pragma unroll
  for (int n = 0; n < NOUT; ++n) s_o[(wave * NOUT + n) * 64 + lane] = o[n];
  if (lane < 16) s_ml[wave * 16 + lane] = make_float2(m_run, l_run);
  lds_barrier();
  // this lane's accumulator rows are heads 4g .. 4g + 3 of the wave's 16
  float wt[TW][4], M[4], L[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float2 ml[TW];
    M[j] = -INFINITY;
    L[j] = 0.f;
#pragma unroll
    for (int t = 0; t < TW; ++t) {
      ml[t] = s_ml[(t * HW + hg) * 16 + 4 * g + j];
      M[j] = fmaxf(M[j], ml[t].x);
    }
#pragma unroll
    for (int t = 0; t < TW; ++t) {
      // a group without a valid token has m = -inf, O = 0, l = 0 and contributes nothing
      wt[t][j] = ml[t].x == -INFINITY ? 0.f : exp2f(ml[t].x - M[j]);
      L[j] += ml[t].y * wt[t][j];
    }
  }
  const int head_base = hb * 16 * HW + hg * 16 + 4 * g;
  float* po = a.direct ? a.out + (int64_t)unit * a.H * DV
                       : a.part_o + ((int64_t)unit * a.n_parts + split) * a.H * DV;
#pragma unroll
  for (int i = 0; i < NF; ++i) {
    const int n = tg * NF + i;
    f32x4 r = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < TW; ++t) {
      const f32x4 v = s_o[((t * HW + hg) * NOUT + n) * 64 + lane];
#pragma unroll
      for (int j = 0; j < 4; ++j) r[j] += v[j] * wt[t][j];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int h = head_base + j;
      const float inv = L[j] > 0.f ? 1.f / L[j] : 0.f;
      if (h < a.H) po[(int64_t)h * DV + n * 16 + (lane & 15)] = a.direct ? r[j] * inv : r[j];
    }
  }
  if (!a.direct && tg == 0 && (lane & 15) == 0) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (head_base + j < a.H)
        a.part_ml[((int64_t)unit * a.n_parts + split) * a.H + head_base + j] =
            make_float2(M[j], L[j]);
  }
}

// Logical row r of a 32-token MFMA tile -> LDS tile row (token) for the latent-attention kernel.
// With r = 16a + 8b + 4h + s the row is 16a + 4s + 2b + h: the P operand of a lane (k-step a,
// half h) then comes straight from its S^T accumulator, and each group of 16 lanes of a V transpose
// read touches rows 4 apart, which the swizzle spreads over the slots of their half (see Tile); the
// 16 K rows that one operand load reads are a permutation of 16 consecutive rows.
__device__ inline int mla_row(int r) {
  return 16 * (r >> 4) + 4 * (r & 3) + 2 * ((r >> 3) & 1) + ((r >> 2) & 1);
}

// Scores of the latent-attention kernel may exceed the split's reference by this many powers
// of two: P <= 2^64 and sums over at most 8192 tokens stay far inside the fp32/bf16 range.
constexpr float kMlaSlack = 64.0f;

// Exact fallback for a latent-attention split whose scores outgrow the reference: plain online
// softmax with fp32 rescaling, one head at a time per wave, K and V read straight from the
// pool. Writes the split's partial results in the fast path's format. Only inputs whose scores
// span more than kMlaSlack powers of two within one split ever come here.
__device__ __forceinline__ void mla_split_exact(const AttnArgs& a, const int32_t* s_idx,
                                                const uint32_t* s_valid, int unit, int split,
                                                int tok_begin, int tok_end, int rec_begin,
                                                int head0, bool direct) {
  constexpr int DQK = 576, DV = 512;
  const int lane = threadIdx.x & 63;
  const uint8_t* pool_u = a.pool + (int64_t)unit * a.rec_per_unit * a.R;
  const int tpr_mask = (1 << a.tpr_shift) - 1;
  for (int hh = 0; hh < 32; ++hh) {
    const int head = head0 + hh;
    if (head >= a.H) break;
    const uint16_t* qh = a.q + ((int64_t)unit * a.H + head) * DQK;
    float qv[DQK / 64];
#pragma unroll
    for (int i = 0; i < DQK / 64; ++i) qv[i] = bf16_to_f32(qh[lane + 64 * i]);
    float m = -INFINITY, l = 0.f, acc[DV / 64];
#pragma unroll
    for (int e = 0; e < DV / 64; ++e) acc[e] = 0.f;
    for (int t = tok_begin; t < tok_end; ++t) {
      const int bit = t - tok_begin;
      if (!((s_valid[bit >> 5] >> (bit & 31)) & 1u)) continue;
      const int rec = s_idx[(t >> a.tpr_shift) - rec_begin];
      const uint16_t* kt = reinterpret_cast<const uint16_t*>(
          pool_u + (int64_t)rec * a.R + (int64_t)(t & tpr_mask) * a.token_bytes);
      float d = 0.f;
#pragma unroll
      for (int i = 0; i < DQK / 64; ++i) d += qv[i] * bf16_to_f32(kt[lane + 64 * i]);
#pragma unroll
      for (int x = 32; x >= 1; x >>= 1) d += __shfl_xor(d, x, 64);
      const float m_new = fmaxf(m, d * a.scale_log2);
      const float alpha = exp2f(m - m_new);
      const float pr = exp2f(over_reference(d, a.scale_log2, m_new));
      l = l * alpha + pr;
#pragma unroll
      for (int e = 0; e < DV / 64; ++e)
        acc[e] = acc[e] * alpha + pr * bf16_to_f32(kt[lane * (DV / 64) + e]);
      m = m_new;
    }
    if (direct) {
      const float inv = l > 0.f ? 1.f / l : 0.f;
      float* oh = a.out + ((int64_t)unit * a.H + head) * DV + lane * (DV / 64);
#pragma unroll
      for (int e = 0; e < DV / 64; ++e) oh[e] = acc[e] * inv;
      continue;
    }
    float* po = a.part_o + ((int64_t)unit * a.n_parts + split) * a.Hp * DV;
#pragma unroll
    for (int e = 0; e < DV / 64; ++e) po[mla_part_offset(head, lane * (DV / 64) + e)] = acc[e];
    if (lane == 0)
      a.part_ml[((int64_t)unit * a.n_parts + split) * a.H + head] = make_float2(m, l);
  }
}

// Latent attention (d_qk 576, d_v 512 = the first 512 key dims). One workgroup per
// (unit, token split, head block of 32 * HW heads); wave w owns 32 heads (w % HW) of token
// group w / HW. Each of the two token groups has its own ring of two chunk tiles in LDS, staged
// once for its HW head waves; the split's 32-token chunks alternate between the groups, and the
// two groups' results are merged in LDS at the end, so a workgroup writes one partial result
// for twice the tokens of one group (half the partial traffic of two workgroups).
// Bound: a round (one chunk per group) of a 128-head call takes 1.7 us with 64 workgroups on the
// chip and 2.3 with 192 or 256, 0.9 of them MFMA issue, 0.35 softmax and the rest waiting for the
// next chunk, of which LDS holds only one (four tiles of 36 KB fill it). Many workgroups of 16-32
// heads reach the HBM rate instead (64 units x 16 heads: 6.3 TB/s in the loop); calls of few rounds
// are bound by the chain of index, first chunk, result and merge. Measured, merge included, before
// these tiles -> now: 96 units x 128 heads x 2048 tokens 137 -> 87.5 us, 64 x 16 81 -> 40.8, 16 x 128
// 33.5 -> 28.2 (of which 67 MB of partials written and read are 13), 5 x 72 x 1337 26.0 -> 17.3, 1 x
// 128 19.0 -> 16.7.
//   S^T[token][head] = K[token][:] . Q^T[:][head]   v_mfma_f32_32x32x16_bf16, 36 k-steps, K rows
//                                                   from LDS, Q resident in VGPRs
//   O[head][dim]    += P[head][token] . V[token][dim]  v_mfma_f32_32x32x16_bf16, 2 k-steps x 16
//                                                   output tiles, V by LDS transpose reads
// A lane holds 16 of a head's 32 scores (the other 16 are in lane ^ 32), which are exactly its
// P operands of the two PV k-steps; O (16 tiles x 16 fp32 per lane) lives in accumulators.
// PACED: the query follows the first chunk; DIRECT: a unit is one split, its output is written here;
// ANYQ: a query that does not start at a multiple of 16 bytes, which direct-to-LDS loads need (a
// kernel of its own: the branch alone cost the large direct calls up to 0.7%).
template <int HW, bool PACED, bool DIRECT, bool ANYQ>
__global__ __launch_bounds__(128 * HW, 1)
void attn_mla_kernel(AttnArgs a) {
  constexpr int DQK = 576, DV = 512;
  constexpr int TG = 2, NST = 2, NW = HW * TG;
  using T = Tile<DQK / 8>;
  static_assert(HW == 1 || HW == 2, "one query tile per token group at most");
  constexpr int RGW = 4 / HW;                // row groups of a chunk that one head wave stages
  constexpr int LPW = RGW * T::NSEG;         // its loads per chunk
  // With one head wave a tile is its wave's own: no barrier in the loop, and the scores begin when
  // the first four of a chunk's nine segments are here, the others being awaited in their middle
  // (64 units of 16 heads: 42.1 us -> 40.8). With two, the second barrier costs what it saves (96
  // units of 128 heads: 87.3 us against 88.5).
  constexpr int EARLY = HW == 1 ? 4 : T::NSEG;
  constexpr int NKK = DQK / 16;  // QK k-steps
  constexpr int NDV = DV / 32;   // PV output tiles
  static_assert(LPW < 64, "the wait counter's range");
  static_assert(TG * NST * T::BYTES >= NW * (NDV / 2 * 4 * 64 * 16 + 32 * 8 + 96 * 4),
                "the tiles hold half of each wave's results for the merge");
  __shared__ __align__(1024) uint8_t s_kv[TG * NST * T::BYTES];
  __shared__ int32_t s_idx[kMaxSplitRecords];         // the split's record indices, -1 = skip
  __shared__ uint32_t s_valid[kMaxSplitTokens / 32];  // bit t of word c: token 32c+t attends
  __shared__ int s_fallback;                           // some score outgrew its reference

  load_args(a);
  // XCD-aware mapping, as in attn_partial_kernel
  const int nwg_pad = (a.n_wg + 7) & ~7;
  if ((int)blockIdx.x >= nwg_pad) {  // wave-uniform: the whole workgroup replays
    replay_worker(a.rp, (int)blockIdx.x - nwg_pad);
    return;
  }
  const int w = (int)(blockIdx.x & 7) * (nwg_pad >> 3) + (int)(blockIdx.x >> 3);
  if (w >= a.n_wg) return;
  const int col_split = (int)fastdiv(w, a.div_hb), hb = w - col_split * a.hb;
  const int unit = (int)fastdiv(col_split, a.div_splits);
  const int split = col_split - unit * a.n_wg_splits;
  const int idx_row = unit - (int)fastdiv(unit, a.div_idx) * a.idx_units;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int half = lane >> 5, col = lane & 31;
  const int hg = wave % HW, tg = wave / HW;  // head wave within the token group, token group
  uint8_t* s_tiles = s_kv + tg * NST * T::BYTES;

  const int tok_begin = split * a.split_tokens;
  const int tok_end = min(a.n_tok, tok_begin + a.split_tokens);
  const int rec_begin = tok_begin >> a.tpr_shift;
  const int n_rec = ((tok_end - 1) >> a.tpr_shift) - rec_begin + 1;
  const SplitRows rows{a.idx + (int64_t)idx_row * a.k + rec_begin,
                       a.pool + (int64_t)unit * a.rec_per_unit * a.R,
                       tok_end, rec_begin, a.tpr_shift, a.R, a.token_bytes, a.rec_per_unit};
  const int rg0 = __builtin_amdgcn_readfirstlane(hg) * RGW;
  // iteration `it` of token group g covers the split's chunk it * TG + g
  const int chunk0 = tok_begin + __builtin_amdgcn_readfirstlane(tg) * kChunk;
  int32_t entry0[RGW];
  first_entries(entry0, rows, chunk0, rg0);
  IndexCopy<64 * NW> ic;
  ic.load(rows, n_rec);

  const int head0 = hb * 32 * HW + hg * 32;  // first head of this wave
  const int head = head0 + col;
  const bool head_ok = head < a.H;
  // The query reaches its registers through LDS: the 32 rows of head wave hg are one tile, staged
  // like a chunk by both token groups' waves of that head wave, in the second chunk buffer of
  // group hg, which the loop fills only after they are read. Read straight
  // from memory in operand order, every lane of a load touches a cache line of its own: that
  // took 3.2 us per workgroup of a 16-unit call. A head past H reads head 0's row: its scores
  // are never stored and, equal to head 0's, change no split-level decision.
  uint8_t* q_tile = s_kv + (hg * NST + 1) * T::BYTES;
  auto stage_q = [&]() {
#pragma unroll
    for (int i = 0; i < 4 / TG; ++i) {
      const int rg = __builtin_amdgcn_readfirstlane(tg) * (4 / TG) + i;
      const int h = head0 + 8 * rg + (lane >> 3);
      const uint8_t* row = reinterpret_cast<const uint8_t*>(
                               a.q + ((int64_t)unit * a.H + (h < a.H ? h : 0)) * DQK) +
                           stage_piece(lane, rg);
      if constexpr (ANYQ) copy_rows<DQK / 8>(q_tile, rg, row);
      else stage_rows<DQK / 8>(q_tile, rg, row);
    }
  };
  bf16x8_t qreg[NKK];
  auto read_q = [&]() {  // Q[head][16kk + 8 half .. +7]
    uint32_t qa[4];
    const int sw = tile_swizzle(col);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      qa[i] = lds_addr(q_tile + T::row(col) + (((2 * i + half) ^ sw) << 4));
    static_for<NKK / 4>([&](auto j) {  // four reads and their wait in one block
      u32x4 v0, v1, v2, v3;
      asm volatile(
          "ds_read_b128 %0, %4 offset:%8\n\tds_read_b128 %1, %5 offset:%8\n\t"
          "ds_read_b128 %2, %6 offset:%8\n\tds_read_b128 %3, %7 offset:%8\n\t"
          "s_waitcnt lgkmcnt(0)"
          : "=&v"(v0), "=&v"(v1), "=&v"(v2), "=&v"(v3)
          : "v"(qa[0]), "v"(qa[1]), "v"(qa[2]), "v"(qa[3]), "n"(j * 1024));
      qreg[4 * j] = __builtin_bit_cast(bf16x8_t, v0);
      qreg[4 * j + 1] = __builtin_bit_cast(bf16x8_t, v1);
      qreg[4 * j + 2] = __builtin_bit_cast(bf16x8_t, v2);
      qreg[4 * j + 3] = __builtin_bit_cast(bf16x8_t, v3);
    });
  };
  // Unpaced, the query goes out behind the index loads and is in flight while they are checked
  // and the first chunk issued. Paced, it follows the first chunk's arrival (below), which
  // spreads the workgroups' start-up traffic.
  if constexpr (!PACED) stage_q();
  const uint8_t* src[RGW];  // this lane's rows of the chunk to issue next
  // Load l of a chunk: with one head wave segment by segment, else row group by row group.
  auto stage = [&](auto l, uint8_t* tile) {
    constexpr int seg = HW == 1 ? l / RGW : l % T::NSEG, i = HW == 1 ? l % RGW : l / T::NSEG;
    stage_block<DQK / 8, seg>(tile, rg0 + i, src[i]);
  };
  first_rows(src, entry0, rows, chunk0, rg0);
  static_for<LPW>([&](auto l) { stage(l, s_tiles); });
  ic.store(s_idx, rows, n_rec);
  if (tid == 0) s_fallback = 0;
  f32x16 o[NDV];
#pragma unroll
  for (int n = 0; n < NDV; ++n) {
    o[n] = f32x16{};
    asm volatile("" : "+a"(o[n]));  // cleared here, while the loads are in flight
  }
  float m_run = -INFINITY, l_run = 0.f;
  float sc[16];
  const int n_it = (tok_end - tok_begin + kChunk * TG - 1) / (kChunk * TG);
  lds_barrier();  // s_idx is ready
  // every chunk the groups iterate over gets its word, including a last one wholly past the
  // split end
  valid_words<NW>(s_valid, s_idx, rows, tok_begin, n_it * TG * kChunk);

  auto finish_chunk = [&](const uint8_t* tile, int it) {
    // V operand by transpose reads: in each 16-lane group lane 4s+q addresses row
    // 16kb + 4s + half (+2 for the second read), columns 32n + 16 (col >> 4) + 4q .. +3; lane
    // t of the group then holds V[those rows][32n + 16 (col >> 4) + t], the k order of P.
    const int vr = 4 * ((lane & 15) >> 2) + half;  // row of the first read, k-step 0
    const int vp = 2 * (col >> 4) + ((lane & 3) >> 1);  // piece of tile 0; tile n: 4 further
    // Accumulator tile n holds dims 32n .. of token group 0's output and dims 32 ((n + 8) % 16) ..
    // of group 1's, so that at the end each group finishes its tiles 0-7 and leaves the other
    // group tiles 8-15 with the same code (registers cannot be chosen at run time).
    uint32_t va[2][2][2];  // [tile half][tile parity][first / second read]
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < 2; ++y) {
        const uint32_t v = lds_addr(tile + T::row(vr + 2 * y) + 8 * (lane & 1) +
                                    (((vp + 4 * x) ^ tile_swizzle(vr + 2 * y)) << 4));
        va[0][x][y] = v + 4096 * tg;
        va[1][x][y] = v - 4096 * tg;
      }
    // MFMA i = (k-step kb, tile n) = (i / NDV, i % NDV), so consecutive MFMAs update
    // different tiles; its two reads run VD MFMAs ahead
    constexpr int VD = 3;
    constexpr int NM = 2 * NDV;
    static_assert(VD == 3 && NM > VD, "the waits below count a ring of 3 read pairs");
    v4i16 vlo[VD], vhi[VD];
    auto vread = [&](auto i) {
      constexpr int OFF = (i / NDV) * 2 * T::NSEG * 1024 + (i % NDV) / 2 * 1024;
      constexpr int h = (i % NDV) / (NDV / 2);
      vlo[i % VD] = lds_read_tr16_b64<OFF>(va[h][i & 1][0]);
      vhi[i % VD] = lds_read_tr16_b64<OFF>(va[h][i & 1][1]);
    };
    static_for<VD>(vread);  // in flight while the weights are worked out
    uint32_t pw[8];
    softmax_weights<16>(pw, sc, a.scale_log2, m_run);
#pragma unroll
    for (int j = 0; j < 8; ++j) l_run = add_weights(pw[j], l_run);
    const bf16x8_t pa0 = __builtin_bit_cast(bf16x8_t, u32x4{pw[0], pw[1], pw[2], pw[3]});
    const bf16x8_t pa1 = __builtin_bit_cast(bf16x8_t, u32x4{pw[4], pw[5], pw[6], pw[7]});
    static_for<NM>([&](auto i) {
      // the reads issued after index i's pair: those of indices i+1 .. min(i+VD-1, NM-1)
      constexpr int later = NM - 1 - i < VD - 1 ? NM - 1 - i : VD - 1;
      lgkm_wait2<2 * later>(vlo[i % VD], vhi[i % VD]);
      const bf16x8_t vb = __builtin_bit_cast(
          bf16x8_t, __builtin_shufflevector(vlo[i % VD], vhi[i % VD], 0, 1, 2, 3, 4, 5, 6, 7));
      o[i % NDV] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(i < NDV ? pa0 : pa1, vb, o[i % NDV],
                                                           0, 0, 0);
      if constexpr (i + VD < NM) vread(std::integral_constant<int, i + VD>{});
      // the next iteration's chunk to issue: its rows are found in the MFMAs' shadow
      if constexpr (i == NDV / 2)
        if (it + NST < n_it) chunk_rows(src, s_idx, rows, chunk0 + (it + NST) * kChunk * TG, rg0);
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  // Exponentials are taken against a per-head reference max fixed by the first valid chunk of
  // the split (exact softmax arithmetic with a different reference point; the combine uses the
  // same reference). Scores more than kMlaSlack powers of two above it send the whole split to
  // an exact fallback after the loop, whose results are then discarded; the loop itself never
  // leaves early, so O has a single update path (the MFMAs) and stays in accumulators.
  if constexpr (PACED) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    stage_q();
    wait_loads_and_barrier<0>();
  } else {
    wait_loads_and_barrier<LPW>();
  }
  read_q();
  if constexpr (HW == 1) lds_barrier();  // both groups have the query: its buffer is free
  if (n_it > 1) chunk_rows(src, s_idx, rows, chunk0 + kChunk * TG, rg0);

  for (int it = 0; it < n_it; ++it) {
    wait_loads<(T::NSEG - EARLY) * RGW, (HW > 1)>();
    const uint8_t* tile = s_tiles + (it % NST) * T::BYTES;
    constexpr int KD = 4;
    static_assert(KD == 4 && NKK > KD, "a ring of 4 reads, one address register each");
    const int kr = mla_row(col);
    uint32_t ka[4];  // piece 2 kk + half of k-steps kk, kk + 4, ...
#pragma unroll
    for (int i = 0; i < 4; ++i)
      ka[i] = lds_addr(tile + T::row(kr) + (((2 * i + half) ^ tile_swizzle(kr)) << 4));
    u32x4 kbuf[KD];
    static_for<KD>([&](auto kk) { kbuf[kk] = lds_read_b128<(kk / 4) * 1024>(ka[kk & 3]); });
    const uint32_t valid = s_valid[it * TG + tg];  // the chunk's validity word
    __builtin_amdgcn_sched_barrier(0);
    // Every wave is past its reads of buffer (it-1) % NST: it takes chunk it+NST-1, whose loads
    // go out LPI at a time between the score MFMAs. Issued in one run they would hold the wave
    // back: the CU's address path takes a 64-lane 16-byte load about every 16 cycles, 0.5 us
    // for a chunk of each token group, with the MFMAs waiting behind it.
    const bool more = it + NST - 1 < n_it;
    uint8_t* next = s_tiles + ((it + NST - 1) % NST) * T::BYTES;

    // ---- scores: S^T for the chunk's 32 tokens x this wave's 32 heads ----
    // K operand reads run KD k-steps ahead of the MFMAs (a small register ring; the
    // scheduling fences keep the compiler from hoisting all 36 reads). The score MFMAs are
    // written as assembly so that their accumulator stays in VGPRs: the output tiles fill
    // the accumulation registers. Hazards hidden from the compiler by the assembly are
    // covered in it: wait states before each MFMA for a just-written operand, and after the
    // last one before the scores are read.
    constexpr int LPI = 3;  // one branch for three loads
    static_assert(LPW % LPI == 0 && LPW <= NKK, "the chunk's loads fit between the MFMAs");
    constexpr int KLATE = 4 * EARLY - KD;  // the k-step before the first read of a later segment
    constexpr int ISSUED = (KLATE / LPI + 1) * LPI;  // the next chunk's loads that are out by then
    f32x16 sacc, sacc1;  // even / odd k-steps: two independent MFMA chains
    static_for<NKK>([&](auto kk) {
      // the K reads issued after read kk: those of k-steps kk+1 .. min(kk+KD-1, NKK-1)
      constexpr int later = NKK - 1 - kk < KD - 1 ? NKK - 1 - kk : KD - 1;
      mfma_qk<later, (kk < 2)>((kk & 1) ? sacc1 : sacc, kbuf[kk % KD], qreg[kk]);
      if constexpr (kk % LPI == 0 && kk < LPW) {
        if (more)
          static_for<LPI>([&](auto i) {
            stage(std::integral_constant<int, kk + i>{}, next);
          });
      }
      if constexpr (EARLY < T::NSEG && kk == KLATE) {
        if (more) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(ISSUED) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      }
      if constexpr (kk + KD < NKK)
        kbuf[kk % KD] = lds_read_b128<((kk + KD) / 4) * 1024>(ka[kk & 3]);
      __builtin_amdgcn_sched_barrier(0);
    });
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" : "+v"(sacc), "+v"(sacc1));
    sacc += sacc1;
#pragma unroll
    for (int j = 0; j < 16; ++j) sc[j] = sacc[j];
    const uint32_t vmask = __builtin_amdgcn_readfirstlane(valid);
    if (vmask != 0xFFFFFFFFu) {  // uniform: a chunk with padding
      int hq = half;
      asm volatile("" : "+v"(hq));
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int bit = mla_row(8 * (j >> 2) + 4 * hq + (j & 3));
        sc[j] = ((vmask >> bit) & 1u) ? sc[j] : -INFINITY;
      }
    }
    float cmax = sc[0];
#pragma unroll
    for (int j = 1; j < 16; ++j) cmax = fmaxf(cmax, sc[j]);
    cmax *= a.scale_log2;  // this lane's half of the head's scores
    // Validity is per token, so every head of the wave agrees on whether m_run is -inf; while
    // it is, O and l are exactly zero and the reference can simply be set.
    if (__ballot(m_run == -INFINITY)) {
      const float both = fmaxf(cmax, __shfl_xor(cmax, 32, 64));
      if (m_run == -INFINITY) m_run = both;
    }
    if (__ballot(cmax > m_run + kMlaSlack) && lane == 0) s_fallback = 1;
    finish_chunk(tile, it);
  }
  l_run += __shfl_xor(l_run, 32, 64);  // each lane summed its half of the head's weights
  wait_loads_and_barrier<0>();  // no staging in flight; s_fallback is final
  if (s_fallback) {
    if (tg == 0)  // the whole split, for this wave's heads
      mla_split_exact(a, s_idx, s_valid, unit, split, tok_begin, tok_end, rec_begin, head0, DIRECT);
    return;
  }
  // ---- partial results of this split, in the accumulator layout (see mla_part_offset), or the
  // unit's output when the split is all of it: the merge of one part, bit for bit (weight 1,
  // one reciprocal of the sum), without its 2 KB per head written and read again ----
  constexpr int HT = NDV / 2;  // output tiles that each group finishes: dims 32 (HT tg + n) ..
  float* oh = DIRECT ? a.out + ((int64_t)unit * a.H + head0 + 4 * half) * DV + 32 * HT * tg + col
                     : nullptr;
  float* po = a.part_o + ((int64_t)unit * a.n_parts + split) * a.Hp * DV +
              (int64_t)(head0 >> 5) * 32 * DV + HT * tg * 1024 + lane * 4;
  const int n_head = a.H - head0;  // heads of this wave that exist
  // heads 8q + 4 half .. +3 of tile n (r: their values; inv: 1 / their sums)
  auto store = [&](int n, int q, const f32x4& r, const f32x4& inv) {
    if constexpr (DIRECT) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (8 * q + 4 * half + e < n_head)
          oh[(int64_t)(8 * q + e) * DV + 32 * n] = (0.f + r[e]) * inv[e];
    } else {
      *reinterpret_cast<f32x4*>(po + (n * 4 + q) * 256) = r;
    }
  };
  // Accumulators are read with explicit v_accvgpr_read (arithmetic on them would make the
  // compiler move all of O into VGPRs and spill); the reads are assembly, so the wait states
  // after the last MFMA that wrote them are given here (the barrier above already separates
  // them by far more).
  asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
  auto acc = [&](int n, int j) {
    float x;
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(x) : "a"(o[n][j]));
    return x;
  };
  // The two token groups' results merged per head on the way out, through LDS (the tiles are
  // free now): each group leaves half of its output tiles and its (reference max, sum) there,
  // and finishes the other half: its own accumulators and the other group's from LDS, both
  // rescaled to the larger reference.
  f32x4* s_o = reinterpret_cast<f32x4*>(s_kv);  // [wave][HT * 4][64 lanes]
  float2* s_ml = reinterpret_cast<float2*>(s_o + NW * HT * 4 * 64);
#pragma unroll
  for (int n = 0; n < HT; ++n)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      s_o[(wave * HT * 4 + n * 4 + q) * 64 + lane] =
          f32x4{o[HT + n][4 * q], o[HT + n][4 * q + 1], o[HT + n][4 * q + 2], o[HT + n][4 * q + 3]};
  if (lane < 32) s_ml[wave * 32 + col] = make_float2(m_run, l_run);
  lds_barrier();
  if (head0 >= a.H) return;
  const int peer = wave ^ HW;  // the other token group's wave of these heads
  const float2 g0 = s_ml[hg * 32 + col], g1 = s_ml[(HW + hg) * 32 + col];
  const float m = fmaxf(g0.x, g1.x);
  // a group without a valid token has m = -inf, O = 0, l = 0 and contributes nothing
  const float a0 = g0.x == -INFINITY ? 0.f : exp2f(g0.x - m);
  const float a1 = g1.x == -INFINITY ? 0.f : exp2f(g1.x - m);
  const float l = g0.y * a0 + g1.y * a1;
  const float l_inv = l > 0.f ? 1.f / l : 0.f;
  // each head's scales to the lanes that hold its rows, by way of LDS (16-byte reads of four
  // heads; lane permutes took 48 dependent LDS round trips)
  float* s_w = reinterpret_cast<float*>(s_ml + 32 * NW) + wave * 96;
  if (lane < 32) {
    s_w[col] = tg == 0 ? a0 : a1;       // this group's
    s_w[32 + col] = tg == 0 ? a1 : a0;  // the other group's
    s_w[64 + col] = l_inv;
  }
  // accumulator row 4q + e of a lane is head 8q + 4 half + e of the wave's 32
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (8 * q >= n_head) break;
    const f32x4 sm = *reinterpret_cast<const f32x4*>(s_w + 8 * q + 4 * half);
    const f32x4 sp = *reinterpret_cast<const f32x4*>(s_w + 32 + 8 * q + 4 * half);
    const f32x4 inv = *reinterpret_cast<const f32x4*>(s_w + 64 + 8 * q + 4 * half);
#pragma unroll
    for (int n = 0; n < HT; ++n) {
      const f32x4 v = s_o[(peer * HT * 4 + n * 4 + q) * 64 + lane];
      f32x4 r;
#pragma unroll
      for (int e = 0; e < 4; ++e) r[e] = acc(n, 4 * q + e) * sm[e] + v[e] * sp[e];
      store(n, q, r, inv);
    }
  }
  if (!DIRECT && tg == 0 && lane < 32 && head_ok)
    a.part_ml[((int64_t)unit * a.n_parts + split) * a.H + head] = make_float2(m, l);
}

struct CombineArgs {
  const float* part_o;
  const float2* part_ml;
  float* out;
  int32_t H, n_parts, n_rows;  // n_rows = units * H
  int32_t n_wg;                // the merge's own workgroups; those after them run rp
  CarriedReplay rp;
};

// One wave per (unit, head) of partials stored row by row: the largest partial reference max M,
// the weights w_p = 2^(m_p - M), then out = sum_p w_p o_p / sum_p w_p l_p, over the parts in split
// order. Lane j holds the weight of part j of each group of 64 parts and DV / 64 output floats;
// eight parts' outputs are in flight at a time, the first eight while the weights are worked out
// (the call is all latency: parts and weights one after the other took 0.9 us more).
template <int DV>
__global__ __launch_bounds__(256) void attn_combine_kernel(CombineArgs a) {
  constexpr int E = DV / 64;  // output floats per lane
  typedef float vec __attribute__((ext_vector_type(E)));
  if ((int)blockIdx.x >= a.n_wg) {  // wave-uniform: the whole workgroup replays
    replay_worker(a.rp, (int)blockIdx.x - a.n_wg);
    return;
  }
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= a.n_rows) return;
  const int unit = row / a.H, h = row % a.H;
  const int np = a.n_parts;
  const int64_t pstride = (int64_t)a.H * DV;
  const float2* ml = a.part_ml + (int64_t)unit * np * a.H + h;
  const float* po = a.part_o + (int64_t)unit * np * pstride + (int64_t)h * DV + lane * E;

  const float2 ml0 = ml[(int64_t)min(lane, np - 1) * a.H];  // this lane's part of the first 64
  vec val[8];
#pragma unroll
  for (int u = 0; u < 8; ++u)
    val[u] = *reinterpret_cast<const vec*>(po + (int64_t)min(u, np - 1) * pstride);
  float M = lane < np ? ml0.x : -INFINITY;
  for (int pb = lane + 64; pb < np; pb += 64) M = fmaxf(M, ml[(int64_t)pb * a.H].x);
#pragma unroll
  for (int x = 32; x >= 1; x >>= 1) M = fmaxf(M, __shfl_xor(M, x, 64));

  vec acc = {};
  float lsum = 0.f;
  for (int pb = 0; pb < np; pb += 64) {
    float w = 0.f;
    if (pb + lane < np) {
      float2 v = ml0;
      if (pb > 0) v = ml[(int64_t)(pb + lane) * a.H];
      w = v.x == -INFINITY ? 0.f : exp2f(v.x - M);
      lsum += w * v.y;
    }
    const int n = min(64, np - pb);
    for (int i = 0; i < n; i += 8) {
      if (pb + i > 0) {
#pragma unroll
        for (int u = 0; u < 8; ++u)
          val[u] = *reinterpret_cast<const vec*>(
              po + (int64_t)(pb + min(i + u, n - 1)) * pstride);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (i + u < n) {
          const float wu = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), i + u));
          acc += wu * val[u];
        }
      }
    }
  }
#pragma unroll
  for (int x = 32; x >= 1; x >>= 1) lsum += __shfl_xor(lsum, x, 64);
  const float inv = lsum > 0.f ? 1.f / lsum : 0.f;
  *reinterpret_cast<vec*>(a.out + (int64_t)row * DV + lane * E) = acc * inv;
}

struct CombineMlaArgs {
  const float* part_o;    // [units][n_parts][Hp * 512], block layout
  const float2* part_ml;  // [units][n_parts][H]
  float* out;             // [units][H][512]
  int32_t H, Hp, n_parts;
  int32_t n_wg;           // the merge's own workgroups; those after them run rp
  CarriedReplay rp;
};

// Merge of latent-attention partials: one workgroup per (unit, 32-head block, 256 / NS of the
// block's 4096 16-byte groups). Weights w_ph = 2^(m_ph - M_h) and L_h = sum_p w_ph l_ph first
// (in LDS); then thread (slice s, group g) sums parts p = s, s + NS, ... of group g, and the NS
// slice sums are added in slice order (NS > 1 puts more loads in flight when units are few).
template <int NS>
__global__ __launch_bounds__(256) void attn_combine_mla_kernel(CombineMlaArgs a) {
  constexpr int DV = 512, BLK4 = 32 * DV / 4, GPW = 256 / NS;
  __shared__ __align__(16) float s_w[kMlaMaxParts][32];
  __shared__ float s_inv[32];
  __shared__ __align__(16) f32x4 s_acc[NS][GPW];
  if ((int)blockIdx.x >= a.n_wg) {  // wave-uniform: the whole workgroup replays
    replay_worker(a.rp, (int)blockIdx.x - a.n_wg);
    return;
  }
  constexpr int chunks = BLK4 / GPW;
  const int nb = a.Hp >> 5;
  const int chunk = blockIdx.x % chunks;
  const int b = (blockIdx.x / chunks) % nb;
  const int unit = blockIdx.x / (chunks * nb);
  const int t = threadIdx.x, hl = t >> 3, sub = t & 7;
  const int head = b * 32 + hl;
  const int np = a.n_parts;
  const float2* ml = a.part_ml + (int64_t)unit * np * a.H;
  float M = -INFINITY;
  if (head < a.H)
    for (int p = sub; p < np; p += 8) M = fmaxf(M, ml[(int64_t)p * a.H + head].x);
#pragma unroll
  for (int x = 1; x < 8; x <<= 1) M = fmaxf(M, __shfl_xor(M, x, 64));
  float lsum = 0.f;
  for (int p = sub; p < np; p += 8) {
    float w = 0.f;
    if (head < a.H) {
      const float2 v = ml[(int64_t)p * a.H + head];
      w = v.x == -INFINITY ? 0.f : exp2f(v.x - M);
      lsum += w * v.y;
    }
    s_w[p][hl] = w;
  }
#pragma unroll
  for (int x = 1; x < 8; x <<= 1) lsum += __shfl_xor(lsum, x, 64);
  if (sub == 0) s_inv[hl] = lsum > 0.f ? 1.f / lsum : 0.f;
  __syncthreads();

  const int g = t % GPW, sl = t / GPW;
  const int f = chunk * GPW + g;  // 16-byte group within the block
  const int ln = f & 63, q = (f >> 6) & 3, n = f >> 8;
  const int h0 = 8 * q + 4 * (ln >> 5);  // first of the group's four heads (block-local)
  const int64_t pstride = (int64_t)a.Hp * DV;
  const float* pb = a.part_o + (int64_t)unit * np * pstride + (int64_t)b * 32 * DV + 4 * f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  int p = b * 32 + h0 < a.H ? sl : np;  // a group of heads past H is neither stored nor read
  for (; p + 3 * NS < np; p += 4 * NS) {
    f32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const f32x4*>(pb + (p + u * NS) * pstride);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      acc += *reinterpret_cast<const f32x4*>(&s_w[p + u * NS][h0]) * v[u];
  }
  for (; p < np; p += NS)
    acc += *reinterpret_cast<const f32x4*>(&s_w[p][h0]) * *reinterpret_cast<const f32x4*>(pb + p * pstride);
  s_acc[sl][g] = acc;
  __syncthreads();
  if (sl == 0) {
    f32x4 r = s_acc[0][g];
#pragma unroll
    for (int s2 = 1; s2 < NS; ++s2) r += s_acc[s2][g];
    const int dim = 32 * n + (ln & 31);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int h = b * 32 + h0 + e;
      if (h < a.H) a.out[((int64_t)unit * a.H + h) * DV + dim] = r[e] * s_inv[h0 + e];
    }
  }
}

// The extra workgroups of a launch that carries a replay: about `threads` threads spread over
// the replay's (unit, layer) pairs, in workgroups of the launch's size `bd`, at most `cap`
// workgroups (at least one per pair). False if the grid would be too large.
bool carried_replay(const FetchArgs& f, int bd, int64_t cap, int32_t threads, int32_t block_bytes,
                    CarriedReplay* r) {
  const int64_t pairs = (int64_t)f.units * f.n_layers;
  int64_t per_pair = std::max<int64_t>(1, threads / (bd * pairs));
  per_pair = std::max<int64_t>(1, std::min(per_pair, cap / pairs));
  if (pairs * per_pair > (1 << 20)) return false;
  r->pf = f;
  r->pf_div = make_fastdiv((uint32_t)(f.R / 16));
  r->pf_per_pair = (int32_t)per_pair;
  r->pf_wg = (int32_t)(pairs * per_pair);
  r->pf_u = std::max(1, block_bytes / 16);
  return true;
}

template <int DQK, int DV, int VOFF, int HW, int TW, int NST>
void launch_partial(const AttnArgs& args, hipStream_t stream) {
  const int nwg_pad = (args.n_wg + 7) & ~7;
  hipLaunchKernelGGL((attn_partial_kernel<DQK, DV, VOFF, HW, TW, NST>), dim3(nwg_pad + args.rp.pf_wg),
                     dim3(64 * HW * TW), 0, stream, args);
}

template <int HW, bool PACED = false, bool DIRECT = false, bool ANYQ = false>
void launch_mla(const AttnArgs& args, hipStream_t stream) {
  const int nwg_pad = (args.n_wg + 7) & ~7;
  hipLaunchKernelGGL((attn_mla_kernel<HW, PACED, DIRECT, ANYQ>), dim3(nwg_pad + args.rp.pf_wg),
                     dim3(128 * HW), 0, stream, args);
}

bool is_mla(const hisparse_attn_desc_t& d) {
  return d.d_qk == 576 && d.d_v == 512 && d.v_offset == 0;
}

// Bytes of `parts` partial results: h_store rows of outputs each, then (max, sum) of H heads.
size_t partials_bytes(size_t parts, int h_store, int H, int d_v) {
  const size_t o_bytes = parts * h_store * d_v * sizeof(float);
  return ((o_bytes + 255) & ~(size_t)255) + parts * H * sizeof(float2);
}

}  // namespace

hisparse_status_t plan_attention(int32_t units, int32_t top_k, int32_t record_bytes,
                                 const hisparse_attn_desc_t* attn, AttnPlan* plan) {
  if (!attn || !plan) return HISPARSE_ERR_INVALID_ARG;
  const hisparse_status_t st = hisparse_validate_attn(record_bytes, top_k, attn);
  if (st != HISPARSE_OK) return st;
  if (units <= 0 || (int64_t)units * 256 > (1LL << 30)) return HISPARSE_ERR_INVALID_ARG;
  const int H = attn->q_heads;
  AttnPlan p{};
  p.n_tok = top_k * attn->tokens_per_record;
  if (is_mla(*attn)) {
    // 32 heads per wave, 1 head wave up to 32 heads, 2 (64 heads) above, and two token groups: the
    // groups share a split's chunks in turn and a partial result covers both, so the split
    // partials (fp32, 2 KB per head) are half of what one group's workgroups would write. With
    // HISPARSE_ATTN_BESIDE_FETCH (another stream's host-link fetch shares the GPU) the same
    // shapes take half as many workgroups (below): the other half of the CUs is left to the
    // fetch's waves.
    // At most 128 tokens, the grouped-query kernel's shape: 16 heads per workgroup, four waves on a
    // chunk each, merged in the workgroup, no merge launch. One round is all it does well: its
    // tiles leave no room for the next chunk (16 heads, 256 tokens 12.2 us against 11.5 in four
    // splits, 64 units x 2048 tokens 44.9 against 40.8). Up to 224 workgroups it takes 9.2 to 10.4
    // us for any number of heads, the tiled kernel 9.7 to 21.6 (1 unit of 128 heads x 128 tokens 9.2
    // against 11.8, 24 units 10.2 against 19.8). Past a CU each its workgroups, which hold a CU's LDS
    // each for 16 heads, queue: 48 units of 128 heads x 64 tokens 19.3 against 13.7. And a replay that
    // the launch carries needs a CU per unit besides: share groups of 28 units of 128 heads x 64
    // tokens take 66 us against 76 with 32 CUs left, 32 units 95 against 79 with none. With up to 16
    // heads the tiled kernel has as many workgroups (300 units x 96 tokens 20.1 against 24.3).
    const int head_blocks = (H + 15) / 16;
    p.rows = p.n_tok <= 4 * kChunk &&
             (H <= 16 || (int64_t)units * (head_blocks + 1) <= kTargetWorkgroups);
    p.hw = H <= 32 || p.rows ? 1 : 2;
    p.tg = p.rows ? 1 : 2;
    p.tw = p.rows ? 4 : 1;
    p.hb = p.rows ? head_blocks : (H + 32 * p.hw - 1) / (32 * p.hw);
  } else {              // up to 64 heads per workgroup, 16 per wave
    p.hw = H > 32 ? 4 : (H > 16 ? 2 : 1);
    p.tw = 4 / p.hw;
    p.tg = 1;
    p.rows = true;
    p.hb = (H + 16 * p.hw - 1) / (16 * p.hw);
  }
  // a split is a whole number of the workgroup's chunk rounds
  const int chunk = kChunk * p.tg * p.tw;
  const int max_splits = (p.n_tok + chunk - 1) / chunk;
  // Beside another stream's host-link fetch, latent attention aims at half a workgroup per CU:
  // the fetch's waves, whose slow host reads occupy the memory pipelines of the CUs they run
  // on, then find CUs without an attention workgroup. Inside the two-micro-batch decode step
  // (16 units of 128 heads, 2 token groups, 4 splits) that fetch moves 51.9 GB/s against 50.6
  // with a workgroup per CU, the step 1.692 against 1.735 ms, and the split partials halve;
  // the attention itself takes 58 against 40 us, hidden behind the other micro-batch's fetch.
  // So does a latent call of one head wave that carries a replay, which then runs on the other half
  // (share groups of four layers, 16 units of 32 heads x 1024 tokens: 200 us against 232).
  const bool half_grid =
      is_mla(*attn) && ((attn->flags & HISPARSE_ATTN_BESIDE_FETCH) ||
                        (p.hw == 1 && (attn->flags & HISPARSE_ATTN_CARRIES_REPLAY)));
  const int target = half_grid ? kTargetWorkgroups / 2 : kTargetWorkgroups;
  // Beside another stream's fetch and with more than 16 workgroup columns (more than 8 units of
  // 128 heads, two token groups) the call hides behind the other micro-batch's longer fetch,
  // whose host reads then set the step; there every workgroup loading its query together with
  // its first chunks slows those reads, and the paced kernel loads the query after them. The
  // two-micro-batch decode step at 20, 24, 28, 32 and 64 requests took 1.247, 1.450, 1.730,
  // 1.82 and 3.43 ms unpaced against 1.241, 1.371, 1.519, 1.69 and 3.23 ms paced. At 16 columns
  // and below the chain of attention, merge and resolve is the longer one and the unpaced start
  // wins (16 requests: 1.005 against 1.052 ms; 8 requests: 0.711 against 0.724).
  p.paced = is_mla(*attn) && (attn->flags & HISPARSE_ATTN_BESIDE_FETCH) && p.hw == 2 &&
            (int64_t)units * p.hb > 16;
  int splits;
  if (attn->num_splits > 0) {
    splits = std::min(attn->num_splits, max_splits);
  } else {
    // at most one workgroup per CU (a workgroup holds a CU's LDS, so one more would wait for a
    // second round), and enough chunks per split for the load pipeline to reach steady state.
    const int per_split = units * p.hb;
    splits = std::max(1, target / per_split);
    // A round is one chunk per token group. Latent attention: the split partials and the merge
    // grow with the splits: one round per split up to 4 workgroup columns and from 16 on (where
    // the grid limits the splits anyway), two between unless there are at most four in all (8 units
    // of 32 heads x 192 tokens: 12.1 us in three splits, 16.3 in one). Grouped-query, four token
    // groups: two rounds of 128 tokens per split; a round takes about 1 us, and 4 units x 4096 tokens
    // take 10.9 us in 16 splits (two rounds each) against 11.8 in 8, 16 units x 2048 tokens 10.8 in 8
    // against 12.4 in 4. With fewer token groups, whose rounds are shorter, four (8 units of 32 heads
    // x 4096 tokens: 12.4 us in 16 splits, 12.5 in 32).
    // Beside another stream's host-link fetch, six: fewer workgroups leave its waves their CUs (two
    // micro-batches of 32 units x 16 heads x 1536 tokens: decode step 1.587 ms with four rounds,
    // 1.552 with six, 1.561 with twelve; of 32 x 4 x 4096: 6.107, 6.105, 6.128).
    const bool beside = attn->flags & HISPARSE_ATTN_BESIDE_FETCH;
    int split_rounds = is_mla(*attn) ? 1 : (beside ? 6 : (p.tw == 4 ? 2 : 4));
    // A carried replay runs on the CUs the attention leaves; a grouped-query call that would leave
    // fewer than a quarter takes four rounds too (share groups of four layers, 32 units of 4 heads x
    // 2048 tokens in pages of 16: 357 us with a workgroup on every CU, 304 on half of them).
    if (!is_mla(*attn) && (attn->flags & HISPARSE_ATTN_CARRIES_REPLAY) &&
        per_split * std::min(splits, p.n_tok / (split_rounds * chunk)) > kTargetWorkgroups * 3 / 4)
      split_rounds = std::max(split_rounds, 4);
    const int rounds = (p.n_tok + chunk - 1) / chunk;
    const bool few_columns = is_mla(*attn) && per_split < 16;
    if (few_columns && per_split > 4 && rounds > 4) split_rounds = 2;
    // A call that carries a replay lasts as long as the replay's host reads; its attention only
    // has to finish within them, and the merge after it is on the decode chain. One request of
    // 128 heads with a replay of its 2048 selections into the next shared layer: 16 four-chunk
    // splits instead of 32 two-chunk ones take the launch from 28.0 to 27.4 us and its merge
    // from 5.8 to 4.6 us (one 1M-token request, 56 layers in groups of 4: decode step 2.299 ->
    // 2.226 ms), although that attention alone takes longer. Not where the replay is short: share
    // groups of four layers, 1 unit of 128 heads x 1999 tokens 95.3 us with the hint, 90.0 without, 3
    // x 64 x 610 84.1 and 79.9; but 2 x 64 x 1480 95.7 and 99.5.
    if (few_columns && rounds > 4 && (int64_t)units * p.n_tok >= 2048 &&
        (attn->flags & HISPARSE_ATTN_CARRIES_REPLAY))
      split_rounds = 2;
    // Whole splits of that many rounds at least. A short call takes one more for what is left over
    // instead of longer ones (5 units of 32 heads x 320 tokens, two rounds per split: 14.0 us in
    // three, 16.1 in two of three rounds); in longer calls, and in those that fill the grid, it is
    // not worth its partials (4 units of 64 heads x 900 tokens: 15.8 us in 8 splits, 17.4 in 15).
    const int min_work_splits = few_columns && rounds <= 8
                                    ? (rounds + split_rounds - 1) / split_rounds
                                    : std::max(1, p.n_tok / (split_rounds * chunk));
    splits = std::max(1, std::min({splits, max_splits, min_work_splits}));
    // A grouped-query unit of one split needs no merge, a launch of its own that costs about 2.5
    // us, against about 1 us for a round: 11 units x 501 tokens, four rounds, take 8.7 us in one
    // split against 10.8 in two to four. (A latent round is longer: one request of 33 heads over
    // 150 tokens takes 11.7 us in three splits of one round and a merge, 13.9 in one of three.)
    if (!is_mla(*attn) && max_splits <= 5) splits = 1;
  }
  // Splits asked for by number hold 1024 records at most as long as there is a CU for each of the
  // workgroups that makes: shorter ones are faster there (16 units of 64 heads x 4096 tokens, one
  // split asked for: 42.4 us in four, 69.7 in two), not beyond (48 units of 128 heads x 4096 tokens,
  // two asked for: 88.5 us in two, 105.7 in four).
  const int64_t short_wgs = (int64_t)units * p.hb * ((top_k + kMaxSplitRecords / 2 - 1) /
                                                     (kMaxSplitRecords / 2));
  const int max_split_records = attn->num_splits > 0 && short_wgs <= kTargetWorkgroups
                                    ? kMaxSplitRecords / 2 : kMaxSplitRecords;
  const int max_split_tokens = std::min(max_split_records * attn->tokens_per_record, kMaxSplitTokens);
  splits = std::max(splits, (p.n_tok + max_split_tokens - 1) / max_split_tokens);
  if (is_mla(*attn)) splits = std::min(splits, kMlaMaxParts);  // the merge keeps weights in LDS
  const int per = (p.n_tok + splits - 1) / splits;
  p.split_tokens = (per + chunk - 1) / chunk * chunk;
  if (p.split_tokens > max_split_tokens) p.split_tokens = max_split_tokens / chunk * chunk;
  p.n_wg_splits = (p.n_tok + p.split_tokens - 1) / p.split_tokens;
  p.n_parts = p.n_wg_splits;
  // the latent-attention merge holds one weight per part in LDS (hisparse_validate_attn keeps the
  // token count within reach of that limit)
  if (is_mla(*attn) && p.n_parts > kMlaMaxParts) return HISPARSE_ERR_UNSUPPORTED;
  const int64_t n_wg = (int64_t)units * p.n_wg_splits * p.hb;
  if (n_wg > (1LL << 30)) return HISPARSE_ERR_INVALID_ARG;
  p.workspace_bytes = partials_bytes((size_t)units * p.n_parts,
                                     is_mla(*attn) ? (H + 31) / 32 * 32 : H, H, attn->d_v);
  *plan = p;
  return HISPARSE_OK;
}

// A size for the call that also serves the smaller ones a caller makes with it. The plan's own need
// is no such size: it falls where a unit becomes one split (64 units of 128 heads x 2048 tokens take
// 128 parts, 96 take 96), and a hint lowers it.
//  - every smaller number of units; above one workgroup column per CU a unit takes the fewest splits
//    there are, so the needs to look at are those up to that many units and the call's own;
//  - the needs without a hint, for the numbers of units up to the last one whose plan it leaves
//    alone; for all of them unless the call is one it is made for: latent, more than 32 heads, at
//    least 64 one-round workgroups. Where it does lower the need, a part per 1024 records of each
//    unit still covers smaller calls without it.
// Calls are checked against their own need, never against this.
size_t attention_workspace_bytes(int32_t units, int32_t top_k, int32_t record_bytes,
                                 const hisparse_attn_desc_t* attn) {
  AttnPlan p{}, bare{};
  if (plan_attention(units, top_k, record_bytes, attn, &p) != HISPARSE_OK) return 0;
  hisparse_attn_desc_t plain = *attn;
  plain.flags &= ~(HISPARSE_ATTN_BESIDE_FETCH | HISPARSE_ATTN_CARRIES_REPLAY);
  const int H = attn->q_heads;
  const int record_tokens = std::min(1024 * attn->tokens_per_record, kMaxSplitTokens);
  const size_t record_parts = (size_t)((p.n_tok + record_tokens - 1) / record_tokens);
  const int32_t columns = kTargetWorkgroups / p.hb;
  size_t bytes = 0;
  bool without_hint = false;
  for (int32_t u = units; u >= 1; u = std::min(u - 1, columns)) {
    if (plan_attention(u, top_k, record_bytes, attn, &p) != HISPARSE_OK) continue;
    bare = p;
    if (plain.flags != attn->flags &&
        plan_attention(u, top_k, record_bytes, &plain, &bare) != HISPARSE_OK)
      continue;
    const bool hinted = is_mla(*attn) && H > 32 && p.n_parts != bare.n_parts &&
                        (int64_t)u * p.hb * (p.n_tok / (2 * kChunk)) >= 64;
    without_hint = without_hint || !hinted;
    bytes = std::max(bytes, p.workspace_bytes);
    if (without_hint) bytes = std::max(bytes, bare.workspace_bytes);
    if (hinted)
      bytes = std::max(bytes, partials_bytes(u * record_parts, (H + 31) / 32 * 32, H, attn->d_v));
  }
  return bytes;
}

hipError_t launch_attention(const AttnPlan& p, const hisparse_attn_desc_t& attn,
                            const uint8_t* pool, int64_t records_per_unit, int32_t record_bytes,
                            int32_t units, int32_t top_k, const uint16_t* q, const int32_t* idx,
                            float* out, void* workspace, hipStream_t stream,
                            int32_t idx_units, const FetchArgs* prefetch,
                            int32_t prefetch_threads, int32_t prefetch_block_bytes) {
  AttnArgs a{};
  if (prefetch && prefetch->units > 0 && prefetch->n_layers > 0) {
    // on the CUs the attention leaves idle (a workgroup of these kernels holds a CU's LDS, so
    // replay and attention never share a CU's memory pipeline); with few or none, as many workgroups
    // as the threads asked for make, which follow the attention's
    const int64_t n_attn = (int64_t)units * p.n_wg_splits * p.hb;
    const int64_t idle = std::max<int64_t>(0, kTargetWorkgroups - ((n_attn + 7) & ~7LL));
    if (!carried_replay(*prefetch, 64 * p.hw * p.tg * p.tw,
                        idle >= kMinIdle ? idle : kTargetWorkgroups, prefetch_threads,
                        prefetch_block_bytes, &a.rp))
      return hipErrorInvalidValue;
  }
  a.idx_units = idx_units > 0 ? idx_units : units;
  a.pool = pool;
  a.q = q;
  a.idx = idx;
  a.Hp = p.rows ? attn.q_heads : (attn.q_heads + 31) / 32 * 32;
  const size_t o_bytes = (size_t)units * p.n_parts * a.Hp * attn.d_v * sizeof(float);
  a.part_o = reinterpret_cast<float*>(workspace);
  a.part_ml = reinterpret_cast<float2*>(reinterpret_cast<uint8_t*>(workspace) +
                                        ((o_bytes + 255) & ~(size_t)255));
  a.rec_per_unit = records_per_unit;
  a.R = record_bytes;
  a.token_bytes = record_bytes / attn.tokens_per_record;
  int shift = 0;
  while ((1 << shift) < attn.tokens_per_record) ++shift;
  a.tpr_shift = shift;
  a.k = top_k;
  a.H = attn.q_heads;
  a.n_tok = p.n_tok;
  a.split_tokens = p.split_tokens;
  a.n_wg_splits = p.n_wg_splits;
  a.hb = p.hb;
  a.n_parts = p.n_parts;
  a.n_wg = units * p.n_wg_splits * p.hb;
  a.div_hb = make_fastdiv((uint32_t)p.hb);
  a.div_splits = make_fastdiv((uint32_t)p.n_wg_splits);
  a.div_idx = make_fastdiv((uint32_t)a.idx_units);
  a.scale_log2 = attn.scale * 1.4426950408889634f;

  // a unit that is one part needs no merge: the kernel writes the output itself
  const bool direct = p.n_parts == 1 && !(attn.flags & HISPARSE_ATTN_DEFER_MERGE);
  a.direct = direct;
  a.out = out;
  if (is_mla(attn) && p.rows) {
    if (p.split_tokens > 4 * kChunk) return hipErrorInvalidValue;  // the plan's: one round
    launch_partial<576, 512, 0, 1, 4, 1>(a, stream);
  } else if (is_mla(attn) && (reinterpret_cast<uintptr_t>(q) & 15) != 0) {
    // the same splits and bits, never paced
    if (p.hw == 1 && direct) launch_mla<1, false, true, true>(a, stream);
    else if (p.hw == 1) launch_mla<1, false, false, true>(a, stream);
    else if (direct) launch_mla<2, false, true, true>(a, stream);
    else launch_mla<2, false, false, true>(a, stream);
  } else if (is_mla(attn)) {
    if (p.hw == 1 && direct) launch_mla<1, false, true>(a, stream);
    else if (p.hw == 1) launch_mla<1>(a, stream);
    else if (p.paced && direct) launch_mla<2, true, true>(a, stream);
    else if (p.paced) launch_mla<2, true>(a, stream);
    else if (direct) launch_mla<2, false, true>(a, stream);
    else launch_mla<2>(a, stream);
  } else {
    switch (p.hw) {
      case 1: launch_partial<128, 128, 128, 1, 4, 2>(a, stream); break;
      case 2: launch_partial<128, 128, 128, 2, 2, 3>(a, stream); break;
      default: launch_partial<128, 128, 128, 4, 1, 4>(a, stream); break;
    }
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (direct || (attn.flags & HISPARSE_ATTN_DEFER_MERGE)) return hipSuccess;
  return launch_merge(p, attn, units, out, workspace, stream);
}

hipError_t launch_merge(const AttnPlan& p, const hisparse_attn_desc_t& attn, int32_t units,
                        float* out, const void* workspace, hipStream_t stream,
                        const FetchArgs* prefetch, int32_t prefetch_threads,
                        int32_t prefetch_block_bytes) {
  // the same workspace layout as launch_attention: partial outputs, then (max, sum) pairs
  const int Hp = p.rows ? attn.q_heads : (attn.q_heads + 31) / 32 * 32;
  const size_t o_bytes = (size_t)units * p.n_parts * Hp * attn.d_v * sizeof(float);
  const float* part_o = reinterpret_cast<const float*>(workspace);
  const float2* part_ml = reinterpret_cast<const float2*>(
      reinterpret_cast<const uint8_t*>(workspace) + ((o_bytes + 255) & ~(size_t)255));
  // a carried replay: merge workgroups are small (no CU's whole LDS), so the replay's
  // workgroups run beside them wherever there is room
  CarriedReplay rp{};
  if (prefetch && prefetch->units > 0 && prefetch->n_layers > 0 &&
      !carried_replay(*prefetch, 256, 1 << 20, prefetch_threads, prefetch_block_bytes, &rp))
    return hipErrorInvalidValue;
  if (!p.rows) {
    const int nb = Hp / 32;
    CombineMlaArgs c{part_o, part_ml, out, attn.q_heads, Hp, p.n_parts, 0, rp};
    if ((int64_t)units * nb * 16 >= 2 * kTargetWorkgroups) {
      c.n_wg = units * nb * 16;
      hipLaunchKernelGGL(attn_combine_mla_kernel<1>, dim3(c.n_wg + rp.pf_wg), dim3(256), 0,
                         stream, c);
    } else {
      c.n_wg = units * nb * 64;
      hipLaunchKernelGGL(attn_combine_mla_kernel<4>, dim3(c.n_wg + rp.pf_wg), dim3(256), 0,
                         stream, c);
    }
    return hipGetLastError();
  }
  CombineArgs c{part_o, part_ml, out, attn.q_heads, p.n_parts, units * attn.q_heads, 0, rp};
  c.n_wg = (units * attn.q_heads + 3) / 4;
  if (is_mla(attn))
    hipLaunchKernelGGL(attn_combine_kernel<512>, dim3(c.n_wg + rp.pf_wg), dim3(256), 0, stream, c);
  else
    hipLaunchKernelGGL(attn_combine_kernel<128>, dim3(c.n_wg + rp.pf_wg), dim3(256), 0, stream, c);
  return hipGetLastError();
}

}  // namespace hisparse

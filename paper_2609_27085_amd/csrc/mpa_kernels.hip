// HIP kernels for one mixed prefill+decode attention step on gfx950.
//
// Cache layout (X = 16 / element bytes):
//   K  [block][kv_head][d/X][16][X]   -- a 16-byte chunk of one key row is X
//                                       consecutive dims; the 16 slots of a
//                                       block sit side by side per chunk
//   V  [block][kv_head][d][16]         -- each dim row holds the block's 16
//                                       tokens contiguously
// With this layout both MFMA operands that come from the cache load as whole
// 512-1024 byte runs per wave instruction, in exactly the register layout the
// matrix cores want, with no shuffles:
//
//   S^T[key][row] = K[key][:] . Q^T[:][row]       (A = K chunks, B = Q chunks)
//   O^T[dim][row] = V^T[dim][key] . P^T[key][row] (A = V^T, B = P from S^T)
//
// In the 16x16 MFMA output a lane holds 4 consecutive rows of one column, so
// lane (n, g) of a wave owns query row n and keys 4g..4g+3 of each 16-key
// block; the softmax state of row n (running max, sum) is lane-local up to a
// 4-way reduction across the lane groups, and P^T is already in B-operand
// order for the PV product.
//
// Softmax runs in base 2: scores are scaled by scale*log2(e), exponentials are
// v_exp_f32, and log-sum-exp values are returned in natural log units.

#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>

#include "mpa_internal.h"

namespace mpa {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// acc + the two bf16 values packed in w (one v_dot2 against (1, 1)); the
// products are exact and the sum is taken in f32
__device__ inline float add_bf16_pair(unsigned w, float acc) {
  const bf16x2 one = {(__bf16)1.0f, (__bf16)1.0f};
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w), one, acc, false);
}

constexpr float kLn2 = 0.69314718055994530942f;

__device__ inline int wave_uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ inline float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

// max(x[lane], x[lane ^ 32]) with one VALU lane swap (no LDS round trip, so
// no wait on outstanding LDS reads)
__device__ inline float max_across_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

__device__ inline short bf16_bits(float x) { return __builtin_bit_cast(short, (__bf16)x); }

// s_waitcnt immediate that waits until at most n vector-memory operations are
// outstanding (expcnt and lgkmcnt left at their maxima).  Used through the
// intrinsic, which the compiler's own wait-count tracking understands.
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }
#define MPA_WAIT_VMCNT(n)                          \
  do {                                             \
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(n));      \
    asm volatile("" ::: "memory");                 \
  } while (0)
// The same for the LDS / scalar-memory counter (vmcnt and expcnt left at
// their maxima).
constexpr int lgkmcnt_imm(int n) { return 15 | (7 << 4) | ((n & 15) << 8) | (3 << 14); }
#define MPA_WAIT_LGKMCNT(n)                        \
  do {                                             \
    __builtin_amdgcn_s_waitcnt(lgkmcnt_imm(n));    \
    asm volatile("" ::: "memory");                 \
  } while (0)

// 16 bytes per lane from global memory straight into LDS: lane l reads the
// 16 bytes at base + voff (base uniform, held in SGPRs; voff the lane's byte
// offset) and they land at lds + 16*l (lds the same for the whole wave).
// With the base in SGPRs the per-lane offsets are loop invariant, so a copy
// needs no per-copy address arithmetic in VGPRs (whose reuse would make each
// copy wait for the previous one to be sent).  Issued as inline assembly so
// that the compiler does not make every later LDS read wait for it (it cannot
// tell that the read targets another buffer); the caller waits with an
// explicit vector-memory wait before the barrier that publishes the tile.  M0
// is written only here in this file.
__device__ inline void global_to_lds16(const void* base, unsigned voff, void* lds) {
  const unsigned off = (unsigned)(size_t)(__attribute__((address_space(3))) void*)lds;
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "s"(off) : "memory");
}
// The same copy as a non-temporal (streaming) load, for data read once.
__device__ inline void global_to_lds16_nt(const void* base, unsigned voff, void* lds) {
  const unsigned off = (unsigned)(size_t)(__attribute__((address_space(3))) void*)lds;
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(voff), "s"(base), "s"(off) : "memory");
}

// Cache reads on the decode path take non-temporal loads: a decode step
// reads each (block, KV head) granule of K and V once, and marking the loads
// as streaming lifts the sustained read rate of scattered 4 KB granules on
// gfx950 by about a tenth over plain loads (the same holds for contiguous
// streams).
template <typename V>
__device__ inline V ld_stream(const void* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const V*>(p));
}

// New tokens are written with non-temporal stores beside a decode step whose
// rows stream as ranges: a token's K is D / 8 pieces of 16 bytes and its
// transposed V D single elements 16 apart, so every line they touch is written
// in part, and such lines left dirty in the L2 slow the streaming reads that
// evict them.  Decode with its tokens, 128 rows of 8 heads: 424 us with plain
// stores, 403 with these, 392 with none; 256 rows 1,242 / 1,205 / 1,190; fp8
// 264 / 253 / 247.  Rows that are split on their own or not at all take plain
// stores: there a wave waits for its token before its first block, a larger
// part of its time, and a plain store is complete in the L2 (32 / 8 heads,
// non-temporal -> plain: 32 rows of 900 23.0 -> 21.0 us, 256 of 600 137.1 ->
// 132.9, fp8 79.2 -> 75.0, 16 of 4,096 31.8 -> 31.0; 128 of 1,500, two rounds
// of waves, 142.1 -> 144.8).
template <typename V>
__device__ inline void st_stream(void* p, V v) {
  __builtin_nontemporal_store(v, reinterpret_cast<V*>(p));
}
template <bool NT, typename V>
__device__ inline void st_token(void* p, V v) {
  if constexpr (NT)
    st_stream(p, v);
  else
    *reinterpret_cast<V*>(p) = v;
}

// ---------------------------------------------------------------------------
// Element-type traits.  A "round" of the QK^T product consumes one 16-byte
// chunk of K and of Q per lane: one 16x16x32 bf16 MFMA, or four 16x16x4 f32
// MFMAs.  The PV product consumes 4 tokens of one V^T row per lane: one
// 16x16x16 bf16 MFMA, or four 16x16x4 f32 MFMAs.
template <int DT>
struct Tr;

template <>
struct Tr<0> {  // bf16
  using Elem = uint16_t;   // cache element
  using QElem = uint16_t;  // queries, new rows and outputs
  static constexpr int X = 8;
  using Chunk = bf16x8;
  using VFrag = s16x4;
  using PFrag = s16x4;
  static __device__ inline Chunk load_chunk(const Elem* p) { return __builtin_bit_cast(Chunk, ld_stream<u32x4>(p)); }
  static __device__ inline Chunk load_q(const QElem* p) { return load_chunk(p); }
  static __device__ inline Chunk zero_chunk() {
    u32x4 z = {0u, 0u, 0u, 0u};
    return __builtin_bit_cast(Chunk, z);
  }
  static __device__ inline f32x4 qk(Chunk k, Chunk q, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(k, q, c, 0, 0, 0);
  }
  static __device__ inline VFrag load_v(const Elem* p) { return __builtin_bit_cast(VFrag, ld_stream<u32x2>(p)); }
  static __device__ inline VFrag keep_first(VFrag v, int nvalid) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = e < nvalid ? v[e] : (short)0;
    return v;
  }
  static constexpr bool kRoundsP = true;  // the PV product takes P in bf16
  static __device__ inline PFrag make_p(f32x4 p) {
    PFrag r;
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = bf16_bits(p[e]);
    return r;
  }
  // p - hi rounded to bf16: hi + lo carries p to about 16 significant bits
  static __device__ inline PFrag make_p_lo(f32x4 p, PFrag hi) {
    PFrag r;
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = bf16_bits(p[e] - __uint_as_float((unsigned)(uint16_t)hi[e] << 16));
    return r;
  }
  static __device__ inline f32x4 pv(VFrag v, PFrag p, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(v, p, c, 0, 0, 0);
  }
  // acc + the probabilities exactly as the PV product consumes them (after
  // rounding to bf16), so that the softmax denominator matches the numerator
  static __device__ inline float psum(f32x4, PFrag pf, float acc) {
    const u32x2 w = __builtin_bit_cast(u32x2, pf);
    return add_bf16_pair(w[1], add_bf16_pair(w[0], acc));
  }
  static __device__ inline void store4(Elem* dst, f32x4 v) {
    s16x4 r;
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = bf16_bits(v[e]);
    *reinterpret_cast<u32x2*>(dst) = __builtin_bit_cast(u32x2, r);
  }
  static __device__ inline void store1(Elem* dst, float v) { *dst = (uint16_t)bf16_bits(v); }
  static __device__ inline void unpack(u32x4 w, float (&f)[X]) {
#pragma unroll
    for (int e = 0; e < X; ++e) f[e] = __uint_as_float(((w[e / 2] >> (16 * (e & 1))) & 0xFFFFu) << 16);
  }
  static __device__ inline u32x4 pack(const float (&f)[X]) {
    u32x4 w;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      w[i] = (unsigned)(uint16_t)bf16_bits(f[2 * i]) | ((unsigned)(uint16_t)bf16_bits(f[2 * i + 1]) << 16);
    return w;
  }
};

template <>
struct Tr<1> {  // f32
  using Elem = float;
  using QElem = float;
  static constexpr int X = 4;
  using Chunk = f32x4;
  using VFrag = f32x4;
  using PFrag = f32x4;
  static __device__ inline Chunk load_chunk(const Elem* p) { return ld_stream<f32x4>(p); }
  static __device__ inline Chunk load_q(const QElem* p) { return load_chunk(p); }
  static __device__ inline Chunk zero_chunk() { return f32x4{0.f, 0.f, 0.f, 0.f}; }
  static __device__ inline f32x4 qk(Chunk k, Chunk q, f32x4 c) {
#pragma unroll
    for (int j = 0; j < 4; ++j) c = __builtin_amdgcn_mfma_f32_16x16x4f32(k[j], q[j], c, 0, 0, 0);
    return c;
  }
  static __device__ inline VFrag load_v(const Elem* p) { return ld_stream<f32x4>(p); }
  static __device__ inline VFrag keep_first(VFrag v, int nvalid) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = e < nvalid ? v[e] : 0.f;
    return v;
  }
  static constexpr bool kRoundsP = false;
  static __device__ inline PFrag make_p(f32x4 p) { return p; }
  static __device__ inline PFrag make_p_lo(f32x4, PFrag) { return f32x4{0.f, 0.f, 0.f, 0.f}; }
  static __device__ inline float psum(f32x4 p, PFrag, float acc) { return acc + ((p[0] + p[1]) + (p[2] + p[3])); }
  static __device__ inline f32x4 pv(VFrag v, PFrag p, f32x4 c) {
#pragma unroll
    for (int j = 0; j < 4; ++j) c = __builtin_amdgcn_mfma_f32_16x16x4f32(v[j], p[j], c, 0, 0, 0);
    return c;
  }
  static __device__ inline void store4(Elem* dst, f32x4 v) { *reinterpret_cast<f32x4*>(dst) = v; }
  static __device__ inline void store1(Elem* dst, float v) { *dst = v; }
  static __device__ inline void unpack(u32x4 w, float (&f)[X]) {
#pragma unroll
    for (int e = 0; e < X; ++e) f[e] = __uint_as_float(w[e]);
  }
  static __device__ inline u32x4 pack(const float (&f)[X]) {
    u32x4 w;
#pragma unroll
    for (int e = 0; e < X; ++e) w[e] = __float_as_uint(f[e]);
    return w;
  }
};

// fp8 caches (OCP E4M3 codes) beside bf16 queries, new rows and outputs.
// Codes become bf16 on load (exact: every E4M3 value is a bf16 value) and
// the arithmetic is the bf16 path's; the tensors' scales are applied outside
// (key scale in the softmax scale, value scale on the outputs).
template <>
struct Tr<2> {
  using Elem = uint8_t;
  using QElem = uint16_t;
  static constexpr int X = 8;  // codes per K chunk: 8 bytes
  using Chunk = bf16x8;
  using VFrag = s16x4;
  using PFrag = s16x4;
  static constexpr bool kRoundsP = true;
  static __device__ inline unsigned cvt2(unsigned w, bool hi) {
    return hi ? __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)w, 1.0f, true))
              : __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)w, 1.0f, false));
  }
  static __device__ inline Chunk k_from_codes(u32x2 w) {
    const u32x4 r = {cvt2(w[0], false), cvt2(w[0], true), cvt2(w[1], false), cvt2(w[1], true)};
    return __builtin_bit_cast(Chunk, r);
  }
  static __device__ inline VFrag v_from_codes(unsigned w) {
    const u32x2 r = {cvt2(w, false), cvt2(w, true)};
    return __builtin_bit_cast(VFrag, r);
  }
  static __device__ inline Chunk load_chunk(const Elem* p) { return k_from_codes(ld_stream<u32x2>(p)); }
  static __device__ inline Chunk load_q(const QElem* p) { return Tr<0>::load_q(p); }
  static __device__ inline Chunk zero_chunk() { return Tr<0>::zero_chunk(); }
  static __device__ inline f32x4 qk(Chunk k, Chunk q, f32x4 c) { return Tr<0>::qk(k, q, c); }
  static __device__ inline VFrag load_v(const Elem* p) { return v_from_codes(ld_stream<unsigned>(p)); }
  static __device__ inline VFrag keep_first(VFrag v, int nvalid) { return Tr<0>::keep_first(v, nvalid); }
  static __device__ inline PFrag make_p(f32x4 p) { return Tr<0>::make_p(p); }
  static __device__ inline PFrag make_p_lo(f32x4 p, PFrag hi) { return Tr<0>::make_p_lo(p, hi); }
  static __device__ inline f32x4 pv(VFrag v, PFrag p, f32x4 c) { return Tr<0>::pv(v, p, c); }
  static __device__ inline float psum(f32x4 p, PFrag pf, float acc) { return Tr<0>::psum(p, pf, acc); }
  static __device__ inline void store4(QElem* dst, f32x4 v) { Tr<0>::store4(dst, v); }
  static __device__ inline void store1(QElem* dst, float v) { Tr<0>::store1(dst, v); }
};

// float32 -> OCP E4M3 code: round to nearest, ties to the even mantissa;
// magnitudes past the largest finite value, 448, saturate to it; NaN -> the
// NaN code; the sign is kept.  One conversion instruction after a clamp: the
// same steps on the bits, with their branches, took a wave that appends a
// block (64 conversions a lane) 13 us more.
__device__ inline unsigned f32_to_e4m3(float x) {
  const float c = __builtin_amdgcn_fmed3f(x, -448.f, 448.f);
  const unsigned code = (unsigned)__builtin_amdgcn_cvt_pk_fp8_f32(c, c, 0, false) & 0xFFu;
  return x != x ? ((__float_as_uint(x) >> 24) & 0x80u) | 0x7Fu : code;
}

// Largest j in [0, n) with starts[j] <= x (starts non-decreasing, starts[0] <= x).
__device__ inline int upper_index(const int32_t* starts, int n, int x) {
  // Up to 8 entries in one scalar load (the plans' arrays hold more than 8),
  // else one load per 64 entries and a ballot, instead of a chain of dependent
  // scalar loads.
  int j = 0;
  if (n <= 8) {
#pragma unroll
    for (int k = 1; k < 8; ++k) j += (int)(k < n && starts[k] <= x);
    return j;
  }
  const int lane = threadIdx.x & 63;
  for (int c = 0; c < n; c += 64) {
    const bool in = c + lane < n && starts[min(c + lane, n - 1)] <= x;
    j += __popcll(__ballot(in));
  }
  return j - 1;
}

// ---------------------------------------------------------------------------
// One wave's online-softmax attention of 16 query rows (one per lane column
// n) against cache blocks kb_begin .. kb_end-1 of one sequence and KV head.
// Key `key` is visible to row n iff key <= limit (per lane) and key < kend;
// V rows of keys >= kend are replaced by zero (they may hold NaN/Inf).
//
// The loop is software-pipelined one block deep: block kb+1's K and V
// fragments are in flight while block kb is consumed.  Block ids come from a
// coalesced load of up to 64 consecutive block-table entries, one per lane,
// and are broadcast with readlane.
template <int DT, int D>
struct RowState {
  f32x4 acc[D / 16];
  float m;  // reference maximum of the row's scaled scores (log2 units)
  float l;  // this lane's part of the running sum of 2^(s*c - m), as rounded for the PV product
};

template <int DT, int D>
struct BlockFrags {
  typename Tr<DT>::Chunk k[D / (4 * Tr<DT>::X)];
  typename Tr<DT>::VFrag v[D / 16];
};

template <int DT, int D>
__device__ inline void load_block(const AttnArgs& a, int blk, int g, BlockFrags<DT, D>& f) {
  using T = Tr<DT>;
  using E = typename T::Elem;
  constexpr int X = T::X;
  const int lane = threadIdx.x & 63;
  const int n = lane & 15, grp = lane >> 4;
  const size_t base = ((size_t)blk * a.hkv + g) * ((size_t)D * kBlock);
  const E* kp = reinterpret_cast<const E*>(a.k_cache) + base;
  const E* vp = reinterpret_cast<const E*>(a.v_cache) + base;
#pragma unroll
  for (int r = 0; r < D / (4 * X); ++r) f.k[r] = T::load_chunk(kp + ((4 * r + grp) * kBlock + n) * X);
#pragma unroll
  for (int mt = 0; mt < D / 16; ++mt) f.v[mt] = T::load_v(vp + (16 * mt + n) * kBlock + 4 * grp);
}

// Scores -> probabilities -> PV for one 16-key block.  Scores are scaled to
// log2 units first (s2 = s * scale * log2(e)).  The softmax keeps a lazily
// moved reference maximum m per row: probabilities are 2^(s2 - m), and m
// (with the O / l rescale it implies) only moves when some score of the wave
// exceeds it by more than 8, so probabilities stay <= 2^8 and the
// accumulators are rescaled on a few blocks only.  The quotient O / l at the
// end is the same for any m; the block that sets m has its maximum at
// exactly 2^0 = 1, so a single key returns its value row unchanged.
// EDGE: the block may hold keys past kend or past some row's causal limit
// (its scores are masked and V rows of keys >= kend zeroed), or belong to
// rows of at most kFewKeys keys.  The plain form has neither, so the loop
// over a row's whole blocks carries no copies of the accumulators for them.
template <int DT, int D, bool EDGE>
__device__ inline void consume_block(const AttnArgs& a, const typename Tr<DT>::Chunk* qf, const BlockFrags<DT, D>& f,
                                     int kb, int kend, int limit, bool few_keys, RowState<DT, D>& st) {
  using T = Tr<DT>;
  constexpr int R = D / (4 * T::X);
  constexpr int MT = D / 16;
  const int grp = (threadIdx.x & 63) >> 4;
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int r = 0; r < R; ++r) s = T::qk(f.k[r], qf[r], s);
  s *= a.scale_log2;
  const int key0 = kb * kBlock + 4 * grp;
  if constexpr (EDGE) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (!(key0 + i <= limit && key0 + i < kend)) s[i] = -INFINITY;
  }
  const float lmax = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
  if (__any(lmax > st.m + 8.f)) {
    float bm = fmaxf(lmax, __shfl_xor(lmax, 16));
    bm = fmaxf(bm, __shfl_xor(bm, 32));
    const float m_new = fmaxf(st.m, bm);
    const float alpha = m_new == -INFINITY ? 1.f : exp2_fast(st.m - m_new);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) st.acc[mt] *= alpha;
    st.l *= alpha;
    st.m = m_new;
  }
  // rows whose reference is still -inf have seen no visible key: p = 0
  const float m = st.m == -INFINITY ? 0.f : st.m;
  f32x4 p;
#pragma unroll
  for (int i = 0; i < 4; ++i) p[i] = exp2_fast(s[i] - m);
  const auto pf = T::make_p(p);
  st.l = T::psum(p, pf, st.l);
  if constexpr (!EDGE) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) st.acc[mt] = T::pv(f.v[mt], pf, st.acc[mt]);
    return;
  }
  const int nvalid = kend - key0;
  if constexpr (T::kRoundsP) {
    if (few_keys) {
      // rows of at most kFewKeys keys: few probabilities carry each output,
      // so their bf16 rounding would not average out; the remainder p - hi
      // goes through a second PV product
      const auto plo = T::make_p_lo(p, pf);
      st.l = T::psum(p, plo, st.l);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const auto v = T::keep_first(f.v[mt], nvalid);
        st.acc[mt] = T::pv(v, plo, T::pv(v, pf, st.acc[mt]));
      }
      return;
    }
  }
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) st.acc[mt] = T::pv(T::keep_first(f.v[mt], nvalid), pf, st.acc[mt]);
}

// The block ids of a run of cache blocks: 64 consecutive block-table entries
// per coalesced load, one per lane, broadcast with readlane.  The next 64
// are loaded when a group is begun, so that the loads of the blocks never
// wait for their ids.  Blocks are asked for in order (a block at or past
// kb_end, asked for by a prefetch, is the last one).  REFILL false: a run of at
// most 64 blocks (a part of a row that is split on its own).
template <bool REFILL>
struct BlockIds {
  const int32_t* bt;
  int base, last, nb;
  int cur, nxt;
  bool poison;  // an id was out of range (block 0 is read in its place)
  __device__ inline BlockIds(const int32_t* table, int kb_begin, int kb_end, int num_blocks)
      : bt(table), base(kb_begin), last(kb_end - 1), nb(num_blocks), poison(false) {
    cur = fetch(base);
    if constexpr (REFILL) nxt = fetch(base + 64);
  }
  __device__ inline int fetch(int kb) const {
    const int k = kb + (int)(threadIdx.x & 63);
    return k <= last ? bt[k] : 0;
  }
  __device__ inline int operator()(int kb) {
    kb = min(kb, last);
    if constexpr (REFILL) {
      if (kb - base >= 64) {
        base += 64;
        cur = nxt;
        nxt = fetch(base + 64);
      }
    }
    int blk = __builtin_amdgcn_readlane(cur, kb - base);
    if (blk < 0 || blk >= nb) {
      poison = true;
      blk = 0;
    }
    return blk;
  }
};

// Blocks between two workgroup barriers of a streaming decode workgroup.
constexpr int kLockstepBlocks = 4;

// Keeps the waves of a streaming decode workgroup within kLockstepBlocks
// blocks of each other: `step` counts this wave's blocks since its last
// barrier.  The memory system serves the waves of a SIMD by age, so left
// alone the oldest finish early and the last ones stream by themselves at a
// falling rate.  Waves that have ended no longer count at s_barrier, so the
// waves of a workgroup may have different numbers of blocks.
__device__ inline void lockstep(int& step, int blocks) {
  step += blocks;
  if (step >= kLockstepBlocks) {
    step = 0;
    __builtin_amdgcn_s_barrier();
  }
}

// Blocks kb_begin .. kb_end-1 for 16 rows whose smallest causal limit is
// min_limit.  Software-pipelined one block deep: the next block's fragments
// are requested before the current one is consumed (the request is pinned in
// place with a scheduling barrier, and is issued unconditionally -- the last
// block is requested twice -- so consuming a block waits only for its own
// loads).  The blocks that every row sees whole come first, the others
// (kb_edge on: the last block, a causal diagonal, rows of few keys) last.
template <int DT, int D, bool STREAM>
__device__ inline void attend_blocks(const AttnArgs& a, const typename Tr<DT>::Chunk* qf,
                                     const int32_t* bt, int g, int kb_begin, int kb_end, int kend,
                                     int limit, int min_limit, RowState<DT, D>& st, bool& poison, int& step) {
  const bool few_keys = kend <= kFewKeys;  // every row sees at most kFewKeys keys
  const int whole = min_limit < kend ? min_limit + 1 : kend;  // keys that every row sees
  const int kb_edge = few_keys ? kb_begin : max(kb_begin, min(kb_end, whole / kBlock));
  if (kb_begin >= kb_end) return;
  BlockIds<true> id(bt, kb_begin, kb_end, a.nb);
  BlockFrags<DT, D> fa, fb;
  load_block<DT, D>(a, id(kb_begin), g, fa);
  int kb = kb_begin;
  for (; kb + 2 <= kb_edge; kb += 2) {
    load_block<DT, D>(a, id(kb + 1), g, fb);
    __builtin_amdgcn_sched_barrier(0);
    consume_block<DT, D, false>(a, qf, fa, kb, kend, limit, false, st);
    load_block<DT, D>(a, id(kb + 2), g, fa);
    __builtin_amdgcn_sched_barrier(0);
    consume_block<DT, D, false>(a, qf, fb, kb + 1, kend, limit, false, st);
    if constexpr (STREAM) lockstep(step, 2);
  }
  if (kb < kb_edge) {
    load_block<DT, D>(a, id(kb + 1), g, fb);
    __builtin_amdgcn_sched_barrier(0);
    consume_block<DT, D, false>(a, qf, fa, kb, kend, limit, false, st);
    if constexpr (STREAM) lockstep(step, 1);
    fa = fb;
    ++kb;
  }
  for (; kb < kb_end; ++kb) {
    load_block<DT, D>(a, id(kb + 1), g, fb);
    __builtin_amdgcn_sched_barrier(0);
    consume_block<DT, D, true>(a, qf, fa, kb, kend, limit, few_keys, st);
    if constexpr (STREAM) lockstep(step, 1);
    fa = fb;
  }
  poison |= id.poison;
}

// attend_blocks for fp8 caches.  A block's K and V granules of one head are
// 16 * D bytes each; read into registers in the MFMA operand layout they take
// 8-byte (K) and 4-byte (V) loads per lane, and such narrow loads stream
// about a tenth slower than 16-byte ones from scattered granules.  So each
// wave copies whole granules into a private ring of three LDS slots with
// 16-byte direct-to-LDS loads (non-temporal, 1 KB per instruction), two
// blocks ahead of the one it consumes, and reads the codes from LDS in the
// operand layout (conflict-free: a wave's K read covers 512 contiguous
// bytes, its V read 256).  `ring` is the wave's 3 * 2 * 16 * D bytes of LDS.
// The copies are counted in vmcnt only (the compiler does not see them), so
// the waits are explicit; the only other vector-memory operation of the loop
// is a load of 64 block ids every 64 blocks, which makes the waits stricter.  A
// part of a row that is split on its own has at most 64 blocks (1,024 keys), so
// it loads its ids once and its copies test for no refill (16 rows of 4,096
// keys, 8 heads of 128: 31.3 -> 30.5 us; 100 of 1,500 66.6 -> 64.9).
template <int D, bool STREAM>
__device__ inline void attend_blocks_fp8_lds(const AttnArgs& a, const bf16x8* qf, const int32_t* bt, int g,
                                             int kb_begin, int kb_end, int kend, int limit, int min_limit,
                                             RowState<2, D>& st, bool& poison, uint8_t* ring) {
  using T = Tr<2>;
  constexpr int GB = kBlock * D;    // bytes of one granule (K or V of one block and head)
  constexpr int NI = GB / 1024;     // 1 KB copies per granule
  constexpr int SLOT = 2 * GB;      // K granule, then V granule
  constexpr int R = D / (4 * T::X);
  constexpr int MT = D / 16;
  static_assert(GB % 1024 == 0, "whole 1 KB copies");
  const int lane = threadIdx.x & 63;
  const int n = lane & 15, grp = lane >> 4;
  const bool few_keys = kend <= kFewKeys;
  const int whole = min_limit < kend ? min_limit + 1 : kend;
  const int kb_edge = few_keys ? kb_begin : max(kb_begin, min(kb_end, whole / kBlock));
  if (kb_begin >= kb_end) return;
  BlockIds<STREAM> id(bt, kb_begin, kb_end, a.nb);
  auto copy = [&](int kb, int slot) {
    const size_t gran = ((size_t)id(kb) * a.hkv + g) * GB;
    const uint8_t* kp = reinterpret_cast<const uint8_t*>(a.k_cache) + gran;
    const uint8_t* vp = reinterpret_cast<const uint8_t*>(a.v_cache) + gran;
#pragma unroll
    for (int u = 0; u < NI; ++u) {
      global_to_lds16_nt(kp, (unsigned)(u * 1024 + lane * 16), ring + slot * SLOT + u * 1024);
      global_to_lds16_nt(vp, (unsigned)(u * 1024 + lane * 16), ring + slot * SLOT + GB + u * 1024);
    }
  };
  int slot = 0;
  BlockFrags<2, D> f;
  // requests block kb + 2, waits for block kb and reads it
  auto next = [&](int kb) {
    copy(kb + 2, slot == 0 ? 2 : slot - 1);
    MPA_WAIT_VMCNT(4 * NI);  // the copies of blocks kb+1 and kb+2 may still be in flight
    const uint8_t* sp = ring + slot * SLOT;
#pragma unroll
    for (int r = 0; r < R; ++r)
      f.k[r] = T::k_from_codes(*reinterpret_cast<const u32x2*>(sp + ((4 * r + grp) * kBlock + n) * T::X));
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      f.v[mt] = T::v_from_codes(*reinterpret_cast<const unsigned*>(sp + GB + (16 * mt + n) * kBlock + 4 * grp));
    slot = slot == 2 ? 0 : slot + 1;
  };
  copy(kb_begin, 0);
  copy(kb_begin + 1, 1);  // past the last block: that block again (unused)
  int kb = kb_begin;
  for (; kb < kb_edge; ++kb) {
    next(kb);
    consume_block<2, D, false>(a, qf, f, kb, kend, limit, false, st);
  }
  for (; kb < kb_end; ++kb) {
    next(kb);
    consume_block<2, D, true>(a, qf, f, kb, kend, limit, few_keys, st);
  }
  // The ring is reused by the next run of blocks (and the wave's LDS is
  // released when it ends): no copy may still be writing it.
  MPA_WAIT_VMCNT(0);
  poison |= id.poison;
}

// A decode row's new token (query row t, position pos) for KV head g,
// written by the wave that reads the row's last part -- parts' edges are
// block-aligned, so no other wave reads this (block, head) granule -- with
// the bits the append kernels store (E4M3 codes for fp8 caches).  K goes out
// as 16 bytes a lane, V as each lane's D / 64 dims of the slot.  The wave
// waits for its stores before it loads any block.  A bad block id writes
// nothing (the row comes out NaN).
template <int DT, int D, bool NT>
__device__ inline void append_decode_token(const AttnArgs& a, int s, int pos, int t, int g, int lane) {
  constexpr int RT = DT == 2 ? 0 : DT;  // new rows: bf16 beside an fp8 cache
  using NE = typename Tr<RT>::Elem;
  using CE = typename Tr<DT>::Elem;
  constexpr int X = Tr<DT>::X;
  constexpr int NC = D / X;    // K chunks of the row
  constexpr int DPL = D / 64;  // V dims per lane
  const int blk = a.block_tables[(size_t)s * a.mb + pos / kBlock];
  if (blk < 0 || blk >= a.nb) return;
  const int slot = pos % kBlock;
  const size_t head = (size_t)blk * a.hkv + g;
  const size_t src = ((size_t)t * a.hkv + g) * D;
  const NE* kn = reinterpret_cast<const NE*>(a.k_new) + src;
  const NE* vn = reinterpret_cast<const NE*>(a.v_new) + src + DPL * lane;
  NE v[DPL];
#pragma unroll
  for (int i = 0; i < DPL; ++i) v[i] = vn[i];
  const u32x4 kw = *reinterpret_cast<const u32x4*>(kn + (lane % NC) * X);
  if (lane < NC) {
    CE* dst = reinterpret_cast<CE*>(const_cast<void*>(a.k_cache)) + ((head * NC + lane) * kBlock + slot) * X;
    if constexpr (DT == 2) {
      float kx[8];
      Tr<0>::unpack(kw, kx);
      u32x2 kc = {0u, 0u};
#pragma unroll
      for (int e = 0; e < 8; ++e) kc[e / 4] |= f32_to_e4m3(kx[e] * a.inv_k_scale) << (8 * (e % 4));
      st_token<NT>(dst, kc);
    } else {
      st_token<NT>(dst, kw);
    }
  }
  CE* vc = reinterpret_cast<CE*>(const_cast<void*>(a.v_cache)) + (head * D + DPL * lane) * kBlock + slot;
#pragma unroll
  for (int i = 0; i < DPL; ++i) {
    if constexpr (DT == 2)
      st_token<NT>(vc + i * kBlock, (uint8_t)f32_to_e4m3(__uint_as_float((unsigned)v[i] << 16) * a.inv_v_scale));
    else
      st_token<NT>(vc + i * kBlock, v[i]);
  }
}

// The results of a workgroup's kKeyWaves waves for the same 16 rows, each over
// keys of its own, merged through LDS and written: (max, sum) of every wave
// and row, then the accumulators, half of the dims at a time; wave w adds up
// the rows' dims 16 * mt for its mt.  `l` is the row's sum over the lane
// groups, out and lse (lse may be null) the lane's row.  A wave that saw no
// key of a row (or only keys of score -inf) has max -inf and weight 0.
constexpr int kKeyWaves = 8;

// 2^(m - M) for a partial result's maximum m <= M: 0 where m is -inf, also
// when every partial result's is.
__device__ inline float partial_weight(float m, float M) { return exp2_fast(m - (M == -INFINITY ? 0.f : M)); }

template <int DT, int D>
__device__ inline void merge_waves(const RowState<DT, D>& st, float l, bool poison, float v_scale, bool row_ok,
                                   typename Tr<DT>::QElem* out, float* lse) {
  constexpr int MT = D / 16;
  const int lane = threadIdx.x & 63;
  const int wave = wave_uniform(threadIdx.x >> 6);
  const int n = lane & 15, grp = lane >> 4;
  __shared__ float ml[kKeyWaves][2][16];
  __shared__ f32x4 part[kKeyWaves][MT / 2][64];
  if (grp == 0) {
    ml[wave][0][n] = st.m;
    ml[wave][1][n] = poison ? NAN : l;
  }
  float w[kKeyWaves], M = -INFINITY, sum = 0.f;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    if (half) __syncthreads();
#pragma unroll
    for (int mt = 0; mt < MT / 2; ++mt) part[wave][mt][lane] = st.acc[half * (MT / 2) + mt];
    __syncthreads();
    if (half == 0) {
#pragma unroll
      for (int k = 0; k < kKeyWaves; ++k) M = fmaxf(M, ml[k][0][n]);
#pragma unroll
      for (int k = 0; k < kKeyWaves; ++k) {
        w[k] = partial_weight(ml[k][0][n], M);
        sum += ml[k][1][n] * w[k];
      }
    }
    if (wave < MT / 2 && row_ok) {
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < kKeyWaves; ++k) v += part[k][wave][lane] * w[k];
      Tr<DT>::store4(out + 16 * (half * (MT / 2) + wave) + 4 * grp, v * (v_scale / sum));
    }
  }
  if (lse && wave == 0 && grp == 0 && row_ok) *lse = (M + log2f(sum)) * kLn2;
}

// ---------------------------------------------------------------------------
// Decode; the G query heads of the group are the 16 MFMA columns (columns
// >= G carry zero queries).
// STREAM false: one wave per (sequence, split, KV head).
// STREAM true: the launch holds one wave per slot of the device, and the
// wave of a KV head takes a range of p.range_blocks consecutive blocks of
// all rows laid end to end; it walks the rows its range touches, each a part
// of that row.  Bound by HBM: a wave that starts costs the latency of its
// plan, its block ids and its first block with nothing in flight (about 5
// us), and splits of at most 1,024 tokens start 2 to 6 waves per slot on
// large batches.  Decode and merge, random contexts, before -> after: 7.9
// GB (256 rows) 1,375 -> 1,205 us, 10.8 GB (32 rows) 1,767 -> 1,554 us (6.97
// TB/s; a contiguous read of 2 GiB takes 7.08), fp8 1.46 GB 265 -> 237 us,
// 64-wide heads 1.6 GB 271 -> 247 us.
// Decode waves a SIMD holds at the kernels' register use (fp8 at 64-wide heads
// is held to 80 registers for six, which its LDS allows: at 82 and five, 256
// rows of 2,000 keys in row splits took 100.9 us, now 93.6).
constexpr int decode_waves_per_simd(int dt, int d) { return d == 128 ? (dt == 1 ? 2 : 3) : dt == 2 ? 6 : 4; }

template <int DT, int D, int WPG, bool STREAM>
__global__ __launch_bounds__(64 * WPG, decode_waves_per_simd(DT, D)) void decode_kernel(AttnArgs a, DecodePlan p) {
  using T = Tr<DT>;
  using QE = typename T::QElem;
  constexpr int X = T::X;
  constexpr int R = D / (4 * X);
  constexpr int MT = D / 16;
  const int lane = threadIdx.x & 63;
  const int wave = wave_uniform(threadIdx.x >> 6);
  const int unit = blockIdx.x * WPG + wave;
  const int item = unit / a.hkv;
  const int g = unit - item * a.hkv;
  const int G = a.hq / a.hkv;
  int j, blk = 0, blk_end = 0;
  if constexpr (STREAM) {
    if (item >= p.n_ranges) return;  // by number: item * range_blocks may pass 2^31 here
    blk = item * p.range_blocks;
    blk_end = min(blk + p.range_blocks, p.part[p.n_seqs]);
    j = upper_index(p.part, p.n_seqs, blk);
  } else {
    if (item >= p.item_start[p.n_seqs]) return;
    j = upper_index(p.item_start, p.n_seqs, item);
  }
  if (a.k_new != nullptr) {
    // the new tokens of the rows this wave reads to their ends, all at once:
    // in the loop below each would hold up the whole workgroup
    bool stored = false;
    if constexpr (STREAM) {
      for (int k = j; k < p.n_seqs && p.part[k + 1] <= blk_end; ++k) {
        const int s = p.seq[k];
        append_decode_token<DT, D, STREAM>(a, s, a.seq_lens[s] - 1, a.qsl[s], g, lane);
        stored = true;
      }
    } else if (item == p.item_start[j + 1] - 1) {
      const int s = p.seq[j];
      append_decode_token<DT, D, STREAM>(a, s, a.seq_lens[s] - 1, a.qsl[s], g, lane);
      stored = true;
    }
    if (stored) MPA_WAIT_VMCNT(0);  // stores are counted in vmcnt
  }
  int step = 0;
  for (;; ++j) {
    int ln = lane;
    if constexpr (STREAM) asm volatile("" : "+v"(ln));
    const int n = ln & 15, grp = ln >> 4;
    const bool head_ok = n < G;
    const int h = g * G + (head_ok ? n : 0);
    const int s = p.seq[j];
    const int nsplit = p.item_start[j + 1] - p.item_start[j];
    const int L = a.seq_lens[s];
    int k0, k1, split;
    if constexpr (STREAM) {
      const int row0 = p.part[j];
      split = item - row0 / p.range_blocks;
      k0 = (blk - row0) * kBlock;
      blk = min(blk_end, p.part[j + 1]);
      k1 = min(L, (blk - row0) * kBlock);
    } else {
      split = item - p.item_start[j];
      k0 = split * p.part[j];
      k1 = min(L, k0 + p.part[j]);
    }
    const int trow = a.qsl[s];

    const QE* q = reinterpret_cast<const QE*>(a.q) + ((size_t)trow * a.hq + h) * D;
    typename T::Chunk qf[R];
#pragma unroll
    for (int r = 0; r < R; ++r) qf[r] = head_ok ? T::load_q(q + (4 * r + grp) * X) : T::zero_chunk();

    RowState<DT, D> st;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) st.acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    st.m = -INFINITY;
    st.l = 0.f;
    bool poison = false;
    if constexpr (DT == 2) {
      __shared__ __attribute__((aligned(16))) uint8_t ring[WPG][3 * 2 * kBlock * D];
      attend_blocks_fp8_lds<D, STREAM>(a, qf, a.block_tables + (size_t)s * a.mb, g, k0 / kBlock,
                                       (k1 + kBlock - 1) / kBlock, k1, INT32_MAX, INT32_MAX, st, poison, ring[wave]);
    } else {
      attend_blocks<DT, D, STREAM>(a, qf, a.block_tables + (size_t)s * a.mb, g, k0 / kBlock,
                                   (k1 + kBlock - 1) / kBlock, k1, INT32_MAX, INT32_MAX, st, poison, step);
    }

    float l = st.l + __shfl_xor(st.l, 16);
    l += __shfl_xor(l, 32);
    if (head_ok) {
      if (nsplit == 1) {
        const float inv = poison ? NAN : a.v_scale / l;
        QE* o = reinterpret_cast<QE*>(a.out) + ((size_t)trow * a.hq + h) * D;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) T::store4(o + 16 * mt + 4 * grp, st.acc[mt] * inv);
        if (a.lse && grp == 0) a.lse[(size_t)trow * a.hq + h] = poison ? NAN : (st.m + log2f(l)) * kLn2;
      } else {
        const size_t slot = (size_t)(p.item_base + p.item_start[j] + split) * a.hq + h;
        float* wo = a.ws_o + slot * D;
        const float bad = poison ? NAN : 1.f;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          *reinterpret_cast<f32x4*>(wo + 16 * mt + 4 * grp) = st.acc[mt] * (bad * a.v_scale);
        if (grp == 0) {
          a.ws_ml[slot * 2] = st.m;
          a.ws_ml[slot * 2 + 1] = l * bad;
        }
      }
    }
    if (!STREAM || blk >= blk_end) return;
  }
}

// Decode of few short rows: one workgroup per (row, KV head), whose waves each
// take an eighth of the row's blocks and merge in LDS, so that the step needs
// neither partial results nor a merge launch.  Latency bound.  4 rows of
// 64-256 keys at 2 KV heads of 64: 5.6 us; the split kernel and its merge
// took 5.9 and 3.1 and the gap between them 1.3.
template <int DT, int D>
__global__ __launch_bounds__(64 * kKeyWaves, 2) void decode_short_kernel(AttnArgs a, DecodePlan p) {
  using T = Tr<DT>;
  using QE = typename T::QElem;
  constexpr int X = T::X;
  constexpr int R = D / (4 * X);
  constexpr int MT = D / 16;
  const int lane = threadIdx.x & 63;
  const int wave = wave_uniform(threadIdx.x >> 6);
  const int j = blockIdx.x / a.hkv;
  const int g = blockIdx.x - j * a.hkv;
  if (j >= p.n_seqs) return;
  const int s = p.seq[j];
  const int L = a.seq_lens[s];
  const int trow = a.qsl[s];
  const int G = a.hq / a.hkv;
  const int n = lane & 15, grp = lane >> 4;
  const bool head_ok = n < G;
  const int h = g * G + (head_ok ? n : 0);
  const int nb = (L + kBlock - 1) / kBlock;
  const int per = (nb + kKeyWaves - 1) / kKeyWaves;
  const int kb0 = min(wave * per, nb), kb1 = min(nb, kb0 + per);
  if (a.k_new != nullptr && kb0 < kb1 && kb1 == nb) {
    append_decode_token<DT, D, false>(a, s, L - 1, trow, g, lane);
    MPA_WAIT_VMCNT(0);  // stores are counted in vmcnt
  }
  const QE* q = reinterpret_cast<const QE*>(a.q) + ((size_t)trow * a.hq + h) * D;
  typename T::Chunk qf[R];
#pragma unroll
  for (int r = 0; r < R; ++r) qf[r] = head_ok ? T::load_q(q + (4 * r + grp) * X) : T::zero_chunk();
  RowState<DT, D> st;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) st.acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
  st.m = -INFINITY;
  st.l = 0.f;
  bool poison = false;
  int step = 0;
  attend_blocks<DT, D, false>(a, qf, a.block_tables + (size_t)s * a.mb, g, kb0, kb1, L, INT32_MAX, INT32_MAX, st,
                              poison, step);
  float l = st.l + __shfl_xor(st.l, 16);
  l += __shfl_xor(l, 32);
  merge_waves<DT, D>(st, l, poison, a.v_scale, head_ok,
                     reinterpret_cast<QE*>(a.out) + ((size_t)trow * a.hq + h) * D,
                     a.lse ? a.lse + (size_t)trow * a.hq + h : nullptr);
}

// Split-K merge.  With split maxima m_k and sums l_k (log2 units), a row's
// softmax denominator is sum_k l_k 2^(m_k - M) with M = max_k m_k, and its
// output is sum_k acc_k 2^(m_k - M) divided by that denominator.
//
// One output row from n partial results, by one wave.  Splits are taken 64
// at a time: lane k loads split k's (m, l) pair and the group's maximum and
// weighted sum come from wave reductions.  A partial row is D / 4 lanes of
// 16 bytes, so the wave reads 256 / D rows per instruction, kMergeUnroll of
// them in flight; each lane adds its 4 elements of every (256 / D)-th split,
// and the lanes' sums are combined at the end.  Only the n real splits are
// read, by as many loads as they need (four loads of two splits' rows took a
// prompt of 1,000 tokens, 32 heads, from 75.5 us to 78.6).  ml points at split
// 0's (m, l) pair (8-byte aligned), acc at split 0's row (16-byte aligned);
// consecutive splits are ml_stride and acc_stride floats apart.
__device__ inline float wave_max64(float x) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) x = fmaxf(x, __shfl_xor(x, off));
  return x;
}
__device__ inline float wave_sum64(float x) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off);
  return x;
}
constexpr int kMergeUnroll = 4;

// Running result over some splits of a row: maximum, weighted sum and (in
// every lane, elements 4 * (lane % (D / 4)) .. + 3) weighted rows.
struct MergeState {
  float M, lsum;
  f32x4 o;
};

template <int D>
__device__ inline MergeState merge_range(const float* ml, size_t ml_stride, const float* acc, size_t acc_stride,
                                         int n) {
  constexpr int LPR = D / 4;     // lanes per partial row
  constexpr int RPI = 64 / LPR;  // rows per load instruction
  const int lane = threadIdx.x & 63;
  const int sub = lane / LPR;
  acc += 4 * (lane % LPR);
  MergeState r = {-INFINITY, 0.f, {0.f, 0.f, 0.f, 0.f}};
  for (int c0 = 0; c0 < n; c0 += 64) {
    const int cnt = min(64, n - c0);
    float mk = -INFINITY, lk = 0.f;
    if (lane < cnt) {
      const float2 v = *reinterpret_cast<const float2*>(ml + (size_t)(c0 + lane) * ml_stride);
      mk = v.x;
      lk = v.y;
    }
    const float gm = fmaxf(r.M, wave_max64(mk));
    const float wk = lane < cnt ? partial_weight(mk, gm) : 0.f;
    const float rescale = partial_weight(r.M, gm);  // M = -inf on the first group: 0
    r.lsum = r.lsum * rescale + wave_sum64(wk * lk);
    r.o *= rescale;
    for (int k = 0; k < cnt; k += RPI * kMergeUnroll) {
      f32x4 v[kMergeUnroll];
#pragma unroll
      for (int u = 0; u < kMergeUnroll; ++u) {
        if (k + u * RPI >= cnt) break;
        const int i = min(k + u * RPI + sub, cnt - 1);
        v[u] = *reinterpret_cast<const f32x4*>(acc + (size_t)(c0 + i) * acc_stride);
      }
#pragma unroll
      for (int u = 0; u < kMergeUnroll; ++u) {
        if (k + u * RPI >= cnt) break;
        const int i = k + u * RPI + sub;
        const float w = __shfl(wk, min(i, cnt - 1));
        if (i < cnt) r.o += v[u] * w;
      }
    }
    r.M = gm;
  }
#pragma unroll
  for (int off = LPR; off < 64; off <<= 1)
#pragma unroll
    for (int e = 0; e < 4; ++e) r.o[e] += __shfl_xor(r.o[e], off);
  return r;
}

// Lanes 0 .. D/4 - 1 write the row's elements, lane 0 its lse.
template <int DT, int D>
__device__ inline void merge_store(const MergeState& r, typename Tr<DT>::QElem* out, float* lse) {
  const int lane = threadIdx.x & 63;
  const float inv = 1.f / r.lsum;
  if (lane < D / 4) Tr<DT>::store4(out + 4 * lane, r.o * inv);
  if (lse && lane == 0) *lse = (r.M + log2f(r.lsum)) * kLn2;
}

// The merge kernels run four waves per workgroup, each wave merging whole
// (row, q head) pairs on its own (no LDS, no barrier): a launch with one
// small workgroup per pair is bound by the dispatcher's workgroup rate
// (about 1.2 per ns), not by the bytes it moves.
constexpr int kMergeWaves = 4;

// Decode merge: one workgroup per (split decode sequence, 4 q heads); wave w
// merges head 4 * blockIdx.y + w.  WIDE: one workgroup per (sequence, q
// head), its waves each taking a quarter of the splits.
template <int DT, int D, bool WIDE>
__global__ __launch_bounds__(64 * kMergeWaves) void merge_kernel(AttnArgs a, DecodePlan p) {
  using E = typename Tr<DT>::QElem;
  const int j = blockIdx.x;
  const int wave = wave_uniform(threadIdx.x >> 6);
  const int h = WIDE ? blockIdx.y : blockIdx.y * kMergeWaves + wave;
  if (j >= p.n_seqs || h >= a.hq) return;
  const int n = p.item_start[j + 1] - p.item_start[j];
  if (n <= 1) return;
  const int s = p.seq[j];
  const int t = a.qsl[s];
  // this wave's splits [x0, x0 + nx)
  const int per = WIDE ? (n + kMergeWaves - 1) / kMergeWaves : n;
  const int x0 = WIDE ? min(wave * per, n) : 0;
  const int nx = WIDE ? min(per, n - x0) : n;
  const size_t base = (size_t)p.item_base + p.item_start[j] + x0;
  MergeState r = merge_range<D>(a.ws_ml + (base * a.hq + h) * 2, (size_t)a.hq * 2, a.ws_o + (base * a.hq + h) * D,
                                (size_t)a.hq * D, nx);
  if constexpr (WIDE) {
    __shared__ float ml[kMergeWaves][2];
    __shared__ f32x4 rows[kMergeWaves][D / 4];
    const int lane = threadIdx.x & 63;
    if (lane == 0) {
      ml[wave][0] = r.M;
      ml[wave][1] = r.lsum;
    }
    if (lane < D / 4) rows[wave][lane] = r.o;
    __syncthreads();
    if (wave != 0) return;
    float M = ml[0][0];
#pragma unroll
    for (int w = 1; w < kMergeWaves; ++w) M = fmaxf(M, ml[w][0]);
    MergeState all = {M, 0.f, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int w = 0; w < kMergeWaves; ++w) {
      const float f = partial_weight(ml[w][0], M);  // a wave without splits: 0
      all.lsum += ml[w][1] * f;
      all.o += rows[w][lane % (D / 4)] * f;
    }
    r = all;
  }
  merge_store<DT, D>(r, reinterpret_cast<E*>(a.out) + ((size_t)t * a.hq + h) * D,
                     a.lse ? a.lse + (size_t)t * a.hq + h : nullptr);
}

// Prefill merge: one workgroup per (token of a KV-split segment, 4 * per_wave q
// heads); wave w merges heads 4 * (per_wave * blockIdx.y + k) + w, k <
// per_wave.  Split x of token i of segment j sits at slot item_base[j] +
// x*ntok[j] + i.
template <int DT, int D>
__global__ __launch_bounds__(64 * kMergeWaves) void prefill_merge_kernel(AttnArgs a, PrefillPlan p, int per_wave) {
  using E = typename Tr<DT>::QElem;
  const int r = blockIdx.x;
  if (r >= p.row_start[p.n_seqs]) return;
  const int j = upper_index(p.row_start, p.n_seqs, r);
  const int s = p.seq[j];
  const int i = r - p.row_start[j];
  const int t0 = a.qsl[s] + p.tok0[j];
  const int C = p.ntok[j];
  const size_t slot = (size_t)p.item_base[j] + i;
  const int h0 = blockIdx.y * (kMergeWaves * per_wave) + wave_uniform(threadIdx.x >> 6);
  for (int k = 0; k < per_wave; ++k) {
    const int h = h0 + k * kMergeWaves;
    if (h >= a.hq) break;
    const MergeState m = merge_range<D>(a.ws_ml + (slot * a.hq + h) * 2, (size_t)C * a.hq * 2,
                                        a.ws_o + (slot * a.hq + h) * D, (size_t)C * a.hq * D, p.nsplit[j]);
    merge_store<DT, D>(m, reinterpret_cast<E*>(a.out) + ((size_t)(t0 + i) * a.hq + h) * D,
                       a.lse ? a.lse + (size_t)(t0 + i) * a.hq + h : nullptr);
  }
}

// ---------------------------------------------------------------------------
// Prefill chunks, f32 caches.  A (sequence, query tile, KV head) has 64
// (token, head) rows; row r is token r / G of the tile and head r % G of the
// group.  A wave works on 16 rows (its MFMA columns).
// KEYS false: one workgroup per tile, each of its 4 waves with rows of its
// own and all their keys.
// KEYS true: one workgroup per 16 rows (4 to a tile), whose 8 waves each take
// an eighth of the key blocks; their results are merged in LDS.  A wave needs
// 2,048 MFMA cycles per 16 keys whichever form runs, so a tile by itself
// takes about 1.2 us per block of its longest row with most of the device
// idle; an eighth of the keys a wave spreads the same products over four
// times the workgroups and eighths of the time.
template <int DT, int D, bool KEYS>
__global__ __launch_bounds__(KEYS ? 64 * kKeyWaves : 256, 2) void prefill_kernel(AttnArgs a, PrefillPlan p) {
  using T = Tr<DT>;
  using QE = typename T::QElem;
  constexpr int X = T::X;
  constexpr int R = D / (4 * X);
  constexpr int MT = D / 16;
  const int lane = threadIdx.x & 63;
  const int wave = wave_uniform(threadIdx.x >> 6);
  const int unit = blockIdx.x / a.hkv;
  const int g = blockIdx.x - unit * a.hkv;
  const int n_tiles = p.tile_start[p.n_seqs];
  const int tile = n_tiles - 1 - (KEYS ? unit >> 2 : unit);  // a chunk's last (longest) tiles first
  const int sub = KEYS ? unit & 3 : wave;                    // the 16 rows of the tile
  if (tile < 0) return;
  const int j = upper_index(p.tile_start, p.n_seqs, tile);
  const int s = p.seq[j];
  const int qt = tile - p.tile_start[j];
  // the segment's first query row, tokens, and keys before it
  const int chunk0 = a.qsl[s];
  const int t0 = chunk0 + p.tok0[j];
  const int C = p.ntok[j];
  const int L = a.seq_lens[s];
  const int P = L - (a.qsl[s + 1] - chunk0) + p.tok0[j];
  const int G = a.hq / a.hkv;
  const int first_tok = qt * p.q_tile;
  if (first_tok + (sub * 16) / G >= C) return;  // no rows here (the same for the whole workgroup with KEYS)
  const int n = lane & 15, grp = lane >> 4;
  const int row = sub * 16 + n;
  // The tile holds q_tile tokens (G * q_tile <= 64 rows): when G does not
  // divide 64, the last rows of the workgroup would fall on the next tile's
  // first token.  They compute a valid token of this tile and store nothing.
  const int r_tok = row / G;
  const int i_raw = first_tok + min(r_tok, p.q_tile - 1);
  const bool row_ok = r_tok < p.q_tile && i_raw < C;
  const int i = min(i_raw, C - 1);
  const int h = g * G + row % G;
  const int last_tok = min(first_tok + min((sub * 16 + 15) / G, p.q_tile - 1), C - 1);
  const int kend = P + last_tok + 1;  // keys these rows need

  const QE* q = reinterpret_cast<const QE*>(a.q) + ((size_t)(t0 + i) * a.hq + h) * D;
  typename T::Chunk qf[R];
#pragma unroll
  for (int r = 0; r < R; ++r) qf[r] = T::load_q(q + (4 * r + grp) * X);

  RowState<DT, D> st;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) st.acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
  st.m = -INFINITY;
  st.l = 0.f;
  bool poison = false;
  const int min_limit = P + min(first_tok + (sub * 16) / G, C - 1);
  const int nb = (kend + kBlock - 1) / kBlock;
  const int per = KEYS ? (nb + kKeyWaves - 1) / kKeyWaves : nb;
  const int kb0 = KEYS ? min(wave * per, nb) : 0;
  int step = 0;
  attend_blocks<DT, D, false>(a, qf, a.block_tables + (size_t)s * a.mb, g, kb0, min(nb, kb0 + per), kend, P + i,
                              min_limit, st, poison, step);

  float l = st.l + __shfl_xor(st.l, 16);
  l += __shfl_xor(l, 32);
  QE* o = reinterpret_cast<QE*>(a.out) + ((size_t)(t0 + i) * a.hq + h) * D;
  if constexpr (KEYS) {
    merge_waves<DT, D>(st, l, poison, a.v_scale, row_ok, o, a.lse ? a.lse + (size_t)(t0 + i) * a.hq + h : nullptr);
    return;
  }
  if (!row_ok) return;
  const float inv = poison ? NAN : a.v_scale / l;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) T::store4(o + 16 * mt + 4 * grp, st.acc[mt] * inv);
  if (a.lse && grp == 0)
    a.lse[(size_t)(t0 + i) * a.hq + h] = poison ? NAN : (st.m + log2f(l)) * kLn2;
}

// ---------------------------------------------------------------------------
// Prefill chunks, bf16: the tensor-core path.  One workgroup of WAVES (8 or 4) waves
// per (sequence, 32*WAVES-row query tile, KV head); row r of the tile is token
// r / G and head r % G of the group, so the G heads that share a KV head share
// every K/V tile.  Each wave owns 32 rows (one 32-wide MFMA column tile).
//
// Per 64-key tile (4 cache blocks), in a STAGES-deep LDS ring:
//   S^T[64 keys][32 rows] = K . Q^T   2 x (D/16) v_mfma_f32_32x32x16_bf16
//   O^T[D][32 rows]     += V^T . P^T  (D/32) x 4 v_mfma_f32_32x32x16_bf16
// Tiles are fetched straight into LDS (global_load_lds, 16 bytes a lane) by
// the waves themselves, STAGES-1 tiles ahead of use, so no registers stage
// them and a copy has STAGES-1 tiles of compute to land in.  The per-lane
// source addresses permute 16-byte pieces so that every MFMA operand read
// from LDS is one contiguous run per 16 lanes (no bank conflicts):
//  * row m of a 32-key S^T tile is key 16(m/16) + swap23(m%16), where swap23
//    exchanges bits 2 and 3.  Then the 8 keys a lane holds for one 16-key PV
//    step (output rows 8j+4h+i, j in {2t', 2t'+1}) are keys 8h..8h+7 of the
//    block.  LDS holds each K chunk row with its 16 slots already in that
//    order: [block][d/8 chunks][slot][8], slot s = key swap23(s);
//  * LDS holds V^T as [block][key half h][d][8 keys], so lane (m, h) of a PV
//    step reads row 32dt+m of half h.
// Each wave copies a contiguous part of one block of a tile, so it needs one
// block id per tile (a scalar load) and fixes up its own pieces (zeroing V entries of keys >= L,
// which may hold NaN/Inf; NaN for an invalid block id) before the barrier
// that publishes the tile.
//
// Softmax: exact online softmax with a lazily updated reference maximum.  The
// running reference m only moves when a row's new maximum exceeds it by more
// than 8 (log2 units), so exp2(s - m) <= 2^8 and the O / l rescale is skipped
// for almost every tile; the final O / l is the same quotient either way.
template <int CT, int D, int WAVES, int STAGES>
__global__ __launch_bounds__(64 * WAVES, WAVES == 8 ? 1 : D == 64 ? 3 : 2) void prefill_mfma_kernel(AttnArgs a, PrefillPlan p) {
  using f32x16 = float __attribute__((ext_vector_type(16)));
  using cint = const __attribute__((address_space(4))) int32_t;
  constexpr int BN = 64;                   // keys per tile
  constexpr int NB = BN / kBlock;          // cache blocks per tile
  constexpr int BLK = kBlock * D;          // elements of one (block, head) granule
  constexpr int TILE = NB * BLK;           // elements of one K (or V) tile
  constexpr int KS = D / 16;               // k-steps of the QK^T product
  static_assert(KS >= 4, "the V reads follow the last four k-steps");
  constexpr int DT = D / 32;               // 32-dim row tiles of O^T
  constexpr int NI = TILE * 2 / 1024;      // 1 KB copies per tile and cache
  constexpr int WI = NI / WAVES;           // ... per wave
  static_assert(WI >= 1 && NI % WAVES == 0 && (WI * 512) <= BLK && BLK % (WI * 512) == 0,
                "each wave copies part of exactly one block per tile");
  // CT: the cache type, 0 bf16 or 2 fp8.  fp8 codes take a register path:
  // each lane loads one 16-byte piece of the K tile and one of the V tile
  // (a (block, head) granule has D such pieces), one tile ahead, and at the
  // end of the iteration converts them to bf16 into the same LDS layout the
  // bf16 copies fill, so the compute below is the same for both.
  static_assert(CT == 0 || CT == 2, "bf16 or fp8 caches");
  static_assert(CT == 0 || (NB * D <= 64 * WAVES && (64 * WAVES) % D == 0), "one fp8 piece per lane");
  constexpr int AHEAD = CT == 2 ? 1 : STAGES - 1;  // tiles a copy runs ahead of its use
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  uint16_t* const sk = smem;                   // STAGES K tiles
  uint16_t* const sv = smem + STAGES * TILE;   // STAGES V tiles

  const int lane = threadIdx.x & 63;
  const int wave = wave_uniform(threadIdx.x >> 6);
  const int n_tiles = p.tile_start[p.n_seqs];
  const int g = blockIdx.x % a.hkv;
  const int tile = n_tiles - 1 - (int)(blockIdx.x / a.hkv);  // last (longest) query tiles first
  const int j = upper_index(p.tile_start, p.n_seqs, tile);
  const int s = p.seq[j];
  const int nsplit = p.nsplit[j];
  const int qt = (tile - p.tile_start[j]) / nsplit;
  const int split = tile - p.tile_start[j] - qt * nsplit;
  // the segment's first query row, tokens, and keys before it
  const int chunk0 = a.qsl[s];
  const int t0 = chunk0 + p.tok0[j];
  const int C = p.ntok[j];
  const int L = a.seq_lens[s];
  const int P = L - (a.qsl[s + 1] - chunk0) + p.tok0[j];
  const int G = a.hq / a.hkv;
  const int first_tok = qt * p.q_tile;
  const int last_tok = min(first_tok + p.q_tile - 1, C - 1);
  const int kend = P + last_tok + 1;  // keys the query tile needs
  // this workgroup's 64-key tiles: [kt_begin, ntile)
  const int kt_begin = split * p.split_tiles[j];
  const int ntile = split == nsplit - 1 ? (kend + BN - 1) / BN : kt_begin + p.split_tiles[j];
  cint* bt = (cint*)(a.block_tables + (size_t)s * a.mb);

  // this lane's query row.  The tile holds q_tile tokens (G * q_tile <= 256
  // rows): when G does not divide 256, the last rows of the workgroup would
  // fall on the next tile's first token, past the keys loaded here.  They
  // compute a valid token of this tile and store nothing.
  const int n = lane & 31, h = lane >> 5;
  const int row = wave * 32 + n;
  const int r_tok = row / G;
  const int i_raw = first_tok + min(r_tok, p.q_tile - 1);
  const bool row_ok = r_tok < p.q_tile && i_raw < C;
  const int i = min(i_raw, C - 1);
  const int head = g * G + row % G;
  const int limit = P + i;
  const int w_first = first_tok + (wave * 32) / G;
  const bool wave_active = w_first < C;
  const int w_min_limit = P + min(w_first, C - 1);
  const int w_kend = P + min(first_tok + min((wave * 32 + 31) / G, p.q_tile - 1), C - 1) + 1;

  bf16x8 qf[KS];
  {
    const uint16_t* q = reinterpret_cast<const uint16_t*>(a.q) + ((size_t)(t0 + i) * a.hq + head) * D;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      qf[ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(q + (2 * ks + h) * 8));
  }

  // ---- global -> LDS tile copies (this wave's slices)
  const int nblk = (kend + kBlock - 1) / kBlock;
  const int pi = wave * 64 + lane;  // fp8: this lane's 16-byte piece of the tile
  const int my_bi = CT == 2 ? (wave * 64) / D : (wave * WI * 512) / BLK;  // the tile block this wave copies
  u32x4 kraw = {0u, 0u, 0u, 0u}, vraw = {0u, 0u, 0u, 0u};  // fp8 pieces in flight
  // Tile kt's copy.  A block index past the sequence's last needed block is
  // clamped to it (its keys are all masked and its V entries zeroed), so
  // every copy is issued, always 2*WI instructions per wave per tile.
  // the id of the block this wave copies for tile kt (a scalar load)
  auto tile_block = [&](int kt) -> int { return bt[min(kt * NB + my_bi, nblk - 1)]; };
  // Byte offsets of the bf16 granules: consecutive cache blocks are
  // blk_bytes apart, this KV head's granule head_bytes into its block (both
  // below 2^32 for any head count the shape check admits).
  const unsigned blk_bytes = (unsigned)a.hkv * (unsigned)(BLK * 2);
  const unsigned head_bytes = (unsigned)g * (unsigned)(BLK * 2);
  // which: 1 the K slices, 2 the V slices, 3 both
  auto copy_tile = [&](int blk_raw, int stage, int which = 3) -> int {
    const unsigned blk = (unsigned)blk_raw < (unsigned)a.nb ? (unsigned)blk_raw : 0u;
    if constexpr (CT == 2) {
      if (pi < NB * D) {
        const size_t gran = ((size_t)blk * a.hkv + g) * (kBlock * D) + (size_t)(pi % D) * 16;
        if (which & 1) kraw = *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint8_t*>(a.k_cache) + gran);
        if (which & 2) vraw = *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint8_t*>(a.v_cache) + gran);
      }
      (void)stage;
      return blk_raw;
    }
    const uint64_t gran = (uint64_t)blk * blk_bytes + head_bytes;
    const uint8_t* kbase = reinterpret_cast<const uint8_t*>(a.k_cache) + gran;
    const uint8_t* vbase = reinterpret_cast<const uint8_t*>(a.v_cache) + gran;
#pragma unroll
    for (int u = 0; u < WI; ++u) {
      const int ii = wave * WI + u;                 // 1 KB slice of the tile
      const int cq = (ii * 64) % (BLK / 8) + lane;  // 16-byte piece within the block
      // K: piece (chunk c, slot) <- key swap23(slot) of chunk c
      const int kc = cq >> 4, ks16 = cq & 15;
      const int kkey = (ks16 & 3) | ((ks16 & 4) << 1) | ((ks16 & 8) >> 1);
      if (which & 1) global_to_lds16(kbase, (unsigned)((kc * 16 + kkey) * 16), sk + stage * TILE + ii * 512);
      // V: piece (half vh, row d) <- keys 8vh..8vh+7 of V^T row d
      const int vh = cq / D, vd = cq % D;
      if (which & 2) global_to_lds16(vbase, (unsigned)((vd * kBlock + vh * 8) * 2), sv + stage * TILE + ii * 512);
    }
    return blk_raw;
  };
  // After this wave's copy of tile kt has landed: zero its V entries of keys
  // >= L (the tail of the sequence's last block, and clamped blocks), or fill
  // them with NaN when the block id was invalid.
  // the first tile whose block copied by this wave holds keys >= L
  const int nfull = L / kBlock;
  const int kt_fix_from = nfull <= my_bi ? 0 : (nfull - my_bi + NB - 1) / NB;
  auto fix_tile = [&](int kt, int blk_raw, int stage) {
    const bool bad = (unsigned)blk_raw >= (unsigned)a.nb;
    if (kt < kt_fix_from && !bad) return;
    const int nvalid_blk = L - (kt * NB + my_bi) * kBlock;
#pragma unroll
    for (int u = 0; u < WI; ++u) {
      const int ii = wave * WI + u;
      const int cq = (ii * 64) % (BLK / 8) + lane;
      const int vh = cq / D;
      uint16_t* piece = sv + stage * TILE + ii * 512 + lane * 8;
      const int nvalid = nvalid_blk - 8 * vh;
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (bad || e >= nvalid) piece[e] = bad ? (uint16_t)0x7FC0 : (uint16_t)0;
    }
  };
  // fp8: once this lane's pieces of tile kt have landed, store them as bf16
  // in the tile's stage -- K piece q (keys 2j, 2j+1 of chunk c = q/8, j = q%8)
  // at the slots of those keys, V piece q (V^T row q, 16 keys) as its two key
  // halves -- with the V entries of keys >= L zeroed (NaN for a bad block id)
  auto store_fp8_tile = [&](int kt, int blk_raw, int stage) {
    if (pi >= NB * D) return;
    const int b = pi / D, q = pi % D;
    uint8_t* kdst = reinterpret_cast<uint8_t*>(sk + stage * TILE + b * BLK);
    uint8_t* vdst = reinterpret_cast<uint8_t*>(sv + stage * TILE + b * BLK);
    const int c = q >> 3, j = q & 7;
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      const int key = 2 * j + x;
      const int slot = (key & 3) | ((key & 4) << 1) | ((key & 8) >> 1);  // the slot that holds this key
      const u32x4 w = {Tr<2>::cvt2(kraw[2 * x], false), Tr<2>::cvt2(kraw[2 * x], true),
                       Tr<2>::cvt2(kraw[2 * x + 1], false), Tr<2>::cvt2(kraw[2 * x + 1], true)};
      *reinterpret_cast<u32x4*>(kdst + (c * 16 + slot) * 16) = w;
    }
    const int nvalid = L - (kt * NB + b) * kBlock;
    const bool bad = !(blk_raw >= 0 && blk_raw < a.nb);
#pragma unroll
    for (int vh = 0; vh < 2; ++vh) {
      u32x4 w = {Tr<2>::cvt2(vraw[2 * vh], false), Tr<2>::cvt2(vraw[2 * vh], true),
                 Tr<2>::cvt2(vraw[2 * vh + 1], false), Tr<2>::cvt2(vraw[2 * vh + 1], true)};
      if (bad || nvalid < 8 * vh + 8) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const unsigned keep = (unsigned)(!bad && 8 * vh + e < nvalid);
          const unsigned fill = bad ? 0x7FC0u : 0u;
          const unsigned sh = 16 * (e & 1);
          const unsigned cur = (w[e >> 1] >> sh) & 0xFFFFu;
          w[e >> 1] = (w[e >> 1] & ~(0xFFFFu << sh)) | ((keep ? cur : fill) << sh);
        }
      }
      *reinterpret_cast<u32x4*>(vdst + (vh * D + q) * 16) = w;
    }
  };

  f32x16 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
  const float c = a.scale_log2;
  const float thresh = 8.f / c;  // 8 in log2 units, in raw score units
  float m_ref = -INFINITY;       // reference maximum, raw score units
  float l = 0.f;
  // K operand row of this lane: slot n%16 of block n/16 of a 32-key tile
  const int koff = (n >> 4) * BLK + (n & 15) * 8;

  // the Q fragments (ordinary loads) land before any tile copy is issued, so
  // that no wait inside the loop is ever needed for them
  MPA_WAIT_VMCNT(0);
  // Stages rotate: tile kt sits in stage kt % STAGES, kept as counters that
  // step each iteration (s_use for tile kt, s_next for kt+1, s_copy for
  // kt+AHEAD).  The block ids of the tiles copied but not yet fixed up wait
  // in ids[]: ids[0] is tile kt+1's, ids[AHEAD-1] tile kt+AHEAD's.
  auto wrap = [](int x) { return x >= STAGES ? x - STAGES : x; };
  int s_use = kt_begin % STAGES;
  int ids[AHEAD];
  // prologue: the split's first AHEAD tiles in flight, its first published
#pragma unroll
  for (int k = 0; k < AHEAD; ++k) ids[k] = copy_tile(tile_block(kt_begin + k), wrap(s_use + k));
  // each iteration loads the block id the next one copies (see below)
  int next_blk = tile_block(kt_begin + AHEAD);
  if constexpr (CT == 2) {
    MPA_WAIT_VMCNT(0);
    store_fp8_tile(kt_begin, ids[0], s_use);
  } else {
    MPA_WAIT_VMCNT(2 * WI * (STAGES - 2));
    fix_tile(kt_begin, ids[0], s_use);
  }
#pragma unroll
  for (int k = 0; k + 1 < AHEAD; ++k) ids[k] = ids[k + 1];
  __syncthreads();

  // Waves w and w + WAVES/2 share a SIMD and run the same phases; the issue
  // arbiter favours the older one, so the upper half finishes each tile
  // last and the lower half waits for it at the barrier.  Raising the upper
  // half's priority shortens that critical path.
  if (WAVES == 8 && wave >= WAVES / 2) __builtin_amdgcn_s_setprio(1);
  for (int kt = kt_begin; kt < ntile; ++kt) {
    // tile kt+STAGES-1 is copied into the stage tile kt-1 used (all waves are
    // past it): by an active wave between its QK products, so that the
    // copy instructions are issued while the matrix core is busy
    const int cblk = next_blk;
    ids[AHEAD - 1] = cblk;
    const int s_next = wrap(s_use + 1), s_copy = wrap(s_use + AHEAD);
    const int key_base = kt * BN;
    if (wave_active && key_base < w_kend) {
      const uint16_t* K = sk + s_use * TILE;
      const uint16_t* V = sv + s_use * TILE;
      // The K operands of the first KUP k-steps are read from LDS before the
      // first MFMA, and each later k-step's KUP steps ahead of its use, each
      // into registers of its own: the reads' latency overlaps instead of
      // separating every MFMA pair (left to itself the scheduler reuses one
      // register quad for them all), and the eight waves do not queue all
      // of the tile's K reads at the LDS at once when the tile is published.
      constexpr int KUP = 3;
      bf16x8 kf[2][KS];
      auto read_k = [&](int ks) {
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
          kf[rt][ks] =
              __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(K + 2 * rt * BLK + koff + (2 * ks + h) * 128));
      };
#pragma unroll
      for (int ks = 0; ks < KUP; ++ks) read_k(ks);
      __builtin_amdgcn_sched_barrier(0);
      f32x16 st[2];
#pragma unroll
      for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int r = 0; r < 16; ++r) st[rt][r] = 0.f;
      // V operands: the reads of cache block t of the tile are issued after
      // k-step KS-4+t of the QK product, into registers whose K operands
      // that step has consumed.  Spread over the last four k-steps, the
      // eight waves' V reads do not all reach the LDS at once when the
      // products end, and they land while the softmax runs.
      bf16x8 vf[4][DT];
      // the two 32-key row tiles are independent accumulation chains:
      // interleave them so back-to-back MFMAs never wait on each other
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
          st[rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[rt][ks], qf[ks], st[rt], 0, 0, 0);
        if (ks + KUP < KS) {
          __builtin_amdgcn_sched_barrier(0);
          read_k(ks + KUP);
          __builtin_amdgcn_sched_barrier(0);
        }
        // the next tile copy: bf16 tiles as their K slices after the third
        // k-step and their V slices after k-step KS/2 (the same step at
        // D = 64); fp8 pieces both after the first, since they must land
        // in registers by the end of this tile
        constexpr int k_ks = CT == 0 ? 2 : 0;
        constexpr int v_ks = CT == 0 ? KS / 2 : 0;
        if (ks == k_ks || ks == v_ks) {
          __builtin_amdgcn_sched_barrier(0);
          copy_tile(cblk, s_copy, (ks == k_ks ? 1 : 0) | (ks == v_ks ? 2 : 0));
          __builtin_amdgcn_sched_barrier(0);
        }
        if (ks >= KS - 4) {
          const int t = ks - (KS - 4);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int dt = 0; dt < DT; ++dt)
            vf[t][dt] = __builtin_bit_cast(
                bf16x8, *reinterpret_cast<const u32x4*>(V + t * BLK + (h * D + n) * 8 + 32 * dt * 8));
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      // the next copy's block id: a scalar load shares the LDS wait counter
      // and may complete out of order, so issued here, after the last LDS
      // read of the tile, it only turns the PV waits into full ones, by
      // which time the V reads have long landed
      next_blk = tile_block(kt + AHEAD + 1);
      if (key_base + BN - 1 > w_min_limit) {
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int jr = r >> 2;
            const int key = key_base + 32 * rt + 16 * (jr >> 1) + 8 * h + 4 * (jr & 1) + (r & 3);
            if (key > limit) st[rt][r] = -INFINITY;
          }
      }
      // The reference maximum m_ref moves only when some score of the wave
      // exceeds it by more than thresh (probabilities stay <= 2^8).  On a
      // wave's first tile it is still -inf and is taken from the tile's row
      // maximum, but not below -2^63 in log2 units: a row whose scores there
      // are all -inf then has probabilities 0 (not 2^(-inf + inf)), and any
      // later score moves the reference.  On later tiles the probabilities are
      // formed with the current reference first, and since a score past the threshold makes its
      // probability -- and so this lane's row-sum partial -- at least 2^8
      // after bf16 rounding, the tile's maximum is taken only when some
      // lane's partial reaches 2^8.  Then S is recomputed from the operands
      // still in LDS (the same products in the same order, so the same
      // values), the reference is moved if the threshold is passed, and the
      // probabilities are formed again.  Either way the probabilities, the
      // row sums and the reference are those of taking the maximum on every
      // tile.
      auto row_max = [&](const f32x16 (&s)[2]) -> float {
        float m4[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
          for (int r = 0; r < 16; ++r) m4[r & 3] = fmaxf(m4[r & 3], s[rt][r]);
        return max_across_halves(fmaxf(fmaxf(m4[0], m4[1]), fmaxf(m4[2], m4[3])));
      };
      auto move_reference = [&](float mx) {
        const float m_new = fmaxf(m_ref, mx);
        const float alpha = m_new == -INFINITY ? 1.f : exp2_fast((m_ref - m_new) * c);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[dt] *= alpha;
        l *= alpha;
        m_ref = m_new;
      };
      // P^T in bf16; the row sum adds the rounded values the PV product
      // uses (four independent partial sums, two probabilities per dot2).
      bf16x8 pb[4];
      float l4[4];
      auto make_p = [&](const f32x16 (&s)[2], float mc) {
#pragma unroll
        for (int k = 0; k < 4; ++k) l4[k] = 0.f;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
#pragma unroll
          for (int e = 0; e < 8; ++e) pb[t][e] = (__bf16)exp2_fast(fmaf(s[t >> 1][8 * (t & 1) + e], c, -mc));
          const u32x4 w = __builtin_bit_cast(u32x4, pb[t]);
#pragma unroll
          for (int k = 0; k < 4; ++k) l4[k] = add_bf16_pair(w[k], l4[k]);
        }
      };
      if (kt == kt_begin) {
        const float mx = row_max(st);
        if (__any(mx > m_ref + thresh)) move_reference(mx);
        m_ref = fmaxf(m_ref, -0x1p60f * thresh);
      }
      make_p(st, m_ref * c);
      if (kt != kt_begin && __any(!((l4[0] + l4[1]) + (l4[2] + l4[3]) < 256.f))) {
        asm volatile("" ::: "memory");
        f32x16 s2[2];
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
          for (int r = 0; r < 16; ++r) s2[rt][r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
          for (int rt = 0; rt < 2; ++rt)
            s2[rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                __builtin_bit_cast(bf16x8,
                                   *reinterpret_cast<const u32x4*>(K + 2 * rt * BLK + koff + (2 * ks + h) * 128)),
                qf[ks], s2[rt], 0, 0, 0);
        if (key_base + BN - 1 > w_min_limit) {
#pragma unroll
          for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              const int jr = r >> 2;
              const int key = key_base + 32 * rt + 16 * (jr >> 1) + 8 * h + 4 * (jr & 1) + (r & 3);
              if (key > limit) s2[rt][r] = -INFINITY;
            }
        }
        const float mx = row_max(s2);
        if (__any(mx > m_ref + thresh)) {
          move_reference(mx);
          make_p(s2, m_ref * c);
        }
      }
      const float mc = m_ref * c;
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[t][dt], pb[t], o[dt], 0, 0, 0);
      l += (l4[0] + l4[1]) + (l4[2] + l4[3]);
      if (key_base == 0 && w_min_limit < kFewKeys) {
        // A row that sees at most kFewKeys keys has them all in tile 0, and
        // its output rests on so few probabilities that their bf16 rounding
        // does not average out.  For such waves the tile is passed a second
        // time with the remainder p - bf16(p): S is recomputed from the
        // operands still in LDS (the same products in the same order, so
        // the same values), and the remainder goes into the PV product and
        // the row sum, which carries P to about 16 bits.  The empty asm
        // keeps the compiler from holding the first pass's fragments live
        // across the tile for this rare branch.
        asm volatile("" ::: "memory");
        f32x16 s2[2];
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
          for (int r = 0; r < 16; ++r) s2[rt][r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
          for (int rt = 0; rt < 2; ++rt)
            s2[rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                __builtin_bit_cast(bf16x8,
                                   *reinterpret_cast<const u32x4*>(K + 2 * rt * BLK + koff + (2 * ks + h) * 128)),
                qf[ks], s2[rt], 0, 0, 0);
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int jr = r >> 2;
            const int key = 32 * rt + 16 * (jr >> 1) + 8 * h + 4 * (jr & 1) + (r & 3);
            if (key > limit) s2[rt][r] = -INFINITY;
          }
        float r4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          bf16x8 plo;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float pe = exp2_fast(fmaf(s2[t >> 1][8 * (t & 1) + e], c, -mc));
            plo[e] = (__bf16)(pe - (float)(__bf16)pe);
          }
          const u32x4 w = __builtin_bit_cast(u32x4, plo);
#pragma unroll
          for (int k = 0; k < 4; ++k) r4[k] = add_bf16_pair(w[k], r4[k]);
#pragma unroll
          for (int dt = 0; dt < DT; ++dt)
            o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(V + t * BLK + (h * D + n) * 8 + 32 * dt * 8)),
                plo, o[dt], 0, 0, 0);
        }
        l += (r4[0] + r4[1]) + (r4[2] + r4[3]);
      }
    } else {
      copy_tile(cblk, s_copy);
      next_blk = tile_block(kt + AHEAD + 1);
      // The block id is a scalar load, which shares the LDS counter and may
      // return out of order.  Left pending on this path, it would reach the
      // active path's join as well, and every wait for the K operand reads
      // there would become a wait for all of them.
      MPA_WAIT_LGKMCNT(0);
    }
    if constexpr (CT == 2) {
      // this lane's pieces of tile kt+1 (the only loads in flight)
      MPA_WAIT_VMCNT(0);
      store_fp8_tile(kt + 1, ids[0], s_next);
    } else {
      // this wave's part of tile kt+1 has landed once only the copies issued
      // after it (tiles kt+2 .. kt+STAGES-1) remain in flight
      MPA_WAIT_VMCNT(2 * WI * (STAGES - 2));
      fix_tile(kt + 1, ids[0], s_next);
    }
#pragma unroll
    for (int k = 0; k + 1 < AHEAD; ++k) ids[k] = ids[k + 1];
    s_use = s_next;
    __syncthreads();
  }
  MPA_WAIT_VMCNT(0);  // drain the clamped copies past the end

  const float lt = l + __shfl_xor(l, 32);
  if (!wave_active || !row_ok) return;
  if (nsplit > 1) {  // partial result of this KV split, merged by prefill_merge_kernel
    const size_t slot = ((size_t)p.item_base[j] + (size_t)split * C + i) * a.hq + head;
    float* wo = a.ws_o + slot * D;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int jb = 0; jb < 4; ++jb) {
        const f32x4 v4 = {o[dt][4 * jb], o[dt][4 * jb + 1], o[dt][4 * jb + 2], o[dt][4 * jb + 3]};
        *reinterpret_cast<f32x4*>(wo + 32 * dt + 8 * jb + 4 * h) = v4 * a.v_scale;
      }
    if (h == 0) {
      a.ws_ml[slot * 2] = m_ref * c;
      a.ws_ml[slot * 2 + 1] = lt;
    }
    return;
  }
  const float inv = a.v_scale / lt;
  uint16_t* out = reinterpret_cast<uint16_t*>(a.out) + ((size_t)(t0 + i) * a.hq + head) * D;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) {
      f32x4 v4 = {o[dt][4 * jb], o[dt][4 * jb + 1], o[dt][4 * jb + 2], o[dt][4 * jb + 3]};
      Tr<0>::store4(out + 32 * dt + 8 * jb + 4 * h, v4 * inv);
    }
  if (a.lse && h == 0) a.lse[(size_t)(t0 + i) * a.hq + head] = (m_ref * c + log2f(lt)) * kLn2;
}

// Stores chunk c (8 consecutive bf16 elements, packed) of a new key row and
// of a new value row into slot `slot` of cache head `head` of an fp8 cache:
// each element x becomes the E4M3 code of x * (1 / scale).
template <int D, bool NT>
__device__ inline void store_fp8_chunk(const AppendArgs& a, size_t head, int c, int slot, u32x4 kw, u32x4 vw) {
  constexpr int NC = D / 8;
  float kx[8], vx[8];
  Tr<0>::unpack(kw, kx);
  Tr<0>::unpack(vw, vx);
  u32x2 kc = {0u, 0u};
#pragma unroll
  for (int e = 0; e < 8; ++e) kc[e / 4] |= f32_to_e4m3(kx[e] * a.inv_k_scale) << (8 * (e % 4));
  st_token<NT>(reinterpret_cast<uint8_t*>(a.k_cache) + ((head * NC + c) * kBlock + slot) * 8, kc);
  uint8_t* vc = reinterpret_cast<uint8_t*>(a.v_cache) + (head * D + c * 8) * kBlock + slot;
#pragma unroll
  for (int e = 0; e < 8; ++e) st_token<NT>(vc + e * kBlock, (uint8_t)f32_to_e4m3(vx[e] * a.inv_v_scale));
}

// ---------------------------------------------------------------------------
// Append of the sequences that add one token: one wave per token, whose
// sequence comes from the kernel-argument plan and its block id from one
// scalar load; the wave then copies the token's Hkv*d key elements as 16-byte
// chunks and its value elements into the V^T rows of the slot, issuing the
// loads of up to 4 chunks per lane before their stores.
template <int DT, int D, bool NT>
__global__ __launch_bounds__(256) void append_kernel(AppendArgs a, AppendPlan p) {
  using T = Tr<DT>;
  using E = typename T::Elem;
  constexpr int X = T::X;
  constexpr int NC = D / X;
  constexpr int U = 4;
  const int lane = threadIdx.x & 63;
  const int tok = blockIdx.x * kWavesPerGroup + wave_uniform(threadIdx.x >> 6);
  if (tok >= p.n_seqs) return;
  const int s = p.seq[tok];
  const int t = p.row[tok];
  const int pos = p.pos[tok];
  const int blk = a.block_tables[(size_t)s * a.mb + pos / kBlock];
  if (blk < 0 || blk >= a.nb) return;
  const int slot = pos % kBlock;
  const int nchunk = a.hkv * NC;
  if constexpr (DT == 2) {
    // fp8 cache: each bf16 element of the new rows is stored as the E4M3
    // code of x * (1 / scale); a lane handles 8 consecutive elements
    const uint16_t* kn = reinterpret_cast<const uint16_t*>(a.k_new) + (size_t)t * a.hkv * D;
    const uint16_t* vn = reinterpret_cast<const uint16_t*>(a.v_new) + (size_t)t * a.hkv * D;
    for (int ci = lane; ci < nchunk; ci += 64) {
      const int h = ci / NC, c = ci - h * NC;
      store_fp8_chunk<D, NT>(a, (size_t)blk * a.hkv + h, c, slot, *reinterpret_cast<const u32x4*>(kn + h * D + c * 8),
                         *reinterpret_cast<const u32x4*>(vn + h * D + c * 8));
    }
  } else {
  for (int c0 = 0; c0 < nchunk; c0 += 64 * U) {
    u32x4 kv[U];
    E vv[U][X];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int ci = min(c0 + 64 * u + lane, nchunk - 1);
      const int h = ci / NC, c = ci - h * NC;
      const size_t src = ((size_t)t * a.hkv + h) * D + c * X;
      kv[u] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const E*>(a.k_new) + src);
#pragma unroll
      for (int e = 0; e < X; ++e) vv[u][e] = reinterpret_cast<const E*>(a.v_new)[src + e];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int ci = c0 + 64 * u + lane;
      if (ci >= nchunk) continue;
      const int h = ci / NC, c = ci - h * NC;
      const size_t head = (size_t)blk * a.hkv + h;
      st_token<NT>(reinterpret_cast<E*>(a.k_cache) + ((head * NC + c) * kBlock + slot) * X, kv[u]);
      E* vc = reinterpret_cast<E*>(a.v_cache) + (head * D + c * X) * kBlock + slot;
#pragma unroll
      for (int e = 0; e < X; ++e) st_token<NT>(vc + e * kBlock, vv[u][e]);
    }
  }
  }
}

// Rotary embedding of 16-byte chunk c of one head row (rotate-half form):
// element i < half pairs with i + half; with the position's angle row cs
// (cos, sin interleaved per pair), y_i = x_i cos - x_{i+half} sin and
// y_{i+half} = x_{i+half} cos + x_i sin, and elements >= 2*half are copied.
// half is a multiple of the chunk's element count.  Each product and each
// sum is rounded to f32 (no fused multiply-add), then the result to the
// storage type.
template <int DT>
__device__ inline u32x4 rope_chunk(const typename Tr<DT>::Elem* row, int c, int half, const float* cs) {
#pragma clang fp contract(off)
  using T = Tr<DT>;
  constexpr int X = T::X;
  // no branch, so that a lane's loads for several chunks are in flight together
  const int e0 = c * X;
  const bool turned = e0 < 2 * half, lo = e0 < half;
  const u32x4 w = *reinterpret_cast<const u32x4*>(row + e0);
  const u32x4 wp = *reinterpret_cast<const u32x4*>(row + (!turned ? e0 : lo ? e0 + half : e0 - half));
  const float* ang = cs + 2 * (!turned ? 0 : lo ? e0 : e0 - half);
  float x[X], xp[X], y[X];
  T::unpack(w, x);
  T::unpack(wp, xp);
#pragma unroll
  for (int e = 0; e < X; ++e) {
    const float a = x[e] * ang[2 * e];
    const float b = xp[e] * ang[2 * e + 1];
    y[e] = lo ? a - b : a + b;
  }
  u32x4 r = T::pack(y);
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = turned ? r[i] : w[i];
  return r;
}

// Rotates the hq head rows of one token's query in place (angle row cs): a
// lane holds the two chunks of a rotated pair and the token's angles for
// them, loaded once, and goes over heads, four at a time with their loads
// issued together.  The element arithmetic is rope_chunk's.
template <int DT, int D>
__device__ inline void rotate_query(typename Tr<DT>::Elem* q, int hq, int half, const float* cs, int lane) {
#pragma clang fp contract(off)
  using T = Tr<DT>;
  constexpr int X = T::X;
  constexpr int U = 4;
  const int np = half / X;                    // chunk pairs of a head row
  const int hp = min(64 / np, hq);            // heads per pass
  const int hl = lane / np, c = lane - hl * np;
  if (hl >= hp) return;
  float co[X], si[X];
#pragma unroll
  for (int e = 0; e < X; ++e) {
    co[e] = cs[2 * (c * X + e)];
    si[e] = cs[2 * (c * X + e) + 1];
  }
  for (int h0 = hl; h0 < hq; h0 += U * hp) {
    u32x4 lo[U], hi[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const auto* row = q + (size_t)min(h0 + u * hp, hq - 1) * D + c * X;
      lo[u] = *reinterpret_cast<const u32x4*>(row);
      hi[u] = *reinterpret_cast<const u32x4*>(row + half);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (h0 + u * hp >= hq) break;
      float x[X], y[X], xr[X], yr[X];
      T::unpack(lo[u], x);
      T::unpack(hi[u], y);
#pragma unroll
      for (int e = 0; e < X; ++e) {
        const float a = x[e] * co[e], b = y[e] * si[e];
        const float d = y[e] * co[e], f = x[e] * si[e];
        xr[e] = a - b;
        yr[e] = d + f;
      }
      auto* row = q + (size_t)(h0 + u * hp) * D + c * X;
      *reinterpret_cast<u32x4*>(row) = T::pack(xr);
      *reinterpret_cast<u32x4*>(row + half) = T::pack(yr);
    }
  }
}

// Append for sequences that add several tokens: one wave per (cache block,
// KV head) writes every new token of the block.  K pieces (chunk c, slot t)
// are taken slot-fastest, so the stores of a chunk row are one contiguous
// run; each lane gathers D / 64 dims of every token, so that a block's V^T
// row of a dim (16 slots) is stored at once when the block is written whole
// (element by element for the slots of a partly written block).  The bits
// stored are the plain append's.
// ROPE: the keys are rotated on the way, and the launch's further waves, one
// per new token, rotate the query rows.  3,001 tokens of 32 / 8 heads of 128
// (74 MB): 17.6 us; a wave per token for all three, with the single-token
// append's scattered V elements and each query chunk loaded twice, took 31.8.
template <int DT, int D, bool ROPE>
__global__ __launch_bounds__(256) void append_block_kernel(AppendArgs a, AppendBlockPlan p, RopeArgs rope) {
  constexpr int RT = DT == 2 ? 0 : DT;  // new rows: bf16 beside an fp8 cache
  using NE = typename Tr<RT>::Elem;
  using CE = typename Tr<DT>::Elem;
  constexpr int X = Tr<DT>::X;           // elements per K chunk of the cache
  constexpr int NC = D / X;
  constexpr int DPL = D / 64;            // V dims per lane
  static_assert((NC * kBlock) % 64 == 0, "K pieces fill whole passes of the wave");
  const int lane = threadIdx.x & 63;
  const int w = blockIdx.x * kWavesPerGroup + wave_uniform(threadIdx.x >> 6);
  const int unit = w / a.hkv, h = w - unit * a.hkv;
  if (unit >= p.unit_start[p.n_seqs]) {
    if constexpr (ROPE) {
      const int tok = w - p.unit_start[p.n_seqs] * a.hkv;
      if (tok >= p.tok_start[p.n_seqs]) return;
      const int j = upper_index(p.tok_start, p.n_seqs, tok);
      const int k = tok - p.tok_start[j];
      rotate_query<RT, D>(reinterpret_cast<NE*>(rope.q) + (size_t)(p.row0[j] + k) * rope.hq * D, rope.hq, rope.half,
                          rope.cos_sin + (size_t)(p.pos0[j] + k) * rope.half * 2, lane);
    }
    return;
  }
  const int j = upper_index(p.unit_start, p.n_seqs, unit);
  const int first = p.pos0[j], end = p.pos0[j] + p.ntok[j];  // new positions [first, end)
  const int b = first / kBlock + (unit - p.unit_start[j]);   // cache block index in the sequence
  const int s0 = max(first, b * kBlock) - b * kBlock;          // its new slots [s0, s1)
  const int s1 = min(end, b * kBlock + kBlock) - b * kBlock;
  const int blk = a.block_tables[(size_t)p.seq[j] * a.mb + b];
  if (blk < 0 || blk >= a.nb) return;
  const size_t head = (size_t)blk * a.hkv + h;
  const size_t rstride = (size_t)a.hkv * D;                    // elements between token rows
  const int row_s0 = p.row0[j] + b * kBlock + s0 - first;      // query row of slot s0
  const NE* kn = reinterpret_cast<const NE*>(a.k_new) + (size_t)h * D;
  const NE* vn = reinterpret_cast<const NE*>(a.v_new) + (size_t)h * D;

  // K: piece (chunk c, slot t) of the block from token row row_s0 + t - s0;
  // all of a lane's loads are issued before its stores
  constexpr int KP = NC * kBlock / 64;  // pieces per lane
  u32x4 kw[KP];
#pragma unroll
  for (int u = 0; u < KP; ++u) {
    const int pc = 64 * u + lane, c = pc / kBlock, t = pc % kBlock;
    const int row = row_s0 + min(max(t, s0), s1 - 1) - s0;  // slots outside [s0, s1) reload a valid row
    if constexpr (ROPE)
      kw[u] = rope_chunk<RT>(kn + (size_t)row * rstride, c, rope.half,
                             rope.cos_sin + (size_t)(first + row - p.row0[j]) * rope.half * 2);
    else
      kw[u] = *reinterpret_cast<const u32x4*>(kn + (size_t)row * rstride + c * X);
  }
#pragma unroll
  for (int u = 0; u < KP; ++u) {
    const int pc = 64 * u + lane, c = pc / kBlock, t = pc % kBlock;
    if (t < s0 || t >= s1) continue;
    CE* dst = reinterpret_cast<CE*>(a.k_cache) + ((head * NC + c) * kBlock + t) * X;
    if constexpr (DT == 2) {
      float kx[8];
      Tr<0>::unpack(kw[u], kx);
      u32x2 kc = {0u, 0u};
#pragma unroll
      for (int e = 0; e < 8; ++e) kc[e / 4] |= f32_to_e4m3(kx[e] * a.inv_k_scale) << (8 * (e % 4));
      *reinterpret_cast<u32x2*>(dst) = kc;
    } else {
      *reinterpret_cast<u32x4*>(dst) = kw[u];
    }
  }

  // V: this lane's dims d = DPL * lane + i of every new token of the block
  // (slots outside [s0, s1) reload a valid row, so that all loads are in
  // flight before the first is converted)
  NE raw[kBlock][DPL];
#pragma unroll
  for (int t = 0; t < kBlock; ++t) {
    const NE* src = vn + (size_t)(row_s0 + min(max(t, s0), s1 - 1) - s0) * rstride + DPL * lane;
#pragma unroll
    for (int i = 0; i < DPL; ++i) raw[t][i] = src[i];
  }
  CE vals[kBlock][DPL];
#pragma unroll
  for (int t = 0; t < kBlock; ++t)
#pragma unroll
    for (int i = 0; i < DPL; ++i) {
      if constexpr (DT == 2)
        vals[t][i] = (uint8_t)f32_to_e4m3(__uint_as_float((unsigned)raw[t][i] << 16) * a.inv_v_scale);
      else
        vals[t][i] = raw[t][i];
    }
  CE* vdst = reinterpret_cast<CE*>(a.v_cache) + (head * D + DPL * lane) * kBlock;
  if (s0 == 0 && s1 == kBlock) {
#pragma unroll
    for (int i = 0; i < DPL; ++i) {
      constexpr int PER = 16 / sizeof(CE);  // elements per 16-byte store
#pragma unroll
      for (int q = 0; q < kBlock / PER; ++q) {
        CE piece[PER];
#pragma unroll
        for (int e = 0; e < PER; ++e) piece[e] = vals[q * PER + e][i];
        *reinterpret_cast<u32x4*>(vdst + i * kBlock + q * PER) = __builtin_bit_cast(u32x4, piece);
      }
    }
  } else {
#pragma unroll
    for (int t = 0; t < kBlock; ++t)
      if (t >= s0 && t < s1)
#pragma unroll
        for (int i = 0; i < DPL; ++i) vdst[i * kBlock + t] = vals[t][i];
  }
}

// Append with the rotary embedding of the sequences that add one token: one
// wave per new token at position pos.
// The wave rotates the token's query row (all Hq heads, in place), writes
// its rotated key row into the cache and copies its value row, as the plain
// append does.  A head's chunks all fall in one pass of the 64 lanes (D / X
// divides 64), so a pass loads every partner chunk before it stores any.
template <int DT, int D, bool NT>
__global__ __launch_bounds__(256) void rope_append_kernel(AppendArgs a, AppendPlan p, RopeArgs r) {
  constexpr int RT = DT == 2 ? 0 : DT;  // queries and new rows: bf16 beside an fp8 cache
  using T = Tr<RT>;
  using E = typename T::Elem;
  constexpr int X = T::X;
  constexpr int NC = D / X;
  static_assert(64 % NC == 0, "a head row's chunks fit one pass of the wave");
  const int lane = threadIdx.x & 63;
  const int tok = blockIdx.x * kWavesPerGroup + wave_uniform(threadIdx.x >> 6);
  if (tok >= p.n_seqs) return;
  const int s = p.seq[tok];
  const int t = p.row[tok];
  const int pos = p.pos[tok];
  const float* cs = r.cos_sin + (size_t)pos * r.half * 2;

  rotate_query<RT, D>(reinterpret_cast<E*>(r.q) + (size_t)t * r.hq * D, r.hq, r.half, cs, lane);

  const int blk = a.block_tables[(size_t)s * a.mb + pos / kBlock];
  if (blk < 0 || blk >= a.nb) return;
  const int slot = pos % kBlock;
  const E* kn = reinterpret_cast<const E*>(a.k_new) + (size_t)t * a.hkv * D;
  const E* vn = reinterpret_cast<const E*>(a.v_new) + (size_t)t * a.hkv * D;
  for (int ci = lane; ci < a.hkv * NC; ci += 64) {
    const int h = ci / NC, c = ci - h * NC;
    const size_t head = (size_t)blk * a.hkv + h;
    if constexpr (DT == 2) {
      // fp8 cache: the rotated key, rounded to bf16, is quantized like a plain new key
      store_fp8_chunk<D, NT>(a, head, c, slot, rope_chunk<RT>(kn + h * D, c, r.half, cs),
                         *reinterpret_cast<const u32x4*>(vn + h * D + c * X));
      continue;
    }
    st_token<NT>(reinterpret_cast<E*>(a.k_cache) + ((head * NC + c) * kBlock + slot) * X,
              rope_chunk<RT>(kn + h * D, c, r.half, cs));
    E vv[X];
#pragma unroll
    for (int e = 0; e < X; ++e) vv[e] = vn[h * D + c * X + e];
    E* vc = reinterpret_cast<E*>(a.v_cache) + (head * D + c * X) * kBlock + slot;
#pragma unroll
    for (int e = 0; e < X; ++e) st_token<NT>(vc + e * kBlock, vv[e]);
  }
}

template <template <int, int> class F, typename... Args>
hipError_t dispatch(int dtype, int head_dim, Args&&... args) {
  if (dtype == 0 && head_dim == 128) return F<0, 128>::run(args...);
  if (dtype == 0 && head_dim == 64) return F<0, 64>::run(args...);
  if (dtype == 1 && head_dim == 128) return F<1, 128>::run(args...);
  if (dtype == 1 && head_dim == 64) return F<1, 64>::run(args...);
  if (dtype == 2 && head_dim == 128) return F<2, 128>::run(args...);
  if (dtype == 2 && head_dim == 64) return F<2, 64>::run(args...);
  return hipErrorInvalidValue;
}

template <int DT, int D>
struct AppendL {
  static hipError_t run(const AppendArgs& a, const AppendPlan& p, hipStream_t stream) {
    const int tokens = p.n_seqs;
    if (tokens == 0) return hipSuccess;
    const dim3 grid((tokens + kWavesPerGroup - 1) / kWavesPerGroup), block(64 * kWavesPerGroup);
    if (DT == 0 || a.nt)
      hipLaunchKernelGGL((append_kernel<DT, D, true>), grid, block, 0, stream, a, p);
    else
      hipLaunchKernelGGL((append_kernel<DT, D, DT == 0>), grid, block, 0, stream, a, p);
    return hipGetLastError();
  }
};

template <int DT, int D>
struct AppendBlockL {
  static hipError_t run(const AppendArgs& a, const AppendBlockPlan& p, const RopeArgs* rope, hipStream_t stream) {
    const long waves = (long)p.unit_start[p.n_seqs] * a.hkv + (rope ? p.tok_start[p.n_seqs] : 0);
    if (waves == 0) return hipSuccess;
    const dim3 grid((unsigned)((waves + kWavesPerGroup - 1) / kWavesPerGroup)), block(64 * kWavesPerGroup);
    if (rope)
      hipLaunchKernelGGL((append_block_kernel<DT, D, true>), grid, block, 0, stream, a, p, *rope);
    else
      hipLaunchKernelGGL((append_block_kernel<DT, D, false>), grid, block, 0, stream, a, p, RopeArgs{});
    return hipGetLastError();
  }
};

template <int DT, int D>
struct RopeAppendL {
  static hipError_t run(const AppendArgs& a, const AppendPlan& p, const RopeArgs& r, hipStream_t stream) {
    const int tokens = p.n_seqs;
    if (tokens == 0) return hipSuccess;
    const dim3 grid((tokens + kWavesPerGroup - 1) / kWavesPerGroup), block(64 * kWavesPerGroup);
    if (DT == 0 || a.nt)
      hipLaunchKernelGGL((rope_append_kernel<DT, D, true>), grid, block, 0, stream, a, p, r);
    else
      hipLaunchKernelGGL((rope_append_kernel<DT, D, DT == 0>), grid, block, 0, stream, a, p, r);
    return hipGetLastError();
  }
};

// Waves per streaming workgroup: bf16 and f32 caches, all that a CU holds (2
// to 4 per SIMD), so that the lockstep covers the CU; fp8 caches, whose waves
// keep even by themselves (their copies run two blocks ahead; with the
// lockstep at any distance the same time within 0.5 %), the usual four.
template <int DT, int D>
constexpr int kStreamWaves = DT == 2 ? kWavesPerGroup : 4 * decode_waves_per_simd(DT, D);

template <int DT, int D>
struct DecodeL {
  static hipError_t run(const AttnArgs& a, const DecodePlan& p, int n_items, hipStream_t stream) {
    const long units = (long)n_items * a.hkv;
    if (units == 0) return hipSuccess;
    if (p.range_blocks < 0) {
      hipLaunchKernelGGL((decode_short_kernel<DT, D>), dim3((unsigned)p.n_seqs * a.hkv), dim3(64 * kKeyWaves), 0,
                         stream, a, p);
      return hipGetLastError();
    }
    if (p.range_blocks > 0) {
      constexpr int W = kStreamWaves<DT, D>;
      const long waves = (long)p.n_ranges * a.hkv;
      hipLaunchKernelGGL((decode_kernel<DT, D, W, true>), dim3((unsigned)((waves + W - 1) / W)), dim3(64 * W), 0, stream,
                         a, p);
      return hipGetLastError();
    }
    hipLaunchKernelGGL((decode_kernel<DT, D, kWavesPerGroup, false>),
                       dim3((unsigned)((units + kWavesPerGroup - 1) / kWavesPerGroup)), dim3(64 * kWavesPerGroup), 0,
                       stream, a, p);
    return hipGetLastError();
  }
};

// Decode waves per CU.
template <int DT, int D>
struct DecodeOccupancy {
  static hipError_t run(bool stream, int* waves) {
    constexpr int W = kStreamWaves<DT, D>;
    int groups = 0;
    const hipError_t e =
        stream ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&groups, decode_kernel<DT, D, W, true>, 64 * W, 0)
               : hipOccupancyMaxActiveBlocksPerMultiprocessor(&groups, decode_kernel<DT, D, kWavesPerGroup, false>,
                                                              64 * kWavesPerGroup, 0);
    *waves = groups * (stream ? W : kWavesPerGroup);
    return e;
  }
};

template <int DT, int D>
struct MergeL {
  static hipError_t run(const AttnArgs& a, const DecodePlan& p, hipStream_t stream) {
    if (p.n_seqs == 0) return hipSuccess;
    // the wide form where a wave would go over many parts and there are few
    // (row, q head) pairs (3 rows of 128 parts, 32 heads: 6.8 us, 16.5 before;
    // 64 rows of 64 heads, one in ten with 16 parts: 8.5 wide, 6.5 not)
    int most = 0;
    for (int j = 0; j < p.n_seqs; ++j) most = std::max(most, p.item_start[j + 1] - p.item_start[j]);
    if (most >= 16 && (long)p.n_seqs * a.hq <= 1024)
      hipLaunchKernelGGL((merge_kernel<DT, D, true>), dim3(p.n_seqs, a.hq), dim3(64 * kMergeWaves), 0, stream, a, p);
    else
      hipLaunchKernelGGL((merge_kernel<DT, D, false>), dim3(p.n_seqs, (a.hq + kMergeWaves - 1) / kMergeWaves),
                         dim3(64 * kMergeWaves), 0, stream, a, p);
    return hipGetLastError();
  }
};

constexpr int kPrefillWaves = 8;   // waves per bf16 prefill workgroup
constexpr int kPrefillStages = 3;  // LDS ring depth of the bf16 prefill kernel

template <int CT, int D, int WAVES, int STAGES>
hipError_t launch_prefill_mfma(const AttnArgs& a, const PrefillPlan& p, int n_tiles, hipStream_t stream) {
  constexpr size_t lds = 2 * STAGES * 4 * kBlock * D * sizeof(uint16_t);
  auto kern = prefill_mfma_kernel<CT, D, WAVES, STAGES>;
  // The ring exceeds the default 64 KB of dynamic LDS; raise the limit once
  // per device (each GPU keeps its own function attributes).
  static std::atomic<unsigned long long> ready{0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return hipErrorInvalidDevice;
  const unsigned long long bit = 1ull << (dev & 63);
  if (!(ready.load(std::memory_order_relaxed) & bit)) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    ready.fetch_or(bit, std::memory_order_relaxed);
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)n_tiles * a.hkv), dim3(64 * WAVES), lds, stream, a, p);
  return hipGetLastError();
}

// Prefill chunks: the MFMA kernel for bf16 and fp8 caches, the generic kernel
// for f32 ones.
template <int DT, int D>
struct PrefillL {
  static hipError_t run(const AttnArgs& a, const PrefillPlan& p, int n_tiles, hipStream_t stream) {
    if (n_tiles == 0) return hipSuccess;
    if constexpr (DT == 0 || DT == 2) {
      if constexpr (DT == 0) {
        // two workgroups of a two-stage ring (64 KB) to a CU, or three of a three-stage one (48 KB)
        if (p.rows == kPrefillRowsHalf) return launch_prefill_mfma<DT, D, 4, D == 64 ? 3 : 2>(a, p, n_tiles, stream);
      }
      return launch_prefill_mfma<DT, D, kPrefillWaves, kPrefillStages>(a, p, n_tiles, stream);
    } else {
      if (p.rows == kPrefillRowsKeys)
        hipLaunchKernelGGL((prefill_kernel<DT, D, true>), dim3((unsigned)n_tiles * 4 * a.hkv), dim3(64 * kKeyWaves), 0, stream, a,
                           p);
      else
        hipLaunchKernelGGL((prefill_kernel<DT, D, false>), dim3((unsigned)n_tiles * a.hkv), dim3(64 * kWavesPerGroup), 0, stream,
                           a, p);
      return hipGetLastError();
    }
  }
};

}  // namespace

hipError_t launch_append(const AppendArgs& a, const AppendPlan& p, int dtype, int head_dim, hipStream_t stream) {
  return dispatch<AppendL>(dtype, head_dim, a, p, stream);
}

hipError_t launch_append_blocks(const AppendArgs& a, const AppendBlockPlan& p, const RopeArgs* rope, int dtype,
                                int head_dim, hipStream_t stream) {
  return dispatch<AppendBlockL>(dtype, head_dim, a, p, rope, stream);
}

hipError_t launch_rope_append(const AppendArgs& a, const AppendPlan& p, const RopeArgs& r, int dtype, int head_dim,
                              hipStream_t stream) {
  return dispatch<RopeAppendL>(dtype, head_dim, a, p, r, stream);
}

int decode_wave_slots(int dtype, int head_dim, bool stream) {
  // Concurrent decode waves the device can hold: workgroups per CU at this
  // kernel's register and LDS use, times waves per workgroup, times CUs.
  // Cached per device.  Without a device: 2048, and 0 for the streaming kernel
  // (whose ranges are made for the device that runs them).
  const int none = stream ? 0 : 2048;
  static std::atomic<int> cache[64][3][2][2];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return none;
  const int di = dtype == 0 ? 0 : dtype == 1 ? 1 : 2, hi = head_dim == 128 ? 0 : 1;
  std::atomic<int>& entry = cache[dev][di][hi][stream ? 1 : 0];
  const int known = entry.load(std::memory_order_relaxed);
  if (known > 0) return known;
  int cus = 0, per_cu = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return none;
  if (dispatch<DecodeOccupancy>(dtype, head_dim, stream, &per_cu) != hipSuccess || per_cu <= 0) return none;
  const int slots = per_cu * cus;
  entry.store(slots, std::memory_order_relaxed);
  return slots;
}
hipError_t launch_decode(const AttnArgs& a, const DecodePlan& p, int n_items, int dtype, int head_dim,
                         hipStream_t stream) {
  return dispatch<DecodeL>(dtype, head_dim, a, p, n_items, stream);
}
hipError_t launch_merge(const AttnArgs& a, const DecodePlan& p, int dtype, int head_dim, hipStream_t stream) {
  return dispatch<MergeL>(dtype, head_dim, a, p, stream);
}
template <int DT, int D>
struct PrefillMergeL {
  static hipError_t run(const AttnArgs& a, const PrefillPlan& p, hipStream_t stream) {
    const int rows = p.row_start[p.n_seqs];
    if (rows == 0) return hipSuccess;
    // Four heads in turn keep the workgroups of a large launch few; one of few
    // tokens has its heads side by side (300 tokens of 16 heads in 12 splits:
    // 9.9 -> 6.6 us).
    const int per_wave = (long)rows * a.hq >= 16384 ? 4 : 1;
    const int heads = kMergeWaves * per_wave;
    hipLaunchKernelGGL((prefill_merge_kernel<DT, D>), dim3(rows, (a.hq + heads - 1) / heads),
                       dim3(64 * kMergeWaves), 0, stream, a, p, per_wave);
    return hipGetLastError();
  }
};

hipError_t launch_prefill_merge(const AttnArgs& a, const PrefillPlan& p, int dtype, int head_dim,
                                hipStream_t stream) {
  return dispatch<PrefillMergeL>(dtype, head_dim, a, p, stream);
}

hipError_t launch_prefill(const AttnArgs& a, const PrefillPlan& p, int n_tiles, int dtype, int head_dim,
                          hipStream_t stream) {
  return dispatch<PrefillL>(dtype, head_dim, a, p, n_tiles, stream);
}

}  // namespace mpa

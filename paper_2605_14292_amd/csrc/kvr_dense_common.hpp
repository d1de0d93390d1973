// Pieces shared by the fused kernels for short heads (n <= 256 bf16 tokens): wave-level
// reductions, the padded LDS row stage and its MFMA fragment reads.
#pragma once
#include "kvr_device.hpp"
#include "kvr_bounds.hpp"
#ifndef KVR_BOUNDS_FILE
#define KVR_BOUNDS_FILE 0   // (a source file that reports its bounds checks defines its number before this header)
#endif

namespace kvr {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int kDenseThreads = 256;
constexpr int kRowPitch = 272;   // bytes per staged row: 256 + 16 so that 8 consecutive rows hit distinct banks

__host__ __device__ constexpr int dense_tri_floats(int NT) { return (NT * 32) * (NT * 32 + 1) / 2; }
__host__ __device__ constexpr int dense_region_a(int NT) {
  const int tri = dense_tri_floats(NT) * 4, stage = NT * 32 * kRowPitch;
  return ((tri > stage ? tri : stage) + 15) & ~15;
}

#define KVR_DPP_MAX(v, ctrl, rmask)                                                        \
  {                                                                                        \
    const int _o = __builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), ctrl, \
                                               rmask, 0xf, false);                        \
    v = fmaxf(v, __int_as_float(_o));                                                      \
  }
#define KVR_DPP_ADD(v, ctrl, rmask)                                                            \
  {                                                                                            \
    const int _o = __builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, rmask, 0xf, false); \
    v += __int_as_float(_o);                                                                   \
  }

// Max over the wave, returned wave-uniform.  Each step is one v_max_f32 with a
// DPP source (the compiler's own lowering of a DPP move plus fmaxf costs four
// instructions a step, which is most of a pick's latency); lanes whose DPP
// source is out of range keep their value.  s_nop 1 covers the two wait states
// a DPP read needs after a VALU write of the same register.
__device__ __forceinline__ float wave_max_uniform(float v) {
  asm volatile(
      "s_nop 1\n\tv_max_f32_dpp %0, %0, %0 row_shr:1 row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 1\n\tv_max_f32_dpp %0, %0, %0 row_shr:2 row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 1\n\tv_max_f32_dpp %0, %0, %0 row_shr:4 row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 1\n\tv_max_f32_dpp %0, %0, %0 row_shr:8 row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 1\n\tv_max_f32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
      "s_nop 1\n\tv_max_f32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf"
      : "+v"(v));
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
// Orders LDS traffic between the lanes of one wave.  Lanes of a wave run in
// lock-step and the LDS pipeline is in order, but the compiler reasons per
// thread: without a fence it may forward a lane's own earlier store to a load
// that another lane has overwritten in between.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// Workgroup barrier that orders LDS traffic only.  __syncthreads() also waits until every
// global store of the wave has been acknowledged by memory, which costs microseconds after a
// burst of output rows and is needed by nobody: no wave reads what another one wrote to HBM.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}
// max(a, b) as the hardware does it (a NaN operand yields the other one), without
// the canonicalising self-max the compiler adds around fmaxf on loaded values
__device__ __forceinline__ float hw_max(float a, float b) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
// max(a, b, c), likewise
__device__ __forceinline__ float max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
// ra[lane ln] = va, rb[lane ln] = vb for wave-uniform va, vb, ln; the other lanes keep their
// values.  The lane select goes through m0 because a VALU instruction reads one SGPR only.  (va may come from a v_readfirstlane
// right before the block, which the compiler does not look into: two wait states before it is read, s_nop and s_mov.)
__device__ __forceinline__ void write_lane2(int& ra, int& rb, int va, int vb, int ln) {
  va = __builtin_amdgcn_readfirstlane(va);             // no-ops when the compiler knows them uniform
  vb = __builtin_amdgcn_readfirstlane(vb);
  ln = __builtin_amdgcn_readfirstlane(ln);
  asm("s_nop 0\n\ts_mov_b32 m0, %4\n\tv_writelane_b32 %0, %2, m0\n\tv_writelane_b32 %1, %3, m0"
      : "+v"(ra), "+v"(rb)
      : "s"(va), "s"(vb), "s"(ln)
      : "m0");
}
// Index of the winning token when token lane + 64*q lives in slot q of lane `lane`: e[q] are the lanes
// whose slot-q token equals the maximum.  The lowest token wins: the lowest non-empty slot, and the
// lowest lane within it.  Negative or meaningless (but below 64*NQ) when all masks are empty.
// (Why lane + 64*q and not NQ*lane + q: the race reads element (i, j) of the packed triangle for every j
// at once, at T(i) + j for j < i and at T(j) + i for j > i, T(j) = j(j+1)/2.  With consecutive j across the
// lanes the first is a stride-1 read and the second hits T(j) mod 64, and the triangular numbers of 64
// consecutive j are a complete residue system mod 64: neither has a bank conflict.  With j = NQ*lane + q
// the lanes read stride NQ and T(NQ*lane) mod 64, which collide.)
template <int NQ>
__device__ __forceinline__ int first_of_slots(const unsigned long long (&e)[NQ]) {
  if constexpr (NQ == 2) {
    // five scalar instructions, four of them in a chain (the race's time is its instruction count);
    // with both masks empty (only a NaN maximum does that) the result is 63, which callers never use
    int i, L;
    unsigned long long m;
    asm("s_cmp_lg_u64 %3, 0\n\t"
        "s_cselect_b64 %1, %3, %4\n\t"
        "s_cselect_b32 %0, 0, 64\n\t"
        "s_ff1_i32_b64 %2, %1\n\t"
        "s_add_i32 %0, %0, %2"
        : "=&s"(i), "=&s"(m), "=&s"(L)
        : "s"(e[0]), "s"(e[1])
        : "scc");
    return i;
  } else {
    // slot q's first winner is token ff1(e[q]) | 64*q; an empty mask gives all ones, which is huge as an
    // unsigned number, so the unsigned minimum over the slots is the answer (-1 when all are empty)
    unsigned best = 0xffffffffu;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      int L;
      asm("s_ff1_i32_b64 %0, %1" : "=s"(L) : "s"(e[q]));   // -1 for an empty mask
      const unsigned cand = static_cast<unsigned>(L) | static_cast<unsigned>(64 * q);
      best = cand < best ? cand : best;
    }
    return static_cast<int>(best);
  }
}
// Which lanes' values satisfy a comparison, for the S token slots of a wave: m[k] = lanes with x <= v[k] (unsigned or float; a
// NaN never does) or v[k] == x.  The comparisons write S different scalar registers back to back; the compiler's own
// ballots go through vcc one after the other, and each waits some twenty cycles for the scalar unit to have read the one
// before (a count over eight slots: 500 -> 200 cycles).  x may come from a v_readfirstlane right before, and a
// mask may go to a vector instruction right after: two wait states at either end.
#define KVR_MASKS8(op)                                                                                               \
  asm("s_nop 1\n\t" op " %0, %8, %9\n\t" op " %1, %8, %10\n\t" op " %2, %8, %11\n\t" op " %3, %8, %12\n\t"             \
      op " %4, %8, %13\n\t" op " %5, %8, %14\n\t" op " %6, %8, %15\n\t" op " %7, %8, %16\n\ts_nop 1"                            \
      : "=&s"(m[0]), "=&s"(m[1]), "=&s"(m[2]), "=&s"(m[3]), "=&s"(m[4]), "=&s"(m[5]), "=&s"(m[6]), "=&s"(m[7])        \
      : "s"(x), "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(v[4]), "v"(v[5]), "v"(v[6]), "v"(v[7]))
#define KVR_MASKS4(op)                                                                                               \
  asm("s_nop 1\n\t" op " %0, %4, %5\n\t" op " %1, %4, %6\n\t" op " %2, %4, %7\n\t" op " %3, %4, %8\n\ts_nop 1"                   \
      : "=&s"(m[0]), "=&s"(m[1]), "=&s"(m[2]), "=&s"(m[3]) : "s"(x), "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]))
#define KVR_MASKS3(op)                                                                                               \
  asm("s_nop 1\n\t" op " %0, %3, %4\n\t" op " %1, %3, %5\n\t" op " %2, %3, %6\n\ts_nop 1"                                          \
      : "=&s"(m[0]), "=&s"(m[1]), "=&s"(m[2]) : "s"(x), "v"(v[0]), "v"(v[1]), "v"(v[2]))
#define KVR_MASKS2(op)                                                                                               \
  asm("s_nop 1\n\t" op " %0, %2, %3\n\t" op " %1, %2, %4\n\ts_nop 1" : "=&s"(m[0]), "=&s"(m[1]) : "s"(x), "v"(v[0]), "v"(v[1]))
#define KVR_MASKS(name, T, op, cmp, uniform)                                                                         \
  template <int S>                                                                                                   \
  __device__ __forceinline__ void name(const T (&v)[S], T x, unsigned long long (&m)[S]) {                           \
    x = uniform;                                       /* (no-op when the compiler knows x uniform) */               \
    if constexpr (S == 8) KVR_MASKS8(op);                                                                            \
    else if constexpr (S == 4) KVR_MASKS4(op);                                                                       \
    else if constexpr (S == 3) KVR_MASKS3(op);                                                                       \
    else if constexpr (S == 2) KVR_MASKS2(op);                                                                       \
    else if constexpr (S > 8 && S % 8 == 0) {                                                                        \
      _Pragma("unroll") for (int c = 0; c < S; c += 8) {                                                             \
        T v8[8];                                                                                                     \
        unsigned long long m8[8];                                                                                    \
        _Pragma("unroll") for (int k = 0; k < 8; ++k) v8[k] = v[c + k];                                              \
        name<8>(v8, x, m8);                                                                                          \
        _Pragma("unroll") for (int k = 0; k < 8; ++k) m[c + k] = m8[k];                                              \
      }                                                                                                              \
    } else {                                                                                                         \
      _Pragma("unroll") for (int k = 0; k < S; ++k) m[k] = __ballot(v[k] cmp x);                                     \
    }                                                                                                                \
  }
KVR_MASKS(masks_ge, uint32_t, "v_cmp_le_u32", >=, static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(x))))
KVR_MASKS(masks_ge, float, "v_cmp_le_f32", >=, __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x))))
KVR_MASKS(masks_eq, float, "v_cmp_eq_f32", ==, __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x))))
// how many lanes below this one are in the mask
__device__ __forceinline__ int lane_rank(unsigned long long m) {
  return static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u)));
}
template <int S, class T>
__device__ __forceinline__ int count_slots_ge(const T (&v)[S], T x) {
  unsigned long long m[S];
  masks_ge<S>(v, x, m);
  int c = 0;
#pragma unroll
  for (int k = 0; k < S; ++k) c += __popcll(m[k]);
  return c;
}

// max / sum over each half of the wave (lanes 0-31 and 32-63); valid in lanes 31 and 63
__device__ __forceinline__ float half_max_at_31(float v) {
  KVR_DPP_MAX(v, 0x111, 0xf) KVR_DPP_MAX(v, 0x112, 0xf) KVR_DPP_MAX(v, 0x114, 0xf)
  KVR_DPP_MAX(v, 0x118, 0xf) KVR_DPP_MAX(v, 0x142, 0xa)
  return v;
}
__device__ __forceinline__ float half_sum_at_31(float v) {
  KVR_DPP_ADD(v, 0x111, 0xf) KVR_DPP_ADD(v, 0x112, 0xf) KVR_DPP_ADD(v, 0x114, 0xf)
  KVR_DPP_ADD(v, 0x118, 0xf) KVR_DPP_ADD(v, 0x142, 0xa)
  return v;
}

// The sum over the wave that a butterfly of lane exchanges (32, 16, 8, 4, 2, 1) gives, bit for bit, without its trips through
// LDS: the halves and the rows are swapped in registers, and from there on every value repeats, so a rotation of the row by 8, 4,
// 2 and 1 lanes meets the butterfly's partner.  Valid in every lane.
__device__ __forceinline__ float half_butterfly_sum(float v) {   // (over lanes 0-31 and 32-63)
  const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(b[0]) + __uint_as_float(b[1]);
  KVR_DPP_ADD(v, 0x128, 0xf) KVR_DPP_ADD(v, 0x124, 0xf) KVR_DPP_ADD(v, 0x122, 0xf) KVR_DPP_ADD(v, 0x121, 0xf)
  return v;
}
__device__ __forceinline__ float butterfly_sum(float v) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return half_butterfly_sum(__uint_as_float(a[0]) + __uint_as_float(a[1]));
}

// half_sum_at_31 of four values at once: one instruction a step, the four chains filling each other's wait states
__device__ __forceinline__ void half_sums_at_31(float (&v)[4]) {
#define KVR_SUM4(ctrl, rmask)                                                        \
  "v_add_f32_dpp %0, %0, %0 " ctrl " row_mask:" rmask " bank_mask:0xf\n\t"           \
  "v_add_f32_dpp %1, %1, %1 " ctrl " row_mask:" rmask " bank_mask:0xf\n\t"           \
  "v_add_f32_dpp %2, %2, %2 " ctrl " row_mask:" rmask " bank_mask:0xf\n\t"           \
  "v_add_f32_dpp %3, %3, %3 " ctrl " row_mask:" rmask " bank_mask:0xf\n\t"
  asm("s_nop 1\n\t" KVR_SUM4("row_shr:1", "0xf") KVR_SUM4("row_shr:2", "0xf") KVR_SUM4("row_shr:4", "0xf")
      KVR_SUM4("row_shr:8", "0xf") KVR_SUM4("row_bcast:15", "0xa") "s_nop 1"
      : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]));
#undef KVR_SUM4
}

// likewise half_max_at_31
__device__ __forceinline__ void half_maxes_at_31(float (&v)[4]) {
#define KVR_MAX4(ctrl, rmask)                                                        \
  "v_max_f32_dpp %0, %0, %0 " ctrl " row_mask:" rmask " bank_mask:0xf\n\t"           \
  "v_max_f32_dpp %1, %1, %1 " ctrl " row_mask:" rmask " bank_mask:0xf\n\t"           \
  "v_max_f32_dpp %2, %2, %2 " ctrl " row_mask:" rmask " bank_mask:0xf\n\t"           \
  "v_max_f32_dpp %3, %3, %3 " ctrl " row_mask:" rmask " bank_mask:0xf\n\t"
  asm("s_nop 1\n\t" KVR_MAX4("row_shr:1", "0xf") KVR_MAX4("row_shr:2", "0xf") KVR_MAX4("row_shr:4", "0xf")
      KVR_MAX4("row_shr:8", "0xf") KVR_MAX4("row_bcast:15", "0xa") "s_nop 1"
      : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]));
#undef KVR_MAX4
}

typedef __attribute__((ext_vector_type(4))) float f32x4;

// A cosine triangle whose row i (columns 0..i) takes (i + 4) & ~3 floats, so that four neighbouring columns of a row are
// one aligned 16-byte store: row i = 4g + r starts at float 4 (g + 1)(2g + r).  Element (i, j), j <= i, sits at
// start(i) + j; start(i) + j >= start(j) + i holds for i > j as in the packed triangle, so the race reads
// max(start(i) + j, start(j) + i) without knowing which index is the larger.
__device__ __forceinline__ int padded_row_start(int i) { return 4 * ((i >> 2) + 1) * (2 * (i >> 2) + (i & 3)); }
__host__ __device__ constexpr int padded_tri_floats(int n) { return 8 * (n / 4) * (n / 4 + 1); }   // n a multiple of 4

// Writes one 32x32 tile of raw dot products as cosines into a padded triangle.  acc comes from the MFMA with the
// column block J as operand A and the row block I as operand B: lane (row = lane & 31, hf = lane >> 5) holds
// columns 8R + 4hf .. + 3 of its row in acc[4R .. 4R+3].  The diagonal holds +inf (the row of a pick retires it);
// what a store writes past the diagonal stays inside the row's padding and is never read.
__device__ __forceinline__ void write_cos_tile_padded(float* tri, const float* rinv, const f32x16& acc, int I, int J, int lane) {
  const int hf = lane >> 5;
  const int row = I * 32 + (lane & 31);
  const float rrow = rinv[row];
  float4 rc[4];                                       // the columns' inverse norms, all requested before the first use
#pragma unroll
  for (int R = 0; R < 4; ++R) rc[R] = *reinterpret_cast<const float4*>(rinv + J * 32 + 8 * R + 4 * hf);
  float* dst = tri + padded_row_start(row) + J * 32 + 4 * hf;
  if (I != J) {                                       // two code paths: no per-element predicate off the diagonal
#pragma unroll
    for (int R = 0; R < 4; ++R)
      *reinterpret_cast<float4*>(dst + 8 * R) = make_float4(acc[4 * R] * rrow * rc[R].x, acc[4 * R + 1] * rrow * rc[R].y,
                                                            acc[4 * R + 2] * rrow * rc[R].z, acc[4 * R + 3] * rrow * rc[R].w);
  } else {
#pragma unroll
    for (int R = 0; R < 4; ++R) {
      const int col = J * 32 + 8 * R + 4 * hf;
      float4 v = make_float4(acc[4 * R] * rrow * rc[R].x, acc[4 * R + 1] * rrow * rc[R].y,
                             acc[4 * R + 2] * rrow * rc[R].z, acc[4 * R + 3] * rrow * rc[R].w);
      if (col == row) v.x = INFINITY;
      if (col + 1 == row) v.y = INFINITY;
      if (col + 2 == row) v.z = INFINITY;
      if (col + 3 == row) v.w = INFINITY;
      if (col <= row) *reinterpret_cast<float4*>(dst + 8 * R) = v;
    }
  }
}

// Scales one 32x32 tile of raw dot products to cosines and writes it into the packed
// triangle (element (i,j), j <= i, at i(i+1)/2 + j).  The diagonal entry holds +inf: reading
// the row of a pick drives the pick's own m to +inf and its gain to -inf, which is how a
// selected token leaves the race.
__device__ __forceinline__ void write_cos_tile(float* tri, const float* rinv, const f32x16& acc,
                                               int I, int J, int lane) {
  const int hf = lane >> 5;
  const int j = J * 32 + (lane & 31);
  const float rc = rinv[j];
  int i = I * 32 + hf * 4;                            // first of this lane's rows in the tile
  int off = i * (i + 1) / 2 + j;
  float4 rr4[4];                                      // the rows' inverse norms, all requested before the first use
#pragma unroll
  for (int R = 0; R < 4; ++R) rr4[R] = *reinterpret_cast<const float4*>(rinv + i + 8 * R);
  if (I != J) {                                       // two code paths: no per-element predicate off the diagonal
#pragma unroll
    for (int R = 0; R < 4; ++R) {
      const float rrow[4] = {rr4[R].x, rr4[R].y, rr4[R].z, rr4[R].w};
      int o = off;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        tri[o] = acc[R * 4 + q] * rrow[q] * rc;
        o += i + q + 1;
      }
      off += 8 * i + 36;                              // T(i+8) - T(i)
      i += 8;
    }
  } else {
#pragma unroll
    for (int R = 0; R < 4; ++R) {
      const float rrow[4] = {rr4[R].x, rr4[R].y, rr4[R].z, rr4[R].w};
      int o = off;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float c = j == i + q ? INFINITY : acc[R * 4 + q] * rrow[q] * rc;
        if (j <= i + q) tri[o] = c;
        o += i + q + 1;
      }
      off += 8 * i + 36;
      i += 8;
    }
  }
}

// The same into the packed triangle from the other orientation (column block J as operand A, row block I as operand B: lane (row = lane &
// 31, hf) holds columns 8R + 4hf .. + 3 of its row), in two steps: products to cosines in registers, and the stores.  A lane's addresses are
// one base and constants, two neighbouring columns a store; with one store and one address per element a tile costs the LDS pipe
// and the vector unit half as much again.  A wave that has the CU's LDS nearly to itself scales all its tiles before it stores the first: a
// read of norms behind a tile's stores waits for them (six tiles of a wave, one after the other, 6 700 cycles).
__device__ __forceinline__ void scale_cos_tile(const float* rinv, f32x16& acc, int I, int J, int lane) {
  const int hf = lane >> 5;
  const float rrow = rinv[I * 32 + (lane & 31)];
  float4 rc[4];                                       // the columns' inverse norms, all requested before the first use
#pragma unroll
  for (int R = 0; R < 4; ++R) rc[R] = *reinterpret_cast<const float4*>(rinv + J * 32 + 8 * R + 4 * hf);
#pragma unroll
  for (int R = 0; R < 4; ++R) {
    acc[4 * R] = acc[4 * R] * rrow * rc[R].x;
    acc[4 * R + 1] = acc[4 * R + 1] * rrow * rc[R].y;
    acc[4 * R + 2] = acc[4 * R + 2] * rrow * rc[R].z;
    acc[4 * R + 3] = acc[4 * R + 3] * rrow * rc[R].w;
  }
}
__device__ __forceinline__ void store_cos_tile(float* tri, const f32x16& acc, int I, int J, int lane) {
  const int hf = lane >> 5;
  const int row = I * 32 + (lane & 31);
  float* dst = tri + row * (row + 1) / 2 + J * 32 + 4 * hf;
  if (I != J) {
#pragma unroll
    for (int R = 0; R < 4; ++R) {
#pragma unroll
      for (int q = 0; q < 4; ++q) dst[8 * R + q] = acc[4 * R + q];
    }
  } else {
    const int last = (lane & 31) - 4 * hf;            // the row's diagonal element, counted from dst
#pragma unroll
    for (int R = 0; R < 4; ++R) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (8 * R + q <= last) dst[8 * R + q] = 8 * R + q == last ? INFINITY : acc[4 * R + q];
    }
  }
}

// One tile, scaled and stored row quarter by row quarter: what workgroups that share a CU do better with.
__device__ __forceinline__ void write_cos_tile_rows(float* tri, const float* rinv, const f32x16& acc, int I, int J, int lane) {
  const int hf = lane >> 5;
  const int row = I * 32 + (lane & 31);
  const float rrow = rinv[row];
  float4 rc[4];                                       // the columns' inverse norms, all requested before the first use
#pragma unroll
  for (int R = 0; R < 4; ++R) rc[R] = *reinterpret_cast<const float4*>(rinv + J * 32 + 8 * R + 4 * hf);
  float* dst = tri + row * (row + 1) / 2 + J * 32 + 4 * hf;
  if (I != J) {
#pragma unroll
    for (int R = 0; R < 4; ++R) {
      dst[8 * R] = acc[4 * R] * rrow * rc[R].x;
      dst[8 * R + 1] = acc[4 * R + 1] * rrow * rc[R].y;
      dst[8 * R + 2] = acc[4 * R + 2] * rrow * rc[R].z;
      dst[8 * R + 3] = acc[4 * R + 3] * rrow * rc[R].w;
    }
  } else {
    const int last = (lane & 31) - 4 * hf;            // the row's diagonal element, counted from dst
#pragma unroll
    for (int R = 0; R < 4; ++R) {
      const float v[4] = {acc[4 * R] * rrow * rc[R].x, acc[4 * R + 1] * rrow * rc[R].y,
                          acc[4 * R + 2] * rrow * rc[R].z, acc[4 * R + 3] * rrow * rc[R].w};
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (8 * R + q <= last) dst[8 * R + q] = 8 * R + q == last ? INFINITY : v[q];
    }
  }
}

// The race: Algorithm 1's picks (Eq. 2-3) on one wave, over the 64*NQ tokens whose cosines sit in a triangle in LDS.
// Token lane + 64*q lives in slot q of lane `lane`: its score s[q], its running maximum m[q] and the LDS address
// row[q] of its row of the triangle.  Element (i, j) sits at max(row(i) + 4j, row(j) + 4i), the diagonal holds +inf, so
// reading the row of a pick retires it.  Picks number u .. cnt-1 (cnt <= 64, cnt > u) are made; pick u is parked in
// lane u of rec_i (4 x its token) and rec_g (its gain).  With BOUND the race stops before the first pick whose gain is
// not above gout; amax and the returned reference i4 then describe that pick, which is not applied.  Returns the number
// of picks made.  Ties go to the lowest token.  Nothing is branched on non-finite gains: a maximum that equals no
// token (NaN) retires lane 63's token, which callers replace afterwards (see pick_chain).
//
// What bounds it is the issue rate of a single wave, four cycles an instruction, plus 20 for each value that crosses
// from the vector to the scalar unit and 50 for the LDS read; so the loop is written out by hand.  The first winning
// slot of every lane is worked out in the wait states of the reduction's DPP steps, which leaves one comparison, one
// s_ff1 and two lane reads after it, whatever NQ is; lanes are in order, but tokens of several lanes with the same
// gain are not, so more than one winning lane takes a slow path that goes through the slots in token order.  That check,
// the logging and the loop control run while the LDS read is on its way.  Measured in cycles per pick for 1 / 2 / 3 / 4
// slots: 240 / 255 / 280 / 300, against 262 / 304 / 384 / 440 for the compiler's loop over ballots of every slot; one
// decode-time event (112 heads, n = 256, b = 128) 37.9 -> 30.0 us.  Also measured: narrowing exec to the winning lane
// and v_readfirstlane instead of s_ff1 and v_readlane (8 cycles slower), one or two copies of the loop instead of four
// (10 and 5 cycles slower), picking the second-best token ahead of the row of the best one (more instructions than the
// LDS read it hides).
#ifdef KVR_BOUNDS
template <int NQ, bool BOUND>
__device__ __forceinline__ int race_loop(float (&m)[NQ], const float (&s)[NQ], const int (&row)[NQ], int lane, float nlam,
                                         int u, int cnt, float gout, int& rec_i, int& rec_g, float& amax, int& i4,
                                         int tri0, int tri_floats) {
  // (debug build: the same picks from plain code, with every address checked)
  typedef __attribute__((address_space(3))) const float* lds_fp;
  while (u < cnt) {
    float av[NQ], best = -INFINITY;
#pragma unroll
    for (int q = 0; q < NQ; ++q) { av[q] = fmaf(nlam, m[q], s[q]); best = hw_max(best, av[q]); }
    amax = wave_max_uniform(best);
    int i = 63;
#pragma unroll
    for (int q = NQ - 1; q >= 0; --q) {
      const unsigned long long e = __ballot(av[q] == amax);
      if (e) i = __ffsll(static_cast<long long>(e)) - 1 + 64 * q;
    }
    i4 = i * 4;
    if (BOUND && !(amax > gout)) return u;
    write_lane2(rec_i, rec_g, i4, __float_as_int(amax), u);
    ++u;
    int ri = 0;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int r = __builtin_amdgcn_readlane(row[q], i & 63);
      if ((i >> 6) == q) ri = r;
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int x0 = ri + (lane + 64 * q) * 4, x1 = row[q] + i4;
      const int xa = kvr_ix(((x0 > x1 ? x0 : x1) - tri0) >> 2, tri_floats, KVR_BOUNDS_FILE * 100 + 5) * 4 + tri0;   // x05: triangle element of the race
      m[q] = hw_max(m[q], *reinterpret_cast<lds_fp>(static_cast<uintptr_t>(static_cast<unsigned>(xa))));
    }
  }
  return u;
}
#else
#define KVR_RACE_MAX(ctrl, rmask) "v_max_f32_dpp %[rd], %[rd], %[rd] " ctrl " row_mask:" rmask " bank_mask:0xf\n\t"
#define KVR_RACE_S1 KVR_RACE_MAX("row_shr:1", "0xf")
#define KVR_RACE_S2 KVR_RACE_MAX("row_shr:2", "0xf")
#define KVR_RACE_S3 KVR_RACE_MAX("row_shr:4", "0xf")
#define KVR_RACE_S4 KVR_RACE_MAX("row_shr:8", "0xf")
#define KVR_RACE_S5 KVR_RACE_MAX("row_bcast:15", "0xa")
#define KVR_RACE_S6 KVR_RACE_MAX("row_bcast:31", "0xc")
#define KVR_RACE_FMA(q, d) "v_fma_f32 %[" d "], %[nl], %[m" #q "], %[s" #q "]\n\t"
// (gfx950 wants two wait states between a VALU write of vcc or another scalar register and the VALU instruction that reads
// it, and before a DPP read.  The compiler does not look into the block, so it starts with its own: -lambda may come from
// a v_readfirstlane right before it.)
#define KVR_RACE_EQ(q) "v_cmp_eq_f32 vcc, %[bs], %[a" #q "]\n\t"
#define KVR_RACE_SR(o, q) "v_cndmask_b32 %[sr], %[" o "], %[r" #q "], vcc\n\t"
#define KVR_RACE_SI(o, q) "v_cndmask_b32 %[si], %[" o "], %[j" #q "], vcc\n\t"
#define KVR_RACE_WIN(best, sr, si)                                                                             \
  "v_readlane_b32 %[am], %[rd], 63\n\ts_nop 1\n\tv_cmp_eq_f32 vcc, %[am], %[" best "]\n\ts_ff1_i32_b64 %[L], vcc\n\t" \
  "v_readlane_b32 %[R], %[" sr "], %[L]\n\tv_readlane_b32 %[I], %[" si "], %[L]\n\ts_nop 0\n\t"
#define KVR_RACE_ADR(q) "v_add_u32 %[x" #q "], %[I], %[t" #q "]\n\tv_max_u32 %[x" #q "], %[x" #q "], %[ad]\n\t"
#define KVR_RACE_RD(q, off) "ds_read_b32 %[x" #q "], %[x" #q "] offset:" off "\n\t"
#define KVR_RACE_UPD(q) "v_max_f32 %[m" #q "], %[m" #q "], %[x" #q "]\n\t"
// A pick is written out KVR_RACE_COPIES times (c is the copy's number, which its labels carry): a taken branch costs 25
// cycles, one that falls through 12.  Winner -> addresses -> reads; while they travel: tie check, bound check, log, loop
// control; the next copy starts by waiting for the reads.
#define KVR_RACE_TIE(c, q)                                                                                     \
  "v_cmp_eq_f32 vcc, %[am], %[a" #q "]\n\ts_cmp_lg_u64 vcc, 0\n\ts_cbranch_scc0 5" #c #q "f\n\ts_ff1_i32_b64 %[L], vcc\n\t" \
  "v_readlane_b32 %[R], %[r" #q "], %[L]\n\tv_readlane_b32 %[I], %[j" #q "], %[L]\n5" #c #q ":\n\t"
#define KVR_RACE_PICK(c, find, adrs, reads, bound, upds)                                                        \
  "6" #c ":\n\t" find "2" #c ":\n\tv_add_u32 %[ad], %[R], %[j0]\n\t" adrs reads                                 \
  "s_bcnt1_i32_b64 %[L], vcc\n\ts_cmp_gt_u32 %[L], 1\n\ts_cbranch_scc1 4" #c "f\n\t" bound                       \
  "v_writelane_b32 %[ri], %[I], m0\n\tv_writelane_b32 %[rg], %[am], m0\n\ts_add_u32 m0, m0, 1\n\t"               \
  "s_cmp_ge_u32 m0, %[cnt]\n\ts_cbranch_scc1 8f\n\ts_waitcnt lgkmcnt(0)\n\t" upds
#define KVR_RACE_TIED(c, ties) "4" #c ":\n\ts_waitcnt lgkmcnt(0)\n\t" ties "s_mov_b64 vcc, 0\n\ts_nop 1\n\ts_branch 2" #c "b\n"
#define KVR_RACE_ASM(find, adrs, reads, bound, upds, ties)                                                       \
  "s_nop 1\n\ts_mov_b32 m0, %[u]\n" KVR_RACE_PICK(0, find, adrs, reads, bound, upds) KVR_RACE_PICK(1, find, adrs, reads, bound, upds) \
  KVR_RACE_PICK(2, find, adrs, reads, bound, upds) KVR_RACE_PICK(3, find, adrs, reads, bound, upds) "s_branch 60b\n"        \
  KVR_RACE_TIED(0, ties(0)) KVR_RACE_TIED(1, ties(1)) KVR_RACE_TIED(2, ties(2)) KVR_RACE_TIED(3, ties(3))                   \
  "8:\n\ts_waitcnt lgkmcnt(0)\n\t" upds "3:\n\ts_waitcnt lgkmcnt(0)\n\ts_mov_b32 %[u], m0"
#define KVR_RACE_BOUND "v_cmp_gt_f32 vcc, %[am], %[go]\n\ts_cbranch_vccz 3f\n\t"
#define KVR_RACE_TMP [rd] "=&v"(rd), [ad] "=&v"(ad), [am] "=&s"(am), [L] "=&s"(L), [R] "=&s"(R), [I] "=&s"(I), \
                     [ri] "+v"(rec_i), [rg] "+v"(rec_g), [u] "+s"(u)
#define KVR_RACE_IN [nl] "s"(nlam), [cnt] "s"(cnt), [go] "v"(gout)

#define KVR_RACE_FIND1 \
  KVR_RACE_FMA(0, "rd") KVR_RACE_FMA(0, "a0") "s_nop 0\n\t" KVR_RACE_S1 "s_nop 1\n\t" KVR_RACE_S2 "s_nop 1\n\t" \
  KVR_RACE_S3 "s_nop 1\n\t" KVR_RACE_S4 "s_nop 1\n\t" KVR_RACE_S5 "s_nop 1\n\t" KVR_RACE_S6 "s_nop 0\n\t" \
  KVR_RACE_WIN("a0", "r0", "j0")
#define KVR_RACE_TIES1(c) KVR_RACE_TIE(c, 0)
#define KVR_RACE_RUN1(bound) \
  asm volatile(KVR_RACE_ASM(KVR_RACE_FIND1, KVR_RACE_ADR(0), \
                            KVR_RACE_RD(0, "0"), bound, \
                            KVR_RACE_UPD(0), KVR_RACE_TIES1) \
               : KVR_RACE_TMP, \
                 [a0] "=&v"(a[0]), \
                 [x0] "=&v"(x[0]), \
                 [m0] "+v"(m[0]) \
               : KVR_RACE_IN, [s0] "v"(s[0]), \
                 [r0] "v"(row[0]), \
                 [t0] "v"(t[0]), \
                 [j0] "v"(j[0]) \
               : "vcc", "scc", "m0", "memory")
#define KVR_RACE_FIND2 \
  KVR_RACE_FMA(0, "a0") KVR_RACE_FMA(1, "a1") "v_max_f32 %[rd], %[a0], %[a1]\n\tv_max_f32 %[bs], %[a0], %[a1]\n\t" \
  KVR_RACE_EQ(0) KVR_RACE_S1 "s_nop 0\n\t" KVR_RACE_SR("r1", 0) KVR_RACE_S2 KVR_RACE_SI("j1", 0) "s_nop 0\n\t" \
  KVR_RACE_S3 "s_nop 1\n\t" KVR_RACE_S4 "s_nop 1\n\t" KVR_RACE_S5 "s_nop 1\n\t" KVR_RACE_S6 "s_nop 0\n\t" \
  KVR_RACE_WIN("bs", "sr", "si")
#define KVR_RACE_TIES2(c) KVR_RACE_TIE(c, 1) KVR_RACE_TIE(c, 0)
#define KVR_RACE_RUN2(bound) \
  asm volatile(KVR_RACE_ASM(KVR_RACE_FIND2, KVR_RACE_ADR(0) KVR_RACE_ADR(1), \
                            KVR_RACE_RD(0, "0") KVR_RACE_RD(1, "256"), bound, \
                            KVR_RACE_UPD(0) KVR_RACE_UPD(1), KVR_RACE_TIES2) \
               : KVR_RACE_TMP, [bs] "=&v"(bs), [sr] "=&v"(sr), [si] "=&v"(si), \
                 [a0] "=&v"(a[0]), [a1] "=&v"(a[1]), \
                 [x0] "=&v"(x[0]), [x1] "=&v"(x[1]), \
                 [m0] "+v"(m[0]), [m1] "+v"(m[1]) \
               : KVR_RACE_IN, [s0] "v"(s[0]), [s1] "v"(s[1]), \
                 [r0] "v"(row[0]), [r1] "v"(row[1]), \
                 [t0] "v"(t[0]), [t1] "v"(t[1]), \
                 [j0] "v"(j[0]), [j1] "v"(j[1]) \
               : "vcc", "scc", "m0", "memory")
#define KVR_RACE_FIND3 \
  KVR_RACE_FMA(0, "a0") KVR_RACE_FMA(1, "a1") \
  KVR_RACE_FMA(2, "a2") "v_max3_f32 %[rd], %[a0], %[a1], %[a2]\n\tv_max3_f32 %[bs], %[a0], %[a1], %[a2]\n\t" \
  KVR_RACE_EQ(1) KVR_RACE_S1 "s_nop 0\n\t" KVR_RACE_SR("r2", 1) KVR_RACE_S2 KVR_RACE_SI("j2", 1) KVR_RACE_EQ(0) \
  KVR_RACE_S3 "s_nop 0\n\t" KVR_RACE_SR("sr", 0) KVR_RACE_S4 KVR_RACE_SI("si", 0) "s_nop 0\n\t" \
  KVR_RACE_S5 "s_nop 1\n\t" KVR_RACE_S6 "s_nop 0\n\t" KVR_RACE_WIN("bs", "sr", "si")
#define KVR_RACE_TIES3(c) KVR_RACE_TIE(c, 2) KVR_RACE_TIE(c, 1) KVR_RACE_TIE(c, 0)
#define KVR_RACE_RUN3(bound) \
  asm volatile(KVR_RACE_ASM(KVR_RACE_FIND3, KVR_RACE_ADR(0) KVR_RACE_ADR(1) KVR_RACE_ADR(2), \
                            KVR_RACE_RD(0, "0") KVR_RACE_RD(1, "256") KVR_RACE_RD(2, "512"), bound, \
                            KVR_RACE_UPD(0) KVR_RACE_UPD(1) KVR_RACE_UPD(2), KVR_RACE_TIES3) \
               : KVR_RACE_TMP, [bs] "=&v"(bs), [sr] "=&v"(sr), [si] "=&v"(si), \
                 [a0] "=&v"(a[0]), [a1] "=&v"(a[1]), [a2] "=&v"(a[2]), \
                 [x0] "=&v"(x[0]), [x1] "=&v"(x[1]), [x2] "=&v"(x[2]), \
                 [m0] "+v"(m[0]), [m1] "+v"(m[1]), [m2] "+v"(m[2]) \
               : KVR_RACE_IN, [s0] "v"(s[0]), [s1] "v"(s[1]), [s2] "v"(s[2]), \
                 [r0] "v"(row[0]), [r1] "v"(row[1]), [r2] "v"(row[2]), \
                 [t0] "v"(t[0]), [t1] "v"(t[1]), [t2] "v"(t[2]), \
                 [j0] "v"(j[0]), [j1] "v"(j[1]), [j2] "v"(j[2]) \
               : "vcc", "scc", "m0", "memory")
#define KVR_RACE_FIND4 \
  KVR_RACE_FMA(0, "a0") KVR_RACE_FMA(1, "a1") KVR_RACE_FMA(2, "a2") \
  KVR_RACE_FMA(3, "a3") "v_max3_f32 %[bs], %[a0], %[a1], %[a2]\n\tv_max_f32 %[rd], %[bs], %[a3]\n\tv_max_f32 %[bs], %[bs], %[a3]\n\t" \
  KVR_RACE_EQ(2) KVR_RACE_S1 "s_nop 0\n\t" KVR_RACE_SR("r3", 2) KVR_RACE_S2 KVR_RACE_SI("j3", 2) KVR_RACE_EQ(1) \
  KVR_RACE_S3 "s_nop 0\n\t" KVR_RACE_SR("sr", 1) KVR_RACE_S4 KVR_RACE_SI("si", 1) KVR_RACE_EQ(0) \
  KVR_RACE_S5 "s_nop 0\n\t" KVR_RACE_SR("sr", 0) KVR_RACE_S6 KVR_RACE_SI("si", 0) KVR_RACE_WIN("bs", "sr", "si")
#define KVR_RACE_TIES4(c) KVR_RACE_TIE(c, 3) KVR_RACE_TIE(c, 2) KVR_RACE_TIE(c, 1) KVR_RACE_TIE(c, 0)
#define KVR_RACE_RUN4(bound) \
  asm volatile(KVR_RACE_ASM(KVR_RACE_FIND4, KVR_RACE_ADR(0) KVR_RACE_ADR(1) KVR_RACE_ADR(2) KVR_RACE_ADR(3), \
                            KVR_RACE_RD(0, "0") KVR_RACE_RD(1, "256") KVR_RACE_RD(2, "512") KVR_RACE_RD(3, "768"), bound, \
                            KVR_RACE_UPD(0) KVR_RACE_UPD(1) KVR_RACE_UPD(2) KVR_RACE_UPD(3), KVR_RACE_TIES4) \
               : KVR_RACE_TMP, [bs] "=&v"(bs), [sr] "=&v"(sr), [si] "=&v"(si), \
                 [a0] "=&v"(a[0]), [a1] "=&v"(a[1]), [a2] "=&v"(a[2]), [a3] "=&v"(a[3]), \
                 [x0] "=&v"(x[0]), [x1] "=&v"(x[1]), [x2] "=&v"(x[2]), [x3] "=&v"(x[3]), \
                 [m0] "+v"(m[0]), [m1] "+v"(m[1]), [m2] "+v"(m[2]), [m3] "+v"(m[3]) \
               : KVR_RACE_IN, [s0] "v"(s[0]), [s1] "v"(s[1]), [s2] "v"(s[2]), [s3] "v"(s[3]), \
                 [r0] "v"(row[0]), [r1] "v"(row[1]), [r2] "v"(row[2]), [r3] "v"(row[3]), \
                 [t0] "v"(t[0]), [t1] "v"(t[1]), [t2] "v"(t[2]), [t3] "v"(t[3]), \
                 [j0] "v"(j[0]), [j1] "v"(j[1]), [j2] "v"(j[2]), [j3] "v"(j[3]) \
               : "vcc", "scc", "m0", "memory")

template <int NQ, bool BOUND>
__device__ __forceinline__ int race_loop(float (&m)[NQ], const float (&s)[NQ], const int (&row)[NQ], int lane, float nlam,
                                         int u, int cnt, float gout, int& rec_i, int& rec_g, float& amax, int& i4,
                                         int, int) {
  float rd, bs, a[NQ], x[NQ];
  int ad, am, L, R, I, sr, si;
  int j[NQ], t[NQ];                                    // 4 x token; row address less 256 q (slot q is read at offset 256 q)
#pragma unroll
  for (int q = 0; q < NQ; ++q) { j[q] = (lane + 64 * q) * 4; t[q] = row[q] - 256 * q; }
  u = __builtin_amdgcn_readfirstlane(u);
  cnt = __builtin_amdgcn_readfirstlane(cnt);
  nlam = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(nlam)));
  if constexpr (NQ == 1) {
    if constexpr (BOUND) KVR_RACE_RUN1(KVR_RACE_BOUND); else KVR_RACE_RUN1("");
  } else if constexpr (NQ == 2) {
    if constexpr (BOUND) KVR_RACE_RUN2(KVR_RACE_BOUND); else KVR_RACE_RUN2("");
  } else if constexpr (NQ == 3) {
    if constexpr (BOUND) KVR_RACE_RUN3(KVR_RACE_BOUND); else KVR_RACE_RUN3("");
  } else {
    static_assert(NQ == 4, "one to four tokens per lane");
    if constexpr (BOUND) KVR_RACE_RUN4(KVR_RACE_BOUND); else KVR_RACE_RUN4("");
  }
  amax = __int_as_float(am);
  i4 = I;
  return u;
}
#endif

// Algorithm 1's pick chain on one wave, for a head whose cosines sit in the packed triangle `tri` (element (i,j),
// j <= i, at i(i+1)/2 + j, or at padded_row_start(i) + j if PADDED, +inf on the diagonal) and whose scores sit in s_l (-inf for padding): the race in chunks of 64
// picks, each written to order_l / gain_l once.  Nothing is checked per pick.  Non-finite input is detected afterwards
// from the logged gains: the picks before the first one without a finite gain are kept and the list is filled up with
// the lowest tokens < n_live not yet in it.  DIVERSE false is the lambda = 0 branch (top-b, the triangle is not read).
// Returns the gain of the last pick.
template <int NQ, bool DIVERSE, bool PADDED>
__device__ __forceinline__ float pick_chain_impl(const float* s_l, const float* tri, int32_t* order_l, float* gain_l,
                                                 int n_live, int b, float lambda, int lane) {
  const int tri0 = static_cast<int>(reinterpret_cast<uintptr_t>(
      (__attribute__((address_space(3))) const char*)reinterpret_cast<const char*>(tri)));
  float sreg[NQ], mreg[NQ];
  int tja[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int j = lane + 64 * q;
    sreg[q] = s_l[j];
    mreg[q] = 0.f;
    tja[q] = (PADDED ? padded_row_start(j) * 4 : j * (j + 1) * 2) + tri0;   // start of the token's row
  }
  const float nlam = -lambda;
  int bad_t = b;                                       // first pick without a finite gain
  float last_g = -INFINITY;
  for (int c0 = 0; c0 < b; c0 += 64) {
    const int cnt = __builtin_amdgcn_readfirstlane(b - c0 < 64 ? b - c0 : 64);
    int rec_i = 0, rec_g = 0;
    if constexpr (DIVERSE) {
      float amax; int i4;
      race_loop<NQ, false>(mreg, sreg, tja, lane, nlam, 0, cnt, 0.f, rec_i, rec_g, amax, i4, tri0,
                           PADDED ? padded_tri_floats(NQ * 64) : NQ * 32 * (NQ * 64 + 1));
      rec_i >>= 2;
    } else {
      for (int u = 0; u < cnt; ++u) {
        float best = sreg[0];
#pragma unroll
        for (int q = 1; q < NQ; ++q) best = hw_max(best, sreg[q]);
        const float amax = wave_max_uniform(best);
        unsigned long long e[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) e[q] = __ballot(sreg[q] == amax);
        const int i = first_of_slots<NQ>(e);           // negative when nothing compares equal (NaN)
        write_lane2(rec_i, rec_g, i, __float_as_int(amax), u);
#pragma unroll
        for (int q = 0; q < NQ; ++q) sreg[q] = (lane + 64 * q == i) ? -INFINITY : sreg[q];
      }
    }
    const float g = __int_as_float(rec_g);
    if (lane < cnt) { order_l[c0 + lane] = rec_i; gain_l[c0 + lane] = g; }
    last_g = __int_as_float(__builtin_amdgcn_readlane(rec_g, cnt - 1));
    const unsigned long long bad = __ballot(lane < cnt && !(g > -INFINITY));
    if (bad && bad_t == b) bad_t = c0 + __ffsll(static_cast<long long>(bad)) - 1;
  }
  if (bad_t < b) {
    wave_lds_sync();
    for (int t = bad_t; t < b; ++t) {
      int i = -1;
#pragma unroll
      for (int q = NQ - 1; q >= 0; --q) {
        const int j = lane + 64 * q;
        bool free_tok = j < n_live;
        for (int u = 0; u < t; ++u) free_tok = free_tok && order_l[u] != j;
        const unsigned long long al = __ballot(free_tok);
        if (al) i = (__ffsll(static_cast<long long>(al)) - 1) + 64 * q;
      }
      if (lane == 0) { order_l[t] = i; gain_l[t] = -INFINITY; }
      wave_lds_sync();
    }
    last_g = -INFINITY;
  }
  return last_g;
}

template <int NQ, bool PADDED = false>
__device__ __forceinline__ float pick_chain(const float* s_l, const float* tri, int32_t* order_l, float* gain_l,
                                            int n_live, int b, float lambda, bool diverse, int lane) {
  return diverse ? pick_chain_impl<NQ, true, PADDED>(s_l, tri, order_l, gain_l, n_live, b, lambda, lane)
                 : pick_chain_impl<NQ, false, PADDED>(s_l, tri, order_l, gain_l, n_live, b, lambda, lane);
}

// sort(S) on one wave: flags the b picks of order_l (indices < 64*NQ), writes them in ascending
// order to idx_l by prefix popcounts.  With a map (ascending in its argument), idx_l and
// order_l are translated through it.  `flag` is scratch for 64*NQ ints.
template <int NQ, class Idx>
__device__ __forceinline__ void sort_picks(int32_t* order_l, Idx* idx_l, int32_t* flag, int b, int lane,
                                           const int32_t* map) {
#pragma unroll
  for (int q = 0; q < NQ; ++q) flag[lane + 64 * q] = 0;
  wave_lds_sync();                                     // order_l was written by other lanes
  for (int u = lane; u < b; u += kWave) flag[min(max(order_l[u], 0), 64 * NQ - 1)] = 1;
  wave_lds_sync();                                     // flags are set by other lanes
  int off = 0;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int j = lane + 64 * q;
    const bool picked = flag[j] != 0;
    const unsigned long long sel = __ballot(picked);
    if (picked) idx_l[off + __popcll(sel & ((1ull << lane) - 1ull))] = static_cast<Idx>(map ? map[j] : j);
    off += __popcll(sel);
  }
  if (map)
    for (int u = lane; u < b; u += kWave) order_l[u] = map[min(max(order_l[u], 0), 64 * NQ - 1)];
}

// Cache update for one head: rows il[t], t < b, of K and V go to rows ob + t of the dense
// outputs, bit for bit, by the nthr threads t0 = 0..nthr-1 (nthr a multiple of 16; 16 threads
// per row).  BATCH rows per thread are loaded by straight-line code before the first store (row
// numbers past b are clamped rather than branched around): with branches between them the
// compiler loses count of what is in flight and waits for everything, acknowledged stores
// included, before each store.  Indices are clamped into [0, n) so that nothing is read
// outside the head whatever the scores were.
template <int BATCH, class Idx>
__device__ __forceinline__ void compact_rows(const char* K, const char* V, char* K_out, char* V_out,
                                             long long head_off_bytes, long long stride_tok,
                                             const Idx* il, int n, int b, long long ob, int t0, int nthr) {
  const int chunk = t0 & 15, g = t0 >> 4, G = nthr >> 4;
  const long long base = head_off_bytes + chunk * 16;
  for (int first = 0; first < b; first += BATCH * G) {
    uint4 kr[BATCH], vr[BATCH];
    if (K_out && V_out) {
#pragma unroll
      for (int k = 0; k < BATCH; ++k) {
        const int t = min(first + g + k * G, b - 1);
        const long long src = base + min(max(kvr_ix(il[t], n, KVR_BOUNDS_FILE * 100 + 90), 0), n - 1) * stride_tok * 2;   // (x90: kept token)
        kr[k] = *reinterpret_cast<const uint4*>(K + src);
        vr[k] = *reinterpret_cast<const uint4*>(V + src);
      }
    } else {
#pragma unroll
      for (int k = 0; k < BATCH; ++k) {
        const int t = min(first + g + k * G, b - 1);
        const long long src = base + min(max(kvr_ix(il[t], n, KVR_BOUNDS_FILE * 100 + 90), 0), n - 1) * stride_tok * 2;   // (x90: kept token)
        kr[k] = vr[k] = make_uint4(0u, 0u, 0u, 0u);
        if (K_out) kr[k] = *reinterpret_cast<const uint4*>(K + src);
        if (V_out) vr[k] = *reinterpret_cast<const uint4*>(V + src);
      }
    }
#pragma unroll
    for (int k = 0; k < BATCH; ++k) {
      const int t = first + g + k * G;
      if (t < b) {
        const long long dst = ((ob + t) * kD + chunk * 8) * 2;
        if (K_out) *reinterpret_cast<uint4*>(K_out + dst) = kr[k];
        if (V_out) *reinterpret_cast<uint4*>(V_out + dst) = vr[k];
      }
    }
  }
}

// One head's [n,128] bf16 rows, from registers (16 threads a row) into the padded LDS stage.
template <int NT>
__device__ __forceinline__ void store_rows(char* stage, int tid,
                                           const uint4 (&reg)[NT * 32 * 16 / kDenseThreads]) {
  constexpr int kIters = NT * 32 * 16 / kDenseThreads;
  const int chunk = tid & 15, r0 = tid >> 4;
#pragma unroll
  for (int k = 0; k < kIters; ++k)
    *reinterpret_cast<uint4*>(stage + (r0 + 16 * k) * kRowPitch + chunk * 16) = reg[k];
}

__device__ __forceinline__ bf16x8 frag_at(const char* stage, int block, int ks, int lane) {
  const int row = block * 32 + (lane & 31), hf = lane >> 5;
  return *reinterpret_cast<const bf16x8*>(stage + row * kRowPitch + ks * 32 + hf * 16);
}

}  // namespace kvr

// Shared by the bf16 GEMM kernels that stream operand tiles HBM -> LDS (gemm_dma.hip, gemm_tile.hip): their parameters, the
// copy instructions and the output stage.
#pragma once

#include "dev_common.h"
#include "hmy_internal.h"

namespace hmy {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

struct DmaP {
  const bf16_t *A, *B;
  void *C;
  const bf16_t *bias, *res;
  bf16_t *gelu_out;
  int M, N, K;
  uint32_t lda, ldb;
  int64_t ldc, ldr;
  int c_fp32, accumulate, res_fp32;
};

// one wavefront-wide 16-byte-per-lane copy HBM -> LDS.  lds_addr is wave-uniform (the
// hardware adds 16 * lane); the global address is base + byte offset per lane.
// The statement overwrites m0 and cannot say so: the compiler rejects m0 in a clobber list as a
// reserved register ("may lead to undefined behaviour").  That is safe here because the compiler
// keeps no value of its own in m0 across statements: whenever code it generates reads m0 (indexed
// register moves, messages, its own LDS-direct loads) it writes m0 immediately before, and this
// file uses none of those constructs.
__device__ __forceinline__ void dma16(const void *base, uint32_t byte_off, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(byte_off), "s"(base), "s"(lds_addr)
               : "memory");
}

// The same through a buffer descriptor, in two parts: the LDS address, then the copy from `lane_off` of each lane plus `tile_off`
// of the wave.  Bytes past the descriptor's size read as zeros and cost no memory traffic, and that is decided on the lane
// offset as an unsigned number: it must never be negative, so the instruction's own constant (added to both addresses) is not
// used to step from one KiB to the next.  Between the two the compiler writes m0 as little as it does elsewhere in this file
// (see above).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u32x4 buffer_of(const void *base, uint32_t bytes) {
  const uint64_t at = reinterpret_cast<uint64_t>(base);
  u32x4 r;
  r[0] = __builtin_amdgcn_readfirstlane(uint32_t(at));
  r[1] = __builtin_amdgcn_readfirstlane(uint32_t(at >> 32) & 0xffffu);   // stride 0
  r[2] = __builtin_amdgcn_readfirstlane(bytes);
  r[3] = 0x00020000u;
  return r;
}
__device__ __forceinline__ void set_m0(uint32_t lds_addr) { asm volatile("s_mov_b32 m0, %0\n\ts_nop 0" : : "s"(lds_addr) : "memory"); }
__device__ __forceinline__ void dma16_buffer(u32x4 rsrc, uint32_t lane_off, uint32_t tile_off) {
  asm volatile("buffer_load_dwordx4 %0, %1, %2 offen lds" : : "v"(lane_off), "s"(rsrc), "s"(tile_off) : "memory");
}
template <int N> __device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// Output stage for 8 consecutive columns of one row.  `fast`: every pointer and leading
// dimension allows 16-byte accesses; `inside`: the workgroup's tile lies inside C.  A
// tile that sticks out still leaves through the 16-byte path wherever a row's group of
// 8 columns lies inside C (a 1600-wide output ends in the middle of a tile: element by
// element that tile took longer than the whole K loop); what remains, and everything
// when `fast` is false, goes element by element through a loop kept rolled, so that it
// costs no instruction-cache space.  A group of 8 columns beyond C does not enter that loop:
// with nothing to store it cost an edge tile 5 us all the same, its code being in no cache
// (4096x2816x832 on 192 columns 30.9 -> 25.2 us, 4096x2880x832, whole tiles, 25.0).
struct Epi {
  bool fast, inside;
  __device__ __forceinline__ bool whole8(const DmaP &p, int m, int nn) const {
    return inside || (m < p.M && nn + 8 <= p.N);
  }
  __device__ __forceinline__ void init(const DmaP &p, int m0, int n0, int side) {
    const int esz = p.c_fp32 ? 4 : 2;
    bool ok = (reinterpret_cast<uintptr_t>(p.C) & 15) == 0 && (p.ldc * esz) % 16 == 0;
    if (p.res) ok = ok && (reinterpret_cast<uintptr_t>(p.res) & 15) == 0 && p.ldr % 8 == 0;
    if (p.res && p.res_fp32 && p.accumulate) ok = false;   // both would want the prefetch registers
    if (p.bias) ok = ok && (reinterpret_cast<uintptr_t>(p.bias) & 15) == 0;
    if (p.gelu_out) ok = ok && (reinterpret_cast<uintptr_t>(p.gelu_out) & 15) == 0;
    fast = ok;
    inside = m0 + side <= p.M && n0 + side <= p.N;
  }
  // tanh-form GELU with the hardware exponential: the argument is a bf16 value and so is
  // the result, which the 2-ulp exponential does not disturb.  Written as u * sigmoid(2z),
  // the same function as u/2 (1 + tanh z), z = c (u + a u^3), in fewer instructions: the
  // epilogue's arithmetic runs with the matrix cores idle, so it is paid in full.
  static __device__ __forceinline__ float gelu_fast(float u) {
    // exp(-2z) as one exp2 with the constants folded, and the hardware reciprocal: __fdividef and
    // __expf expand to a ten-instruction IEEE division and an extra multiply
    const float k = -2.f * 0.7978845608028654f * 1.4426950408889634f, a = 0.044715f;
    return u * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(k * (u + a * u * u * u)));
  }
  // what the output stage reads from global memory for 8 columns of one row: the residual
  // (bf16) or, for an accumulating fp32 C, C itself.  Fetched before the last K tile so
  // that its latency hides behind that tile's multiplies.
  struct Pre { float4 lo, hi; };
  __device__ __forceinline__ void prefetch(const DmaP &p, int m, int nn, Pre &r) const {
    if (!whole8(p, m, nn)) return;
    if (p.res && p.res_fp32) {   // the fp32 residual stream: 8 columns are 32 bytes
      const float *x = reinterpret_cast<const float *>(p.res) + int64_t(m) * p.ldr + nn;
      r.lo = *reinterpret_cast<const float4 *>(x);
      r.hi = *reinterpret_cast<const float4 *>(x + 4);
    } else if (p.res) {
      r.lo = *reinterpret_cast<const float4 *>(p.res + int64_t(m) * p.ldr + nn);
    } else if (p.c_fp32 && p.accumulate) {
      const float *c = static_cast<const float *>(p.C) + int64_t(m) * p.ldc + nn;
      r.lo = *reinterpret_cast<const float4 *>(c);
      r.hi = *reinterpret_cast<const float4 *>(c + 4);
    }
  }
  // v[0..7] += the eight bf16 values held in the 16 bytes of `raw`, taken apart with integer operations on
  // the registers: reading them through a pointer of another type made the compiler keep `raw` in scratch memory
  static __device__ __forceinline__ void add_bf16x8(float (&v)[8], const float4 &raw) {
    const uint32_t u[4] = {__float_as_uint(raw.x), __float_as_uint(raw.y), __float_as_uint(raw.z), __float_as_uint(raw.w)};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      v[2 * c] += __uint_as_float(u[c] << 16);
      v[2 * c + 1] += __uint_as_float(u[c] & 0xffff0000u);
    }
  }
  // `bias8`: the lane's 8 bias values, the same for every row it emits.  Loaded once with the prefetch: a
  // load inside this function would wait on the memory counter, which also counts the stores of the
  // previous call, and so serialise the eight store rounds of a wave.
  __device__ __forceinline__ void emit_fast(const DmaP &p, int m, int nn, float (&v)[8], const Pre &r,
                                            const float4 &bias8) const {
    if (p.bias) add_bf16x8(v, bias8);
    if (p.res && p.res_fp32) {
      v[0] += r.lo.x; v[1] += r.lo.y; v[2] += r.lo.z; v[3] += r.lo.w;
      v[4] += r.hi.x; v[5] += r.hi.y; v[6] += r.hi.z; v[7] += r.hi.w;
    } else if (p.res) {
      add_bf16x8(v, r.lo);
    }
    const int64_t ci = int64_t(m) * p.ldc + nn;
    if (p.c_fp32) {
      float *c = static_cast<float *>(p.C) + ci;
      float4 lo = *reinterpret_cast<float4 *>(v), hi = *reinterpret_cast<float4 *>(v + 4);
      if (p.accumulate) {
        if (p.res) {   // the prefetch slot held the residual: read C now
          const float4 a = *reinterpret_cast<const float4 *>(c), b = *reinterpret_cast<const float4 *>(c + 4);
          lo.x += a.x; lo.y += a.y; lo.z += a.z; lo.w += a.w;
          hi.x += b.x; hi.y += b.y; hi.z += b.z; hi.w += b.w;
        } else {
          lo.x += r.lo.x; lo.y += r.lo.y; lo.z += r.lo.z; lo.w += r.lo.w;
          hi.x += r.hi.x; hi.y += r.hi.y; hi.z += r.hi.z; hi.w += r.hi.w;
        }
      }
      *reinterpret_cast<float4 *>(c) = lo;
      *reinterpret_cast<float4 *>(c + 4) = hi;
    } else {
      Vec16<bf16_t> o;
#pragma unroll
      for (int k = 0; k < 8; ++k) o.v[k] = from_f32<bf16_t>(v[k]);
      // gelu_out == C: only the activation is wanted (a forward pass that keeps nothing for a backward pass)
      if (p.gelu_out != static_cast<bf16_t *>(p.C)) store16(static_cast<bf16_t *>(p.C) + ci, o);
      if (p.gelu_out) {
        Vec16<bf16_t> g;
#pragma unroll
        for (int k = 0; k < 8; ++k) g.v[k] = from_f32<bf16_t>(gelu_fast(to_f32(o.v[k])));
        store16(p.gelu_out + ci, g);
      }
    }
  }
  // one element; src points at its fp32 value in LDS
  __device__ __forceinline__ void emit_one(const DmaP &p, int m, int nn, float v) const {
    if (p.bias) v += to_f32(p.bias[nn]);
    if (p.res)
      v += p.res_fp32 ? reinterpret_cast<const float *>(p.res)[int64_t(m) * p.ldr + nn]
                      : to_f32(p.res[int64_t(m) * p.ldr + nn]);
    const int64_t ci = int64_t(m) * p.ldc + nn;
    if (p.c_fp32) {
      float *c = static_cast<float *>(p.C) + ci;
      *c = p.accumulate ? *c + v : v;
    } else {
      const bf16_t o = from_f32<bf16_t>(v);
      static_cast<bf16_t *>(p.C)[ci] = o;
      if (p.gelu_out) p.gelu_out[ci] = from_f32<bf16_t>(gelu_f(to_f32(o)));
    }
  }
  // the same with the eight values in the 16-byte chunks `chunk` and `chunk` ^ 1 of a row in LDS
  __device__ __forceinline__ void emit8(const DmaP &p, int m, int nn, const float *row, int chunk, const Pre &r,
                                        const float4 &bias8) const {
    if (fast && whole8(p, m, nn)) {
      float v[8];
      *reinterpret_cast<float4 *>(v) = *reinterpret_cast<const float4 *>(row + 4 * chunk);
      *reinterpret_cast<float4 *>(v + 4) = *reinterpret_cast<const float4 *>(row + 4 * (chunk ^ 1));
      emit_fast(p, m, nn, v, r, bias8);
    } else if (m < p.M && nn < p.N) {
#pragma unroll 1
      for (int k = 0; k < 8; ++k)
        if (nn + k < p.N) emit_one(p, m, nn + k, row[4 * (chunk ^ (k >> 2)) + (k & 3)]);
    }
  }
  // a row's group of 8 columns, whose fp32 values lie at src in LDS: in one piece where the group lies inside C,
  // else whatever of it does, element by element
  __device__ __forceinline__ void emit8(const DmaP &p, int m, int nn, const float *src, const Pre &r,
                                        const float4 &bias8) const {
    if (whole8(p, m, nn)) {
      float v[8];
      *reinterpret_cast<float4 *>(v) = *reinterpret_cast<const float4 *>(src);
      *reinterpret_cast<float4 *>(v + 4) = *reinterpret_cast<const float4 *>(src + 4);
      emit_fast(p, m, nn, v, r, bias8);
    } else if (m < p.M && nn < p.N) {
#pragma unroll 1
      for (int k = 0; k < 8; ++k)
        if (nn + k < p.N) emit_one(p, m, nn + k, src[k]);
    }
  }
};

inline DmaP dma_params(const hmy_gemm_desc &g) {
  DmaP p;
  p.A = static_cast<const bf16_t *>(g.A); p.B = static_cast<const bf16_t *>(g.B); p.C = g.C;
  p.bias = static_cast<const bf16_t *>(g.bias); p.res = static_cast<const bf16_t *>(g.res);
  p.gelu_out = static_cast<bf16_t *>(g.gelu_out);
  p.M = g.M; p.N = g.N; p.K = g.K;
  p.lda = uint32_t(g.lda); p.ldb = uint32_t(g.ldb); p.ldc = g.ldc; p.ldr = g.ldr;
  p.c_fp32 = g.c_fp32; p.accumulate = g.accumulate; p.res_fp32 = g.res_fp32;
  return p;
}

}  // namespace

}  // namespace hmy

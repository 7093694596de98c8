// fp32 GEMM on the matrix cores (v_mfma_f32_32x32x2_f32): C[M,N] = op(A) op(B) (+bias) (+res), optional gelu second
// output, optional accumulation into C.  Every product and every sum is fp32, as in the plain kernel.
//
// One such instruction multiplies 32x32 outputs by two contraction steps in 64 cycles, so what feeds it is never the
// limit: operand tiles go through registers into one of two LDS stages, and ragged edges are masked on the way.  What
// bounds the kernel is the matrix pipe when the output has tiles for every SIMD, and the length of one wave's multiply
// chain when it has not.  Hence these splits of the same loop:
//   128x128  four waves of 64x64 (2x2 instructions per step)        outputs with two workgroups for every compute unit
//   64x64    four waves of 32x32, or eight that halve the contraction    ordinary outputs
//   32x32    four or eight waves share the tile and split the contraction (added up through LDS in a fixed order): small
//            outputs, where a wave that ran the whole contraction would be alone on its compute unit
// Contraction order inside a tile: lane half h of a wave takes steps 4h..4h+3 of every group of eight, for both
// operands alike, so that an operand with the contraction index contiguous is read from LDS 16 bytes at a time; one
// stored contraction-major is kept [k][row] and read 4 bytes at a time.
// Measured against the plain kernel (us): 128x128x128 15.5 -> 5.5, 1024x2048x512 72 -> 24.0, 1024x512x2048 284 -> 26.0,
// 1024x512x8192 (input gradient) 1135 -> 103, 4096x1536x2048 224, 2048x8192x4096 (weight gradient) 2520 -> 1186
// = 116 TFLOP/s of the 154 that a large fp32 product of the vendor library reaches.
#include <algorithm>

#include "dev_common.h"
#include "hmy_internal.h"

namespace hmy {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

struct F32P {
  const float *A, *B;
  float *C;
  const float *bias, *res;
  float *gelu_out;
  int M, N, K;
  int64_t lda, ldb, ldc, ldr;
  int accumulate;
};

constexpr int kSlab = 32;   // contraction steps a wave multiplies per tile

// One operand's tile of ROWS rows and KT contraction steps: global -> registers -> LDS.
// TR = false: memory [row][k], LDS [k slab][row][32] with 16-byte chunks XOR-swizzled by the row.
// TR = true : memory [k][row], LDS [k][ROWS + 8] (the pad puts a wave's two halves, four k apart, on different banks).
template <bool TR, bool VEC, int ROWS, int KT, int THREADS>
struct Operand {
  static constexpr int kVecs = ROWS * KT / 4 / THREADS;   // 16-byte pieces per thread
  static_assert(kVecs >= 1 && ROWS * KT / 4 % THREADS == 0, "a tile divides over the workgroup");
  static constexpr int kFloats = TR ? KT * (ROWS + 8) : ROWS * KT;
  float4 r[kVecs];
  // element (row, k) = base[row * ld + k] or base[k * ld + row]; nrows x K valid.  VEC (16-byte aligned rows): every load is
  // one 16-byte piece that holds at least one valid element, rows past the operand clamped into it (they only feed outputs
  // that are never stored); contraction steps past K are set to zero on the way to LDS, so that nothing waits for a load
  // here.  Otherwise element by element.
  __device__ __forceinline__ void load(const float *base, int64_t ld, int row0, int nrows, int k0, int K, int tid) {
#pragma unroll
    for (int i = 0; i < kVecs; ++i) {
      const int idx = tid + THREADS * i;
      if (VEC && TR) {
        const int row = min(row0 + 4 * (idx % (ROWS / 4)), (nrows - 1) & ~3), k = k0 + idx / (ROWS / 4);
        r[i] = *reinterpret_cast<const float4 *>(base + int64_t(min(k, K - 1)) * ld + row);
      } else if (VEC) {
        const int row = min(row0 + idx / (KT / 4), nrows - 1), k = k0 + 4 * (idx % (KT / 4));
        r[i] = *reinterpret_cast<const float4 *>(base + int64_t(row) * ld + min(k, (K - 1) & ~3));
      } else {
        // `across`: the index along the contiguous axis, `along`: the other one
        const int across = TR ? row0 + 4 * (idx % (ROWS / 4)) : k0 + 4 * (idx % (KT / 4));
        const int along = TR ? k0 + idx / (ROWS / 4) : row0 + idx / (KT / 4);
        const float *p = base + int64_t(min(along, (TR ? K : nrows) - 1)) * ld;
        const int last = (TR ? nrows : K) - 1;
        r[i] = make_float4(p[min(across, last)], p[min(across + 1, last)], p[min(across + 2, last)], p[min(across + 3, last)]);
      }
    }
  }
  __device__ __forceinline__ void store(float *s, int k0, int K, int tid) {
    if (k0 + KT > K) {   // the last tile
#pragma unroll
      for (int i = 0; i < kVecs; ++i) {
        const int idx = tid + THREADS * i;
        const int left = K - (TR ? k0 + idx / (ROWS / 4) : k0 + 4 * (idx % (KT / 4)));   // valid steps from this piece's first on
        r[i].x = left > 0 ? r[i].x : 0.f;
        r[i].y = left > (TR ? 0 : 1) ? r[i].y : 0.f;
        r[i].z = left > (TR ? 0 : 2) ? r[i].z : 0.f;
        r[i].w = left > (TR ? 0 : 3) ? r[i].w : 0.f;
      }
    }
#pragma unroll
    for (int i = 0; i < kVecs; ++i) {
      const int idx = tid + THREADS * i;
      int at;
      if (TR) {
        at = (idx / (ROWS / 4)) * (ROWS + 8) + 4 * (idx % (ROWS / 4));
      } else {
        const int chunk = idx % (KT / 4), row = idx / (KT / 4);
        at = (chunk / 8) * (ROWS * kSlab) + row * kSlab + (((chunk & 7) ^ ((row >> 1) & 7)) << 2);
      }
      *reinterpret_cast<float4 *>(s + at) = r[i];
    }
  }
  // the four steps of chunk pair c (steps 8c + 4h + 0..3 of slab kw) for row `row`
  static __device__ __forceinline__ float4 frag(const float *s, int kw, int row, int c, int h) {
    if (TR) {
      const float *p = s + (kw * kSlab + 8 * c + 4 * h) * (ROWS + 8) + row;
      return make_float4(p[0], p[ROWS + 8], p[2 * (ROWS + 8)], p[3 * (ROWS + 8)]);
    }
    return *reinterpret_cast<const float4 *>(s + kw * (ROWS * kSlab) + row * kSlab + (((2 * c + h) ^ ((row >> 1) & 7)) << 2));
  }
};

// Output stage of one lane's column n: value k goes to row m0 + row_of(k).  What it adds (residual, C itself) is read for all
// rows before the first is stored: a load behind a store to what may be the same memory waits for it, and sixteen such
// round trips in a row took longer than a short contraction.
template <int COUNT, typename RowOf, typename Value>
__device__ __forceinline__ void emit(const F32P &p, int m0, int n, RowOf row_of, Value value) {
  const float bias = p.bias ? p.bias[n] : 0.f;
  float add[COUNT];
#pragma unroll
  for (int k = 0; k < COUNT; ++k) add[k] = bias;
  if (p.res) {
#pragma unroll
    for (int k = 0; k < COUNT; ++k)
      if (m0 + row_of(k) < p.M) add[k] += p.res[int64_t(m0 + row_of(k)) * p.ldr + n];
  }
  if (p.accumulate) {
#pragma unroll
    for (int k = 0; k < COUNT; ++k)
      if (m0 + row_of(k) < p.M) add[k] += p.C[int64_t(m0 + row_of(k)) * p.ldc + n];
  }
#pragma unroll
  for (int k = 0; k < COUNT; ++k) {
    const int m = m0 + row_of(k);
    if (m >= p.M) continue;
    const int64_t ci = int64_t(m) * p.ldc + n;
    const float v = value(k) + add[k];
    p.C[ci] = v;
    if (p.gelu_out) p.gelu_out[ci] = gelu_f(v);
  }
}

// WM x WN waves over rows and columns, KW over the contraction; TI x TJ instructions of 32x32 per wave and step
template <bool TA, bool TB, bool VEC, int WM, int WN, int KW, int TI, int TJ>
__global__ __launch_bounds__(64 * WM * WN * KW, 2) void k_gemm_f32(F32P p, int grid_n) {
  constexpr int THREADS = 64 * WM * WN * KW;
  static_assert(KW == 1 || (TI == 1 && TJ == 1), "waves that split the contraction have one accumulator to exchange");
  constexpr int BM = WM * TI * 32, BN = WN * TJ * 32, KT = KW * kSlab;
  typedef Operand<TA, VEC, BM, KT, THREADS> OpA;
  typedef Operand<TB, VEC, BN, KT, THREADS> OpB;
  constexpr int kStage = OpA::kFloats + OpB::kFloats;
  __shared__ __attribute__((aligned(16))) float smem[2 * kStage];
  const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
  const int h = lane / 32, l32 = lane % 32;
  const int kw = wave % KW, wn = (wave / KW) % WN, wm = wave / (KW * WN);
  // each XCD (workgroup id mod 8) takes a contiguous range of tiles, ordered in bands of eight tile rows
  int bid = blockIdx.x;
  const int nb = gridDim.x, grid_m = nb / grid_n;
  {
    const int x = bid % 8, per = nb / 8, extra = nb % 8;
    bid = x * per + min(x, extra) + bid / 8;
  }
  constexpr int kBand = 8;
  const int band = bid / (kBand * grid_n), first_m = band * kBand;
  const int band_rows = min(grid_m - first_m, kBand);
  const int in_band = bid - band * kBand * grid_n;
  const int m0 = (first_m + in_band % band_rows) * BM, n0 = (in_band / band_rows) * BN;

  f32x16 acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // Tiles are fetched two ahead of their way to LDS, into two sets of registers by turns: one tile's multiplies are
  // shorter than a trip to memory.
  OpA oa[2];
  OpB ob[2];
  const int nk = (p.K + KT - 1) / KT;
  auto fetch = [&](int set, int t) {
    if (t >= nk) return;
    oa[set].load(p.A, p.lda, m0, p.M, t * KT, p.K, tid);
    ob[set].load(p.B, p.ldb, n0, p.N, t * KT, p.K, tid);
  };
  auto put = [&](int set, int t) {
    float *stage = smem + (t & 1) * kStage;
    oa[set].store(stage, t * KT, p.K, tid);
    ob[set].store(stage + OpA::kFloats, t * KT, p.K, tid);
  };
  // fragments of half a tile: chunks 2 half, 2 half + 1
  float4 fa[2][2][TI], fb[2][2][TJ];
  auto read = [&](int half, int t) {
    const float *a_s = smem + (t & 1) * kStage, *b_s = a_s + OpA::kFloats;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
#pragma unroll
      for (int i = 0; i < TI; ++i) fa[half][c][i] = OpA::frag(a_s, kw, (wm * TI + i) * 32 + l32, 2 * half + c, h);
#pragma unroll
      for (int j = 0; j < TJ; ++j) fb[half][c][j] = OpB::frag(b_s, kw, (wn * TJ + j) * 32 + l32, 2 * half + c, h);
    }
    __builtin_amdgcn_sched_barrier(0);   // before the multiplies it is to hide behind
  };
  auto multiply = [&](int half) {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
          for (int j = 0; j < TJ; ++j) {
            const float4 &x = fa[half][c][i], &y = fb[half][c][j];
            const float a = q == 0 ? x.x : q == 1 ? x.y : q == 2 ? x.z : x.w;
            const float b = q == 0 ? y.x : q == 1 ? y.y : q == 2 ? y.z : y.w;
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc[i][j], 0, 0, 0);
          }
    __builtin_amdgcn_sched_barrier(0);
  };
  // Tile t: tile t + 1 goes from registers (set `set`) to the stage that every wave left before the last barrier and tile t + 3
  // is requested into those registers; each half's fragments are read behind the other half's multiplies, and the barrier in
  // the middle waits for writes that are half a tile old.
  auto tile = [&](int set, int t) {
    const bool more = t + 1 < nk;
    if (more) {
      put(set, t + 1);
      fetch(set, t + 3);
    }
    read(1, t);
    multiply(0);
    if (more) {
      __syncthreads();
      read(0, t + 1);
    }
    multiply(1);
  };
  fetch(0, 0);
  fetch(1, 1);
  put(0, 0);
  fetch(0, 2);
  __syncthreads();
  read(0, 0);
  for (int t = 0; t < nk; t += 2) {
    tile(1, t);
    if (t + 1 < nk) tile(0, t + 1);
  }
  __syncthreads();   // the output stage may use the tiles' memory
  // accumulator register r of lane l: row 8*(r/4) + 4*(l/32) + r%4, column l%32
  if (KW == 1) {
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      const int n = n0 + (wn * TJ + j) * 32 + l32;
      if (n >= p.N) continue;
#pragma unroll
      for (int i = 0; i < TI; ++i)
        emit<16>(p, m0 + (wm * TI + i) * 32 + 4 * h, n, [](int r) { return 8 * (r / 4) + r % 4; }, [&](int r) { return acc[i][j][r]; });
    }
  } else {
    // the partial sums of the waves that share outputs meet in LDS (free since the last barrier), each adding up its share of
    // the registers, in the order of the contraction
    constexpr int SHARE = 16 / KW;
    float *x = smem + (wm * WN + wn) * (KW * 16 * 64);
#pragma unroll
    for (int r = 0; r < 16; ++r) x[(kw * 16 + r) * 64 + lane] = acc[0][0][r];
    __syncthreads();
    const int n = n0 + wn * 32 + l32;
    if (n >= p.N) return;
    auto row_of = [&](int q) {
      const int r = SHARE * kw + q;
      return 8 * (r / 4) + r % 4;
    };
    emit<SHARE>(p, m0 + wm * 32 + 4 * h, n, row_of, [&](int q) {
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < KW; ++w) v += x[(w * 16 + SHARE * kw + q) * 64 + lane];
      return v;
    });
  }
}

template <bool VEC, int WM, int WN, int KW, int TI, int TJ>
int launch_split(const hmy_gemm_desc &g, const F32P &p, hipStream_t s) {
  const int bm = WM * TI * 32, bn = WN * TJ * 32;
  const int gm = (g.M + bm - 1) / bm, gn = (g.N + bn - 1) / bn;
  const dim3 grid(gm * gn), block(64 * WM * WN * KW);
  if (!g.ta && !g.tb) hipLaunchKernelGGL((k_gemm_f32<false, false, VEC, WM, WN, KW, TI, TJ>), grid, block, 0, s, p, gn);
  else if (!g.ta && g.tb) hipLaunchKernelGGL((k_gemm_f32<false, true, VEC, WM, WN, KW, TI, TJ>), grid, block, 0, s, p, gn);
  else if (g.ta && !g.tb) hipLaunchKernelGGL((k_gemm_f32<true, false, VEC, WM, WN, KW, TI, TJ>), grid, block, 0, s, p, gn);
  else hipLaunchKernelGGL((k_gemm_f32<true, true, VEC, WM, WN, KW, TI, TJ>), grid, block, 0, s, p, gn);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(HMY_E_HIP, "launch of gemm_f32 failed: %s", hipGetErrorString(e));
  return HMY_OK;
}

}  // namespace

int launch_gemm_f32(const hmy_gemm_desc &g, stream_t st) {
  F32P p;
  p.A = static_cast<const float *>(g.A); p.B = static_cast<const float *>(g.B); p.C = static_cast<float *>(g.C);
  p.bias = static_cast<const float *>(g.bias); p.res = static_cast<const float *>(g.res);
  p.gelu_out = static_cast<float *>(g.gelu_out);
  p.M = g.M; p.N = g.N; p.K = g.K;
  p.lda = g.lda; p.ldb = g.ldb; p.ldc = g.ldc; p.ldr = g.ldr;
  p.accumulate = g.accumulate;
  const bool vec = ((reinterpret_cast<uintptr_t>(g.A) | reinterpret_cast<uintptr_t>(g.B)) & 15) == 0 && g.lda % 4 == 0 &&
                   g.ldb % 4 == 0;
  auto tiles = [&](int side) { return int64_t((g.M + side - 1) / side) * ((g.N + side - 1) / side); };
  hipStream_t s = (hipStream_t)st;
  // One wave's chain of multiplies leaves its SIMD idle around every tile's reads and barrier, so the finest split that still
  // gives every SIMD two waves does best; larger tiles only save operand traffic, which matters once there are two of them for
  // every compute unit.
  // operands whose rows are not 16-byte aligned: rare (no tensor of a model has such rows), one split does
  if (!vec) return launch_split<false, 2, 2, 1, 1, 1>(g, p, s);
  if (tiles(128) >= 512) return launch_split<true, 2, 2, 1, 2, 2>(g, p, s);
  // 64x64 tiles: eight waves, two to each quarter of the tile and a half of the contraction, where a compute unit has one such
  // workgroup.  Where it has two, those hide each other's reads and barriers, and the eight (K tiles of 64 instead of 32) pay
  // only where the output stage reads what it adds, with half the registers per wave, or where the contraction is very long.
  // Four waves -> eight, us: 1536x512x1024 (192 tiles, weight gradient) 35 -> 25, 1024x1024x512 15.0 -> 14.1 (weight gradient
  // 19.9 -> 16.7), x2048 48 -> 43; 2048x1024 (512 tiles), K = 32 5.8 -> 7.9, 96 8.4 -> 10.2, 512 24.0 -> 24.7, 2048 80.1 ->
  // 79.3, with a residual K = 64 12.0 -> 10.2, 512 28.5 -> 27.0, weight gradient K = 32 7.5 -> 8.7, 128 14.1 -> 12.7, 2048 88.8
  // -> 83.2; 2048x1536x512 (768) 33.5 -> 35.0
  if (tiles(64) > 512) return launch_split<true, 2, 2, 1, 1, 1>(g, p, s);
  if (tiles(64) >= 192) {
    const bool eight = tiles(64) <= 256 || g.K >= 2048 || (g.K > 32 && (g.res || g.accumulate));
    return eight ? launch_split<true, 2, 2, 2, 1, 1>(g, p, s) : launch_split<true, 2, 2, 1, 1, 1>(g, p, s);
  }
  // 32x32 tiles: eight waves to a tile where a compute unit has one and the contraction is long, unless its last K tile, 256
  // deep instead of 128, would be less than half full and the others are few.  Four waves -> eight, us: 512x512x512 7.0 -> 6.6,
  // x640 7.9 -> 8.3, x768 8.8 -> 8.2, x896 10.0 -> 10.3, x1152 11.9 -> 12.0, x2048 17.8 -> 16.1; weight gradient x640 8.1 -> 8.5,
  // x1152 13.2 -> 12.8; input gradient x640 7.8 -> 8.4, x1152 11.9 -> 12.3, x1408 13.7 -> 13.9, x1600 15.8 -> 15.6; with a residual
  // x800 11.4 -> 10.9; 512x512x128 5.7 -> 5.7; 1024x512x512 (512 tiles) 9.8 -> 11.1
  const bool filled = (g.K + 127) / 128 % 2 == 0 || g.K > (g.res ? 768 : g.tb && !g.ta ? 1536 : 1024);
  if (tiles(32) <= 256 && g.K >= 512 && filled) return launch_split<true, 1, 1, 8, 1, 1>(g, p, s);
  return launch_split<true, 1, 1, 4, 1, 1>(g, p, s);
}

}  // namespace hmy

// bf16 GEMM on tiles of 256 rows and 128, 160, 192, 224 or 256 columns, for outputs with at least some hundred of them.
//
// Eight waves, four along the rows and two along the columns, each with 4 x NB blocks of v_mfma_f32_16x16x32_bf16 (NB = columns
// over 32); two waves per SIMD.  Why this instruction: under the power limit a loop of it on registers alone sustains 2.04
// PFLOP/s over the chip, one of v_mfma_f32_32x32x16_bf16 1.82; it sums in the same order, to the same bits.
//
// What bounds the K loop, measured by taking parts out of it (cycles of a compute unit per K tile of 64 on 256x256, 2048 of them
// multiplies): LDS reads and the barrier 140; the eight load-to-LDS instructions of each wave, when they are issued together
// behind the barrier that frees a stage, 280, and waiting for what they bring 350 to 640.  So the ring is as deep as LDS allows,
// 160 KiB of it, and the two operands' stages need not be as many: with 256 columns A has three and B two.  A's tile t + 2 is
// fetched while tile t is being read, one instruction in each half step, and only B's behind the barrier.
// Products of one 256x256 tile per compute unit, K = 16384, us, two stages of both -> these: forward 437 -> 374 (1472 TFLOP/s),
// input gradient 410 -> 394, weight gradient 450 -> 416; 8192^3 796 -> 724 (1518 TFLOP/s; 32x32x16 instructions, two stages:
// 826).  Five stages of 32 steps cost more with the contraction contiguous in memory (half a cache line of every row at a time:
// 466 us), and a workgroup that went on to its next output tile with two stages filled gained less (773 us for 8192^3).
//
// The width: a product is rounds of 256 tiles, and what the last round leaves idle costs as much as what it does (the rule stands
// at tile_time).
#include <type_traits>

#include "gemm_dma.h"

namespace hmy {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f32x4 mfma16(bf16x8 rows, bf16x8 cols, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(rows, cols, c, 0, 0, 0);
}

// One operand's tile of ROWS rows and KD contraction steps in LDS.
// TR = false (contraction contiguous in memory): [row][k], the 16-byte chunks of a row XOR-swizzled by the row.
// TR = true  (contraction-major): [k][row] as loaded, chunks swizzled by k.
// The swizzles put the lanes that one LDS cycle serves on different banks: sixteen consecutive rows of one chunk, or rows of 32
// bytes from eight k (k + 0..3 and k + 8..11; what the length of a row in LDS already spreads needs no swizzle).
constexpr int KD = 64;
template <bool TR, int ROWS>
struct OpTile {
  static constexpr int kElems = ROWS * KD, kKib = kElems / 512;
  static __device__ __forceinline__ int swz_row(int row) { return (row >> 1) & 7; }
  static __device__ __forceinline__ int swz_k(int k) {
    const int by8 = (k >> 2) & 2;
    return ROWS % 128 == 0 ? ((k & 3) << 2) | by8 : ROWS % 64 == 0 ? ((k & 2) << 1) | by8 : by8;
  }
  // what lane `lane` of KiB c of the tile holds: byte offset in the operand from the K tile's first element.  Rows outside the
  // operand are clamped into it: they only feed outputs that are never stored.
  static __device__ __forceinline__ uint32_t source(int c, int lane, uint32_t ld, int row0, int nrows) {
    if (TR) {
      const int e = c * 512 + lane * 8, k = e / ROWS, chunk = (e % ROWS / 8) ^ swz_k(k);
      return (uint32_t(k) * ld + uint32_t(min(row0 + chunk * 8, ((nrows + 7) & ~7) - 8))) * 2u;
    }
    const int row = c * 8 + lane / 8, chunk = (lane % 8) ^ swz_row(row);
    return (uint32_t(min(row0 + row, nrows - 1)) * ld + uint32_t(chunk * 8)) * 2u;
  }
  // bytes from the operand's first element to the end of its last row
  static __device__ __forceinline__ uint32_t bytes(uint32_t ld, int nrows, int k) {
    return TR ? (uint32_t(k - 1) * ld + uint32_t((nrows + 7) & ~7)) * 2u : (uint32_t(nrows - 1) * ld + uint32_t(k)) * 2u;
  }
  // fragment of sixteen rows from row16 on, steps 32 ks .. + 31: lane l gets row l % 16, steps 8 (l / 16) .. + 7 of these
  static __device__ __forceinline__ bf16x8 frag(const bf16_t *s, int row16, int ks, int lane) {
    const int q = lane % 16, g = lane / 16;
    if (!TR) {
      const int row = row16 + q;
      return *reinterpret_cast<const bf16x8 *>(s + row * KD + (((4 * ks + g) ^ swz_row(row)) << 3));
    }
    const int k = 32 * ks + 8 * g + q / 4, col = row16 + 4 * (q % 4);
    const bf16_t *p = s + k * ROWS + (((col >> 3) ^ swz_k(k)) << 3) + (col & 7);
    typedef __attribute__((address_space(3))) short4v *lds_ptr;
    union { short4v s4[2]; bf16x8 b; } u;
    u.s4[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p));
    u.s4[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p + 4 * ROWS));
    return u.b;
  }
};

// Output stage of a wave's 16 MI x 16 NB outputs.  The second operand's rows went to the matrix instruction's rows: lane l holds
// row 16 i + l % 16 and the four consecutive columns 16 j + 4 (l / 16) .. + 3 in acc[i][j].  16 rows of up to 64 columns at a time
// pass through the wave's own 4 KiB of LDS and leave with 8 consecutive columns per lane.  16-byte chunks of a row of the slab are
// swizzled by the row: conflict-free both ways.
// What the output stage reads (residual, C) is fetched AHEAD parts ahead, the first before the last K tile.
template <int MI, int NB, int AHEAD>
struct Out {
  static constexpr int CH = NB < 4 ? NB : 4, PER = (NB + CH - 1) / CH, PARTS = MI * PER;   // blocks at a time, parts of a row block
  const DmaP &p;
  const Epi &e;
  const int m0, n0, lane, r8, c8;   // lane's place in a part: row 8 q + r8, columns c8 .. + 7
  Epi::Pre pre[AHEAD + 1][2];
  __device__ __forceinline__ Out(const DmaP &p_, const Epi &e_, int m, int n, int l)
      : p(p_), e(e_), m0(m), n0(n), lane(l), r8(l / 8), c8(8 * (l % 8)) {}
  __device__ __forceinline__ void prefetch(int part) {
    const int i = part / PER, j0 = part % PER * CH;
    if (!e.fast || c8 >= 16 * (NB - j0)) return;
#pragma unroll
    for (int q = 0; q < 2; ++q) e.prefetch(p, m0 + 16 * i + 8 * q + r8, n0 + 16 * j0 + c8, pre[part % (AHEAD + 1)][q]);
  }
  __device__ __forceinline__ void put(const f32x4 (&acc)[MI][NB], float *slab) {
    float4 bias8[PER];
#pragma unroll
    for (int c = 0; c < PER; ++c) {
      bias8[c] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (p.bias && e.fast && c8 < 16 * (NB - c * CH) && n0 + 16 * c * CH + c8 + 8 <= p.N)
        bias8[c] = *reinterpret_cast<const float4 *>(p.bias + n0 + 16 * c * CH + c8);
    }
#pragma unroll
    for (int part = 1; part < AHEAD; ++part) prefetch(part);
#pragma unroll
    for (int part = 0; part < PARTS; ++part) {
      const int i = part / PER, j0 = part % PER * CH;
      if (part + AHEAD < PARTS) prefetch(part + AHEAD);
#pragma unroll
      for (int b = 0; b < CH; ++b)
        if (j0 + b < NB) *reinterpret_cast<f32x4 *>(slab + (lane % 16) * 64 + (((4 * b + lane / 16) ^ (lane % 16)) << 2)) = acc[i][j0 + b];
      if (c8 < 16 * (NB - j0)) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int row = 8 * q + r8;
          e.emit8(p, m0 + 16 * i + row, n0 + 16 * j0 + c8, slab + row * 64, (c8 >> 2) ^ row, pre[part % (AHEAD + 1)][q], bias8[part % PER]);
        }
      }
    }
  }
};

// `tiles` output tiles, `grid_n` of them side by side.  Without a split of the contraction (splits = 1) a workgroup takes one;
// XCD x (workgroup id mod 8), whose L2 cache is its own, the x-th contiguous range of them, in bands of four tile rows walked
// column by column, so that neighbours in time share operand tiles in it.  With a split (few tiles, long K; NB = 4 only) the part
// varies fastest, so that an XCD works on one range of the contraction.
template <bool TA, bool TB, int NB, int SA, int SB>
__device__ __forceinline__ void tile_product(const DmaP &p, int tiles, int grid_n, int tiles_per_split, int splits) {
  extern __shared__ __attribute__((aligned(1024))) bf16_t smem[];
  constexpr int NW = 8, TM = 256, TN = 32 * NB;
  typedef OpTile<TA, TM> TileA;
  typedef OpTile<TB, TN> TileB;
  constexpr int STA = TileA::kElems, STB = TileB::kElems;                  // elements of a stage of either operand
  constexpr int LA = TileA::kKib / NW, LB = (TileB::kKib + NW - 1) / NW;   // KiB that a wave fetches of each operand's tile
  constexpr bool kEven = TileB::kKib % NW == 0;                            // (the last waves one less of B's otherwise)
  constexpr bool kHalves = NB > 4;   // a step's multiplies in two parts, so that B's fragments take half the registers
  constexpr int H0 = kHalves ? (NB + 1) / 2 : NB, H1 = NB - H0;
  constexpr int kAhead = NB < 8 || (TA && TB) ? 3 : TA || TB ? 1 : 2;   // (see k_gemm_tile)
  static_assert(LA == 4, "four fetches of A's");
  const int tid = threadIdx.x, lane = tid % 64;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int wm = wave / 2, wn = wave % 2;
  int bid = blockIdx.x, split_idx = 0;
  const bool split = splits > 1;
  if (split) {
    split_idx = bid % splits;
    bid /= splits;
  } else {
    const int x = bid % 8, per = tiles / 8, extra = tiles % 8;
    bid = x * per + min(x, extra) + bid / 8;
  }
  constexpr int kBand = 4;
  const int grid_m = tiles / grid_n, band = bid / (kBand * grid_n), first_m = band * kBand;
  const int band_rows = min(grid_m - first_m, kBand), in_band = bid - band * kBand * grid_n;
  const int m0 = (first_m + in_band % band_rows) * TM, n0 = (in_band / band_rows) * TN;
  const int kt0 = split_idx * tiles_per_split, nk = (p.K + KD - 1) / KD, kt1 = min(nk, kt0 + tiles_per_split);
  const int n = kt1 - kt0;                             // K tiles of this workgroup
  const bool half = kt1 == nk && p.K % KD != 0;        // the last of them has only 32 steps

  uint32_t off_a[LA], off_b[LB];
#pragma unroll
  for (int j = 0; j < LA; ++j) off_a[j] = TileA::source(j * NW + wave, lane, p.lda, m0, p.M);
#pragma unroll
  for (int j = 0; j < LB; ++j) off_b[j] = TileB::source(j * NW + wave, lane, p.ldb, n0, p.N);
  const uint32_t a_kstep = (TA ? uint32_t(KD) * p.lda : uint32_t(KD)) * 2u, b_kstep = (TB ? uint32_t(KD) * p.ldb : uint32_t(KD)) * 2u;
  u32x4 a_buf = buffer_of(p.A, TileA::bytes(p.lda, p.M, p.K)), b_buf = buffer_of(p.B, TileB::bytes(p.ldb, p.N, p.K));
  uint32_t a_next = uint32_t(kt0) * a_kstep, b_next = uint32_t(kt0) * b_kstep;   // of the next K tile to fetch
  int a_left = n, b_left = n;                                                    // K tiles not yet fetched
  const uint32_t lds_a = uint32_t(reinterpret_cast<uintptr_t>(smem)) + 1024u * wave, lds_b = lds_a + uint32_t(2 * SA * STA);
  auto fetch_a = [&](int j, int stage) {
    set_m0(lds_a + uint32_t(stage * (2 * STA) + j * NW * 1024));
    dma16_buffer(a_buf, off_a[j], a_next);
  };
  auto fetch_b = [&](int j, int stage) {
    if (!kEven && j * NW + wave >= TileB::kKib) return;
    set_m0(lds_b + uint32_t(stage * (2 * STB) + j * NW * 1024));
    dma16_buffer(b_buf, off_b[j], b_next);
  };
  // past the last K tile the fetches go on, from descriptors of no bytes: no branch around them
  auto advance_a = [&]() {
    a_next = --a_left > 0 ? a_next + a_kstep : 0;
    if (a_left <= 0) a_buf[2] = 0;
  };
  auto advance_b = [&]() {
    b_next = --b_left > 0 ? b_next + b_kstep : 0;
    if (b_left <= 0) b_buf[2] = 0;
  };
  // In K tile t, A's tile t + SA - 1 is fetched in front of the barrier, B's tile t + SB behind it.
#pragma unroll
  for (int s = 0; s < (SA - 1 > SB ? SA - 1 : SB); ++s) {
    if (s < SA - 1) {
#pragma unroll
      for (int j = 0; j < LA; ++j) fetch_a(j, s);
      advance_a();
    }
    if (s < SB) {
#pragma unroll
      for (int j = 0; j < LB; ++j) fetch_b(j, s);
      advance_b();
    }
  }
  // at the barrier of K tile t: until tile t + 1 has landed
  auto wait_next = [&](auto lb) {
    constexpr int l = decltype(lb)::value, a = (SA - 2) * (LA + l), b = (SB - 1) * LA + (SB - 2) * l;
    wait_vm<(a < b ? a : b)>();
  };
  const bool full = kEven || wave < TileB::kKib % NW;
  const int arow = 64 * wm, brow = 16 * NB * wn;
  bf16x8 fa[2][4], fb[2][H0];
  auto read_a = [&](int set, int i, int stage, int ks) { fa[set][i] = TileA::frag(smem + stage * STA, arow + 16 * i, ks, lane); };
  auto read_b = [&](int set, int slot, int j, int stage, int ks) {
    fb[set][slot] = TileB::frag(smem + SA * STA + stage * STB, brow + 16 * j, ks, lane);
  };
  f32x4 acc[4][NB];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[a][b][r] = 0.f;
#define HMY_FENCE() __builtin_amdgcn_sched_barrier(0)
  // between the last read of K tile t and the first of t + 1
  auto cross = [&]() {
    advance_a();
    if (full) wait_next(std::integral_constant<int, LB>());
    else wait_next(std::integral_constant<int, LB - 1>());
    __syncthreads();
  };
  // steps 32 ks .. + 31 of the K tile in stages sa, sb
  auto step = [&](int ks, int sa, int sb, int sa_next, int sb_next, int sa_fetch, bool last) {
    if constexpr (kHalves) {
#pragma unroll
      for (int m = 0; m < 4 * H0; ++m) {
        HMY_FENCE();
        acc[m % 4][m / 4] = mfma16(fb[0][m / 4], fa[ks][m % 4], acc[m % 4][m / 4]);
        HMY_FENCE();
        if (m < H1) read_b(1, m, H0 + m, sb, ks);
        if (!last && m == 4 * H0 - 3) fetch_a(ks ? 3 : 0, sa_fetch);
      }
      HMY_FENCE();
      if (!last && ks == 1) cross();
#pragma unroll
      for (int m = 0; m < 4 * H1; ++m) {
        HMY_FENCE();
        acc[m % 4][H0 + m / 4] = mfma16(fb[1][m / 4], fa[ks][m % 4], acc[m % 4][H0 + m / 4]);
        HMY_FENCE();
        if (!last || ks == 0) {
          if (m < 4) read_a(1 - ks, m, ks ? sa_next : sa, 1 - ks);
          else if (m < H0 + 4) read_b(0, m - 4, m - 4, ks ? sb_next : sb, 1 - ks);
        }
        if (!last && ks == 0 && m == H0 + 4 - 1) fetch_a(1, sa_fetch);
        if (!last && ks == 0 && m == 4 * H1 - 1) fetch_a(2, sa_fetch);
        if (!last && ks == 1) {
#pragma unroll
          for (int j = 0; j < LB; ++j)
            if (m == 1 + j * (4 * H1) / LB) fetch_b(j, sb);
        }
      }
    } else {
#pragma unroll
      for (int m = 0; m < 4 * NB; ++m) {
        HMY_FENCE();
        acc[m % 4][m / 4] = mfma16(fb[ks][m / 4], fa[ks][m % 4], acc[m % 4][m / 4]);
        HMY_FENCE();
        if (!last || ks == 0) {
          if (m < 4) read_a(1 - ks, m, ks ? sa_next : sa, 1 - ks);
          else if (m < NB + 4) read_b(1 - ks, m - 4, m - 4, ks ? sb_next : sb, 1 - ks);
        }
        if (!last && ks == 0 && m % 4 == 2) fetch_a(m / 4, sa_fetch);
        if (!last && ks == 1) {
#pragma unroll
          for (int j = 0; j < LB; ++j)
            if (m == 2 + j * (4 * NB) / LB) fetch_b(j, sb);
        }
      }
      HMY_FENCE();
      if (!last && ks == 0) cross();
    }
    if (!last && ks == 1) advance_b();
    HMY_FENCE();
  };
  {
    constexpr int a = (SA - 2) * LA, b = SB - 1;
    if (full) wait_vm<a + b * LB>();
    else wait_vm<a + b * (LB - 1)>();
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < H0; ++j) read_b(0, j, j, 0, 0);
#pragma unroll
  for (int i = 0; i < 4; ++i) read_a(0, i, 0, 0);
  int sa = 0, sb = 0;   // of K tile t
#pragma unroll 1
  for (int t = 0; t + 1 < n; ++t) {
    const int sa1 = sa + 1 == SA ? 0 : sa + 1, sa_fetch = sa == 0 ? SA - 1 : sa - 1, sb1 = sb + 1 == SB ? 0 : sb + 1;
    step(0, sa, sb, sa1, sb1, sa_fetch, false);
    step(1, sa, sb, sa1, sb1, sa_fetch, false);
    sa = sa1;
    sb = sb1;
  }
  wait_vm<0>();   // the last fetches, of nothing, have been written to LDS
  Epi e;
  e.init(p, m0, n0, TM);
  e.inside = m0 + TM <= p.M && n0 + TN <= p.N;
  // (the one layout that has no register left to keep the lane's number in)
  const int lane_again = TA || !TB ? lane : __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0));
  Out<4, NB, kAhead> out(p, e, m0 + arow, n0 + brow, lane_again);
  if (!split) out.prefetch(0);
  step(0, sa, sb, sa, sb, sa, true);
  if (!half) step(1, sa, sb, sa, sb, sa, true);
#undef HMY_FENCE
  __syncthreads();   // every wave has finished reading the stages
  if (split) {       // fp32 atomics, a row of 64 columns at a time: through LDS, 16 rows of the wave's outputs each
    if constexpr (NB == 4) {
      float *slab = reinterpret_cast<float *>(smem) + wave * 1024;
#pragma unroll
      for (int a = 0; a < 4; ++a) {
#pragma unroll
        for (int b = 0; b < 4; ++b)
          *reinterpret_cast<f32x4 *>(slab + (lane % 16) * 64 + (((4 * b + lane / 16) ^ (lane % 16)) << 2)) = acc[a][b];
        const int nn = n0 + brow + lane;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float v = slab[r * 64 + (lane ^ (r << 2))];
          const int m = m0 + arow + 16 * a + r;
          if (m < p.M && nn < p.N) atomicAdd(static_cast<float *>(p.C) + int64_t(m) * p.ldc + nn, v);
        }
      }
    }
    return;
  }
  out.put(acc, reinterpret_cast<float *>(smem) + wave * 1024);
}

// At most 224 registers (the attribute counts vector and accumulation registers apart, 112 of each), so that two waves per SIMD
// leave 64 of 512: k_adam_out, whose waves sit on ten compute units for as long as an update lasts, takes 56, and a launch of 256
// workgroups that cannot share those units runs a second round.  256 columns would take 238 to 241 registers: the output stage then
// reads two parts ahead, or one, instead of three.  Iterations of the 24-layer encoder's width with the update on the device and
// without copy engines: with 241 registers 108.6 ms (input gradient of the second MLP layer 78 us), with 224 106.4 (48; 33 alone).
// On its own a product takes 0 to 0.9 % longer, with copy engines an iteration as long as before.
template <bool TA, bool TB, int NB, int SA, int SB>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2), amdgpu_num_vgpr(112)))
void k_gemm_tile(DmaP p, int tiles, int grid_n, int tiles_per_split, int splits) {
  tile_product<TA, TB, NB, SA, SB>(p, tiles, grid_n, tiles_per_split, splits);
}
// Weight gradients: 256 columns with all their registers (241).  Held to 224 they read C one part ahead, and every launch takes 1.7 %
// longer, up to 5 % on short contractions.  Layers of width 1024 to 1600 have none on 256 columns; those of wider ones are longer
// than a round (12288x4096), or a round that shares the device with k_adam_out only where there are no copy engines.
template <int NB, int SA, int SB>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
void k_gemm_tile_dw(DmaP p, int tiles, int grid_n, int tiles_per_split, int splits) {
  tile_product<true, true, NB, SA, SB>(p, tiles, grid_n, tiles_per_split, splits);
}

inline int check_launch(const char *what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(HMY_E_HIP, "launch of %s failed: %s", what, hipGetErrorString(e));
  return HMY_OK;
}

template <int NB, int SA, int SB>
int launch_tile(const hmy_gemm_desc &g, const DmaP &p, int splits, hipStream_t s) {
  constexpr int TM = 256, TN = 32 * NB;
  const int gm = (g.M + TM - 1) / TM, gn = (g.N + TN - 1) / TN, nk = (g.K + KD - 1) / KD, tiles = gm * gn;
  const int tps = (nk + splits - 1) / splits;
  splits = (nk + tps - 1) / tps;
  const size_t lds = size_t(SA * TM + SB * TN) * KD * sizeof(bf16_t);
  static_assert((SA * TM + SB * TN) * KD * 2 <= 160 * 1024, "a compute unit's LDS");
  const dim3 grid(tiles * splits), block(512);
  if (!g.ta && !g.tb) hipLaunchKernelGGL((k_gemm_tile<false, false, NB, SA, SB>), grid, block, lds, s, p, tiles, gn, tps, splits);
  else if (!g.ta && g.tb) hipLaunchKernelGGL((k_gemm_tile<false, true, NB, SA, SB>), grid, block, lds, s, p, tiles, gn, tps, splits);
  else if (g.ta && !g.tb) hipLaunchKernelGGL((k_gemm_tile<true, false, NB, SA, SB>), grid, block, lds, s, p, tiles, gn, tps, splits);
  else hipLaunchKernelGGL((k_gemm_tile_dw<NB, SA, SB>), grid, block, lds, s, p, tiles, gn, tps, splits);
  return check_launch("gemm_tile");
}

}  // namespace

int launch_gemm_tile(const hmy_gemm_desc &g, int nb, int splits, stream_t st) {
  const DmaP p = dma_params(g);
  const hipStream_t s = (hipStream_t)st;
  if (splits > 1 && (nb != 4 || !g.accumulate || !g.c_fp32 || g.bias || g.res))
    return fail(HMY_E_INVALID, "gemm: the parts of a split contraction meet in an fp32 sum on tiles of 128 columns");
  if (nb == 8) return launch_tile<8, 3, 2>(g, p, 1, s);
  if (nb == 7) return launch_tile<7, 3, 2>(g, p, 1, s);
  if (nb == 6) return launch_tile<6, 3, 2>(g, p, 1, s);
  if (nb == 5) return launch_tile<5, 3, 3>(g, p, 1, s);
  if (nb == 4) return launch_tile<4, 3, 4>(g, p, splits, s);
  return fail(HMY_E_INVALID, "gemm: no tiles of %d columns", 32 * nb);
}

}  // namespace hmy

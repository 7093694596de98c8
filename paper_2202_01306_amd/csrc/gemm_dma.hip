// bf16 GEMM on the matrix cores with operand tiles streamed HBM -> LDS by the
// load-to-LDS instruction (global_load_lds_dwordx4): no staging registers, so a ring
// of S LDS stages keeps up to S-1 K tiles in flight per workgroup while one is
// multiplied, which is what hides HBM latency when an operand is not cache-resident
// (activations of another microbatch, weights that have just arrived from the host).
//
// 128x128 block tile, four wavefronts of 64x64 (2x2 v_mfma_f32_32x32x16_bf16), K tile
// BK in {32, 64}.  One s_waitcnt vmcnt + one barrier per K tile, placed inside the tile
// so that the first fragments of the next tile are requested before this tile's last
// multiplies.  Fragments are read one (BK 32) or two (BK 64) 16-deep steps ahead of
// their multiplies; every LDS read and load-to-LDS is issued right behind a multiply.
//
// A load-to-LDS instruction writes 64 lanes x 16 bytes to one contiguous KiB of LDS
// (lane i at byte 16 i) from per-lane global addresses, so the bank swizzle is applied
// on the global side: the lane that owns LDS slot p of a row fetches the chunk that
// the swizzle maps to p.
//
// LDS layouts.  Operand with the contraction index contiguous in memory: [row][k],
// 16-byte chunks XOR-swizzled by the row, read with ds_read_b128.  Operand stored
// contraction-major: kept as loaded, [k][row], chunks swizzled by k, read through
// ds_read_b64_tr_b16 with k rows 8h..8h+3 and 8h+4..8h+7 (h = lane/32), which is the
// same contraction order as the 16-byte read of the other layout.
//
// Larger outputs go to tiles of 256 rows (gemm_tile.hip), small ones to 64x64 tiles (further down).
//
// Tuning switches (read once per process): HMY_GEMM_BK = 32 | 64 overrides the K tile of the 128x128 kernel,
// HMY_GEMM_STAGES = 3 | 4 its ring's depth, and with either of them every shape takes it; HMY_GEMM_TILE = 128 | 256 names it or
// tiles of 256x256.  With any of them set no shape takes the 64x64 tiles.
#include <algorithm>
#include <climits>
#include <cstdlib>

#include "gemm_dma.h"

namespace hmy {

namespace {

constexpr int BM = 128, NT = 256;  // square block tile, threads

// element address inside a [row][k] tile of BK columns (BK/8 chunks per row)
template <int BK>
__device__ __forceinline__ int addr_rk(int row, int chunk) {
  if (BK == 32) return row * 32 + ((chunk ^ ((row >> 2) & 3)) << 3);
  return row * 64 + ((chunk ^ ((row >> 1) & 7)) << 3);
}
// element address inside a [k][row] tile (16 chunks per k-row, swizzled by k)
__device__ __forceinline__ int addr_kr(int k, int col) {
  return k * BM + ((((col >> 3) ^ ((k & 3) << 2)) & 15) << 3) + (col & 7);
}

// the 16-byte-per-lane copy with a full address per lane
__device__ __forceinline__ void dma16_at(const void *addr, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(addr), "s"(lds_addr) : "memory");
}
// contraction steps past the operands' end come from here
__device__ __attribute__((aligned(256))) bf16_t g_zero_page[128];   // zero-initialised, never written

// Per-thread, loop-invariant byte offsets of this thread's lanes of every KiB it copies.
// TR = false: memory [row][k]; KiB c holds rows c*R..c*R+R-1 (R = 512/BK), lane i owns slot i%(BK/8) of row i/(BK/8).
// TR = true : memory [k][row]; KiB c holds k rows 4c..4c+3, lane i owns slot i%16 of k row i/16.
// Wave w copies KiBs c = 4 j + w, j = 0..BK/16-1.  Rows outside the operand are
// clamped into it: they only feed outputs that are never stored.
template <bool TR, int BK>
struct Dma {
  static constexpr int NJ = BK / 16;
  uint32_t off[TR ? 1 : NJ];
  uint32_t step;  // TR: bytes between this thread's consecutive KiBs
  __device__ __forceinline__ void init(uint32_t ld, int row0, int nrows, int lane, int wave) {
    if (!TR) {
      constexpr int CH = BK / 8, R = 64 / CH;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int row = (4 * j + wave) * R + lane / CH, slot = lane % CH;
        const int chunk = BK == 32 ? (slot ^ ((row >> 2) & 3)) : (slot ^ ((row >> 1) & 7));
        off[j] = (uint32_t(min(row0 + row, nrows - 1)) * ld + uint32_t(chunk * 8)) * 2u;
      }
      step = 0;
    } else {
      const int kq = lane / 16, slot = lane % 16;
      const int chunk = slot ^ (kq << 2);   // k & 3 == lane / 16 for every KiB
      const int col = min(row0 + chunk * 8, ((nrows + 7) & ~7) - 8);
      off[0] = (uint32_t(4 * wave + kq) * ld + uint32_t(col)) * 2u;
      step = 16u * ld * 2u;
    }
  }
  // base: operand base advanced to the K tile; lds: byte address of the tile's stage
  __device__ __forceinline__ void issue_one(const bf16_t *base, uint32_t lds, int wave, int j) const {
    dma16(base, TR ? off[0] + uint32_t(j) * step : off[j], lds + uint32_t(4 * j + wave) * 1024u);
  }
  __device__ __forceinline__ void issue(const bf16_t *base, uint32_t lds, int wave) const {
#pragma unroll
    for (int j = 0; j < NJ; ++j) issue_one(base, lds, wave, j);
  }
};

template <bool TR, int BK>
__device__ __forceinline__ bf16x8 frag(const bf16_t *s, int row32, int ks, int lane) {
  if (!TR) {
    return *reinterpret_cast<const bf16x8 *>(s + addr_rk<BK>(row32 + lane % 32, 2 * ks + lane / 32));
  } else {
    const int q = lane % 16, g16 = (lane / 16) % 2, h = lane / 32;
    const int k = 16 * ks + 8 * h + q / 4, col = row32 + 16 * g16 + 4 * (q % 4);
    typedef __attribute__((address_space(3))) short4v *lds_ptr;
    union { short4v s4[2]; bf16x8 b; } u;
    u.s4[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(s + addr_kr(k, col)));
    u.s4[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(s + addr_kr(k + 4, col)));
    return u.b;
  }
}

template <bool TA, bool TB, int BK, int S>
__global__ __launch_bounds__(NT) void k_gemm_dma(DmaP p, int tiles_per_split, int grid_n, int splits) {
  extern __shared__ __attribute__((aligned(1024))) bf16_t smem[];
  constexpr int TILE = BM * BK;            // elements per operand per stage
  constexpr int L = 2 * (BK / 16);         // load-to-LDS instructions per thread per K tile
  static_assert(S >= 3, "the tile being fetched gets its last part after the barrier: two tiles must be ahead of it");
  static_assert((S - 1) * L <= 63, "vmcnt is a 6-bit counter");
  const int tid = threadIdx.x, lane = tid % 64;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int wm = wave / 2, wn = wave % 2;
  // Workgroup b runs on XCD b % 8, each with an L2 of its own.  Without a split of the contraction: XCD x gets
  // the x-th contiguous range of tile ids (ranges differ by at most one), tiles ordered in bands of 8 tile rows
  // walked column by column, so that neighbours in time share operand tiles in that L2.  With a split (few
  // tiles, long K): the split index varies fastest, so an XCD works on ONE K range of every tile and each
  // byte of A and B is fetched by one XCD only (with the tile fastest, every XCD streamed all of A).
  int bid = blockIdx.x, split_idx = 0;
  const int nb = gridDim.x / splits, grid_m = nb / grid_n;
  if (splits > 1) {
    split_idx = bid % splits;
    bid /= splits;
  } else {
    const int x = bid % 8, per = nb / 8, extra = nb % 8;
    bid = x * per + min(x, extra) + bid / 8;
  }
  constexpr int kBand = 8;
  const int band = bid / (kBand * grid_n), first_m = band * kBand;
  const int band_rows = min(grid_m - first_m, kBand);
  const int in_band = bid - band * kBand * grid_n;
  const int m0 = (first_m + in_band % band_rows) * BM, n0 = (in_band / band_rows) * BM;

  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int nk_all = p.K / BK;
  const int kt0 = split_idx * tiles_per_split;
  const int n = min(nk_all, kt0 + tiles_per_split) - kt0;   // K tiles of this workgroup
  Dma<TA, BK> da;
  Dma<TB, BK> db;
  da.init(p.lda, m0, p.M, lane, wave);
  db.init(p.ldb, n0, p.N, lane, wave);
  const uint32_t lds0 = uint32_t(reinterpret_cast<uintptr_t>(smem));
  // element strides of one K tile in each operand
  const uint64_t a_kstep = TA ? uint64_t(BK) * p.lda : uint64_t(BK);
  const uint64_t b_kstep = TB ? uint64_t(BK) * p.ldb : uint64_t(BK);
  const bf16_t *a_next = p.A + uint64_t(kt0) * a_kstep;
  const bf16_t *b_next = p.B + uint64_t(kt0) * b_kstep;
  auto issue = [&](int stage) {
    da.issue(a_next, lds0 + uint32_t(stage) * uint32_t(4 * TILE), wave);
    db.issue(b_next, lds0 + uint32_t(stage) * uint32_t(4 * TILE) + uint32_t(2 * TILE), wave);
    a_next += a_kstep;
    b_next += b_kstep;
  };
#pragma unroll
  for (int s = 0; s < S; ++s)
    if (s < n) issue(s);

  const int arow = wm * 64, brow = wn * 64;
  constexpr int KS = BK / 16;
  // operand fragments: read one step ahead of their multiplies (two buffers) with K tiles
  // of 32, two steps ahead (four buffers, indexed by the step within the tile) with 64
  constexpr int NBUF = KS == 4 ? 4 : 2;
  bf16x8 fa[NBUF][2], fb[NBUF][2];
  auto load_frags = [&](int buf, int stage, int ks) {
    const bf16_t *a_s = smem + stage * (2 * TILE), *b_s = a_s + TILE;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      fa[buf][i] = frag<TA, BK>(a_s, arow + 32 * i, ks, lane);
      fb[buf][i] = frag<TB, BK>(b_s, brow + 32 * i, ks, lane);
    }
  };
  // tile 0 has landed once at most the S-1 tiles issued after it are outstanding
  if (n > S - 1) wait_vm<(S - 1) * L>();
  else wait_vm<0>();
  __syncthreads();
  if (n > 0) {
    load_frags(0, 0, 0);
    if (KS == 4) load_frags(1, 0, 1);
  }
  // One 16-deep step: the four multiplies on fragment buffer `cur`, each followed by one
  // of the four fragment reads of a later step (into buffer `nxt`) and, twice, by one
  // load-to-LDS of the tile being fetched.  A wavefront issues in order and an LDS read
  // occupies its issue slot for some 20 cycles, so reads grouped in front of the
  // multiplies would delay them; placed behind a multiply each read issues while the
  // matrix pipe works through that multiply's 32 cycles.  The fences pin this order.
#define HMY_FENCE() __builtin_amdgcn_sched_barrier(0)
  auto step = [&](int cur, int nxt, bool reads, int nstage, int nks, bool fetch, int fstage, int part) {
    const bf16_t *a_s = smem + nstage * (2 * TILE), *b_s = a_s + TILE;
    const uint32_t fl = lds0 + uint32_t(fstage) * uint32_t(4 * TILE);
    HMY_FENCE();
    acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[cur][0], fb[cur][0], acc[0][0], 0, 0, 0);
    HMY_FENCE();
    if (reads) fa[nxt][0] = frag<TA, BK>(a_s, arow, nks, lane);
    HMY_FENCE();
    acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[cur][0], fb[cur][1], acc[0][1], 0, 0, 0);
    HMY_FENCE();
    if (reads) fb[nxt][0] = frag<TB, BK>(b_s, brow, nks, lane);
    if (fetch) da.issue_one(a_next, fl, wave, part);
    HMY_FENCE();
    acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[cur][1], fb[cur][0], acc[1][0], 0, 0, 0);
    HMY_FENCE();
    if (reads) fb[nxt][1] = frag<TB, BK>(b_s, brow + 32, nks, lane);
    HMY_FENCE();
    acc[1][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[cur][1], fb[cur][1], acc[1][1], 0, 0, 0);
    HMY_FENCE();
    if (reads) fa[nxt][1] = frag<TA, BK>(a_s, arow + 32, nks, lane);
    if (fetch) db.issue_one(b_next, fl + uint32_t(2 * TILE), wave, part);
    HMY_FENCE();
  };
  int stage = 0;      // stage holding tile t
  int freed = S - 1;  // stage of tile t-1: free since the barrier inside that tile
  const bool split = splits > 1;
  Epi e;
  e.init(p, m0, n0, BM);
  const int m_tile = m0 + wm * 64, n_tile = n0 + wn * 64;
  Epi::Pre pre[2][4];
  float4 bias8 = make_float4(0.f, 0.f, 0.f, 0.f);
  // lane's share of the output: slab i (32 rows), pass q -> row 8 q + lane/8, columns 8 (lane%8) .. +7
  auto prefetch_outputs = [&]() {
    if (split || !e.fast) return;
    if (p.bias && (e.inside || n_tile + 8 * (lane % 8) + 8 <= p.N))
      bias8 = *reinterpret_cast<const float4 *>(p.bias + n_tile + 8 * (lane % 8));
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) e.prefetch(p, m_tile + 32 * i + 8 * q + lane / 8, n_tile + 8 * (lane % 8), pre[i][q]);
  };
  if constexpr (KS == 4) {
    for (int t = 0; t + 1 < n; ++t) {
      const int next = stage + 1 == S ? 0 : stage + 1;
      // tile t+S-1 goes to the stage tile t-1 has left, a part per step
      const bool fetch = t > 0 && t + S - 1 < n;
      step(0, 2, true, stage, 2, fetch, freed, 0);
      step(1, 3, true, stage, 3, fetch, freed, 1);
      // every read of tile t has been issued.  Tile t+1 has landed once at most the S-3
      // whole tiles issued after it and two parts of the tile being fetched are outstanding.
      if (t + S - 1 < n) wait_vm<(S - 3) * L + 4>();
      else wait_vm<0>();
      __syncthreads();   // tile t+1 visible to every wave; every wave is done reading tile t
      step(2, 0, true, next, 0, fetch, freed, 2);
      step(3, 1, true, next, 1, fetch, freed, 3);
      if (fetch) {
        a_next += a_kstep;
        b_next += b_kstep;
      }
      freed = stage;
      stage = next;
    }
    prefetch_outputs();
    if (n > 0) {   // last tile: nothing left to fetch or wait for
      step(0, 2, true, stage, 2, false, 0, 0);
      step(1, 3, true, stage, 3, false, 0, 0);
      step(2, 0, false, stage, 0, false, 0, 0);
      step(3, 1, false, stage, 0, false, 0, 0);
    }
  } else {
    for (int t = 0; t + 1 < n; ++t) {
      const int next = stage + 1 == S ? 0 : stage + 1;
      const bool fetch = t > 0 && t + S - 1 < n;
#pragma unroll
      for (int ks = 0; ks + 1 < KS; ++ks) step(ks & 1, (ks + 1) & 1, true, stage, ks + 1, fetch, freed, ks);
      // every read of tile t has been issued.  Tile t+1 has landed once at most the S-2
      // tiles issued after it (the one being fetched lacks its last part) are outstanding.
      if (t + S - 1 < n) wait_vm<(S - 2) * L - 2>();
      else wait_vm<0>();
      __syncthreads();   // tile t+1 visible to every wave; every wave is done reading tile t
      step((KS - 1) & 1, 0, true, next, 0, fetch, freed, KS - 1);
      if (fetch) {
        a_next += a_kstep;
        b_next += b_kstep;
      }
      freed = stage;
      stage = next;
    }
    prefetch_outputs();
    if (n > 0) {   // last tile: nothing left to fetch or wait for
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) step(ks & 1, (ks + 1) & 1, ks + 1 < KS, stage, ks + 1, false, 0, 0);
    }
  }
#undef HMY_FENCE

  // Epilogue.  Accumulator register r of lane l holds row 8*(r/4) + 4*(l/32) + r%4,
  // column l%32 of a 32x32 block: stored from there, a wavefront would write 2-byte
  // elements in 64-byte runs.  Each wave instead passes its 64x64 outputs, 32 rows at a
  // time, through 8 KiB of LDS (the operand stages are free now) and leaves with 8
  // consecutive columns per lane: 16-byte stores, 128 contiguous bytes per row.  Rows
  // that differ in bit 2 are written by the two lane halves at once; flipping bit 5 of
  // the column for them keeps the halves on different banks.
  if (split) {   // fp32 atomics: one column per lane, straight from the accumulator layout
    const int m_base = m0 + wm * 64 + 4 * (lane / 32), n_base = n0 + wn * 64 + lane % 32;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int nn = n_base + j * 32;
      if (nn >= p.N) continue;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int m = m_base + i * 32 + 8 * (r / 4) + r % 4;
          if (m < p.M) atomicAdd(static_cast<float *>(p.C) + int64_t(m) * p.ldc + nn, acc[i][j][r]);
        }
    }
    return;
  }
  __syncthreads();   // every wave has finished reading the operand stages
  float *slab = reinterpret_cast<float *>(smem) + wave * 2048;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = 8 * (r / 4) + 4 * (lane / 32) + r % 4, col = 32 * j + lane % 32;
        slab[row * 64 + (col ^ (((row >> 2) & 1) << 5))] = acc[i][j][r];
      }
    if (e.fast) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int row = 8 * q + lane / 8, c0 = 8 * (lane % 8);
        const float *src = slab + row * 64 + (c0 ^ (((row >> 2) & 1) << 5));
        e.emit8(p, m_tile + 32 * i + row, n_tile + c0, src, pre[i][q], bias8);
      }
    } else {
#pragma unroll 1
      for (int idx = lane; idx < 32 * 64; idx += 64) {   // one row of 64 columns per pass
        const int row = idx / 64, col = idx % 64;
        const int m = m_tile + 32 * i + row, nn = n_tile + col;
        if (m < p.M && nn < p.N) e.emit_one(p, m, nn, slab[row * 64 + (col ^ (((row >> 2) & 1) << 5))]);
      }
    }
  }
}

// ---- small outputs --------------------------------------------------------------------
// The same GEMM on 64x64 tiles for outputs whose 128x128 tiles leave most compute units idle: what bounds those is the
// length of one workgroup's life (launch, first tiles' way from memory, K loop, output stage), so four times as many
// workgroups with a quarter of the work each finish sooner.  Four waves of one 32x32 output each, K tiles of 64, a ring
// of four stages (64 KiB, two workgroups per unit): a contraction of up to 256 is in flight as a whole before the first
// multiply.  Where neither splits the contraction and it is a multiple of 32, it is summed in the same order as by the
// larger kernels: same results, bit for bit.  (Sums of weight gradients are split by this kernel's own count of tiles, and
// the larger kernels take a ragged contraction in two parts.)
// Contractions that are no multiple of 64 are taken as they are: steps past K of the last tile come from a page of zeros,
// and a 16-byte chunk that K cuts is masked in LDS.
constexpr int ST = 64, SK = 64, SS = 4;               // tile side, K tile, stages
constexpr int kSmallOp = ST * SK;                      // elements of one operand and stage

// element address inside a [k][64 rows] tile: 8 chunks per k-row of 128 bytes, swizzled so that the four k-rows of a
// transposed read fall on different banks
__device__ __forceinline__ int addr_kr64(int k, int col) { return k * ST + ((((col >> 3) ^ ((k & 2) << 1)) & 7) << 3) + (col & 7); }

template <bool TR>
struct SmallDma {
  uint32_t off[2];
  int k_of[2];      // contraction step of the lane's chunk inside a tile (TR: its k-row; else its first element)
  __device__ __forceinline__ void init(uint32_t ld, int row0, int nrows, int lane, int wave) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if (!TR) {   // KiB 4 j + wave: rows 8 c .. 8 c + 7, lane owns slot lane%8 of row lane/8
        const int row = (4 * j + wave) * 8 + lane / 8, chunk = (lane % 8) ^ ((row >> 1) & 7);
        off[j] = (uint32_t(min(row0 + row, nrows - 1)) * ld + uint32_t(chunk * 8)) * 2u;
        k_of[j] = chunk * 8;
      } else {     // KiB 4 j + wave: k-rows 8 c .. 8 c + 7
        const int k = (4 * j + wave) * 8 + lane / 8, chunk = (lane % 8) ^ ((k & 2) << 1);
        const int col = min(row0 + chunk * 8, ((nrows + 7) & ~7) - 8);
        off[j] = (uint32_t(k) * ld + uint32_t(col)) * 2u;
        k_of[j] = k;
      }
    }
  }
  // `left`: contraction steps from this tile's first to the end of the operand
  __device__ __forceinline__ void issue(const bf16_t *base, uint32_t lds, int wave, int left) const {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const uint32_t at = lds + uint32_t(4 * j + wave) * 1024u;
      if (left >= SK) {
        dma16(base, off[j], at);
      } else {
        const char *p = reinterpret_cast<const char *>(base) + off[j];
        dma16_at(k_of[j] < left ? p : reinterpret_cast<const char *>(g_zero_page), at);
      }
    }
  }
};
template <bool TR>
__device__ __forceinline__ bf16x8 small_frag(const bf16_t *s, int row32, int ks, int lane) {
  if (!TR) return *reinterpret_cast<const bf16x8 *>(s + addr_rk<64>(row32 + lane % 32, 2 * ks + lane / 32));
  const int q = lane % 16, g16 = (lane / 16) % 2, h = lane / 32;
  const int k = 16 * ks + 8 * h + q / 4, col = row32 + 16 * g16 + 4 * (q % 4);
  typedef __attribute__((address_space(3))) short4v *lds_ptr;
  union { short4v s4[2]; bf16x8 b; } u;
  u.s4[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(s + addr_kr64(k, col)));
  u.s4[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(s + addr_kr64(k + 4, col)));
  return u.b;
}

template <bool TA, bool TB>
__global__ __launch_bounds__(NT) void k_gemm_dma64(DmaP p, int tiles_per_split, int grid_n, int splits) {
  __shared__ __attribute__((aligned(1024))) bf16_t smem[SS * 2 * kSmallOp];
  constexpr int L = 4;   // load-to-LDS instructions per thread per K tile
  const int tid = threadIdx.x, lane = tid % 64;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int wm = wave / 2, wn = wave % 2;
  int bid = blockIdx.x, split_idx = 0;
  const int nb = gridDim.x / splits, grid_m = nb / grid_n;
  if (splits > 1) {   // as in the 128x128 kernel
    split_idx = bid % splits;
    bid /= splits;
  } else {
    const int x = bid % 8, per = nb / 8, extra = nb % 8;
    bid = x * per + min(x, extra) + bid / 8;
  }
  constexpr int kBand = 8;
  const int band = bid / (kBand * grid_n), first_m = band * kBand;
  const int band_rows = min(grid_m - first_m, kBand);
  const int in_band = bid - band * kBand * grid_n;
  const int m0 = (first_m + in_band % band_rows) * ST, n0 = (in_band / band_rows) * ST;

  const int kt0 = split_idx * tiles_per_split;
  const int n = min((p.K + SK - 1) / SK, kt0 + tiles_per_split) - kt0;   // K tiles of this workgroup
  SmallDma<TA> da;
  SmallDma<TB> db;
  da.init(p.lda, m0, p.M, lane, wave);
  db.init(p.ldb, n0, p.N, lane, wave);
  const uint32_t lds0 = uint32_t(reinterpret_cast<uintptr_t>(smem));
  const uint64_t a_kstep = TA ? uint64_t(SK) * p.lda : uint64_t(SK), b_kstep = TB ? uint64_t(SK) * p.ldb : uint64_t(SK);
  auto issue = [&](int t) {   // tile t of this workgroup into stage t % SS
    const uint32_t at = lds0 + uint32_t(t % SS) * uint32_t(4 * kSmallOp);
    const int left = p.K - (kt0 + t) * SK;
    da.issue(p.A + uint64_t(kt0 + t) * a_kstep, at, wave, left);
    db.issue(p.B + uint64_t(kt0 + t) * b_kstep, at + uint32_t(2 * kSmallOp), wave, left);
  };
#pragma unroll
  for (int t = 0; t < SS; ++t)
    if (t < n) issue(t);

  Epi e;
  e.init(p, m0, n0, ST);
  const bool split = splits > 1;
  // lane's share of the output: pass q -> row 16 q + lane/4, columns 8 (lane%4) .. +7 of the wave's 32x32
  const int m_tile = m0 + wm * 32, n_tile = n0 + wn * 32, n_lane = n_tile + 8 * (lane % 4);
  Epi::Pre pre[2];
  float4 bias8 = make_float4(0.f, 0.f, 0.f, 0.f);

  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  for (int t = 0; t < n; ++t) {
    // tile t has landed once at most the tiles issued after it are outstanding: t + 1 .. t + SS - 1 before the first
    // refill, up to t + SS - 2 from then on
    const int later = min(n, t == 0 ? SS : t + SS - 1) - t - 1;
    if (later >= 3) wait_vm<3 * L>();
    else if (later == 2) wait_vm<2 * L>();
    else if (later == 1) wait_vm<L>();
    else wait_vm<0>();
    __syncthreads();   // tile t visible to every wave; every wave has read tile t - 1
    if (t > 0 && t - 1 + SS < n) issue(t - 1 + SS);
    bf16_t *a_s = smem + (t % SS) * (2 * kSmallOp), *b_s = a_s + kSmallOp;
    const int left = p.K - (kt0 + t) * SK;
    if (left < SK && left % 8 && (!TA || !TB)) {   // K cuts a chunk of the operands whose rows run along it
      if (tid < ST) {
        const int at = addr_rk<64>(tid, left / 8), keep = left % 8;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          if (k < keep) continue;
          if (!TA) a_s[at + k] = from_f32<bf16_t>(0.f);
          if (!TB) b_s[at + k] = from_f32<bf16_t>(0.f);
        }
      }
      __syncthreads();
    }
    bf16x8 fa[4], fb[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      fa[ks] = small_frag<TA>(a_s, wm * 32, ks, lane);
      fb[ks] = small_frag<TB>(b_s, wn * 32, ks, lane);
    }
    if (t + 1 == n && !split && e.fast) {   // what the output stage adds arrives during the last multiplies
      if (p.bias && (e.inside || n_lane + 8 <= p.N)) bias8 = *reinterpret_cast<const float4 *>(p.bias + n_lane);
#pragma unroll
      for (int q = 0; q < 2; ++q) e.prefetch(p, m_tile + 16 * q + lane / 4, n_lane, pre[q]);
    }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ks], fb[ks], acc, 0, 0, 0);
  }
  if (split) {
    const int nn = n_tile + lane % 32;
    if (nn >= p.N) return;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = m_tile + 8 * (r / 4) + 4 * (lane / 32) + r % 4;
      if (m < p.M) atomicAdd(static_cast<float *>(p.C) + int64_t(m) * p.ldc + nn, acc[r]);
    }
    return;
  }
  // through LDS, as in the 128x128 kernel: 4 KiB per wave, rows of 32 columns
  __syncthreads();
  float *slab = reinterpret_cast<float *>(smem) + wave * 1024;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = 8 * (r / 4) + 4 * (lane / 32) + r % 4;
    slab[row * 32 + ((lane % 32) ^ ((row & 4) << 1))] = acc[r];
  }
  if (e.fast) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int row = 16 * q + lane / 4, c0 = 8 * (lane % 4);
      e.emit8(p, m_tile + row, n_lane, slab + row * 32 + (c0 ^ ((row & 4) << 1)), pre[q], bias8);
    }
  } else {
#pragma unroll 1
    for (int idx = lane; idx < 32 * 32; idx += 64) {
      const int row = idx / 32, col = idx % 32;
      const int m = m_tile + row, nn = n_tile + col;
      if (m < p.M && nn < p.N) e.emit_one(p, m, nn, slab[row * 32 + (col ^ ((row & 4) << 1))]);
    }
  }
}

// The same for contractions that are a multiple of 64, and for any where both operands are stored contraction-major: steps past
// K of the last tile are rows past the operand, which the descriptors read as zeros.  What bounds a workgroup that has its SIMDs to
// itself is each wave's own instruction stream: 128 cycles of multiplies per K tile among branches, waits and LDS reads that
// follow one another.  So: no branch in the loop (the fetches go through buffer descriptors, as on tiles of 256 rows, and end by
// themselves), the next tile's fragments are read while this one's are multiplied, and what the output stage adds is fetched
// before the loop.  Measured, us, kernel above -> this: 600x768x3072 22.1 -> 15.4 (input gradient 22.6 -> 14.4), 480x768x768 8.2 ->
// 6.9; weight gradient 1024x1024x1024 12.1 -> 8.7, 768x3072x600 16.2 -> 14.0, 256x1024x480 6.6 -> 5.4.  It takes longer before its
// first multiply: short contractions stay with the kernel above (`even_pays`).
// `bid` of `workgroups`: a launch may hold more than this product.
template <bool TA, bool TB>
__device__ __forceinline__ void even_tile(const DmaP &p, int tiles_per_split, int grid_n, int splits, int bid, int workgroups,
                                          bf16_t *smem) {
  constexpr int L = 4;   // load-to-LDS instructions per thread per K tile
  static_assert(SS == 4, "stages are counted modulo 4");
  const int tid = threadIdx.x, lane = tid % 64;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int wm = wave / 2, wn = wave % 2;
  int split_idx = 0;
  const int nb = workgroups / splits, grid_m = nb / grid_n;
  if (splits > 1) {   // as in the 128x128 kernel
    split_idx = bid % splits;
    bid /= splits;
  } else {
    const int x = bid % 8, per = nb / 8, extra = nb % 8;
    bid = x * per + min(x, extra) + bid / 8;
  }
  constexpr int kBand = 8;
  const int band = bid / (kBand * grid_n), first_m = band * kBand;
  const int band_rows = min(grid_m - first_m, kBand);
  const int in_band = bid - band * kBand * grid_n;
  const int m0 = (first_m + in_band % band_rows) * ST, n0 = (in_band / band_rows) * ST;
  const int kt0 = split_idx * tiles_per_split;
  const int n = min((p.K + SK - 1) / SK, kt0 + tiles_per_split) - kt0;   // K tiles of this workgroup

  Epi e;
  e.init(p, m0, n0, ST);
  const bool split = splits > 1;
  // lane's share of the output: pass q -> row 16 q + lane/4, columns 8 (lane%4) .. +7 of the wave's 32x32
  const int m_tile = m0 + wm * 32, n_tile = n0 + wn * 32, n_lane = n_tile + 8 * (lane % 4);
  Epi::Pre pre[2];
  float4 bias8 = make_float4(0.f, 0.f, 0.f, 0.f);
  if (!split && e.fast) {
    if (p.bias && (e.inside || n_lane + 8 <= p.N)) bias8 = *reinterpret_cast<const float4 *>(p.bias + n_lane);
#pragma unroll
    for (int q = 0; q < 2; ++q) e.prefetch(p, m_tile + 16 * q + lane / 4, n_lane, pre[q]);
  }

  // byte offsets of this thread's lanes of the KiBs its wave copies: 2 w and 2 w + 1 of each operand's eight
  uint32_t off[2][2];
#pragma unroll
  for (int op = 0; op < 2; ++op)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const uint32_t ld = op ? p.ldb : p.lda;
      const int first = op ? n0 : m0, rows = op ? p.N : p.M, line = 8 * (2 * wave + j) + lane / 8;   // row, or k row
      if (op ? TB : TA) {
        const int col = min(first + ((lane % 8) ^ ((line & 2) << 1)) * 8, ((rows + 7) & ~7) - 8);
        off[op][j] = (uint32_t(line) * ld + uint32_t(col)) * 2u;
      } else {
        off[op][j] = (uint32_t(min(first + line, rows - 1)) * ld + uint32_t(((lane % 8) ^ ((line >> 1) & 7)) * 8)) * 2u;
      }
    }
  const uint32_t lds0 = uint32_t(reinterpret_cast<uintptr_t>(smem)) + 2048u * wave;
  const uint32_t a_kstep = TA ? uint32_t(SK) * p.lda * 2u : uint32_t(SK) * 2u, b_kstep = TB ? uint32_t(SK) * p.ldb * 2u : uint32_t(SK) * 2u;
  u32x4 a_buf = buffer_of(p.A, uint32_t(TA ? p.K : p.M) * p.lda * 2u), b_buf = buffer_of(p.B, uint32_t(TB ? p.K : p.N) * p.ldb * 2u);
  uint32_t a_next = uint32_t(kt0) * a_kstep, b_next = uint32_t(kt0) * b_kstep;   // byte offset of the next K tile to fetch
  int fetched = 0;
  auto fetch = [&]() {   // the next tile, or, past the last one, nothing
    const uint32_t at = lds0 + uint32_t(fetched & 3) * uint32_t(4 * kSmallOp);
    set_m0(at);
    dma16_buffer(a_buf, off[0][0], a_next);
    set_m0(at + 1024u);
    dma16_buffer(a_buf, off[0][1], a_next);
    set_m0(at + uint32_t(2 * kSmallOp));
    dma16_buffer(b_buf, off[1][0], b_next);
    set_m0(at + uint32_t(2 * kSmallOp) + 1024u);
    dma16_buffer(b_buf, off[1][1], b_next);
    ++fetched;
    a_next = fetched < n ? a_next + a_kstep : 0;
    b_next = fetched < n ? b_next + b_kstep : 0;
    if (fetched >= n) a_buf[2] = b_buf[2] = 0;
  };
#pragma unroll
  for (int t = 0; t < SS; ++t) fetch();

  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  bf16x8 fa[2][4], fb[2][4];
  auto read = [&](int buf, int stage) {
    const bf16_t *a_s = smem + stage * (2 * kSmallOp), *b_s = a_s + kSmallOp;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      fa[buf][ks] = small_frag<TA>(a_s, wm * 32, ks, lane);
      fb[buf][ks] = small_frag<TB>(b_s, wn * 32, ks, lane);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto multiply = [&](int buf) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[buf][ks], fb[buf][ks], acc, 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  // tile t + 1 has landed once at most the SS - 2 behind it are outstanding; past the barrier it is visible to every wave, and
  // every wave has read tile t, whose stage the next fetch takes
  auto land = [&]() {
    wait_vm<(SS - 2) * L>();
    __syncthreads();
    fetch();
  };
  wait_vm<(SS - 1) * L>();
  __syncthreads();
  read(0, 0);
#pragma unroll 1
  for (int t = 0; t < n; t += 2) {
    land();
    read(1, (t + 1) & 3);   // (past the last tile: what nobody multiplies)
    multiply(0);
    land();
    read(0, (t + 2) & 3);
    if (t + 1 < n) multiply(1);
  }
  wait_vm<0>();   // the last fetches, of nothing, have been written to LDS: none outlives the workgroup or meets its output stage
  if (split) {
    const int nn = n_tile + lane % 32;
    if (nn >= p.N) return;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = m_tile + 8 * (r / 4) + 4 * (lane / 32) + r % 4;
      if (m < p.M) atomicAdd(static_cast<float *>(p.C) + int64_t(m) * p.ldc + nn, acc[r]);
    }
    return;
  }
  // through LDS, as in the kernel above: 4 KiB per wave, rows of 32 columns
  __syncthreads();
  float *slab = reinterpret_cast<float *>(smem) + wave * 1024;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = 8 * (r / 4) + 4 * (lane / 32) + r % 4;
    slab[row * 32 + ((lane % 32) ^ ((row & 4) << 1))] = acc[r];
  }
  if (e.fast) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int row = 16 * q + lane / 4, c0 = 8 * (lane % 4);
      e.emit8(p, m_tile + row, n_lane, slab + row * 32 + (c0 ^ ((row & 4) << 1)), pre[q], bias8);
    }
  } else {
#pragma unroll 1
    for (int idx = lane; idx < 32 * 32; idx += 64) {
      const int row = idx / 32, col = idx % 32;
      const int m = m_tile + row, nn = n_tile + col;
      if (m < p.M && nn < p.N) e.emit_one(p, m, nn, slab[row * 32 + (col ^ ((row & 4) << 1))]);
    }
  }
}
template <bool TA, bool TB>
__global__ __launch_bounds__(NT) void k_gemm_dma64_even(DmaP p, int tiles_per_split, int grid_n, int splits) {
  __shared__ __attribute__((aligned(1024))) bf16_t smem[SS * 2 * kSmallOp];
  even_tile<TA, TB>(p, tiles_per_split, grid_n, splits, blockIdx.x, gridDim.x, smem);
}
// An input gradient (the first `wgs` workgroups) and a weight gradient (the others), which do not depend on each other.
struct EvenPart { DmaP p; int tiles_per_split, grid_n, splits, wgs; };
__global__ __launch_bounds__(NT) void k_gemm_dma64_pair(EvenPart input, EvenPart weight) {
  __shared__ __attribute__((aligned(1024))) bf16_t smem[SS * 2 * kSmallOp];
  const int l = blockIdx.x;
  if (l < input.wgs) even_tile<false, true>(input.p, input.tiles_per_split, input.grid_n, input.splits, l, input.wgs, smem);
  else even_tile<true, true>(weight.p, weight.tiles_per_split, weight.grid_n, weight.splits, l - input.wgs, weight.wgs, smem);
}

inline int check_launch(const char *what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(HMY_E_HIP, "launch of %s failed: %s", what, hipGetErrorString(e));
  return HMY_OK;
}

template <int BK, int S>
int launch_cfg(const hmy_gemm_desc &g, const DmaP &p, dim3 grid, int tiles_per_split, int gn, int splits, hipStream_t s) {
  const size_t lds = size_t(S) * 2 * BM * BK * sizeof(bf16_t);
  dim3 block(NT);
  if (!g.ta && !g.tb) hipLaunchKernelGGL((k_gemm_dma<false, false, BK, S>), grid, block, lds, s, p, tiles_per_split, gn, splits);
  else if (!g.ta && g.tb) hipLaunchKernelGGL((k_gemm_dma<false, true, BK, S>), grid, block, lds, s, p, tiles_per_split, gn, splits);
  else if (g.ta && !g.tb) hipLaunchKernelGGL((k_gemm_dma<true, false, BK, S>), grid, block, lds, s, p, tiles_per_split, gn, splits);
  else hipLaunchKernelGGL((k_gemm_dma<true, true, BK, S>), grid, block, lds, s, p, tiles_per_split, gn, splits);
  return check_launch("gemm_dma");
}

bool small_may_split(const hmy_gemm_desc &g) { return g.accumulate && g.c_fp32 && !g.bias && !g.res; }
// a long contraction over few tiles that may be split (fp32 atomics into C): while it fills idle compute units and
// leaves each workgroup at least eight K tiles
int small_splits(const hmy_gemm_desc &g) {
  const int64_t tiles = int64_t((g.M + ST - 1) / ST) * ((g.N + ST - 1) / ST);
  if (!small_may_split(g) || tiles > 128) return 1;
  return std::max(1, std::min(256 / int(tiles), (g.K + SK - 1) / SK / 8));
}

// Where the kernel without branches pays: its descriptors, the whole ring fetched whatever the length, and the output stage's
// operands in front of the loop have to be made up for, by more K tiles where two workgroups share a compute unit and hide each
// other's waits.  Kernel with branches -> without, us, up to 256 tiles: 1024x1024x64 4.1 -> 4.6, x192 4.9 -> 5.0, x256 5.2 ->
// 5.1, x512 6.9 -> 6.1; 257 to 512 tiles: 2048x1024x64 4.8 -> 5.9, x256 6.3 -> 6.5, x320 6.8 -> 7.1, x384 7.2 -> 7.1, x512 8.1
// -> 7.6; with a residual to add 1536x1024x384 (384 tiles) 8.5 -> 8.3, 2304x768x384 (432) 8.7 -> 8.9, x512 9.8 -> 9.6.
bool even_pays(const hmy_gemm_desc &g) {
  const int64_t tiles = int64_t((g.M + ST - 1) / ST) * ((g.N + ST - 1) / ST);
  return (g.K % SK == 0 || (g.ta && g.tb)) && g.K >= (tiles <= 256 ? 256 : g.res && tiles > 400 ? 512 : 384);
}

// how a product is laid out over 64x64 tiles
EvenPart small_part(const hmy_gemm_desc &g, const DmaP &p) {
  const int gm = (g.M + ST - 1) / ST, gn = (g.N + ST - 1) / ST, nk = (g.K + SK - 1) / SK;
  int splits = small_splits(g);
  const int tps = (nk + splits - 1) / splits;
  splits = (nk + tps - 1) / tps;
  return {p, tps, gn, splits, gm * gn * splits};
}

int launch_small(const hmy_gemm_desc &g, const DmaP &p, hipStream_t s) {
  const EvenPart part = small_part(g, p);
  const int tps = part.tiles_per_split, gn = part.grid_n, splits = part.splits;
  const dim3 grid(part.wgs), block(NT);
  if (even_pays(g)) {
    if (!g.ta && !g.tb) hipLaunchKernelGGL((k_gemm_dma64_even<false, false>), grid, block, 0, s, p, tps, gn, splits);
    else if (!g.ta && g.tb) hipLaunchKernelGGL((k_gemm_dma64_even<false, true>), grid, block, 0, s, p, tps, gn, splits);
    else if (g.ta && !g.tb) hipLaunchKernelGGL((k_gemm_dma64_even<true, false>), grid, block, 0, s, p, tps, gn, splits);
    else hipLaunchKernelGGL((k_gemm_dma64_even<true, true>), grid, block, 0, s, p, tps, gn, splits);
    return check_launch("gemm_dma64_even");
  }
  if (!g.ta && !g.tb) hipLaunchKernelGGL((k_gemm_dma64<false, false>), grid, block, 0, s, p, tps, gn, splits);
  else if (!g.ta && g.tb) hipLaunchKernelGGL((k_gemm_dma64<false, true>), grid, block, 0, s, p, tps, gn, splits);
  else if (g.ta && !g.tb) hipLaunchKernelGGL((k_gemm_dma64<true, false>), grid, block, 0, s, p, tps, gn, splits);
  else hipLaunchKernelGGL((k_gemm_dma64<true, true>), grid, block, 0, s, p, tps, gn, splits);
  return check_launch("gemm_dma64");
}

int env_int(const char *name, int dflt) {
  const char *v = std::getenv(name);
  return v ? std::atoi(v) : dflt;
}

}  // namespace

// Shapes this kernel takes: K a multiple of 32 (no K tail: the copy engine cannot
// mask), 16-byte aligned operands with leading dimensions that are multiples of 8
// elements, every operand spanning less than 4 GiB (32-bit byte offsets).
bool gemm_dma_eligible(const hmy_gemm_desc &g) {
  const int64_t a_span = int64_t(g.ta ? g.K : g.M) * g.lda, b_span = int64_t(g.tb ? g.K : g.N) * g.ldb;
  return g.K % 32 == 0 && a_span < (int64_t(1) << 31) && b_span < (int64_t(1) << 31);
}

bool gemm_small_excluded() {
  static const bool larger_forced = std::getenv("HMY_GEMM_BK") || std::getenv("HMY_GEMM_STAGES") || std::getenv("HMY_GEMM_TILE");
  return larger_forced;
}

// Weight gradients on 64x64 tiles: while the contraction of a workgroup (K over the splits) is not long.  A workgroup
// multiplies a K tile in 215 to 230 ns here, and the larger kernels, whose workgroups have four times the multiplies and whose
// splits are four times as many, start 10 us later and are a third faster from there on.  Measured over 80 outputs, 128x128
// tiles -> these, us:
// - up to 256 tiles the two meet between 4600 and 5600 (768x768x4096 21.7 -> 19.1, x4608 22.5 -> 21.1, x6144 26.2 -> 26.5;
//   512x512 in four parts of 4608 24.5 -> 22.5, of 5632 26.2 -> 25.9; 992x864x4096 21.1 -> 19.7, x5120 22.8 -> 23.5);
// - sooner where rows are no whole half cache lines: a row of a tile then lies in three of them instead of two, of the larger
//   tiles' in five instead of four (1000x1000x4096 26.6 -> 24.2, x5120 28.5 -> 28.8; 504x392 in four parts of 4096 24.0 ->
//   23.1), and at 3072 if the tiles leave many compute units idle (1000x520x3072 19.6 -> 18.5, x3584 19.1 -> 20.8);
// - the parts of a split contraction are dealt over the eight XCDs in turn.  Unless their number is a power of two an L2 cache
//   sees several of them: three up to 3072 (800x352 in three parts of 3072 19.8 -> 18.7, of 4096 21.5 -> 23.1), more not at all
//   (five parts of 2048: 416x416 17.3 -> 21.4, though 480x352 18.4 -> 14.7);
// - 257 to 512 tiles are two workgroups for some of the compute units: up to 2304 (1280x1024 21.2 -> 21.0, x2560 21.4 -> 23.0),
//   from 400 on 3072 (2304x768x2816 23.9 -> 23.4, x3072 24.7 -> 25.2; 2048x1024x3072 26.7 -> 25.7).  If edge tiles are half
//   empty, not at all (1056x992x2048 18.1 -> 20.1, 1320x800 18.8 -> 20.7; x1536 18.5 -> 16.8) and 2304 (1984x1000 26.1 -> 21.6
//   at 2048, 29.7 -> 28.8 at 3072; 1312x1312x2304 22.2 -> 22.2, x2560 23.1 -> 24.1).
// Short of a first split, at most 64 tiles of such misaligned rows are the other exception: 504x392x704 8.2 -> 7.7, x768 7.4 ->
// 7.8, x960 8.0 -> 9.0 (416x416x960 7.8 -> 7.9, 600x600x960 10.6 -> 9.2).  Contractions that are no multiple of 32 gain more,
// since the larger kernels take them in two launches (1024x1024x2008 23.3 -> 12.0, 2048x2048x3000 57 -> 45, 4096x1024x3000 54 ->
// 51), and have up to 2047 tiles.  Beyond 1024 of them the other side is tiles of 256 rows, and the two meet where tiles x K is 2.6
// million, from 1408 tiles on 2.2 (tiles of 256 rows and a tail -> these: 4672x1024x824, 1168 tiles, 32.7 -> 23.4, 1856x2304x1813
// 43.5 -> 36.5, 1120x3920x2216, 1116 tiles, 49.3 -> 49.6, 8960x512x3048 60.2 -> 64.6; 2560x2432x848, 1520 tiles, 34.9 -> 27.5,
// 5040x1344x1354, 1659 tiles, 44.5 -> 45.1, 4608x1536x3000, 1728 tiles, 67 -> 83, 6400x1280x2968 72 -> 95).
bool small_sum_pays(const hmy_gemm_desc &g) {
  const int64_t tiles = int64_t((g.M + ST - 1) / ST) * ((g.N + ST - 1) / ST);
  const int splits = small_splits(g), length = g.K / splits;
  const bool half_lines = g.lda % 32 == 0 && g.ldb % 32 == 0;
  if (tiles > 1024 && tiles * g.K > (tiles <= 1408 ? 2600000 : 2200000)) return false;
  if (length < 1792) return g.K % SK != 0 || half_lines || splits > 1 || tiles > 64 || g.K < 768;
  if (tiles > 256) {
    const bool whole = g.M % ST == 0 && g.N % ST == 0;
    return tiles <= 400 ? whole && length <= 2304 : length <= (whole ? 3072 : 2304);
  }
  if ((splits & (splits - 1)) != 0) return splits % 3 == 0 && 24 % splits == 0 && length <= 3072;   // 3, 6, 12: three per XCD
  return length <= (half_lines ? 4608 : splits == 1 && tiles < 200 ? 3072 : 4096);
}

// 64x64 tiles while all of them are resident at once, two per compute unit (us, 128x128 -> 64x64 tiles: 480x768x256 7.3 -> 5.0,
// 1024x1024x1024 12.6 -> 8.1, 2048x1024 (512 tiles), K = 1024 12.9 -> 10.2, 4096 31.7 -> 28.0; 3072x768x1536 (576 tiles) 16.6
// -> 20.4), and for four times as many where the contraction is no multiple of 32 and the larger kernels leave it to
// register-staged ones (768x3072x600 25 -> 15, 4096x1024x1001 38 -> 24, 2048x4096x1001 (2048 tiles) 41 -> 44).  Contractions
// that are no multiple of 64, weight gradients aside, go through the kernel with branches: up to 2048 of them beyond 256 tiles
// (2048x1024x2048 19.6 -> 18.9, 4096 32.5 -> 33.4).  Beyond 256 tiles an operand stored contraction-major loses on long ones what
// the tiles gain: from 8192 on (input gradients 2048x1024x8192 59.9 -> 58.9, x12288 86.7 -> 89.4), from 4096 on where its rows are
// no whole half cache lines (1960x1000x4096 36.8 -> 35.5, x8192 63.0 -> 68.1; forward, x16384 109 -> 102).  Sums into an fp32 C
// other than weight gradients (the vocabulary-long input gradient) keep the larger kernels' splits of the contraction, and so do
// long weight gradients (above).
bool gemm_prefers_small(const hmy_gemm_desc &g) {
  if (gemm_small_excluded()) return false;
  if (g.accumulate && !(g.ta && g.tb)) return false;
  const int64_t tiles = int64_t((g.M + ST - 1) / ST) * ((g.N + ST - 1) / ST);
  const bool even = g.K % SK == 0 || (g.ta && g.tb);
  if (small_may_split(g) && !small_sum_pays(g)) return false;
  if (g.K % 32 != 0) return tiles < 2048;
  const bool major = g.ta || g.tb, half_lines = (!g.ta || g.lda % 32 == 0) && (!g.tb || g.ldb % 32 == 0);
  return tiles <= 256 || (tiles <= 512 && g.K <= (!even ? 2048 : !major ? INT_MAX : half_lines ? 8192 : 4096));
}
GemmTiles gemm_small_tiles(const hmy_gemm_desc &g) { return {ST, ST, small_part(g, dma_params(g)).splits, 0, 0, 0}; }
int launch_gemm_small(const hmy_gemm_desc &g, stream_t st) { return launch_small(g, dma_params(g), (hipStream_t)st); }

// A linear layer's two gradients in one launch: each is one workgroup's chain over its K tiles long, however few workgroups there
// are, and they depend on nothing of each other.  Up to one workgroup per compute unit in all: iterations of an encoder of width
// 256 over 480 tokens (96 to 192 workgroups a pair) 5416 -> 5157 us; with 257 to 512 workgroups (width 512) there was nothing to
// gain, 12.01 ms either way.
bool launch_gemm_small_pair(const hmy_gemm_desc &input, const hmy_gemm_desc &weight, stream_t st, int *rc) {
  if (input.ta || !input.tb || !weight.ta || !weight.tb || !even_pays(input) || !even_pays(weight)) return false;
  const EvenPart i = small_part(input, dma_params(input)), w = small_part(weight, dma_params(weight));
  if (i.wgs + w.wgs > 256) return false;
  hipLaunchKernelGGL(k_gemm_dma64_pair, dim3(i.wgs + w.wgs), dim3(NT), 0, (hipStream_t)st, i, w);
  *rc = check_launch("gemm_dma64_pair");
  return true;
}

static int64_t tiles_of(const hmy_gemm_desc &g, int rows, int cols) {
  return int64_t((g.M + rows - 1) / rows) * ((g.N + cols - 1) / cols);
}
// Estimated time, in us, of a product on tiles of 256 x 32 nb outputs (gemm_tile.hip), or (nb = 0) on the 128x128 ones: rounds
// of 256 tiles, each of which costs its multiplies, its output stage (longer if it reads as much as it writes; several 128x128
// workgroups of a compute unit overlap theirs) and its start.  The last of several rounds costs a whole one, however few tiles
// it has (128x128 tiles, two to a unit, save a little): fewest outputs in flight for nothing is what the width is chosen for.  A
// first round that is not full saves up to half of its stores and start, but a workgroup's multiplies take nearly as long
// beside fewer others: half a round of 256x128 tiles is no match for a whole one of 128x128 (4096x1024x50257, the input
// gradient of a vocabulary, 128x128 | 256x128, us: 449 | 603; K = 16384 146 | 199).
// Fitted to 6800 random products of all layouts and output stages, K = 64 to 50240, on all six tiles, for the choice and not for
// the time itself, one that would be slower than on 128x128 tiles counting three times: the tile with the smallest estimate takes
// 0.3 % longer than the fastest on average from K = 480 on, 1.2 % below, where only 256x128 and 256x256 are asked for besides
// (with the other widths the mean there is 0.5 % lower, and three times as many take longer than on 128x128).  56 of the products
// take more than 2 % longer than on the tiles they had when the widths were 128 for one round and 256 for whole ones, the worst
// of them 13 %.
// Some, us, on 128x128 | 256x128, 160, 192, 224, 256: 2048x4800x1600 (forward) 49 | 41 33 33 36 37, 2048x12288x4096 250 | 165
// 201 156 167 173, 1944x3768x512 (fp32) 17.8 | 16.3 19.3 19.2 20.8 21.3, 3856x4416x704 (input gradient) 40 | 39 38 39 42 44,
// 5696x4072x832 (weight gradient) 72 | 75 91 80 84 84, 512x25504x192 (fp32 +=) 37 | 34 44 50 35 35.
static float tile_time(const hmy_gemm_desc &g, int nb) {
  static constexpr float per_1024_steps[] = {8.5f, 0.f, 0.f, 0.f, 11.1f, 14.7f, 16.8f, 18.6f, 19.6f};
  const int64_t tiles = nb ? tiles_of(g, 256, 32 * nb) : tiles_of(g, BM, BM), whole = tiles / 256;
  const float part = float(tiles % 256) / 256.f;
  // rounds' worth of time, if the last one's costs `least` at least
  auto rounds = [&](float least) { return float(whole) + (part == 0.f ? 0.f : least + (1.f - least) * part); };
  const float last = nb ? 0.99f : 0.85f;
  const bool both = g.c_fp32 || g.gelu_out;   // twice the bytes of a bf16 C
  const float kind = g.accumulate ? (g.ta && g.tb ? (nb ? 2.28f : 1.49f) : nb ? 2.35f : 2.05f)
                     : g.res && g.res_fp32 ? 2.6f : both ? (nb ? 1.58f : 1.96f) : 1.f;
  float out = 9.5f * kind * (nb ? float(nb) / 8.f : 0.264f);
  if (nb % 2 && !g.c_fp32) out += 0.1f;   // tiles whose rows end inside a cache line
  const float multiplies = per_1024_steps[nb] * float(g.K) / 1024.f, around = out + (nb ? 4.7f : 0.98f);
  return rounds(whole ? last : 0.65f) * multiplies + rounds(whole ? last : 0.5f) * around;
}
// Columns, over 32, of the tiles of 256 rows that a product takes, or 0 for 128x128 tiles.
static int tile_columns(const hmy_gemm_desc &g) {
  if (g.M < 256 || g.N < 128) return 0;
  int best = 0;
  for (int nb = 4; nb <= 8; nb += g.K < 480 ? 4 : 1)
    if (tile_time(g, nb) < tile_time(g, best)) best = nb;
  return best;
}

// 128x128 tiles: the contraction is split over workgroups (fp32 atomics into C) only while that fills idle compute units: with one
// workgroup per unit already, a deeper K loop beats more workgroups that each pay a prologue and an atomic epilogue.
GemmTiles gemm_128_tiles(const hmy_gemm_desc &g) {
  static const int force_bk = env_int("HMY_GEMM_BK", 0), force_s = env_int("HMY_GEMM_STAGES", 0);
  const int wgs = int(tiles_of(g, BM, BM));
  int splits = 1;
  if (small_may_split(g) && wgs <= 128) splits = std::max(1, std::min(256 / wgs, g.K / 256));
  // few workgroups: one per compute unit, deep K tiles and a deep ring; many: smaller
  // stages so that several are resident and overlap each other's prologue and epilogue
  int bk = g.K % 64 == 0 && wgs * splits <= 256 ? 64 : 32;
  if (force_bk == 32 || (force_bk == 64 && g.K % 64 == 0)) bk = force_bk;
  return {BM, BM, splits, bk, force_s == 3 ? 3 : 4, 0};
}

GemmTiles gemm_dma_tiles(const hmy_gemm_desc &g) {
  // 128 | 256: that block tile for every shape it can take; the other two switches are the 128x128 kernel's
  static const int force_tile = env_int("HMY_GEMM_BK", 0) || env_int("HMY_GEMM_STAGES", 0) ? 128 : env_int("HMY_GEMM_TILE", 0);
  const bool can_split = small_may_split(g);
  if (force_tile == 256 && g.M >= 256 && g.N >= 256) return {256, 256, 1, 0, 0, 0};
  if (force_tile == 0) {
    // Very long sums over few outputs: 256x128 tiles with the contraction split (fp32 atomics into C), where they come to nearly
    // a workgroup per compute unit and every part stays long enough to make up for twice the atomics.  Measured, us, 128x128
    // tiles -> these: 2048x1024, K = 50240 219 -> 184 (12560 in each part), 1024x1600 199 -> 164, 1024x1024 115 -> 105 (6280),
    // 512x1600 104 -> 92 (5582); 1024x1024x40960 98 -> 93 (5120), 512x1024x65536 77.7 -> 78.4 (4096), 1024x1024x16384 50 -> 55
    // (2048).  Not where 128x128 tiles fill the compute units: 4096x1024x50257 takes 465 in two parts (563 in one, 449 on 128x128
    // tiles), and an input gradient is rounded to bf16 next: from another order of its sum every gradient below moves by some 6e-3.
    const bool few = tiles_of(g, BM, BM) <= 128;
    if (can_split && few && g.M >= 256 && g.K % 64 == 0) {
      const int w2 = int(tiles_of(g, 256, 128)), splits = 256 / w2;
      if (splits > 1 && w2 * splits >= 200 && g.K / splits >= 4608) return {256, 128, splits, 0, 0, 0};
    }
    // sums over few outputs split the contraction over 128x128 tiles instead (below)
    const int nb = can_split && few ? 0 : tile_columns(g);
    if (nb) return {256, 32 * nb, 1, 0, 0, 0};
  }
  return gemm_128_tiles(g);
}

int launch_gemm_dma(const hmy_gemm_desc &g, const GemmTiles &t, stream_t st) {
  if (t.rows == 256) return launch_gemm_tile(g, t.cols / 32, t.splits, st);
  const DmaP p = dma_params(g);
  const int gm = (g.M + BM - 1) / BM, gn = (g.N + BM - 1) / BM, nk = g.K / t.bk;
  const int tps = (nk + t.splits - 1) / t.splits, splits = (nk + tps - 1) / tps;
  dim3 grid(gm * gn * splits);
  hipStream_t s = (hipStream_t)st;
  const auto launch = t.bk == 64 ? (t.stages == 3 ? launch_cfg<64, 3> : launch_cfg<64, 4>)
                                 : (t.stages == 3 ? launch_cfg<32, 3> : launch_cfg<32, 4>);
  return launch(g, p, grid, tps, gn, splits, s);
}

}  // namespace hmy

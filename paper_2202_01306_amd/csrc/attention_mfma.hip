// bf16 flash attention on the gfx950 matrix cores (v_mfma_f32_32x32x16_bf16).
//
// Every kernel keeps the scores transposed so that one lane owns one softmax row:
// for S^T = K Q^T the 32x32 accumulator gives lane l the query l%32 and sixteen of
// the 32 keys (the lane 32 further holds the other sixteen), so row maxima and sums
// are register reductions plus one cross-lane exchange, and the per-row rescaling
// of the output accumulator (also transposed: O^T = V^T P^T) is a per-lane scalar.
// Operands that must be read along the "wrong" axis of their LDS tile (V^T, K^T,
// dO^T, Q^T) come through ds_read_b64_tr_b16, which hands each lane four values
// from four different tile rows; the contraction order this induces (rows
// 4h+0..3 then 8+4h+0..3 of each group of 16, h = lane/32) is exactly the order in
// which the accumulator of the preceding MFMA holds them, so probabilities go from
// accumulator to operand without leaving registers.
//
// qkv is [T, 3d] with q | k | v thirds, head h at columns h*DH..; lse is [b,H,s].
// HMY_ATTN_SPLIT=0 (read once per process) takes the four-wave kernels wherever there is one (forward at head dimensions
// 64 and 128, dQ at 128, dK/dV at 64 and 128) instead of the eight-wave ones, for timing the two against each other.
#include <cstdlib>

#include "dev_common.h"
#include "hmy_internal.h"

namespace hmy {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kThreads = 256;       // 4 wavefronts, 32 rows of the block tile each
// At least two waves per SIMD, i.e. at most 256 registers per lane: the compiler then keeps the MFMA
// accumulators in ordinary vector registers.  Left free to use the accumulation registers it moved the
// score and output tiles back and forth with v_accvgpr_read / write around every softmax and rescaling
// (about 100 extra vector instructions per 32 x 32 subtile in kernels that are bound by exactly those).
// The four-wave dK/dV kernel at head dimension 128 needs more than 256 registers and keeps the default.
#define HMY_MFMA_IN_VGPRS __attribute__((amdgpu_waves_per_eu(2)))
constexpr int kBlockRows = 128;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

template <int DH> struct Cfg {
  static constexpr int TILE = DH == 128 ? 32 : 64;   // rows of the streamed tiles
  static constexpr int PITCH = DH + 8;               // padded LDS row (conflict-free 16-byte reads)
  static constexpr int KSTEPS = DH / 16;             // MFMA k-steps along the head dimension
  static constexpr int DTILES = DH / 32;             // 32-row output tiles along the head dimension
};

__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.f;
  return z;
}
__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Stage ROWS rows x DH columns (global row stride ld) into LDS [ROWS][PITCH]; rows at
// or beyond n_valid are zero.  Two phases, so that the loads of the next tile are in
// flight while the current one is multiplied: fetch into registers, put into LDS after
// the compute.
template <int DH, int ROWS, int NT = kThreads>
struct TileRegs {
  static constexpr int CPR = DH / 8;
  static constexpr int N = ROWS * CPR / NT;
  static_assert(N >= 1 && ROWS * CPR % NT == 0, "tile does not divide over the workgroup");
  Vec16<bf16_t> v[N];
  __device__ __forceinline__ void fetch(const bf16_t *src, int64_t ld, int n_valid, int tid) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int q = tid + i * NT, r = q / CPR, c = (q % CPR) * 8;
      if (r < n_valid) {
        v[i] = load16(src + int64_t(r) * ld + c);
      } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) v[i].v[k] = bf16_t(0.f);
      }
    }
  }
  __device__ __forceinline__ void put(bf16_t *lds, int tid) const {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int q = tid + i * NT, r = q / CPR, c = (q % CPR) * 8;
      store16(lds + r * Cfg<DH>::PITCH + c, v[i]);
    }
  }
};

// Operand fragment along a tile row: lane (row%32, kg) gets 8 consecutive columns.
template <int DH>
__device__ __forceinline__ bf16x8 frag_row(const bf16_t *lds, int row, int col) {
  return *reinterpret_cast<const bf16x8 *>(lds + row * Cfg<DH>::PITCH + col);
}
// Operand fragment across tile rows (the tile transposed): the lane's MFMA row is tile
// column colbase + lane%32; its 8 contraction slots are tile rows rowbase + 4h + 0..3
// and rowbase + 8 + 4h + 0..3 (h = lane/32).
template <int DH>
__device__ __forceinline__ bf16x8 frag_col(const bf16_t *lds, int rowbase, int colbase, int lane) {
  const int s = lane % 16, g16 = (lane / 16) % 2, h = lane / 32;
  const bf16_t *p = lds + (rowbase + 4 * h + s / 4) * Cfg<DH>::PITCH + colbase + 16 * g16 + 4 * (s % 4);
  typedef __attribute__((address_space(3))) short4v *lds_ptr;
  const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p));
  const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p + 8 * Cfg<DH>::PITCH));
  union { short4v s4[2]; bf16x8 b; } u;
  u.s4[0] = lo;
  u.s4[1] = hi;
  return u.b;
}
// Fragment straight from global memory: row-major matrix, lane (row, kg) gets columns col..col+7.
__device__ __forceinline__ bf16x8 frag_global(const bf16_t *base, int64_t ld, int row, int col) {
  return *reinterpret_cast<const bf16x8 *>(base + int64_t(row) * ld + col);
}
// Accumulator registers 8c..8c+7 as an operand fragment (rows 16c+4h+0..3, 16c+8+4h+0..3).
__device__ __forceinline__ bf16x8 acc_to_frag(const f32x16 &a, int c) {
  bf16x8 f;
#pragma unroll
  for (int k = 0; k < 8; ++k) f[k] = static_cast<__bf16>(a[8 * c + k]);
  return f;
}
// the larger of x and the value that the lane 32 further holds, without a trip through LDS
__device__ __forceinline__ float pair_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
// the wave's number within its workgroup, known to the compiler to be the same for all of its lanes: what a wave decides
// from it (which subtile, masked or not) becomes scalar arithmetic and branches instead of vector compares and saved masks
__device__ __forceinline__ int wave_number() { return __builtin_amdgcn_readfirstlane(threadIdx.x / 64); }
// what stands before is issued before what stands behind: the compiler otherwise sinks each read of an operand to the multiply
// that takes it, and every one of a chain's multiplies then waits for a read of its own
__device__ __forceinline__ void reads_first() { __builtin_amdgcn_sched_barrier(0); }
// tile row (0..31) held in accumulator register r by a lane of half h
__device__ __forceinline__ int acc_row(int r, int h) { return 8 * (r / 4) + 4 * h + r % 4; }

// dK/dV of a 32x32 subtile: lane owns a key, accumulator registers run over its 32 queries, sixteen per lane in four runs of
// four consecutive rows (16-byte reads of the rows' statistics): scores -> P (in place), dP -> dS (in place). `edge`, the same
// for the whole wave: queries past the sequence end or (causal) before the key may be among them; the test stands outside of
// the loop over registers, where the compiler made sixteen branches of it, each around one exponential.  The whole backward, us,
// causal: 16 heads of 64, s = 4096 202 -> 175, four sequences of 1024 71 -> 63; 32 heads of s = 2048: of 32 108 -> 76, of 128 197 -> 169.
__device__ __forceinline__ void probabilities(f32x16 &sm, f32x16 &dp, const float *lse, const float *delta, int h2, float sc,
                                              bool edge, int ib, int s, int key, int causal) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    float L[4];
    *reinterpret_cast<float4 *>(L) = *reinterpret_cast<const float4 *>(lse + 8 * g + 4 * h2);
#pragma unroll
    for (int k = 0; k < 4; ++k) sm[4 * g + k] = fmaf(sm[4 * g + k], sc, -L[k]);
  }
  if (edge) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int qi = ib + acc_row(r, h2);
      sm[r] = qi < s && (!causal || key <= qi) ? sm[r] : -INFINITY;
    }
  }
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    float D[4];
    *reinterpret_cast<float4 *>(D) = *reinterpret_cast<const float4 *>(delta + 8 * g + 4 * h2);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int r = 4 * g + k;
      sm[r] = fast_exp2(sm[r]);         // P
      dp[r] = sm[r] * (dp[r] - D[k]);   // dS
    }
  }
}

// scores of a 32-key subtile from key kb on, lane owns query q of the wave's 32 from qw on: keys past the sequence end or
// (causal) past the query get no weight.  Only a diagonal and the last subtile hold any.
__device__ __forceinline__ void mask_keys(f32x16 &st, int kb, int qw, int q, int s, int h2, int causal) {
  if (kb + 32 > s || (causal && kb + 31 > qw)) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = kb + acc_row(r, h2);
      if (!(key < s && (!causal || key <= q))) st[r] = -INFINITY;
    }
  }
}

// db[c] += sum over the workgroup's 128 rows of the values stored from the accumulators (scaled and rounded to bf16
// as they are stored; rows that are not stored count as zero): the bias gradient of the QKV projection, taken while
// the gradient of its output is still in registers.  acc[t][r] of lane l in wave w belongs to row 32 w + l % 32,
// column 32 t + 8 (r / 4) + 4 (l / 32) + r % 4.  The values pass through LDS, 64 columns at a time (rows padded to
// an odd number of floats so that the lanes of a wave, which hold different rows, fall on different banks); every
// thread then adds up a share of one column, and one atomic per thread leaves the workgroup -- a few wide atomic
// instructions instead of one narrow one per value and wave.  At head dimension 32 that would be eight atomics on every
// address from each workgroup, and a launch of many workgroups waits for them: there the shares meet in LDS first, and one
// atomic per column leaves.  us, the whole backward, with eight -> with one (without the bias gradient): 32 heads of 32, 32
// sequences of 128 70 -> 42 (38), sixteen of 256 81 -> 52 (48), eight of 1024, causal, 206 -> 150 (142); 4 heads, four of 64
// 13.1 -> 10.1 (8.1).  Wider heads, four shares, gain nothing (16 heads of 64, sixteen of 512 105.4 -> 105.5) and pay for the
// barriers (4 heads of 128, s = 128 31.5 -> 32.1).  Every thread of the workgroup must call this.
constexpr int kBiasCols = 64, kBiasPitch = kBiasCols + 1;
template <int NT>
__device__ __forceinline__ void bias_grad_sums(float *db, const f32x16 (&acc)[NT], float scale, bool row_stored, float *lds,
                                               int tid, bool adds = true) {
  const int lane = tid % 64, h = lane / 32, row = 32 * (tid / 64) + lane % 32;
  constexpr int G = NT < 2 ? NT : 2, W = 32 * G;   // accumulator tiles and columns per pass
#pragma unroll
  for (int g = 0; g < NT; g += G) {
#pragma unroll
    for (int t = 0; t < G; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        lds[row * kBiasPitch + 32 * t + 8 * (r / 4) + 4 * h + r % 4] =
            row_stored ? static_cast<float>(static_cast<__bf16>(acc[g + t][r] * scale)) : 0.f;
    __syncthreads();
    const int col = tid % W, part = tid / W;
    constexpr int kParts = kThreads / W;
    float sum = 0.f;
    for (int rr = part; rr < kBlockRows; rr += kParts) sum += lds[rr * kBiasPitch + col];
    if constexpr (kParts > 4) {   // (see above)
      __syncthreads();
      lds[part * kBiasPitch + col] = sum;
      __syncthreads();
      adds = adds && part == 0;
      if (adds) {
#pragma unroll
        for (int k = 1; k < kParts; ++k) sum += lds[k * kBiasPitch + col];
      }
    }
    if (adds) atomicAdd(db + 32 * g + col, sum);
    __syncthreads();
  }
}

// Which 128-row block, head and sequence a workgroup takes (1-D grid of nrb * H * b workgroups).
// With a causal mask the work of a row block grows with the number of keys (queries) it sees, from 1
// to nrb units.  Workgroups are handed out in linear order, round-robin over the 8 XCDs, and a launch
// of the usual size is resident all at once (about two workgroups per compute unit), so the order IS
// the placement: a grid with the row block in its fastest dimension puts every heaviest block on one
// XCD and pairs equal weights on a compute unit (16 units on some, 2 on others, where 9 would do).
// Here the (row block, head, sequence) triples are ranked by weight, heaviest first, and dealt out in
// rounds of one workgroup per compute unit, every other round backwards: a unit that got a heavy block
// in one round gets a light one in the next, and each XCD sees every weight equally often.  A kernel of which
// only one workgroup fits a compute unit (`snake` false) keeps the ranking as it is: the unit that finishes
// first, having had the lightest block of the round, takes the heaviest that is left.
struct BlockCoord { int rb, head, seq; };
__device__ __forceinline__ BlockCoord block_coord(int nrb, int H, int causal, bool heaviest_is_last_row_block, bool snake, int n, int l) {
  const int bh_count = n / nrb;
  int r = l;
  if (causal && snake) {
    constexpr int kUnits = 256;
    const int round = l / kUnits, first = round * kUnits, len = min(kUnits, n - first);
    if (round & 1) r = first + (len - 1 - (l - first));
  }
  const int rank = r / bh_count, bh = r % bh_count;
  BlockCoord c;
  c.rb = !causal ? rank : (heaviest_is_last_row_block ? nrb - 1 - rank : rank);
  c.head = bh % H;
  c.seq = bh / H;
  return c;
}
__device__ __forceinline__ BlockCoord block_coord(int nrb, int H, int causal, bool heaviest_is_last_row_block, bool snake = true) {
  return block_coord(nrb, H, causal, heaviest_is_last_row_block, snake, gridDim.x, blockIdx.x);
}

// delta of one row, sum_c dO[c] O[c]: lane (row, h2) takes half of the columns and keeps its dO as multiply operands
template <int DH>
__device__ __forceinline__ float row_delta(const bf16_t *g, const bf16_t *o, int d, int row, int h2, bf16x8 (&fg)[DH / 16]) {
  float dl = 0.f;
#pragma unroll
  for (int c = 0; c < DH / 16; ++c) {
    fg[c] = frag_global(g, d, row, 16 * c + 8 * h2);
    const bf16x8 fo = frag_global(o, d, row, 16 * c + 8 * h2);
#pragma unroll
    for (int k = 0; k < 8; ++k) dl = fmaf(static_cast<float>(fg[c][k]), static_cast<float>(fo[k]), dl);
  }
  return dl + __shfl_xor(dl, 32, 64);   // the other half of the row
}

// ---------------------------------------------------------------------------------
// Forward.  grid (ceil(s/128) * H * b).  Wave w owns queries q0 + 32w .. +31.
template <int DH>
__global__ __launch_bounds__(kThreads) HMY_MFMA_IN_VGPRS void k_attn_fwd_mfma(const bf16_t *qkv, bf16_t *o, float *lse, int s, int H,
                                                            int causal) {
  typedef Cfg<DH> C;
  __shared__ __attribute__((aligned(16))) bf16_t sK[2][C::TILE * C::PITCH];
  __shared__ __attribute__((aligned(16))) bf16_t sV[2][C::TILE * C::PITCH];
  const int tid = threadIdx.x, lane = tid % 64, wave = wave_number(), h2 = lane / 32;
  const int d = H * DH;
  const int64_t ld = 3 * int64_t(d);
  const BlockCoord bc = block_coord((s + kBlockRows - 1) / kBlockRows, H, causal, true);   // the last query blocks see the most keys
  const int head = bc.head, seq = bc.seq, q0 = bc.rb * kBlockRows;
  const bf16_t *base = qkv + int64_t(seq) * s * ld + head * DH;
  const int qw = q0 + 32 * wave;                 // first query of this wave
  const int q = qw + lane % 32;                  // this lane's query
  const int q_ld = min(q, s - 1);
  bf16x8 fq[C::KSTEPS];
#pragma unroll
  for (int c = 0; c < C::KSTEPS; ++c) fq[c] = frag_global(base, ld, q_ld, 16 * c + 8 * h2);
  f32x16 acc_o[C::DTILES];
#pragma unroll
  for (int t = 0; t < C::DTILES; ++t) acc_o[t] = zero16();
  // Row sums come out of the matrix cores as well: a row of ones in the role of V^T makes every
  // register of acc_l the sum over keys of this lane's query's probabilities (both half-waves' keys),
  // which takes sixteen additions per 32 keys off the vector ALU, the unit this kernel is bound by.
  f32x16 acc_l = zero16();
  bf16x8 ones;
#pragma unroll
  for (int k = 0; k < 8; ++k) ones[k] = static_cast<__bf16>(1.f);
  // m_run is the REFERENCE the exponentials are taken against, not the exact running maximum: it is
  // raised (and everything accumulated rescaled) only when some row's scores outgrow it by more than
  // kSlack, so probabilities stay below 2^kSlack and most tiles skip the rescaling altogether
  constexpr float kSlack = 8.f;
  float m_run = -INFINITY;
  const float sc = rsqrtf(float(DH)) * kLog2e;   // scores in log2 units
  const int k_end = causal ? min(s, q0 + kBlockRows) : s;
  const int n_tiles = (k_end + C::TILE - 1) / C::TILE;
  TileRegs<DH, C::TILE> rk, rv;
  rk.fetch(base + d, ld, min(C::TILE, s), tid);
  rv.fetch(base + 2 * d, ld, min(C::TILE, s), tid);
  rk.put(sK[0], tid);
  rv.put(sV[0], tid);
  __syncthreads();
  for (int kt = 0; kt < n_tiles; ++kt) {
    const int cur = kt & 1, k0 = kt * C::TILE;
    const bool more = kt + 1 < n_tiles;
    if (more) {   // next tile's loads fly during this tile's multiplies
      const int kn = k0 + C::TILE;
      rk.fetch(base + d + int64_t(kn) * ld, ld, min(C::TILE, s - kn), tid);
      rv.fetch(base + 2 * d + int64_t(kn) * ld, ld, min(C::TILE, s - kn), tid);
    }
    const bool wave_active = !causal || k0 <= qw + 31;   // some query of this wave sees this tile
    if (wave_active) {
      // The 32-key subtiles of the tile go through each stage together: their score products are independent chains
      // of multiplies that overlap, the row maximum and the decision to rescale are taken once over all of them, and
      // the exponentials of one overlap the multiplies of another.  A subtile that lies wholly past this wave's
      // queries (second half of a diagonal tile) is carried along fully masked: its probabilities are exact zeros.
      constexpr int NS = C::TILE / 32;
      f32x16 st[NS];
#pragma unroll
      for (int sub = 0; sub < NS; ++sub) st[sub] = zero16();
      // S^T[key, query] = K Q^T
#pragma unroll
      for (int c = 0; c < C::KSTEPS; ++c)
#pragma unroll
        for (int sub = 0; sub < NS; ++sub)
          st[sub] = mfma(frag_row<DH>(sK[cur], 32 * sub + lane % 32, 16 * c + 8 * h2), fq[c], st[sub]);
#pragma unroll
      for (int sub = 0; sub < NS; ++sub) {
        const int kb = k0 + 32 * sub;                     // first key of the 32-key subtile
        // keys past the sequence end or (causal) past the query: only the diagonal and
        // the last subtile need the per-element test
        if (kb + 32 > s || (causal && kb + 31 > qw)) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int key = kb + acc_row(r, h2);
            if (!(key < s && (!causal || key <= q))) st[sub][r] = -INFINITY;
          }
        }
      }
      float mx = st[0][0];
#pragma unroll
      for (int sub = 0; sub < NS; ++sub)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, st[sub][r]);
      mx = pair_max(mx) * sc;     // log2 units (sc > 0)
      if (__any(mx > m_run + kSlack)) {   // some row outgrew its reference: raise it, rescale what was accumulated
        const float m_new = fmaxf(m_run, mx);
        const float corr = m_new == -INFINITY ? 1.f : fast_exp2(m_run - m_new);
        acc_l[0] *= corr;
#pragma unroll
        for (int t = 0; t < C::DTILES; ++t)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc_o[t][r] *= corr;
        m_run = m_new;
      }
      // rows that have seen no key yet keep m = -inf; use 0 as the reference to stay finite
      const float m_ref = m_run == -INFINITY ? 0.f : m_run;
#pragma unroll
      for (int sub = 0; sub < NS; ++sub) {
#pragma unroll
        for (int r = 0; r < 16; ++r) st[sub][r] = fast_exp2(fmaf(st[sub][r], sc, -m_ref));
        // O^T[dh, query] += V^T P^T, and the row sums
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const bf16x8 fp = acc_to_frag(st[sub], c);
#pragma unroll
          for (int t = 0; t < C::DTILES; ++t)
            acc_o[t] = mfma(frag_col<DH>(sV[cur], 32 * sub + 16 * c, 32 * t, lane), fp, acc_o[t]);
          acc_l = mfma(ones, fp, acc_l);
        }
      }
    }
    if (more) {
      rk.put(sK[cur ^ 1], tid);
      rv.put(sV[cur ^ 1], tid);
    }
    __syncthreads();
  }
  const float l_tot = acc_l[0];
  if (q < s) {
    const float inv = 1.f / l_tot;
    bf16_t *orow = o + (int64_t(seq) * s + q) * d + head * DH;
#pragma unroll
    for (int t = 0; t < C::DTILES; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        bf16x4 v;
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = static_cast<__bf16>(acc_o[t][4 * j + k] * inv);
        *reinterpret_cast<bf16x4 *>(orow + 32 * t + 8 * j + 4 * h2) = v;
      }
    if (h2 == 0) lse[(int64_t(seq) * H + head) * s + q] = (m_run + log2f(l_tot)) * kLn2;
  }
}

// ---------------------------------------------------------------------------------
// Forward for head dimensions 64 and 128: eight waves per workgroup, key tiles of two 32-key subtiles.  Wave w takes
// the queries q0 + 32 (w % 4) .. + 31 and, of every key tile, only subtile w / 4: two waves share each group of
// queries and split its keys, each with a running reference, row sum and output accumulator of its own, which the
// pair merges through LDS at the end.  The same work in twice as many, half as long chains: the kernel is bound by
// each wave's serial chain (multiplies, maximum, exponentials, multiplies), and with four waves per SIMD instead of
// two the vector unit of one wave works while the matrix unit of another does.  So what counts is the length of the chain:
// a subtile's operands are read from LDS together, ahead of where they are wanted, the halves of a row's maximum meet by a swap
// of lanes instead of through LDS, and branches are scalar.  us, before -> after: 16 heads of 64, s = 4096, causal 64.8 -> 56.8
// (the swap alone 61.5, with scalar branches 59.6); four sequences of 1024 20.7 -> 18.7, eight of 512, not causal, 17.8 -> 16.7;
// 32 heads of 128, s = 2048, 92.3 -> 88.6.  Four tiles in flight and a barrier for every second one instead of two and one:
// 57.2 -> 63.1, not causal 48.4 -> 48.7.
template <int DH>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(DH == 128 ? 2 : 4))) void k_attn_fwd_mfma_split(const bf16_t *qkv, bf16_t *o, float *lse, int s, int H,
                                                                                                    int causal) {
  typedef Cfg<DH> C;
  constexpr int NTHR = 512, TILE = 64;
  constexpr int kTileElems = TILE * C::PITCH;
  // K and V tiles, double buffered; afterwards the same bytes carry one wave's state to its partner
  __shared__ __attribute__((aligned(16))) bf16_t smem[4 * kTileElems];
  static_assert(4 * kTileElems * 2 >= 4 * 64 * (2 + 16 * C::DTILES) * 4, "the merge needs 2 + 16 DTILES floats per lane of four waves");
  auto sK = [&](int buf) { return smem + buf * kTileElems; };
  auto sV = [&](int buf) { return smem + (2 + buf) * kTileElems; };
  const int tid = threadIdx.x, lane = tid % 64, wave = wave_number(), h2 = lane / 32;
  const int rg = wave % 4, sub = wave / 4;
  const int d = H * DH;
  const int64_t ld = 3 * int64_t(d);
  const BlockCoord bc = block_coord((s + kBlockRows - 1) / kBlockRows, H, causal, true, DH != 128);
  const int head = bc.head, seq = bc.seq, q0 = bc.rb * kBlockRows;
  const bf16_t *base = qkv + int64_t(seq) * s * ld + head * DH;
  const int qw = q0 + 32 * rg, q = qw + lane % 32, q_ld = min(q, s - 1);
  bf16x8 fq[C::KSTEPS];
#pragma unroll
  for (int c = 0; c < C::KSTEPS; ++c) fq[c] = frag_global(base, ld, q_ld, 16 * c + 8 * h2);
  f32x16 acc_o[C::DTILES];
#pragma unroll
  for (int t = 0; t < C::DTILES; ++t) acc_o[t] = zero16();
  f32x16 acc_l = zero16();   // row sums from the matrix cores, as in the kernel above
  bf16x8 ones;
#pragma unroll
  for (int k = 0; k < 8; ++k) ones[k] = static_cast<__bf16>(1.f);
  constexpr float kSlack = 8.f;   // the exponent reference is raised only when a row outgrows it by this much
  float m_run = -INFINITY;
  const float sc = rsqrtf(float(DH)) * kLog2e;   // scores in log2 units
  const int k_end = causal ? min(s, q0 + kBlockRows) : s;
  const int n_tiles = (k_end + TILE - 1) / TILE;
  TileRegs<DH, TILE, NTHR> rk, rv;
  rk.fetch(base + d, ld, min(TILE, s), tid);
  rv.fetch(base + 2 * d, ld, min(TILE, s), tid);
  rk.put(sK(0), tid);
  rv.put(sV(0), tid);
  __syncthreads();
  for (int kt = 0; kt < n_tiles; ++kt) {
    const int cur = kt & 1, k0 = kt * TILE;
    const bool more = kt + 1 < n_tiles;
    if (more) {   // next tile's loads fly during this tile's multiplies
      const int kn = k0 + TILE;
      rk.fetch(base + d + int64_t(kn) * ld, ld, min(TILE, s - kn), tid);
      rv.fetch(base + 2 * d + int64_t(kn) * ld, ld, min(TILE, s - kn), tid);
    }
    const int kb = k0 + 32 * sub;   // first key of this wave's subtile
    if (kb < s && (!causal || kb <= qw + 31)) {   // some query of this wave sees some key of it
      // S^T[key, query] = K Q^T
      f32x16 st = zero16();
      bf16x8 fk[C::KSTEPS];
#pragma unroll
      for (int c = 0; c < C::KSTEPS; ++c) fk[c] = frag_row<DH>(sK(cur), 32 * sub + lane % 32, 16 * c + 8 * h2);
      reads_first();
#pragma unroll
      for (int c = 0; c < C::KSTEPS; ++c) st = mfma(fk[c], fq[c], st);
      if (kb + 32 > s || (causal && kb + 31 > qw)) {   // ragged or diagonal subtile: per-element test
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = kb + acc_row(r, h2);
          if (!(key < s && (!causal || key <= q))) st[r] = -INFINITY;
        }
      }
      bf16x8 fv[2][C::DTILES];   // V^T, wanted behind the exponentials
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int t = 0; t < C::DTILES; ++t) fv[c][t] = frag_col<DH>(sV(cur), 32 * sub + 16 * c, 32 * t, lane);
      reads_first();
      float mx = st[0];
#pragma unroll
      for (int r = 1; r < 16; ++r) mx = fmaxf(mx, st[r]);
      mx = pair_max(mx) * sc;     // log2 units (sc > 0)
      if (__any(mx > m_run + kSlack)) {   // some row outgrew its reference: raise it, rescale what was accumulated
        const float m_new = fmaxf(m_run, mx);
        const float corr = m_new == -INFINITY ? 1.f : fast_exp2(m_run - m_new);
        acc_l[0] *= corr;
#pragma unroll
        for (int t = 0; t < C::DTILES; ++t)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc_o[t][r] *= corr;
        m_run = m_new;
      }
      const float m_ref = m_run == -INFINITY ? 0.f : m_run;   // a row that has seen no key yet
#pragma unroll
      for (int r = 0; r < 16; ++r) st[r] = fast_exp2(fmaf(st[r], sc, -m_ref));
      // O^T[dh, query] += V^T P^T, and the row sums
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const bf16x8 fp = acc_to_frag(st, c);
#pragma unroll
        for (int t = 0; t < C::DTILES; ++t)
          acc_o[t] = mfma(fv[c][t], fp, acc_o[t]);
        acc_l = mfma(ones, fp, acc_l);
      }
    }
    if (more) {
      rk.put(sK(cur ^ 1), tid);
      rv.put(sV(cur ^ 1), tid);
    }
    __syncthreads();
  }
  // merge the two key subsets of each query: the wave of the second subtile hands over its reference, row sum and
  // accumulator ([value][lane] floats: conflict-free both ways); the first rescales both to the larger reference
  constexpr int NV = 2 + 16 * C::DTILES;
  float *xch = reinterpret_cast<float *>(smem) + rg * (NV * 64);
  if (sub == 1) {
    xch[lane] = m_run;
    xch[64 + lane] = acc_l[0];
#pragma unroll
    for (int t = 0; t < C::DTILES; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) xch[(2 + 16 * t + r) * 64 + lane] = acc_o[t][r];
  }
  __syncthreads();
  if (sub == 1) return;
  const float m_b = xch[lane], l_b = xch[64 + lane];
  const float m_tot = fmaxf(m_run, m_b);   // finite: the first subtile of the first tile holds key 0, which every query sees
  const float ca = fast_exp2(m_run - m_tot), cb = m_b == -INFINITY ? 0.f : fast_exp2(m_b - m_tot);
  const float l_tot = acc_l[0] * ca + l_b * cb;
  if (q < s) {
    const float inv = 1.f / l_tot;
    bf16_t *orow = o + (int64_t(seq) * s + q) * d + head * DH;
#pragma unroll
    for (int t = 0; t < C::DTILES; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        bf16x4 v;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int r = 4 * j + k;
          v[k] = static_cast<__bf16>((acc_o[t][r] * ca + xch[(2 + 16 * t + r) * 64 + lane] * cb) * inv);
        }
        *reinterpret_cast<bf16x4 *>(orow + 32 * t + 8 * j + 4 * h2) = v;
      }
    if (h2 == 0) lse[(int64_t(seq) * H + head) * s + q] = (m_tot + log2f(l_tot)) * kLn2;
  }
}

// ---------------------------------------------------------------------------------
// dQ.  grid (ceil(s/128), H, b).  Wave w owns queries q0+32w..; K and V tiles stream.
// Also delta[seq,head,q] = sum_c dO[q,c] * O[q,c], which this kernel needs per query and the dK/dV kernel, launched
// behind it, reads per streamed query row: each lane holds half of its query's dO row as multiply operands already, so
// the sum is 4 DH / 16 multiply-adds and one exchange with the lane that holds the other half, and no kernel of its own.
// The bias gradient's sums take the tiles' LDS, which are done with by then: 37 KB instead of 70 let three workgroups share a
// compute unit where two did; and a subtile's operands are read together, as in the forward.  The whole backward, us, before ->
// with the LDS -> with both: 16 heads of 64, causal, s = 4096 171.9 -> 164.1 -> 161.2, sixteen sequences of 1024 195.0 -> 185.8
// -> 183.9.  (Both subtiles of a tile side by side, for chains half as long, need 196 registers: 171 -> 179.)
//
// NT threads: waves 4 and up only help to fetch the tiles (`smem` then holds twice the room for the bias gradient).
template <int DH> struct DqLds {
  static constexpr int TILE = Cfg<DH>::TILE * Cfg<DH>::PITCH, BIAS = 2 * kBlockRows * kBiasPitch;   // in elements
  static constexpr int ELEMS = 4 * TILE > BIAS ? 4 * TILE : BIAS;
};
template <int DH, int NT>
__device__ __forceinline__ void dq_rows(const bf16_t *qkv, const bf16_t *o, const bf16_t *d_o, const float *lse, float *delta,
                                        bf16_t *dqkv, float *dbias, int s, int H, int causal, bf16_t *smem, int n_wg, int wg) {
  typedef Cfg<DH> C;
  constexpr int kTile = DqLds<DH>::TILE;
  // K and V tiles, double buffered; afterwards the bias gradient's way through LDS
  bf16_t (*sK)[kTile] = reinterpret_cast<bf16_t (*)[kTile]>(smem), (*sV)[kTile] = sK + 2;
  float *sB = reinterpret_cast<float *>(smem);
  const int tid = threadIdx.x, lane = tid % 64, wave = wave_number(), h2 = lane / 32;
  const int d = H * DH;
  const int64_t ld = 3 * int64_t(d);
  const BlockCoord bc = block_coord((s + kBlockRows - 1) / kBlockRows, H, causal, true, NT == kThreads, n_wg, wg);
  const int head = bc.head, seq = bc.seq, q0 = bc.rb * kBlockRows;
  const bf16_t *base = qkv + int64_t(seq) * s * ld + head * DH;
  const bf16_t *gbase = d_o + int64_t(seq) * s * d + head * DH;
  const bf16_t *obase = o + int64_t(seq) * s * d + head * DH;
  const bool works = NT == kThreads || wave < kThreads / 64;
  const int qw = q0 + 32 * (wave % 4), q = qw + lane % 32, q_ld = min(q, s - 1);
  bf16x8 fq[C::KSTEPS], fg[C::KSTEPS];
#pragma unroll
  for (int c = 0; c < C::KSTEPS; ++c) fq[c] = frag_global(base, ld, q_ld, 16 * c + 8 * h2);
  const float dl = row_delta<DH>(gbase, obase, d, q_ld, h2, fg);
  if (works && h2 == 0 && q < s) delta[(int64_t(seq) * H + head) * s + q] = dl;
  const float L = lse[(int64_t(seq) * H + head) * s + q_ld] * kLog2e;   // log2 units
  const float scale = rsqrtf(float(DH)), sc = scale * kLog2e;
  f32x16 acc_q[C::DTILES];
#pragma unroll
  for (int t = 0; t < C::DTILES; ++t) acc_q[t] = zero16();
  const int k_end = causal ? min(s, q0 + kBlockRows) : s;
  const int n_tiles = (k_end + C::TILE - 1) / C::TILE;
  TileRegs<DH, C::TILE, NT> rk, rv;
  rk.fetch(base + d, ld, min(C::TILE, s), tid);
  rv.fetch(base + 2 * d, ld, min(C::TILE, s), tid);
  rk.put(sK[0], tid);
  rv.put(sV[0], tid);
  __syncthreads();
  for (int kt = 0; kt < n_tiles; ++kt) {
    const int cur = kt & 1, k0 = kt * C::TILE;
    const bool more = kt + 1 < n_tiles;
    if (more) {   // next tile's loads fly during this tile's multiplies
      const int kn = k0 + C::TILE;
      rk.fetch(base + d + int64_t(kn) * ld, ld, min(C::TILE, s - kn), tid);
      rv.fetch(base + 2 * d + int64_t(kn) * ld, ld, min(C::TILE, s - kn), tid);
    }
    if (works && (!causal || k0 <= qw + 31)) {
#pragma unroll
      for (int sub = 0; sub < C::TILE / 32; ++sub) {
        const int kb = k0 + 32 * sub;
        if (causal && kb > qw + 31) continue;
        f32x16 st = zero16(), dp = zero16();
        // at head dimension 128 the fragments of a whole subtile do not fit the registers (20 of them spilled: 274 -> 282 us)
        constexpr bool kAhead = DH <= 64;
        bf16x8 fk[C::KSTEPS], fv[C::KSTEPS];
#pragma unroll
        for (int c = 0; c < C::KSTEPS; ++c) {
          fk[c] = frag_row<DH>(sK[cur], 32 * sub + lane % 32, 16 * c + 8 * h2);
          fv[c] = frag_row<DH>(sV[cur], 32 * sub + lane % 32, 16 * c + 8 * h2);
        }
        if constexpr (kAhead) reads_first();
#pragma unroll
        for (int c = 0; c < C::KSTEPS; ++c) {
          st = mfma(fk[c], fq[c], st);   // S^T = K Q^T
          dp = mfma(fv[c], fg[c], dp);   // dP^T = V dO^T
        }
        bf16x8 ft[2][C::DTILES];   // K^T, wanted behind the exponentials
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int t = 0; t < C::DTILES; ++t) ft[c][t] = frag_col<DH>(sK[cur], 32 * sub + 16 * c, 32 * t, lane);
        if constexpr (kAhead) reads_first();
        mask_keys(st, kb, qw, q, s, h2, causal);
#pragma unroll
        for (int r = 0; r < 16; ++r) st[r] = fast_exp2(fmaf(st[r], sc, -L)) * (dp[r] - dl);     // dS^T
        // dQ^T[dh, query] += K^T dS^T
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const bf16x8 fs = acc_to_frag(st, c);
#pragma unroll
          for (int t = 0; t < C::DTILES; ++t)
            acc_q[t] = mfma(ft[c][t], fs, acc_q[t]);
        }
      }
    }
    if (more) {
      rk.put(sK[cur ^ 1], tid);
      rv.put(sV[cur ^ 1], tid);
    }
    __syncthreads();
  }
  if (works && q < s) {
    bf16_t *row = dqkv + (int64_t(seq) * s + q) * ld + head * DH;
#pragma unroll
    for (int t = 0; t < C::DTILES; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        bf16x4 v;
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = static_cast<__bf16>(acc_q[t][4 * j + k] * scale);
        *reinterpret_cast<bf16x4 *>(row + 32 * t + 8 * j + 4 * h2) = v;
      }
  }
  if (dbias)
    bias_grad_sums<C::DTILES>(dbias + head * DH, acc_q, scale, q < s, sB + (works ? 0 : kBlockRows * kBiasPitch),
                              tid % kThreads, works);
}
template <int DH>
__global__ __launch_bounds__(kThreads) HMY_MFMA_IN_VGPRS void k_attn_bwd_dq_mfma(const bf16_t *qkv, const bf16_t *o, const bf16_t *d_o,
                                                               const float *lse, float *delta, bf16_t *dqkv, float *dbias,
                                                               int s, int H, int causal) {
  __shared__ __attribute__((aligned(16))) bf16_t smem[DqLds<DH>::ELEMS];
  dq_rows<DH, kThreads>(qkv, o, d_o, lse, delta, dqkv, dbias, s, H, causal, smem, gridDim.x, blockIdx.x);
}

// ---------------------------------------------------------------------------------
// dK, dV.  grid (ceil(s/128), H, b).  Wave w owns keys j0+32w..; Q and dO tiles stream.
template <int DH>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(DH == 128 ? 1 : 2))) void k_attn_bwd_dkv_mfma(const bf16_t *qkv, const bf16_t *d_o, const float *lse,
                                                                const float *delta, bf16_t *dqkv, float *dbias, int s,
                                                                int H, int causal) {
  typedef Cfg<DH> C;
  __shared__ __attribute__((aligned(16))) bf16_t sQ[2][C::TILE * C::PITCH];
  __shared__ __attribute__((aligned(16))) bf16_t sG[2][C::TILE * C::PITCH];
  __shared__ __attribute__((aligned(16))) float sL[2][C::TILE], sD[2][C::TILE];
  __shared__ float sB[kBlockRows * kBiasPitch];   // the bias gradient's way through LDS
  const int tid = threadIdx.x, lane = tid % 64, wave = wave_number(), h2 = lane / 32;
  const int d = H * DH;
  const int64_t ld = 3 * int64_t(d);
  const BlockCoord bc = block_coord((s + kBlockRows - 1) / kBlockRows, H, causal, false);   // the first key blocks are seen by the most queries
  const int head = bc.head, seq = bc.seq, j0 = bc.rb * kBlockRows;
  const bf16_t *base = qkv + int64_t(seq) * s * ld + head * DH;
  const bf16_t *gbase = d_o + int64_t(seq) * s * d + head * DH;
  const float *lbase = lse + (int64_t(seq) * H + head) * s, *dbase = delta + (int64_t(seq) * H + head) * s;
  const int jw = j0 + 32 * wave, key = jw + lane % 32, key_ld = min(key, s - 1);
  bf16x8 fk[C::KSTEPS], fv[C::KSTEPS];
#pragma unroll
  for (int c = 0; c < C::KSTEPS; ++c) {
    fk[c] = frag_global(base + d, ld, key_ld, 16 * c + 8 * h2);
    fv[c] = frag_global(base + 2 * d, ld, key_ld, 16 * c + 8 * h2);
  }
  const float scale = rsqrtf(float(DH)), sc = scale * kLog2e;
  f32x16 acc_k[C::DTILES], acc_v[C::DTILES];
#pragma unroll
  for (int t = 0; t < C::DTILES; ++t) { acc_k[t] = zero16(); acc_v[t] = zero16(); }
  // causal: queries before the block's first key see none of its keys
  const int t_begin = causal ? j0 / C::TILE : 0;
  const int n_tiles = (s + C::TILE - 1) / C::TILE;
  TileRegs<DH, C::TILE> rq, rg;
  float rl = 0.f, rd = 0.f;
  auto fetch = [&](int i0) {
    const int nv = min(C::TILE, s - i0);
    rq.fetch(base + int64_t(i0) * ld, ld, nv, tid);
    rg.fetch(gbase + int64_t(i0) * d, d, nv, tid);
    if (tid < C::TILE) {
      rl = tid < nv ? lbase[i0 + tid] : 0.f;
      rd = tid < nv ? dbase[i0 + tid] : 0.f;
    }
  };
  auto put = [&](int buf) {
    rq.put(sQ[buf], tid);
    rg.put(sG[buf], tid);
    if (tid < C::TILE) {
      sL[buf][tid] = rl * kLog2e;   // log2 units; not where it is fetched, which would make the wave wait for it there
      sD[buf][tid] = rd;
    }
  };
  if (t_begin < n_tiles) {
    fetch(t_begin * C::TILE);
    put(0);
  }
  __syncthreads();
  for (int it = t_begin; it < n_tiles; ++it) {
    const int cur = (it - t_begin) & 1, i0 = it * C::TILE;
    const bool more = it + 1 < n_tiles;
    // (no register prefetch across the compute here: with both accumulator sets it would
    // cost the second resident wave per SIMD)
    if (more) {
      fetch(i0 + C::TILE);
      put(cur ^ 1);
    }
#pragma unroll
    for (int sub = 0; sub < C::TILE / 32; ++sub) {
      const int ib = i0 + 32 * sub;                       // first query of the subtile
      if (causal && ib + 31 < jw) continue;               // every query precedes every key of this wave
      // S[query, key] = Q K^T and dP[query, key] = dO V^T: lane owns a key, registers run over queries
      f32x16 sm = zero16(), dp = zero16();
#pragma unroll
      for (int c = 0; c < C::KSTEPS; ++c) {
        sm = mfma(frag_row<DH>(sQ[cur], 32 * sub + lane % 32, 16 * c + 8 * h2), fk[c], sm);
        dp = mfma(frag_row<DH>(sG[cur], 32 * sub + lane % 32, 16 * c + 8 * h2), fv[c], dp);
      }
      probabilities(sm, dp, sL[cur] + 32 * sub, sD[cur] + 32 * sub, h2, sc, ib + 32 > s || (causal && ib < jw + 31), ib, s, key,
                    causal);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const bf16x8 fp = acc_to_frag(sm, c), fs = acc_to_frag(dp, c);
#pragma unroll
        for (int t = 0; t < C::DTILES; ++t) {
          acc_v[t] = mfma(frag_col<DH>(sG[cur], 32 * sub + 16 * c, 32 * t, lane), fp, acc_v[t]);   // dV^T += dO^T P
          acc_k[t] = mfma(frag_col<DH>(sQ[cur], 32 * sub + 16 * c, 32 * t, lane), fs, acc_k[t]);   // dK^T += Q^T dS
        }
      }
    }
    __syncthreads();
  }
  if (key < s) {
    bf16_t *row = dqkv + (int64_t(seq) * s + key) * ld + head * DH;
#pragma unroll
    for (int t = 0; t < C::DTILES; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        bf16x4 vk, vv;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          vk[k] = static_cast<__bf16>(acc_k[t][4 * j + k] * scale);
          vv[k] = static_cast<__bf16>(acc_v[t][4 * j + k]);
        }
        *reinterpret_cast<bf16x4 *>(row + d + 32 * t + 8 * j + 4 * h2) = vk;
        *reinterpret_cast<bf16x4 *>(row + 2 * d + 32 * t + 8 * j + 4 * h2) = vv;
      }
  }
  if (dbias) {
    bias_grad_sums<C::DTILES>(dbias + d + head * DH, acc_k, scale, key < s, sB, tid);
    bias_grad_sums<C::DTILES>(dbias + 2 * d + head * DH, acc_v, 1.f, key < s, sB, tid);
  }
}

// ---------------------------------------------------------------------------------
// The backward kernels (dK/dV: head dimensions 64 and 128, dQ: 128) on eight waves per workgroup, as in k_attn_fwd_mfma_split: waves
// w and w + 4 share 32 rows of the output and take one 32-row subtile of every streamed tile each, with an accumulator
// of their own; at the end each hands the other half of its sums through LDS.  What bounds these kernels is a wave's
// serial chain (two products, exponentials, conversion, two products), and under a causal mask the heaviest row block's
// chain is the whole launch: four waves walked 3500 cycles per 32x32 subtile.  Halving the chain also halves the share
// of a streamed tile that a thread carries in registers, so the next tile is fetched during the multiplies here too.
// What fits no registers twice (two accumulator sets of dK/dV need more than 128) leaves one such workgroup per compute
// unit, whose waves pass every barrier together; two four-wave workgroups do not, and where both always have work they
// are the faster (the rules and their measurements at the launchers).
template <int DH> struct SplitBwd {
  static constexpr int TILE = 64, NTHR = 512;
  static constexpr int TILE_ELEMS = TILE * Cfg<DH>::PITCH;
  static constexpr int XCH = 4 * 64 * 16 * Cfg<DH>::DTILES * 4;       // bytes: one accumulator set of four waves
  static constexpr int BIAS = 2 * kBlockRows * kBiasPitch * 4;        // both halves of the workgroup sum columns at once
  static constexpr int max3(int a, int b, int c) { return a > b ? (a > c ? a : c) : (b > c ? b : c); }
  static constexpr int DQ_LDS = max3(4 * TILE_ELEMS * 2, XCH, BIAS);
  // four tile buffers, the rows' statistics; at head dimension 128 also the workgroup's V rows, which do not fit the
  // registers beside two accumulator sets of 64
  static constexpr int STATS = 4 * TILE * 4;
  static constexpr int DKV_LDS = max3(4 * TILE_ELEMS * 2 + STATS + (DH == 128 ? kBlockRows * Cfg<DH>::PITCH * 2 : 0), 2 * XCH, BIAS);
};

// dQ: head dimension 128 (64 takes the four-wave kernel).
template <int DH>
__global__ __launch_bounds__(512) HMY_MFMA_IN_VGPRS void k_attn_bwd_dq_split(const bf16_t *qkv, const bf16_t *o, const bf16_t *d_o,
                                                               const float *lse, float *delta, bf16_t *dqkv, float *dbias,
                                                               int s, int H, int causal) {
  static_assert(DH == 128, "two waves per SIMD, one workgroup per compute unit, workgroups ranked for that");
  typedef Cfg<DH> C;
  typedef SplitBwd<DH> S;
  constexpr int TILE = S::TILE;
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  auto sK = [&](int buf) { return smem + buf * S::TILE_ELEMS; };
  auto sV = [&](int buf) { return smem + (2 + buf) * S::TILE_ELEMS; };
  const int tid = threadIdx.x, lane = tid % 64, wave = wave_number(), h2 = lane / 32;
  const int rg = wave % 4, sub = wave / 4;
  const int d = H * DH;
  const int64_t ld = 3 * int64_t(d);
  const BlockCoord bc = block_coord((s + kBlockRows - 1) / kBlockRows, H, causal, true, false);
  const int head = bc.head, seq = bc.seq, q0 = bc.rb * kBlockRows;
  const bf16_t *base = qkv + int64_t(seq) * s * ld + head * DH;
  const bf16_t *gbase = d_o + int64_t(seq) * s * d + head * DH;
  const bf16_t *obase = o + int64_t(seq) * s * d + head * DH;
  const int qw = q0 + 32 * rg, q = qw + lane % 32, q_ld = min(q, s - 1);
  bf16x8 fq[C::KSTEPS], fg[C::KSTEPS];
  float dl = 0.f;
#pragma unroll
  for (int c = 0; c < C::KSTEPS; ++c) {
    fq[c] = frag_global(base, ld, q_ld, 16 * c + 8 * h2);
    fg[c] = frag_global(gbase, d, q_ld, 16 * c + 8 * h2);
    const bf16x8 fo = frag_global(obase, d, q_ld, 16 * c + 8 * h2);
#pragma unroll
    for (int k = 0; k < 8; ++k) dl = fmaf(static_cast<float>(fg[c][k]), static_cast<float>(fo[k]), dl);
  }
  dl += __shfl_xor(dl, 32, 64);   // the other half of the row
  if (sub == 0 && h2 == 0 && q < s) delta[(int64_t(seq) * H + head) * s + q] = dl;
  const float L = lse[(int64_t(seq) * H + head) * s + q_ld] * kLog2e;   // log2 units
  const float scale = rsqrtf(float(DH)), sc = scale * kLog2e;
  f32x16 acc_q[C::DTILES];
#pragma unroll
  for (int t = 0; t < C::DTILES; ++t) acc_q[t] = zero16();
  const int k_end = causal ? min(s, q0 + kBlockRows) : s;
  const int n_tiles = (k_end + TILE - 1) / TILE;
  TileRegs<DH, TILE, S::NTHR> rk, rv;
  rk.fetch(base + d, ld, min(TILE, s), tid);
  rv.fetch(base + 2 * d, ld, min(TILE, s), tid);
  rk.put(sK(0), tid);
  rv.put(sV(0), tid);
  __syncthreads();
  for (int kt = 0; kt < n_tiles; ++kt) {
    const int cur = kt & 1, k0 = kt * TILE;
    const bool more = kt + 1 < n_tiles;
    if (more) {   // next tile's loads fly during this tile's multiplies
      const int kn = k0 + TILE;
      rk.fetch(base + d + int64_t(kn) * ld, ld, min(TILE, s - kn), tid);
      rv.fetch(base + 2 * d + int64_t(kn) * ld, ld, min(TILE, s - kn), tid);
    }
    const int kb = k0 + 32 * sub;   // first key of this wave's subtile
    if (kb < s && (!causal || kb <= qw + 31)) {   // some query of this wave sees some key of it
      f32x16 st = zero16(), dp = zero16();
#pragma unroll
      for (int c = 0; c < C::KSTEPS; ++c) {
        st = mfma(frag_row<DH>(sK(cur), 32 * sub + lane % 32, 16 * c + 8 * h2), fq[c], st);   // S^T = K Q^T
        dp = mfma(frag_row<DH>(sV(cur), 32 * sub + lane % 32, 16 * c + 8 * h2), fg[c], dp);   // dP^T = V dO^T
      }
      mask_keys(st, kb, qw, q, s, h2, causal);
#pragma unroll
      for (int r = 0; r < 16; ++r) st[r] = fast_exp2(fmaf(st[r], sc, -L)) * (dp[r] - dl);     // dS^T
      // dQ^T[dh, query] += K^T dS^T
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const bf16x8 fs = acc_to_frag(st, c);
#pragma unroll
        for (int t = 0; t < C::DTILES; ++t)
          acc_q[t] = mfma(frag_col<DH>(sK(cur), 32 * sub + 16 * c, 32 * t, lane), fs, acc_q[t]);
      }
    }
    if (more) {
      rk.put(sK(cur ^ 1), tid);
      rv.put(sV(cur ^ 1), tid);
    }
    __syncthreads();
  }
  // the first wave of a pair finishes the lower half of the head's columns, the second the upper half
  constexpr int HALF = C::DTILES / 2;
  float *xch = reinterpret_cast<float *>(smem) + rg * (16 * C::DTILES * 64);   // [value][lane]: conflict-free both ways
#pragma unroll
  for (int t = 0; t < HALF; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) xch[((1 - sub) * HALF * 16 + 16 * t + r) * 64 + lane] = sub ? acc_q[t][r] : acc_q[HALF + t][r];
  __syncthreads();
  f32x16 res[HALF];
#pragma unroll
  for (int t = 0; t < HALF; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r)
      res[t][r] = (sub ? acc_q[HALF + t][r] : acc_q[t][r]) + xch[(sub * HALF * 16 + 16 * t + r) * 64 + lane];
  const int col0 = head * DH + 32 * HALF * sub;
  if (q < s) {
    bf16_t *row = dqkv + (int64_t(seq) * s + q) * ld + col0;
#pragma unroll
    for (int t = 0; t < HALF; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        bf16x4 v;
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = static_cast<__bf16>(res[t][4 * j + k] * scale);
        *reinterpret_cast<bf16x4 *>(row + 32 * t + 8 * j + 4 * h2) = v;
      }
  }
  if (dbias) {
    __syncthreads();   // the exchanged sums have been read
    bias_grad_sums<HALF>(dbias + col0, res, scale, q < s, reinterpret_cast<float *>(smem) + sub * (kBlockRows * kBiasPitch),
                         tid % kThreads);
  }
}

// `o` for a caller that does not have delta yet: the workgroup then takes it of all the rows that it streams, ahead of them,
// into LDS behind the tiles (`delta` is not read).
template <int DH, bool OWN_DELTA>
__device__ __forceinline__ void dkv_split_rows(const bf16_t *qkv, const bf16_t *o, const bf16_t *d_o, const float *lse,
                                               const float *delta, bf16_t *dqkv, float *dbias, int s, int H, int causal,
                                               bf16_t *smem, int n_wg, int wg) {
  typedef Cfg<DH> C;
  typedef SplitBwd<DH> S;
  constexpr int TILE = S::TILE;
  constexpr bool kVInLds = DH == 128;
  static_assert(!(OWN_DELTA && kVInLds), "V lies where the rows' delta would");
  auto sQ = [&](int buf) { return smem + buf * S::TILE_ELEMS; };
  auto sG = [&](int buf) { return smem + (2 + buf) * S::TILE_ELEMS; };
  float *sL = reinterpret_cast<float *>(smem + 4 * S::TILE_ELEMS), *sD = sL + 2 * TILE;
  bf16_t *sV = reinterpret_cast<bf16_t *>(sD + 2 * TILE);
  float *sDelta = sD + 2 * TILE;
  const int tid = threadIdx.x, lane = tid % 64, wave = wave_number(), h2 = lane / 32;
  const int rg = wave % 4, sub = wave / 4;
  const int d = H * DH;
  const int64_t ld = 3 * int64_t(d);
  // the first key blocks are seen by the most queries
  const BlockCoord bc = block_coord((s + kBlockRows - 1) / kBlockRows, H, causal, false, false, n_wg, wg);
  const int head = bc.head, seq = bc.seq, j0 = bc.rb * kBlockRows;
  const bf16_t *base = qkv + int64_t(seq) * s * ld + head * DH;
  const bf16_t *gbase = d_o + int64_t(seq) * s * d + head * DH;
  const float *lbase = lse + (int64_t(seq) * H + head) * s, *dbase = delta + (int64_t(seq) * H + head) * s;
  const int jw = j0 + 32 * rg, key = jw + lane % 32, key_ld = min(key, s - 1);
  bf16x8 fk[C::KSTEPS], fv[kVInLds ? 1 : C::KSTEPS];
#pragma unroll
  for (int c = 0; c < C::KSTEPS; ++c) {
    fk[c] = frag_global(base + d, ld, key_ld, 16 * c + 8 * h2);
    if constexpr (!kVInLds) fv[c] = frag_global(base + 2 * d, ld, key_ld, 16 * c + 8 * h2);
  }
  if constexpr (kVInLds) {
    TileRegs<DH, kBlockRows, S::NTHR> rv;
    rv.fetch(base + 2 * d + int64_t(j0) * ld, ld, min(kBlockRows, s - j0), tid);
    rv.put(sV, tid);
  }
  const float scale = rsqrtf(float(DH)), sc = scale * kLog2e;
  f32x16 acc_k[C::DTILES], acc_v[C::DTILES];
#pragma unroll
  for (int t = 0; t < C::DTILES; ++t) { acc_k[t] = zero16(); acc_v[t] = zero16(); }
  // causal: queries before the block's first key see none of its keys
  const int t_begin = causal ? j0 / TILE : 0;
  const int n_tiles = (s + TILE - 1) / TILE;
  TileRegs<DH, TILE, S::NTHR> rq, rgr;
  float rl = 0.f, rd = 0.f;
  auto fetch = [&](int i0) {
    const int nv = min(TILE, s - i0);
    rq.fetch(base + int64_t(i0) * ld, ld, nv, tid);
    rgr.fetch(gbase + int64_t(i0) * d, d, nv, tid);
    if (tid < TILE) {
      rl = tid < nv ? lbase[i0 + tid] : 0.f;
      if constexpr (!OWN_DELTA) rd = tid < nv ? dbase[i0 + tid] : 0.f;
    }
  };
  auto put = [&](int buf) {
    rq.put(sQ(buf), tid);
    rgr.put(sG(buf), tid);
    if (tid < TILE) {
      // log2 units.  Multiplied here and not where it is fetched: there the first wave waited for the load, and the others, at the
      // barrier, for that wave.  The whole backward, us: 32 heads of 128, s = 2048 282 -> 275, causal 165.9 -> 163.2; 50
      // sequences x heads of 64, s = 1024, causal 57.2 -> 55.4
      sL[buf * TILE + tid] = rl * kLog2e;
      if constexpr (!OWN_DELTA) sD[buf * TILE + tid] = rd;
    }
  };
  fetch(t_begin * TILE);
  if constexpr (OWN_DELTA) {
    const bf16_t *obase = o + int64_t(seq) * s * d + head * DH;
    for (int r = t_begin * TILE + 32 * wave; r < n_tiles * TILE; r += 32 * (S::NTHR / 64)) {
      const int row = r + lane % 32;
      bf16x8 unused[C::KSTEPS];
      const float dl = row_delta<DH>(gbase, obase, d, min(row, s - 1), h2, unused);
      if (h2 == 0) sDelta[row] = row < s ? dl : 0.f;
    }
  }
  put(0);
  __syncthreads();
  for (int it = t_begin; it < n_tiles; ++it) {
    const int cur = (it - t_begin) & 1, i0 = it * TILE;
    const bool more = it + 1 < n_tiles;
    if (more) fetch(i0 + TILE);   // next tile's loads fly during this tile's multiplies
    const int ib = i0 + 32 * sub;   // first query of this wave's subtile
    if (ib < s && (!causal || ib + 31 >= jw)) {   // some query of it sees some key of this wave
      // S[query, key] = Q K^T and dP[query, key] = dO V^T: lane owns a key, registers run over queries
      f32x16 sm = zero16(), dp = zero16();
#pragma unroll
      for (int c = 0; c < C::KSTEPS; ++c) {
        sm = mfma(frag_row<DH>(sQ(cur), 32 * sub + lane % 32, 16 * c + 8 * h2), fk[c], sm);
        const bf16x8 v = kVInLds ? frag_row<DH>(sV, 32 * rg + lane % 32, 16 * c + 8 * h2) : fv[kVInLds ? 0 : c];
        dp = mfma(frag_row<DH>(sG(cur), 32 * sub + lane % 32, 16 * c + 8 * h2), v, dp);
      }
      probabilities(sm, dp, sL + cur * TILE + 32 * sub, OWN_DELTA ? sDelta + ib : sD + cur * TILE + 32 * sub, h2, sc,
                    ib + 32 > s || (causal && ib < jw + 31), ib, s, key, causal);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const bf16x8 fp = acc_to_frag(sm, c), fs = acc_to_frag(dp, c);
#pragma unroll
        for (int t = 0; t < C::DTILES; ++t) {
          acc_v[t] = mfma(frag_col<DH>(sG(cur), 32 * sub + 16 * c, 32 * t, lane), fp, acc_v[t]);   // dV^T += dO^T P
          acc_k[t] = mfma(frag_col<DH>(sQ(cur), 32 * sub + 16 * c, 32 * t, lane), fs, acc_k[t]);   // dK^T += Q^T dS
        }
      }
    }
    if (more) put(cur ^ 1);
    __syncthreads();
  }
  // the first wave of a pair finishes dK, the second dV
  float *xch = reinterpret_cast<float *>(smem) + rg * (2 * 16 * C::DTILES * 64);
#pragma unroll
  for (int t = 0; t < C::DTILES; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) xch[((1 - sub) * C::DTILES * 16 + 16 * t + r) * 64 + lane] = sub ? acc_k[t][r] : acc_v[t][r];
  __syncthreads();
  f32x16 res[C::DTILES];
#pragma unroll
  for (int t = 0; t < C::DTILES; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r)
      res[t][r] = (sub ? acc_v[t][r] : acc_k[t][r]) + xch[(sub * C::DTILES * 16 + 16 * t + r) * 64 + lane];
  const float out_scale = sub ? 1.f : scale;
  const int col0 = (1 + sub) * d + head * DH;
  if (key < s) {
    bf16_t *row = dqkv + (int64_t(seq) * s + key) * ld + col0;
#pragma unroll
    for (int t = 0; t < C::DTILES; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        bf16x4 v;
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = static_cast<__bf16>(res[t][4 * j + k] * out_scale);
        *reinterpret_cast<bf16x4 *>(row + 32 * t + 8 * j + 4 * h2) = v;
      }
  }
  if (dbias) {
    __syncthreads();   // the exchanged sums have been read
    bias_grad_sums<C::DTILES>(dbias + col0, res, out_scale, key < s,
                              reinterpret_cast<float *>(smem) + sub * (kBlockRows * kBiasPitch), tid % kThreads);
  }
}

template <int DH>
__global__ __launch_bounds__(512) HMY_MFMA_IN_VGPRS void k_attn_bwd_dkv_split(const bf16_t *qkv, const bf16_t *d_o, const float *lse,
                                                                const float *delta, bf16_t *dqkv, float *dbias, int s,
                                                                int H, int causal) {
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  dkv_split_rows<DH, false>(qkv, nullptr, d_o, lse, delta, dqkv, dbias, s, H, causal, smem, gridDim.x, blockIdx.x);
}
// Both in one launch, for as many workgroups as leave half of the compute units to each: the first half of the grid takes
// dK/dV, the second dQ.  Of the one thing that the former needs of the latter, delta, every workgroup makes its own.
template <int DH>
__global__ __launch_bounds__(512) HMY_MFMA_IN_VGPRS void k_attn_bwd_both(const bf16_t *qkv, const bf16_t *o, const bf16_t *d_o, const float *lse,
                                                           float *delta, bf16_t *dqkv, float *dbias, int s, int H, int causal) {
  static_assert(DqLds<DH>::ELEMS * 2 <= SplitBwd<DH>::DKV_LDS && SplitBwd<DH>::BIAS <= SplitBwd<DH>::DKV_LDS, "one size for both");
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  const int n = gridDim.x / 2, l = blockIdx.x;
  if (l < n)
    dkv_split_rows<DH, true>(qkv, o, d_o, lse, nullptr, dqkv, dbias, s, H, causal, smem, n, l);
  else
    dq_rows<DH, 512>(qkv, o, d_o, lse, delta, dqkv, dbias, s, H, causal, smem, n, l - n);
}

inline int check_launch(const char *what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(HMY_E_HIP, "launch of %s failed: %s", what, hipGetErrorString(e));
  return HMY_OK;
}

// Where the eight-wave kernels pay.  They halve a wave's chain over the streamed rows and pay for it with one workgroup per
// compute unit and a pass of the partial sums through LDS at the end: rows have to be long enough for the first to matter.
//
// Head dimension 64, dK/dV.  Two streamed tiles and more, and up to one workgroup per unit, or two with a causal mask over at
// least eight row blocks.  The whole backward, us, four waves -> eight: 256 workgroups of s = 512 34.1 -> 32.7, of s = 1024
// 55.2 -> 51.6; 512 of s = 512 46.9 -> 54.8; causal, 512 of s = 1024 61.6 -> 62.2, of s = 2048 105 -> 99, of s = 4096 192 ->
// 174, 1024 of s = 1024 98 -> 111.  Rows of 65 to 256 would be faster on four waves: 128 workgroups of s = 65 14.5 -> 14.8, of
// s = 128 15.7 -> 17.1, of s = 256 20.9 -> 21.4, of s = 320 23.2 -> 23.2.  They are left here because eight waves add up in
// another order, and these are the rows whose gradients have been added up in it: results stay bit for bit what they were.
inline bool dkv_split_pays_64(int workgroups, int s, int causal) {
  return s > 64 && (workgroups <= 256 || (causal && s >= 1024 && workgroups <= 512));
}
// Head dimension 128, dK/dV: from rows of nearly a row block on, at every number of workgroups.  The whole backward, us, four
// waves -> eight: s = 64, 128 workgroups 17.7 -> 18.2, 1024 66.0 -> 67.3; s = 96, 128 23.5 -> 23.8, 1024 93.0 -> 92.8; s = 112,
// 128 28.6 -> 27.4, 1024 114 -> 107; s = 128, 256 33.7 -> 33.0, causal 35.1 -> 33.5; s = 144, 512 53.6 -> 50.4, causal 46.7 ->
// 45.9; s = 256, 256 46.6 -> 40.9, 1024 165 -> 143, causal 145 -> 129.  (104 to 111, where eight waves gain as much, keep the
// order of sums that they have had.)
inline bool dkv_split_pays_128(int s) { return s >= 112; }
// Head dimension 128, forward and dQ: one eight-wave workgroup per compute unit against two of the four-wave ones.  Where
// there is no second workgroup for a unit, or where a causal mask makes the heaviest row block the whole launch (16 row
// blocks and more), half the chain wins, dQ's from a later length on (it reads its rows' o as well, and exchanges more).
// Measured, us, four waves -> eight, forward: 128 workgroups of s = 32 4.4 -> 5.5, of s = 96 7.8 -> 8.5 (causal 8.2 -> 8.7), of
// 120 9.6 -> 9.7 (9.9 -> 9.5), 64 of 192 11.0 -> 10.6, 128 of 512 21 -> 18; 512 of s = 512 31 -> 37; 512 of s = 1024, causal
// 39 -> 38; 512 of s = 4096, causal 131 -> 104.  dQ, within the whole backward: 128 workgroups of s = 128 31.2 -> 33.0, 256 of
// 256 51.0 -> 51.0 (causal 47.9 -> 48.5), 96 of 384 57.8 -> 56.8, 128 of 512 71.8 -> 69.8; alone, 512 of s = 512 46 -> 56, 512 of
// s = 1024, causal 51 -> 55, 512 of s = 4096, causal 150 -> 126.
inline bool fwd_split_pays_128(int workgroups, int s, int causal) {
  return (workgroups <= 256 && s >= (causal ? 112 : 192)) || (causal && s >= 2048);
}
inline bool dq_split_pays_128(int workgroups, int s, int causal) { return (workgroups <= 256 && s >= 384) || (causal && s >= 2048); }

// Head dimension 64, where dK/dV takes eight waves: dQ and dK/dV side by side instead of one after the other.  Each of the two is
// a chain over the streamed rows that more compute units do not shorten, so a launch that leaves half of the device idle costs
// as long as a full one.  It pays up to 160 workgroups of each, and, where a causal mask leaves most of them short, up to one
// per unit from rows of 256 on.  The whole backward, us, apart -> together: 12 heads, three sequences of 200 20.5 -> 13.2; 4
// heads, four of 120 15.6 -> 9.7; 8 heads of s = 1024 44.7 -> 31.5, of s = 4096 (128 workgroups) 143.8 -> 105.8; 160 workgroups
// of s = 128 16.4 -> 15.2, of 1024 45.4 -> 41.7, of 4096 144 -> 133; 168 of 128 16.6 -> 17.3, of 512 29.5 -> 32.0, of 1024 46.2 ->
// 51.1; causal, 168 of 128 17.1 -> 17.9, of 256 21.2 -> 18.5, 256 of 256 21.9 -> 20.8, of 512 30.2 -> 26.7, of 1024 46.5 -> 38.1,
// of 4096 144.5 -> 107.4, 252 of 200 21.1 -> 21.4, 320 of 1024 49.1 -> 48.5, 384 53.3 -> 57.0.  The rows' delta has to fit LDS
// behind the tiles.  Results are the same bit for bit.
inline bool both_at_once_pays_64(int workgroups, int s, int causal) {
  constexpr int kRoom = (SplitBwd<64>::DKV_LDS - 4 * SplitBwd<64>::TILE_ELEMS * 2 - SplitBwd<64>::STATS) / 4 / 64 * 64;
  return s <= kRoom && (workgroups <= 160 || (causal && s >= 256 && workgroups <= 256));
}

inline bool eight_waves_allowed() {
  static const bool allowed = std::getenv("HMY_ATTN_SPLIT") == nullptr || std::atoi(std::getenv("HMY_ATTN_SPLIT")) != 0;
  return allowed;
}

template <int DH>
int fwd_t(const void *qkv, void *o, float *lse, int b, int s, int H, int causal, hipStream_t st) {
  const dim3 grid(((s + kBlockRows - 1) / kBlockRows) * H * b);
  if constexpr (DH >= 64) {   // enough 16-byte pieces in a 64-row tile for 512 threads
    if (eight_waves_allowed() && (DH == 64 || fwd_split_pays_128(int(grid.x), s, causal))) {
      hipLaunchKernelGGL((k_attn_fwd_mfma_split<DH>), grid, dim3(512), 0, st, (const bf16_t *)qkv, (bf16_t *)o, lse, s, H,
                         causal);
      return check_launch("attn_fwd_mfma_split");
    }
  }
  hipLaunchKernelGGL((k_attn_fwd_mfma<DH>), grid, dim3(kThreads), 0, st, (const bf16_t *)qkv, (bf16_t *)o, lse, s, H,
                     causal);
  return check_launch("attn_fwd_mfma");
}
template <int DH>
int bwd_t(const void *qkv, const void *o, const void *d_o, const float *lse, float *delta, void *dqkv, float *dbias, int b,
          int s, int H, int causal, hipStream_t st) {
  const dim3 grid(((s + kBlockRows - 1) / kBlockRows) * H * b);
  bool dq_split = false, dkv_split = false;
  if constexpr (DH >= 64)
    dkv_split = eight_waves_allowed() && (DH == 128 ? dkv_split_pays_128(s) : dkv_split_pays_64(int(grid.x), s, causal));
  if constexpr (DH == 64)
    if (dkv_split && both_at_once_pays_64(int(grid.x), s, causal)) {
      hipLaunchKernelGGL((k_attn_bwd_both<DH>), dim3(2 * grid.x), dim3(512), SplitBwd<DH>::DKV_LDS, st, (const bf16_t *)qkv,
                         (const bf16_t *)o, (const bf16_t *)d_o, lse, delta, (bf16_t *)dqkv, dbias, s, H, causal);
      return check_launch("attn_bwd_both");
    }
  if constexpr (DH == 128) {
    dq_split = eight_waves_allowed() && dq_split_pays_128(int(grid.x), s, causal);
    if (dq_split)
      hipLaunchKernelGGL((k_attn_bwd_dq_split<DH>), grid, dim3(512), SplitBwd<DH>::DQ_LDS, st, (const bf16_t *)qkv,
                         (const bf16_t *)o, (const bf16_t *)d_o, lse, delta, (bf16_t *)dqkv, dbias, s, H, causal);
  }
  if (!dq_split)   // either writes delta for the next kernel
    hipLaunchKernelGGL((k_attn_bwd_dq_mfma<DH>), grid, dim3(kThreads), 0, st, (const bf16_t *)qkv, (const bf16_t *)o,
                       (const bf16_t *)d_o, lse, delta, (bf16_t *)dqkv, dbias, s, H, causal);
  if constexpr (DH >= 64)   // enough 16-byte pieces in a 64-row tile for 512 threads
    if (dkv_split)
      hipLaunchKernelGGL((k_attn_bwd_dkv_split<DH>), grid, dim3(512), SplitBwd<DH>::DKV_LDS, st, (const bf16_t *)qkv,
                         (const bf16_t *)d_o, lse, delta, (bf16_t *)dqkv, dbias, s, H, causal);
  if (!dkv_split)
    hipLaunchKernelGGL((k_attn_bwd_dkv_mfma<DH>), grid, dim3(kThreads), 0, st, (const bf16_t *)qkv, (const bf16_t *)d_o,
                       lse, delta, (bf16_t *)dqkv, dbias, s, H, causal);
  return check_launch("attn_bwd_mfma");
}

}  // namespace

int launch_attn_fwd_mfma(const void *qkv, void *o, float *lse, int b, int s, int H, int dh, int causal, stream_t st) {
  if (dh == 32) return fwd_t<32>(qkv, o, lse, b, s, H, causal, (hipStream_t)st);
  if (dh == 64) return fwd_t<64>(qkv, o, lse, b, s, H, causal, (hipStream_t)st);
  if (dh == 128) return fwd_t<128>(qkv, o, lse, b, s, H, causal, (hipStream_t)st);
  return fail(HMY_E_INVALID, "attention: unsupported head dim %d", dh);
}
int launch_attn_bwd_mfma(const void *qkv, const void *o, const void *d_o, const float *lse, float *delta, void *dqkv,
                         float *dbias, int b, int s, int H, int dh, int causal, stream_t st) {
  if (dh == 32) return bwd_t<32>(qkv, o, d_o, lse, delta, dqkv, dbias, b, s, H, causal, (hipStream_t)st);
  if (dh == 64) return bwd_t<64>(qkv, o, d_o, lse, delta, dqkv, dbias, b, s, H, causal, (hipStream_t)st);
  if (dh == 128) return bwd_t<128>(qkv, o, d_o, lse, delta, dqkv, dbias, b, s, H, causal, (hipStream_t)st);
  return fail(HMY_E_INVALID, "attention: unsupported head dim %d", dh);
}

}  // namespace hmy

// fp32 softmax attention forward and backward on the matrix cores (v_mfma_f32_32x32x2_f32), never materialising the
// s x s probabilities.  Same layout as attention.hip: qkv is [T, 3d] with q | k | v thirds, head h at columns h*DH..
//
// A wave owns 32 queries (forward, dQ) or 32 keys (dK/dV) and walks over tiles of 32 rows of the other side, staged
// through LDS with the next tile's global loads in flight.  Scores are computed with the wave's own rows as columns of
// the product (lane % 32), so that softmax runs along a lane's registers plus one exchange between the wave's halves,
// and register r of a lane, row 8*(r/4) + 4*(lane/32) + r%4 of the tile, is directly the second operand of the next
// product's step over the rows {8*(r/4) + r%4, that + 4}: probabilities never leave their registers.
// What bounds it is the fp32 matrix pipe: at head dimension 64 a tile is 64 multiplies of 64 cycles forward against
// some 200 vector instructions.  Against the thread-per-row kernels, 4 x 256 tokens, 8 heads of 64, causal, inside an
// iteration: forward 214 -> 32 us, backward 597 -> 89 us; with the tiles split over four waves 12 and 35.  Where there are rows
// for two workgroups of four waves on every compute unit, those share the staged tiles; elsewhere a workgroup has 32 rows, whose
// tiles one, two or four waves share out (`split` below).
#include "dev_common.h"
#include "hmy_internal.h"

namespace hmy {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kRows = 32;   // rows of a tile, and of a wave

inline int check_launch(const char *what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(HMY_E_HIP, "launch of %s failed: %s", what, hipGetErrorString(e));
  return HMY_OK;
}

__device__ __forceinline__ float part(const float4 &v, int q) { return q == 0 ? v.x : q == 1 ? v.y : q == 2 ? v.z : v.w; }
__device__ __forceinline__ int reg_row(int r, int h) { return 8 * (r / 4) + 4 * h + r % 4; }

// rows [r0, r0 + 32) x DH columns of a global array (row stride ld): global -> registers -> LDS, rows past `rows` as zeros
template <int DH, int W>
struct Stage {
  static constexpr int kPitch = DH + 4;    // 16-byte row reads of 16 consecutive rows fall on distinct banks
  static constexpr int kVecs = kRows * DH / 4 / (64 * W);
  float4 v[kVecs];
  __device__ __forceinline__ void load(const float *src, int64_t ld, int rows, int tid) {
#pragma unroll
    for (int i = 0; i < kVecs; ++i) {
      const int idx = tid + 64 * W * i, r = idx / (DH / 4), c = 4 * (idx % (DH / 4));
      v[i] = r < rows ? *reinterpret_cast<const float4 *>(src + int64_t(r) * ld + c) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
  __device__ __forceinline__ void store(float *s, int tid) const {
#pragma unroll
    for (int i = 0; i < kVecs; ++i) {
      const int idx = tid + 64 * W * i, r = idx / (DH / 4), c = 4 * (idx % (DH / 4));
      *reinterpret_cast<float4 *>(s + r * kPitch + c) = v[i];
    }
  }
};

// a wave's own rows as the second operand: columns 8c + 4h .. +3 of row lane%32
template <int DH>
__device__ __forceinline__ void load_own(float4 (&f)[DH / 8], const float *row, int h, bool active) {
#pragma unroll
  for (int c = 0; c < DH / 8; ++c)
    f[c] = active ? *reinterpret_cast<const float4 *>(row + 8 * c + 4 * h) : make_float4(0.f, 0.f, 0.f, 0.f);
}
// [32 tile rows] x [32 own rows]: tile rows read from LDS
template <int DH>
__device__ __forceinline__ f32x16 product(const float *tile, const float4 (&own)[DH / 8], int l32, int h) {
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
  for (int c = 0; c < DH / 8; ++c) {
    const float4 a = *reinterpret_cast<const float4 *>(tile + l32 * (DH + 4) + 8 * c + 4 * h);
#pragma unroll
    for (int q = 0; q < 4; ++q) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(part(a, q), part(own[c], q), acc, 0, 0, 0);
  }
  return acc;
}
// acc[DH columns of the tile] x [32 own rows] += tile^T w, w = [32 tile rows] x [32 own rows] in registers
template <int DH>
__device__ __forceinline__ void accumulate(f32x16 (&acc)[DH / 32], const float *tile, const f32x16 &w, int l32, int h) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const float *row = tile + reg_row(r, h) * (DH + 4) + l32;
#pragma unroll
    for (int b = 0; b < DH / 32; ++b) acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(row[32 * b], w[r], acc[b], 0, 0, 0);
  }
}
template <int DH>
__device__ __forceinline__ void store_own(float *row, const f32x16 (&acc)[DH / 32], int h, float scale) {
#pragma unroll
  for (int b = 0; b < DH / 32; ++b)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<float4 *>(row + 32 * b + 8 * g + 4 * h) =
          make_float4(acc[b][4 * g] * scale, acc[b][4 * g + 1] * scale, acc[b][4 * g + 2] * scale, acc[b][4 * g + 3] * scale);
}
template <int DH>
__device__ __forceinline__ void clear(f32x16 (&acc)[DH / 32]) {
#pragma unroll
  for (int b = 0; b < DH / 32; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[b][r] = 0.f;
}

// Which of a workgroup's rows and tiles a wave takes.  KW == 1: W waves of 32 rows each, all walking over the same tiles.
// KW > 1 (W == 1): KW waves share 32 rows and take every KW-th tile each, staged for themselves, with sums of their own
// that meet in LDS at the end.
template <int W, int KW> struct Role {
  static_assert(W == 1 || KW == 1, "either the rows or the tiles are shared out");
  int lane, h, l32, tid, wave, part;
  __device__ __forceinline__ Role() {
    lane = threadIdx.x % 64;
    h = lane / 32;
    l32 = lane % 32;
    tid = KW > 1 ? lane : threadIdx.x;
    wave = KW > 1 ? 0 : threadIdx.x / 64;
    part = KW > 1 ? threadIdx.x / 64 : 0;
  }
  // tiles in LDS: written by those who read them (a wave's own accesses to LDS are executed in order)
  __device__ __forceinline__ void sync() const {
    if (KW == 1) {
      __syncthreads();
    } else {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
  }
};
// the waves' sums on their way to each other: 16 N floats per lane of each wave, [wave][value][lane]
template <int N>
__device__ __forceinline__ void put_sums(float *x, int part, int lane, const f32x16 (&acc)[N]) {
#pragma unroll
  for (int b = 0; b < N; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) x[(part * 16 * N + 16 * b + r) * 64 + lane] = acc[b][r];
}
// values 4 q .. 4 q + 3 of all waves, added up in their order with weights w
template <int N, int KW>
__device__ __forceinline__ float4 add_sums(const float *x, int q, int lane, const float (&w)[KW]) {
  float v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[e] = 0.f;
#pragma unroll
    for (int p = 0; p < KW; ++p) v[e] = fmaf(w[p], x[(p * 16 * N + 4 * q + e) * 64 + lane], v[e]);
  }
  return make_float4(v[0], v[1], v[2], v[3]);
}
// a wave's share of the rows of DH values: float4 q holds columns 32 (q / 4) + 8 (q % 4) + 4 h ..
template <int DH, int KW>
__device__ __forceinline__ void store_sums(float *row, const float *x, const Role<1, KW> &me, const float (&w)[KW], float scale) {
  constexpr int N = DH / 32, PER = 4 * N / KW;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int q = me.part * PER + i;
    const float4 v = add_sums<N, KW>(x, q, me.lane, w);
    *reinterpret_cast<float4 *>(row + 32 * (q / 4) + 8 * (q % 4) + 4 * me.h) = make_float4(v.x * scale, v.y * scale, v.z * scale, v.w * scale);
  }
}

// grid (row blocks of 32 W, H, b), 64 W KW threads
template <int DH, int W, int KW>
__global__ __launch_bounds__(64 * W * KW) void k_attn_f32_fwd(const float *qkv, float *o, float *lse, int s, int H, int causal) {
  constexpr int kTile = kRows * (DH + 4);
  __shared__ __attribute__((aligned(16))) float smem[2 * KW * kTile];   // per wave of a split: its K tile, its V tile
  const Role<W, KW> me;
  float *const sK = smem + 2 * me.part * kTile, *const sV = sK + kTile;
  const int d = H * DH, ld = 3 * d;
  const int h = me.h, l32 = me.l32, wave = me.wave;
  const int head = blockIdx.y, seq = blockIdx.z;
  // with a causal mask the last rows see the most keys: their workgroups start first
  const int blk = causal ? gridDim.x - 1 - blockIdx.x : blockIdx.x;
  const int q0 = (blk * W + wave) * kRows, i = q0 + l32;
  const bool active = i < s;
  const float *base = qkv + int64_t(seq) * s * ld + head * DH;
  const float scale = rsqrtf(float(DH));
  float4 q[DH / 8];
  load_own<DH>(q, base + int64_t(i) * ld, h, active);
  f32x16 acc[DH / 32];
  clear<DH>(acc);
  float mrun = -INFINITY, lrun = 0.f;
  const int j_end = causal ? min(s, (blk + 1) * W * kRows) : s;   // keys any row of this workgroup may see
  const int my_end = q0 >= s ? 0 : causal ? min(s, q0 + kRows) : s;
  Stage<DH, W> tk, tv;
  auto fetch = [&](int j) {
    tk.load(base + d + int64_t(j) * ld, ld, min(kRows, s - j), me.tid);
    tv.load(base + 2 * d + int64_t(j) * ld, ld, min(kRows, s - j), me.tid);
  };
  if (KW == 1 || me.part * kRows < j_end) fetch(me.part * kRows);   // (the first tile is always there)
  for (int j0 = me.part * kRows; j0 < j_end; j0 += KW * kRows) {
    me.sync();
    tk.store(sK, me.tid);
    tv.store(sV, me.tid);
    me.sync();
    const int j1 = j0 + kRows;
    if (j0 + KW * kRows < j_end) fetch(j0 + KW * kRows);
    if (j0 >= my_end) continue;   // beyond this wave's rows; the barriers are still met
    f32x16 p = product<DH>(sK, q, l32, h);
    const bool whole = j1 <= s && (!causal || j1 - 1 <= q0);
    float tmax = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int j = j0 + reg_row(r, h);
      p[r] = whole || (j < s && (!causal || j <= i)) ? p[r] * scale : -INFINITY;
      tmax = fmaxf(tmax, p[r]);
    }
    tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
    const float mnew = fmaxf(mrun, tmax);       // finite: key 0 is visible to every row
    const float corr = __expf(mrun - mnew);     // exp(-inf) = 0 on the first tile
    float sum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      p[r] = __expf(p[r] - mnew);
      sum += p[r];
    }
    lrun = lrun * corr + (sum + __shfl_xor(sum, 32, 64));
    mrun = mnew;
#pragma unroll
    for (int b = 0; b < DH / 32; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[b][r] *= corr;
    accumulate<DH>(acc, sV, p, l32, h);
  }
  float *orow = o + (int64_t(seq) * s + i) * d + head * DH;
  if constexpr (KW == 1) {
    if (active) store_own<DH>(orow, acc, h, 1.f / lrun);
  } else {
    __shared__ float sM[KW][32], sS[KW][32];
    __syncthreads();   // every wave is done with its tiles
    put_sums<DH / 32>(smem, me.part, me.lane, acc);
    if (h == 0) {
      sM[me.part][l32] = mrun;
      sS[me.part][l32] = lrun;
    }
    __syncthreads();
    float w[KW];
    mrun = sM[0][l32];   // finite: the first tile is the first wave's
#pragma unroll
    for (int p = 1; p < KW; ++p) mrun = fmaxf(mrun, sM[p][l32]);
    lrun = 0.f;
#pragma unroll
    for (int p = 0; p < KW; ++p) {
      w[p] = __expf(sM[p][l32] - mrun);   // 0 for a wave that had no tile
      lrun = fmaf(w[p], sS[p][l32], lrun);
    }
    if (active) store_sums<DH, KW>(orow, smem, me, w, 1.f / lrun);
  }
  if (active && me.part == 0 && h == 0) lse[(int64_t(seq) * H + head) * s + i] = mrun + __logf(lrun);
}

// dQ, and delta[seq, head, i] = sum_c do[i,c] * o[i,c] for the dK/dV kernel
template <int DH, int W, int KW>
__global__ __launch_bounds__(64 * W * KW) void k_attn_f32_dq(const float *qkv, const float *o, const float *d_o, const float *lse,
                                                        float *delta, float *dqkv, int s, int H, int causal) {
  constexpr int kTile = kRows * (DH + 4);
  __shared__ __attribute__((aligned(16))) float smem[2 * KW * kTile];   // per wave of a split: its K tile, its V tile
  const Role<W, KW> me;
  float *const sK = smem + 2 * me.part * kTile, *const sV = sK + kTile;
  const int d = H * DH, ld = 3 * d;
  const int h = me.h, l32 = me.l32, wave = me.wave;
  const int head = blockIdx.y, seq = blockIdx.z;
  const int blk = causal ? gridDim.x - 1 - blockIdx.x : blockIdx.x;
  const int q0 = (blk * W + wave) * kRows, i = q0 + l32;
  const bool active = i < s;
  const float *base = qkv + int64_t(seq) * s * ld + head * DH;
  const int64_t row = int64_t(seq) * s + i, stat = (int64_t(seq) * H + head) * s + i;
  const float scale = rsqrtf(float(DH));
  float4 q[DH / 8], g[DH / 8];
  load_own<DH>(q, base + int64_t(i) * ld, h, active);
  load_own<DH>(g, d_o + row * d + head * DH, h, active);
  float dl = 0.f, L = 0.f;
  {
    float4 ov[DH / 8];
    load_own<DH>(ov, o + row * d + head * DH, h, active);
#pragma unroll
    for (int c = 0; c < DH / 8; ++c)
      dl = fmaf(g[c].x, ov[c].x, fmaf(g[c].y, ov[c].y, fmaf(g[c].z, ov[c].z, fmaf(g[c].w, ov[c].w, dl))));
    dl += __shfl_xor(dl, 32, 64);
    if (active) {
      L = lse[stat];
      if (me.part == 0 && h == 0) delta[stat] = dl;
    }
  }
  f32x16 acc[DH / 32];
  clear<DH>(acc);
  const int j_end = causal ? min(s, (blk + 1) * W * kRows) : s;
  const int my_end = q0 >= s ? 0 : causal ? min(s, q0 + kRows) : s;
  Stage<DH, W> tk, tv;
  auto fetch = [&](int j) {
    tk.load(base + d + int64_t(j) * ld, ld, min(kRows, s - j), me.tid);
    tv.load(base + 2 * d + int64_t(j) * ld, ld, min(kRows, s - j), me.tid);
  };
  if (KW == 1 || me.part * kRows < j_end) fetch(me.part * kRows);   // (the first tile is always there)
  for (int j0 = me.part * kRows; j0 < j_end; j0 += KW * kRows) {
    me.sync();
    tk.store(sK, me.tid);
    tv.store(sV, me.tid);
    me.sync();
    const int j1 = j0 + kRows;
    if (j0 + KW * kRows < j_end) fetch(j0 + KW * kRows);
    if (j0 >= my_end) continue;
    f32x16 p = product<DH>(sK, q, l32, h);
    const f32x16 dp = product<DH>(sV, g, l32, h);
    const bool whole = j1 <= s && (!causal || j1 - 1 <= q0);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int j = j0 + reg_row(r, h);
      const float e = __expf(p[r] * scale - L);
      p[r] = whole || (j < s && (!causal || j <= i)) ? e * (dp[r] - dl) : 0.f;
    }
    accumulate<DH>(acc, sK, p, l32, h);
  }
  if constexpr (KW == 1) {
    if (active) store_own<DH>(dqkv + row * ld + head * DH, acc, h, scale);
  } else {
    __syncthreads();   // every wave is done with its tiles
    put_sums<DH / 32>(smem, me.part, me.lane, acc);
    __syncthreads();
    float w[KW];
#pragma unroll
    for (int p = 0; p < KW; ++p) w[p] = 1.f;
    if (active) store_sums<DH, KW>(dqkv + row * ld + head * DH, smem, me, w, scale);
  }
}

// dK and dV: a wave owns 32 keys, queries staged through LDS
template <int DH, int W, int KW>
__global__ __launch_bounds__(64 * W * KW) void k_attn_f32_dkv(const float *qkv, const float *d_o, const float *lse, const float *delta,
                                                         float *dqkv, int s, int H, int causal) {
  constexpr int kTile = kRows * (DH + 4);
  __shared__ __attribute__((aligned(16))) float smem[2 * KW * kTile];   // per wave of a split: its Q tile, its dO tile
  __shared__ __attribute__((aligned(16))) float stats[2 * KW * kRows];
  const Role<W, KW> me;
  float *const sQ = smem + 2 * me.part * kTile, *const sG = sQ + kTile, *const sL = stats + 2 * me.part * kRows, *const sD = sL + kRows;
  const int d = H * DH, ld = 3 * d;
  const int h = me.h, l32 = me.l32, wave = me.wave;
  const int head = blockIdx.y, seq = blockIdx.z;
  const int b0 = blockIdx.x * W * kRows, j0 = b0 + wave * kRows, j = j0 + l32;
  const bool active = j < s;
  const float *base = qkv + int64_t(seq) * s * ld + head * DH;
  const float *gbase = d_o + int64_t(seq) * s * d + head * DH;
  const int64_t stat = (int64_t(seq) * H + head) * s;
  const float scale = rsqrtf(float(DH));
  float4 k[DH / 8], v[DH / 8];
  load_own<DH>(k, base + d + int64_t(j) * ld, h, active);
  load_own<DH>(v, base + 2 * d + int64_t(j) * ld, h, active);
  f32x16 dk[DH / 32], dv[DH / 32];
  clear<DH>(dk);
  clear<DH>(dv);
  const int i_begin = causal ? b0 : 0;   // earlier queries see none of this workgroup's keys
  Stage<DH, W> tq, tg;
  float nl = 0.f, nd = 0.f;
  auto fetch = [&](int i0) {
    const int rows = min(kRows, s - i0);
    tq.load(base + int64_t(i0) * ld, ld, rows, me.tid);
    tg.load(gbase + int64_t(i0) * d, d, rows, me.tid);
    if (me.tid < kRows) {
      const bool ok = me.tid < rows;
      nl = ok ? lse[stat + i0 + me.tid] : 0.f;
      nd = ok ? delta[stat + i0 + me.tid] : 0.f;
    }
  };
  const int i_first = i_begin + me.part * kRows;
  if (i_first < s) fetch(i_first);
  for (int i0 = i_first; i0 < s; i0 += KW * kRows) {
    me.sync();
    tq.store(sQ, me.tid);
    tg.store(sG, me.tid);
    if (me.tid < kRows) {
      sL[me.tid] = nl;
      sD[me.tid] = nd;
    }
    me.sync();
    if (i0 + KW * kRows < s) fetch(i0 + KW * kRows);
    if (j0 >= s || (causal && i0 + kRows <= j0)) continue;   // none of these queries sees this wave's keys
    f32x16 p = product<DH>(sQ, k, l32, h);
    f32x16 ds = product<DH>(sG, v, l32, h);
    const bool whole = i0 + kRows <= s && j0 + kRows <= s && (!causal || j0 + kRows - 1 <= i0);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 L = *reinterpret_cast<const float4 *>(sL + 8 * g + 4 * h);
      const float4 dl = *reinterpret_cast<const float4 *>(sD + 8 * g + 4 * h);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = 4 * g + q, i = i0 + reg_row(r, h);
        const float e = __expf(p[r] * scale - part(L, q));
        p[r] = whole || (i < s && active && (!causal || j <= i)) ? e : 0.f;
        ds[r] = p[r] * (ds[r] - part(dl, q));
      }
    }
    accumulate<DH>(dv, sG, p, l32, h);
    accumulate<DH>(dk, sQ, ds, l32, h);
  }
  float *row = dqkv + (int64_t(seq) * s + j) * ld + head * DH;
  if constexpr (KW == 1) {
    if (active) {
      store_own<DH>(row + d, dk, h, scale);
      store_own<DH>(row + 2 * d, dv, h, 1.f);
    }
  } else {
    float w[KW];
#pragma unroll
    for (int p = 0; p < KW; ++p) w[p] = 1.f;
    __syncthreads();   // every wave is done with its tiles
    put_sums<DH / 32>(smem, me.part, me.lane, dk);
    __syncthreads();
    if (active) store_sums<DH, KW>(row + d, smem, me, w, scale);
    __syncthreads();
    put_sums<DH / 32>(smem, me.part, me.lane, dv);
    __syncthreads();
    if (active) store_sums<DH, KW>(row + 2 * d, smem, me, w, 1.f);
  }
}

// four waves of rows per workgroup once that still leaves two workgroups for every compute unit
inline bool wide(int b, int s, int H) { return int64_t(b) * H * ((s + 4 * kRows - 1) / (4 * kRows)) >= 512; }
// Waves that share 32 rows and split their tiles, for a launch of few waves, which is as long as one wave's chain over its
// tiles.  Measured, us, one wave -> two -> four: forward at head dimension 64, 256 groups of 32 rows, s = 256 31 -> 18 -> 12,
// 512 of s = 1024 115 -> 91 -> 53, 1024 of s = 512 63 -> 53 -> 57, of s = 256 37 -> 36 -> 40; at 32, 1024 of s = 256 23 -> 20
// -> 23; at 128, 256 of s = 256 49 -> 31 -> 25, 512 of s = 512 94 -> 62 -> 67, 1024 of s = 512 101 -> 116 -> 128.  Backward at
// 64, 256 of s = 256 85 -> 49 -> 35, 384 of s = 500 164 -> 91 -> 101, 512 of s = 1024 320 -> 171 -> 182, 1024 of s = 512 175 ->
// 181 -> 201; at 128, 256 157 -> 127 -> 97, 512 300 -> 255 -> 276.  Two tiles: 64 groups of s = 64 27 -> 19 -> 21. (All of
// dK/dV at 128: a wave that has its tiles to itself stages both of them, 128 registers beside 128 of sums and 128 of K and V,
// and spills 288, where two that share them spill 100 and four none.  What the spilling costs is in these figures.)
inline int split(int b, int s, int H, int dh, bool backward) {
  const int tiles = (s + kRows - 1) / kRows;
  const int64_t groups = int64_t(b) * H * tiles;
  int parts = groups <= 256 ? 4 : groups <= 512 ? 2 : 1;
  if (!backward && dh != 128) parts = groups <= 512 ? 4 : groups <= 1024 ? 2 : 1;
  return tiles == 1 ? 1 : tiles == 2 ? (parts < 2 ? parts : 2) : parts;
}

template <int DH, int W, int KW>
int fwd_t(const float *qkv, float *o, float *lse, int b, int s, int H, int causal, hipStream_t st) {
  const dim3 grid((s + W * kRows - 1) / (W * kRows), H, b);
  hipLaunchKernelGGL((k_attn_f32_fwd<DH, W, KW>), grid, dim3(64 * W * KW), 0, st, qkv, o, lse, s, H, causal);
  return check_launch("attn_f32_fwd");
}
template <int DH, int W, int KW>
int bwd_t(const float *qkv, const float *o, const float *d_o, const float *lse, float *delta, float *dqkv, int b, int s, int H,
          int causal, hipStream_t st) {
  const dim3 grid((s + W * kRows - 1) / (W * kRows), H, b);
  hipLaunchKernelGGL((k_attn_f32_dq<DH, W, KW>), grid, dim3(64 * W * KW), 0, st, qkv, o, d_o, lse, delta, dqkv, s, H, causal);
  hipLaunchKernelGGL((k_attn_f32_dkv<DH, W, KW>), grid, dim3(64 * W * KW), 0, st, qkv, d_o, lse, delta, dqkv, s, H, causal);
  return check_launch("attn_f32_bwd");
}

}  // namespace

// (one wave per group: two of them to a workgroup at head dimension 128)
#define DISPATCH_DIM(FN, DH, ONE, ...)                  \
  do {                                                  \
    if (wide(b, s, H)) return FN<DH, 4, 1>(__VA_ARGS__); \
    if (parts == 4) return FN<DH, 1, 4>(__VA_ARGS__);   \
    if (parts == 2) return FN<DH, 1, 2>(__VA_ARGS__);   \
    return FN<DH, ONE, 1>(__VA_ARGS__);                 \
  } while (0)
#define DISPATCH_F32(FN, BACKWARD, ...)                                   \
  do {                                                                    \
    const int parts = split(b, s, H, dh, BACKWARD);                       \
    if (dh == 32) DISPATCH_DIM(FN, 32, 1, __VA_ARGS__);                   \
    if (dh == 64) DISPATCH_DIM(FN, 64, 1, __VA_ARGS__);                   \
    if (dh == 128) DISPATCH_DIM(FN, 128, 2, __VA_ARGS__);                 \
    return fail(HMY_E_INVALID, "attention: unsupported head dim %d", dh); \
  } while (0)

int launch_attn_fwd_f32(const float *qkv, float *o, float *lse, int b, int s, int H, int dh, int causal, stream_t st) {
  DISPATCH_F32(fwd_t, false, qkv, o, lse, b, s, H, causal, (hipStream_t)st);
}
int launch_attn_bwd_f32(const float *qkv, const float *o, const float *d_o, const float *lse, float *delta, float *dqkv, int b,
                        int s, int H, int dh, int causal, stream_t st) {
  DISPATCH_F32(bwd_t, true, qkv, o, d_o, lse, delta, dqkv, b, s, H, causal, (hipStream_t)st);
}

}  // namespace hmy

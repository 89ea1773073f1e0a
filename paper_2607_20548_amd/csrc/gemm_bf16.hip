// bfloat16 products of the Muon Newton-Schulz iteration on the CDNA4 matrix
// cores (v_mfma_f32_32x32x16_bf16): C = round_bf16(alpha * P Q^T + beta * D)
// with P (M x K), Q (N x K) and D, C (M x N) bfloat16, row-major, every row
// k-contiguous.  The sum is accumulated in fp32 and rounded to bfloat16 once
// (nearest, ties to even), after the epilogue's linear combination.
//
// Tiling: large products take 256 x 256 tiles (gemm_bf16_nt256 below), the
// others a 256-thread workgroup (4 wave64s, 2 x 2) per 128 x 128 tile: each
// wave owns 64 x 64 as 2 x 2 MFMA 32x32 accumulators (64 x 64 tiles of 32 x 32
// per wave for products with few tiles).  K advances in
// slabs of 64 staged through double-buffered LDS as [x][k] rows padded to 72
// bfloat16 (144 bytes, so that the 16-byte reads of 16 consecutive lanes fall
// in distinct banks); at MFMA step q a lane (row xl, half h) feeds the 8
// values k = 16 q + 8 h .. +7 of its row, the same k for both operands.
// Global loads are 16 bytes (8 bfloat16) at addresses clamped into the
// operand; rows past the operand only reach outputs that are never written,
// and k past K is zeroed at the LDS store of the last slab.
//
// SYRK mode launches only the tiles on or below the diagonal and mirrors
// each stored value, so C is bitwise symmetric (for P = Q).  A second output
// Ct = C^T is optional (the iterate is kept in both layouts so that every
// product reads k-contiguous rows).
#include "internal.h"

#include <algorithm>
#include <type_traits>

namespace soap {
namespace {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

constexpr int KB = 64;           // K slab (bfloat16 values)
constexpr int LDK = KB + 8;      // LDS row stride in bfloat16
constexpr int NTH = 256;

enum { BMODE_GENERAL = 0, BMODE_SYRK = 1 };

struct BfParams {
  int M, N, K;
  const uint16_t *P; int64_t ldp, sP;
  const uint16_t *Q; int64_t ldq, sQ;
  const uint16_t *D; int64_t ldd, sD;
  uint16_t *C; int64_t ldc, sC;
  uint16_t *Ct; int64_t ldct, sCt;
  float alpha, beta;
  int tiles_m, tiles_n, ntiles;
};

__device__ __forceinline__ uint16_t to_bf16(float f) {   // nearest, ties to even
  return __builtin_bit_cast(uint16_t, (__bf16)f);
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// One operand slab: TB rows x 64 k as 8 TB chunks of 8 values, TB / 32 per
// thread (chunk = tid + 256 s: row chunk >> 3, k offset 8 (chunk & 7)).
template <int TB>
struct Slab {
  uint4 r[TB / 32];
  __device__ __forceinline__ void load(const uint16_t *__restrict__ base, int64_t ld, int x0,
                                       int k0, int X, int K, int tid) {
#pragma unroll
    for (int s = 0; s < TB / 32; ++s) {
      const int c = tid + NTH * s;
      const int x = min(x0 + (c >> 3), X - 1);
      const int k = min(k0 + 8 * (c & 7), K - 8);
      r[s] = *reinterpret_cast<const uint4 *>(base + (int64_t)x * ld + k);
    }
  }
  // kvalid: k-values of this slab inside K (KB except in the last slab).
  __device__ __forceinline__ void store(uint16_t *lds, int tid, int kvalid) {
#pragma unroll
    for (int s = 0; s < TB / 32; ++s) {
      const int c = tid + NTH * s;
      if (8 * (c & 7) >= kvalid) r[s] = make_uint4(0u, 0u, 0u, 0u);   // K % 8 == 0
      *reinterpret_cast<uint4 *>(lds + (c >> 3) * LDK + 8 * (c & 7)) = r[s];
    }
  }
};

template <int MODE>
__device__ __forceinline__ void bf_tile_coords(const BfParams &p, int t, int &tm, int &tn) {
  const int nt = p.ntiles;
  if ((nt & 7) == 0) t = (t & 7) * (nt >> 3) + (t >> 3);   // contiguous run per XCD
  if (MODE == BMODE_SYRK) {
    int r = (int)((sqrtf(8.f * (float)t + 1.f) - 1.f) * 0.5f);
    while ((r + 1) * (r + 2) / 2 <= t) ++r;
    while (r * (r + 1) / 2 > t) --r;
    tm = r;
    tn = t - r * (r + 1) / 2;
  } else {
    const int per_group = 8 * p.tiles_n;
    const int group = t / per_group;
    const int first_m = group * 8;
    const int gsz = min(p.tiles_m - first_m, 8);
    const int in_group = t - group * per_group;
    tm = first_m + in_group % gsz;
    tn = in_group / gsz;
  }
}

// TB = 128, or 64 (four waves of one 32 x 32 block) for products with few
// tiles.
template <int MODE, int TB>
__global__ __launch_bounds__(NTH, 2) void gemm_bf16_nt(BfParams p) {
  constexpr int TILE_U16 = TB * LDK, WT = TB / 2, NBLK = WT / 32;
  __shared__ __attribute__((aligned(16))) uint16_t lds[2 * 2 * TILE_U16];
  int tm, tn;
  bf_tile_coords<MODE>(p, blockIdx.x, tm, tn);
  const int64_t bz = blockIdx.z;
  const uint16_t *P = p.P + bz * p.sP;
  const uint16_t *Q = p.Q + bz * p.sQ;
  const int m0 = tm * TB, n0 = tn * TB;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int xl = lane & 31, h = lane >> 5;

  v16f acc[NBLK][NBLK];
#pragma unroll
  for (int i = 0; i < NBLK; ++i)
#pragma unroll
    for (int j = 0; j < NBLK; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  auto buf = [&](int stage, int which) { return lds + (stage * 2 + which) * TILE_U16; };
  const int nk = (p.K + KB - 1) / KB;
  Slab<TB> sa, sb;
  if (nk > 0) {
    sa.load(P, p.ldp, m0, 0, p.M, p.K, tid);
    sb.load(Q, p.ldq, n0, 0, p.N, p.K, tid);
    const int kv = min(KB, p.K);
    sa.store(buf(0, 0), tid, kv);
    sb.store(buf(0, 1), tid, kv);
  }
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const int cur = kt & 1;
    const bool more = kt + 1 < nk;
    if (more) {
      sa.load(P, p.ldp, m0, (kt + 1) * KB, p.M, p.K, tid);
      sb.load(Q, p.ldq, n0, (kt + 1) * KB, p.N, p.K, tid);
    }
    const uint16_t *la = buf(cur, 0), *lb = buf(cur, 1);
#pragma unroll
    for (int q = 0; q < KB / 16; ++q) {
      v8bf fa[NBLK], fb[NBLK];
#pragma unroll
      for (int i = 0; i < NBLK; ++i)
        fa[i] = __builtin_bit_cast(
            v8bf, *reinterpret_cast<const uint4 *>(la + (wm * WT + 32 * i + xl) * LDK + 16 * q + 8 * h));
#pragma unroll
      for (int j = 0; j < NBLK; ++j)
        fb[j] = __builtin_bit_cast(
            v8bf, *reinterpret_cast<const uint4 *>(lb + (wn * WT + 32 * j + xl) * LDK + 16 * q + 8 * h));
#pragma unroll
      for (int i = 0; i < NBLK; ++i)
#pragma unroll
        for (int j = 0; j < NBLK; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
    }
    if (more) {
      const int kv = min(KB, p.K - (kt + 1) * KB);
      sa.store(buf(cur ^ 1, 0), tid, kv);
      sb.store(buf(cur ^ 1, 1), tid, kv);
    }
    __syncthreads();
  }

  // Epilogue.  Accumulator register r of block (i, j) holds
  // C[row0 + 8 (r/4) + 4 h + r%4][col0 + xl].
  uint16_t *C = p.C + bz * p.sC;
  const uint16_t *D = p.D ? p.D + bz * p.sD : nullptr;
  uint16_t *Ct = p.Ct ? p.Ct + bz * p.sCt : nullptr;
#pragma unroll
  for (int i = 0; i < NBLK; ++i)
#pragma unroll
    for (int j = 0; j < NBLK; ++j) {
      const int col = n0 + wn * WT + 32 * j + xl;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int rowb = m0 + wm * WT + 32 * i + 8 * g + 4 * h;
        uint16_t v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int row = rowb + e;
          float x = p.alpha * acc[i][j][4 * g + e];
          if (D && row < p.M && col < p.N) x += p.beta * from_bf16(D[(int64_t)row * p.ldd + col]);
          v[e] = to_bf16(x);
        }
        if (col >= p.N) continue;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int row = rowb + e;
          if (row >= p.M) continue;
          if (MODE == BMODE_SYRK && row < col) continue;   // the mirror is written by its owner
          C[(int64_t)row * p.ldc + col] = v[e];
          if (MODE == BMODE_SYRK && row != col) C[(int64_t)col * p.ldc + row] = v[e];
        }
        if (Ct) {   // Ct[col][rowb .. rowb+3]: one 8-byte store when all four rows exist
          uint16_t *dst = Ct + (int64_t)col * p.ldct + rowb;
          if (rowb + 3 < p.M) {
            *reinterpret_cast<uint2 *>(dst) =
                make_uint2((uint32_t)v[0] | ((uint32_t)v[1] << 16), (uint32_t)v[2] | ((uint32_t)v[3] << 16));
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (rowb + e < p.M) dst[e] = v[e];
          }
        }
      }
    }
}

// The same product by 256 x 256 tiles: 256 threads, 4 waves (2 x 2), one per
// SIMD, each 128 x 128 as 4 x 4 accumulators (256 of the 512 registers a lane
// may hold).  A wave reads 8 KB of LDS for 16 matrix instructions: the reads
// and the slab's writes take three quarters of the matrix instructions'
// time, where eight waves of 128 x 64 took all of it (12 KB).  K advances in
// slabs of 64 through two LDS buffers of unpadded 128-byte rows whose 16-byte
// units are permuted (unit g of row x at g ^ (x / 2 % 8)), so that sixteen
// consecutive rows of one g lie in different banks (with x % 8 for x / 2 % 8,
// which covers eight rows, conflicts took 0.4 of the LDS cycles: the step of
// 4096 x 14336 15.3 -> 14.9 ms).  With one wave per SIMD nothing else hides a
// latency, so each of a slab's four steps of 16 k multiplies fragments read
// during the step before, the first two steps also move the next slab from
// registers to LDS and load the one after it (in flight for a whole slab),
// and the barrier lies before the fourth step, which reads the next slab's
// first fragments.  The sums run over k in the same order as with 128-tiles:
// the results are the same bit for bit.  Measured against 128-tiles and eight
// waves of 128 x 64: B X of 4096 x 14336 750, 610 -> 500 us (960 TFLOP/s; 3.5
// tiles per CU, so 1100 while the chip is full); of 64 x (768 x 2048), K = 768,
// 665, 360 -> 300 us, most of it the epilogue, which one tile per CU leaves
// uncovered (two tiles of 256 x 128 per CU took as long).  The matrix
// instructions run 0.55-0.6 of the main loop's time; the rest is waiting for
// memory.  A second slab in flight does not fit the registers.
// Epilogue: 64 rows at a time through LDS in fp32 (each result is rounded
// once, by the conversion instruction: in integer arithmetic the bank's step
// took 10.4 ms instead of 9.8), D read (a band ahead) and C written 16 bytes
// per lane, and the transposed output (C itself mirrored in SYRK mode) from
// the columns of the same 64 rows.
constexpr int T2 = 256;
constexpr int OP2 = T2 * KB;                    // one operand slab, bfloat16 values
constexpr int SLD2 = T2 + 4;                    // staging row in floats

__device__ __forceinline__ int unit2(int x, int g) { return x * KB + 8 * (g ^ ((x >> 1) & 7)); }

// TAIL: K is not a multiple of the slab.
template <int MODE, bool TAIL>
__global__ __launch_bounds__(NTH, 1) void gemm_bf16_nt256(BfParams p) {
  __shared__ __attribute__((aligned(16))) uint16_t lds[2 * 2 * OP2];
  static_assert(64 * SLD2 * 4 <= 2 * 2 * OP2 * 2, "the staging rows fit the slabs");
  int tm, tn;
  bf_tile_coords<MODE>(p, blockIdx.x, tm, tn);
  const int64_t bz = blockIdx.z;
  const uint16_t *P = p.P + bz * p.sP;
  const uint16_t *Q = p.Q + bz * p.sQ;
  const int m0 = tm * T2, n0 = tn * T2;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int xl = lane & 31, h = lane >> 5;

  v16f acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // thread -> rows lr + 32 s, unit lg of each operand; slabs past the last
  // are loaded from clamped addresses and never multiplied
  const int lr = tid >> 3, lg = tid & 7;
  uint4 ra[8], rb[8];
  const uint16_t *pa[8], *pb[8];
#pragma unroll
  for (int s = 0; s < 8; ++s)
    pa[s] = P + (int64_t)min(m0 + lr + 32 * s, p.M - 1) * p.ldp;
#pragma unroll
  for (int s = 0; s < 8; ++s)
    pb[s] = Q + (int64_t)min(n0 + lr + 32 * s, p.N - 1) * p.ldq;
  auto load = [&](auto &r, const auto &src, int kt) {
    const int k = min(kt * KB + 8 * lg, p.K - 8);
#pragma unroll
    for (unsigned s = 0; s < sizeof(r) / sizeof(uint4); ++s)
      r[s] = *reinterpret_cast<const uint4 *>(src[s] + k);
  };
  auto store = [&](const auto &r, uint16_t *dst, int kt) {
    const bool dead = TAIL && kt * KB + 8 * lg >= p.K;   // K % 8 == 0
#pragma unroll
    for (unsigned s = 0; s < sizeof(r) / sizeof(uint4); ++s)
      *reinterpret_cast<uint4 *>(dst + unit2(lr + 32 * s, lg)) =
          dead ? make_uint4(0u, 0u, 0u, 0u) : r[s];
  };
  auto op = [&](int kt, int which) { return lds + ((kt & 1) * 2 + which) * OP2; };
  v8bf fa[2][4], fb[2][4];
  auto frag = [&](int f, int kt, int q) {
    const uint16_t *la = op(kt, 0), *lb = op(kt, 1);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      fa[f][i] = __builtin_bit_cast(v8bf, *reinterpret_cast<const uint4 *>(
          la + unit2(wm * 128 + 32 * i + xl, 2 * q + h)));
      fb[f][i] = __builtin_bit_cast(v8bf, *reinterpret_cast<const uint4 *>(
          lb + unit2(wn * 128 + 32 * i + xl, 2 * q + h)));
    }
  };
  auto multiply = [&](int f) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[f][i], fb[f][j], acc[i][j], 0, 0, 0);
  };
  // One step's instructions in turn: two matrix instructions, an LDS read and
  // (moves) an LDS write and a global load, eight times.
  auto interleave = [&](auto moves) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if constexpr (decltype(moves)::value) {
        __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  const int nk = (p.K + KB - 1) / KB;
  load(ra, pa, 0);
  load(rb, pb, 0);
  store(ra, op(0, 0), 0);
  store(rb, op(0, 1), 0);
  load(ra, pa, 1);
  load(rb, pb, 1);
  __syncthreads();
  frag(0, 0, 0);
  for (int kt = 0; kt < nk; ++kt) {
    __builtin_amdgcn_sched_barrier(0);
    frag(1, kt, 1);
    store(ra, op(kt + 1, 0), kt + 1);
    load(ra, pa, kt + 2);
    multiply(0);
    interleave(std::true_type{});
    frag(0, kt, 2);
    store(rb, op(kt + 1, 1), kt + 1);
    load(rb, pb, kt + 2);
    multiply(1);
    interleave(std::true_type{});
    frag(1, kt, 3);
    multiply(0);
    interleave(std::false_type{});
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
    frag(0, kt + 1, 0);
    multiply(1);
    interleave(std::false_type{});
  }

  uint16_t *C = p.C + bz * p.sC;
  const uint16_t *D = p.D ? p.D + bz * p.sD : nullptr;
  // the transposed output: Ct, or C itself in SYRK mode
  uint16_t *Ct = MODE == BMODE_SYRK ? C : (p.Ct ? p.Ct + bz * p.sCt : nullptr);
  const int64_t ldct = MODE == BMODE_SYRK ? p.ldc : p.ldct;
  float *stage = reinterpret_cast<float *>(lds);
  // thread -> (row (tid >> 5) + 8 u of a band, 8 columns)
  const int er = tid >> 5, ec = 8 * (tid & 31);
  uint4 dv[8];
  auto load_d = [&](int ps) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int row = m0 + 64 * ps + er + 8 * u, col = n0 + ec;
      dv[u] = make_uint4(0u, 0u, 0u, 0u);
      if (D && row < p.M && col < p.N)                    // N % 8 == 0
        dv[u] = *reinterpret_cast<const uint4 *>(D + (int64_t)row * p.ldd + col);
    }
  };
  load_d(0);
  __syncthreads();                         // the last fragments are read
#pragma unroll
  for (int ps = 0; ps < 4; ++ps) {         // rows 64 ps .. 64 ps + 63 of the tile
    if (wm == ps >> 1) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            stage[(32 * i + 8 * (r >> 2) + 4 * h + (r & 3)) * SLD2 + wn * 128 + 32 * j + xl] =
                acc[2 * (ps & 1) + i][j][r];
    }
    __syncthreads();
    const int rb0 = m0 + 64 * ps;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int row = rb0 + er + 8 * u, col = n0 + ec;
      float *sp = stage + (er + 8 * u) * SLD2 + ec;
      if (row >= p.M || col >= p.N) continue;             // N % 8 == 0
      const uint32_t dw[4] = {dv[u].x, dv[u].y, dv[u].z, dv[u].w};
      uint32_t ow[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float x0 = p.alpha * sp[2 * q], x1 = p.alpha * sp[2 * q + 1];
        if (D) {
          x0 += p.beta * from_bf16((uint16_t)(dw[q] & 0xffffu));
          x1 += p.beta * from_bf16((uint16_t)(dw[q] >> 16));
        }
        const uint16_t b0 = to_bf16(x0), b1 = to_bf16(x1);
        ow[q] = (uint32_t)b0 | ((uint32_t)b1 << 16);
        sp[2 * q] = from_bf16(b0);                        // for the transposed output
        sp[2 * q + 1] = from_bf16(b1);
      }
      uint16_t *dst = C + (int64_t)row * p.ldc + col;
      if (MODE != BMODE_SYRK || col + 7 <= row) {
        *reinterpret_cast<uint4 *>(dst) = make_uint4(ow[0], ow[1], ow[2], ow[3]);
      } else {
#pragma unroll
        for (int q = 0; q < 8; ++q)
          if (col + q <= row) dst[q] = (uint16_t)(ow[q >> 1] >> (16 * (q & 1)));
      }
    }
    if (ps < 3) load_d(ps + 1);
    __syncthreads();
    if (Ct) {
#pragma unroll
      for (int u = 0; u < 8; ++u) {        // thread -> (column, 8 rows)
        const int e = tid + NTH * u, c = e >> 3, r8 = 8 * (e & 7);
        const int col = n0 + c, row = rb0 + r8;
        if (col >= p.N || row >= p.M) continue;           // M % 8 == 0
        uint32_t ow[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint32_t lo = __float_as_uint(stage[(r8 + 2 * q) * SLD2 + c]) >> 16;
          const uint32_t hi = __float_as_uint(stage[(r8 + 2 * q + 1) * SLD2 + c]) >> 16;
          ow[q] = lo | (hi << 16);
        }
        uint16_t *dst = Ct + (int64_t)col * ldct + row;
        if (MODE != BMODE_SYRK || row > col) {
          *reinterpret_cast<uint4 *>(dst) = make_uint4(ow[0], ow[1], ow[2], ow[3]);
        } else {
#pragma unroll
          for (int q = 0; q < 8; ++q)
            if (row + q > col) dst[q] = (uint16_t)(ow[q >> 1] >> (16 * (q & 1)));
        }
      }
      __syncthreads();
    }
  }
}

// X_0 in both layouts: Xo = round_bf16(inv * S) (rows x cols) and Xt = Xo^T,
// through 32 x 32 LDS tiles; S is fp32 (transposed on input when trans).
__global__ __launch_bounds__(256) void bf16_scale_both_kernel(const float *__restrict__ S,
                                                              int rows, int cols, int trans,
                                                              const float *__restrict__ inv,
                                                              uint16_t *__restrict__ Xo,
                                                              uint16_t *__restrict__ Xt) {
  __shared__ uint16_t tile[32][34];
  const int64_t bz = blockIdx.z;
  const int64_t rc = (int64_t)rows * cols;
  const float *Sb = S + bz * rc;
  uint16_t *Xob = Xo + bz * rc, *Xtb = Xt + bz * rc;
  const float sc = inv[bz];
  const int r0 = blockIdx.y * 32, c0 = blockIdx.x * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int k = ty; k < 32; k += 8) {
    const int r = r0 + k, c = c0 + tx;
    if (r < rows && c < cols) {
      // element (r, c) of the (possibly transposed) source
      const float s = trans ? Sb[(int64_t)c * rows + r] : Sb[(int64_t)r * cols + c];
      const uint16_t b = to_bf16(s * sc);
      Xob[(int64_t)r * cols + c] = b;
      tile[k][tx] = b;
    }
  }
  __syncthreads();
  for (int k = ty; k < 32; k += 8) {
    const int c = c0 + k, r = r0 + tx;
    if (r < rows && c < cols) Xtb[(int64_t)c * rows + r] = tile[tx][k];
  }
}

// W <- alpha W + beta X (X bfloat16).
__global__ __launch_bounds__(256) void axpby_bf16_kernel(float *__restrict__ W,
                                                         const uint16_t *__restrict__ X, int64_t n,
                                                         float alpha, float beta) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
    W[i] = alpha * W[i] + beta * from_bf16(X[i]);
}

}  // namespace

// 256-tiles where 128-tiles would not all be resident at once (two per compute
// unit), if they are themselves or hold at least 2.5 of those on average (small
// and odd sides leave them half empty).  16 iterations in 256-tiles and in
// 128-tiles: triangles of 528 128-tiles (4096 x 4096) 5.65 and 7.11 ms, of 406
// (3584 x 3584) 4.74 and 4.30; full products of 576 (3072 x 3072) 3.63 and 4.43,
// of 400 (2560 x 2560) 2.78 and 2.62; banks of 128 x (256 x 256), 384 and 512 of
// them, 1.88 and 1.49; of 300 x (320 x 640), whose triangles hold 2 each,
// 8.88 and 8.05; of 128 x (128 x 256) 1.25 and, in 64-tiles, 0.76.
static constexpr int64_t ROUND_256 = 256, ROUND_128 = 512;
// 64-tiles while 128-tiles would leave compute units idle: 1024 x 1024 1.38 ->
// 0.79 ms, 1536 x 3072 2.21 -> 1.75; the same with a bound of 400.
static constexpr int64_t MAX_TILES_64 = 192;

hipError_t launch_gemm_bf16_nt(const BfGemmDesc &d, hipStream_t s) {
  if (d.M <= 0 || d.N <= 0 || d.batch <= 0) return hipSuccess;
  if (d.K % 8 != 0 || d.ldp % 8 != 0 || d.ldq % 8 != 0 || (d.Ct && d.ldct % 4 != 0))
    return hipErrorInvalidValue;
  BfParams p;
  p.M = (int)d.M; p.N = (int)d.N; p.K = (int)d.K;
  p.P = d.P; p.ldp = d.ldp; p.sP = d.sP;
  p.Q = d.Q; p.ldq = d.ldq; p.sQ = d.sQ;
  p.D = d.D; p.ldd = d.ldd; p.sD = d.sD;
  p.C = d.C; p.ldc = d.ldc; p.sC = d.sC;
  p.Ct = d.Ct; p.ldct = d.ldct; p.sCt = d.sCt;
  p.alpha = d.alpha; p.beta = d.beta;
  if (d.syrk && p.M != p.N) return hipErrorInvalidValue;
  auto tiles = [&](int bt) {
    p.tiles_m = (p.M + bt - 1) / bt;
    p.tiles_n = (p.N + bt - 1) / bt;
    p.ntiles = d.syrk ? p.tiles_m * (p.tiles_m + 1) / 2 : p.tiles_m * p.tiles_n;
  };
  // 16-byte accesses to C, D and Ct in the 256-tile epilogue
  auto al = [](const void *q) { return (reinterpret_cast<uintptr_t>(q) & 15u) == 0; };
  const bool wide = d.M % 8 == 0 && d.N % 8 == 0 && d.ldc % 8 == 0 && d.sC % 8 == 0 && al(d.C) &&
                    (!d.D || (d.ldd % 8 == 0 && d.sD % 8 == 0 && al(d.D))) &&
                    (!d.Ct || (d.ldct % 8 == 0 && d.sCt % 8 == 0 && al(d.Ct)));
  tiles(T2);
  const int64_t n256 = p.ntiles * d.batch;
  tiles(128);
  const int64_t n128 = p.ntiles * d.batch;
  if (wide && d.K > 0 && n128 > ROUND_128 && (n256 <= ROUND_256 || 2 * n128 >= 5 * n256) &&
      !(d.syrk && d.Ct)) {
    tiles(T2);
    const dim3 grid(p.ntiles, 1, (unsigned)d.batch);
    const bool tail = p.K % KB != 0;
#define SOAP_BF(MODE, TAIL) hipLaunchKernelGGL((gemm_bf16_nt256<MODE, TAIL>), grid, dim3(NTH), 0, s, p)
    if (d.syrk) { if (tail) SOAP_BF(BMODE_SYRK, true); else SOAP_BF(BMODE_SYRK, false); }
    else { if (tail) SOAP_BF(BMODE_GENERAL, true); else SOAP_BF(BMODE_GENERAL, false); }
#undef SOAP_BF
  } else {
    const bool few = n128 <= MAX_TILES_64;
    if (few) tiles(64);
    const dim3 grid(p.ntiles, 1, (unsigned)d.batch);
#define SOAP_BF(MODE, TB) hipLaunchKernelGGL((gemm_bf16_nt<MODE, TB>), grid, dim3(NTH), 0, s, p)
    if (d.syrk) { if (few) SOAP_BF(BMODE_SYRK, 64); else SOAP_BF(BMODE_SYRK, 128); }
    else { if (few) SOAP_BF(BMODE_GENERAL, 64); else SOAP_BF(BMODE_GENERAL, 128); }
#undef SOAP_BF
  }
  return hipGetLastError();
}

hipError_t launch_bf16_scale_both(const float *S, int64_t batch, int64_t rows, int64_t cols,
                                  bool trans, const float *inv, uint16_t *Xo, uint16_t *Xt,
                                  hipStream_t s) {
  if (batch <= 0 || rows <= 0 || cols <= 0) return hipSuccess;
  hipLaunchKernelGGL(bf16_scale_both_kernel,
                     dim3((unsigned)((cols + 31) / 32), (unsigned)((rows + 31) / 32), (unsigned)batch),
                     dim3(256), 0, s, S, (int)rows, (int)cols, trans ? 1 : 0, inv, Xo, Xt);
  return hipGetLastError();
}

hipError_t launch_axpby_bf16(float *W, const uint16_t *X, int64_t count, float alpha, float beta,
                             hipStream_t s) {
  if (count <= 0) return hipSuccess;
  const int64_t blocks = std::min<int64_t>((count + 255) / 256, 2048);
  hipLaunchKernelGGL(axpby_bf16_kernel, dim3((unsigned)blocks), dim3(256), 0, s, W, X, count, alpha,
                     beta);
  return hipGetLastError();
}

}  // namespace soap

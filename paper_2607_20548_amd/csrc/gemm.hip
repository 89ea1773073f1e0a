// fp32 GEMM on the CDNA4 matrix cores, used for every dense product of the
// SOAP step: the factor EMAs (one triangle), the power products L Q_L and
// R Q_R, the rotations and the compact-WY updates of the QR.
//
// Arithmetic: each fp32 operand is split into three bfloat16 parts,
// x = hi + mid + lo (exact: 3 x 8 bits and the parts' signs cover the 24 bits),
// and a product takes the six partial products above 2^-27 of the largest on
// v_mfma_f32_32x32x16_bf16, which run at 16 times the rate of the fp32 matrix
// instructions (six of them: 2.7 times).  bfloat16 products are exact in fp32;
// the sums of one K slab start from zero and are added to the fp32
// accumulators on the vector unit.  Left in the matrix instructions' own
// accumulator, a long sum of one sign lost 1.2e-5 (K = 6144), because they
// cut addends off below its last bits; as it is, the error against fp64 is
// 2.2e-7 at 4096^3 and 3.1e-7 at 8192^3 (Gaussian operands), against 1.15e-6
// and 1.6e-6 on v_mfma_f32_32x32x2_f32.  Operands are split once, on the way
// to LDS, scaled so that bfloat16's range holds their parts (see SCALE); sums
// that overflow are handled after the K loop (see there).
// Measured: 4096^3 1150 -> 855 us and 14336^3 (both operands x-contiguous)
// 44.0 -> 34.5 ms against the fp32 instructions, i.e. 161-187 TFLOP/s
// of products, 1.0-1.1 PFLOP/s of bfloat16 matrix work; the same launches on
// zero operands ran at 205-234, so that the card's power bounds the large
// products (a large library product in bfloat16 runs at 1.37 PFLOP/s).
//
// Tiling: a 256-thread workgroup (4 wave64s in a 2 x 2 arrangement) computes a
// 128 x 128 tile of C (64 x 64 for products with few tiles); each wave owns a
// 64 x 64 sub-tile held as 2 x 2 32x32 accumulators.  K advances in slabs of
// 32; the global loads of the next slab are in flight while a slab is
// multiplied.
//
// Epilogue: the tile goes through LDS (free after the K loop) so that C is read
// and written 16 bytes per lane (see the epilogue).
//
// Tile order: the 8 XCDs receive workgroups round-robin, so the linear tile
// index is remapped to give each XCD a contiguous run of tiles, and that run is
// walked in groups of 8 tile-rows so that neighbouring tiles share A rows and B
// columns in the XCD's L2.
#include "internal.h"

namespace soap {
namespace {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

constexpr int BIG = 128;      // tile rows and columns
constexpr int SMALL = 64;     // of products whose 128-tiles leave compute units idle
constexpr int BK = 32;
constexpr int NTHREADS = 256;
constexpr int GROUP_M = 8;

// LDS image of one operand slab (BT x-rows, 32 k): three bfloat16 planes; in
// a plane the 16-byte unit (x, g) holds k = 8 g .. 8 g + 7 of row x, at
// g * GROUP + (x / 2) * 16 + (x % 2) * ODD.  A fragment read (one g, 32
// consecutive x) then covers all banks every eight lanes, and so do the
// writes of both loaders (x pairs or consecutive x of one g; four g of two
// rows).
template <int BT>
struct Lds {
  static constexpr int ODD = BT / 2 * 16 + 64;
  static constexpr int GROUP = 2 * ODD + 16;
  static constexpr int PLANE = 4 * GROUP;
  static constexpr int OPERAND = 3 * PLANE;
  static __device__ __forceinline__ int unit(int x, int g) {
    return g * GROUP + (x >> 1) * 16 + (x & 1) * ODD;
  }
};

// Operands are scaled by this on their way to the parts and the sums scaled
// back at the end (both exact short of fp32's own range): the last bit of the
// smallest fp32 value, 2^-149, becomes 2^-133, the smallest bfloat16, so that
// the three parts hold every operand exactly (the matrix instructions keep
// bfloat16's subnormals).  Unscaled, operands below 2^-110 lost bits: 1e-37
// times 1e12 came out with a relative error of 3e-4.  It takes one
// multiplication per loaded value, 1 to 2% of a product.
constexpr float SCALE = 65536.f;
constexpr float UNSCALE = 1.f / (SCALE * SCALE);

enum { MODE_GENERAL = 0, MODE_SYRK = 1, MODE_ADAM = 2 };
// How an operand is read: V_ALIGNED with 16-byte (k-contiguous) or 8-byte
// (x-contiguous) aligned loads and whole quads / pairs, V_ANY the same loads
// at 4-byte alignment with the ragged ends handled.
enum { V_ALIGNED = 0, V_ANY = 1 };

struct KParams {
  int M, N, K;
  const float *A;
  int64_t lda, sA;
  const float *B;
  int64_t ldb, sB;
  float *C;
  int64_t ldc, sC;
  float alpha, beta;
  const float *D;   // what beta applies to (C unless the caller gave another)
  int64_t ldd, sD;
  float *V;
  float *Nout;
  float b2, c1, c2, eps;
  int tiles_m, tiles_n, ntiles;
  int kslice;       // K extent of one split-K slice (multiple of BK); = K when not split
  float *part;      // split-K partials, or nullptr
  const unsigned *skip;   // batch entry b is skipped when skip[b * sSkip] != 0 (or nullptr)
  int64_t sSkip;
};

struct f4u { float x, y, z, w; };   // 4-byte aligned
typedef v2f v2fu __attribute__((aligned(4)));

// A wave-uniform address kept in scalar registers, for loads at a 32-bit
// offset from it.
typedef const __attribute__((address_space(1))) char *GlobalBytes;
__device__ __forceinline__ GlobalBytes uniform_row(const float *p) {
  uint64_t a = reinterpret_cast<uint64_t>(p);
  asm("" : "+s"(a));
  return reinterpret_cast<GlobalBytes>(a);
}

// Two floats as three bfloat16 pairs with SCALE x = hi + mid + lo exactly
// (for |x| below 2^111, past which a part is infinite): each part is the
// remainder rounded to nearest, so mid <= 2^-9 hi and lo <= 2^-18 hi.
__device__ __forceinline__ void split2(float x0, float x1, uint32_t &hi, uint32_t &mid,
                                       uint32_t &lo) {
  x0 *= SCALE;
  x1 *= SCALE;
  const v2f v = {x0, x1};
  hi = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, v2bf));
  const float r0 = x0 - __uint_as_float(hi << 16);
  const float r1 = x1 - __uint_as_float(hi & 0xffff0000u);
  const v2f r = {r0, r1};
  mid = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, v2bf));
  const v2f q = {r0 - __uint_as_float(mid << 16), r1 - __uint_as_float(mid & 0xffff0000u)};
  lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(q, v2bf));
}

// Splits eight consecutive k of row x and writes them as unit (x, g).
template <int BT>
__device__ __forceinline__ void store_unit(char *lds, int x, int g, const float (&v)[8]) {
  uint4 h, m, l;
  split2(v[0], v[1], h.x, m.x, l.x);
  split2(v[2], v[3], h.y, m.y, l.y);
  split2(v[4], v[5], h.z, m.z, l.z);
  split2(v[6], v[7], h.w, m.w, l.w);
  char *dst = lds + Lds<BT>::unit(x, g);
  *reinterpret_cast<uint4 *>(dst) = h;
  *reinterpret_cast<uint4 *>(dst + Lds<BT>::PLANE) = m;
  *reinterpret_cast<uint4 *>(dst + 2 * Lds<BT>::PLANE) = l;
}

// One operand slab of BT x-rows by BK k-values: RPT rows of 8 values per thread.
//   KCONTIG = true : global element (x, k) at base[x*ld + k]; a thread holds
//     k-octet tid & 3 of rows tid >> 2 and (BT = 128) 64 + (tid >> 2)
//   KCONTIG = false: global element (x, k) at base[k*ld + x]; a thread holds
//     the k-octet of its wave (tid >> 6) for rows 2 lane, 2 lane + 1 (BT =
//     128) or row lane (BT = 64)
// Every load is issued unconditionally at an address clamped into the
// matrix, so nothing consumes a loaded register before store(): rows x >= X
// only reach output rows or columns that are never written, and k-values
// past the end of K are zeroed by store().  V_ALIGNED needs K % 4 == 0 (and
// the row starts 16-byte aligned) for k-contiguous operands and an even X
// (8-byte aligned rows) for x-contiguous ones.
template <int BT, bool KCONTIG, int LOADS>
struct SlabLoader {
  static constexpr int RPT = BT / 64;
  float r[RPT][8];

  __device__ __forceinline__ void load(const float *__restrict__ base, int64_t ld, int x0,
                                       int k0, int X, int K, int tid) {
    if constexpr (KCONTIG) {
      const int k = k0 + 8 * (tid & 3);
#pragma unroll
      for (int s = 0; s < RPT; ++s) {
        const float *row = base + (int64_t)min(x0 + (tid >> 2) + 64 * s, X - 1) * ld;
        if (LOADS == V_ALIGNED) {
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const float4 v = *reinterpret_cast<const float4 *>(row + min(k + 4 * q, K - 4));
            r[s][4 * q] = v.x; r[s][4 * q + 1] = v.y; r[s][4 * q + 2] = v.z; r[s][4 * q + 3] = v.w;
          }
        } else if (k0 + BK <= K) {
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const f4u v = *reinterpret_cast<const f4u *>(row + k + 4 * q);
            r[s][4 * q] = v.x; r[s][4 * q + 1] = v.y; r[s][4 * q + 2] = v.z; r[s][4 * q + 3] = v.w;
          }
        } else {   // the ragged slab (or past the end): element by element
#pragma unroll
          for (int e = 0; e < 8; ++e) r[s][e] = row[min(k + e, K - 1)];
        }
      }
    } else {
      // k is uniform within a wave: the row address is formed on the scalar
      // unit.  In 128-tiles, whose vector unit is as busy as the matrix
      // cores, it stays there, with the lane's offset as the load's own
      // 32-bit one (a 64-bit addition per load otherwise: 14336^3 37.0 ->
      // 34.4 ms), and the rows of a whole slab follow each other by additions
      // (a clamp and a 64-bit product per row otherwise: 4096^3 793 -> 774 us).
      // The short chains of 64-tiles were slower with it (517 x 517 x 1283 66
      // -> 69 us).
      const int k = k0 + 8 * __builtin_amdgcn_readfirstlane(tid >> 6);
      if (RPT == 2 && (LOADS == V_ALIGNED || X > 1)) {
        const int x = x0 + 2 * (tid & 63), xb = min(x0, X - 2);
        unsigned xc = 4u * (unsigned)(min(x, X - 2) - xb);
        asm volatile("" : "+v"(xc));   // widened at its loads, as their offset field
        // an odd X: the last row is the second of the clamped pair
        const bool odd = LOADS == V_ANY && x == X - 1;
        auto get = [&](int e, const float *row) {
          const GlobalBytes rowp = uniform_row(row);
          float vx, vy;
          if (LOADS == V_ALIGNED) {
            const v2f v = *reinterpret_cast<const __attribute__((address_space(1))) v2f *>(rowp + xc);
            vx = v.x; vy = v.y;
          } else {
            const v2fu v = *reinterpret_cast<const __attribute__((address_space(1))) v2fu *>(rowp + xc);
            vx = v.x; vy = v.y;
          }
          r[0][e] = odd ? vy : vx;
          r[RPT - 1][e] = vy;
        };
        if (k0 + BK <= K) {
          const float *row = base + (int64_t)k * ld + xb;
#pragma unroll
          for (int e = 0; e < 8; ++e, row += ld) get(e, row);
        } else {   // the ragged slab (or past the end)
#pragma unroll
          for (int e = 0; e < 8; ++e) get(e, base + (int64_t)min(k + e, K - 1) * ld + xb);
        }
      } else {   // one row per thread (or a single row in all)
        const unsigned xc = (unsigned)min(x0 + (tid & 63), X - 1);
#pragma unroll
        for (int e = 0; e < 8; ++e)
          r[0][e] = r[RPT - 1][e] = (base + (int64_t)min(k + e, K - 1) * ld)[xc];
      }
    }
  }

  // Splits the slab into the LDS planes; kvalid = number of k-values of this
  // slab inside K (BK except in the last, ragged slab).
  __device__ __forceinline__ void store(char *lds, int tid, int kvalid) {
    const int g = KCONTIG ? (tid & 3) : (tid >> 6);
    if (kvalid < BK) {
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int s = 0; s < RPT; ++s)
          if (8 * g + e >= kvalid) r[s][e] = 0.f;
    }
#pragma unroll
    for (int s = 0; s < RPT; ++s)
      store_unit<BT>(lds, KCONTIG ? (tid >> 2) + 64 * s : RPT * (tid & 63) + s, g, r[s]);
  }
};

// Four consecutive k of one row of an operand, from p on (used by the fp32
// path below); those past `valid` are zero and not read.  p moves on by eight.
template <bool KCONTIG>
__device__ __forceinline__ void exact_operand(const float *&p, int64_t ld, int valid, float (&e)[4]) {
  const int64_t step = KCONTIG ? 1 : ld;
  if (KCONTIG && valid >= 4) {
    const f4u v = *reinterpret_cast<const f4u *>(p);
    e[0] = v.x; e[1] = v.y; e[2] = v.z; e[3] = v.w;
  } else {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      e[u] = 0.f;
      if (u < valid) e[u] = p[u * step];
    }
  }
  p += 8 * step;
}

// Maps the linear workgroup id to a (tile-row, tile-column) pair.
template <int MODE>
__device__ __forceinline__ void tile_coords(const KParams &p, int t, int &tm, int &tn) {
  const int nt = p.ntiles;
  if ((nt & 7) == 0) t = (t & 7) * (nt >> 3) + (t >> 3);  // contiguous run per XCD
  if (MODE == MODE_SYRK) {
    // lower-triangle tiles (tm >= tn), enumerated row by row
    int r = (int)((sqrtf(8.f * (float)t + 1.f) - 1.f) * 0.5f);
    while ((r + 1) * (r + 2) / 2 <= t) ++r;
    while (r * (r + 1) / 2 > t) --r;
    tm = r;
    tn = t - r * (r + 1) / 2;
  } else {
    const int per_group = GROUP_M * p.tiles_n;
    const int group = t / per_group;
    const int first_m = group * GROUP_M;
    const int gsz = min(p.tiles_m - first_m, GROUP_M);
    const int in_group = t - group * per_group;
    tm = first_m + in_group % gsz;
    tn = in_group / gsz;
  }
}

// Two workgroups per CU (256 registers per lane: accumulators, one or two
// blocks' slab sums, the slab in flight and the fragments of a block), whose
// loads, splits and matrix instructions overlap one another; bounded to
// three, the slab sums spill (180 -> 89 TFLOP/s).  Most V_ANY forms (odd sizes)
// keep 8 to 44 bytes per lane in scratch even so: a few words moved per slab,
// none among its matrix instructions.
//
// BT = 64 is for products with few tiles (four waves of one 32 x 32 block
// each): four times the workgroups, a quarter of the work in each, and three
// slabs in flight, since such products wait for memory.
template <int BT, int TA, int TB, int LOADS, int MODE, int TAG, bool PERSIST = false>
__global__ __launch_bounds__(NTHREADS, BT == BIG ? 2 : 3) void gemm_f32_split(KParams p) {
  using LD = Lds<BT>;
  constexpr int WT = BT / 2;        // a wave's tile
  constexpr int NBLK = WT / 32;     // its 32 x 32 blocks each way
  constexpr int AHEAD = BT == BIG ? 1 : 3;
  constexpr int SLD = BT + 4;       // LDS row of the epilogue's staging (WT rows)
  constexpr int LDS_BYTES = 2 * LD::OPERAND > WT * SLD * 4 ? 2 * LD::OPERAND : WT * SLD * 4;
  __shared__ __attribute__((aligned(16))) char lds_raw[LDS_BYTES];
  float *const lds = reinterpret_cast<float *>(lds_raw);
  if (p.skip && p.skip[(int64_t)blockIdx.z * p.sSkip] != 0u) return;

  // One tile per workgroup; PERSIST: a loop over tiles when the grid was
  // capped (the caller limited the compute units this product may hold).
  for (int tile = blockIdx.x;;) {
  int tm, tn;
  tile_coords<MODE>(p, tile, tm, tn);
  const int64_t bz = blockIdx.z;
  const float *A = p.A + bz * p.sA;
  const float *B = p.B + bz * p.sB;
  const int m0 = tm * BT, n0 = tn * BT;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int xl = lane & 31, h = lane >> 5;

  // op(A) rows are x = i: k-contiguous when TA == 0.  op(B) columns are x = j:
  // k-contiguous when TB == 1.
  SlabLoader<BT, TA == 0, LOADS> la[AHEAD];
  SlabLoader<BT, TB == 1, LOADS> lb[AHEAD];

  v16f acc[NBLK][NBLK];
#pragma unroll
  for (int i = 0; i < NBLK; ++i)
#pragma unroll
    for (int j = 0; j < NBLK; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  char *const sa = lds_raw, *const sb = lds_raw + LD::OPERAND;
  const int kbeg = blockIdx.y * p.kslice;
  const int kend = min(p.K, kbeg + p.kslice);
  const int nk = (kend - kbeg + BK - 1) / BK;
#pragma unroll
  for (int u = 0; u < AHEAD; ++u)
    if (u < nk) {
      la[u].load(A, p.lda, m0, kbeg + u * BK, p.M, kend, tid);
      lb[u].load(B, p.ldb, n0, kbeg + u * BK, p.N, kend, tid);
    }
  for (int kt0 = 0; kt0 < nk; kt0 += AHEAD) {
#pragma unroll
  for (int u = 0; u < AHEAD; ++u) {
    const int kt = kt0 + u;
    if (AHEAD > 1 && kt >= nk) break;
    const int k0 = kbeg + kt * BK;
    const int kvalid = min(BK, kend - k0);
    la[u].store(sa, tid, kvalid);
    lb[u].store(sb, tid, kvalid);
    __syncthreads();
    if (kt + AHEAD < nk) {
      la[u].load(A, p.lda, m0, k0 + AHEAD * BK, p.M, kend, tid);
      lb[u].load(B, p.ldb, n0, k0 + AHEAD * BK, p.N, kend, tid);
    }
    // block by block: the slab's sums from zero, then into the accumulators
    v8bf fa[2][3], fb[2][3];
    auto frag = [&](const char *base, int x, v8bf (&f)[2][3]) {
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int pl = 0; pl < 3; ++pl)
          f[q][pl] = __builtin_bit_cast(v8bf, *reinterpret_cast<const uint4 *>(
              base + pl * LD::PLANE + LD::unit(x, 2 * q + h)));
    };
    auto block = [&](v16f &c) {
      v16f t;
#pragma unroll
      for (int r = 0; r < 16; ++r) t[r] = 0.f;
      // the six products above 2^-27 of the largest, the small ones first
#pragma unroll
      for (int v = 0; v < 6; ++v) {
        constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
        for (int q = 0; q < 2; ++q)
          t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[q][pa[v]], fb[q][pb[v]], t, 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) c[r] += t[r];
    };
    frag(sa, wm * WT + xl, fa);
    frag(sb, wn * WT + xl, fb);
    block(acc[0][0]);
    if constexpr (NBLK == 2) {
      frag(sb, wn * WT + 32 + xl, fb);
      block(acc[0][1]);
      frag(sa, wm * WT + 32 + xl, fa);
      block(acc[1][1]);
      frag(sb, wn * WT + xl, fb);
      block(acc[1][0]);
    }
    __syncthreads();
  }
  }

  // A wave whose sums hold an infinity or a NaN (an infinite operand times a
  // zero part gives NaN here and not in fp32; operands from 2^111 and sums
  // from 2^96 on overflow by their scale) takes its sums again on the fp32
  // matrix instructions, straight from memory (4096^3 of NaN: 1.9-2.2 ms, 62
  // to 72 TFLOP/s); the others are scaled back.
  {
    uint32_t mx = 0u;
#pragma unroll
    for (int i = 0; i < NBLK; ++i)
#pragma unroll
      for (int j = 0; j < NBLK; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          mx = max(mx, __float_as_uint(acc[i][j][r]) & 0x7fffffffu);
          acc[i][j][r] *= UNSCALE;
        }
    if (__any(mx >= 0x7f800000u)) {
#pragma unroll
      for (int i = 0; i < NBLK; ++i)
#pragma unroll
        for (int j = 0; j < NBLK; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
      // Groups of 8 k: lane half h takes 4 consecutive ones, the next group
      // is loaded while one is multiplied (not in the tile loop, whose own
      // registers leave no room).
      constexpr int BUFS = PERSIST ? 1 : 2;
      const float *pa[NBLK], *pb[NBLK];
#pragma unroll
      for (int i = 0; i < NBLK; ++i) {
        const int64_t xa = min(m0 + wm * WT + 32 * i + xl, p.M - 1), k4 = kbeg + 4 * h;
        const int64_t xb = min(n0 + wn * WT + 32 * i + xl, p.N - 1);
        pa[i] = A + (TA == 0 ? xa * p.lda + k4 : k4 * p.lda + xa);
        pb[i] = B + (TB == 1 ? xb * p.ldb + k4 : k4 * p.ldb + xb);
      }
      float ea[BUFS][NBLK][4], eb[BUFS][NBLK][4];
      auto fetch = [&](int f, int valid) {   // valid: k-values of this lane's four
#pragma unroll
        for (int i = 0; i < NBLK; ++i) {
          exact_operand<TA == 0>(pa[i], p.lda, valid, ea[f][i]);
          exact_operand<TB == 1>(pb[i], p.ldb, valid, eb[f][i]);
        }
      };
      auto multiply = [&](int f) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int i = 0; i < NBLK; ++i)
#pragma unroll
            for (int j = 0; j < NBLK; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(ea[f][i][u], eb[f][j][u], acc[i][j],
                                                              0, 0, 0);
      };
      const int groups = (kend - kbeg + 7) / 8;
      auto valid = [&](int g) { return kend - kbeg - 8 * g - 4 * h; };
      if constexpr (BUFS == 1) {
#pragma unroll 1
        for (int g = 0; g < groups; ++g) {
          fetch(0, valid(g));
          multiply(0);
        }
      } else {
        fetch(0, valid(0));
#pragma unroll 1
        for (int g = 0; g < groups; g += 2) {
          if (g + 1 < groups) fetch(1, valid(g + 1));
          multiply(0);
          if (g + 2 < groups) fetch(0, valid(g + 2));
          if (g + 1 < groups) multiply(1);
        }
      }
    }
  }

  // Epilogue.  Accumulator register r of block (i, j) holds
  // C[row0 + 8*(r/4) + 4*h + r%4][col0 + xl].
  float *C = p.C + bz * p.sC;
  const float *Dm = p.D + bz * p.sD;
  float *P = p.part ? p.part + (bz * gridDim.y + blockIdx.y) * (int64_t)p.M * p.N : nullptr;
  float *V = (MODE == MODE_ADAM) ? p.V + bz * p.sC : nullptr;
  float *Nout = (MODE == MODE_ADAM) ? p.Nout + bz * p.sC : nullptr;
  bool staged = false;
  constexpr int NQ = WT * BT / 4 / NTHREADS;   // float4 of a half per thread
  constexpr int QG = NQ < 4 ? NQ : 4;
  if constexpr (MODE == MODE_SYRK) {
   if (!P && ((reinterpret_cast<uintptr_t>(C) | reinterpret_cast<uintptr_t>(Dm)) & 15u) == 0 &&
       ((p.ldc | p.ldd) & 3) == 0) {
    staged = true;
    // One triangle, mirrored, through LDS in two halves of WT rows: the
    // lower part (row >= col) is written as beta C + alpha acc with 16-byte
    // reads and writes, the final values go back to LDS, and the mirror is
    // written from the transposed half, again 16 bytes per lane (scattered
    // 4-byte mirror stores, and a read of C after each store, otherwise).
    float *stage = lds;
    const bool read_back = p.beta != 0.f;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      __syncthreads();
      if (wm == half) {
#pragma unroll
        for (int i = 0; i < NBLK; ++i)
#pragma unroll
          for (int j = 0; j < NBLK; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
              stage[(i * 32 + 8 * (r >> 2) + 4 * h + (r & 3)) * SLD + wn * WT + j * 32 + xl] =
                  acc[i][j][r];
      }
      __syncthreads();
#pragma unroll
      for (int g4 = 0; g4 < NQ / QG; ++g4) {   // groups of 4 (registers of the main loop)
        float4 cv[QG];
#pragma unroll
        for (int qq = 0; qq < QG; ++qq) {
          const int q = QG * g4 + qq;
          const int e = tid + NTHREADS * q, lrow = e / (BT / 4), c4 = (e % (BT / 4)) * 4;
          const int row = m0 + half * WT + lrow, col = n0 + c4;
          cv[qq] = make_float4(0.f, 0.f, 0.f, 0.f);
          // only the lower triangle is read (a float4 with col <= row holds at
          // least one element of it; the others are masked)
          if (read_back && row < p.M && col <= row && col < p.N) {
            const float *src = Dm + (int64_t)row * p.ldd + col;
            if (col + 3 < p.N && col + 3 <= row) {
              cv[qq] = *reinterpret_cast<const float4 *>(src);
            } else {
              cv[qq].x = src[0];
              if (col + 1 < p.N && col + 1 <= row) cv[qq].y = src[1];
              if (col + 2 < p.N && col + 2 <= row) cv[qq].z = src[2];
              if (col + 3 < p.N && col + 3 <= row) cv[qq].w = src[3];
            }
          }
        }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int qq = 0; qq < QG; ++qq) {
          const int q = QG * g4 + qq;
          const int e = tid + NTHREADS * q, lrow = e / (BT / 4), c4 = (e % (BT / 4)) * 4;
          const int row = m0 + half * WT + lrow, col = n0 + c4;
          float *sp = stage + lrow * SLD + c4;
          const float4 a = *reinterpret_cast<const float4 *>(sp);
          float4 v;
          v.x = p.alpha * a.x + (read_back ? p.beta * cv[qq].x : 0.f);
          v.y = p.alpha * a.y + (read_back ? p.beta * cv[qq].y : 0.f);
          v.z = p.alpha * a.z + (read_back ? p.beta * cv[qq].z : 0.f);
          v.w = p.alpha * a.w + (read_back ? p.beta * cv[qq].w : 0.f);
          *reinterpret_cast<float4 *>(sp) = v;   // final values for the mirror
          if (row >= p.M || col > row || col >= p.N) continue;
          float *dst = C + (int64_t)row * p.ldc + col;
          if (col + 3 < p.N && col + 3 <= row) {
            *reinterpret_cast<float4 *>(dst) = v;
          } else {
            dst[0] = v.x;
            if (col + 1 < p.N && col + 1 <= row) dst[1] = v.y;
            if (col + 2 < p.N && col + 2 <= row) dst[2] = v.z;
            if (col + 3 < p.N && col + 3 <= row) dst[3] = v.w;
          }
        }
        asm volatile("" ::: "memory");
      }
      __syncthreads();
      // mirror: C[col][row] for row > col; thread -> (lc = output row within
      // the tile's columns, 4 consecutive rows of this half as output columns)
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int e = tid + NTHREADS * q, lc = e / (WT / 4), r4 = (e % (WT / 4)) * 4;
        const int orow = n0 + lc, ocol = m0 + half * WT + r4;   // C[orow][ocol] = value(ocol, orow)
        if (orow >= p.N || ocol >= p.M) continue;
        float4 v;
        v.x = stage[(r4 + 0) * SLD + lc];
        v.y = stage[(r4 + 1) * SLD + lc];
        v.z = stage[(r4 + 2) * SLD + lc];
        v.w = stage[(r4 + 3) * SLD + lc];
        float *dst = C + (int64_t)orow * p.ldc + ocol;
        // element (ocol + u, orow) of the lower triangle mirrors to here when ocol + u > orow
        if (ocol > orow && ocol + 3 < p.M) {
          *reinterpret_cast<float4 *>(dst) = v;
        } else {
          if (ocol > orow) dst[0] = v.x;
          if (ocol + 1 > orow && ocol + 1 < p.M) dst[1] = v.y;
          if (ocol + 2 > orow && ocol + 2 < p.M) dst[2] = v.z;
          if (ocol + 3 > orow && ocol + 3 < p.M) dst[3] = v.w;
        }
      }
    }
    if constexpr (PERSIST) __syncthreads();
   }
  }
  if constexpr (MODE == MODE_GENERAL) {
   if (!P && ((reinterpret_cast<uintptr_t>(C) | reinterpret_cast<uintptr_t>(Dm)) & 15u) == 0 &&
       ((p.ldc | p.ldd) & 3) == 0) {
    staged = true;
    // Rank-k updates are bound by their pass over C, so the tile goes
    // through LDS (free after the K loop) in two halves of WT rows and C is
    // read and written 16 bytes per lane, all reads of a thread before its
    // stores.
    float *stage = lds;
    const bool read_back = p.beta != 0.f;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      __syncthreads();
      if (wm == half) {
#pragma unroll
        for (int i = 0; i < NBLK; ++i)
#pragma unroll
          for (int j = 0; j < NBLK; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
              stage[(i * 32 + 8 * (r >> 2) + 4 * h + (r & 3)) * SLD + wn * WT + j * 32 + xl] =
                  acc[i][j][r];
      }
      __syncthreads();
      float4 cv[NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int e = tid + NTHREADS * q, lrow = e / (BT / 4), c4 = (e % (BT / 4)) * 4;
        const int row = m0 + half * WT + lrow, col = n0 + c4;
        cv[q] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (read_back && row < p.M) {
          const float *src = Dm + (int64_t)row * p.ldd + col;
          if (col + 3 < p.N) {
            cv[q] = *reinterpret_cast<const float4 *>(src);
          } else {
            if (col < p.N) cv[q].x = src[0];
            if (col + 1 < p.N) cv[q].y = src[1];
            if (col + 2 < p.N) cv[q].z = src[2];
          }
        }
      }
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int e = tid + NTHREADS * q, lrow = e / (BT / 4), c4 = (e % (BT / 4)) * 4;
        const int row = m0 + half * WT + lrow, col = n0 + c4;
        if (row >= p.M) continue;
        const float4 a = *reinterpret_cast<const float4 *>(stage + lrow * SLD + c4);
        float4 v;
        v.x = p.alpha * a.x + (read_back ? p.beta * cv[q].x : 0.f);
        v.y = p.alpha * a.y + (read_back ? p.beta * cv[q].y : 0.f);
        v.z = p.alpha * a.z + (read_back ? p.beta * cv[q].z : 0.f);
        v.w = p.alpha * a.w + (read_back ? p.beta * cv[q].w : 0.f);
        float *dst = C + (int64_t)row * p.ldc + col;
        if (col + 3 < p.N) {
          *reinterpret_cast<float4 *>(dst) = v;
        } else {
          if (col < p.N) dst[0] = v.x;
          if (col + 1 < p.N) dst[1] = v.y;
          if (col + 2 < p.N) dst[2] = v.z;
        }
      }
    }
    // a persistent launch's next tile writes the same LDS
    if constexpr (PERSIST) __syncthreads();
   }
  }
  if (staged) {
    // done
  } else {
#pragma unroll
    for (int i = 0; i < NBLK; ++i)
#pragma unroll
      for (int j = 0; j < NBLK; ++j) {
        const int col = n0 + wn * WT + j * 32 + xl;
        // C = alpha acc + beta C: the 16 values of C of this block are read
        // before its stores (one memory latency per block instead of one per
        // element); the empty asm keeps the compiler from hoisting the reads
        // of later blocks, whose registers would cost the main loop a wave
        // per SIMD.
        float cv[16];
        if (MODE == MODE_GENERAL && !P) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int row = m0 + wm * WT + i * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
            cv[r] = (p.beta != 0.f && row < p.M && col < p.N) ? Dm[(int64_t)row * p.ldd + col] : 0.f;
          }
        }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = m0 + wm * WT + i * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
          if (row >= p.M || col >= p.N) continue;
          const int64_t off = (int64_t)row * p.ldc + col;
          if (MODE != MODE_ADAM && P) {
            P[(int64_t)row * p.N + col] = acc[i][j][r];
          } else if (MODE == MODE_GENERAL) {
            float v = p.alpha * acc[i][j][r];
            if (p.beta != 0.f) v += p.beta * cv[r];
            C[off] = v;
          } else if (MODE == MODE_SYRK) {
            if (row < col) continue;  // the mirror of (col,row) is written by its owner
            const float v = (p.beta != 0.f ? p.beta * Dm[(int64_t)row * p.ldd + col] : 0.f) + p.alpha * acc[i][j][r];
            C[off] = v;
            if (row != col) C[(int64_t)col * p.ldc + row] = v;
          } else if ((r & 1) == 0) {
            // rows 2i, 2i+1 of the interleaved operand are G' and M' of
            // output row i; they sit in registers r, r+1 of the same lane
            const float g = acc[i][j][r];
            const float mm = acc[i][j][r + 1];
            const int64_t o = (int64_t)(row >> 1) * p.ldc + col;
            const float v = p.b2 * V[o] + (1.f - p.b2) * g * g;
            V[o] = v;
            Nout[o] = (mm / p.c1) / (sqrtf(v / p.c2) + p.eps);
          }
        }
      }
  }
  if constexpr (!PERSIST) break;
  tile += gridDim.x;
  if (tile >= p.ntiles) break;
  }  // tile loop
}

// C = alpha * sum_s part[s] + beta * C, slices summed in index order.
__global__ __launch_bounds__(256) void splitk_reduce(const float *__restrict__ part, int S,
                                                     int M, int N, float *C, int64_t ldc,
                                                     int64_t sC, float alpha, float beta,
                                                     const unsigned *skip, int64_t sSkip) {
  const int64_t bz = blockIdx.y;
  if (skip && skip[bz * sSkip] != 0u) return;
  const int64_t mn = (int64_t)M * N;
  const float *pb = part + bz * S * mn;
  float *Cb = C + bz * sC;
  for (int64_t e = blockIdx.x * 256 + threadIdx.x; e < mn; e += (int64_t)gridDim.x * 256) {
    float acc = 0.f;
    for (int s = 0; s < S; ++s) acc += pb[s * mn + e];
    const int64_t row = e / N, col = e - row * N;
    float v = alpha * acc;
    if (beta != 0.f) v += beta * Cb[row * ldc + col];
    Cb[row * ldc + col] = v;
  }
}

// The same without beta for the lower triangle of a symmetric product: the
// sum of every element with row >= col goes to (row, col) and (col, row), by
// 32 x 32 blocks on or below the diagonal (the mirror through LDS).
__global__ __launch_bounds__(256) void splitk_reduce_syrk(const float *__restrict__ part, int S,
                                                          int N, float *C, int64_t ldc, int64_t sC,
                                                          float alpha) {
  __shared__ float tile[32][33];
  const int bi = blockIdx.y, bj = blockIdx.x;
  if (bj > bi) return;
  const int64_t bz = blockIdx.z, nn = (int64_t)N * N;
  const float *pb = part + bz * S * nn;
  float *Cb = C + bz * sC;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int row = 32 * bi + ty + 8 * q, col = 32 * bj + tx;
    float v = 0.f;
    if (row < N && col <= row) {
      for (int s = 0; s < S; ++s) v += pb[s * nn + (int64_t)row * N + col];
      v *= alpha;
      Cb[(int64_t)row * ldc + col] = v;
    }
    tile[ty + 8 * q][tx] = v;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int col = 32 * bj + ty + 8 * q, row = 32 * bi + tx;
    if (row < N && row > col) Cb[(int64_t)col * ldc + row] = tile[tx][ty + 8 * q];
  }
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

template <int BT, int MODE, int TAG, bool PERSIST>
hipError_t launch_layout(int code, bool aligned, dim3 grid, hipStream_t s, const KParams &kp) {
  const dim3 block(NTHREADS);
#define SOAP_LAUNCH(TA, TB)                                                                      \
  do {                                                                                           \
    if (aligned)                                                                                 \
      hipLaunchKernelGGL((gemm_f32_split<BT, TA, TB, V_ALIGNED, MODE, TAG, PERSIST>), grid, block, 0, \
                         s, kp);                                                                 \
    else                                                                                         \
      hipLaunchKernelGGL((gemm_f32_split<BT, TA, TB, V_ANY, MODE, TAG, PERSIST>), grid, block, 0, s,  \
                         kp);                                                                    \
  } while (0)
  if constexpr (MODE == MODE_GENERAL && TAG == 0) {
    switch (code) {
      case 0: SOAP_LAUNCH(0, 0); break;
      case 1: SOAP_LAUNCH(0, 1); break;
      case 2: SOAP_LAUNCH(1, 0); break;
      default: SOAP_LAUNCH(1, 1); break;
    }
  } else if constexpr (MODE == MODE_GENERAL) {   // the power products, by their own symbols
    if (code != 2) return hipErrorInvalidValue;
    SOAP_LAUNCH(1, 0);
  } else if constexpr (MODE == MODE_SYRK) {      // X X^T and X^T X
    if (code == 1) SOAP_LAUNCH(0, 1);
    else if (code == 2) SOAP_LAUNCH(1, 0);
    else return hipErrorInvalidValue;
  } else {
    if (code == 0) SOAP_LAUNCH(0, 0);
    else if (code == 1) SOAP_LAUNCH(0, 1);
    else return hipErrorInvalidValue;
  }
#undef SOAP_LAUNCH
  return hipGetLastError();
}

// Products of at most this many 128-tiles (split slices and batch included)
// take 64-tiles: below it compute units stay idle with 128-tiles and each
// tile's chain of slabs is what takes the time (128 x 128 x 128: 16 -> 9 us;
// 517 x 517 x 1283, 25 tiles: 162 -> 66; 1536^3, 144 tiles: 114 -> 85; a
// triangle of 136 tiles, K = 2048: 138 -> 100); from 256 tiles on the larger
// tile's fewer bytes per flop win (2048^3: 155 us with 128-tiles, 172 with
// 64-tiles; 3072 x 2048 x 2048, 384 tiles: 187 and 231).
constexpr int64_t SMALL_MAX_TILES = 192;

void set_tiles(KParams &kp, int bt, bool triangle) {
  kp.tiles_m = (kp.M + bt - 1) / bt;
  kp.tiles_n = (kp.N + bt - 1) / bt;
  kp.ntiles = triangle ? kp.tiles_m * (kp.tiles_m + 1) / 2 : kp.tiles_m * kp.tiles_n;
}

template <int MODE>
hipError_t dispatch(const GemmDesc &d, KParams &kp, hipStream_t s, bool aligned) {
  hipError_t err;
  const int S = (MODE != MODE_ADAM && d.splitk > 1 && d.part) ? d.splitk : 1;
  // A cap counts every workgroup (split slices and batch included); the
  // tile dimension stays a multiple of 8 for XCD locality.
  const int64_t per_tile = (int64_t)S * d.batch;
  const bool capped = (MODE == MODE_GENERAL || MODE == MODE_SYRK) && d.max_wg > 0 &&
                      (int64_t)kp.ntiles * per_tile > d.max_wg;
  const int code = d.trans_a * 2 + d.trans_b;
  if (d.tile == SMALL || (d.tile == 0 && kp.ntiles * per_tile <= SMALL_MAX_TILES && d.max_wg == 0)) {
    set_tiles(kp, SMALL, MODE == MODE_SYRK);
    err = launch_layout<SMALL, MODE, 0, false>(code, aligned, dim3(kp.ntiles, S, (unsigned)d.batch),
                                               s, kp);
  } else {
    const int wgs = capped ? (int)std::max<int64_t>(8, (d.max_wg / per_tile) & ~int64_t(7)) : kp.ntiles;
    const dim3 grid(std::min(wgs, kp.ntiles), S, (unsigned)d.batch);
    if constexpr (MODE != MODE_ADAM) {
      if (capped) err = launch_layout<BIG, MODE, 0, true>(code, aligned, grid, s, kp);
      else if (MODE == MODE_GENERAL && d.tag == 1 && code == 2)
        err = launch_layout<BIG, MODE_GENERAL, 1, false>(code, aligned, grid, s, kp);
      else if (MODE == MODE_GENERAL && d.tag == 2 && code == 2)
        err = launch_layout<BIG, MODE_GENERAL, 2, false>(code, aligned, grid, s, kp);
      else err = launch_layout<BIG, MODE, 0, false>(code, aligned, grid, s, kp);
    } else {
      err = launch_layout<BIG, MODE, 0, false>(code, aligned, grid, s, kp);
    }
  }
  if (err != hipSuccess || S == 1 || d.partials_only) return err;
  if (MODE == MODE_SYRK) {
    const unsigned g = (unsigned)((d.N + 31) / 32);
    hipLaunchKernelGGL(splitk_reduce_syrk, dim3(g, g, (unsigned)d.batch), dim3(256), 0, s, kp.part,
                       S, kp.N, kp.C, kp.ldc, kp.sC, d.alpha);
    return hipGetLastError();
  }
  int64_t mn = d.M * d.N;
  unsigned gx = (unsigned)std::min<int64_t>((mn + 255) / 256, 2048);
  hipLaunchKernelGGL(splitk_reduce, dim3(gx, (unsigned)d.batch), dim3(256), 0, s, kp.part, S,
                     kp.M, kp.N, d.C, d.ldc, d.sC, d.alpha, d.beta, kp.skip, kp.sSkip);
  return hipGetLastError();
}

KParams make_params(const GemmDesc &d, bool triangle = false) {
  KParams kp{};
  kp.M = (int)d.M; kp.N = (int)d.N; kp.K = (int)d.K;
  kp.A = d.A; kp.lda = d.lda; kp.sA = d.sA;
  kp.B = d.B; kp.ldb = d.ldb; kp.sB = d.sB;
  kp.C = d.C; kp.ldc = d.ldc; kp.sC = d.sC;
  kp.alpha = d.alpha; kp.beta = d.beta;
  kp.D = d.D ? d.D : d.C;
  kp.ldd = d.D ? d.ldd : d.ldc;
  kp.sD = d.D ? d.sD : d.sC;
  set_tiles(kp, BIG, triangle);
  kp.kslice = (int)d.K;
  kp.part = nullptr;
  kp.skip = d.skip;
  kp.sSkip = d.sSkip;
  if (d.splitk > 1 && d.part) {
    const int64_t per = (d.K + d.splitk - 1) / d.splitk;
    kp.kslice = (int)(((per + BK - 1) / BK) * BK);
    kp.part = d.part;
  }
  return kp;
}

// V_ALIGNED's preconditions: a k-contiguous operand is read 16 bytes at a time
// along k (k extent, leading dimension, batch stride multiples of 4 floats,
// 16-byte aligned base); an x-contiguous operand 8 bytes along x (even x
// extent, leading dimension and batch stride, 8-byte aligned base).
bool aligned8(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 7u) == 0; }

bool aligned_loads(const GemmDesc &d) {
  bool ok = d.K > 0;
  if (d.trans_a == 0)
    ok = ok && d.K % 4 == 0 && d.lda % 4 == 0 && d.sA % 4 == 0 && aligned16(d.A);
  else
    ok = ok && d.M % 2 == 0 && d.lda % 2 == 0 && d.sA % 2 == 0 && aligned8(d.A);
  if (d.trans_b == 1)
    ok = ok && d.K % 4 == 0 && d.ldb % 4 == 0 && d.sB % 4 == 0 && aligned16(d.B);
  else
    ok = ok && d.N % 2 == 0 && d.ldb % 2 == 0 && d.sB % 2 == 0 && aligned8(d.B);
  return ok;
}

}  // namespace

int choose_splitk(int64_t M, int64_t N, int64_t K, int64_t batch, int max_split) {
  const int64_t tiles = ((M + BIG - 1) / BIG) * ((N + BIG - 1) / BIG) * batch;
  if (tiles <= 0) return 1;   // an empty product: nothing to split
  int64_t s = (512 + tiles - 1) / tiles;
  const int64_t kcap = K / 512;     // keep at least 512 of K per slice
  if (s > kcap) s = kcap;
  if (s > max_split) s = max_split;
  if (s < 1) s = 1;
  return (int)s;
}

// A triangle of at most 256 64-tiles (over the batch) is split, as 64-tiles,
// into about two workgroups per CU of at least 256 of K each (517^2, K = 1283,
// 45 tiles: 80 -> 27 + 8 us); one of more, but of few 128-tiles (whose compute units would hold one tile or
// none), into 128-tiles of at least 1024 of K each where two slices or more
// fit two workgroups per CU (2048^2, K = 8192, 136 of them: the Muon step of
// 2048 x 8192 13.0 -> 11.6 ms).
SyrkSplit choose_syrk_split(int64_t d, int64_t K, int64_t batch) {
  const int64_t t1 = (d + SMALL - 1) / SMALL, n1 = t1 * (t1 + 1) / 2 * batch;
  const int64_t t2 = (d + BIG - 1) / BIG, n2 = t2 * (t2 + 1) / 2 * batch;
  if (n1 <= 0) return {1, 0};
  int64_t s = 1;
  if (n1 <= 256) s = std::min<int64_t>({8, 512 / n1, K / 256});
  else if (n2 * 2 > SMALL_MAX_TILES) s = std::min<int64_t>({8, 512 / n2, K / 1024});
  if (s <= 1) return {1, 0};
  return {(int)s, n1 <= 256 ? SMALL : BIG};
}

hipError_t launch_gemm(const GemmDesc &d, hipStream_t s) {
  if (d.M <= 0 || d.N <= 0 || d.batch <= 0) return hipSuccess;
  if (d.D && d.splitk > 1) return hipErrorInvalidValue;
  KParams kp = make_params(d);
  return dispatch<MODE_GENERAL>(d, kp, s, aligned_loads(d));
}

hipError_t launch_syrk_ema(const GemmDesc &d, hipStream_t s) {
  if (d.M <= 0 || d.batch <= 0) return hipSuccess;
  if (d.splitk > 1 && (d.D || d.beta != 0.f)) return hipErrorInvalidValue;
  KParams kp = make_params(d, true);
  return dispatch<MODE_SYRK>(d, kp, s, aligned_loads(d));
}

hipError_t launch_gemm_adam(const GemmDesc &d, const AdamEpi &e, hipStream_t s) {
  if (d.M <= 0 || d.N <= 0 || d.batch <= 0) return hipSuccess;
  if (d.M % 2 != 0 || d.trans_a != 0) return hipErrorInvalidValue;
  KParams kp = make_params(d);
  kp.V = e.V;
  kp.Nout = e.Nout;
  kp.b2 = e.b2; kp.c1 = e.c1; kp.c2 = e.c2; kp.eps = e.eps;
  return dispatch<MODE_ADAM>(d, kp, s, aligned_loads(d));
}

}  // namespace soap

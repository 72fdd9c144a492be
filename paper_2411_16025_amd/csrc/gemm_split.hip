// fp32 products on the bf16 matrix cores: every operand is the exact sum of
// three bf16 numbers, and six of the nine products of the parts are added in
// fp32.
//
// Why: v_mfma_f32_32x32x16_bf16 does 16 times the work of the fp32 matrix
// instruction per cycle (2.07 PFLOP/s against 0.15 in a register-only loop), so six
// of them still give 345 TFLOP/s of fp32 products.
//
// Precision. An fp32 number has 24 significant bits; h = bf16(x), m =
// bf16(x - h), l = bf16(x - h - m), each rounded to nearest even, hold 8 of
// them each, and both differences are exact, so h + m + l = x. With |m| <=
// 2^-8 |h| and |l| <= 2^-17 |h| the products left out (m l, l m, l l) are below
// 2^-24 of h h by no more than a 2^-10th, an fp32 rounding where the operands
// are the worst ones (1.0038834 squared) and far below it on average. The six others are
// exact in the matrix core and are added to the fp32 accumulator sixteen at a time,
// the small ones first. Against 64 bits, normal values, K = 100 / 256 / 516:
// 1.5e-7 / 2.4e-7 / 3.5e-7 here, 1.8e-7 / 2.9e-7 / 4.1e-7 with
// v_mfma_f32_16x16x4_f32; all operands positive 1.2e-7 / 1.9e-7 / 2.7e-7 and 1.1e-7
// / 1.7e-7 / 2.5e-7; all operands 1.0038834, K = 16 / 256 / 1024, 5.9e-8 / 1.8e-7 /
// 1.8e-7 and 5.9e-8 / 5.9e-8 / 1.5e-5.
//
// Small operands. The parts of an fp32 number are multiples of 2^-149, its
// smallest step, but a bf16 part below 2^-126 counts as 0 in the matrix core. So
// both operands are taken times 2^24 (with the signs below, in the same
// multiplication), which makes every part 0 or at least 2^-125, and the sums
// times 2^-48. Operands from 2^104 on, and sums from 2^80, then leave the range
// and take the route of the infinities. (Not scaled, operands about 2^-118 lost m's
// low bits and products were off by 8.8e-6, about 2^-124 by 5.6e-4.)
//
// The matrix core rounds the aligned products towards minus infinity some 8 bits
// below the sum's last bit. That bias is far below a rounding, but it has the same
// sign in every sum, and sums over millions of such results, or chunks of
// them, would keep it (512 x 256 x 2.45M in 19,136-row chunks: 1.1e-5). So half
// of the sums are formed of negated products and negated at the end: odd rows
// of A and odd columns of B where A is tall (a checkerboard in C), every other
// chunk in A^T B; the bias then cancels in any sum over rows, columns or chunks.
//
// Infinities, NaN and operands that round up to infinity give a NaN in the
// sums of the parts, whatever the fp32 product would be; a wavefront whose
// tile holds a sum that is not finite therefore computes that tile again on the
// fp32 matrix instruction.
//
// What bounds them: random operands hold the chip's bf16 matrix cores at about 1.1
// PFLOP/s (an 8192^3 library product reaches 1.12), 185 TFLOP/s of fp32
// products. 2,449,029 x 256 x 516: 3.51 ms, 184 TFLOP/s (5.57 ms on the fp32
// instruction); x 512 x 256 transposed weights 3.57 ms (6.21); A^T B 512 x 256
// 3.57 ms (5.44). Shallow products (K = 100: 1.11 ms, 1.61 before) are bound by
// writing C, which a tile cannot overlap with its own products.

#include <algorithm>

#include "common.h"

namespace gcn {
namespace {

typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));  // 4-byte aligned 16-byte load
typedef float f16 __attribute__((ext_vector_type(16)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;  // four wavefronts
constexpr int kKs = 16;        // K of one step: one matrix instruction deep
constexpr int kFrag = 1024;    // bytes of one 32 x 16 operand block of one part
constexpr float kUp = 0x1p24f, kDown = 0x1p-48f;  // of an operand, of a sum

// The parts of two neighbouring values, each pair packed in 32 bits.
__device__ inline void split2(float x0, float x1, uint32_t& h, uint32_t& m, uint32_t& l) {
  const f2 x = {x0, x1};
  h = __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf2));
  const f2 r = {x0 - __uint_as_float(h << 16), x1 - __uint_as_float(h & 0xFFFF0000u)};
  m = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, bf2));
  const f2 q = {r.x - __uint_as_float(m << 16), r.y - __uint_as_float(m & 0xFFFF0000u)};
  l = __builtin_bit_cast(uint32_t, __builtin_convertvector(q, bf2));
}

__device__ inline void split8(const float* x, u4* out) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint32_t h, m, l;
    split2(x[2 * j], x[2 * j + 1], h, m, l);
    out[0][j] = h;
    out[1][j] = m;
    out[2][j] = l;
  }
}

// One step of a wavefront's RBW x NBW blocks, operands from LDS: the six
// products of each block, the smallest first; the B parts of a column block
// are read while the one before it is multiplied.
template <int RBW, int NBW, int NBUF = 2>
__device__ inline void mul_step(const bf8* as, const bf8* bs, f16 (*acc)[NBW]) {
  constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
  bf8 a[RBW][3], b[NBUF][3];
#pragma unroll
  for (int i = 0; i < RBW; ++i)
#pragma unroll
    for (int s = 0; s < 3; ++s) a[i][s] = as[(i * 3 + s) * 64];
  if (NBUF == 2) {
#pragma unroll
    for (int s = 0; s < 3; ++s) b[0][s] = bs[s * 64];
  }
#pragma unroll
  for (int j = 0; j < NBW; ++j) {
    if (NBUF == 1 || j + 1 < NBW) {
      const int jn = NBUF == 1 ? j : j + 1;
#pragma unroll
      for (int s = 0; s < 3; ++s) b[jn % NBUF][s] = bs[(jn * 3 + s) * 64];
    }
#pragma unroll
    for (int p = 0; p < 6; ++p)
#pragma unroll
      for (int i = 0; i < RBW; ++i)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][pa[p]], b[j % NBUF][pb[p]],
                                                            acc[i][j], 0, 0, 0);
  }
}

// The order of a step's instructions: the LDS reads of the first blocks, then
// products with the LDS reads of the next column block and the splitting of
// the next step's operands between them, the LDS stores last.
template <int RBW, int NBW>
__device__ inline void pipeline() {
  __builtin_amdgcn_sched_group_barrier(0x100, 3 * RBW + 3, 0);
#pragma unroll
  for (int j = 0; j < NBW; ++j) {
    if (j + 1 < NBW) __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
#pragma unroll
    for (int p = 0; p < 6 * RBW; ++p) {
      __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x2, 3, 0);
    }
  }
}

// Operand layout of the instruction: lane l holds A[l % 32][8 (l / 32) + j]
// and B[8 (l / 32) + j][l % 32], j = 0 .. 7; result element e of lane l is
// C[(e % 4) + 8 (e / 4) + 4 (l / 32)][l % 32].
__device__ inline int result_row(int e, int lane) {
  return (e & 3) + 8 * (e >> 2) + 4 * (lane >> 5);
}

// ---- C = A B, A tall -------------------------------------------------------------

struct TallArgs {
  int64_t M;
  int N, K;
  const float* A;
  int64_t lda;
  const float* B;
  int64_t ldb;
  int col_tiles;
  float* C;
  int64_t ldc;
  const float* mask;
  int64_t ldm;
  bool relu;
};

__device__ inline float finish(const TallArgs& a, float v, int64_t gm, int64_t gn) {
  if (a.mask && !(a.mask[gm * a.ldm + gn] > 0.f)) v = 0.f;
  return a.relu ? fmaxf(v, 0.f) : v;
}

// A uniform pointer plus the lane's 32-bit offset in bytes (one scalar and one
// vector register of address).
__device__ inline const float* at_bytes(const float* base, uint32_t off) {
  return reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + off);
}

// Whether a sum of the wavefront is not finite.
template <int RBW, int NBW>
__device__ inline bool not_finite(const f16 (*acc)[NBW]) {
  float bad = 0.f;  // NaN once a sum is not finite
#pragma unroll
  for (int i = 0; i < RBW; ++i)
#pragma unroll
    for (int j = 0; j < NBW; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) bad = __builtin_fmaf(acc[i][j][e], 0.f, bad);
  return __any(bad != bad);
}

// The wavefront's sums over [k0, k1) again on the fp32 matrix instruction, the
// operands from global memory. Lane l holds A[l % 32][k] and B[k][l % 32], k the
// same for both in each half of the wavefront: four k of each half are fetched
// at a time by load(k, a, b), zeros from k1 on. (Element by element, a product of
// 32,768 x 256 x 516 whose operands are NaN took 8.8 ms; 0.32 here, 0.09 with
// finite ones.)
template <int RBW, int NBW, class Load>
__device__ inline void mul_again(int64_t k0, int64_t k1, Load load, f16 (*acc)[NBW]) {
#pragma unroll
  for (int i = 0; i < RBW; ++i)
#pragma unroll
    for (int j = 0; j < NBW; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
#pragma unroll 1
  for (int64_t k = k0; k < k1; k += 8) {
    float x[RBW][4], y[NBW][4];
    load(k + 4 * ((threadIdx.x >> 5) & 1), x, y);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < RBW; ++i)
#pragma unroll
        for (int j = 0; j < NBW; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[i][q], y[j][q], acc[i][j], 0, 0, 0);
  }
}

// WR x WC wavefronts, each with RBW x NBW blocks of 32 x 32 of C. A step
// covers 16 of K: the workgroup's rows of A and columns of B are loaded, split
// and laid out in LDS in operand order, and the next step's loads are in flight
// meanwhile (two LDS buffers, one barrier a step). B is split by every
// workgroup anew: laid out once by a kernel of its own it needed scratch, which a
// captured call and one without free memory cannot have. BT: B is stored N x K.
template <int WR, int WC, int RBW, int NBW, bool BT>
__global__ __launch_bounds__(64 * WR * WC, 2) void k_split_tall(TallArgs a) {
  constexpr int RB = WR * RBW, NB = WC * NBW;  // blocks of the workgroup's tile
  constexpr int ROWS = RB * 32;
  constexpr int NT = 64 * WR * WC, RP = NT / 4;  // threads; rows of A loaded at a time
  constexpr int AP = ROWS * 4 / NT;  // 16-byte pieces of A per thread
  // of B, 16-byte pieces like A's, or units of 8 rows (4 where those do not fill
  // the threads: 2.45M x 192 x 256: 1.60 ms instead of 1.67) of one column
  constexpr int BV = BT || (NB * 64 % NT != 0 && NB * 128 % NT == 0) ? 4 : 8;
  constexpr int BUNITS = NB * 512 / BV, BP = (BUNITS + NT - 1) / NT;
  constexpr bool BFULL = BUNITS % NT == 0;
  __shared__ __align__(16) char lds[2][(RB + NB) * 3 * kFrag];
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wr = w / WC, wc = w % WC;
  // column tiles of one row tile run on one XCD, one after the other, so that
  // the second finds its rows of A in that XCD's L2
  const int64_t xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
  const int ct = (int)(idx % a.col_tiles);
  const int64_t m0 = ((idx / a.col_tiles) * 8 + xcd) * ROWS;
  const int n0 = ct * NB * 32;
  if (m0 >= a.M) return;  // the whole workgroup

  // a thread's pieces of A: row t / 4 + RP p, k = 4 (t % 4) .. + 3
  const float* at = a.A + m0 * a.lda;
  uint32_t ao[AP];
#pragma unroll
  for (int p = 0; p < AP; ++p) {
    const int r = (t >> 2) + RP * p;
    ao[p] = 4 * ((uint32_t)(m0 + r < a.M ? r : (int)(a.M - 1 - m0)) * (uint32_t)a.lda + 4 * (t & 3));
  }
  const float sign = (t >> 2) & 1 ? -kUp : kUp;
  // of B: as of A, or unit u: block u / (512 / BV), column u % 32 of it,
  // k = BV (u / 32 % (16 / BV)) .. + BV - 1
  const int bk = BT ? 4 * (t & 3) : BV * ((t >> 5) & (16 / BV - 1));
  const float* bt = BT ? a.B + n0 * a.ldb : a.B + n0;
  uint32_t bo[BP];
#pragma unroll
  for (int p = 0; p < BP; ++p) {
    const int u = t + NT * p;
    const int c = BT ? (t >> 2) + RP * p : u / (512 / BV) * 32 + (u & 31);
    const uint32_t in = (uint32_t)(n0 + c < a.N ? c : a.N - 1 - n0);
    bo[p] = 4 * (BT ? in * (uint32_t)a.ldb + bk : in + (uint32_t)bk * (uint32_t)a.ldb);
  }
  const float bsign = BT ? sign : (t & 1 ? -kUp : kUp);
  // where the 16-byte pieces go: block row / 32, lane row % 32 + 32 (k / 8), half k / 4 % 2
  const int a_off = (t >> 7) * 3 * kFrag + ((t >> 2) & 31) * 16 + ((t >> 1) & 1) * 512 + (t & 1) * 8;

  const int steps = (a.K + kKs - 1) / kKs;
  f4u av[2][AP];  // A of the next step and of the one after it
  float bv[BP][BV];
  auto load_a = [&](f4u* v, int ks) {
    const int k0 = ks * kKs, k = k0 + 4 * (t & 3);
    if (k0 + kKs <= a.K) {
#pragma unroll
      for (int p = 0; p < AP; ++p) v[p] = *reinterpret_cast<const f4u*>(at_bytes(at + k0, ao[p]));
    } else {  // the last, partial step, and the steps past it (not used)
#pragma unroll
      for (int p = 0; p < AP; ++p)
#pragma unroll
        for (int j = 0; j < 4; ++j) v[p][j] = k + j < a.K ? at_bytes(at + k0, ao[p])[j] : 0.f;
    }
  };
  auto load_b = [&](int ks) {
    const int k0 = ks * kKs;
    const bool full = k0 + kKs <= a.K;  // else the last, partial step, or one past it
#pragma unroll
    for (int p = 0; p < BP; ++p) {
      if (!BFULL && t + p * NT >= BUNITS) continue;
      if constexpr (BT) {
        const float* q = at_bytes(bt + k0, bo[p]);
        if (full) {
          const f4u v = *reinterpret_cast<const f4u*>(q);
#pragma unroll
          for (int j = 0; j < 4; ++j) bv[p][j] = v[j];
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) bv[p][j] = k0 + bk + j < a.K ? q[j] : 0.f;
        }
      } else {
        const float* q = bt + (int64_t)k0 * a.ldb;
        if (full) {
#pragma unroll
          for (int j = 0; j < BV; ++j) bv[p][j] = *at_bytes(q + j * a.ldb, bo[p]);
        } else {
#pragma unroll
          for (int j = 0; j < BV; ++j)
            bv[p][j] = k0 + bk + j < a.K ? *at_bytes(q + j * a.ldb, bo[p]) : 0.f;
        }
      }
    }
  };
  auto store4 = [](char* q, float x0, float x1, float x2, float x3) {
    uint32_t h0, m0, l0, h1, m1, l1;
    split2(x0, x1, h0, m0, l0);
    split2(x2, x3, h1, m1, l1);
    *reinterpret_cast<u2*>(q) = u2{h0, h1};
    *reinterpret_cast<u2*>(q + kFrag) = u2{m0, m1};
    *reinterpret_cast<u2*>(q + 2 * kFrag) = u2{l0, l1};
  };
  auto store_a = [&](char* buf, const f4u* v) {
#pragma unroll
    for (int p = 0; p < AP; ++p)
      store4(buf + RP / 32 * p * 3 * kFrag + a_off, v[p][0] * sign, v[p][1] * sign, v[p][2] * sign,
             v[p][3] * sign);
  };
  auto store_b = [&](char* buf) {
    buf += RB * 3 * kFrag;
#pragma unroll
    for (int p = 0; p < BP; ++p) {
      if (!BFULL && t + p * NT >= BUNITS) continue;
      const int u = t + p * NT;
#pragma unroll
      for (int j = 0; j < BV; ++j) bv[p][j] *= bsign;
      if constexpr (BT) {
        store4(buf + RP / 32 * p * 3 * kFrag + a_off, bv[p][0], bv[p][1], bv[p][2], bv[p][3]);
      } else if constexpr (BV == 4) {
        const int r = (t >> 5) & 3;  // its quarter of the step
        store4(buf + (u >> 7) * 3 * kFrag + ((t & 31) + 32 * (r >> 1)) * 16 + (r & 1) * 8, bv[p][0],
               bv[p][1], bv[p][2], bv[p][3]);
      } else {
        u4 s[3];
        split8(bv[p], s);
        u4* q = reinterpret_cast<u4*>(buf) + (u >> 6) * 3 * 64 + (u & 63);
        q[0] = s[0];
        q[64] = s[1];
        q[128] = s[2];
      }
    }
  };

  f16 acc[RBW][NBW];
#pragma unroll
  for (int i = 0; i < RBW; ++i)
#pragma unroll
    for (int j = 0; j < NBW; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // step ks: B of the next step and A of the one after it are issued, the
  // blocks in LDS are multiplied, and A and B of the next step are stored
  auto step = [&](int ks, char* cur, char* next, const f4u* v, f4u* vload) {
    load_b(ks + 1);
    load_a(vload, ks + 2);
    const bf8* as = reinterpret_cast<const bf8*>(cur) + wr * RBW * 3 * 64 + lane;
    const bf8* bs = reinterpret_cast<const bf8*>(cur + RB * 3 * kFrag) + wc * NBW * 3 * 64 + lane;
    mul_step<RBW, NBW>(as, bs, acc);
    store_a(next, v);
    store_b(next);
    pipeline<RBW, NBW>();
    __syncthreads();
  };
  load_a(av[0], 0);
  load_b(0);
  load_a(av[1], 1);
  store_a(lds[0], av[0]);
  store_b(lds[0]);
  __syncthreads();
  int ks = 0;
  for (; ks + 1 < steps; ks += 2) {
    step(ks, lds[0], lds[1], av[1], av[0]);
    step(ks + 1, lds[1], lds[0], av[0], av[1]);
  }
  if (ks < steps) step(ks, lds[0], lds[1], av[1], av[0]);

  const int64_t wm = m0 + wr * RBW * 32;
  const int wn = n0 + wc * NBW * 32;
  // the signs and scale of even and odd rows in the lane's column (with 0 added
  // to the product: -0 becomes +0)
  float even = lane & 1 ? -kDown : kDown, odd = -even;
  if (not_finite<RBW, NBW>(acc)) {
    even = odd = 1.f;
    auto load = [&](int64_t k, float (*x)[4], float (*y)[4]) {
#pragma unroll
      for (int i = 0; i < RBW; ++i) {
        const int64_t m = wm + i * 32 + (lane & 31);
        const float* q = a.A + (m < a.M ? m : a.M - 1) * a.lda + k;
#pragma unroll
        for (int j = 0; j < 4; ++j) x[i][j] = k + j < a.K ? q[j] : 0.f;
      }
#pragma unroll
      for (int i = 0; i < NBW; ++i) {
        const int64_t n = wn + i * 32 + (lane & 31), c = n < a.N ? n : a.N - 1;
        const float* q = BT ? a.B + c * a.ldb + k : a.B + k * a.ldb + c;
#pragma unroll
        for (int j = 0; j < 4; ++j) y[i][j] = k + j < a.K ? q[BT ? j : j * a.ldb] : 0.f;
      }
    };
    mul_again<RBW, NBW>(0, a.K, load, acc);
  }
  if (wm + RBW * 32 <= a.M && wn + NBW * 32 <= a.N) {
    // the lane's part of an address once, the rest uniform
    const uint32_t lc = (uint32_t)(4 * (lane >> 5)) * (uint32_t)a.ldc + (lane & 31);
    const uint32_t lm = (uint32_t)(4 * (lane >> 5)) * (uint32_t)a.ldm + (lane & 31);
#pragma unroll
    for (int i = 0; i < RBW; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        float* c = a.C + (wm + i * 32 + result_row(e, 0)) * a.ldc + wn;
        const float* mk = a.mask + (wm + i * 32 + result_row(e, 0)) * a.ldm + wn;
#pragma unroll
        for (int j = 0; j < NBW; ++j) {
          float v = __builtin_fmaf(acc[i][j][e], e & 1 ? odd : even, 0.f);
          if (a.mask) v = mk[lm + j * 32] > 0.f ? v : 0.f;
          if (a.relu) v = fmaxf(v, 0.f);
          c[lc + j * 32] = v;
        }
      }
  } else {
#pragma unroll
    for (int i = 0; i < RBW; ++i)
#pragma unroll
      for (int j = 0; j < NBW; ++j) {
        const int gn = wn + j * 32 + (lane & 31);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int64_t gm = wm + i * 32 + result_row(e, lane);
          if (gm < a.M && gn < a.N)
            a.C[gm * a.ldc + gn] =
                finish(a, __builtin_fmaf(acc[i][j][e], e & 1 ? odd : even, 0.f), gm, gn);
        }
      }
  }
}

// ---- C = A^T B, K = rows in the millions ---------------------------------------------

struct TnArgs {
  int M, N;
  int64_t K, split, chunks;  // rows of a chunk (a multiple of 16), their number
  int64_t run, groups;       // chunks that a workgroup sums, groups of so many chunks
  const float* A;
  int64_t lda;
  const float* B;
  int64_t ldb;
  float* part;  // [groups][M][N]
  int m_tiles, n_tiles;
};

// The tile's columns of A and of B are loaded 8 rows per thread with 4-byte
// loads (32 lanes on neighbouring columns), which gives a thread the 8 k of
// one operand lane; they are split and stored to LDS as such, PF steps after
// their loads were issued (PF = 1 where the accumulators leave no registers for two).
// A is negated in every other chunk (see the head of this file). RUN: a workgroup
// takes several chunks, one after the other, and adds their sums to its partial
// C (without it the loop is gone, and with it the registers it costs).
template <int WR, int WC, int RBW, int NBW, int PF, bool RUN>
__global__ __launch_bounds__(64 * WR * WC, 2) void k_split_tn(TnArgs a) {
  constexpr int RB = WR * RBW, NB = WC * NBW, NT = 64 * WR * WC;
  constexpr int AU = (RB * 64 + NT - 1) / NT;  // (column, half step) units per thread
  constexpr int BU = (NB * 64 + NT - 1) / NT;
  __shared__ __align__(16) char lds[2][(RB + NB) * 3 * kFrag];
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wr = w / WC, wc = w % WC;
  // the tiles of a group run on one XCD, one after the other: they read the
  // same rows of A and B
  const int tiles = a.m_tiles * a.n_tiles;
  const int64_t idx = blockIdx.x >> 3;
  const int tile = (int)(idx % tiles);
  const int64_t group = idx / tiles * 8 + (blockIdx.x & 7);
  if (group >= a.groups) return;  // the whole workgroup
  const int m0 = (tile / a.n_tiles) * RB * 32, n0 = (tile % a.n_tiles) * NB * 32;

  // unit u of a block of columns: column (u / 64) * 32 + u % 32, half u / 32 % 2;
  // in operand order that is 16-byte slot u % 64 of block u / 64
  // (its address: a uniform row plus a 32-bit lane part)
  uint32_t ao[AU], bo[BU];
#pragma unroll
  for (int p = 0; p < AU; ++p) {
    const int u = t + p * NT, c = m0 + (u >> 6) * 32 + (u & 31);
    ao[p] = 4 * ((uint32_t)(8 * ((u >> 5) & 1)) * (uint32_t)a.lda + ((c < a.M ? c : a.M - 1) - m0));
  }
#pragma unroll
  for (int p = 0; p < BU; ++p) {
    const int u = t + p * NT, c = n0 + (u >> 6) * 32 + (u & 31);
    bo[p] = 4 * ((uint32_t)(8 * ((u >> 5) & 1)) * (uint32_t)a.ldb + ((c < a.N ? c : a.N - 1) - n0));
  }
  const int h8 = 8 * ((t >> 5) & 1);  // the half is the same for all of a thread's units

  auto sum_chunk = [&](int64_t chunk, bool add) {
    const int64_t kb = chunk * a.split;
    const int64_t ke = kb + a.split < a.K ? kb + a.split : a.K;
    const float sign = chunk & 1 ? -kUp : kUp;
    float down = chunk & 1 ? -kDown : kDown;
    struct Pieces {
      float a[AU][8], b[BU][8];
    } v[PF];
    auto load = [&](Pieces& v, int64_t k) {
      const float *ar = a.A + k * a.lda + m0, *br = a.B + k * a.ldb + n0;
      const bool full = k + kKs <= ke;  // else the last, partial step, or one past it (not used)
      if (full) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
#pragma unroll
          for (int p = 0; p < AU; ++p) v.a[p][j] = *at_bytes(ar + j * a.lda, ao[p]);
#pragma unroll
          for (int p = 0; p < BU; ++p) v.b[p][j] = *at_bytes(br + j * a.ldb, bo[p]);
        }
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const bool in = k + h8 + j < ke;
#pragma unroll
          for (int p = 0; p < AU; ++p) v.a[p][j] = in ? *at_bytes(ar + j * a.lda, ao[p]) : 0.f;
#pragma unroll
          for (int p = 0; p < BU; ++p) v.b[p][j] = in ? *at_bytes(br + j * a.ldb, bo[p]) : 0.f;
        }
      }
    };
    auto store = [&](char* buf, Pieces& v) {
#pragma unroll
      for (int p = 0; p < AU; ++p) {
        const int u = t + p * NT;
        u4 s[3];
#pragma unroll
        for (int j = 0; j < 8; ++j) v.a[p][j] *= sign;
        split8(v.a[p], s);
        u4* q = reinterpret_cast<u4*>(buf) + (u >> 6) * 3 * 64 + (u & 63);
        if (RB * 64 % NT == 0 || u < RB * 64) { q[0] = s[0]; q[64] = s[1]; q[128] = s[2]; }
      }
#pragma unroll
      for (int p = 0; p < BU; ++p) {
        const int u = t + p * NT;
        u4 s[3];
#pragma unroll
        for (int j = 0; j < 8; ++j) v.b[p][j] *= kUp;
        split8(v.b[p], s);
        u4* q = reinterpret_cast<u4*>(buf + RB * 3 * kFrag) + (u >> 6) * 3 * 64 + (u & 63);
        if (NB * 64 % NT == 0 || u < NB * 64) { q[0] = s[0]; q[64] = s[1]; q[128] = s[2]; }
      }
    };

    f16 acc[RBW][NBW];
#pragma unroll
    for (int i = 0; i < RBW; ++i)
#pragma unroll
      for (int j = 0; j < NBW; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    auto step = [&](int64_t k, char* cur, char* next, Pieces& vnext, Pieces& vload) {
      load(vload, k + PF * kKs);
      const bf8* as = reinterpret_cast<const bf8*>(cur) + wr * RBW * 3 * 64 + lane;
      const bf8* bs = reinterpret_cast<const bf8*>(cur + RB * 3 * kFrag) + wc * NBW * 3 * 64 + lane;
      mul_step<RBW, NBW, PF>(as, bs, acc);
      store(next, vnext);
      if (PF == 2) pipeline<RBW, NBW>();
      __syncthreads();
    };
    load(v[0], kb);
    if (PF == 2) load(v[PF - 1], kb + kKs);
    store(lds[0], v[0]);
    __syncthreads();
    int64_t k = kb;
    for (; k + kKs < ke; k += 2 * kKs) {
      step(k, lds[0], lds[1], v[PF - 1], v[0]);
      step(k + kKs, lds[1], lds[0], v[0], v[PF - 1]);
    }
    if (k < ke) step(k, lds[0], lds[1], v[PF - 1], v[0]);

    float* part = a.part + group * a.M * a.N;
    int wm = m0 + wr * RBW * 32, wn = n0 + wc * NBW * 32, N = a.N;
    // (the addresses of the sums are formed here, not kept over the chunks)
    if (RUN) asm volatile("" : "+s"(wm), "+s"(wn), "+s"(N));
    if (not_finite<RBW, NBW>(acc)) {
      down = 1.f;
      auto load = [&](int64_t k, float (*x)[4], float (*y)[4]) {
#pragma unroll
        for (int i = 0; i < RBW; ++i) {
          const int m = wm + i * 32 + (lane & 31);
          const float* q = a.A + k * a.lda + (m < a.M ? m : a.M - 1);
#pragma unroll
          for (int j = 0; j < 4; ++j) x[i][j] = k + j < ke ? q[j * a.lda] : 0.f;
        }
#pragma unroll
        for (int i = 0; i < NBW; ++i) {
          const int n = wn + i * 32 + (lane & 31);
          const float* q = a.B + k * a.ldb + (n < a.N ? n : a.N - 1);
#pragma unroll
          for (int j = 0; j < 4; ++j) y[i][j] = k + j < ke ? q[j * a.ldb] : 0.f;
        }
      };
      mul_again<RBW, NBW>(kb, ke, load, acc);
    }
#pragma unroll
    for (int i = 0; i < RBW; ++i)
#pragma unroll
      for (int j = 0; j < NBW; ++j) {
        const int n = wn + j * 32 + (lane & 31);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int m = wm + i * 32 + result_row(e, lane);
          if (m < a.M && n < N) {
            float* q = part + (int64_t)m * N + n;
            const float v = acc[i][j][e] * down;
            *q = RUN && add ? *q + v : v;
          }
        }
      }
  };
  if constexpr (RUN) {
    const int64_t first = group * a.run;
    for (int64_t c = first; c < first + a.run && c < a.chunks; ++c) sum_chunk(c, c != first);
  } else {
    sum_chunk(group, false);
  }
}

}  // namespace

// ---- launch ----------------------------------------------------------------------

// The lane parts of the addresses are 32-bit offsets over the rows of a tile
// (256 of A and of B stored N x K, 8 of B stored K x N and of both operands of
// A^T B, 4 of C); larger strides, and sizes beyond 2^30, stay with the general
// kernels.
bool gemm_split_tall_takes(int op, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb,
                           int64_t ldc, int64_t ldm) {
  return M < (int64_t(1) << 33) && N < (int64_t(1) << 30) && K >= 16 && K <= 4096 &&
         lda < (int64_t(1) << 22) && ldb < (int64_t(1) << (op == GCN_GEMM_NT ? 22 : 26)) &&
         ldc < (int64_t(1) << 27) && ldm < (int64_t(1) << 27);
}

bool gemm_split_tn_takes(int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb) {
  return M < (int64_t(1) << 30) && N < (int64_t(1) << 30) && K >= 64 &&
         lda < (int64_t(1) << 26) && ldb < (int64_t(1) << 26);
}

namespace {

template <bool BT>
hipError_t launch_split_tall(const TallArgs& a, int per, hipStream_t stream) {
  auto go = [&](auto kern, int threads, int64_t rows) {
    const int64_t row_tiles = ceil_div(ceil_div(a.M, rows), (int64_t)8) * 8;
    hipLaunchKernelGGL(kern, dim3((unsigned)(row_tiles * a.col_tiles)), dim3(threads), 0, stream,
                       a);
    return hipGetLastError();
  };
  // 256 columns: 256-row tiles of eight wavefronts, which split B half as often,
  // once there are tiles for most CUs; below that 64 rows.
  switch (per) {
    case 1: return go(k_split_tall<4, 1, 1, 1, BT>, 256, 128);
    case 2: return go(k_split_tall<4, 1, 1, 2, BT>, 256, 128);
    case 4: return go(k_split_tall<2, 2, 2, 2, BT>, 256, 128);
    case 6: return go(k_split_tall<2, 2, 2, 3, BT>, 256, 128);
    default:
      return a.M >= 32768 ? go(k_split_tall<4, 2, 2, 4, BT>, 512, 256)
                          : go(k_split_tall<1, 4, 2, 2, BT>, 256, 64);
  }
}

}  // namespace

gcn_status gemm_split_tall(int op, int64_t M, int64_t N, int64_t K, const float* A, int64_t lda,
                           const float* B, int64_t ldb, float* C, int64_t ldc, const float* mask,
                           int64_t ldm, bool relu, hipStream_t stream) {
  // column tiles of at most 8 blocks of 32, all of the same width
  const int64_t nb = ceil_div(N, (int64_t)32);
  const int64_t col_tiles = ceil_div(nb, (int64_t)8);
  int per = (int)ceil_div(nb, col_tiles);
  per = per <= 2 ? per : (per + 1) / 2 * 2;
  ProfScope ps(op == GCN_GEMM_NN ? "gemm_nn" : "gemm_nt", stream);
  const TallArgs a{M, (int)N, (int)K, A, lda, B, ldb, (int)col_tiles, C, ldc, mask, ldm, relu};
  const hipError_t e = op == GCN_GEMM_NN ? launch_split_tall<false>(a, per, stream)
                                         : launch_split_tall<true>(a, per, stream);
  if (e != hipSuccess) return hip_fail(e, "k_split_tall", __FILE__, __LINE__);
  return GCN_OK;
}

gcn_status gemm_split_tn(int64_t M, int64_t N, int64_t K, const float* A, int64_t lda,
                         const float* B, int64_t ldb, float* C, int64_t ldc, hipStream_t stream) {
  // 256 x 256 tiles split each value half as often as 128 x 128 ones and have
  // one workgroup per CU: faster once every CU has long chunks (512 x 256 x
  // 2.45M: 3.73 ms against 4.16; x 65,536: 160 us against 136).
  const bool wide = M > 128 && N > 128 && K >= 131072;
  const int64_t tm = wide ? 256 : 128;
  const int64_t tn = wide ? 256 : (N <= 32 ? 32 : (N <= 64 ? 64 : 128));
  const int64_t m_tiles = ceil_div(M, tm), n_tiles = ceil_div(N, tn), tiles = m_tiles * n_tiles;
  // Rows of a chunk: at most those after which the sums are as close to 64 bits as
  // the fp32 instruction's were in chunks of `most` rows (1024, or more where C
  // has many tiles and K many rows): 1408 rows here are like 1024 there (300 x 300
  // x 500,000 in 1312 rows 5.9e-7 against 6.1e-7; in 1968 rows 7.0e-7). And 1024 for small
  // outputs, 2048 for most, so that long sums stay below that (256 x 96 x 2.45M
  // 6.5e-7 against 7.2e-7; 512 x 256 7.4e-7 against 11.7e-7). A multiple of 512
  // workgroups, a fixed count so that the order of the sums does not depend on
  // the device.
  const int64_t fp32_tiles = ceil_div(M, (int64_t)128) * ceil_div(N, (int64_t)(N <= 64 ? 64 : 128));
  int64_t most = 8192;
  while (most > 1024 && fp32_tiles * ceil_div(K, most) < 4096) most /= 2;
  const int64_t rows = std::min<int64_t>(
      M * N <= 32768 ? 1024 : (M * N <= 262144 ? 2048 : 8192), most + most * 3 / 8);
  const int64_t rounds = std::max<int64_t>(1, ceil_div(K * tiles, (int64_t)512 * rows));
  const int64_t want = std::max<int64_t>(1, 512 * rounds / tiles);
  // Short sums are chains of steps: at least 64 rows (3,000 x 64 x 10: 17.6 us with
  // 256, 11.9; 128 for outputs whose partials take longer to add, 512 x 256: 25 and 22).
  const int64_t least = M * N <= 32768 ? 64 : 128;
  const int64_t split =
      std::max<int64_t>(least, std::min(rows, ceil_div(ceil_div(K, want), (int64_t)kKs) * kKs));
  const int64_t chunks = ceil_div(K, split);
  // The partials take about the memory of those of `most` rows (at most 1.3 times
  // it), or of 512 workgroups (134 MB), if that is more: a workgroup adds up several
  // chunks (512 x 256 x 2.45M: 335 MB instead of 671, 3.69 ms instead of 3.66).
  const int64_t run = std::max<int64_t>(
      1, std::min(ceil_div(chunks * most - 3 * K / 10, K), chunks * tiles / 512));
  const int64_t groups = ceil_div(chunks, run);
  float* part = nullptr;
  GCN_CHECK(talloc(&part, groups * M * N, stream, "GEMM partials"));
  const TnArgs a{(int)M, (int)N, K, split, chunks, run, groups, A, lda, B, ldb, part, (int)m_tiles,
                 (int)n_tiles};
  const dim3 grid((unsigned)(tiles * ceil_div(groups, (int64_t)8) * 8));
  hipError_t e;
  {
    ProfScope ps("gemm_tn_partial", stream);
    auto go = [&](auto kern, auto kern_run, int threads) {
      hipLaunchKernelGGL(run > 1 ? kern_run : kern, grid, dim3(threads), 0, stream, a);
    };
    if (wide)
      go(k_split_tn<4, 2, 2, 4, 1, false>, k_split_tn<4, 2, 2, 4, 1, true>, 512);
    else if (tn == 128)
      go(k_split_tn<2, 2, 2, 2, 2, false>, k_split_tn<2, 2, 2, 2, 2, true>, 256);
    else if (tn == 64)
      go(k_split_tn<4, 1, 1, 2, 2, false>, k_split_tn<4, 1, 1, 2, 2, true>, 256);
    else
      go(k_split_tn<4, 1, 1, 1, 2, false>, k_split_tn<4, 1, 1, 1, 2, true>, 256);
    e = hipGetLastError();
  }
  gcn_status st = e == hipSuccess ? sum_partials(M, N, groups, part, C, ldc, stream)
                                  : hip_fail(e, "k_split_tn", __FILE__, __LINE__);
  tfree(part, stream);
  return st;
}

}  // namespace gcn

// FP32 step with the coupling product on the int8 matrix cores.
//
// The plain method's product F = J.Q (Eq. 8) in fixed point: every position
// is held beside its FP32 value as a 32-bit integer v = rint(q 2^k) with one
// exponent k per replica, chosen so that the replica's largest |q| just fits,
// and split into four balanced base-256 digits.  For integer couplings
// |J_ij| <= 127 the four digit products run on v_mfma_i32_32x32x32_i8 with
// int32 accumulation, which is exact, and F is their weighted sum: pairs of
// digits exactly in 32 bits, then one FP32 conversion of each half and one
// fused multiply-add.  Positions within a factor of 64 of the replica's
// largest enter without any error, smaller ones with at most 2^-31 of the
// largest; the FP32 matrix cores round every partial sum to 24 bits instead.
// Against 64 bits, final positions after 20 steps: 5.3e-8 (FP32 4.6e-7) at N =
// 2000, R = 1024.  The sum does not depend on its order, so neither the tile
// nor a split changes a result.
//
// Uneven replicas.  2^-31 of the largest is less than what FP32 sums lose as
// long as every row sums products of large positions.  Where a few positions
// tower over the rest, a row that does not contain them (their own; in real
// couplings also one whose couplings to them vanish) is a sum of small
// positions only, which FP32 forms to 24 bits of its own size.  So a replica
// takes the fixed point in a step only if at least half of its groups of four
// neighbouring positions hold one that reaches a sixteenth of its scale
// (I8_LARGE; of random positions and positions between the walls 58 % and more
// do, so that 97 % of the groups count); the step that forms positions counts
// their groups.  The others' products are formed on the FP32 matrix cores by
// the same launch (i8_uneven): one position of 1.4 among ones of 1e-6, k = 0, N
// = 1000, R = 704, largest relative error of a momentum 4e-5 (15 in fixed
// point, 3e-4 on the FP32 tiles).  N = 2000, R = 1024 with every replica uneven
// 123 us a step (110 with real couplings; the FP32 tiles 74), with none 22.4
// (22.3 without the counts); the 32 x 16 tiles 11.5 (11.4) at N = 600, R = 1024.
//
// Measured (MI355X, us per step, FP32 matrix cores before): N = 2000, R = 1024
// 22.4 (73.6), R = 2048 42 (141), N = 4000, R = 2048 128 (532), N = 8000,
// R = 2048 480 (2076).  Bound: four int8 products take 7.6 us of matrix time a
// step at N = 2000, R = 1024 (256 tiles, one per CU; 52 us at the FP32 peak);
// a 256-deep slab of a tile takes 1.6 us instead of 0.95, because the loads of
// J and the copies and LDS reads of the digits fill the CU's memory and LDS
// pipelines as well, and the start and the end of a launch take 10 us (one tile
// per CU with 4, 8, 16 and 32 slabs: N, R = 1024, 2048 16.4 us, 2048, 1024 23.1,
// 4096, 512 35.9, 8192, 256 62).  Slower: J through LDS too (24.0 at N = 2000, R = 1024; 127 at
// N = 4000, R = 2048), eight 32 x 32 matrix waves (23.6; 138), eight waves
// without state waves (25; 147), counters in LDS for the slab barriers (23.4;
// 132), J fetched into L2 ahead (23.2; 136).
//
// Operand layout: 1 KB blocks of 32 rows (or replicas) by 32 contraction
// indices in the matrix instruction's own lane order (lane l holds the 16
// bytes of row l % 32 from index 16 (l / 32) on), so that slabs are copied to
// LDS, and fragments read from it, as consecutive 1 KB pieces: no swizzle,
// no bank conflict.  J: [row block][k block], Q: [column block][k block][digit].
//
// Scales.  The digits of q_{n+1} are written by the step that computes it,
// so the largest |q_{n+1}| of a replica has to be known before: in the paper
// order q_{n+1} = clamp(q_n + (Delta_n/m) p_n) depends on the state n alone,
// and the previous step, which produced that state, leaves the maximum per
// row tile and replica in peak.  After set_state, set_schedule or steps by
// other kernels a preparation kernel derives digits, scales and maxima from
// the FP32 state.  Every entry q_{n+1} lies within the walls, so only
// positions given by the caller can be non-finite: their replicas carry
// I8_SPECIAL and are stepped as uneven ones.
#include <algorithm>
#include <type_traits>

#include "si_epilogue.h"
#include "si_f32_gemm.h"
#include "si_grid_barrier.h"
#include "si_internal.h"

namespace si {

typedef int intx4 __attribute__((ext_vector_type(4)));
typedef int intx16 __attribute__((ext_vector_type(16)));
typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void_q;
typedef __attribute__((address_space(1))) const void gbl_void_q;

namespace {
constexpr int QP = I8_DIGITS;
constexpr int BLK = 1024;  // bytes of one 32 x 32 operand block
}  // namespace

// First digit's 1 KB block (of jd, or QP) of J's row block rb, or of the
// positions' column block cb, at contraction block kb.  The contraction is outermost:
// all workgroups walk it together, so what they read at one time lies in
// one consecutive range and spreads over every channel of the caches and the
// memory (row blocks outermost would put it at strides of a power of two).
template <int JD>
__device__ __forceinline__ size_t i8_jblk(int kb, int rb, int nrb) {
  return (((size_t)(kb >> 1) * nrb + rb) * 2 + (kb & 1)) * JD;
}
__device__ __forceinline__ size_t i8_qblk(int kb, int cb, int ncb) {
  return (((size_t)(kb >> 1) * ncb + cb) * 2 + (kb & 1)) * QP;
}

// Exponent k of a replica whose largest |q| is m: |rint(q 2^k)| fits four
// balanced digits (at most 0x7F7F7F7F).  I8_ZERO where every position is zero.
__device__ __forceinline__ int i8_exponent(float m) {
  if (!(m <= 3.402823466e38f)) return I8_SPECIAL;
  if (m == 0.f) return I8_ZERO;
  int e;
  (void)frexpf(m, &e);
  int k = 31 - e;
  if (ldexpf(m, k) > 2139062016.f) --k;  // 0x7F7F7F00
  return k;
}

// q in fixed point, and its four digits as the bytes of one word, lowest
// digit first.
__device__ __forceinline__ float i8_fixed(float q, int k) {
  return fminf(fmaxf(rintf(ldexpf(q, k)), -2139062016.f), 2139062016.f);
}
__device__ __forceinline__ uint32_t i8_digits(float v) {
  return ((uint32_t)(int)v + 0x80808080u) ^ 0x80808080u;
}

// Whether one of four positions in fixed point reaches I8_LARGE.
__device__ __forceinline__ bool i8_is_large(const float (&v)[4]) {
  return fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3]))) >= I8_LARGE;
}

// Whether a replica's product is formed in FP32: scale k, and the number of
// groups of four positions that i8_is_large holds for.
__device__ __forceinline__ bool i8_is_uneven(int k, int large, int n) {
  return k == I8_SPECIAL || (k != I8_ZERO && 2 * large < (n + 3) / 4);
}

// Bytes of four words regrouped by digit: out[d] = digit d of the four.
__device__ __forceinline__ void byte_transpose(const uint32_t (&w)[4], uint32_t (&out)[4]) {
  const uint32_t lo01 = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u);
  const uint32_t hi01 = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u);
  const uint32_t lo23 = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u);
  const uint32_t hi23 = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
  out[0] = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u);
  out[1] = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u);
  out[2] = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u);
  out[3] = __builtin_amdgcn_perm(hi23, hi01, 0x07060302u);
}

// 4 x 4 transpose over the four lanes of a quad: lane t's w[c] becomes lane
// c's out[t].
__device__ __forceinline__ void quad_transpose(uint32_t (&w)[4]) {
  const int t = threadIdx.x & 3;
  // exchange with lane t ^ 1 (quad_perm 1,0,3,2), then with t ^ 2 (2,3,0,1)
#pragma unroll
  for (int c = 0; c < 4; c += 2) {
    const uint32_t send = (t & 1) ? w[c] : w[c + 1];
    const uint32_t got = (uint32_t)__builtin_amdgcn_mov_dpp((int)send, 0xB1, 0xF, 0xF, true);
    if (t & 1)
      w[c] = got;
    else
      w[c + 1] = got;
  }
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const uint32_t send = (t & 2) ? w[c] : w[c + 2];
    const uint32_t got = (uint32_t)__builtin_amdgcn_mov_dpp((int)send, 0x4E, 0xF, 0xF, true);
    if (t & 2)
      w[c] = got;
    else
      w[c + 2] = got;
  }
}

// Wall bits of four positions and momenta before clamping, as the FP32 tiles
// record them for the adjoint (bit 0: q within its walls, bit 1: p).
__device__ __forceinline__ uint32_t i8_wall_bits(const I8Args &a, floatx4 q4, floatx4 p4, floatx4 f,
                                                 float dt, float zeta) {
  uint32_t mk = 0;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const float uu = fmaf(dt * a.inv_m, p4[v], q4[v]);
    const float vv = fmaf(dt, fmaf(zeta, f[v], -a.k * q4[v]), p4[v]);
    mk |= ((fabsf(uu) <= a.qmax ? 1u : 0u) | (fabsf(vv) <= a.pmax ? 2u : 0u)) << (8 * v);
  }
  return mk;
}

// Wait until at most N memory operations of this wave are in flight, then
// synchronise the workgroup.  The wait goes through the builtin, which the
// compiler's own wait insertion accounts for.
template <int N>
__device__ __forceinline__ void q_wait_barrier() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));
  asm volatile("s_barrier" ::: "memory");
}
__device__ __forceinline__ void q_barrier() { asm volatile("s_barrier" ::: "memory"); }
__device__ __forceinline__ void q_wait_lds() { __builtin_amdgcn_s_waitcnt(0xC07F); }

// ---------------------------------------------------------------------------
// Step kernel: 256 x 32 tiles in two roles.  Four matrix waves of 64 x 32 run
// the products: each reads its own rows of J straight from memory into
// registers, PD contraction blocks ahead, and the digits, which all four
// need, from an LDS ring of 256-deep slabs.  Four state waves fill the ring
// and own the tile's state: in the paper order q' and its digits need no
// coupling term, so they are formed while the product runs, and p' follows
// while the product of the workgroup's next tile runs.  (A workgroup takes
// every gridDim-th tile of its XCD, and the ring flows across tiles.)  The
// two roles share the matrix pipes, the copies' queue and the vector units
// instead of taking turns on them.
//
// Barriers, passed by both roles: one when the first slab has landed, then
// per tile nk slab barriers (the slab has been read, the next one has
// landed) and one when F is in LDS.
// ---------------------------------------------------------------------------
template <int JD_>
struct I8Cfg {
  static constexpr int JD = JD_;               // digits of J
  static constexpr bool REAL = JD > 1;
  static constexpr int BM = REAL ? I8_BM_REAL : I8_BM, BN = REAL ? 64 : 32;
  static constexpr int BKB = REAL ? 4 : 8, STAGES = 3;  // contraction blocks per slab, slabs
  static constexpr int NM = 4, NS = 4, NT = 64 * (NM + NS);
  static constexpr int RB = BM / 32 / NM, NCB = BN / 32;  // blocks of a matrix wave
  static constexpr int SLOT = BKB * NCB * QP * BLK;       // digits of one slab
  static constexpr int L = BKB * NCB * QP / NS;  // 1 KB copies per state wave and slab
  static constexpr int PD = REAL ? 4 : 8;      // contraction blocks of J held ahead (a slab)
  static constexpr int LDT = BM + 4;           // floats per column of F
  static constexpr int COLS = BN / NS;         // columns per state wave
  static constexpr int LPC = BM / 4;           // lanes per column, four spins each
  static constexpr int PERL = COLS * LPC / 64;  // columns per lane
  static constexpr int SETS = PERL / 4;
  static_assert(BM == 32 * RB * NM && PERL == 8 && BKB % PD == 0, "tile");
  static_assert(BKB * NCB == 2 * NS && (STAGES - 1) * L <= 63 && STAGES >= 2, "ring");
};
using I8Int = I8Cfg<1>;
using I8Real = I8Cfg<I8_JDIGITS>;

template <class C>
struct I8Smem {
  __attribute__((aligned(16))) uint8_t ring[C::STAGES * C::SLOT];
  __attribute__((aligned(16))) float tile[C::BN * C::LDT];
  int uneven, odd[C::BN];  // some column of this workgroup's tiles; the columns of one tile
};

// Tile i of this workgroup.  Every XCD (workgroup b runs on XCD b % 8) takes
// an xr-th of the row tiles by an xc-th of the column tiles (xr xc = 8), so
// that its L2 fetches that part of J and of the digits only, and walks it in
// bands of four row tiles, column by column, so that a band of J stays there.
template <class C>
struct I8Walk {
  int pr, pc, r0, c0, nr, nc, first, stride, count;
  __device__ __forceinline__ I8Walk(const I8Args &a) {
    const int ntr = a.ld / C::BM, ntc = a.r_pad / C::BN, xc = NUM_XCD / a.xr;
    const int x = blockIdx.x % NUM_XCD;
    pr = (ntr + a.xr - 1) / a.xr;
    pc = (ntc + xc - 1) / xc;
    r0 = (x / xc) * pr;
    c0 = (x % xc) * pc;
    nr = min(pr, ntr - r0);
    nc = min(pc, ntc - c0);
    first = blockIdx.x / NUM_XCD;
    stride = gridDim.x / NUM_XCD;
    const int tiles = nr > 0 && nc > 0 ? nr * nc : 0;
    count = first < tiles ? (tiles - first + stride - 1) / stride : 0;
  }
  __device__ __forceinline__ void at(int i, int &m0, int &n0) const {
    const int t = first + i * stride, band = t / (4 * nc), rows = min(4, nr - band * 4);
    const int u = t - band * 4 * nc;
    m0 = (r0 + band * 4 + u % rows) * C::BM;
    n0 = (c0 + u / rows) * C::BN;
  }
};

// The matrix waves' part of one step.
__device__ __forceinline__ void i8_matrix(const I8Args &a, const I8Walk<I8Int> &walk,
                                          I8Smem<I8Int> &sm) {
  using C = I8Int;
  constexpr int NB = C::BKB, PD = C::PD;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int nk = (a.n + 32 * NB - 1) / (32 * NB), nrb = a.ld / 32;
  const size_t pair = (size_t)nrb * 2 * BLK;  // two contraction blocks further
  int m0, n0;
  auto source = [&](int i) {
    walk.at(i, m0, n0);
    return a.Jt + i8_jblk<1>(0, m0 / 32 + wave * 2, nrb) * BLK + lane * 16;
  };
  intx4 fa[PD][2], fb[2][QP];
  auto load_a = [&](const uint8_t *s, int i, intx4 (&x)[2]) {
    s += (size_t)(i / 2) * pair + (i & 1) * BLK;
    x[0] = *reinterpret_cast<const intx4 *>(s);
    x[1] = *reinterpret_cast<const intx4 *>(s + 2 * BLK);
  };
  auto read_b = [&](const uint8_t *st, int i, int f) {
#pragma unroll
    for (int d = 0; d < QP; ++d)
      fb[f][d] = *reinterpret_cast<const intx4 *>(st + (i * QP + d) * BLK);
  };
  const uint8_t *cur = source(0), *nxt = cur;
#pragma unroll
  for (int i = 0; i < PD; ++i) load_a(cur, i, fa[i]);
  int rd = 0;
  const uint8_t *st = sm.ring + lane * 16;
  if (threadIdx.x == 0) sm.uneven = 0;
  q_wait_lds();
  q_barrier();  // the first slab has landed
  read_b(st, 0, 0);
  for (int tile = 0; tile < walk.count; ++tile) {
    walk.at(tile, m0, n0);
    const int kcol = a.kexp[a.cur][n0 + (lane & 31)];
    intx16 acc[2][QP];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int d = 0; d < QP; ++d)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][d][v] = 0;
    for (int kt = 0; kt < nk; ++kt) {
      // the slab after this one (of the next tile; past the last: this one)
      nxt = kt + 1 < nk ? cur + (NB / 2) * pair : tile + 1 < walk.count ? source(tile + 1) : cur;
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        if (i + 1 < NB) {
          read_b(st, i + 1, (i & 1) ^ 1);
        } else {
          q_wait_lds();  // this wave has read the slab
          q_barrier();
          rd = rd + 1 == C::STAGES ? 0 : rd + 1;
          st = sm.ring + rd * C::SLOT + lane * 16;
          read_b(st, 0, (i & 1) ^ 1);  // (past the last slab: not used)
        }
        // (the scheduler would gather the loads of J at the end)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int d = 0; d < QP; ++d)
#pragma unroll
          for (int r = 0; r < 2; ++r)
            acc[r][d] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[i % PD][r], fb[i & 1][d],
                                                              acc[r][d], 0, 0, 0);
        load_a(i + PD < NB ? cur : nxt, (i + PD) % NB, fa[i % PD]);
        __builtin_amdgcn_sched_barrier(0);
      }
      cur = nxt;
    }
    // F = sum_d 256^d acc_d 2^-k: pairs of digits exactly in 32 bits, then
    // one FP32 conversion each and one fused multiply-add
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float f[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int e = 4 * g + v;
          const float hi = (float)(acc[r][3][e] * 256 + acc[r][2][e]);
          const float lo = (float)(acc[r][1][e] * 256 + acc[r][0][e]);
          f[v] = ldexpf(fmaf(hi, 65536.f, lo), -kcol);
        }
        epi_put(sm.tile, C::LDT, wave * 64 + r * 32 + g * 8 + (lane / 32) * 4, lane & 31, f[0],
                f[1], f[2], f[3]);
      }
    q_wait_lds();
    q_barrier();  // F is in LDS
  }
}

// The same for couplings in four digits: 32 x 64 per wave, ten products per
// pair of blocks, summed by their weight 256^o (o = digit of J + digit of
// q - 3).  A column block's digits are read for the next contraction block as
// soon as its ten products are issued, while the other's run.
//
// Measured (us per step, FP32 matrix cores before): N = 2000, R = 1024 41.3
// (74.1), N = 4000, R = 2048 275 (532), N = 8000, R = 2048 1050 (2080); final
// positions against 64 bits after 5 steps at the last: 4.8e-8 (1.0e-6).
// Bound: the products; a loop of them alone takes 906 us at the last size
// (42 .. 48 cycles each instead of 32; 800 us with couplings of one digit),
// with the loads of J 950, with those and the digits' reads 1050.  Reordered
// for longer distances between dependent sums 1050, a shorter look-ahead of
// J (2 blocks) 1155.
__device__ __forceinline__ void i8_matrix(const I8Args &a, const I8Walk<I8Real> &walk,
                                          I8Smem<I8Real> &sm) {
  using C = I8Real;
  constexpr int NB = C::BKB, PD = C::PD, JD = C::JD;
  static_assert(JD == 4 && QP == 4 && C::RB == 1 && C::NCB == 2, "products");
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int nk = (a.n + 32 * NB - 1) / (32 * NB), nrb = a.ld / 32;
  const size_t pair = (size_t)nrb * 2 * JD * BLK;  // two contraction blocks further
  int m0, n0;
  auto source = [&](int i) {
    walk.at(i, m0, n0);
    return a.Jt + i8_jblk<JD>(0, m0 / 32 + wave, nrb) * BLK + lane * 16;
  };
  intx4 fa[PD][JD], fb[2][QP];
  auto load_a = [&](const uint8_t *s, int i, intx4 (&x)[JD]) {
    s += (size_t)(i / 2) * pair + (i & 1) * JD * BLK;
#pragma unroll
    for (int d = 0; d < JD; ++d) x[d] = *reinterpret_cast<const intx4 *>(s + d * BLK);
  };
  // (slab: [pair of blocks][column block][block of the pair][digit])
  auto read_b = [&](const uint8_t *st, int i, int c) {
#pragma unroll
    for (int d = 0; d < QP; ++d)
      fb[c][d] = *reinterpret_cast<const intx4 *>(
          st + ((((i >> 1) * 2 + c) * 2 + (i & 1)) * QP + d) * BLK);
  };
  const uint8_t *cur = source(0), *nxt = cur;
#pragma unroll
  for (int i = 0; i < PD; ++i) load_a(cur, i, fa[i]);
  int rd = 0;
  const uint8_t *st = sm.ring + lane * 16;
  if (threadIdx.x == 0) sm.uneven = 0;
  q_wait_lds();
  q_barrier();  // the first slab has landed
  read_b(st, 0, 0);
  read_b(st, 0, 1);
  for (int tile = 0; tile < walk.count; ++tile) {
    intx16 acc[2][4];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int o = 0; o < 4; ++o)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[c][o][v] = 0;
    for (int kt = 0; kt < nk; ++kt) {
      // the slab after this one (of the next tile; past the last: this one)
      nxt = kt + 1 < nk ? cur + (NB / 2) * pair : tile + 1 < walk.count ? source(tile + 1) : cur;
#pragma unroll
      for (int i = 0; i < NB; ++i) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          __builtin_amdgcn_sched_barrier(0);
          // digits of J and of q
          constexpr int PJ[10] = {0, 1, 2, 1, 2, 3, 2, 3, 3, 3}, PQ[10] = {3, 3, 3, 2, 2, 3, 1, 1, 2, 0};
#pragma unroll
          for (int e = 0; e < 10; ++e) {
            const int o = PJ[e] + PQ[e] - 3;
            acc[c][o] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[i % PD][PJ[e]], fb[c][PQ[e]],
                                                              acc[c][o], 0, 0, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
          if (i + 1 < NB) {
            read_b(st, i + 1, c);
          } else {
            if (c == 0) {
              q_wait_lds();  // this wave has read the slab
              q_barrier();
              rd = rd + 1 == C::STAGES ? 0 : rd + 1;
              st = sm.ring + rd * C::SLOT + lane * 16;
            }
            read_b(st, 0, c);  // (past the last slab: not used)
          }
        }
        load_a(i + PD < NB ? cur : nxt, (i + PD) % NB, fa[i % PD]);
      }
      cur = nxt;
    }
    // F = sum_o 256^(o + 3) acc_o 2^-(k + row's exponent): the leading sums
    // are exact in FP32 up to 2^24, each further one weighs 256 times less
    walk.at(tile, m0, n0);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int kcol = a.kexp[a.cur][n0 + c * 32 + (lane & 31)];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int row = wave * 32 + g * 8 + (lane / 32) * 4;
        const intx4 kj = *reinterpret_cast<const intx4 *>(a.jexp + m0 + row);
        float f[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int e = 4 * g + v;
          float x = fmaf((float)acc[c][1][e], 256.f, (float)acc[c][0][e]);
          x = fmaf((float)acc[c][2][e], 65536.f, x);
          x = fmaf((float)acc[c][3][e], 16777216.f, x);
          f[v] = ldexpf(x, 24 - kcol - kj[v]);
        }
        epi_put(sm.tile, C::LDT, row, c * 32 + (lane & 31), f[0], f[1], f[2], f[3]);
      }
    }
    q_wait_lds();
    q_barrier();  // F is in LDS
  }
}

// p' and the next step's maxima of the uneven replicas in this workgroup's
// tiles, again, from products on the FP32 matrix cores (all waves; q', its
// digits and counts need no product and stand).  128 rows at a time, with the
// main loops of the FP32 tiles in the ring's LDS.
template <class C, int WALL>
__device__ __forceinline__ void i8_uneven(const I8Args &a, const I8Walk<C> &walk, I8Smem<C> &sm) {
  using F = std::conditional_t<C::REAL, F32Cfg<128, 64, 4, 2, 32, 32, 4, 1>,
                               F32Cfg<128, 32, 8, 1, 16, 64, 0, 1>>;
  static_assert(F::NT == C::NT && F::BN == C::BN && C::BM % F::BM == 0 &&
                F::LDS_FLOATS * 4 <= (int)sizeof sm.ring, "FP32 product");
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nx = a.cur ^ 1, ntr = a.ld / C::BM;
  const int wy = wave / F::WN, wx = wave % F::WN;
  const int row = threadIdx.x % C::LPC * 4;
  const float dt = a.dt[a.t], zeta = a.zeta[a.t];
  const float cn = a.dt[a.t + 1 < a.total_steps ? a.t + 1 : a.t] * a.inv_m;
  for (int i = 0; i < walk.count; ++i) {
    int m0, n0;
    walk.at(i, m0, n0);
    __syncthreads();  // (the tile before this one has been read)
    if (threadIdx.x == 0) sm.uneven = 0;
    __syncthreads();
    if (threadIdx.x < C::BN) {
      const int col = n0 + threadIdx.x;
      int large = 0;
      for (int rt = 0; rt < ntr; ++rt) large += a.peak[a.cur][(size_t)rt * a.r_pad + col].large;
      const bool odd = i8_is_uneven(a.kexp[a.cur][col], large, a.n);
      sm.odd[threadIdx.x] = odd;
      if (odd) sm.uneven = 1;
    }
    __syncthreads();
    if (!sm.uneven) continue;
    for (int mh = 0; mh < C::BM; mh += F::BM) {
      typename F::acc_t acc[F::TM][F::TN];
      const int K = (a.n + F::BK - 1) / F::BK * F::BK;
      float *ring = reinterpret_cast<float *>(sm.ring);
      if constexpr (F::STAGES > 0)
        f32_mainloop_dma<F>(a.J, a.q[a.cur], a.ld, K, m0 + mh, n0, acc, ring);
      else
        f32_mainloop<F, B_PLAIN>(a.J, a.q[a.cur], a.ld, K, m0 + mh, n0, acc, ring);
#pragma unroll
      for (int i = 0; i < F::TM; ++i)
#pragma unroll
        for (int j = 0; j < F::TN; ++j)
#pragma unroll
          for (int g = 0; g < F::M::NACC / 4; ++g)
            epi_put(sm.tile, C::LDT,
                    mh + wy * F::WTM + i * F::MB + g * 8 + (lane / F::MB) * 4,
                    wx * F::WTN + j * F::MB + lane % F::MB, acc[i][j][4 * g],
                    acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
    }
    __syncthreads();
    floatx4 h4 = {0.f, 0.f, 0.f, 0.f};
    if (a.h) h4 = *reinterpret_cast<const floatx4 *>(a.h + m0 + row);
    for (int col = threadIdx.x / C::LPC; col < C::BN; col += C::NT / C::LPC) {
      if (!sm.odd[col]) continue;
      const size_t off = (size_t)(n0 + col) * a.ld + m0 + row;
      const floatx4 q4 = *reinterpret_cast<const floatx4 *>(a.q[a.cur] + off);
      const floatx4 p4 = *reinterpret_cast<const floatx4 *>(a.p[a.cur] + off);
      const floatx4 f = *reinterpret_cast<const floatx4 *>(sm.tile + col * C::LDT + row);
      floatx4 pn, fh;
      float mx = 0.f;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float qv, pv;
        // (an infinite position times the rows' zero padding is not a number)
        fh[v] = (m0 + row + v < a.n ? f[v] : 0.f) + h4[v];
        spring_update<SI_ORDER_PAPER, WALL>(q4[v], p4[v], fh[v], dt, zeta, a.k, a.inv_m, a.qmax,
                                            a.pmax, qv, pv);
        pn[v] = pv;
        mx = fmaxf(mx, fabsf(fminf(fmaxf(fmaf(cn, pv, qv), -a.qmax), a.qmax)));
      }
      *reinterpret_cast<floatx4 *>(a.p[nx] + off) = pn;
      if (a.mask_out)
        *reinterpret_cast<uint32_t *>(a.mask_out + off) = i8_wall_bits(a, q4, p4, fh, dt, zeta);
#pragma unroll
      for (int o = 1; o < C::LPC; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
      if (row == 0) a.peak[nx][(size_t)(m0 / C::BM) * a.r_pad + n0 + col].mx = mx;
    }
  }
}

// The state waves' part of one step: wave sw owns COLS columns of a tile, a
// lane four spins of eight of them.
template <class C, int WALL, bool REC>
__device__ __forceinline__ void i8_state(const I8Args &a, const I8Walk<C> &walk, I8Smem<C> &sm) {
  const int sw = __builtin_amdgcn_readfirstlane(((int)threadIdx.x >> 6) - C::NM);
  const int lane = threadIdx.x & 63, row = lane % C::LPC * 4, nx = a.cur ^ 1;
  const int lc = lane / C::LPC * C::PERL;  // first of the lane's columns among the wave's
  // entry of the lane's column cc in a vector that holds one column per lane
  auto of = [&](int v, int cc) {
    const int x = __builtin_amdgcn_readlane(v, cc);
    if constexpr (C::LPC == 64) return x;
    const int y = __builtin_amdgcn_readlane(v, C::PERL + cc);
    return lc ? y : x;
  };
  const int nk = (a.n + 32 * C::BKB - 1) / (32 * C::BKB), ncb = a.r_pad / 32;
  const int ntr = a.ld / C::BM;
  int m0, n0;
  // copies: wave sw takes two contraction blocks of one column block of each slab
  const size_t step = (size_t)ncb * (C::BKB * QP) * BLK;
  const uint8_t *src = nullptr;
  int itile = 0, ikt = 0, islot = 0;  // tile and slab of the next copy, its slot
  auto issue = [&]() {
    if (itile >= walk.count) return;
    if (ikt == 0) {
      int m, n;
      walk.at(itile, m, n);
      src = a.Qt[a.cur] + i8_qblk(sw / C::NCB * 2, n / 32 + sw % C::NCB, ncb) * BLK + lane * 16;
    }
    uint8_t *dst = sm.ring + islot * C::SLOT + sw * C::L * BLK;
#pragma unroll
    for (int d = 0; d < C::L; ++d)
      __builtin_amdgcn_global_load_lds((gbl_void_q *)(src + d * BLK), (lds_void_q *)(dst + d * BLK),
                                       16, 0, 0);
    src += step;
    islot = islot + 1 == C::STAGES ? 0 : islot + 1;
    if (++ikt == nk) {
      ikt = 0;
      ++itile;
    }
  };
  const int total = walk.count * nk;
  int g = 1, left = 0;  // next slab to hand over (of all tiles'), barriers left in this tile
  // the barrier after a slab: the next one has landed, its slot is refilled
  auto pass = [&]() {
    if (g + C::STAGES - 2 < total)
      q_wait_barrier<(C::STAGES - 2) * C::L>();
    else
      q_wait_barrier<0>();
    issue();
    ++g;
    --left;
  };
  auto tick = [&]() {
    if (left > 0) pass();
  };
  issue();
  if (total > 1) {
    issue();
    q_wait_barrier<C::L>();  // the first slab has landed
  } else {
    q_wait_barrier<0>();
  }
  if (C::STAGES > 2) issue();

  const float dt = a.dt[a.t], zeta = a.zeta[a.t];
  const float cdt = dt * a.inv_m;
  const float cn = a.dt[a.t + 1 < a.total_steps ? a.t + 1 : a.t] * a.inv_m;
  floatx4 q4[C::PERL], p4[C::PERL], h4;
  int many = 0;  // groups of large new positions of column lc + lane % LPC
  // p' of tile (m, n) from F in LDS, and the next step's maxima
  auto finish = [&](int m, int n) {
#pragma unroll
    for (int set = 0; set < C::SETS; ++set) {
      uint32_t um[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int cc = set * 4 + c, col = sw * C::COLS + lc + cc;
        const size_t off = (size_t)(n + col) * a.ld + m + row;
        floatx4 f = *reinterpret_cast<const floatx4 *>(sm.tile + col * C::LDT + row);
        float mx = 0.f;
        floatx4 pn;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          float qv, pv;
          f[v] += h4[v];
          spring_update<SI_ORDER_PAPER, WALL>(q4[cc][v], p4[cc][v], f[v], dt, zeta, a.k, a.inv_m,
                                              a.qmax, a.pmax, qv, pv);
          pn[v] = pv;
          mx = fmaxf(mx, fabsf(fminf(fmaxf(fmaf(cn, pv, qv), -a.qmax), a.qmax)));
        }
        *reinterpret_cast<floatx4 *>(a.p[nx] + off) = pn;
        if constexpr (REC)
          *reinterpret_cast<uint32_t *>(a.mask_out + off) =
              i8_wall_bits(a, q4[cc], p4[cc], f, dt, zeta);
        um[c] = __float_as_uint(mx);
      }
      quad_transpose(um);
      float mx = fmaxf(fmaxf(__uint_as_float(um[0]), __uint_as_float(um[1])),
                       fmaxf(__uint_as_float(um[2]), __uint_as_float(um[3])));
#pragma unroll
      for (int off = 4; off < C::LPC; off <<= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
      if (lane % C::LPC / 4 == set)
        a.peak[nx][(size_t)(m / C::BM) * a.r_pad + n + sw * C::COLS + lc + lane % C::LPC] =
            I8Peak{mx, many};
      tick();
    }
  };
  for (int tile = 0; tile < walk.count; ++tile) {
    left = nk;
    if (tile > 0) finish(m0, n0);
    walk.at(tile, m0, n0);
    const int col0 = n0 + sw * C::COLS;
    // scales of the new positions (maxima of this wave's columns) and counts
    // of the current ones' large entries: one column and every (64 / COLS)th
    // row tile per lane
    float mx = 0.f;
    int large = 0;
    const int mine = col0 + lane % C::COLS;
    for (int rt = lane / C::COLS; rt < ntr; rt += 64 / C::COLS) {
      const I8Peak pk = a.peak[a.cur][(size_t)rt * a.r_pad + mine];
      mx = fmaxf(mx, pk.mx);
      large += pk.large;
    }
    const int kin = a.kexp[a.cur][mine];
    h4 = floatx4{0.f, 0.f, 0.f, 0.f};
    if (a.h) h4 = *reinterpret_cast<const floatx4 *>(a.h + m0 + row);
#pragma unroll
    for (int c = 0; c < C::PERL; ++c) {
      const size_t off = (size_t)(col0 + lc + c) * a.ld + m0 + row;
      q4[c] = *reinterpret_cast<const floatx4 *>(a.q[a.cur] + off);
      p4[c] = *reinterpret_cast<const floatx4 *>(a.p[a.cur] + off);
    }
#pragma unroll
    for (int off = C::COLS; off < 64; off <<= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
    const int kout = i8_exponent(mx);
    if (m0 == 0 && lane < C::COLS) a.kexp[nx][col0 + lane] = kout;
    tick();
    const int spin = m0 + (lane % C::LPC >> 2) * 16;
#pragma unroll
    for (int set = 0; set < C::SETS; ++set) {
      uint32_t w[QP][4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int cc = set * 4 + c, k = of(kout, cc);
        uint32_t dg[4], by[4];
        floatx4 qn;
        float fx[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float u = fmaf(cdt, p4[cc][v], q4[cc][v]);
          qn[v] = fminf(fmaxf(u, -a.qmax), a.qmax);
          fx[v] = i8_fixed(qn[v], k);
          dg[v] = i8_digits(fx[v]);
        }
        const uint64_t big = __ballot(i8_is_large(fx));
        if (lane % C::LPC == cc)
          many = C::LPC == 64 ? __popcll(big) : __popc((uint32_t)(lane < 32 ? big : big >> 32));
        *reinterpret_cast<floatx4 *>(a.q[nx] + (size_t)(col0 + lc + cc) * a.ld + m0 + row) = qn;
        byte_transpose(dg, by);
#pragma unroll
        for (int d = 0; d < QP; ++d) w[d][c] = by[d];
        if (c == 1) tick();
      }
      // lane t of a quad takes column t: 16 consecutive spins per digit
      const int rep = col0 + lc + set * 4 + (lane & 3);
      uint8_t *out = a.Qt[nx] + i8_qblk(spin / 32, rep / 32, ncb) * BLK + (spin & 16) * 32 +
                     (rep & 31) * 16;
#pragma unroll
      for (int d = 0; d < QP; ++d) {
        quad_transpose(w[d]);
        *reinterpret_cast<uintx4 *>(out + d * BLK) = uintx4{w[d][0], w[d][1], w[d][2], w[d][3]};
      }
      tick();
    }
    while (left > 0) pass();
    // (added up here, where these waves wait: no slab's copies are held up)
#pragma unroll
    for (int off = C::COLS; off < 64; off <<= 1) large += __shfl_xor(large, off);
    if (i8_is_uneven(kin, large, a.n)) sm.uneven = 1;
    q_barrier();  // F is in LDS
  }
  left = 0;
  finish(m0, n0);
}

// One step of this workgroup's tiles (REC: recording the wall bits).
template <class C, int WALL, bool REC>
__device__ __forceinline__ void i8_step(const I8Args &a, const I8Walk<C> &walk, I8Smem<C> &sm) {
  if (__builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) < C::NM)
    i8_matrix(a, walk, sm);
  else
    i8_state<C, WALL, REC>(a, walk, sm);
  __syncthreads();
  if (__builtin_expect(sm.uneven, 0)) i8_uneven<C, WALL>(a, walk, sm);
}

template <class C, int WALL, bool REC>
__global__ __launch_bounds__(C::NT) void step_i8_kernel(I8Args a) {
  __shared__ I8Smem<C> sm;
  const I8Walk<C> walk(a);
  if (walk.count == 0) return;
  i8_step<C, WALL, REC>(a, walk, sm);
}

// Resident form: one cooperative launch runs n_steps steps with a grid-wide
// barrier between them (see grid_barrier).  One tile per workgroup.
template <class C, int WALL>
__global__ __launch_bounds__(C::NT) void resident_i8_kernel(I8Args a, ResidentArgs r) {
  __shared__ I8Smem<C> sm;
  const I8Walk<C> walk(a);
  if (walk.count == 0) return;
  for (int s = 0; s < r.n_steps; ++s) {
    i8_step<C, WALL, false>(a, walk, sm);
    a.cur ^= 1;
    a.t += 1;
    if (s + 1 < r.n_steps && !grid_barrier(r.count, (uint32_t)(s + 1), r.err)) return;
  }
}

// ---------------------------------------------------------------------------
// Few replicas, integer couplings: 32 x 16 tiles, so that 64 replicas of N =
// 2000 give every CU one, and the contraction split over the eight waves of a
// workgroup.  Each wave reads its contraction steps of J and of the digits
// straight from memory into v_mfma_i32_16x16x64_i8's registers, FEW_PD steps
// ahead; the waves' sums (pairs of digits, exact in 32 bits) are added in LDS,
// and the update of the tile follows.  Sums are exact, so the result is that
// of the 256 x 32 tiles bit for bit (uneven replicas' FP32 sums aside).
//
// Measured (us per step, FP32 one-launch form or 256 x 32 tiles before): N =
// 2000, R = 50 6.8 (9.3), N = 4000, R = 64 12.3 (26.1), N = 1000, R = 512 10.4
// (13.1), N = 2000, R = 256 12.6 (19.4), N = 8000, R = 64 36.0 (47.2).  Bound: a
// launch, then its loads: 96 N bytes per workgroup (3.3 us at N = 2000, R = 64
// at 57 bytes a cycle and CU).  Two workgroups per CU and two steps ahead beat
// one and four (N = 4000, R = 64 12.0 against 15.0, N = 2000, R = 256 14.2
// against 20.0), three steps ahead spill to slower (20.4).
// ---------------------------------------------------------------------------
constexpr int FEW_PD = 2, FEW_BN = 16;

// FP32 products of 16 RB rows and 16 CB columns over the contraction indices
// k0 .. k1 (multiples of 64), operands straight from memory: rows (columns) of
// 64 lanes' four consecutive indices each, as the 16 x 16 x 4 products take
// them.  J, Q: this lane's row and column, l % 16, from index 4 (l / 16) on.
template <int RB, int CB>
__device__ __forceinline__ void i8_f32_product(const float *__restrict__ J,
                                               const float *__restrict__ Q, int ld, int k0, int k1,
                                               floatx4 (&acc)[RB][CB]) {
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < CB; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  for (int k = k0; k < k1; k += 32) {
    floatx4 a[2][RB], b[2][CB];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
#pragma unroll
      for (int i = 0; i < RB; ++i)
        a[u][i] = *reinterpret_cast<const floatx4 *>(J + (size_t)i * 16 * ld + k + u * 16);
#pragma unroll
      for (int j = 0; j < CB; ++j)
        b[u][j] = *reinterpret_cast<const floatx4 *>(Q + (size_t)j * 16 * ld + k + u * 16);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
          for (int j = 0; j < CB; ++j)
            acc[i][j] = MfmaF32<16>::mma(a[u][i][v], b[u][j][v], acc[i][j]);
  }
}

template <int FEW_W, int WALL, bool REC>
__global__ __launch_bounds__(64 * FEW_W, 4) void step_i8_few_kernel(I8Args a) {
  constexpr int BM = I8_BM_FEW, BN = FEW_BN;
  __shared__ __attribute__((aligned(16))) int sums[FEW_W][2][BN][BM + 4];
  __shared__ __attribute__((aligned(16))) uint8_t dig[QP][BN][BM];
  __shared__ float colmax[BN];
  __shared__ int kshared[2][BN], collarge[BN], uneven;
  const int tid = threadIdx.x, lane = tid & 63, nx = a.cur ^ 1;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ntc = a.r_pad / BN, ntr = a.ld / BM, t = xcd_tile(blockIdx.x, gridDim.x);
  const int m0 = t / ntc * BM, n0 = t % ntc * BN;
  const int nrb = a.ld / 32, ncb = a.r_pad / 32, ns = (a.n + 63) / 64;  // steps of 64

  // lane l holds row (or column) l % 16 from index 16 (l / 16) of a step on:
  // block l / 32 of the pair, half l / 16 % 2 of its indices
  const int lrow = lane & 15, half = (lane >> 4) & 1;
  const uint8_t *pa = a.Jt + i8_jblk<1>(0, m0 / 32, nrb) * BLK + (lane >> 5) * BLK + half * 512 +
                      lrow * 16;
  const uint8_t *pb = a.Qt[a.cur] + i8_qblk(0, n0 / 32, ncb) * BLK + (size_t)(lane >> 5) * QP * BLK +
                      half * 512 + (n0 % 32 + lrow) * 16;
  const size_t da = (size_t)nrb * 2 * BLK, db = (size_t)ncb * 2 * QP * BLK;
  const int count = wave < ns ? (ns - wave + FEW_W - 1) / FEW_W : 0;
  intx4 fa[FEW_PD][2], fb[FEW_PD][QP];
  auto load = [&](int i, int f) {
    const int k = wave + (i < count ? i : count - 1) * FEW_W;  // (past the end: not used)
    const uint8_t *sa = pa + (size_t)k * da, *sb = pb + (size_t)k * db;
    fa[f][0] = *reinterpret_cast<const intx4 *>(sa);
    fa[f][1] = *reinterpret_cast<const intx4 *>(sa + 256);
#pragma unroll
    for (int d = 0; d < QP; ++d) fb[f][d] = *reinterpret_cast<const intx4 *>(sb + d * BLK);
  };
  if (count > 0)
#pragma unroll
    for (int f = 0; f < FEW_PD; ++f) load(f, f);

  // the tile's state: thread u < 128 owns four spins of one column
  const int scol = tid >> 3, srow = (tid & 7) * 4;
  const size_t off = (size_t)(n0 + scol) * a.ld + m0 + srow;
  floatx4 q4, p4, h4 = {0.f, 0.f, 0.f, 0.f};
  const bool owner = tid < BN * BM / 4;
  if (owner) {
    q4 = *reinterpret_cast<const floatx4 *>(a.q[a.cur] + off);
    p4 = *reinterpret_cast<const floatx4 *>(a.p[a.cur] + off);
    if (a.h) h4 = *reinterpret_cast<const floatx4 *>(a.h + m0 + srow);
  }
  // scales: the largest |q'| of every column of the tile (bits of floats >= 0
  // order as integers)
  const int kin = a.kexp[a.cur][n0 + (tid & 15)];
  float mx = 0.f;
  int large = 0;
  for (int rt = tid >> 4; rt < ntr; rt += 4 * FEW_W) {
    const I8Peak pk = a.peak[a.cur][(size_t)rt * a.r_pad + n0 + (tid & 15)];
    mx = fmaxf(mx, pk.mx);
    large += pk.large;
  }
  if (tid < BN) {
    colmax[tid] = 0.f;
    collarge[tid] = 0;
  }
  if (tid == 0) uneven = 0;
  __syncthreads();
  atomicMax(reinterpret_cast<int *>(colmax) + (tid & 15), __float_as_int(mx));
  atomicAdd(collarge + (tid & 15), large);

  intx4 acc[2][QP];
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int d = 0; d < QP; ++d) acc[r][d] = intx4{0, 0, 0, 0};
  auto mul = [&](int f) {
#pragma unroll
    for (int d = 0; d < QP; ++d)
#pragma unroll
      for (int r = 0; r < 2; ++r)
        acc[r][d] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[f][r], fb[f][d], acc[r][d], 0, 0, 0);
  };
  int i = 0;
  for (; i + FEW_PD < count; i += FEW_PD)
#pragma unroll
    for (int f = 0; f < FEW_PD; ++f) {
      mul(f);
      load(i + FEW_PD + f, f);
    }
#pragma unroll
  for (int f = 0; f < FEW_PD; ++f)
    if (i + f < count) mul(f);
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    intx4 hi, lo;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      hi[v] = acc[r][3][v] * 256 + acc[r][2][v];
      lo[v] = acc[r][1][v] * 256 + acc[r][0][v];
    }
    const int row = r * 16 + (lane >> 4) * 4;
    *reinterpret_cast<intx4 *>(&sums[wave][0][lrow][row]) = hi;
    *reinterpret_cast<intx4 *>(&sums[wave][1][lrow][row]) = lo;
  }
  __syncthreads();
  if (tid < BN) {
    const int kout = i8_exponent(colmax[tid]);
    const bool odd = i8_is_uneven(kin, collarge[tid], a.n);
    if (odd) uneven = 1;
    kshared[0][tid] = odd ? I8_SPECIAL : kin;
    kshared[1][tid] = kout;
    if (m0 == 0) a.kexp[nx][n0 + tid] = kout;
  }
  __syncthreads();
  if (owner) {
    const float dt = a.dt[a.t], zeta = a.zeta[a.t];
    const float cn = a.dt[a.t + 1 < a.total_steps ? a.t + 1 : a.t] * a.inv_m;
    const int kin = kshared[0][scol], kout = kshared[1][scol];
    intx4 hi = {0, 0, 0, 0}, lo = {0, 0, 0, 0};
#pragma unroll
    for (int w = 0; w < FEW_W; ++w) {
      hi += *reinterpret_cast<const intx4 *>(&sums[w][0][scol][srow]);
      lo += *reinterpret_cast<const intx4 *>(&sums[w][1][scol][srow]);
    }
    floatx4 f;
    float mnext = 0.f;
    floatx4 qn, pn;
    uint32_t dg[4], by[4];
    float fx[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      float qv, pv;
      f[v] = ldexpf(fmaf((float)hi[v], 65536.f, (float)lo[v]), -kin) + h4[v];
      spring_update<SI_ORDER_PAPER, WALL>(q4[v], p4[v], f[v], dt, zeta, a.k, a.inv_m, a.qmax,
                                          a.pmax, qv, pv);
      qn[v] = fminf(fmaxf(fmaf(dt * a.inv_m, p4[v], q4[v]), -a.qmax), a.qmax);
      pn[v] = pv;
      mnext = fmaxf(mnext, fabsf(fminf(fmaxf(fmaf(cn, pv, qv), -a.qmax), a.qmax)));
      fx[v] = i8_fixed(qn[v], kout);
      dg[v] = i8_digits(fx[v]);
    }
    *reinterpret_cast<floatx4 *>(a.q[nx] + off) = qn;
    *reinterpret_cast<floatx4 *>(a.p[nx] + off) = pn;
    if constexpr (REC)
      *reinterpret_cast<uint32_t *>(a.mask_out + off) = i8_wall_bits(a, q4, p4, f, dt, zeta);
    byte_transpose(dg, by);
#pragma unroll
    for (int d = 0; d < QP; ++d) *reinterpret_cast<uint32_t *>(&dig[d][scol][srow]) = by[d];
    // (the eight lanes of a column)
    const int many = __popc((uint32_t)(__ballot(i8_is_large(fx)) >> (lane & 56)) & 255u);
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) mnext = fmaxf(mnext, __shfl_xor(mnext, o));
    if ((tid & 7) == 0)
      a.peak[nx][(size_t)(m0 / BM) * a.r_pad + n0 + scol] = I8Peak{mnext, many};
  }
  __syncthreads();
  for (int u = tid; u < QP * 2 * BN; u += 64 * FEW_W) {  // 16 spins of one column and digit
    const int d = u >> 5, h = (u >> 4) & 1, c = u & 15;
    *reinterpret_cast<uintx4 *>(a.Qt[nx] + (i8_qblk(m0 / 32, n0 / 32, ncb) + d) * BLK + h * 512 +
                                (n0 % 32 + c) * 16) =
        *reinterpret_cast<const uintx4 *>(&dig[d][c][h * 16]);
  }
  if (__builtin_expect(!uneven, 1)) return;
  // p' and the maxima of the uneven columns again, from products on the FP32
  // matrix cores: a range of the contraction per wave, added in the order of the
  // ranges
  const int K = (a.n + 63) / 64 * 64, klen = (K / 64 + FEW_W - 1) / FEW_W * 64;
  floatx4 part[2][1];
  i8_f32_product(a.J + (size_t)(m0 + lrow) * a.ld + (lane >> 4) * 4,
                 a.q[a.cur] + (size_t)(n0 + lrow) * a.ld + (lane >> 4) * 4, a.ld, wave * klen,
                 min(K, (wave + 1) * klen), part);
#pragma unroll
  for (int r = 0; r < 2; ++r)
    *reinterpret_cast<floatx4 *>(&sums[wave][0][lrow][r * 16 + (lane >> 4) * 4]) = part[r][0];
  __syncthreads();
  if (!owner || kshared[0][scol] != I8_SPECIAL) return;
  q4 = *reinterpret_cast<const floatx4 *>(a.q[a.cur] + off);
  p4 = *reinterpret_cast<const floatx4 *>(a.p[a.cur] + off);
  h4 = floatx4{0.f, 0.f, 0.f, 0.f};
  if (a.h) h4 = *reinterpret_cast<const floatx4 *>(a.h + m0 + srow);
  floatx4 f = {0.f, 0.f, 0.f, 0.f}, pn;
#pragma unroll
  for (int w = 0; w < FEW_W; ++w) f += *reinterpret_cast<const floatx4 *>(&sums[w][0][scol][srow]);
  const float dt = a.dt[a.t], zeta = a.zeta[a.t];
  const float cn = a.dt[a.t + 1 < a.total_steps ? a.t + 1 : a.t] * a.inv_m;
  float mnext = 0.f;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    float qv, pv;
    // (an infinite position times the rows' zero padding is not a number)
    f[v] = (m0 + srow + v < a.n ? f[v] : 0.f) + h4[v];
    spring_update<SI_ORDER_PAPER, WALL>(q4[v], p4[v], f[v], dt, zeta, a.k, a.inv_m, a.qmax, a.pmax,
                                        qv, pv);
    pn[v] = pv;
    mnext = fmaxf(mnext, fabsf(fminf(fmaxf(fmaf(cn, pv, qv), -a.qmax), a.qmax)));
  }
  *reinterpret_cast<floatx4 *>(a.p[nx] + off) = pn;
  if constexpr (REC)
    *reinterpret_cast<uint32_t *>(a.mask_out + off) = i8_wall_bits(a, q4, p4, f, dt, zeta);
#pragma unroll
  for (int o = 1; o < 8; o <<= 1) mnext = fmaxf(mnext, __shfl_xor(mnext, o));
  if ((tid & 7) == 0) a.peak[nx][(size_t)(m0 / BM) * a.r_pad + n0 + scol].mx = mnext;
}

// Digits, scales, counts and maxima of the FP32 state (t: the next step's index).
// One workgroup per four replicas (256 of them at R = 1024: one per CU, 11.6
// us with half as many of eight, 7.0 now), two waves per replica for the maxima.
constexpr int PREP_R = 4;
__global__ __launch_bounds__(512) void i8_prepare_kernel(I8Args a) {
  __shared__ float most[2][8];
  __shared__ int isnan[8], kx[PREP_R], count[PREP_R];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r0 = blockIdx.x * PREP_R, rw = wave / 2;
  const float *q = a.q[a.cur], *p = a.p[a.cur];
  const float c = a.dt[a.t < a.total_steps ? a.t : a.total_steps - 1] * a.inv_m;
  {
    const size_t base = (size_t)(r0 + rw) * a.ld;
    float mq = 0.f, mu = 0.f;
    bool nan = false;
#pragma unroll 4
    for (int i = ((wave & 1) * 64 + lane) * 4; i < a.ld; i += 512) {
      const floatx4 q4 = *reinterpret_cast<const floatx4 *>(q + base + i);
      const floatx4 p4 = *reinterpret_cast<const floatx4 *>(p + base + i);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        nan |= q4[v] != q4[v];
        mq = fmaxf(mq, fabsf(q4[v]));
        mu = fmaxf(mu, fabsf(fminf(fmaxf(fmaf(c, p4[v], q4[v]), -a.qmax), a.qmax)));
      }
    }
    for (int off = 32; off >= 1; off >>= 1) {
      mq = fmaxf(mq, __shfl_xor(mq, off));
      mu = fmaxf(mu, __shfl_xor(mu, off));
    }
    const bool any = __any(nan);
    if (lane == 0) {
      most[0][wave] = mq;
      most[1][wave] = mu;
      isnan[wave] = any;
    }
  }
  __syncthreads();
  if (threadIdx.x < PREP_R) {
    const int w = threadIdx.x * 2;
    const int k = isnan[w] || isnan[w + 1] ? I8_SPECIAL : i8_exponent(fmaxf(most[0][w], most[0][w + 1]));
    kx[threadIdx.x] = k;
    count[threadIdx.x] = 0;
    a.kexp[a.cur][r0 + threadIdx.x] = k;
  }
  for (int u = threadIdx.x; u < a.ld / a.bm * PREP_R; u += 512) {
    const int rt = u / PREP_R, j = u % PREP_R;
    I8Peak *pk = a.peak[a.cur] + (size_t)rt * a.r_pad + r0 + j;
    pk->mx = rt == 0 ? fmaxf(most[1][2 * j], most[1][2 * j + 1]) : 0.f;
    if (rt > 0) pk->large = 0;  // (all counted in the first row tile's entry, below)
  }
  __syncthreads();
  const int j = threadIdx.x % PREP_R, r = r0 + j, k = kx[j], ncb = a.r_pad / 32;
  int large = 0;
  for (int pc = threadIdx.x / PREP_R; pc < a.ld / 16; pc += 512 / PREP_R) {
    uint32_t w[QP][4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const floatx4 q4 = *reinterpret_cast<const floatx4 *>(q + (size_t)r * a.ld + pc * 16 + g * 4);
      uint32_t dg[4], by[4];
      float fx[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        fx[v] = k == I8_SPECIAL ? 0.f : i8_fixed(q4[v], k);
        dg[v] = i8_digits(fx[v]);
      }
      large += i8_is_large(fx);
      byte_transpose(dg, by);
#pragma unroll
      for (int d = 0; d < QP; ++d) w[d][g] = by[d];
    }
    uint8_t *out = a.Qt[a.cur] + i8_qblk(pc / 2, r / 32, ncb) * BLK + (pc & 1) * 512 +
                   (r & 31) * 16;
#pragma unroll
    for (int d = 0; d < QP; ++d)
      *reinterpret_cast<uintx4 *>(out + d * BLK) = uintx4{w[d][0], w[d][1], w[d][2], w[d][3]};
  }
  atomicAdd(count + j, large);
  __syncthreads();
  if (threadIdx.x < PREP_R) a.peak[a.cur][r0 + threadIdx.x].large = count[threadIdx.x];
}

// Couplings into blocks of digits: one wave per block, 16 couplings per lane.
template <int JD>
__global__ __launch_bounds__(256) void i8_pack_j_kernel(const float *__restrict__ J, int ld,
                                                        int64_t blocks, const int *__restrict__ jexp,
                                                        uint8_t *__restrict__ out) {
  const int lane = threadIdx.x & 63, nkb = ld / 32;
  for (int64_t b = blockIdx.x * 4 + (threadIdx.x >> 6); b < blocks; b += (int64_t)gridDim.x * 4) {
    const int rb = (int)(b / 2 % nkb), kb = (int)(b / 2 / nkb) * 2 + (int)(b & 1);
    const int row = rb * 32 + (lane & 31);
    const float *src = J + (size_t)row * ld + kb * 32 + (lane >> 5) * 16;
    const int k = JD > 1 ? jexp[row] : 0;
    uint32_t w[JD][4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const floatx4 x = *reinterpret_cast<const floatx4 *>(src + g * 4);
      if constexpr (JD == 1) {
        w[0][g] = ((uint32_t)(int)x[0] & 255u) | (((uint32_t)(int)x[1] & 255u) << 8) |
                  (((uint32_t)(int)x[2] & 255u) << 16) | ((uint32_t)(int)x[3] << 24);
      } else {
        uint32_t dg[4], by[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) dg[v] = i8_digits(i8_fixed(x[v], k));
        byte_transpose(dg, by);
#pragma unroll
        for (int d = 0; d < JD; ++d) w[d][g] = by[d];
      }
    }
#pragma unroll
    for (int d = 0; d < JD; ++d)
      *reinterpret_cast<uintx4 *>(out + (b * JD + d) * BLK + lane * 16) =
          uintx4{w[d][0], w[d][1], w[d][2], w[d][3]};
  }
}

// Exponent of every row of real couplings (caller's layout), as for a replica's
// positions.  flags[8] is set if a row is not a dense one of like couplings:
// its largest exceeds I8_CREST times the root mean square of its n entries, or
// more than a sixteenth of them lie below 1/1024 of the largest (a Gaussian
// row: 0.4 %; the diagonal is one).  Such rows' sums may be finer in FP32 than
// 2^-31 of their largest product.  One wave per row; nothing to do for
// couplings that the checks before it (flags) found to take one digit.
__global__ __launch_bounds__(256) void i8_rows_kernel(const float *__restrict__ J, int n,
                                                      int *__restrict__ jexp, int *flags) {
  if (flags[3] == 0 && (int64_t)n * flags[6] <= I8_NJ_MAX) return;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= n) return;
  const float *x = J + (size_t)row * n;
  float m = 0.f;
#pragma unroll 4
  for (int i = lane; i < n; i += 64) m = fmaxf(m, fabsf(x[i]));
  for (int off = 32; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  float s = 0.f;  // sum of squares in units of the largest
  int small = 0;
#pragma unroll 4
  for (int i = lane; i < n; i += 64) {
    const float v = m > 0.f ? x[i] / m : 0.f;
    s = fmaf(v, v, s);
    small += fabsf(x[i]) < m * (1.f / 1024.f);
  }
  for (int off = 32; off >= 1; off >>= 1) {
    s += __shfl_xor(s, off);
    small += __shfl_xor(small, off);
  }
  if (lane == 0) {
    jexp[row] = i8_exponent(m);
    if (s * (I8_CREST * I8_CREST) < (float)n || small > n / 16 || m == 0.f) flags[8] = 1;
  }
}

static bool i8_real(const I8Args &a) { return a.bm == I8_BM_REAL; }

static bool i8_few(const I8Args &a) { return a.bm == I8_BM_FEW; }

// (Two slabs at least: the state waves read a tile's F between the slabs of
// the next one, whose last barrier lets the matrix waves write again.)
static bool i8_fits(const I8Args &a) {
  return (i8_few(a) || a.n > 32 * (i8_real(a) ? I8Real::BKB : I8Int::BKB)) &&
         (a.bm == I8_BM || i8_few(a) || (i8_real(a) && a.jexp)) && a.ld % a.bm == 0 && a.r_pad % 64 == 0 &&
         a.n >= 1 && a.n <= a.ld && (a.xr == 1 || a.xr == 2 || a.xr == 4 || a.xr == 8);
}

static int i8_bn(const I8Args &a) {
  return i8_real(a) ? I8Real::BN : i8_few(a) ? FEW_BN : I8Int::BN;
}

// One workgroup per CU (the register file holds one), fewer if an XCD's part
// has fewer tiles than CUs.
static int i8_grid(const I8Args &a, int num_cus) {
  const int ntr = a.ld / a.bm, ntc = a.r_pad / i8_bn(a), xc = NUM_XCD / a.xr;
  const int part = ((ntr + a.xr - 1) / a.xr) * ((ntc + xc - 1) / xc);
  const int per = std::max(num_cus / NUM_XCD, 1);
  return NUM_XCD * std::min(part, per);
}

// The split of the tiles over the XCDs' L2s that fetches least: every row
// group reads all of its column group's digits and the other way round.
int32_t i8_xcd_rows(const I8Args &a) {
  const int64_t ntr = a.ld / a.bm, ntc = a.r_pad / i8_bn(a);
  const int64_t nn = (int64_t)a.ld * a.ld * (i8_real(a) ? I8_JDIGITS : 1);
  const int64_t nr = (int64_t)a.ld * a.r_pad * I8_DIGITS;
  int32_t best = 1;
  double least = 0.0;
  for (int32_t xr = 1; xr <= NUM_XCD; xr *= 2) {
    const int64_t xc = NUM_XCD / xr, pr = (ntr + xr - 1) / xr, pc = (ntc + xc - 1) / xc;
    const double pad = (double)(pr * xr * pc * xc) / (double)(ntr * ntc);
    const int64_t bands = (pr + 3) / 4;  // sweeps over its columns
    const double cost = pad * ((double)nn * xc + (double)nr * xr * bands);
    if (xr == 1 || cost < least) {
      least = cost;
      best = xr;
    }
  }
  return best;
}

template <class C>
static const void *i8_step_of(const I8Args &a) {
  if (a.wall == SI_WALL_INELASTIC)
    return reinterpret_cast<const void *>(&step_i8_kernel<C, SI_WALL_INELASTIC, false>);
  return a.mask_out ? reinterpret_cast<const void *>(&step_i8_kernel<C, SI_WALL_CLAMP, true>)
                    : reinterpret_cast<const void *>(&step_i8_kernel<C, SI_WALL_CLAMP, false>);
}

static const void *i8_step_entry(const I8Args &a) {
  return i8_real(a) ? i8_step_of<I8Real>(a) : i8_step_of<I8Int>(a);
}

static const void *i8_resident(const I8Args &a) {
  const bool clamp = a.wall == SI_WALL_CLAMP;
  if (i8_real(a))
    return clamp ? reinterpret_cast<const void *>(&resident_i8_kernel<I8Real, SI_WALL_CLAMP>)
                 : reinterpret_cast<const void *>(&resident_i8_kernel<I8Real, SI_WALL_INELASTIC>);
  return clamp ? reinterpret_cast<const void *>(&resident_i8_kernel<I8Int, SI_WALL_CLAMP>)
               : reinterpret_cast<const void *>(&resident_i8_kernel<I8Int, SI_WALL_INELASTIC>);
}

template <int FEW_W>
static const void *i8_few_of(const I8Args &a) {
  if (a.wall == SI_WALL_INELASTIC)
    return reinterpret_cast<const void *>(&step_i8_few_kernel<FEW_W, SI_WALL_INELASTIC, false>);
  return a.mask_out ? reinterpret_cast<const void *>(&step_i8_few_kernel<FEW_W, SI_WALL_CLAMP, true>)
                    : reinterpret_cast<const void *>(&step_i8_few_kernel<FEW_W, SI_WALL_CLAMP, false>);
}

static int i8_few_tiles(const I8Args &a) { return a.ld / a.bm * (a.r_pad / FEW_BN); }

// Waves of a workgroup of the 32 x 16 tiles: eight while two workgroups fill a
// CU and the contraction is long, else four (us per step, eight against four:
// N = 2000, R = 50 6.8 and 7.1, N = 4000, R = 64 12.0 and 13.3, N = 2000, R =
// 256 14.2 and 12.4, N = 1000, R = 64 5.6 and 5.3).
static int i8_few_waves(const I8Args &a) { return i8_few_tiles(a) <= 512 && a.n > 1024 ? 8 : 4; }

// (wall bits are recorded for the adjoint, which takes clamping walls only)
hipError_t launch_step_i8(const I8Args &a, int num_cus, hipStream_t s) {
  if (!i8_fits(a) || (a.mask_out && a.wall != SI_WALL_CLAMP)) return hipErrorInvalidValue;
  I8Args aa = a;
  void *args[] = {&aa};
  if (i8_few(a)) {
    const int waves = i8_few_waves(a);
    return hipLaunchKernel(waves == 8 ? i8_few_of<8>(a) : i8_few_of<4>(a), dim3(i8_few_tiles(a)),
                           dim3(64 * waves), args, 0, s);
  }
  return hipLaunchKernel(i8_step_entry(a), dim3(i8_grid(a, num_cus)), dim3(I8Int::NT), args, 0, s);
}

const char *i8_kernel_name(const I8Args &a) {
  return i8_real(a)  ? "step_i8x10_128x64_w4_k128_s3"
         : i8_few(a) ? (i8_few_waves(a) == 8 ? "step_i8x4_32x16_ks8" : "step_i8x4_32x16_ks4")
                     : "step_i8x4_256x32_w4_k256_s3";
}

// Every workgroup of the grid must own exactly one tile: an even XCD split,
// and no more tiles than workgroups that fit at once.  Elsewhere a barrier
// between the steps costs more than their launches, so those contexts launch
// (us per step, launches against resident: N = 384, R = 400 5.9 and 18.8, N =
// 600, R = 1024 11.7 and 42, N = 8000, R = 64 36.5 and 73 with a resident form of
// the 32 x 16 tiles; N = 1100, R = 700 15.8 and 28.5, N = 3000, R = 1100 51 and 74
// with several or uneven tiles of the others; N = 2000, R = 1024, which has one,
// 21.8 and 37.7).
hipError_t resident_i8_groups(const I8Args &a, int num_cus, int32_t *groups) {
  *groups = 0;
  if (!i8_fits(a) || i8_few(a)) return hipSuccess;
  const int ntr = a.ld / a.bm, ntc = a.r_pad / i8_bn(a);
  if (ntr % a.xr || ntc % (NUM_XCD / a.xr) || i8_grid(a, num_cus) != ntr * ntc) return hipSuccess;
  int per = 0;
  hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, i8_resident(a), I8Int::NT, 0);
  if (e == hipSuccess && ntr * ntc <= per * num_cus) *groups = ntr * ntc;
  return e;
}

hipError_t launch_resident_i8(const I8Args &a, const ResidentArgs &r, int32_t groups,
                              hipStream_t s) {
  if (!i8_fits(a) || i8_few(a) || groups < 1) return hipErrorInvalidValue;
  I8Args aa = a;
  ResidentArgs rr = r;
  void *args[] = {&aa, &rr};
  return hipLaunchCooperativeKernel(i8_resident(a), dim3(groups), dim3(I8Int::NT), args, 0, s);
}

hipError_t launch_i8_prepare(const I8Args &a, hipStream_t s) {
  if (a.r_pad % PREP_R || a.ld % 128 || a.ld % a.bm) return hipErrorInvalidValue;
  i8_prepare_kernel<<<a.r_pad / PREP_R, 512, 0, s>>>(a);
  return hipGetLastError();
}

hipError_t launch_i8_rows(const float *J, int32_t n, int32_t *jexp, int32_t *flags,
                          hipStream_t s) {
  if (n < 1) return hipErrorInvalidValue;
  i8_rows_kernel<<<(n + 3) / 4, 256, 0, s>>>(J, n, jexp, flags);
  return hipGetLastError();
}

hipError_t launch_i8_pack_j(const float *J, int32_t ld, const int32_t *jexp, uint8_t *out,
                            hipStream_t s) {
  const int64_t blocks = (int64_t)(ld / 32) * (ld / 32);
  const int wg = (int)std::min<int64_t>((blocks + 3) / 4, 8192);
  if (jexp)
    i8_pack_j_kernel<I8_JDIGITS><<<wg, 256, 0, s>>>(J, ld, blocks, jexp, out);
  else
    i8_pack_j_kernel<1><<<wg, 256, 0, s>>>(J, ld, blocks, jexp, out);
  return hipGetLastError();
}

}  // namespace si

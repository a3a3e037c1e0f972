// Split contraction for problems with fewer output tiles than CUs.
//
// With R = 64 replicas and N = 2000 spins the coupling product J.Q has
// only 2048 x 64 outputs: 128 tiles of 32 x 32 leave half the CUs idle and
// each tile runs through the whole contraction.  Here the contraction is cut
// into S ranges of k; launch 1 computes every (tile, range) product into a
// workspace W[s][r_pad][n_pad] (S times as many workgroups, each S times
// shorter), and launch 2 adds the S partial products in a fixed order
// (deterministic) and applies the update of Eq. (8) with the walls, or the
// adjoint's multiplier update, element by element in the state's layout.
// Where few tiles make it worth it (few_fits), one launch does both.
#include "si_epilogue.h"
#include "si_f32_gemm.h"

namespace si {

// Partial products of one (tile, range) work item.  BMODE = B_MASKED
// multiplies the position operand by the momentum-wall bit of `mask` (the
// adjoint's J vb).
template <class C, int BMODE>
__global__ __launch_bounds__(C::NT) void coupling_partial_kernel(const float *__restrict__ J,
                                                                 const float *__restrict__ X,
                                                                 const uint8_t *__restrict__ mask,
                                                                 int ld, int r_pad, int K,
                                                                 int klen, float *__restrict__ W) {
  __shared__ __attribute__((aligned(16))) float smem[C::LDS_FLOATS];
  using T = EpiTile<C::BM, C::BN, C::NT>;
  static_assert(T::BYTES <= C::LDS_FLOATS * 4, "the partial tile fits in the main loop's LDS");
  const int ncol = r_pad / C::BN, tiles = (ld / C::BM) * ncol;
  const int b = xcd_tile(blockIdx.x, gridDim.x);
  const int t = b % tiles, s = b / tiles;
  const int m0 = (t / ncol) * C::BM, n0 = (t % ncol) * C::BN;
  const int k0 = s * klen;
  const int kl = K - k0 < klen ? K - k0 : klen;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wy = wave / C::WN, wx = wave % C::WN;
  constexpr int G = C::M::NACC / 4;
  typename C::acc_t acc[C::TM][C::TN];
  if (kl > 0) {
    if constexpr (C::STAGES > 0 && BMODE == B_PLAIN)
      f32_mainloop_dma<C>(J + k0, X + k0, ld, kl, m0, n0, acc, smem);
    else
      f32_mainloop<C, BMODE>(J + k0, X + k0, ld, kl, m0, n0, acc, smem,
                             BMODE == B_MASKED ? mask + k0 : nullptr);
  } else {
#pragma unroll
    for (int i = 0; i < C::TM; ++i)
#pragma unroll
      for (int j = 0; j < C::TN; ++j)
#pragma unroll
        for (int v = 0; v < C::M::NACC; ++v) acc[i][j][v] = 0.f;
  }
#pragma unroll
  for (int i = 0; i < C::TM; ++i)
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int j = 0; j < C::TN; ++j)
        epi_put(smem, T::LD, wy * C::WTM + i * C::MB + g * 8 + (lane / C::MB) * 4,
                wx * C::WTN + j * C::MB + (lane % C::MB), acc[i][j][4 * g], acc[i][j][4 * g + 1],
                acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
  __syncthreads();
  float *w = W + (size_t)s * r_pad * ld;
#pragma unroll
  for (int c = 0; c < T::CPT; ++c) {
    const int col = T::col(c), row = T::row(c);
    *reinterpret_cast<floatx4 *>(w + (size_t)(n0 + col) * ld + m0 + row) =
        *reinterpret_cast<const floatx4 *>(smem + col * T::LD + row);
  }
}

// Sum of the S partial products at element offset off (chunk of four).
__device__ __forceinline__ floatx4 split_sum(const float *__restrict__ W, int64_t plane, int S,
                                             int64_t off) {
  floatx4 f = *reinterpret_cast<const floatx4 *>(W + off);
  for (int s = 1; s < S; ++s) f += *reinterpret_cast<const floatx4 *>(W + s * plane + off);
  return f;
}

// Update of Eq. (8) with the walls for four elements; returns the wall mask
// (if the launch records it).
template <int ORDER, int WALL>
__device__ __forceinline__ uint32_t split_update(const StepArgs &a, floatx4 q4, floatx4 p4,
                                                 floatx4 f, floatx4 h4, float dt, float zeta,
                                                 floatx4 &qn, floatx4 &pn) {
  uint32_t mk = 0;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    float qv, pv;
    spring_update<ORDER, WALL>(q4[v], p4[v], f[v] + h4[v], dt, zeta, a.k, a.inv_m, a.qmax, a.pmax,
                               qv, pv);
    qn[v] = qv;
    pn[v] = pv;
    if (a.mask_out) {
      // the unclamped values, recomputed exactly as in spring_update()
      const float cc = dt * a.inv_m;
      const float force = fmaf(zeta, f[v] + h4[v], -a.k * q4[v]);
      const float vv = fmaf(dt, force, p4[v]);
      const float uu = fmaf(cc, p4[v], q4[v]);
      mk |= ((fabsf(uu) <= a.qmax ? 1u : 0u) | (fabsf(vv) <= a.pmax ? 2u : 0u)) << (8 * v);
    }
  }
  return mk;
}

// The same for every element, F from the partials.
template <int ORDER, int WALL>
__global__ __launch_bounds__(256) void update_split_kernel(StepArgs a, const float *__restrict__ W,
                                                           int S) {
  const int64_t plane = (int64_t)a.r_pad * a.ld, chunks = plane / 4;
  const float dt = a.dt[a.t], zeta = a.zeta[a.t];
  for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c < chunks;
       c += (int64_t)gridDim.x * blockDim.x) {
    const int64_t off = c * 4;
    const int row = (int)(off % a.ld);
    const floatx4 f = split_sum(W, plane, S, off);
    floatx4 h4 = {0.f, 0.f, 0.f, 0.f};
    if (a.h) h4 = *reinterpret_cast<const floatx4 *>(a.h + row);
    const floatx4 q4 = *reinterpret_cast<const floatx4 *>(a.q_in + off);
    const floatx4 p4 = *reinterpret_cast<const floatx4 *>(a.p_in + off);
    floatx4 qn, pn;
    const uint32_t mk = split_update<ORDER, WALL>(a, q4, p4, f, h4, dt, zeta, qn, pn);
    *reinterpret_cast<floatx4 *>(a.q_out + off) = qn;
    *reinterpret_cast<floatx4 *>(a.p_out + off) = pn;
    if (a.mask_out) *reinterpret_cast<uint32_t *>(a.mask_out + off) = mk;
  }
}

struct AdjArgs {
  const float *J, *lamq_in, *lamp_in;
  const uint8_t *mask, *mask_next;  // wall bits of the step; null or of the step after
  const float *qn, *pn;             // the state before the step
  float *lamq_out, *lamp_out;
  double *part;          // three partial sums per workgroup
  const float *dt, *zeta;
  int n, ld, r_pad;      // n: the step
  float k, inv_m;
};

// Adjoint multiplier update of four elements with G = J vb; adds their
// <ub, p_n>, <vb, q_n>, <G, q_n> to s.  The next backward step only ever uses
// the multipliers behind its own walls, so where its wall bits are known
// already (mask_next) they are applied here, and its product then reads
// plain operands.
__device__ __forceinline__ void adj_update4(const AdjArgs &a, floatx4 G, int64_t off,
                                            double (&s)[3]) {
  const float dt = a.dt[a.n], zeta = a.zeta[a.n];
  const float c = dt * a.inv_m;
  const floatx4 lq = *reinterpret_cast<const floatx4 *>(a.lamq_in + off);
  const floatx4 lp = *reinterpret_cast<const floatx4 *>(a.lamp_in + off);
  const floatx4 q4 = *reinterpret_cast<const floatx4 *>(a.qn + off);
  const floatx4 p4 = *reinterpret_cast<const floatx4 *>(a.pn + off);
  const uint32_t mk = *reinterpret_cast<const uint32_t *>(a.mask + off);
  floatx4 oq, op;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const uint32_t b = mk >> (8 * v);
    const float ub = (b & 1u) ? lq[v] : 0.f;
    const float vb = (b & 2u) ? lp[v] : 0.f;
    oq[v] = fmaf(dt * zeta, G[v], fmaf(-dt * a.k, vb, ub));
    op[v] = fmaf(c, ub, vb);
    s[0] += (double)ub * (double)p4[v];
    s[1] += (double)vb * (double)q4[v];
    s[2] += (double)G[v] * (double)q4[v];
  }
  if (a.mask_next) {
    const uint32_t next = *reinterpret_cast<const uint32_t *>(a.mask_next + off);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      oq[v] = (next >> (8 * v) & 1u) ? oq[v] : 0.f;
      op[v] = (next >> (8 * v) & 2u) ? op[v] : 0.f;
    }
  }
  *reinterpret_cast<floatx4 *>(a.lamq_out + off) = oq;
  *reinterpret_cast<floatx4 *>(a.lamp_out + off) = op;
}

// Adjoint multiplier update with G = J vb from the partials; FP64 partial
// sums per workgroup (fixed order).
__global__ __launch_bounds__(256) void adj_update_split_kernel(AdjArgs a,
                                                               const float *__restrict__ W,
                                                               int S) {
  __shared__ double red[3][4];
  const int64_t plane = (int64_t)a.r_pad * a.ld, chunks = plane / 4;
  double s[3] = {0.0, 0.0, 0.0};
  for (int64_t ch = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; ch < chunks;
       ch += (int64_t)gridDim.x * blockDim.x)
    adj_update4(a, split_sum(W, plane, S, ch * 4), ch * 4, s);
  double s0 = s[0], s1 = s[1], s2 = s[2];
  // workgroup sums: fixed shuffle and wave order
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    s0 += __shfl_xor(s0, off);
    s1 += __shfl_xor(s1, off);
    s2 += __shfl_xor(s2, off);
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
    red[0][wave] = s0;
    red[1][wave] = s1;
    red[2][wave] = s2;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double *o = a.part + (size_t)blockIdx.x * 3;
#pragma unroll
    for (int q = 0; q < 3; ++q) o[q] = red[q][0] + red[q][1] + red[q][2] + red[q][3];
  }
}

// ---------------------------------------------------------------------------
// One-launch form for few replicas: a workgroup owns an MB x 32 output tile
// and holds all S ranges of its contraction, one wave per range, so that the
// partial products meet in LDS, are added there in the order of the ranges
// and the update follows in the same launch.  No two waves share an operand:
// each copies its own slabs of J and X into a ring of its own, several ahead,
// and waits for its copies alone, without a barrier in the loop.  (Reading the
// operands straight into registers takes 64 cycles an instruction instead of
// 16: the matrix layout puts neighbouring lanes on different rows.)  The
// products, their order and the order of the sums are the two-launch form's,
// bit for bit.  MB is the matrix block edge of the tile it stands in for, MW
// the most waves (ranges) of a workgroup.
//
// Measured (us per step, two launches before): N = 2000, R = 50 9.4 (12.5), N =
// 1000, R = 64 6.7 (8.8), N = 300, R = 8 5.2 (6.8), N = 2000, R = 128 13.2
// (17.6), N = 4000, R = 64 26.1 (26.3).  Bound at N = 2000, R = 50: the products
// take 3.9 us at the FP32 matrix rate, a launch 2.5 .. 3, its first copies and
// its update the rest.
// ---------------------------------------------------------------------------
constexpr int FEW_MAX = 8;  // ranges, at most
constexpr int ADJ_FEW_MB = 16;

template <int MB_, int MW_, bool MASKED_ = false>
struct FewCfg {
  static constexpr int MB = MB_, MW = MW_;
  static constexpr bool MASKED = MASKED_;
  static constexpr int BM = MB, BN = 32, TN = BN / MB, BK = 32;
  static constexpr int KSTEP = 64 / MB * 4;  // contraction indices per step of four products
  static constexpr int SLAB = (BM + BN) * BK + (MASKED ? BN * BK / 4 : 0);  // floats
  static constexpr int L = (BM + BN) / 8 + (MASKED ? 1 : 0);  // 1 KB copies
  static constexpr int SLOTS = 147456 / 4 / MW / SLAB;        // (of 160 KB)
  static constexpr int RING = SLOTS * SLAB;
  static constexpr int LDT = BM + 4;          // floats per column of a partial product
  static constexpr int CHUNKS = BM / 4 * BN;  // of four spins
  static constexpr int CPT = CHUNKS / 128;    // per thread, at two waves
  using M = MfmaF32<MB>;
  using acc_t = typename M::acc_t;
  static_assert(SLOTS >= 2 && BN * LDT <= RING && (SLOTS - 1) * L <= 63, "ring");
};

// Partial product of this wave's range, left in the wave's own LDS.
template <class C>
__device__ __forceinline__ void few_product(const float *__restrict__ J,
                                            const float *__restrict__ X,
                                            const uint8_t *__restrict__ mask, int ld, int kl,
                                            int m0, int n0, float *__restrict__ ring) {
  constexpr int MB = C::MB, TN = C::TN, S = C::SLOTS, NA = C::BM / 8, NB = C::BN / 8;
  const int lane = threadIdx.x & 63, lrow = lane % MB, lk = lane / MB * 4;
  // copies: lane L fetches the 16-byte chunk that belongs at its place
  // (chunk c of row r is stored at c ^ lds_swz(r))
  const int drow = lane / 8, dch = lane % 8;
  const float *src[NA + NB];
#pragma unroll
  for (int d = 0; d < NA + NB; ++d) {
    const int row = (d < NA ? d : d - NA) * 8 + drow;
    src[d] = (d < NA ? J + (size_t)(m0 + row) * ld : X + (size_t)(n0 + row) * ld) +
             (dch ^ lds_swz<8>(row)) * 4;
  }
  const uint8_t *srcm = C::MASKED ? mask + (size_t)(n0 + lane / 2) * ld + lane % 2 * 16 : nullptr;
  auto issue = [&](int kt, int slot) {
    float *st = ring + slot * C::SLAB;
#pragma unroll
    for (int d = 0; d < NA + NB; ++d)
      __builtin_amdgcn_global_load_lds((gbl_void_t *)(src[d] + kt * C::BK),
                                       (lds_void_t *)(st + d * 8 * C::BK), 16, 0, 0);
    if (C::MASKED)
      __builtin_amdgcn_global_load_lds((gbl_void_t *)(srcm + kt * C::BK),
                                       (lds_void_t *)(st + (NA + NB) * 8 * C::BK), 16, 0, 0);
  };
  typename C::acc_t acc[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int v = 0; v < C::M::NACC; ++v) acc[j][v] = 0.f;
  const int nk = kl > 0 ? kl / C::BK : 0;
#pragma unroll
  for (int i = 0; i < S - 1; ++i)
    if (i < nk) issue(i, i);
  int rd = 0, wr = S - 1;
  for (int kt = 0; kt < nk; ++kt) {
    // this slab has landed (its successors are still under way), and the one
    // before it has been read: its slot is filled below.  No other wave reads
    // this ring, so the wave's own wait is all that takes.
    if (kt + S - 1 < nk)
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((S - 2) * C::L) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    const float *st = ring + rd * C::SLAB;
    floatx4 a[C::BK / C::KSTEP], b[C::BK / C::KSTEP][TN];
#pragma unroll
    for (int u = 0; u < C::BK / C::KSTEP; ++u) {
      const int ch = (u * C::KSTEP + lk) / 4;
      a[u] = *reinterpret_cast<const floatx4 *>(st + lrow * C::BK + ((ch ^ lds_swz<8>(lrow)) << 2));
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int r = j * MB + lrow;
        b[u][j] = *reinterpret_cast<const floatx4 *>(st + (C::BM + r) * C::BK +
                                                     ((ch ^ lds_swz<8>(r)) << 2));
        if (C::MASKED) {
          const uint32_t mk = *reinterpret_cast<const uint32_t *>(
              reinterpret_cast<const uint8_t *>(st + (C::BM + C::BN) * C::BK) + r * C::BK +
              u * C::KSTEP + lk);
#pragma unroll
          for (int v = 0; v < 4; ++v) b[u][j][v] = (mk & (2u << (8 * v))) ? b[u][j][v] : 0.f;
        }
      }
    }
    // (the slot filled here has been read, see the wait above)
    if (kt + S - 1 < nk) issue(kt + S - 1, wr);
    wr = wr + 1 == S ? 0 : wr + 1;
    rd = rd + 1 == S ? 0 : rd + 1;
#pragma unroll
    for (int u = 0; u < C::BK / C::KSTEP; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[j] = C::M::mma(a[u][v], b[u][j][v], acc[j]);
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the ring has been read
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int g = 0; g < C::M::NACC / 4; ++g)
      *reinterpret_cast<floatx4 *>(ring + (j * MB + lrow) * C::LDT + g * 8 + lk) =
          floatx4{acc[j][4 * g], acc[j][4 * g + 1], acc[j][4 * g + 2], acc[j][4 * g + 3]};
}

// Sum of the S partial products at column col, rows row .. row + 3.
template <class C>
__device__ __forceinline__ floatx4 few_sum(const float *parts, int S, int col, int row) {
  const float *w = parts + col * C::LDT + row;
  floatx4 f = *reinterpret_cast<const floatx4 *>(w);
  for (int s = 1; s < S; ++s)
    f += *reinterpret_cast<const floatx4 *>(w + s * C::RING);
  return f;
}

// This workgroup's tile; wave s takes range s of the contraction.
#define SI_FEW_TILE(C)                                                                     \
  __shared__ __attribute__((aligned(16))) float parts[C::MW * C::RING];                 \
  const int ncol = r_pad / C::BN, t = xcd_tile(blockIdx.x, gridDim.x), S = blockDim.x >> 6; \
  const int m0 = (t / ncol) * C::BM, n0 = (t % ncol) * C::BN;                               \
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), k0 = wave * klen; \
  const int kl = K - k0 < klen ? K - k0 : klen;                                             \
  float *part = parts + wave * C::RING

template <class C, int ORDER, int WALL>
__global__ __launch_bounds__(64 * C::MW) void step_few_kernel(StepArgs a, int K, int klen) {
  constexpr int MB = C::MB;
  const int r_pad = a.r_pad;
  SI_FEW_TILE(C);
  floatx4 q4[C::CPT], p4[C::CPT];
#pragma unroll
  for (int c = 0; c < C::CPT; ++c) {
    const int u = c * blockDim.x + threadIdx.x;
    if (u < C::CHUNKS) {
      const size_t off = (size_t)(n0 + u / (MB / 4)) * a.ld + m0 + u % (MB / 4) * 4;
      q4[c] = *reinterpret_cast<const floatx4 *>(a.q_in + off);
      p4[c] = *reinterpret_cast<const floatx4 *>(a.p_in + off);
    }
  }
  few_product<C>(a.J + k0, a.q_in + k0, nullptr, a.ld, kl, m0, n0, part);
  const float dt = a.dt[a.t], zeta = a.zeta[a.t];
  __syncthreads();
#pragma unroll
  for (int c = 0; c < C::CPT; ++c) {
    const int u = c * blockDim.x + threadIdx.x;
    if (u >= C::CHUNKS) break;
    const int col = u / (MB / 4), row = u % (MB / 4) * 4;
    const size_t off = (size_t)(n0 + col) * a.ld + m0 + row;
    const floatx4 f = few_sum<C>(parts, S, col, row);
    floatx4 h4 = {0.f, 0.f, 0.f, 0.f};
    if (a.h) h4 = *reinterpret_cast<const floatx4 *>(a.h + m0 + row);
    floatx4 qn, pn;
    const uint32_t mk =
        split_update<ORDER, WALL>(a, q4[c], p4[c], f, h4, dt, zeta, qn, pn);
    *reinterpret_cast<floatx4 *>(a.q_out + off) = qn;
    *reinterpret_cast<floatx4 *>(a.p_out + off) = pn;
    if (a.mask_out) *reinterpret_cast<uint32_t *>(a.mask_out + off) = mk;
  }
}

// The adjoint's backward step: G = J vb and the multiplier update.
template <class C>
__global__ __launch_bounds__(64 * C::MW) void adj_few_kernel(AdjArgs a, int K, int klen) {
  constexpr int MB = C::MB;
  const int r_pad = a.r_pad;
  __shared__ double red[3][C::MW];
  SI_FEW_TILE(C);
  few_product<C>(a.J + k0, a.lamp_in + k0, a.mask + k0, a.ld, kl, m0, n0, part);
  __syncthreads();
  double s[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int c = 0; c < C::CPT; ++c) {
    const int u = c * blockDim.x + threadIdx.x;
    if (u >= C::CHUNKS) break;
    const int col = u / (MB / 4), row = u % (MB / 4) * 4;
    adj_update4(a, few_sum<C>(parts, S, col, row), (size_t)(n0 + col) * a.ld + m0 + row, s);
  }
  // workgroup sums: fixed shuffle and wave order
#pragma unroll
  for (int q = 0; q < 3; ++q) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s[q] += __shfl_xor(s[q], off);
    if ((threadIdx.x & 63) == 0) red[q][wave] = s[q];
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    double o = red[threadIdx.x][0];
    for (int w = 1; w < S; ++w) o += red[threadIdx.x][w];
    a.part[(size_t)blockIdx.x * 3 + threadIdx.x] = o;
  }
}

// The one-launch form stands in for a tile of MB x MB matrix blocks with S
// ranges where one workgroup per CU (its rings fill the LDS) holds all tiles,
// or two in turn of four waves or more with the larger blocks up to N = 4096
// (us per step, two launches against one: N = 2000, R = 200 26.9 against 23.5,
// N = 4000, R = 128 42.3 against 41.7).  Beyond, the larger tiles of the
// two-launch form fetch less: N = 8000, R = 64 76.2 against 79.7; and two
// waves leave a CU half empty: N = 1000, R = 200 12.6 against 16.1.
static bool few_fits(int32_t n_pad, int32_t r_pad, int32_t mb, int32_t S) {
  if (S < 2 || S > FEW_MAX || n_pad % mb || r_pad % 32) return false;
  const int64_t groups = (int64_t)(n_pad / mb) * (r_pad / 32);
  return groups <= 256 || (groups <= 512 && S >= 4 && mb == 32 && n_pad <= 4096);
}

// Tiles of the step kernel with a split form: the automatic choices for
// problems with fewer tiles than CUs.
#define SI_HAS_SPLIT(id) \
  ((id) == 3 || (id) == 6 || (id) == 12 || (id) == 2 || (id) == 14 || (id) == 9 || (id) == 26 || \
   (id) == 27)

// Depth of the contraction and of a range, in whole slabs of bk.
static void split_ranges(int32_t n, int32_t ld, int32_t ksplit, int32_t bk, int *K, int *klen) {
  const int up = (n + bk - 1) / bk * bk;
  *K = up < ld ? up : ld;
  const int per = (*K + ksplit - 1) / ksplit;
  *klen = (per + bk - 1) / bk * bk;
}

template <class C, int ORDER, int WALL>
static hipError_t split_step_as(const StepArgs &a, hipStream_t s) {
  int K, klen;
  split_ranges(a.n, a.ld, a.ksplit, C::BK, &K, &klen);
  if (few_fits(a.n_pad, a.r_pad, C::MB, a.ksplit)) {
    const int groups = (a.n_pad / C::MB) * (a.r_pad / 32);
    if (a.ksplit <= 4)
      step_few_kernel<FewCfg<C::MB, 4>, ORDER, WALL><<<groups, 64 * a.ksplit, 0, s>>>(a, K, klen);
    else
      step_few_kernel<FewCfg<C::MB, 8>, ORDER, WALL><<<groups, 64 * a.ksplit, 0, s>>>(a, K, klen);
    return hipGetLastError();
  }
  if (!a.fsplit) return hipErrorInvalidValue;
  const int tiles = (a.n_pad / C::BM) * (a.r_pad / C::BN);
  coupling_partial_kernel<C, B_PLAIN><<<tiles * a.ksplit, C::NT, 0, s>>>(
      a.J, a.q_in, nullptr, a.ld, a.r_pad, K, klen, a.fsplit);
  const int64_t chunks = (int64_t)a.r_pad * a.ld / 4;
  int64_t blocks = (chunks + 255) / 256;
  if (blocks > 2048) blocks = 2048;
  update_split_kernel<ORDER, WALL><<<(int)blocks, 256, 0, s>>>(a, a.fsplit, a.ksplit);
  return hipGetLastError();
}

template <class C>
static hipError_t split_step(const StepArgs &a, hipStream_t s) {
  if (a.n_pad % C::BM || a.r_pad % C::BN || a.ld % C::BK || a.ksplit < 2)
    return hipErrorInvalidValue;
  switch (a.order * 2 + a.wall) {
    case 0: return split_step_as<C, SI_ORDER_PAPER, SI_WALL_CLAMP>(a, s);
    case 1: return split_step_as<C, SI_ORDER_PAPER, SI_WALL_INELASTIC>(a, s);
    case 2: return split_step_as<C, SI_ORDER_SYMPLECTIC, SI_WALL_CLAMP>(a, s);
    case 3: return split_step_as<C, SI_ORDER_SYMPLECTIC, SI_WALL_INELASTIC>(a, s);
    default: return hipErrorInvalidValue;
  }
}

bool tile_has_split(int32_t tile) {
  switch (tile) {
#define SI_HS(id, bm, bn, wm, wn, mb, bk, st, ks) \
  case id:                                       \
    return SI_HAS_SPLIT(id);
    SI_F32_TILES(SI_HS)
#undef SI_HS
    default: return false;
  }
}

hipError_t launch_step_f32_split(int32_t tile, const StepArgs &a, hipStream_t s) {
  switch (tile) {
#define SI_SL(id, bm, bn, wm, wn, mb, bk, st, ks)                              \
  case id:                                                                    \
    if constexpr (SI_HAS_SPLIT(id))                                           \
      return split_step<F32Cfg<bm, bn, wm, wn, mb, bk, st, ks>>(a, s);        \
    else                                                                      \
      return hipErrorInvalidValue;
    SI_F32_TILES(SI_SL)
#undef SI_SL
    default: return hipErrorInvalidValue;
  }
}

// Adjoint backward step with the split contraction (32 x 32 tiles of the
// 16x16x4 MFMA, register-staged, masked position operand).
using ASplitCfg = F32Cfg<ADJ_BM, ADJ_BN, 2, 2, 16, 32, 0, 1>;

int32_t adj_split_groups(int32_t n_pad, int32_t r_pad, int32_t ksplit) {
  if (few_fits(n_pad, r_pad, ADJ_FEW_MB, ksplit)) return (n_pad / ADJ_FEW_MB) * (r_pad / 32);
  const int64_t chunks = (int64_t)n_pad * r_pad / 4;
  int64_t blocks = (chunks + 255) / 256;
  return (int32_t)(blocks > 1024 ? 1024 : blocks);
}

// Matrix block edge of a tile (0: no such tile).
static int32_t tile_mb(int32_t tile) {
  switch (tile) {
#define SI_MB(id, bm, bn, wm, wn, mb, bk, st, ks) \
  case id: return mb;
    SI_F32_TILES(SI_MB)
#undef SI_MB
    default: return 0;
  }
}

int32_t split_few_rows(int32_t tile, int32_t n_pad, int32_t r_pad, int32_t ksplit) {
  const int32_t mb = tile_mb(tile);
  return mb && few_fits(n_pad, r_pad, mb, ksplit) ? mb : 0;
}

// Partial products that a split step or backward step keeps in memory.
int64_t split_workspace(int32_t tile, int32_t n_pad, int32_t r_pad, int32_t ksplit) {
  if (ksplit < 2 || !tile_mb(tile) || split_few_rows(tile, n_pad, r_pad, ksplit)) return 0;
  return (int64_t)ksplit * n_pad * r_pad;
}

int64_t adj_split_workspace(int32_t n_pad, int32_t r_pad, int32_t ksplit) {
  return ksplit < 2 || few_fits(n_pad, r_pad, ADJ_FEW_MB, ksplit) ? 0
                                                                  : (int64_t)ksplit * n_pad * r_pad;
}

hipError_t launch_adj_step_split(const float *J, const float *lamq_in, const float *lamp_in,
                                 const uint8_t *mask, bool masked, const uint8_t *mask_next,
                                 const float *q_n, const float *p_n, float *lamq_out,
                                 float *lamp_out, double *part, const float *dt, const float *zeta,
                                 int32_t n, float k, float inv_m, int32_t n_pad, int32_t n_spins,
                                 int32_t r_pad, int32_t ksplit, float *W, hipStream_t s) {
  using C = ASplitCfg;
  static_assert(C::MB == ADJ_FEW_MB, "same products");
  if (n_pad % C::BM || r_pad % C::BN || ksplit < 2) return hipErrorInvalidValue;
  int K, klen;
  split_ranges(n_spins, n_pad, ksplit, C::BK, &K, &klen);
  const AdjArgs a{J,    lamq_in, lamp_in, mask, mask_next, q_n,   p_n, lamq_out, lamp_out,
                  part, dt,      zeta,    n,    n_pad,     r_pad, k,   inv_m};
  const int groups = adj_split_groups(n_pad, r_pad, ksplit);
  if (few_fits(n_pad, r_pad, ADJ_FEW_MB, ksplit)) {
    const int nt = 64 * ksplit;
    if (ksplit <= 4 && masked)
      adj_few_kernel<FewCfg<ADJ_FEW_MB, 4>><<<groups, nt, 0, s>>>(a, K, klen);
    else if (ksplit <= 4)
      adj_few_kernel<FewCfg<ADJ_FEW_MB, 4, true>><<<groups, nt, 0, s>>>(a, K, klen);
    else if (masked)
      adj_few_kernel<FewCfg<ADJ_FEW_MB, 8>><<<groups, nt, 0, s>>>(a, K, klen);
    else
      adj_few_kernel<FewCfg<ADJ_FEW_MB, 8, true>><<<groups, nt, 0, s>>>(a, K, klen);
    return hipGetLastError();
  }
  if (!W) return hipErrorInvalidValue;
  const int tiles = (n_pad / C::BM) * (r_pad / C::BN);
  if (masked)
    coupling_partial_kernel<C, B_PLAIN><<<tiles * ksplit, C::NT, 0, s>>>(J, lamp_in, nullptr, n_pad,
                                                                          r_pad, K, klen, W);
  else
    coupling_partial_kernel<C, B_MASKED><<<tiles * ksplit, C::NT, 0, s>>>(J, lamp_in, mask, n_pad,
                                                                           r_pad, K, klen, W);
  adj_update_split_kernel<<<groups, 256, 0, s>>>(a, W, ksplit);
  return hipGetLastError();
}

}  // namespace si

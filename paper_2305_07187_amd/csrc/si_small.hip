// Many steps of a small problem in one launch.
//
// Up to N = 224 the couplings fit the registers of one workgroup: its waves
// hold their rows of J as the operands of v_mfma_f32_16x16x4_f32, 16 rows per
// row block, and q of 16 replicas passes from step to step through LDS.
// Replicas do not interact, so workgroups never wait for each other: no
// launch and no grid-wide barrier between steps.  Products, their order and
// the update are those of the FP32 tiles of 16 x 16 matrix blocks without a
// split, bit for bit.
//
// Bound: the products on one CU's matrix cores (2048 cycles a step at N =
// 128), then the chain LDS write, barrier, LDS read.  Measured (us per step, a
// launch each before): N = 20, R = 8 0.36 (3.8), N = 64, R = 64 0.48 (4.0), N =
// 100, R = 8 .. 2048 1.1 (4.7 .. 5.3), N = 160, R = 64 2.2 (5.0), N = 192, R =
// 2048 2.6 (7.0).
#include "si_epilogue.h"
#include "si_f32_gemm.h"

namespace si {

constexpr int SMALL_WAVES = 8, SMALL_COLS = 16;

template <int KB, int ORDER, int WALL>
__global__ __launch_bounds__(64 * SMALL_WAVES) void small_steps_kernel(StepArgs a, int steps) {
  constexpr int RB = (KB + SMALL_WAVES - 1) / SMALL_WAVES;  // row blocks of a wave
  constexpr int LD = KB * 16 + 4;  // floats per replica: conflict-free 16-byte reads
  __shared__ __attribute__((aligned(16))) float qs[2][SMALL_COLS * LD];
  const int lane = threadIdx.x & 63, lcol = lane & 15, lk = (lane >> 4) * 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int col = blockIdx.x * SMALL_COLS + lcol;
  floatx4 ja[RB][KB], q4[RB], p4[RB], h4[RB];
#pragma unroll
  for (int i = 0; i < RB; ++i) {
    const int rb = wave + i * SMALL_WAVES;
    if (rb >= KB) continue;
    const float *row = a.J + (size_t)(rb * 16 + lcol) * a.ld + lk;
#pragma unroll
    for (int k = 0; k < KB; ++k) ja[i][k] = *reinterpret_cast<const floatx4 *>(row + k * 16);
    const size_t off = (size_t)col * a.ld + rb * 16 + lk;
    q4[i] = *reinterpret_cast<const floatx4 *>(a.q_in + off);
    p4[i] = *reinterpret_cast<const floatx4 *>(a.p_in + off);
    h4[i] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (a.h) h4[i] = *reinterpret_cast<const floatx4 *>(a.h + rb * 16 + lk);
    *reinterpret_cast<floatx4 *>(qs[0] + lcol * LD + rb * 16 + lk) = q4[i];
  }
  float dt = a.dt[a.t], zeta = a.zeta[a.t];
  __syncthreads();
  for (int s = 0; s < steps; ++s) {
    const int t = a.t + (s + 1 < steps ? s + 1 : s);
    const float dt_next = a.dt[t], zeta_next = a.zeta[t];
    const float *src = qs[s & 1] + lcol * LD + lk;
    float *dst = qs[(s & 1) ^ 1] + lcol * LD + lk;
    floatx4 acc[RB];
#pragma unroll
    for (int i = 0; i < RB; ++i) acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (wave < KB) {
#pragma unroll
      for (int k = 0; k < KB; ++k) {
        const floatx4 b = *reinterpret_cast<const floatx4 *>(src + k * 16);
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
          for (int i = 0; i < RB; ++i)
            if (wave + i * SMALL_WAVES < KB)
              acc[i] = MfmaF32<16>::mma(ja[i][k][v], b[v], acc[i]);
      }
    }
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      const int rb = wave + i * SMALL_WAVES;
      if (rb >= KB) continue;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float qv, pv;
        spring_update<ORDER, WALL>(q4[i][v], p4[i][v], acc[i][v] + h4[i][v], dt, zeta, a.k,
                                   a.inv_m, a.qmax, a.pmax, qv, pv);
        q4[i][v] = qv;
        p4[i][v] = pv;
      }
      *reinterpret_cast<floatx4 *>(dst + rb * 16) = q4[i];
    }
    dt = dt_next;
    zeta = zeta_next;
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < RB; ++i) {
    const int rb = wave + i * SMALL_WAVES;
    if (rb >= KB) continue;
    const size_t off = (size_t)col * a.ld + rb * 16 + lk;
    *reinterpret_cast<floatx4 *>(a.q_out + off) = q4[i];
    *reinterpret_cast<floatx4 *>(a.p_out + off) = p4[i];
  }
  // the padding of the rows stays zero
  const int pad = (a.ld - KB * 16) / 4;
  for (int u = threadIdx.x; u < SMALL_COLS * pad; u += blockDim.x) {
    const size_t off =
        (size_t)(blockIdx.x * SMALL_COLS + u / pad) * a.ld + KB * 16 + u % pad * 4;
    *reinterpret_cast<floatx4 *>(a.q_out + off) = floatx4{0.f, 0.f, 0.f, 0.f};
    *reinterpret_cast<floatx4 *>(a.p_out + off) = floatx4{0.f, 0.f, 0.f, 0.f};
  }
}

template <int KB>
static hipError_t small_launch(const StepArgs &a, int32_t steps, hipStream_t s) {
  const int groups = a.r_pad / SMALL_COLS, nt = 64 * SMALL_WAVES;
  switch (a.order * 2 + a.wall) {
    case 0: small_steps_kernel<KB, SI_ORDER_PAPER, SI_WALL_CLAMP><<<groups, nt, 0, s>>>(a, steps); break;
    case 1: small_steps_kernel<KB, SI_ORDER_PAPER, SI_WALL_INELASTIC><<<groups, nt, 0, s>>>(a, steps); break;
    case 2: small_steps_kernel<KB, SI_ORDER_SYMPLECTIC, SI_WALL_CLAMP><<<groups, nt, 0, s>>>(a, steps); break;
    case 3: small_steps_kernel<KB, SI_ORDER_SYMPLECTIC, SI_WALL_INELASTIC><<<groups, nt, 0, s>>>(a, steps); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// For the tiles of 16 x 16 blocks, which the automatic choice takes up to N =
// 224 unless the replicas fill the chip with larger ones; up to 16 replicas
// per CU (4096) every workgroup runs at once.  One CU's matrix cores take
// N^2 / 8 cycles a step, so N = 224 still gains (3.8 us against 5.4 at R = 64
// and 7.9 at R = 2000), and N = 256, which the split form spreads over 32 CUs
// (5.2 us), would not.
bool small_fits(int32_t tile, int32_t n, int32_t r_pad) {
  switch (tile) {
#define SI_SMALL(id, bm, bn, wm, wn, mb, bk, st, ks) \
  case id:                                           \
    return mb == 16 && ks == 1 && n <= 224 && r_pad <= 4096;
    SI_F32_TILES(SI_SMALL)
#undef SI_SMALL
    default: return false;
  }
}

// The kernel's row blocks for n spins.
static int small_blocks(int32_t n) {
  const int kb = (n + 15) / 16;
  return kb == 7 ? 7 : (kb + 1) / 2 * 2;
}

int32_t small_rows(int32_t n) { return small_blocks(n) * 16; }

hipError_t launch_small_steps(const StepArgs &a, int32_t steps, hipStream_t s) {
  const int kb = small_blocks(a.n);
  // (row blocks beyond n lie in J's padding)
  if (steps < 1 || a.r_pad % SMALL_COLS || a.n < 1 || a.ld % 64 ||
      kb * 16 > a.ld || a.mask_out)
    return hipErrorInvalidValue;
  switch (kb) {
    case 2: return small_launch<2>(a, steps, s);
    case 4: return small_launch<4>(a, steps, s);
    case 6: return small_launch<6>(a, steps, s);
    case 7: return small_launch<7>(a, steps, s);
    case 8: return small_launch<8>(a, steps, s);
    case 10: return small_launch<10>(a, steps, s);
    case 12: return small_launch<12>(a, steps, s);
    case 14: return small_launch<14>(a, steps, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace si

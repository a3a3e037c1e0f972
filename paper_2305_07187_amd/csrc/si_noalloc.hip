// Exact Ising energy (Eq. 1) of caller-owned positions and couplings that
// allocates nothing: for callers that cannot allocate device memory (code
// under HIP graph capture, serving loops).  Its only scratch memory is the
// file-scope array below, one copy per GPU, held until the process ends.
//
// Energy of s = sign(x) (+1 for x >= 0, also -0.0) for every replica r:
//   E_r = -1/2 sum_i s_i sum_j J_ij s_j     (= -sum_{i<j} J_ij s_i s_j for a
//                                            symmetric, zero-diagonal J)
// G = J.S runs on the int8 matrix cores (v_mfma_i32_32x32x32_i8) with int32
// accumulation, exact for integer |J_ij| <= 127; the couplings are converted
// to int8 while they are staged into LDS, so J is read in the caller's FP32
// layout (n x n, unpadded) and the positions in theirs (r x n, unpadded).
// Per-replica sums of s_i G_i go to 64-bit integer atomics, whose result
// does not depend on their order, so the contraction may be split as well.
//
// Bound: every tile reads and converts its rows of J and x in FP32: 256 MB
// and 64 M elements at N = 2000, R = 1024, 9 us and 10 us on the L2s and the
// vector units, so tiles are large (128 x 128, the contraction split to fill
// the chip) and an element costs few instructions: four at a time from a
// 16-byte load, next slab's loads under way during the products, one 4-byte
// LDS write, one atomic per column and workgroup.  The three launches take
// 35.5 us there (282 with 64 x 64 tiles staged one element and one byte write
// at a time), 68 at N = 8000, R = 100 (1158), 197 at N = 4000, R = 2048 (751).
#include <atomic>

#include "si_internal.h"

namespace si {

typedef int intx4 __attribute__((ext_vector_type(4)));
typedef int intx16 __attribute__((ext_vector_type(16)));
// the caller's rows start on any float
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));

namespace {
// scratch: [0, NOALLOC_R_MAX) per-replica 64-bit sums; [NOALLOC_R_MAX] the
// flag of couplings outside the exact int8 range.
constexpr int NOALLOC_R_MAX = 65536;
constexpr int NB = 128, NK = 64, NLDK = NK + 16;  // tile 128 x 128, slab 64 deep (bytes)
constexpr int NNT = 512, NF4 = NB * NK / 4 / NNT;  // threads; 16-byte loads of each operand
}  // namespace

static __device__ __align__(256) unsigned long long scratch[NOALLOC_R_MAX + 32];

// Low bytes of four words, first word lowest.
__device__ __forceinline__ uint32_t low_bytes(const uint32_t (&w)[4]) {
  const uint32_t lo = __builtin_amdgcn_perm(w[1], w[0], 0x0C0C0400u);
  const uint32_t hi = __builtin_amdgcn_perm(w[3], w[2], 0x04000C0Cu);
  return lo | hi;
}

// Four couplings as int8, lowest first (flagging values that are not integers
// in [-127, 127]).  Adding 1.5 x 2^23 leaves an integer's two's complement in
// the low bits of the sum; the difference finds what is not one.
__device__ __forceinline__ uint32_t j_to_i8(floatx4u v, bool &bad) {
  uint32_t w[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float t = v[k] + 12582912.f;
    bad |= !(t - 12582912.f == v[k]) || !(fabsf(v[k]) <= 127.f);
    w[k] = __float_as_uint(t);
  }
  return low_bytes(w);
}

// sign(x) of four positions as int8 (entries beyond the matrix meet couplings
// staged as zero).
__device__ __forceinline__ uint32_t x_to_i8(floatx4u v) {
  uint32_t w[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) w[k] = v[k] < 0.f ? 0xFFu : 1u;
  return low_bytes(w);
}

// Entries k .. k + 3 of a row of n (zero beyond it).
__device__ __forceinline__ floatx4u load4(const float *row, int k, int n) {
  if (k + 3 < n) return *reinterpret_cast<const floatx4u *>(row + k);
  floatx4u v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < 3; ++j)
    if (k + j < n) v[j] = row[k + j];
  return v;
}

__global__ __launch_bounds__(NNT) void noalloc_energy_kernel(const float *__restrict__ J,
                                                             const float *__restrict__ x, int n,
                                                             int r, int klen,
                                                             unsigned long long *__restrict__ sc) {
  __shared__ __attribute__((aligned(16))) uint8_t As[2][NB * NLDK];
  __shared__ __attribute__((aligned(16))) uint8_t Bs[2][NB * NLDK];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wy = wave >> 1, wx = wave & 1;  // 4 x 2 waves of 32 x 64
  const int m0 = blockIdx.x * NB, n0 = blockIdx.y * NB;
  const int kb = blockIdx.z * klen, ke = min(kb + klen, n);
  bool bad = false;
  intx16 acc[2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[j][v] = 0;

  // staging: thread t takes four entries at column t % 16 * 4 of every
  // (t / 16 + 32 f)th row of both slabs
  const int srow = tid >> 4, sk = (tid & 15) * 4;
  // (rows beyond the matrix repeat its last one; their sums are not used)
  const float *pa[NF4], *pb[NF4];
#pragma unroll
  for (int f = 0; f < NF4; ++f) {
    pa[f] = J + (size_t)min(m0 + srow + 32 * f, n - 1) * n;
    pb[f] = x + (size_t)min(n0 + srow + 32 * f, r - 1) * n;
  }
  floatx4u ga[NF4], gb[NF4];
  auto load = [&](int k0) {
    if (k0 + NK <= n) {
#pragma unroll
      for (int f = 0; f < NF4; ++f) ga[f] = *reinterpret_cast<const floatx4u *>(pa[f] + k0 + sk);
#pragma unroll
      for (int f = 0; f < NF4; ++f) gb[f] = *reinterpret_cast<const floatx4u *>(pb[f] + k0 + sk);
    } else {
#pragma unroll
      for (int f = 0; f < NF4; ++f) {
        ga[f] = load4(pa[f], k0 + sk, n);
        gb[f] = load4(pb[f], k0 + sk, n);
      }
    }
  };
  auto stage = [&](int buf) {
#pragma unroll
    for (int f = 0; f < NF4; ++f) {
      const int off = (srow + 32 * f) * NLDK + sk;
      *reinterpret_cast<uint32_t *>(As[buf] + off) = j_to_i8(ga[f], bad);
      *reinterpret_cast<uint32_t *>(Bs[buf] + off) = x_to_i8(gb[f]);
    }
  };
  load(kb);
  stage(0);
  __syncthreads();
  const int lrow = lane & 31, lk = (lane >> 5) * 16;
  for (int k0 = kb, buf = 0; k0 < ke; k0 += NK, buf ^= 1) {
    const bool more = k0 + NK < ke;
    if (more) load(k0 + NK);
#pragma unroll
    for (int kk = 0; kk < NK; kk += 32) {
      const intx4 a =
          *reinterpret_cast<const intx4 *>(As[buf] + (wy * 32 + lrow) * NLDK + kk + lk);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const intx4 b =
            *reinterpret_cast<const intx4 *>(Bs[buf] + (wx * 64 + j * 32 + lrow) * NLDK + kk + lk);
        acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, acc[j], 0, 0, 0);
      }
    }
    if (more) stage(buf ^ 1);
    __syncthreads();
  }
  if (bad) atomicOr(sc + NOALLOC_R_MAX, 1ull);

  // sum_i s_i G_i over this wave's rows for each replica column, added up in
  // LDS over the four waves of a column: one atomic per column and workgroup
  __shared__ int sums[NB];
  if (tid < NB) sums[tid] = 0;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int lc = wx * 64 + j * 32 + (lane & 31), col = n0 + lc;
    int c = 0;
    if (col < r)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int row = m0 + wy * 32 + g * 8 + (lane >> 5) * 4;
        const floatx4u v = load4(x + (size_t)col * n, row, n);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (row + e < n) c += v[e] < 0.f ? -acc[j][4 * g + e] : acc[j][4 * g + e];
      }
    c += __shfl_xor(c, 32);
    if (lane < 32) atomicAdd(sums + lc, c);
  }
  __syncthreads();
  if (tid < NB && n0 + tid < r)
    atomicAdd(sc + n0 + tid, (unsigned long long)(long long)sums[tid]);
}

__global__ void noalloc_clear_kernel(unsigned long long *sc, int r) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < r; i += gridDim.x * blockDim.x)
    sc[i] = 0ull;
  if (blockIdx.x == 0 && threadIdx.x == 0) sc[NOALLOC_R_MAX] = 0ull;
}

// e_r = -(sum / 2); INT32_MIN when a coupling was outside the exact range or
// the energy does not fit in int32.
__global__ void noalloc_finalize_kernel(const unsigned long long *sc, int r, int32_t *e) {
  const int col = blockIdx.x * blockDim.x + threadIdx.x;
  if (col >= r) return;
  const long long s = (long long)sc[col];
  const long long v = -(s / 2);
  const bool ok = sc[NOALLOC_R_MAX] == 0ull && v >= INT32_MIN + 1LL && v <= INT32_MAX;
  e[col] = ok ? (int32_t)v : INT32_MIN;
}

int32_t noalloc_r_max() { return NOALLOC_R_MAX; }

// Device address of this GPU's scratch array, looked up once per device.
hipError_t noalloc_scratch_ptr(int device, void **ptr) {
  static void *table[64] = {nullptr};
  static std::atomic<int> lock{0};
  if (device < 0 || device >= 64) return hipErrorInvalidDevice;
  while (lock.exchange(1, std::memory_order_acquire)) {
  }
  hipError_t e = hipSuccess;
  if (!table[device]) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e == hipSuccess) table[device] = p;
  }
  *ptr = table[device];
  lock.store(0, std::memory_order_release);
  return e;
}

hipError_t launch_noalloc_energy(const float *J, const float *x, int32_t n, int32_t r,
                                 int32_t *e_int, void *sc_ptr, hipStream_t s) {
  if (n < 1 || r < 1 || r > NOALLOC_R_MAX || !sc_ptr) return hipErrorInvalidValue;
  auto *sc = static_cast<unsigned long long *>(sc_ptr);
  const int cb = (r + 255) / 256 < 256 ? (r + 255) / 256 : 256;
  noalloc_clear_kernel<<<cb, 256, 0, s>>>(sc, r);
  // contraction parts of at least four slabs, until every CU has a workgroup
  // (N = 2000, R = 1024: 35.5 us; two per CU 38.9, four 44.7)
  const int tn = (n + NB - 1) / NB, tr = (r + NB - 1) / NB, nk = (n + NK - 1) / NK;
  int parts = 256 / (tn * tr);
  parts = parts < nk / 4 ? parts : nk / 4;
  if (parts < 1) parts = 1;
  const int klen = (nk + parts - 1) / parts * NK;
  dim3 grid(tn, tr, (n + klen - 1) / klen);
  noalloc_energy_kernel<<<grid, NNT, 0, s>>>(J, x, n, r, klen, sc);
  noalloc_finalize_kernel<<<(r + 255) / 256, 256, 0, s>>>(sc, r, e_int);
  return hipGetLastError();
}

}  // namespace si

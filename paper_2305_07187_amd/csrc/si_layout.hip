// Staging kernels: validation of J, zero-padded packing of J and of the
// state into the device layout, and unpacking back to the caller's layout.
#include "si_internal.h"

namespace si {

__device__ __forceinline__ bool fp8_e4m3_exact(float v) {
  // e4m3 (no infinities): 1 sign, 4 exponent (bias 7), 3 mantissa bits;
  // normals 2^-6 .. 448, subnormals multiples of 2^-9.
  const float a = fabsf(v);
  if (a == 0.f) return true;
  if (!(a <= 448.f)) return false;
  if (a < 0.015625f) {  // subnormal range: a = m * 2^-9, m integer 1..7
    const float m = a * 512.f;
    return m == rintf(m);
  }
  int e;
  const float fr = frexpf(a, &e);  // a = fr * 2^e, fr in [0.5, 1)
  const float m = fr * 16.f;        // 4 significant bits
  return m == rintf(m);
}

// Checks of J (see launch_validate).  Workgroup (bi, bj), bi <= bj, takes the
// 64 x 64 tile (bi, bj) and its mirror image (bj, bi), both row by row, so
// that the comparison J_ij == J_ji costs no strided reads; the mirror tile
// passes through LDS (one float of padding per row: no bank conflicts).
// Bound: one pass over J.  N = 2000: 17.5 us, N = 8000: 103 us (383 and 1440
// with J_ji read at a stride of one row and a 64-bit division per element).
__global__ __launch_bounds__(256) void validate_kernel(const float *__restrict__ J, int n, int nt,
                                                       int32_t *flags) {
  __shared__ float mirror[64][65];
  __shared__ int found, most;
  int bi = 0, rest = blockIdx.x;  // row bi of the upper triangle has nt - bi tiles
  {
    // largest bi with bi nt - bi (bi - 1) / 2 <= rest
    const double b = nt + 0.5;
    bi = (int)(b - sqrt(b * b - 2.0 * (double)rest));
    while (bi > 0 && (int64_t)bi * nt - (int64_t)bi * (bi - 1) / 2 > rest) --bi;
    while ((int64_t)(bi + 1) * nt - (int64_t)(bi + 1) * bi / 2 <= rest) ++bi;
    rest -= (int)((int64_t)bi * nt - (int64_t)bi * (bi - 1) / 2);
  }
  const int i0 = bi * 64, j0 = (bi + rest) * 64, c = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (threadIdx.x == 0) found = most = 0;
  // bit k of mask: flag k
  int mask = 0, maxabs = 0;
  auto check = [&](float v, bool diagonal) {
    if (diagonal && v != 0.f) mask |= 1 << 1;
    if (!diagonal && v == 0.f) mask |= 1 << 7;
    if (!isfinite(v)) {
      mask |= 1 << 2;
      return;
    }
    if (v != rintf(v) || fabsf(v) > 127.f)
      mask |= 1 << 3;
    else
      maxabs = max(maxabs, (int)fabsf(v));
    if (!fp8_e4m3_exact(v)) mask |= 1 << 4;
    if ((__float_as_uint(v) & 0xFFFFu) != 0u) mask |= 1 << 5;
  };
  float up[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int row = w * 16 + k;
    up[k] = i0 + row < n && j0 + c < n ? J[(int64_t)(i0 + row) * n + j0 + c] : 0.f;
    mirror[row][c] = j0 + row < n && i0 + c < n ? J[(int64_t)(j0 + row) * n + i0 + c] : 0.f;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int row = w * 16 + k;
    if (i0 + row >= n || j0 + c >= n) continue;
    const float other = mirror[c][row];
    if (!(up[k] == other)) mask |= 1 << 0;
    check(up[k], i0 + row == j0 + c);
    check(other, i0 + row == j0 + c);
  }
  for (int off = 32; off >= 1; off >>= 1) {
    mask |= __shfl_xor(mask, off);
    maxabs = max(maxabs, __shfl_xor(maxabs, off));
  }
  if (c == 0 && mask) atomicOr(&found, mask);
  if (c == 0 && maxabs) atomicMax(&most, maxabs);
  __syncthreads();
  // (most workgroups find what others have found: they only look)
  if (threadIdx.x < 8) {
    const int k = threadIdx.x;
    if (k == 6) {
      if (most > __hip_atomic_load(flags + 6, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(flags + 6, most);
    } else if ((found >> k & 1) &&
               !__hip_atomic_load(flags + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
      atomicOr(flags + k, 1);
    }
  }
}

// ---------------------------------------------------------------------------
// Copies between the caller's rows of n and the device's rows of n_pad, one
// wave per row and four entries per lane, so that no entry's row has to be
// found by a division.  Both arrays of a state (and the BF16 planes that the
// precision forms read) and all instances of a batch go in one launch.
// Caller rows that start on 16 bytes move as vectors, others one entry per
// lane.  Bound: memory.  With one BF16 plane, N = 2000, R = 1024 set_state takes
// 8.4 us (20 in three launches with a division per entry), get_state 6.9
// (12); N = 8000, R = 2048 41 us (5.5 TB/s) and 43 us (6.1 TB/s); 256
// instances of N = 64 .. 4096, R = 64 one launch each way instead of 1280 of
// 2.6 us.
// ---------------------------------------------------------------------------
typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bool row_aligned(const void *p, int bytes) {
  return ((uintptr_t)p & (uintptr_t)(bytes - 1)) == 0;
}

// Entries i .. i + 3 of a row of n, zero beyond its end.
__device__ __forceinline__ floatx4 row_load(const float *src, int i, int n, bool aligned) {
  if (aligned && i + 3 < n) return *reinterpret_cast<const floatx4 *>(src + i);
  floatx4 v;
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = i + k < n ? src[i + k] : 0.f;
  return v;
}

__global__ __launch_bounds__(256) void pack_matrix_kernel(const float *__restrict__ src, int n,
                                                          float *__restrict__ dst,
                                                          int8_t *__restrict__ dst8, int n_pad) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  const float *from = src + (int64_t)row * n;
  const bool aligned = row_aligned(from, 16);
  for (int i = (blockIdx.y * 64 + lane) * 4; i < n_pad; i += gridDim.y * 256) {
    const floatx4 v = row_load(from, i, row < n ? n : 0, aligned);
    const int64_t off = (int64_t)row * n_pad + i;
    *reinterpret_cast<floatx4 *>(dst + off) = v;
    if (dst8)
      *reinterpret_cast<char4 *>(dst8 + off) = make_char4((int8_t)(int)v[0], (int8_t)(int)v[1],
                                                          (int8_t)(int)v[2], (int8_t)(int)v[3]);
  }
}

// This wave's row of the copy.
struct RowAt {
  const StateRows *d;
  int row, lane;
  __device__ __forceinline__ RowAt(const StateCopy &c) {
    const int groups = c.r_pad / 4, inst = blockIdx.x / groups;
    d = c.many ? c.many + inst : &c.one;
    row = (blockIdx.x - inst * groups) * 4 + (threadIdx.x >> 6);
    lane = threadIdx.x & 63;
  }
};

__global__ __launch_bounds__(256) void pack_rows_kernel(StateCopy c, const float *__restrict__ x,
                                                        const float *__restrict__ p) {
  const RowAt at(c);
  const int n = at.row < c.r ? at.d->n : 0, n_pad = at.d->n_pad;
  const int64_t from = at.d->off + (int64_t)at.row * at.d->n, to = (int64_t)at.row * n_pad;
  const bool ax = row_aligned(x + from, 16), ap = row_aligned(p + from, 16);
  float *q = at.d->q[c.cur] + to, *pp = at.d->p[c.cur] + to;
  uint16_t *qb = c.planes ? at.d->qb[c.cur] + to : nullptr;
  for (int i = (blockIdx.y * 64 + at.lane) * 4; i < n_pad; i += gridDim.y * 256) {
    floatx4 v = row_load(x + from, i, n, ax);
    const floatx4 w = row_load(p + from, i, p ? n : 0, ap);
    *reinterpret_cast<floatx4 *>(q + i) = v;
    *reinterpret_cast<floatx4 *>(pp + i) = w;
    for (int k = 0; k < c.planes; ++k) {
      ushort4 b;
      uint16_t *e = reinterpret_cast<uint16_t *>(&b);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t u = bf16_bits(v[j]);
        e[j] = (uint16_t)u;
        v[j] = v[j] - bf16_to_f32(u);
      }
      *reinterpret_cast<ushort4 *>(qb + k * at.d->plane + i) = b;
    }
  }
}

__device__ __forceinline__ void unpack_row(const float *src, float *dst, int n, int lane) {
  if (row_aligned(dst, 16)) {
    for (int i = (blockIdx.y * 64 + lane) * 4; i < n; i += gridDim.y * 256) {
      const floatx4 v = *reinterpret_cast<const floatx4 *>(src + i);
      if (i + 3 < n) {
        *reinterpret_cast<floatx4 *>(dst + i) = v;
      } else {
        for (int k = 0; k < 3; ++k)
          if (i + k < n) dst[i + k] = v[k];
      }
    }
    return;
  }
  for (int i0 = blockIdx.y * 256; i0 < n; i0 += gridDim.y * 256)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = i0 + k * 64 + lane;
      if (i < n) dst[i] = src[i];
    }
}

__global__ __launch_bounds__(256) void unpack_rows_kernel(StateCopy c, float *__restrict__ x,
                                                          float *__restrict__ p) {
  const RowAt at(c);
  if (at.row >= c.r) return;
  const int64_t from = (int64_t)at.row * at.d->n_pad, to = at.d->off + (int64_t)at.row * at.d->n;
  if (x) unpack_row(at.d->q[c.cur] + from, x + to, at.d->n, at.lane);
  if (p) unpack_row(at.d->p[c.cur] + from, p + to, at.d->n, at.lane);
}

// Spins into the caller's rows: the signs of q, or of the kept spins src8.
__global__ __launch_bounds__(256) void unpack_spins_kernel(StateCopy c,
                                                           const int8_t *__restrict__ src8,
                                                           int8_t *__restrict__ out,
                                                           const double *__restrict__ e_src,
                                                           double *__restrict__ e_out) {
  const RowAt at(c);
  if (at.row >= c.r) return;
  if (e_out && blockIdx.y == 0 && at.lane == 0) {
    const int64_t k = (int64_t)(blockIdx.x / (c.r_pad / 4)) * c.r + at.row;
    e_out[k] = e_src[k];
  }
  const int n = at.d->n;
  const int64_t from = (int64_t)at.row * at.d->n_pad;
  const float *q = at.d->q[c.cur] + from;
  if (src8) src8 += at.d->soff + from;
  int8_t *dst = out + at.d->off + (int64_t)at.row * n;
  const bool aligned = row_aligned(dst, 4);
  for (int i = (blockIdx.y * 64 + at.lane) * 4; i < n; i += gridDim.y * 256) {
    char4 s;
    if (src8) {
      s = *reinterpret_cast<const char4 *>(src8 + i);
    } else {
      const floatx4 v = *reinterpret_cast<const floatx4 *>(q + i);
      s = make_char4(v[0] < 0.f ? -1 : 1, v[1] < 0.f ? -1 : 1, v[2] < 0.f ? -1 : 1,
                     v[3] < 0.f ? -1 : 1);
    }
    if (aligned && i + 3 < n) {
      *reinterpret_cast<char4 *>(dst + i) = s;
    } else {
      dst[i] = s.x;
      if (i + 1 < n) dst[i + 1] = s.y;
      if (i + 2 < n) dst[i + 2] = s.z;
      if (i + 3 < n) dst[i + 3] = s.w;
    }
  }
}

__global__ void pack_field_kernel(const float *__restrict__ h, int n, float *__restrict__ hf,
                                  int8_t *__restrict__ h8, int n_pad, int32_t *flags) {
  int nonint = 0, nonfin = 0, maxabs = 0;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n_pad; i += gridDim.x * blockDim.x) {
    const float v = i < n ? h[i] : 0.f;
    hf[i] = v;
    if (!isfinite(v)) nonfin = 1;
    const bool integer = isfinite(v) && v == rintf(v) && fabsf(v) <= 127.f;
    if (!integer)
      nonint = 1;
    else
      maxabs = max(maxabs, (int)fabsf(v));
    h8[i] = integer ? (int8_t)(int)v : (int8_t)0;
  }
  if (nonfin) atomicOr(flags + 2, 1);
  if (nonint) atomicOr(flags + 3, 1);
  if (maxabs) atomicMax(flags + 6, maxabs);
}

static int grid_for(int64_t total) {
  int64_t b = (total + 255) / 256;
  if (b > 8192) b = 8192;
  return b < 1 ? 1 : (int)b;
}

hipError_t launch_validate(const float *J, int32_t n, int32_t *flags, hipStream_t s) {
  const int64_t nt = ((int64_t)n + 63) / 64, tiles = nt * (nt + 1) / 2;
  if (n < 1 || tiles > 0x7fffffff) return hipErrorInvalidValue;
  validate_kernel<<<(int)tiles, 256, 0, s>>>(J, n, (int)nt, flags);
  return hipGetLastError();
}

// Row groups of the copy, and slices of a row (256 entries or a multiple of
// it) until the launch has about 4096 workgroups.
static hipError_t rows_grid(int64_t groups, int32_t n_pad, dim3 *grid) {
  if (groups < 1 || groups > 0x7fffffff) return hipErrorInvalidValue;
  int64_t slices = (4096 + groups - 1) / groups;
  const int64_t most = (n_pad + 255) / 256;
  *grid = dim3((unsigned)groups, (unsigned)(slices < most ? slices : most));
  return hipSuccess;
}

static hipError_t copy_grid(const StateCopy &c, dim3 *grid) {
  if (c.r_pad % 4 || c.count < 1) return hipErrorInvalidValue;
  return rows_grid((int64_t)c.count * (c.r_pad / 4), c.max_n_pad, grid);
}

hipError_t launch_pack_matrix(const float *src, int32_t n, float *dst, int8_t *dst8,
                              int32_t n_pad, hipStream_t s) {
  dim3 grid;
  if (n_pad % 4 || rows_grid(n_pad / 4, n_pad, &grid) != hipSuccess) return hipErrorInvalidValue;
  pack_matrix_kernel<<<grid, 256, 0, s>>>(src, n, dst, dst8, n_pad);
  return hipGetLastError();
}

hipError_t launch_pack_rows(const StateCopy &c, const float *x, const float *p, hipStream_t s) {
  dim3 grid;
  if (!x || copy_grid(c, &grid) != hipSuccess) return hipErrorInvalidValue;
  pack_rows_kernel<<<grid, 256, 0, s>>>(c, x, p);
  return hipGetLastError();
}

hipError_t launch_unpack_rows(const StateCopy &c, float *x, float *p, hipStream_t s) {
  dim3 grid;
  if (!x && !p) return hipSuccess;
  if (copy_grid(c, &grid) != hipSuccess) return hipErrorInvalidValue;
  unpack_rows_kernel<<<grid, 256, 0, s>>>(c, x, p);
  return hipGetLastError();
}

hipError_t launch_unpack_spins(const StateCopy &c, const int8_t *src8, int8_t *out,
                               const double *e_src, double *e_out, hipStream_t s) {
  dim3 grid;
  if (copy_grid(c, &grid) != hipSuccess) return hipErrorInvalidValue;
  unpack_spins_kernel<<<grid, 256, 0, s>>>(c, src8, out, e_src, e_out);
  return hipGetLastError();
}

hipError_t launch_pack_field(const float *h, int32_t n, float *hf, int8_t *h8, int32_t n_pad,
                             int32_t *flags, hipStream_t s) {
  pack_field_kernel<<<grid_for(n_pad), 256, 0, s>>>(h, n, hf, h8, n_pad, flags);
  return hipGetLastError();
}

}  // namespace si

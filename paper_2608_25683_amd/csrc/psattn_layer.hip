// The tree-dependent steps around the attention of one layer in the shared layout: rotary
// position embedding by each row's sequence position, K/V rows written into their pool slots
// (the page table), and dK/dV read back from the pool into row order.
//
// Rotary embedding: for sequence position p, the pair (x_i, x_{i + d/2}), i < d/2, turns by the
// angle p * theta^(-2i/d); the inverse (transposed) rotation, for the backward, turns by minus
// that angle.  Every token of a shared node has one position however many samples read it (the
// block's pos field, Sec. 6), so shared rows are rotated once.  Angles are formed and reduced in
// fp64 (positions reach 10^4 and beyond), the rotation itself is fp32.
#include <algorithm>

#include "psattn_device.h"

namespace psattn {
namespace {

using namespace dev;

// sin and cos of x (|x| up to about 2^31) in fp64, for results rounded to fp32: x less the nearest
// multiple n of pi/2, taken in two parts (pi/2 to 106 bits, n exact), and the Taylor series of sin and
// cos on [-pi/4, pi/4], whose first omitted terms are below 5e-17.  About 30 fp64 operations; the
// library's sincos (every argument, to the last bits of fp64) takes several times as many.
__device__ __forceinline__ void sincos_reduced(double x, float& sf, float& cf) {
  const double n = rint(x * 0.63661977236758134308);                      // 2/pi
  double r = fma(n, -1.57079632679489655800, x);                          // pi/2: its fp64 value ...
  r = fma(n, -6.12323399573676603587e-17, r);                             // ... and the remainder
  const double z = r * r;
  double s = 1.0 / -1307674368000.0;                                      // -1/15!
  s = fma(s, z, 1.0 / 6227020800.0);
  s = fma(s, z, -1.0 / 39916800.0);
  s = fma(s, z, 1.0 / 362880.0);
  s = fma(s, z, -1.0 / 5040.0);
  s = fma(s, z, 1.0 / 120.0);
  s = fma(s, z, -1.0 / 6.0);
  s = fma(s * z, r, r);
  double c = 1.0 / 20922789888000.0;                                      // 1/16!
  c = fma(c, z, -1.0 / 87178291200.0);
  c = fma(c, z, 1.0 / 479001600.0);
  c = fma(c, z, -1.0 / 3628800.0);
  c = fma(c, z, 1.0 / 40320.0);
  c = fma(c, z, -1.0 / 720.0);
  c = fma(c, z, 1.0 / 24.0);
  c = fma(c, z, -0.5);
  c = fma(c, z, 1.0);
  const int q = (int)((int64_t)n & 3);
  const double a = q & 1 ? c : s, b = q & 1 ? s : c;
  sf = (float)(q & 2 ? -a : a);
  cf = (float)(q == 1 || q == 2 ? -b : b);
}

// A workgroup takes 256 / (d/2) rows: one angle per thread into LDS, then every head of those rows,
// 16 bytes of either half of a head per lane and turn.  Bound by the rows' bytes: 42109 rows of 32 heads,
// d = 128, bf16 (690 MB) take 128 us, 5.4 TB/s; with the angle formed again for every head by one thread
// per pair, moving 2 bytes at a time, they took 540 us.
template <bool BF16>
__global__ __launch_bounds__(256) void rope_kernel(PlanView plan, int32_t ns, int32_t heads, int32_t d, double log2_theta,
                                                   double sign, void* X) {
  __shared__ __attribute__((aligned(16))) float s_sin[256], s_cos[256];   // (read 16 bytes at a time)
  const int half = d / 2, rows = 256 / half;
  const int row0 = blockIdx.x * rows;
  {
    const int i = threadIdx.x % half, row = min(row0 + (int)threadIdx.x / half, ns - 1);
    const double ang = sign * (double)plan.row_pos[row] * exp2(-(2.0 * i / d) * log2_theta);
    sincos_reduced(ang, s_sin[threadIdx.x], s_cos[threadIdx.x]);
  }
  __syncthreads();
  constexpr int V = BF16 ? 8 : 4;   // elements in 16 bytes
  const int per_head = half / V, per_row = per_head * heads;
  const int n = min(rows, ns - row0) * per_row;
#pragma unroll 4
  for (int idx = threadIdx.x; idx < n; idx += 256) {
    const int r = idx / per_row, c = V * (idx % per_head);
    const int64_t o = ((int64_t)row0 * heads + idx / per_head) * d + c;
    const float* sn = s_sin + r * half + c;
    const float* cs = s_cos + r * half + c;
    if (BF16) {
      bf16_t* x = (bf16_t*)X + o;
      const u32x4 a = ld16(x), b = ld16(x + half);
      u32x4 y, z;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float a0 = bf2f(a[k] & 0xffffu), a1 = bf2f(a[k] >> 16), b0 = bf2f(b[k] & 0xffffu), b1 = bf2f(b[k] >> 16);
        const float s0 = sn[2 * k], s1 = sn[2 * k + 1], c0 = cs[2 * k], c1 = cs[2 * k + 1];
        y[k] = pack2(a0 * c0 - b0 * s0, a1 * c1 - b1 * s1);
        z[k] = pack2(a0 * s0 + b0 * c0, a1 * s1 + b1 * c1);
      }
      *(u32x4*)x = y;
      *(u32x4*)(x + half) = z;
    } else {
      float* x = (float*)X + o;
      const f32x4 a = *(const f32x4*)x, b = *(const f32x4*)(x + half);
      const f32x4 s = *(const f32x4*)sn, c4 = *(const f32x4*)cs;
      *(f32x4*)x = a * c4 - b * s;
      *(f32x4*)(x + half) = a * s + b * c4;
    }
  }
}

// rows [Ns][hkv][d] <-> pool [slots][hkv][d], 16 bytes per thread
__global__ __launch_bounds__(256) void kv_move_kernel(PlanView plan, int32_t ns, int32_t row_bytes, int32_t to_pool,
                                                      const uint8_t* a0, const uint8_t* a1, uint8_t* b0, uint8_t* b1) {
  const int per_row = row_bytes / 16;
  const int64_t n = (int64_t)ns * per_row;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < n; idx += (int64_t)gridDim.x * blockDim.x) {
    const int row = (int)(idx / per_row), c = (int)(idx % per_row);
    const int64_t r_off = (int64_t)row * row_bytes + 16 * c;
    const int64_t p_off = (int64_t)plan.row_slot[row] * row_bytes + 16 * c;
    const int64_t src = to_pool ? r_off : p_off, dst = to_pool ? p_off : r_off;
    *(u32x4*)(b0 + dst) = *(const u32x4*)(a0 + src);
    *(u32x4*)(b1 + dst) = *(const u32x4*)(a1 + src);
  }
}

// ---- fp32 tensors as three bf16 planes, for products with a bf16 tensor on the bf16 matrix cores.
// x = x1 + x2 + x3 exactly: each plane takes the next 8 bits of x's 24-bit significand (truncation, so
// that nothing overflows; infinities and NaN stay in x1).  The product of a plane and a bf16 number is
// exact in fp32, so three bf16 products with fp32 sums hold what one fp32 product holds.
__device__ __forceinline__ void split3(float x, uint32_t& x1, uint32_t& x2, uint32_t& x3) {
  const uint32_t u = __float_as_uint(x);
  const bool special = (u & 0x7f800000u) == 0x7f800000u;
  const uint32_t h = (u & 0xffff0000u) | (special && (u & 0x007fffffu) ? 0x00400000u : 0u);
  const float r = special ? 0.f : x - __uint_as_float(u & 0xffff0000u);
  const uint32_t m = __float_as_uint(r) & 0xffff0000u;
  const float l = r - __uint_as_float(m);
  x1 = h >> 16;
  x2 = m >> 16;
  x3 = __float_as_uint(l) >> 16;
}

// four consecutive elements into the three planes (n elements each) at element i
__device__ __forceinline__ void put_planes(const f32x4& x, bf16_t* y, int64_t n, int64_t i) {
  uint32_t p[3][4];
#pragma unroll
  for (int k = 0; k < 4; ++k) split3(x[k], p[0][k], p[1][k], p[2][k]);
#pragma unroll
  for (int j = 0; j < 3; ++j) *(u32x2*)(y + j * n + i) = u32x2{p[j][0] | p[j][1] << 16, p[j][2] | p[j][3] << 16};
}

// (VEC: n is a multiple of 4, four elements per lane and turn; else one)
__device__ __forceinline__ void put_plane1(float x, bf16_t* y, int64_t n, int64_t i) {
  uint32_t p[3];
  split3(x, p[0], p[1], p[2]);
#pragma unroll
  for (int j = 0; j < 3; ++j) y[j * n + i] = (bf16_t)p[j];
}

// y [3][n] = the planes of x [n].  Bound by its 10 bytes per element.
template <bool VEC>
__global__ __launch_bounds__(256) void split3_kernel(const float* x, bf16_t* y, int64_t n) {
  if (!VEC) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) put_plane1(x[i], y, n, i);
    return;
  }
  for (int64_t i = 4 * ((int64_t)blockIdx.x * 256 + threadIdx.x); i < n; i += 4 * (int64_t)gridDim.x * 256)
    put_planes(*(const f32x4*)(x + i), y, n, i);
}

// Backward of silu(a) * b: dm = the sum of its planes [3][n], da = dm b (s + a s (1 - s)) and db = dm a s
// with s = sigmoid(a), written as planes.  Bound by its 28 bytes per element, in place of ten
// elementwise passes over fp32 tensors.
template <bool VEC>
__global__ __launch_bounds__(256) void silu_bwd_kernel(const float* dm, const bf16_t* a, const bf16_t* b, bf16_t* da,
                                                       bf16_t* db, int64_t n) {
  auto grads = [](float d, float av, float bv, float& ga, float& gb) {
    const float s = 1.f / (1.f + expf(-av));
    ga = d * bv * (s + av * s * (1.f - s));
    gb = d * av * s;
  };
  if (!VEC) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
      float ga, gb;
      grads(dm[i] + (dm[n + i] + dm[2 * n + i]), bf2f(a[i]), bf2f(b[i]), ga, gb);
      put_plane1(ga, da, n, i);
      put_plane1(gb, db, n, i);
    }
    return;
  }
  for (int64_t i = 4 * ((int64_t)blockIdx.x * 256 + threadIdx.x); i < n; i += 4 * (int64_t)gridDim.x * 256) {
    const f32x4 d = *(const f32x4*)(dm + i) + (*(const f32x4*)(dm + n + i) + *(const f32x4*)(dm + 2 * n + i));
    const u32x2 a2 = ld8(a + i), b2 = ld8(b + i);
    f32x4 ga, gb;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float av = k & 1 ? __uint_as_float(a2[k / 2] & 0xffff0000u) : bf2f(a2[k / 2] & 0xffffu);
      const float bv = k & 1 ? __uint_as_float(b2[k / 2] & 0xffff0000u) : bf2f(b2[k / 2] & 0xffffu);
      float x, y;
      grads(d[k], av, bv, x, y);
      ga[k] = x;
      gb[k] = y;
    }
    put_planes(ga, da, n, i);
    put_planes(gb, db, n, i);
  }
}

unsigned grid_for(int64_t n) { return (unsigned)std::min<int64_t>((n + 255) / 256, 8192); }

}  // namespace

hipError_t launch_rope(const PlanView& plan, int32_t ns, int32_t heads, int32_t d, float theta, bool inverse, bool bf16,
                       void* X, hipStream_t st) {
  const double l2t = log2((double)theta), sign = inverse ? -1.0 : 1.0;
  const int rows = 256 / (d / 2);
  const dim3 grid((unsigned)((ns + rows - 1) / rows));
  if (bf16) hipLaunchKernelGGL(rope_kernel<true>, grid, dim3(256), 0, st, plan, ns, heads, d, l2t, sign, X);
  else hipLaunchKernelGGL(rope_kernel<false>, grid, dim3(256), 0, st, plan, ns, heads, d, l2t, sign, X);
  return hipGetLastError();
}

hipError_t launch_kv_move(const PlanView& plan, int32_t ns, int32_t row_bytes, bool to_pool, const void* a0,
                          const void* a1, void* b0, void* b1, hipStream_t st) {
  hipLaunchKernelGGL(kv_move_kernel, dim3(grid_for((int64_t)ns * (row_bytes / 16))), dim3(256), 0, st, plan, ns, row_bytes,
                     to_pool ? 1 : 0, (const uint8_t*)a0, (const uint8_t*)a1, (uint8_t*)b0, (uint8_t*)b1);
  return hipGetLastError();
}

namespace {
unsigned plane_grid(int64_t n) { return (unsigned)std::min<int64_t>((n % 4 ? n + 255 : n / 4 + 255) / 256, 65536); }
}  // namespace

hipError_t launch_split_planes(const float* x, void* planes, int64_t n, hipStream_t st) {
  hipLaunchKernelGGL(n % 4 ? split3_kernel<false> : split3_kernel<true>, dim3(plane_grid(n)), dim3(256), 0, st, x,
                     (dev::bf16_t*)planes, n);
  return hipGetLastError();
}

hipError_t launch_silu_bwd(const float* dm, const void* a, const void* b, void* da, void* db, int64_t n, hipStream_t st) {
  hipLaunchKernelGGL(n % 4 ? silu_bwd_kernel<false> : silu_bwd_kernel<true>, dim3(plane_grid(n)), dim3(256), 0, st, dm,
                     (const dev::bf16_t*)a, (const dev::bf16_t*)b, (dev::bf16_t*)da, (dev::bf16_t*)db, n);
  return hipGetLastError();
}

}  // namespace psattn

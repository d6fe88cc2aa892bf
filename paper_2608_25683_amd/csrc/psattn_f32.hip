// fp32 kernels on the fp32 matrix instruction v_mfma_f32_32x32x2_f32 (gfx950): forward, dQ and dK/dV.
//
// What bounds them: the matrix cores at 64 fp32 flops per cycle and SIMD (157 TFLOP/s on the card,
// 148 measured on a large library product), 1/16 of the bf16 rate.  A 32 x 32 block of one product
// over d = 128 takes 4096 cycles of one SIMD and needs 16 KB of one operand, so four wavefronts per
// CU read 16 bytes per cycle: the operands come straight from L2 into registers, in the layout the
// instruction takes, with no LDS staging and no barrier in the loop.  Each operand is loaded one
// product ahead of its use (4096 cycles, beyond the load latency), with one wavefront per SIMD.
//
// Every lane holds one key (or row) of an A or B operand for two halves of head_dim: MFMA step
// s = 4 j + c contracts d = 8 j + c (lanes 0-31) and 8 j + 4 + c (lanes 32-63), so that an operand
// is D/8 16-byte loads per lane.  The 32 x 32 result has column l32 = lane % 32 on each lane and
// rows 8 (v / 4) + 4 hh + v % 4 (hh = lane / 32) in elements v = 0..15; result element v is thus the
// B operand of the next product for the two rows it holds, and that product's A operand is a whole
// row of K, V, Q or dO per half wave, D/32 floats per lane (one coalesced load).
//
// A workgroup is four wavefronts on the same 32 rows (forward, dQ) or 32 keys (dK/dV), which deal
// out the key blocks (or row subtiles and heads) in turn and combine their results through LDS in
// wave order at the end.  Small trees thus still spread over the chip: a tree of 384 rows x 4 heads
// has 48 forward workgroups.  4 trajectories of 4 steps, 16 query heads, d = 128: forward, dQ and dK/dV
// 1398, 2600 and 4541 us on the VALU kernels that these replace (two lanes per row, operands re-read
// from LDS by every lane), 109, 148 and 226 us here; 97 to 109 TFLOP/s on a 4096-token prompt.
#include "psattn_device.h"

namespace psattn {
namespace {

using namespace dev;

constexpr int NW = 4;   // wavefronts per workgroup

__device__ __forceinline__ f32x16 mma(float a, float b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// row of element v of a result on lanes of half hh
__device__ __forceinline__ int res_row(int v, int hh) { return 8 * (v >> 2) + 4 * hh + (v & 3); }

template <int D>
struct Ops {
  typedef __attribute__((ext_vector_type(D / 32))) float vec;   // a lane's share of one row
  static constexpr int LS = D + 4;                              // LDS row stride (floats)
  f32x4 a[D / 8];
  // operand with one row per lane: p points at the lane's row, head_dim 0
  __device__ __forceinline__ void load(const float* p, int hh) {
#pragma unroll
    for (int j = 0; j < D / 8; ++j) a[j] = *(const f32x4*)(p + 8 * j + 4 * hh);
  }
};

// X^T Y over head_dim, X and Y with one row per lane
template <int D>
__device__ __forceinline__ f32x16 dot_rows(const Ops<D>& x, const Ops<D>& y) {
  f32x16 s = f32x16{};
#pragma unroll
  for (int j = 0; j < D / 8; ++j)
#pragma unroll
    for (int c = 0; c < 4; ++c) s = mma(x.a[j][c], y.a[j][c], s);
  return s;
}

// The rows res_row(v, hh), v = 0..15, of a gathered tile, one coalesced row per half wave: lane r of
// either half holds row r's index.
template <int D>
__device__ __forceinline__ void load_rows(typename Ops<D>::vec (&x)[16], const float* base, int index, size_t stride,
                                          int l32, int hh) {
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int r = __shfl(index, res_row(v, hh));
    x[v] = *(const typename Ops<D>::vec*)(base + (size_t)r * stride + (D / 32) * l32);
  }
}

// acc[mb] += (16 gathered rows)^T * p: element e of acc[mb] is head_dim (D/32) res_row(e, hh) + mb of
// column l32
template <int D>
__device__ __forceinline__ void acc_rows(f32x16 (&acc)[D / 32], const typename Ops<D>::vec (&x)[16], const f32x16& p) {
#pragma unroll
  for (int v = 0; v < 16; ++v)
#pragma unroll
    for (int mb = 0; mb < D / 32; ++mb) acc[mb] = mma(x[v][mb], p[v], acc[mb]);
}

// this wave's accumulators into its LDS tile, row l32
template <int D>
__device__ __forceinline__ void put_tile(float* tile, const f32x16 (&acc)[D / 32], int l32, int hh) {
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    typename Ops<D>::vec x;
#pragma unroll
    for (int mb = 0; mb < D / 32; ++mb) x[mb] = acc[mb][e];
    *(typename Ops<D>::vec*)(tile + l32 * Ops<D>::LS + (D / 32) * res_row(e, hh)) = x;
  }
}

// Lanes whose row (eight lanes each) holds a value that is not finite, in an item of packed siblings
template <bool SIB>
__device__ __forceinline__ uint64_t redo_lanes(const FwdItem& it, bool bad) {
  if (!SIB || it.part != PART_SIBLINGS) return 0;
  uint64_t b = __ballot(bad);
  b |= b >> 4;
  b |= b >> 2;
  b |= b >> 1;
  return (b & 0x0101010101010101ull) * 0xff;
}

// ============================================================================================
// Forward: one FwdItem of up to 32 rows x one head; wave w takes the 32-key blocks w, w + 4, ...
template <int D, bool SIB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, D == 128 ? 1 : 2))) void fwd_f32_kernel(FwdArgs a) {
  typedef typename Ops<D>::vec vec;
  constexpr int DB = D / 32, LS = Ops<D>::LS;
  __shared__ __attribute__((aligned(16))) float s_o[NW][32 * LS];
  __shared__ float s_m[NW][32], s_l[NW][32];
  const FwdItem it = a.plan.fwd[blockIdx.x];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int head = it.head0, hk = head / a.s.g;
  const int ridx = min(l32, it.nq - 1), row = a.plan.q_list[it.q_off + ridx];
  const RowKeys rk = row_keys<SIB>(it, it.nkv, ridx, a.plan.q_pos[it.q_off + ridx]);
  auto hidden = [&](int k) { return k > rk.lim || (SIB && (uint32_t)(k - (it.nkv - it.nq)) < rk.gap); };
  const size_t kv_stride = (size_t)a.s.hkv * D;
  const int* kvl = a.plan.kv_list + it.kv_off;
  const float* Kh = (const float*)a.K + (size_t)hk * D;
  const float* Vh = (const float*)a.V + (size_t)hk * D;
  const int nblk = (it.nkv + 31) / 32;

  Ops<D> q, k;
  vec v[16];
  f32x16 o[DB];
#pragma unroll
  for (int mb = 0; mb < DB; ++mb) o[mb] = f32x16{};
  float m_run = kNegInf, l_run = 0.f;
  auto slot_of = [&](int b) { return kvl[min(32 * b + l32, it.nkv - 1)]; };
  int slot = slot_of(wave), slot_nx = slot_of(wave + NW);
  q.load((const float*)a.Q + ((size_t)row * a.s.hq + head) * D, hh);
  k.load(Kh + (size_t)slot * kv_stride, hh);
  for (int b = wave; b < nblk; b += NW) {
    load_rows<D>(v, Vh, slot, kv_stride, l32, hh);
    sched_fence();
    f32x16 s = dot_rows<D>(k, q);
    sched_fence();
    slot = slot_nx;
    slot_nx = slot_of(b + 2 * NW);
    k.load(Kh + (size_t)slot * kv_stride, hh);   // (past the last block: the last key's row)
    sched_fence();
    float mx = kNegInf;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      s[e] = hidden(32 * b + res_row(e, hh)) ? kNegInf : s[e] * a.s.scale;
      mx = fmaxf(mx, s[e]);
    }
    const float m_new = fmaxf(m_run, pair_max(mx));
    const float m_use = m_new == kNegInf ? 0.f : m_new;
    if (__any(m_new > m_run)) {
      const float alpha = expf(m_run - m_use);
      l_run *= alpha;
#pragma unroll
      for (int mb = 0; mb < DB; ++mb) o[mb] *= alpha;
      m_run = m_new;
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      s[e] = expf(s[e] - m_use);
      l_run += s[e];
    }
    acc_rows<D>(o, v, s);
  }
  put_tile<D>(s_o[wave], o, l32, hh);
  l_run = pair_sum(l_run);
  if (hh == 0) {
    s_m[wave][l32] = m_run;
    s_l[wave][l32] = l_run;
  }
  __syncthreads();
  // eight threads per row: the waves' results against the common maximum, in wave order
  const int r = min(tid >> 3, it.nq - 1);
  float m = kNegInf, l = 0.f, w[NW];
#pragma unroll
  for (int i = 0; i < NW; ++i) m = fmaxf(m, s_m[i][r]);
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    w[i] = s_m[i][r] == kNegInf ? 0.f : expf(s_m[i][r] - m);
    l += w[i] * s_l[i][r];
  }
  const float inv = l > 0.f ? 1.f / l : 0.f;
  const float lse = l > 0.f ? m + logf(l) : kNegInf;
  const int orow = a.plan.q_list[it.q_off + r];
  const bool row_ok = tid >> 3 < it.nq;
  float* op;
  if (it.part < 0) {
    op = (float*)a.O + ((size_t)orow * a.s.hq + head) * D;
    if (row_ok && (tid & 7) == 0) a.LSE[(size_t)head * a.s.ns + orow] = lse;
  } else {
    const size_t prow = (size_t)it.part + r;
    op = a.part_o + (prow * a.s.hq + head) * D;
    if (row_ok && (tid & 7) == 0) a.part_lse[prow * a.s.hq + head] = lse;
  }
  f32x4 x[D / 32];
  float z = 0.f;
#pragma unroll
  for (int c = 0; c < D / 32; ++c) {
    x[c] = f32x4{};
#pragma unroll
    for (int i = 0; i < NW; ++i) x[c] += w[i] * *(const f32x4*)&s_o[i][r * LS + 4 * ((tid & 7) + 8 * c)];
    x[c] *= inv;
    z = add_if_finite(x[c], z);
  }
  const uint64_t redo = redo_lanes<SIB>(it, row_ok && !(z == 0.f));
  if (row_ok) {
#pragma unroll
    for (int c = 0; c < D / 32; ++c) *(f32x4*)(op + 4 * ((tid & 7) + 8 * c)) = x[c];
  }
  if constexpr (SIB) {
    if (redo) __threadfence_block();   // (this wavefront's rows, written above, are read back)
    for (uint64_t todo = redo & 0x0101010101010101ull; todo; todo &= todo - 1) {   // the row's first thread
      const int l = __builtin_ctzll(todo), i = 8 * wave + l / 8;
      if (!(lane_value(inv, l) > 0.f)) continue;   // no sum of probabilities: not finite by its own scores
      const int qpos = a.plan.q_pos[it.q_off + i];
      const RowKeys keys = row_keys<SIB>(it, it.nkv, i, qpos);
      const size_t at = ((size_t)__builtin_amdgcn_readlane(orow, l) * a.s.hq + head) * D;
      float* const yp = (float*)a.O + at + (D / 64) * lane;
      float y[D / 64];
      bool want[D / 64];
#pragma unroll
      for (int e = 0; e < D / 64; ++e) want[e] = !is_finite(yp[e]);
      if (!row_fwd<D, false>(y, want, RowPath(kvl, it, keys.lim, (int)keys.gap), (const float*)a.Q + at, Kh, Vh, kv_stride,
                             a.s.scale, lane_value(m, l), lane_value(inv, l), lane))
        continue;
#pragma unroll
      for (int e = 0; e < D / 64; ++e)
        if (want[e]) yp[e] = y[e];
    }
  }
}

// ============================================================================================
// dQ: the forward's items and split; dQ^T += K^T dS^T with dS = P (dO V^T - Delta)
template <int D, bool SIB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void bwd_dq_f32_kernel(BwdArgs a) {
  typedef typename Ops<D>::vec vec;
  constexpr int DB = D / 32, LS = Ops<D>::LS;
  __shared__ __attribute__((aligned(16))) float s_q[NW][32 * LS];
  const FwdItem it = a.plan.fwd[blockIdx.x];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int head = it.head0, hk = head / a.s.g;
  const int ridx = min(l32, it.nq - 1), row = a.plan.q_list[it.q_off + ridx];
  const RowKeys rk = row_keys<SIB>(it, it.nkv, ridx, a.plan.q_pos[it.q_off + ridx]);
  auto hidden = [&](int k) { return k > rk.lim || (SIB && (uint32_t)(k - (it.nkv - it.nq)) < rk.gap); };
  const float lse = a.LSE[(size_t)head * a.s.ns + row];
  const float del = a.delta[(size_t)row * a.s.hq + head];
  const size_t kv_stride = (size_t)a.s.hkv * D;
  const int* kvl = a.plan.kv_list + it.kv_off;
  const float* Kh = (const float*)a.K + (size_t)hk * D;
  const float* Vh = (const float*)a.V + (size_t)hk * D;
  const int nblk = (it.nkv + 31) / 32;

  Ops<D> q, dO, k, v;
  vec kt[16];
  f32x16 dq[DB];
#pragma unroll
  for (int mb = 0; mb < DB; ++mb) dq[mb] = f32x16{};
  auto slot_of = [&](int b) { return kvl[min(32 * b + l32, it.nkv - 1)]; };
  int slot = slot_of(wave), slot_nx = slot_of(wave + NW);
  const size_t qo = ((size_t)row * a.s.hq + head) * D;
  q.load((const float*)a.Q + qo, hh);
  dO.load((const float*)a.dO + qo, hh);
  k.load(Kh + (size_t)slot * kv_stride, hh);
  v.load(Vh + (size_t)slot * kv_stride, hh);
  for (int b = wave; b < nblk; b += NW) {
    load_rows<D>(kt, Kh, slot, kv_stride, l32, hh);
    sched_fence();
    f32x16 s = dot_rows<D>(k, q);
    sched_fence();
    slot = slot_nx;
    slot_nx = slot_of(b + 2 * NW);
    k.load(Kh + (size_t)slot * kv_stride, hh);
    sched_fence();
    const f32x16 dp = dot_rows<D>(v, dO);
    sched_fence();
    v.load(Vh + (size_t)slot * kv_stride, hh);
    sched_fence();
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float p = hidden(32 * b + res_row(e, hh)) ? 0.f : expf(s[e] * a.s.scale - lse);
      s[e] = p * (dp[e] - del);
    }
    acc_rows<D>(dq, kt, s);
  }
  put_tile<D>(s_q[wave], dq, l32, hh);
  __syncthreads();
  const int r = min(tid >> 3, it.nq - 1);
  const bool row_ok = tid >> 3 < it.nq;
  float* dst = it.part < 0 ? a.dQ + ((size_t)a.plan.q_list[it.q_off + r] * a.s.hq + head) * D
                           : a.part_dq + (((size_t)it.part + r) * a.s.hq + head) * D;
  f32x4 x[D / 32];
  float z = 0.f;
#pragma unroll
  for (int c = 0; c < D / 32; ++c) {
    x[c] = f32x4{};
#pragma unroll
    for (int i = 0; i < NW; ++i) x[c] += *(const f32x4*)&s_q[i][r * LS + 4 * ((tid & 7) + 8 * c)];
    x[c] *= a.s.scale;
    z = add_if_finite(x[c], z);
  }
  const uint64_t redo = redo_lanes<SIB>(it, row_ok && !(z == 0.f));
  if (row_ok) {
#pragma unroll
    for (int c = 0; c < D / 32; ++c) *(f32x4*)(dst + 4 * ((tid & 7) + 8 * c)) = x[c];
  }
  if constexpr (SIB) {
    if (redo) __threadfence_block();   // (this wavefront's rows, written above, are read back)
    for (uint64_t todo = redo & 0x0101010101010101ull; todo; todo &= todo - 1) {   // the row's first thread
      const int i = 8 * wave + __builtin_ctzll(todo) / 8;
      const int qrow = a.plan.q_list[it.q_off + i], qpos = a.plan.q_pos[it.q_off + i];
      const RowKeys keys = row_keys<SIB>(it, it.nkv, i, qpos);
      const size_t at = ((size_t)qrow * a.s.hq + head) * D;
      float* const yp = a.dQ + at + (D / 64) * lane;
      float y[D / 64], sum;
      bool want[D / 64];
#pragma unroll
      for (int e = 0; e < D / 64; ++e) want[e] = !is_finite(yp[e]);
      if (!row_dq<D, false>(y, sum, want, false, RowPath(kvl, it, keys.lim, (int)keys.gap), (const float*)a.Q + at,
                            (const float*)a.dO + at, Kh, Vh, kv_stride, a.s.scale, a.LSE[(size_t)head * a.s.ns + qrow],
                            -a.delta[(size_t)qrow * a.s.hq + head], lane))
        continue;
#pragma unroll
      for (int e = 0; e < D / 64; ++e)
        if (want[e]) yp[e] = y[e] * a.s.scale;
    }
  }
}

// ============================================================================================
// dK/dV: workgroup (i, y) takes keys 32 y .. 32 y + 31 of BkvItem i; wave w takes the steps (32-row
// subtile, head of the group) w, w + 4, ...  K and V of the keys are in LDS (the B operands of
// S = Q K^T and dP = dO V^T; parts y = 0 of all items start first); the rows of Q and dO are loaded twice, one row per lane for those two
// products and coalesced for dV^T += dO^T P and dK^T += Q^T dS.
template <int D>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void bwd_kv_f32_kernel(BwdArgs a) {
  typedef typename Ops<D>::vec vec;
  constexpr int DB = D / 32, LS = Ops<D>::LS;
  __shared__ __attribute__((aligned(16))) float s_kv[2][32 * LS];
  __shared__ __attribute__((aligned(16))) float s_acc[NW][32 * LS];
  const BkvItem it = a.plan.bkv[blockIdx.x];
  const int k0 = 32 * blockIdx.y, nk = min(it.nk - k0, 32);
  if (nk <= 0) return;
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hk = it.hk, G = a.s.g, hq = a.s.hq;
  const size_t kv_stride = (size_t)a.s.hkv * D, q_stride = (size_t)hq * D;
  const int* kvl = a.plan.kv_list + it.kv_off + k0;
  const int* ql = a.plan.q_list + it.q_off;
  const int* qp = a.plan.q_pos + it.q_off;
  const int kpos0 = it.kv_pos0 + k0, kpos = kpos0 + l32;

  for (int i = tid; i < 32 * (D / 4); i += 256) {
    const int key = i / (D / 4), d = 4 * (i % (D / 4));
    const size_t o = (size_t)kvl[min(key, nk - 1)] * kv_stride + (size_t)hk * D + d;
    *(f32x4*)&s_kv[0][key * LS + d] = *(const f32x4*)((const float*)a.K + o);
    *(f32x4*)&s_kv[1][key * LS + d] = *(const f32x4*)((const float*)a.V + o);
  }
  // rows before the first key of this part see none of its keys: they are the last entries of the
  // list (the node's own rows, positions descending by one), fewer than BKV_TILE of them
  int nq = it.nq;
#pragma unroll
  for (int i = 0; i < BKV_TILE; i += 64) {
    const int e = it.nq - 1 - i - lane;
    nq -= __popcll(__ballot(e >= 0 && qp[max(e, 0)] < kpos0));
  }
  const int nsteps = (nq + Q_SUB - 1) / Q_SUB * G;
  __syncthreads();

  f32x16 dk[DB], dv[DB];
#pragma unroll
  for (int mb = 0; mb < DB; ++mb) dk[mb] = dv[mb] = f32x16{};
  Ops<D> q, dO;
  vec qt[16], dot[16];
  int row, qpos, row_nx, qpos_nx;
  float lse, del, lse_nx, del_nx;
  auto fetch = [&](int step, int& r, int& p, float& l, float& d) __attribute__((always_inline)) {
    const int e = step / G * Q_SUB + l32;
    r = ql[min(e, nq - 1)];
    p = e < nq ? qp[e] : -1;
    const int head = hk * G + step % G;
    l = a.LSE[(size_t)head * a.s.ns + r];
    d = a.delta[(size_t)r * hq + head];
  };
  auto head_off = [&](int step) __attribute__((always_inline)) { return (size_t)(hk * G + step % G) * D; };
  if (wave < nsteps) {
    fetch(wave, row, qpos, lse, del);
    q.load((const float*)a.Q + row * q_stride + head_off(wave), hh);
    dO.load((const float*)a.dO + row * q_stride + head_off(wave), hh);
  }
  // (rows past the list, masked by position -1, are the last row again)
  for (int st = wave; st < nsteps; st += NW) {
    const int nx = min(st + NW, nsteps - 1);
    load_rows<D>(dot, (const float*)a.dO + head_off(st), row, q_stride, l32, hh);
    fetch(nx, row_nx, qpos_nx, lse_nx, del_nx);
    sched_fence();
    Ops<D> kv;
    kv.load(&s_kv[0][l32 * LS], hh);
    f32x16 s = dot_rows<D>(q, kv);
    sched_fence();
    load_rows<D>(qt, (const float*)a.Q + head_off(st), row, q_stride, l32, hh);
    sched_fence();
    kv.load(&s_kv[1][l32 * LS], hh);
    f32x16 dp = dot_rows<D>(dO, kv);
    sched_fence();
    q.load((const float*)a.Q + row_nx * q_stride + head_off(nx), hh);
    sched_fence();
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int r = res_row(e, hh);   // (every lane takes part in the exchanges: no branch around them)
      const int qpos_r = __shfl(qpos, r);
      const float lse_r = __shfl(lse, r), del_r = __shfl(del, r);
      const float p = kpos > qpos_r ? 0.f : expf(s[e] * a.s.scale - lse_r);
      dp[e] = p * (dp[e] - del_r);
      s[e] = p;
    }
    acc_rows<D>(dv, dot, s);
    sched_fence();
    dO.load((const float*)a.dO + row_nx * q_stride + head_off(nx), hh);
    sched_fence();
    acc_rows<D>(dk, qt, dp);
    row = row_nx;
    qpos = qpos_nx;
    lse = lse_nx;
    del = del_nx;
  }
  // sum over the waves, in wave order: dV, then dK through the same tiles
  const int key = tid >> 3;
  auto write = [&](const f32x16 (&acc)[DB], float* full, float* part, float scale) __attribute__((always_inline)) {
    __syncthreads();
    put_tile<D>(s_acc[wave], acc, l32, hh);
    __syncthreads();
    if (key >= nk) return;
    float* dst = it.part < 0 ? full + (size_t)kvl[key] * kv_stride + (size_t)hk * D
                             : part + ((size_t)it.part * BKV_TILE + k0 + key) * D;
    const bool add = it.part < 0 && it.acc;   // a cached node's keys: add to earlier calls' gradients
#pragma unroll
    for (int c = 0; c < D / 32; ++c) {
      const int d = 4 * ((tid & 7) + 8 * c);
      f32x4 x = f32x4{};
#pragma unroll
      for (int i = 0; i < NW; ++i) x += *(const f32x4*)&s_acc[i][key * LS + d];
      x *= scale;
      if (add) x += *(const f32x4*)(dst + d);
      *(f32x4*)(dst + d) = x;
    }
  };
  write(dv, a.dV, a.part_dv, 1.f);
  write(dk, a.dK, a.part_dk, a.s.scale);
}

}  // namespace

// One workgroup per item (the planner makes fp32 items 32 rows x one head)
hipError_t launch_fwd_f32(const FwdArgs& a, hipStream_t st) {
  if (a.s.bmq != 32 || a.s.hc != 1) return hipErrorInvalidValue;
  auto launch = [&](auto sib) {   // SIB: plans with items of packed siblings
    constexpr bool SIB = decltype(sib)::value;
    if (a.s.d == 128) hipLaunchKernelGGL((fwd_f32_kernel<128, SIB>), dim3(a.n_items), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((fwd_f32_kernel<64, SIB>), dim3(a.n_items), dim3(256), 0, st, a);
  };
  if (a.siblings) launch(dev::Flag<true>{});
  else launch(dev::Flag<false>{});
  return hipGetLastError();
}

hipError_t launch_bwd_dq_f32(const BwdArgs& a, hipStream_t st) {
  if (a.s.bmq != 32 || a.s.hc != 1) return hipErrorInvalidValue;
  auto launch = [&](auto sib) {   // SIB: plans with items of packed siblings
    constexpr bool SIB = decltype(sib)::value;
    if (a.s.d == 128) hipLaunchKernelGGL((bwd_dq_f32_kernel<128, SIB>), dim3(a.n_fwd), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((bwd_dq_f32_kernel<64, SIB>), dim3(a.n_fwd), dim3(256), 0, st, a);
  };
  if (a.siblings) launch(dev::Flag<true>{});
  else launch(dev::Flag<false>{});
  return hipGetLastError();
}

hipError_t launch_bwd_kv_f32(const BwdArgs& a, hipStream_t st) {
  const dim3 grid(a.n_bkv, BKV_TILE / 32);
  if (a.s.d == 128) hipLaunchKernelGGL((bwd_kv_f32_kernel<128>), grid, dim3(256), 0, st, a);
  else hipLaunchKernelGGL((bwd_kv_f32_kernel<64>), grid, dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace psattn

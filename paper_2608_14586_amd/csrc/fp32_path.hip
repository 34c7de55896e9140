// fp32 debug path: the same blocks with no reduced precision anywhere, to
// check the composition (rotary layout, cache layout, grouped heads, residual
// order) at a 1e-4 bar.

#include <math.h>

#include "kernels.h"

namespace vla {
namespace {

// C = A * W^T (+ bias), or C += ..., by v_mfma_f32_32x32x2_f32 (fp32 products
// and sums).  A wave owns a 32x32 tile; per 8 k each lane loads 16 bytes of
// its A row and of its W row (k range 4 * (lane / 32)), whose four elements
// feed four MFMAs: element j pairs k = j with k = 4 + j in both operands.  No
// LDS in the loop: the operands are small and stay in L1 / L2.
// SPLIT: the four waves take a quarter of K each of one 32x32 tile and add
// their sums in LDS, so that a product of few tiles still fills the chip and
// its chain of loads is a quarter as long; otherwise they take the four
// quadrants of a 64x64 tile.  Both sum the quarters on their own and add them
// in the same order, so that a row's bits do not depend on how many rows share
// the call.  A 128-row product of the d=256 stack (K = 256 and 688) took 57 us
// with 64x64 VALU tiles in 16-deep LDS slabs (8 to 24 workgroups, two barriers
// a slab) and takes 6 to 9 under the tracer.
// VEC: rows are 16-byte aligned; otherwise elements load one by one.
template <bool SPLIT, bool VEC>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ A, int lda,
                                                       const float* __restrict__ W, int ldw, float* __restrict__ C,
                                                       int ldc, const float* __restrict__ bias, int mode, int M,
                                                       int N, int K) {
  __shared__ float red[SPLIT ? 4 : 1][SPLIT ? 16 : 1][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int li = lane & 31, half = lane >> 5;
  const int m0 = SPLIT ? blockIdx.y * 32 : blockIdx.y * 64 + (wave >> 1) * 32;
  const int n0 = SPLIT ? blockIdx.x * 32 : blockIdx.x * 64 + (wave & 1) * 32;
  // rows past the end load the last row; their results are not stored
  const float* ar = A + (size_t)min(m0 + li, M - 1) * lda + 4 * half;
  const float* wr = W + (size_t)min(n0 + li, N - 1) * ldw + 4 * half;
  const int steps = (K + 7) / 8;
  auto load = [&](const float* r, int s) {
    const int k = s * 8;
    if (VEC && k + 8 <= K) return *(const f32x4*)(r + k);
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (k + 4 * half + j < K) v[j] = r[k + j];
    return v;
  };
  // the sum over quarter q of K
  auto quarter = [&](int q) {
    constexpr int U = 8;
    const int s1 = steps * (q + 1) / 4;
    int s = steps * q / 4;
    f32x16 acc = {};
    for (; s + U <= s1; s += U) {
      f32x4 a[U], w[U];
#pragma unroll
      for (int u = 0; u < U; ++u) a[u] = load(ar, s + u), w[u] = load(wr, s + u);
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u][j], w[u][j], acc, 0, 0, 0);
    }
    for (; s < s1; ++s) {
      const f32x4 a = load(ar, s), w = load(wr, s);
#pragma unroll
      for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[j], w[j], acc, 0, 0, 0);
    }
    return acc;
  };
  const int col = n0 + li;
  const float bv = bias && col < N ? bias[col] : 0.f;
  auto store = [&](int r, float v) {
    const int row = m0 + (r >> 2) * 8 + half * 4 + (r & 3);
    if (row >= M || col >= N) return;
    float* p = C + (size_t)row * ldc + col;
    v += bv;
    *p = mode == 1 ? *p + v : v;
  };
  if constexpr (SPLIT) {
    const f32x16 acc = quarter(wave);
#pragma unroll
    for (int r = 0; r < 16; ++r) red[wave][r][lane] = acc[r];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = wave * 4 + q;
      store(r, (red[0][r][lane] + red[1][r][lane]) + (red[2][r][lane] + red[3][r][lane]));
    }
  } else {
    f32x16 sum = {};
#pragma unroll 1
    for (int p = 0; p < 4; p += 2) {
      const f32x16 a = quarter(p), b = quarter(p + 1);
      sum = p ? sum + (a + b) : a + b;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) store(r, sum[r]);
  }
}

// one thread per (row, head-column pair) of the natural-order qkv matrix
__global__ void qkv_split_f32_kernel(const float* __restrict__ qkv, const float* __restrict__ rc,
                                     const float* __restrict__ rs, float* q, float* k, float* v, float* vt, int ldvt,
                                     int B, int L, int H, int Hkv, int dh) {
  const int half = dh / 2;
  const int npairs = (H + 2 * Hkv) * half;
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)B * L * npairs) return;
  const int pr = (int)(idx % npairs);
  const int row = (int)(idx / npairs);
  const int b = row / L, pos = row % L;
  const int head_all = pr / half, i = pr % half;
  const int ncol = (H + 2 * Hkv) * dh;
  const float* src = qkv + (size_t)row * ncol + head_all * dh;
  float x1 = src[i], x2 = src[i + half];
  if (head_all < H + Hkv && rc != nullptr) {
    float c = rc[(size_t)pos * half + i], s = rs[(size_t)pos * half + i];
    float y1 = x1 * c - x2 * s, y2 = x2 * c + x1 * s;
    x1 = y1;
    x2 = y2;
  }
  if (head_all < H) {
    float* d = q + (((size_t)b * H + head_all) * L + pos) * dh;
    d[i] = x1;
    d[i + half] = x2;
  } else if (head_all < H + Hkv) {
    int hh = head_all - H;
    float* d = k + (((size_t)b * Hkv + hh) * L + pos) * dh;
    d[i] = x1;
    d[i + half] = x2;
  } else {
    int hh = head_all - H - Hkv;
    float* d = v + (((size_t)b * Hkv + hh) * L + pos) * dh;
    d[i] = x1;
    d[i + half] = x2;
    if (vt) {
      vt[(((size_t)b * Hkv + hh) * dh + i) * ldvt + pos] = x1;
      vt[(((size_t)b * Hkv + hh) * dh + i + half) * ldvt + pos] = x2;
    }
  }
}

// 16 queries of one (batch, head) per workgroup, 16 lanes per query; keys in
// tiles of 64 staged in LDS (rows padded by 16 bytes), online softmax per
// tile.  A lane scores four keys of its query, and then owns DH / 16 of the
// query's output dims.  dh <= DH, the dims past it are zeros.  (One thread
// per query, its q and output rows in registers over all keys, took 844 us at
// L = 128, 4 heads of 64: eight waves in all, each a serial chain over the
// keys; this takes 17 to 18.)
constexpr int AF_Q = 16, AF_K = 64;
template <int DH>
__global__ __launch_bounds__(256) void attention_f32_kernel(const float* __restrict__ q, const float* __restrict__ k,
                                                            const float* __restrict__ v, float* __restrict__ o,
                                                            int B, int H, int Hkv, int L, int dh, int causal,
                                                            float scale) {
  constexpr int LD = DH + 4, OD = DH / 16;
  __shared__ __attribute__((aligned(16))) float sq[AF_Q][LD], sk[AF_K][LD], sv[AF_K][LD], sp[AF_Q][AF_K + 4];
  const int tid = threadIdx.x, qr = tid >> 4, lq = tid & 15;
  const int h = blockIdx.y, b = blockIdx.z, q0 = blockIdx.x * AF_Q;
  const int hk = h / (H / Hkv);
  const float* qh = q + ((size_t)b * H + h) * (size_t)L * dh;
  const float* kh = k + ((size_t)b * Hkv + hk) * (size_t)L * dh;
  const float* vh = v + ((size_t)b * Hkv + hk) * (size_t)L * dh;
  // rows [r0, r0 + R) of a head into LDS; rows from L on and dims from dh on are zero
  auto stage = [&](float (*dst)[LD], const float* src, int r0, int R) {
    for (int e = tid; e < R * (DH / 4); e += 256) {
      const int r = e / (DH / 4), d = e % (DH / 4) * 4, row = r0 + r;
      f32x4 x = {0.f, 0.f, 0.f, 0.f};
      if (row < L) {
        if (dh % 4 == 0) {
          if (d < dh) x = *(const f32x4*)(src + (size_t)row * dh + d);
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (d + j < dh) x[j] = src[(size_t)row * dh + d + j];
        }
      }
      *(f32x4*)&dst[r][d] = x;
    }
  };
  stage(sq, qh, q0, AF_Q);
  const int qi = q0 + qr, kend = causal ? min(L, q0 + AF_Q) : L;
  float m = -INFINITY, l = 0.f, acc[OD];
#pragma unroll
  for (int d = 0; d < OD; ++d) acc[d] = 0.f;
  for (int k0 = 0; k0 < kend; k0 += AF_K) {
    __syncthreads();  // the previous tile's reads are done
    stage(sk, kh, k0, AF_K);
    stage(sv, vh, k0, AF_K);
    __syncthreads();
    float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int d = 0; d < DH; d += 4) {
      const f32x4 x = *(const f32x4*)&sq[qr][d];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 y = *(const f32x4*)&sk[lq + 16 * j][d];
#pragma unroll
        for (int e = 0; e < 4; ++e) s[j] = fmaf(x[e], y[e], s[j]);
      }
    }
    float mt = -INFINITY;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int key = k0 + lq + 16 * j;
      s[j] = key < L && (!causal || key <= qi) ? s[j] * scale : -INFINITY;
      mt = fmaxf(mt, s[j]);
    }
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) mt = fmaxf(mt, __shfl_xor(mt, off, 16));
    const float mn = fmaxf(m, mt);
    // a query past L has no valid key in a causal tile: its row stays empty
    const float mu = mn == -INFINITY ? 0.f : mn;
    const float alpha = m == -INFINITY ? 0.f : expf(m - mu);
    float ps = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float p = s[j] == -INFINITY ? 0.f : expf(s[j] - mu);
      sp[qr][lq + 16 * j] = p;
      ps += p;
    }
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) ps += __shfl_xor(ps, off, 16);
    l = l * alpha + ps;
    m = mn;
#pragma unroll
    for (int d = 0; d < OD; ++d) acc[d] *= alpha;
    __syncthreads();  // sp
    // the sum ends with the query's last key: a weight of zero times a later
    // token's value is not zero where that value is not finite
    const int jn = causal ? min(qi - k0 + 1, AF_K) : AF_K;
#pragma unroll 4
    for (int j = 0; j < jn; ++j) {
      const float p = sp[qr][j];
#pragma unroll
      for (int d = 0; d < OD; d += 4) {
        const f32x4 x = *(const f32x4*)&sv[j][lq * 4 + d * 16];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[d + e] = fmaf(p, x[e], acc[d + e]);
      }
    }
  }
  if (qi >= L) return;
  float* orow = o + ((size_t)b * L + qi) * (size_t)(H * dh) + h * dh;
#pragma unroll
  for (int d = 0; d < OD; d += 4)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int c = lq * 4 + d * 16 + e;
      if (c < dh) orow[c] = acc[d + e] / l;
    }
}

__global__ void swiglu_f32_kernel(const float* __restrict__ gu, float* __restrict__ a, int M, int F) {
  size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)M * F) return;
  size_t row = idx / F, f = idx % F;
  float g = gu[row * 2 * F + f], u = gu[row * 2 * F + F + f];
  a[idx] = g / (1.f + expf(-g)) * u;
}

__global__ void gelu_f32_kernel(float* x, size_t n) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float z = x[i];
  x[i] = z * 0.5f * erfcf(-z * 0.70710678118654752f);
}

}  // namespace

hipError_t gemm_f32(const float* A, int lda, const float* W, int ldw, float* C, int ldc, const float* bias, int mode,
                    int M, int N, int K, hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  // 64x64 tiles once they give every CU a workgroup, split-K 32x32 tiles below
  const bool split = (long)((M + 63) / 64) * ((N + 63) / 64) < 256;
  const bool vec = lda % 4 == 0 && ldw % 4 == 0 && ((uintptr_t)A | (uintptr_t)W) % 16 == 0;
  const int t = split ? 32 : 64;
  const dim3 grid((N + t - 1) / t, (M + t - 1) / t);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, A, lda, W, ldw, C, ldc, bias, mode, M, N, K);
  };
  if (split)
    vec ? go(gemm_f32_kernel<true, true>) : go(gemm_f32_kernel<true, false>);
  else
    vec ? go(gemm_f32_kernel<false, true>) : go(gemm_f32_kernel<false, false>);
  return hipGetLastError();
}

hipError_t qkv_split_f32(const float* qkv, const float* rope_cos, const float* rope_sin, float* q, float* k,
                         float* v, float* vt, int ldvt, int B, int L, int H, int Hkv, int dh, hipStream_t s) {
  size_t n = (size_t)B * L * (H + 2 * Hkv) * (dh / 2);
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(qkv_split_f32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, qkv, rope_cos,
                     rope_sin, q, k, v, vt, ldvt, B, L, H, Hkv, dh);
  return hipGetLastError();
}

hipError_t attention_f32(const float* q, const float* k, const float* v, float* o, int B, int H, int Hkv, int L,
                         int dh, bool causal, hipStream_t s) {
  if (B <= 0 || L <= 0) return hipSuccess;
  if (Hkv <= 0 || H % Hkv != 0 || dh > 128) return hipErrorInvalidValue;
  dim3 grid((L + AF_Q - 1) / AF_Q, H, B);
  float scale = 1.f / sqrtf((float)dh);
  if (dh <= 64)
    hipLaunchKernelGGL((attention_f32_kernel<64>), grid, dim3(256), 0, s, q, k, v, o, B, H, Hkv, L, dh, causal ? 1 : 0,
                       scale);
  else
    hipLaunchKernelGGL((attention_f32_kernel<128>), grid, dim3(256), 0, s, q, k, v, o, B, H, Hkv, L, dh,
                       causal ? 1 : 0, scale);
  return hipGetLastError();
}

hipError_t swiglu_f32(const float* gu, float* a, int M, int F, hipStream_t s) {
  size_t n = (size_t)M * F;
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(swiglu_f32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, gu, a, M, F);
  return hipGetLastError();
}

hipError_t gelu_f32(float* x, size_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(gelu_f32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, x, n);
  return hipGetLastError();
}

}  // namespace vla

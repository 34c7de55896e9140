// Flash-style attention for gfx950 (bf16 MFMA, fp32 online softmax).
//
// One workgroup = 4 waves = 128 queries of one (batch, head); each wave owns
// 32 queries.  Keys advance in tiles of 64 staged in LDS: K as [key][dh] and
// V transposed as [dh][key], so every MFMA operand is a contiguous LDS read.
// The tiles move global -> LDS with buffer_load ... lds (no VGPRs, no
// ds_write) into two stages, the 16-byte chunks of each row XOR-swizzled so
// that fragment reads hit every bank once per 16-lane phase.  Each stage of
// each operand is an LDS array of its own and the tile loop is unrolled over
// the stages, so the compiler can tell fragment reads from the DMA writes into
// other stages and never waits for those.  Key rows past L read as zero
// through the buffer resource; V^T columns past L are zeroed in LDS in the
// last tile.
//
// A wave works one tile ahead of itself: while it exponentiates the scores of
// tile t, the MFMAs between the exponentials form the scores of tile t + 1,
// and every K and V^T fragment is read from LDS four MFMAs before the one
// that takes it.  A wave that did scores, softmax and PV one after the other
// spent 2300 cycles a tile on latencies that only other waves could cover,
// and most calls leave a SIMD one or two waves: the longest causal query
// block, one camera, two cameras.  With the lane exchange of the row maximum
// by v_permlane32_swap (through LDS the same exchange was flat before, and
// costs 8% now that it stands alone), us a launch: 14 heads of 64, causal,
// L=4096 57 -> 49; 16 heads of 64 at 1 x 1024 16.5 -> 14.3, 2 x 577 12.5 ->
// 11.1, 6 x 1024 34.6 -> 33.9; 32 heads of 128, causal, L=2048 47-50 -> 43-45,
// L=1024 23.1 -> 20.7.  Four stages instead of two for heads of 64 (two
// workgroups a CU) measured 49 -> 55 and 34 -> 41, the maximum taken between
// the PV MFMAs flat.
//
// The scores are formed transposed, S^T = K Q^T, with v_mfma_f32_32x32x16_bf16
// (A = K tile from LDS, B = the wave's Q held in registers).  In the 32x32
// accumulator layout each lane then holds 16 keys of ONE query, so a query's
// running max/sum needs a single cross-half exchange (lane ^ 32) instead of a
// 32-lane reduction, and the probabilities already sit where the PV product
// O^T = V^T P^T wants its B operand: a lane's 8 bf16 values for keys
// {16s + 4h + j, 16s + 8 + 4h + j : j < 4} feed k-step s directly.  V^T is
// stored with the keys of every 16-key group in the order
// [0-3, 8-11, 4-7, 12-15] (bits 2 and 3 of the key index swapped), so the A
// fragment of those same keys is one contiguous 16-byte read.  The softmax
// runs in base 2 with log2(e)/sqrt(dh) folded into one FMA per score.
//
// Causal tiles are masked per element only on the diagonal; a wave skips the
// key tiles entirely beyond its last query (but for the scores of the first,
// formed ahead and dropped).  Causal query blocks are
// issued so that co-resident workgroups carry complementary amounts of work.

#include <math.h>

#include <type_traits>

#include "kernels.h"

namespace vla {
namespace {

constexpr int BQ = 128, BKV = 64;

// key index <-> stored V^T column: bits 2 and 3 swapped (an involution)
__device__ __forceinline__ int swap23(int t) { return (t & ~12) | ((t & 4) << 1) | ((t & 8) >> 1); }

__device__ __forceinline__ void lds_dma16(__amdgpu_buffer_rsrc_t r, void* lds, unsigned voff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds, 16, voff, 0, 0, 0);
}
// wait until at most N of this wave's global->LDS loads are outstanding and
// every LDS access has completed, then barrier (no vmcnt(0) drain)
template <int N>
__device__ __forceinline__ void wait_barrier() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0070);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// three workgroups a CU for heads of 64 (32 KB of LDS each), two for heads of
// 128 (64 KB)
template <int DH, bool CAUSAL>
__global__ __launch_bounds__(256, DH == 64 ? 3 : 2) void attn_bf16_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ k,
                                                          const bf16_t* __restrict__ vt, int ldvt,
                                                          bf16_t* __restrict__ o, int B, int H, int Hkv, int L,
                                                          float scale_log2) {
  constexpr int KROWB = DH * 2;                  // bytes per K row
  constexpr int KT = BKV * KROWB, VT = DH * BKV * 2;   // bytes per K / V^T tile
  constexpr int KI = KT / 1024 / 4, VI = VT / 1024 / 4;  // 1 KB loads per wave per tile
  constexpr int ND = DH / 32, KS = DH / 16;
  // one array per operand and stage: every access names its array, so the
  // compiler can tell fragment reads from the DMA writes into other arrays
  __shared__ __attribute__((aligned(1024))) char sk0[KT];
  __shared__ __attribute__((aligned(1024))) char sk1[KT];
  __shared__ __attribute__((aligned(1024))) char sv0[VT];
  __shared__ __attribute__((aligned(1024))) char sv1[VT];

  // the wave index is uniform: from a scalar register, the DMA destinations
  // (M0) are scalar arithmetic and take no VGPRs
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, li = lane & 31;
  const int nqb = (L + BQ - 1) / BQ;
  const int id = blockIdx.x;
  const int rest = id % (H * B);
  const int qb_r = id / (H * B);
  const int heavy = (nqb + 1) / 2;
  const int qb = !CAUSAL ? qb_r : (qb_r < heavy ? nqb - 1 - qb_r : qb_r - heavy);
  const int h = rest % H, b = rest / H;
  const int hk = h / (H / Hkv);
  const int q0 = qb * BQ;
  const int qw0 = q0 + wave * 32;
  const int qi = qw0 + li;

  const bf16_t* qh = q + ((size_t)b * H + h) * L * DH;
  const bf16_t* kh = k + ((size_t)b * Hkv + hk) * L * DH;
  const bf16_t* vh = vt + ((size_t)b * Hkv + hk) * DH * (size_t)ldvt;
  // rows past L read as zero
  const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc((void*)kh, (short)0, L * DH * 2, 0x00020000);
  const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc((void*)vh, (short)0, DH * ldvt * 2, 0x00020000);

  // the wave's queries as MFMA B fragments, loaded without branches: lanes
  // past L load row L-1 (their scores and outputs are never stored)
  bf16x8 fq[KS];
  const int qrow = min(qi, L - 1);
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) fq[ks] = *(const bf16x8*)(qh + (size_t)qrow * DH + ks * 16 + half * 8);

  const int kend = CAUSAL ? min(L, q0 + BQ) : L;
  const int ntiles = (kend + BKV - 1) / BKV;

  // K row r of a tile: 16-byte chunk c stored at chunk c ^ ksw(r); V^T row d: chunk c at c ^ ((d >> 1) & 7)
  auto ksw = [](int r) { return DH == 128 ? (r & 15) : ((r >> 1) & 7); };
  auto issue_k = [&](char* st, int t) {
    const int kb = t * BKV;
#pragma unroll
    for (int j = 0; j < KI; ++j) {
      const int blk = wave * KI + j;
      constexpr int RPK = 1024 / KROWB;        // rows per 1 KB
      constexpr int CPR = KROWB / 16;          // chunks per row
      const int r = blk * RPK + lane / CPR, cs = lane % CPR;
      const int c = cs ^ ksw(r);
      lds_dma16(rk, st + blk * 1024, (unsigned)(((kb + r) * DH + c * 8) * 2));
    }
  };
  auto issue_v = [&](char* st, int t) {
    const int kb = t * BKV;
#pragma unroll
    for (int j = 0; j < VI; ++j) {
      const int blk = wave * VI + j;
      const int d = blk * 8 + lane / 8, cs = lane % 8;
      const int c = cs ^ ((d >> 1) & 7);
      lds_dma16(rv, st + blk * 1024, (unsigned)((d * ldvt + kb + c * 8) * 2));
    }
  };

  f32x16 acc_o[ND];
#pragma unroll
  for (int t = 0; t < ND; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc_o[t][r] = 0.f;
  float m_run = -INFINITY, l_part = 0.f;

  // K tile t + 2 and V^T tile t + 1 are loaded at the head of tile t, into the
  // stages that tile t - 1 read last.  The first loads are issued
  // unconditionally (a tile past the last reads zeros, or rows of later keys,
  // and is never used); then wait for the query fragments and K tile 0 only.
  issue_k(sk0, 0);
  issue_k(sk1, 1);
  issue_v(sv0, 0);

  f32x16 sa[2], sb[2];  // raw scores of the tile in work and of the next
  const f32x16 zero = {};
  auto kfrag = [&](const char* st, int t, int ks) -> bf16x8 {
    const int r = t * 32 + li, c = ks * 2 + half;
    return *(const bf16x8*)(st + r * KROWB + ((c ^ ksw(r)) * 16));
  };
  auto vfrag = [&](const char* st, int c4, int dt) -> bf16x8 {
    const int d = dt * 32 + li, c = c4 * 2 + half;
    return *(const bf16x8*)(st + d * 128 + ((c ^ ((d >> 1) & 7)) * 16));
  };
  wait_barrier<KI + VI>();
  if (qw0 < L) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int t = 0; t < 2; ++t)
        sa[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kfrag(sk0, t, ks), fq[ks], ks == 0 ? zero : sa[t], 0, 0, 0);
  }

  // tile it in stage S (= it % 2): s holds its scores, sn receives the next tile's
  auto body = [&](auto S_, int it, f32x16(&s)[2], f32x16(&sn)[2]) {
    constexpr int S = decltype(S_)::value;
    // K tile it + 1 and V^T tile it landed (for every wave), and every wave is
    // done with the stages the next loads overwrite
    wait_barrier<0>();
    const int kb = it * BKV;
    char* vst = S == 0 ? sv0 : sv1;
    const char* kst = S == 0 ? sk1 : sk0;
    if (kb + BKV > L) {
      // ragged last tile: V^T columns of keys >= L hold whatever lies past the
      // keys; zero them (their probabilities are zero, but 0 * NaN is not)
      for (int e = tid; e < DH * BKV; e += 256) {
        const int d = e / BKV, sc = e % BKV;
        const int key = kb + swap23(sc);
        if (key >= L) *(bf16_t*)(vst + d * 128 + (((sc / 8) ^ ((d >> 1) & 7)) * 16) + (sc % 8) * 2) = 0;
      }
      wait_barrier<0>();
    }
    if (it + 1 < ntiles) {
      issue_k(S == 0 ? sk0 : sk1, it + 2);
      issue_v(S == 0 ? sv1 : sv0, it + 1);
    }
    const bool active = !CAUSAL || kb <= qw0 + 31;
    if (active && qw0 < L) {
      // fragments of the block's MFMAs in order: the next tile's K (NMF), then
      // this tile's V^T; read LA ahead of the MFMA that takes them.  The
      // scheduling barriers let only VALU and scalar instructions cross, so
      // this order of reads and MFMAs is the one issued.
      constexpr int NMF = 2 * KS, NPV = 4 * ND, EPM = 32 / NMF, LA = 4;
      bf16x8 fr[LA];
      auto fetch = [&](int i) {
        if (i < NMF) fr[i % LA] = kfrag(kst, i & 1, i >> 1);
        else if (i < NMF + NPV) fr[i % LA] = vfrag(vst, (i - NMF) / ND, (i - NMF) % ND);
      };
#pragma unroll
      for (int i = 0; i < LA; ++i) fetch(i);
      __builtin_amdgcn_sched_barrier(0);
      const bool need_mask = (kb + BKV > L) || (CAUSAL && kb + BKV - 1 > qw0);
      if (need_mask) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            int key = kb + t * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
            bool ok = key < L && (!CAUSAL || key <= qi);
            s[t][r] = ok ? s[t][r] : -INFINITY;
          }
      }
      float mt = -INFINITY;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) mt = fmaxf(mt, s[t][r]);
      // both halves' maxima in every lane
      const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mt), __float_as_uint(mt), false, false);
      mt = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1])) * scale_log2;
      if (__any((mt > m_run + 8.f) ? 1 : 0)) {
        const float m_new = fmaxf(m_run, mt);
        const float alpha = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - m_new);
        l_part *= alpha;
#pragma unroll
        for (int t = 0; t < ND; ++t)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc_o[t][r] *= alpha;
        m_run = m_new;
      }
      const float m_use = (m_run == -INFINITY) ? 0.f : m_run;
      float psum = 0.f;
      // the next tile's scores on the matrix cores between this tile's
      // exponentials (past the last tile: scores of stale rows, never used)
#pragma unroll
      for (int i = 0; i < NMF; ++i) {
        const int ks = i >> 1, t = i & 1;
        sn[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i % LA], fq[ks], ks == 0 ? zero : sn[t], 0, 0, 0);
        fetch(i + LA);
#pragma unroll
        for (int x = i * EPM; x < (i + 1) * EPM; ++x) {
          const float p = __builtin_amdgcn_exp2f(fmaf(s[x >> 4][x & 15], scale_log2, -m_use));
          s[x >> 4][x & 15] = p;
          psum += p;
        }
        __builtin_amdgcn_sched_barrier(0x406);
      }
      l_part += psum;
#pragma unroll
      for (int c4 = 0; c4 < 4; ++c4) {
        const int t = c4 >> 1, ih = c4 & 1;
        union {
          uint32_t u[4];
          bf16x8 v;
        } cv;
        cv.u[0] = pack_bf2(s[t][(2 * ih) * 4 + 0], s[t][(2 * ih) * 4 + 1]);
        cv.u[1] = pack_bf2(s[t][(2 * ih) * 4 + 2], s[t][(2 * ih) * 4 + 3]);
        cv.u[2] = pack_bf2(s[t][(2 * ih + 1) * 4 + 0], s[t][(2 * ih + 1) * 4 + 1]);
        cv.u[3] = pack_bf2(s[t][(2 * ih + 1) * 4 + 2], s[t][(2 * ih + 1) * 4 + 3]);
#pragma unroll
        for (int dt = 0; dt < ND; ++dt) {
          const int i = NMF + c4 * ND + dt;
          acc_o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i % LA], cv.v, acc_o[dt], 0, 0, 0);
          fetch(i + LA);
          __builtin_amdgcn_sched_barrier(0x406);
        }
      }
    }
  };
  for (int base = 0; base < ntiles; base += 2) {
    body(std::integral_constant<int, 0>{}, base, sa, sb);
    if (base + 1 < ntiles) body(std::integral_constant<int, 1>{}, base + 1, sb, sa);
  }

  const float l_tot = l_part + __shfl_xor(l_part, 32, 64);
  if (qi < L) {
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
    bf16_t* orow = o + ((size_t)b * L + qi) * (size_t)(H * DH) + h * DH;
#pragma unroll
    for (int dt = 0; dt < ND; ++dt)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        int d = dt * 32 + g * 8 + half * 4;
        u32x2 w = {pack_bf2(acc_o[dt][g * 4 + 0] * inv, acc_o[dt][g * 4 + 1] * inv),
                   pack_bf2(acc_o[dt][g * 4 + 2] * inv, acc_o[dt][g * 4 + 3] * inv)};
        *(u32x2*)(orow + d) = w;
      }
  }
}

template <int DH, bool CAUSAL>
hipError_t launch_attn(const bf16_t* q, const bf16_t* k, const bf16_t* vt, int ldvt, bf16_t* o, int B, int H, int Hkv,
                       int L, hipStream_t s) {
  const int nqb = (L + BQ - 1) / BQ;
  const float scale_log2 = 1.4426950408889634f / sqrtf((float)DH);
  hipLaunchKernelGGL((attn_bf16_kernel<DH, CAUSAL>), dim3(nqb * H * B), dim3(256), 0, s, q, k, vt, ldvt, o, B, H, Hkv,
                     L, scale_log2);
  return hipGetLastError();
}

}  // namespace

hipError_t attention_bf16(const bf16_t* q, const bf16_t* k, const bf16_t* vt, int ldvt, bf16_t* o, int B, int H,
                          int Hkv, int L, int dh, bool causal, hipStream_t s) {
  if (B <= 0 || L <= 0 || H <= 0) return hipSuccess;
  if (Hkv <= 0 || H % Hkv != 0 || ldvt < (L + 15) / 16 * 16 || ldvt % 16 != 0)
    return hipErrorInvalidValue;
  if (dh == 128) return causal ? launch_attn<128, true>(q, k, vt, ldvt, o, B, H, Hkv, L, s)
                               : launch_attn<128, false>(q, k, vt, ldvt, o, B, H, Hkv, L, s);
  if (dh == 64) return causal ? launch_attn<64, true>(q, k, vt, ldvt, o, B, H, Hkv, L, s)
                              : launch_attn<64, false>(q, k, vt, ldvt, o, B, H, Hkv, L, s);
  return hipErrorInvalidValue;
}

}  // namespace vla

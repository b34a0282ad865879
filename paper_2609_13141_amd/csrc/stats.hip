// Selection-analysis statistics (Sec. 6.1): attention mass coverage of the
// attended set (Eq. mass_coverage, raw and value-norm weights), the
// full-attention reference sets (per-head Top-K blocks by attention mass,
// merged per KV group by majority vote) and the cross-layer overlap recall
// (Eq. overlap_recall) on OR-accumulated block bitmasks.
//
// The coverage pass is a dense causal pass in the forward attention's layout
// (S^T = K Q^T on v_mfma_f32_32x32x16_bf16, lane = query, partner lane l^32)
// without the PV product: per query it keeps two running references (raw and
// value-aware logits, log2 domain) and four sums (all keys / attended keys,
// each weighting), and the log-sum-exp of every historical block's raw
// logits for the reference Top-K.
#include <float.h>

#include <stdint.h>

#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace sas {

constexpr float SLOG2E = 1.4426950408889634f;

// lvn[b, t, g] = log2 ||v[b, t, g, :]||_2 (fp32 sum of squares; -inf for a zero row)
template <typename T, int DH>
__global__ void vnorm_kernel(const T* __restrict__ V, size_t rows, float* __restrict__ lvn) {
  const size_t r = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= rows) return;
  const T* v = V + r * DH;
  float ss = 0.f;
  for (int j = 0; j < DH; j += 8) {
    Vec8<T> x;
    x.load(v + j);
#pragma unroll
    for (int e = 0; e < 8; ++e) ss = fmaf(x.get(e), x.get(e), ss);
  }
  lvn[r] = 0.5f * log2f(ss);
}

// log2(2^a + 2^b), either may be -inf
__device__ __forceinline__ float lse2(float a, float b) {
  const float m = fmaxf(a, b);
  if (m == -INFINITY) return -INFINITY;
  return m + log2f(exp2f(a - m) + exp2f(b - m));
}

typedef __attribute__((address_space(3))) void stats_lds_t;

// Bound by VALU issue: one exponential per (query, key).  A tile's p = 2^(z - its
// largest z) serves the raw and, times the key's value norm, the value-aware
// sums (norms relative to the tile's largest, both references carried in the
// log2 domain), so neither weighting needs an exponential or a maximum of its
// own; sums are per sub-block and join the attended set's as a whole.  Where a
// query's sum falls under 2^-60 of its reference (large logits at keys of tiny
// values: products would leave the range of float) the wave redoes the tile's
// value-aware sums relative to their own maximum.  K rows go straight to LDS
// into the other of two buffers, one barrier per tile.
// 2 x 2048 tokens, 32 heads: 97 us; with an exponential and a
// running maximum per weighting, staged K and two barriers 162.
template <int DH, int LSB>
__device__ __forceinline__ void stats_bf16_job(const StatsArgs& P, const int qtile, const int h, const int bi) {
  constexpr int C8 = DH / 8;
  constexpr int NSUB = 64 >> LSB;
  constexpr int TB = 64 * DH * 2;    // bytes of a K tile
  constexpr int NL = 64 * C8 / 256;  // 16-byte pieces per thread and tile
  constexpr int NA = NSUB == 1 ? 4 : 1;  // partial sums per sub-block
  // two K tiles (2 TB bytes; dynamic, because the compiler makes every read of a
  // static array wait for the direct-to-LDS loads in flight)
  extern __shared__ __align__(16) unsigned char stats_tiles[];
  __shared__ __align__(16) float w_s[2][64];  // value norms of the tile's keys over the largest
  __shared__ float wmax_s[2];                 // log2 of that
  __shared__ float lv_s[2][64];               // log2 norms themselves

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 31, lk = lane >> 5;
  const int G = P.H / P.Hkv, g = h / G;
  const int n = P.n, B = P.B;
  const int qrow = wave * 32 + lr;
  const int t = qtile * 128 + qrow;
  const bool qvalid = t < n;
  const int beta = qvalid ? t / B : -1;
  const bool dense = P.mode == SAS_MODE_DENSE;
  const int Kn = dense ? 0 : P.K;
  const int NB = (n + B - 1) / B;
  const int t_hi = min(n, qtile * 128 + 128) - 1;
  const int last_tile = t_hi / 64;
  const size_t grow = ((size_t)bi * P.Hkv + g) * n;
  const size_t hrow = ((size_t)bi * P.H + h) * n + (qvalid ? t : 0);
  const int fb = qvalid ? doc_first(P.doc, bi, NB, t, B) : 0;  // the query's document starts at block fb
  const int first_tile = doc_first(P.doc, bi, NB, qtile * 128, B) * B / 64;

  bf16x8_t qb[DH / 16];
  {
    const bf16_t* qp = (const bf16_t*)P.Q + (((size_t)bi * n + (qvalid ? t : 0)) * P.H + h) * DH;
#pragma unroll
    for (int ks = 0; ks < DH / 16; ++ks) {
      uint4 u = qvalid ? *(const uint4*)(qp + ks * 16 + lk * 8) : make_uint4(0, 0, 0, 0);
      qb[ks] = *(bf16x8_t*)&u;
    }
  }

  const float qk_scale = P.sm_scale * SLOG2E;
  const bf16_t* Kg = (const bf16_t*)P.Kt + (size_t)g * DH;
  const size_t kstride = (size_t)P.Hkv * DH;
  const size_t kbase = (size_t)bi * n;
  float rl = 0.f;  // wave 0: log2 norm of the next tile's key `lane`
  auto load_tile = [&](int kt, int buf) {  // keys past the end repeat the last one (masked)
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int p = (wave * NL + i) * 64 + lane, r = p / C8, c = (p % C8) ^ lds_swz<DH>(r);
      __builtin_amdgcn_global_load_lds((const void*)(Kg + (kbase + min(kt * 64 + r, n - 1)) * kstride + c * 8),
                                       (stats_lds_t*)(stats_tiles + buf * TB + (wave * NL + i) * 1024), 16, 0, 0);
    }
    if (wave == 0) rl = P.lvn[(kbase + min(kt * 64 + lane, n - 1)) * P.Hkv + g];
  };
  auto commit_norms = [&](int kt, int buf) {
    if (wave != 0) return;
    const float l = kt * 64 + lane < n ? rl : -INFINITY;
    const float mxl = wave_max(l);
    w_s[buf][lane] = __builtin_amdgcn_exp2f(l - (mxl == -INFINITY ? 0.f : mxl));
    lv_s[buf][lane] = l;
    if (lane == 0) wmax_s[buf] = mxl;
  };
  uint32_t o_row = lr * DH * 2 + ((lk ^ lds_swz<DH>(lr)) << 4);  // row lr, chunk 2 ks + lk: o_row ^ (ks << 5)

  float m_raw = -INFINITY, m_val = -INFINITY;         // running references (log2 domain)
  float l_all = 0.f, l_S = 0.f, l_vall = 0.f, l_vS = 0.f;
  float blk_acc = -INFINITY;                           // log2 mass of a block wider than a tile so far
  // selection cursor: slot `cur` (block next_sel) and the one after it, read one slot ahead
  const size_t srow = (grow + (qvalid ? t : 0)) * (size_t)Kn;
  auto sel_at = [&](int k) -> int { return P.sel[srow + min(k, Kn - 1)]; };  // Kn > 0
  int cur = 0, next_sel = 0x7fffffff, s_nx = -1;
  if (Kn > 0) {
    const int s0 = sel_at(0);
    s_nx = sel_at(1);
    if (qvalid && s0 >= 0) next_sel = s0;
  }
  // the queries have arrived (else the compiler waits for all loads at their first
  // use, which is in the loop)
#pragma unroll
  for (int ks = 0; ks < DH / 16; ++ks) asm volatile("" : "+v"(*(u32x4_t*)&qb[ks]));
  int buf = 0;
  load_tile(first_tile, 0);
  commit_norms(first_tile, 0);
  for (int kt = first_tile; kt <= last_tile; ++kt) {
    // this wave's loads of the tile are done; after the barrier everyone's are,
    // and every wave is done with the other buffer
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const int k0 = kt * 64;
    const unsigned char* const tb = stats_tiles + buf * TB;
    // membership of the attended set per sub-block (causal context only)
    bool inS[NSUB], ctx[NSUB];
#pragma unroll
    for (int sb = 0; sb < NSUB; ++sb) {
      const int kstart = k0 + (sb << LSB);
      ctx[sb] = qvalid && kstart <= t && kstart / B >= fb;
      inS[sb] = false;
      if (!ctx[sb]) continue;
      const int m = kstart / B;
      if (m == beta || dense) {
        inS[sb] = true;
      } else if (m == next_sel) {
        inS[sb] = true;
        if (kstart + (1 << LSB) >= (m + 1) * B) {
          ++cur;
          next_sel = cur < Kn && s_nx >= 0 ? s_nx : 0x7fffffff;
          s_nx = sel_at(cur + 1);
        }
      }
    }
    if (kt < last_tile) load_tile(kt + 1, buf ^ 1);

    auto logits = [&](floatx16_t (&s)[2]) {
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int v = 0; v < 16; ++v) s[st][v] = 0.f;
      __builtin_amdgcn_s_setprio(2);
#pragma unroll
      for (int ks = 0; ks < DH / 16; ++ks) {
        const unsigned char* row = tb + (o_row ^ (ks << 5));
        const bf16x8_t a0 = *(const bf16x8_t*)row, a1 = *(const bf16x8_t*)(row + 32 * DH * 2);
        s[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, qb[ks], s[0], 0, 0, 0);
        s[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, qb[ks], s[1], 0, 0, 0);
      }
      __builtin_amdgcn_s_setprio(0);
      if (k0 + 63 > qtile * 128) {  // keys past some query of the workgroup
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
          for (int v = 0; v < 16; ++v)
            if (k0 + st * 32 + 8 * (v >> 2) + 4 * lk + (v & 3) > t) s[st][v] = -INFINITY;
      }
    };
    floatx16_t s[2];
    logits(s);
    // the tile's largest logit (the scale is positive: per sub-block the largest raw score)
    float mxs[NSUB];
#pragma unroll
    for (int sb = 0; sb < NSUB; ++sb) mxs[sb] = -INFINITY;
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int sb = (st * 32 + 8 * (v >> 2)) >> LSB;
        mxs[sb] = fmaxf(mxs[sb], s[st][v]);
      }
    float mx = -INFINITY;
#pragma unroll
    for (int sb = 0; sb < NSUB; ++sb) mx = fmaxf(mx, ctx[sb] ? mxs[sb] * qk_scale : -INFINITY);
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float ref = mx == -INFINITY ? 0.f : mx;
    float bs[NSUB][NA], vs[NSUB][NA];
#pragma unroll
    for (int sb = 0; sb < NSUB; ++sb)
#pragma unroll
      for (int i = 0; i < NA; ++i) bs[sb][i] = vs[sb][i] = 0.f;
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int sb = (st * 32 + 8 * j) >> LSB;
        const float4 w4 = *(const float4*)&w_s[buf][st * 32 + 8 * j + 4 * lk];
        const float w[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float p = __builtin_amdgcn_exp2f(fmaf(s[st][4 * j + i], qk_scale, -ref));
          bs[sb][i % NA] += p;
          vs[sb][i % NA] = fmaf(p, w[i], vs[sb][i % NA]);
        }
      }
    float sa = 0.f, sS = 0.f, sva = 0.f, svS = 0.f, bsum[NSUB];
#pragma unroll
    for (int sb = 0; sb < NSUB; ++sb) {
      float x = bs[sb][0], y = vs[sb][0];
#pragma unroll
      for (int i = 1; i < NA; ++i) {
        x += bs[sb][i];
        y += vs[sb][i];
      }
      x += __shfl_xor(x, 32, 64);
      y += __shfl_xor(y, 32, 64);
      if (!ctx[sb]) x = y = 0.f;  // whatever these keys hold
      bsum[sb] = x;
      sa += x;
      sva += y;
      if (inS[sb]) {
        sS += x;
        svS += y;
      }
    }
    // join the running sums: raw reference mx, value-aware mx + log2 of the largest norm
    const float wmax = wmax_s[buf];
    float mxv = wmax == -INFINITY ? -INFINITY : mx + wmax;
    if (__any(sva < 0x1p-60f && mxv > -INFINITY)) {
      floatx16_t z[2];
      logits(z);
      mxv = -INFINITY;
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          z[st][v] = ctx[(st * 32 + 8 * (v >> 2)) >> LSB]
                         ? fmaf(z[st][v], qk_scale, lv_s[buf][st * 32 + 8 * (v >> 2) + 4 * lk + (v & 3)]) : -INFINITY;
          mxv = fmaxf(mxv, z[st][v]);
        }
      mxv = fmaxf(mxv, __shfl_xor(mxv, 32, 64));
      const float zr = mxv == -INFINITY ? 0.f : mxv;
      sva = svS = 0.f;
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float p = __builtin_amdgcn_exp2f(z[st][v] - zr);
          sva += p;
          if (inS[(st * 32 + 8 * (v >> 2)) >> LSB]) svS += p;
        }
      sva += __shfl_xor(sva, 32, 64);
      svS += __shfl_xor(svS, 32, 64);
    }
    const float mn = fmaxf(m_raw, mx), mnv = fmaxf(m_val, mxv);
    const float mu = mn == -INFINITY ? 0.f : mn, muv = mnv == -INFINITY ? 0.f : mnv;
    const float a = __builtin_amdgcn_exp2f(m_raw - mu), c = __builtin_amdgcn_exp2f(mx - mu);
    const float av = __builtin_amdgcn_exp2f(m_val - muv), cv = __builtin_amdgcn_exp2f(mxv - muv);
    l_all = l_all * a + sa * c;
    l_S = l_S * a + sS * c;
    l_vall = l_vall * av + sva * cv;
    l_vS = l_vS * av + svS * cv;
    m_raw = mn;
    m_val = mnv;
    // block masses of the historical blocks (reference Top-K)
#pragma unroll
    for (int sb = 0; sb < NSUB; ++sb) {
      const int kstart = k0 + (sb << LSB), m = kstart / B;
      if (P.blk_lse && lk == 0 && ctx[sb] && m < beta) {
        blk_acc = lse2(blk_acc, bsum[sb] > 0.f ? ref + log2f(bsum[sb]) : -INFINITY);
        if (kstart + (1 << LSB) >= (m + 1) * B) {
          P.blk_lse[hrow * NB + m] = blk_acc;
          blk_acc = -INFINITY;
        }
      }
    }
    buf ^= 1;
    if (kt < last_tile) commit_norms(kt + 1, buf);
  }
  if (!qvalid || lk != 0) return;
  if (P.cov) P.cov[hrow] = l_S / l_all;
  if (P.cov_v) P.cov_v[hrow] = l_vS / l_vall;
}

// One job (query tile, head, batch entry) per workgroup (grid = job count, no
// queue) or the work queue; the heavy (late) query tiles first.
template <int DH, int LSB>
__global__ void __launch_bounds__(256, 2) stats_bf16_kernel(StatsArgs P) {
  const int nqt = (P.n + 127) / 128, per = P.H * P.b;
  const int njobs = nqt * per;
  for (int it = 0;; ++it) {
    const int job = P.queue ? queue_next_job(P.queue) : (it == 0 ? (int)blockIdx.x : njobs);
    if (job >= njobs) break;
    const int r = job % per;
    __syncthreads();  // the previous job is done with LDS
    stats_bf16_job<DH, LSB>(P, nqt - 1 - job / per, r % P.H, r / P.H);
  }
}

// fp32: one thread per (batch, head, query), sums in fp32 against running maxima
template <int DH>
__global__ void stats_f32_kernel(StatsArgs P) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int n = P.n;
  if (idx >= (size_t)P.b * P.H * n) return;
  const int t = (int)(idx % n), h = (int)((idx / n) % P.H), bi = (int)(idx / ((size_t)n * P.H));
  const int G = P.H / P.Hkv, g = h / G, B = P.B, beta = t / B;
  const int NB = (n + B - 1) / B;
  const float* q = (const float*)P.Q + (((size_t)bi * n + t) * P.H + h) * DH;
  const size_t row = ((size_t)bi * P.Hkv + g) * n + t;
  const size_t hrow = ((size_t)bi * P.H + h) * n + t;
  float qv[DH];
#pragma unroll
  for (int j = 0; j < DH; ++j) qv[j] = q[j];
  float m_raw = -INFINITY, m_val = -INFINITY, l_all = 0.f, l_S = 0.f, l_vall = 0.f, l_vS = 0.f;
  int cur = 0;
  for (int m = doc_first(P.doc, bi, NB, t, B); m <= beta; ++m) {
    bool in = m == beta || P.mode == SAS_MODE_DENSE;
    if (!in && P.K > 0) {
      while (cur < P.K && P.sel[row * P.K + cur] >= 0 && P.sel[row * P.K + cur] < m) ++cur;
      in = cur < P.K && P.sel[row * P.K + cur] == m;
    }
    float bm = -INFINITY, bl = 0.f;  // the block's own log2 mass
    const int i1 = m == beta ? t : (m + 1) * B - 1;
    for (int i = m * B; i <= i1; ++i) {
      const float* k = (const float*)P.Kt + (((size_t)bi * n + i) * P.Hkv + g) * DH;
      float z = 0.f;
#pragma unroll
      for (int j = 0; j < DH; ++j) z = fmaf(qv[j], k[j], z);
      const float x = z * P.sm_scale * SLOG2E;
      const float y = x + P.lvn[((size_t)bi * n + i) * P.Hkv + g];
      if (x > m_raw) {
        const float a = exp2f(m_raw - x);
        l_all *= a;
        l_S *= a;
        m_raw = x;
      }
      if (y > m_val) {
        const float a = exp2f(m_val - y);
        l_vall *= a;
        l_vS *= a;
        m_val = y;
      }
      const float p = exp2f(x - m_raw), pv = exp2f(y - m_val);
      l_all += p;
      l_vall += pv;
      if (in) {
        l_S += p;
        l_vS += pv;
      }
      if (x > bm) {
        bl = bl * exp2f(bm - x) + 1.f;
        bm = x;
      } else {
        bl += exp2f(x - bm);
      }
    }
    if (P.blk_lse && m < beta) P.blk_lse[hrow * NB + m] = bm + log2f(bl);
  }
  if (P.cov) P.cov[hrow] = l_S / l_all;
  if (P.cov_v) P.cov_v[hrow] = l_vS / l_vall;
}

// Per-head Top-K historical blocks by block mass (descending, lower block
// first on ties; NaN never), as a bitmask row [W words]; one thread per (b, h, t).
// Bound by VALU issue: the first walk keeps only the KMAX largest values, sorted,
// one median per slot and block (an inserted x leaves max(min(x, tv[i-1]), tv[i])
// in slot i); the second sets the blocks above the last one taken and the first
// of those equal to it.  Rows are read 8 blocks at a time.  2 x 2048 tokens, 32
// heads, 32 blocks, K = 16: 17 us, with indices carried through the slots 37.
template <int KMAX>
__global__ void ref_topk_kernel(const float* __restrict__ blk_lse, size_t rows, int n, int H, int B, int K, int NB,
                                int W, uint32_t* __restrict__ head_mask, const int32_t* __restrict__ doc) {
  const size_t r = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= rows) return;
  const int t = (int)(r % n);
  const int C = t / B;
  const int F = doc_first(doc, (int)(r / ((size_t)n * H)), NB, t, B);  // historical blocks [F, C)
  const int kk = min(K, C - F);
  const float* row = blk_lse + r * NB;
  float tv[KMAX];
#pragma unroll
  for (int i = 0; i < KMAX; ++i) tv[i] = -INFINITY;
  for (int m0 = F; m0 < C; m0 += 8) {
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = row[min(m0 + j, C - 1)];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float x = m0 + j < C && v[j] == v[j] ? v[j] : -INFINITY;  // one more -inf changes nothing
#pragma unroll
      for (int i = KMAX - 1; i > 0; --i) tv[i] = __builtin_amdgcn_fmed3f(x, tv[i - 1], tv[i]);
      tv[0] = fmaxf(x, tv[0]);
    }
  }
  float last = -INFINITY;  // value in slot kk - 1
#pragma unroll
  for (int i = 0; i < KMAX; ++i)
    if (i < kk) last = tv[i];
  int ties = kk;  // slots that hold `last`
#pragma unroll
  for (int i = 0; i < KMAX; ++i)
    if (i < kk && tv[i] > last) --ties;
  uint32_t* out = head_mask + r * W;
  for (int w = 0; w < W; ++w) {
    uint32_t bits = 0;
    if (kk > 0)
      for (int m0 = max(F, w * 32); m0 < min(C, w * 32 + 32); m0 += 8) {
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = row[min(m0 + j, C - 1)];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int m = m0 + j;
          const bool tie = v[j] == last && ties > 0, in = m < C && m < w * 32 + 32 && (v[j] > last || tie);
          if (in) bits |= 1u << (m & 31);
          if (in && tie) --ties;
        }
      }
    out[w] = bits;
  }
}

// group set = blocks chosen by more than half of the group's heads; OR into the union
__global__ void vote_union_kernel(const uint32_t* __restrict__ head_mask, int b, int n, int H, int Hkv, int W,
                                  uint32_t* __restrict__ uni) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)b * Hkv * n * W) return;
  const int w = (int)(idx % W), t = (int)((idx / W) % n), g = (int)((idx / ((size_t)W * n)) % Hkv);
  const int bi = (int)(idx / ((size_t)W * n * Hkv));
  const int G = H / Hkv;
  uint32_t bits = 0;
  for (int j = 0; j < 32; ++j) {
    int cnt = 0;
    for (int hh = g * G; hh < (g + 1) * G; ++hh)
      cnt += (head_mask[(((size_t)bi * H + hh) * n + t) * W + w] >> j) & 1u;
    if (2 * cnt > G) bits |= 1u << j;
  }
  uni[idx] |= bits;
}

// OR the selection rows [b, Hkv, n, K] into the union bitmask
__global__ void sel_union_kernel(const int32_t* __restrict__ sel, size_t rows, int K, int NB, int W,
                                 uint32_t* __restrict__ uni) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= rows * W) return;
  const size_t row = idx / W;
  const int w = (int)(idx % W);
  uint32_t bits = 0;
  for (int k = 0; k < K; ++k) {
    const int m = sel[row * K + k];
    if (m >= 0 && m < NB && (m >> 5) == w) bits |= 1u << (m & 31);
  }
  uni[idx] |= bits;
}

__global__ void zero_u64_kernel(unsigned long long* p, int n) {
  if ((int)threadIdx.x < n) p[threadIdx.x] = 0ull;
}

// counts[0] += |a & b|, counts[1] += |b| over every word
__global__ void overlap_count_kernel(const uint32_t* __restrict__ a, const uint32_t* __restrict__ b, size_t words,
                                     unsigned long long* __restrict__ counts) {
  __shared__ unsigned long long part[2][4];
  unsigned long long ci = 0, cb = 0;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += (size_t)gridDim.x * blockDim.x) {
    const uint32_t bw = b[i];
    ci += __popc(a[i] & bw);
    cb += __popc(bw);
  }
  for (int off = 32; off > 0; off >>= 1) {
    ci += __shfl_xor(ci, off, 64);
    cb += __shfl_xor(cb, off, 64);
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
    part[0][wave] = ci;
    part[1][wave] = cb;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long si = 0, sb = 0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
      si += part[0][w];
      sb += part[1][w];
    }
    atomicAdd(&counts[0], si);
    atomicAdd(&counts[1], sb);
  }
}

hipError_t launch_vnorm(int dtype, const void* V, size_t rows, int dh, float* lvn, hipStream_t s) {
  if (rows == 0) return hipSuccess;
  const unsigned grid = (unsigned)cdiv(rows, 256);
  if (dtype == SAS_BF16) {
    if (dh == 128) vnorm_kernel<bf16_t, 128><<<grid, 256, 0, s>>>((const bf16_t*)V, rows, lvn);
    else vnorm_kernel<bf16_t, 64><<<grid, 256, 0, s>>>((const bf16_t*)V, rows, lvn);
  } else {
    if (dh == 128) vnorm_kernel<float, 128><<<grid, 256, 0, s>>>((const float*)V, rows, lvn);
    else vnorm_kernel<float, 64><<<grid, 256, 0, s>>>((const float*)V, rows, lvn);
  }
  return hipGetLastError();
}

hipError_t launch_stats(int dtype, const StatsArgs& a, hipStream_t s) {
  if (a.n <= 0 || a.b <= 0) return hipSuccess;
  if (a.K > 32) return hipErrorInvalidValue;
  if (dtype != SAS_BF16) {
    const size_t tot = (size_t)a.b * a.H * a.n;
    if (a.dh == 128) stats_f32_kernel<128><<<(unsigned)cdiv(tot, 64), 64, 0, s>>>(a);
    else stats_f32_kernel<64><<<(unsigned)cdiv(tot, 64), 64, 0, s>>>(a);
    return hipGetLastError();
  }
  const int lsb = a.B >= 64 ? 6 : (a.B == 32 ? 5 : 4);
  auto kern = a.dh == 128 ? (lsb == 6 ? stats_bf16_kernel<128, 6> : lsb == 5 ? stats_bf16_kernel<128, 5>
                                                                              : stats_bf16_kernel<128, 4>)
                          : (lsb == 6 ? stats_bf16_kernel<64, 6> : lsb == 5 ? stats_bf16_kernel<64, 5>
                                                                             : stats_bf16_kernel<64, 4>);
  const long long jobs = (long long)cdiv(a.n, 128) * a.H * a.b;
  const size_t lds = (size_t)256 * a.dh;  // two K tiles (at most 32 KB)
  const int res = resident_workgroups(kern, 256, lds);
  if (res <= 0 || jobs > INT32_MAX) return hipErrorInvalidValue;
  StatsArgs A = a;
  A.queue = nullptr;
  if (jobs > res) {
    if (!a.queue) return hipErrorInvalidValue;
    const hipError_t e = launch_fill_f32((float*)a.queue, 1, 0.f, s);  // the job counter to zero
    if (e != hipSuccess) return e;
    A.queue = a.queue;
  }
  kern<<<(unsigned)std::min<long long>(jobs, res), 256, lds, s>>>(A);
  return hipGetLastError();
}

hipError_t launch_ref_sets(const float* blk_lse, int b, int n, int H, int Hkv, int B, int K, uint32_t* head_mask,
                           uint32_t* uni, const int32_t* doc, hipStream_t s) {
  const int NB = cdiv(n, B), W = cdiv(NB, 32);
  const size_t rows = (size_t)b * H * n;
  if (rows == 0) return hipSuccess;
  const unsigned grid = (unsigned)cdiv(rows, 128);
  if (K <= 8) ref_topk_kernel<8><<<grid, 128, 0, s>>>(blk_lse, rows, n, H, B, K, NB, W, head_mask, doc);
  else if (K <= 16) ref_topk_kernel<16><<<grid, 128, 0, s>>>(blk_lse, rows, n, H, B, K, NB, W, head_mask, doc);
  else ref_topk_kernel<32><<<grid, 128, 0, s>>>(blk_lse, rows, n, H, B, K, NB, W, head_mask, doc);
  const size_t tot = (size_t)b * Hkv * n * W;
  vote_union_kernel<<<(unsigned)cdiv(tot, 256), 256, 0, s>>>(head_mask, b, n, H, Hkv, W, uni);
  return hipGetLastError();
}

hipError_t launch_sel_union(const int32_t* sel, size_t rows, int K, int NB, uint32_t* uni, hipStream_t s) {
  const int W = cdiv(NB, 32);
  if (rows * W == 0) return hipSuccess;
  sel_union_kernel<<<(unsigned)cdiv(rows * W, 256), 256, 0, s>>>(sel, rows, K, NB, W, uni);
  return hipGetLastError();
}

hipError_t launch_overlap_count(const uint32_t* a, const uint32_t* b, size_t words, unsigned long long* counts,
                                hipStream_t s) {
  zero_u64_kernel<<<1, 64, 0, s>>>(counts, 2);
  if (words == 0) return hipGetLastError();
  const size_t blocks = cdiv(words, 256);
  const unsigned grid = (unsigned)(blocks < 1024 ? blocks : 1024);
  overlap_count_kernel<<<grid, 256, 0, s>>>(a, b, words, counts);
  return hipGetLastError();
}

}  // namespace sas

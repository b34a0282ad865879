// Backward of SAS attention (Sec. 4.3, Eq. ours_train; the recomputation
// backward of App. E) and of the selector's normalized log gate
// (Eq. normalized_log_gate), for the selector update of Alg. 1.
//
// Per (head h of group g, query t) over the forward's attended set S with
// z_i = sm q.k_i + bias_i and p = exp(z - LSE):
//   Delta = dO . O,  dp_i = dO . v_i,  ds_i = p_i (dp_i - Delta)
//   dq = sm sum_i ds_i k_i,  dk_i += sm ds_i q,  dv_i += p_i dO
//   dlog g[g, t, slot of m] = sum_{h in g} sum_{i in B_m} ds_i   (GATED)
// Pass 1 walks queries (dQ and the per-head block sums of ds); pass 2 walks
// keys (dK, dV) and visits only the query chunks that attend them.
//
// Selector (the end of this file): the gate's softmax backward gives the
// score gradient ds of each row's historical blocks; the scores are inner
// products of gate queries and block summaries, so their gradients (and
// those of the optional projections) are small batched GEMMs over ds.
#include <float.h>
#include <stdint.h>

#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace sas {

// Delta[b, h, t] = sum_d O[b, t, h, d] dO[b, t, h, d] (fp32): dh / 8 threads per
// row (rows (b, t, h) are contiguous in [b, n, H, dh]), 16-byte loads of 8
// values each, the partial sums added across the row's lanes.
template <typename T>
__global__ void __launch_bounds__(256) bwd_delta_kernel(const T* __restrict__ O, const T* __restrict__ dO, int b,
                                                        int n, int H, int dh, float* __restrict__ delta) {
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int tpr = dh / 8;  // threads per row: 16 or 8, aligned groups of lanes
  const size_t rows = (size_t)b * n * H, row = gid / tpr;
  const int c8 = (int)(gid % tpr);
  const bool valid = row < rows;
  float acc = 0.f;
  if (valid) {
    Vec8<T> o, d;
    o.load(O + row * dh + c8 * 8);
    d.load(dO + row * dh + c8 * 8);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc = fmaf(o.get(e), d.get(e), acc);
  }
  for (int sh = tpr >> 1; sh > 0; sh >>= 1) acc += __shfl_xor(acc, sh, 64);
  if (valid && c8 == 0) {
    const int h = (int)(row % H), t = (int)((row / H) % n), bi = (int)(row / ((size_t)H * n));
    delta[((size_t)bi * H + h) * n + t] = acc;
  }
}

// How block m enters the attention of query t and its gradient (natural-log
// domain): att = attended (dQ, dK, dV terms); grad = receives a log-gate
// gradient; bias = logit bias; w = value weight; lg = the block's log gate;
// slot = its selection slot (-1 if none).
struct BlockGate {
  bool att, grad;
  float bias, w, lg;
  int slot;
};

__device__ BlockGate block_gate(const BwdArgs& P, int bi, int g, int t, int m) {
  BlockGate r = {false, false, 0.f, 1.f, 0.f, -1};
  const int beta = t / P.B;
  const int NBr = (P.n + P.B - 1) / P.B;
  if (m > beta || (m < beta && m < doc_first(P.doc, bi, NBr, t, P.B))) return r;  // outside the document
  if (m == beta || P.mode == SAS_MODE_DENSE) {
    r.att = true;
    return r;
  }
  const bool gated = P.mode == SAS_MODE_GATED;
  const size_t row = ((size_t)bi * P.Hkv + g) * P.n + t;
  const int NB = (P.n + P.B - 1) / P.B;
  if (gated && P.full && !P.ste) {  // every historical block, gate from the table
    r.att = r.grad = true;
    r.lg = P.log_gate[row * NB + m];
  } else {
    for (int k = 0; k < P.K; ++k) {
      const int s = P.sel[row * P.K + k];
      if (s < 0 || s > m) break;
      if (s == m) {
        r.att = true;
        r.grad = gated;
        r.slot = k;
        r.lg = gated ? P.sel_bias[row * P.K + k] : 0.f;
        break;
      }
    }
    if (!r.att && gated && P.ste && P.full) {  // straight-through gradient of a dropped block
      r.grad = true;
      r.lg = P.log_gate[row * NB + m];
    }
  }
  if (gated && !P.ste) {
    if (P.outer) r.w = expf(r.lg);
    else r.bias = r.lg;
  }
  return r;
}

// ---- fp32 path ------------------------------------------------------------------
// pass 1: one thread per (batch, head, query)
template <int DH>
__global__ void __launch_bounds__(64) bwd_dq_f32_kernel(BwdArgs P) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int n = P.n;
  if (idx >= (size_t)P.b * P.H * n) return;
  const int t = (int)(idx % n), h = (int)((idx / n) % P.H), bi = (int)(idx / ((size_t)n * P.H));
  const int G = P.H / P.Hkv, g = h / G, B = P.B;
  const int NB = (n + B - 1) / B;
  const float* q = (const float*)P.Q + (((size_t)bi * n + t) * P.H + h) * DH;
  const float* dO = (const float*)P.dO + (((size_t)bi * n + t) * P.H + h) * DH;
  const size_t hrow = ((size_t)bi * P.H + h) * n + t;
  const float lse = P.lse[hrow];
  const float delta = P.delta[hrow];
  float qv[DH], dov[DH], dq[DH];
#pragma unroll
  for (int j = 0; j < DH; ++j) {
    qv[j] = q[j];
    dov[j] = dO[j];
    dq[j] = 0.f;
  }
  float* dlg = P.dlg_head ? P.dlg_head + hrow * P.K : nullptr;
  const int beta = t / B;
  for (int m = 0; m <= beta; ++m) {
    const BlockGate bg = block_gate(P, bi, g, t, m);
    if (!bg.att && !bg.grad) continue;
    const int i1 = m == beta ? t : (m + 1) * B - 1;
    float dsum = 0.f;
    for (int i = m * B; i <= i1; ++i) {
      const float* k = (const float*)P.Kt + (((size_t)bi * n + i) * P.Hkv + g) * DH;
      const float* v = (const float*)P.V + (((size_t)bi * n + i) * P.Hkv + g) * DH;
      float z = 0.f, dp = 0.f;
#pragma unroll
      for (int j = 0; j < DH; ++j) {
        z = fmaf(qv[j], k[j], z);
        dp = fmaf(dov[j], v[j], dp);
      }
      const float p = expf(z * P.sm_scale + bg.bias - lse);
      const float dpw = bg.w * dp;
      const float ds = p * (dpw - delta);
      dsum += P.outer ? p * dpw : ds;
      if (bg.att) {
#pragma unroll
        for (int j = 0; j < DH; ++j) dq[j] = fmaf(ds * P.sm_scale, k[j], dq[j]);
      }
    }
    if (bg.grad && m < beta) {
      if (P.full) P.dlg_head_full[hrow * NB + m] = dsum;
      else if (dlg && bg.slot >= 0) dlg[bg.slot] = dsum;
    }
  }
  float* dqp = (float*)P.dQ + (((size_t)bi * n + t) * P.H + h) * DH;
#pragma unroll
  for (int j = 0; j < DH; ++j) dqp[j] = dq[j];
}

// pass 2: one thread per (batch, group, key)
template <int DH>
__global__ void __launch_bounds__(64) bwd_dkv_f32_kernel(BwdArgs P) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int n = P.n;
  if (idx >= (size_t)P.b * P.Hkv * n) return;
  const int i = (int)(idx % n), g = (int)((idx / n) % P.Hkv), bi = (int)(idx / ((size_t)n * P.Hkv));
  const int G = P.H / P.Hkv, B = P.B, m = i / B;
  const float* k = (const float*)P.Kt + (((size_t)bi * n + i) * P.Hkv + g) * DH;
  const float* v = (const float*)P.V + (((size_t)bi * n + i) * P.Hkv + g) * DH;
  float kv[DH], vv[DH], dk[DH], dv[DH];
#pragma unroll
  for (int j = 0; j < DH; ++j) {
    kv[j] = k[j];
    vv[j] = v[j];
    dk[j] = 0.f;
    dv[j] = 0.f;
  }
  for (int t = i; t < n; ++t) {
    const BlockGate bg = block_gate(P, bi, g, t, m);
    if (!bg.att) continue;
    for (int h = g * G; h < (g + 1) * G; ++h) {
      const float* q = (const float*)P.Q + (((size_t)bi * n + t) * P.H + h) * DH;
      const float* dO = (const float*)P.dO + (((size_t)bi * n + t) * P.H + h) * DH;
      float z = 0.f, dp = 0.f;
#pragma unroll
      for (int j = 0; j < DH; ++j) {
        z = fmaf(q[j], kv[j], z);
        dp = fmaf(dO[j], vv[j], dp);
      }
      const size_t hr = ((size_t)bi * P.H + h) * n + t;
      const float p = expf(z * P.sm_scale + bg.bias - P.lse[hr]);
      const float ds = p * (bg.w * dp - P.delta[hr]);
      const float pw = p * bg.w;
#pragma unroll
      for (int j = 0; j < DH; ++j) {
        dk[j] = fmaf(ds * P.sm_scale, q[j], dk[j]);
        dv[j] = fmaf(pw, dO[j], dv[j]);
      }
    }
  }
  float* dkp = (float*)P.dK + (((size_t)bi * n + i) * P.Hkv + g) * DH;
  float* dvp = (float*)P.dV + (((size_t)bi * n + i) * P.Hkv + g) * DH;
#pragma unroll
  for (int j = 0; j < DH; ++j) {
    dkp[j] = dk[j];
    dvp[j] = dv[j];
  }
}

// dLogG[b, g, t, slot] = sum over the group's heads of the per-head block sums
// (times the block's gate for the straight-through gate: the gradient of log g)
__global__ void bwd_dlog_gate_sum_kernel(const float* __restrict__ dlg_head, const float* __restrict__ sel_bias,
                                         int ste, int b, int n, int H, int Hkv, int K,
                                         float* __restrict__ dlog_gate) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)b * Hkv * n * K) return;
  const int k = (int)(idx % K), t = (int)((idx / K) % n), g = (int)((idx / ((size_t)K * n)) % Hkv);
  const int bi = (int)(idx / ((size_t)K * n * Hkv));
  const int G = H / Hkv;
  float s = 0.f;
  for (int h = g * G; h < (g + 1) * G; ++h) s += dlg_head[(((size_t)bi * H + h) * n + t) * K + k];
  dlog_gate[idx] = ste ? s * expf(sel_bias[idx]) : s;
}

// the same for every block (full scope): 0 for blocks that are not historical
__global__ void bwd_dlog_gate_full_sum_kernel(const float* __restrict__ dlg_head_full,
                                              const float* __restrict__ log_gate, int ste, int b, int n, int H,
                                              int Hkv, int B, int NB, float* __restrict__ out,
                                              const int32_t* __restrict__ doc) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)b * Hkv * n * NB) return;
  const int m = (int)(idx % NB), t = (int)((idx / NB) % n), g = (int)((idx / ((size_t)NB * n)) % Hkv);
  const int bi = (int)(idx / ((size_t)NB * n * Hkv));
  float s = 0.f;
  if (m < t / B && m >= doc_first(doc, bi, NB, t, B)) {
    const int G = H / Hkv;
    for (int h = g * G; h < (g + 1) * G; ++h) s += dlg_head_full[(((size_t)bi * H + h) * n + t) * NB + m];
    if (ste) s *= expf(log_gate[idx]);
  }
  out[idx] = s;
}

__global__ void bwd_scatter_slots_kernel(const int32_t* __restrict__ sel, const float* __restrict__ slots,
                                         size_t rows, int K, int NB, float* __restrict__ table) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= rows * NB) return;
  const size_t row = idx / NB;
  const int m = (int)(idx % NB);
  float v = 0.f;
  for (int k = 0; k < K; ++k)
    if (sel[row * K + k] == m) v += slots[row * K + k];
  table[idx] = v;
}

hipError_t launch_scatter_slots(const int32_t* sel, const float* slots, int b, int n, int Hkv, int K, int NB,
                                float* table, hipStream_t s) {
  const size_t rows = (size_t)b * Hkv * n;
  if (rows * NB == 0) return hipSuccess;
  bwd_scatter_slots_kernel<<<(unsigned)cdiv(rows * NB, 256), 256, 0, s>>>(sel, slots, rows, K, NB, table);
  return hipGetLastError();
}

// log gate of each selected slot: bias[b, g, t, k] = log_gate[b, g, t, sel[b, g, t, k]]
__global__ void bwd_gather_gate_kernel(const int32_t* __restrict__ sel, const float* __restrict__ log_gate, int b,
                                       int n, int Hkv, int K, int NB, float* __restrict__ bias) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)b * Hkv * n * K) return;
  const int m = sel[idx];
  bias[idx] = (m >= 0 && m < NB) ? log_gate[(idx / K) * NB + m] : 0.f;
}

__global__ void fill_f32_kernel(float* p, size_t n, float v) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// ---- bf16 path ------------------------------------------------------------------
constexpr float BLOG2E = 1.4426950408889634f;

// Pass 1 (dQ and the per-head block sums of ds): one workgroup = 4 waves =
// 128 query rows of one batch entry and KV group, 128 / G consecutive positions x
// the group's G heads as in the forward (the key tiles the rows attend are the
// union over the positions only); a wave none of whose rows attends a key of
// the tile or takes a gradient from it skips it (SKIP, grouped queries).  Each lane owns one query
// of S^T = K Q^T (v_mfma_f32_32x32x16_bf16), with dP^T = V dO^T computed the
// same way; dS^T = P^T (dP^T - Delta) is formed in registers and fed back as the
// B operand of dQ^T += K^T dS^T, whose A operand is read from the same K rows
// with the transposing LDS read, in the accumulator's key permutation.  The key
// tiles any query of the workgroup attends are flagged in LDS first; a tile's
// K and V are loaded into registers while the previous tile is multiplied and
// written to the other of two buffers after it: one barrier per tile.
// Sub-blocks of 2^LSB = min(B, 64) keys carry one bias per query; a sub-block of
// an accumulator element is known at compile time (the lane-dependent part of
// its key index is below 8).  Each lane walks its query's ascending selection
// row from global memory (the next slot read one slot ahead) and writes a
// slot's block sum once the slot's last sub-block is done; a tile is processed
// as two halves of 32 keys to keep the live registers low enough for two
// workgroups per compute unit.  28/4 heads, 16384 tokens, K = 32: 3.57 ms, 4.20 with
// one head per workgroup, a transposed K copy and two barriers; 4 x 4096, 32/32
// heads: 1.33 ms, 1.39 before.
// heads of a KV group that share a workgroup's rows (1 when a group has more heads than rows)
__host__ __device__ inline int bwd_dq_heads(int G) { return G <= 128 ? G : 1; }

template <int DH, int LSB, bool PLAIN, bool SKIP>
__device__ __forceinline__ void bwd_dq_bf16_job(const BwdArgs& P, const int qtile, const int unit, const int bi) {
  constexpr int C8 = DH / 8;
  constexpr int KPT = 64 * C8 / 256;  // keys per thread in the tile staging ...
  constexpr int KS = 256 / C8;        // ... this many apart
  constexpr int NSUB = 64 >> LSB;
  constexpr int TB = 64 * DH * 2;     // bytes of a tile
  __shared__ __align__(16) unsigned char tiles[2 * 2 * TB];  // two buffers of K and V
  __shared__ uint32_t need[BWD_MAX_SEQ / 64 / 32];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 31, lk = lane >> 5;
  const int G = P.H / P.Hkv, PG = bwd_dq_heads(G), QPT = 128 / PG;
  const int n = P.n, B = P.B;
  const int qrow = wave * 32 + lr;  // query row of this lane in the workgroup
  const int pl = qrow / PG, h = unit * PG + (qrow - pl * PG), g = unit * PG / G;
  const int t0 = qtile * QPT;       // first position of the workgroup
  const int t = t0 + pl;
  const bool qvalid = pl < QPT && t < n;
  const int beta = qvalid ? t / B : -1;
  const bool gated = P.mode == SAS_MODE_GATED;
  const bool dense = P.mode == SAS_MODE_DENSE;
  const bool full = gated && P.full;           // a gradient for every historical block
  const bool fullatt = full && !P.ste;         // ... which are all attended
  const bool ste = gated && P.ste, outer = gated && P.outer;
  const bool every = dense || full;            // every tile up to the query
  const int Kn = (dense || fullatt) ? 0 : P.K;
  const int ntiles = (n + 63) / 64;
  const int NB = (n + B - 1) / B;
  const size_t grow = ((size_t)bi * P.Hkv + g) * n;
  const int t_hi = min(n, t0 + QPT) - 1;
  const int last_tile = t_hi / 64;
  const int fb = qvalid ? doc_first(P.doc, bi, NB, t, B) : 0;  // first block of the query's document
  const int first_tile = doc_first(P.doc, bi, NB, t0, B) * B / 64;

  bf16x8_t qb[DH / 16], dob[DH / 16];
  {
    const size_t off = (((size_t)bi * n + (qvalid ? t : 0)) * P.H + h) * DH;
    const bf16_t* qp = (const bf16_t*)P.Q + off;
    const bf16_t* dp = (const bf16_t*)P.dO + off;
#pragma unroll
    for (int ks = 0; ks < DH / 16; ++ks) {
      uint4 u = qvalid ? *(const uint4*)(qp + ks * 16 + lk * 8) : make_uint4(0, 0, 0, 0);
      qb[ks] = *(bf16x8_t*)&u;
      uint4 w = qvalid ? *(const uint4*)(dp + ks * 16 + lk * 8) : make_uint4(0, 0, 0, 0);
      dob[ks] = *(bf16x8_t*)&w;
    }
  }
  const size_t hrow = ((size_t)bi * P.H + h) * n + (qvalid ? t : 0);
  const float lse2 = qvalid ? P.lse[hrow] * BLOG2E : 0.f;
  const float delta = qvalid ? P.delta[hrow] : 0.f;

  // key tiles of every earlier block (DENSE, full scope), from the workgroup's earliest document start
  for (int w = tid; w < (ntiles + 31) / 32; w += 256) {
    const int lo = w * 32;
    uint32_t bits = 0;
    if (every && lo <= last_tile) bits = last_tile - lo >= 31 ? 0xffffffffu : ((1u << (last_tile - lo + 1)) - 1u);
    if (every && lo + 31 >= first_tile && lo < first_tile) bits &= ~((1u << (first_tile - lo)) - 1u);
    if (lo + 31 < first_tile) bits = 0;
    need[w] = bits;
  }
  __syncthreads();
  // this query's selection row: slots are ascending historical blocks, -1 padded
  const size_t srow = (grow + (qvalid ? t : 0)) * (size_t)Kn;
  // key tiles this workgroup attends: every query's current block, its selected blocks
  if (!every && qvalid && lk == 0) {
    for (int tl = (beta * B) / 64; tl <= t / 64; ++tl) atomicOr(&need[tl >> 5], 1u << (tl & 31));
    for (int k = 0; k < Kn; ++k) {
      const int m = P.sel[srow + k];
      if (m < 0 || m >= beta) break;  // slots are ascending historical blocks, -1 padded
      for (int tl = (m * B) / 64; tl <= ((m + 1) * B - 1) / 64; ++tl) atomicOr(&need[tl >> 5], 1u << (tl & 31));
    }
  }
  __syncthreads();

  floatx16_t dq[DH / 32];
#pragma unroll
  for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) dq[dt][v] = 0.f;
  const float qk_scale = P.sm_scale * BLOG2E;
  const bf16_t* Kg = (const bf16_t*)P.Kt + (size_t)g * DH;
  const bf16_t* Vg = (const bf16_t*)P.V + (size_t)g * DH;
  const size_t kstride = (size_t)P.Hkv * DH;
  const size_t kbase = (size_t)bi * n;
  const int c8 = tid % C8, kg = tid / C8;  // staging role: keys kg + KS q, 16-byte piece c8
  uint4 rk[KPT], rv[KPT];
  float r_lg[NSUB];  // full scope: this query's log gates of the tile's blocks
  auto prefetch = [&](int kt) {
    // unconditional loads (a branch around a load waits for those in flight):
    // keys past the end repeat the last one and are zeroed on their way to LDS
#pragma unroll
    for (int q = 0; q < KPT; ++q) {
      const size_t go = (kbase + min(kt * 64 + kg + KS * q, n - 1)) * kstride + c8 * 8;
      rk[q] = *(const uint4*)(Kg + go);
      rv[q] = *(const uint4*)(Vg + go);
    }
    if (full) {
#pragma unroll
      for (int sb = 0; sb < NSUB; ++sb) {
        const int m = (kt * 64 + (sb << LSB)) / B;
        r_lg[sb] = (qvalid && m < beta && m >= fb) ? P.log_gate[(grow + t) * NB + m] : 0.f;
      }
    }
  };
  auto commit = [&](int kt, int buf) {
    bf16_t* kb = (bf16_t*)(tiles + buf * 2 * TB);
    if (kt * 64 + 64 > n) {
#pragma unroll
      for (int q = 0; q < KPT; ++q)
        if (kt * 64 + kg + KS * q >= n) rk[q] = rv[q] = make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < KPT; ++q) {
      *(uint4*)(kb + lds_chunk<DH>(kg + KS * q, c8)) = rk[q];
      *(uint4*)(kb + 64 * DH + lds_chunk<DH>(kg + KS * q, c8)) = rv[q];
    }
  };
  // byte offsets of this lane's operands in a tile (see the dK/dV pass): rows lr,
  // chunk 2 ks + lk; columns of row 4 lk + 8 half + (lane % 16) / 4
  uint32_t o_row = lr * DH * 2 + ((lk ^ lds_swz<DH>(lr)) << 4);
  uint32_t o_tr[2];
#pragma unroll
  for (int hf = 0; hf < 2; ++hf) {
    const int r = 4 * lk + 8 * hf + ((lane & 15) >> 2);
    o_tr[hf] = r * DH * 2 + (((2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ lds_swz<DH>(r)) << 4) + (lane & 1) * 8;
  }

  // the walk over this query's slots: slot `cur` (block next_sel, bias b_cur) and the
  // one after it (read one slot ahead, so the read is done by the time it is needed)
  auto sel_at = [&](int k) -> int { return qvalid && k < Kn ? P.sel[srow + k] : -1; };
  auto bias_at = [&](int k) -> float { return gated && qvalid && k < Kn ? P.sel_bias[srow + k] : 0.f; };
  int cur = 0;
  int next_sel = sel_at(0);
  float b_cur = bias_at(0);
  int s_nx = sel_at(1);
  float b_nx = bias_at(1);
  if (next_sel < 0) next_sel = 0x7fffffff;
  float blk_acc = 0.f;   // full scope: running sum of a block wider than a tile
  float slot_acc = 0.f;  // the current slot's running sum (a block may span two tiles)
  int kt = next_set(need, 0, ntiles), buf = 0;
  if (kt < ntiles) {
    prefetch(kt);
    commit(kt, 0);
  }
  while (kt < ntiles) {
    lds_barrier();  // the tile is staged; every wave is done with the other buffer
    const int k0 = kt * 64;
    const unsigned char* const tb = tiles + buf * 2 * TB;
    asm volatile("" : "+v"(o_row), "+v"(o_tr[0]), "+v"(o_tr[1]));  // (formed anew per tile: kept, they would spill)

    // per sub-block: offset (log2-domain bias - LSE; -inf: neither attended nor
    // receiving a gradient, or a zero gate), value weight, attended, selection slot
    float offs[NSUB], wts[NSUB];
    bool attb[NSUB], gradb[NSUB];
    int slot[NSUB];
#pragma unroll
    for (int sb = 0; sb < NSUB; ++sb) {
      offs[sb] = -INFINITY;
      wts[sb] = 1.f;
      attb[sb] = gradb[sb] = false;
      slot[sb] = -1;
      const int kstart = k0 + (sb << LSB);
      if (!qvalid || kstart > t) continue;
      const int m = kstart / B;
      float lg = 0.f;
      if (m == beta || (dense && m >= fb)) {
        attb[sb] = true;
      } else if (m < fb) {
        // outside the query's document
      } else if (fullatt) {
        attb[sb] = gradb[sb] = true;
        lg = r_lg[sb];
      } else {
        if (m == next_sel) {
          attb[sb] = true;
          gradb[sb] = gated;
          lg = b_cur;
          slot[sb] = cur;
          if (kstart + (1 << LSB) >= (m + 1) * B) {
            ++cur;
            next_sel = s_nx >= 0 ? s_nx : 0x7fffffff;
            b_cur = b_nx;
            s_nx = sel_at(cur + 1);
            b_nx = bias_at(cur + 1);
          }
        } else if (ste && full) {
          gradb[sb] = true;  // straight-through gradient of a dropped block
          lg = r_lg[sb];
        }
      }
      if (attb[sb] || gradb[sb]) {
        const bool biased = gated && !ste && !outer && m != beta;
        offs[sb] = (biased ? lg * BLOG2E : 0.f) - lse2;
        if (outer && m != beta) wts[sb] = __builtin_amdgcn_exp2f(lg * BLOG2E);
      }
    }
    const int nkt = next_set(need, kt + 1, ntiles);
    if (nkt < ntiles) prefetch(nkt);

    // a block with a zero gate (its offset is -inf) counts: its block sum, 0, is written below
    bool any = !SKIP;
    if constexpr (SKIP) {
#pragma unroll
      for (int sb = 0; sb < NSUB; ++sb) any = any || attb[sb] || gradb[sb];
    }
    if (!SKIP || __builtin_amdgcn_ballot_w64(any) != 0) {
    const bool diag = k0 + 63 > t0;  // keys past some query of the workgroup: mask key > t
    float dsum[NSUB];
#pragma unroll
    for (int sb = 0; sb < NSUB; ++sb) dsum[sb] = 0.f;
    // the tile's two halves of 32 keys one after the other (fewer live registers):
    // S^T, dP^T of the half, dS^T in registers, then its two 16-key steps of dQ^T += K^T dS^T
#pragma unroll
    for (int st = 0; st < 2; ++st) {
      floatx16_t sc, dp;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        sc[v] = 0.f;
        dp[v] = 0.f;
      }
#pragma unroll
      for (int ks = 0; ks < DH / 16; ++ks) {
        const unsigned char* row = tb + (o_row ^ (ks << 5)) + st * 32 * DH * 2;
        const bf16x8_t a = *(const bf16x8_t*)row;
        sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qb[ks], sc, 0, 0, 0);
        const bf16x8_t av = *(const bf16x8_t*)(row + TB);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, dob[ks], dp, 0, 0, 0);
      }
      // P, dS^T and the block sums.  PLAIN (no value weights, no straight-through gradient): a
      // sub-block that is not attended has an offset of -inf, so its dS is already zero
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int klc = st * 32 + 8 * (v >> 2);  // key offset without the lane part (4 lk + v % 4 < 8)
        const int sb = klc >> LSB;
        float p = __builtin_amdgcn_exp2f(fmaf(sc[v], qk_scale, offs[sb]));
        if (diag && k0 + klc + 4 * lk + (v & 3) > t) p = 0.f;
        if constexpr (PLAIN) {
          const float ds = p * (dp[v] - delta);
          sc[v] = ds;
          dsum[sb] += ds;
        } else {
          const float dpw = outer ? wts[sb] * dp[v] : dp[v];
          const float ds = p * (dpw - delta);
          sc[v] = attb[sb] ? ds : 0.f;
          dsum[sb] += outer ? p * dpw : ds;
        }
      }
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const int ks = 2 * st + kk, v0 = 8 * kk;
        uint4 su;
        su.x = pack_bf16x2(sc[v0 + 0], sc[v0 + 1]);
        su.y = pack_bf16x2(sc[v0 + 2], sc[v0 + 3]);
        su.z = pack_bf16x2(sc[v0 + 4], sc[v0 + 5]);
        su.w = pack_bf16x2(sc[v0 + 6], sc[v0 + 7]);
        const bf16x8_t pb = *(const bf16x8_t*)&su;
#pragma unroll
        for (int dt = 0; dt < DH / 32; ++dt) {
          const uint2 lo = lds_read_tr(tb + (o_tr[0] ^ (dt << 6)) + ks * 16 * DH * 2);
          const uint2 hi = lds_read_tr(tb + (o_tr[1] ^ (dt << 6)) + ks * 16 * DH * 2);
          uint4 u = make_uint4(lo.x, lo.y, hi.x, hi.y);
          dq[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(bf16x8_t*)&u, pb, dq[dt], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int sb = 0; sb < NSUB; ++sb) {
      const float tot = dsum[sb] + __shfl_xor(dsum[sb], 32, 64);
      const int kstart = k0 + (sb << LSB), m = kstart / B;
      const bool last = kstart + (1 << LSB) >= (m + 1) * B;  // the block's last sub-block
      if (lk == 0 && full && gradb[sb]) {
        blk_acc += tot;
        if (last) {
          P.dlg_head_full[hrow * NB + m] = blk_acc;
          blk_acc = 0.f;
        }
      } else if (lk == 0 && !full && slot[sb] >= 0) {
        if (gradb[sb]) slot_acc += tot;
        if (last) {  // the slot is complete
          if (P.dlg_head) P.dlg_head[hrow * P.K + slot[sb]] = slot_acc;
          slot_acc = 0.f;
        }
      }
    }
    }
    buf ^= 1;
    if (nkt < ntiles) commit(nkt, buf);
    kt = nkt;
  }

  if (!qvalid) return;
  if (P.dlg_head && !full && lk == 0) {  // slots never reached (padding) get zero
    float* dlg = P.dlg_head + hrow * P.K;
    for (int k = cur; k < Kn; ++k) dlg[k] = 0.f;
  }
  bf16_t* op = (bf16_t*)P.dQ + (((size_t)bi * n + t) * P.H + h) * DH;
  const float sm = P.sm_scale;
#pragma unroll
  for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
    for (int v4 = 0; v4 < 4; ++v4) {
      const int d0 = dt * 32 + 8 * v4 + 4 * lk;
      const uint32_t w0 = pack_bf16x2(dq[dt][4 * v4 + 0] * sm, dq[dt][4 * v4 + 1] * sm);
      const uint32_t w1 = pack_bf16x2(dq[dt][4 * v4 + 2] * sm, dq[dt][4 * v4 + 3] * sm);
      *(uint2*)(op + d0) = make_uint2(w0, w1);
    }
}

// One job per workgroup (grid = job count, no queue) or the work queue.
// two workgroups per compute unit where the registers allow it without spills
// (one sub-block per tile, or dh = 64)
template <int DH, int LSB, bool PLAIN, bool SKIP>
__global__ void __launch_bounds__(256, LSB == 6 || DH == 64 ? 2 : 1) bwd_dq_bf16_kernel(BwdArgs P) {
  const int PG = bwd_dq_heads(P.H / P.Hkv), qpt = 128 / PG;
  const int nqt = (P.n + qpt - 1) / qpt, units = P.H / PG, per = units * P.b;
  const int njobs = nqt * per;
  for (int it = 0;; ++it) {
    const int job = P.queue ? queue_next_job(P.queue) : (it == 0 ? (int)blockIdx.x : njobs);
    if (job >= njobs) break;
    const int r = job % per;  // the longest (last) query tiles first, groups and batch inside
    __syncthreads();          // the previous job is done with LDS
    bwd_dq_bf16_job<DH, LSB, PLAIN, SKIP>(P, nqt - 1 - job / per, r % units, r / units);
  }
}

// selection bitmask of each row: bit m of word m / 32 is set when block m is selected
__global__ void bwd_selmask_kernel(const int32_t* __restrict__ sel, size_t rows, int K, int NW,
                                   uint32_t* __restrict__ mask) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= rows * NW) return;
  const size_t row = idx / NW;
  const int w = (int)(idx % NW);
  uint32_t bits = 0;
  for (int k = 0; k < K; ++k) {
    const int m = sel[row * K + k];
    if (m >= 0 && (m >> 5) == w) bits |= 1u << (m & 31);
  }
  mask[idx] = bits;
}

// The rows of (b, g) that attend key tile j (keys 64 j .. 64 j + 63), in
// ascending order: the rows t >= 64 j whose own block lies in the tile (the
// causal part of the current block) and every later row that selected one of
// the tile's blocks (at most four; they share one mask word since a tile
// starts at a multiple of 64 / B blocks).  Without `rows` the kernel writes
// the count of tile j; with it, the rows at off[tile].  One workgroup of 256
// threads per (tile, group, batch entry); the ballot prefix sums keep the
// order, so the lists are an exact function of the selection.
__global__ void __launch_bounds__(256) bwd_tile_rows_kernel(const uint32_t* __restrict__ selmask, int n, int Hkv,
                                                            int B, int NW, int ntiles, int* __restrict__ cnt,
                                                            const int* __restrict__ off, int* __restrict__ rows) {
  __shared__ int wsum[4];
  const int j = blockIdx.x, g = blockIdx.y, bi = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const size_t tile = ((size_t)bi * Hkv + g) * ntiles + j;
  const int k0 = j * 64, m_lo = k0 / B, m_hi = min(n - 1, k0 + 63) / B;
  const int own_end = min(n, (m_hi + 1) * B);
  const uint32_t bits = ((2u << (m_hi - m_lo)) - 1u) << (m_lo & 31);
  const uint32_t* sm = selmask + ((size_t)bi * Hkv + g) * (size_t)n * NW + (m_lo >> 5);
  const int base = rows ? off[tile] : 0;
  int total = 0;
  for (int t0 = k0; t0 < n; t0 += 256) {
    const int t = t0 + tid;
    bool f = false;
    if (t < n) f = t < own_end || (sm[(size_t)t * NW] & bits) != 0;
    const uint64_t bal = __ballot(f);
    if (lane == 0) wsum[wave] = __popcll(bal);
    __syncthreads();
    int before = __popcll(bal & ((1ull << lane) - 1ull)), all = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      before += w < wave ? wsum[w] : 0;
      all += wsum[w];
    }
    if (rows && f) rows[base + total + before] = t;
    total += all;
    __syncthreads();  // wsum is rewritten by the next step
  }
  if (!rows && tid == 0) cnt[tile] = total;
}

// exclusive sum over the 1024 threads of a workgroup; the total in `all`
__device__ __forceinline__ int block_scan1024(int v, int* wsum, int& all) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  __syncthreads();  // wsum of an earlier call has been read
  if (lane == 63) wsum[wave] = x;
  __syncthreads();
  int before = 0;
  all = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    before += w < wave ? wsum[w] : 0;
    all += wsum[w];
  }
  return before + x - v;
}

// Offsets of the tiles' row lists and the dK/dV jobs, in the order of the
// passes: key tile by key tile (the longest lists first), (batch, group) pairs
// inside.  cnt, off and tile_part are indexed [pair, tile].  One workgroup of
// 1024 threads; each takes a contiguous range, then the ranges are offset.
// `slots`: parts that the scratch holds (see bwd_part_slots).
__global__ void __launch_bounds__(1024) bwd_jobs_kernel(const int* __restrict__ cnt, int Z, int ntiles, int slots,
                                                        int* __restrict__ off, int4* __restrict__ jobs,
                                                        int* __restrict__ job_count, int2* __restrict__ tile_part) {
  __shared__ int wsum[16];
  const int T = Z * ntiles, tid = threadIdx.x;
  const int per = (T + 1023) / 1024, lo = min(T, tid * per), hi = min(T, lo + per);
  int unit = slots > 0 ? BWD_PART_CHUNKS : 0x40000000;  // chunks (of the dK/dV pass) per part, at most
  auto parts_of = [&](int c) { return max(1, ((c + 63) / 64 + unit - 1) / unit); };
  int s_row = 0, s_job = 0, s_slot = 0, s_chunk = 0;
  for (int i = lo; i < hi; ++i) {
    const int c = cnt[(i % Z) * ntiles + i / Z], p = parts_of(c);
    s_row += c;
    s_job += p;
    s_slot += p > 1 ? p : 0;
    s_chunk += (c + 63) / 64;
  }
  int all, parts, jobs_all;
  int row = block_scan1024(s_row, wsum, all);
  int slot = block_scan1024(s_slot, wsum, parts);
  if (parts > slots) {
    int chunks;
    block_scan1024(s_chunk, wsum, chunks);
    const int last = (int)((2LL * chunks + slots - 1) / slots);  // fits: ceil(c / unit) < 2 c / unit where c > unit
    do {
      unit = (int)min((long long)last, max((long long)unit + 1, ((long long)unit * parts + slots - 1) / slots));
      s_job = s_slot = 0;
      for (int i = lo; i < hi; ++i) {
        const int p = parts_of(cnt[(i % Z) * ntiles + i / Z]);
        s_job += p;
        s_slot += p > 1 ? p : 0;
      }
      slot = block_scan1024(s_slot, wsum, parts);
    } while (parts > slots && unit < last);
  }
  int job = block_scan1024(s_job, wsum, jobs_all);
  if (tid == 0) *job_count = jobs_all;
  for (int i = lo; i < hi; ++i) {
    const int tile = (i % Z) * ntiles + i / Z;
    const int c = cnt[tile], p = parts_of(c);
    off[tile] = row;
    tile_part[tile] = make_int2(p, slot);
    for (int q = 0; q < p; ++q) jobs[job + q] = make_int4(tile, q, p, slot + q);
    row += c;
    job += p;
    slot += p > 1 ? p : 0;
  }
}

// dK and dV of the divided key tiles: their parts' sums added in order
template <int DH>
__global__ void __launch_bounds__(256) bwd_dkv_sum_kernel(const int2* __restrict__ tile_part,
                                                          const float* __restrict__ part, int n, int Hkv, int ntiles,
                                                          float sm, bf16_t* __restrict__ dK, bf16_t* __restrict__ dV) {
  const int2 tp = tile_part[blockIdx.x];
  if (tp.x <= 1) return;
  const int z = blockIdx.x / ntiles, k0 = (blockIdx.x % ntiles) * 64, g = z % Hkv, bi = z / Hkv;
  const float* src = part + (size_t)tp.y * (2 * 64 * DH);
  for (int i = threadIdx.x * 4; i < 2 * 64 * DH; i += 1024) {
    const int which = i / (64 * DH), key = k0 + i / DH % 64, d = i % DH;
    if (key >= n) continue;
    float4 s = *(const float4*)(src + i);
    for (int q = 1; q < tp.x; ++q) {
      const float4 p = *(const float4*)(src + (size_t)q * (2 * 64 * DH) + i);
      s.x += p.x;
      s.y += p.y;
      s.z += p.z;
      s.w += p.w;
    }
    const float f = which ? 1.f : sm;
    bf16_t* o = (which ? dV : dK) + (((size_t)bi * n + key) * Hkv + g) * DH + d;
    *(uint2*)o = make_uint2(pack_bf16x2(s.x * f, s.y * f), pack_bf16x2(s.z * f, s.w * f));
  }
}

// Pass 2 (dK, dV): one workgroup of 4 waves per 64 keys of one (batch, KV
// group).  The rows are those of the tile's list (selections), or, when every
// earlier block is attended (DENSE, full scope), the consecutive rows from the
// tile on, in chunks of 64 that reach the tile; work items are (chunk, head of
// the group).  Wave (kh, rh) multiplies 32 of the chunk's rows by 32 of the keys
// and accumulates dK and dV of its keys over its rows, all dimensions (128
// registers); the two row halves are added through LDS once per job.  Bound by
// LDS bandwidth and matrix cores: K and V stay in LDS for the job, the chunk's Q
// and dO rows are staged once, row-major, and read both as rows (A of S = Q K^T
// and dP = dO V^T) and, with the transposing read, as columns (A of dK^T += Q^T dS
// and dV^T += dO^T P, in the accumulator's row permutation): 48 KB of reads per
// wave and 32 x 32 block, 64 KB of LDS per workgroup, two workgroups per compute
// unit.  P and dS never leave registers.  4 x 4096 tokens, 32/32 heads, K = 16:
// 1.04 ms; waves that split the dimensions, exchanged partial S and dP
// through LDS and staged transposed copies took 1.64 ms.
// The next item's rows are loaded into registers while this one is multiplied;
// row indices are read one chunk ahead.
constexpr int DKV_ROWS = 64;
template <int DH, bool PLAIN>
__device__ __forceinline__ void bwd_dkv_bf16_job(const BwdArgs& P, const int ktile, const int g, const int bi,
                                                 const int part, const int parts, const int slot) {
  constexpr int KT = 64, RC = DKV_ROWS;
  constexpr int C8 = DH / 8;              // 16-byte pieces of a row
  constexpr int NR = RC * C8 / 256;       // chunk rows staged per thread
  constexpr int RS = 256 / C8;            // ... this many rows apart
  __shared__ __align__(16) bf16_t tiles[4 * 64 * DH];  // Q, dO, K, V; at the end the row halves' sums
  bf16_t* const Qs = tiles;
  bf16_t* const Ds = tiles + 64 * DH;
  bf16_t* const Ks = tiles + 2 * 64 * DH;
  bf16_t* const Vs = tiles + 3 * 64 * DH;
  __shared__ __align__(16) float delta_s[RC];
  __shared__ __align__(16) int rows_s[2][RC];   // row index of each staged row (n: none), by chunk parity
  __shared__ __align__(16) float off_s[4][RC];  // log2-domain bias - LSE per (sub-block, row); -inf: not attended
  __shared__ __align__(16) float wt_s[PLAIN ? 1 : 4][RC];  // value weight per (sub-block, row) (outer gate)
  __shared__ uint32_t flags[BWD_MAX_SEQ / RC / 32];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 31, lk = lane >> 5;
  const int kh = wave >> 1, rh = wave & 1;  // key half, row half
  const int k0 = ktile * KT;
  const int n = P.n, B = P.B, H = P.H, G = H / P.Hkv;
  const int key = k0 + kh * 32 + lr;
  const int bshift = 31 - __clz(B < 64 ? B : 64);
  const int nsb = KT >> bshift;  // sub-blocks of min(B, 64) keys in the tile: 1, 2 or 4
  const int m_hi = min(n - 1, k0 + KT - 1) / B;
  const int NB = (n + B - 1) / B;
  const int NW = (NB + 31) / 32;
  const int nqc = (n + RC - 1) / RC;
  const bool dense = P.mode == SAS_MODE_DENSE, gated = P.mode == SAS_MODE_GATED;
  const bool ste = gated && P.ste, outer = gated && P.outer;
  const bool fullatt = gated && P.full && !P.ste;  // every historical block attended, gates from the table
  const bool use_list = P.tile_rows != nullptr;    // selections: the tile's row list
  const size_t grow = ((size_t)bi * P.Hkv + g) * n;  // first row of (b, g) in [b, Hkv, n, ...]
  const int ntk = (n + KT - 1) / KT;
  int lbase = 0, lcnt = 0;
  if (use_list) {  // this part of the tile's list: whole chunks
    const size_t tile = ((size_t)bi * P.Hkv + g) * ntk + ktile;
    const int cnt = P.tile_cnt[tile], ch = (cnt + RC - 1) / RC, cp = (ch + parts - 1) / parts;
    const int lo = min(cnt, part * cp * RC);
    lbase = P.tile_off[tile] + lo;
    lcnt = min(cnt - lo, cp * RC);
  }
  const int nchunk = use_list ? (lcnt + RC - 1) / RC : nqc;

  // the previous job of this workgroup is done with LDS
  __syncthreads();
  const int c8 = tid % C8, sr = tid / C8;  // staging role: rows sr + RS i, 16-byte piece c8
  {
    uint4 kv[NR], vv[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const size_t off = (((size_t)bi * n + min(k0 + sr + RS * i, n - 1)) * P.Hkv + g) * DH + c8 * 8;
      kv[i] = *(const uint4*)((const bf16_t*)P.Kt + off);
      vv[i] = *(const uint4*)((const bf16_t*)P.V + off);
    }
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const uint32_t keep = k0 + sr + RS * i < n ? 0xffffffffu : 0u;  // keys past the end: zero
      kv[i] = make_uint4(kv[i].x & keep, kv[i].y & keep, kv[i].z & keep, kv[i].w & keep);
      vv[i] = make_uint4(vv[i].x & keep, vv[i].y & keep, vv[i].z & keep, vv[i].w & keep);
      *(uint4*)(Ks + lds_chunk<DH>(sr + RS * i, c8)) = kv[i];
      *(uint4*)(Vs + lds_chunk<DH>(sr + RS * i, c8)) = vv[i];
    }
  }
  // without a list: the chunks that reach the tile (their rows lie in its blocks, or,
  // every earlier block being attended, their earliest row's document starts in time)
  const int qc0 = use_list ? 0 : k0 / RC;
  if (!use_list) {
    for (int w = tid; w < (nqc + 31) / 32; w += 256) flags[w] = 0;
    __syncthreads();
    for (int qc = qc0 + tid; qc < nqc; qc += 256) {
      const bool any = ((dense || fullatt) && doc_first(P.doc, bi, NB, qc * RC, B) <= m_hi) || (qc * RC) / B <= m_hi;
      if (any) atomicOr(&flags[qc >> 5], 1u << (qc & 31));
    }
    __syncthreads();
  }
  auto next_chunk = [&](int c) { return use_list ? c : next_set(flags, c, nqc); };
  // row index of staged row r of chunk c (n: none)
  auto row_of = [&](int c, int r) -> int {
    if (c >= nchunk) return n;
    const int i = c * RC + r;
    if (use_list) return i < lcnt ? P.tile_rows[lbase + i] : n;
    return min(i, n);
  };

  floatx16_t dk[DH / 32], dv[DH / 32];
#pragma unroll
  for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      dk[dt][v] = 0.f;
      dv[dt][v] = 0.f;
    }
  const float qk_scale = P.sm_scale * BLOG2E;
  const int bq = tid & 63, bsb = wave;  // row scalars: row bq; its bias in sub-block bsb
  uint4 rq[NR], rd[NR];
  float r_lse = 0.f, r_delta = 0.f, r_lg = 0.f;
  uint32_t r_mw = 0;
  int r_doc = 0;  // the row's entry of the packing table
  // the next item's values: unconditional loads from clamped addresses, left as
  // they arrive until commit (a branch or an operation on one waits for all in flight)
  auto prefetch = [&](int par, int hg) {
    const int h = g * G + hg;
    int t[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) t[i] = min(rows_s[par][sr + RS * i], n - 1);
    const int tb = min(rows_s[par][bq], n - 1);
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const size_t off = (((size_t)bi * n + t[i]) * H + h) * DH + c8 * 8;
      rq[i] = *(const uint4*)((const bf16_t*)P.Q + off);
      rd[i] = *(const uint4*)((const bf16_t*)P.dO + off);
    }
    const size_t hr = ((size_t)bi * H + h) * n + tb;
    if (wave == 0) r_delta = P.delta[hr];
    if (bsb < nsb) {
      const int m = min((k0 + (bsb << bshift)) / B, NB - 1);
      r_lse = P.lse[hr];
      if (P.doc) r_doc = P.doc[(size_t)bi * NB + tb / B];
      if (use_list) r_mw = P.selmask[(grow + tb) * NW + (m >> 5)];
      if (gated && (use_list || fullatt)) r_lg = P.log_gate[(grow + tb) * NB + m];
    }
  };
  auto commit = [&](int par) {
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const uint32_t keep = rows_s[par][sr + RS * i] < n ? 0xffffffffu : 0u;  // no row: zero
      const int o = lds_chunk<DH>(sr + RS * i, c8);
      *(uint4*)(Qs + o) = make_uint4(rq[i].x & keep, rq[i].y & keep, rq[i].z & keep, rq[i].w & keep);
      *(uint4*)(Ds + o) = make_uint4(rd[i].x & keep, rd[i].y & keep, rd[i].z & keep, rd[i].w & keep);
    }
    const int t = rows_s[par][bq];
    if (wave == 0) delta_s[bq] = t < n ? r_delta : 0.f;
    if (bsb < nsb) {
      const int kstart = k0 + (bsb << bshift), m = kstart / B;
      const int fb = min(max(r_doc, 0), t / B);  // first block of the row's document (doc_first)
      float bb = -INFINITY, w = 1.f;
      if (t < n && kstart <= t) {
        if (m == t / B || (dense && m >= fb)) {
          bb = 0.f;
        } else if ((fullatt && m >= fb) || (use_list && ((r_mw >> (m & 31)) & 1u))) {
          const bool gate = gated && !ste;
          bb = gate && !outer ? r_lg * BLOG2E : 0.f;
          if (gate && outer) w = __builtin_amdgcn_exp2f(r_lg * BLOG2E);
        }
      }
      off_s[bsb][bq] = bb - (t < n ? r_lse : 0.f) * BLOG2E;
      if constexpr (!PLAIN) wt_s[bsb][bq] = w;
    }
  };
  // byte offsets of this lane's operands in a tile; a step or dimension block is an
  // exclusive-or of the chunk bits.  Rows: row rh 32 + lr of Q / dO and kh 32 + lr of
  // K / V, chunk 2 ks + lk.  Columns (transposing read): dimensions 32 dt + 16 (lane
  // / 16 % 2) + 4 (lane % 4) .. of row 4 lk + 8 half + (lane % 16) / 4 of the wave's rows.
  uint32_t o_row = (rh * 32 + lr) * DH * 2 + ((lk ^ lds_swz<DH>(lr)) << 4);
  uint32_t o_key = (kh * 32 + lr) * DH * 2 + ((lk ^ lds_swz<DH>(lr)) << 4);
  uint32_t o_tr[2];
#pragma unroll
  for (int hf = 0; hf < 2; ++hf) {
    const int r = 4 * lk + 8 * hf + ((lane & 15) >> 2);
    o_tr[hf] = (rh * 32 + r) * DH * 2 + (((2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ lds_swz<DH>(r)) << 4) +
               (lane & 1) * 8;
  }
  const unsigned char* const tb = (const unsigned char*)tiles;
  constexpr int TB = 64 * DH * 2;  // bytes of a tile

  int qc = next_chunk(qc0), hg = 0, par = 0;
  int nqcx = qc < nchunk ? next_chunk(qc + 1) : nchunk;  // the chunk after qc
  int r_next = n;                                        // its row of this thread (wave 0)
  if (wave == 0) {
    rows_s[0][bq] = row_of(qc, bq);
    r_next = row_of(nqcx, bq);
  }
  __syncthreads();
  if (qc < nchunk) prefetch(0, 0);
  while (qc < nchunk) {
    commit(par);
    if (hg == 0 && wave == 0) rows_s[par ^ 1][bq] = r_next;
    lds_barrier();
    const bool last_head = hg + 1 == G;
    int after = nchunk;
    if (last_head) {
      after = nqcx < nchunk ? next_chunk(nqcx + 1) : nchunk;
      if (nqcx < nchunk) prefetch(par ^ 1, 0);
      if (wave == 0) r_next = row_of(after, bq);
    } else {
      prefetch(par, hg + 1);
    }

    // (the operand addresses are formed anew for each item: kept, they would spill)
    asm volatile("" : "+v"(o_row), "+v"(o_key), "+v"(o_tr[0]), "+v"(o_tr[1]));
    const int* trow = rows_s[par] + rh * 32;
    if (trow[0] < n) {  // rows ascend: else this wave's half holds none
      floatx16_t sc, dp;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        sc[v] = 0.f;
        dp[v] = 0.f;
      }
#pragma unroll
      for (int ks = 0; ks < DH / 16; ++ks) {
        const unsigned char *row = tb + (o_row ^ (ks << 5)), *col = tb + (o_key ^ (ks << 5));
        const bf16x8_t aq = *(const bf16x8_t*)row, bk = *(const bf16x8_t*)(col + 2 * TB);
        sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aq, bk, sc, 0, 0, 0);
        const bf16x8_t ad = *(const bf16x8_t*)(row + TB), bv = *(const bf16x8_t*)(col + 3 * TB);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ad, bv, dp, 0, 0, 0);
      }
      // lane: key column `key`; rows 8 j + 4 lk + i of this half (v = 4 j + i)
      const int sbk = (kh * 32 + lr) >> bshift;
      const bool diag = trow[0] < k0 + KT - 1;  // some row precedes a key of the tile: mask key > row
      // dV^T += dO^T P and dK^T += Q^T dS, 16 rows per step in the accumulator's row permutation;
      // each step's P and dS are formed and packed just before its MFMAs
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        float pv[8], sv[8];
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
          const int j = 2 * ks + jj, r = rh * 32 + 8 * j + 4 * lk;
          const float4 of = *(const float4*)&off_s[sbk][r];
          const float4 de = *(const float4*)&delta_s[r];
          const int4 tr = *(const int4*)&rows_s[par][r];
          float4 wt = make_float4(1.f, 1.f, 1.f, 1.f);
          if constexpr (!PLAIN)
            if (outer) wt = *(const float4*)&wt_s[sbk][r];
          const float ofv[4] = {of.x, of.y, of.z, of.w}, dev[4] = {de.x, de.y, de.z, de.w};
          const float wv[4] = {wt.x, wt.y, wt.z, wt.w};
          const int trv[4] = {tr.x, tr.y, tr.z, tr.w};
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int v = 4 * j + i;
            float p = __builtin_amdgcn_exp2f(fmaf(sc[v], qk_scale, ofv[i]));
            if (diag && key > trv[i]) p = 0.f;
            if constexpr (PLAIN) {  // unit value weights
              pv[4 * jj + i] = p;
              sv[4 * jj + i] = p * (dp[v] - dev[i]);
            } else {
              pv[4 * jj + i] = p * wv[i];
              sv[4 * jj + i] = p * (wv[i] * dp[v] - dev[i]);
            }
          }
        }
        uint4 pu, su;
        pu.x = pack_bf16x2(pv[0], pv[1]);
        pu.y = pack_bf16x2(pv[2], pv[3]);
        pu.z = pack_bf16x2(pv[4], pv[5]);
        pu.w = pack_bf16x2(pv[6], pv[7]);
        su.x = pack_bf16x2(sv[0], sv[1]);
        su.y = pack_bf16x2(sv[2], sv[3]);
        su.z = pack_bf16x2(sv[4], sv[5]);
        su.w = pack_bf16x2(sv[6], sv[7]);
        const bf16x8_t pb = *(const bf16x8_t*)&pu, sb8 = *(const bf16x8_t*)&su;
#pragma unroll
        for (int dt = 0; dt < DH / 32; ++dt) {
          const unsigned char* lo = tb + (o_tr[0] ^ (dt << 6)) + ks * 16 * DH * 2;
          const unsigned char* hi = tb + (o_tr[1] ^ (dt << 6)) + ks * 16 * DH * 2;
          const uint2 dlo = lds_read_tr(lo + TB), dhi = lds_read_tr(hi + TB);
          const uint4 du = make_uint4(dlo.x, dlo.y, dhi.x, dhi.y);
          dv[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8_t*)&du, pb, dv[dt], 0, 0, 0);
          const uint2 qlo = lds_read_tr(lo), qhi = lds_read_tr(hi);
          const uint4 qu = make_uint4(qlo.x, qlo.y, qhi.x, qhi.y);
          dk[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8_t*)&qu, sb8, dk[dt], 0, 0, 0);
        }
      }
    }
    lds_barrier();
    if (last_head) {
      qc = nqcx;
      nqcx = after;
      par ^= 1;
      hg = 0;
    } else {
      ++hg;
    }
  }

  // add the row halves: wave (kh, 0) takes dK, wave (kh, 1) takes dV
  {
    float* x = (float*)tiles + (size_t)wave * (32 * DH / 2) * 2;  // 32 keys x DH sums of this wave's other matrix
#pragma unroll
    for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4) {
        const floatx16_t& o = rh ? dk[dt] : dv[dt];
        *(float4*)(x + ((dt * 4 + v4) * 64 + lane) * 4) = make_float4(o[4 * v4], o[4 * v4 + 1], o[4 * v4 + 2], o[4 * v4 + 3]);
      }
    lds_barrier();
    x = (float*)tiles + (size_t)(wave ^ 1) * (32 * DH / 2) * 2;
    const float sm = rh ? 1.f : P.sm_scale;
    float* fp = P.part + (size_t)slot * (2 * 64 * DH) + (size_t)(rh * 64 + kh * 32 + lr) * DH;
    bf16_t* op = (bf16_t*)(rh ? P.dV : P.dK) + (((size_t)bi * n + min(key, n - 1)) * P.Hkv + g) * DH;
#pragma unroll
    for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4) {
        const floatx16_t& o = rh ? dv[dt] : dk[dt];
        const float4 y = *(const float4*)(x + ((dt * 4 + v4) * 64 + lane) * 4);
        // rows ascend from half 0 to half 1 in both waves' sums
        const float4 r = rh ? make_float4(y.x + o[4 * v4], y.y + o[4 * v4 + 1], y.z + o[4 * v4 + 2], y.w + o[4 * v4 + 3])
                            : make_float4(o[4 * v4] + y.x, o[4 * v4 + 1] + y.y, o[4 * v4 + 2] + y.z, o[4 * v4 + 3] + y.w);
        const int d0 = dt * 32 + 8 * v4 + 4 * lk;
        if (parts > 1) *(float4*)(fp + d0) = r;  // bwd_dkv_sum_kernel adds the parts
        else if (key < n)
          *(uint2*)(op + d0) = make_uint2(pack_bf16x2(r.x * sm, r.y * sm), pack_bf16x2(r.z * sm, r.w * sm));
      }
  }
}

template <int DH, bool PLAIN>
__global__ void __launch_bounds__(256, 2) bwd_dkv_bf16_kernel(BwdArgs P) {
  const int nkt = (P.n + 63) / 64, per = P.Hkv * P.b;
  const int njobs = P.tile_rows ? *P.job_count : nkt * per;
  for (int it = 0;; ++it) {
    const int job = P.queue ? queue_next_job(P.queue) : (it == 0 ? (int)blockIdx.x : njobs);
    if (job >= njobs) break;
    // the first (longest) key tiles first
    if (P.tile_rows) {
      const int4 j = P.jobs[job];
      const int z = j.x / nkt;
      bwd_dkv_bf16_job<DH, PLAIN>(P, j.x % nkt, z % P.Hkv, z / P.Hkv, j.y, j.z, j.w);
    } else {
      const int r = job % per;
      bwd_dkv_bf16_job<DH, PLAIN>(P, job / per, r % P.Hkv, r / P.Hkv, 0, 1, 0);
    }
  }
}

static hipError_t launch_attention_backward_bf16(const BwdArgs& P, hipStream_t s) {
  if (P.n > BWD_MAX_SEQ) return hipErrorInvalidValue;
  if (P.K > 32) return hipErrorInvalidValue;
  if (!P.queue) return hipErrorInvalidValue;
  const int NB = cdiv(P.n, P.B), NW = cdiv(NB, 32), ntk = cdiv(P.n, 64);
  BwdArgs Q = P;
  const bool marks = P.mode != SAS_MODE_DENSE && P.K > 0;  // selected blocks to mark
  const bool fullatt = P.mode == SAS_MODE_GATED && P.full && !P.ste;
  Q.tile_rows = nullptr;
  Q.tile_cnt = nullptr;
  Q.tile_off = nullptr;
  if (!marks) {
    Q.selmask = nullptr;
  } else {
    const size_t rows = (size_t)P.b * P.Hkv * P.n;
    bwd_selmask_kernel<<<(unsigned)cdiv(rows * NW, 256), 256, 0, s>>>(P.sel, rows, P.K, NW, P.selmask);
    if (!fullatt) {
      // each tile's list of attending rows: counts, offsets, rows
      if (!P.tile_rows || !P.tile_cnt || !P.tile_off || !P.jobs || !P.job_count || !P.tile_part ||
          (P.part_slots > 0 && !P.part))
        return hipErrorInvalidValue;
      const long long T = (long long)P.b * P.Hkv * ntk;
      if (T > INT32_MAX || rows * 2 * (P.K + 1) > (size_t)INT32_MAX) return hipErrorInvalidValue;
      const dim3 grid(ntk, P.Hkv, P.b);
      bwd_tile_rows_kernel<<<grid, 256, 0, s>>>(P.selmask, P.n, P.Hkv, P.B, NW, ntk, P.tile_cnt, nullptr, nullptr);
      bwd_jobs_kernel<<<1, 1024, 0, s>>>(P.tile_cnt, P.b * P.Hkv, ntk, (int)P.part_slots, P.tile_off, P.jobs, P.job_count,
                                         P.tile_part);
      bwd_tile_rows_kernel<<<grid, 256, 0, s>>>(P.selmask, P.n, P.Hkv, P.B, NW, ntk, P.tile_cnt, P.tile_off,
                                                P.tile_rows);
      Q.tile_rows = P.tile_rows;
      Q.tile_cnt = P.tile_cnt;
      Q.tile_off = P.tile_off;
    }
  }
  const int lsb = P.B >= 64 ? 6 : (P.B == 32 ? 5 : 4);
  // no value weights and no straight-through gradient: the plain elementwise step
  const bool plain = !(P.mode == SAS_MODE_GATED && (P.outer || P.ste));
  const int pg = bwd_dq_heads(P.H / P.Hkv);
  void (*dq)(BwdArgs);
#define DQ_PICK2(DH, LSB, PLAIN) \
  (pg > 1 ? bwd_dq_bf16_kernel<DH, LSB, PLAIN, true> : bwd_dq_bf16_kernel<DH, LSB, PLAIN, false>)
#define DQ_PICK(DH, LSB) (plain ? DQ_PICK2(DH, LSB, true) : DQ_PICK2(DH, LSB, false))
  if (P.dh == 128) dq = lsb == 6 ? DQ_PICK(128, 6) : lsb == 5 ? DQ_PICK(128, 5) : DQ_PICK(128, 4);
  else dq = lsb == 6 ? DQ_PICK(64, 6) : lsb == 5 ? DQ_PICK(64, 5) : DQ_PICK(64, 4);
#undef DQ_PICK
#undef DQ_PICK2
  auto dkv = P.dh == 128 ? (plain ? bwd_dkv_bf16_kernel<128, true> : bwd_dkv_bf16_kernel<128, false>)
                         : (plain ? bwd_dkv_bf16_kernel<64, true> : bwd_dkv_bf16_kernel<64, false>);
  const bool lists = Q.tile_rows != nullptr;
  // list jobs are counted on the GPU: at most one per tile and one per slot
  const long long jq = (long long)cdiv(P.n, 128 / pg) * (P.H / pg) * P.b;
  const long long jk = (long long)ntk * P.Hkv * P.b + (lists ? P.part_slots : 0);
  const int rq = resident_workgroups(dq, 256), rk = resident_workgroups(dkv, 256);
  if (rq <= 0 || rk <= 0 || jq > INT32_MAX || jk > INT32_MAX) return hipErrorInvalidValue;
  if (jq > rq || jk > rk) fill_f32_kernel<<<1, 64, 0, s>>>((float*)P.queue, 2, 0.f);  // job counters to zero
  BwdArgs A = Q;
  A.queue = jq > rq ? P.queue : nullptr;
  if (jq > 0) dq<<<(unsigned)std::min<long long>(jq, rq), 256, 0, s>>>(A);
  A.queue = jk > rk ? P.queue + 1 : nullptr;
  if (jk > 0) dkv<<<(unsigned)std::min<long long>(jk, rk), 256, 0, s>>>(A);
  if (lists && P.part_slots > 0) {
    const unsigned tiles = (unsigned)ntk * P.Hkv * P.b;
    if (P.dh == 128)
      bwd_dkv_sum_kernel<128><<<tiles, 256, 0, s>>>(P.tile_part, P.part, P.n, P.Hkv, ntk, P.sm_scale, (bf16_t*)P.dK,
                                                    (bf16_t*)P.dV);
    else
      bwd_dkv_sum_kernel<64><<<tiles, 256, 0, s>>>(P.tile_part, P.part, P.n, P.Hkv, ntk, P.sm_scale, (bf16_t*)P.dK,
                                                   (bf16_t*)P.dV);
  }
  return hipGetLastError();
}

hipError_t launch_fill_f32(float* p, size_t n, float v, hipStream_t s) {
  if (n == 0) return hipSuccess;
  fill_f32_kernel<<<(unsigned)cdiv(n, 256), 256, 0, s>>>(p, n, v);
  return hipGetLastError();
}

hipError_t launch_gather_gate(const int32_t* sel, const float* log_gate, int b, int n, int Hkv, int K, int NB,
                              float* bias, hipStream_t s) {
  const size_t tot = (size_t)b * Hkv * n * K;
  if (tot == 0) return hipSuccess;
  bwd_gather_gate_kernel<<<(unsigned)cdiv(tot, 256), 256, 0, s>>>(sel, log_gate, b, n, Hkv, K, NB, bias);
  return hipGetLastError();
}

// ---- selector ------------------------------------------------------------------
// One wave per DS_ROWS consecutive rows (b, g, t), whose loads are issued
// together; lane k < K holds slot k (per-slot input).  Bound by memory: log
// gates and slots read, ds written.  A slot's gradient reaches its block's lane
// through LDS (added there, so a block that appears twice counts twice).
// 4 x 4096 rows, 32 groups, 64 blocks, K = 16: 119 us; exchanging the slots by
// 2 K wave shuffles per 64 blocks took 214.
constexpr int DS_ROWS = 4;
__global__ void __launch_bounds__(256) selector_ds_kernel(const int32_t* __restrict__ sel,
                                                          const float* __restrict__ log_gate,
                                                          const float* __restrict__ dlog_gate,
                                                          const float* __restrict__ dfull, int act, int rows,
                                                          int n, int Hkv, int K, int B, int NB,
                                                          float* __restrict__ ds, float* __restrict__ row_sum,
                                                          const int32_t* __restrict__ doc) {
  __shared__ float slot_s[4][DS_ROWS][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row0 = ((int)blockIdx.x * 4 + wave) * DS_ROWS;
  if (row0 >= rows) return;
  int sk[DS_ROWS], C[DS_ROWS], F[DS_ROWS];
  float dk[DS_ROWS], lg0[DS_ROWS], D[DS_ROWS];
  const bool has_slot = !dfull && K > 0 && lane < K;
#pragma unroll
  for (int r = 0; r < DS_ROWS; ++r) {
    const int row = min(row0 + r, rows - 1);
    sk[r] = -1;
    dk[r] = 0.f;
    if (has_slot) {
      sk[r] = sel[(size_t)row * K + lane];
      dk[r] = dlog_gate[(size_t)row * K + lane];
    }
    lg0[r] = log_gate[(size_t)row * NB + min(lane, NB - 1)];
  }
#pragma unroll
  for (int r = 0; r < DS_ROWS; ++r) {
    const int row = min(row0 + r, rows - 1);
    C[r] = (row % n) / B;
    F[r] = doc_first(doc, row / (n * Hkv), NB, row % n, B);  // historical blocks are [F, C)
    if (sk[r] < 0) dk[r] = 0.f;
    D[r] = 0.f;  // sum of the row's log-gate gradient (softmax)
    if (act == SAS_ACT_SOFTMAX) {
      float d = dk[r];
      if (dfull)
        for (int m = F[r] + lane; m < C[r]; m += 64) d += dfull[(size_t)row * NB + m];
      D[r] = wave_sum(d);
    }
  }
  float total[DS_ROWS];
#pragma unroll
  for (int r = 0; r < DS_ROWS; ++r) total[r] = 0.f;
  for (int m0 = 0; m0 < NB; m0 += 64) {
    const int m = m0 + lane;
    float dl[DS_ROWS], lg[DS_ROWS];
#pragma unroll
    for (int r = 0; r < DS_ROWS; ++r) {
      const size_t o = (size_t)min(row0 + r, rows - 1) * NB + min(m, NB - 1);
      lg[r] = m0 == 0 ? lg0[r] : log_gate[o];
      if (dfull) {
        const float d = dfull[o];
        dl[r] = m < C[r] && m >= F[r] ? d : 0.f;
      } else {
        slot_s[wave][r][lane] = 0.f;
      }
    }
    if (!dfull) {
      wave_lds_fence();
#pragma unroll
      for (int r = 0; r < DS_ROWS; ++r)
        if (sk[r] >= m0 && sk[r] < m0 + 64) atomicAdd(&slot_s[wave][r][sk[r] - m0], dk[r]);
      wave_lds_fence();
#pragma unroll
      for (int r = 0; r < DS_ROWS; ++r) dl[r] = slot_s[wave][r][lane];
      wave_lds_fence();  // before the next blocks' zeros
    }
#pragma unroll
    for (int r = 0; r < DS_ROWS; ++r) {
      float v = 0.f;
      if (m < C[r] && m >= F[r]) {
        if (act == SAS_ACT_SOFTMAX) v = dl[r] - expf(lg[r]) * D[r];
        else if (act == SAS_ACT_SIGMOID) v = dl[r] * (1.f - expf(lg[r]));
        else v = dl[r];
      }
      if (m < NB && row0 + r < rows) ds[(size_t)(row0 + r) * NB + m] = v;
      total[r] += v;
    }
  }
  if (!row_sum) return;
#pragma unroll
  for (int r = 0; r < DS_ROWS; ++r) {
    const float sum = wave_sum(total[r]);
    if (lane == 0 && row0 + r < rows) row_sum[row0 + r] = sum;
  }
}

hipError_t launch_selector_ds(const int32_t* sel, const float* log_gate, const float* dlog_gate,
                              const float* dlog_gate_full, int act, int b, int n, int Hkv, int K, int B, float* ds,
                              float* row_sum, const int32_t* doc, hipStream_t s) {
  const int rows = b * Hkv * n;
  if (rows <= 0) return hipSuccess;
  if (K > 64) return hipErrorInvalidValue;
  if (K > 0 && !dlog_gate_full && (!sel || !dlog_gate)) return hipErrorInvalidValue;
  selector_ds_kernel<<<cdiv(rows, 4 * DS_ROWS), 256, 0, s>>>(sel, log_gate, dlog_gate, dlog_gate_full, act, rows, n,
                                                             Hkv, K, B, cdiv(n, B), ds, row_sum, doc);
  return hipGetLastError();
}

// 64 x N output tile per workgroup (N = dh) on v_mfma_f32_32x32x2_f32 (fp32
// products, one rounding per addition), wave (wi, wj) 32 rows x N/2 columns;
// 32-deep k stages in LDS as fp32 ([k][i] and [k][j]; pitches that put rows k
// and k + 1, the two halves of an operand, in different banks, and 97 also the
// transposed staging of a k-contiguous A), the next stage's values loaded into
// registers during this one.  Loads of A run along its contiguous index.
// ds^T [qhat0 | qhat], 4 x 4096 rows, 32 groups, 64 blocks, dh = 128: 179 us
// for both (17 GFLOP); the VALU tile it replaces took 211 us for one.
template <typename T, int DH, bool SHIFT>
__global__ void __launch_bounds__(256) small_gemm_kernel(SmallGemm P) {
  constexpr int AP = 97, BP = DH + 32, TN = DH / 2, FN = TN / 32, NB8 = 32 * (DH / 8) / 256;
  __shared__ float As[32 * AP];
  __shared__ __align__(16) float Bs[32 * BP];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 31, lk = lane >> 5, wi = wave >> 1, wj = wave & 1;
  const int i0 = blockIdx.x * 64, mat = blockIdx.y;
  const int z = blockIdx.z / P.splits, sp = blockIdx.z % P.splits;
  // the k range that this tile's rows reach, then this split's share (whole stages)
  const long long klo = P.kmin_b > 0 ? min((long long)P.K, (long long)(i0 + 1) * P.kmin_b) : 0;
  const int khi = P.kmax_b > 0 ? min(P.K, min(P.M - 1, i0 + 63) / P.kmax_b) : P.K;
  const int len = max(0, khi - (int)klo), kc = ((len + P.splits - 1) / P.splits + 31) / 32 * 32;
  const int kb = (int)klo + sp * kc, ke = min(khi, kb + kc);
  const float* A = P.A + z * P.sAz;
  const T* Bm = (const T*)P.Bm[mat] + z * P.sBz;
  const bool icont = P.sAi == 1;
  floatx16_t acc[FN];
#pragma unroll
  for (int f = 0; f < FN; ++f)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[f][v] = 0.f;
  float sh[8];  // this thread's columns of the shift (256 is a multiple of DH / 8)
  if constexpr (SHIFT) {
    const float* sp8 = P.shift + (size_t)z * DH + (tid % (DH / 8)) * 8;
#pragma unroll
    for (int j = 0; j < 8; ++j) sh[j] = sp8[j];
  }
  float ra[8];
  Vec8<T> rb[NB8];
  auto load = [&](int k0) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int idx = tid + e * 256;
      const int i = i0 + (icont ? idx & 63 : idx >> 5), k = k0 + (icont ? idx >> 6 : idx & 31);
      ra[e] = (i < P.M && k < ke) ? A[i * P.sAi + k * P.sAk] : 0.f;
    }
#pragma unroll
    for (int e = 0; e < NB8; ++e) {  // rows past the range repeat its last one (A is zero there)
      const int idx = tid + e * 256;
      rb[e].load(Bm + (long long)min(k0 + idx / (DH / 8), ke - 1) * P.sBk + (idx % (DH / 8)) * 8);
    }
  };
  if (kb < ke) load(kb);
  for (int k0 = kb; k0 < ke; k0 += 32) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int idx = tid + e * 256;
      As[icont ? (idx >> 6) * AP + (idx & 63) : (idx & 31) * AP + (idx >> 5)] = ra[e];
    }
#pragma unroll
    for (int e = 0; e < NB8; ++e) {
      const int idx = tid + e * 256;
      float* d = Bs + (idx / (DH / 8)) * BP + (idx % (DH / 8)) * 8;
      const bool in = k0 + idx / (DH / 8) < ke;  // (a repeated row may hold an infinity)
      float x[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] = in ? (SHIFT ? rb[e].get(j) - sh[j] : rb[e].get(j)) : 0.f;
      *(float4*)d = make_float4(x[0], x[1], x[2], x[3]);
      *(float4*)(d + 4) = make_float4(x[4], x[5], x[6], x[7]);
    }
    __syncthreads();
    if (k0 + 32 < ke) load(k0 + 32);
    // a wave whose rows are zero over the whole stage skips it
    if (!(P.kmin_b > 0 && k0 + 31 < (long long)(i0 + wi * 32 + 1) * P.kmin_b)) {
#pragma unroll
      for (int s = 0; s < 16; ++s) {
        const float a = As[(2 * s + lk) * AP + wi * 32 + lr];
#pragma unroll
        for (int f = 0; f < FN; ++f)
          acc[f] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, Bs[(2 * s + lk) * BP + wj * TN + f * 32 + lr], acc[f], 0, 0, 0);
      }
    }
    __syncthreads();
  }
  float* C = P.C[mat] + z * P.sCz + sp * P.sCs;
#pragma unroll
  for (int f = 0; f < FN; ++f)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int i = i0 + wi * 32 + 8 * (v >> 2) + 4 * lk + (v & 3), j = wj * TN + f * 32 + lr;
      if (i >= P.M) continue;
      float y = P.alpha * acc[f][v];
      if constexpr (SHIFT) y = fmaf(P.shift_w[(size_t)z * P.M + i], P.shift[(size_t)z * DH + j], y);
      C[i * P.sCi + j * P.sCj] = y;
    }
}

hipError_t launch_small_gemm(int dtype, const SmallGemm& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.Z <= 0) return hipSuccess;
  if (g.splits < 1 || (g.N != 64 && g.N != 128) || (g.sAi != 1 && g.sAk != 1) || g.nmat < 1 || g.nmat > 2)
    return hipErrorInvalidValue;
  if ((size_t)g.Z * g.splits > 65535) return hipErrorInvalidValue;
  if (g.shift && (!g.shift_w || g.splits != 1 || g.nmat != 1)) return hipErrorInvalidValue;
  dim3 grid(cdiv(g.M, 64), g.nmat, g.Z * g.splits);
  auto run = [&](auto kern) { kern<<<grid, 256, 0, s>>>(g); };
  if (dtype == SAS_BF16) {
    if (g.N == 128) run(g.shift ? small_gemm_kernel<bf16_t, 128, true> : small_gemm_kernel<bf16_t, 128, false>);
    else run(g.shift ? small_gemm_kernel<bf16_t, 64, true> : small_gemm_kernel<bf16_t, 64, false>);
  } else {
    if (g.N == 128) run(g.shift ? small_gemm_kernel<float, 128, true> : small_gemm_kernel<float, 128, false>);
    else run(g.shift ? small_gemm_kernel<float, 64, true> : small_gemm_kernel<float, 64, false>);
  }
  return hipGetLastError();
}

// part[z, split, j] = alpha sum_{t in split} w[z, t] x[z, t, j]; bound by reading x.
// 16 or 32 rows at a time, 8 columns per thread, the rows' sums added in LDS.
template <typename T, int DH>
__global__ void __launch_bounds__(256) weighted_rows_kernel(const T* __restrict__ x, const float* __restrict__ w, int n,
                                                            int splits, float alpha, float* __restrict__ part) {
  constexpr int C8 = DH / 8, R = 256 / C8;
  __shared__ float sum_s[R][DH + 4];
  const int tid = threadIdx.x, c8 = tid % C8, r = tid / C8;
  const int z = blockIdx.x / splits, sp = blockIdx.x % splits, per = (n + splits - 1) / splits;
  const int t1 = min(n, (sp + 1) * per);
  float acc[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) acc[j] = 0.f;
  for (int t = sp * per + r; t < t1; t += R) {
    const float wt = w[(size_t)z * n + t];
    Vec8<T> v;
    v.load(x + ((size_t)z * n + t) * DH + c8 * 8);
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = fmaf(wt, v.get(j), acc[j]);
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) sum_s[r][c8 * 8 + j] = acc[j];
  __syncthreads();
  if (tid >= DH) return;
  float s = 0.f;
  for (int q = 0; q < R; ++q) s += sum_s[q][tid];
  part[(size_t)blockIdx.x * DH + tid] = alpha * s;
}

// shift[z, j] = mean of the first nf rows of x[z, nb, DH] (fp64 sums), and
// shift_w[z, j] = sum over the splits of part[z, split, j]
template <typename T, int DH>
__global__ void __launch_bounds__(256) shift_kernel(const T* __restrict__ x, int nb, int nf, int splits,
                                                    const float* __restrict__ part, float* __restrict__ shift,
                                                    float* __restrict__ shift_w) {
  constexpr int R = 256 / DH;
  __shared__ double sum_s[R][DH];
  const int tid = threadIdx.x, j = tid % DH, r = tid / DH, z = blockIdx.x;
  double s = 0.0;
  for (int m = r; m < nf; m += R) s += (double)Act<T>::to_f32(x[((size_t)z * nb + m) * DH + j]);
  sum_s[r][j] = s;
  __syncthreads();
  if (r != 0) return;
  for (int q = 1; q < R; ++q) s += sum_s[q][j];
  shift[(size_t)z * DH + j] = nf > 0 ? (float)(s / (double)nf) : 0.f;
  float p = 0.f;
  for (int q = 0; q < splits; ++q) p += part[((size_t)z * splits + q) * DH + j];
  shift_w[(size_t)z * DH + j] = p;
}

template <typename T, int DH>
static void run_selector_shift(const SelShift& a, hipStream_t s) {
  weighted_rows_kernel<T, DH><<<(unsigned)a.Z * a.splits, 256, 0, s>>>((const T*)a.q, a.row_sum, a.n, a.splits, a.alpha,
                                                                      a.part);
  shift_kernel<T, DH><<<a.Z, 256, 0, s>>>((const T*)a.kbar, a.NB, a.nf, a.splits, a.part, a.shift, a.shift_w);
}

hipError_t launch_selector_shift(int dtype, const SelShift& a, hipStream_t s) {
  if (a.Z <= 0 || a.n <= 0 || a.splits < 1) return hipErrorInvalidValue;
  if (dtype == SAS_BF16) {
    if (a.dh == 128) run_selector_shift<bf16_t, 128>(a, s);
    else run_selector_shift<bf16_t, 64>(a, s);
  } else {
    if (a.dh == 128) run_selector_shift<float, 128>(a, s);
    else run_selector_shift<float, 64>(a, s);
  }
  return hipGetLastError();
}

__global__ void partial_sum_kernel(const float* __restrict__ part, int U, int ZO, int S, size_t E,
                                   float* __restrict__ out) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)ZO * E) return;
  const size_t zo = idx / E, e = idx % E;
  float acc = 0.f;
  for (int u = 0; u < U; ++u)
    for (int q = 0; q < S; ++q) acc += part[(((size_t)u * ZO + zo) * S + q) * E + e];
  out[idx] = acc;
}

hipError_t launch_partial_sum(const float* part, int U, int ZO, int S, size_t E, float* out, hipStream_t s) {
  const size_t tot = (size_t)ZO * E;
  if (tot == 0) return hipSuccess;
  partial_sum_kernel<<<(unsigned)cdiv(tot, 256), 256, 0, s>>>(part, U, ZO, S, E, out);
  return hipGetLastError();
}

hipError_t launch_attention_backward(int dtype, const BwdArgs& a, hipStream_t s) {
  if (a.n <= 0 || a.b <= 0) return hipSuccess;
  if (a.dh != 64 && a.dh != 128) return hipErrorInvalidValue;
  const size_t dthreads = (size_t)a.b * a.n * a.H * (a.dh / 8);
  if (dtype == SAS_BF16)
    bwd_delta_kernel<bf16_t><<<(unsigned)cdiv(dthreads, 256), 256, 0, s>>>((const bf16_t*)a.O, (const bf16_t*)a.dO,
                                                                            a.b, a.n, a.H, a.dh, a.delta);
  else
    bwd_delta_kernel<float><<<(unsigned)cdiv(dthreads, 256), 256, 0, s>>>((const float*)a.O, (const float*)a.dO,
                                                                           a.b, a.n, a.H, a.dh, a.delta);
  const bool need_dlg = a.dlog_gate && a.mode == SAS_MODE_GATED && a.K > 0 && !a.full;
  BwdArgs P = a;
  if (!need_dlg) P.dlg_head = nullptr;
  if (!(a.mode == SAS_MODE_GATED && a.full)) P.dlg_head_full = nullptr;
  if (P.dlg_head) {
    const size_t tot = (size_t)a.b * a.H * a.n * a.K;
    fill_f32_kernel<<<(unsigned)cdiv(tot, 256), 256, 0, s>>>(P.dlg_head, tot, 0.f);
  }
  if (dtype == SAS_BF16) {
    const hipError_t e = launch_attention_backward_bf16(P, s);
    if (e != hipSuccess) return e;
  } else {
    const size_t tq = (size_t)a.b * a.H * a.n, tk = (size_t)a.b * a.Hkv * a.n;
    if (a.dh == 128) {
      bwd_dq_f32_kernel<128><<<(unsigned)cdiv(tq, 64), 64, 0, s>>>(P);
      bwd_dkv_f32_kernel<128><<<(unsigned)cdiv(tk, 64), 64, 0, s>>>(P);
    } else {
      bwd_dq_f32_kernel<64><<<(unsigned)cdiv(tq, 64), 64, 0, s>>>(P);
      bwd_dkv_f32_kernel<64><<<(unsigned)cdiv(tk, 64), 64, 0, s>>>(P);
    }
  }
  if (need_dlg) {
    const size_t tot = (size_t)a.b * a.Hkv * a.n * a.K;
    bwd_dlog_gate_sum_kernel<<<(unsigned)cdiv(tot, 256), 256, 0, s>>>(P.dlg_head, a.sel_bias, a.ste, a.b, a.n,
                                                                        a.H, a.Hkv, a.K, a.dlog_gate);
  }
  if (P.dlg_head_full) {
    const int NB = cdiv(a.n, a.B);
    const size_t tot = (size_t)a.b * a.Hkv * a.n * NB;
    bwd_dlog_gate_full_sum_kernel<<<(unsigned)cdiv(tot, 256), 256, 0, s>>>(
        P.dlg_head_full, a.log_gate, a.ste, a.b, a.n, a.H, a.Hkv, a.B, NB, a.dlog_gate_full, a.doc);
  }
  return hipGetLastError();
}

}  // namespace sas

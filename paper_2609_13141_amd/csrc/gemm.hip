// C = A[M, K] * B[N, K]^T on MFMA (bf16 in, fp32 accumulate) with fused
// epilogues: QKV projection + RoPE, SwiGLU (gate and up in one pass),
// residual add.  A variant on the fp32 MFMA serves the fp32 dtype.
//
// Epilogues that combine two output columns (RoPE rotates the pair
// (i, i + dh/2) of a head; SwiGLU multiplies gate column f by up column f)
// get both columns into the same lane by permuting the B rows as they are
// loaded: logical column J of the tile maps to pair p = (J/64)*32 + J%32 and
// half (J/32)%2.  A 32x32 MFMA output tile holds column J%32 in lane J%32, so
// the two halves of a pair sit in neighbouring 32-column subtiles of the same
// lane.  Plain (residual) GEMMs use the identity mapping.
#include "common.h"
#include "kernels.h"

namespace sas {

struct GemmParams {
  int epi, M, K, N;  // N = logical columns of the tiling
  int npairs;        // pair epilogues: number of output column pairs
  const bf16_t* A;
  const bf16_t* B0;
  const bf16_t* B1;
  const bf16_t* B2;
  const bf16_t* resid;
  bf16_t* out;
  bf16_t* out1;
  bf16_t* out2;
  int H, Hkv, dh, seq_len;
  const float2* rope;
  const int32_t* row_pos;
  int group_m;       // M tiles per group of the tile order (0: M-fastest over all tiles, no XCD remap)
  // prefill cache write of the staged QKV epilogue (NULL k_pages: none)
  bf16_t* k_pages;
  bf16_t* v_pages;
  PageGeom geom;
  // K split over several workgroups per tile: each leaves its fp32 accumulators in
  // part [splits, tiles][BM x BN] (in the accumulators' own order) and
  // gemm_finish_kernel adds them and runs the epilogue
  int splits;
  float* part;
  int n_off, n_cnt;  // gemm_bf16_lds_kernel: logical columns [n_off, n_off + n_cnt) of this launch
};

// Tile of workgroup `bid`.  Workgroups are dispatched round-robin over the 8
// XCDs (bid % 8), each with its own L2.  The remap gives XCD x a contiguous
// range of a grouped tile order -- groups of group_m M tiles, M fastest inside
// a group -- so the workgroups sharing an L2 share operand tiles instead of
// each XCD streaming the whole weight matrix.
__device__ __forceinline__ void grouped_tile(int lid, int Mt, int Nt, int group_m, int& mt, int& nt) {
  const int gm = min(group_m, Mt);
  const int per_group = gm * Nt, grp = lid / per_group, m_first = grp * gm;
  const int gsz = min(Mt - m_first, gm), in = lid - grp * per_group;
  mt = m_first + in % gsz;
  nt = in / gsz;
}

__device__ __forceinline__ void tile_of(int bid, int Mt, int Nt, int group_m, int& mt, int& nt) {
  if (group_m <= 0) {
    mt = bid % Mt;
    nt = bid / Mt;
    return;
  }
  const int T = Mt * Nt, q = T / 8, r = T % 8, x = bid % 8, loc = bid / 8;
  const int lid = (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + loc;
  grouped_tile(lid, Mt, Nt, group_m, mt, nt);
}

// Source row (in units of K elements) of logical column J, or null past the
// last column (RESID: J >= N; pair epilogues: pair index >= npairs).
template <typename T>
__device__ __forceinline__ const T* b_row(int epi, int J, int N, int npairs, int K, const T* B0,
                                          const T* B1, const T* B2, int H, int Hkv, int dh) {
  if (epi == EPI_RESID) return (J < N) ? B0 + (size_t)J * K : nullptr;
  int p = (J >> 6) * 32 + (J & 31);
  int half = (J >> 5) & 1;
  if (p >= npairs) return nullptr;
  if (epi == EPI_SWIGLU) return (half ? B1 : B0) + (size_t)p * K;
  int hh = dh >> 1;
  int hd = p / hh, ir = p % hh;
  int c = hd * dh + ir + half * hh;
  if (c < H * dh) return B0 + (size_t)c * K;
  c -= H * dh;
  if (c < Hkv * dh) return B1 + (size_t)c * K;
  return B2 + (size_t)(c - Hkv * dh) * K;
}

// x * sigmoid(x) with the hardware reciprocal (1 ulp) in place of an IEEE division
__device__ __forceinline__ float silu_f(float x) { return x * __builtin_amdgcn_rcpf(1.0f + __expf(-x)); }

constexpr int BK = 64;

// Epilogue shared by the GEMM kernels.  Lane (lr, lk) of wave (wm, wn) holds
// column lr of every 32x32 subtile (i, j) of its TM x TN tile, at rows
// 8*(v/4) + 4*lk + (v%4) of the subtile for accumulator element v.
template <int EPI, int TM, int TN, int FM, int FN>
__device__ __forceinline__ void gemm_epilogue_t(const GemmParams& P, floatx16_t (&acc)[FM][FN], int m0, int n0,
                                                int wm, int wn, int lr, int lk) {
  // The loads an element needs (residual, rotary table) are issued for a
  // whole 32x32 subtile before any of them is used, from clamped addresses,
  // so that their latencies overlap.
  const int colbase = n0 + wn * TN;
  const int rowbase = m0 + wm * TM + 4 * lk;
  if constexpr (EPI == EPI_RESID) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int col = colbase + j * 32 + lr;
        const int colc = min(col, P.N - 1);
        float r[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int rowc = min(rowbase + i * 32 + 8 * (v >> 2) + (v & 3), P.M - 1);
          r[v] = bf16_to_f32(P.resid[(size_t)rowc * P.N + colc]);
        }
        if (col >= P.N) continue;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int row = rowbase + i * 32 + 8 * (v >> 2) + (v & 3);
          if (row < P.M) P.out[(size_t)row * P.N + col] = f32_to_bf16(acc[i][j][v] + r[v]);
        }
      }
    return;
  }
  const int hh = P.dh >> 1;
#pragma unroll
  for (int jp = 0; jp < FN / 2; ++jp) {
    const int J = colbase + jp * 64 + lr;  // half-0 logical column
    const int p = (J >> 6) * 32 + (J & 31);
    const bool pvalid = p < P.npairs;
    // per-column-pair destination (row stride ld, element offset base)
    bf16_t* dst;
    size_t ld;
    int ir = 0;
    bool rot = false;
    if constexpr (EPI == EPI_SWIGLU) {
      dst = P.out + p;
      ld = (size_t)P.npairs;
    } else {
      const int hd = min(p, P.npairs - 1) / hh;
      ir = min(p, P.npairs - 1) - hd * hh;
      if (hd < P.H) {
        dst = P.out + (size_t)hd * P.dh + ir;
        ld = (size_t)P.H * P.dh;
      } else if (hd < P.H + P.Hkv) {
        dst = P.out1 + (size_t)(hd - P.H) * P.dh + ir;
        ld = (size_t)P.Hkv * P.dh;
      } else {
        dst = P.out2 + (size_t)(hd - P.H - P.Hkv) * P.dh + ir;
        ld = (size_t)P.Hkv * P.dh;
      }
      rot = hd < P.H + P.Hkv;
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      float2 cs[16];
      if constexpr (EPI == EPI_QKV_ROPE) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int rowc = min(rowbase + i * 32 + 8 * (v >> 2) + (v & 3), P.M - 1);
          const int pos = P.row_pos ? P.row_pos[rowc] : rowc % P.seq_len;
          cs[v] = P.rope[(size_t)pos * hh + ir];
        }
      }
      if (!pvalid) continue;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = rowbase + i * 32 + 8 * (v >> 2) + (v & 3);
        if (row >= P.M) continue;
        float x1 = acc[i][2 * jp][v], x2 = acc[i][2 * jp + 1][v];
        if constexpr (EPI == EPI_SWIGLU) {
          dst[(size_t)row * ld] = f32_to_bf16(silu_f(x1) * x2);
        } else {
          if (rot) {
            const float o1 = x1 * cs[v].x - x2 * cs[v].y;
            const float o2 = x2 * cs[v].x + x1 * cs[v].y;
            x1 = o1;
            x2 = o2;
          }
          dst[(size_t)row * ld] = f32_to_bf16(x1);
          dst[(size_t)row * ld + hh] = f32_to_bf16(x2);
        }
      }
    }
  }
}

template <int TM, int TN, int FM, int FN>
__device__ __forceinline__ void gemm_epilogue(const GemmParams& P, floatx16_t (&acc)[FM][FN], int m0, int n0,
                                              int wm, int wn, int lr, int lk) {
  if (P.epi == EPI_RESID) gemm_epilogue_t<EPI_RESID, TM, TN, FM, FN>(P, acc, m0, n0, wm, wn, lr, lk);
  else if (P.epi == EPI_SWIGLU) gemm_epilogue_t<EPI_SWIGLU, TM, TN, FM, FN>(P, acc, m0, n0, wm, wn, lr, lk);
  else gemm_epilogue_t<EPI_QKV_ROPE, TM, TN, FM, FN>(P, acc, m0, n0, wm, wn, lr, lk);
}


template <int BM, int BN, int WM, int WN>
__global__ void __launch_bounds__(WM * WN * 64)
gemm_bf16_kernel(GemmParams P) {
  constexpr int NT = WM * WN * 64;
  constexpr int TM = BM / WM, TN = BN / WN;
  constexpr int FM = TM / 32, FN = TN / 32;
  constexpr int ACH = BM * 8 / NT;  // 16-byte A chunks per thread per k-tile
  constexpr int BCH = BN * 8 / NT;
  static_assert(ACH * NT == BM * 8 && BCH * NT == BN * 8, "tile/threads mismatch");
  static_assert(TN % 64 == 0, "pair epilogues need 64-column wave tiles");

  extern __shared__ __align__(16) unsigned char smem[];
  bf16_t* As = (bf16_t*)smem;                 // [2][BM][64]
  bf16_t* Bs = As + 2 * BM * BK;              // [2][BN][64]

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;

  const int Mt = (P.M + BM - 1) / BM, Nt = (P.N + BN - 1) / BN;
  int mt, nt;
  tile_of(blockIdx.x, Mt, Nt, P.group_m, mt, nt);
  const int m0 = mt * BM, n0 = nt * BN;

  // per-thread global source pointers (fixed along K)
  const bf16_t* a_src[ACH];
  const bf16_t* b_src[BCH];
  int a_lds[ACH], b_lds[BCH];
#pragma unroll
  for (int i = 0; i < ACH; ++i) {
    int c = tid + i * NT;
    int row = c >> 3, c16 = c & 7;
    int gr = m0 + row;
    a_src[i] = (gr < P.M) ? P.A + (size_t)gr * P.K + c16 * 8 : nullptr;
    a_lds[i] = row * BK + ((c16 ^ ((row >> 1) & 7)) << 3);
  }
#pragma unroll
  for (int i = 0; i < BCH; ++i) {
    int c = tid + i * NT;
    int row = c >> 3, c16 = c & 7;
    const bf16_t* r = b_row<bf16_t>(P.epi, n0 + row, P.N, P.npairs, P.K, P.B0, P.B1, P.B2, P.H,
                                    P.Hkv, P.dh);
    b_src[i] = r ? r + c16 * 8 : nullptr;
    b_lds[i] = row * BK + ((c16 ^ ((row >> 1) & 7)) << 3);
  }

  floatx16_t acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  uint4 ra[ACH], rb[BCH];
  const int nk = (P.K + BK - 1) / BK;
  const bool k_full = (P.K % BK) == 0;

  auto gload = [&](int kt) {
    const int k0 = kt * BK;
#pragma unroll
    for (int i = 0; i < ACH; ++i) {
      int kc = k0 + (((tid + i * NT) & 7) << 3);
      bool ok = a_src[i] && (k_full || kc < P.K);
      ra[i] = ok ? *(const uint4*)(a_src[i] + k0) : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < BCH; ++i) {
      int kc = k0 + (((tid + i * NT) & 7) << 3);
      bool ok = b_src[i] && (k_full || kc < P.K);
      rb[i] = ok ? *(const uint4*)(b_src[i] + k0) : make_uint4(0, 0, 0, 0);
    }
  };
  auto lstore = [&](int buf) {
    bf16_t* a = As + buf * BM * BK;
    bf16_t* b = Bs + buf * BN * BK;
#pragma unroll
    for (int i = 0; i < ACH; ++i) *(uint4*)(a + a_lds[i]) = ra[i];
#pragma unroll
    for (int i = 0; i < BCH; ++i) *(uint4*)(b + b_lds[i]) = rb[i];
  };

  gload(0);
  lstore(0);
  __syncthreads();

  const int lr = lane & 31, lk = lane >> 5;
  for (int kt = 0; kt < nk; ++kt) {
    if (kt + 1 < nk) gload(kt + 1);
    const bf16_t* a = As + (kt & 1) * BM * BK;
    const bf16_t* b = Bs + (kt & 1) * BN * BK;
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk) {
      const int kc = kk * 2 + lk;
      bf16x8_t fa[FM], fb[FN];
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        int row = wm * TM + i * 32 + lr;
        fa[i] = *(const bf16x8_t*)(a + row * BK + ((kc ^ ((row >> 1) & 7)) << 3));
      }
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        int row = wn * TN + j * 32 + lr;
        fb[j] = *(const bf16x8_t*)(b + row * BK + ((kc ^ ((row >> 1) & 7)) << 3));
      }
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < nk) lstore((kt + 1) & 1);
    __syncthreads();
  }

  gemm_epilogue<TM, TN, FM, FN>(P, acc, m0, n0, wm, wn, lr, lk);
}

// ---- direct-to-LDS loading (shared by the kernel below) --------------------
// Global tiles are copied straight into LDS with global_load_lds_dwordx4
// (each lane writes 16 bytes at M0 + 16*lane), so no VGPRs stage them.  The
// XOR swizzle of the 16-byte chunks is applied by choosing which global chunk
// each lane fetches: with CPR = BKT/8 chunks per row, LDS chunk c of a stage
// holds row r = c / CPR and k-chunk (c % CPR) ^ ((r / (16/CPR)) % CPR).  A
// 128-bit LDS read serves 16 lanes per pass; 16 consecutive rows then cover
// 16 distinct 4-bank groups.  Out-of-range rows are clamped to a valid row
// (their results are never stored), so the main loop has no predication.
// STAGES LDS buffers: the loads of k-tile t + STAGES - 1 are issued right after
// the barrier that ends the reads of k-tile t - 1, so STAGES - 1 tiles are in
// flight while k-tile t is multiplied.
typedef __attribute__((address_space(3))) void lds_void_t;

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Workgroup barrier that waits for this wave's LDS reads but not for its
// outstanding global->LDS loads: __syncthreads() is a release fence and would
// drain vmcnt to zero, i.e. wait for every stage in flight.
__device__ __forceinline__ void barrier_lds() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}


// ---- 8-wave direct-to-LDS kernel with an LDS-staged epilogue (K % 64 == 0) --
// Two waves per SIMD: a wave's direct-to-LDS load instructions stall its own
// issue for tens of cycles, and the second wave keeps the matrix core busy
// meanwhile.  Per 64-wide k-tile a wave runs four 16-deep MFMA steps and reads
// the fragments of the next step while the current one multiplies.  The
// workgroup barrier of k-tile kt sits before its last step (every wave's reads
// of kt are complete there); after it the stage of kt is refilled with k-tile
// kt + STAGES and the reads of k-tile kt + 1 start under the last step's MFMAs.
// Fragment reads are plain LDS loads: the compiler's waits (one per step) are
// the ones this schedule needs.
//
// The epilogue stages 32 rows of a wave's tile at a time in LDS and writes
// 16-byte stores (8 bf16 per lane) instead of one 2-byte store per
// accumulator element.  RESID stages fp32 sums and fetches the residual before
// the staging so that its latency overlaps it; SWIGLU stages bf16 results;
// QKV stages the two halves of each rotary pair in fp32 and rotates on the way
// out, reading 8 consecutive rotary entries (64 bytes) per lane.  It needs
// 8 | N (RESID) or 8 | npairs and 16 | dh (pair epilogues); other shapes use
// gemm_epilogue_t.
template <int EPI, int TN>
constexpr int epi_region_bytes() {
  return EPI == EPI_SWIGLU ? 32 * (TN / 2) * 2 : 32 * TN * 4;
}

__device__ __forceinline__ uint4 pack8_bf16(const float* x) {
  uint4 r;
  r.x = pack_bf16x2(x[0], x[1]);
  r.y = pack_bf16x2(x[2], x[3]);
  r.z = pack_bf16x2(x[4], x[5]);
  r.w = pack_bf16x2(x[6], x[7]);
  return r;
}

template <int EPI, int TM, int TN>
__device__ __forceinline__ void gemm_epilogue_lds(const GemmParams& P, floatx4_t (&acc)[TM / 16][TN / 16], int m0,
                                                  int n0, int wm, int wn, int lane, unsigned char* region) {
  const int colbase = n0 + wn * TN;
  const int rowbase = m0 + wm * TM;
  // The accumulator elements of the wave tile's 32-row block ib, as (row in the
  // block, column in the wave tile, value): element v of subtile (2 ib + h, j) is
  // row 16 h + 4 (lane/16) + v, column 16 j + lane%16.
  auto for_each_elem = [&](int ib, auto&& f) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < TN / 16; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) f(16 * h + 4 * (lane >> 4) + v, j * 16 + (lane & 15), acc[2 * ib + h][j][v]);
  };
  // The same for the pair epilogues, as (row, pair in the wave tile, first
  // half, second half): column c with c % 64 < 32 pairs with c + 32, pair
  // index 32 (c / 64) + c % 32.
  auto for_each_pair = [&](int ib, auto&& f) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int t = 0; t < TN / 64; ++t)
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            f(16 * h + 4 * (lane >> 4) + v, t * 32 + u * 16 + (lane & 15), acc[2 * ib + h][4 * t + u][v],
              acc[2 * ib + h][4 * t + u + 2][v]);
  };
#pragma unroll
  for (int ib = 0; ib < TM / 32; ++ib) {
    const int brow = rowbase + ib * 32;
    if constexpr (EPI == EPI_RESID) {
      constexpr int GPR = TN / 8, G = 32 * GPR, IT = (G + 63) / 64;
      uint4 rv[IT];
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int g = it * 64 + lane;
        const int r = min(g / GPR, 31), c8 = (g % GPR) * 8;
        const int row = min(brow + r, P.M - 1), col = min(colbase + c8, P.N - 8);
        rv[it] = *(const uint4*)(P.resid + (size_t)row * P.N + col);
      }
      float* st = (float*)region;
      for_each_elem(ib, [&](int r, int c, float x) { st[r * TN + c] = x; });
      // a wave's LDS accesses complete in order: the reads below see its writes
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int g = it * 64 + lane;
        if (G % 64 != 0 && g >= G) break;
        const int r = g / GPR, c8 = (g % GPR) * 8;
        const int row = brow + r, col = colbase + c8;
        const float4 a = *(const float4*)(st + r * TN + c8);
        const float4 b = *(const float4*)(st + r * TN + c8 + 4);
        if (row < P.M && col < P.N) {
          float x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
          const uint32_t rw[4] = {rv[it].x, rv[it].y, rv[it].z, rv[it].w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            x[2 * e] += __uint_as_float(rw[e] << 16);
            x[2 * e + 1] += __uint_as_float(rw[e] & 0xffff0000u);
          }
          *(uint4*)(P.out + (size_t)row * P.N + col) = pack8_bf16(x);
        }
      }
    } else if constexpr (EPI == EPI_SWIGLU) {
      constexpr int NP = TN / 2, GPR = NP / 8, G = 32 * GPR;
      bf16_t* st = (bf16_t*)region;
      for_each_pair(ib, [&](int r, int pp, float g, float u) { st[r * NP + pp] = f32_to_bf16(silu_f(g) * u); });
      const int pbase = colbase >> 1;  // colbase is a multiple of 64
#pragma unroll
      for (int g0 = 0; g0 < G; g0 += 64) {
        const int g = g0 + lane;
        if (G % 64 != 0 && g >= G) break;
        const int r = g / GPR, q8 = (g % GPR) * 8;
        const int row = brow + r, p = pbase + q8;
        if (row >= P.M || p >= P.npairs) continue;
        *(uint4*)(P.out + (size_t)row * P.npairs + p) = *(const uint4*)(st + r * NP + q8);
      }
    } else {
      constexpr int NP = TN / 2, GPR = NP / 8, G = 32 * GPR;
      constexpr int IT = (G + 63) / 64, BATCH = 2;
      const int hh = P.dh >> 1;
      const int pbase = colbase >> 1;
      const int pb = P.row_pos ? 0 : brow % P.seq_len;  // wave-uniform
      float* st = (float*)region;  // [2][32][NP]: first and second halves of the pairs
      for_each_pair(ib, [&](int r, int pp, float x1, float x2) {
        st[r * NP + pp] = x1;
        st[32 * NP + r * NP + pp] = x2;
      });
#pragma unroll
      for (int b0 = 0; b0 < IT; b0 += BATCH) {
        float4 cs[BATCH][4];  // 8 (cos, sin) entries per group, fetched before use
#pragma unroll
        for (int it = b0; it < b0 + BATCH && it < IT; ++it) {
          const int g = min(it * 64 + lane, G - 1);
          const int r = g / GPR, q8 = (g % GPR) * 8;
          const int p = min(pbase + q8, P.npairs - 8);
          const int hd = p / hh, ir = p - hd * hh;
          int pos;
          if (P.row_pos) pos = P.row_pos[min(brow + r, P.M - 1)];
          else if (P.seq_len >= 32) pos = pb + r >= P.seq_len ? pb + r - P.seq_len : pb + r;
          else pos = min(brow + r, P.M - 1) % P.seq_len;
          const float4* rp = (const float4*)(P.rope + (size_t)pos * hh + ir);
#pragma unroll
          for (int e = 0; e < 4; ++e) cs[it - b0][e] = rp[e];
        }
#pragma unroll
        for (int it = b0; it < b0 + BATCH && it < IT; ++it) {
          const int g = it * 64 + lane;
          if (G % 64 != 0 && g >= G) break;
          const int r = g / GPR, q8 = (g % GPR) * 8;
          const int row = brow + r, p = pbase + q8;
          if (row >= P.M || p >= P.npairs) continue;
          const int hd = p / hh, ir = p - hd * hh;
          float x1[8], x2[8];
          *(float4*)&x1[0] = *(const float4*)(st + r * NP + q8);
          *(float4*)&x1[4] = *(const float4*)(st + r * NP + q8 + 4);
          *(float4*)&x2[0] = *(const float4*)(st + 32 * NP + r * NP + q8);
          *(float4*)&x2[4] = *(const float4*)(st + 32 * NP + r * NP + q8 + 4);
          bf16_t* dst;
          size_t ld;
          if (hd < P.H) {
            dst = P.out + (size_t)hd * P.dh + ir;
            ld = (size_t)P.H * P.dh;
          } else if (hd < P.H + P.Hkv) {
            dst = P.out1 + (size_t)(hd - P.H) * P.dh + ir;
            ld = (size_t)P.Hkv * P.dh;
          } else {
            dst = P.out2 + (size_t)(hd - P.H - P.Hkv) * P.dh + ir;
            ld = (size_t)P.Hkv * P.dh;
          }
          if (hd < P.H + P.Hkv) {
            const float* c = (const float*)cs[it - b0];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const float co = c[2 * e], si = c[2 * e + 1];
              const float o1 = x1[e] * co - x2[e] * si;
              const float o2 = x2[e] * co + x1[e] * si;
              x1[e] = o1;
              x2[e] = o2;
            }
          }
          dst += (size_t)row * ld;
          const uint4 w1 = pack8_bf16(x1), w2 = pack8_bf16(x2);
          *(uint4*)dst = w1;
          *(uint4*)(dst + hh) = w2;
          if (P.k_pages && hd >= P.H) {
            // the same K/V values into the paged cache: sequence row / seq_len,
            // position row % seq_len (positions without a page are skipped)
            const bool isk = hd < P.H + P.Hkv;
            const int g = isk ? hd - P.H : hd - P.H - P.Hkv;
            const long long off = P.geom.offset(row / P.seq_len, g, row % P.seq_len, P.Hkv, P.dh);
            if (off >= 0) {
              bf16_t* pg = (isk ? P.k_pages : P.v_pages) + off + ir;
              *(uint4*)pg = w1;
              *(uint4*)(pg + hh) = w2;
            }
          }
        }
      }
    }
  }
}

template <int EPI, int BM, int BN, int WM, int WN, int STAGES, bool SPLIT>
__global__ void __launch_bounds__(WM * WN * 64)
gemm_bf16_lds_kernel(GemmParams P) {
  // v_mfma_f32_16x16x32_bf16: the same work per LDS byte as 32x32x16 in shorter,
  // lower-power instructions (a higher clock under load: 5-10% at 256x256)
  constexpr int MI = 16, BKT = 64;
  constexpr int KS = 512 / MI;  // k per MFMA
  constexpr int KK = BKT / KS;
  static_assert(KK % 2 == 0, "the fragment double buffer alternates with the k-step: an even count per k-tile");
  constexpr int NW = WM * WN;
  constexpr int TM = BM / WM, TN = BN / WN;
  constexpr int FM = TM / MI, FN = TN / MI, NF = FM + FN, NMF = FM * FN;
  constexpr int CPR = BKT / 8, RPG = 16 / CPR;  // the chunk swizzle described above
  constexpr int AI = BM * CPR / (64 * NW);
  constexpr int BI = BN * CPR / (64 * NW);
  constexpr int LI = AI + BI;
  static_assert(AI * 64 * NW == BM * CPR && BI * 64 * NW == BN * CPR, "tile/threads mismatch");
  static_assert(EPI == EPI_RESID || TN % 64 == 0, "pair epilogues need 64-column wave tiles");
  static_assert(STAGES >= 2 && (STAGES - 1) * LI <= 63, "vmcnt range");
  constexpr int STAGE = (BM + BN) * BKT;  // elements per stage
  static_assert(NW * epi_region_bytes<EPI, TN>() <= STAGES * STAGE * 2, "epilogue staging exceeds the stages");

  extern __shared__ __align__(16) unsigned char smem[];
  bf16_t* S = (bf16_t*)smem;

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int Mt = (P.M + BM - 1) / BM, Nt = (P.n_cnt + BN - 1) / BN;
  // SPLIT: workgroup (split, tile) in one order, split by split, so that the tiles
  // an XCD works on at a time share operands over the same part of K
  int mt, nt, kt0 = 0, nk = P.K / BKT;
  size_t slot = 0;
  if constexpr (SPLIT) {
    const int tiles = Mt * Nt, T = tiles * P.splits, q = T / 8, r = T % 8, x = blockIdx.x % 8;
    const int lid = (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + blockIdx.x / 8;
    const int sp = lid / tiles, tile = lid - sp * tiles;
    grouped_tile(tile, Mt, Nt, P.group_m, mt, nt);
    kt0 = (int)((long long)nk * sp / P.splits);
    nk = (int)((long long)nk * (sp + 1) / P.splits) - kt0;
    slot = (size_t)sp * tiles + (size_t)nt * Mt + mt;
  } else {
    tile_of(blockIdx.x, Mt, Nt, P.group_m, mt, nt);
  }
  const int m0 = mt * BM, n0 = P.n_off + nt * BN;

  // per-lane sources of the direct-to-LDS loads (rows clamped; results of
  // clamped rows are never stored); A's offsets count from the tile's first row,
  // so that they fit 32 bits for any number of rows
  const bf16_t* const a_tile = P.A + (size_t)m0 * P.K;
  uint32_t a_off[AI];
  const bf16_t* b_src[BI];
#pragma unroll
  for (int j = 0; j < AI; ++j) {
    const int c = (wave * AI + j) * 64 + lane;
    const int r = c / CPR, cc = (c % CPR) ^ ((r / RPG) % CPR);
    a_off[j] = (uint32_t)min(r, P.M - 1 - m0) * (uint32_t)P.K + cc * 8;
  }
#pragma unroll
  for (int j = 0; j < BI; ++j) {
    const int c = (wave * BI + j) * 64 + lane;
    const int r = c / CPR, cc = (c % CPR) ^ ((r / RPG) % CPR);
    const bf16_t* row = b_row<bf16_t>(P.epi, n0 + r, P.N, P.npairs, P.K, P.B0, P.B1, P.B2, P.H, P.Hkv, P.dh);
    b_src[j] = (row ? row : P.B0) + cc * 8;
  }
  // load j (0 <= j < LI) of k-tile kt into its stage
  auto issue1 = [&](int kt, int j) {
    const int k0 = (SPLIT ? kt0 + kt : kt) * BKT;
    bf16_t* st = S + (kt % STAGES) * STAGE;
    if (j < AI)
      __builtin_amdgcn_global_load_lds((const void*)(a_tile + a_off[j] + k0),
                                       (lds_void_t*)(st + (wave * AI + j) * 64 * 8), 16, 0, 0);
    else
      __builtin_amdgcn_global_load_lds((const void*)(b_src[j - AI] + k0),
                                       (lds_void_t*)(st + BM * BKT + (wave * BI + j - AI) * 64 * 8), 16, 0, 0);
  };

  floatx4_t acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.f;

  // an operand lane supplies row lr of its fragment, 16-byte k-chunk lk of the step
  const int lr = lane % MI, lk = lane / MI;
  int foff[NF];  // element offset of fragment g's row in a stage: A0..A(FM-1), B0..B(FN-1)
#pragma unroll
  for (int g = 0; g < NF; ++g)
    foff[g] = g < FM ? (wm * TM + g * MI + lr) * BKT : BM * BKT + (wn * TN + (g - FM) * MI + lr) * BKT;
  const int sw = (lr / RPG) % CPR;  // fragment row bases are multiples of 16
  auto rd_off = [&](int kt, int kk) -> int {
    return (kt % STAGES) * STAGE + (((kk * (KS / 8) + lk) ^ sw) << 3);
  };
  bf16x8_t fr[2][NF];

  const int npro = nk < STAGES ? nk : STAGES;
  for (int t = 0; t < npro; ++t)
#pragma unroll
    for (int j = 0; j < LI; ++j) issue1(t, j);
  if (nk >= STAGES) wait_vmcnt<(STAGES - 1) * LI>();
  else wait_vmcnt<0>();
  barrier_lds();
  {
    const bf16_t* a0 = S + rd_off(0, 0);
#pragma unroll
    for (int g = 0; g < NF; ++g) fr[0][g] = *(const bf16x8_t*)(a0 + foff[g]);
  }

  // The loop's place among 32-byte blocks of code decides up to 7% of a round (256x256, 512 x 22016 x
  // 4096: 99 to 107 us by the loop's first byte), and whatever is added before it would move it: this
  // fixes it, with the padding that measured best over the products of a tile (256x128: 4 bytes, 3%
  // ahead of 24; the others 24, within 1% of the best).
  if constexpr (BM == 256 && BN == 128) asm volatile(".p2align 5\n\ts_nop 0" ::: "memory");
  else asm volatile(".p2align 5\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0" ::: "memory");
  for (int kt = 0; kt < nk; ++kt) {
    const bool has_next = kt + 1 < nk;
    const bool refill = kt + STAGES < nk;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const int cur = kk & 1, nxt = cur ^ 1;
      if (kk == KK - 1 && has_next) {
        // k-tile kt+1 must have landed for every wave; loads issued after it
        // are those of k-tiles kt+2 .. kt+STAGES-1
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (kt + STAGES - 1 < nk) wait_vmcnt<(STAGES - 2) * LI>();
        else wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
      }
      const bool more = kk + 1 < KK || has_next;
      const bf16_t* na = S + (kk + 1 < KK ? rd_off(kt, kk + 1) : rd_off(kt + 1, 0));
      int m = 0;
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr[cur][i], fr[cur][FM + j], acc[i][j], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
          if (more && m < NF) fr[nxt][m] = *(const bf16x8_t*)(na + foff[m]);
          if (kk == KK - 1 && refill) {
#pragma unroll
            for (int q = m * LI / NMF; q < (m + 1) * LI / NMF; ++q) issue1(kt + STAGES, q);
          }
          __builtin_amdgcn_sched_barrier(0);
          ++m;
        }
#pragma unroll
      for (int g = NMF; g < NF; ++g)
        if (more) fr[nxt][g] = *(const bf16x8_t*)(na + foff[g]);
    }
  }
  if constexpr (SPLIT) {
    float* o = P.part + slot * (BM * BN) + (size_t)(wave * FM * FN) * (MI * MI) + lane * 4;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) *(floatx4_t*)(o + (i * FN + j) * (MI * MI)) = acc[i][j];
    return;
  }
  barrier_lds();  // every wave is done with the stages
  gemm_epilogue_lds<EPI, TM, TN>(P, acc, m0, n0, wm, wn, lane, smem + wave * epi_region_bytes<EPI, TN>());
}

// The splits' accumulators of a tile added in order, and the epilogue; the layout
// is that of gemm_bf16_lds_kernel with the same template arguments.
template <int EPI, int BM, int BN, int WM, int WN>
__global__ void __launch_bounds__(WM * WN * 64) gemm_finish_kernel(GemmParams P) {
  constexpr int TM = BM / WM, TN = BN / WN, FM = TM / 16, FN = TN / 16;
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int Mt = (P.M + BM - 1) / BM, tiles = gridDim.x;
  const int mt = blockIdx.x % Mt, nt = blockIdx.x / Mt;
  floatx4_t acc[FM][FN];
  const float* o = P.part + (size_t)blockIdx.x * (BM * BN) + (size_t)(wave * FM * FN) * 256 + lane * 4;
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = *(const floatx4_t*)(o + (i * FN + j) * 256);
  for (int sp = 1; sp < P.splits; ++sp) {
    o += (size_t)tiles * (BM * BN);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const floatx4_t p = *(const floatx4_t*)(o + (i * FN + j) * 256);
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[i][j][v] += p[v];
      }
  }
  gemm_epilogue_lds<EPI, TM, TN>(P, acc, mt * BM, nt * BN, wave / WN, wave % WN, lane,
                                     smem + wave * epi_region_bytes<EPI, TN>());
}

// ---- fp32 path ------------------------------------------------------------------
// v_mfma_f32_16x16x4_f32 (fp32 products and sums, one rounding per addition).
// Bound by latency at the sizes this dtype is used for (tens to a few thousand
// rows of a narrow layer): a workgroup owns 16 FM rows x 16 FN logical columns
// and its 4 waves split K, so that even a 64-row product has hundreds of waves
// and a chain of K / 64 steps each; their sums meet in LDS in wave order.  The
// operands go straight from global memory to registers, 16 bytes per lane: lane
// (c, q) holds row or column c at k = 16 st + 4 q .. + 3, and step e multiplies
// the k = 16 st + 4 q + e of the four lane groups.  At 64 rows of the d = 256,
// d_ff = 688 layer the four products take 27 us; with one thread per output
// they took 324 us.
struct GemmF32 {
  int M, K, N, npairs;
  const float *A, *B0, *B1, *B2, *resid;
  float *out, *out1, *out2;
  int H, Hkv, dh, seq_len;
  const float2* rope;
  const int32_t* row_pos;
};

template <int EPI, int FM, int FN>
__global__ void __launch_bounds__(256) gemm_f32_kernel(GemmF32 P) {
  constexpr bool PLAIN = EPI == EPI_RESID || EPI == EPI_F32OUT;
  static_assert(PLAIN || FN % 2 == 0, "column tiles 2u and 2u + 1 are the halves of pair group u");
  __shared__ floatx4_t part[4][FM * FN][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = lane & 15, q = lane >> 4;
  const int Mt = (P.M + 16 * FM - 1) / (16 * FM);
  const int m0 = (blockIdx.x % Mt) * 16 * FM, nt = blockIdx.x / Mt;
  const float* ar[FM];
  const float* br[FN];
#pragma unroll
  for (int i = 0; i < FM; ++i) ar[i] = P.A + (size_t)min(m0 + i * 16 + c, P.M - 1) * P.K + 4 * q;
#pragma unroll
  for (int f = 0; f < FN; ++f) {
    const float* r;
    if constexpr (PLAIN) {
      r = P.B0 + (size_t)min(nt * 16 * FN + f * 16 + c, P.N - 1) * P.K;
    } else {
      const int p = min(nt * 8 * FN + (f / 2) * 16 + c, P.npairs - 1);
      r = b_row<float>(EPI, (p / 32) * 64 + p % 32 + (f & 1) * 32, P.N, P.npairs, P.K, P.B0, P.B1, P.B2, P.H, P.Hkv,
                       P.dh);
    }
    br[f] = r + 4 * q;
  }
  floatx4_t acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int f = 0; f < FN; ++f) acc[i][f] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  // this wave's range of 16-deep steps; U steps are loaded together (K is a
  // multiple of 4: a lane's 4 values are all inside K or all zero)
  constexpr int U = FM == 1 ? 8 : (FM == 2 ? 4 : 2);
  const int steps = (P.K + 15) / 16, per = (steps + 3) / 4;
  const int s0 = wave * per, s1 = min(steps, s0 + per);
  for (int st = s0; st < s1; st += U) {
    floatx4_t a[U][FM], b[U][FN];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool ok = st + u < s1 && (st + u) * 16 + 4 * q < P.K;
      const int k = ok ? (st + u) * 16 : 0;
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        a[u][i] = *(const floatx4_t*)(ar[i] + k - (ok ? 0 : 4 * q));
        if (!ok) a[u][i] = floatx4_t{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int f = 0; f < FN; ++f) {
        b[u][f] = *(const floatx4_t*)(br[f] + k - (ok ? 0 : 4 * q));
        if (!ok) b[u][f] = floatx4_t{0.f, 0.f, 0.f, 0.f};
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int f = 0; f < FN; ++f)
            acc[i][f] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][i][e], b[u][f][e], acc[i][f], 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int f = 0; f < FN; ++f) part[wave][i * FN + f][lane] = acc[i][f];
  __syncthreads();
  auto total = [&](int tile) {
    floatx4_t t = part[0][tile][lane];
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      const floatx4_t p = part[w][tile][lane];
#pragma unroll
      for (int v = 0; v < 4; ++v) t[v] += p[v];
    }
    return t;
  };
  // element v of a tile: row 4 q + v, column c
  constexpr int FU = PLAIN ? FN : FN / 2;
  for (int u = wave; u < FM * FU; u += 4) {
    const int i = u / FU, f = u % FU;
    const int row0 = m0 + i * 16 + 4 * q;
    if constexpr (PLAIN) {
      const floatx4_t t = total(i * FN + f);
      const int col = nt * 16 * FN + f * 16 + c;
      if (col >= P.N) continue;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if (row0 + v >= P.M) continue;
        const size_t o = (size_t)(row0 + v) * P.N + col;
        P.out[o] = EPI == EPI_RESID ? P.resid[o] + t[v] : t[v];
      }
    } else {
      const floatx4_t t1 = total(i * FN + 2 * f), t2 = total(i * FN + 2 * f + 1);
      const int p = nt * 8 * FN + f * 16 + c;
      if (p >= P.npairs) continue;
      const int hh = P.dh / 2, hd = p / hh, ir = p % hh;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = row0 + v;
        if (row >= P.M) continue;
        float x1 = t1[v], x2 = t2[v];
        if constexpr (EPI == EPI_SWIGLU) {
          P.out[(size_t)row * P.npairs + p] = silu_f(x1) * x2;
        } else {
          float* dst;
          if (hd < P.H) dst = P.out + ((size_t)row * P.H + hd) * P.dh;
          else if (hd < P.H + P.Hkv) dst = P.out1 + ((size_t)row * P.Hkv + (hd - P.H)) * P.dh;
          else dst = P.out2 + ((size_t)row * P.Hkv + (hd - P.H - P.Hkv)) * P.dh;
          if (hd < P.H + P.Hkv) {
            const int pos = P.row_pos ? P.row_pos[row] : row % P.seq_len;
            const float2 cs = P.rope[(size_t)pos * hh + ir];
            const float o1 = x1 * cs.x - x2 * cs.y;
            const float o2 = x2 * cs.x + x1 * cs.y;
            x1 = o1;
            x2 = o2;
          }
          dst[ir] = x1;
          dst[ir + hh] = x2;
        }
      }
    }
  }
}

template <int EPI>
static hipError_t run_f32(const GemmF32& P, hipStream_t s) {
  constexpr bool PLAIN = EPI == EPI_RESID || EPI == EPI_F32OUT;
  const int nt = PLAIN ? cdiv(P.N, 32) : cdiv(P.npairs, 16);  // tiles of 32 logical columns
  // taller tiles (fewer operand bytes per product) while two workgroups per compute unit remain
  if ((long long)cdiv(P.M, 64) * nt >= 512) gemm_f32_kernel<EPI, 4, 2><<<cdiv(P.M, 64) * nt, 256, 0, s>>>(P);
  else if ((long long)cdiv(P.M, 32) * nt >= 512) gemm_f32_kernel<EPI, 2, 2><<<cdiv(P.M, 32) * nt, 256, 0, s>>>(P);
  else if constexpr (PLAIN) gemm_f32_kernel<EPI, 1, 1><<<cdiv(P.M, 16) * cdiv(P.N, 16), 256, 0, s>>>(P);
  else gemm_f32_kernel<EPI, 1, 2><<<cdiv(P.M, 16) * nt, 256, 0, s>>>(P);
  return hipGetLastError();
}

template <int BM, int BN, int WM, int WN>
static hipError_t run_bf16(const GemmParams& P, hipStream_t s) {
  constexpr int NT = WM * WN * 64;
  const int tiles = ((P.M + BM - 1) / BM) * ((P.N + BN - 1) / BN);
  const size_t lds = (size_t)2 * (BM + BN) * BK * sizeof(bf16_t);
  hipLaunchKernelGGL((gemm_bf16_kernel<BM, BN, WM, WN>), dim3(tiles), dim3(NT), lds, s, P);
  return hipGetLastError();
}

template <int EPI, int BM, int BN, int WM, int WN, int STAGES, bool SPLIT>
static hipError_t run_lds_t(const GemmParams& P, hipStream_t s) {
  constexpr int NT = WM * WN * 64;
  const int tiles = ((P.M + BM - 1) / BM) * ((P.n_cnt + BN - 1) / BN);
  const size_t lds = (size_t)STAGES * (BM + BN) * 64 * sizeof(bf16_t);
  static bool attr = false;
  if (!attr) {
    (void)hipFuncSetAttribute((const void*)gemm_bf16_lds_kernel<EPI, BM, BN, WM, WN, STAGES, SPLIT>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if constexpr (SPLIT)
      (void)hipFuncSetAttribute((const void*)gemm_finish_kernel<EPI, BM, BN, WM, WN>,
                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                WM * WN * epi_region_bytes<EPI, BN / WN>());
    attr = true;
  }
  if constexpr (SPLIT) {
    g_launch_events = LaunchEvents{nullptr, nullptr, 0};  // two launches: timed around both
    gemm_bf16_lds_kernel<EPI, BM, BN, WM, WN, STAGES, true><<<tiles * P.splits, NT, lds, s>>>(P);
    gemm_finish_kernel<EPI, BM, BN, WM, WN>
        <<<tiles, NT, WM * WN * epi_region_bytes<EPI, BN / WN>(), s>>>(P);
    return hipGetLastError();
  } else {
    return launch_ext(gemm_bf16_lds_kernel<EPI, BM, BN, WM, WN, STAGES, false>, dim3(tiles), dim3(NT),
                      (uint32_t)lds, s, P);
  }
}

template <int BM, int BN, int WM, int WN, int STAGES>
static hipError_t run_lds(const GemmParams& P, hipStream_t s) {
  if (P.splits > 1) {
    if (P.epi == EPI_RESID) return run_lds_t<EPI_RESID, BM, BN, WM, WN, STAGES, true>(P, s);
    if (P.epi == EPI_SWIGLU) return run_lds_t<EPI_SWIGLU, BM, BN, WM, WN, STAGES, true>(P, s);
    return run_lds_t<EPI_QKV_ROPE, BM, BN, WM, WN, STAGES, true>(P, s);
  }
  if (P.epi == EPI_RESID) return run_lds_t<EPI_RESID, BM, BN, WM, WN, STAGES, false>(P, s);
  if (P.epi == EPI_SWIGLU) return run_lds_t<EPI_SWIGLU, BM, BN, WM, WN, STAGES, false>(P, s);
  return run_lds_t<EPI_QKV_ROPE, BM, BN, WM, WN, STAGES, false>(P, s);
}

// the shapes of the LDS kernel: whole 64-deep k-tiles and the staged epilogue
// (8 consecutive outputs per lane)
static bool lds_shape(int epi, int K, int nlog, int npairs, int dh) {
  if (K % 64 != 0) return false;
  return epi == EPI_RESID ? nlog % 8 == 0 : npairs % 8 == 0 && (epi == EPI_SWIGLU || dh % 16 == 0);
}

// Tile and K split of a product.  One workgroup runs on a compute unit at a
// time, so a launch takes ceil(tiles * splits / 256) rounds, each of K / splits
// steps whose time depends on the tile alone (ns per k with every unit busy,
// measured at M = 300 .. 3000, K = 3584 .. 18944: 256x256 25.5, 128x256 15.0,
// 256x128 14.7, 128x128 9.8: the larger the tile, the fewer operand bytes per
// product).  Splits add a launch (8 us) and their sums' way through memory: 4 bytes
// per sum written at 3.4 TB/s and read at 3.7, or by one workgroup per tile at 55
// GB/s each where that takes longer (few large tiles).  Over 25 row counts from 66
// to 8192 of the 7B, 28/4 and d = 1536 layers (300 products) the plan takes 0.8%
// longer than the best tile and split measured on average, 14% at worst.  In us
// under the profiler, against the fixed rule before: 600 x 12288 x 4096 113 -> 78
// (240 tiles of 128x256, not 144 of 256x256), 600 x 4096 x 11008 119 -> 83 (80
// tiles in 3 parts, not 160 whole ones of 128x128), 3001 x 37888 x 3584 930 -> 788
// (7 rounds of 256x256, not one of them and 12 of 256x128), 3001 x 3584 x 18944
// 664 -> 454 (168 tiles in 3 parts).
// Where 256x256 tiles would fill one round and little of a second, one round of
// them followed by 256x128 tiles for the other columns is another plan, taken if
// it is 4% better (two launches: 3% better by this count was 3% slower).  7B
// gate/up product at 1000 rows (344 tiles of 256x256): 161 us, one launch 173.
// A product of more than 1024 workgroups is not split (the last round is a small
// share of four, and sums of 256 MiB a bound on the scratch).
struct GemmPlan {
  int tile, splits;
  size_t bytes;  // scratch of the splits' sums
  int first;     // columns that a first launch of 256x256 tiles takes
};
static GemmPlan gemm_plan(int M, int nlog, int K, size_t part_bytes) {
  static const struct {
    int bm, bn;
    double ns;
  } T[4] = {{256, 256, 25.5}, {128, 256, 15.0}, {256, 128, 14.7}, {128, 128, 9.8}};
  GemmPlan best = {0, 1, 0, 0};
  double cost = 0.0;
  for (int t = 0; t < 4; ++t) {
    const long long tiles = (long long)cdiv(M, T[t].bm) * cdiv(nlog, T[t].bn);
    for (int sp = 1; sp <= 8; ++sp) {
      const size_t bytes = sp > 1 ? (size_t)tiles * sp * T[t].bm * T[t].bn * sizeof(float) : 0;
      if (sp > 1 && (K / 64 < 8 * sp || tiles * sp > 1024 || bytes > part_bytes)) break;
      double c = (double)((tiles * sp + 255) / 256) * K / sp * T[t].ns * 1e-3;
      if (sp > 1)
        c += 8.0 + (double)bytes / 3.4e6 +
             std::max((double)bytes / 3.7e6, (double)((tiles + 255) / 256) * sp * T[t].bm * T[t].bn * 4 / 55e3);
      if ((t == 0 && sp == 1) || c < cost) {
        cost = c;
        best = {t, sp, bytes, 0};
      }
    }
  }
  const int mt = cdiv(M, 256), full = 256 / mt * 256;  // columns of one round of 256x256 tiles
  if (full > 0 && full < nlog) {
    const long long rest = (long long)mt * cdiv(nlog - full, 128);
    const double c = K * T[0].ns * 1e-3 + (double)((rest + 255) / 256) * K * T[2].ns * 1e-3;
    if (c < 0.96 * cost) best = {2, 1, 0, full};
  }
  return best;
}

size_t gemm_scratch_bytes(int dtype, const GemmArgs& g) {
  if (dtype != SAS_BF16 || g.M <= 0) return 0;
  const int npairs = g.epi == EPI_SWIGLU ? g.N : (g.epi == EPI_QKV_ROPE ? g.N / 2 : 0);
  const int nlog = g.epi == EPI_RESID ? g.N : (npairs + 31) / 32 * 64;
  if (!lds_shape(g.epi, g.K, nlog, npairs, g.head_dim)) return 0;
  // a plan depends on the rows' number of 128-row tiles; past 512 tiles of 256x256 none is split
  size_t most = 0;
  for (int i = 1; i <= cdiv(g.M, 128) && (long long)cdiv(i, 2) * cdiv(nlog, 256) <= 512; ++i)
    most = std::max(most, gemm_plan(i * 128, nlog, g.K, SIZE_MAX).bytes);
  return most;
}

static bool attrs_done = false;

bool gemm_fills_cache(int dtype, const GemmArgs& g) {
  // the staged epilogue of the LDS kernels (every bf16 launch with K % 64 == 0 and the
  // fast epilogue shape below), with rows at their sequence positions
  return dtype == SAS_BF16 && g.epi == EPI_QKV_ROPE && g.K % 64 == 0 && !g.row_pos && g.seq_len > 0 &&
         (g.N / 2) % 8 == 0 && g.head_dim % 16 == 0;
}

hipError_t launch_gemm(int dtype, const GemmArgs& g, hipStream_t s) {
  if (g.prefill_cache && !gemm_fills_cache(dtype, g)) return hipErrorInvalidValue;
  if (g.M <= 0) return hipSuccess;
  // pair epilogues: SWIGLU has F pairs, QKV has (H + 2 Hkv) dh / 2 pairs
  const int npairs = g.epi == EPI_SWIGLU ? g.N : (g.epi == EPI_QKV_ROPE ? g.N / 2 : 0);
  const bool plain = g.epi == EPI_RESID || g.epi == EPI_F32OUT;
  const int nlog = plain ? g.N : (npairs + 31) / 32 * 64;
  if (dtype == SAS_F32) {
    if (g.K % 4 != 0) return hipErrorInvalidValue;  // 16-byte operand loads (d and d_ff are multiples of 8)
    const GemmF32 F = {g.M, g.K, plain ? g.N : nlog, npairs, (const float*)g.A, (const float*)g.B0,
                       (const float*)g.B1, (const float*)g.B2, (const float*)g.resid, (float*)g.out,
                       (float*)g.out1, (float*)g.out2, g.n_heads, g.n_kv_heads, g.head_dim, g.seq_len, g.rope,
                       g.row_pos};
    switch (g.epi) {
      case EPI_QKV_ROPE: return run_f32<EPI_QKV_ROPE>(F, s);
      case EPI_SWIGLU: return run_f32<EPI_SWIGLU>(F, s);
      case EPI_F32OUT: return run_f32<EPI_F32OUT>(F, s);
      default: return run_f32<EPI_RESID>(F, s);
    }
  }
  if (!attrs_done) {
    (void)hipFuncSetAttribute((const void*)gemm_bf16_kernel<256, 256, 2, 4>,
                        hipFuncAttributeMaxDynamicSharedMemorySize, 2 * (256 + 256) * BK * 2);
    (void)hipFuncSetAttribute((const void*)gemm_bf16_kernel<128, 128, 2, 2>,
                        hipFuncAttributeMaxDynamicSharedMemorySize, 2 * (128 + 128) * BK * 2);
    attrs_done = true;
  }
  GemmParams P;
  P.epi = g.epi;
  P.M = g.M;
  P.K = g.K;
  P.N = nlog;
  P.npairs = npairs;
  P.A = (const bf16_t*)g.A;
  P.B0 = (const bf16_t*)g.B0;
  P.B1 = (const bf16_t*)g.B1;
  P.B2 = (const bf16_t*)g.B2;
  P.resid = (const bf16_t*)g.resid;
  P.out = (bf16_t*)g.out;
  P.out1 = (bf16_t*)g.out1;
  P.out2 = (bf16_t*)g.out2;
  P.H = g.n_heads;
  P.Hkv = g.n_kv_heads;
  P.dh = g.head_dim;
  // tile order: groups of 8 M tiles; the long-K residual product (the MLP's
  // down projection, K > 2N) runs faster with groups of 2 (measured 4-5%)
  P.group_m = (g.epi == EPI_RESID && g.K > 2 * nlog) ? 2 : 8;
  P.splits = 1;
  P.part = g.part;
  P.n_off = 0;
  P.n_cnt = nlog;
  P.seq_len = g.seq_len;
  P.rope = g.rope;
  P.row_pos = g.row_pos;
  P.k_pages = g.prefill_cache ? (bf16_t*)g.prefill_cache->k_pages : nullptr;
  P.v_pages = g.prefill_cache ? (bf16_t*)g.prefill_cache->v_pages : nullptr;
  P.geom = g.prefill_cache ? PageGeom{g.prefill_cache->block_table, g.prefill_cache->num_pages,
                                      g.prefill_cache->page_size, g.prefill_cache->max_pages}
                           : PageGeom{nullptr, 0, 1, 0};
  const long big_tiles = (long)((g.M + 255) / 256) * ((nlog + 255) / 256);
  if (g.epi == EPI_F32OUT) return hipErrorInvalidValue;  // bf16 fp32-output products go through gemv
  if (lds_shape(g.epi, g.K, nlog, npairs, g.head_dim)) {
    const GemmPlan plan = gemm_plan(g.M, nlog, g.K, g.part ? g.part_bytes : 0);
    P.splits = plan.splits;
    if (plan.first > 0) {
      g_launch_events = LaunchEvents{nullptr, nullptr, 0};  // two launches: timed around both
      P.n_cnt = plan.first;
      const hipError_t e = run_lds<256, 256, 2, 4, 2>(P, s);
      if (e != hipSuccess) return e;
      P.n_off = plan.first;
      P.n_cnt = nlog - plan.first;
    }
    switch (plan.tile) {
      case 0: return run_lds<256, 256, 2, 4, 2>(P, s);
      case 1: return run_lds<128, 256, 2, 4, 3>(P, s);
      case 2: return run_lds<256, 128, 4, 2, 3>(P, s);
      default: return run_lds<128, 128, 4, 2, 4>(P, s);
    }
  }
  if (big_tiles >= 256) return run_bf16<256, 256, 2, 4>(P, s);
  return run_bf16<128, 128, 2, 2>(P, s);
}

}  // namespace sas

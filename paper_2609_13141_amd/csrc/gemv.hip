// Skinny GEMM: out = A[M, K] W^T with M <= GEMV_MAX_ROWS rows (the batch of new
// tokens of a decode step, a few prompt tokens), bound by streaming W from HBM.
//
// One workgroup per 16 output columns (several such groups for more than 16
// rows); its waves split K into contiguous ranges of 32-wide steps.
// v_mfma_f32_16x16x32_bf16 takes A (activations, 16 rows, rows >= M zero) and
// W^T (16 columns).  The MFMA only needs A and B to
// enumerate k the same way, so the k slice of a step is chosen to make each
// load instruction contiguous: lane l reads the 16 bytes at k = 32 st +
// 8 (l/16) of row l % 16, so that with row-major weights one instruction
// covers 16 rows x 64 contiguous bytes, and with the packed decode layout
// (sas_pack_decode_weights) 1 KB of consecutive bytes.  Partial sums of the
// waves are added in LDS.
//
// Column groups of the pair epilogues hold 8 first-half and 8 second-half
// columns (RoPE: i and i + dh/2 of a head; SwiGLU: gate f and up f); a lane's
// partner is lane ^ 8 after the reduction.
#include "common.h"
#include "kernels.h"

namespace sas {

struct GemvParams {
  int epi, M, K, N, npairs;
  const bf16_t* A;
  const bf16_t* B0;
  const bf16_t* B1;
  const bf16_t* B2;
  const bf16_t* resid;
  void* out;
  bf16_t* out1;
  bf16_t* out2;
  int H, Hkv, dh;
  const float2* rope;  // rotary table: per row [M, dh/2], or of positions 0 .. seq_len - 1
  int seq_len;         // > 0: row r is position r % seq_len of sequence r / seq_len (prefill); 0: one row per sequence
  const int32_t* pos;  // [M] positions (cache append, seq_len 0)
  const bf16_t* packed;  // the weights in the packed decode layout, or NULL
  // cache append (QKV epilogue): K/V rows into their pages, and the summary of
  // a block completed by this position (NULL k_pages: no append; NULL
  // k_summary: no summaries)
  void* k_pages;
  void* v_pages;
  void* k_summary;
  PageGeom geom;
  int B, max_blocks;
};

// weight row of local column c (0..15) of column group gi (EPI < 0: the
// epilogue kind is read from P at run time)
template <int EPI = -1>
__device__ __forceinline__ const bf16_t* gemv_row(const GemvParams& P, int gi, int c, bool& valid) {
  const int epi = EPI >= 0 ? EPI : P.epi;
  if (epi == EPI_RESID || epi == EPI_F32OUT) {
    const int col = gi * 16 + c;
    valid = col < P.N;
    return P.B0 + (size_t)min(col, P.N - 1) * P.K;
  }
  const int p = gi * 8 + (c & 7), half = c >> 3;
  valid = p < P.npairs;
  const int pc = min(p, P.npairs - 1);
  if (epi == EPI_SWIGLU) return (half ? P.B1 : P.B0) + (size_t)pc * P.K;
  const int hh = P.dh >> 1;
  const int hd = pc / hh, ir = pc % hh;
  int cc = hd * P.dh + ir + half * hh;
  if (cc < P.H * P.dh) return P.B0 + (size_t)cc * P.K;
  cc -= P.H * P.dh;
  if (cc < P.Hkv * P.dh) return P.B1 + (size_t)cc * P.K;
  return P.B2 + (size_t)(cc - P.Hkv * P.dh) * P.K;
}

// Epilogue inputs of a lane for column group gi (pair gi * 8 + c % 8, rows
// r0 + 4 kg + v): the QKV epilogue's rotary entries, positions and page ids, the
// RESID epilogue's residual values.  They are loaded with the weight stream and
// left as they arrive until the epilogue: a value converted or tested earlier
// makes its wave wait for memory before its stream begins (the page id depends
// on the position, so it is read after the first batch of weights).
struct GemvPre {
  float2 cs[4];
  int ps[4], page[4];
  uint32_t res[4];
};

template <int EPI, bool SEQ>
__device__ __forceinline__ void gemv_prepare(const GemvParams& P, int gi, int c, int kg, int r0, GemvPre& e) {
  if constexpr (EPI == EPI_RESID) {
    const int col = min(gi * 16 + c, P.N - 1);
#pragma unroll
    for (int v = 0; v < 4; ++v) e.res[v] = P.resid[(size_t)min(r0 + 4 * kg + v, P.M - 1) * P.N + col];
  }
  if constexpr (EPI == EPI_QKV_ROPE) {
    const int hh = P.dh >> 1, ir = min(gi * 8 + (c & 7), P.npairs - 1) % hh;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = min(r0 + 4 * kg + v, P.M - 1);
      const int rr = SEQ ? row % P.seq_len : row;  // row of the rotary table
      e.cs[v] = P.rope[(size_t)rr * hh + ir];
      e.ps[v] = rr;
      if (!SEQ && P.k_pages) e.ps[v] = P.pos[row];
    }
  }
}

// the page ids (from a clamped place of the table; the epilogue checks the position)
template <int EPI, bool SEQ>
__device__ __forceinline__ void gemv_prepare_pages(const GemvParams& P, int kg, int r0, GemvPre& e) {
  if constexpr (EPI == EPI_QKV_ROPE) {
    if (P.k_pages) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = min(r0 + 4 * kg + v, P.M - 1), seq = SEQ ? row / P.seq_len : row;
        const int pi = min(max(e.ps[v], 0) / P.geom.ps, P.geom.max_pages - 1);
        e.page[v] = P.geom.table[(size_t)seq * P.geom.max_pages + pi];
      }
    }
  }
}

// The fused epilogue of column group gi; `tot` holds column c, rows r0 + 4 kg + v.
template <int EPI = -1>
__device__ __forceinline__ void gemv_epilogue(const GemvParams& P, int gi, int c, int kg, int r0,
                                              const floatx4_t& tot, const GemvPre& e) {
  const int epi = EPI >= 0 ? EPI : P.epi;
  bool cvalid;
  (void)gemv_row<EPI>(P, gi, c, cvalid);
  if (epi == EPI_RESID || epi == EPI_F32OUT) {
    const int col = gi * 16 + c;
    if (!cvalid) return;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = r0 + 4 * kg + v;
      if (row >= P.M) continue;
      const size_t o = (size_t)row * P.N + col;
      if (epi == EPI_RESID) {
        uint32_t r = e.res[v];
        asm("" : "+v"(r));  // keeps the conversion (and the wait for the load) here
        ((bf16_t*)P.out)[o] = f32_to_bf16(tot[v] + __uint_as_float(r << 16));
      } else
        ((float*)P.out)[o] = tot[v];
    }
    return;
  }
  const int hh = P.dh >> 1;
  float partner[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) partner[v] = __shfl_xor(tot[v], 8, 64);
  if (c >= 8 || !cvalid) return;
  const int p = gi * 8 + c;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int row = r0 + 4 * kg + v;
    if (row >= P.M) continue;
    float x1 = tot[v], x2 = partner[v];
    if (epi == EPI_SWIGLU) {
      ((bf16_t*)P.out)[(size_t)row * P.npairs + p] = f32_to_bf16(x1 * __builtin_amdgcn_rcpf(1.0f + __expf(-x1)) * x2);
      continue;
    }
    const int hd = p / hh, ir = p % hh;
    bf16_t* dst;
    if (hd < P.H) dst = (bf16_t*)P.out + ((size_t)row * P.H + hd) * P.dh;
    else if (hd < P.H + P.Hkv) dst = P.out1 + ((size_t)row * P.Hkv + (hd - P.H)) * P.dh;
    else dst = P.out2 + ((size_t)row * P.Hkv + (hd - P.H - P.Hkv)) * P.dh;
    if (hd < P.H + P.Hkv) {
      const float2 cs = e.cs[v];
      const float o1 = x1 * cs.x - x2 * cs.y;
      const float o2 = x2 * cs.x + x1 * cs.y;
      x1 = o1;
      x2 = o2;
    }
    const bf16_t b1 = f32_to_bf16(x1), b2 = f32_to_bf16(x2);
    dst[ir] = b1;
    dst[ir + hh] = b2;
    if (P.k_pages && hd >= P.H) {
      // cache append of this row's K or V, dimensions ir and ir + dh/2
      const bool isk = hd < P.H + P.Hkv;
      const int g = isk ? hd - P.H : hd - P.H - P.Hkv;
      const int ps = e.ps[v], page = e.page[v];
      if (ps < 0 || ps / P.geom.ps >= P.geom.max_pages || page < 0 || page >= P.geom.num_pages) continue;
      const long long off = (((long long)page * P.Hkv + g) * P.geom.ps + ps % P.geom.ps) * P.dh;
      bf16_t* pg = (bf16_t*)(isk ? P.k_pages : P.v_pages) + off;
      pg[ir] = b1;
      pg[ir + hh] = b2;
      if (!isk || !P.k_summary || (ps + 1) % P.B != 0 || ps / P.B >= P.max_blocks) continue;
      // this position completes block m: its summary in these two dimensions
      // (fp64 sum over ascending positions, the new key last).  Positions go
      // in chunks of SUMC: the chunk's page ids, then its keys, are loaded
      // unconditionally from clamped addresses and masked afterwards, so each
      // chunk costs two memory round trips instead of two per position.
      constexpr int SUMC = 16;
      const int m = ps / P.B;
      const bf16_t* kp = (const bf16_t*)P.k_pages;
      const int32_t* trow = P.geom.table + (size_t)row * P.geom.max_pages;
      double s1 = 0.0, s2 = 0.0;
      for (int q0 = m * P.B; q0 < ps; q0 += SUMC) {
        long long o[SUMC];
#pragma unroll
        for (int j = 0; j < SUMC; ++j) {
          const int q = q0 + j, pi = q / P.geom.ps;
          const int page = trow[min(pi, P.geom.max_pages - 1)];
          const bool ok = q < ps && pi < P.geom.max_pages && page >= 0 && page < P.geom.num_pages;
          o[j] = ok ? (((long long)page * P.Hkv + g) * P.geom.ps + (q % P.geom.ps)) * P.dh : -1;
        }
        float k1[SUMC], k2[SUMC];
#pragma unroll
        for (int j = 0; j < SUMC; ++j) {
          const long long oc = o[j] >= 0 ? o[j] : 0;
          const float a = bf16_to_f32(kp[oc + ir]), b = bf16_to_f32(kp[oc + ir + hh]);
          k1[j] = o[j] >= 0 ? a : 0.f;  // a position without a page adds zero
          k2[j] = o[j] >= 0 ? b : 0.f;
        }
#pragma unroll
        for (int j = 0; j < SUMC; ++j) {
          if (q0 + j < ps) {
            s1 += (double)k1[j];
            s2 += (double)k2[j];
          }
        }
      }
      s1 += (double)bf16_to_f32(b1);
      s2 += (double)bf16_to_f32(b2);
      bf16_t* sm = (bf16_t*)P.k_summary + (((size_t)row * P.Hkv + g) * P.max_blocks + m) * P.dh;
      sm[ir] = Act<bf16_t>::from_f64(s1 / (double)P.B);
      sm[ir + hh] = Act<bf16_t>::from_f64(s2 / (double)P.B);
    }
  }
}

// The packed decode layout: the 16 columns x 32 k of step st of column group
// gi form one 1-KB block at element ((gi * K/32 + st) * 64 + l) * 8 for lane
// l, holding row(gi, l % 16)[st * 32 + (l / 16) * 8 ..+8]: the fragment lane l
// of the 16x16x32 MFMA takes, so a wave's load is 1 KB of consecutive bytes.
__global__ void gemv_pack_kernel(GemvParams P, bf16_t* __restrict__ out, size_t chunks) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;  // one 16-byte chunk
  if (idx >= chunks) return;
  const int nsteps = P.K / 32;
  const int l = (int)(idx % 64);
  const size_t r = idx / 64;
  const int st = (int)(r % nsteps), gi = (int)(r / nsteps);
  bool valid;
  const bf16_t* row = gemv_row(P, gi, l & 15, valid);  // clamped: columns past the end repeat the last row
  *(uint4*)(out + idx * 8) = *(const uint4*)(row + st * 32 + (l >> 4) * 8);
}

// One workgroup per CG column groups of 16, its NW waves splitting K, all MT
// tiles of 16 rows in it.  Lane (c, kg) multiplies step st's weights --
// row-major: row(gi, c)[st * 32 + kg * 8 ..]; packed: its 16 bytes of block
// (gi, st) -- by the activation rows' elements st * 32 + kg * 8 ..; both
// layouts give the same products in the same order.  Every workgroup reads
// all of A (from L2), so with more rows it takes more columns: CG and NW are
// chosen by the launch.  SEQ: rows are positions of sequences (prefill).
// 32 rows of the 28/4 layer (K = 3584, d_ff = 18944, packed): QKV 18, O 14,
// gate/up 61, down 51 us; tiled launches of 36, 28, 148 and 28 workgroups took
// 35, 49, 94 and 140 us.
template <int NW, int EPI, int MT, int CG, bool SEQ, bool PK>
__global__ void __launch_bounds__(NW * 64) gemv_kernel(GemvParams P) {
  constexpr int NT = MT * CG;                // 16 x 16 output tiles
  constexpr int TPW = (NT + NW - 1) / NW;    // ... finished per wave
  constexpr int U = MT + CG <= 3 ? 8 : (MT + CG <= 6 ? 4 : 2);  // steps loaded together (64 to 96 registers)
  // the waves' sums meet here: all at once, or (more than 32 KB of them, so that
  // several workgroups fit a compute unit) the upper half of the waves first
  constexpr int PW = NW * NT > 32 ? NW / 2 : NW;
  __shared__ floatx4_t part[PW][NT][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, kg = lane >> 4;
  const int groups = (EPI == EPI_RESID || EPI == EPI_F32OUT) ? (P.N + 15) / 16 : (P.npairs + 7) / 8;
  const bf16_t* wr[CG];
  constexpr int WSTEP = PK ? 512 : 32;  // elements between a lane's pieces of two steps
#pragma unroll
  for (int j = 0; j < CG; ++j) {
    const int gi = CG == 1 ? (int)blockIdx.x : min((int)blockIdx.x * CG + j, groups - 1);
    bool cvalid;
    if constexpr (PK) wr[j] = P.packed + ((size_t)gi * (P.K / 32) * 64 + lane) * 8;
    else wr[j] = gemv_row<EPI>(P, gi, c, cvalid) + kg * 8;
  }
  const bf16_t* ar[MT];
  bool avalid[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    avalid[i] = 16 * i + c < P.M;
    ar[i] = P.A + (size_t)min(16 * i + c, P.M - 1) * P.K + kg * 8;
  }
  // tile of this wave's q-th epilogue, and its column group (past the last: nothing to do)
  auto tile_of = [&](int q) { return q * NW + wave; };
  auto group_of = [&](int tile) { return (int)blockIdx.x * CG + tile % CG; };
  GemvPre pre;
  const bool early = TPW == 1 && (NT == NW || wave < NT);  // one tile per wave: its inputs come with the stream
  if (early) gemv_prepare<EPI, SEQ>(P, min(group_of(wave), groups - 1), c, kg, 16 * (wave / CG), pre);

  // this wave's range of 32-wide k steps
  const int steps = P.K / 32;
  const int per = (steps + NW - 1) / NW;
  const int s0 = wave * per, s1 = min(steps, s0 + per);

  floatx4_t acc[MT][CG];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < CG; ++j) acc[i][j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  // the pointers move with the steps, so that a load's address is one of them and a constant
#pragma unroll
  for (int j = 0; j < CG; ++j) wr[j] += (size_t)s0 * WSTEP;
#pragma unroll
  for (int i = 0; i < MT; ++i) ar[i] += s0 * 32;
  int st = s0;
  auto batch = [&]() {
    uint4 w[U][CG], a[U][MT];
#pragma unroll
    for (int q = 0; q < U; ++q) {
#pragma unroll
      for (int j = 0; j < CG; ++j) w[q][j] = *(const uint4*)(wr[j] + q * WSTEP);
#pragma unroll
      for (int i = 0; i < MT; ++i) a[q][i] = *(const uint4*)(ar[i] + q * 32);
    }
#pragma unroll
    for (int q = 0; q < U; ++q)
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        if (!avalid[i]) a[q][i] = make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int j = 0; j < CG; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(bf16x8_t*)&a[q][i], *(bf16x8_t*)&w[q][j], acc[i][j],
                                                              0, 0, 0);
      }
#pragma unroll
    for (int j = 0; j < CG; ++j) wr[j] += U * WSTEP;
#pragma unroll
    for (int i = 0; i < MT; ++i) ar[i] += U * 32;
    st += U;
  };
  if (st + U <= s1) batch();
  if (early) gemv_prepare_pages<EPI, SEQ>(P, kg, 16 * (wave / CG), pre);
  while (st + U <= s1) batch();
  for (; st < s1; ++st) {
    uint4 w[CG];
#pragma unroll
    for (int j = 0; j < CG; ++j) w[j] = *(const uint4*)wr[j];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      uint4 a = avalid[i] ? *(const uint4*)ar[i] : make_uint4(0, 0, 0, 0);
#pragma unroll
      for (int j = 0; j < CG; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(bf16x8_t*)&a, *(bf16x8_t*)&w[j], acc[i][j], 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < CG; ++j) wr[j] += WSTEP;
#pragma unroll
    for (int i = 0; i < MT; ++i) ar[i] += 32;
  }
  if constexpr (PW < NW) {
    if (wave >= PW) {
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < CG; ++j) part[wave - PW][i * CG + j][lane] = acc[i][j];
    }
    __syncthreads();
    if (wave < PW) {
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < CG; ++j) {
          const floatx4_t p = part[wave][i * CG + j][lane];
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[i][j][v] += p[v];
          part[wave][i * CG + j][lane] = acc[i][j];  // read and written by this lane only
        }
    }
  } else {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < CG; ++j) part[wave][i * CG + j][lane] = acc[i][j];
  }
  __syncthreads();
  for (int q = 0; q < TPW; ++q) {
    const int tile = tile_of(q), gi = group_of(tile), r0 = 16 * (tile / CG);
    if (tile < NT && gi < groups) {
      if (TPW > 1) {
        gemv_prepare<EPI, SEQ>(P, gi, c, kg, r0, pre);
        gemv_prepare_pages<EPI, SEQ>(P, kg, r0, pre);
      }
      floatx4_t tot = part[0][tile][lane];
#pragma unroll
      for (int wv = 1; wv < PW; ++wv) {
        const floatx4_t p = part[wv][tile][lane];
#pragma unroll
        for (int v = 0; v < 4; ++v) tot[v] += p[v];
      }
      gemv_epilogue<EPI>(P, gi, c, kg, r0, tot, pre);
    }
  }
}

// 4 waves per group for up to 16 rows: as fast as or faster than 8 or 16 waves
// at the decode shapes (measured: QKV 22.6 vs 23.8 us, down 21.9 vs 22.7 us, O equal)
template <int EPI, bool SEQ, bool PK>
static hipError_t run_gemv_t(const GemvParams& P, int groups, hipStream_t s) {
  const int mt = cdiv(P.M, 16);
  if (mt == 1) return launch_ext(gemv_kernel<4, EPI, 1, 1, SEQ, PK>, dim3(groups), dim3(256), 0, s, P);
  if constexpr (EPI == EPI_F32OUT) {
    return hipErrorInvalidValue;
  } else {
    // columns per workgroup: the busiest compute unit reads (16 CG columns + 16 MT
    // rows) x K values per workgroup it runs; CG with the least of that
    int cg = 1;
    long best = 0;
    for (int t = 1; t <= 4; t *= 2) {
      const long cost = (long)cdiv(cdiv(groups, t), 256) * (t + mt);
      if (t == 1 || cost < best) {
        best = cost;
        cg = t;
      }
    }
    // waves per workgroup, measured (us, 4 / 8 waves): CG 4 with a workgroup per
    // compute unit 62.6 / 68.7 (gate/up, 64 rows), with fewer 57.5 / 43.7 (QKV);
    // CG 2 27.6 / 30.0 (QKV, 17 rows) but 47.0 / 41.6 (48 rows); CG 1 33.3 / 27.2
    // (down, 17 rows), 38.0 / 44.1 (48), 56.4 / 55.2 (64)
    const dim3 grid(cdiv(groups, cg));
#define GEMV_NW(NW, MT, CG) launch_ext(gemv_kernel<NW, EPI, MT, CG, SEQ, PK>, grid, dim3(NW * 64), 0, s, P)
#define GEMV_MT(MT)                                 \
  (cg == 1 ? GEMV_NW((MT == 3 ? 4 : 8), MT, 1)      \
   : cg == 2 ? GEMV_NW((MT == 2 ? 4 : 8), MT, 2)    \
   : grid.x >= 256 ? GEMV_NW(4, MT, 4) : GEMV_NW(8, MT, 4))
    if (mt == 2) return GEMV_MT(2);
    if (mt == 3) return GEMV_MT(3);
    return GEMV_MT(4);
#undef GEMV_MT
#undef GEMV_NW
  }
}

template <int EPI>
static hipError_t run_gemv(const GemvParams& P, int groups, hipStream_t s) {
  if constexpr (EPI == EPI_F32OUT) {
    return run_gemv_t<EPI, false, false>(P, groups, s);
  } else {
    if constexpr (EPI == EPI_QKV_ROPE)
      if (P.seq_len > 0) return run_gemv_t<EPI, true, false>(P, groups, s);
    return P.packed ? run_gemv_t<EPI, false, true>(P, groups, s) : run_gemv_t<EPI, false, false>(P, groups, s);
  }
}

hipError_t launch_gemv(const GemmArgs& g, hipStream_t s) {
  if (g.M <= 0) return hipSuccess;
  if (g.M > GEMV_MAX_ROWS || g.K % 128 != 0) return hipErrorInvalidValue;
  GemvParams P;
  P.epi = g.epi;
  P.M = g.M;
  P.K = g.K;
  P.N = g.N;
  P.npairs = g.epi == EPI_SWIGLU ? g.N : (g.epi == EPI_QKV_ROPE ? g.N / 2 : 0);
  P.A = (const bf16_t*)g.A;
  P.B0 = (const bf16_t*)g.B0;
  P.B1 = (const bf16_t*)g.B1;
  P.B2 = (const bf16_t*)g.B2;
  P.resid = (const bf16_t*)g.resid;
  P.out = g.out;
  P.out1 = (bf16_t*)g.out1;
  P.out2 = (bf16_t*)g.out2;
  P.H = g.n_heads;
  P.Hkv = g.n_kv_heads;
  P.dh = g.head_dim;
  P.rope = g.rope;
  P.seq_len = g.epi != EPI_QKV_ROPE || g.append || g.row_pos ? 0 : g.seq_len;
  P.pos = g.row_pos;
  P.packed = (const bf16_t*)g.packed;
  P.k_pages = nullptr;
  P.v_pages = nullptr;
  P.k_summary = nullptr;
  P.geom = PageGeom{nullptr, 0, 1, 0};
  P.B = 1;
  P.max_blocks = 0;
  if (g.packed && (g.epi == EPI_F32OUT || P.seq_len > 0)) return hipErrorInvalidValue;  // row-major only
  if (g.epi == EPI_QKV_ROPE) {
    if (!g.rope) return hipErrorInvalidValue;
    if (g.append) {
      if (!g.row_pos) return hipErrorInvalidValue;
      const DecodeArgs& c = *g.append;
      P.k_pages = c.k_pages;
      P.v_pages = c.v_pages;
      P.k_summary = c.k_summary;
      P.geom = PageGeom{c.block_table, c.num_pages, c.page_size, c.max_pages};
      P.B = c.B;
      P.max_blocks = c.max_blocks;
    } else if (g.prefill_cache) {
      const DecodeArgs& c = *g.prefill_cache;
      P.k_pages = c.k_pages;
      P.v_pages = c.v_pages;
      P.geom = PageGeom{c.block_table, c.num_pages, c.page_size, c.max_pages};
    }
  }
  const int groups = (g.epi == EPI_RESID || g.epi == EPI_F32OUT) ? (g.N + 15) / 16 : (P.npairs + 7) / 8;
  switch (g.epi) {
    case EPI_QKV_ROPE: return run_gemv<EPI_QKV_ROPE>(P, groups, s);
    case EPI_SWIGLU: return run_gemv<EPI_SWIGLU>(P, groups, s);
    case EPI_F32OUT: return run_gemv<EPI_F32OUT>(P, groups, s);
    default: return run_gemv<EPI_RESID>(P, groups, s);
  }
}

static GemvParams pack_params(const GemmArgs& g) {
  GemvParams P = {};
  P.epi = g.epi;
  P.M = 1;
  P.K = g.K;
  P.N = g.N;
  P.npairs = g.epi == EPI_SWIGLU ? g.N : (g.epi == EPI_QKV_ROPE ? g.N / 2 : 0);
  P.B0 = (const bf16_t*)g.B0;
  P.B1 = (const bf16_t*)g.B1;
  P.B2 = (const bf16_t*)g.B2;
  P.H = g.n_heads;
  P.Hkv = g.n_kv_heads;
  P.dh = g.head_dim;
  return P;
}

size_t gemv_packed_elems(const GemmArgs& g) {
  const GemvParams P = pack_params(g);
  const size_t groups = (P.epi == EPI_RESID || P.epi == EPI_F32OUT) ? (P.N + 15) / 16 : (P.npairs + 7) / 8;
  return groups * (size_t)(g.K / 32) * 512;
}

hipError_t launch_gemv_pack(const GemmArgs& g, void* out, hipStream_t s) {
  if (g.K % 128 != 0 || g.N <= 0) return hipErrorInvalidValue;
  const GemvParams P = pack_params(g);
  const size_t chunks = gemv_packed_elems(g) / 8;
  gemv_pack_kernel<<<(unsigned)((chunks + 255) / 256), 256, 0, s>>>(P, (bf16_t*)out, chunks);
  return hipGetLastError();
}

}  // namespace sas

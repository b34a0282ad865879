// SAS selector on the GPU: block summaries, gate query, exact scores,
// normalized log gate (Eq. normalized_log_gate) and Top-K selection
// (Eq. selected_context), one lane per query row.
//
// Exactness: summaries and gate queries are fp64 sums of activation-dtype
// values in ascending index order, rounded once to the activation dtype;
// scores are sequential fp64 FMA chains over ascending j (each product of two
// bf16/fp32 values is exact in fp64, so FMA equals multiply-then-add).  The
// ranking key is the exact score with ties going to the lower block index,
// so the selected indices are an integer function of the input bits.
#include <float.h>

#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace sas {

// ---------------------------------------------------------------------------
// Block summaries: thread per (b, m, g, 8-dim chunk), the chunk fastest and
// then the KV head, so that a load instruction reads a contiguous stretch of
// one key row (Hkv * dh values per position); the B keys of the block are
// read 16 at a time (independent 16-byte loads) and summed per dimension in
// fp64 in ascending token order.
template <typename T>
__global__ void summaries_kernel(const T* __restrict__ K, T* __restrict__ out, int n, int Hkv, int dh,
                                 int B, int NB, size_t total) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  const int nc = dh / 8;
  const int c8 = (int)(idx % nc);
  size_t r = idx / nc;
  const int g = (int)(r % Hkv);
  r /= Hkv;
  const int m = (int)(r % NB);
  const int bi = (int)(r / NB);
  T* o = out + (((size_t)bi * Hkv + g) * NB + m) * dh + c8 * 8;
  if ((m + 1) * B > n) {  // incomplete block: no summary
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = Act<T>::from_f32(0.f);
    return;
  }
  const T* p = K + (((size_t)bi * n + (size_t)m * B) * Hkv + g) * dh + c8 * 8;
  const size_t stride = (size_t)Hkv * dh;
  double acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.0;
  for (int i0 = 0; i0 < B; i0 += 16) {  // B is a multiple of 16
    Vec8<T> v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q].load(p + (size_t)(i0 + q) * stride);
#pragma unroll
    for (int q = 0; q < 16; ++q)
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += (double)v[q].get(e);
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = Act<T>::from_f64(acc[e] / (double)B);
}

// Per-group projection of rows: out[b, g, r, k] = rho(sum_j W[g, k, j] v[r, j])
// with v the rounded fp64 sum of `nh` consecutive heads of the source row
// (in + b sb + g sg + r sr, nh = 1: the row itself), which is also written to
// `plain` [b, Hkv, rows, DH] when that is given.
//
// Bound: fp64 matrix rate (2 rows dh^2 flops per group).  The products run on
// v_mfma_f64_16x16x4_f64, which adds its four products to the accumulator one
// after the other in ascending k with one rounding each (checked bit for bit
// against an fma chain), so 32 of them in order are the chain over ascending
// j.  A workgroup keeps W of its group in LDS for `tpw` tiles of 64 rows; a
// wave multiplies 16 rows by all DH columns.  Elements j of a row are stored at
// (j % 4) DH/4 + j / 4, so that the lanes that supply k = j % 4 read 8
// consecutive steps with one 16-byte load (bf16).  At 4 x 4096 rows, 32 groups,
// dh = 128: 0.41 ms (42 TFLOP/s) with the gate query inside; one thread per output with an
// fma chain over global memory took 15.3 ms, and the gate query 0.07 ms; two
// 16-row tiles per wave (half the operand conversions, half the waves) 0.48 ms.
typedef double f64x4_t __attribute__((ext_vector_type(4)));

template <typename T, int DH>
__global__ void __launch_bounds__(256) project_rows_kernel(const T* __restrict__ in, long long sb, long long sg,
                                                           long long sr, int nh, const T* __restrict__ W,
                                                           T* __restrict__ plain, T* __restrict__ out, int Hkv,
                                                           int rows, int tpw, int groups) {
  constexpr int PITCH = DH + 16 / (int)sizeof(T);  // 16-byte reads of 16 rows hit distinct banks
  constexpr int Q4 = DH / 4, C8 = DH / 8;
  __shared__ __align__(16) T Ws[DH * PITCH];
  __shared__ __align__(16) T As[64 * PITCH];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = lane & 15, q = lane >> 4;
  const int grp = blockIdx.x % groups;
  const int z = blockIdx.x / groups, g = z % Hkv, bi = z / Hkv;
  // the 8 consecutive elements from j0 (a multiple of 8) of an LDS row, permuted
  auto put8 = [](T* row, int j0, const T* x) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      T* d = row + e * Q4 + j0 / 4;
      d[0] = x[e];
      d[1] = x[e + 4];
    }
  };
  const T* Wg = W + (size_t)g * DH * DH;
  for (int i = tid; i < DH * C8; i += 256) {
    alignas(16) T x[8];
#pragma unroll
    for (int k = 0; k < (int)(8 * sizeof(T) / 16); ++k) ((uint4*)x)[k] = ((const uint4*)(Wg + i * 8))[k];
    put8(Ws + (i / C8) * PITCH, (i % C8) * 8, x);
  }
  const T* src = in + bi * sb + g * sg;
  const size_t orow = (size_t)z * rows;
  const int r_end = min(rows, (grp + 1) * tpw * 64);
  for (int r0 = grp * tpw * 64; r0 < r_end; r0 += 64) {
    constexpr int NI = 64 * C8 / 256;  // 8-value chunks per thread
    double acc8[NI][8];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int e = 0; e < 8; ++e) acc8[i][e] = 0.0;
    for (int h = 0; h < nh; ++h) {
      Vec8<T> v[NI];
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int ch = tid + i * 256;
        v[i].load(src + (long long)min(r0 + ch / C8, rows - 1) * sr + h * DH + (ch % C8) * 8);
      }
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc8[i][e] += (double)v[i].get(e);
    }
    __syncthreads();  // the previous tile's rows are stored
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int ch = tid + i * 256, r = ch / C8, j0 = (ch % C8) * 8;
      alignas(16) T x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = nh == 1 ? Act<T>::from_f32((float)acc8[i][e]) : Act<T>::from_f64(acc8[i][e]);
      put8(As + r * PITCH, j0, x);
      if (plain && r0 + r < rows) {
#pragma unroll
        for (int k = 0; k < (int)(8 * sizeof(T) / 16); ++k)
          ((uint4*)(plain + (orow + r0 + r) * DH + j0))[k] = ((const uint4*)x)[k];
      }
    }
    __syncthreads();
    f64x4_t acc[DH / 16];
#pragma unroll
    for (int t = 0; t < DH / 16; ++t) acc[t] = f64x4_t{0.0, 0.0, 0.0, 0.0};
    const T* ar = As + (wave * 16 + c) * PITCH + q * Q4;
    const T* wr = Ws + c * PITCH + q * Q4;
    for (int s0 = 0; s0 < Q4; s0 += 8) {
      Vec8<T> av, wv[DH / 16];
      av.load(ar + s0);
#pragma unroll
      for (int t = 0; t < DH / 16; ++t) wv[t].load(wr + t * 16 * PITCH + s0);
#pragma unroll
      for (int e = 0; e < 8; ++e) {  // step s0 + e: j = 4 (s0 + e) .. + 3
        const double a = (double)av.get(e);
#pragma unroll
        for (int t = 0; t < DH / 16; ++t)
          acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, (double)wv[t].get(e), acc[t], 0, 0, 0);
      }
    }
    // accumulator element i of column block t: row q + 4 i, column 16 t + c;
    // back through the wave's own LDS rows (its reads above are done) to 16-byte stores
    T* ow = As + wave * 16 * PITCH;
    wave_lds_fence();
#pragma unroll
    for (int t = 0; t < DH / 16; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) ow[(q + 4 * i) * PITCH + t * 16 + c] = Act<T>::from_f64(acc[t][i]);
    wave_lds_fence();
    constexpr int CW = 16 / (int)sizeof(T);  // values per 16-byte store
#pragma unroll
    for (int k = 0; k < 16 * DH / CW / 64; ++k) {
      const int ch = lane + k * 64, r = ch / (DH / CW), j0 = (ch % (DH / CW)) * CW;
      const int row = r0 + wave * 16 + r;
      if (row < rows) *(uint4*)(out + (orow + row) * DH + j0) = *(const uint4*)(ow + r * PITCH + j0);
    }
  }
}

// rows of (b, group) projected by w; in: see project_rows_kernel
template <typename T>
static void run_project_rows(const T* in, long long sb, long long sg, long long sr, int nh, const T* w, T* plain,
                             T* out, int b, int Hkv, int rows, int dh, hipStream_t s) {
  const int tiles = cdiv(rows, 64);
  // W is read once per workgroup: up to 4 row tiles each, as long as 1024 workgroups (two rounds) remain
  const int tpw = (int)std::min<long long>(4, std::max<long long>(1, (long long)tiles * b * Hkv / 1024));
  const int groups = cdiv(tiles, tpw);
  const unsigned grid = (unsigned)groups * b * Hkv;
  if (dh == 128)
    project_rows_kernel<T, 128><<<grid, 256, 0, s>>>(in, sb, sg, sr, nh, w, plain, out, Hkv, rows, tpw, groups);
  else
    project_rows_kernel<T, 64><<<grid, 256, 0, s>>>(in, sb, sg, sr, nh, w, plain, out, Hkv, rows, tpw, groups);
}

// Gate query qhat[b, g, t, j] = rho(sum over the group's heads of Q[b, t, h, j]),
// fp64 sum in ascending head order: thread per (b, g, t, 8-dim chunk), with
// 16-byte loads and stores.
template <typename T>
__global__ void gate_query_kernel(const T* __restrict__ Q, T* __restrict__ out, int n, int H, int Hkv, int dh,
                                  size_t chunks) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= chunks) return;
  const int nc = dh / 8;
  const int c8 = (int)(idx % nc);
  size_t r = idx / nc;
  const int t = (int)(r % n);
  r /= n;
  const int g = (int)(r % Hkv);
  const int bi = (int)(r / Hkv);
  const int G = H / Hkv;
  const T* q = Q + (((size_t)bi * n + t) * H + (size_t)g * G) * dh + c8 * 8;
  double acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.0;
  for (int h = 0; h < G; ++h) {
    Vec8<T> v;
    v.load(q + (size_t)h * dh);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += (double)v.get(e);
  }
  alignas(16) T res[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) res[e] = Act<T>::from_f64(acc[e]);
  uint4* o = (uint4*)(out + idx * 8);  // [b, Hkv, n, dh]: chunk idx
#pragma unroll
  for (int k = 0; k < (int)(8 * sizeof(T) / 16); ++k) o[k] = ((const uint4*)res)[k];
}

template <typename T>
static void run_gate_query(const T* Q, int b, int n, int H, int Hkv, int dh, const T* w_gq, T* qplain, T* qhat,
                           hipStream_t s) {
  if (w_gq) {
    const int G = H / Hkv;
    run_project_rows<T>(Q, (long long)n * H * dh, (long long)G * dh, (long long)H * dh, G, w_gq, qplain, qhat, b, Hkv,
                        n, dh, s);
    return;
  }
  const size_t chunks = (size_t)b * Hkv * n * dh / 8;  // dh is a multiple of 8
  gate_query_kernel<T><<<(unsigned)((chunks + 255) / 256), 256, 0, s>>>(Q, qhat, n, H, Hkv, dh, chunks);
}

hipError_t launch_gate_query(int dtype, const void* Q, int b, int n, int H, int Hkv, int dh, const void* w_gq,
                             void* qplain, void* qhat, hipStream_t s) {
  if ((size_t)b * Hkv * n * dh == 0) return hipSuccess;
  if (dtype == SAS_BF16)
    run_gate_query<bf16_t>((const bf16_t*)Q, b, n, H, Hkv, dh, (const bf16_t*)w_gq, (bf16_t*)qplain, (bf16_t*)qhat, s);
  else
    run_gate_query<float>((const float*)Q, b, n, H, Hkv, dh, (const float*)w_gq, (float*)qplain, (float*)qhat, s);
  return hipGetLastError();
}

hipError_t launch_block_summaries(int dtype, const void* K, int b, int n, int Hkv, int dh, int B,
                                  const void* w_gk, void* kplain, void* ksum, hipStream_t s) {
  const int NB = cdiv(n, B);
  const size_t total = (size_t)b * Hkv * NB * dh;
  if (total == 0) return hipSuccess;
  const size_t tchunks = total / 8;
  const unsigned sgrid = (unsigned)((tchunks + 63) / 64);
  void* dst = w_gk ? kplain : ksum;
  if (dtype == SAS_BF16)
    summaries_kernel<bf16_t><<<sgrid, 64, 0, s>>>((const bf16_t*)K, (bf16_t*)dst, n, Hkv, dh, B, NB, tchunks);
  else
    summaries_kernel<float><<<sgrid, 64, 0, s>>>((const float*)K, (float*)dst, n, Hkv, dh, B, NB, tchunks);
  if (w_gk) {
    // rows of incomplete blocks are zero and project to zero
    const long long sg = (long long)NB * dh;
    if (dtype == SAS_BF16)
      run_project_rows<bf16_t>((const bf16_t*)kplain, Hkv * sg, sg, dh, 1, (const bf16_t*)w_gk, nullptr, (bf16_t*)ksum,
                               b, Hkv, NB, dh, s);
    else
      run_project_rows<float>((const float*)kplain, Hkv * sg, sg, dh, 1, (const float*)w_gk, nullptr, (float*)ksum, b,
                              Hkv, NB, dh, s);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Selection: one workgroup of SEL_NW waves per 64 consecutive query rows of
// one (batch, group); lane = query row.  The 64 gate queries are staged in
// LDS once (as fp32, each the rounded gate query); the waves split the
// historical blocks into contiguous ranges and walk theirs in ascending
// order, in chunks of SEL_MC = 8 summaries, one exact fp64 FMA chain per
// (row, block), j ascending.  The summary values reach the rows through DPP
// row broadcasts: for a 16-dimension group, lane n of every 16-lane row holds
// summary n % 8 at dimensions 8 (n / 8) .. + 8 (the four rows hold the same
// values), and each v_fmac_f64 takes its summary operand from one lane of its
// row, so the wave's 64 chains share one loaded copy without LDS traffic.
// Each lane keeps a register Top-K (best first) and a running LSE.  The lists
// are ordered by score, then by lower block index (the order of a single
// ascending scan with strict comparisons).  Two sorted lists are merged by
// taking the elementwise better of one and the reverse of the other, which
// holds the best K as a bitonic sequence that a half-cleaner cascade sorts:
// a chunk's candidates (sorted by a bitonic network) into a wave's list, and
// the other waves' lists into wave 0's, in wave order.
constexpr int SEL_NW = 4;  // waves per workgroup

// r[mm] += k(lane L + mm of the 16-lane row) * q, mm = 0..7, for the four
// dimensions whose summary values are k0..k3 and query values q0..q3, in that
// order (L = 0: summaries of the group's first 8 dimensions, L = 8: its last
// 8).  v_fmac_f64 with a row_newbcast DPP source: every lane of a row reads
// the source from one lane of that row.  The s_nop covers the two wait states
// a DPP read needs after a VALU write of its source.
#define SEL_F(R, K, Q, N) "v_fmac_f64_dpp %" #R ", %" #K ", %" #Q " row_newbcast:" #N " row_mask:0xf bank_mask:0xf\n\t"
#define SEL_DIM0(K, Q) \
  SEL_F(0, K, Q, 0) SEL_F(1, K, Q, 1) SEL_F(2, K, Q, 2) SEL_F(3, K, Q, 3) \
  SEL_F(4, K, Q, 4) SEL_F(5, K, Q, 5) SEL_F(6, K, Q, 6) SEL_F(7, K, Q, 7)
#define SEL_DIM8(K, Q) \
  SEL_F(0, K, Q, 8) SEL_F(1, K, Q, 9) SEL_F(2, K, Q, 10) SEL_F(3, K, Q, 11) \
  SEL_F(4, K, Q, 12) SEL_F(5, K, Q, 13) SEL_F(6, K, Q, 14) SEL_F(7, K, Q, 15)
template <int L>
__device__ __forceinline__ void sel_fma4(double (&r)[8], double k0, double k1, double k2, double k3, double q0,
                                         double q1, double q2, double q3) {
  static_assert(L == 0 || L == 8, "lane base 0 or 8");
  if constexpr (L == 0) {
    asm("s_nop 1\n\t" SEL_DIM0(8, 12) SEL_DIM0(9, 13) SEL_DIM0(10, 14) SEL_DIM0(11, 15)
        : "+v"(r[0]), "+v"(r[1]), "+v"(r[2]), "+v"(r[3]), "+v"(r[4]), "+v"(r[5]), "+v"(r[6]), "+v"(r[7])
        : "v"(k0), "v"(k1), "v"(k2), "v"(k3), "v"(q0), "v"(q1), "v"(q2), "v"(q3));
  } else {
    asm("s_nop 1\n\t" SEL_DIM8(8, 12) SEL_DIM8(9, 13) SEL_DIM8(10, 14) SEL_DIM8(11, 15)
        : "+v"(r[0]), "+v"(r[1]), "+v"(r[2]), "+v"(r[3]), "+v"(r[4]), "+v"(r[5]), "+v"(r[6]), "+v"(r[7])
        : "v"(k0), "v"(k1), "v"(k2), "v"(k3), "v"(q0), "v"(q1), "v"(q2), "v"(q3));
  }
}
#undef SEL_DIM8
#undef SEL_DIM0
#undef SEL_F

// Lists of up to 16 slots: three waves per SIMD (a few values spill, and the
// third wave hides more of the merge and load latency than they cost).
template <typename T, int DH, int KMAX, int SEL_MC, bool NOISY>
__global__ void __launch_bounds__(SEL_NW * WAVE, KMAX <= 16 ? 3 : 2) select_kernel(SelectArgs P) {
  static_assert((KMAX & (KMAX - 1)) == 0, "the merge network needs a power-of-two list");
  static_assert(SEL_MC == 8 && DH % 16 == 0, "chunks of 8 summaries, 16-dimension groups");
  // a list exchange region: [KMAX][WAVE] keys, [KMAX][WAVE] blocks, [WAVE]
  // running max and sum; the second region reuses the query staging when it
  // is large enough (the queries are dead once every wave has scored)
  constexpr int MG_BYTES = KMAX * WAVE * 12 + WAVE * 12;
  constexpr bool R1_IN_QS = WAVE * (DH + 4) * 4 >= MG_BYTES;
  __shared__ __align__(16) unsigned char pool[R1_IN_QS ? MG_BYTES : 2 * MG_BYTES];
  // the 64 gate queries as fp32 (exact: each is a rounded value of T); the
  // pitch of DH + 4 puts the 16-byte reads of 16 lanes in distinct banks
  __shared__ __align__(16) float qs[WAVE][DH + 4];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = blockIdx.y, bi = blockIdx.z;
  const int t0 = (gridDim.x - 1 - blockIdx.x) * WAVE;  // the late rows (more blocks to score) first
  const int t = t0 + lane;
  const bool valid = t < P.n;
  const int G = P.H / P.Hkv;
  const int ct = valid ? t / P.B : 0;
  const int fb = valid ? doc_first(P.doc, bi, P.NB, t, P.B) : 0;  // first block of the query's document
  const int t_last = min(P.n - 1, t0 + WAVE - 1);
  const int cmax = t_last / P.B;  // wave-uniform block count
  const int mlo = doc_first(P.doc, bi, P.NB, t0, P.B);  // the rows' earliest document start
  const double den = (double)G * sqrt((double)DH);  // s = r / (G sqrt(dh))
  const double inv_scale = 1.0 / den;
  const size_t row = ((size_t)bi * P.Hkv + g) * P.n + t;
  const float* noise = (NOISY && valid) ? P.noise + row * P.NB : nullptr;
  // the log-gate table row of this query: raw scores written as they are computed (softmax:
  // the LSE is subtracted at the end), the other activations' gates written directly
  float* lgrow = (P.log_gate && valid) ? P.log_gate + row * P.NB : nullptr;
  const int act = P.act;

  // stage the 64 gate queries: either the precomputed (projected) rows, or
  // the group's query heads summed here in fp64 and rounded once; a thread's
  // loads of one head are issued together
  {
    constexpr int NC = DH / 8;       // 8-value chunks per row
    constexpr int NI = NC / SEL_NW;  // chunks per thread (64 rows x NC chunks)
    const int rows = t_last - t0 + 1;
    const int nh = P.qhat ? 1 : G;
    double acc[NI][8];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[i][e] = 0.0;
    for (int h = 0; h < nh; ++h) {
      Vec8<T> v[NI];
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int c = tid + i * SEL_NW * WAVE;
        const int r = c / NC, c8 = c % NC;
        const int rr = min(r, rows - 1);
        v[i].load(P.qhat ? (const T*)P.qhat + (((size_t)bi * P.Hkv + g) * P.n + t0 + rr) * DH + c8 * 8
                         : (const T*)P.Q + (((size_t)bi * P.n + t0 + rr) * P.H + (size_t)g * G + h) * DH + c8 * 8);
      }
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[i][e] += (double)v[i].get(e);
    }
    // a single row (one head, or the projected query) is already a value of
    // T, and its rounding the identity: stored as it is
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = tid + i * SEL_NW * WAVE;
      const int r = c / NC, c8 = c % NC;
#pragma unroll
      for (int e = 0; e < 8; ++e)
        qs[r][c8 * 8 + e] =
            r < rows ? (nh == 1 ? (float)acc[i][e] : Act<T>::to_f32(Act<T>::from_f64(acc[i][e]))) : 0.f;
    }
  }
  __syncthreads();

  constexpr int EMPTY = 0x7fffffff;  // block id of an empty slot
  double tr[KMAX];
  int tm[KMAX];
#pragma unroll
  for (int i = 0; i < KMAX; ++i) {
    tr[i] = -DBL_MAX;
    tm[i] = EMPTY;
  }
  double mrun = -DBL_MAX;  // running max of s
  float lrun = 0.f;        // running sum of exp(s - mrun)
  // does key a rank strictly ahead of the slot (b, bm)?  An equal key keeps
  // the earlier (lower) block ahead.  Without noise every key is a finite
  // exact dot product, above the empty slots' -DBL_MAX.  With noise a key can
  // be -inf (or NaN): every key then beats an empty slot (so such blocks are
  // kept when fewer than K others exist) and NaN ranks below every number.
  auto beats = [](double a, double b, int bm) -> bool {
    if constexpr (!NOISY) {
      return a > b;
    } else {
      if (bm == EMPTY) return true;
      if (a != a) return false;
      return a > b || b != b;
    }
  };
  // the total order of the lists: a ranks ahead of b (ties: lower block first)
  auto ahead = [](double a, int am, double b, int bm) -> bool {
    if constexpr (!NOISY) {
      return a > b || (a == b && am < bm);
    } else {
      const int ca = am == EMPTY ? 2 : (a != a ? 1 : 0), cb = bm == EMPTY ? 2 : (b != b ? 1 : 0);
      if (ca != cb) return ca < cb;
      return (ca == 0 && a > b) || ((ca == 1 || a == b) && am < bm);
    }
  };

  const T* kbar = (const T*)P.kbar + ((size_t)bi * P.Hkv + g) * (size_t)P.NB * DH;
  const int per = (cmax - mlo + SEL_NW - 1) / SEL_NW;
  const int mb = mlo + wave * per, me = min(cmax, mb + per);
  // this lane's part of a 16-dimension group jg of the chunk at m0: summary
  // (lane % 8) of the chunk (the last block for a ragged chunk's missing
  // ones), dimensions 16 jg + 8 ((lane % 16) / 8) .. + 8
  const int lsum = lane & 7, lhalf = (lane >> 3) & 1;
  auto group_ptr = [&](int m0, int jg) {
    return kbar + (size_t)min(m0 + lsum, me - 1) * DH + jg * 16 + lhalf * 8;
  };
  constexpr int NG = DH / 16;  // dimension groups per summary
  Vec8<T> kn;  // the next group's values, loaded one group ahead
  if (mb < me) kn.load(group_ptr(mb, 0));
  for (int m0 = mb; m0 < me; m0 += SEL_MC) {
    const int mc = min(SEL_MC, me - m0);
    // r[mm] = sum_j q_j kbar[m0+mm]_j: one fp64 FMA chain per block, j ascending
    double r[SEL_MC];
#pragma unroll
    for (int mm = 0; mm < SEL_MC; ++mm) r[mm] = 0.0;
    const float* qrow = qs[lane];
#pragma unroll
    for (int jg = 0; jg < NG; ++jg) {
      const Vec8<T> kc = kn;
      if (jg + 1 < NG) kn.load(group_ptr(m0, jg + 1));
      else if (m0 + SEL_MC < me) kn.load(group_ptr(m0 + SEL_MC, 0));
      double kd[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) kd[e] = (double)kc.get(e);
      const float4 q0 = *(const float4*)(qrow + jg * 16), q1 = *(const float4*)(qrow + jg * 16 + 4);
      const float4 q2 = *(const float4*)(qrow + jg * 16 + 8), q3 = *(const float4*)(qrow + jg * 16 + 12);
      // dimensions 16 jg + 0..7 from lanes 0..7 of the row, then 16 jg + 8..15 from lanes 8..15
      sel_fma4<0>(r, kd[0], kd[1], kd[2], kd[3], q0.x, q0.y, q0.z, q0.w);
      sel_fma4<0>(r, kd[4], kd[5], kd[6], kd[7], q1.x, q1.y, q1.z, q1.w);
      sel_fma4<8>(r, kd[0], kd[1], kd[2], kd[3], q2.x, q2.y, q2.z, q2.w);
      sel_fma4<8>(r, kd[4], kd[5], kd[6], kd[7], q3.x, q3.y, q3.z, q3.w);
    }
    // the chunk's candidates (ranking key, block; EMPTY where the block is not
    // a historical block of this row's document)
    double cr[SEL_MC];
    int cmi[SEL_MC];
    bool any = false;
#pragma unroll
    for (int mm = 0; mm < SEL_MC; ++mm) {
      const int m = m0 + mm;
      cr[mm] = -DBL_MAX;
      cmi[mm] = EMPTY;
      if (mm >= mc || m >= ct || m < fb) continue;
      // ranking key: the raw score r, or the noisy score s + noise when noise is given
      const double sv = noise ? r[mm] / den + (double)noise[m] : r[mm] * inv_scale;
      const double rv = noise ? sv : r[mm];
      if (lgrow) {
        double gv = sv;
        if (act == SAS_ACT_SIGMOID) gv = sv >= 0.0 ? -log1p(exp(-sv)) : sv - log1p(exp(sv));
        lgrow[m] = (float)gv;
      }
      // running LSE: one exponential of minus the gap to the running max, the
      // sum rescaled when sv is the new max (no divergent branch)
      {
        const float d = (float)(sv - mrun);
        const float e = __expf(-fabsf(d));
        const bool up = d > 0.f;
        lrun = up ? fmaf(lrun, e, 1.f) : lrun + e;
        mrun = up ? sv : mrun;
      }
      cr[mm] = rv;
      cmi[mm] = m;
      any = any || beats(rv, tr[KMAX - 1], tm[KMAX - 1]);
    }
    // Keep the best KMAX of the list and the chunk's candidates: sort the
    // candidates best first; the better of list slot KMAX-1-i and candidate i
    // leaves the best KMAX as a bitonic sequence, which a half-cleaner cascade
    // sorts.  The order is the total order (key descending, block ascending)
    // that inserting the blocks one by one in ascending order gives.
    if (__builtin_amdgcn_ballot_w64(any) != 0) {
      auto cas = [&](double& ra, int& ma, double& rb, int& mb) {  // the better one into (ra, ma)
        const bool sw = ahead(rb, mb, ra, ma);
        const double x = ra, y = rb;
        const int u = ma, v = mb;
        ra = sw ? y : x;
        rb = sw ? x : y;
        ma = sw ? v : u;
        mb = sw ? u : v;
      };
#pragma unroll
      for (int k = 2; k <= SEL_MC; k <<= 1)
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1)
#pragma unroll
          for (int i = 0; i < SEL_MC; ++i) {
            const int l = i ^ j;
            if (l > i) {
              if ((i & k) == 0) cas(cr[i], cmi[i], cr[l], cmi[l]);
              else cas(cr[l], cmi[l], cr[i], cmi[i]);
            }
          }
      static_assert(SEL_MC <= KMAX, "a chunk fits the list");
      if (!NOISY && m0 == mb) {
        // the wave's first chunk: the list is empty, so the sorted candidates
        // are the list (what the merge below would leave; the noisy variant,
        // at its register limit, takes the merge)
#pragma unroll
        for (int i = 0; i < SEL_MC; ++i) {
          tr[i] = cr[i];
          tm[i] = cmi[i];
        }
      } else {
#pragma unroll
        for (int i = 0; i < SEL_MC; ++i) {
          const int q = KMAX - 1 - i;
          if (ahead(cr[i], cmi[i], tr[q], tm[q])) {
            tr[q] = cr[i];
            tm[q] = cmi[i];
          }
        }
#pragma unroll
        for (int len = KMAX / 2; len >= 1; len >>= 1)
#pragma unroll
          for (int i = 0; i < KMAX; ++i)
            if ((i & len) == 0) cas(tr[i], tm[i], tr[i + len], tm[i + len]);
      }
    }
  }
  __syncthreads();
  // merge the waves' lists as a tree: 1 into 0 and 3 into 2, then 2 into 0.
  // The lists are ordered by a strict total order, so the best KMAX of the
  // union do not depend on the merge order.
  unsigned char* const region[2] = {pool, R1_IN_QS ? (unsigned char*)&qs[0][0] : pool + MG_BYTES};
  auto put = [&](const unsigned char* base) {  // this wave's list and LSE into a region
    double* rk = (double*)base;
    int* rb = (int*)(base + KMAX * WAVE * 8);
#pragma unroll
    for (int i = 0; i < KMAX; ++i) {
      rk[i * WAVE + lane] = tr[i];
      rb[i * WAVE + lane] = tm[i];
    }
    ((double*)(base + KMAX * WAVE * 12))[lane] = mrun;
    ((float*)(base + KMAX * WAVE * 12 + WAVE * 8))[lane] = lrun;
  };
  auto take = [&](const unsigned char* base) {  // a region's list and LSE into this wave's
    const double* rk = (const double*)base;
    const int* rb = (const int*)(base + KMAX * WAVE * 8);
    // the better of slot i and the other list's slot KMAX-1-i: the best KMAX
    // of both, descending then ascending (a bitonic sequence)
#pragma unroll
    for (int i = 0; i < KMAX; ++i) {
      const double ob = rk[(KMAX - 1 - i) * WAVE + lane];
      const int om = rb[(KMAX - 1 - i) * WAVE + lane];
      if (ahead(ob, om, tr[i], tm[i])) {
        tr[i] = ob;
        tm[i] = om;
      }
    }
    // bitonic sort, best first
#pragma unroll
    for (int len = KMAX / 2; len >= 1; len >>= 1)
#pragma unroll
      for (int i = 0; i < KMAX; ++i)
        if ((i & len) == 0) {
          const int j = i + len;
          const bool sw = ahead(tr[j], tm[j], tr[i], tm[i]);
          const double ri = tr[i], rj = tr[j];
          const int mi = tm[i], mj = tm[j];
          tr[i] = sw ? rj : ri;
          tr[j] = sw ? ri : rj;
          tm[i] = sw ? mj : mi;
          tm[j] = sw ? mi : mj;
        }
    const double om = ((const double*)(base + KMAX * WAVE * 12))[lane];
    const float ol = ((const float*)(base + KMAX * WAVE * 12 + WAVE * 8))[lane];
    if (om > mrun) {
      lrun = lrun * expf((float)(mrun - om)) + ol;
      mrun = om;
    } else if (ol > 0.f) {
      lrun += ol * expf((float)(om - mrun));
    }
  };
  static_assert(SEL_NW == 4, "a two-level merge tree");
  if (wave == 1) put(region[0]);
  if (wave == 3) put(region[1]);
  __syncthreads();
  if (wave == 0) take(region[0]);
  if (wave == 2) take(region[1]);
  __syncthreads();
  if (wave == 2) put(region[0]);
  __syncthreads();
  if (wave == 0) take(region[0]);
  if (wave != 0 || !valid) return;
  const double lse = (ct > fb) ? mrun + log((double)lrun) : 0.0;
  auto log_gate_of = [&](double key) -> double {  // log g of a block from its ranking key
    const double sv = noise ? key : key * inv_scale;
    if (act == SAS_ACT_SOFTMAX) return sv - lse;
    if (act == SAS_ACT_SIGMOID) return sv >= 0.0 ? -log1p(exp(-sv)) : sv - log1p(exp(sv));
    return sv;
  };
  const int K = P.K;
  const int C = ct - fb;  // historical blocks of the query (its own document)
  const int kk = min(K, C);

  if (P.tau) {
    float tau;
    if (C <= K) tau = -INFINITY;
    else if (K == 0) tau = INFINITY;
    else {
      double rk = tr[0];
#pragma unroll
      for (int i = 0; i < KMAX; ++i)
        if (i == K - 1) rk = tr[i];
      tau = (float)log_gate_of(rk);
    }
    P.tau[row] = tau;
  }

  // order the kept blocks by index (a bitonic sorting network; empty slots,
  // the largest index, last)
#pragma unroll
  for (int i = 0; i < KMAX; ++i)
    if (i >= kk) tm[i] = EMPTY;
#pragma unroll
  for (int k = 2; k <= KMAX; k <<= 1)
#pragma unroll
    for (int j = k >> 1; j > 0; j >>= 1)
#pragma unroll
      for (int i = 0; i < KMAX; ++i) {
        const int l = i ^ j;
        if (l > i) {
          const bool sw = (i & k) == 0 ? tm[i] > tm[l] : tm[i] < tm[l];
          const int a = tm[i], c = tm[l];
          const double ra = tr[i], rc = tr[l];
          tm[i] = sw ? c : a;
          tm[l] = sw ? a : c;
          tr[i] = sw ? rc : ra;
          tr[l] = sw ? ra : rc;
        }
      }
  int32_t* sel = P.sel + row * K;
  float* sb = P.sel_bias + row * K;
#pragma unroll
  for (int i = 0; i < KMAX; ++i) {
    if (i < K) {
      const bool kept = i < kk && tm[i] != EMPTY;
      sel[i] = kept ? tm[i] : -1;
      sb[i] = kept ? (float)log_gate_of(tr[i]) : 0.f;
    }
  }

  if (lgrow) P.row_lse[row] = (float)lse;  // finish_table_kernel subtracts it (softmax)
}

// finish the log-gate table: softmax gates are the written scores minus the
// row's LSE; blocks m >= C_t are not historical (-inf)
__global__ void finish_table_kernel(float* __restrict__ table, const float* __restrict__ row_lse, size_t rows,
                                    int n, int Hkv, int B, int NB, int softmax, const int32_t* __restrict__ doc) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= rows * NB) return;
  const size_t row = idx / NB;
  const int t = (int)(row % n), bi = (int)(row / ((size_t)n * Hkv));
  const int m = (int)(idx % NB), ct = t / B, fb = doc_first(doc, bi, NB, t, B);
  table[idx] = (m < ct && m >= fb) ? (softmax ? table[idx] - row_lse[row] : table[idx]) : -INFINITY;
}

template <typename T, int DH, bool NOISY>
static void run_select_t(const SelectArgs& a, hipStream_t s) {
  dim3 grid(cdiv(a.n, WAVE), a.Hkv, a.b);
  if (a.K <= 8) select_kernel<T, DH, 8, 8, NOISY><<<grid, SEL_NW * WAVE, 0, s>>>(a);
  else if (a.K <= 16) select_kernel<T, DH, 16, 8, NOISY><<<grid, SEL_NW * WAVE, 0, s>>>(a);
  else select_kernel<T, DH, 32, 8, NOISY><<<grid, SEL_NW * WAVE, 0, s>>>(a);
}

template <typename T, int DH>
static void run_select(const SelectArgs& a, hipStream_t s) {
  if (a.noise) run_select_t<T, DH, true>(a, s);
  else run_select_t<T, DH, false>(a, s);
}

hipError_t launch_select(int dtype, const SelectArgs& a, hipStream_t s) {
  if (a.n <= 0 || a.b <= 0) return hipSuccess;
  if (a.log_gate && !a.row_lse) return hipErrorInvalidValue;
  if (dtype == SAS_BF16) {
    if (a.dh == 128) run_select<bf16_t, 128>(a, s);
    else run_select<bf16_t, 64>(a, s);
  } else {
    if (a.dh == 128) run_select<float, 128>(a, s);
    else run_select<float, 64>(a, s);
  }
  if (a.log_gate) {
    const size_t rows = (size_t)a.b * a.Hkv * a.n;
    finish_table_kernel<<<(unsigned)cdiv(rows * a.NB, 256), 256, 0, s>>>(a.log_gate, a.row_lse, rows, a.n, a.Hkv, a.B,
                                                                          a.NB, a.act == SAS_ACT_SOFTMAX, a.doc);
  }
  return hipGetLastError();
}

}  // namespace sas

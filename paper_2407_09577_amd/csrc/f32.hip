// fp32 fused norm-then-project kernels (exact fp32 products, no reduced-precision matrix-core
// modes): one on the fp32 matrix cores for all but the smallest calls, one on the vector units for
// those, and vector tiles that a caller can name.
//
// f32_kernel, the vector tiles (named configurations 1 and 2 alone).  A workgroup owns a BM x 64 output tile (BM = 16 RI rows) and KS groups of 256
// threads split K between them: group g takes the 64-deep k steps g, g + KS, ...,
// staging its activation and weight tiles in its own LDS buffers.  The threads
// that stage an activation row also accumulate its sum of squares (and sum, for
// LayerNorm) from the values they just loaded, alongside the products (Cor. 1).
// The groups' partial products and sums are added in LDS in a fixed order
// (deterministic; no split across workgroups), and group 0 applies the deferred
// per-row scale (Prop. 2) in the epilogue.  LayerNorm runs on activations shifted
// by a per-row pivot p (the row's first element): the sum exchange of Sec. 3.5 holds
// for any shift, sum_k (a_k - mu) W*_kn = sum_k (a_k - p) W*_kn - (mu - p) colsum_n,
// and with |mu - p| ~ sigma neither the fp32 products nor the statistics cancel when
// |mu| >> sigma (sums of the shifted values in fp64).  Thread (tx, ty) of group 0 finishes
// rows ty + 16 i and packed columns tx + 16 j, so columns j = 0, 1 (and 2, 3) are a
// GLU gate block and its up block.  RI = 1 with four k groups makes each thread's
// chain of products a quarter of K long for problems with few 64-row tiles; the
// few-row kernel below goes further for problems with few 16 x 64 tiles.
#include "fn_device.h"
#include "fn_epilogue.h"
#include "fn_launch.h"
#include "fn_tile.h"

#ifndef FEW_MIN_WG
#define FEW_MIN_WG 256
#endif

namespace fn {

// Epilogue of the fp32 kernels.  Thread (tx, ty) holds the accumulators of rows
// ty + 16 i (i < RI) and packed columns tx + 16 j (j < NJ) of the tile at (m0, p0), and
// rss / rsa the sums of its rows; first_tile marks the tile column that writes inv_rms.
template <int EPI, int RI, int NJ>
__device__ __forceinline__ void f32_epilogue(float (&acc)[RI][NJ], const StatT<EPI> (&rss)[RI],
                                             const StatT<EPI> (&rsa)[RI], int tx, int ty, int m0, int p0, int M,
                                             int ncols, float* __restrict__ y, int ldy, const EpiArgs& ep,
                                             bool first_tile) {
  static_assert(!epi_is_glu(EPI) || NJ % 2 == 0, "GLU: gate/up column block pairs");
  static_assert(EPI != EPI_HEADNORM || NJ == 4, "per-head norms: heads up to 64 wide in one tile");
  if constexpr (EPI == EPI_ROPE) {
    // Pair partners (column c ^ 1) sit in the neighbouring lane (tx ^ 1, same rows);
    // every lane takes part in the exchange before any guard.
    float part[RI][NJ];
#pragma unroll
    for (int i = 0; i < RI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) part[i][j] = __shfl_xor(acc[i][j], 1);
#pragma unroll
    for (int i = 0; i < RI; ++i) {
      const int r = ty + 16 * i;
      const int m = m0 + r;
      if (m >= M) continue;
      const RowStat st = row_stat_at<EPI>(rss[i], rsa[i], ep, m, M);
      if (ep.inv_rms && first_tile && tx == 0) ep.inv_rms[m] = st.s;
      float* yr = y + (int64_t)m * ldy;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int c = p0 + tx + 16 * j;
        if (c >= ncols) continue;
        const float bv = ep.bias ? ep.bias[c] : 0.f, bw = ep.bias ? ep.bias[c ^ 1] : 0.f;
        yr[c] = rope1(c, acc[i][j], part[i][j], bv, bw, st, ep);
      }
    }
  } else if constexpr (EPI == EPI_HEADNORM) {
    // Heads of h | 64 columns: a lane holds columns tx + 16 j of its rows.  A head's
    // squares are summed over its lanes (xor 1 .. min(h, 16) / 2) and, for h > 16, over
    // the lane's h / 16 column groups of the head; pair partners sit in lane tx ^ 1.
    // Every lane takes part in the exchanges before any guard.
    const int h = ep.head_h;
    float hs[RI][NJ], part[RI][NJ];
#pragma unroll
    for (int i = 0; i < RI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        float v = acc[i][j] * acc[i][j];
        for (int off = 1; off < (h < 16 ? h : 16); off <<= 1) v += __shfl_xor(v, off);
        hs[i][j] = v;
      }
#pragma unroll
    for (int i = 0; i < RI; ++i) {
      if (h >= 32) {  // combine the column groups of one head: j and j ^ 1 (h = 32), all four (h = 64)
        const float s01 = hs[i][0] + hs[i][1], s23 = hs[i][2] + hs[i][3];
        hs[i][0] = hs[i][1] = h == 64 ? s01 + s23 : s01;
        hs[i][2] = hs[i][3] = h == 64 ? s01 + s23 : s23;
      }
    }
#pragma unroll
    for (int i = 0; i < RI; ++i) {
      const int m = m0 + ty + 16 * i;
      const RowStat st = row_stat_at<EPI>(rss[i], rsa[i], ep, m, M);
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int c = p0 + tx + 16 * j;
        const int ch = c & (h - 1);
        const bool is_q = c < ep.q_end, is_k = !is_q && c < ep.k_end;
        const float* w = is_q ? ep.hn_gq : is_k ? ep.hn_gk : ep.hn_gv;
        float v = acc[i][j];
        if (w && c < ncols) v *= rsqrtf(fmaf(hs[i][j], ep.head_inv_h, ep.hn_eps)) * w[ch];
        else v *= st.s;
        part[i][j] = v;  // the normalised value, also the partner of lane tx ^ 1
      }
    }
#pragma unroll
    for (int i = 0; i < RI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) hs[i][j] = __shfl_xor(part[i][j], 1);
#pragma unroll
    for (int i = 0; i < RI; ++i) {
      const int r = ty + 16 * i;
      const int m = m0 + r;
      if (m >= M) continue;
      const RowStat st = row_stat_at<EPI>(rss[i], rsa[i], ep, m, M);
      if (ep.inv_rms && first_tile && tx == 0) ep.inv_rms[m] = st.s;
      float* yr = y + (int64_t)m * ldy;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int c = p0 + tx + 16 * j;
        if (c >= ncols) continue;
        const bool is_q = c < ep.q_end, is_k = !is_q && c < ep.k_end;
        float v = part[i][j];
        if ((is_q || is_k) && ep.rope_pos) {
          if ((unsigned)st.pos < (unsigned)ep.rope_P) {
            const int64_t off = (int64_t)st.pos * (ep.head_h >> 1) + ((c & (ep.head_h - 1)) >> 1);
            const float cs = ep.rope_cos[off], sn = ep.rope_sin[off], w2 = hs[i][j];
            v = (c & 1) ? w2 * sn + v * cs : v * cs - w2 * sn;
          } else {
            v = __builtin_nanf("");
          }
        }
        yr[c] = is_q ? v * ep.q_scale : v;
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < RI; ++i) {
      const int r = ty + 16 * i;
      const int m = m0 + r;
      if (m >= M) continue;
      const RowStat st = row_stat_at<EPI>(rss[i], rsa[i], ep, m, M);
      if constexpr (epi_exports_s(EPI)) {
        if (ep.inv_rms && first_tile && tx == 0) ep.inv_rms[m] = st.s;
      }
      float* yr = y + (int64_t)m * ldy;
      if constexpr (epi_is_glu(EPI)) {
#pragma unroll
        for (int q = 0; q < NJ / 2; ++q) {
          const int f = p0 / 2 + 16 * q + tx;
          if (f < ncols) yr[f] = epi_value<EPI>(acc[i][2 * q], acc[i][2 * q + 1], st, 0.f, 0.f);
        }
      } else {
        const float* vp = epi_vec<EPI>(ep);
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int c = p0 + tx + 16 * j;
          if (c >= ncols) continue;
          const float vec = vp ? vp[c] : 0.f;
          const float cs = EPI == EPI_LN ? ep.colsum[c] : 0.f;
          yr[c] = epi_value<EPI>(acc[i][j], acc[i][j], st, vec, cs);
        }
      }
    }
  }
}

template <int EPI, int RI, int KS>
__global__ __launch_bounds__(256 * KS) void f32_kernel(const float* __restrict__ a, int M, int K, int lda,
                                                       const float* __restrict__ ws, int NP, int ncols,
                                                       float* __restrict__ y, int ldy, EpiArgs ep) {
  constexpr int BM = 16 * RI, BN = 64, BK = 64;
  constexpr int TPR = 256 / BM;            // staging threads per activation row
  constexpr int QA = BK / (4 * TPR);       // activation quads per staging thread and step (= RI)
  constexpr int QW = BK * BN / (4 * 256);  // weight quads per thread and step
  using ST = StatT<EPI>;
  struct Stage {
    float As[BK][BM + 4];
    float Wsh[BK][BN];
  };
  __shared__ Stage stg[KS];
  __shared__ ST row_ss[KS][BM], row_sa[KS][BM];

  const int grp = threadIdx.x >> 8;  // k group (wave-uniform)
  const int t = threadIdx.x & 255;
  const int tx = t & 15, ty = t >> 4;
  const int m0 = blockIdx.y * BM, p0 = blockIdx.x * BN;

  const int lr = t / TPR, lkq = (t % TPR) * 4;  // activation staging: row lr, k quads lkq + 4 TPR q
  const int wk = t >> 4, wc = (t & 15) * 4;      // weight staging: k rows wk + 16 q, column quad
  const bool lr_ok = m0 + lr < M;
  const bool wc_ok = p0 + wc < NP;
  float(&As)[BK][BM + 4] = stg[grp].As;
  float(&Wsh)[BK][BN] = stg[grp].Wsh;
  // LayerNorm pivot of the staged row (rows past M stage zeros).
  const float piv = (EPI == EPI_LN && lr_ok) ? a[(int64_t)(m0 + lr) * lda] : 0.0f;

  float acc[RI][4] = {};
  ST ss = ST(0), sa = ST(0);
  // Every group runs the same number of rounds (the barriers need it); a group whose
  // step lies past K stages zeros and skips the products.
  const int rounds = ((K + BK - 1) / BK + KS - 1) / KS;
  for (int rd = 0; rd < rounds; ++rd) {
    const int k0 = (rd * KS + grp) * BK;
    const bool live = k0 < K;  // uniform in the group
    // All of the step's loads first (K is a multiple of 4: a quad is wholly inside
    // or outside; the packed weight has KP >= k0 + BK rows when k0 < K, zero past K).
    float4 av[QA], wv[QW];
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      const int k = k0 + lkq + 4 * TPR * q;
      av[q] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (lr_ok && k < K) {
        av[q] = *reinterpret_cast<const float4*>(a + (int64_t)(m0 + lr) * lda + k);
        if constexpr (EPI == EPI_LN) {
          av[q].x -= piv;
          av[q].y -= piv;
          av[q].z -= piv;
          av[q].w -= piv;
        }
      }
    }
#pragma unroll
    for (int q = 0; q < QW; ++q) {
      wv[q] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (wc_ok && live) wv[q] = *reinterpret_cast<const float4*>(ws + (int64_t)(k0 + wk + 16 * q) * NP + p0 + wc);
    }
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      if constexpr (EPI == EPI_LN) {  // fp64 sums: the squares of fp32 values are exact in fp64
        const double x = av[q].x, yv = av[q].y, z = av[q].z, w = av[q].w;
        ss += (x * x + yv * yv) + (z * z + w * w);
        sa += (x + yv) + (z + w);
      } else {
        ss = fmaf(av[q].x, av[q].x, ss);
        ss = fmaf(av[q].y, av[q].y, ss);
        ss = fmaf(av[q].z, av[q].z, ss);
        ss = fmaf(av[q].w, av[q].w, ss);
      }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      const int kq = lkq + 4 * TPR * q;
      As[kq + 0][lr] = av[q].x;
      As[kq + 1][lr] = av[q].y;
      As[kq + 2][lr] = av[q].z;
      As[kq + 3][lr] = av[q].w;
    }
#pragma unroll
    for (int q = 0; q < QW; ++q) *reinterpret_cast<float4*>(&Wsh[wk + 16 * q][wc]) = wv[q];
    __syncthreads();
    if (live) {
#pragma unroll 16
      for (int kk = 0; kk < BK; ++kk) {
        float ar[RI], wr[4];
#pragma unroll
        for (int i = 0; i < RI; ++i) ar[i] = As[kk][ty + 16 * i];
#pragma unroll
        for (int j = 0; j < 4; ++j) wr[j] = Wsh[kk][tx + 16 * j];
#pragma unroll
        for (int i = 0; i < RI; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(ar[i], wr[j], acc[i][j]);
      }
    }
  }
  // A row's staging threads are TPR consecutive lanes of one wave.
#pragma unroll
  for (int off = 1; off < TPR; off <<= 1) {
    ss += __shfl_xor(ss, off);
    if constexpr (EPI == EPI_LN) sa += __shfl_xor(sa, off);
  }
  if (t % TPR == 0) {
    row_ss[grp][lr] = ss;
    row_sa[grp][lr] = sa;
  }
  __syncthreads();  // every group's products done: the stage buffers are free
  if constexpr (KS > 1) {
    // Groups 1.. hand their partial products to group 0, which adds them in group
    // order; thread t < BM of group 0 adds its row's sums the same way.
    static_assert((KS - 1) * RI * 4 * 256 * sizeof(float) <= sizeof(stg), "reduction buffer");
    float* red = reinterpret_cast<float*>(&stg[0]);
    if (grp > 0) {
#pragma unroll
      for (int i = 0; i < RI; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) red[(((grp - 1) * RI + i) * 4 + j) * 256 + t] = acc[i][j];
    } else if (t < BM) {
      ST s1 = row_ss[0][t], s2 = row_sa[0][t];
#pragma unroll
      for (int g = 1; g < KS; ++g) {
        s1 += row_ss[g][t];
        s2 += row_sa[g][t];
      }
      row_ss[0][t] = s1;
      row_sa[0][t] = s2;
    }
    __syncthreads();
    if (grp > 0) return;
#pragma unroll
    for (int g = 1; g < KS; ++g)
#pragma unroll
      for (int i = 0; i < RI; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] += red[(((g - 1) * RI + i) * 4 + j) * 256 + t];
  }

  using STE = StatT<EPI>;
  STE rss[RI], rsa[RI];
#pragma unroll
  for (int i = 0; i < RI; ++i) {
    rss[i] = row_ss[0][ty + 16 * i];
    rsa[i] = row_sa[0][ty + 16 * i];
  }
  f32_epilogue<EPI, RI, 4>(acc, rss, rsa, tx, ty, m0, p0, M, ncols, y, ldy, ep, blockIdx.x == 0);
}

// Few-row kernel.  A workgroup of 256 threads owns a 16-row tile of 4 CQ packed columns
// (CQ column quads) and splits K over KG = 64 / CQ groups of 4 CQ threads.  Group g takes
// the k quads g, g + KG, ...; its thread (rb, cb) keeps a 4 x 4 block of products (four
// rows of 4 rb.., column quad cb) and loads its operands straight from global memory as
// float4 (no LDS staging), PF quads ahead in registers.  The loads are range-checked
// buffer loads: a quad past K, a row past M or a column past NP reads zeros without
// touching memory, so no load sits behind a branch and the quads in flight stay in
// flight.  The thread also sums RS of its four rows (Cor. 1; LayerNorm on pivot-shifted
// values as in f32_kernel): its slots are rotated so that those rows are slots 0..RS-1.
// The groups' partials are added in LDS in a fixed order (deterministic).  CQ = 1, 2 or 4
// for the plain kinds (narrow tiles spread few rows over many workgroups: the 16-row
// tiny workload runs in 144 of them), 2 or 4 for a GLU (gate quads and the matching up
// quads, 16 columns apart in the packed layout), 16 for per-head norms (whole heads of
// up to 64 columns in one tile).
template <int EPI, bool GS, int CQ>
__global__ __launch_bounds__(256) void f32_few_rows_kernel(const float* __restrict__ a, int M, int K, int lda,
                                                           const float* __restrict__ ws, int NP, int ncols,
                                                           float* __restrict__ y, int ldy, EpiArgs ep) {
  constexpr bool kGlu = epi_is_glu(EPI);
  static_assert(EPI == EPI_HEADNORM ? CQ == 16 : kGlu ? (CQ == 2 || CQ == 4) : (CQ == 1 || CQ == 2 || CQ == 4),
                "tile width");
  constexpr int TG = 4 * CQ;                   // threads per k group
  constexpr int KG = 256 / TG;                 // k groups
  constexpr int NV = 4 * CQ;                   // values per tile row
  constexpr int RS = CQ >= 4 ? 1 : 4 / CQ;     // rows a thread sums
  constexpr int PF = 3;                        // k quads in flight per thread
  using ST = StatT<EPI>;
  __shared__ float red[KG][16][NV];
  __shared__ ST red_ss[KG][16], red_sa[KG][16];

  const int t = threadIdx.x;
  const int g = t / TG, u = t % TG;
  const int rb = u & 3, cb = u >> 2;
  // XCD-aware tile order: the workgroups of one XCD take neighbouring column tiles, so
  // the 128-byte weight lines that several narrow tiles share are fetched into one L2.
  int tm, tn;
  tile_of_block(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y, gridDim.y, gridDim.x, tm, tn);
  const int m0 = tm * 16;
  // Packed columns: plain tiles are 4 CQ consecutive columns; a GLU tile takes FQ = CQ / 2
  // gate quads of a 32-column block and the up quads 16 columns on.  p0e is the epilogue's
  // column origin (twice the first feature for a GLU).
  int colq, p0e;
  if constexpr (kGlu) {
    constexpr int FQ = CQ / 2, TPB = 4 / FQ;  // tiles per 32-column block
    const int blk = tn / TPB, sub = tn % TPB;
    const int fbase = 16 * blk + 4 * FQ * sub;
    colq = 32 * blk + 4 * FQ * sub + (cb < FQ ? 4 * cb : 16 + 4 * (cb - FQ));
    p0e = 2 * fbase;
  } else {
    p0e = tn * NV;
    colq = p0e + 4 * cb;
  }
  const int KQ = K >> 2;                                          // K is a multiple of 4
  const int rounds = ((KQ + KG - 1) / KG + PF - 1) / PF * PF;     // per group, whole batches of PF
  const int arows = M - m0 < 16 ? M - m0 : 16;
  // Extents end at the last valid element (lda >= K: a row past M starts beyond them).
  const __amdgpu_buffer_rsrc_t ars =
      make_rsrc(a + (int64_t)m0 * lda, (uint32_t)(((int64_t)(arows - 1) * lda + K) * 4));
  const __amdgpu_buffer_rsrc_t wrs = make_rsrc(ws, (uint32_t)((int64_t)K * NP * 4));
  const __amdgpu_buffer_rsrc_t grs = make_rsrc(GS ? ep.g_rt : nullptr, GS ? (uint32_t)K * 4 : 0u);
  const bool col_ok = colq < NP;
  // Slot i of the thread's four rows is row 4 rb + ((i + RS cb) & 3).
  int rrow[4];
  float piv[4];
  unsigned aoff[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    rrow[i] = 4 * rb + ((i + RS * cb) & 3);
    const int m = m0 + rrow[i];
    piv[i] = (EPI == EPI_LN && m < M) ? a[(int64_t)m * lda] : 0.f;
    aoff[i] = (unsigned)(rrow[i] * lda) * 4u;
  }
  const bool writes_stats = RS * cb < 4;

  // The load offsets pass through an empty asm so that the compiler keeps one load of a
  // selected offset (not two loads behind a branch).
  auto opaque = [](unsigned v) {
    asm volatile("" : "+v"(v));
    return v;
  };
  const unsigned woff = (unsigned)colq * 4u, wrow = (unsigned)NP * 4u;
  f32x4 A[PF][4], W[PF][4], G[PF];
  auto load = [&](int s, int r) {
    const int q = r * KG + g;
    const bool live = q < KQ, wlive = live & col_ok;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      A[s][i] = __builtin_bit_cast(f32x4, load_buf16(ars, opaque(live ? aoff[i] + (unsigned)q * 16u : kOobOffset)));
#pragma unroll
    for (int i = 0; i < 4; ++i)
      W[s][i] = __builtin_bit_cast(
          f32x4, load_buf16(wrs, opaque(wlive ? (unsigned)(4 * q + i) * wrow + woff : kOobOffset)));
    if constexpr (GS) G[s] = __builtin_bit_cast(f32x4, load_buf16(grs, opaque(live ? (unsigned)q * 16u : kOobOffset)));
  };

  float acc[4][4] = {};
  ST ss[RS] = {}, sa[RS] = {};
  auto compute = [&](int s, int r) {
    f32x4 av[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) av[i] = A[s][i];
    if constexpr (EPI == EPI_LN) {  // shift by the pivot; a quad past K stays zero
      const bool live = r * KG + g < KQ;
#pragma unroll
      for (int i = 0; i < 4; ++i) av[i] = live ? av[i] - piv[i] : f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int j = 0; j < RS; ++j) {
      if constexpr (EPI == EPI_LN) {  // fp64 sums: the squares of fp32 values are exact in fp64
        const double x = av[j].x, yv = av[j].y, z = av[j].z, w = av[j].w;
        ss[j] += (x * x + yv * yv) + (z * z + w * w);
        sa[j] += (x + yv) + (z + w);
      } else {
        ss[j] = fmaf(av[j].x, av[j].x, ss[j]);
        ss[j] = fmaf(av[j].y, av[j].y, ss[j]);
        ss[j] = fmaf(av[j].z, av[j].z, ss[j]);
        ss[j] = fmaf(av[j].w, av[j].w, ss[j]);
      }
    }
    if constexpr (GS) {  // run-time g (unfolded W): a_k g_k in fp32
#pragma unroll
      for (int i = 0; i < 4; ++i) av[i] *= G[s];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        acc[i][c] = fmaf(av[i].x, W[s][0][c], acc[i][c]);
        acc[i][c] = fmaf(av[i].y, W[s][1][c], acc[i][c]);
        acc[i][c] = fmaf(av[i].z, W[s][2][c], acc[i][c]);
        acc[i][c] = fmaf(av[i].w, W[s][3][c], acc[i][c]);
      }
  };

#pragma unroll
  for (int s = 0; s < PF; ++s) load(s, s);
  for (int r0 = 0; r0 < rounds; r0 += PF) {
#pragma unroll
    for (int s = 0; s < PF; ++s) {
      compute(s, r0 + s);
      load(s, r0 + s + PF);
    }
  }

#pragma unroll
  for (int i = 0; i < 4; ++i)
    *reinterpret_cast<f32x4*>(&red[g][rrow[i]][4 * cb]) = f32x4{acc[i][0], acc[i][1], acc[i][2], acc[i][3]};
  if (writes_stats) {
#pragma unroll
    for (int j = 0; j < RS; ++j) {
      red_ss[g][rrow[j]] = ss[j];
      red_sa[g][rrow[j]] = sa[j];
    }
  }
  __syncthreads();

  if constexpr (CQ == 16) {
    // 1024 values: thread (tx, ty) adds the KG partials of row ty, columns tx + 16 j.
    const int tx = t & 15, ty = t >> 4;
    float out[1][4];
    ST rss[1] = {ST(0)}, rsa[1] = {ST(0)};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float v = red[0][ty][tx + 16 * j];
#pragma unroll
      for (int k = 1; k < KG; ++k) v += red[k][ty][tx + 16 * j];
      out[0][j] = v;
    }
#pragma unroll
    for (int k = 0; k < KG; ++k) {
      rss[0] += red_ss[k][ty];
      rsa[0] += red_sa[k][ty];
    }
    f32_epilogue<EPI, 1, 4>(out, rss, rsa, tx, ty, m0, p0e, M, ncols, y, ldy, ep, tn == 0);
  } else {
    // 16 NV values, TPV = 4 / CQ threads each adding a contiguous run of KG / TPV
    // partials; then one thread per value adds the TPV runs in order.
    constexpr int V = 16 * NV, TPV = 256 / V, RUN = KG / TPV;
    __shared__ float part[TPV][V];
    __shared__ ST row_ss[16], row_sa[16];
    {
      const int v = t % V, pr = t / V;
      const int row = v / NV, col = v % NV;
      float sum = red[pr * RUN][row][col];
#pragma unroll 8
      for (int k = 1; k < RUN; ++k) sum += red[pr * RUN + k][row][col];
      part[pr][v] = sum;
    }
    if (t < 16) {
      ST s1 = ST(0), s2 = ST(0);
#pragma unroll 8
      for (int k = 0; k < KG; ++k) {
        s1 += red_ss[k][t];
        s2 += red_sa[k][t];
      }
      row_ss[t] = s1;
      row_sa[t] = s2;
    }
    __syncthreads();
    auto value = [&](int v) {
      float sum = part[0][v];
#pragma unroll
      for (int p = 1; p < TPV; ++p) sum += part[p][v];
      return sum;
    };
    if constexpr (kGlu) {
      constexpr int FW = NV / 2;  // features per tile row
      if (t >= 16 * FW) return;   // whole waves
      const int tx = t % FW, ty = t / FW;
      float out[1][2] = {{value(ty * NV + tx), value(ty * NV + FW + tx)}};
      const ST rss[1] = {row_ss[ty]}, rsa[1] = {row_sa[ty]};
      f32_epilogue<EPI, 1, 2>(out, rss, rsa, tx, ty, m0, p0e, M, ncols, y, ldy, ep, tn == 0);
    } else {
      if (t >= V) return;  // whole waves
      const int tx = t % NV, ty = t / NV;
      float out[1][1] = {{value(t)}};
      const ST rss[1] = {row_ss[ty]}, rsa[1] = {row_sa[ty]};
      f32_epilogue<EPI, 1, 1>(out, rss, rsa, tx, ty, m0, p0e, M, ncols, y, ldy, ep, tn == 0);
    }
  }
}

// Matrix-core kernel: fp32 operands, fp32 products and sums (v_mfma_f32_16x16x4_f32, whose
// operands are not rounded).  A workgroup owns 16 MB rows x 64 packed columns, and its KS waves
// split K: wave w takes the 16-deep k blocks w, w + KS, ... and holds the whole tile's partial
// products, so nothing is staged or read twice inside a workgroup and the K loop has no barrier.
//
// Operands.  Lane l = 16 q + r loads the activations of row r, k = 4 q .. 4 q + 3 of the block
// (one float4 per 16 rows: 64 contiguous bytes of each row) and, for e = 0..3, the weights of
// k = 4 q + e, columns 4 r .. 4 r + 3 (256 contiguous bytes of each k).  Matrix-core op (t, e, j)
// multiplies element e of row block t with component j of weight e: its four k are 4 q + e and
// its sixteen columns 4 r + j, an order of K and of the columns that both operands share.  The
// lane ends with row r and, over j, four consecutive columns 16 q + 4 i .. 4 i + 3 for every
// accumulator component i.  Loads run one block ahead in registers, 16 MB matrix-core ops of 32
// cycles before their use.
//
// Bound by the fp32 matrix rate (154 TFLOP/s measured with a large product) where the tiles
// fill the chip.  500 x 2048 -> 2048: 163 us on the vector units (f32_kernel, whose operands
// come from LDS one value per multiply-add), 38.7 us here.
template <int EPI, bool GS, int MB, int KS>
__global__ __launch_bounds__(64 * KS, 1) void f32_mfma_kernel(const float* __restrict__ a, int M, int K, int lda,
                                                              const float* __restrict__ ws, int NP, int KP,
                                                              int ncols, float* __restrict__ y, int ldy, EpiArgs ep) {
  using ST = StatT<EPI>;
  constexpr bool kLN = EPI == EPI_LN, kSS = epi_needs_ss(EPI);
  constexpr int BM = 16 * MB, LDT = 68;  // rows; floats per staged row (16 rows of one column: 16 bank groups)
  __shared__ __attribute__((aligned(16))) float part[KS][BM][LDT];
  __shared__ ST row_ss[KS][BM], row_sa[KS][BM];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (NP + 63) / 64;
  const int64_t bid = blockIdx.x + (int64_t)gridDim.x * blockIdx.y;
  if (bid >= (int64_t)tiles_m * tiles_n) return;  // the last row of a grid of more than kF32GridX tiles
  int tm, tn;
  tile_of_block((int)bid, tiles_m * tiles_n, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * BM, p0 = tn * 64;
  const int r = lane & 15, q = lane >> 4;
  const int rows = min(BM, M - m0);
  const __amdgpu_buffer_rsrc_t ars =
      make_rsrc(a + (int64_t)m0 * lda, (uint32_t)(((int64_t)(rows - 1) * lda + K) * 4));
  const __amdgpu_buffer_rsrc_t wrs = make_rsrc(ws, (uint32_t)((int64_t)KP * NP * 4));
  const __amdgpu_buffer_rsrc_t grs = make_rsrc(GS ? ep.g_rt : nullptr, GS ? (uint32_t)K * 4 : 0u);
  const bool col_ok = p0 + 4 * r < NP;  // NP is a multiple of 16: a quad is wholly inside or outside
  const unsigned woff = (unsigned)(p0 + 4 * r) * 4u, wrow = (unsigned)NP * 4u;

  float piv[MB];
#pragma unroll
  for (int t = 0; t < MB; ++t) piv[t] = kLN && m0 + 16 * t + r < M ? a[(int64_t)(m0 + 16 * t + r) * lda] : 0.0f;

  // Offsets past an operand are selected to one that reads zeros (through an empty asm, so that
  // the compiler keeps one load of a selected offset).  K is a multiple of 4.
  auto opaque = [](unsigned v) {
    asm volatile("" : "+v"(v));
    return v;
  };
  auto load = [&](int kb, f32x4 (&A)[MB], f32x4 (&W)[4], f32x4& G) __attribute__((always_inline)) {
    const int k = kb * 16 + 4 * q;
    const bool live = k < K;
#pragma unroll
    for (int t = 0; t < MB; ++t)
      A[t] = __builtin_bit_cast(
          f32x4, load_buf16(ars, opaque(live ? (unsigned)((16 * t + r) * lda + k) * 4u : kOobOffset)));
#pragma unroll
    for (int e = 0; e < 4; ++e)
      W[e] = __builtin_bit_cast(
          f32x4, load_buf16(wrs, opaque(live && col_ok ? (unsigned)(k + e) * wrow + woff : kOobOffset)));
    if constexpr (GS) G = __builtin_bit_cast(f32x4, load_buf16(grs, opaque(live ? (unsigned)k * 4u : kOobOffset)));
  };

  constexpr int ES = 4 / MB;  // chains of sums per output, over e % ES: K / (4 KS ES) ops long
  f32x4 acc[ES][MB][4];
  ST ss[MB], sa[MB];
#pragma unroll
  for (int t = 0; t < MB; ++t) {
    ss[t] = sa[t] = ST(0);
#pragma unroll
    for (int s = 0; s < ES; ++s)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[s][t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  auto compute = [&](int kb, f32x4 (&A)[MB], const f32x4 (&W)[4], const f32x4& G) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < MB; ++t) {
      f32x4 av = A[t];
      if constexpr (kLN) {  // shifted by the row's pivot; a quad past K stays zero
        const float p = kb * 16 + 4 * q < K ? piv[t] : 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e) av[e] -= p;
        const double x = av[0], yv = av[1], z = av[2], w = av[3];
        ss[t] += (x * x + yv * yv) + (z * z + w * w);
        sa[t] += (x + yv) + (z + w);
      } else if constexpr (kSS) {
#pragma unroll
        for (int e = 0; e < 4; ++e) ss[t] = fmaf(av[e], av[e], ss[t]);
      }
      if constexpr (GS) {  // run-time g (unfolded W): a_k g_k in fp32
#pragma unroll
        for (int e = 0; e < 4; ++e) av[e] *= G[e];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[e % ES][t][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(W[e][j], av[e], acc[e % ES][t][j], 0, 0, 0);
    }
  };

  const int KB = (K + 15) / 16;
  f32x4 A0[MB], A1[MB], W0[4], W1[4], G0, G1;
  load(wave, A0, W0, G0);
  for (int kb = wave; kb < KB; kb += 2 * KS) {
    load(kb + KS, A1, W1, G1);
    __builtin_amdgcn_sched_barrier(0);
    compute(kb, A0, W0, G0);
    __builtin_amdgcn_sched_barrier(0);
    load(kb + 2 * KS, A0, W0, G0);
    __builtin_amdgcn_sched_barrier(0);
    compute(kb + KS, A1, W1, G1);
    __builtin_amdgcn_sched_barrier(0);
  }

  // Partials to LDS, added over the waves in order (deterministic) by the threads that finish
  // them: thread (tx, ty) of 256-thread group g takes rows ty + 16 i of the group's share and
  // columns tx + 16 j, as the other fp32 kernels' epilogue.
#pragma unroll
  for (int t = 0; t < MB; ++t) {
    if constexpr (kSS) {
      ss[t] += __shfl_xor(ss[t], 16);
      ss[t] += __shfl_xor(ss[t], 32);
      if constexpr (kLN) {
        sa[t] += __shfl_xor(sa[t], 16);
        sa[t] += __shfl_xor(sa[t], 32);
      }
    }
    if (lane < 16) {
      row_ss[wave][16 * t + r] = ss[t];
      row_sa[wave][16 * t + r] = sa[t];
    }
#pragma unroll
    for (int s = 1; s < ES; ++s)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[0][t][j] += acc[s][t][j];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      *reinterpret_cast<f32x4*>(&part[wave][16 * t + r][16 * q + 4 * i]) =
          f32x4{acc[0][t][0][i], acc[0][t][1][i], acc[0][t][2][i], acc[0][t][3][i]};
  }
  __syncthreads();
  constexpr int EG = MB < KS / 4 ? MB : KS / 4, RI = MB / EG;  // finishing groups, row blocks of each
  const int grp = threadIdx.x >> 8, tx = threadIdx.x & 15, ty = (threadIdx.x >> 4) & 15;
  if (grp >= EG) return;
  float out[RI][4];
  ST rss[RI], rsa[RI];
#pragma unroll
  for (int i = 0; i < RI; ++i) {
    const int row = 16 * (grp * RI + i) + ty;
    rss[i] = rsa[i] = ST(0);
#pragma unroll
    for (int j = 0; j < 4; ++j) out[i][j] = part[0][row][tx + 16 * j];
#pragma unroll
    for (int w = 0; w < KS; ++w) {
      rss[i] += row_ss[w][row];
      rsa[i] += row_sa[w][row];
      if (w > 0) {
#pragma unroll
        for (int j = 0; j < 4; ++j) out[i][j] += part[w][row][tx + 16 * j];
      }
    }
  }
  f32_epilogue<EPI, RI, 4>(out, rss, rsa, tx, ty, m0 + 16 * grp * RI, p0, M, ncols, y, ldy, ep, tn == 0);
}

// Tile configurations (kF32CfgCount): 0 automatic; by name, 1 = 64-row vector tiles with one k
// group, 2 = 16-row vector tiles of 64 columns with four k groups, 3 = the few-row kernel.
//
// Automatic (2222 random shapes of 1..2048 rows, K 64..4096, 8..8192 columns, linear and GLU,
// on MI355X): the few-row kernel when 16 x 64 tiles would be 32 or fewer (its narrow tiles
// spread them over more units: 16 x 576 -> 576 6.1 us, 7.0 on the matrix cores), for one or
// two rows of up to 64 tiles (1 x 332 -> 4084: 5.5 and 6.6), and for up to 64 tiles of at most 16
// columns from K = 256 on (its 4-column tiles still fit one round, and three quarters of a 64-column
// tile would be padding: 958 x 2380 -> 6 9.4 us, 15.1 on the matrix cores; from 65 tiles, or 17
// columns, on those are the faster; of a GLU's 32 packed columns only where the rows' pitch is an
// odd number of 16 bytes, which splits the 64 bytes that the matrix-core kernel loads of a row:
// 731 x 2052 -> 2 x 4 10.9 and 13.1 us, at K = 2048 the other way by 2%).  Otherwise the
// matrix-core kernel:
// 32-row tiles with four waves from 384 tiles on (1024 x 2048 -> 4096: 146 us, 170 with 16
// rows), else 16-row tiles, with four waves from 128 tiles and eight below (64 x 2048 -> 2048:
// 14.3 us, 14.9 with four).  500 x 2048 -> 2048: 163 us on the vector kernels, 38.7 so;
// 16 x 2048 -> 8192: 162 and 15.  Over 1500 fresh shapes the choice takes 0.74 of the vector
// kernels' time, three run over 5% slower, at worst 10% (580 x 3772 -> 27).  The error against fp64 is at most the vector kernels': a chain of
// sums is K / 64 (32 rows: K / 32) ops long and shorter with eight waves.

// Workgroups along x of a matrix-core grid (times 512 threads stays below 2^32); more go along y.
constexpr int64_t kF32GridX = 1 << 22;

template <int EPI, bool GS, int MB, int KS>
static hipError_t launch_f32_mfma(const F32Args& p) {
  const int64_t tiles = (int64_t)((p.NP + 63) / 64) * ((p.M + 16 * MB - 1) / (16 * MB));
  if (tiles > INT32_MAX) return hipErrorInvalidValue;
  const int64_t gx = tiles < kF32GridX ? tiles : kF32GridX;
  const dim3 grid((unsigned)gx, (unsigned)((tiles + gx - 1) / gx));
  hipLaunchKernelGGL((f32_mfma_kernel<EPI, GS, MB, KS>), grid, dim3(64 * KS), 0, p.stream, p.a, p.M, p.K, p.lda, p.ws,
                     p.NP, p.KP, p.ncols, p.y, p.ldy, p.ep);
  return hipGetLastError();
}

template <int EPI, bool GS = false>
static hipError_t launch_f32_epi(const F32Args& p) {
  int cfg = p.cfg;
  if (cfg == 0) {
    const int64_t nt = (p.NP + 63) / 64, tiles = nt * ((p.M + 15) / 16);
    const bool sliver = tiles <= 64 && p.K >= 256 &&
                        (epi_is_glu(EPI) ? p.NP == 32 && p.lda % 8 : p.NP == 16 && EPI != EPI_HEADNORM);
    if (tiles <= 32 || (p.M <= 2 && nt <= 64) || sliver) {
      cfg = 3;
    } else if (nt * ((p.M + 31) / 32) >= 384) {
      return launch_f32_mfma<EPI, GS, 2, 4>(p);
    } else {
      return tiles >= 128 ? launch_f32_mfma<EPI, GS, 1, 4>(p) : launch_f32_mfma<EPI, GS, 1, 8>(p);
    }
  }
  if (cfg == 1 || cfg == 2) {
    // Only the core kinds can name a configuration (the others return FN_ERR_UNSUPPORTED for one).
    if constexpr (EPI < EPI_REGLU && !GS) {
      if (cfg == 1) {
        dim3 grid((p.NP + 63) / 64, (p.M + 63) / 64);
        hipLaunchKernelGGL((f32_kernel<EPI, 4, 1>), grid, dim3(256), 0, p.stream, p.a, p.M, p.K, p.lda, p.ws,
                           p.NP, p.ncols, p.y, p.ldy, p.ep);
      } else {
        dim3 grid((p.NP + 63) / 64, (p.M + 15) / 16);
        hipLaunchKernelGGL((f32_kernel<EPI, 1, 4>), grid, dim3(1024), 0, p.stream, p.a, p.M, p.K, p.lda, p.ws,
                           p.NP, p.ncols, p.y, p.ldy, p.ep);
      }
    } else {
      return hipErrorInvalidValue;
    }
  } else {
    // Column quads per tile: the widest of 4, 2, 1 that still makes FEW_MIN_WG workgroups.
    const int64_t mt = (p.M + 15) / 16;
    auto wgs = [&](int cq) { return (int64_t)((p.NP + 4 * cq - 1) / (4 * cq)) * mt; };
    const int cq = EPI == EPI_HEADNORM ? 16
                   : wgs(4) >= FEW_MIN_WG ? 4
                   : (wgs(2) >= FEW_MIN_WG || epi_is_glu(EPI)) ? 2
                                                                : 1;
    auto go = [&](auto kern, int cqv) {
      dim3 grid((p.NP + 4 * cqv - 1) / (4 * cqv), mt);
      hipLaunchKernelGGL(kern, grid, dim3(256), 0, p.stream, p.a, p.M, p.K, p.lda, p.ws, p.NP, p.ncols, p.y,
                         p.ldy, p.ep);
    };
    if constexpr (EPI == EPI_HEADNORM) {
      go(f32_few_rows_kernel<EPI, GS, 16>, 16);
    } else {
      if (cq == 4) go(f32_few_rows_kernel<EPI, GS, 4>, 4);
      else if (cq == 2) go(f32_few_rows_kernel<EPI, GS, 2>, 2);
      else if constexpr (!epi_is_glu(EPI)) go(f32_few_rows_kernel<EPI, GS, 1>, 1);
    }
  }
  return hipGetLastError();
}

hipError_t launch_f32(const F32Args& p) {
  if (p.cfg < 0 || p.cfg >= kF32CfgCount) return hipErrorInvalidValue;
  if (p.gs) {  // run-time g: RMS kinds
    if (p.epi == EPI_RMS) return launch_f32_epi<EPI_RMS, true>(p);
    if (p.epi == EPI_GLU) return launch_f32_epi<EPI_GLU, true>(p);
    return hipErrorInvalidValue;
  }
  switch (p.epi) {
    case EPI_RMS: return launch_f32_epi<EPI_RMS>(p);
    case EPI_GLU: return launch_f32_epi<EPI_GLU>(p);
    case EPI_LN: return launch_f32_epi<EPI_LN>(p);
    case EPI_NONE: return launch_f32_epi<EPI_NONE>(p);
    case EPI_GLU_NOSCALE: return launch_f32_epi<EPI_GLU_NOSCALE>(p);
    case EPI_REGLU: return launch_f32_epi<EPI_REGLU>(p);
    case EPI_BILINEAR: return launch_f32_epi<EPI_BILINEAR>(p);
    case EPI_GLU_DEFER: return launch_f32_epi<EPI_GLU_DEFER>(p);
    case EPI_RELU_DEFER: return launch_f32_epi<EPI_RELU_DEFER>(p);
    case EPI_ROWSCALE: return launch_f32_epi<EPI_ROWSCALE>(p);
    case EPI_ROPE: return launch_f32_epi<EPI_ROPE>(p);
    case EPI_HEADNORM: return launch_f32_epi<EPI_HEADNORM>(p);
  }
  return hipErrorInvalidValue;
}

}  // namespace fn

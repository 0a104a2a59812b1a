// Middle-row fused norm-then-project kernel for gfx950: more rows than the decode kernel
// takes and too few tiles for the many-row kernel to fill the chip.
//
// What bounds it: the weight stream while the rows are few, then how many compute units work
// and how many bytes each keeps in flight (128-row tiles give 3 x 128 = 384 tiles of uneven
// rounds at 333 x 4096 -> 12288, and 8 tiles, 8 busy units of 256, at 32 x 8192 -> 1024).
//
// Split.  A workgroup owns 16 MB rows and CW NCB packed column blocks of 16; its CW KS waves
// are CW column waves times KS k groups.  K is walked in sets of S = U KS k blocks, group kg
// takes k blocks kg U .. kg U + U - 1 of each.  The weights go from memory straight into the
// registers of the one wave that multiplies them (16 bytes per lane, the packed order is the
// operand order), one set ahead.  The activations are read by every column wave: the workgroup
// loads them row-contiguously two sets ahead (4 S lanes read one row's 64 S bytes), and puts
// them into a double-buffered LDS stage in the matrix-core order, where every fragment read is
// linear in the lane; the position of row r is XORed with its chunk and k block, so that the
// 16 lanes that write one row's units hit 16 different bank groups.  The fragment reads run D
// steps ahead of the matrix cores.  The k groups' partial products meet in LDS in a fixed
// order (deterministic), each group finishing its share of the row blocks.
//
// The waves of a workgroup share the row statistics: column wave cw walks the row blocks from
// block cw TWM on and takes the sums of the first TWM it meets (RMS kinds: the diagonal of the
// fragment's Gram block; LayerNorm: packed dot products added in fp64).
//
// Measured on MI355X against the 128-row tiles (graph replay): 64 x 4096 -> 2 x 11008 GLU
// 43.3 -> 33.0 us, 64 x 4096 -> 4096 24.8 -> 10.5, 32 x 8192 -> 1024 44.2 -> 14.7, 333 x 4096
// -> 12288 62.4 -> 48.3, 1024 x 5120 -> 576 33.5 -> 19.3.  Slower and not kept: register rings
// of three and four sets (35.1 -> 37..39 us at 64 rows GLU) and a step sequence over a
// three-slot LDS ring with the barrier inside it (37.1).
#pragma once

#include <type_traits>

#include "fn_device.h"
#include "fn_epilogue.h"
#include "fn_launch.h"
#include "fn_tile.h"

namespace fn {

template <int MB, int NCB, int CW, int KS, int U, int EPI, int CPOL>
__global__ __launch_bounds__(64 * CW * KS, 1) void mid_bf16_kernel(
    const __bf16* __restrict__ a, int M, int K, int lda, const __bf16* __restrict__ ws, int NP, int KP, int ncols,
    __bf16* __restrict__ y, int ldy, EpiArgs ep, int groups) {
  constexpr int NW = CW * KS, S = U * KS;  // waves; k blocks per set
  constexpr bool kSS = epi_needs_ss(EPI), kSA = EPI == EPI_LN, kGram = kSS && !kSA;
  constexpr int TWM = (MB + CW - 1) / CW;     // row blocks whose statistics a wave takes
  constexpr int NU = (MB * S + NW - 1) / NW;  // activation units (16 bytes) per thread and set
  constexpr int RPI = 16 * CW / U;            // rows between a thread's units
  static_assert((16 * CW) % U == 0, "a thread's units share their chunk of the row");
  static_assert(!epi_is_glu(EPI) || NCB % 2 == 0, "GLU needs gate/up block pairs");
  using ST = StatT<EPI>;
  constexpr int MBS = ((16 * MB + RPI - 1) / RPI * RPI + 15) / 16;  // staged row blocks (whole rounds of units)
  static_assert(MBS * 16 >= NU * RPI, "every unit a thread writes has a place");
  constexpr int STAGE_UNITS = S * MBS * 64;
  constexpr int RED_UNITS = (KS - 1) * MB * CW * NCB * 64;
  __shared__ u32x4 smem[2 * STAGE_UNITS > RED_UNITS ? 2 * STAGE_UNITS : RED_UNITS];
  __shared__ ST row_ss[kSS ? KS : 1][kSS ? MB * 16 : 1], row_sa[kSA ? KS : 1][kSA ? MB * 16 : 1];

  // Workgroup -> (column tile, row group): ids go to the 8 XCDs in turn; each XCD takes a
  // contiguous range of the (tile, group) pairs, so the row groups of a column tile share its
  // weights in one L2 and every XCD gets the same number of workgroups (within one).
  const int q8 = gridDim.x / kXcds, r8 = gridDim.x % kXcds, x8 = blockIdx.x % kXcds;
  const int logical = x8 * q8 + min(x8, r8) + blockIdx.x / kXcds;
  const int tile = logical / groups, grp = logical % groups;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int cw = wave % CW, kg = wave / CW;
  const int cb0 = (tile * CW + cw) * NCB;
  const int KB = KP / kKB, npb = NP / 16;
  const int m0 = grp * (16 * MB);
  const int rows = min(16 * MB, M - m0);

  // Range-checked views.  Rows past M lie past the extent (lda >= K) and read zeros; column
  // blocks past the packed width (last tile only) read the next k block's fragments or zeros,
  // and feed columns that are never stored.
  const __amdgpu_buffer_rsrc_t rs_a =
      make_rsrc(a + (int64_t)m0 * lda, (uint32_t)(((int64_t)(rows - 1) * lda + K) * 2));
  const int64_t w_extent = ((int64_t)KB * npb - cb0) * kFragBytes;
  const __amdgpu_buffer_rsrc_t rs_w =
      make_rsrc(ws + (int64_t)cb0 * (kFragBytes / 2), (uint32_t)(w_extent > 0 ? w_extent : 0));

  const int lrow = lane & 15, lch = lane >> 4;
  // Staging: unit n = (i NW + wave) 64 + lane of the set's 16 MB rows x 4 S chunks, row-major.
  const int n0u = wave * 64 + lane;
  const int ur = n0u / (4 * S), uq = n0u % (4 * S);  // first row; chunk of the set (the same for every unit)
  const int uu = uq >> 2, uc = uq & 3;
  const int ukt = uu * kKB + uc * 8;
  auto slot = [](int u, int rb, int r, int c) { return (u * MBS + rb) * 64 + 16 * c + (r ^ (c + 4 * (u & 3))); };
  auto load_act = [&](int kb0, u32x4 (&af)[NU]) __attribute__((always_inline)) {
    const int kt = kb0 * kKB + ukt;
    const unsigned off = (unsigned)(ur * lda + kt) * 2;
#pragma unroll
    for (int i = 0; i < NU; ++i)
      af[i] = load_buf16(rs_a, kt < K ? off + (unsigned)(i * RPI * lda) * 2 : kOobOffset);
  };
  auto put_act = [&](int buf, const u32x4 (&af)[NU]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NU; ++i) {
      const int r = ur + i * RPI;
      smem[buf * STAGE_UNITS + slot(uu, r >> 4, r & 15, uc)] = af[i];
    }
  };
  auto load_w = [&](int kb0, u32x4 (&wf)[U][NCB]) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kb = kb0 + kg * U + u;
#pragma unroll
      for (int c = 0; c < NCB; ++c)
        wf[u][c] = load_buf16<CPOL>(rs_w, kb < KB ? (unsigned)((kb * npb + c) * kFragBytes + lane * 16) : kOobOffset);
    }
  };

  f32x4 acc[MB][NCB], gsq[kGram ? TWM : 1];
  ST ss[TWM], sa[TWM];
#pragma unroll
  for (int t = 0; t < MB; ++t)
#pragma unroll
    for (int c = 0; c < NCB; ++c) acc[t][c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < TWM; ++t) {
    ss[t] = sa[t] = ST(0);
    if (kGram) gsq[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  int boff[MB];  // stage units of the row block that step t works on
#pragma unroll
  for (int t = 0; t < MB; ++t) boff[t] = (t + cw * TWM) % MB * 64;
  int rd[U];
#pragma unroll
  for (int u = 0; u < U; ++u) rd[u] = slot(kg * U + u, 0, lrow, lch);

  auto compute = [&](int buf, const u32x4 (&wf)[U][NCB]) __attribute__((always_inline)) {
    constexpr int STEPS = U * MB, D = STEPS < 4 ? STEPS : 4;
    u32x4 av[D];
    auto read = [&](int s) __attribute__((always_inline)) {
      av[s % D] = smem[buf * STAGE_UNITS + boff[s % MB] + rd[s / MB]];
    };
#pragma unroll
    for (int s = 0; s < D; ++s) read(s);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      const int u = s / MB, t = s % MB;
      const bf16x8 af = __builtin_bit_cast(bf16x8, av[s % D]);
      if (t < TWM) {
        if constexpr (kSA) {
          ss[t] += (double)sumsq8(af, 0.0f);
          sa[t] += (double)sum8(af, 0.0f);
        } else if constexpr (kGram) {
          gsq[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, af, gsq[t], 0, 0, 0);
        }
      }
#pragma unroll
      for (int c = 0; c < NCB; ++c)
        acc[t][c] =
            __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wf[u][c]), af, acc[t][c], 0, 0, 0);
      if (s + D < STEPS) read(s + D);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // Set s: its weights were issued during set s - 1, its activations during set s - 2, and put
  // into slot s % 2 during set s - 1.  The barrier of set s orders those writes before this
  // set's reads, and every wave's reads of slot (s + 1) % 2 during set s - 1 before it is
  // rewritten here.  Sets past K multiply zeros.
  u32x4 a0[NU], a1[NU], w0[U][NCB], w1[U][NCB];
  load_act(0, a0);
  load_act(S, a1);
  load_w(0, w0);
  put_act(0, a0);
  for (int kb0 = 0; kb0 < KB; kb0 += 2 * S) {
    load_act(kb0 + 2 * S, a0);
    load_w(kb0 + S, w1);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    put_act(1, a1);
    compute(0, w0);
    __builtin_amdgcn_sched_barrier(0);
    load_act(kb0 + 3 * S, a1);
    load_w(kb0 + 2 * S, w0);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    put_act(0, a0);
    compute(1, w1);
    __builtin_amdgcn_sched_barrier(0);
  }

  // Row totals: wave (kg, cw) holds those of its k blocks for the row blocks it took.
  if constexpr (kSS) {
#pragma unroll
    for (int t = 0; t < TWM; ++t) {
      if constexpr (kGram) {  // row m's diagonal element: lane 20 (m / 4) + m % 4, component m % 4
        const f32x4 g = gsq[t];
        const float d = (lane & 2) ? ((lane & 1) ? g[3] : g[2]) : ((lane & 1) ? g[1] : g[0]);
        ss[t] = __shfl(d, lrow + 16 * (lrow >> 2));
      } else {
        ss[t] += __shfl_xor(ss[t], 16);
        ss[t] += __shfl_xor(ss[t], 32);
        sa[t] += __shfl_xor(sa[t], 16);
        sa[t] += __shfl_xor(sa[t], 32);
      }
      if (lane < 16 && t + cw * TWM < MB) {
        row_ss[kg][boff[t] / 4 + lane] = ss[t];
        if constexpr (kSA) row_sa[kg][boff[t] / 4 + lane] = sa[t];
      }
    }
  }
  // Partial products of the k groups: the row block of step t is finished by group t % KS.
  f32x4* red = reinterpret_cast<f32x4*>(smem);
  auto red_at = [&](int g, int t, int c) {  // group g's partial of (t, c), g != t % KS
    const int gi = g < t % KS ? g : g - 1;
    return (((gi * MB + t) * CW + cw) * NCB + c) * 64 + lane;
  };
  __syncthreads();
  if constexpr (KS > 1) {
#pragma unroll
    for (int t = 0; t < MB; ++t)
      if (t % KS != kg) {
#pragma unroll
        for (int c = 0; c < NCB; ++c) red[red_at(kg, t, c)] = acc[t][c];
      }
    __syncthreads();
  }
  const int n_lane = lch * 4;
  auto epilogue = [&](auto vec_tag) __attribute__((always_inline)) {
    constexpr bool VEC = decltype(vec_tag)::value;
#pragma unroll
    for (int t = 0; t < MB; ++t) {
      if (KS > 1 && t % KS != kg) continue;
      if constexpr (KS > 1) {
#pragma unroll
        for (int c = 0; c < NCB; ++c) {
          f32x4 v = t % KS == 0 ? acc[t][c] : red[red_at(0, t, c)];
#pragma unroll
          for (int g = 1; g < KS; ++g) v += g == t % KS ? acc[t][c] : red[red_at(g, t, c)];
          acc[t][c] = v;
        }
      }
      const int rl = boff[t] / 4 + lrow, m = m0 + rl;
      if (m >= M) continue;
      ST s1 = ST(0), s2 = ST(0);
      if constexpr (kSS) {
#pragma unroll
        for (int g = 0; g < KS; ++g) {
          s1 += row_ss[g][rl];
          if constexpr (kSA) s2 += row_sa[g][rl];
        }
      }
      const RowStat st = row_stat_at<EPI>(s1, s2, ep, m, M);
      if constexpr (epi_exports_s(EPI)) {
        if (ep.inv_rms && tile == 0 && cw == 0 && lane < 16) ep.inv_rms[m] = st.s;
      }
      constexpr int STEP = epi_is_glu(EPI) ? 2 : 1;
#pragma unroll
      for (int c = 0; c < NCB; c += STEP) {
        const int n = (cb0 + c) / STEP * 16;
        if (n + 16 <= ncols)
          store4_bf16_full<EPI, VEC>(y, ldy, m, n + n_lane, acc[t][c], acc[t][c + STEP - 1], st, ep);
        else
          store4_bf16_edge<EPI, VEC>(y, ldy, M, ncols, m, n + n_lane, acc[t][c], acc[t][c + STEP - 1], st, ep);
      }
    }
  };
  if (epi_vec<EPI>(ep) != nullptr)
    epilogue(std::true_type{});
  else
    epilogue(std::false_type{});
}

template <int MB, int NCB, int CW, int KS, int EPI, int CPOL = 0>
static hipError_t launch_mid_cfg(const PrefillArgs& p) {
  // Two k blocks per group and set for the four- and eight-block shapes: 48 x 4096 -> 12288 24.5 ->
  // 22.6 us, 96 x 5120 -> 15360 42.0 -> 38.0, elsewhere -4 to +4%.  The others lose by it: two-block
  // shapes 2 to 7%, the 112-row one 2 to 5% (333 x 4096 -> 12288 49.2 -> 51.8), 96 rows x 16 blocks
  // 3 to 5%; six-block shapes are within 3% either way.
  constexpr int U = NCB * CW == 4 || NCB * CW == 8 ? 2 : 1;
  const int groups = (p.M + 16 * MB - 1) / (16 * MB);
  const int col_tiles = (p.NP / 16 + NCB * CW - 1) / (NCB * CW);
  hipLaunchKernelGGL((mid_bf16_kernel<MB, NCB, CW, KS, U, EPI, CPOL>), dim3(col_tiles * groups),
                     dim3(64 * CW * KS), 0, p.stream, p.a, p.M, p.K, p.lda, p.ws, p.NP, p.KP, p.ncols, p.y, p.ldy,
                     p.ep, groups);
  return hipGetLastError();
}

// The shapes of mid_bf16.hip's table, in its order.
template <int EPI>
hipError_t launch_mid_epi(const PrefillArgs& p, int shape) {
  switch (shape) {
    case 0: return launch_mid_cfg<2, 2, 1, 8, EPI>(p);
    case 1: return launch_mid_cfg<2, 2, 2, 4, EPI>(p);
    case 2: return launch_mid_cfg<2, 2, 3, 4, EPI>(p);
    case 3: return launch_mid_cfg<3, 2, 1, 8, EPI>(p);
    case 4: return launch_mid_cfg<3, 2, 2, 4, EPI>(p);
    case 5: return launch_mid_cfg<3, 2, 3, 4, EPI>(p);
    case 6: return launch_mid_cfg<4, 2, 1, 8, EPI>(p);
    case 7: return launch_mid_cfg<4, 2, 2, 4, EPI>(p);
    case 8: return launch_mid_cfg<4, 2, 3, 4, EPI>(p);
    case 9: return launch_mid_cfg<6, 2, 3, 4, EPI>(p);
    case 10: return launch_mid_cfg<6, 4, 4, 2, EPI>(p);
    case 11: return launch_mid_cfg<8, 2, 3, 4, EPI>(p);
    case 12: return launch_mid_cfg<8, 4, 4, 2, EPI>(p);
    case 13: return launch_mid_cfg<2, 2, 3, 4, EPI, kCachePolicyNT>(p);
    case 14: return launch_mid_cfg<3, 2, 3, 4, EPI, kCachePolicyNT>(p);
    case 15: return launch_mid_cfg<4, 2, 3, 4, EPI, kCachePolicyNT>(p);
    case 16: return launch_mid_cfg<4, 2, 4, 2, EPI>(p);
    case 17:
      if constexpr (!epi_is_glu(EPI)) return launch_mid_cfg<7, 3, 4, 2, EPI>(p);
  }
  return hipErrorInvalidValue;
}

}  // namespace fn

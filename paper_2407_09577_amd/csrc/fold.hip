// Offline weight fold (Prop. 1: W*[k,n] = g_k W[k,n]; Sec. 3.4: c* = beta W) and
// the packing into the kernels' layout.  Runs once per weight, off the hot path.
//
// Each stored element is the exact product g_k * W[k,n] rounded once, to nearest with
// ties to even, into the storage type.  colsum sums the stored values and c* the products
// of beta with the unfolded W, both in fp64, rounded once to fp32.
#include "fn_device.h"
#include "fn_launch.h"
#include "fn_tile.h"

namespace fn {

// Packed column -> logical column, or -1 for padding.
__device__ __forceinline__ int64_t logical_col(int64_t p, int64_t N, int glu) {
  if (!glu) return p < N ? p : -1;
  const int64_t F = N / 2;
  const int64_t pair = p / 32, within = p % 32;
  const int64_t f = pair * 16 + (within & 15);
  if (f >= F) return -1;
  return within < 16 ? f : F + f;
}

// Round a double to the nearest bf16 (ties to even), returning the bit pattern.
// Normal range: add the rounding bias below bit 45 of the binary64 pattern (the
// 45 bits that bf16's 7-bit significand drops) and truncate, letting a carry
// ripple into the exponent.  Below 2^-126 bf16 is subnormal with fixed spacing
// 2^-133: scale, round to an integer (rint rounds ties to even), scale back.
__device__ __forceinline__ unsigned short dbl_to_bf16_rne(double x) {
  if (x != x) return 0x7fc0;
  if (fabs(x) < 0x1p-126) {
    const double r = rint(x * 0x1p133) * 0x1p-133;
    return (unsigned short)(__float_as_uint((float)r) >> 16);
  }
  unsigned long long u = (unsigned long long)__double_as_longlong(x);
  u += 0xfffffffffffull + ((u >> 45) & 1ull);
  u &= ~((1ull << 45) - 1ull);
  const float f = (float)__longlong_as_double((long long)u);  // exact, or overflow -> inf
  return (unsigned short)(__float_as_uint(f) >> 16);
}

// g w rounded once to bf16, from fp32: p is the rounded product and e its exact error, so the
// product truncated to 24 bits with the lost part folded into the last bit (round to odd)
// rounds to 8 bits as the exact product does.  Products outside the range where e is exact
// (below 2^-80, infinite, NaN) report `special` and take the fp64 rounding above; a product
// that underflows fp32 rounds to the same signed zero.
__device__ __forceinline__ float fold_odd(float g, float w, bool& special) {
  const float p = g * w, e = fmaf(g, w, -p);
  unsigned u = __float_as_uint(p);
  if (e != 0.0f) u = (u - ((__float_as_uint(e) ^ u) >> 31)) | 1u;
  special |= p != 0.0f && !(fabsf(p) >= 0x1p-80f && fabsf(p) <= 0x1.fffffep127f);
  return __uint_as_float(u);
}

// g w rounded once to fp32 (NaN as the fp64 product gives it).
__device__ __forceinline__ float fold_f32(float g, float w) {
  const float p = g * w;
  return p == p ? p : (float)((double)g * (double)w);
}

__device__ __forceinline__ float widen(unsigned short b) { return __uint_as_float((unsigned)b << 16); }
__device__ __forceinline__ float widen(float f) { return f; }

// Eight consecutive k of logical column n (zeros past K or without a column).  vec: the k are
// contiguous, K is a multiple of 8 and every such run starts on 16 bytes.  The addresses are
// clamped and the values selected, so that no load stands behind a branch and the loads of
// several fragments are in flight together.
template <typename T>
__device__ __forceinline__ void load_k8(const T* __restrict__ W, int64_t sk, int64_t sn, int64_t k0, int64_t n,
                                        int64_t K, bool vec, float (&w)[8]) {
  const int64_t nc = n >= 0 ? n : 0;
  if (vec) {
    const bool ok = n >= 0 && k0 < K;
    const T* p = W + nc * sn + (k0 < K ? k0 : 0);
    if constexpr (sizeof(T) == 2) {
      const u32x4 v = *reinterpret_cast<const u32x4*>(p);
#pragma unroll
      for (int i = 0; i < 4; ++i) w[2 * i] = ok ? bf16_lo(v[i]) : 0.0f, w[2 * i + 1] = ok ? bf16_hi(v[i]) : 0.0f;
    } else {
      const f32x4 v0 = *reinterpret_cast<const f32x4*>(p), v1 = *reinterpret_cast<const f32x4*>(p + 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) w[i] = ok ? v0[i] : 0.0f, w[4 + i] = ok ? v1[i] : 0.0f;
    }
    return;
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int64_t k = k0 + e;
    const float v = widen(W[(k < K ? k : 0) * sk + nc * sn]);
    w[e] = n >= 0 && k < K ? v : 0.0f;
  }
}

// Eight consecutive values of an optional vector over K (`none` without one, or past K).
__device__ __forceinline__ void load_v8(const float* __restrict__ v, int64_t k0, int64_t K, bool vec, float none,
                                        float (&x)[8]) {
  if (v && vec && k0 + 8 <= K) {
    const f32x4 v0 = *reinterpret_cast<const f32x4*>(v + k0), v1 = *reinterpret_cast<const f32x4*>(v + k0 + 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = v0[i], x[4 + i] = v1[i];
    return;
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = v && k0 + e < K ? v[k0 + e] : none;
}

// The stored bf16 values of eight k of a column, as 16 bytes; +0 without a column, whatever g
// (k past K have w = +0 and g = 1).
__device__ __forceinline__ u32x4 fold8_bf16(const float (&g)[8], const float (&w)[8], bool column) {
  bool special = false;
  u32x4 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const f32x2 o = {fold_odd(g[2 * i], w[2 * i], special), fold_odd(g[2 * i + 1], w[2 * i + 1], special)};
    r[i] = __builtin_bit_cast(unsigned, __builtin_convertvector(o, bf16x2));
  }
  if (special) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      r[i] = dbl_to_bf16_rne((double)g[2 * i] * (double)w[2 * i]) |
             ((unsigned)dbl_to_bf16_rne((double)g[2 * i + 1] * (double)w[2 * i + 1]) << 16);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = column ? r[i] : 0u;
  return r;
}

struct FoldIn {
  int64_t sk, sn, K, N;
  const float* g;
  const float* beta;
  int glu;
  bool vec, gvec, bvec;  // 16-byte loads of W along k, of g, of beta
};

// bf16 storage.  Bound by memory: W read once, W* written once, in 16-byte chunks of the
// fragment-major layout (lane 16 c + p of a fragment holds k chunk c of column p).  A wave
// writes whole fragments, NF of them in flight together.  With the k of W contiguous (a linear
// layer's [N, K] weight) the four waves of a block take consecutive k blocks, so 256 contiguous
// bytes of each of 16 columns are read together; otherwise consecutive column blocks, 128 bytes
// of a row.  4096 x 4096 bf16 from [N, K]: 39.7 us with an fp64 product and rounding per
// element and 64-byte pieces, 17.5 us (3.8 TB/s) so.
template <typename T, int NF>
__global__ __launch_bounds__(256) void fold_pack_bf16_kernel(const T* __restrict__ W, FoldIn in, int NPB, int KB,
                                                             int kgroups, u32x4* __restrict__ out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int cq = blockIdx.x / kgroups, kq = blockIdx.x % kgroups;
  const int cb = in.sk == 1 ? cq : 4 * cq + wave;
  if (cb >= NPB) return;
  const int64_t n = logical_col((int64_t)cb * 16 + (lane & 15), in.N, in.glu);
  auto block = [&](int i) { return in.sk == 1 ? 4 * (NF * kq + i) + wave : NF * kq + i; };
  float w[NF][8];
#pragma unroll
  for (int i = 0; i < NF; ++i)
    load_k8(W, in.sk, in.sn, (int64_t)block(i) * kKB + (lane >> 4) * 8, n, in.K, in.vec, w[i]);
#pragma unroll
  for (int i = 0; i < NF; ++i) {
    const int kb = block(i);
    if (kb >= KB) break;
    float g[8];
    load_v8(in.g, (int64_t)kb * kKB + (lane >> 4) * 8, in.K, in.gvec, 1.0f, g);
    out[((int64_t)kb * NPB + cb) * 64 + lane] = fold8_bf16(g, w[i], n >= 0);
  }
}

// LayerNorm's sums over K of a linear layout (packed column == logical column), with the bf16
// packing done on the way (kSumsPack) or alone for fp32 storage.  A block owns 16 columns and all of
// K, its 16 waves take k blocks w, w + 16, ...: every lane sums eight k of a column in fp64,
// then lanes and waves are added in a fixed order that does not depend on the strides.  (One
// thread per column, K steps in series on N / 128 blocks, took 1358 us at 4096 x 4096 beside
// the packing; both together 21.2 us from [N, K] and 25 us from [K, N].)
// kSumsAfter: the packing is done and the sums read it back, for sums written over g or W, which
// no block may still be reading.
enum FoldSums { kSumsPack, kSumsAlone, kSumsAfter };
template <typename T, FoldSums MODE>
__global__ __launch_bounds__(1024) void fold_sums_kernel(const T* __restrict__ W, FoldIn in, int NPB, int KB,
                                                         u32x4* __restrict__ out, float* __restrict__ colsum,
                                                         float* __restrict__ cstar, int ws_dtype) {
  __shared__ double part[2][16][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // Neighbouring column blocks (which share W's lines when its rows are contiguous) on one XCD.
  const int q8 = gridDim.x / kXcds, r8 = gridDim.x % kXcds, x8 = blockIdx.x % kXcds;
  const int cb = x8 * q8 + min(x8, r8) + blockIdx.x / kXcds;
  const int64_t col = (int64_t)cb * 16 + (lane & 15), n = col < in.N ? col : -1;
  double cs = 0.0, cb_sum = 0.0;
#pragma unroll 2
  for (int kb = wave; kb < KB; kb += 16) {
    const int64_t k0 = (int64_t)kb * kKB + (lane >> 4) * 8;
    float w[8], g[8], b[8];
    if (MODE != kSumsAfter || cstar) load_k8(W, in.sk, in.sn, k0, n, in.K, in.vec, w);
    if constexpr (MODE != kSumsAfter) load_v8(in.g, k0, in.K, in.gvec, 1.0f, g);
    if constexpr (MODE == kSumsAfter) {
      if (ws_dtype == kDtypeBf16) {
        const u32x4 h = out[((int64_t)kb * NPB + cb) * 64 + lane];
#pragma unroll
        for (int i = 0; i < 4; ++i) cs += (double)bf16_lo(h[i]) + (double)bf16_hi(h[i]);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) cs += (double)reinterpret_cast<const float*>(out)[(k0 + e) * 16 * NPB + col];
      }
    } else if constexpr (MODE == kSumsPack) {
      const u32x4 h = fold8_bf16(g, w, n >= 0);
      out[((int64_t)kb * NPB + cb) * 64 + lane] = h;
#pragma unroll
      for (int i = 0; i < 4; ++i) cs += (double)bf16_lo(h[i]) + (double)bf16_hi(h[i]);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) cs += (double)fold_f32(g[e], w[e]);
    }
    if (cstar) {
      load_v8(in.beta, k0, in.K, in.bvec, 0.0f, b);
#pragma unroll
      for (int e = 0; e < 8; ++e) cb_sum = fma((double)b[e], (double)w[e], cb_sum);
    }
  }
  cs += __shfl_xor(cs, 16);
  cs += __shfl_xor(cs, 32);
  cb_sum += __shfl_xor(cb_sum, 16);
  cb_sum += __shfl_xor(cb_sum, 32);
  if (lane < 16) {
    part[0][wave][lane] = cs;
    part[1][wave][lane] = cb_sum;
  }
  __syncthreads();
  if (threadIdx.x < 16 && n >= 0) {
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      s0 += part[0][i][lane];
      s1 += part[1][i][lane];
    }
    if (colsum) colsum[n] = (float)s0;
    if (cstar) cstar[n] = (float)s1;
  }
}

// fp32 storage: row-major [KP][NP] with columns in packed order, in tiles of 32 k x 64 packed
// columns.  With the k of W contiguous the tile is read along k and turned in LDS, so that both
// sides move whole lines (2048 x 2048 from [N, K]: 21.5 -> 8.0 us).
template <typename T>
__global__ __launch_bounds__(256) void fold_pack_f32_kernel(const T* __restrict__ W, FoldIn in, int64_t KP,
                                                            int64_t NP, int ptiles, float* __restrict__ out) {
  __shared__ float tile[32][65];
  const int t = threadIdx.x;
  const int64_t k0 = (int64_t)(blockIdx.x / ptiles) * 32, p0 = (int64_t)(blockIdx.x % ptiles) * 64;
  const int64_t p = p0 + (t & 63);
  float v[8];
  if (in.sk == 1) {
    const int64_t k = k0 + (t & 31), kc = k < in.K ? k : 0;
    const float g = in.g ? in.g[kc] : 1.0f;
    bool live[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int64_t pl = p0 + (t >> 5) + 8 * i, n = pl < NP ? logical_col(pl, in.N, in.glu) : -1;
      v[i] = widen(W[kc + (n >= 0 ? n : 0) * in.sn]);
      live[i] = n >= 0 && k < in.K;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) tile[t & 31][(t >> 5) + 8 * i] = live[i] ? fold_f32(g, v[i]) : 0.0f;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = tile[(t >> 6) + 4 * i][t & 63];
  } else {
    const int64_t n = p < NP ? logical_col(p, in.N, in.glu) : -1;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int64_t k = k0 + (t >> 6) + 4 * i, kc = k < in.K ? k : 0;
      v[i] = widen(W[kc * in.sk + (n >= 0 ? n : 0) * in.sn]);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int64_t k = k0 + (t >> 6) + 4 * i;
      v[i] = n >= 0 && k < in.K ? fold_f32(in.g ? in.g[k] : 1.0f, v[i]) : 0.0f;
    }
  }
  if (p >= NP) return;
#pragma unroll
  for (int i = 0; i < 8; ++i) out[(k0 + (t >> 6) + 4 * i) * NP + p] = v[i];  // KP is a multiple of 64
}

__global__ void unpack_kernel(const void* __restrict__ ws, int ws_dtype, int64_t K, int64_t N, int glu,
                              int64_t KP, int64_t NP, void* __restrict__ out, int64_t ldo) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= K * NP) return;
  const int64_t k = i / NP, p = i % NP;
  const int64_t n = logical_col(p, N, glu);
  if (n < 0) return;
  if (ws_dtype == kDtypeBf16) {
    const int64_t off = ((k / kKB) * (NP / 16) + p / 16) * 512 + (((k % kKB) / 8) * 16 + p % 16) * 8 + k % 8;
    reinterpret_cast<unsigned short*>(out)[k * ldo + n] = reinterpret_cast<const unsigned short*>(ws)[off];
  } else {
    reinterpret_cast<float*>(out)[k * ldo + n] = reinterpret_cast<const float*>(ws)[k * NP + p];
  }
}

static unsigned blocks_for(int64_t n, int threads) { return (unsigned)((n + threads - 1) / threads); }

template <typename T>
static hipError_t launch_fold_t(const FoldArgs& p) {
  const int64_t KP = packed_rows(p.K), NP = packed_cols(p.N, p.glu);
  const T* W = reinterpret_cast<const T*>(p.W);
  auto aligned = [](const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; };
  const FoldIn in{p.sk, p.sn, p.K, p.N, p.g, p.beta, p.glu,
                  p.sk == 1 && p.K % 8 == 0 && aligned(W) && p.sn * (int64_t)sizeof(T) % 16 == 0, aligned(p.g), aligned(p.beta)};
  const int NPB = (int)(NP / 16), KB = (int)(KP / kKB);
  u32x4* out = reinterpret_cast<u32x4*>(p.ws);
  const bool sums = p.colsum || p.cstar;
  auto launch_sums = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(NPB), dim3(1024), 0, p.stream, W, in, NPB, KB, out, p.colsum, p.cstar, p.ws_dtype);
    return hipGetLastError();
  };
  // Sums over g, or over W where c* does not need it, wait for the packing.
  auto over = [&](const float* s, const void* q, int64_t bytes) {
    const uintptr_t a = reinterpret_cast<uintptr_t>(s), b = reinterpret_cast<uintptr_t>(q);
    return s && q && a < b + (uintptr_t)bytes && b < a + (uintptr_t)p.N * 4;
  };
  const int64_t wbytes = ((p.K - 1) * p.sk + (p.N - 1) * p.sn + 1) * (int64_t)sizeof(T);
  const bool after = over(p.colsum, p.g, p.K * 4) || over(p.cstar, p.g, p.K * 4) ||
                     (!p.cstar && over(p.colsum, p.W, wbytes));
  if (p.ws_dtype == kDtypeBf16) {
    if (sums && !after) return launch_sums(fold_sums_kernel<T, kSumsPack>);
    // Four fragments per wave once that leaves two waves per SIMD (2048); below, one (576 x 1536:
    // 3.6 us with one, 7.1 with four).
    auto go = [&](auto kernel, int nf) {
      const int kstep = in.sk == 1 ? 4 * nf : nf, cstep = in.sk == 1 ? 1 : 4;
      const int kgroups = (KB + kstep - 1) / kstep;
      hipLaunchKernelGGL(kernel, dim3((unsigned)kgroups * ((NPB + cstep - 1) / cstep)), dim3(256), 0, p.stream, W,
                         in, NPB, KB, kgroups, out);
    };
    if ((int64_t)KB * NPB >= 4 * 2048) go(fold_pack_bf16_kernel<T, 4>, 4);
    else go(fold_pack_bf16_kernel<T, 1>, 1);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess || !sums ? e : launch_sums(fold_sums_kernel<T, kSumsAfter>);
  }
  const int ptiles = (int)((NP + 63) / 64);
  hipLaunchKernelGGL(fold_pack_f32_kernel<T>, dim3((unsigned)(KP / 32) * ptiles), dim3(256), 0, p.stream, W, in, KP,
                     NP, ptiles, reinterpret_cast<float*>(p.ws));
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || !sums) return e;
  return after ? launch_sums(fold_sums_kernel<T, kSumsAfter>) : launch_sums(fold_sums_kernel<T, kSumsAlone>);
}

hipError_t launch_fold(const FoldArgs& p) {
  return p.w_dtype == kDtypeBf16 ? launch_fold_t<unsigned short>(p) : launch_fold_t<float>(p);
}

hipError_t launch_unpack(const void* ws, int64_t K, int64_t N, int glu, int ws_dtype, void* out,
                         int64_t ldo, hipStream_t stream) {
  const int64_t KP = packed_rows(K), NP = packed_cols(N, glu);
  hipLaunchKernelGGL(unpack_kernel, dim3(blocks_for(K * NP, 256)), dim3(256), 0, stream, ws, ws_dtype, K,
                     N, glu, KP, NP, out, ldo);
  return hipGetLastError();
}

}  // namespace fn

// fp32 GEMM for the fp32 mode of the encoder (small models and the fp32
// parity mode).  Same contract as the bf16 MFMA GEMM (GemmArgs): optional
// LayerNorm prologue on an fp32 A, fused bias / activation / position /
// residual epilogue.  Plain FMA: a 64 x 64 tile, k-step 16, each of the 256
// threads owning a 4 x 4 block, or 16 x 16 tiles of one output a thread for small
// products; both sum k in ascending order for every output, so results do not
// depend on M.
#include "common.h"

namespace eas {
namespace {

constexpr int TM = 64, TN = 64, TK = 16;

// The epilogue of one output.
__device__ __forceinline__ void store_out(const GemmArgs& a, int m, int n, float acc) {
  if (m >= a.M || n >= a.N) return;
  const float* bias = static_cast<const float*>(a.bias);
  float v = apply_act(a.act, acc + (bias ? bias[n] : 0.0f));
  if (a.pos) {
    const int pr = a.pos_idx ? a.pos_idx[m] : m % a.pos_period;
    const long pi = (long)pr * a.ld_pos + n;
    v += a.pos_f32 ? static_cast<const float*>(a.pos)[pi] : (float)static_cast<const bf16*>(a.pos)[pi];
  }
  if (a.resid) v += a.resid[(long)m * a.ldr + n];
  const long oi = (long)m * a.ldo + n;
  if (a.out_f32) static_cast<float*>(a.out)[oi] = v;
  else static_cast<bf16*>(a.out)[oi] = (bf16)v;
}

__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmArgs a) {
  __shared__ float As[TK][TM + 4];
  __shared__ float Bs[TK][TN + 4];
  const int tid = threadIdx.x;
  const int tiles_n = (a.N + TN - 1) / TN;
  const int m0 = (blockIdx.x / tiles_n) * TM, n0 = (blockIdx.x % tiles_n) * TN;
  const int ty = tid / 16, tx = tid % 16;
  const float* A = static_cast<const float*>(a.A);
  const float* B = static_cast<const float*>(a.B);
  const float* g = static_cast<const float*>(a.ln_g);
  const float* b = static_cast<const float*>(a.ln_b);

  float acc[4][4] = {};
  for (int k0 = 0; k0 < a.K; k0 += TK) {
    for (int e = tid; e < TM * TK; e += 256) {
      const int r = e / TK, kk = e % TK;
      const int gm = m0 + r, gk = k0 + kk;
      float v = 0.0f;
      if (gm < a.M && gk < a.K) {
        v = A[(long)gm * a.lda + gk];
        if (a.stats) {
          const float2 st = a.stats[(long)gm * a.ln_group + gk / a.ln_dim];
          const int c = gk % a.ln_dim;
          v = (v - st.x) * st.y * g[c] + b[c];
        }
      }
      As[kk][r] = v;
    }
    for (int e = tid; e < TN * TK; e += 256) {
      const int r = e / TK, kk = e % TK;
      const int gn = n0 + r, gk = k0 + kk;
      Bs[kk][r] = (gn < a.N && gk < a.K) ? B[(long)gn * a.ldb + gk] : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < TK; ++kk) {
      float av[4], bv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) av[i] = As[kk][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) bv[j] = Bs[kk][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(av[i], bv[j], acc[i][j]);
    }
    __syncthreads();
  }

#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) store_out(a, m0 + ty * 4 + i, n0 + tx * 4 + j, acc[i][j]);
}

// Small products (the tiny encoder's have 8 to 128 rows): bound by latency, not work.
// The 64 x 64 kernel puts one on a few CUs and waits for global memory at every 16 k
// (588 k: 35 us on one CU).  Here a block owns 16 x 16 outputs and stages SK k of its 32
// operand rows at a time, every load of a stage in flight at once and the next
// stage's issued before this one is multiplied; with a LayerNorm prologue it also
// takes its rows' statistics (the statistics kernel's own reduction, so the same
// bits), which saves that launch.  Two tiny images, all 20 launches: 326 -> 110 us (15 launches left).
constexpr int SM = 16, SK = 256, SLD = SK + 4;   // 4 floats of padding: 16 rows' 16-byte reads on distinct banks

__global__ __launch_bounds__(256) void gemm_f32_small_kernel(GemmArgs a) {
  __shared__ __attribute__((aligned(16))) float As[SM * SLD];
  __shared__ __attribute__((aligned(16))) float Bs[SM * SLD];
  __shared__ float2 st[SM * 4];   // ln_group <= 4
  const int tid = threadIdx.x, tiles_n = (a.N + SM - 1) / SM;
  const int m0 = (blockIdx.x / tiles_n) * SM, n0 = (blockIdx.x % tiles_n) * SM;
  const float* A = static_cast<const float*>(a.A);
  const float* B = static_cast<const float*>(a.B);
  const float* g = static_cast<const float*>(a.ln_g);
  const float* b = static_cast<const float*>(a.ln_b);
  // chunk c of a stage: row c / (SK / 4), 4 k at (c % (SK / 4)) * 4; 4 chunks of A and 4 of B a thread
  constexpr int CPT = SM * SK / 4 / 256;
  float4 ra[CPT], rb[CPT];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
      const int c = u * 256 + tid, r = c / (SK / 4), k = k0 + c % (SK / 4) * 4;
      const bool in = k < a.K;   // K % 4 == 0: all four or none
      ra[u] = in && m0 + r < a.M ? *reinterpret_cast<const float4*>(A + (long)(m0 + r) * a.lda + k)
                                 : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      rb[u] = in && n0 + r < a.N ? *reinterpret_cast<const float4*>(B + (long)(n0 + r) * a.ldb + k)
                                 : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
  };
  fetch(0);
  if (g) {   // one wave per token row, as ln_stats_kernel
    const int rows = min(SM, a.M - m0) * a.ln_group;
    for (int t = tid >> 6; t < rows; t += 4) {
      float v[LN_MAXE], mu, rstd;
      row_stats(A + ((long)m0 * a.ln_group + t) * a.ln_dim, a.ln_dim, a.ln_eps, v, &mu, &rstd);
      if ((tid & 63) == 0) st[t] = make_float2(mu, rstd);
    }
    __syncthreads();
  }
  const float* arow = As + (tid / SM) * SLD;
  const float* brow = Bs + (tid % SM) * SLD;
  float acc = 0.0f;
  for (int k0 = 0; k0 < a.K; k0 += SK) {
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
      const int c = u * 256 + tid, r = c / (SK / 4), kk = c % (SK / 4) * 4;
      float v[4] = {ra[u].x, ra[u].y, ra[u].z, ra[u].w};
      if (g && k0 + kk < a.K && m0 + r < a.M) {
        const float2 s = st[r * a.ln_group + (k0 + kk) / a.ln_dim];   // ln_dim % 4 == 0: one token's four
        const int gc = (k0 + kk) % a.ln_dim;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (v[e] - s.x) * s.y * g[gc + e] + b[gc + e];
      }
      *reinterpret_cast<float4*>(As + r * SLD + kk) = make_float4(v[0], v[1], v[2], v[3]);
      *reinterpret_cast<float4*>(Bs + r * SLD + kk) = rb[u];
    }
    __syncthreads();
    if (k0 + SK < a.K) fetch(k0 + SK);
    const int n4 = min(SK, a.K - k0) / 4;
#pragma unroll 8
    for (int q = 0; q < n4; ++q) {
      const float4 x = *reinterpret_cast<const float4*>(arow + 4 * q);
      const float4 y = *reinterpret_cast<const float4*>(brow + 4 * q);
      acc = fmaf(x.x, y.x, acc);
      acc = fmaf(x.y, y.y, acc);
      acc = fmaf(x.z, y.z, acc);
      acc = fmaf(x.w, y.w, acc);
    }
    __syncthreads();
  }
  store_out(a, m0 + tid / SM, n0 + tid % SM, acc);
}

// 16 x 16 tiles while the product has at most 2^20 outputs (16 blocks a CU; the 64 x 64
// kernel then has at most one) and its rows can be read 16 bytes at a time.
bool small_ok(const GemmArgs& a) {
  auto al = [](const void* p) { return (uintptr_t)p % 16 == 0; };
  return (long)a.M * a.N <= 1 << 20 && a.K % 4 == 0 && a.lda % 4 == 0 && a.ldb % 4 == 0 && al(a.A) && al(a.B) &&
         !a.stats;
}

}  // namespace

bool gemm_f32_own_stats(const GemmArgs& a) {
  return small_ok(a) && a.ln_g && a.ln_dim % 4 == 0 && a.ln_dim <= 64 * LN_MAXE && a.ln_group <= 4 &&
         a.lda == a.ln_group * a.ln_dim;
}

hipError_t launch_gemm_f32(const GemmArgs& a, hipStream_t s, const char** kname) {
  if (small_ok(a) && (!a.ln_g || gemm_f32_own_stats(a))) {
    const long tiles = (long)((a.M + SM - 1) / SM) * ((a.N + SM - 1) / SM);
    *kname = "gemm_f32_16x16";
    hipLaunchKernelGGL(gemm_f32_small_kernel, dim3((unsigned)tiles), dim3(256), 0, s, a);
    return hipGetLastError();
  }
  const long tiles = (long)((a.M + TM - 1) / TM) * ((a.N + TN - 1) / TN);
  *kname = "gemm_f32_64x64";
  hipLaunchKernelGGL(gemm_f32_kernel, dim3((unsigned)tiles), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace eas

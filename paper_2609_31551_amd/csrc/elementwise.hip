// Bandwidth-bound kernels of the Encode path: token positions, LayerNorm
// statistics / application, rotary position application, CLS insertion,
// the audio front end's im2col, and the micro-batch packers.
#include "common.h"

namespace eas {
namespace {

// (t, h, w) of token j of a t x h x w grid in storage order: merge-window
// order (2x2 windows in raster order, the window's 4 tokens consecutive) when
// merge == 2, raster order otherwise.
__device__ __forceinline__ void decode_token(int j, int h, int w, int merge, int* ti, int* hi, int* wi) {
  const int hw = h * w;
  *ti = j / hw;
  const int rem = j - *ti * hw;
  if (merge == 2) {
    const int win = rem >> 2, q = rem & 3, wb_n = w >> 1;
    *hi = 2 * (win / wb_n) + (q >> 1);
    *wi = 2 * (win % wb_n) + (q & 1);
  } else {
    *hi = rem / w;
    *wi = rem - *hi * w;
  }
}

__global__ void positions_kernel(SeqMeta m, int N, int4* pos3, int* tab_idx, int pos_gw) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  const int r = find_seq(m.cu, m.n, i);
  int j = i - m.cu[r];
  int4 p = make_int4(0, 0, 0, 0);
  if (m.cls) {
    if (j == 0) { pos3[i] = p; tab_idx[i] = 0; return; }
    j -= 1;
  }
  decode_token(j, m.thw[r][1], m.thw[r][2], m.merge, &p.x, &p.y, &p.z);
  pos3[i] = p;
  tab_idx[i] = m.cls + p.y * pos_gw + p.z;
}

__global__ __launch_bounds__(256) void ln_stats_kernel(const float* x, int N, int d, float eps, float2* st) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= N) return;
  float v[LN_MAXE], mu, rstd;
  row_stats(x + (long)row * d, d, eps, v, &mu, &rstd);
  if ((threadIdx.x & 63) == 0) st[row] = make_float2(mu, rstd);
}

template <class W, class Y>
__global__ __launch_bounds__(256) void ln_apply_kernel(const float* x, int N, int d, float eps, const W* g,
                                                       const W* b, Y* y) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= N) return;
  const int lane = threadIdx.x & 63;
  float v[LN_MAXE], mu, rstd;
  row_stats(x + (long)row * d, d, eps, v, &mu, &rstd);
#pragma unroll
  for (int e = 0; e < LN_MAXE; ++e) {
    const int c = lane + 64 * e;
    if (c < d) y[(long)row * d + c] = (Y)((v[e] - mu) * rstd * (float)g[c] + (float)b[c]);
  }
}

// Vector form: one wave per row, each lane 4 consecutive elements per 16-byte
// chunk (rows with d % 4 == 0, up to 64 * 4 * LNV_MAXC wide).
constexpr int LNV_MAXC = 8;

template <class W, class Y>
__global__ __launch_bounds__(256) void ln_apply_vec_kernel(const float* x, int N, int d, float eps, const W* g,
                                                           const W* b, Y* y) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= N) return;
  const int lane = threadIdx.x & 63, nc = d >> 2;
  const float4* xr = reinterpret_cast<const float4*>(x + (long)row * d);
  // gamma and beta are fetched with the row, so their latency hides under its
  // loads and reductions (one LayerNorm over one image's 577 rows is latency-bound)
  static_assert(sizeof(W) == 2, "gamma / beta fetched as four 16-bit values per 8 bytes");
  uint2 gv[LNV_MAXC], bv[LNV_MAXC];
#pragma unroll
  for (int e = 0; e < LNV_MAXC; ++e) {
    const int c = lane + 64 * e;
    if (c < nc) {
      gv[e] = *reinterpret_cast<const uint2*>(g + 4 * c);
      bv[e] = *reinterpret_cast<const uint2*>(b + 4 * c);
    }
  }
  float4 v[LNV_MAXC];
  float s = 0.0f;
#pragma unroll
  for (int e = 0; e < LNV_MAXC; ++e) {
    const int c = lane + 64 * e;
    v[e] = c < nc ? xr[c] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    s += (v[e].x + v[e].y) + (v[e].z + v[e].w);
  }
  const float mean = wave_sum(s) / (float)d;
  float q = 0.0f;
#pragma unroll
  for (int e = 0; e < LNV_MAXC; ++e) {
    if (lane + 64 * e < nc) {
      const float a0 = v[e].x - mean, a1 = v[e].y - mean, a2 = v[e].z - mean, a3 = v[e].w - mean;
      q += (a0 * a0 + a1 * a1) + (a2 * a2 + a3 * a3);
    }
  }
  const float rstd = 1.0f / sqrtf(wave_sum(q) / (float)d + eps);
#pragma unroll
  for (int e = 0; e < LNV_MAXC; ++e) {
    const int c = lane + 64 * e;
    if (c < nc) {
      const float in[4] = {v[e].x, v[e].y, v[e].z, v[e].w};
      union { uint2 u; W h[4]; } gw, bw;
      gw.u = gv[e];
      bw.u = bv[e];
      Y out[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) out[j] = (Y)((in[j] - mean) * rstd * (float)gw.h[j] + (float)bw.h[j]);
      if constexpr (sizeof(Y) == 2) {
        union { uint2 u; Y h[4]; } o;
#pragma unroll
        for (int j = 0; j < 4; ++j) o.h[j] = out[j];
        *reinterpret_cast<uint2*>(y + (long)row * d + 4 * c) = o.u;
      } else {
        *reinterpret_cast<float4*>(y + (long)row * d + 4 * c) = make_float4(out[0], out[1], out[2], out[3]);
      }
    }
  }
}

// Rotate the pairs (k, k + hd/2) of every head of q and k in place; slot k
// turns by pos[axis(k)] * inv_freq[k].
template <class T>
__global__ void rope_kernel(T* qkv, int ldqkv, int N, int heads, int hd, const int4* pos3,
                            const float* inv_freq, const int* slot_axis) {
  const int half = hd >> 1;
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long total = (long)N * heads * half;
  if (idx >= total) return;
  const int k = (int)(idx % half);
  const int h = (int)((idx / half) % heads);
  const int i = (int)(idx / ((long)half * heads));
  const int4 p = pos3[i];
  const int ax = slot_axis[k];
  const float pos = (float)(ax == 0 ? p.x : (ax == 1 ? p.y : p.z));
  float sn, cs;
  sincosf(pos * inv_freq[k], &sn, &cs);
  const int dq = heads * hd;
#pragma unroll
  for (int part = 0; part < 2; ++part) {   // q block, then k block
    T* base = qkv + (long)i * ldqkv + part * dq + h * hd;
    const float x1 = (float)base[k], x2 = (float)base[k + half];
    base[k] = (T)(x1 * cs - x2 * sn);
    base[k + half] = (T)(x2 * cs + x1 * sn);
  }
}

// bf16 RoPE, one block per ROPE_TOK tokens: the (cos, sin) of every rotation
// slot of its tokens are computed once into LDS, then the block's threads
// rotate the (x_k, x_{k+half}) 16-byte chunk pairs of q and k, consecutive
// threads on consecutive chunks (a row's q and k heads are one contiguous
// stretch of 2 * heads * hd elements), ROPE_R pairs per thread with all their
// loads issued before the first store.  hd % 16 == 0, hd <= 128.
constexpr int ROPE_TOK = 8, ROPE_R = 5;
__global__ __launch_bounds__(256) void rope_vec_kernel(bf16* qkv, int ldqkv, int N, int heads, int hd,
                                                       const int4* pos3, const float* inv_freq, const int* slot_axis) {
  __shared__ float2 tab[ROPE_TOK * 64];   // [token][slot]: (cos, sin)
  const int half = hd >> 1, chunks = half >> 3;
  const int t0 = blockIdx.x * ROPE_TOK, nt = min(ROPE_TOK, N - t0);
  for (int e = threadIdx.x; e < nt * half; e += blockDim.x) {
    const int t = e / half, k = e % half;
    const int4 p = pos3[t0 + t];
    const int ax = slot_axis[k];
    const float pos = (float)(ax == 0 ? p.x : (ax == 1 ? p.y : p.z));
    float sn, cs;
    sincosf(pos * inv_freq[k], &sn, &cs);
    tab[t * 64 + k] = make_float2(cs, sn);
  }
  __syncthreads();
  const int per_tok = 2 * heads * chunks;   // chunk pairs of q and k per token
  const int items = nt * per_tok;
  for (int i0 = 0; i0 < items; i0 += ROPE_R * 256) {
    union { uint4 u; bf16 e[8]; } a[ROPE_R], c[ROPE_R];
    bf16* ptr[ROPE_R];
    int ti[ROPE_R], kk[ROPE_R];
#pragma unroll
    for (int r = 0; r < ROPE_R; ++r) {
      const int it = i0 + r * 256 + (int)threadIdx.x;
      ptr[r] = nullptr;
      if (it < items) {
        const int t = it / per_tok, w = it % per_tok;
        ti[r] = t;
        kk[r] = (w % chunks) * 8;
        ptr[r] = qkv + (long)(t0 + t) * ldqkv + (w / chunks) * hd + kk[r];
        a[r].u = *reinterpret_cast<const uint4*>(ptr[r]);
        c[r].u = *reinterpret_cast<const uint4*>(ptr[r] + half);
      }
    }
#pragma unroll
    for (int r = 0; r < ROPE_R; ++r) {
      if (ptr[r]) {
        const float2* f = tab + ti[r] * 64 + kk[r];
        union { uint4 u; bf16 e[8]; } oa, oc;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const float2 q = f[j];
          const float x1 = (float)a[r].e[j], x2 = (float)c[r].e[j];
          oa.e[j] = (bf16)(x1 * q.x - x2 * q.y);
          oc.e[j] = (bf16)(x2 * q.x + x1 * q.y);
        }
        *reinterpret_cast<uint4*>(ptr[r]) = oa.u;
        *reinterpret_cast<uint4*>(ptr[r] + half) = oc.u;
      }
    }
  }
}

template <class W>
__global__ void cls_kernel(SeqMeta m, float* x, int d, const W* cls, const W* pos0) {
  const int r = blockIdx.x;
  for (int c = threadIdx.x; c < d; c += blockDim.x)
    x[(long)m.cu[r] * d + c] = (float)cls[c] + (float)pos0[c];
}

// dst[(clip, t), c*3 + k] = src[(clip, stride*t + k - 1), c], zero outside the
// clip: the im2col of a kernel-3, padding-1 1-D convolution over time-major
// frames, in the (channel, tap) order of a [out, C, 3] weight.
template <class T>
__global__ void im2col_k3_kernel(const T* src, int fin, int C, int fout, int stride, long total, T* dst) {
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  const int k = (int)(idx % 3);
  const int c = (int)((idx / 3) % C);
  const long row = idx / (3L * C);
  const int t = (int)(row % fout);
  const long clip = row / fout;
  const int ts = stride * t + k - 1;
  dst[idx] = (ts >= 0 && ts < fin) ? src[(clip * fin + ts) * C + c] : (T)0.0f;
}

template <class T>
__global__ void pack_vision_kernel(PackArgs p, int cls, int merge, int patch, int tp, int K, long total, T* out) {
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  const int kk = (int)(idx % K);
  const int row = (int)(idx / K);
  const int r = find_seq(p.cu, p.n, row);
  int j = row - p.cu[r];
  if (cls) {
    if (j == 0) { out[idx] = (T)0.0f; return; }
    j -= 1;
  }
  const int H = p.tchw[r][2], W = p.tchw[r][3], C = p.tchw[r][1];
  const int h = H / patch, w = W / patch;
  int ti, hi, wi;
  decode_token(j, h, w, merge, &ti, &hi, &wi);
  const int dx = kk % patch, dy = (kk / patch) % patch;
  const int tau = (kk / (patch * patch)) % tp, c = kk / (patch * patch * tp);
  const long src = (((long)(ti * tp + tau) * C + c) * H + hi * patch + dy) * W + wi * patch + dx;
  out[idx] = (T)p.src[r][src];
}

// bf16 packer: a block packs a strip of up to STRIP patches side by side (with the
// merger, the two patch rows of its windows), whose token rows are consecutive in
// storage order.  Consecutive threads read consecutive float2 pairs of an image row
// (224 bytes a strip of four) and write them as bf16 into the block's LDS copy of the
// token rows, which then leaves as one contiguous span of 8-byte writes.  Bound by
// memory, and by a block's own latency in small launches: so six loads a thread are in
// flight at once, and the index arithmetic has two divisions.  Needs an even patch,
// even widths and 8-byte aligned sources.  Kernel times (us), one thread a 14-pixel
// line -> this: 224 x 224 image 4.9 -> 4.5, 336 x 504 7.5 -> 4.9, 672 x 896 15.0 ->
// 8.6, 1344 x 1344 45.9 -> 17.4, 16 frames of 448 x 448 41.1 -> 13.7 (3.8 TB/s); 336 x
// 336 images: one 4.4 -> 4.3, two 4.8 -> 5.0, 16 16.1 -> 10.4, 64 50.8 -> 29.1.
template <int STRIP, int NT>
__global__ __launch_bounds__(NT) void pack_vision_vec_kernel(PackArgs p, int cls, int merge, int patch, int tp, int C,
                                                             int dy, int dc, int dtau, int K, bf16* out) {
  extern __shared__ __attribute__((aligned(16))) unsigned buf[];   // STRIP * merge token rows of K bf16
  const int r = find_seq(p.strip0, p.n, blockIdx.x);
  const int H = p.tchw[r][2], W = p.tchw[r][3], hr = p.hw[r][0], w = p.hw[r][1];
  const int q = blockIdx.x - p.strip0[r], per_row = (w + STRIP - 1) / STRIP;
  const int pr = q / per_row, ti = pr / hr, hi = (pr - ti * hr) * merge;
  const int wi = (q - pr * per_row) * STRIP, wp = min(STRIP, w - wi);
  // TR threads an image row of the strip (at most 8 float2 pairs a patch), RP rows at a time
  constexpr int U = 6, TR = 8 * STRIP, RP = NT / TR;
  const int hp = patch / 2, tx = threadIdx.x % TR;
  int px = 0;
#pragma unroll
  for (int i = 1; i <= STRIP; ++i) px += tx >= i * hp;
  const int dx = tx - px * hp;
  const bool on = px < wp;
  const int rows = merge * patch, nr = C * tp * rows;
  const int row2 = K / 2;                               // 4-byte words a token row
  const int tokx = merge == 2 ? (px >> 1) * 4 + (px & 1) : px;
  const float* base = p.src[r] + ((long)ti * tp * C * H + (long)hi * patch) * W + (long)wi * patch + (on ? 2 * tx : 0);
  // the thread's image rows e, e + RP, ...: line y of channel c of frame tau, walked by
  // additions (RP rows are dy lines, dc channels and dtau frames)
  int e = threadIdx.x / TR, y = e, c = 0, tau = 0;
  while (y >= rows) {
    y -= rows;
    if (++c == C) { c = 0; ++tau; }
  }
  for (; e < nr; e += U * RP) {
    float2 v[U];
    int dst[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = e + u * RP < nr;
      const int py = y >= patch ? 1 : 0;
      v[u] = *reinterpret_cast<const float2*>(base + (in ? ((long)(tau * C + c) * H + y) * W : 0));
      dst[u] = in && on ? (tokx + 2 * py) * row2 + ((c * tp + tau) * patch + y - py * patch) * hp + dx : -1;
      y += dy;
      c += dc;
      tau += dtau;
      if (y >= rows) { y -= rows; ++c; }
      if (c >= C) { c -= C; ++tau; }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      union { unsigned u; bf16 h[2]; } o;
      o.h[0] = (bf16)v[u].x;
      o.h[1] = (bf16)v[u].y;
      if (dst[u] >= 0) buf[dst[u]] = o.u;
    }
  }
  __syncthreads();
  // first token of the strip: whole patch rows (or pairs) before it, then merge * wi tokens
  const long tok0 = p.cu[r] + cls + ((long)ti * hr * merge + hi) * w + (long)merge * wi;
  const int n8 = merge * wp * K / 4;   // 8-byte pieces (K % 4 == 0)
  uint2* o8 = reinterpret_cast<uint2*>(out + tok0 * K);
  const uint2* b8 = reinterpret_cast<const uint2*>(buf);
  for (int i = threadIdx.x; i < n8; i += NT) o8[i] = b8[i];
  if (cls && q == 0) {   // the request's CLS row
    uint2* c8 = reinterpret_cast<uint2*>(out + (long)p.cu[r] * K);
    for (int i = threadIdx.x; i < K / 4; i += NT) c8[i] = make_uint2(0u, 0u);
  }
}

// bf16 im2col for C % 8 == 0: one thread per (output frame, 8 channels) reads
// the three taps' 16-byte chunks and writes the 24 values ((channel, tap)
// order) as three 16-byte stores.
__global__ void im2col_k3_vec_kernel(const bf16* src, int fin, int C, int fout, int stride, long total, bf16* dst) {
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  const int cg = C >> 3;
  const long row = idx / cg;
  const int c0 = (int)(idx % cg) * 8;
  const int t = (int)(row % fout);
  const long clip = row / fout;
  union { uint4 u; bf16 e[8]; } in[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int ts = stride * t + k - 1;
    in[k].u = (ts >= 0 && ts < fin) ? *reinterpret_cast<const uint4*>(src + (clip * fin + ts) * C + c0)
                                    : make_uint4(0u, 0u, 0u, 0u);
  }
  union { uint4 u[3]; bf16 e[24]; } o;
#pragma unroll
  for (int cc = 0; cc < 8; ++cc)
#pragma unroll
    for (int k = 0; k < 3; ++k) o.e[cc * 3 + k] = in[k].e[cc];
  uint4* d = reinterpret_cast<uint4*>(dst + row * 3 * C + c0 * 3);
#pragma unroll
  for (int q = 0; q < 3; ++q) d[q] = o.u[q];
}

// [n_mels, n_frames] -> [n_frames, n_mels] per clip.
template <class T>
__global__ void pack_audio_kernel(PackArgs p, int n_mels, int n_frames, T* out) {
  const long per = (long)n_mels * n_frames;
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= per * p.n) return;
  const int clip = (int)(idx / per);
  const long e = idx % per;
  const int t = (int)(e / n_mels), mel = (int)(e % n_mels);
  out[idx] = (T)p.src[clip][(long)mel * n_frames + t];
}

// [rows, k] 16-bit elements -> [rows, kp] with zero columns k .. kp; a thread
// writes one 16-byte chunk of the output.
__global__ void pad_cols16_kernel(const uint16_t* src, int rows, int k, int kp, uint16_t* dst) {
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const int cpr = kp / 8;
  if (idx >= (long)rows * cpr) return;
  const int r = (int)(idx / cpr), c0 = (int)(idx % cpr) * 8;
  union { uint4 u; uint16_t h[8]; } o;
#pragma unroll
  for (int e = 0; e < 8; ++e) o.h[e] = c0 + e < k ? src[(long)r * k + c0 + e] : (uint16_t)0;
  *reinterpret_cast<uint4*>(dst + (long)r * kp + c0) = o.u;
}

inline unsigned blocks_for(long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

namespace {

// Whisper-style sinusoid table [F, d]: columns i < d/2 hold sin(t * w_i) and
// columns d/2 + i hold cos(t * w_i), w_i = exp(-i ln(10^4) / (d/2 - 1));
// evaluated in double, stored as fp32.
__global__ void sinusoid_table_kernel(float* tab, int F, int d) {
  const int hc = d / 2;
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (long)F * hc) return;
  const int t = (int)(idx / hc), i = (int)(idx % hc);
  const double a = (double)t * exp(-log(10000.0) / (double)(hc - 1) * (double)i);
  tab[(long)t * d + i] = (float)sin(a);
  tab[(long)t * d + hc + i] = (float)cos(a);
}

// Rotary slot tables: the sections s0, s1, s2 of slots turn with the t, h
// and w position; slot j of an axis with n slots turns by theta^(-j / n).
__global__ void rope_table_kernel(float* inv_freq, int* slot_axis, int s0, int s1, int s2, float theta) {
  const int k = threadIdx.x;
  if (k >= s0 + s1 + s2) return;
  const int ax = k < s0 ? 0 : (k < s0 + s1 ? 1 : 2);
  const int j = k - (ax == 0 ? 0 : (ax == 1 ? s0 : s0 + s1));
  const int n = ax == 0 ? s0 : (ax == 1 ? s1 : s2);
  inv_freq[k] = (float)pow((double)theta, -(double)j / (double)n);
  slot_axis[k] = ax;
}

// dst[l, n] = src[l * stride + rope_src_row(n)]: every layer's q | k | v bias with
// the q and k heads interleaved for the rotary epilogue.
__global__ void rope_bias_kernel(const bf16* src, long stride, int w, int cols, int hd, unsigned hd_inv, bf16* dst,
                                 long total) {
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  const int l = (int)(idx / w), n = (int)(idx % w);
  dst[idx] = src[l * stride + rope_src_row(n, hd, hd_inv, cols)];
}

}  // namespace

hipError_t launch_rope_bias(const void* src, long stride, int layers, int cols, int hd, void* dst, hipStream_t s) {
  const int w = cols / 2 * 3;
  const long total = (long)layers * w;
  if (cols % 2 || hd % 2 || hd > 128 || cols % hd || w >= 65536) return hipErrorInvalidValue;
  if (total == 0) return hipSuccess;
  hipLaunchKernelGGL(rope_bias_kernel, dim3(blocks_for(total, 256)), dim3(256), 0, s, static_cast<const bf16*>(src),
                     stride, w, cols, hd, rope_hd_inv(hd), static_cast<bf16*>(dst), total);
  return hipGetLastError();
}

hipError_t launch_sinusoid_table(float* tab, int F, int d, hipStream_t s) {
  if (d < 4 || d % 2) return hipErrorInvalidValue;
  const long total = (long)F * (d / 2);
  if (total == 0) return hipSuccess;
  hipLaunchKernelGGL(sinusoid_table_kernel, dim3(blocks_for(total, 256)), dim3(256), 0, s, tab, F, d);
  return hipGetLastError();
}

hipError_t launch_rope_table(float* inv_freq, int* slot_axis, const int sections[3], float theta, hipStream_t s) {
  if (sections[0] + sections[1] + sections[2] > 256) return hipErrorInvalidValue;
  hipLaunchKernelGGL(rope_table_kernel, dim3(1), dim3(256), 0, s, inv_freq, slot_axis, sections[0], sections[1],
                     sections[2], theta);
  return hipGetLastError();
}

hipError_t launch_positions(const SeqMeta& m, int N, int4* pos3, int* tab_idx, int pos_gw, hipStream_t s) {
  hipLaunchKernelGGL(positions_kernel, dim3(blocks_for(N, 256)), dim3(256), 0, s, m, N, pos3, tab_idx, pos_gw);
  return hipGetLastError();
}

hipError_t launch_ln_stats(const float* x, int N, int d, float eps, float2* stats, hipStream_t s) {
  if (d > 64 * LN_MAXE) return hipErrorInvalidValue;
  hipLaunchKernelGGL(ln_stats_kernel, dim3(blocks_for(N, 4)), dim3(256), 0, s, x, N, d, eps, stats);
  return hipGetLastError();
}

hipError_t launch_ln_apply(const float* x, int N, int d, float eps, const void* g, const void* b, int w_bf16,
                           void* y, int y_f32, hipStream_t s) {
  if (d > 64 * LN_MAXE) return hipErrorInvalidValue;
  const dim3 grid(blocks_for(N, 4)), blk(256);
  const bool al = (uintptr_t)x % 16 == 0 && (uintptr_t)y % (y_f32 ? 16 : 8) == 0 &&
                  (uintptr_t)g % (w_bf16 ? 8 : 16) == 0 && (uintptr_t)b % (w_bf16 ? 8 : 16) == 0;
  if (d % 4 == 0 && d <= 256 * LNV_MAXC && al && w_bf16) {
    if (y_f32)
      hipLaunchKernelGGL((ln_apply_vec_kernel<bf16, float>), grid, blk, 0, s, x, N, d, eps, (const bf16*)g,
                         (const bf16*)b, (float*)y);
    else
      hipLaunchKernelGGL((ln_apply_vec_kernel<bf16, bf16>), grid, blk, 0, s, x, N, d, eps, (const bf16*)g,
                         (const bf16*)b, (bf16*)y);
    return hipGetLastError();
  }
  if (w_bf16 && y_f32)
    hipLaunchKernelGGL((ln_apply_kernel<bf16, float>), grid, blk, 0, s, x, N, d, eps, (const bf16*)g, (const bf16*)b, (float*)y);
  else if (w_bf16)
    hipLaunchKernelGGL((ln_apply_kernel<bf16, bf16>), grid, blk, 0, s, x, N, d, eps, (const bf16*)g, (const bf16*)b, (bf16*)y);
  else if (y_f32)
    hipLaunchKernelGGL((ln_apply_kernel<float, float>), grid, blk, 0, s, x, N, d, eps, (const float*)g, (const float*)b, (float*)y);
  else
    hipLaunchKernelGGL((ln_apply_kernel<float, bf16>), grid, blk, 0, s, x, N, d, eps, (const float*)g, (const float*)b, (bf16*)y);
  return hipGetLastError();
}

hipError_t launch_rope(void* qkv, int ldqkv, int N, int heads, int hd, int is_bf16, const int4* pos3,
                       const float* inv_freq, const int* slot_axis, hipStream_t s) {
  const long total = (long)N * heads * (hd / 2);
  if (is_bf16 && hd % 16 == 0 && hd <= 128 && ldqkv % 8 == 0 && (uintptr_t)qkv % 16 == 0) {
    if (N == 0) return hipSuccess;
    hipLaunchKernelGGL(rope_vec_kernel, dim3((N + ROPE_TOK - 1) / ROPE_TOK), dim3(256), 0, s, (bf16*)qkv, ldqkv, N,
                       heads, hd, pos3, inv_freq, slot_axis);
    return hipGetLastError();
  }
  if (is_bf16)
    hipLaunchKernelGGL((rope_kernel<bf16>), dim3(blocks_for(total, 256)), dim3(256), 0, s, (bf16*)qkv, ldqkv, N,
                       heads, hd, pos3, inv_freq, slot_axis);
  else
    hipLaunchKernelGGL((rope_kernel<float>), dim3(blocks_for(total, 256)), dim3(256), 0, s, (float*)qkv, ldqkv, N,
                       heads, hd, pos3, inv_freq, slot_axis);
  return hipGetLastError();
}

hipError_t launch_pad_cols16(const void* src, int rows, int k, int kp, void* dst, hipStream_t s) {
  if (kp % 8 || kp < k || (uintptr_t)dst % 16) return hipErrorInvalidValue;
  if (rows == 0) return hipSuccess;
  hipLaunchKernelGGL(pad_cols16_kernel, dim3(blocks_for((long)rows * (kp / 8), 256)), dim3(256), 0, s,
                     static_cast<const uint16_t*>(src), rows, k, kp, static_cast<uint16_t*>(dst));
  return hipGetLastError();
}

hipError_t launch_cls(const SeqMeta& m, float* x, int d, const void* cls, const void* pos0, int w_bf16, hipStream_t s) {
  if (w_bf16)
    hipLaunchKernelGGL((cls_kernel<bf16>), dim3(m.n), dim3(256), 0, s, m, x, d, (const bf16*)cls, (const bf16*)pos0);
  else
    hipLaunchKernelGGL((cls_kernel<float>), dim3(m.n), dim3(256), 0, s, m, x, d, (const float*)cls, (const float*)pos0);
  return hipGetLastError();
}

hipError_t launch_im2col_k3(const void* src, int frames_in, int C, int n_clips, int stride, int is_bf16, void* dst,
                            hipStream_t s) {
  const int fout = (frames_in - 1) / stride + 1;
  const long total = (long)n_clips * fout * C * 3;
  if (total == 0) return hipSuccess;
  if (is_bf16 && C % 8 == 0 && (uintptr_t)src % 16 == 0 && (uintptr_t)dst % 16 == 0) {
    const long threads = (long)n_clips * fout * (C / 8);
    hipLaunchKernelGGL(im2col_k3_vec_kernel, dim3(blocks_for(threads, 256)), dim3(256), 0, s, (const bf16*)src,
                       frames_in, C, fout, stride, threads, (bf16*)dst);
    return hipGetLastError();
  }
  if (is_bf16)
    hipLaunchKernelGGL((im2col_k3_kernel<bf16>), dim3(blocks_for(total, 256)), dim3(256), 0, s, (const bf16*)src,
                       frames_in, C, fout, stride, total, (bf16*)dst);
  else
    hipLaunchKernelGGL((im2col_k3_kernel<float>), dim3(blocks_for(total, 256)), dim3(256), 0, s, (const float*)src,
                       frames_in, C, fout, stride, total, (float*)dst);
  return hipGetLastError();
}

namespace {

template <int STRIP, int NT>
hipError_t launch_strips(PackArgs& q, int cls, int merge, int patch, int tp, int K, bf16* packed, hipStream_t s) {
  q.strip0[0] = 0;
  for (int r = 0; r < q.n; ++r)
    q.strip0[r + 1] = q.strip0[r] + q.tchw[r][0] / tp * q.hw[r][0] * ((q.hw[r][1] + STRIP - 1) / STRIP);
  constexpr int RP = NT / (8 * STRIP);
  const int rows = merge * patch, C = q.tchw[0][1];
  hipLaunchKernelGGL((pack_vision_vec_kernel<STRIP, NT>), dim3((unsigned)q.strip0[q.n]), dim3(NT),
                     (size_t)STRIP * merge * K * 2, s, q, cls, merge, patch, tp, C, RP % rows, RP / rows % C,
                     RP / rows / C, K, packed);
  return hipGetLastError();
}

hipError_t launch_pack_strips(const PackArgs& p, int cls, int merge, int patch, int tp, int K, bf16* packed,
                              hipStream_t s) {
  PackArgs q = p;
  long n4 = 0;   // strips of four patches
  for (int r = 0; r < p.n; ++r) {
    q.hw[r][0] = p.tchw[r][2] / patch / merge;
    q.hw[r][1] = p.tchw[r][3] / patch;
    n4 += (long)(p.tchw[r][0] / tp) * q.hw[r][0] * ((q.hw[r][1] + 3) / 4);
  }
  // Eight rows at a time cover one frame of patches without the merger (42 rows) in one
  // round of loads; taller strips take 512 threads.  Those hold two patches while
  // four-patch strips would give fewer than three blocks a CU (224 x 224: 4.5 us against
  // 5.5; 1036 x 756, 518 strips of four: 9.8 against 10.3), and four past that
  // (1344 x 1344, 1,152 strips: 17.4 us against 19.3).
  if (K / patch * merge <= 48) return launch_strips<4, 256>(q, cls, merge, patch, tp, K, packed, s);
  if (n4 < 3L * device_cus()) return launch_strips<2, 512>(q, cls, merge, patch, tp, K, packed, s);
  return launch_strips<4, 512>(q, cls, merge, patch, tp, K, packed, s);
}

}  // namespace

hipError_t launch_pack_vision(const PackArgs& p, int cls, int merge, int patch, int tp, int K, int is_bf16,
                              void* packed, long total, hipStream_t s) {
  if (total == 0) return hipSuccess;
  // with the merger every grid is even, so a strip holds whole windows
  bool vec = is_bf16 && patch % 2 == 0 && patch <= 16 && K / patch <= 256 && (uintptr_t)packed % 8 == 0 && merge <= 2;
  for (int r = 0; vec && r < p.n; ++r) vec = p.tchw[r][3] % 2 == 0 && (uintptr_t)p.src[r] % 8 == 0;
  if (vec) return launch_pack_strips(p, cls, merge, patch, tp, K, (bf16*)packed, s);
  if (is_bf16)
    hipLaunchKernelGGL((pack_vision_kernel<bf16>), dim3(blocks_for(total, 256)), dim3(256), 0, s, p, cls, merge, patch,
                       tp, K, total, (bf16*)packed);
  else
    hipLaunchKernelGGL((pack_vision_kernel<float>), dim3(blocks_for(total, 256)), dim3(256), 0, s, p, cls, merge,
                       patch, tp, K, total, (float*)packed);
  return hipGetLastError();
}

hipError_t launch_pack_audio(const PackArgs& p, int n_mels, int n_frames, int is_bf16, void* packed, hipStream_t s) {
  const long total = (long)p.n * n_mels * n_frames;
  if (is_bf16)
    hipLaunchKernelGGL((pack_audio_kernel<bf16>), dim3(blocks_for(total, 256)), dim3(256), 0, s, p, n_mels, n_frames,
                       (bf16*)packed);
  else
    hipLaunchKernelGGL((pack_audio_kernel<float>), dim3(blocks_for(total, 256)), dim3(256), 0, s, p, n_mels, n_frames,
                       (float*)packed);
  return hipGetLastError();
}

}  // namespace eas

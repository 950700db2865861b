// Pooling, the fully connected head and the loss of the sub-ResNet's training step (NHWC).
// Pooling reads and writes activations in their storage type (fp32 or bf16); pooled features,
// logits, loss and everything behind them are fp32.  These are small or bandwidth-bound kernels;
// every reduction runs in a fixed order.
#include <algorithm>

#include "elem.h"
#include "internal.h"

namespace resist {

namespace {

// ---- max pool 3x3 stride 2 pad 1 -----------------------------------------------------------------
// argmax stores the window tap (r*3+s) of the first maximum in row-major window order.
// A thread owns V = 4 (fp32) or 8 (bf16) consecutive channels of one pixel.
template <typename T>
__global__ __launch_bounds__(256) void maxpool_fwd_kernel(const T *__restrict__ x, T *__restrict__ y,
                                                          uint8_t *__restrict__ arg, int N, int H, int W, int C, int P, int Q) {
  constexpr int V = Vec<T>::N;
  const long long total = (long long)N * P * Q * (C / V);
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int c = (int)(i % (C / V)) * V;
  long long pix = i / (C / V);
  const int q = (int)(pix % Q); pix /= Q;
  const int p = (int)(pix % P);
  const int n = (int)(pix / P);
  float best[V];
  int bi[V];
#pragma unroll
  for (int e = 0; e < V; ++e) { best[e] = -INFINITY; bi[e] = 0; }
  bool any = false;
  for (int r = 0; r < 3; ++r) {
    const int ih = p * 2 + r - 1;
    if (ih < 0 || ih >= H) continue;
    for (int s = 0; s < 3; ++s) {
      const int iw = q * 2 + s - 1;
      if (iw < 0 || iw >= W) continue;
      float v[V];
      Vec<T>::load(x + ((size_t)(n * H + ih) * W + iw) * C + c, v);
#pragma unroll
      for (int e = 0; e < V; ++e)
        if (!any || v[e] > best[e]) { best[e] = v[e]; bi[e] = r * 3 + s; }
      any = true;
    }
  }
  const size_t off = ((size_t)(n * P + p) * Q + q) * C + c;
  Vec<T>::store(y + off, best);
#pragma unroll
  for (int e = 0; e < V; e += 4)
    *reinterpret_cast<uchar4 *>(arg + off + e) = make_uchar4((uint8_t)bi[e], (uint8_t)bi[e + 1], (uint8_t)bi[e + 2], (uint8_t)bi[e + 3]);
}

// Gather form.  A thread owns V channels of the 2x2 input pixels (2p, 2q) .. (2p+1, 2q+1): the windows that cover them are (p, q),
// (p, q+1), (p+1, q) and (p+1, q+1), each read once for up to four pixels (a thread to a pixel reads them 2.25 times and the taps byte
// by byte: 112x112, 64 ch, batch 64, bf16 51 -> 32.5 us, 141 MB).
template <typename T>
__global__ __launch_bounds__(256) void maxpool_bwd_kernel(const T *__restrict__ dy, const uint8_t *__restrict__ arg,
                                                          T *__restrict__ dx, int N, int H, int W, int C, int P, int Q) {
  constexpr int V = Vec<T>::N;
  const int PB = (H + 1) / 2, QB = (W + 1) / 2;
  const long long total = (long long)N * PB * QB * (C / V);
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int c = (int)(i % (C / V)) * V;
  long long blk = i / (C / V);
  const int q0 = (int)(blk % QB); blk /= QB;
  const int p0 = (int)(blk % PB);
  const int n = (int)(blk / PB);
  float g[2][2][V];
  unsigned tap[2][2][V / 4];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const bool ok = p0 + a < P && q0 + b < Q;
      const size_t off = ((size_t)(n * P + (ok ? p0 + a : p0)) * Q + (ok ? q0 + b : q0)) * C + c;
      Vec<T>::load(dy + off, g[a][b]);
#pragma unroll
      for (int e = 0; e < V / 4; ++e) {
        tap[a][b][e] = reinterpret_cast<const unsigned *>(arg + off)[e];
        if (!ok) tap[a][b][e] = 0xffffffffu;   // no window: matches no tap
      }
    }
#pragma unroll
  for (int dh = 0; dh < 2; ++dh)
#pragma unroll
    for (int dw = 0; dw < 2; ++dw) {
      const int h = 2 * p0 + dh, w = 2 * q0 + dw;
      if (h >= H || w >= W) continue;
      float acc[V];
#pragma unroll
      for (int e = 0; e < V; ++e) acc[e] = 0.f;
      // window p covers rows 2p-1 .. 2p+1: the even row is row 1 of window p0, the odd one row 2 of it and row 0 of the next
#pragma unroll
      for (int a = 0; a <= dh; ++a)
#pragma unroll
        for (int b = 0; b <= dw; ++b) {
          const unsigned t = (unsigned)((dh ? (a ? 0 : 2) : 1) * 3 + (dw ? (b ? 0 : 2) : 1));
#pragma unroll
          for (int e = 0; e < V; ++e)
            if (((tap[a][b][e / 4] >> (8 * (e % 4))) & 0xffu) == t) acc[e] += g[a][b][e];
        }
      Vec<T>::store(dx + ((size_t)(n * H + h) * W + w) * C + c, acc);
    }
}

// ---- global mean pool ------------------------------------------------------------------------------
// A workgroup owns one sample's `cols` channel vectors (a power of two up to 32), its 256 / cols thread rows share the pixels, eight
// loads in flight each, and meet in LDS.  (One thread to a vector, a load at a time: 16 ch 16x16, batch 4 35 -> 3.2 us;
// 2048 ch 7x7, one image 15 -> 3.2, batch 64 16 -> 5.)
template <typename T>
__global__ __launch_bounds__(256) void avgpool_fwd_kernel(const T *__restrict__ x, float *__restrict__ y, int HW, int C, int cols) {
  constexpr int V = Vec<T>::N, U = 8;
  __shared__ float red[128][V + 1];
  const int tc = threadIdx.x & (cols - 1), tr = threadIdx.x / cols, rows = 256 / cols;
  const int cv = blockIdx.x * cols + tc, n = blockIdx.y;
  float acc[V];
#pragma unroll
  for (int e = 0; e < V; ++e) acc[e] = 0.f;
  if (cv < C / V) {
    const T *src = x + (size_t)n * HW * C + cv * V;
    for (int p = tr; p < HW; p += U * rows) {
      typename Vec<T>::Raw raw[U];
#pragma unroll
      for (int u = 0; u < U; ++u) raw[u] = Vec<T>::load_raw(src + (size_t)min(p + u * rows, HW - 1) * C);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float v[V];
        Vec<T>::unpack(raw[u], v);
#pragma unroll
        for (int e = 0; e < V; ++e) acc[e] += p + u * rows < HW ? v[e] : 0.f;
      }
    }
  }
  // the upper half of the rows hands its sums to the lower half, until one row is left
  for (int half = rows / 2; half >= 1; half >>= 1) {
    if (tr >= half && tr < 2 * half)
#pragma unroll
      for (int e = 0; e < V; ++e) red[threadIdx.x - half * cols][e] = acc[e];
    __syncthreads();
    if (tr < half)
#pragma unroll
      for (int e = 0; e < V; ++e) acc[e] += red[threadIdx.x][e];
    __syncthreads();
  }
  if (tr == 0 && cv < C / V) {
    const float inv = 1.0f / (float)HW;
#pragma unroll
    for (int e = 0; e < V; ++e) y[(size_t)n * C + cv * V + e] = acc[e] * inv;
  }
}

template <typename T>
__global__ __launch_bounds__(256) void avgpool_bwd_kernel(const float *__restrict__ dy, const T *__restrict__ mask, T *__restrict__ dx,
                                                          int N, int HW, int C) {
  constexpr int V = Vec<T>::N;
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long long)N * HW * (C / V)) return;
  const int c = (int)(i % (C / V)) * V;
  const int n = (int)(i / ((long long)HW * (C / V)));
  const float inv = 1.0f / (float)HW;
  float g[V];
#pragma unroll
  for (int e = 0; e < V; ++e) g[e] = dy[(size_t)n * C + c + e] * inv;
  if (mask) {   // the ReLU that produced the pooled tensor: the gradient passes where its output is positive
    float m[V];
    Vec<T>::load(mask + i * V, m);
#pragma unroll
    for (int e = 0; e < V; ++e) g[e] = m[e] > 0.f ? g[e] : 0.f;
  }
  Vec<T>::store(dx + i * V, g);
}

// ---- fully connected -------------------------------------------------------------------------------
__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  return v;
}

// The three small GEMMs of the classifier are register-tiled 4 x 4 (classes x samples, or classes x
// channel vectors) so that every 16-byte load feeds 16 multiply-adds; rows past N or J are handled by
// clamping the row index and discarding the result.  Every sum runs in a fixed order.

// z[n][j] = b[j] + sum_c x[n][c] * w[j][c].  A workgroup owns 4 classes and 16 samples, each of its waves
// 4 of the samples; the 64 lanes stride over the channels, then the 16 dot products are reduced over the lanes.
__global__ __launch_bounds__(256) void fc_fwd_kernel(const float *__restrict__ x, const float *__restrict__ w,
                                                     const float *__restrict__ b, float *__restrict__ z, int N, int C, int J) {
  const int j0 = blockIdx.x * 4, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float *wr[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) wr[k] = w + (size_t)min(j0 + k, J - 1) * C;
  for (int n0 = blockIdx.y * 16 + wave * 4; n0 < N && n0 < (int)blockIdx.y * 16 + 16; n0 += 16) {
    const float *xr[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) xr[s] = x + (size_t)min(n0 + s, N - 1) * C;
    float acc[4][4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int s = 0; s < 4; ++s) acc[k][s] = 0.f;
#pragma unroll 2
    for (int c = lane * 4; c < C; c += 256) {
      f32x4 xv[4], wv[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) xv[s] = *reinterpret_cast<const f32x4 *>(xr[s] + c);
#pragma unroll
      for (int k = 0; k < 4; ++k) wv[k] = *reinterpret_cast<const f32x4 *>(wr[k] + c);
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int s = 0; s < 4; ++s)
          acc[k][s] += xv[s][0] * wv[k][0] + xv[s][1] * wv[k][1] + xv[s][2] * wv[k][2] + xv[s][3] * wv[k][3];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const float t = wave_sum(acc[k][s]);
        if (lane == 0 && j0 + k < J && n0 + s < N) z[(size_t)(n0 + s) * J + j0 + k] = t + b[j0 + k];
      }
  }
}

// dx[n][c] = sum_j dz[n][j] * w[j][c].  A workgroup owns 8 samples and 64 channels: 16 lanes cover the channels (4 each), the 16
// groups of lanes take every 16th class, a piece of dz at a time from LDS, and their partial sums are added in group order.
// (4 samples and 256 channels, every 4th class: 1000 classes, 2048 ch, batch 64 31.7 -> 28.5 us.)  C is a multiple of 4; channels past C are skipped.
constexpr int kDxClasses = 512;   // classes of dz in LDS at a time
__global__ __launch_bounds__(256) void fc_bwd_dx_kernel(const float *__restrict__ dz, const float *__restrict__ w,
                                                        float *__restrict__ dx, int N, int C, int J) {
  __shared__ __attribute__((aligned(16))) float lds[kDxClasses * 8];   // dz [class][sample]; then the partial sums
  static_assert(sizeof(lds) >= 8 * 8 * 16 * 16, "partial sums of half the groups fit");
  const int n0 = blockIdx.y * 8, tx = threadIdx.x & 15, jg = threadIdx.x >> 4;
  const int c = blockIdx.x * 64 + tx * 4;
  f32x4 acc[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) acc[s] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int jb = 0; jb < J; jb += kDxClasses) {
    const int jn = min(J - jb, kDxClasses);
    __syncthreads();
    {
      const int s = threadIdx.x >> 5, l = threadIdx.x & 31;
      const float *src = dz + (size_t)min(n0 + s, N - 1) * J + jb;
      float v[kDxClasses / 32];
#pragma unroll
      for (int i = 0; i < kDxClasses / 32; ++i) v[i] = src[min(l + 32 * i, jn - 1)];
#pragma unroll
      for (int i = 0; i < kDxClasses / 32; ++i) lds[(l + 32 * i) * 8 + s] = v[i];
    }
    __syncthreads();
    if (c < C) {
      constexpr int U = 8;
      for (int j = jg; j < jn; j += 16 * U) {
        f32x4 wv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) wv[u] = *reinterpret_cast<const f32x4 *>(w + (size_t)(jb + min(j + 16 * u, jn - 1)) * C + c);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (j + 16 * u >= jn) break;
          const f32x4 d0 = *reinterpret_cast<const f32x4 *>(&lds[(j + 16 * u) * 8]), d1 = *reinterpret_cast<const f32x4 *>(&lds[(j + 16 * u) * 8 + 4]);
#pragma unroll
          for (int s = 0; s < 8; ++s) {
            const float d = s < 4 ? d0[s & 3] : d1[s & 3];
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[s][e] = fmaf(d, wv[u][e], acc[s][e]);
          }
        }
      }
    }
  }
  // groups 8..15 hand their sums to 0..7, those to group 0 .. 3, and so on: ((0 + 8) + (4 + 12)) + ...
  f32x4 (*red)[8][16] = reinterpret_cast<f32x4 (*)[8][16]>(lds);
#pragma unroll
  for (int half = 8; half >= 1; half >>= 1) {
    __syncthreads();
    if (jg >= half && jg < 2 * half)
#pragma unroll
      for (int s = 0; s < 8; ++s) red[jg - half][s][tx] = acc[s];
    __syncthreads();
    if (jg < half)
#pragma unroll
      for (int s = 0; s < 8; ++s) acc[s] += red[jg][s][tx];
  }
  if (jg == 0 && c < C) {
#pragma unroll
    for (int s = 0; s < 8; ++s)
      if (n0 + s < N) *reinterpret_cast<f32x4 *>(dx + (size_t)(n0 + s) * C + c) = acc[s];
  }
}

// dw[j][c] = sum_n dz[n][j] * x[n][c].  A thread owns 4 classes x 4 consecutive channels; blockIdx.y selects the group of 4 classes.
// The G waves of a workgroup share the samples, four in flight each, and their sums are added in wave order.
// (All samples in one thread, two in flight: 10 classes, 512 ch, batch 128 22 -> 5.6 us.)
template <int G>
__global__ __launch_bounds__(64 * G) void fc_bwd_dw_kernel(const float *__restrict__ dz, const float *__restrict__ x,
                                                           float *__restrict__ dw, int N, int C, int J) {
  __shared__ f32x4 red[G][4][64];
  const int tx = threadIdx.x & 63, g = threadIdx.x >> 6;
  const int c = (blockIdx.x * 64 + tx) * 4;
  const int j0 = blockIdx.y * 4;
  f32x4 acc[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) acc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (c < C) {
    int jr[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) jr[k] = min(j0 + k, J - 1);
    constexpr int U = 4;
    for (int n = g; n < N; n += G * U) {
      f32x4 xv[U];
      float d[U][4];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int m = min(n + G * u, N - 1);
        xv[u] = *reinterpret_cast<const f32x4 *>(x + (size_t)m * C + c);
#pragma unroll
        for (int k = 0; k < 4; ++k) d[u][k] = dz[(size_t)m * J + jr[k]];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (n + G * u >= N) break;
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[k][e] = fmaf(d[u][k], xv[u][e], acc[k][e]);
      }
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) red[g][k][tx] = acc[k];
  __syncthreads();
  if (g < 4 && c < C && j0 + g < J) {   // wave g finishes class j0 + g
    f32x4 t = red[0][g][tx];
#pragma unroll
    for (int i = 1; i < G; ++i) t += red[i][g][tx];
    *reinterpret_cast<f32x4 *>(dw + (size_t)(j0 + g) * C + c) = t;
  }
}

// db over the padded length (multiple of 4): entries past J are written as zero.  One wave to a class.
__global__ __launch_bounds__(256) void fc_bwd_db_kernel(const float *__restrict__ dz, float *__restrict__ db, int N, int J, int Jpad) {
  const int lane = threadIdx.x & 63, j = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (j >= Jpad) return;
  float acc = 0.f;
  if (j < J)
    for (int n = lane; n < N; n += 64) acc += dz[(size_t)n * J + j];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if (lane == 0) db[j] = acc;
}

// ---- softmax cross-entropy ---------------------------------------------------------------------------
// one wave per sample: row_loss[n] = logsumexp(z_n) - z_n[label]; dz = (softmax - onehot)/N
__global__ __launch_bounds__(64) void softmax_ce_kernel(const float *__restrict__ z, const int32_t *__restrict__ labels,
                                                        float *__restrict__ row_loss, float *__restrict__ dz, int N, int J) {
  const int n = blockIdx.x, lane = threadIdx.x;
  const float *zr = z + (size_t)n * J;
  float mx = -INFINITY;
  for (int j = lane; j < J; j += 64) mx = fmaxf(mx, zr[j]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
  float se = 0.f;
  for (int j = lane; j < J; j += 64) se += expf(zr[j] - mx);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) se += __shfl_xor(se, o, 64);
  const int lab = labels[n];
  const float invN = 1.0f / (float)N;
  const float inv = 1.0f / se;
  for (int j = lane; j < J; j += 64) {
    const float p = expf(zr[j] - mx) * inv;
    dz[(size_t)n * J + j] = (p - (j == lab ? 1.f : 0.f)) * invN;
  }
  // a label outside [0,J) is a caller error: it must not turn into an out-of-bounds read
  if (lane == 0) row_loss[n] = (lab >= 0 && lab < J) ? (logf(se) + mx) - zr[lab] : NAN;
}

__global__ __launch_bounds__(64) void mean_loss_kernel(const float *__restrict__ row_loss, float *__restrict__ loss, int N) {
  double acc = 0;
  for (int n = threadIdx.x; n < N; n += 64) acc += (double)row_loss[n];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if (threadIdx.x == 0) *loss = (float)(acc / (double)N);
}

unsigned blocks_for(long long n, int t = 256) { return (unsigned)((n + t - 1) / t); }

}  // namespace

int maxpool_fwd(int dt, const void *x, void *y, uint8_t *argmax, int N, int H, int W, int C, int P, int Q, hipStream_t st) {
  const int V = dt == DT_BF16 ? 8 : 4;
  if (C % V) return set_error(RESIST_ESHAPE, "max-pool: C=%d must be a multiple of %d", C, V);
  prof::Scope ps("maxpool_fwd", 0, (double)esize(dt) * N * C * ((double)H * W + (double)P * Q) + (double)N * P * Q * C, st);
  const dim3 grid(blocks_for((long long)N * P * Q * (C / V)));
  if (dt == DT_BF16) hipLaunchKernelGGL(maxpool_fwd_kernel<__bf16>, grid, dim3(256), 0, st, (const __bf16 *)x, (__bf16 *)y, argmax, N, H, W, C, P, Q);
  else hipLaunchKernelGGL(maxpool_fwd_kernel<float>, grid, dim3(256), 0, st, (const float *)x, (float *)y, argmax, N, H, W, C, P, Q);
  RESIST_CHECK_LAUNCH("maxpool_fwd");
  return RESIST_OK;
}
int maxpool_bwd(int dt, const void *dy, const uint8_t *argmax, void *dx, int N, int H, int W, int C, int P, int Q, hipStream_t st) {
  const int V = dt == DT_BF16 ? 8 : 4;
  if (C % V) return set_error(RESIST_ESHAPE, "max-pool: C=%d must be a multiple of %d", C, V);
  prof::Scope ps("maxpool_bwd", 0, (double)esize(dt) * N * C * ((double)H * W + (double)P * Q) + (double)N * P * Q * C, st);
  const dim3 grid(blocks_for((long long)N * ((H + 1) / 2) * ((W + 1) / 2) * (C / V)));
  if (dt == DT_BF16) hipLaunchKernelGGL(maxpool_bwd_kernel<__bf16>, grid, dim3(256), 0, st, (const __bf16 *)dy, argmax, (__bf16 *)dx, N, H, W, C, P, Q);
  else hipLaunchKernelGGL(maxpool_bwd_kernel<float>, grid, dim3(256), 0, st, (const float *)dy, argmax, (float *)dx, N, H, W, C, P, Q);
  RESIST_CHECK_LAUNCH("maxpool_bwd");
  return RESIST_OK;
}
int avgpool_fwd(int dt, const void *x, float *y, int N, int HW, int C, hipStream_t st) {
  const int V = dt == DT_BF16 ? 8 : 4;
  if (C % V) return set_error(RESIST_ESHAPE, "mean pool: C=%d must be a multiple of %d", C, V);
  prof::Scope ps("avgpool_fwd", 0, 0, st);
  int cols = 1;
  while (cols < 32 && cols < C / V) cols *= 2;
  for (int n = 0; n < N; n += 65535) {   // samples along the grid's second axis
    const dim3 grid((C / V + cols - 1) / cols, std::min(N - n, 65535));
    const size_t in = (size_t)n * HW * C;
    if (dt == DT_BF16) hipLaunchKernelGGL(avgpool_fwd_kernel<__bf16>, grid, dim3(256), 0, st, (const __bf16 *)x + in, y + (size_t)n * C, HW, C, cols);
    else hipLaunchKernelGGL(avgpool_fwd_kernel<float>, grid, dim3(256), 0, st, (const float *)x + in, y + (size_t)n * C, HW, C, cols);
  }
  RESIST_CHECK_LAUNCH("avgpool_fwd");
  return RESIST_OK;
}
int avgpool_bwd(int dt, const float *dy, const void *relu_mask, void *dx, int N, int HW, int C, hipStream_t st) {
  const int V = dt == DT_BF16 ? 8 : 4;
  if (C % V) return set_error(RESIST_ESHAPE, "mean pool: C=%d must be a multiple of %d", C, V);
  prof::Scope ps("avgpool_bwd", 0, 0, st);
  const dim3 grid(blocks_for((long long)N * HW * (C / V)));
  if (dt == DT_BF16) hipLaunchKernelGGL(avgpool_bwd_kernel<__bf16>, grid, dim3(256), 0, st, dy, (const __bf16 *)relu_mask, (__bf16 *)dx, N, HW, C);
  else hipLaunchKernelGGL(avgpool_bwd_kernel<float>, grid, dim3(256), 0, st, dy, (const float *)relu_mask, (float *)dx, N, HW, C);
  RESIST_CHECK_LAUNCH("avgpool_bwd");
  return RESIST_OK;
}
int fc_fwd_f32(const float *x, const float *w, const float *b, float *z, int N, int C, int J, hipStream_t st) {
  prof::Scope ps("fc_fwd", 0, 0, st);
  if (C % 4 || N < 1 || J < 1) return set_error(RESIST_ESHAPE, "fully connected layer: N=%d C=%d J=%d (C must be a multiple of 4)", N, C, J);
  hipLaunchKernelGGL(fc_fwd_kernel, dim3((J + 3) / 4, (N + 15) / 16), dim3(256), 0, st, x, w, b, z, N, C, J);
  RESIST_CHECK_LAUNCH("fc_fwd");
  return RESIST_OK;
}
int fc_bwd_dx_f32(const float *dz, const float *w, float *dx, int N, int C, int J, hipStream_t st) {
  prof::Scope ps("fc_bwd_dx", 0, 0, st);
  if (C % 4) return set_error(RESIST_ESHAPE, "fully connected layer: C=%d must be a multiple of 4", C);
  hipLaunchKernelGGL(fc_bwd_dx_kernel, dim3((C + 63) / 64, (N + 7) / 8), dim3(256), 0, st, dz, w, dx, N, C, J);
  RESIST_CHECK_LAUNCH("fc_bwd_dx");
  return RESIST_OK;
}
int fc_bwd_params_f32(const float *dz, const float *x, float *dw, float *db, int N, int C, int J, hipStream_t st) {
  prof::Scope ps("fc_bwd_params", 0, 0, st);
  if (C % 4) return set_error(RESIST_ESHAPE, "fully connected layer: C=%d must be a multiple of 4", C);
  const dim3 grid((C / 4 + 63) / 64, (J + 3) / 4);
  // sixteen waves share the samples where there are few workgroups
  if (grid.x * grid.y < 256) hipLaunchKernelGGL(fc_bwd_dw_kernel<16>, grid, dim3(1024), 0, st, dz, x, dw, N, C, J);
  else hipLaunchKernelGGL(fc_bwd_dw_kernel<4>, grid, dim3(256), 0, st, dz, x, dw, N, C, J);
  RESIST_CHECK_LAUNCH("fc_bwd_dw");
  const int Jpad = (J + 3) & ~3;
  hipLaunchKernelGGL(fc_bwd_db_kernel, dim3(Jpad / 4), dim3(256), 0, st, dz, db, N, J, Jpad);
  RESIST_CHECK_LAUNCH("fc_bwd_db");
  return RESIST_OK;
}
int softmax_ce_f32(const float *z, const int32_t *labels, float *dz, float *row_loss, int N, int J, hipStream_t st) {
  prof::Scope ps("softmax_ce", 0, 0, st);
  hipLaunchKernelGGL(softmax_ce_kernel, dim3(N), dim3(64), 0, st, z, labels, row_loss, dz, N, J);
  RESIST_CHECK_LAUNCH("softmax_ce");
  return RESIST_OK;
}
int mean_loss_f32(const float *row_loss, float *loss, int N, hipStream_t st) {
  prof::Scope ps("mean_loss", 0, 0, st);
  hipLaunchKernelGGL(mean_loss_kernel, dim3(1), dim3(64), 0, st, row_loss, loss, N);
  RESIST_CHECK_LAUNCH("mean_loss");
  return RESIST_OK;
}

}  // namespace resist

// GroupNorm forward/backward, max pool 3x3/2, frame preparation (2x2 average
// pool + NCHW -> NHWC), and small elementwise helpers.
//
// Activations are [B][P][C] (NHWC, P = H*W pixels).  GroupNorm statistics are
// gathered in two steps: every workgroup reduces one chunk of pixels of one
// image for all channels into per-channel shifted sums, then one wavefront
// per (image, group) merges the chunk results with the exact
// parallel-variance formula (each chunk's centred second moment plus n_i
// (mean_i - mean)^2), all in float32.
#include "common.h"
#include "kernels.h"

// ------------------------------------------------------------------ forward
// part[(b*S + s)*C + c] = {sum(y - K), sum((y - K)^2), K}, K = y at the chunk's
// first pixel.
__global__ void __launch_bounds__(256) gn_partial_kernel(const float* __restrict__ y, int P, int C,
                                                         int S, float4* __restrict__ part) {
  // lanes take channel quads (float4 loads), the rest of the block walks pixels
  __shared__ float4 s1[256], s2[256];
  const int b = blockIdx.y, s = blockIdx.x, tid = threadIdx.x;
  const int chunk = (P + S - 1) / S;
  const int p0 = s * chunk, p1 = min(P, p0 + chunk);
  const float* yb = y + (size_t)b * P * C;
  const int C4 = C >> 2;
  const int QT = C4 < 256 ? C4 : 256;  // channel quads per pass
  const int PR = 256 / QT;             // pixel lanes
  const int q0 = tid % QT, pr = tid / QT;
  for (int qb = 0; qb < C4; qb += QT) {
    const int c = 4 * (qb + q0);
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f), q = a, K = a;
    if (p0 < p1 && pr < PR) {
      K = *(const float4*)(yb + (size_t)p0 * C + c);
#pragma unroll 4
      for (int p = p0 + pr; p < p1; p += PR) {
        const float4 v = *(const float4*)(yb + (size_t)p * C + c);
        const float4 d = make_float4(v.x - K.x, v.y - K.y, v.z - K.z, v.w - K.w);
        a.x += d.x; a.y += d.y; a.z += d.z; a.w += d.w;
        q.x += d.x * d.x; q.y += d.y * d.y; q.z += d.z * d.z; q.w += d.w * d.w;
      }
    }
    s1[tid] = a;
    s2[tid] = q;
    __syncthreads();
    if (pr == 0) {
      for (int r = 1; r < PR; ++r) {
        const float4 u = s1[r * QT + q0], w = s2[r * QT + q0];
        a.x += u.x; a.y += u.y; a.z += u.z; a.w += u.w;
        q.x += w.x; q.y += w.y; q.z += w.z; q.w += w.w;
      }
      const float n = (float)max(0, p1 - p0);
      float4* o = part + ((size_t)b * S + s) * C + c;
      o[0] = make_float4(a.x, q.x, K.x, n);
      o[1] = make_float4(a.y, q.y, K.y, n);
      o[2] = make_float4(a.z, q.z, K.z, n);
      o[3] = make_float4(a.w, q.w, K.w, n);
    }
    __syncthreads();
  }
}

// One wavefront per (b, g): mean and 1/sqrt(var + eps) of the group.
__global__ void __launch_bounds__(256) gn_finalize_kernel(const float4* __restrict__ part, int B, int S,
                                                          int C, int G, float eps,
                                                          float2* __restrict__ stats) {
  const int wid = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (wid >= B * G) return;
  const int b = wid / G, g = wid % G, Cg = C / G;
  const int nparts = S * Cg;
  float sn = 0.f, sx = 0.f;
#pragma unroll 4
  for (int i = lane; i < nparts; i += 64) {
    const int s = i / Cg, c = g * Cg + i % Cg;
    const float4 v = part[((size_t)b * S + s) * C + c];
    sn += v.w;
    sx += fmaf(v.w, v.z, v.x);  // n K + sum(y - K)
  }
  sn = wave_sum(sn);
  sx = wave_sum(sx);
  const float mean = sn > 0.f ? sx / sn : 0.f;
  float m2 = 0.f;
#pragma unroll 4
  for (int i = lane; i < nparts; i += 64) {
    const int s = i / Cg, c = g * Cg + i % Cg;
    const float4 v = part[((size_t)b * S + s) * C + c];
    if (v.w > 0.f) {
      const float n = v.w, a = v.x / n;  // chunk mean - K
      const float m2i = fmaxf(v.y - v.x * a, 0.f);
      const float d = (v.z - mean) + a;
      m2 += fmaf(n * d, d, m2i);
    }
  }
  m2 = wave_sum(m2);
  if (lane == 0) {
    const float var = sn > 0.f ? fmaxf(m2 / sn, 0.f) : 0.f;
    stats[wid] = make_float2(mean, 1.0f / sqrtf(var + eps));
  }
}

// Divisors of the elementwise kernels: quads a pixel, pixels an image, channels a group.
struct GnDiv {
  FastDiv c4, p, cg;
};
// Workgroups of a pass over n4 quads: a quad a thread, or 8192 workgroups where a
// step of that many threads would take the 32-bit index past 2^31.
static int quad_blocks(size_t n4) {
  const size_t nb = std::min<size_t>(1 << 20, (n4 + 255) / 256);
  return n4 + 256 * nb <= 1ull << 31 ? (int)nb : 8192;
}
static GnDiv gn_div(int P, int C, int G) { return GnDiv{fast_div(C / 4), fast_div(P), fast_div(C / G)}; }

// (y - mean) rstd gamma + beta: what gn_apply_kernel puts out, and what
// gn_fused_kernel does (which adds a 0 residual, of no effect on the sign).  The
// backward recomputes the ReLU mask of units without a residual with the same
// functions, each operation spelled out, so that the two agree at the border
// whatever the compiler contracts elsewhere.
DEV float gn_value(float y, float2 st, float gamma, float beta) {
  return fmaf((y - st.x) * st.y, gamma, beta);
}
DEV float gn_value_fused(float y, float2 st, float gamma, float beta) { return fmaf(y - st.x, gamma * st.y, beta); }

// out = [relu]( (y - mean) rstd gamma + beta [+ res] ), written NHWC or,
// with out_chw, as [B][C][P].  Memory-bound: a quad per thread (256 frames,
// all GroupNorm passes of an update: 45 us less than 8192 workgroups striding).
__global__ void __launch_bounds__(256) gn_apply_kernel(const float* __restrict__ y, int n4, int P,
                                                       int C, int G, GnDiv dv, const float2* __restrict__ stats,
                                                       const float* __restrict__ gamma,
                                                       const float* __restrict__ beta,
                                                       const float* __restrict__ res, int relu,
                                                       float* __restrict__ out, int out_chw) {
  const int C4 = C >> 2;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n4; i += gridDim.x * 256) {
    const int row = dv.c4.div(i), c = 4 * (i - row * C4);
    const int b = dv.p.div(row), p = row - b * P;
    const size_t e = (size_t)row * C + c;
    const float4 v = *(const float4*)(y + e);
    const float r[4] = {v.x, v.y, v.z, v.w};
    float4 rr = make_float4(0.f, 0.f, 0.f, 0.f);
    if (res) rr = *(const float4*)(res + e);
    const float ra[4] = {rr.x, rr.y, rr.z, rr.w};
    float o[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      o[j] = gn_value(r[j], stats[b * G + dv.cg.div(c + j)], gamma[c + j], beta[c + j]) + ra[j];
      if (relu) o[j] = fmaxf(o[j], 0.f);
    }
    if (!out_chw) {
      *(float4*)(out + e) = make_float4(o[0], o[1], o[2], o[3]);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) out[((size_t)b * C + c + j) * P + p] = o[j];
    }
  }
}

void launch_gn_forward(const float* y, int B, int P, int C, int G, float eps, const float* gamma,
                       const float* beta, const float* res, int relu, float* out, int out_chw,
                       float2* stats, float4* part, int S, hipStream_t s) {
  hipLaunchKernelGGL(gn_partial_kernel, dim3(S, B), dim3(256), 0, s, y, P, C, S, part);
  hipLaunchKernelGGL(gn_finalize_kernel, dim3(cdiv((long)B * G, 4)), dim3(256), 0, s, part, B, S, C,
                     G, eps, stats);
  const size_t n4 = (size_t)B * P * C / 4;
  const int nb = quad_blocks(n4);
  hipLaunchKernelGGL(gn_apply_kernel, dim3(nb), dim3(256), 0, s, y, (int)n4, P, C, G, gn_div(P, C, G), stats, gamma,
                     beta, res, relu, out, out_chw);
}

// ----------------------------------------------------------------- backward
// dz = dout * mask, xhat = (y - mean) rstd.  The mask: none (kMaskNone), [out >
// 0] of the saved output (kMaskOut), or of the output formed again from y,
// which saves reading it (kMaskApply, kMaskFused: as the forward's kernel of
// that name formed it; units without a residual).  The passes run at the rate
// of HBM, so the bytes count.  256 frames: sums 1.05 -> 0.93 ms in all (with
// four pixels' loads in flight); a whole bfloat16 update 12.79 -> 12.65 ms,
// SE-ResNeXt 11.12 -> 10.83 ms.
enum { kMaskNone, kMaskOut, kMaskApply, kMaskFused };
// bpart[(b*S + s)*C + c] = {sum dz, sum dz xhat}.
DEV size_t io_index(int b, int p, int c, int P, int C, int chw) {
  return chw ? ((size_t)b * C + c) * P + p : ((size_t)b * P + p) * C + c;
}

template <int MASK>
__global__ void __launch_bounds__(256) gnb_partial_kernel(const float* __restrict__ dout,
                                                          const float* __restrict__ out, int chw,
                                                          const float* __restrict__ y, int P, int C,
                                                          int G, int S, const float2* __restrict__ stats,
                                                          const float* __restrict__ gamma,
                                                          const float* __restrict__ beta,
                                                          float2* __restrict__ bpart) {
  __shared__ float4 s1[256], s2[256];
  const int b = blockIdx.y, s = blockIdx.x, tid = threadIdx.x;
  const int chunk = (P + S - 1) / S;
  const int p0 = s * chunk, p1 = min(P, p0 + chunk);
  const int C4 = C >> 2;
  const int QT = C4 < 256 ? C4 : 256;
  const int PR = 256 / QT;
  const int q0 = tid % QT, pr = tid / QT;
  const int Cg = C / G;
  for (int qb = 0; qb < C4; qb += QT) {
    const int c = 4 * (qb + q0);
    float a[4] = {0.f, 0.f, 0.f, 0.f}, q[4] = {0.f, 0.f, 0.f, 0.f};
    if (pr < PR) {
      float2 st[4];
      float gm[4] = {}, bt[4] = {};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        st[j] = stats[b * G + (c + j) / Cg];
        if (MASK >= kMaskApply) {
          gm[j] = gamma[c + j];
          bt[j] = beta[c + j];
        }
      }
#pragma unroll 4
      for (int p = p0 + pr; p < p1; p += PR) {
        const size_t e = ((size_t)b * P + p) * C + c;
        float dz[4], om[4] = {1.f, 1.f, 1.f, 1.f};
        if (!chw) {
          const float4 d = *(const float4*)(dout + e);
          dz[0] = d.x; dz[1] = d.y; dz[2] = d.z; dz[3] = d.w;
          if (MASK == kMaskOut) {
            const float4 m = *(const float4*)(out + e);
            om[0] = m.x; om[1] = m.y; om[2] = m.z; om[3] = m.w;
          }
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const size_t io = ((size_t)b * C + c + j) * P + p;
            dz[j] = dout[io];
            if (MASK == kMaskOut) om[j] = out[io];
          }
        }
        const float4 yv = *(const float4*)(y + e);
        const float yy[4] = {yv.x, yv.y, yv.z, yv.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (MASK == kMaskApply) om[j] = gn_value(yy[j], st[j], gm[j], bt[j]);
          if (MASK == kMaskFused) om[j] = gn_value_fused(yy[j], st[j], gm[j], bt[j]);
          const float z = om[j] > 0.f ? dz[j] : 0.f;
          a[j] += z;
          q[j] += z * (yy[j] - st[j].x) * st[j].y;
        }
      }
    }
    s1[tid] = make_float4(a[0], a[1], a[2], a[3]);
    s2[tid] = make_float4(q[0], q[1], q[2], q[3]);
    __syncthreads();
    if (pr == 0) {
      for (int r = 1; r < PR; ++r) {
        const float4 u = s1[r * QT + q0], w = s2[r * QT + q0];
        a[0] += u.x; a[1] += u.y; a[2] += u.z; a[3] += u.w;
        q[0] += w.x; q[1] += w.y; q[2] += w.z; q[3] += w.w;
      }
      float2* o = bpart + ((size_t)b * S + s) * C + c;
#pragma unroll
      for (int j = 0; j < 4; ++j) o[j] = make_float2(a[j], q[j]);
    }
    __syncthreads();
  }
}

// Two reductions of the chunk partials in one launch (one wavefront per item):
//   items [0, B G):    coef[b*G+g] = {sum_c gamma_c sum dz / n, sum_c gamma_c sum dz xhat / n}
//   items [B G, +C):   dgamma[c] = sum_{b,s} sum dz xhat, dbeta[c] = sum_{b,s} sum dz
__global__ void __launch_bounds__(256) gnb_coef_affine_kernel(const float2* __restrict__ bpart, int B, int S,
                                                              int C, int G, int P,
                                                              const float* __restrict__ gamma,
                                                              float2* __restrict__ coef, float* __restrict__ dgamma,
                                                              float* __restrict__ dbeta) {
  const int wid = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (wid < B * G) {
    const int b = wid / G, g = wid % G, Cg = C / G;
    float a = 0.f, q = 0.f;
#pragma unroll 4
    for (int i = lane; i < S * Cg; i += 64) {
      const int s = i / Cg, c = g * Cg + i % Cg;
      const float2 v = bpart[((size_t)b * S + s) * C + c];
      a = fmaf(gamma[c], v.x, a);
      q = fmaf(gamma[c], v.y, q);
    }
    a = wave_sum(a);
    q = wave_sum(q);
    if (lane == 0) {
      const float n = (float)P * (float)Cg;
      coef[wid] = make_float2(a / n, q / n);
    }
    return;
  }
  const int c = wid - B * G;
  if (c >= C) return;
  float a = 0.f, q = 0.f;
#pragma unroll 4
  for (int i = lane; i < B * S; i += 64) {
    const float2 v = bpart[(size_t)i * C + c];
    a += v.x;
    q += v.y;
  }
  a = wave_sum(a);
  q = wave_sum(q);
  if (lane == 0) {
    dgamma[c] = q;
    dbeta[c] = a;
  }
}

// dgamma / dbeta only (the one-launch backward's per-image partials, S = 1).
__global__ void __launch_bounds__(256) gnb_affine_kernel(const float2* __restrict__ bpart, int B, int S,
                                                         int C, float* __restrict__ dgamma,
                                                         float* __restrict__ dbeta) {
  const int c = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (c >= C) return;
  float a = 0.f, q = 0.f;
#pragma unroll 4
  for (int i = lane; i < B * S; i += 64) {
    const float2 v = bpart[(size_t)i * C + c];
    a += v.x;
    q += v.y;
  }
  a = wave_sum(a);
  q = wave_sum(q);
  if (lane == 0) {
    dgamma[c] = q;
    dbeta[c] = a;
  }
}

// dy = rstd (dz gamma - coef.x - xhat coef.y); dres (optional) = dz.  NHWC outputs.
template <int MASK>
__global__ void __launch_bounds__(256) gnb_apply_kernel(const float* __restrict__ dout,
                                                        const float* __restrict__ out, int chw,
                                                        const float* __restrict__ y, int n4, int P, int C,
                                                        int G, GnDiv dv, const float2* __restrict__ stats,
                                                        const float2* __restrict__ coef,
                                                        const float* __restrict__ gamma,
                                                        const float* __restrict__ beta,
                                                        float* __restrict__ dy, float* __restrict__ dres) {
  const int C4 = C >> 2;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n4; i += gridDim.x * 256) {
    const int row = dv.c4.div(i), c = 4 * (i - row * C4);
    const int b = dv.p.div(row), p = row - b * P;
    const size_t e = (size_t)row * C + c;
    float dz[4], om[4] = {1.f, 1.f, 1.f, 1.f};
    if (!chw) {
      const float4 d = *(const float4*)(dout + e);
      dz[0] = d.x; dz[1] = d.y; dz[2] = d.z; dz[3] = d.w;
      if (MASK == kMaskOut) {
        const float4 m = *(const float4*)(out + e);
        om[0] = m.x; om[1] = m.y; om[2] = m.z; om[3] = m.w;
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const size_t io = ((size_t)b * C + c + j) * P + p;
        dz[j] = dout[io];
        if (MASK == kMaskOut) om[j] = out[io];
      }
    }
    const float4 yv = *(const float4*)(y + e);
    const float yy[4] = {yv.x, yv.y, yv.z, yv.w};
    float o[4], zz[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int bg = b * G + dv.cg.div(c + j);
      const float2 st = stats[bg], cf = coef[bg];
      if (MASK == kMaskApply) om[j] = gn_value(yy[j], st, gamma[c + j], beta[c + j]);
      if (MASK == kMaskFused) om[j] = gn_value_fused(yy[j], st, gamma[c + j], beta[c + j]);
      const float z = om[j] > 0.f ? dz[j] : 0.f;
      zz[j] = z;
      o[j] = st.y * (z * gamma[c + j] - cf.x - (yy[j] - st.x) * st.y * cf.y);
    }
    *(float4*)(dy + e) = make_float4(o[0], o[1], o[2], o[3]);
    if (dres) *(float4*)(dres + e) = make_float4(zz[0], zz[1], zz[2], zz[3]);
  }
}

void launch_gn_backward(const float* dout, const float* out, GnMask mask, int chw, const float* y, int B, int P,
                        int C, int G, const float2* stats, const float* gamma, const float* beta, float* dy,
                        float* dres, float* dgamma, float* dbeta, float2* bpart, float2* coef, int S,
                        hipStream_t s) {
  const size_t n = (size_t)B * P * C / 4;
  const int nb = quad_blocks(n);
  auto run = [&](auto partial, auto apply) {
    hipLaunchKernelGGL(partial, dim3(S, B), dim3(256), 0, s, dout, out, chw, y, P, C, G, S, stats, gamma, beta,
                       bpart);
    hipLaunchKernelGGL(gnb_coef_affine_kernel, dim3(cdiv((long)B * G + C, 4)), dim3(256), 0, s, bpart, B, S, C,
                       G, P, gamma, coef, dgamma, dbeta);
    hipLaunchKernelGGL(apply, dim3(nb), dim3(256), 0, s, dout, out, chw, y, (int)n, P, C, G, gn_div(P, C, G), stats,
                       coef, gamma, beta, dy, dres);
  };
  switch (mask) {
    case GnMask::none: return run(gnb_partial_kernel<kMaskNone>, gnb_apply_kernel<kMaskNone>);
    case GnMask::out: return run(gnb_partial_kernel<kMaskOut>, gnb_apply_kernel<kMaskOut>);
    case GnMask::apply: return run(gnb_partial_kernel<kMaskApply>, gnb_apply_kernel<kMaskApply>);
    case GnMask::fused: return run(gnb_partial_kernel<kMaskFused>, gnb_apply_kernel<kMaskFused>);
  }
}

// ------------------------------------------------------------------ pooling
// 3x3 window, stride 2, padding 1; arg = index 0..8 of the first maximum in
// row-major window order.  Memory-bound: a thread takes four channels of an
// output pixel (16-byte loads, all nine in flight), quad indices in 32 bits
// with multiply-shift divisors.  256 frames of 64x64x32: 50.0 us with a channel
// per thread, 38.4 us so.  Quads and their indices stay below 2^31, as the
// 32-bit offsets of the convolutions around the pool need.
__global__ void __launch_bounds__(256) maxpool_fwd_kernel(const float* __restrict__ x, int n4, int H, int W,
                                                          int C4, int Ho, int Wo, FastDiv dC4, FastDiv dWo,
                                                          FastDiv dHo, float* __restrict__ y,
                                                          uint8_t* __restrict__ arg) {
  for (int e = blockIdx.x * 256 + threadIdx.x; e < n4; e += gridDim.x * 256) {
    const int px = dC4.div(e), c = e - px * C4, r = dWo.div(px), wo = px - r * Wo, b = dHo.div(r), ho = r - b * Ho;
    // outside taps read a clamped in-bounds element and are skipped
    float4 v[9];
    bool ok[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int hi = 2 * ho - 1 + t / 3, wi = 2 * wo - 1 + t % 3;
      ok[t] = hi >= 0 && hi < H && wi >= 0 && wi < W;
      const size_t p = ((size_t)b * H + min(max(hi, 0), H - 1)) * W + min(max(wi, 0), W - 1);
      v[t] = ((const float4*)x)[p * C4 + c];
    }
    float best[4];
    uint8_t bi[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      best[j] = -INFINITY;
      bi[j] = 0;
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const float u = j == 0 ? v[t].x : j == 1 ? v[t].y : j == 2 ? v[t].z : v[t].w;
        if (ok[t] && u > best[j]) {
          best[j] = u;
          bi[j] = (uint8_t)t;
        }
      }
    }
    ((float4*)y)[e] = make_float4(best[0], best[1], best[2], best[3]);
    ((uchar4*)arg)[e] = make_uchar4(bi[0], bi[1], bi[2], bi[3]);
  }
}

// dx[b,h,w,c] = sum of dy over the (at most 4) windows whose winner is (h, w):
// four channels per thread, as above (164 us with one, 49.9 us so: 176 MB, 3.5 TB/s).
__global__ void __launch_bounds__(256) maxpool_bwd_kernel(const float* __restrict__ dy,
                                                          const uint8_t* __restrict__ arg, int n4, int H, int W,
                                                          int C4, int Ho, int Wo, FastDiv dC4, FastDiv dW,
                                                          FastDiv dH, float* __restrict__ dx) {
  for (int e = blockIdx.x * 256 + threadIdx.x; e < n4; e += gridDim.x * 256) {
    const int px = dC4.div(e), c = e - px * C4, r = dW.div(px), w = px - r * W, b = dH.div(r), h = r - b * H;
    // windows ho = h/2, (h+1)/2 and wo likewise (one of each for even h, w)
    uchar4 a[4];
    float4 d[4];
    int tap[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int ho = h / 2 + (q >> 1), wo = w / 2 + (q & 1);
      const int kh = h - (2 * ho - 1), kw = w - (2 * wo - 1);
      const bool ok = ho <= min(Ho - 1, (h + 1) / 2) && wo <= min(Wo - 1, (w + 1) / 2);
      tap[q] = ok && kh >= 0 && kh <= 2 && kw >= 0 && kw <= 2 ? kh * 3 + kw : -1;
      const size_t o = (((size_t)b * Ho + min(ho, Ho - 1)) * Wo + min(wo, Wo - 1)) * C4 + c;
      a[q] = ((const uchar4*)arg)[o];
      d[q] = ((const float4*)dy)[o];
    }
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (a[q].x == tap[q]) s.x += d[q].x;
      if (a[q].y == tap[q]) s.y += d[q].y;
      if (a[q].z == tap[q]) s.z += d[q].z;
      if (a[q].w == tap[q]) s.w += d[q].w;
    }
    ((float4*)dx)[e] = s;
  }
}

// C % 4 == 0 (every trunk width is a multiple of 4).
void launch_maxpool_fwd(const float* x, int B, int H, int W, int C, float* y, uint8_t* arg,
                        hipStream_t s) {
  const int Ho = (H - 1) / 2 + 1, Wo = (W - 1) / 2 + 1, C4 = C / 4;
  const size_t n4 = (size_t)B * Ho * Wo * C4;
  hipLaunchKernelGGL(maxpool_fwd_kernel, dim3((int)std::min<size_t>(8192, (n4 + 255) / 256)), dim3(256), 0, s, x,
                     (int)n4, H, W, C4, Ho, Wo, fast_div(C4), fast_div(Wo), fast_div(Ho), y, arg);
}

void launch_maxpool_bwd(const float* dy, const uint8_t* arg, int B, int H, int W, int C, float* dx,
                        hipStream_t s) {
  const int Ho = (H - 1) / 2 + 1, Wo = (W - 1) / 2 + 1, C4 = C / 4;
  const size_t n4 = (size_t)B * H * W * C4;
  hipLaunchKernelGGL(maxpool_bwd_kernel, dim3((int)std::min<size_t>(8192, (n4 + 255) / 256)), dim3(256), 0, s, dy,
                     arg, (int)n4, H, W, C4, Ho, Wo, fast_div(C4), fast_div(W), fast_div(H), dx);
}

// ------------------------------------------------------------ frame prep
// x0[f][h][w][c] = mean of the 2x2 block (or the pixel) of frame src[f]
// (obs + src[f]*C*Hin*Win, NCHW, float32 or bfloat16).
template <typename T>
__global__ void __launch_bounds__(256) prep_kernel(const T* __restrict__ obs,
                                                   const int32_t* __restrict__ src, int F, int C,
                                                   int Hin, int Win, int pool, float* __restrict__ x0) {
  const int Ho = pool ? Hin / 2 : Hin, Wo = pool ? Win / 2 : Win;
  const size_t n = (size_t)F * Ho * Wo * C;
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256) {
    const int c = (int)(e % C);
    size_t r = e / C;
    const int w = (int)(r % Wo);
    r /= Wo;
    const int h = (int)(r % Ho);
    const int f = (int)(r / Ho);
    const size_t fr = src ? (size_t)src[f] : (size_t)f;
    const T* p = obs + (fr * C + c) * Hin * Win;
    float v;
    if (pool) {
      const T* q = p + (size_t)(2 * h) * Win + 2 * w;
      v = 0.25f * ((ldf(q) + ldf(q + 1)) + (ldf(q + Win) + ldf(q + Win + 1)));
    } else {
      v = ldf(p + (size_t)h * Win + w);
    }
    x0[e] = v;
  }
}

// The same for 4-channel frames with the pool: a thread makes one output pixel
// (16 bytes) from one 2-pixel load per channel and row; pairs aligned to
// their size.  256 frames of 256x256: 67.8 us with an element per thread, 38.9 us so.
// Other channel counts, unpooled frames and frames less aligned take prep_kernel.
DEV float2 ld_pair(const float* p) { return *(const float2*)p; }
DEV float2 ld_pair(const bf16_t* p) {
  const uint32_t u = *(const uint32_t*)p;
  return make_float2(__uint_as_float(u << 16), __uint_as_float(u & 0xffff0000u));
}
template <typename T>
__global__ void __launch_bounds__(256) prep4_kernel(const T* __restrict__ obs, const int32_t* __restrict__ src,
                                                    int n, int Hin, int Win, FastDiv dWo, FastDiv dHo,
                                                    float* __restrict__ x0) {
  const int Ho = Hin / 2, Wo = Win / 2;
  for (int e = blockIdx.x * 256 + threadIdx.x; e < n; e += gridDim.x * 256) {
    const int r = dWo.div(e), w = e - r * Wo, f = dHo.div(r), h = r - f * Ho;
    const size_t fr = src ? (size_t)src[f] : (size_t)f;
    const T* q = obs + (fr * 4 * Hin + 2 * h) * Win + 2 * w;
    float2 a[4], b[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      a[c] = ld_pair(q + (size_t)c * Hin * Win);
      b[c] = ld_pair(q + (size_t)c * Hin * Win + Win);
    }
    float v[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = 0.25f * ((a[c].x + a[c].y) + (b[c].x + b[c].y));
    ((float4*)x0)[e] = make_float4(v[0], v[1], v[2], v[3]);
  }
}

void launch_prep(const void* obs, int bf16, const int32_t* src, int F, int C, int Hin, int Win,
                 int pool, float* x0, hipStream_t s) {
  const int Ho = pool ? Hin / 2 : Hin, Wo = pool ? Win / 2 : Win;
  const size_t n = (size_t)F * Ho * Wo * C;
  if (pool && C == 4 && Win % 2 == 0 && ((uintptr_t)obs & (bf16 ? 3 : 7)) == 0 &&
      n / 4 <= (1u << 31) - 256 * 8192) {  // pixel index plus one step of the grid in 32 bits
    const int np = (int)(n / 4), nb = (int)std::min<size_t>(8192, ((size_t)np + 255) / 256);
    if (bf16)
      hipLaunchKernelGGL(prep4_kernel<bf16_t>, dim3(nb), dim3(256), 0, s, (const bf16_t*)obs, src, np, Hin, Win,
                         fast_div(Wo), fast_div(Ho), x0);
    else
      hipLaunchKernelGGL(prep4_kernel<float>, dim3(nb), dim3(256), 0, s, (const float*)obs, src, np, Hin, Win,
                         fast_div(Wo), fast_div(Ho), x0);
    return;
  }
  const int nb = (int)std::min<size_t>(8192, (n + 255) / 256);
  if (bf16)
    hipLaunchKernelGGL(prep_kernel<bf16_t>, dim3(nb), dim3(256), 0, s, (const bf16_t*)obs, src, F, C,
                       Hin, Win, pool, x0);
  else
    hipLaunchKernelGGL(prep_kernel<float>, dim3(nb), dim3(256), 0, s, (const float*)obs, src, F, C, Hin,
                       Win, pool, x0);
}

// dx = dy * [y > 0]
__global__ void __launch_bounds__(256) relu_grad_kernel(const float* __restrict__ dy,
                                                        const float* __restrict__ y, size_t n,
                                                        float* __restrict__ dx) {
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256)
    dx[e] = y[e] > 0.f ? dy[e] : 0.f;
}

void launch_relu_grad(const float* dy, const float* y, size_t n, float* dx, hipStream_t s) {
  const int nb = (int)std::min<size_t>(8192, (n + 255) / 256);
  hipLaunchKernelGGL(relu_grad_kernel, dim3(nb), dim3(256), 0, s, dy, y, n, dx);
}

// ------------------------------------------------------ fused GroupNorm
// One workgroup per (image b, group g) holds the group's P*Cg values in
// registers (NPT per thread, element e = p*Cg + cc, so a thread keeps one
// channel when 256 % Cg == 0): exact two-pass mean / variance, then the
// apply.  The input is the convolution output, or the sum of its split-K
// partial tiles (src + z*zstride), in which case the summed output can also
// be stored (u_out) for the backward.
// Two block sums in one reduction.
template <int NT>
DEV float2 block_sum2(float v0, float v1, float2* red) {
  const float d0 = wave_sum(v0), d1 = wave_sum(v1);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = make_float2(d0, d1);
  __syncthreads();
  float2 t = make_float2(0.f, 0.f);
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) {
    t.x += red[i].x;
    t.y += red[i].y;
  }
  return t;
}

template <int NT = 256>
DEV float block_sum(float v, float* red) {
  const float d = wave_sum(v);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = d;
  __syncthreads();
  float t = 0.f;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) t += red[i];
  return t;
}

template <int NPT, int NT, bool DUAL>
__global__ void __launch_bounds__(NT) gn_fused_kernel(const float* __restrict__ src, int nsplit, size_t zstride,
                                                       float* __restrict__ u_out, int P, int C, int G, float eps,
                                                       const float* __restrict__ gamma,
                                                       const float* __restrict__ beta,
                                                       const float* __restrict__ res, int relu,
                                                       float* __restrict__ out, int out_chw,
                                                       float2* __restrict__ stats, int src_gm,
                                                       float* __restrict__ pool_out, int H, int W,
                                                       const float* __restrict__ src2, int nsplit2, int src2_gm,
                                                       const float* __restrict__ gamma2,
                                                       const float* __restrict__ beta2,
                                                       float2* __restrict__ stats2) {
  __shared__ float red[NT / 64];
  __shared__ float2 red2[DUAL ? NT / 64 : 1];
  extern __shared__ float s_slab[];  // pool_out: the normalised slab [p][cc] (P Cg floats)
  const int b = blockIdx.x / G, g = blockIdx.x - b * G;
  const int Cg = C / G, n = P * Cg;
  // element j of this thread: pixel p0 + j*pstep, channel c (NT % Cg == 0)
  const int cc = threadIdx.x % Cg, p0 = threadIdx.x / Cg, pstep = NT / Cg, c = g * Cg + cc;
  const size_t base = ((size_t)b * P + p0) * C + c, jstr = (size_t)pstep * C;
  // a group-major input holds this (b, g) slab contiguously, element (p, cc) at
  // p Cg + cc: this thread's element j at threadIdx.x + j NT (coalesced)
  const size_t sbase = src_gm ? (size_t)blockIdx.x * n + threadIdx.x : base;
  const size_t sjstr = src_gm ? (size_t)NT : jstr;
  // the split-K partials, ZB splits per round with every load of a round in
  // flight together (summed in split order: deterministic)
  constexpr int ZB = NPT >= 16 ? 1 : 16 / NPT;
  // the affine parameters and the residual are loaded up front, so their
  // latency overlaps the input loads and the reductions
  const float gm = gamma[c], be = beta[c];
  float rv[NPT];
#pragma unroll
  for (int j = 0; j < NPT; ++j) rv[j] = (res && p0 + j * pstep < P) ? res[base + j * jstr] : 0.f;
  float x[NPT];
#pragma unroll
  for (int j = 0; j < NPT; ++j) x[j] = 0.f;
  for (int z0 = 0; z0 < nsplit; z0 += ZB) {
    float y[ZB][NPT];
#pragma unroll
    for (int q = 0; q < ZB; ++q)
#pragma unroll
      for (int j = 0; j < NPT; ++j)
        y[q][j] = (z0 + q < nsplit && p0 + j * pstep < P) ? src[(size_t)(z0 + q) * zstride + sbase + j * sjstr] : 0.f;
#pragma unroll
    for (int q = 0; q < ZB; ++q)
#pragma unroll
      for (int j = 0; j < NPT; ++j) x[j] += y[q][j];
  }
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < NPT; ++j) {
    if (u_out && p0 + j * pstep < P) u_out[base + j * jstr] = x[j];
    s += x[j];
  }
  float mean, var;
  if constexpr (DUAL) {
    // a second GroupNorm of the same shape (a projection shortcut) whose
    // output is this one's residual: its partials summed, its statistics and
    // apply taken with the same per-thread sums and reductions as a launch of
    // its own, so the residual is that launch's output bit for bit
    const size_t sbase2 = src2_gm ? (size_t)blockIdx.x * n + threadIdx.x : base;
    const size_t sjstr2 = src2_gm ? (size_t)NT : jstr;
    float x2[NPT];
#pragma unroll
    for (int j = 0; j < NPT; ++j) x2[j] = 0.f;
    for (int z0 = 0; z0 < nsplit2; z0 += ZB) {
      float y[ZB][NPT];
#pragma unroll
      for (int q = 0; q < ZB; ++q)
#pragma unroll
        for (int j = 0; j < NPT; ++j)
          y[q][j] = (z0 + q < nsplit2 && p0 + j * pstep < P) ? src2[(size_t)(z0 + q) * zstride + sbase2 + j * sjstr2]
                                                               : 0.f;
#pragma unroll
      for (int q = 0; q < ZB; ++q)
#pragma unroll
        for (int j = 0; j < NPT; ++j) x2[j] += y[q][j];
    }
    float s2 = 0.f;
#pragma unroll
    for (int j = 0; j < NPT; ++j) s2 += x2[j];
    const float2 m12 = block_sum2<NT>(s, s2, red2);
    const float mean1 = m12.x / n, mean2 = m12.y / n;
    float q1 = 0.f, q2 = 0.f;
#pragma unroll
    for (int j = 0; j < NPT; ++j)
      if (p0 + j * pstep < P) {
        q1 += (x[j] - mean1) * (x[j] - mean1);
        q2 += (x2[j] - mean2) * (x2[j] - mean2);
      }
    const float2 v12 = block_sum2<NT>(q1, q2, red2);
    const float rstd2 = 1.0f / sqrtf(v12.y / n + eps);
    const float2 st2 = make_float2(mean2, rstd2);
    if (threadIdx.x == 0) stats2[blockIdx.x] = st2;
    const float gamma2c = gamma2[c], be2 = beta2[c];
#pragma unroll
    for (int j = 0; j < NPT; ++j) rv[j] = gn_value_fused(x2[j], st2, gamma2c, be2) + 0.f;
    mean = mean1;       // this GroupNorm's statistics from the same sums as a launch of its own
    var = v12.x / n;
  } else {
    mean = block_sum<NT>(s, red) / n;
    float q = 0.f;
#pragma unroll
    for (int j = 0; j < NPT; ++j)
      if (p0 + j * pstep < P) q += (x[j] - mean) * (x[j] - mean);
    var = block_sum<NT>(q, red) / n;
  }
  const float rstd = 1.0f / sqrtf(var + eps);
  const float2 st = make_float2(mean, rstd);
  if (threadIdx.x == 0) stats[blockIdx.x] = st;
#pragma unroll
  for (int j = 0; j < NPT; ++j) {
    const int p = p0 + j * pstep;
    if (p < P) {
      const size_t idx = base + j * jstr;
      float o = gn_value_fused(x[j], st, gm, be) + rv[j];
      if (relu) o = fmaxf(o, 0.f);
      if (pool_out)
        s_slab[p * Cg + cc] = o;
      else
        out[out_chw ? ((size_t)b * C + c) * P + p : idx] = o;
    }
  }
  if (pool_out) {
    // 3x3 / 2 max pool (pad 1) of this group's channels from LDS; the plain
    // output is not written.  The window maximum over the in-bounds taps is
    // the same value max_pool's first maximum takes.
    __syncthreads();
    const int Ho = (H - 1) / 2 + 1, Wo = (W - 1) / 2 + 1, no = Ho * Wo * Cg;
    for (int e = threadIdx.x; e < no; e += NT) {
      const int c2 = e % Cg, q = e / Cg, wo = q % Wo, ho = q / Wo;
      float best = -INFINITY;
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const int hi = 2 * ho - 1 + t / 3, wi = 2 * wo - 1 + t % 3;
        if (hi >= 0 && hi < H && wi >= 0 && wi < W) {
          const float v = s_slab[(hi * W + wi) * Cg + c2];
          if (v > best) best = v;
        }
      }
      pool_out[(((size_t)b * Ho + ho) * Wo + wo) * C + g * Cg + c2] = best;
    }
  }
}

// Backward per (b, g): dz = dout [* (out > 0)], xhat = (y - mean) rstd;
// dy = rstd (dz gamma - mean(dz gamma) - xhat mean(dz gamma xhat)), dres = dz;
// bpart[b*C + c] = {sum_p dz, sum_p dz xhat} for the dgamma / dbeta reduction.
template <int NPT, int NT>
__global__ void __launch_bounds__(NT) gnb_fused_kernel(const float* __restrict__ dout,
                                                        const float* __restrict__ outm, int chw,
                                                        const float* __restrict__ y, int P, int C, int G,
                                                        const float2* __restrict__ stats,
                                                        const float* __restrict__ gamma, float* __restrict__ dy,
                                                        float* __restrict__ dres, float2* __restrict__ bpart) {
  __shared__ float2 red2[NT / 64];
  __shared__ float2 cred[NT];
  const int b = blockIdx.x / G, g = blockIdx.x - b * G;
  const int Cg = C / G, n = P * Cg;
  const float2 st = stats[blockIdx.x];
  const int cc = threadIdx.x % Cg, p0 = threadIdx.x / Cg, pstep = NT / Cg, c = g * Cg + cc;
  const size_t base = ((size_t)b * P + p0) * C + c, jstr = (size_t)pstep * C;
  const float gm = gamma[c];
  float dz[NPT], xh[NPT];
#pragma unroll
  for (int j = 0; j < NPT; ++j) {
    const int p = p0 + j * pstep;
    float zv = 0.f, om = 1.f, yv = st.x;
    if (p < P) {
      const size_t io = chw ? ((size_t)b * C + c) * P + p : base + j * jstr;
      zv = dout[io];
      if (outm) om = outm[io];
      yv = y[base + j * jstr];
    }
    dz[j] = om > 0.f ? zv : 0.f;
    xh[j] = (yv - st.x) * st.y;
  }
  float s1 = 0.f, s2 = 0.f, cz = 0.f, czx = 0.f;
#pragma unroll
  for (int j = 0; j < NPT; ++j) {
    s1 += dz[j] * gm;
    s2 += dz[j] * gm * xh[j];
    cz += dz[j];
    czx += dz[j] * xh[j];
  }
  const float2 sm = block_sum2<NT>(s1, s2, red2);
  const float m1 = sm.x / n, m2 = sm.y / n;
#pragma unroll
  for (int j = 0; j < NPT; ++j) {
    if (p0 + j * pstep < P) {
      const size_t idx = base + j * jstr;
      dy[idx] = st.y * (dz[j] * gm - m1 - xh[j] * m2);
      if (dres) dres[idx] = dz[j];
    }
  }
  cred[threadIdx.x] = make_float2(cz, czx);
  __syncthreads();
  if (threadIdx.x < Cg) {
    float a = 0.f, q = 0.f;
    for (int t = threadIdx.x; t < NT; t += Cg) {
      a += cred[t].x;
      q += cred[t].y;
    }
    bpart[(size_t)b * C + g * Cg + threadIdx.x] = make_float2(a, q);
  }
}

// Elements per thread (1..32) of the fused kernels, 0 when unsupported; the
// block has 256 threads up to 512 elements per (image, group), else 1024.
int gn_fused_npt(int P, int Cg) {
  const int n = P * Cg;
  if (256 % Cg) return 0;
  const int nt = n <= 256 * 2 ? 256 : 1024;
  for (int k = 1; k <= 32; k *= 2)
    if (n <= nt * k) return k;
  return 0;
}

#define GN_NPT_SWITCH(NT_, NPT_, CALL) \
  if (NT_ == 256) {                    \
    switch (NPT_) {                    \
      case 1: CALL(1, 256); break;     \
      case 2: CALL(2, 256); break;     \
      case 4: CALL(4, 256); break;     \
      default: CALL(8, 256); break;    \
    }                                  \
  } else {                             \
    switch (NPT_) {                    \
      case 1: CALL(1, 1024); break;    \
      case 2: CALL(2, 1024); break;    \
      case 4: CALL(4, 1024); break;    \
      case 8: CALL(8, 1024); break;    \
      case 16: CALL(16, 1024); break;  \
      default: CALL(32, 1024); break;  \
    }                                  \
  }

bool gn_pool_fits(int P, int Cg) { return (long)P * Cg * (long)sizeof(float) <= kGnPoolLds; }

void launch_gn_fused(const float* src, int nsplit, size_t zstride, float* u_out, int B, int P, int C, int G,
                     float eps, const float* gamma, const float* beta, const float* res, int relu, float* out,
                     int out_chw, float2* stats, hipStream_t s, int src_gm, float* pool_out, int H, int W,
                     const GnSecond* second) {
  const float* src2 = second ? second->src : nullptr;
  const int nsplit2 = second ? second->nsplit : 0, src2_gm = second ? second->src_gm : 0;
  const float* gamma2 = second ? second->gamma : nullptr;
  const float* beta2 = second ? second->beta : nullptr;
  float2* stats2 = second ? second->stats : nullptr;
  const int npt = gn_fused_npt(P, C / G), nt = (long)P * (C / G) <= 256 * 2 ? 256 : 1024;
  const size_t lds = pool_out ? (size_t)P * (C / G) * sizeof(float) : 0;
#define GN_CALL_D(K, T, D)                                                                                        \
  hipLaunchKernelGGL((gn_fused_kernel<K, T, D>), dim3(B * G), dim3(T), lds, s, src, nsplit, zstride, u_out, P, C, \
                     G, eps, gamma, beta, res, relu, out, out_chw, stats, src_gm, pool_out, H, W, src2, nsplit2,      \
                     src2_gm, gamma2, beta2, stats2)
#define GN_CALL(K, T) GN_CALL_D(K, T, false)
#define GN_CALL2(K, T) GN_CALL_D(K, T, true)
  if (second) {
    GN_NPT_SWITCH(nt, npt, GN_CALL2)
  } else {
    GN_NPT_SWITCH(nt, npt, GN_CALL)
  }
#undef GN_CALL
#undef GN_CALL2
#undef GN_CALL_D
}

void launch_gnb_fused(const float* dout, const float* outm, int chw, const float* y, int B, int P, int C, int G,
                      const float2* stats, const float* gamma, float* dy, float* dres, float* dgamma,
                      float* dbeta, float2* bpart, hipStream_t s) {
  const int npt = gn_fused_npt(P, C / G), nt = (long)P * (C / G) <= 256 * 2 ? 256 : 1024;
#define GNB_CALL(K, T)                                                                                       \
  hipLaunchKernelGGL((gnb_fused_kernel<K, T>), dim3(B * G), dim3(T), 0, s, dout, outm, chw, y, P, C, G, stats, \
                     gamma, dy, dres, bpart)
  GN_NPT_SWITCH(nt, npt, GNB_CALL)
#undef GNB_CALL
  hipLaunchKernelGGL(gnb_affine_kernel, dim3(cdiv(C, 4)), dim3(256), 0, s, bpart, B, 1, C, dgamma, dbeta);
}

// SE-ResNeXt blocks (App. "Agent Design", visual encoder; Xie et al.'s
// aggregated transform, Hu et al.'s squeeze-excite gate), NHWC float32
// activations:
//
//   grouped 3x3 convolution  input and output channels in G equal slices,
//                            output slice g convolves input slice g with its
//                            own filters [Co][3][3][C/G].  Its FLOPs are 1/G of
//                            a dense 3x3 and its per-group products (K = 9C/G,
//                            N = Co/G, as small as 36 x 4) would leave most of
//                            a matrix-core tile empty, so it is a direct
//                            vector-ALU convolution, bound by its multiply-adds
//                            and the LDS and L1 reads that feed them: one workgroup
//                            per (pixel tile, one to four neighbouring groups) with
//                            their filters staged in LDS.  Groups of 4, 8, 16 or 32
//                            channels on both sides run register-tiled kernels
//                            (several outputs a thread), others a general form
//                            with one output a thread.
//   squeeze-excite           z = per-channel pixel mean of the branch y,
//                            s = sigmoid(W2 relu(W1 z + b1) + b2), then
//                            out = relu(s * y + shortcut); the FCs are tiny
//                            (C x C/16 per frame) and run in float32 FMAs,
//                            spread over (frame, unit tile) workgroups.
//
// Precision: with bfloat16 weights every product operand of the convolution
// is rounded to bfloat16 (activation at load, weight as stored), as the
// matrix-core path does; gradients multiply the incoming float32 gradient
// with the rounded operand.  All reductions run in a fixed order
// (deterministic).
#include "common.h"
#include "kernels.h"

namespace {

constexpr int kThreads = 256;

// nearest bfloat16 value (ties to even) by the hardware conversion
typedef __bf16 se_bf16x2 __attribute__((ext_vector_type(2)));
typedef float se_f32x2 __attribute__((ext_vector_type(2)));
DEV float rnd_bf16(float x) {
  const se_bf16x2 r = __builtin_convertvector((se_f32x2){x, 0.f}, se_bf16x2);
  return __uint_as_float(__builtin_bit_cast(uint32_t, r) << 16);
}

// A group's filters [og][9cg] (contiguous in w) into LDS as dst[perm(co, k)],
// with every thread's loads issued before its stores.
template <typename TW, typename Perm>
DEV void stage_filters(const TW* __restrict__ w, int n, float* dst, Perm perm) {
  constexpr int kU = 8;
  for (int e0 = threadIdx.x; e0 < n; e0 += kU * 256) {
    float v[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int e = e0 + u * 256;
      v[u] = ldf(w + min(e, n - 1));
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int e = e0 + u * 256;
      if (e < n) dst[perm(e)] = v[u];
    }
  }
}

template <bool BF>
DEV float opnd(float x) {
  return BF ? rnd_bf16(x) : x;
}

DEV void ld4(const float* p, float* v) {
  const float4 t = *(const float4*)p;
  v[0] = t.x;
  v[1] = t.y;
  v[2] = t.z;
  v[3] = t.w;
}

// Index sizes are checked on the host to fit in 31 bits; quotients by
// runtime sizes use precomputed multiply-shift divisors.
struct PixDiv {
  FastDiv plane, row;  // pixels per image, pixels per row (of the indexed map)
};

// ---------------------------------------------------------------- forward
// Workgroup: `pix` consecutive output pixels of one group; thread t owns
// output channel t % og of pixel rows t / og + k (256 / og).  An
// out-of-range tap reads the image origin and is zeroed.  General form: any
// group width; see gconv_tile_kernel.
template <typename TW>
__global__ void __launch_bounds__(kThreads) gconv_fwd_kernel(const float* __restrict__ x, const TW* __restrict__ w,
                                                            float* __restrict__ y, ConvGeo g, int G, int pix,
                                                            PixDiv dv) {
  extern __shared__ float ws[];  // [9][cg][og]
  constexpr bool BF = sizeof(TW) == 2;
  const int cg = g.C / G, og = g.Co / G, grp = blockIdx.y;
  const int kw9 = 9 * cg;
  stage_filters(w + (size_t)grp * og * kw9, og * kw9, ws, [=](int e) {
    const int co = e / kw9, k = e - co * kw9;                 // w[grp*og + co][k] -> ws[k][co]
    return k * og + co;
  });
  __syncthreads();
  const int rows = kThreads / og, co = threadIdx.x % og, r0 = threadIdx.x / og;
  if (r0 >= rows) return;
  const int plane = g.Ho * g.Wo, P = g.B * plane;
  const int p0 = blockIdx.x * pix, pend = min(P, p0 + pix);
  for (int p = p0 + r0; p < pend; p += rows) {
    const int b = dv.plane.div(p), q = p - b * plane;
    const int ho = dv.row.div(q), wo = q - ho * g.Wo;
    const float* xb = x + (size_t)b * g.H * g.W * g.C + grp * cg;
    float acc = 0.f;
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      const int hi = ho * g.stride - g.pad + tap / 3, wi = wo * g.stride - g.pad + tap % 3;
      const bool ok = (unsigned)hi < (unsigned)g.H && (unsigned)wi < (unsigned)g.W;
      const float* xp = xb + (ok ? ((size_t)hi * g.W + wi) * g.C : 0);
      const float* wp = ws + tap * cg * og + co;
      for (int c4 = 0; c4 < cg; c4 += 4) {
        float v[4];
        ld4(xp + c4, v);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = fmaf(ok ? opnd<BF>(v[e]) : 0.f, wp[(c4 + e) * og], acc);
      }
    }
    y[(size_t)p * g.Co + grp * og + co] = acc;
  }
}

// ----------------------------------------------------------- data gradient
// dx[b][hi][wi][grp*cg + ci] = sum over taps (kh, kw) whose output pixel
// ho = (hi + pad - kh) / stride is whole and in range, and over the group's
// output channels co, of dy[b][ho][wo][grp*og + co] * w[grp*og + co][kh][kw][ci].
// Stride 1 or 2.  General form.
template <typename TW>
__global__ void __launch_bounds__(kThreads) gconv_dgrad_kernel(const float* __restrict__ dy,
                                                              const TW* __restrict__ w, float* __restrict__ dx,
                                                              ConvGeo g, int G, int pix, PixDiv dv,
                                                              int accumulate) {
  extern __shared__ float ws[];  // [9][og][cg]
  const int cg = g.C / G, og = g.Co / G, grp = blockIdx.y;
  const int kw9 = 9 * cg;
  stage_filters(w + (size_t)grp * og * kw9, og * kw9, ws, [=](int e) {
    const int co = e / kw9, k = e - co * kw9, tap = k / cg, ci = k - tap * cg;
    return (tap * og + co) * cg + ci;                         // -> ws[tap][co][ci]
  });
  __syncthreads();
  const int rows = kThreads / cg, ci = threadIdx.x % cg, r0 = threadIdx.x / cg;
  if (r0 >= rows) return;
  const int plane = g.H * g.W, P = g.B * plane;
  const int sh = g.stride == 2 ? 1 : 0;
  const int p0 = blockIdx.x * pix, pend = min(P, p0 + pix);
  for (int p = p0 + r0; p < pend; p += rows) {
    const int b = dv.plane.div(p), q = p - b * plane;
    const int hi = dv.row.div(q), wi = q - hi * g.W;
    const float* db = dy + (size_t)b * g.Ho * g.Wo * g.Co + grp * og;
    float acc = 0.f;
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      const int th = hi + g.pad - tap / 3, tw = wi + g.pad - tap % 3;
      const int ho = th >> sh, wo = tw >> sh;
      const bool ok = th >= 0 && tw >= 0 && ((th | tw) & sh) == 0 && ho < g.Ho && wo < g.Wo;
      const float* dp = db + (ok ? ((size_t)ho * g.Wo + wo) * g.Co : 0);
      const float* wp = ws + tap * og * cg + ci;
      for (int c4 = 0; c4 < og; c4 += 4) {
        float v[4];
        ld4(dp + c4, v);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = fmaf(ok ? v[e] : 0.f, wp[(c4 + e) * cg], acc);
      }
    }
    float* o = dx + (size_t)p * g.C + grp * cg + ci;
    *o = accumulate ? *o + acc : acc;
  }
}

// --------------------------------------------------------- weight gradient
// Partial dw of one group over one chunk of output pixels:
//   part[chunk][(grp*og + co) * 9cg + k] = sum_{p in chunk} dy[p][grp*og + co] * xcol[p][k],
// xcol[p][(kh*3 + kw)*cg + ci] the (rounded) input under tap (kh, kw).
// Pixels are staged PT at a time in LDS (the group's dy columns, and its
// im2col rows copied as float4); thread t owns outputs t, t + 256, ... (at
// most kEPT).
constexpr int kEPT = 36;   // og * 9cg <= 256 * 36 (group widths up to 32)
constexpr int kLdsFloats = 10240;

struct WgradDiv {
  PixDiv pix;          // output map
  FastDiv og, k9c4, cg4;  // og; 9cg/4 float4 per im2col row; cg/4 float4 per tap
};

template <bool BF>
__global__ void __launch_bounds__(kThreads) gconv_wgrad_kernel(const float* __restrict__ x,
                                                              const float* __restrict__ dy,
                                                              float* __restrict__ part, ConvGeo g, int G, int pix,
                                                              int PT, WgradDiv dv) {
  extern __shared__ float sm[];  // dys [PT][og], xs [PT][9cg], coordinates [PT][3]
  const int cg = g.C / G, og = g.Co / G, grp = blockIdx.y;
  const int kw9 = 9 * cg, ne = og * kw9, k9c4 = kw9 / 4, cg4 = cg / 4;
  float* xs = sm;                      // 16-byte aligned: PT * 9cg floats
  float* dys = sm + PT * kw9;
  int* pc = (int*)(dys + PT * og);
  float acc[kEPT];
#pragma unroll
  for (int j = 0; j < kEPT; ++j) acc[j] = 0.f;
  const int plane = g.Ho * g.Wo, P = g.B * plane;
  const int p0 = blockIdx.x * pix, pend = min(P, p0 + pix);
  for (int pt = p0; pt < pend; pt += PT) {
    const int np = min(PT, pend - pt);
    __syncthreads();
    for (int i = threadIdx.x; i < PT; i += kThreads) {
      int b = -1, ho = 0, wo = 0;
      if (i < np) {
        const int p = pt + i;
        b = dv.pix.plane.div(p);
        const int q = p - b * plane;
        ho = dv.pix.row.div(q);
        wo = q - ho * g.Wo;
      }
      pc[3 * i] = b;
      pc[3 * i + 1] = ho * g.stride - g.pad;
      pc[3 * i + 2] = wo * g.stride - g.pad;
    }
    for (int e = threadIdx.x; e < PT * og; e += kThreads) {
      const int i = dv.og.div(e), co = e - i * og;
      dys[e] = i < np ? dy[(size_t)(pt + i) * g.Co + grp * og + co] : 0.f;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < PT * k9c4; e += kThreads) {
      const int i = dv.k9c4.div(e), r = e - i * k9c4;
      const int tap = dv.cg4.div(r), c4 = r - tap * cg4;
      const int b = pc[3 * i], hi = pc[3 * i + 1] + tap / 3, wi = pc[3 * i + 2] + tap % 3;
      const bool ok = b >= 0 && (unsigned)hi < (unsigned)g.H && (unsigned)wi < (unsigned)g.W;
      float v[4] = {0.f, 0.f, 0.f, 0.f};
      if (ok) {
        ld4(x + (((size_t)b * g.H + hi) * g.W + wi) * g.C + grp * cg + 4 * c4, v);
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = opnd<BF>(v[q]);
      }
      *(float4*)(xs + i * kw9 + tap * cg + 4 * c4) = make_float4(v[0], v[1], v[2], v[3]);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kEPT; ++j) {
      const int e = threadIdx.x + j * kThreads;
      if (e < ne) {
        const int co = e / kw9, k = e - co * kw9;
        float a = acc[j];
        for (int i = 0; i < np; ++i) a = fmaf(dys[i * og + co], xs[i * kw9 + k], a);
        acc[j] = a;
      }
    }
  }
  float* out = part + (size_t)blockIdx.x * g.Co * kw9 + (size_t)grp * ne;
#pragma unroll
  for (int j = 0; j < kEPT; ++j) {
    const int e = threadIdx.x + j * kThreads;
    if (e < ne) out[e] = acc[j];
  }
}

// ------------------------------------------------- register-tiled kernels
// The same sums for groups of CG input and CG output channels (CG 4, 8, 16 or
// 32): every output is the same chain of FMAs as above, only dealt to the
// threads otherwise.  The kernels above read LDS (and L1) once or twice an FMA,
// which bounds them; these read a float4 for 4 to 8 FMAs.
//
// Forward and data gradient (BWD; source dy, filters transposed).  Workgroup:
// `pix` pixels of gpw neighbouring groups (64 contiguous bytes a pixel, 128 at CG
// 32; 16 or 32 at CG 4 and 8 where the group count has no such factor);
// a thread makes 4 channels of NP pixels (2, or 1 where that would leave the
// chip idle).  Filters in LDS as ws[group][tap][source channel][channel], 16
// floats of padding a group against conflicts between groups.  128 frames of
// the paper's net, bfloat16, widths 4 / 8 / 16 / 32, in us: forward 95 / 85 /
// 155 / 290 -> 53 / 37 / 22 / 34, data gradient 55 / 45 / 81 / 206 -> 28 / 22 /
// 21 / 26, at stride 2 151 / 228 / 552 (8 / 16 / 32) -> 54 / 44 / 52.
template <typename TW, int CG, bool BWD, int NP>
__global__ void __launch_bounds__(kThreads) gconv_tile_kernel(const float* __restrict__ src,
                                                             const TW* __restrict__ w, float* __restrict__ dst,
                                                             ConvGeo g, int gpw, int pix, PixDiv dv,
                                                             int accumulate) {
  extern __shared__ float ws[];
  constexpr bool RND = !BWD && sizeof(TW) == 2;
  constexpr int QL = CG / 4, K9 = 9 * CG, NE = CG * K9, GS = NE + 16, UN = CG <= 8 ? 3 : 1;
  const int grp0 = blockIdx.y * gpw;
  stage_filters(w + (size_t)grp0 * NE, gpw * NE, ws, [=](int e) {
    const int gi = e / NE, q = e - gi * NE, co = q / K9, k = q - co * K9, tap = k / CG, ci = k - tap * CG;
    return gi * GS + (BWD ? (tap * CG + co) * CG + ci : k * CG + co);
  });
  __syncthreads();
  const int nl = gpw * QL, rows = kThreads / nl, l = threadIdx.x % nl, r0 = threadIdx.x / nl;
  const int gi = l / QL, c4 = l % QL * 4;
  const float* wg = ws + gi * GS + c4;
  const int Hd = BWD ? g.H : g.Ho, Wd = BWD ? g.W : g.Wo, Cd = BWD ? g.C : g.Co;
  const int Hs = BWD ? g.Ho : g.H, Ws = BWD ? g.Wo : g.W, Cs = BWD ? g.Co : g.C;
  const int sh = g.stride == 2 ? 1 : 0;
  const int p0 = blockIdx.x * pix, pend = min(g.B * Hd * Wd, p0 + pix);
  for (int p = p0 + r0; p < pend; p += NP * rows) {
    int pp[NP], h0[NP], w0[NP];
    const float* sb[NP];
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      pp[u] = min(p + u * rows, pend - 1);  // past the end: the last pixel again, not stored
      const int b = dv.plane.div(pp[u]), q = pp[u] - b * Hd * Wd, h = dv.row.div(q);
      sb[u] = src + (size_t)b * Hs * Ws * Cs + (grp0 + gi) * CG;
      h0[u] = BWD ? h + g.pad : h * g.stride - g.pad;
      w0[u] = BWD ? q - h * Wd + g.pad : (q - h * Wd) * g.stride - g.pad;
    }
    float acc[NP][4];
#pragma unroll
    for (int u = 0; u < NP; ++u) acc[u][0] = acc[u][1] = acc[u][2] = acc[u][3] = 0.f;
#pragma unroll UN
    for (int tap = 0; tap < 9; ++tap) {
      const int kh = tap / 3, kw = tap - 3 * kh;
      float v[NP][CG];
#pragma unroll
      for (int u = 0; u < NP; ++u) {
        int hs, wsx;
        bool ok;
        if (BWD) {
          const int th = h0[u] - kh, tw = w0[u] - kw;
          hs = th >> sh;
          wsx = tw >> sh;
          ok = th >= 0 && tw >= 0 && ((th | tw) & sh) == 0 && hs < Hs && wsx < Ws;
        } else {
          hs = h0[u] + kh;
          wsx = w0[u] + kw;
          ok = (unsigned)hs < (unsigned)Hs && (unsigned)wsx < (unsigned)Ws;
        }
        const float* q = sb[u] + (ok ? ((size_t)hs * Ws + wsx) * Cs : 0);  // outside: the origin, zeroed
#pragma unroll
        for (int c = 0; c < CG; c += 4) ld4(q + c, v[u] + c);
#pragma unroll
        for (int c = 0; c < CG; ++c) v[u][c] = ok ? opnd<RND>(v[u][c]) : 0.f;
      }
      const float* wp = wg + tap * CG * CG;
#pragma unroll
      for (int c = 0; c < CG; ++c) {
        float f[4];
        ld4(wp + c * CG, f);
#pragma unroll
        for (int u = 0; u < NP; ++u)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[u][j] = fmaf(v[u][c], f[j], acc[u][j]);
      }
    }
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      if (p + u * rows >= pend) break;
      float4* o = (float4*)(dst + (size_t)pp[u] * Cd + (grp0 + gi) * CG + c4);
      float4 r = make_float4(acc[u][0], acc[u][1], acc[u][2], acc[u][3]);
      if (accumulate) {
        const float4 t = *o;
        r = make_float4(t.x + r.x, t.y + r.y, t.z + r.z, t.w + r.w);
      }
      *o = r;
    }
  }
}

// Weight gradient of GPW groups over one chunk of output pixels: a thread owns
// CO x 4 elements (unit (group, co block, k quad)), PT pixels staged at a time;
// the next PT are loaded into registers while these are summed.  GPW, CO and T
// are sized to fill most of the threads with units and to keep the staged
// pixels within 40 KB of LDS; the wider the group, the fewer the chunks, so
// a width of 32 has 9 wavefronts a workgroup.  128 frames, bfloat16, widths 4 /
// 8 / 16 / 32, in us: 208 / 128 / 82 / 202 -> 65 / 40 / 31 / 29.
template <int CG> struct WgradTile;
template <> struct WgradTile<4> { static constexpr int GPW = 4, CO = 2, T = 128, PT = 32; };
template <> struct WgradTile<8> { static constexpr int GPW = 4, CO = 4, T = 192, PT = 32; };
template <> struct WgradTile<16> { static constexpr int GPW = 1, CO = 4, T = 192, PT = 64; };
template <> struct WgradTile<32> { static constexpr int GPW = 1, CO = 4, T = 576, PT = 32; };

template <bool BF, int CG>
__global__ void __launch_bounds__(WgradTile<CG>::T) gconv_wgrad_tile_kernel(const float* __restrict__ x,
                                                                           const float* __restrict__ dy,
                                                                           float* __restrict__ part, ConvGeo g,
                                                                           int pix, PixDiv dv) {
  using W = WgradTile<CG>;
  constexpr int GPW = W::GPW, CO = W::CO, T = W::T, PT = W::PT, QL = CG / 4, K9 = 9 * CG, NE = CG * K9;
  constexpr int XR = GPW * K9, DR = GPW * CG;                  // floats of a pixel's x and dy rows
  constexpr int NX = PT * XR / 4, ND = PT * DR / 4;            // float4 of a round
  constexpr int LX = NX / T, LD = (ND + T - 1) / T;
  constexpr int UG = CG / CO * (K9 / 4), U = GPW * UG;         // units
  static_assert(NX % T == 0 && U <= T, "round");
  __shared__ __attribute__((aligned(16))) float xs[PT * XR];   // [pixel][group][tap][ci]
  __shared__ __attribute__((aligned(16))) float ds[PT * DR];   // [pixel][group][co]
  const int tid = threadIdx.x, grp0 = blockIdx.y * GPW, plane = g.Ho * g.Wo;
  const int p0 = blockIdx.x * pix, pend = min(g.B * plane, p0 + pix);
  float4 vx[LX], vd[LD];
  auto gload = [&](int pt) {
#pragma unroll
    for (int n = 0; n < LX; ++n) {
      const int e = tid + n * T, i = e / (XR / 4), r = e % (XR / 4), tap = r / (GPW * QL), cq = r % (GPW * QL);
      const int p = pt + i;
      vx[n] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (p < pend) {
        const int b = dv.plane.div(p), q = p - b * plane, ho = dv.row.div(q), wo = q - ho * g.Wo;
        const int hi = ho * g.stride - g.pad + tap / 3, wi = wo * g.stride - g.pad + tap % 3;
        if ((unsigned)hi < (unsigned)g.H && (unsigned)wi < (unsigned)g.W)
          vx[n] = *(const float4*)(x + (((size_t)b * g.H + hi) * g.W + wi) * g.C + grp0 * CG + 4 * cq);
      }
    }
#pragma unroll
    for (int n = 0; n < LD; ++n) {
      const int e = tid + n * T, i = e / (DR / 4), cq = e % (DR / 4), p = pt + i;
      vd[n] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (e < ND && p < pend) vd[n] = *(const float4*)(dy + (size_t)p * g.Co + grp0 * CG + 4 * cq);
    }
  };
  const int gi = tid / UG, uc = tid % UG / (K9 / 4) * CO, uk = tid % (K9 / 4) * 4;
  float acc[CO][4];
#pragma unroll
  for (int c = 0; c < CO; ++c)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[c][j] = 0.f;
  gload(p0);
  for (int pt = p0; pt < pend; pt += PT) {
    __syncthreads();  // the last round's sums are done with the buffers
#pragma unroll
    for (int n = 0; n < LX; ++n) {
      const int e = tid + n * T, i = e / (XR / 4), r = e % (XR / 4), tap = r / (GPW * QL), cq = r % (GPW * QL);
      const float4 v = vx[n];
      *(float4*)(xs + i * XR + cq / QL * K9 + tap * CG + cq % QL * 4) =
          make_float4(opnd<BF>(v.x), opnd<BF>(v.y), opnd<BF>(v.z), opnd<BF>(v.w));
    }
#pragma unroll
    for (int n = 0; n < LD; ++n)
      if (tid + n * T < ND) *(float4*)(ds + 4 * (tid + n * T)) = vd[n];
    __syncthreads();
    if (pt + PT < pend) gload(pt + PT);
    if (tid < U) {
      const int np = min(PT, pend - pt);
#pragma unroll 4
      for (int i = 0; i < np; ++i) {
        float f[4], d[CO];
        ld4(xs + i * XR + gi * K9 + uk, f);
#pragma unroll
        for (int c = 0; c < CO; ++c) d[c] = ds[i * DR + gi * CG + uc + c];
#pragma unroll
        for (int c = 0; c < CO; ++c)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[c][j] = fmaf(d[c], f[j], acc[c][j]);
      }
    }
  }
  if (tid >= U) return;
  float* out = part + (size_t)blockIdx.x * g.Co * K9 + (size_t)(grp0 + gi) * NE + uk;
#pragma unroll
  for (int c = 0; c < CO; ++c)
    *(float4*)(out + (uc + c) * K9) = make_float4(acc[c][0], acc[c][1], acc[c][2], acc[c][3]);
}

// dst[i] = sum over chunks z (in order) of part[z][i]
__global__ void __launch_bounds__(kThreads) chunk_sum_kernel(const float* __restrict__ part, int chunks, int n,
                                                            float* __restrict__ dst) {
  for (int i = blockIdx.x * kThreads + threadIdx.x; i < n; i += gridDim.x * kThreads) {
    // 16 loads in flight, added in order
    float s = 0.f;
    int z = 0;
    for (; z + 16 <= chunks; z += 16) {
      float v[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) v[q] = part[(size_t)(z + q) * n + i];
#pragma unroll
      for (int q = 0; q < 16; ++q) s += v[q];
    }
    for (; z < chunks; ++z) s += part[(size_t)z * n + i];
    dst[i] = s;
  }
}

// ---------------------------------------------------------- squeeze-excite
// Per-channel sums over a slice of the pixels (grid F x ceil(C/64) x S;
// thread (lane, row): channel lane, pixels row, row + 4, ... of slice z):
// zpart[z][f][c] = sum_{p in slice z} y[f][p][c].  The slices' sums are
// added in order by the kernel that consumes them.
__global__ void __launch_bounds__(kThreads) se_squeeze_kernel(const float* __restrict__ y, int HW, int C, int F,
                                                             int slice, float* __restrict__ zpart) {
  __shared__ float red[4][64];
  const int lane = threadIdx.x & 63, row = threadIdx.x >> 6;
  const int f = blockIdx.x, c = blockIdx.y * 64 + lane, z = blockIdx.z;
  const int pend = min(HW, (z + 1) * slice);
  float s0 = 0.f, s1 = 0.f;
  if (c < C) {
    const float* yf = y + (size_t)f * HW * C + c;
    int p = z * slice + row;
    for (; p + 4 < pend; p += 8) {
      s0 += yf[(size_t)p * C];
      s1 += yf[(size_t)(p + 4) * C];
    }
    if (p < pend) s0 += yf[(size_t)p * C];
  }
  red[row][lane] = s0 + s1;
  __syncthreads();
  if (row == 0 && c < C)
    zpart[((size_t)z * F + f) * C + c] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
}

// Hidden layer of the gate, workgroup (f, y): z = (sum of the slices) / HW
// (workgroup y == 0 stores it), then a1 = W1 z + b1 for the 16 hidden units
// 16y .. 16y + 15, four per wavefront, each a lane-strided dot product over
// the channels with its loads unrolled.
__global__ void __launch_bounds__(kThreads) se_hidden_kernel(const float* __restrict__ zpart, int S, int F,
                                                            float inv_hw, int C, int R,
                                                            const float* __restrict__ w1,
                                                            const float* __restrict__ b1, float* __restrict__ z,
                                                            float* __restrict__ a1) {
  extern __shared__ float zs[];  // [C]
  const int f = blockIdx.x, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int c = threadIdx.x; c < C; c += kThreads) {
    float t = 0.f;
    for (int k = 0; k < S; ++k) t += zpart[((size_t)k * F + f) * C + c];
    t *= inv_hw;
    zs[c] = t;
    if (blockIdx.y == 0) z[(size_t)f * C + c] = t;
  }
  __syncthreads();
  const int jb = blockIdx.y * 16 + wv * 4;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  const float* wr[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) wr[q] = w1 + (size_t)min(jb + q, R - 1) * C;
  for (int c = lane; c < C; c += 64) {
    const float zv = zs[c];
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = fmaf(wr[q][c], zv, acc[q]);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float v = wave_sum(acc[q]);
    if (lane == 0 && jb + q < R) a1[(size_t)f * R + jb + q] = v + b1[jb + q];
  }
}

// Gate, workgroup (f, y): s = sigmoid(W2 relu(a1) + b2) for channels
// 64y .. 64y + 63, four wavefronts each summing a quarter of the hidden
// units, added in a fixed order.
__global__ void __launch_bounds__(kThreads) se_gate_kernel(const float* __restrict__ a1, int C, int R,
                                                          const float* __restrict__ w2,
                                                          const float* __restrict__ b2, float* __restrict__ s) {
  extern __shared__ float sm[];  // hs [R], red [4][64]
  float* hs = sm;
  float* red = sm + R;
  const int f = blockIdx.x, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int j = threadIdx.x; j < R; j += kThreads) hs[j] = fmaxf(a1[(size_t)f * R + j], 0.f);
  __syncthreads();
  const int c = blockIdx.y * 64 + lane;
  const int q = (R + 3) / 4, j0 = wv * q, j1 = min(R, j0 + q);
  float acc = 0.f;
  if (c < C) {
    const float* wr = w2 + (size_t)c * R;
#pragma unroll 8
    for (int j = j0; j < j1; ++j) acc = fmaf(wr[j], hs[j], acc);
  }
  red[wv * 64 + lane] = acc;
  __syncthreads();
  if (wv == 0 && c < C)
    s[(size_t)f * C + c] = sigm(b2[c] + ((red[lane] + red[64 + lane]) + (red[128 + lane] + red[192 + lane])));
}

// out = relu(s[f][c] * y + res), four channels per thread (C % 4 == 0)
__global__ void __launch_bounds__(kThreads) se_excite_kernel(const float* __restrict__ y,
                                                            const float* __restrict__ s,
                                                            const float* __restrict__ res, int n4, FastDiv dhwc4,
                                                            FastDiv dc4, int C4, float* __restrict__ out) {
  for (int i = blockIdx.x * kThreads + threadIdx.x; i < n4; i += gridDim.x * kThreads) {
    const int f = dhwc4.div(i), c4 = i - dc4.div(i) * C4;
    const float4 yv = ((const float4*)y)[i], rv = ((const float4*)res)[i];
    const float4 sv = ((const float4*)s)[f * C4 + c4];
    ((float4*)out)[i] = make_float4(fmaxf(fmaf(sv.x, yv.x, rv.x), 0.f), fmaxf(fmaf(sv.y, yv.y, rv.y), 0.f),
                                    fmaxf(fmaf(sv.z, yv.z, rv.z), 0.f), fmaxf(fmaf(sv.w, yv.w, rv.w), 0.f));
  }
}

// Backward, first pass (grid F x ceil(C/64) x S): dpre = dout * [out > 0]
// into dres (the shortcut's gradient) and dspart[z][f][c] = sum over slice z
// of dpre * y.
__global__ void __launch_bounds__(kThreads) se_bwd_reduce_kernel(const float* __restrict__ dout,
                                                                const float* __restrict__ out,
                                                                const float* __restrict__ y, int HW, int C, int F,
                                                                int slice, float* __restrict__ dres,
                                                                float* __restrict__ dspart) {
  __shared__ float red[4][64];
  const int lane = threadIdx.x & 63, row = threadIdx.x >> 6;
  const int f = blockIdx.x, c = blockIdx.y * 64 + lane, z = blockIdx.z;
  const int pend = min(HW, (z + 1) * slice);
  float acc = 0.f;
  if (c < C) {
    const size_t base = (size_t)f * HW * C + c;
    // eight pixels' loads in flight (128 frames, all 16 blocks: 501 -> 299 us)
#pragma unroll 8
    for (int p = z * slice + row; p < pend; p += 4) {
      const size_t i = base + (size_t)p * C;
      const float o = out[i], g = dout[i], yv = y[i];
      const float d = o > 0.f ? g : 0.f;
      dres[i] = d;
      acc = fmaf(d, yv, acc);
    }
  }
  red[row][lane] = acc;
  __syncthreads();
  if (row == 0 && c < C)
    dspart[((size_t)z * F + f) * C + c] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
}

// Backward through the gate, one workgroup per frame:
//   ds = sum of the slices;  da2 = ds * s (1 - s);  da1 = (W2^T da2) * [a1 > 0];  dz = W1^T da1.
__global__ void __launch_bounds__(kThreads) se_fc_bwd_kernel(const float* __restrict__ dspart, int S, int F,
                                                            const float* __restrict__ s,
                                                            const float* __restrict__ a1, int C, int R,
                                                            const float* __restrict__ w1,
                                                            const float* __restrict__ w2, float* __restrict__ da2,
                                                            float* __restrict__ da1, float* __restrict__ dz) {
  extern __shared__ float sm[];  // d2 [C], d1 [R]
  float* d2 = sm;
  float* d1 = sm + C;
  const int f = blockIdx.x, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int c = threadIdx.x; c < C; c += kThreads) {
    float ds = 0.f;
    for (int k = 0; k < S; ++k) ds += dspart[((size_t)k * F + f) * C + c];
    const float sv = s[(size_t)f * C + c];
    const float v = ds * sv * (1.f - sv);
    d2[c] = v;
    da2[(size_t)f * C + c] = v;
  }
  __syncthreads();
  for (int j = wv; j < R; j += kThreads / 64) {
    float acc = 0.f;
#pragma unroll 8
    for (int c = lane; c < C; c += 64) acc = fmaf(w2[(size_t)c * R + j], d2[c], acc);
    acc = wave_sum(acc);
    if (lane == 0) {
      const float v = a1[(size_t)f * R + j] > 0.f ? acc : 0.f;
      d1[j] = v;
      da1[(size_t)f * R + j] = v;
    }
  }
  __syncthreads();
  for (int c = threadIdx.x; c < C; c += kThreads) {
    float acc = 0.f;
#pragma unroll 16
    for (int j = 0; j < R; ++j) acc = fmaf(w1[(size_t)j * C + c], d1[j], acc);
    dz[(size_t)f * C + c] = acc;
  }
}

// Gate weight gradients, one thread per element, frames summed in order:
//   dW1[j][c] = sum_f da1[f][j] z[f][c],  db1[j] = sum_f da1[f][j],
//   dW2[c][j] = sum_f da2[f][c] relu(a1[f][j]),  db2[c] = sum_f da2[f][c].
__global__ void __launch_bounds__(kThreads) se_fc_wgrad_kernel(const float* __restrict__ z,
                                                              const float* __restrict__ a1,
                                                              const float* __restrict__ da1,
                                                              const float* __restrict__ da2, int F, int C, int R,
                                                              float* __restrict__ gw1, float* __restrict__ gb1,
                                                              float* __restrict__ gw2, float* __restrict__ gb2) {
  const int n1 = R * C, n2 = n1 + R, n3 = n2 + C * R, n4 = n3 + C;
  // sum over the frames in order of term(f), 16 frames' loads in flight
  auto sum = [&](auto load, auto add) {
    float acc = 0.f;
    int f = 0;
    for (; f + 16 <= F; f += 16) {
      float2 v[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) v[q] = load(f + q);
#pragma unroll
      for (int q = 0; q < 16; ++q) acc = add(v[q], acc);
    }
    for (; f < F; ++f) acc = add(load(f), acc);
    return acc;
  };
  auto prod = [](float2 v, float acc) { return fmaf(v.x, v.y, acc); };
  auto plain = [](float2 v, float acc) { return acc + v.x; };
  for (int e = blockIdx.x * kThreads + threadIdx.x; e < n4; e += gridDim.x * kThreads) {
    if (e < n1) {
      const int j = e / C, c = e - j * C;
      gw1[e] = sum([=](int f) { return make_float2(da1[(size_t)f * R + j], z[(size_t)f * C + c]); }, prod);
    } else if (e < n2) {
      const int j = e - n1;
      gb1[j] = sum([=](int f) { return make_float2(da1[(size_t)f * R + j], 0.f); }, plain);
    } else if (e < n3) {
      const int q = e - n2, c = q / R, j = q - c * R;
      gw2[q] = sum([=](int f) { return make_float2(da2[(size_t)f * C + c], fmaxf(a1[(size_t)f * R + j], 0.f)); },
                   prod);
    } else {
      const int c = e - n3;
      gb2[c] = sum([=](int f) { return make_float2(da2[(size_t)f * C + c], 0.f); }, plain);
    }
  }
}

// dy = s[f][c] * dpre + dz[f][c] / HW  (the gradient at the branch y), four channels per thread
__global__ void __launch_bounds__(kThreads) se_excite_bwd_kernel(const float* __restrict__ dpre,
                                                                const float* __restrict__ s,
                                                                const float* __restrict__ dz, int n4,
                                                                FastDiv dhwc4, FastDiv dc4, int C4, float inv_hw,
                                                                float* __restrict__ dy) {
  for (int i = blockIdx.x * kThreads + threadIdx.x; i < n4; i += gridDim.x * kThreads) {
    const int f = dhwc4.div(i), c4 = i - dc4.div(i) * C4;
    const float4 d = ((const float4*)dpre)[i];
    const float4 sv = ((const float4*)s)[f * C4 + c4], zv = ((const float4*)dz)[f * C4 + c4];
    ((float4*)dy)[i] = make_float4(fmaf(sv.x, d.x, zv.x * inv_hw), fmaf(sv.y, d.y, zv.y * inv_hw),
                                   fmaf(sv.z, d.z, zv.z * inv_hw), fmaf(sv.w, d.w, zv.w * inv_hw));
  }
}

unsigned grid_for(long n) { return (unsigned)std::max<long>(1, std::min<long>(cdiv(n, kThreads), 8192)); }

// Output pixels per workgroup: about 2048 workgroups in all, at most 16
// passes of the workgroup's rows.
int pix_per_block(long P, int rows, int G) {
  const long per_group = std::max<long>(1, 2048 / G);
  long pix = (P + per_group - 1) / per_group;
  pix = std::max<long>(rows, std::min<long>(pix, (long)rows * 16));
  return (int)((pix + rows - 1) / rows * rows);
}

// Pixel slices of the squeeze reductions: about 512 workgroups, slices of
// at least 16 pixels, at most kMaxSlices.
int se_slices(int F, int HW, int C) {
  const int base = F * cdiv(C, 64);
  int S = std::max(1, 512 / std::max(base, 1));
  S = std::min(S, std::max(1, HW / 16));
  return std::min(S, kSeMaxSlices);
}

// Register-tiled kernels for these groups?  (Equal input and output widths, one of the instantiated.)
bool gconv_tiled(int cg, int og) { return cg == og && (cg == 4 || cg == 8 || cg == 16 || cg == 32); }

template <typename TW, bool BWD>
void gconv_tile(const ConvGeo& g, int G, const float* src, const TW* w, float* dst, int accumulate, hipStream_t s) {
  const int cg = g.C / G;
  // neighbouring groups of a workgroup: up to 16 channels, a power of two that divides the group count
  int gpw = 1;
  while (2 * gpw * cg <= 16 && G % (2 * gpw) == 0) gpw *= 2;
  const int rows = kThreads / (gpw * cg / 4), H = BWD ? g.H : g.Ho, W = BWD ? g.W : g.Wo;
  const long P = (long)g.B * H * W;
  const int np = P * (G / gpw) >= 2L * rows * 2048 ? 2 : 1;
  const int pix = pix_per_block(P, np * rows, G / gpw);
  const dim3 grid((unsigned)cdiv(P, pix), (unsigned)(G / gpw));
  const size_t sh = (size_t)gpw * (9 * cg * cg + 16) * sizeof(float);
  const PixDiv dv{fast_div(H * W), fast_div(W)};
  switch (cg) {
#define TILE(CG) \
  case CG: \
    if (np == 2) \
      hipLaunchKernelGGL((gconv_tile_kernel<TW, CG, BWD, 2>), grid, dim3(kThreads), sh, s, src, w, dst, g, gpw, pix, \
                         dv, accumulate); \
    else \
      hipLaunchKernelGGL((gconv_tile_kernel<TW, CG, BWD, 1>), grid, dim3(kThreads), sh, s, src, w, dst, g, gpw, pix, \
                         dv, accumulate); \
    break;
    TILE(4) TILE(8) TILE(16) TILE(32)
#undef TILE
  }
}

template <bool BF, int CG>
bool gconv_wgrad_tile(const ConvGeo& g, int G, const float* x, const float* dy, float* part, int chunks, int pix,
                      hipStream_t s) {
  using W = WgradTile<CG>;
  if (G % W::GPW) return false;
  hipLaunchKernelGGL((gconv_wgrad_tile_kernel<BF, CG>), dim3((unsigned)chunks, (unsigned)(G / W::GPW)), dim3(W::T),
                     0, s, x, dy, part, g, pix, PixDiv{fast_div(g.Ho * g.Wo), fast_div(g.Wo)});
  return true;
}

// The register-tiled weight gradient; false where the general kernel has to run.
template <bool BF>
bool gconv_wgrad_tiled(const ConvGeo& g, int G, const float* x, const float* dy, float* part, int chunks, int pix,
                       hipStream_t s) {
  if (!gconv_tiled(g.C / G, g.Co / G)) return false;
  switch (g.C / G) {
    case 4: return gconv_wgrad_tile<BF, 4>(g, G, x, dy, part, chunks, pix, s);
    case 8: return gconv_wgrad_tile<BF, 8>(g, G, x, dy, part, chunks, pix, s);
    case 16: return gconv_wgrad_tile<BF, 16>(g, G, x, dy, part, chunks, pix, s);
    default: return gconv_wgrad_tile<BF, 32>(g, G, x, dy, part, chunks, pix, s);
  }
}

}  // namespace

bool gconv_supported(const ConvGeo& g, int G) {
  if (G <= 0 || g.C % G || g.Co % G || g.KH != 3 || g.KW != 3 || g.pad != 1) return false;
  if (g.stride != 1 && g.stride != 2) return false;
  const int cg = g.C / G, og = g.Co / G;
  // float4 channel loads; one output channel (input channel for the data
  // gradient) per thread of a row; every weight-gradient element among a
  // thread's kEPT; filters of a group within the LDS budget
  if (cg % 4 || og % 4 || cg > kThreads || og > kThreads || og * 9 * cg > kThreads * kEPT) return false;
  if ((size_t)9 * cg * og > (size_t)kLdsFloats || og + 9 * cg > kLdsFloats / 8) return false;
  // 31-bit indices (checked per call for the pixel counts)
  return true;
}

bool gconv_fits(const ConvGeo& g) {
  return (long)g.B * g.H * g.W * g.C < (1L << 31) && (long)g.B * g.Ho * g.Wo * g.Co < (1L << 31);
}

void launch_gconv_fwd(int prec, const ConvGeo& g, int G, const float* x, const void* w, float* y,
                      hipStream_t s) {
  if (gconv_tiled(g.C / G, g.Co / G)) {
    if (prec == 1) gconv_tile<bf16_t, false>(g, G, x, (const bf16_t*)w, y, 0, s);
    else gconv_tile<float, false>(g, G, x, (const float*)w, y, 0, s);
    return;
  }
  const int cg = g.C / G, og = g.Co / G, rows = kThreads / og;
  const long P = (long)g.B * g.Ho * g.Wo;
  const int pix = pix_per_block(P, rows, G);
  const dim3 grid((unsigned)cdiv(P, pix), (unsigned)G);
  const size_t sh = (size_t)9 * cg * og * sizeof(float);
  const PixDiv dv{fast_div(g.Ho * g.Wo), fast_div(g.Wo)};
  if (prec == 1)
    hipLaunchKernelGGL(gconv_fwd_kernel<bf16_t>, grid, dim3(kThreads), sh, s, x, (const bf16_t*)w, y, g, G, pix, dv);
  else
    hipLaunchKernelGGL(gconv_fwd_kernel<float>, grid, dim3(kThreads), sh, s, x, (const float*)w, y, g, G, pix, dv);
}

void launch_gconv_dgrad(int prec, const ConvGeo& g, int G, const float* dy, const void* w, float* dx,
                        int accumulate, hipStream_t s) {
  if (gconv_tiled(g.C / G, g.Co / G)) {
    if (prec == 1) gconv_tile<bf16_t, true>(g, G, dy, (const bf16_t*)w, dx, accumulate, s);
    else gconv_tile<float, true>(g, G, dy, (const float*)w, dx, accumulate, s);
    return;
  }
  const int cg = g.C / G, og = g.Co / G, rows = kThreads / cg;
  const long P = (long)g.B * g.H * g.W;
  const int pix = pix_per_block(P, rows, G);
  const dim3 grid((unsigned)cdiv(P, pix), (unsigned)G);
  const size_t sh = (size_t)9 * cg * og * sizeof(float);
  const PixDiv dv{fast_div(g.H * g.W), fast_div(g.W)};
  if (prec == 1)
    hipLaunchKernelGGL(gconv_dgrad_kernel<bf16_t>, grid, dim3(kThreads), sh, s, dy, (const bf16_t*)w, dx, g, G, pix,
                       dv, accumulate);
  else
    hipLaunchKernelGGL(gconv_dgrad_kernel<float>, grid, dim3(kThreads), sh, s, dy, (const float*)w, dx, g, G, pix,
                       dv, accumulate);
}

void launch_gconv_wgrad(int prec, const ConvGeo& g, int G, const float* x, const float* dy, float* dw,
                        float* part, size_t part_bytes, hipStream_t s) {
  const int cg = g.C / G, og = g.Co / G;
  const long n = (long)g.Co * 9 * cg;
  const long P = (long)g.B * g.Ho * g.Wo;
  // pixels staged per round: the LDS budget over one pixel's dy columns and im2col row
  const int PT = std::max(8, std::min(256, kLdsFloats / (og + 9 * cg)) / 8 * 8);
  const long cap = std::max<long>(1, (long)(part_bytes / ((size_t)n * sizeof(float))));
  // chunks of at least 256 pixels, about 4096 workgroups, within the partial buffer
  long chunks = std::min<long>(std::max<long>(1, 4096 / G), std::max<long>(1, P / 256));
  chunks = std::max<long>(1, std::min(chunks, cap));
  long pix = (P + chunks - 1) / chunks;
  pix = (pix + PT - 1) / PT * PT;
  chunks = (P + pix - 1) / pix;
  const size_t sh = (size_t)PT * (og + 9 * cg) * sizeof(float) + (size_t)PT * 3 * sizeof(int);
  const dim3 grid((unsigned)chunks, (unsigned)G);
  const WgradDiv dv{{fast_div(g.Ho * g.Wo), fast_div(g.Wo)}, fast_div(og), fast_div(9 * cg / 4), fast_div(cg / 4)};
  if (prec == 1 ? gconv_wgrad_tiled<true>(g, G, x, dy, part, (int)chunks, (int)pix, s)
                : gconv_wgrad_tiled<false>(g, G, x, dy, part, (int)chunks, (int)pix, s)) {
  } else if (prec == 1)
    hipLaunchKernelGGL(gconv_wgrad_kernel<true>, grid, dim3(kThreads), sh, s, x, dy, part, g, G, (int)pix, PT, dv);
  else
    hipLaunchKernelGGL(gconv_wgrad_kernel<false>, grid, dim3(kThreads), sh, s, x, dy, part, g, G, (int)pix, PT, dv);
  hipLaunchKernelGGL(chunk_sum_kernel, dim3(grid_for(n)), dim3(kThreads), 0, s, part, (int)chunks, (int)n, dw);
}

void launch_se_forward(const float* y, const float* res, int F, int HW, int C, int R, const float* w1,
                       const float* b1, const float* w2, const float* b2, float* zpart, float* z, float* a1,
                       float* gate, float* out, hipStream_t s) {
  const int S = se_slices(F, HW, C), slice = cdiv(HW, S);
  hipLaunchKernelGGL(se_squeeze_kernel, dim3(F, cdiv(C, 64), S), dim3(kThreads), 0, s, y, HW, C, F, slice, zpart);
  hipLaunchKernelGGL(se_hidden_kernel, dim3(F, cdiv(R, 16)), dim3(kThreads), (size_t)C * sizeof(float), s, zpart,
                     S, F, 1.f / HW, C, R, w1, b1, z, a1);
  hipLaunchKernelGGL(se_gate_kernel, dim3(F, cdiv(C, 64)), dim3(kThreads), (size_t)(R + 256) * sizeof(float), s, a1,
                     C, R, w2, b2, gate);
  const int n4 = F * HW * C / 4;
  hipLaunchKernelGGL(se_excite_kernel, dim3(grid_for(n4)), dim3(kThreads), 0, s, y, gate, res, n4,
                     fast_div(HW * C / 4), fast_div(C / 4), C / 4, out);
}

void launch_se_backward(const float* dout, const float* out, const float* y, const float* z, const float* a1,
                        const float* gate, int F, int HW, int C, int R, const float* w1, const float* w2,
                        float* dres, float* dspart, float* da2, float* da1, float* dz, float* gw1, float* gb1,
                        float* gw2, float* gb2, float* dy, hipStream_t s) {
  const int S = se_slices(F, HW, C), slice = cdiv(HW, S);
  hipLaunchKernelGGL(se_bwd_reduce_kernel, dim3(F, cdiv(C, 64), S), dim3(kThreads), 0, s, dout, out, y, HW, C, F,
                     slice, dres, dspart);
  hipLaunchKernelGGL(se_fc_bwd_kernel, dim3(F), dim3(kThreads), (size_t)(C + R) * sizeof(float), s, dspart, S, F,
                     gate, a1, C, R, w1, w2, da2, da1, dz);
  const long nw = 2L * R * C + R + C;
  hipLaunchKernelGGL(se_fc_wgrad_kernel, dim3(grid_for(nw)), dim3(kThreads), 0, s, z, a1, da1, da2, F, C, R, gw1,
                     gb1, gw2, gb2);
  const int n4 = F * HW * C / 4;
  hipLaunchKernelGGL(se_excite_bwd_kernel, dim3(grid_for(n4)), dim3(kThreads), 0, s, dres, gate, dz, n4,
                     fast_div(HW * C / 4), fast_div(C / 4), C / 4, 1.f / HW, dy);
}

// LDS-tiled MFMA GEMM core and its operand loaders (convolution forward,
// data gradient, weight gradient as implicit GEMMs; plain dense products).
//
// C[m][n] = alpha * sum_k A(m, k) B(n, k)  (+= C) (+ bias[n]) (ReLU)
//
// A workgroup of 256 threads (4 wavefronts) owns a BM x BN tile.  Operands
// are staged through double-buffered LDS as [rows][k] (k contiguous), one
// barrier per K tile; the next tile's global loads are in flight while the
// current tile feeds the matrix cores.  Every operand "chunk" is 8
// consecutive k of one row: for operands contiguous along k it is one or two
// vector loads, for operands contiguous along rows (transposed reads) the
// lanes of a wavefront walk the rows so each of the 8 scalar loads is
// coalesced; either way the chunk lands in LDS with one 16-byte write.
// The weight gradient reads 4 rows x 4 k as four row vectors and transposes
// them in registers (QUADS), or 8 rows x 2 k stored as pairs (RT).
//
// bfloat16: v_mfma_f32_32x32x16_bf16 on 32x32 fragments.  float32: four
// v_mfma_f32_16x16x4_f32 per 16-k step on 16x16 fragments.  A and B use the
// same lane -> k assignment, so the order of k inside a step is irrelevant.
// SPLIT (bfloat16 only): A is carried as hi + lo bfloat16 parts (two MFMAs),
// giving the gradient operand of backward products a 16-bit mantissa.
// Accumulation is float32; a split over K writes partial tiles that a second
// kernel sums in a fixed order (no float atomics: results are deterministic).
#pragma once
#include "common.h"
#include "kernels.h"

typedef float v16f __attribute__((ext_vector_type(16)));

// ------------------------------------------------------------- loads
DEV void zero8(float v[8]) {
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = 0.f;
}

template <typename T>
DEV void load8(const T* p, float v[8]);
template <>
DEV void load8<float>(const float* p, float v[8]) {
  const float4 a = *(const float4*)p, b = *(const float4*)(p + 4);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
template <>
DEV void load8<bf16_t>(const bf16_t* p, float v[8]) {
  const uint4 a = *(const uint4*)p;
  const uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = __uint_as_float(w[i] << 16);
    v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
}

DEV bool aligned16(const void* p) { return (((uintptr_t)p) & 15) == 0; }

// ------------------------------------------------------------ problems
// Each problem exposes, for A (rows m) and B (rows n): a per-row state built
// once per thread (rowA / rowB) and a chunk loader (a8 / b8) returning the 8
// values at k .. k+7 (k a multiple of 8; entries past K are 0).

// Forward: A(m = (b,ho,wo), k = (kh,kw,ci)) = x[b][ho*s-p+kh][wo*s-p+kw][ci]; B(n = co, k) = w[co][k].
template <typename TW>
struct ConvFwdProb {
  static constexpr int kKind = 1;
  ConvGeo g;
  FastDiv dC, dKW, dHoWo, dWo;
  const float* x;
  const TW* w;
  int M, N, K;
  struct RA {
    int off, h0, w0, ok;
  };
  struct RB {
    const TW* p;
    int ok;
  };
  DEV RA rowA(int m) const {
    RA r{0, 0, 0, m < M};
    if (r.ok) {
      const int b = dHoWo.div(m), q = m - b * g.Ho * g.Wo;
      const int ho = dWo.div(q), wo = q - ho * g.Wo;
      r.off = b * g.H * g.W * g.C;
      r.h0 = ho * g.stride - g.pad;
      r.w0 = wo * g.stride - g.pad;
    }
    return r;
  }
  DEV RB rowB(int n) const { return RB{w + (size_t)n * K, n < N}; }
  DEV void a8(const RA& r, int k, float v[8]) const {
    if (!r.ok) return zero8(v);
    if ((g.C & 7) == 0) {
      if (k >= K) return zero8(v);
      const int tap = dC.div(k), ci = k - tap * g.C;
      const int kh = dKW.div(tap), kw = tap - kh * g.KW;
      const int hi = r.h0 + kh, wi = r.w0 + kw;
      if ((unsigned)hi < (unsigned)g.H && (unsigned)wi < (unsigned)g.W)
        return load8(x + r.off + ((size_t)hi * g.W + wi) * g.C + ci, v);
      return zero8(v);
    }
    if ((g.C & 3) == 0) {
      // two 4-channel quads (one or two taps), each one float4 load
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int kk = k + 4 * h;
        float* o = v + 4 * h;
        o[0] = o[1] = o[2] = o[3] = 0.f;
        if (kk >= K) continue;
        const int tap = dC.div(kk), ci = kk - tap * g.C;
        const int kh = dKW.div(tap), kw = tap - kh * g.KW;
        const int hi = r.h0 + kh, wi = r.w0 + kw;
        if ((unsigned)hi < (unsigned)g.H && (unsigned)wi < (unsigned)g.W) {
          const float4 t = *(const float4*)(x + r.off + ((size_t)hi * g.W + wi) * g.C + ci);
          o[0] = t.x; o[1] = t.y; o[2] = t.z; o[3] = t.w;
        }
      }
      return;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int kk = k + e;
      float val = 0.f;
      if (kk < K) {
        const int tap = dC.div(kk), ci = kk - tap * g.C;
        const int kh = dKW.div(tap), kw = tap - kh * g.KW;
        const int hi = r.h0 + kh, wi = r.w0 + kw;
        if ((unsigned)hi < (unsigned)g.H && (unsigned)wi < (unsigned)g.W)
          val = x[r.off + ((size_t)hi * g.W + wi) * g.C + ci];
      }
      v[e] = val;
    }
  }
  DEV void b8(const RB& r, int k, float v[8]) const {
    if (!r.ok) return zero8(v);
    if (k + 8 <= K && aligned16(r.p + k)) return load8(r.p + k, v);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (k + e < K) ? ldf(r.p + k + e) : 0.f;
  }
};

// Data gradient over one class of input pixels: rows m = (b, hq, wq) are
// the pixels hi = step*hq + rh, wi = step*wq + rw (step 1: every pixel;
// step 2: one of the four parity classes of a stride-2 convolution), and k =
// (tap t of the class, co) with kh = kh0 + step*(t / nkw), kw = kw0 +
// step*(t % nkw), the only taps for which (hi + pad - kh) / stride is exact.
// A(m, k) = dy[b][(hi+pad-kh)/s][(wi+pad-kw)/s][co] (0 outside the output);
// B(n = ci, k) = wt[ci][kh*KW + kw][co] (weights reordered so B rows are
// contiguous along k).
template <typename TW>
struct ConvDgradProb {
  static constexpr int kKind = 2;
  ConvGeo g;
  FastDiv dCo, dNkw, dHqWq, dWq;
  const float* dy;
  const TW* wt;
  int M, N, K;  // M = B*Hq*Wq, N = C, K = nkh*nkw*Co
  int step, rh, rw, kh0, kw0, nkw, Wq;
  struct RA {
    int off, th, tw, ok;
  };
  struct RB {
    const TW* p;
    int ok;
  };
  DEV RA rowA(int m) const {
    RA r{0, 0, 0, m < M};
    if (r.ok) {
      const int b = dHqWq.div(m), q = m - b * (M / g.B);
      const int hq = dWq.div(q), wq = q - hq * Wq;
      r.off = b * g.Ho * g.Wo * g.Co;
      r.th = step * hq + rh + g.pad;
      r.tw = step * wq + rw + g.pad;
    }
    return r;
  }
  DEV RB rowB(int n) const { return RB{wt + (size_t)n * g.KH * g.KW * g.Co, n < N}; }
  // tap t -> (kh, kw) and the source output pixel; false outside the output
  DEV bool src(const RA& r, int t, int& tap, int& pix) const {
    const int ih = dNkw.div(t), iw = t - ih * nkw;
    const int kh = kh0 + step * ih, kw = kw0 + step * iw;
    tap = kh * g.KW + kw;
    const int th = r.th - kh, tw = r.tw - kw;
    if (th < 0 || tw < 0) return false;
    const int ho = g.stride == 2 ? th >> 1 : th, wo = g.stride == 2 ? tw >> 1 : tw;
    if (ho >= g.Ho || wo >= g.Wo) return false;
    pix = ho * g.Wo + wo;
    return true;
  }
  DEV void a8(const RA& r, int k, float v[8]) const {
    if (!r.ok || k >= K) return zero8(v);
    if ((g.Co & 7) == 0) {
      const int t = dCo.div(k), co = k - t * g.Co;
      int tap, pix;
      if (src(r, t, tap, pix)) return load8(dy + r.off + (size_t)pix * g.Co + co, v);
      return zero8(v);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int kk = k + e;
      float val = 0.f;
      if (kk < K) {
        const int t = dCo.div(kk), co = kk - t * g.Co;
        int tap, pix;
        if (src(r, t, tap, pix)) val = dy[r.off + (size_t)pix * g.Co + co];
      }
      v[e] = val;
    }
  }
  DEV void b8(const RB& r, int k, float v[8]) const {
    if (!r.ok || k >= K) return zero8(v);
    if ((g.Co & 7) == 0) {
      const int t = dCo.div(k), co = k - t * g.Co;
      const int ih = dNkw.div(t), iw = t - ih * nkw;
      const int tap = (kh0 + step * ih) * g.KW + kw0 + step * iw;
      const TW* p = r.p + (size_t)tap * g.Co + co;
      if (aligned16(p)) return load8(p, v);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = ldf(p + e);
      return;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int kk = k + e;
      float val = 0.f;
      if (kk < K) {
        const int t = dCo.div(kk), co = kk - t * g.Co;
        const int ih = dNkw.div(t), iw = t - ih * nkw;
        val = ldf(r.p + (size_t)((kh0 + step * ih) * g.KW + kw0 + step * iw) * g.Co + co);
      }
      v[e] = val;
    }
  }
};

// 8 consecutive weights as stored, and their copy to an LDS row.
template <typename TW> struct Raw8;
template <> struct Raw8<bf16_t> { uint4 v; };
template <> struct Raw8<float> { float4 v, w; };
DEV void load_raw(const bf16_t* p, Raw8<bf16_t>& r) { r.v = *(const uint4*)p; }
DEV void load_raw(const float* p, Raw8<float>& r) {
  r.v = *(const float4*)p;
  r.w = *(const float4*)(p + 4);
}
DEV void zero_raw(Raw8<bf16_t>& r) { r.v = make_uint4(0, 0, 0, 0); }
DEV void zero_raw(Raw8<float>& r) { r.v = r.w = make_float4(0.f, 0.f, 0.f, 0.f); }
DEV void put_raw(bf16_t* d, const Raw8<bf16_t>& r) { *(uint4*)d = r.v; }
DEV void put_raw(float* d, const Raw8<float>& r) {
  *(float4*)d = r.v;
  *(float4*)(d + 4) = r.w;
}

// Forward and data gradient where a K tile lies in one tap (UNI: channels a
// multiple of 32, weights 16-byte aligned, at most 2^31 elements of x or dy): the
// tap and its offsets are scalars of the tile (KT), a row adds its own, and
// weights go to LDS as they are stored.  The general forms divide once a chunk and
// thread and convert bfloat16 weights to float and back.  Same values, same order.
// All such products of 256 frames, bfloat16: forward 1.55 -> 1.23 ms, data
// gradient 2.06 -> 1.70 ms; an act step of 4 envs 676 -> 642 us.
template <typename TW>
struct ConvFwdUProb {
  static constexpr int kKind = 1;
  typedef TW Weight;
  ConvGeo g;
  FastDiv dC, dKW, dHoWo, dWo;
  const float* x;
  const TW* w;
  int M, N, K;
  struct RA {
    int base, h0, w0, ok;
  };
  struct RB {
    const TW* p;
    int ok;
  };
  struct KT {
    int off, kh, kw, k;
  };
  DEV RA rowA(int m, int kc) const {
    RA r{0, 0, 0, m < M};
    if (r.ok) {
      const int b = dHoWo.div(m), q = m - b * g.Ho * g.Wo;
      const int ho = dWo.div(q), wo = q - ho * g.Wo;
      r.h0 = ho * g.stride - g.pad;
      r.w0 = wo * g.stride - g.pad;
      r.base = ((b * g.H + r.h0) * g.W + r.w0) * g.C + kc;
    }
    return r;
  }
  DEV RB rowB(int n, int kc) const { return RB{w + (size_t)(n < N ? n : 0) * K + kc, n < N}; }
  DEV KT ktile(int k0) const {
    const int tap = dC.div(k0), kh = dKW.div(tap), kw = tap - kh * g.KW;
    return KT{(kh * g.W + kw) * g.C + k0 - tap * g.C, kh, kw, k0};
  }
  DEV void a8(const RA& r, const KT& t, float v[8]) const {
    if (r.ok && (unsigned)(r.h0 + t.kh) < (unsigned)g.H && (unsigned)(r.w0 + t.kw) < (unsigned)g.W)
      return load8(x + (r.base + t.off), v);
    zero8(v);
  }
  DEV void b8(const RB& r, const KT& t, Raw8<TW>& v) const {
    if (r.ok) load_raw(r.p + t.k, v);
    else zero_raw(v);
  }
};

template <typename TW>
struct ConvDgradUProb {
  static constexpr int kKind = 2;
  typedef TW Weight;
  ConvGeo g;
  FastDiv dCo, dNkw, dHqWq, dWq;
  const float* dy;
  const TW* wt;
  int M, N, K;  // as ConvDgradProb
  int step, rh, rw, kh0, kw0, nkw, Wq;
  struct RA {
    int off, th, tw, ok;
  };
  struct RB {
    const TW* p;
    int ok;
  };
  struct KT {
    int co, kh, kw, w;
  };
  DEV RA rowA(int m, int kc) const {
    RA r{0, 0, 0, m < M};
    if (r.ok) {
      const int b = dHqWq.div(m), q = m - b * (M / g.B);
      const int hq = dWq.div(q), wq = q - hq * Wq;
      r.off = b * g.Ho * g.Wo * g.Co + kc;
      r.th = step * hq + rh + g.pad;
      r.tw = step * wq + rw + g.pad;
    }
    return r;
  }
  DEV RB rowB(int n, int kc) const {
    return RB{wt + (size_t)(n < N ? n : 0) * g.KH * g.KW * g.Co + kc, n < N};
  }
  DEV KT ktile(int k0) const {
    const int t = dCo.div(k0), co = k0 - t * g.Co, ih = dNkw.div(t), iw = t - ih * nkw;
    const int kh = kh0 + step * ih, kw = kw0 + step * iw;
    return KT{co, kh, kw, (kh * g.KW + kw) * g.Co + co};
  }
  DEV void a8(const RA& r, const KT& t, float v[8]) const {
    const int sh = g.stride == 2 ? 1 : 0;
    const int th = r.th - t.kh, tw = r.tw - t.kw, ho = th >> sh, wo = tw >> sh;
    if (r.ok && (unsigned)ho < (unsigned)g.Ho && (unsigned)wo < (unsigned)g.Wo)
      return load8(dy + (r.off + (ho * g.Wo + wo) * g.Co + t.co), v);
    zero8(v);
  }
  DEV void b8(const RB& r, const KT& t, Raw8<TW>& v) const {
    if (r.ok) load_raw(r.p + t.w, v);
    else zero_raw(v);
  }
};

// Weight gradient: C(m = co, n = (kh,kw,ci)) = sum_r dy[r][co] * im2col(x)[r][n],
// r = (b,ho,wo) is the reduction.  Both operands are contiguous along their
// rows: lanes walk co (A) or n (B); 8 consecutive r per chunk.
struct ConvWgradProb {
  static constexpr int kKind = 3;
  ConvGeo g;
  FastDiv dC, dKW, dHoWo, dWo;
  const float* x;
  const float* dy;
  int M, N, K;  // M = Co, N = KH*KW*C, K = B*Ho*Wo
  struct RA {
    int co, ok;
  };
  struct RB {
    int kh, kw, ci, ok;
  };
  DEV RA rowA(int m) const { return RA{m, m < M}; }
  DEV RB rowB(int n) const {
    RB r{0, 0, 0, n < N};
    if (r.ok) {
      const int tap = dC.div(n);
      r.ci = n - tap * g.C;
      r.kh = dKW.div(tap);
      r.kw = tap - r.kh * g.KW;
    }
    return r;
  }
  DEV void a8(const RA& r, int k, float v[8]) const {
    if (!r.ok) return zero8(v);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (k + e < K) ? dy[(size_t)(k + e) * g.Co + r.co] : 0.f;
  }
  DEV void b8(const RB& r, int k, float v[8]) const {
    if (!r.ok || k >= K) return zero8(v);
    const int hw = g.Ho * g.Wo;
    int b = dHoWo.div(k);
    const int q = k - b * hw;
    int ho = dWo.div(q), wo = q - ho * g.Wo;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float val = 0.f;
      if (k + e < K) {
        const int hi = ho * g.stride - g.pad + r.kh, wi = wo * g.stride - g.pad + r.kw;
        if ((unsigned)hi < (unsigned)g.H && (unsigned)wi < (unsigned)g.W)
          val = x[(((size_t)b * g.H + hi) * g.W + wi) * g.C + r.ci];
      }
      v[e] = val;
      if (++wo == g.Wo) {
        wo = 0;
        if (++ho == g.Ho) {
          ho = 0;
          ++b;
        }
      }
    }
  }
};

// Weight gradient with channel quads: a unit is 4 consecutive channels (co for
// A, ci of one tap for B) at 4 consecutive reduction indices r = (b,ho,wo),
// four float4 loads along the NHWC channel axis, coalesced over the lanes.
// A quarter of the loads and index arithmetic of the scalar gather, the same
// conversions: 28 vector instructions a matrix instruction (counted, bfloat16,
// 256 frames), 81 before.  Of what is left the wavefronts wait 62 % of their
// cycles, for a K tile's loads and at its barrier; two tiles in flight gained
// nothing (float32) or spilled (bfloat16).  All weight gradients of 256 frames (54
// launches): bfloat16 3.01 -> 1.95 ms, float32 4.25 -> 3.21 ms (its stem alone, 4
// channels a tap, was slower so, 317 -> 360 us, and takes 8-row vectors again: below).
// Needs Co % 4 == 0, C % 4 == 0 and 16-byte aligned x and dy.
struct ConvWgradQProb {
  static constexpr int kKind = 3;
  ConvGeo g;
  FastDiv dC, dKW, dHoWo, dWo;
  const float* x;
  const float* dy;
  int M, N, K;  // M = Co, N = KH*KW*C, K = B*Ho*Wo
  int flat;     // 1x1, stride 1, no padding: reduction row r is row r of x
  struct RU {
    int c, kh, kw, ok;
  };
  // Tile-table kind: 4 where the saved rows of these sizes have it (4n, not 8n
  // input channels).  A row also names the K split, so a table saved before keeps
  // its owner's sums bit for bit; its tiles cost a little (an update of 256 frames
  // on such a table 12.22 ms, on one tuned now 12.03, float32 15.57 and 15.05).
  int kind() const { return g.C % 8 == 0 || g.Co % 8 != 0 ? 3 : 4; }
  DEV RU rowA(int m) const { return RU{m, 0, 0, m < M}; }
  DEV RU rowB(int n) const {
    RU r{0, 0, 0, n < N};
    if (r.ok) {
      const int tap = dC.div(n);
      r.c = n - tap * g.C;
      r.kh = dKW.div(tap);
      r.kw = tap - r.kh * g.KW;
    }
    return r;
  }
  DEV void rows4(const float* base, int ld, int k, int kend, float4 v[4]) const {
    const float* q = base + (size_t)k * ld;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      v[e] = k + e < kend ? *(const float4*)(q + (size_t)e * ld) : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  DEV void a44(const RU& r, int k, int kend, float4 v[4]) const {
    rows4(dy + (r.ok ? r.c : 0), g.Co, k, r.ok ? kend : 0, v);
  }
  DEV void b44(const RU& r, int k, int kend, float4 v[4]) const {
    if (!r.ok) kend = 0;
    if (flat) return rows4(x + r.c, g.C, k, kend, v);
    int b = dHoWo.div(k);
    const int q = k - b * g.Ho * g.Wo;
    int ho = dWo.div(q), wo = q - ho * g.Wo;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int hi = ho * g.stride - g.pad + r.kh, wi = wo * g.stride - g.pad + r.kw;
      const bool in = k + e < kend && (unsigned)hi < (unsigned)g.H && (unsigned)wi < (unsigned)g.W;
      v[e] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (in) v[e] = *(const float4*)(x + (((size_t)b * g.H + hi) * g.W + wi) * g.C + r.c);
      if (++wo == g.Wo) {
        wo = 0;
        if (++ho == g.Ho) {
          ho = 0;
          ++b;
        }
      }
    }
  }
};

// Weight gradient with 8-row vectors: a unit is 8 consecutive rows m..m+7 (output
// channels for A, (kh,kw,ci) for B: two taps of 4 channels where C is not 8n) at
// reduction indices k and k+1, two float4 loads each, stored down the LDS rows as
// pairs along k (put8t2).  Needs Co % 8 == 0, C % 4 == 0, 16-byte aligned x and dy.
// Float32, where the quads fit the tile badly (see the dispatch); the loads of
// both k of all units go out before the first is used: the stem of 256 frames
// 300 us when they went out unit by unit, 232 us so.
struct ConvWgradRTProb {
  static constexpr int kKind = 4;
  ConvGeo g;
  FastDiv dHoWo, dWo;
  const float* x;
  const float* dy;
  int M, N, K;  // as ConvWgradProb
  struct RA {
    int co, ok;
  };
  struct RB {
    int kh0, kw0, ci0, kh1, kw1, ci1, nv;  // taps of rows n..n+3 and n+4..n+7; rows within N (0, 4 or 8)
  };
  DEV RA rowA(int m) const { return RA{m, m < M}; }
  DEV RB rowB(int n) const {
    const int t0 = n / g.C, t1 = (n + 4) / g.C;
    RB r;
    r.nv = max(0, min(8, N - n));
    r.ci0 = n - t0 * g.C;
    r.kh0 = t0 / g.KW;
    r.kw0 = t0 - r.kh0 * g.KW;
    r.ci1 = n + 4 - t1 * g.C;
    r.kh1 = t1 / g.KW;
    r.kw1 = t1 - r.kh1 * g.KW;
    return r;
  }
  DEV void a8(const RA& r, int k, float v[8]) const {
    if (!r.ok || k >= K) return zero8(v);
    load8(dy + (size_t)k * g.Co + r.co, v);
  }
  DEV void b8(const RB& r, int k, float v[8]) const {
    zero8(v);
    if (r.nv <= 0 || k >= K) return;
    const int b = dHoWo.div(k), q = k - b * g.Ho * g.Wo;
    const int ho = dWo.div(q), wo = q - ho * g.Wo;
    const int hb = ho * g.stride - g.pad, wb = wo * g.stride - g.pad;
    const float* xb = x + (size_t)b * g.H * g.W * g.C;
    auto quad = [&](int kh, int kw, int ci, float* o) {
      const int hi = hb + kh, wi = wb + kw;
      if ((unsigned)hi < (unsigned)g.H && (unsigned)wi < (unsigned)g.W) {
        const float4 t = *(const float4*)(xb + ((size_t)hi * g.W + wi) * g.C + ci);
        o[0] = t.x; o[1] = t.y; o[2] = t.z; o[3] = t.w;
      }
    };
    quad(r.kh0, r.kw0, r.ci0, v);
    if (r.nv > 4) quad(r.kh1, r.kw1, r.ci1, v + 4);
  }
};

// Dense: A(m, k) = a[m*lda + k] (or a[k*lda + m] when TA), B(n, k) = b[n*ldb + k]
// (or b[k*ldb + n] when TB).
template <typename TAe, typename TBe, bool TA, bool TB>
struct DenseProb {
  static constexpr int kKind = 8 + 4 * (int)(sizeof(TBe) == 2) + 2 * (int)TA + (int)TB;
  const TAe* a;
  const TBe* b;
  int lda, ldb;
  int M, N, K;
  struct RA {
    int m, ok;
  };
  typedef RA RB;
  DEV RA rowA(int m) const { return RA{m, m < M}; }
  DEV RB rowB(int n) const { return RB{n, n < N}; }
  template <typename T, bool TR>
  DEV static void get(const T* base, int ld, int row, int k, int K, float v[8]) {
    if (!TR) {
      const T* p = base + (size_t)row * ld + k;
      if (k + 8 <= K && aligned16(p)) return load8(p, v);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = (k + e < K) ? ldf(p + e) : 0.f;
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = (k + e < K) ? ldf(base + (size_t)(k + e) * ld + row) : 0.f;
    }
  }
  DEV void a8(const RA& r, int k, float v[8]) const {
    if (!r.ok) return zero8(v);
    get<TAe, TA>(a, lda, r.m, k, K, v);
  }
  DEV void b8(const RB& r, int k, float v[8]) const {
    if (!r.ok) return zero8(v);
    get<TBe, TB>(b, ldb, r.m, k, K, v);
  }
};

// Bytes per element of a convolution's weight operand (the B rows of the
// forward product); 0 for other products (GEMM launch timer's byte count).
template <class P> struct WeightBytes { static constexpr int v = 0; };
template <typename TW> struct WeightBytes<ConvFwdProb<TW>> { static constexpr int v = (int)sizeof(TW); };
template <typename TW> struct WeightBytes<ConvFwdUProb<TW>> { static constexpr int v = (int)sizeof(TW); };

// Is the operand contiguous along rows (so lanes should walk rows)?  QUADS:
// units are 4 rows x 4 k (vector loads along rows, transposed in registers).
// RT: units are 8 rows x 2 k.  UNI: a K tile lies in one tap.
template <class P> struct Layout;
template <> struct Layout<ConvWgradQProb> {
  static constexpr bool A_ROWS = true, B_ROWS = true, QUADS = true, RT = false, UNI = false;
};
template <> struct Layout<ConvWgradRTProb> {
  static constexpr bool A_ROWS = false, B_ROWS = false, QUADS = false, RT = true, UNI = false;
};
template <typename TW> struct Layout<ConvFwdProb<TW>> {
  static constexpr bool A_ROWS = false, B_ROWS = false, QUADS = false, RT = false, UNI = false;
};
template <typename TW> struct Layout<ConvDgradProb<TW>> {
  static constexpr bool A_ROWS = false, B_ROWS = false, QUADS = false, RT = false, UNI = false;
};
template <typename TW> struct Layout<ConvFwdUProb<TW>> {
  static constexpr bool A_ROWS = false, B_ROWS = false, QUADS = false, RT = false, UNI = true;
};
template <typename TW> struct Layout<ConvDgradUProb<TW>> {
  static constexpr bool A_ROWS = false, B_ROWS = false, QUADS = false, RT = false, UNI = true;
};
template <> struct Layout<ConvWgradProb> {
  static constexpr bool A_ROWS = true, B_ROWS = true, QUADS = false, RT = false, UNI = false;
};
template <typename A_, typename B_, bool TA, bool TB>
struct Layout<DenseProb<A_, B_, TA, TB>> {
  static constexpr bool A_ROWS = TA, B_ROWS = TB, QUADS = false, RT = false, UNI = false;
};
// Tile-table kind of a problem.
template <class P> int kind_of(const P&) { return P::kKind; }
inline int kind_of(const ConvWgradQProb& p) { return p.kind(); }

// ------------------------------------------------------------- MFMA
template <typename TC>
struct Mma;
template <>
struct Mma<bf16_t> {  // v_mfma_f32_32x32x16_bf16
  static constexpr int FR = 32, NOUT = 16;
  typedef v16f Acc;
  DEV static int row(int l) { return l & 31; }
  DEV static int kof(int l) { return (l >> 5) * 8; }
  DEV static Acc zero() {
    Acc a;
#pragma unroll
    for (int i = 0; i < 16; ++i) a[i] = 0.f;
    return a;
  }
  DEV static Acc mma(const bf16_t* a, const bf16_t* b, Acc c) {
    const v8bf x = *(const v8bf*)a, y = *(const v8bf*)b;
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, y, c, 0, 0, 0);
  }
  // accumulator element r of lane l
  DEV static int orow(int l, int r) { return 8 * (r >> 2) + 4 * (l >> 5) + (r & 3); }
  DEV static int ocol(int l) { return l & 31; }
};
template <>
struct Mma<float> {  // 4 x v_mfma_f32_16x16x4_f32 per 16-k step
  static constexpr int FR = 16, NOUT = 4;
  typedef v4f Acc;
  DEV static int row(int l) { return l & 15; }
  DEV static int kof(int l) { return (l >> 4) * 4; }
  DEV static Acc zero() { return v4f{0.f, 0.f, 0.f, 0.f}; }
  DEV static Acc mma(const float* a, const float* b, Acc c) {
    const float4 x = *(const float4*)a, y = *(const float4*)b;
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(x.x, y.x, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(x.y, y.y, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(x.z, y.z, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(x.w, y.w, c, 0, 0, 0);
    return c;
  }
  DEV static int orow(int l, int r) { return 4 * (l >> 4) + r; }
  DEV static int ocol(int l) { return l & 15; }
};

// 8 floats -> LDS row segment in the operand type (hi part; lo = residual).
DEV void put8(float* d, const float v[8], float*) {
  *(float4*)d = make_float4(v[0], v[1], v[2], v[3]);
  *(float4*)(d + 4) = make_float4(v[4], v[5], v[6], v[7]);
}
// Two floats -> packed bfloat16 pair, round to nearest even (v_cvt_pk_bf16_f32).
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
DEV uint32_t pk_bf16(float a, float b) {
  const bf16x2_t r = __builtin_convertvector((f32x2_t){a, b}, bf16x2_t);
  return __builtin_bit_cast(uint32_t, r);
}
DEV void put8(bf16_t* d, const float v[8], bf16_t* lo) {
  uint32_t h[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) h[i] = pk_bf16(v[2 * i], v[2 * i + 1]);
  *(uint4*)d = make_uint4(h[0], h[1], h[2], h[3]);
  if (lo) {
    uint32_t l[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float a = __uint_as_float(h[i] << 16), b = __uint_as_float(h[i] & 0xffff0000u);
      l[i] = pk_bf16(v[2 * i] - a, v[2 * i + 1] - b);
    }
    *(uint4*)lo = make_uint4(l[0], l[1], l[2], l[3]);
  }
}

// 4 rows x 4 k (v[e] = the rows' values at k+e) -> 4 consecutive LDS rows
// (stride ld elements): one 16-byte (float) or 8-byte (bfloat16) store a row.
DEV void put44(float* d, int ld, const float4 v[4], float*) {
  *(float4*)d = make_float4(v[0].x, v[1].x, v[2].x, v[3].x);
  *(float4*)(d + ld) = make_float4(v[0].y, v[1].y, v[2].y, v[3].y);
  *(float4*)(d + 2 * ld) = make_float4(v[0].z, v[1].z, v[2].z, v[3].z);
  *(float4*)(d + 3 * ld) = make_float4(v[0].w, v[1].w, v[2].w, v[3].w);
}
DEV void put44(bf16_t* d, int ld, const float4 v[4], bf16_t* lo) {
  const float* f = (const float*)v;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t h0 = pk_bf16(f[j], f[4 + j]), h1 = pk_bf16(f[8 + j], f[12 + j]);
    *(uint2*)(d + j * ld) = make_uint2(h0, h1);
    if (lo) {
      const uint32_t l0 = pk_bf16(f[j] - __uint_as_float(h0 << 16), f[4 + j] - __uint_as_float(h0 & 0xffff0000u));
      const uint32_t l1 = pk_bf16(f[8 + j] - __uint_as_float(h1 << 16), f[12 + j] - __uint_as_float(h1 & 0xffff0000u));
      *(uint2*)(lo + j * ld) = make_uint2(l0, l1);
    }
  }
}

// 8 rows at k and k+1 (k even) -> columns k, k+1 of 8 consecutive LDS rows (stride
// ld): a pair a row.  The lanes of a wavefront walk k, so a store instruction
// covers consecutive LDS words of a row.
DEV void put8t2(float* d, int ld, const float v0[8], const float v1[8]) {
#pragma unroll
  for (int e = 0; e < 8; ++e) *(float2*)(d + e * ld) = make_float2(v0[e], v1[e]);
}

// ------------------------------------------------------------- kernel
template <class Prob, typename TC, int BM, int BN, int WGM, int WGN, bool SPLIT>
__global__ void __launch_bounds__(256) gemm_kernel(Prob p, Epi e, int tiles_n, int k_per_split) {
  using MM = Mma<TC>;
  constexpr int BK = 32;
  constexpr int FR = MM::FR;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int FM = WTM / FR, FN = WTN / FR;
  static_assert(WGM * WGN == 4 && FM >= 1 && FN >= 1, "bad tile");
  constexpr int LDK = BK + 16 / (int)sizeof(TC);  // padded LDS row (elements)
  constexpr bool AR = Layout<Prob>::A_ROWS, BR = Layout<Prob>::B_ROWS, QUADS = Layout<Prob>::QUADS;
  // chunks (one row, 8 k) per K tile and thread
  constexpr int CA = BM * BK / 8, CB = BN * BK / 8;
  constexpr int QA = (CA + 255) / 256, QB = (CB + 255) / 256;
  // QUADS: units (4 rows, 4 k) of A, then of B; a wavefront's units are all of one operand
  constexpr int UA = BM * BK / 16, UB = BN * BK / 16, QU = (UA + UB + 255) / 256;
  static_assert(UA % 64 == 0 && UB % 64 == 0, "units of a wavefront");
  constexpr int NSPL = SPLIT ? 2 : 1;
  __shared__ __attribute__((aligned(16))) TC sA[NSPL][2][BM * LDK];
  __shared__ __attribute__((aligned(16))) TC sB[2][BN * LDK];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tm = blockIdx.x / tiles_n, tn = blockIdx.x - tm * tiles_n;
  const int m0 = tm * BM, n0 = tn * BN;
  const int kbeg = blockIdx.y * k_per_split;
  const int kend = min(p.K, kbeg + k_per_split);
  const int wm0 = (wave / WGN) * WTM, wn0 = (wave % WGN) * WTN;

  // chunk c -> (row, k offset): lanes walk k for k-contiguous operands and
  // rows for row-contiguous ones
  auto a_row = [&](int c) { return AR ? c % BM : c / (BK / 8); };
  auto a_kc = [&](int c) { return AR ? (c / BM) * 8 : (c % (BK / 8)) * 8; };
  auto b_row = [&](int c) { return BR ? c % BN : c / (BK / 8); };
  auto b_kc = [&](int c) { return BR ? (c / BN) * 8 : (c % (BK / 8)) * 8; };

  typename MM::Acc acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = MM::zero();

  // the main loop over K tiles: gload(k0) fetches a tile into registers,
  // sstore(buf) converts and writes it to LDS
  auto mainloop = [&](auto& gload, auto& sstore) {
    const int ntiles = kbeg < kend ? (kend - kbeg + BK - 1) / BK : 0;
    if (ntiles <= 0) return;
    gload(kbeg);
    sstore(0);
    __syncthreads();
    for (int t = 0; t < ntiles; ++t) {
      const int cur = t & 1;
      if (t + 1 < ntiles) gload(kbeg + (t + 1) * BK);
#pragma unroll
      for (int ks = 0; ks < BK; ks += 16) {
        const int ko = ks + MM::kof(lane);
#pragma unroll
        for (int i = 0; i < FM; ++i) {
          const int ao = (wm0 + i * FR + MM::row(lane)) * LDK + ko;
#pragma unroll
          for (int j = 0; j < FN; ++j) {
            const TC* bp = &sB[cur][(wn0 + j * FR + MM::row(lane)) * LDK + ko];
            acc[i][j] = MM::mma(&sA[0][cur][ao], bp, acc[i][j]);
            if (SPLIT) acc[i][j] = MM::mma(&sA[NSPL - 1][cur][ao], bp, acc[i][j]);
          }
        }
      }
      if (t + 1 < ntiles) sstore(cur ^ 1);
      __syncthreads();
    }
  };
  if constexpr (QUADS) {
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    typename Prob::RU ru[QU];
    int uo[QU], uk[QU];  // LDS offset, k offset
    float4 vu[QU][4];
    auto is_a = [&](int q) { return wv + 4 * q < UA / 64; };
    auto live = [&](int q) { return wv + 4 * q < (UA + UB) / 64; };
#pragma unroll
    for (int q = 0; q < QU; ++q) {
      // lanes: 4 row quads (64 bytes of a memory row) by the 8 k groups, so
      // that the stores of 16 (float) or 32 (bfloat16) lanes, whose rows lie
      // 4 LDK apart, cover every LDS bank once
      const int u = tid + 256 * q - (is_a(q) ? 0 : UA);
      const int row = ((u & 3) + (u >> 5) * 4) * 4;
      uk[q] = ((u >> 2) & 7) * 4;
      uo[q] = row * LDK + uk[q];
      ru[q] = is_a(q) ? p.rowA(m0 + row) : p.rowB(live(q) ? n0 + row : 1 << 30);
    }
    auto gload = [&](int k0) {
#pragma unroll
      for (int q = 0; q < QU; ++q) {
        if (is_a(q)) p.a44(ru[q], k0 + uk[q], kend, vu[q]);
        else if (live(q)) p.b44(ru[q], k0 + uk[q], kend, vu[q]);
      }
    };
    auto sstore = [&](int buf) {
#pragma unroll
      for (int q = 0; q < QU; ++q) {
        if (is_a(q)) put44(&sA[0][buf][uo[q]], LDK, vu[q], SPLIT ? &sA[NSPL - 1][buf][uo[q]] : (TC*)nullptr);
        else if (live(q)) put44(&sB[buf][uo[q]], LDK, vu[q], (TC*)nullptr);
      }
    };
    mainloop(gload, sstore);
  } else if constexpr (Layout<Prob>::RT) {
    constexpr int RA_ = BM / 8 * (BK / 2), RB_ = BN / 8 * (BK / 2);  // units of A and B
    constexpr int PA = (RA_ + 255) / 256, PB = (RB_ + 255) / 256;
    auto row = [](int c) { return c / (BK / 2) * 8; };
    auto kc = [](int c) { return c % (BK / 2) * 2; };
    typename Prob::RA ra[PA];
    typename Prob::RB rb[PB];
    float va[PA][2][8], vb[PB][2][8];
#pragma unroll
    for (int q = 0; q < PA; ++q) ra[q] = p.rowA(tid + 256 * q < RA_ ? m0 + row(tid + 256 * q) : 1 << 30);
#pragma unroll
    for (int q = 0; q < PB; ++q) rb[q] = p.rowB(tid + 256 * q < RB_ ? n0 + row(tid + 256 * q) : 1 << 30);
    auto gload = [&](int k0) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int q = 0; q < PA; ++q) {
          const int c = tid + 256 * q, k = k0 + kc(c) + h;
          if (c < RA_ && k < kend) p.a8(ra[q], k, va[q][h]);
          else zero8(va[q][h]);
        }
#pragma unroll
        for (int q = 0; q < PB; ++q) {
          const int c = tid + 256 * q, k = k0 + kc(c) + h;
          if (c < RB_ && k < kend) p.b8(rb[q], k, vb[q][h]);
          else zero8(vb[q][h]);
        }
      }
    };
    auto sstore = [&](int buf) {
#pragma unroll
      for (int q = 0; q < PA; ++q) {
        const int c = tid + 256 * q;
        if (c < RA_) put8t2(&sA[0][buf][row(c) * LDK + kc(c)], LDK, va[q][0], va[q][1]);
      }
#pragma unroll
      for (int q = 0; q < PB; ++q) {
        const int c = tid + 256 * q;
        if (c < RB_) put8t2(&sB[buf][row(c) * LDK + kc(c)], LDK, vb[q][0], vb[q][1]);
      }
    };
    mainloop(gload, sstore);
  } else if constexpr (Layout<Prob>::UNI) {
    typename Prob::RA ra[QA];
    typename Prob::RB rb[QB];
    float va[QA][8];
    Raw8<typename Prob::Weight> vb[QB];
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      const int c = tid + 256 * q;
      ra[q] = p.rowA(c < CA ? m0 + a_row(c) : 1 << 30, a_kc(c));
    }
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const int c = tid + 256 * q;
      rb[q] = p.rowB(c < CB ? n0 + b_row(c) : 1 << 30, b_kc(c));
    }
    auto gload = [&](int k0) {
      const auto kt = p.ktile(k0);
#pragma unroll
      for (int q = 0; q < QA; ++q) p.a8(ra[q], kt, va[q]);
#pragma unroll
      for (int q = 0; q < QB; ++q) p.b8(rb[q], kt, vb[q]);
    };
    auto sstore = [&](int buf) {
#pragma unroll
      for (int q = 0; q < QA; ++q) {
        const int c = tid + 256 * q;
        const int o = a_row(c) * LDK + a_kc(c);
        if (c < CA) put8(&sA[0][buf][o], va[q], SPLIT ? &sA[NSPL - 1][buf][o] : (TC*)nullptr);
      }
#pragma unroll
      for (int q = 0; q < QB; ++q) {
        const int c = tid + 256 * q;
        if (c < CB) put_raw(&sB[buf][b_row(c) * LDK + b_kc(c)], vb[q]);
      }
    };
    mainloop(gload, sstore);
  } else {
    typename Prob::RA ra[QA];
    typename Prob::RB rb[QB];
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      const int c = tid + 256 * q;
      ra[q] = p.rowA(c < CA ? m0 + a_row(c) : 1 << 30);
    }
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const int c = tid + 256 * q;
      rb[q] = p.rowB(c < CB ? n0 + b_row(c) : 1 << 30);
    }
    float va[QA][8], vb[QB][8];
    auto gload = [&](int k0) {
#pragma unroll
      for (int q = 0; q < QA; ++q) {
        const int c = tid + 256 * q;
        const int k = k0 + a_kc(c);
        if (c < CA && k < kend) p.a8(ra[q], k, va[q]);
        else zero8(va[q]);
      }
#pragma unroll
      for (int q = 0; q < QB; ++q) {
        const int c = tid + 256 * q;
        const int k = k0 + b_kc(c);
        if (c < CB && k < kend) p.b8(rb[q], k, vb[q]);
        else zero8(vb[q]);
      }
    };
    auto sstore = [&](int buf) {
#pragma unroll
      for (int q = 0; q < QA; ++q) {
        const int c = tid + 256 * q;
        const int o = a_row(c) * LDK + a_kc(c);
        if (c < CA) put8(&sA[0][buf][o], va[q], SPLIT ? &sA[NSPL - 1][buf][o] : (TC*)nullptr);
      }
#pragma unroll
      for (int q = 0; q < QB; ++q) {
        const int c = tid + 256 * q;
        if (c < CB) put8(&sB[buf][b_row(c) * LDK + b_kc(c)], vb[q], (TC*)nullptr);
      }
    };
    mainloop(gload, sstore);
  }

  if (e.gm_p > 0 && (e.partial || !e.gm_split_only)) {
    // group-major stores (plain values): the image and pixel of the fragment's
    // first row once, later rows step from it
    float* dst = e.partial ? e.partial + (size_t)blockIdx.y * p.M * p.N : e.C;
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int n = n0 + wn0 + j * FR + MM::ocol(lane);
      if (n >= p.N) continue;
      const int g = n / e.gm_cg, cc = n - g * e.gm_cg, G = p.N / e.gm_cg;
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        const int mb = m0 + wm0 + i * FR;
        const int b0 = mb / e.gm_p, pb = mb - b0 * e.gm_p;
#pragma unroll
        for (int r = 0; r < MM::NOUT; ++r) {
          const int m = mb + MM::orow(lane, r);
          if (m < p.M) {
            int b = b0, px = pb + MM::orow(lane, r);
            if (px >= e.gm_p) {  // the fragment crosses into later images
              const int q = px / e.gm_p;
              b += q;
              px -= q * e.gm_p;
            }
            dst[(((size_t)b * G + g) * e.gm_p + px) * e.gm_cg + cc] = acc[i][j][r];
          }
        }
      }
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int n = n0 + wn0 + j * FR + MM::ocol(lane);
#pragma unroll
      for (int r = 0; r < MM::NOUT; ++r) {
        const int m = m0 + wm0 + i * FR + MM::orow(lane, r);
        if (m < p.M && n < p.N) {
          float v = acc[i][j][r];
          if (e.partial) {
            e.partial[((size_t)blockIdx.y * p.M + m) * p.N + n] = v;
          } else {
            v *= e.alpha;
            float* cp = e.C + crow(e, m) * e.ldc + n;
            if (e.accumulate) v += *cp;
            if (e.bias) v += e.bias[n];
            if (e.relu) v = fmaxf(v, 0.f);
            *cp = v;
          }
        }
      }
    }
}

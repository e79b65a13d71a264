// The per-atom layers of a small batch, spread over the chip.
//
// The fused update kernels give a workgroup 16 or 32 atoms and every layer of
// the block: with a handful of atoms a handful of CUs stream all the weights
// (8.8 MB per layer in FP32 at F = 384) one after the other, 130 to 180 us per
// launch whatever the batch.  Here each dense layer is a launch of its own
// whose workgroup takes 16 atoms x 16 output features, its 4 waves a quarter
// of the contraction each (summed through LDS in wave order); activations go
// through memory between launches.  A block of 5 such launches (3 in reverse)
// takes about 6 us each, until there are enough atoms that the fused kernels'
// weight reuse wins: small_rows() draws the line.
#pragma once

#include "mfma.h"

namespace rows {

// Whether a batch of N atoms takes this form, forward or reverse, as measured
// (whole calls, us, fused -> this form; energies for the forward).
//  FP32 F = 384: 1,152 atoms 465 -> 385, 1,536 467 -> 453, 2,304 512 -> 597;
//   F = 256: 1,536 1,656 -> 1,273, 2,304 2,131 -> 1,940; F = 128: 1,536 350 ->
//   294, 2,304 383 -> 366; F = 64: 768 174 -> 170, 1,536 176 -> 171, 2,304 184
//   -> 193 (from 768 on the two are within 3 %).
//  FP64 F = 384: 1,152 738 -> 668, 1,536 740 -> 785; F = 256: 1,152 1,820 ->
//   1,764, 1,536 1,823 -> 1,898; F = 128: 768 514 -> 488, 1,152 536 -> 551; F =
//   64: 1,152 264 -> 236, 2,304 276 -> 268.
// In reverse the element-wise operands are formed once per 16 features, so the
// line lies lower (forces calls with the forward in its own form):
//  FP32 F = 384: 96 864 -> 626, 384 918 -> 863, 576 948 -> 989.
//  FP64 F = 384: 96 1,233 -> 954, 288 1,281 -> 1,274, 384 1,414 -> 1,514; F =
//   256: both passes gain 820 us at 240 atoms and 415 at 384, the forward alone
//   567 and 450; below F = 256 the fused kernels win from the start.
// A structure's last bits depend on the form, so on the batch it is in.
template <class P, int F>
inline bool small_rows(int N, bool reverse) {
  if (P::PREC == PAINN_BF16) return false;
  if (P::PREC == PAINN_FP32) return N <= (reverse ? (F >= 128 ? 384 : 0) : F >= 128 ? 1536 : 768);
  return N <= (reverse ? (F >= 256 ? 240 : 0) : F == 128 ? 768 : 1152);
}

struct Args {
  int N;
  DenseDev d0, d1;
  // forward: v, s after the message; U [N][3][us]; |V|, <U, V> and a hidden
  // layer [N][F] each
  const void *s, *v;
  void *s_out, *v_out, *h;
  void *U, *nrm, *pd, *hid;
  int us;                        // elements between the components of U
  void *save_uv, *save_z, *save_a;   // or null
  // reverse (names as in the fused kernels); gz, t: [N] rows of `ts` elements
  const void *uv, *z, *ag, *gs, *gv, *gh, *gm;
  void *gs_out, *gv_out, *gn, *t;
  int sw, ts;
};

enum Op { UV, GATE1, GATE2, PHI1, PHI2, B_GATE2, B_GATE1, B_UV, B_PHI2, B_PHI1 };

template <class A>
__device__ __forceinline__ A dsilu1(A x) {
  const A sg = A(1) / (A(1) + (sizeof(A) == 8 ? (A)exp((double)-x) : (A)expf((float)-x)));
  return sg * (A(1) + x * (A(1) - sg));
}

// KPL consecutive values as one load, and as an operand fragment.
template <class T, int N>
struct alignas(N * sizeof(T)) Vec {
  T x[N];
};

template <class P, int F, int OP>
__global__ void __launch_bounds__(256) k_rows(Args a) {
  using D = dense_t<P>;
  using T = typename P::T;
  using A = typename P::A;
  using C = typename P::C;
  using Fr = typename D::Fr;
  constexpr int KPL = D::KPL, KC = D::KC, NFT = F / 16;
  using Vt = Vec<T, KPL>;
  // accumulator tiles, and k-blocks per wave of the (first) contraction
  constexpr int NT = OP == UV ? 6 : OP == GATE2 ? 3 : OP == B_PHI2 ? 2 : 1;
  constexpr int KW = OP == GATE1 || OP == B_UV ? 2 * F : OP == B_GATE2 ? 3 * F : F;
  constexpr int NKB = KW / KC, PW = NKB / 4;
  static_assert(NKB % 4 == 0, "a quarter of the contraction per wave");
  __shared__ A part[4][NT][256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, q = lane >> 4;
  const int t = blockIdx.x, ft = blockIdx.y;
  // B_UV's rows are (atom, component); rows past the end read the last one
  const int rows = OP == B_UV ? 3 * a.N : a.N;
  const size_t r = min(t * 16 + (lane & 15), rows - 1);
  C acc[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n)
    for (int i = 0; i < 4; ++i) acc[n][i] = 0;
  auto ld = [](const void* p, size_t o) { return *(const Vt*)((const T*)p + o); };
  auto fr = [](const Vt& v) {
    Fr f;
    __builtin_memcpy(&f, &v, sizeof(f));
    return f;
  };
  auto wfrag = [&](const DenseDev& L, int ct, int nkb, int kb) {
    return D::frag((const T*)L.w + (((size_t)ct * nkb + kb) * 64 + lane) * KPL);
  };
  constexpr int UN = PW <= 8 ? PW : 6;
#pragma unroll UN
  for (int x = 0; x < PW; ++x) {
    const int kb = wave * PW + x, k = kb * KC + q * KPL;
    if constexpr (OP == UV) {
      const Fr wu = wfrag(a.d0, ft, NKB, kb), wv = wfrag(a.d0, NFT + ft, NKB, kb);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const Fr f = fr(ld(a.v, (3 * r + c) * F + k));
        acc[c] = D::mfma(f, wu, acc[c]);
        acc[3 + c] = D::mfma(f, wv, acc[3 + c]);
      }
    } else if constexpr (OP == GATE2) {
      const Fr f = fr(ld(a.hid, r * F + k));
#pragma unroll
      for (int n = 0; n < 3; ++n) acc[n] = D::mfma(f, wfrag(a.d0, n * NFT + ft, NKB, kb), acc[n]);
    } else if constexpr (OP == B_PHI2) {
      acc[0] = D::mfma(fr(ld(a.s, r * F + k)), wfrag(a.d0, ft, NKB, kb), acc[0]);
#pragma unroll
      for (int n = 0; n < 3; ++n)
        acc[1] = D::mfma(fr(ld(a.gh, r * 3 * F + n * F + k)), wfrag(a.d1, ft, 3 * NKB, n * NKB + kb), acc[1]);
    } else {
      Vt v;
      if constexpr (OP == GATE1) {
        v = k < F ? ld(a.s, r * F + k) : ld(a.nrm, r * F + k - F);
      } else if constexpr (OP == PHI1) {
        v = ld(a.s, r * F + k);
      } else if constexpr (OP == PHI2) {
        v = ld(a.hid, r * F + k);
      } else if constexpr (OP == B_GATE1 || OP == B_PHI1) {
        v = ld(a.t, r * a.ts + k);
      } else if constexpr (OP == B_GATE2) {
        // g_a = [sum_c g_v U | g_s <U, V> | g_s]
        const int f = k % F, sec = k / F;
        for (int e = 0; e < KPL; ++e) v.x[e] = T(0);
        if (sec < 2)
          for (int c = 0; c < 3; ++c) {
            const Vt u = ld(a.uv, (r * 3 + c) * 2 * F + f);
            const Vt w = sec ? ld(a.uv, (r * 3 + c) * 2 * F + F + f) : ld(a.gv, r * 3 * F + c * F + f);
            for (int e = 0; e < KPL; ++e) v.x[e] += u.x[e] * w.x[e];
          }
        if (sec) {
          const Vt g = ld(a.gs, r * F + f);
          for (int e = 0; e < KPL; ++e) v.x[e] = sec == 1 ? v.x[e] * g.x[e] : g.x[e];
        }
      } else {
        // B_UV: g_U = g_v a_vv + g_s a_sv V; g_V = g_s a_sv U + (g_n / |V|) V
        const size_t i = r / 3, c = r % 3;
        const int f = k % F;
        const Vt w = ld(a.uv, r * 2 * F + F + f), g = ld(a.gs, i * F + f), asv = ld(a.ag, i * 2 * F + F + f);
        if (k < F) {
          const Vt gvc = ld(a.gv, i * 3 * F + c * F + f), avv = ld(a.ag, i * 2 * F + f);
          for (int e = 0; e < KPL; ++e) v.x[e] = gvc.x[e] * avv.x[e] + g.x[e] * asv.x[e] * w.x[e];
        } else {
          const Vt u = ld(a.uv, r * 2 * F + f);
          const Vt v0 = ld(a.uv, (3 * i) * 2 * F + F + f), v1 = ld(a.uv, (3 * i + 1) * 2 * F + F + f),
                   v2 = ld(a.uv, (3 * i + 2) * 2 * F + F + f);
          for (int e = 0; e < KPL; ++e) {
            const A nv = sqrt(v0.x[e] * v0.x[e] + v1.x[e] * v1.x[e] + v2.x[e] * v2.x[e]);
            const A gn = ((const A*)a.gn)[i * a.sw + f + e];
            v.x[e] = g.x[e] * asv.x[e] * u.x[e] + (nv > A(0) ? gn * w.x[e] / nv : A(0));
          }
        }
      }
      acc[0] = D::mfma(fr(v), wfrag(a.d0, ft, NKB, kb), acc[0]);
    }
  }
#pragma unroll
  for (int n = 0; n < NT; ++n)
#pragma unroll
    for (int i = 0; i < 4; ++i) part[wave][n][P::row(lane, i) * 16 + (lane & 15)] = acc[n][i];
  __syncthreads();
  const int x = threadIdx.x, col = ft * 16 + (x & 15);
  const size_t row = t * 16 + (x >> 4);
  if (row >= (size_t)rows) return;
  A y[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n) y[n] = ((part[0][n][x] + part[1][n][x]) + part[2][n][x]) + part[3][n][x];
  if constexpr (OP == UV) {
    A n2 = 0, pd = 0;
    for (int c = 0; c < 3; ++c) {
      n2 += y[3 + c] * y[3 + c];
      pd += y[c] * y[3 + c];
      ((T*)a.U)[(row * 3 + c) * a.us + col] = P::st(y[c]);
      if (a.save_uv) {
        T* o = (T*)a.save_uv + (row * 3 + c) * 2 * F;
        o[col] = P::st(y[c]);
        o[F + col] = P::st(y[3 + c]);
      }
    }
    ((T*)a.nrm)[row * F + col] = P::st(sqrt(n2));
    ((A*)a.pd)[row * F + col] = pd;
  } else if constexpr (OP == GATE1) {
    const A z = y[0] + ((const A*)a.d0.b)[col];
    ((T*)a.hid)[row * F + col] = P::st(silu<A>(z));
    if (a.save_z) ((T*)a.save_z)[row * F + col] = P::st(z);
  } else if constexpr (OP == GATE2) {
    const A* b = (const A*)a.d0.b;
    const A gvv = y[0] + b[col], gsv = y[1] + b[F + col], gss = y[2] + b[2 * F + col];
    if (a.save_a) {
      ((T*)a.save_a)[row * 2 * F + col] = P::st(gvv);
      ((T*)a.save_a)[row * 2 * F + F + col] = P::st(gsv);
    }
    ((T*)a.s_out)[row * F + col] =
        P::st(P::ld(((const T*)a.s)[row * F + col]) + gsv * ((const A*)a.pd)[row * F + col] + gss);
    for (int c = 0; c < 3; ++c) {
      const size_t o = row * 3 * F + c * F + col;
      ((T*)a.v_out)[o] = P::st(P::ld(((const T*)a.v)[o]) + gvv * P::ld(((const T*)a.U)[(row * 3 + c) * a.us + col]));
    }
  } else if constexpr (OP == PHI1) {
    ((T*)a.hid)[row * F + col] = P::st(silu<A>(y[0] + ((const A*)a.d0.b)[col]));
  } else if constexpr (OP == PHI2) {
    ((T*)a.h)[row * 3 * F + col] = P::st(y[0] + ((const A*)a.d0.b)[col]);
  } else if constexpr (OP == B_GATE2) {
    ((A*)a.t)[row * a.ts + col] = y[0] * dsilu1<A>(((const A*)a.z)[row * F + col]);
  } else if constexpr (OP == B_GATE1) {
    if (col < F) ((A*)a.gs_out)[row * F + col] = ((const A*)a.gs)[row * F + col] + y[0];
    else ((A*)a.gn)[row * a.sw + col - F] = y[0];
  } else if constexpr (OP == B_UV) {
    ((A*)a.gv_out)[row * F + col] = ((const A*)a.gv)[row * F + col] + y[0];
  } else if constexpr (OP == B_PHI2) {
    ((A*)a.t)[row * a.ts + col] = y[1] * dsilu1<A>(y[0] + ((const A*)a.d0.b)[col]);
  } else {
    ((A*)a.gs_out)[row * F + col] = ((const A*)a.gm)[row * F + col] + y[0];
  }
}

template <class P, int F, int OP>
void launch(hipStream_t st, const Args& a) {
  const int rows = OP == B_UV ? 3 * a.N : a.N;
  const int cols = OP == PHI2 ? 3 * F : OP == B_GATE1 ? 2 * F : F;
  k_rows<P, F, OP><<<dim3((unsigned)((rows + 15) / 16), (unsigned)(cols / 16)), 256, 0, st>>>(a);
}

}  // namespace rows

// Wide branch layers of the heads (the lead model's 776-wide branches),
// forward and reverse, as matrix products over tiles of rows of one head.
//
// A row is one (atom, head) entry of the heads' grouping (k_head_*).  Per
// branch layer one launch of k_branch runs out[row][feature] over tiles of
// 128 rows (32 where rows are few) x 128 or 160 features; activations go
// between launches through a scratch in HBM in the operand layout of
// branchgemm.h, and the launches of one chunk of tiles share that scratch.
// With gradients the reverse products follow in the same chunk (they reuse
// the stored pre-activations) and leave dE/dY per entry, Y being the shared
// layers' output.
//
// Why not one kernel per tile with its activations in LDS: a 776-wide layer's
// weights are 2.4 MB in FP32 (4.8 MB in FP64).  Tiles of 16 to 64 rows, all
// that fits the LDS, re-read them from L2 for 16 to 64 rows at a time: the
// lead model's blended reverse heads ran at 0.17 (FP64) and 0.36 (FP32) of
// the matrix cores' peak.  With 128 rows x 160 features per workgroup each
// byte staged in LDS feeds 128 to 160 products, and the pre-activations are
// formed once instead of once forward and once in reverse.  FP32 products run
// on the BF16 matrix cores over three planes of each operand (branchgemm.h,
// also for what they do with infinities and the smallest values): the six
// products of order 2^-16 and above of the nine (the rest are below FP32's
// rounding), 96 cycles per 16x16x32 against 256 for the FP32 instruction.
#include "branchgemm.h"
#include "mfma.h"

namespace {

typedef double dd2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u2_t __attribute__((ext_vector_type(2)));

template <class A>
__device__ __forceinline__ A dsilu_(A x) {
  const A sg = A(1) / (A(1) + (sizeof(A) == 8 ? (A)exp((double)-x) : (A)expf((float)-x)));
  return sg * (A(1) + x * (A(1) - sg));
}

template <class P> struct Op;
template <> struct Op<PB16> {
  static constexpr int NP = 1, KB = 32, NSUB = 1;
  using Fr = bf8_t;
  __device__ static __forceinline__ f4_t mma(const Fr* a, const Fr* b, f4_t c, int) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[0], c, 0, 0, 0);
  }
};
template <> struct Op<P32> {
  static constexpr int NP = 3, KB = 32, NSUB = 6;
  using Fr = bf8_t;
  // smallest products first: lo hi, mid mid, hi lo, mid hi, hi mid, hi hi
  __device__ static __forceinline__ f4_t mma(const Fr* a, const Fr* b, f4_t c, int j) {
    constexpr int pa[6] = {2, 1, 0, 1, 0, 0}, pb[6] = {0, 1, 2, 0, 1, 0};
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[pa[j]], b[pb[j]], c, 0, 0, 0);
  }
};
template <> struct Op<P64> {
  static constexpr int NP = 1, KB = 8, NSUB = 2;
  using Fr = dd2_t;
  __device__ static __forceinline__ d4_t mma(const Fr* a, const Fr* b, d4_t c, int j) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a[0][j], b[0][j], c, 0, 0, 0);
  }
};

// Four consecutive features (f, f % 4 == 0) of row `row` of an operand
// buffer of nkb k-blocks.
template <class P>
__device__ __forceinline__ void store_op4(void* buf, int nkb, int row, int f, const typename P::A* x) {
  using O = Op<P>;
  constexpr int KPL = O::KB / 4;
  const size_t blk = ((size_t)(row >> 4) * nkb + f / O::KB) * O::NP * 1024;
  const int q = (f % O::KB) / KPL;
  char* d = (char*)buf + blk + (16 * q + (row & 15)) * 16;
  if constexpr (P::PREC == PAINN_FP64) {
    *(dd2_t*)d = dd2_t{x[0], x[1]};
    *(dd2_t*)(d + 256) = dd2_t{x[2], x[3]};
  } else {
    d += (f & 4) * 2;
    if constexpr (O::NP == 3) {
      uint32_t p[4][3];
#pragma unroll
      for (int i = 0; i < 4; ++i) split3(x[i], p[i]);
#pragma unroll
      for (int k = 0; k < 3; ++k)
        *(u2_t*)(d + 1024 * k) = u2_t{(p[0][k] >> 16) | p[1][k], (p[2][k] >> 16) | p[3][k]};
    } else {
      const uint32_t b0 = f_to_bf16(x[0]), b1 = f_to_bf16(x[1]), b2 = f_to_bf16(x[2]), b3 = f_to_bf16(x[3]);
      *(u2_t*)d = u2_t{b0 | (b1 << 16), b2 | (b3 << 16)};
    }
  }
}

enum { EPI_HIDDEN = 0, EPI_LAST = 1, EPI_BACK = 2, EPI_OUT = 3 };

struct GemmArgs {
  int tile0, tiles;              // this chunk's tiles [tile0, tile0 + tiles)
  int N;                         // without tiles: rows [TM t, N), head 0
  int nft, nkb, nfb;             // feature tiles (16), k-blocks, feature blocks of the grid
  const HeadTile* tl;
  const HeadPlan* plan;
  const int32_t* order;          // atom of each entry (null: the row itself)
  const void* const* table;      // [head][stride] pointers
  int stride, iw, ib, io;        // weights, bias, output layer's weights in a head's entry
  const void* in;                // EPI 0/1 first layer: Y [N][planes][KY]; else operand blocks
  int ky;                        // row width of Y (elements)
  void* out;                     // operand blocks of the result
  int nkb_out;
  void* z;                       // pre-activations in accumulator layout
  int nft_z;
  void* part;                    // [nft][slots] partial energies (EPI_LAST)
  size_t slots;
  void* dy;                      // EPI_OUT: dE/dY, [atom (* H + head)][KY]
  int H;                         // > 0: one row per (atom, head)
};

// One workgroup (4 waves, 2 feature halves x 2 row halves) of FTW x RTW 16x16
// tiles per wave.  Per k-block both operands' blocks go through LDS; the next
// k-block's are loaded into registers meanwhile, and two workgroups per CU
// overlap one's barriers and epilogue with the other's products.
template <class P, int FTW, int RTW, int EPI, bool FIRST, bool GRAD>
__global__ void __launch_bounds__(256, 2) k_branch(GemmArgs a) {
  using O = Op<P>;
  using A = typename P::A;
  using C = typename P::C;
  using Fr = typename O::Fr;
  constexpr int NP = O::NP, TM = 32 * RTW;
  constexpr int UA = 2 * FTW * NP * 64, UB = 2 * RTW * NP * 64;       // 16-byte units per k-block
  constexpr int NA = (UA + 255) / 256, NB = (UB + 255) / 256;
  __shared__ __attribute__((aligned(16))) u4_t As[UA], Bs[UB];
  __shared__ int rows[TM];
  // the feature blocks of a row tile on one XCD, next to each other: its
  // activations are read from that L2
  const int xcd = blockIdx.x % 8, lin = blockIdx.x / 8;
  const int t = (lin / a.nfb) * 8 + xcd, fb = lin % a.nfb;
  if (t >= a.tiles) return;
  int head = 0, begin, end;
  if (a.tl) {
    if (a.tile0 + t >= a.plan->n_tiles) return;
    const HeadTile h = a.tl[a.tile0 + t];
    head = h.head;
    begin = h.begin;
    end = h.end;
  } else {
    begin = (a.tile0 + t) * TM;
    end = min(a.N, begin + TM);
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wf = wave & 1, wr = wave >> 1;
  if (FIRST || EPI == EPI_OUT) {
    if (tid < TM) {
      const int k = begin + tid;
      rows[tid] = k < end ? (a.order ? a.order[k] : k) : -1;
    }
    __syncthreads();
  }
  const void* const* tab = a.table + (size_t)head * a.stride;
  const u4_t* W = (const u4_t*)tab[a.iw];
  const u4_t* X = (const u4_t*)a.in;
  const int row0 = t * TM;                // first slot of the tile in the chunk's scratch
  const int ft0 = fb * 2 * FTW;
  u4_t ra[NA], rb[NB];
  // this thread's unit u of a k-block: block u / 64 (tile-major, plane), lane u % 64
  auto load = [&](int kb) {
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int u = tid + 256 * i, b = u >> 6, ft = ft0 + b / NP;
      ra[i] = u4_t{0, 0, 0, 0};
      if (u < UA && ft < a.nft) ra[i] = W[(((size_t)ft * a.nkb + kb) * NP + b % NP) * 64 + lane];
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int u = tid + 256 * i, b = u >> 6;
      rb[i] = u4_t{0, 0, 0, 0};
      if (u < UB) {
        if constexpr (FIRST) {
          const int r = rows[(b / NP) * 16 + (lane & 15)];
          constexpr int EPU = O::KB / 4;
          if (r >= 0) rb[i] = X[((size_t)r * NP + b % NP) * (a.ky / EPU) + kb * 4 + (lane >> 4)];
        } else {
          rb[i] = X[((((size_t)(row0 >> 4) + b / NP) * a.nkb + kb) * NP + b % NP) * 64 + lane];
        }
      }
    }
  };
  C acc[FTW][RTW];
#pragma unroll
  for (int f = 0; f < FTW; ++f)
#pragma unroll
    for (int r = 0; r < RTW; ++r)
      for (int i = 0; i < 4; ++i) acc[f][r][i] = 0;
  load(0);
  for (int kb = 0; kb < a.nkb; ++kb) {
    if (kb) __syncthreads();
#pragma unroll
    for (int i = 0; i < NA; ++i)
      if (UA % 256 == 0 || tid + 256 * i < UA) As[tid + 256 * i] = ra[i];
#pragma unroll
    for (int i = 0; i < NB; ++i)
      if (UB % 256 == 0 || tid + 256 * i < UB) Bs[tid + 256 * i] = rb[i];
    __syncthreads();
    if (kb + 1 < a.nkb) load(kb + 1);
    Fr bf[RTW][NP];
#pragma unroll
    for (int r = 0; r < RTW; ++r)
#pragma unroll
      for (int p = 0; p < NP; ++p) bf[r][p] = *(const Fr*)&Bs[((wr * RTW + r) * NP + p) * 64 + lane];
#pragma unroll
    for (int f = 0; f < FTW; ++f) {
      Fr af[NP];
#pragma unroll
      for (int p = 0; p < NP; ++p) af[p] = *(const Fr*)&As[((wf * FTW + f) * NP + p) * 64 + lane];
      if constexpr (NP == 3) {
        // a k-block's six products are summed apart and added once.  Added to
        // the running sum one by one they left energies 5 % further from 64
        // bits than the FP32 instructions; so, 5 to 18 % nearer (lead model
        // blended forces, 712 structures: 23.2 -> 23.5 ms)
        C part[RTW];
#pragma unroll
        for (int r = 0; r < RTW; ++r)
          for (int i = 0; i < 4; ++i) part[r][i] = 0;
#pragma unroll
        for (int j = 0; j < O::NSUB; ++j)
#pragma unroll
          for (int r = 0; r < RTW; ++r) part[r] = O::mma(af, bf[r], part[r], j);
#pragma unroll
        for (int r = 0; r < RTW; ++r)
          for (int i = 0; i < 4; ++i) acc[f][r][i] += part[r][i];
      } else {
#pragma unroll
        for (int j = 0; j < O::NSUB; ++j)
#pragma unroll
          for (int r = 0; r < RTW; ++r) acc[f][r] = O::mma(af, bf[r], acc[f][r], j);
      }
    }
  }
  // a lane holds features 16 ft + 4 (lane / 16) + i of row lane % 16 of a tile
#pragma unroll
  for (int f = 0; f < FTW; ++f) {
    const int ft = ft0 + wf * FTW + f;
    if (ft >= a.nft) continue;
    const int feat = 16 * ft + 4 * (lane >> 4);
    A bias[4], wo[4];
    if constexpr (EPI == EPI_HIDDEN || EPI == EPI_LAST) {
      const Quad<A> q = *(const Quad<A>*)((const A*)tab[a.ib] + feat);
      for (int i = 0; i < 4; ++i) bias[i] = q.x[i];
    }
    if constexpr (EPI == EPI_LAST) {
      const Quad<A> q = *(const Quad<A>*)((const A*)tab[a.io] + feat);
      for (int i = 0; i < 4; ++i) wo[i] = q.x[i];
    }
#pragma unroll
    for (int r = 0; r < RTW; ++r) {
      const int rl = (wr * RTW + r) * 16 + (lane & 15);   // row of the tile
      const int slot = row0 + rl;
      Quad<A>* zq = (Quad<A>*)a.z + ((size_t)(slot >> 4) * a.nft_z + ft) * 64 + lane;
      A x[4];
      if constexpr (EPI == EPI_HIDDEN) {
        Quad<A> zz;
        for (int i = 0; i < 4; ++i) {
          zz.x[i] = acc[f][r][i] + bias[i];
          x[i] = silu<A>(zz.x[i]);
        }
        if constexpr (GRAD) *zq = zz;
        store_op4<P>(a.out, a.nkb_out, slot, feat, x);
      } else if constexpr (EPI == EPI_LAST) {
        // the output layer's dot product, per tile of 16 features in a fixed
        // order (the same for every tile shape)
        A y = 0;
        for (int i = 0; i < 4; ++i) {
          const A z = acc[f][r][i] + bias[i];
          y += silu<A>(z) * wo[i];
          x[i] = wo[i] * dsilu_<A>(z);
        }
        y += __shfl_xor(y, 16);
        y += __shfl_xor(y, 32);
        if (lane < 16) ((A*)a.part)[(size_t)ft * a.slots + slot] = y;
        if constexpr (GRAD) store_op4<P>(a.out, a.nkb_out, slot, feat, x);
      } else if constexpr (EPI == EPI_BACK) {
        const Quad<A> zz = *zq;
        for (int i = 0; i < 4; ++i) x[i] = acc[f][r][i] * dsilu_<A>(zz.x[i]);
        store_op4<P>(a.out, a.nkb_out, slot, feat, x);
      } else {
        const int g = rows[rl];
        if (g >= 0) {
          Quad<A> o;
          for (int i = 0; i < 4; ++i) o.x[i] = acc[f][r][i];
          *(Quad<A>*)((A*)a.dy + ((size_t)g * (a.H ? a.H : 1) + (a.H ? head : 0)) * a.ky + feat) = o;
        }
      }
    }
  }
}

// Energies of a chunk's entries: the partial sums in feature order, then the
// output layer's bias.
template <class A>
__global__ void __launch_bounds__(256) k_branch_out(GemmArgs a, int TM, void* e, void* eh) {
  const int x = blockIdx.x * 256 + threadIdx.x, t = x / TM, r = x % TM;
  if (t >= a.tiles) return;
  int head = 0, begin, end;
  if (a.tl) {
    if (a.tile0 + t >= a.plan->n_tiles) return;
    const HeadTile h = a.tl[a.tile0 + t];
    head = h.head;
    begin = h.begin;
    end = h.end;
  } else {
    begin = (a.tile0 + t) * TM;
    end = min(a.N, begin + TM);
  }
  if (begin + r >= end) return;
  const int atom = a.order ? a.order[begin + r] : begin + r;
  A y = 0;
#pragma unroll 10
  for (int f = 0; f < a.nft; ++f) y += ((const A*)a.part)[(size_t)f * a.slots + x];
  y += ((const A*)a.table[(size_t)head * a.stride + a.ib])[0];
  if (eh) ((A*)eh)[(size_t)atom * a.H + head] = y;
  else ((A*)e)[atom] = y;
}

template <class P, int FTW, int RTW, int EPI, bool FIRST, bool GRAD>
void launch_one(hipStream_t st, GemmArgs a) {
  a.nfb = (a.nft + 2 * FTW - 1) / (2 * FTW);
  const unsigned grid = (unsigned)((a.tiles + 7) / 8 * 8) * (unsigned)a.nfb;
  k_branch<P, FTW, RTW, EPI, FIRST, GRAD><<<grid, 256, 0, st>>>(a);
}

// Feature tiles per wave: 4 (128 features per workgroup) or 5 (160) by which
// pads less; 2 (64) for narrow results and for tiles of 32 rows.
template <class P, int EPI, bool FIRST, bool GRAD>
void launch_gemm(hipStream_t st, const GemmArgs& a, bool small) {
  if (small) return launch_one<P, 2, 1, EPI, FIRST, GRAD>(st, a);
  if (a.nft <= 4) return launch_one<P, 2, 4, EPI, FIRST, GRAD>(st, a);
  if ((a.nft + 9) / 10 * 10 < (a.nft + 7) / 8 * 8) return launch_one<P, 5, 4, EPI, FIRST, GRAD>(st, a);
  return launch_one<P, 4, 4, EPI, FIRST, GRAD>(st, a);
}

template <class P, bool GRAD>
hipError_t branch_impl(hipStream_t st, const BranchArgs& b) {
  using A = typename P::A;
  using O = Op<P>;
  const PrecModel* pm = b.pm;
  const std::vector<int>& bd = *b.branch_dims;
  const int nb = (int)bd.size(), nh = nb - 1;      // hidden branch layers
  const int TM = b.small ? BRANCH_TM_SMALL : BRANCH_TM;
  const size_t tile_bytes = branch_tile_bytes(P::PREC, bd, GRAD, b.small);
  const long long cap = (long long)(b.scratch_bytes / tile_bytes);
  if (cap < 1) return hipErrorInvalidValue;
  GemmArgs g{};
  g.N = b.N;
  g.tl = b.tiles;
  g.plan = b.plan;
  g.order = b.order;
  g.table = (const void* const*)pm->branch_table;
  g.stride = pm->branch_stride;
  g.ky = b.ky;
  g.H = b.eh ? b.H : 0;
  int wmax = 0;
  for (int m = 0; m < nh; ++m) wmax = wmax > pad32(bd[m]) ? wmax : pad32(bd[m]);
  for (long long t0 = 0; t0 < b.max_tiles; t0 += cap) {
    const long long nt = b.max_tiles - t0 < cap ? b.max_tiles - t0 : cap;
    const size_t slots = (size_t)nt * TM;
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    char* p = (char*)b.scratch;
    void* ob[2] = {nullptr, nullptr};
    const int nob = branch_op_buffers(nh, GRAD);
    for (int k = 0; k < nob; ++k) {
      ob[k] = p;
      p += al(slots * branch_row_bytes(P::PREC, wmax));
    }
    void* part = p;
    p += al(slots * (pad32(bd[nh - 1]) / 16) * sizeof(A));
    void* z[16];
    for (int m = 0; m + 1 < nh; ++m) {
      z[m] = p;
      if (GRAD) p += al(slots * pad32(bd[m]) * sizeof(A));
    }
    g.tile0 = (int)t0;
    g.tiles = (int)nt;
    g.slots = slots;
    int cur = 0;
    const void* in = b.y;
    int kin = b.ky;
    for (int m = 0; m < nh; ++m) {
      GemmArgs a = g;
      a.nft = pad32(bd[m]) / 16;
      a.nkb = kin / O::KB;
      a.iw = 4 * m;
      a.ib = 4 * m + 1;
      a.in = in;
      a.out = nob ? ob[cur] : nullptr;
      a.nkb_out = pad32(bd[m]) / O::KB;
      a.nft_z = a.nft;
      if (m + 1 < nh) {
        a.z = z[m];
        if (m == 0) launch_gemm<P, EPI_HIDDEN, true, GRAD>(st, a, b.small);
        else launch_gemm<P, EPI_HIDDEN, false, GRAD>(st, a, b.small);
      } else {
        a.io = 4 * (nb - 1) + 3;
        a.part = part;
        if (m == 0) launch_gemm<P, EPI_LAST, true, GRAD>(st, a, b.small);
        else launch_gemm<P, EPI_LAST, false, GRAD>(st, a, b.small);
      }
      in = a.out;
      kin = pad32(bd[m]);
      cur ^= 1;
    }
    GemmArgs o = g;
    o.nft = pad32(bd[nh - 1]) / 16;
    o.part = part;
    o.ib = 4 * (nb - 1) + 1;
    o.H = b.H;
    k_branch_out<A><<<(unsigned)((slots + 255) / 256), 256, 0, st>>>(o, TM, b.e, b.eh);
    if constexpr (GRAD) {
      for (int m = nh - 1; m >= 0; --m) {
        // dE/d(layer m's input) from dE/dz_m, by the transposed weights
        GemmArgs a = g;
        a.iw = 4 * m + 2;
        a.nkb = pad32(bd[m]) / O::KB;
        a.in = in;
        if (m > 0) {
          a.nft = a.nft_z = pad32(bd[m - 1]) / 16;
          a.z = z[m - 1];
          a.out = ob[cur];
          a.nkb_out = pad32(bd[m - 1]) / O::KB;
          launch_gemm<P, EPI_BACK, false, GRAD>(st, a, b.small);
          in = a.out;
          cur ^= 1;
        } else {
          a.nft = b.ky / 16;
          a.dy = b.dy;
          launch_gemm<P, EPI_OUT, false, GRAD>(st, a, b.small);
        }
      }
    }
  }
  return hipGetLastError();
}

// Y in operand form from plain rows (no shared layers: Y = s).
template <class P>
__global__ void __launch_bounds__(256) k_branch_rows(int N, int F, const typename P::T* __restrict__ s,
                                                     void* __restrict__ y) {
  using T = typename P::T;
  constexpr int NP = Op<P>::NP;
  const size_t tot = (size_t)N * F;
  for (size_t x = blockIdx.x * (size_t)blockDim.x + threadIdx.x; x < tot; x += (size_t)gridDim.x * blockDim.x) {
    if constexpr (NP == 3) {
      const size_t i = x / F, c = x % F;
      uint32_t p[3];
      split3((float)s[x], p);
      for (int k = 0; k < 3; ++k) ((bf16_t*)y)[(i * 3 + k) * F + c] = (bf16_t)(p[k] >> 16);
    } else {
      ((T*)y)[x] = s[x];
    }
  }
}

}  // namespace

int branch_op_buffers(int nh, bool grad) { return grad ? 2 : nh > 2 ? 2 : nh > 1 ? 1 : 0; }

size_t branch_tile_bytes(int prec, const std::vector<int>& bd, bool grad, bool small) {
  const size_t rows = small ? BRANCH_TM_SMALL : BRANCH_TM, ab = prec == PAINN_FP64 ? 8 : 4;
  const int nh = (int)bd.size() - 1;
  int wmax = 0;
  size_t z = 0;
  for (int m = 0; m < nh; ++m) {
    wmax = wmax > pad32(bd[m]) ? wmax : pad32(bd[m]);
    if (grad && m + 1 < nh) z += pad32(bd[m]) * ab;
  }
  // every buffer of a chunk is a multiple of 256 bytes at these row counts
  return rows * ((size_t)branch_op_buffers(nh, grad) * branch_row_bytes(prec, wmax) +
                 (size_t)(pad32(bd[nh - 1]) / 16) * ab + z) + 2048;
}

BranchPlan branch_plan(int prec, const Hyper& hp, int N, bool blend, double skip, bool grad) {
  BranchPlan p;
  const bool small = branch_small(prec, hp, N, blend, skip);
  p.y_row = branch_row_bytes(prec, branch_ky(hp));
  p.dyh_row = blend && grad ? (size_t)hp.n_heads * branch_ky(hp) * (prec == PAINN_FP64 ? 8 : 4) : 0;
  p.tile = branch_tile_bytes(prec, hp.branch_dims, grad, small);
  p.TM = small ? BRANCH_TM_SMALL : BRANCH_TM;
  p.tiles = (long long)N * (blend ? hp.n_heads : 1) / p.TM + hp.n_heads;
  return p;
}

hipError_t launch_branch(hipStream_t st, int prec, const BranchArgs& b) {
  if (prec == PAINN_FP64)
    return b.dy ? branch_impl<P64, true>(st, b) : branch_impl<P64, false>(st, b);
  if (prec == PAINN_FP32)
    return b.dy ? branch_impl<P32, true>(st, b) : branch_impl<P32, false>(st, b);
  if (b.dy) return hipErrorInvalidValue;
  return branch_impl<PB16, false>(st, b);
}

hipError_t launch_branch_rows(hipStream_t st, int prec, int N, int F, const void* s, void* y) {
  const size_t tot = (size_t)N * F;
  const unsigned grid = (unsigned)((tot + 255) / 256 < 65536 ? (tot + 255) / 256 : 65536);
  if (!grid) return hipSuccess;
  if (prec == PAINN_FP64) k_branch_rows<P64><<<grid, 256, 0, st>>>(N, F, (const double*)s, y);
  else if (prec == PAINN_FP32) k_branch_rows<P32><<<grid, 256, 0, st>>>(N, F, (const float*)s, y);
  else k_branch_rows<PB16><<<grid, 256, 0, st>>>(N, F, (const bf16_t*)s, y);
  return hipGetLastError();
}

// Sampling products of randomized HSS compression (Sec. 2.2) on FP64 MFMA:
//   S^r = (A - M) R^r      and      S^c = (A - M)^T R^c,
// where M is either zero or the block-diagonal part of A formed by the leaf
// diagonal blocks.  With M the leaf blocks, S^(l) = (A - D^(l)) R at the
// leaf level is exactly the leaves' local sample S_loc = S(I,:) - D R(I,:)
// of Alg. 1, so the leaf step is fused into the sampling product.
//
// A may be stored in FP32 (widened exactly to FP64 when read from LDS) or
// FP64.  Both products are tall-skinny GEMMs (n x n times n x ncols, ncols =
// d0 or the growth step dd) and are MFMA-bound for ncols >= 32 on gfx950
// (FP64: ~9.8 flop/B ridge against 2*ncols/sizeof(A) flop per byte of A).
//
// Tiling: a 256-thread workgroup computes a 128 x 64 tile of S; its four
// wavefronts each own a 64 x 32 sub-tile as 4 x 2 blocks of the 16x16x4 f64
// MFMA.  A and R are staged through LDS in k-slices of BK rows (BK = 32 for
// FP32 A, 16 for FP64 A); the A slice is stored k-major so that both the
// plain and the transposed product read MFMA operands conflict-free, and
// only the global->LDS copy differs between them.  The next slice is
// prefetched into registers while the current one is multiplied.  When the
// tile count is too small to give every CU its four resident workgroups, K
// is split over workgroups and
// the partial sums are added in a fixed order by a second kernel
// (deterministic, no atomics).  Consecutive tiles are mapped to the same XCD
// so that the column tiles sharing an A slice meet in one L2.
#include <algorithm>
#include <type_traits>

#include "hss_internal.h"
#include "sample_plan.h"

namespace hss {
namespace {

typedef double dbl4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_a4 __attribute__((aligned(4)));  // 16 bytes from any entry of A

constexpr int BM = 128;
constexpr int BN = 64;
constexpr int NT = 256;
constexpr int kSmallN = 512;  // below: K whole in one workgroup

template <typename TA>
struct Cfg;
template <>
struct Cfg<float> {
  static constexpr int BK = 32;
  static constexpr int PAD = 16;
};
template <>
struct Cfg<double> {
  static constexpr int BK = 16;
  static constexpr int PAD = 8;
};

template <typename TA>
__device__ __forceinline__ double widen(TA v) {
  return (double)v;
}

// This thread's share of the A slice: 64 bytes of one row (NN: of A[i][k], TN:
// of A[k][i]) in 4 pieces of 16, piece q holding the entries (row, col ..) of
// the slice.  (Eight consecutive lanes to a row, FP64 NN: the stores to LDS
// collide, 10.2 against 9.7 ms at n = 65536, 4.9 against 4.0 at 40000.)  The
// loads need only the alignment of an entry, and go through the caches
// (streamed past them, the four loads of a thread fetch their lines more than
// once).  64 columns, ms, four scalar loads where rows are off the 16-byte
// grid, streamed elsewhere -> now: FP64 n = 20011 NN 1.78 -> 1.09, TN 1.15 ->
// 1.04; n = 32768 NN 2.67 -> 2.37, TN 2.52 -> 2.40; FP32 n = 20011 NN 1.56 -> 0.97,
// TN 1.15 -> 0.97; n = 32768 NN 2.09 -> 2.01, TN 2.10 -> 2.03.
template <typename TA, bool TRANS>
__device__ __forceinline__ void a_piece(int q, int& row, int& col) {
  constexpr int E = 64 / sizeof(TA), EV = 16 / sizeof(TA);
  constexpr int BK = Cfg<TA>::BK;
  const int tid = threadIdx.x;
  if (TRANS) {
    row = tid / (BM / E);
    col = (tid % (BM / E)) * E + q * EV;
  } else {
    row = tid / (BK / E);
    col = (tid % (BK / E)) * E + q * EV;
  }
}

// OWN: a thread takes wide loads where its own 64 bytes are inside; otherwise
// where the whole slice is.  OWN serves the tiles at the edge of the matrix
// (scalar loads for all of such a tile held the launch up: n = 8191, FP64,
// one column, both products 435 -> 350 us), and, throughout, two kinds of launches:
// n < kSmallN, where a few workgroups wait for every slice (FP64 n = 256, both
// products, 57 -> 52 us), and the transposed product of few columns, whose loads
// of R have branches of their own (FP32 n = 40000, one column 3.87 -> 3.36 ms;
// 64 columns, without them, 3.36 -> 3.33, but 8.06 -> 8.20 at n = 65536).
template <typename TA, bool TRANS, bool OWN>
__device__ __forceinline__ void load_a(TA (&v)[64 / sizeof(TA)], const TA* __restrict__ A,
                                       long long lda, int n, int i0, int k0, int kend,
                                       const int* __restrict__ leaf_of, bool need_mask) {
  constexpr int EV = 16 / sizeof(TA);
  const int rbeg = !TRANS ? i0 : k0, cbeg = !TRANS ? k0 : i0;
  const auto mine = [&] {  // this thread's 64 bytes of the slice are there
    int row, col;
    a_piece<TA, TRANS>(0, row, col);
    return rbeg + row < (!TRANS ? n : kend) && cbeg + col + 4 * EV <= (!TRANS ? kend : n);
  };
  if (OWN ? mine() : i0 + BM <= n && k0 + Cfg<TA>::BK <= kend) {  // or the whole slice is
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      int row, col;
      a_piece<TA, TRANS>(q, row, col);
      const u32x4_a4* p = reinterpret_cast<const u32x4_a4*>(A + (long long)(rbeg + row) * lda + cbeg + col);
      u32x4 w = *p;
      TA* t = reinterpret_cast<TA*>(&w);
#pragma unroll
      for (int e = 0; e < EV; ++e) v[q * EV + e] = t[e];
    }
  } else {
    const int rend = !TRANS ? n : kend, cend = !TRANS ? kend : n;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      int row, col;
      a_piece<TA, TRANS>(q, row, col);
#pragma unroll
      for (int e = 0; e < EV; ++e)
        v[q * EV + e] = (rbeg + row < rend && cbeg + col + e < cend)
                            ? A[(long long)(rbeg + row) * lda + cbeg + col + e]
                            : (TA)0;
    }
  }
  if (need_mask) {
    // zero the entries of the leaf diagonal blocks: leaf_of[i] == leaf_of[k]
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      int row, col;
      a_piece<TA, TRANS>(q, row, col);
#pragma unroll
      for (int e = 0; e < EV; ++e)
        if (rbeg + row < n && cbeg + col + e < n && leaf_of[rbeg + row] == leaf_of[cbeg + col + e])
          v[q * EV + e] = (TA)0;
    }
  }
}

template <typename TA, bool TRANS>
__device__ __forceinline__ void store_a(TA (*As)[BM + Cfg<TA>::PAD], const TA (&v)[64 / sizeof(TA)]) {
  constexpr int EV = 16 / sizeof(TA);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    int row, col;
    a_piece<TA, TRANS>(q, row, col);
#pragma unroll
    for (int e = 0; e < EV; ++e) {
      if (TRANS) As[row][col + e] = v[q * EV + e];
      else As[col + e][row] = v[q * EV + e];
    }
  }
}

// R slice: rows k0 .. k0+BK-1, columns c0 .. c0+BN-1; ER doubles per thread.
template <int BK>
__device__ __forceinline__ void load_r(double (&v)[BK / 4], const double* __restrict__ R,
                                       long long ldr, int k0, int kend, int c0, int ncols,
                                       bool vec_ok) {
  constexpr int ER = BK / 4;
  const int tid = threadIdx.x;
  const int rr = tid / (BN / ER);
  const int cc = (tid % (BN / ER)) * ER;
  const int k = k0 + rr;
  const int c = c0 + cc;
  if (k < kend && c + ER <= ncols && vec_ok) {
    const double2* p = reinterpret_cast<const double2*>(R + (long long)k * ldr + c);
#pragma unroll
    for (int q = 0; q < ER / 2; ++q) {
      double2 w = p[q];
      v[2 * q] = w.x;
      v[2 * q + 1] = w.y;
    }
  } else {
#pragma unroll
    for (int e = 0; e < ER; ++e) v[e] = (k < kend && c + e < ncols) ? R[(long long)k * ldr + c + e] : 0.0;
  }
}

template <int BK>
__device__ __forceinline__ void store_r(double (*Bs)[BN + 4], const double (&v)[BK / 4]) {
  constexpr int ER = BK / 4;
  const int tid = threadIdx.x;
  const int rr = tid / (BN / ER);
  const int cc = (tid % (BN / ER)) * ER;
#pragma unroll
  for (int e = 0; e < ER; ++e) Bs[rr][cc + e] = v[e];
}

template <typename TA, bool TRANS, bool OWN>
__global__ __launch_bounds__(NT) void sample_kernel(
    const TA* __restrict__ A, long long lda, int n, const int* __restrict__ leaf_of,
    const double* __restrict__ R, long long ldr, double* __restrict__ S, long long lds, int ncols,
    int n_nt, int ksplit, int kchunk, double* __restrict__ work) {
  constexpr int BK = Cfg<TA>::BK;
  constexpr int E = 64 / sizeof(TA);
  __shared__ TA As[BK][BM + Cfg<TA>::PAD];
  __shared__ double Bs[BK][BN + 4];

  // tile of this workgroup; consecutive logical tiles share an XCD
  const int nblk = gridDim.x;
  int L = blockIdx.x;
  if ((nblk & 7) == 0) L = (blockIdx.x & 7) * (nblk >> 3) + (blockIdx.x >> 3);
  const int nt = L % n_nt;
  const int rest = L / n_nt;
  const int ks = rest % ksplit;
  const int mt = rest / ksplit;
  const int i0 = mt * BM;
  const int c0 = nt * BN;
  const int kbeg = ks * kchunk;
  const int kend = min(n, kbeg + kchunk);

  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int wm = wave >> 1;
  const int wn = wave & 1;

  const bool vec_r = (ldr % 2 == 0) && ((reinterpret_cast<uintptr_t>(R) & 15) == 0);

  // Does the leaf mask touch rows [i0, i0+BM) x k-range [k0, k0+BK)?
  // leaf_of holds leaf ordinals in index order (non-decreasing), so the
  // blocks meet iff the leaf ranges of the two index ranges overlap.
  int li0 = 0, li1 = -1;
  if (leaf_of) {
    li0 = leaf_of[min(i0, n - 1)];
    li1 = leaf_of[min(i0 + BM, n) - 1];
  }

  dbl4 acc[4][2];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = dbl4{0.0, 0.0, 0.0, 0.0};

  const auto products = [&](auto own) __attribute__((always_inline)) {
    TA va[E];
    double vr[BK / 4];
    auto mask_for = [&](int k0) -> bool {
      if (!leaf_of || k0 >= kend) return false;
      const int lk0 = leaf_of[k0];
      const int lk1 = leaf_of[min(k0 + BK, kend) - 1];
      return !(lk1 < li0 || li1 < lk0);
    };

    int k0 = kbeg;
    if (k0 < kend) {
      load_a<TA, TRANS, own.value>(va, A, lda, n, i0, k0, kend, leaf_of, mask_for(k0));
      load_r<BK>(vr, R, ldr, k0, kend, c0, ncols, vec_r);
      store_a<TA, TRANS>(As, va);
      store_r<BK>(Bs, vr);
    }
    __syncthreads();
    for (; k0 < kend; k0 += BK) {
      const int kn = k0 + BK;
      if (kn < kend) {
        load_a<TA, TRANS, own.value>(va, A, lda, n, i0, kn, kend, leaf_of, mask_for(kn));
        load_r<BK>(vr, R, ldr, kn, kend, c0, ncols, vec_r);
      }
      // the wavefronts multiplying take issue priority over those still
      // loading or storing the next slice (8.99 -> 8.36 ms per launch at
      // n = 65536, 64 columns)
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int kk = 0; kk < BK; kk += 4) {
        const int kr = kk + (lane >> 4);
        double a[4], b[2];
#pragma unroll
        for (int mb = 0; mb < 4; ++mb) a[mb] = widen(As[kr][wm * 64 + mb * 16 + (lane & 15)]);
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) b[nb] = Bs[kr][wn * 32 + nb * 16 + (lane & 15)];
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
#pragma unroll
          for (int nb = 0; nb < 2; ++nb)
            acc[mb][nb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[mb], b[nb], acc[mb][nb], 0, 0, 0);
      }
      __builtin_amdgcn_s_setprio(0);
      __syncthreads();
      if (kn < kend) {
        store_a<TA, TRANS>(As, va);
        store_r<BK>(Bs, vr);
      }
      __syncthreads();
    }
  };
  if (OWN || i0 + BM > n) products(std::true_type{});
  else products(std::false_type{});

  // D layout of the 16x16x4 f64 MFMA on gfx950 (checked on the device):
  // lane l, register r -> row l/16 + 4r, column l%16.
  double* out = S;
  long long ldo = lds;
  if (ksplit > 1) {
    out = work + (long long)ks * n * ncols;
    ldo = ncols;
  }
#pragma unroll
  for (int mb = 0; mb < 4; ++mb)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
      const int c = c0 + wn * 32 + nb * 16 + (lane & 15);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = i0 + wm * 64 + mb * 16 + (lane >> 4) + 4 * r;
        if (i < n && c < ncols) out[(long long)i * ldo + c] = acc[mb][nb][r];
      }
    }
}

__global__ void reduce_splits_kernel(const double* __restrict__ work, int ksplit, long long n,
                                     int ncols, double* __restrict__ S, long long lds) {
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long total = n * ncols;
  if (idx >= total) return;
  const long long i = idx / ncols;
  const int c = (int)(idx % ncols);
  double s = 0.0;
  for (int q = 0; q < ksplit; ++q) s += work[(long long)q * total + idx];
  S[i * lds + c] = s;
}

struct Plan {
  int n_mt, n_nt, ksplit, kchunk;
};

// K is split so that the workgroups fill the device: 4 per CU at the most,
// with 1024 k or more each (a whole round of them for n >= 8192).  Smaller
// matrices have too few tiles for that: from n = 512 on their splits are
// taken down to 64 k, up to 16 of them and 2 workgroups per CU (the partial
// sums of more cost what they gain; at n = 300 the reduction does).  64
// columns, FP64, plain product: n = 512 57 -> 19 us, 1024 111 -> 24, 2048 117
// -> 29, 4096 120 -> 61, 6000 228 -> 152, 8192 on as before.
Plan make_plan(long long n, int ncols, int bk) {
  Plan p;
  p.n_mt = (int)((n + BM - 1) / BM);
  p.n_nt = (ncols + BN - 1) / BN;
  const long long tiles = (long long)p.n_mt * p.n_nt;
  const int cus = compute_units();
  const long long want = (4LL * cus + tiles - 1) / tiles;  // 4 workgroups per CU (the resident maximum)
  const long long small = small_splits(n, tiles, kSmallN, 64, cus);
  const long long splits = std::max(1LL, std::min(want, std::max(n / 1024, small)));
  long long chunk = (n + splits - 1) / splits;
  chunk = (chunk + bk - 1) / bk * bk;
  p.ksplit = (int)((n + chunk - 1) / chunk);
  p.kchunk = (int)chunk;
  return p;
}

template <typename TA, bool TRANS>
void run(const TA* A, long long lda, long long n, const int* leaf_of, int ncols, const double* R,
         long long ldr, double* S, long long lds, double* work, hipStream_t s) {
  Plan p = make_plan(n, ncols, Cfg<TA>::BK);
  const long long nblocks = (long long)p.n_mt * p.n_nt * p.ksplit;
  const bool own = n < kSmallN || (TRANS && ncols < BN);  // see load_a
  const auto fn = own ? sample_kernel<TA, TRANS, true> : sample_kernel<TA, TRANS, false>;
  hipLaunchKernelGGL(fn, dim3((unsigned)nblocks), dim3(NT), 0, s, A, lda, (int)n, leaf_of, R, ldr, S, lds, ncols,
                     p.n_nt, p.ksplit, p.kchunk, work);
  if (p.ksplit > 1) {
    const long long total = n * ncols;
    hipLaunchKernelGGL(reduce_splits_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s,
                       work, p.ksplit, n, ncols, S, lds);
  }
}

}  // namespace

long long sample_workspace_doubles(long long n, int ncols) {
  // the FP64 plan needs at least as many splits as the FP32 one
  Plan a = make_plan(n, ncols, Cfg<float>::BK);
  Plan b = make_plan(n, ncols, Cfg<double>::BK);
  int ks = a.ksplit > b.ksplit ? a.ksplit : b.ksplit;
  return ks > 1 ? (long long)ks * n * ncols : 0;
}

void launch_sample(const void* A, int dtype, long long n, long long lda, const int* leaf_of,
                   int ncols, const double* Rr, const double* Rc, long long ldr, double* Sr,
                   double* Sc, long long lds, double* work, hipStream_t s) {
  if (n <= 0 || ncols <= 0) return;
  if (dtype == 1) {
    const float* a = static_cast<const float*>(A);
    if (Sr) run<float, false>(a, lda, n, leaf_of, ncols, Rr, ldr, Sr, lds, work, s);
    if (Sc) run<float, true>(a, lda, n, leaf_of, ncols, Rc, ldr, Sc, lds, work, s);
  } else {
    const double* a = static_cast<const double*>(A);
    if (Sr) run<double, false>(a, lda, n, leaf_of, ncols, Rr, ldr, Sr, lds, work, s);
    if (Sc) run<double, true>(a, lda, n, leaf_of, ncols, Rc, ldr, Sc, lds, work, s);
  }
}

}  // namespace hss

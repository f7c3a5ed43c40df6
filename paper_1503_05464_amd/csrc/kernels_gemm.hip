// Batched FP64 GEMM with row gathers and scatters, for the small per-node
// products of compression (Alg. 1: S_a - B_ab R_b, V^T R_in), matvec
// (Alg. 2: V^T x, B y, U z) and the ULV factors (Alg. 3/4).
//
//   D[rowD(r), c] = beta * C[rowC(r), c] + alpha * sum_k Aop(r, k) * B[rowB(k), c]
//
// Every problem of a batch has its own sizes and pointers; one launch covers
// all of them, one output tile per workgroup.  The tile shape of a launch is
// picked from a table indexed by the batch's size class (widest N, largest
// M), written by the project's autotuner (paper_1503_05464_amd/autotune.py)
// from measured launch times, or by the launch's longest product where its
// tiles do not fill the device (pick_shape).  Row maps let the
// ID-structured generators U = Pi [I; E] act without forming U: rows J are
// gathered or scattered and E multiplies the other rows.  A source may be
// split in two segments (rows below `split` from one buffer, the rest from
// another), which stacks the two children's blocks [X_a; X_b] without a copy.
//
// Arithmetic: the 16x16x4 FP64 MFMA, k in increasing order whatever the tile
// shape.  A and B are staged through LDS in k-slices of 16, both k-major so
// that the MFMA operands are read conflict-free.
//
// What bounds it: the per-node products have few tiles and long inner
// dimensions, so a tile's time is its chain of slices.  With one slice loaded
// ahead, through flat accesses (an LDS wait for each, 64-bit products for
// every address), a slice took 1 us, the latency of its loads.  Now two to
// six slices are in flight in registers, A through a buffer resource (no
// address arithmetic), B through addresses looked up ahead in LDS, one
// barrier per slice that waits for LDS only.  A matvec with 64 columns at n = 20011:
// 1077 -> 515 us; the class of the widest, longest products (384 + 6 of up to
// 600 x 256 x 632): 655 -> 527 us.
#include <algorithm>
#include <climits>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "gemm_offsets.h"
#include "hss_internal.h"

namespace hss {
namespace {

constexpr int TK = kGemmSlice, NTH = 256;

typedef double dbl4 __attribute__((ext_vector_type(4)));

struct DevDesc {
  GemmDesc g;
  int tiles_n;  // tiles along N
};

// Pointers out of a descriptor table have no known address space: a load
// through one is a flat access, which counts as an LDS access too and makes
// every wait a full one.  They all point to device memory.
typedef __attribute__((address_space(1))) const double gdouble_c;
typedef __attribute__((address_space(1))) double gdouble;
typedef __attribute__((address_space(1))) const int gint_c;
__device__ __forceinline__ gint_c* as_global(const int* p) { return (gint_c*)(uintptr_t)p; }

// Row q of a segmented source (or output), q already mapped.
__device__ __forceinline__ gdouble_c* seg_row(const Seg& s, int q) {
  const uintptr_t p0 = (uintptr_t)s.p0, p1 = (uintptr_t)s.p1 - (uintptr_t)((long long)s.split * s.ld * 8);
  return (gdouble_c*)((q < s.split ? p0 : p1) + (uintptr_t)((long long)q * s.ld * 8));
}
__device__ __forceinline__ gdouble* seg_row_out(const SegOut& s, int q) {
  const uintptr_t p0 = (uintptr_t)s.p0, p1 = (uintptr_t)s.p1 - (uintptr_t)((long long)s.split * s.ld * 8);
  return (gdouble*)((q < s.split ? p0 : p1) + (uintptr_t)((long long)q * s.ld * 8));
}

// Tile shapes: the four wavefronts form a WGM x WGN grid, each owning MB x NB
// blocks of 16 x 16 (one 16x16x4 FP64 MFMA accumulator each), so a tile is
// TM = 16 WGM MB rows by TN = 16 WGN NB columns.  Wide tiles suit the
// compression's products (N = the new sample columns); narrow ones the
// matvec and solve with few right-hand sides, where a 64-column tile would
// leave most of its columns empty.
template <int WGM, int WGN, int MB, int NB>
struct Tile {
  static_assert(WGM * WGN == 4, "four wavefronts");
  static constexpr int TM = 16 * WGM * MB, TN = 16 * WGN * NB;
  static constexpr int LA = TK * TM / NTH, LB = TK * TN / NTH;  // slice entries per thread
  static_assert(LA >= 1 && LB >= 1 && TK * TM % NTH == 0 && TK * TN % NTH == 0, "whole slices");
  // slices in flight: as many as fit in about 48 registers
  static constexpr int PD = LA + LB <= 4 ? 6 : LA + LB <= 6 ? 4 : LA + LB < 8 ? 3 : 2;
};

// Orders this workgroup's LDS accesses around a barrier, leaving the global
// loads of later slices in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// k is walked in chunks of KC: the rows of B of a chunk are looked up ahead,
// as addresses in LDS, and A is addressed from the chunk's first k
constexpr int KC = kGemmChunk;
static_assert(KC % TK == 0, "whole slices");

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
// bytes of `count` doubles as the range of a buffer resource
__device__ __forceinline__ int buf_range(long long count) {
  return (int)(unsigned)min(count * 8, 0xffffffffll);
}
__device__ __forceinline__ double buf_load(__amdgpu_buffer_rsrc_t r, unsigned lane_off, unsigned off) {
  const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(r, (int)lane_off, (int)off, 0);
  return __hiloint2double((int)w.y, (int)w.x);
}

// Held to four wavefronts per SIMD (at most 128 registers), or to three where
// the LDS of a tile of 128 rows leaves no room for more, or where four blocks
// per wavefront would spill.
// SHORT: one slice ahead and no load past the last, for launches whose
// products have no more than kShortK k.  Their time is that of the outputs,
// which wants wavefronts: 68 to 128 registers instead of 94 to 168.  Device
// time, DEEP -> SHORT: 384 products of 300 x 256 with 8 k 184 -> 159 us, 64 of
// 1000 x 1000 with 16 k 376 -> 302, one of 400 x 700 with 48 k 13.5 -> 13.0.
// FAR: A is read at 64-bit addresses, for a leading dimension at which 32-bit
// offsets would wrap (gemm_offsets_fit: from 1048575 on with 512 rows of a
// transposed A, from 4.2 million on without).
enum Mode { DEEP, SHORT, FAR };
template <int WGM, int WGN, int MB, int NB, Mode MODE>
__global__ __launch_bounds__(NTH) __attribute__((amdgpu_waves_per_eu(MODE != SHORT && (WGM * MB > 4 || MB * NB > 2) ? 3 : 4))) void gemm_batched_kernel(
    const DevDesc* __restrict__ descs, const long long* __restrict__ tile0, int nprob) {
  using TL = Tile<WGM, WGN, MB, NB>;
  static_assert(TL::TM <= kGemmMaxRows, "offsets are checked for tiles of at most kGemmMaxRows rows");
  constexpr int TM = TL::TM, TN = TL::TN, LA = TL::LA, LB = TL::LB, PD = MODE == SHORT ? 1 : TL::PD;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  // the problem of this tile: the last whose first tile is not above it; 64
  // candidates per step, one per lane (a step is one load, where a binary
  // search waits for one load per halving)
  const long long t = blockIdx.x;
  int lo = 0, cnt = nprob;
  while (cnt > 1) {
    const int stride = (cnt + 63) >> 6;
    const int i = lane * stride;
    const unsigned long long le = __ballot(i < cnt && tile0[lo + min(i, cnt - 1)] <= t);
    const int at = (__popcll(le) - 1) * stride;  // lane 0 always counts
    lo += at;
    cnt = min(stride, cnt - at);
  }
  lo = __builtin_amdgcn_readfirstlane(lo);
  const DevDesc dd = descs[lo];  // by value: the uniform fields in scalar registers
  const GemmDesc& g = dd.g;
  const int local = (int)(t - tile0[lo]);
  const int r0 = local / dd.tiles_n * TM;
  const int c0 = local % dd.tiles_n * TN;
  const int M = g.M, N = g.N, K = g.K;

  __shared__ double As[2][TK][TM + 4];
  __shared__ double Bs[2][TK][TN + 4];
  __shared__ uintptr_t krow[KC];

  const int wm = wave / WGN, wn = wave % WGN;  // this wavefront's sub-tile
  const bool tr = g.transA != 0;

  // the output rows' places before the products: the latency of their maps
  // passes behind the k loop
  int rc[MB][4], rd[MB][4];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      rc[mb][q] = rd[mb][q] = min(r0 + wm * 16 * MB + mb * 16 + (lane >> 4) + 4 * q, M - 1);
  if (g.C.map && g.beta != 0.0) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int q = 0; q < 4; ++q) rc[mb][q] = as_global(g.C.map)[rc[mb][q]];
  }
  if (g.D.map) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int q = 0; q < 4; ++q) rd[mb][q] = as_global(g.D.map)[rd[mb][q]];
  }

  // This thread's share of a k-slice: LA entries of A and LB of B.  Rows and
  // columns past the end read the last valid one (they only reach outputs
  // that are not stored), and k past the end is zeroed on its way into LDS.
  // A is read through a buffer resource: a lane's offset never changes, the
  // slice's is a scalar, and reads past the matrix return zero.
  unsigned ao[LA];     // byte offset of the entry from the chunk's first slice (FAR: its row)
  int ak[LA], al[LA];  // k within the slice, place in the LDS slice
#pragma unroll
  for (int q = 0; q < LA; ++q) {
    const int e = tid + q * NTH;
    const int rr = tr ? e % TM : e / TK;
    ak[q] = tr ? e / TM : e % TK;
    al[q] = ak[q] * (TM + 4) + rr;
    const int rv = min(rr, M - 1 - r0);
    ao[q] = MODE == FAR ? (unsigned)rv : gemm_entry_offset(tr, g.lda, rv, ak[q]);
  }
  const unsigned astep = gemm_slice_step(tr, g.lda);  // from one slice to the next
  const int mt = min(TM, M - r0);  // rows of this tile
  const int cb = min(c0 + tid % TN, N - 1);
  const int bk = tid / TN;  // entries q of B lie NTH / TN rows apart
  double va[PD][LA], vb[PD][LB];
  __amdgpu_buffer_rsrc_t ra;
  gdouble_c* fa = nullptr;  // FAR: the chunk's first entry
  int fk = 0;               // and its last k
  auto load = [&](double (&xa)[LA], double (&xb)[LB], int s) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < LA; ++q) {
      if constexpr (MODE == FAR) {
        const long long k = min(s * TK + ak[q], fk), r = ao[q];
        xa[q] = fa[tr ? k * g.lda + r : r * g.lda + k];
      } else {
        xa[q] = buf_load(ra, ao[q], (unsigned)s * astep);
      }
    }
#pragma unroll
    for (int q = 0; q < LB; ++q) xb[q] = ((gdouble_c*)krow[s * TK + bk + q * (NTH / TN)])[cb];
  };
  auto store = [&](const double (&xa)[LA], const double (&xb)[LB], int b, int k0) __attribute__((always_inline)) {
    double* as = &As[b][0][0];
#pragma unroll
    for (int q = 0; q < LA; ++q) as[al[q]] = k0 + ak[q] < K ? xa[q] : 0.0;
#pragma unroll
    for (int q = 0; q < LB; ++q) {
      const int kk = bk + q * (NTH / TN);
      Bs[b][kk][tid % TN] = k0 + kk < K ? xb[q] : 0.0;
    }
  };

  dbl4 acc[MB][NB];
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = dbl4{0.0, 0.0, 0.0, 0.0};

  for (int kc = 0; kc < K; kc += KC) {
    const int kn = min(K - kc, KC);
    const int ns = (kn + TK - 1) / TK;  // slices
    for (int k = tid; k < ns * TK; k += NTH) {
      const int kk = kc + min(k, kn - 1);
      krow[k] = (uintptr_t)seg_row(g.B, g.B.map ? as_global(g.B.map)[kk] : kk);
    }
    const double* a0 = g.A + (tr ? (long long)kc * g.lda + r0 : (long long)r0 * g.lda + kc);
    if constexpr (MODE == FAR) {
      fa = (gdouble_c*)(uintptr_t)a0;
      fk = kn - 1;
    } else {
      ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(a0), 0,
                                             buf_range(tr ? (kn - 1) * g.lda + mt : (mt - 1) * g.lda + kn), 0x00027000);
    }
    lds_barrier();
#pragma unroll
    for (int p = 0; p < PD; ++p) load(va[p], vb[p], min(p, ns - 1));
    store(va[0], vb[0], 0, kc);
    lds_barrier();
    // slice s is multiplied from LDS while slices s+1 .. s+PD are on their
    // way: s+1 has arrived in registers (its loads are the oldest) and goes
    // into the other LDS buffer, and s+1+PD takes its registers
    for (int s0 = 0; s0 < ns; s0 += PD * 2) {
#pragma unroll
      for (int u = 0; u < PD * 2; ++u) {
        const int s = s0 + u;
        if (s >= ns) break;
        double a[TK / 4][MB], b[TK / 4][NB];
#pragma unroll
        for (int q = 0; q < TK / 4; ++q) {
          const int kr = 4 * q + (lane >> 4);
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) a[q][mb] = As[u & 1][kr][wm * 16 * MB + mb * 16 + (lane & 15)];
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) b[q][nb] = Bs[u & 1][kr][wn * 16 * NB + nb * 16 + (lane & 15)];
        }
        // past the last slice: the last one again, never stored
        if (MODE != SHORT || s + PD < ns) load(va[u % PD], vb[u % PD], min(s + PD, ns - 1));
        __builtin_amdgcn_s_setprio(1);  // multiplying wavefronts issue first
#pragma unroll
        for (int q = 0; q < TK / 4; ++q)
#pragma unroll
          for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
              acc[mb][nb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q][mb], b[q][nb], acc[mb][nb], 0, 0, 0);
        __builtin_amdgcn_s_setprio(0);
        if (s + 1 < ns) store(va[(u + 1) % PD], vb[(u + 1) % PD], (u + 1) & 1, kc + (s + 1) * TK);
        lds_barrier();
      }
    }
  }

  // D layout of the 16x16x4 f64 MFMA: lane l, register q -> row l/16 + 4q,
  // column l%16 of the 16 x 16 block
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (r0 + wm * 16 * MB + mb * 16 + (lane >> 4) + 4 * q >= M) continue;
      gdouble_c* crow = seg_row(g.C, rc[mb][q]);
      gdouble* drow = seg_row_out(g.D, rd[mb][q]);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const int c = c0 + wn * 16 * NB + nb * 16 + (lane & 15);
        if (c >= N) continue;
        double v = g.alpha * acc[mb][nb][q];
        if (g.beta != 0.0) v += g.beta * crow[c];
        drow[c] = v;
      }
    }
}

struct GVariant {
  int tm, tn;
  void (*fn[2])(const DevDesc*, const long long*, int);  // DEEP, SHORT
};
#define GV(A_, B_, C_, D_) {gemm_batched_kernel<A_, B_, C_, D_, DEEP>, gemm_batched_kernel<A_, B_, C_, D_, SHORT>}
// the tile shapes (index = variant number of the tuning table)
const GVariant kGVariants[] = {
    {64, 64, GV(2, 2, 2, 2)},
    {64, 16, GV(4, 1, 1, 1)},
    {128, 16, GV(4, 1, 2, 1)},
    {32, 32, GV(2, 2, 1, 1)},
    {64, 32, GV(4, 1, 1, 2)},
    {128, 32, GV(4, 1, 2, 2)},
    {16, 64, GV(1, 4, 1, 1)},
};
#undef GV
// the shape of every launch with an A beyond 32-bit offsets
const GVariant kGFar = {32, 32, {gemm_batched_kernel<2, 2, 1, 1, FAR>, gemm_batched_kernel<2, 2, 1, 1, FAR>}};
// most k of a SHORT launch.  At 48 to 64 k SHORT took 0.82 to 1.0 of DEEP's time
// in 190 launches of 1 to 384 products of 4 x 20 to 1000 x 1000; above, the
// two come together (200 k, few tiles: up to 1.1) and the table is DEEP's.
constexpr int kShortK = 64;
constexpr int kNumGVariants = sizeof(kGVariants) / sizeof(kGVariants[0]);

#include "gemm_tiles.inc"  // kGemmTileTable[SHORT][class] = variant (written by autotune.py)
static_assert(sizeof(kGemmTileTable) == 2 * kGemmClasses * sizeof(int), "one entry per class and mode");

}  // namespace

// The size class of a launch: its widest N and its largest M, bucketed.
static int gemm_class(const GemmDesc* descs, int nprob) {
  int nmax = 0, mmax = 0;
  for (int p = 0; p < nprob; ++p)
    if (descs[p].M > 0 && descs[p].N > 0) {
      nmax = std::max(nmax, descs[p].N);
      mmax = std::max(mmax, descs[p].M);
    }
  const int nb = nmax <= 16 ? 0 : nmax <= 32 ? 1 : nmax <= 64 ? 2 : 3;
  const int mb = mmax <= 32 ? 0 : mmax <= 128 ? 1 : 2;
  return nb * 3 + mb;
}

int compute_units() {
  static const int v = [] {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
      return 256;
    return cus;
  }();
  return v;
}

// The tile shape of a launch.  The table's shapes are the fastest where the
// tiles fill the device.  Where they do not, a launch lasts as long as its
// tile with the longest inner dimension, whose slices cost a compute unit the
// matrix instructions of its blocks: 1024 cycles a slice for 64 x 64, 256
// for the shapes with one block per wavefront.  So a launch whose longest
// tile takes more than the device's share of all its tiles goes to such a
// shape (every shape gives the same bits).  Measured at the top of a matvec
// with 64 columns (n = 20011, two to four products of about 700 x 64 x 1500):
// 64 x 64, 28 workgroups, 64 us; 32 x 32, 22 us.  Of these shapes 32 x 32 has
// the most slices in flight (6 against 4 of 16 x 64, which loads five entries
// a thread and slice for its four): two products of up to 400 rows, 33 to 256
// columns and 1500 k take 44 to 46 us, 47 to 49 in 16 x 64 and 49 to 51 in
// 64 x 16.  Where the tiles fill the device, 16 x 64 is the better (the table).
static int pick_shape(const GemmDesc* descs, int nprob, Mode mode) {
  const int cls = gemm_class(descs, nprob);
  const int v = kGemmTileTable[mode == SHORT][cls];
  const int small = cls < 3 ? 1 : 3;  // 64 x 16 up to 16 columns, else 32 x 32
  const GVariant& gv = kGVariants[v];
  long long slices = 0, longest = 0;
  for (int p = 0; p < nprob; ++p) {
    const GemmDesc& g = descs[p];
    if (g.M <= 0 || g.N <= 0) continue;
    const long long n = (g.K + TK - 1) / TK;
    longest = std::max(longest, n);
    slices += n * ((g.M + gv.tm - 1) / gv.tm) * ((g.N + gv.tn - 1) / gv.tn);
  }
  return longest * compute_units() > slices ? small : v;
}

hipError_t launch_gemm_batched(const GemmDesc* descs, int nprob, Staging& st, hipStream_t s, int variant) {
  if (nprob <= 0) return hipSuccess;
  bool far = false;
  int kmax = 0;
  for (int p = 0; p < nprob; ++p) {
    const GemmDesc& g = descs[p];
    if (g.M <= 0 || g.N <= 0) continue;
    kmax = std::max(kmax, g.K);
    far = far || !gemm_offsets_fit(g.transA != 0, g.M, g.K, g.lda);
  }
  const Mode mode = far ? FAR : kmax <= kShortK ? SHORT : DEEP;
  if (variant < 0 || variant >= kNumGVariants) {
    variant = pick_shape(descs, nprob, mode);
    static const int forced = [] {  // tuning and tests: one variant for every launch
      const char* v = std::getenv("HSS_GEMM_VARIANT");
      return v && v[0] ? std::atoi(v) : -1;
    }();
    if (forced >= 0 && forced < kNumGVariants) variant = forced;
  }
  const GVariant& gv = far ? kGFar : kGVariants[variant];
  std::vector<DevDesc> h;
  std::vector<long long> tile0;  // first flattened tile of each problem
  h.reserve(nprob);
  tile0.reserve(nprob);
  long long tiles = 0;
  for (int p = 0; p < nprob; ++p) {
    const GemmDesc& g = descs[p];
    if (g.M <= 0 || g.N <= 0) continue;
    DevDesc d;
    d.g = g;
    if (d.g.B.p1 == nullptr) d.g.B.split = INT_MAX;
    if (d.g.C.p1 == nullptr) d.g.C.split = INT_MAX;
    if (d.g.D.p1 == nullptr) d.g.D.split = INT_MAX;
    d.tiles_n = (g.N + gv.tn - 1) / gv.tn;
    tile0.push_back(tiles);
    tiles += (long long)((g.M + gv.tm - 1) / gv.tm) * d.tiles_n;
    h.push_back(d);
  }
  if (h.empty() || tiles <= 0) return hipSuccess;
  // one table, one copy: the descriptors, then the first tiles
  const size_t db = sizeof(DevDesc) * h.size(), tb = sizeof(long long) * h.size();
  std::vector<char> table(db + tb);
  std::memcpy(table.data(), h.data(), db);
  std::memcpy(table.data() + db, tile0.data(), tb);
  char* dd = static_cast<char*>(st.push(table.data(), db + tb));
  if (!dd) return hipErrorOutOfMemory;
  const auto fn = gv.fn[mode == SHORT];
  const int np = (int)h.size();
  return st.launch([=] {
    hipLaunchKernelGGL(fn, dim3((unsigned)tiles), dim3(NTH), 0, s, reinterpret_cast<const DevDesc*>(dd),
                       reinterpret_cast<const long long*>(dd + db), np);
    return hipGetLastError();
  });
}

int gemm_variants() { return kNumGVariants; }

}  // namespace hss

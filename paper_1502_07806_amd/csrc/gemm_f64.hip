// FP64 GEMM on CDNA4 matrix cores (v_mfma_f64_16x16x4_f64) with LDS double
// buffering and fused epilogues for the PFSM contractions:
//   basis change  W = A V,  At = V^T W            (EPI_STORE, lower tiles + mirror)
//   folded-spectrum products (At - eps)X, X - a(At - eps)Y   (EPI_SHIFT / EPI_FSUPD)
//   overlap S = X^T X, Cholesky trailing updates    (EPI_STORE, alpha/beta)
//   Rayleigh quotients  x_j^T (At x_j)               (EPI_RQ column-dot partials)
//
// 256 threads = 4 waves in a 2x2 grid; a wave owns WI x WJ MFMA blocks of
// 16x16, so the block tile is (32 WI) x (32 WJ).  The MFMA is issued with the B
// fragment as its first operand so that each lane's accumulator entries run
// down a column of C (row = lane%16, col = lane/16 + 4*reg), which makes the
// column-major stores contiguous per column.
//
// Two kernels: gemm_f64_dl (tiles of 128 or 64, loads straight into LDS) and
// gemm_f64_kernel (tiles of 32 for products too small to fill the chip with
// larger ones, and any leading dimension); gemm_f64 chooses.
#include "common.h"

namespace pfsm {
namespace {

typedef double v2d __attribute__((ext_vector_type(2)));
constexpr int NT = 256;
// An operand tile that is contiguous along k in memory sits in LDS as [row][k]
// with its 16-byte chunks swizzled by the row, so that both the coalesced
// stores (consecutive k) and the 16-byte fragment reads (consecutive rows)
// are free of bank conflicts; one that is contiguous along its rows sits as
// [k][row].  Within a group of 8 k values, MFMA h takes k = 2 (lane / 16) + h
// from both operands, so a [row][k] fragment read gives two MFMAs' operands.
template <bool KMAJOR, int ROWS, int BK> __device__ inline int lds_at(int row, int k) {
  return KMAJOR ? row * BK + ((((k >> 1) ^ (row & 7)) << 1) | (k & 1)) : k * ROWS + row;
}

__device__ inline int xcd_tile(int b, int total) {
  // Workgroups are dispatched round-robin over the 8 XCDs; give each XCD a
  // contiguous range of tiles so neighbouring tiles share its L2.
  if (total % 8 != 0) return b;
  return (b % 8) * (total / 8) + b / 8;
}

__device__ inline void tri_index(int t, int& a, int& b) {
  // t -> (a, b) with a >= b, row-major over the lower triangle
  int r = (int)((sqrt(8.0 * t + 1.0) - 1.0) * 0.5);
  while ((r + 1) * (r + 2) / 2 <= t) ++r;
  while (r * (r + 1) / 2 > t) --r;
  a = r;
  b = t - r * (r + 1) / 2;
}

// Block tile of this workgroup: the lower triangle only, or groups of 8 row
// tiles together, so that consecutive tiles reuse B columns and A rows.
// Rayleigh quotients of a symmetric A (EPI_RQ, lower_only) have K ranges that
// end at the tile's last row: the longest first, dealt round the XCDs.
template <int EPI>
__device__ inline void tile_coords(const GemmArgs& g, int tiles_m, int tiles_n, int& tm, int& tn) {
  if (EPI == EPI_RQ && g.lower_only) {
    tm = tiles_m - 1 - (int)blockIdx.x / tiles_n;
    tn = (int)blockIdx.x % tiles_n;
    return;
  }
  if (g.lower_only) {  // tiles_m == tiles_n
    const int total = tiles_m * (tiles_m + 1) / 2;
    tri_index(xcd_tile(blockIdx.x, total), tm, tn);
    return;
  }
  const int t_lin = xcd_tile(blockIdx.x, tiles_m * tiles_n);
  const int GROUP = 8;
  const int first_m = (t_lin / (GROUP * tiles_n)) * GROUP;
  const int gsz = min(tiles_m - first_m, GROUP);
  tm = first_m + (t_lin % (GROUP * tiles_n)) % gsz;
  tn = (t_lin % (GROUP * tiles_n)) / gsz;
}

template <int WI, int WJ> __device__ inline void double_acc(v4d (&acc)[WI][WJ]) {
#pragma unroll
  for (int i = 0; i < WI; ++i)
#pragma unroll
    for (int j = 0; j < WJ; ++j) acc[i][j] *= 2.0;
}

// acc[ib][jb][r] is C(i, j) with i = wi0 + 16 ib + lane % 16, j = wj0 + 16 jb +
// lane / 16 + 4 r; red: BN doubles per wave row, free to use.
template <int EPI, int WI, int WJ>
__device__ inline void f64_epilogue(const GemmArgs& g, v4d (&acc)[WI][WJ], int64_t m0, int64_t n0, int wi0, int wj0,
                                    int tid, int tm, double (*red)[32 * WJ]) {
  constexpr int BN = 32 * WJ;
  const int lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, lq = lane >> 4;
  if (EPI == EPI_RQ) {
    // column partial sums of acc .* D over this tile's rows
    double cs[WJ][4];
#pragma unroll
    for (int jb = 0; jb < WJ; ++jb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        double s = 0.0;
        int64_t gj = n0 + wj0 + jb * 16 + lq + 4 * r;
#pragma unroll
        for (int ib = 0; ib < WI; ++ib) {
          int64_t gi = m0 + wi0 + ib * 16 + l16;
          if (gi < g.M && gj < g.N) s += acc[ib][jb][r] * g.D[gi + gj * g.ldd];
        }
        // reduce over the 16 lanes that share this column (same lane>>4)
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) s += __shfl_xor(s, off, 64);
        cs[jb][r] = s;
      }
    if (l16 == 0) {
#pragma unroll
      for (int jb = 0; jb < WJ; ++jb)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wave & 1][wj0 + jb * 16 + lq + 4 * r] = cs[jb][r];
    }
    __syncthreads();
    if (tid < BN) {
      int64_t gj = n0 + tid;
      if (gj < g.N) g.part[(int64_t)tm * g.N + gj] = red[0][tid] + red[1][tid];
    }
    if (!g.part2) return;
    // the same for acc^2 (squared norms of the columns of A X over this tile's rows)
#pragma unroll
    for (int jb = 0; jb < WJ; ++jb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        double s = 0.0;
        const int64_t gj = n0 + wj0 + jb * 16 + lq + 4 * r;
#pragma unroll
        for (int ib = 0; ib < WI; ++ib) {
          const int64_t gi = m0 + wi0 + ib * 16 + l16;
          if (gi < g.M && gj < g.N) s += acc[ib][jb][r] * acc[ib][jb][r];
        }
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) s += __shfl_xor(s, off, 64);
        cs[jb][r] = s;
      }
    __syncthreads();  // red is read above
    if (l16 == 0) {
#pragma unroll
      for (int jb = 0; jb < WJ; ++jb)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wave & 1][wj0 + jb * 16 + lq + 4 * r] = cs[jb][r];
    }
    __syncthreads();
    if (tid < BN) {
      const int64_t gj = n0 + tid;
      if (gj < g.N) g.part2[(int64_t)tm * g.N + gj] = red[0][tid] + red[1][tid];
    }
    return;
  }

  if (EPI == EPI_G2S) {
    // C = Z + D^{-1}(A - B Z) for the generalized -> standard iteration, with
    // per-column partial sums of the squared residual.  The loads of one row
    // block are gathered before its stores.
    double cs[WJ][4];
#pragma unroll
    for (int jb = 0; jb < WJ; ++jb)
#pragma unroll
      for (int r = 0; r < 4; ++r) cs[jb][r] = 0.0;
#pragma unroll
    for (int ib = 0; ib < WI; ++ib) {
      const int64_t gi = m0 + wi0 + ib * 16 + l16;
      if (gi >= g.M) continue;
      const double di = g.eps[gi];
      double zv[WJ][4], av[WJ][4];
#pragma unroll
      for (int jb = 0; jb < WJ; ++jb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int64_t gj = min<int64_t>(n0 + wj0 + jb * 16 + lq + 4 * r, g.N - 1);
          zv[jb][r] = g.B[gi + gj * g.ldb];
          av[jb][r] = g.D[gi + gj * g.ldd];
        }
#pragma unroll
      for (int jb = 0; jb < WJ; ++jb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int64_t gj = n0 + wj0 + jb * 16 + lq + 4 * r;
          if (gj >= g.N) continue;
          const double res = av[jb][r] - acc[ib][jb][r];
          g.C[gi + gj * g.ldc] = zv[jb][r] + di * res;
          cs[jb][r] += res * res;
        }
    }
    if (!g.part) return;
#pragma unroll
    for (int jb = 0; jb < WJ; ++jb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        double s = cs[jb][r];
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) s += __shfl_xor(s, off, 64);
        cs[jb][r] = s;
      }
    if (l16 == 0) {
#pragma unroll
      for (int jb = 0; jb < WJ; ++jb)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wave & 1][wj0 + jb * 16 + lq + 4 * r] = cs[jb][r];
    }
    __syncthreads();
    if (tid < BN) {
      const int64_t gj = n0 + tid;
      if (gj < g.N) g.part[(int64_t)tm * g.N + gj] = red[0][tid] + red[1][tid];
    }
    return;
  }

  if (EPI == EPI_POLY) {
    // one output at a time; the loads of one row block are gathered before its stores
    for (int o = 0; o < g.poly_count; ++o) {
      double* P = g.poly[o];
      const double *ci = g.poly_init[o], *cc = g.poly_coef[o];
      const double* src = ci ? g.B : P;
      const int64_t lds = ci ? g.ldb : g.ldc;
#pragma unroll
      for (int ib = 0; ib < WI; ++ib) {
        const int64_t gi = m0 + wi0 + ib * 16 + l16;
        if (gi >= g.M) continue;
        double v[WJ][4];
#pragma unroll
        for (int jb = 0; jb < WJ; ++jb)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int64_t c = n0 + wj0 + jb * 16 + lq + 4 * r, gj = c < g.N ? c : g.N - 1;
            v[jb][r] = (ci ? ci[gj] : 1.0) * src[gi + gj * lds] + (cc ? cc[gj] : 1.0) * acc[ib][jb][r];
          }
#pragma unroll
        for (int jb = 0; jb < WJ; ++jb)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int64_t gj = n0 + wj0 + jb * 16 + lq + 4 * r;
            if (gj < g.N) P[gi + gj * g.ldc] = v[jb][r];
          }
      }
    }
    return;
  }

  double a_eff = g.alpha;
  if (EPI == EPI_FSUPD && g.alpha_dev) a_eff = *g.alpha_dev;
#pragma unroll
  for (int ib = 0; ib < WI; ++ib) {
    const int64_t gi = m0 + wi0 + ib * 16 + l16;
    if (gi >= g.M) continue;
#pragma unroll
    for (int jb = 0; jb < WJ; ++jb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t gj = n0 + wj0 + jb * 16 + lq + 4 * r;
        if (gj >= g.N) continue;
        double v = acc[ib][jb][r];
        double* cp = g.C + gi + gj * g.ldc;
        if (EPI == EPI_STORE) {
          v = g.alpha * v;
          if (g.beta != 0.0) v += g.beta * (*cp);
        } else if (EPI == EPI_SHIFT) {
          v = v - g.B[gi + gj * g.ldb] * g.eps[gj];
        } else if (EPI == EPI_FSUPD) {
          v = g.D[gi + gj * g.ldd] - a_eff * (v - g.B[gi + gj * g.ldb] * g.eps[gj]);
        }
        *cp = v;
      }
  }
}

template <bool TA, bool TB, int EPI, int WI, int WJ, int BK, typename OFF>
__global__ __launch_bounds__(NT, 3) void gemm_f64_kernel(GemmArgs g, int tiles_m, int tiles_n) {
  constexpr int BM = 32 * WI, BN = 32 * WJ;
  constexpr int A_PER_T = BM * BK / NT, B_PER_T = BN * BK / NT;
  __shared__ __attribute__((aligned(16))) double As[2][BM * BK];
  __shared__ __attribute__((aligned(16))) double Bs[2][BN * BK];
  __shared__ double red[2][BN];

  int tm, tn;
  tile_coords<EPI>(g, tiles_m, tiles_n, tm, tn);
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wi0 = (wave & 1) * 16 * WI, wj0 = (wave >> 1) * 16 * WJ;
  const int l16 = lane & 15, lq = lane >> 4;

  int64_t kbeg = 0, kend = g.K;
  if (g.krange) {
    const int64_t kt = n0 / GEMM_BN;
    kbeg = g.krange[2 * kt];
    kend = g.krange[2 * kt + 1];
  }
  const bool sym = EPI == EPI_RQ && g.lower_only;  // sum over k < m0 twice, the diagonal block once
  if (sym) kend = m0 + BM < g.K ? m0 + BM : g.K;

  v4d acc[WI][WJ];
#pragma unroll
  for (int i = 0; i < WI; ++i)
#pragma unroll
    for (int j = 0; j < WJ; ++j) acc[i][j] = (v4d){0.0, 0.0, 0.0, 0.0};

  // element r of this thread's part of the A / B tile: (row, k)
  auto a_row = [&](int r) { return TA ? tid / BK + (NT / BK) * r : tid % BM; };
  auto a_k = [&](int r) { return TA ? tid % BK : tid / BM + (NT / BM) * r; };
  auto b_row = [&](int r) { return TB ? tid % BN : tid / BK + (NT / BK) * r; };
  auto b_k = [&](int r) { return TB ? tid / BN + (NT / BN) * r : tid % BK; };
  double ra[A_PER_T], rb[B_PER_T];
  // Offsets (in bytes) from the tile's first element of the stage; rows past
  // the edge read the last row, whose results are never stored.  Whole stages
  // load without tests; in the last, partial one the elements past the end
  // read the stage's first element instead and count as zero.
  OFF offa[A_PER_T], offb[B_PER_T];
  const int64_t am = min<int64_t>(BM, g.M - m0) - 1, bn = min<int64_t>(BN, g.N - n0) - 1;
#pragma unroll
  for (int r = 0; r < A_PER_T; ++r) {
    const int64_t i = min<int64_t>(a_row(r), am);
    offa[r] = (OFF)(8 * (TA ? i * g.lda + a_k(r) : i + a_k(r) * g.lda));
  }
#pragma unroll
  for (int r = 0; r < B_PER_T; ++r) {
    const int64_t j = min<int64_t>(b_row(r), bn);
    offb[r] = (OFF)(8 * (TB ? j + b_k(r) * g.ldb : j * g.ldb + b_k(r)));
  }
  auto load_tile = [&](int64_t k0) {
    const char* pa = (const char*)(g.A + (TA ? m0 * g.lda + k0 : m0 + k0 * g.lda));
    const char* pb = (const char*)(g.B + (TB ? n0 + k0 * g.ldb : n0 * g.ldb + k0));
    const int left = (int)min<int64_t>(BK, kend - k0);
    if (left == BK) {
#pragma unroll
      for (int r = 0; r < A_PER_T; ++r) ra[r] = *(const double*)(pa + offa[r]);
#pragma unroll
      for (int r = 0; r < B_PER_T; ++r) rb[r] = *(const double*)(pb + offb[r]);
    } else {
#pragma unroll
      for (int r = 0; r < A_PER_T; ++r) {
        const bool in = a_k(r) < left;
        const double v = *(const double*)(pa + (in ? offa[r] : (OFF)0));
        ra[r] = in ? v : 0.0;
      }
#pragma unroll
      for (int r = 0; r < B_PER_T; ++r) {
        const bool in = b_k(r) < left;
        const double v = *(const double*)(pb + (in ? offb[r] : (OFF)0));
        rb[r] = in ? v : 0.0;
      }
    }
  };
  auto store_tile = [&](int buf) {
#pragma unroll
    for (int r = 0; r < A_PER_T; ++r) As[buf][lds_at<TA, BM, BK>(a_row(r), a_k(r))] = ra[r];
#pragma unroll
    for (int r = 0; r < B_PER_T; ++r) Bs[buf][lds_at<!TB, BN, BK>(b_row(r), b_k(r))] = rb[r];
  };
  auto mma = [&](int buf) {
#pragma unroll
    for (int kk = 0; kk < BK; kk += 8) {
      double2 af[WI], bf[WJ];
#pragma unroll
      for (int ib = 0; ib < WI; ++ib) {
        const int i = wi0 + ib * 16 + l16, k = kk + 2 * lq;
        if (TA) af[ib] = *(const double2*)&As[buf][lds_at<true, BM, BK>(i, k)];
        else af[ib] = make_double2(As[buf][lds_at<false, BM, BK>(i, k)], As[buf][lds_at<false, BM, BK>(i, k + 1)]);
      }
#pragma unroll
      for (int jb = 0; jb < WJ; ++jb) {
        const int j = wj0 + jb * 16 + l16, k = kk + 2 * lq;
        if (!TB) bf[jb] = *(const double2*)&Bs[buf][lds_at<true, BN, BK>(j, k)];
        else bf[jb] = make_double2(Bs[buf][lds_at<false, BN, BK>(j, k)], Bs[buf][lds_at<false, BN, BK>(j, k + 1)]);
      }
#pragma unroll
      for (int ib = 0; ib < WI; ++ib)
#pragma unroll
        for (int jb = 0; jb < WJ; ++jb)
          acc[ib][jb] = __builtin_amdgcn_mfma_f64_16x16x4f64(bf[jb].x, af[ib].x, acc[ib][jb], 0, 0, 0);
#pragma unroll
      for (int ib = 0; ib < WI; ++ib)
#pragma unroll
        for (int jb = 0; jb < WJ; ++jb)
          acc[ib][jb] = __builtin_amdgcn_mfma_f64_16x16x4f64(bf[jb].y, af[ib].y, acc[ib][jb], 0, 0, 0);
    }
  };

  const int64_t ntk = kend > kbeg ? (kend - kbeg + BK - 1) / BK : 0;
  if (ntk > 0) {
    load_tile(kbeg);
    store_tile(0);
    __syncthreads();
    for (int64_t t = 0; t < ntk; ++t) {
      const int cur = (int)(t & 1);
      if (t + 1 < ntk) load_tile(kbeg + (t + 1) * BK);
      if (sym && t * BK == m0) double_acc(acc);
      mma(cur);
      if (t + 1 < ntk) store_tile(cur ^ 1);
      __syncthreads();
    }
  }
  f64_epilogue<EPI, WI, WJ>(g, acc, m0, n0, wi0, wj0, tid, tm, red);
}

// ------------------------------------------------------- direct-to-LDS kernel
// Tiles of (32 WI) x (32 WJ) x 16 loaded straight from global memory into LDS
// (buffer loads, CH bytes per lane: 16 where alignment and even sizes allow,
// else 4), so nothing passes through registers on the way.  Rows past the
// edge and k past the end get an offset beyond the buffer's range, for which
// the load writes zeros.  Offsets fit 31 bits for leading dimensions below
// 2^21 (gemm_f64 checks).
//
// The fragments of a stage's second half are read while the MFMAs of its
// first half run, those of the next stage's first half while the second
// half's run.  The one barrier of a stage lies between the halves: by then
// every wave holds all of stage t in registers, so its slot takes stage
// t + 2, and every wave's part of stage t + 1 has landed.  Stages past the
// last are issued too (they read only zeros), so the loop body has no branch.
//
// Bound by the FP64 matrix cores (64 cycles per MFMA): 75.0 TFLOP/s at N =
// 8192 TN, 74 NN and NT (register-staged tiles with tested loads and both
// halves' fragments read behind one barrier: 61, 50 and 57), tiles of 64 70
// at 4096; 4-byte loads 71 and 65; with the polynomial's epilogue, whose loads
// spill 108 registers a lane, 64.  One workgroup of four 64 x 64 wave tiles
// per SIMD pair keeps two waves per SIMD, so that one's barrier skew hides
// behind the other's MFMAs.  The compiler waits for every outstanding load
// before an LDS read of a struct type (HIP's double2) but not of a vector
// type, so the fragments are read as vectors.
constexpr uint32_t OUT_OF_RANGE = 0x80000000u;

// Workgroup barrier without the memory fence of __syncthreads (the waits
// before it are explicit); the empty asm statements keep the compiler from
// moving LDS accesses across it.
__device__ inline void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
// At most W of this wave's global loads still outstanding, and all its LDS reads done.
template <int W> __device__ inline void wait_loads() {
  __builtin_amdgcn_s_waitcnt((W & 15) | (7 << 4) | (0 << 8) | (((W >> 4) & 3) << 14));
}
template <int CH>
__device__ inline void load_lds(__amdgpu_buffer_rsrc_t r, unsigned char* dst, uint32_t off) {
  auto l = (void __attribute__((address_space(3)))*)dst;
  if constexpr (CH == 16) __builtin_amdgcn_raw_ptr_buffer_load_lds(r, l, 16, off, 0, 0, 0);
  else __builtin_amdgcn_raw_ptr_buffer_load_lds(r, l, 4, off, 0, 0, 0);
}

template <bool TA, bool TB, int EPI, int WI, int WJ, int CH>
__global__ __launch_bounds__(NT, WI * WJ > 8 ? 2 : 4) void gemm_f64_dl(GemmArgs g, int tiles_m, int tiles_n) {
  constexpr int BM = 32 * WI, BN = 32 * WJ, BK = 16, STAGE = 8 * (BM + BN) * BK;  // bytes
  constexpr int NA = BM / (2 * CH), NB = BN / (2 * CH);  // loads per wave and stage
  extern __shared__ __attribute__((aligned(16))) unsigned char f64_lds[];
  int tm, tn;
  tile_coords<EPI>(g, tiles_m, tiles_n, tm, tn);
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wi0 = (wave & 1) * 16 * WI, wj0 = (wave >> 1) * 16 * WJ;
  const int l16 = lane & 15, lq = lane >> 4;
  int64_t kbeg = 0, kend = g.K;
  if (g.krange) {
    const int64_t kt = n0 / GEMM_BN;
    kbeg = g.krange[2 * kt];
    kend = g.krange[2 * kt + 1];
  }
  const bool sym = EPI == EPI_RQ && g.lower_only;  // sum over k < m0 twice, the diagonal block once
  if (sym) kend = m0 + BM < g.K ? m0 + BM : g.K;
  // Byte x of an operand's tile of ROWS rows: [row][k] tiles hold 16 k per
  // 128 bytes with the 16-byte chunks swizzled by the row, [k][row] tiles all
  // rows of one k together (lds_at).  off: its byte offset in global memory
  // from the tile's first element of the stage; k: its k within the stage.
  auto place = [](bool kmajor, int rows, int x, int64_t ld, int64_t limit, uint32_t& off, int& k) {
    int row;
    if (kmajor) {
      row = x / 128;
      const int c = ((x % 128) / 16) ^ (row & 7);
      k = 2 * c + (x % 16) / 8;
      off = (uint32_t)(row * ld * 8 + c * 16 + x % 16);
    } else {
      k = x / (8 * rows);
      row = (x % (8 * rows)) / 8;
      off = (uint32_t)(k * ld * 8 + x % (8 * rows));
    }
    if (row >= limit) off = OUT_OF_RANGE;
  };
  uint32_t oa[NA], ob[NB];
  int ka[NA], kb[NB];
#pragma unroll
  for (int u = 0; u < NA; ++u)
    place(TA, BM, ((NA * wave + u) * 64 + lane) * CH, g.lda, g.M - m0, oa[u], ka[u]);
#pragma unroll
  for (int u = 0; u < NB; ++u)
    place(!TB, BN, ((NB * wave + u) * 64 + lane) * CH, g.ldb, g.N - n0, ob[u], kb[u]);
  const double* pa = g.A + (TA ? m0 * g.lda + kbeg : m0 + kbeg * g.lda);
  const double* pb = g.B + (TB ? n0 + kbeg * g.ldb : n0 * g.ldb + kbeg);
  const int64_t stepa = TA ? BK : BK * g.lda, stepb = TB ? BK * g.ldb : BK;
  auto issue = [&](int64_t t) {
    const int64_t rest = kend - kbeg - t * BK;
    const int left = rest >= BK ? BK : rest > 0 ? (int)rest : 0;
    const auto ra = __builtin_amdgcn_make_buffer_rsrc((void*)(pa + t * stepa), 0, 0x7fffffff, 0x00027000);
    const auto rb = __builtin_amdgcn_make_buffer_rsrc((void*)(pb + t * stepb), 0, 0x7fffffff, 0x00027000);
    unsigned char* dst = f64_lds + (t & 1) * STAGE;
#pragma unroll
    for (int u = 0; u < NA; ++u)
      load_lds<CH>(ra, dst + (NA * wave + u) * 64 * CH, ka[u] < left ? oa[u] : OUT_OF_RANGE);
#pragma unroll
    for (int u = 0; u < NB; ++u)
      load_lds<CH>(rb, dst + 8 * BM * BK + (NB * wave + u) * 64 * CH, kb[u] < left ? ob[u] : OUT_OF_RANGE);
  };
  v4d acc[WI][WJ];
#pragma unroll
  for (int i = 0; i < WI; ++i)
#pragma unroll
    for (int j = 0; j < WJ; ++j) acc[i][j] = (v4d){0.0, 0.0, 0.0, 0.0};
  struct Frags {
    v2d a[WI], b[WJ];
  };
  auto read = [&](int64_t t, int kk, Frags& f) {
    const double* As = (const double*)(f64_lds + (t & 1) * STAGE);
    const double* Bs = As + BM * BK;
    const int k = kk + 2 * lq;
#pragma unroll
    for (int ib = 0; ib < WI; ++ib) {
      const int i = wi0 + ib * 16 + l16;
      if (TA) f.a[ib] = *(const v2d*)&As[lds_at<true, BM, BK>(i, k)];
      else f.a[ib] = (v2d){As[lds_at<false, BM, BK>(i, k)], As[lds_at<false, BM, BK>(i, k + 1)]};
    }
#pragma unroll
    for (int jb = 0; jb < WJ; ++jb) {
      const int j = wj0 + jb * 16 + l16;
      if (!TB) f.b[jb] = *(const v2d*)&Bs[lds_at<true, BN, BK>(j, k)];
      else f.b[jb] = (v2d){Bs[lds_at<false, BN, BK>(j, k)], Bs[lds_at<false, BN, BK>(j, k + 1)]};
    }
  };
  auto mma = [&](const Frags& f) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int ib = 0; ib < WI; ++ib)
#pragma unroll
        for (int jb = 0; jb < WJ; ++jb)
          acc[ib][jb] = __builtin_amdgcn_mfma_f64_16x16x4f64(h ? f.b[jb].y : f.b[jb].x, h ? f.a[ib].y : f.a[ib].x,
                                                             acc[ib][jb], 0, 0, 0);
  };
  constexpr int NM = 2 * WI * WJ, NR = WI + WJ, NL = NA + NB;  // MFMAs per half, fragment reads, loads
  const int64_t ntk = kend > kbeg ? (kend - kbeg + BK - 1) / BK : 0;
  if (ntk > 0) {
    Frags f0, f1;
    issue(0);
    issue(1);
    wait_loads<NL>();  // stage 0 has landed
    lds_barrier();
    read(0, 0, f0);
    for (int64_t t = 0; t < ntk; ++t) {
      if (sym && t * BK == m0) double_acc(acc);
      __builtin_amdgcn_sched_barrier(0);
      read(t, 8, f1);
      mma(f0);
#pragma unroll
      for (int u = 0; u < NR; ++u) {
        __builtin_amdgcn_sched_group_barrier(0x008, NM / (NR + 1), 0);  // MFMA
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);              // LDS read
      }
      __builtin_amdgcn_sched_barrier(0);
      wait_loads<0>();
      lds_barrier();
      issue(t + 2);
      read(t + 1, 0, f0);
      mma(f1);
#pragma unroll
      for (int u = 0; u < NR; ++u) {
        __builtin_amdgcn_sched_group_barrier(0x008, NM / (NR + 1), 0);
        __builtin_amdgcn_sched_group_barrier(0x020, NL / NR, 0);  // global -> LDS loads
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
    }
  }
  wait_loads<0>();
  lds_barrier();  // the epilogue reuses the stages
  f64_epilogue<EPI, WI, WJ>(g, acc, m0, n0, wi0, wj0, tid, tm, (double (*)[BN])f64_lds);
}

// Launch with the tile (32 WI) x (32 WJ).
template <bool TA, bool TB, int WI, int WJ, int BK, typename OFF = uint32_t>
hipError_t launch_epi(int epi, const GemmArgs& a, hipStream_t s) {
  constexpr int BM = 32 * WI, BN = 32 * WJ;
  const int tm = (int)((a.M + BM - 1) / BM), tn = (int)((a.N + BN - 1) / BN);
  if (tm == 0 || tn == 0) return hipSuccess;
  const bool tri = a.lower_only && epi != EPI_RQ;
  if (tri && tm != tn) return hipErrorInvalidValue;
  dim3 grid(tri ? tm * (tm + 1) / 2 : tm * tn), block(NT);
  switch (epi) {
#define F64_CASE(E)                                                                             \
  case E:                                                                                       \
    hipLaunchKernelGGL((gemm_f64_kernel<TA, TB, E, WI, WJ, BK, OFF>), grid, block, 0, s, a, tm, tn); \
    break;
    F64_CASE(EPI_STORE)
    F64_CASE(EPI_SHIFT)
    F64_CASE(EPI_FSUPD)
    F64_CASE(EPI_RQ)
    F64_CASE(EPI_G2S)
    F64_CASE(EPI_POLY)
#undef F64_CASE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <bool TA, bool TB, int WI, int WJ, int CH>
hipError_t launch_dl(int epi, const GemmArgs& a, hipStream_t s) {
  constexpr int BM = 32 * WI, BN = 32 * WJ;
  const int tm = (int)((a.M + BM - 1) / BM), tn = (int)((a.N + BN - 1) / BN);
  if (tm == 0 || tn == 0) return hipSuccess;
  const bool tri = a.lower_only && epi != EPI_RQ;
  if (tri && tm != tn) return hipErrorInvalidValue;
  dim3 grid(tri ? tm * (tm + 1) / 2 : tm * tn), block(NT);
  constexpr size_t lds = 2 * 8 * (BM + BN) * 16;
  switch (epi) {
#define F64_CASE(E)                                                                           \
  case E:                                                                                     \
    hipLaunchKernelGGL((gemm_f64_dl<TA, TB, E, WI, WJ, CH>), grid, block, lds, s, a, tm, tn); \
    break;
    F64_CASE(EPI_STORE)
    F64_CASE(EPI_SHIFT)
    F64_CASE(EPI_FSUPD)
    F64_CASE(EPI_RQ)
    F64_CASE(EPI_G2S)
    F64_CASE(EPI_POLY)
#undef F64_CASE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

// Rows (and columns) of the block tile a product of this size runs with.
// Tiles of 128 reach 74-75 TFLOP/s at order 4096 and 8192, tiles of 64 70; a
// grid of t tiles leaves 1 - t / (256 ceil(t / 256)) of the chip idle, which
// at order 3000 costs the larger tile more (53 against 63 TFLOP/s; 1664: 46
// against 58).  Up to 100 tiles of 64, tiles of 32 spread the product wider
// (order 640: 24.6 against 26.0 us, 256: 8.4 against 12.0 us; at 768, 144
// tiles, 36.7 against 31.0 us).
int gemm_f64_tile(int64_t M, int64_t N, bool lower) {
  constexpr int64_t CUS = 256;
  auto tiles = [&](int64_t b) {
    const int64_t m = (M + b - 1) / b, n = (N + b - 1) / b;
    return lower ? m * (m + 1) / 2 : m * n;
  };
  auto filled = [&](int64_t t) { return (double)t / (double)(CUS * ((t + CUS - 1) / CUS)); };
  const int64_t t128 = tiles(128), t64 = tiles(64);
  if (t64 <= 100) return 32;
  return filled(t128) >= 0.9 * filled(t64) ? 128 : 64;
}

template <bool TA, bool TB>
hipError_t launch_tile(int epi, const GemmArgs& a, hipStream_t s) {
  const bool part = (epi == EPI_RQ || epi == EPI_G2S) && a.part;
  int tile = part && a.part_rows ? a.part_rows : part ? GEMM_BM
                                              : gemm_f64_tile(a.M, a.N, a.lower_only && epi != EPI_RQ);
  if (a.in_place && tile < 64) tile = 64;
  // 16-byte loads need aligned columns and chunks that lie wholly inside or outside the matrix
  const bool wide = (((uintptr_t)a.A | (uintptr_t)a.B) & 15) == 0 && ((a.lda | a.ldb | a.M | a.N | a.K) & 1) == 0;
  if (a.lda >= (int64_t(1) << 21) || a.ldb >= (int64_t(1) << 21)) {
    // offsets within a tile past 31 bits: the kernel with 64-bit ones, whose tile of
    // 128 rows (which part_rows = 128 needs) has 32 columns.  A lower triangle
    // needs square tiles and a product in place all columns in one: those take
    // tiles of 64.
    if (tile == 32) return launch_epi<TA, TB, 1, 1, 32, int64_t>(epi, a, s);
    return tile == 64 || a.in_place || (a.lower_only && epi != EPI_RQ)
               ? launch_epi<TA, TB, 2, 2, 16, int64_t>(epi, a, s)
               : launch_epi<TA, TB, 4, 1, 16, int64_t>(epi, a, s);
  }
  if (tile == 32) return launch_epi<TA, TB, 1, 1, 32>(epi, a, s);
  if (tile == 64) return wide ? launch_dl<TA, TB, 2, 2, 16>(epi, a, s) : launch_dl<TA, TB, 2, 2, 4>(epi, a, s);
  return wide ? launch_dl<TA, TB, 4, 4, 16>(epi, a, s) : launch_dl<TA, TB, 4, 4, 4>(epi, a, s);
}

hipError_t gemm_f64(bool ta, bool tb, int epi, const GemmArgs& a, hipStream_t s) {
  // SHIFT / FSUPD / G2S / POLY read B at output positions: only the non-transposed square case is valid.
  if ((epi == EPI_SHIFT || epi == EPI_FSUPD || epi == EPI_G2S || epi == EPI_POLY) && (tb || a.K < a.M)) return hipErrorInvalidValue;
  if (!ta && !tb) return launch_tile<false, false>(epi, a, s);
  if (ta && !tb) return launch_tile<true, false>(epi, a, s);
  if (!ta && tb) return launch_tile<false, true>(epi, a, s);
  return launch_tile<true, true>(epi, a, s);
}

}  // namespace pfsm

// Device factorisation of the ORAS local matrices B_j (paper sec. 2.2: the
// local matrices are factorised once at set-up; the paper uses a sparse
// direct solver, here the factorisation is rebuilt for the GPU).
//
// A box of sx x sy x sz nodes ordered plane by plane (z slowest) makes B_j
// block tridiagonal with p x p plane blocks (p = sx sy), because the
// 27-point stencil couples a plane only to its two neighbours.  Block
// elimination over the planes gives the Schur complements
//     S_0 = D_0,   S_k = D_k - L_k S_{k-1}^{-1} U_{k-1},
// and the factors kept are the explicit inverses S_k^{-1}.  A solve is then
// two sweeps of dense products (forward y_k = S_k^{-1}(r_k - L_k y_{k-1}),
// backward x_k = y_k - S_k^{-1} U_k x_{k+1}), which map onto MFMA.
//
// Every plane matrix is padded to P = ceil(p / 32) * 32 (identity on the pad)
// and stored as 32 x 32 tiles, tile (I, J) at ((I nt + J) * 1024); inside a
// tile, entry (r, c) sits at ((c / 4) * 32 + r) * 4 + c % 4, so four
// consecutive columns of 16 or 32 consecutive rows form one contiguous run
// (the operand fragment of a 16x16x4 MFMA, and a 4x4 register block).
//
// The inverse is formed in place by blocked Gauss-Jordan elimination with
// pivot blocks of several tiles (no row exchanges; a zero or non-finite pivot
// is reported, and the smallest pivot relative to the plane's largest entry
// is recorded):
//     A_kk <- A_kk^{-1};  A_kJ <- A_kk^{-1} A_kJ;  A_IJ <- A_IJ - A_Ik A_kJ;
//     A_Ik <- -A_Ik A_kk^{-1}.
// B_j is complex symmetric and so is every S_k.  The elimination keeps that
// up to signs: A_JI = A_IJ^T where I and J are both eliminated or both not,
// A_JI = -A_IJ^T otherwise.  So only the tiles with I <= J are kept up to date,
// which halves the trailing update that carries almost all the work, and the
// last pivot block writes the mirror tiles (with every tile updated, 96^3 in 64
// subdomains took 180 ms a factorisation in complex128, now 90; 160^3 in 512
// took 224 ms in complex64, now 113).
#include <type_traits>
#include <utility>

#include "oras_internal.h"

namespace oras {

namespace {

__device__ inline long long tile_off(int I, int J, int nt) {
  return ((long long)I * nt + J) * (TILE * TILE);
}
__device__ inline int in_tile(int r, int c) { return ((c >> 2) * TILE + r) * 4 + (c & 3); }
__device__ inline long long mat_off(int row, int col, int nt) {
  return tile_off(row / TILE, col / TILE, nt) + in_tile(row % TILE, col % TILE);
}

template <typename T> __device__ inline T czero() { T z; z.x = 0; z.y = 0; return z; }
template <typename T> __device__ inline T cone() { T z; z.x = 1; z.y = 0; return z; }

template <typename R> struct Tiny;
template <> struct Tiny<float> { static constexpr float v = 1e-30f; };
template <> struct Tiny<double> { static constexpr double v = 1e-280; };

// T = S_{k-1}^{-1} U_{k-1}:  T[a, c] = sum_d Sinv[a, c - d] U[c - d, c], where
// U[c', c] couples node c' of plane k-1 to node c of plane k.  The couplings
// of the tile's 32 columns are staged in LDS once (every row of the tile uses
// them).
template <typename R>
__global__ void __launch_bounds__(256) schur_T_kernel(const SubDesc* subs, int k, const C<R>* fac,
                                                      C<R>* tbuf, const C<R>* lca) {
  using T = C<R>;
  __shared__ T ucol[9][TILE];
  const SubDesc sd = subs[blockIdx.z];
  if (k == 0 || k >= sd.sz) return;
  const int nt = sd.nt;
  const int I = blockIdx.y, J = blockIdx.x;
  // S_k is symmetric and only its tiles on and above the diagonal are formed:
  // they read T up to one row of the plane below their own rows
  if (I >= nt || J >= nt || I * TILE > J * TILE + TILE + sd.sx) return;
  const long long P2 = (long long)sd.P * sd.P;
  const T* Sinv = fac + sd.fac_off + (long long)(k - 1) * P2;
  T* Tm = tbuf + sd.t_off;
  const long long nbox = (long long)sd.sx * sd.sy * sd.sz;
  const T* L = lca + sd.lca_off;
  for (int i = threadIdx.x; i < 9 * TILE; i += 256) {
    // coupling of column c to its neighbour (c - d) in plane k - 1, d = (dx, dy)
    const int d = i / TILE, c = J * TILE + i % TILE;
    const int dx = d % 3 - 1, dy = d / 3 - 1;
    T u = czero<T>();
    if (c < sd.p) {
      const int px = c % sd.sx - dx, py = c / sd.sx - dy;
      if (px >= 0 && px < sd.sx && py >= 0 && py < sd.sy)
        u = L[eidx(dx, dy, 1) * nbox + ((long long)(k - 1) * sd.sy + py) * sd.sx + px];
    }
    ucol[d][i % TILE] = u;
  }
  __syncthreads();
  // four consecutive columns per thread: per dy they need six consecutive
  // entries of the row, half the loads of one column per thread, which the
  // kernel was bound by (512 subdomains of 576-row planes in FP32 927 -> 516 us
  // a plane, 64 of 800 in FP64 292 -> 245; S_k below 827 -> 500 in FP32).
  // Indices are clamped to the plane: a neighbour outside the box has a zero
  // coupling.
  const int c4 = threadIdx.x >> 5, r = threadIdx.x & 31;
  const T* row = Sinv + tile_off(I, 0, nt) + r * 4;
  T acc[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) acc[j] = czero<T>();
#pragma unroll
  for (int dy = -1; dy <= 1; ++dy) {
    T v[6];
#pragma unroll
    for (int o = 0; o < 6; ++o) {
      const int c = min(max(J * TILE + c4 * 4 - dy * sd.sx + o - 1, 0), sd.P - 1);
      v[o] = row[(c >> 2) * (4 * TILE) + (c & 3)];
    }
#pragma unroll
    for (int dx = -1; dx <= 1; ++dx)
#pragma unroll
      for (int j = 0; j < 4; ++j) cfma(acc[j], v[j + 1 - dx], ucol[(dy + 1) * 3 + dx + 1][c4 * 4 + j]);
  }
  T* out = Tm + tile_off(I, J, nt) + c4 * (4 * TILE) + r * 4;
#pragma unroll
  for (int j = 0; j < 4; ++j) out[j] = acc[j];
}

// S_k = D_k - L_k T  (just D_k on the first plane), identity on the pad: the
// tiles on and above the diagonal (S_k is symmetric).
// stats[2 (sub max_sz + k)] receives the bits of max |S_k|^2 (a non-negative
// double, so its bits order as the value).
// The couplings of the tile's 32 rows to plane k - 1 are staged in LDS once
// (every column of the tile uses them).
template <typename R>
__global__ void __launch_bounds__(256) build_S_kernel(const SubDesc* subs, int k, C<R>* fac,
                                                      const C<R>* tbuf, const C<R>* lca,
                                                      unsigned long long* stats, int max_sz) {
  using T = C<R>;
  __shared__ double red[256];
  __shared__ T lrow[9][TILE];
  const SubDesc sd = subs[blockIdx.z];
  if (k >= sd.sz) return;
  const int nt = sd.nt;
  const int I = blockIdx.y, J = blockIdx.x;
  if (I > J || J >= nt) return;
  double big = 0.0;
  const long long P2 = (long long)sd.P * sd.P;
  T* S = fac + sd.fac_off + (long long)k * P2;
  const T* Tm = tbuf + sd.t_off;
  const long long nbox = (long long)sd.sx * sd.sy * sd.sz;
  const T* L = lca + sd.lca_off;
  if (k > 0) {
    for (int i = threadIdx.x; i < 9 * TILE; i += 256) {
      const int e = i / TILE, b = I * TILE + i % TILE;
      T l = czero<T>();
      if (b < sd.p)
        l = L[eidx(e % 3 - 1, e / 3 - 1, -1) * nbox +
              ((long long)k * sd.sy + b / sd.sx) * sd.sx + b % sd.sx];
      lrow[e][i % TILE] = l;
    }
    __syncthreads();
  }
  // NC consecutive columns per thread: four in FP32 (one run of the tile layout
  // per neighbouring row of T), one in FP64, whose 64-byte run would leave a
  // lane's loads that far apart.  Rows outside the box are clamped, their
  // coupling is zero.
  constexpr int NC = sizeof(R) == 4 ? 4 : 1;
#pragma unroll
  for (int q = 0; q < 4 / NC; ++q) {
    const int e = (threadIdx.x + 256 * q) * NC;
    const int b = I * TILE + ((e >> 2) & 31), c0 = J * TILE + (e >> 7) * 4 + (e & 3);
    T v[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) v[j] = czero<T>();
    if (b < sd.p) {
      const int bx = b % sd.sx, by = b / sd.sx;
      const long long node = ((long long)k * sd.sy + by) * sd.sx + bx;
#pragma unroll
      for (int j = 0; j < NC; ++j) {
        const int c = c0 + j, dx = c % sd.sx - bx, dy = c / sd.sx - by;
        if (c < sd.p && dx >= -1 && dx <= 1 && dy >= -1 && dy <= 1)
          v[j] = L[eidx(dx, dy, 0) * nbox + node];
      }
      if (k > 0) {
#pragma unroll
        for (int ey = -1; ey <= 1; ++ey)
#pragma unroll
          for (int ex = -1; ex <= 1; ++ex) {
            const int n = min(max(by + ey, 0), sd.sy - 1) * sd.sx + min(max(bx + ex, 0), sd.sx - 1);
            const T* t = Tm + mat_off(n, c0, nt);
            const T l = lrow[(ey + 1) * 3 + ex + 1][(e >> 2) & 31];
#pragma unroll
            for (int j = 0; j < NC; ++j) cfms(v[j], l, t[j]);
          }
      }
    }
    T* out = S + tile_off(I, J, nt) + e;
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const int c = c0 + j;
      if (b < sd.p && c < sd.p) big = fmax(big, (double)v[j].x * v[j].x + (double)v[j].y * v[j].y);
      else v[j] = b == c ? cone<T>() : czero<T>();
      out[j] = v[j];
    }
  }
  red[threadIdx.x] = big;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x == 0 && red[0] > 0.0)
    atomicMax(&stats[2 * ((long long)blockIdx.z * max_sz + k)],
              (unsigned long long)__double_as_longlong(red[0]));
}

// ------------------------------------------------------- blocked Gauss-Jordan
// Pivot blocks of NBT tiles (32 NBT rows); the last block of a plane may be
// narrower.  Every pass reads and writes the whole plane matrix once, so wide
// blocks cut the HBM traffic of the inversion; NBT is what fits the pivot
// block in LDS (128 x 128 FP32, 64 x 64 FP64).
template <typename R> struct GjBlock;
template <> struct GjBlock<float> { static constexpr int NBT = 4, WAVES = 16; };
template <> struct GjBlock<double> { static constexpr int NBT = 2, WAVES = 8; };

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// 16 x 16 x 4 products in the precision itself: A[row = l % 16][k = l / 16],
// B[k = l / 16][col = l % 16]; result item i of lane l is column l % 16 and row
// l / 16 + 4 i (FP64) or 4 (l / 16) + i (FP32).
template <typename R> struct Mma16;
template <> struct Mma16<double> {
  typedef f64x4 V;
  static __device__ V mac(double a, double b, V c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ int row(int kk, int i) { return kk + 4 * i; }
};
template <> struct Mma16<float> {
  typedef f32x4 V;
  static __device__ V mac(float a, float b, V c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ int row(int kk, int i) { return 4 * kk + i; }
};

// lane N of each 16 lanes, to all 16 of them (DPP row broadcast)
template <int N> __device__ inline float row_bcast(float v) {
  return __int_as_float(
      __builtin_amdgcn_mov_dpp(__float_as_int(v), 0x150 + N, 0xf, 0xf, false));
}
template <int N> __device__ inline double row_bcast(double v) {
  const long long u = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)(u & 0xffffffffLL), 0x150 + N, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_mov_dpp((int)(u >> 32), 0x150 + N, 0xf, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// the 16 lanes G of a wave, to each 16 lanes of it
template <int G> __device__ inline unsigned group_bcast(unsigned v) {
  const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);    // groups 0 0 2 2, 1 1 3 3
  const unsigned w = a[G & 1];
  const auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false);    // the lower, the upper
  return b[G >> 1];
}
template <int G> __device__ inline float group_bcast(float v) {
  return __uint_as_float(group_bcast<G>(__float_as_uint(v)));
}
template <int G> __device__ inline double group_bcast(double v) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const unsigned long long lo = group_bcast<G>((unsigned)u), hi = group_bcast<G>((unsigned)(u >> 32));
  return __longlong_as_double((long long)(hi << 32 | lo));
}
// lane L's value, uniform
template <int L> __device__ inline float lane_value(float v) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), L));
}
template <int L> __device__ inline double lane_value(double v) {
  const long long u = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(u & 0xffffffffLL), L);
  const int hi = __builtin_amdgcn_readlane((int)(u >> 32), L);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Between LDS stores of a wave's lanes and accesses of the same bytes by its
// other lanes.  A wave's LDS operations complete in order, so this costs no
// wait: it keeps the compiler from moving them past each other, which the types
// of the accesses or the address of a single lane may seem to allow.
__device__ inline void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int... I, typename F>
__device__ inline void static_for_impl(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>()), ...);
}
// f(integral_constant<int, i>) for i = 0 .. N - 1, unrolled at compile time
template <int N, typename F> __device__ inline void static_for(F&& f) {
  static_for_impl(std::make_integer_sequence<int, N>(), f);
}

// A = L D L^T of a symmetric 16 x 16 block at m (row stride ld; its upper triangle
// is read) by one wave: W = L^{-1} to w (row stride 17) and D^{-1} to d.
// Unblocked elimination in registers, lane (r = l % 16, g = l / 16) holding row
// r, columns 4 g .. 4 g + 3, of what is left of A right of the pivot and of W left
// of it; the pivot row comes by DPP, the pivot column by lane swaps, the pivot by
// a lane read, so no pivot step waits at a barrier or for LDS.  The smallest
// |pivot|^2 of the first `count` pivots goes to mag_min, a zero or non-finite one
// to bad.
template <typename R>
__device__ inline void factor16(const C<R>* m, int ld, C<R>* w, C<R>* d, int count, R& mag_min,
                                bool& bad) {
  using T = C<R>;
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));   // its comparisons are not kept from call to call (spills)
  const int r = lane & 15, g = lane >> 4;
  T a[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) a[j] = m[min(r, 4 * g + j) * ld + max(r, 4 * g + j)];
  static_for<16>([&](auto P) {
    constexpr int piv = decltype(P)::value, pg = piv / 4, pj = piv % 4;
    T p;
    p.x = lane_value<16 * pg + piv>(a[pj].x);
    p.y = lane_value<16 * pg + piv>(a[pj].y);
    T rv[4], cv;
    cv.x = group_bcast<pg>(a[pj].x);
    cv.y = group_bcast<pg>(a[pj].y);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      rv[j].x = row_bcast<piv>(a[j].x);
      rv[j].y = row_bcast<piv>(a[j].y);
    }
    const R mag = p.x * p.x + p.y * p.y;
    const bool ok = isfinite(p.x) & isfinite(p.y) & (mag > Tiny<R>::v);
    bad |= !ok;
    mag_min = ok & (piv < count) & (mag < mag_min) ? mag : mag_min;
    const R inv = (R)1 / mag;
    T f;                                             // A_r,piv / p below the pivot, else 0
    f.x = r > piv ? (cv.x * p.x + cv.y * p.y) * inv : (R)0;
    f.y = r > piv ? (cv.y * p.x - cv.x * p.y) * inv : (R)0;
#pragma unroll
    for (int j = 0; j < 4; ++j) cfms(a[j], f, rv[j]);
    if (g == pg && r > piv) {                        // W_r,piv
      a[pj].x = -f.x;
      a[pj].y = -f.y;
    }
  });
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int c = 4 * g + j;
    w[r * 17 + c] = c < r ? a[j] : (c == r ? cone<T>() : czero<T>());
    if (c == r) {                                    // the pivot
      const R inv = (R)1 / (a[j].x * a[j].x + a[j].y * a[j].y);
      d[r].x = a[j].x * inv;
      d[r].y = -a[j].y * inv;
    }
  }
}

// Products of one wave's 16 x 16 blocks in LDS.  Every operand is read before a
// result is written, so the result may take the place of any of them.
template <typename R> struct Block {
  C<R>* p;
  int ld;        // row stride
  __device__ C<R>& operator()(int r, int c) const { return p[r * ld + c]; }
};
// acc += sign X Y
template <typename R, typename FX, typename FY>
__device__ inline void block_mac(typename Mma16<R>::V& re, typename Mma16<R>::V& im, R sign, FX X,
                                 FY Y) {
  using M = Mma16<R>;
  const int m = threadIdx.x & 15, kk = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const C<R> x = X(m, 4 * q + kk), y = Y(4 * q + kk, m);
    const R xr = sign * x.x, xi = sign * x.y;
    re = M::mac(xr, y.x, re);
    im = M::mac(xr, y.y, im);
    re = M::mac(-xi, y.y, re);
    im = M::mac(xi, y.x, im);
  }
}
// A <- W A
template <typename R> __device__ inline void block_w(Block<R> A, Block<R> W) {
  using M = Mma16<R>;
  const int m = threadIdx.x & 15, kk = (threadIdx.x & 63) >> 4;
  typename M::V re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
  block_mac<R>(re, im, (R)1, W, A);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    C<R> v;
    v.x = re[i];
    v.y = im[i];
    A(M::row(kk, i), m) = v;
  }
}
// A <- A + sign X^T D Y with D diagonal (SUM; its transpose times msign also to
// mirror if that is not null), or (X^T D Y)^T times msign to mirror.
template <typename R, bool SUM>
__device__ inline void block_tdy(Block<R> A, R sign, Block<R> X, const C<R>* d, Block<R> Y,
                                 C<R>* mirror, R msign) {
  using T = C<R>;
  using M = Mma16<R>;
  const int m = threadIdx.x & 15, kk = (threadIdx.x & 63) >> 4;
  typename M::V re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
  if (SUM) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      re[i] = A(M::row(kk, i), m).x;
      im[i] = A(M::row(kk, i), m).y;
    }
  }
  block_mac<R>(re, im, sign, [&](int row, int k) { return cmul(X(k, row), d[k]); }, Y);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    T v;
    v.x = re[i];
    v.y = im[i];
    if (SUM) A(M::row(kk, i), m) = v;
    if (mirror) {
      v.x *= msign;
      v.y *= msign;
      mirror[m * A.ld + M::row(kk, i)] = v;
    }
  }
}

// A_kk <- A_kk^{-1} for the pivot block (nb tiles from tile kb0), by blocked
// Gauss-Jordan over 16 x 16 blocks of the matrix in LDS, one work-group per
// subdomain.  It is a chain (few work-groups, every other kernel of the plane
// waits for it), so what counts is the length of a step: wave 0 updates and
// factors the next diagonal block in registers, ahead of the other waves in
// instruction priority, while those finish the step, and the products run on
// the matrix unit.  The matrix stays symmetric but for the sign between
// eliminated and other blocks, so of A_ij and A_ji one is computed.
//
// A diagonal block enters as L D L^T, not as its inverse: with W = L^{-1} and
// Y_j = W A_bj the update is A_ij -= +- Y_i^T D^{-1} Y_j and the block row W^T
// D^{-1} Y_j.  Where a block is a large multiple s of a rank-one matrix plus a
// rest (the plane before it was nearly singular), products with its inverse
// leave eps s^2 in the result, those with L and D eps s, as elimination row by
// row does (complex64 solve of a box of 18 x 23 x 37 nodes: error 4.7e-3, 3.6e-5
// and 5.4e-5).  Only the upper triangle of a diagonal block is read: with both,
// equal but for rounding, block row and column would belong to different
// matrices, which near a small pivot p leaves eps / p^2 (boxes of 11 x 35 x 3
// nodes: up to 2.3e-3, 7e-5 with one).
//
// 64 complex FP64 rows 28 us a call: 64 pivots of 0.27 (about 25 dependent FP64
// instructions each), the rest are products, loads and stores; as much with
// explicit inverses, 75 for 64 pivot steps with two barriers each.  128 complex
// FP32 rows on 64 subdomains, beside other kernels, 51 us (48 with inverses).  A
// factorisation of 32^3 in 8 subdomains, which little else but this chain keeps
// waiting, 6.4 ms in FP64 and 4.2 in FP32 (6.4, 4.1 with inverses).
//
// stats[2 (sub max_sz + k) + 1] receives the bits of max 1 / |pivot|^2.
template <typename R>
__global__ void __launch_bounds__(64 * GjBlock<R>::WAVES)
gj_diag_kernel(const SubDesc* subs, int k, int kb0, C<R>* fac, int* status,
               unsigned long long* stats, int max_sz) {
  using T = C<R>;
  constexpr int NB = TILE * GjBlock<R>::NBT, LD = NB + 1, WAVES = GjBlock<R>::WAVES;
  __shared__ __align__(16) T A[NB * LD];      // 132 KB FP32, 65 KB FP64
  __shared__ __align__(16) T wbuf[2][16 * 17], dbuf[2][16];   // W and D^{-1} of a diagonal block
  const SubDesc sd = subs[blockIdx.x];
  if (k >= sd.sz || kb0 >= sd.nt) return;
  const int nb = min(GjBlock<R>::NBT, sd.nt - kb0);
  const int nblk = nb * TILE / 16;
  T* base = fac + sd.fac_off + (long long)k * sd.P * sd.P;
  const int wv = threadIdx.x >> 6;
  auto at = [&](int bi, int bj) { return Block<R>{A + 16 * (bi * LD + bj), LD}; };
  // tiles on and above the diagonal, all loads in flight at once
  constexpr int TT = TILE * TILE, NTHR = 64 * WAVES, TILES = GjBlock<R>::NBT * (GjBlock<R>::NBT + 1) / 2;
  constexpr int NLOAD = (TILES * TT + NTHR - 1) / NTHR;
  T v[NLOAD];
#pragma unroll
  for (int n = 0; n < NLOAD; ++n) {
    const int i = n * NTHR + threadIdx.x, t = i / TT;
    const int tj = (t > 0) + (t > 2) + (t > 5), ti = t - tj * (tj + 1) / 2;
    v[n] = tj < nb ? base[tile_off(kb0 + ti, kb0 + tj, sd.nt) + i % TT] : czero<T>();
  }
#pragma unroll
  for (int n = 0; n < NLOAD; ++n) {
    const int i = n * NTHR + threadIdx.x, t = i / TT, e = i % TT;
    const int tj = (t > 0) + (t > 2) + (t > 5), ti = t - tj * (tj + 1) / 2;
    const int row = ti * TILE + ((e >> 2) & 31), col = tj * TILE + (e >> 7) * 4 + (e & 3);
    if (tj >= nb || row > col) continue;
    A[row * LD + col] = v[n];
    A[col * LD + row] = v[n];
  }
  __syncthreads();
  R mag_min = INFINITY;    // smallest |pivot|^2 seen (wave 0)
  bool bad = false;
  const int live = sd.p - TILE * kb0;     // pivots that are not padding
  // Between steps, block row b - 1 holds the Y_j of its step and block column
  // b - 1 the values of both.
  for (int b = -1; b < nblk; ++b) {
    const Block<R> W{wbuf[b & 1], 17};
    const T* d = dbuf[b & 1];
    // block row b <- Y_j = W A_bj
    for (int j = wv; j < nblk && b >= 0; j += WAVES)
      if (j != b) block_w<R>(at(b, j), W);
    __syncthreads();
    // wave 0: the next diagonal block and its factors; the rest: the other blocks
    // of the update, one of (i, j) and (j, i) each, for b - 1 the one in column
    // b - 1, then block column b, the transposed row W^T D^{-1} Y_j, and the
    // inverse of the diagonal block
    const bool ahead = b + 1 < nblk;
    if (ahead && wv == 0) {
      __builtin_amdgcn_s_setprio(3);
      if (b >= 0)
        block_tdy<R, true>(at(b + 1, b + 1), (R)-1, at(b, b + 1), d, at(b, b + 1), nullptr, (R)1);
      wave_lds_sync();
      factor16<R>(at(b + 1, b + 1).p, LD, wbuf[(b + 1) & 1], dbuf[(b + 1) & 1],
                  live - 16 * (b + 1), mag_min, bad);
      __builtin_amdgcn_s_setprio(0);
    } else if (b >= 0) {
      const int first = ahead ? wv - 1 : wv, step = ahead ? WAVES - 1 : WAVES;
      const int pairs = nblk * (nblk - 1) / 2;
      for (int t = first; t < pairs + nblk; t += step) {
        if (t >= pairs) {
          const int j = t - pairs;
          block_tdy<R, false>(at(j, b), (R)1, W, d, j == b ? W : at(b, j), at(j, b).p,
                              j <= b ? (R)1 : (R)-1);
          continue;
        }
        int j = 0;
        while ((j + 1) * (j + 2) / 2 <= t) ++j;
        int i = t - j * (j + 1) / 2;       // i <= j of the nblk - 1 blocks but b
        i += i >= b;
        j += j >= b;
        if (ahead && i == b + 1 && j == b + 1) continue;
        if (i == b - 1) {
          i = j;
          j = b - 1;
        }
        block_tdy<R, true>(at(i, j), i < b ? (R)1 : (R)-1, at(b, i), d, at(b, j),
                           i == j ? nullptr : at(j, i).p, (i <= b) == (j <= b) ? (R)1 : (R)-1);
      }
    }
    __syncthreads();
  }
  // the last block row: the transposed last column
  for (int i = threadIdx.x; i < (nblk - 1) * 256; i += 64 * WAVES)
    at(nblk - 1, i >> 8)(i & 15, (i >> 4) & 15) = at(i >> 8, nblk - 1)((i >> 4) & 15, i & 15);
  __syncthreads();
  for (int i = threadIdx.x; i < nb * nb * TILE * TILE; i += 64 * WAVES) {
    const int t = i / (TILE * TILE), e = i % (TILE * TILE);
    const int row = t / nb * TILE + ((e >> 2) & 31), col = t % nb * TILE + (e >> 7) * 4 + (e & 3);
    base[tile_off(kb0 + t / nb, kb0 + t % nb, sd.nt) + e] = A[row * LD + col];
  }
  // largest 1 / |pivot|^2 over the block's pivots
  const double inv_min = mag_min < INFINITY ? 1.0 / (double)mag_min : 0.0;
  if (threadIdx.x == 0 && bad) status[blockIdx.x] = 1;
  if (threadIdx.x == 0 && inv_min > 0.0)
    atomicMax(&stats[2 * ((long long)blockIdx.x * max_sz + k) + 1],
              (unsigned long long)__double_as_longlong(inv_min));
}
typedef float f32x16 __attribute__((ext_vector_type(16)));

// A tile in LDS: the tile layout with each group of four columns moved on by
// four entries, so that the lanes of a row (8 or 4 such groups) read different
// banks.
constexpr int LTILE = TILE / 4 * (TILE * 4 + 4);
__device__ inline int lds_tile(int r, int c) { return (c >> 2) * (TILE * 4 + 4) + r * 4 + (c & 3); }
// the LDS place of entry e of the tile layout
__device__ inline int lds_entry(int e) { return e + (e >> 7) * 4; }

// One wave's 32 x 32 complex tile product on MFMA: acc += X Y with X a 32 x 32
// tile in memory (tile layout, fetched into registers) and Y one in LDS in the
// form OPERAND (OPERAND_BYTES), written from memory by the four waves of a
// work-group together (fetch_y, stage_y) or from registers (put).
// The instruction forms Y^T X^T, whose lanes hold a row of the result in runs of
// consecutive columns: whole lines of the tile layout per load and store (with
// X Y a lane held a column, 32-byte pieces of sixteen lines per instruction).
// visit(row, col, value) walks the lane's 16 entries of the result.
template <typename R> struct TileMma;

// Complex FP32 on the bf16 instruction (32x32x16) with exactly split operands
// (three bf16 pieces per FP32 value, six piece products per real product:
// FP32-level error).  The real and imaginary parts of the result are separate
// accumulators, Re += Xr Yr - Xi Yi, Im += Xr Yi + Xi Yr.  Per 16-k half tile
// a lane (r = l % 32, g = l / 32) holds X entries (r, 4 q + 2 g + e) of the
// tile layout (four float4 loads, q = 0..3, e = 0..1) and the Y entries
// (4 q + 2 g + e, r) of column r, so value i = 2 q + e of both operands refers
// to the same k.  Y is kept split: per half tile six blocks (pieces 1 - 3 of the
// real part, of the imaginary part) of one 16-byte group per lane.
template <> struct TileMma<float> {
  static constexpr int OPERAND_BYTES = 12 * 64 * 16, NX = 8;
  f32x16 accR, accI;
  float4 x[8];
  float2 y[4];
  __device__ void zero() {
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      accR[j] = 0.f;
      accI[j] = 0.f;
    }
  }
  __device__ void fetch_x(const float2* __restrict__ X, int q0 = 0, int q1 = 8) {
    const int lane = threadIdx.x & 63;
    const float4* X4 = reinterpret_cast<const float4*>(X) + (lane & 31) * 2 + (lane >> 5);
#pragma unroll
    for (int q = q0; q < q1; ++q) x[q] = X4[q * 64];
  }
  // wave w: half tile w % 2, values 4 (w / 2) .. + 3 of each lane
  __device__ void fetch_y(const float2* __restrict__ Y) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      y[j] = Y[in_tile(16 * (w & 1) + 8 * (w >> 1) + 4 * (j >> 1) + 2 * (lane >> 5) + (j & 1),
                       lane & 31)];
  }
  __device__ void stage_y(void* lds) const { put(lds, threadIdx.x >> 6, y); }
  static __device__ void put(void* lds, int w, const float2 (&v)[4]) {
    unsigned pr[3][2], pi[3][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      split3(v[2 * h].x, v[2 * h + 1].x, pr[0][h], pr[1][h], pr[2][h]);
      split3(v[2 * h].y, v[2 * h + 1].y, pi[0][h], pi[1][h], pi[2][h]);
    }
    uint2* o = reinterpret_cast<uint2*>(lds) + ((w & 1) * 6 * 64 + (threadIdx.x & 63)) * 2 + (w >> 1);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      o[q * 128] = make_uint2(pr[q][0], pr[q][1]);
      o[(3 + q) * 128] = make_uint2(pi[q][0], pi[q][1]);
    }
  }
  // fetch(i0, i1) is called as x[i0 .. i1) comes free
  template <typename F> __device__ void mac(const void* lds, F fetch) {
    const u32x4* Y = reinterpret_cast<const u32x4*>(lds) + (threadIdx.x & 63);
    const u32x4 sgn = {0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u};
#pragma unroll
    for (int hj = 0; hj < 2; ++hj) {
      unsigned r1[4], r2[4], r3[4], i1[4], i2[4], i3[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        split3(x[4 * hj + q].x, x[4 * hj + q].z, r1[q], r2[q], r3[q]);
        split3(x[4 * hj + q].y, x[4 * hj + q].w, i1[q], i2[q], i3[q]);
      }
      fetch(4 * hj, 4 * hj + 4);
      const bf16x8 Xr1 = as_bf16x8(u32x4{r1[0], r1[1], r1[2], r1[3]});
      const bf16x8 Xr2 = as_bf16x8(u32x4{r2[0], r2[1], r2[2], r2[3]});
      const bf16x8 Xr3 = as_bf16x8(u32x4{r3[0], r3[1], r3[2], r3[3]});
      const bf16x8 Xi1 = as_bf16x8(u32x4{i1[0], i1[1], i1[2], i1[3]});
      const bf16x8 Xi2 = as_bf16x8(u32x4{i2[0], i2[1], i2[2], i2[3]});
      const bf16x8 Xi3 = as_bf16x8(u32x4{i3[0], i3[1], i3[2], i3[3]});
      const bf16x8 Xn1 = as_bf16x8(u32x4{i1[0], i1[1], i1[2], i1[3]} ^ sgn);
      const bf16x8 Xn2 = as_bf16x8(u32x4{i2[0], i2[1], i2[2], i2[3]} ^ sgn);
      const bf16x8 Xn3 = as_bf16x8(u32x4{i3[0], i3[1], i3[2], i3[3]} ^ sgn);
      const bf16x8 Yr1 = as_bf16x8(Y[(6 * hj + 0) * 64]), Yr2 = as_bf16x8(Y[(6 * hj + 1) * 64]);
      const bf16x8 Yr3 = as_bf16x8(Y[(6 * hj + 2) * 64]), Yi1 = as_bf16x8(Y[(6 * hj + 3) * 64]);
      const bf16x8 Yi2 = as_bf16x8(Y[(6 * hj + 4) * 64]), Yi3 = as_bf16x8(Y[(6 * hj + 5) * 64]);
#define ORAS_X3(XR, XI, XN, YR, YI)                                              \
  accR = __builtin_amdgcn_mfma_f32_32x32x16_bf16(YR, XR, accR, 0, 0, 0);         \
  accI = __builtin_amdgcn_mfma_f32_32x32x16_bf16(YI, XR, accI, 0, 0, 0);         \
  accR = __builtin_amdgcn_mfma_f32_32x32x16_bf16(YI, XN, accR, 0, 0, 0);         \
  accI = __builtin_amdgcn_mfma_f32_32x32x16_bf16(YR, XI, accI, 0, 0, 0);
      ORAS_X3(Xr1, Xi1, Xn1, Yr1, Yi1)
      ORAS_X3(Xr1, Xi1, Xn1, Yr2, Yi2)
      ORAS_X3(Xr2, Xi2, Xn2, Yr1, Yi1)
      ORAS_X3(Xr1, Xi1, Xn1, Yr3, Yi3)
      ORAS_X3(Xr3, Xi3, Xn3, Yr1, Yi1)
      ORAS_X3(Xr2, Xi2, Xn2, Yr2, Yi2)
#undef ORAS_X3
    }
  }
  // accumulator item i of lane l: row l % 32, column 8 (i / 4) + 4 (l / 32) + i % 4
  template <typename F> __device__ void visit(F f) const {
    const int lane = threadIdx.x & 63, rr = lane & 31, g = lane >> 5;
#pragma unroll
    for (int i = 0; i < 16; ++i) f(rr, 8 * (i / 4) + 4 * g + (i % 4), make_float2(accR[i], accI[i]));
  }
};

// Complex FP64 on the 16x16x4 FP64 instruction: two 16-row halves x two
// 16-column halves, the real and imaginary parts of the result in separate
// accumulators.  Y is kept as the tile with padded column groups (lds_tile).
template <> struct TileMma<double> {
  static constexpr int OPERAND_BYTES = LTILE * (int)sizeof(double2), NX = 16;
  f64x4 acc[2][2][2];
  double2 x[16], y[4];
  __device__ void zero() {
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i >> 2][(i >> 1) & 1][i & 1] = f64x4{0, 0, 0, 0};
  }
  __device__ void fetch_x(const double2* __restrict__ X, int i0 = 0, int i1 = 16) {
    const int lane = threadIdx.x & 63, m = lane & 15, kk = lane >> 4;
#pragma unroll
    for (int i = i0; i < i1; ++i) x[i] = X[((i >> 1) * TILE + 16 * (i & 1) + m) * 4 + kk];
  }
  __device__ void fetch_y(const double2* __restrict__ Y) {
#pragma unroll
    for (int j = 0; j < 4; ++j) y[j] = Y[threadIdx.x + 256 * j];
  }
  __device__ void stage_y(void* lds) const {
    double2* o = reinterpret_cast<double2*>(lds);
#pragma unroll
    for (int j = 0; j < 4; ++j) o[lds_entry(threadIdx.x + 256 * j)] = y[j];
  }
  template <typename F> __device__ void mac(const void* lds, F fetch) {
    const double2* Y = reinterpret_cast<const double2*>(lds);
    const int lane = threadIdx.x & 63, m = lane & 15, kk = lane >> 4;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      double2 v[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) v[h] = Y[lds_tile(4 * q + kk, 16 * h + m)];
#pragma unroll
      for (int rs = 0; rs < 2; ++rs)
#pragma unroll
        for (int ns = 0; ns < 2; ++ns) {
          const double2 u = x[2 * q + rs];
          f64x4 &re = acc[rs][ns][0], &im = acc[rs][ns][1];
          re = __builtin_amdgcn_mfma_f64_16x16x4f64(v[ns].x, u.x, re, 0, 0, 0);
          im = __builtin_amdgcn_mfma_f64_16x16x4f64(v[ns].y, u.x, im, 0, 0, 0);
          re = __builtin_amdgcn_mfma_f64_16x16x4f64(v[ns].y, -u.y, re, 0, 0, 0);
          im = __builtin_amdgcn_mfma_f64_16x16x4f64(v[ns].x, u.y, im, 0, 0, 0);
        }
      fetch(2 * q, 2 * q + 2);
    }
  }
  template <typename F> __device__ void visit(F f) const {
    const int lane = threadIdx.x & 63, m = lane & 15, kk = lane >> 4;
#pragma unroll
    for (int rs = 0; rs < 2; ++rs)
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int ns = 0; ns < 2; ++ns)
          f(rs * 16 + m, 16 * ns + kk + 4 * t,
            make_double2(acc[rs][ns][0][t], acc[rs][ns][1][t]));
  }
};

// The panels of one pivot block, for one tile index J outside it (one
// work-group of NBT waves per (J, subdomain)): wave t writes
//   C_J,t  the old A_Jk (tile t of the row, the update's left operand) to the
//          plane's scratch: nb tiles for each of the nt - nb tile indices
//          outside the block, then the W tiles of the kb0 before it.  That is
//          at most 2 (nt - nb) nb <= nt^2 / 2 tiles, so they fit where T was.
//   W_J,t  the new A_kJ = A_kk^{-1} A_kJ (the update's right operand) to its
//          place for J after the pivot block; for J before it, whose place
//          holds the transposed tile (J, kb0 + t), to both.
// The last pivot block of a plane also writes the tile's mirror.  All loads of a
// wave's tile are in flight at once: 26 us a call (29 with four) on 32
// subdomains of 800 rows in FP64, a factorisation of 160^3 in FP32 118 ms (122).
template <typename R>
__global__ void __launch_bounds__(64 * GjBlock<R>::NBT)
gj_panel_kernel(const SubDesc* subs, int k, int kb0, C<R>* fac, C<R>* tbuf) {
  using T = C<R>;
  using M = TileMma<R>;
  constexpr int NBT = GjBlock<R>::NBT, TT = TILE * TILE;
  __shared__ __align__(16) unsigned char lds[NBT][M::OPERAND_BYTES];
  const SubDesc sd = subs[blockIdx.y];
  const int J = blockIdx.x;
  if (k >= sd.sz || kb0 >= sd.nt || J >= sd.nt) return;
  const int nb = min(NBT, sd.nt - kb0);
  if (J >= kb0 && J < kb0 + nb) return;
  const bool after = J > kb0, last = kb0 + nb == sd.nt;
  T* base = fac + sd.fac_off + (long long)k * sd.P * sd.P;
  T* Cs = tbuf + sd.t_off + (long long)(after ? J - nb : J) * nb * TT;
  T* Ws = tbuf + sd.t_off + (long long)(sd.nt - nb + J) * nb * TT;
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  M mm;
  if (wv < nb) {
    const T* g = base + (after ? tile_off(kb0 + wv, J, sd.nt) : tile_off(J, kb0 + wv, sd.nt));
    T* sY = reinterpret_cast<T*>(lds[wv]);
    T ld[TT / 64];       // all loads of the tile in flight
#pragma unroll
    for (int i = 0; i < TT / 64; ++i) ld[i] = g[i * 64 + lane];
#pragma unroll
    for (int i = 0; i < TT / 64; ++i) {
      // entry e of the tile: row r, column c
      const int e = i * 64 + lane, r = (e >> 2) & 31, c = (e >> 7) * 4 + (e & 3);
      T v = ld[i];
      Cs[wv * TT + (after ? in_tile(c, r) : e)] = v;
      if (!after) {        // eliminated before: A_kJ = -A_Jk^T
        v.x = -v.x;
        v.y = -v.y;
      }
      sY[after ? lds_tile(r, c) : lds_tile(c, r)] = v;
    }
    if constexpr (sizeof(R) == 4) {
      // the wave's own tile: columns into registers, then split in its place
      float2 v[4][4];
      wave_lds_sync();
#pragma unroll
      for (int w = 0; w < 4; ++w)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          v[w][j] = sY[lds_tile(16 * (w & 1) + 8 * (w >> 1) + 4 * (j >> 1) + 2 * (lane >> 5) + (j & 1),
                                lane & 31)];
      wave_lds_sync();
#pragma unroll
      for (int w = 0; w < 4; ++w) M::put(sY, w, v[w]);
    }
  }
  __syncthreads();
  if (wv >= nb) return;
  mm.zero();
  const T* D = base + tile_off(kb0 + wv, kb0, sd.nt);
  mm.fetch_x(D);
  for (int u = 0; u < nb - 1; ++u) {
    const T* next = D + (u + 1) * TT;
    mm.mac(lds[u], [&](int i0, int i1) { mm.fetch_x(next, i0, i1); });
    asm volatile("" ::: "memory");      // keeps the fetch in this iteration
  }
  mm.mac(lds[nb - 1], [](int, int) {});
  T* lo = base + tile_off(kb0 + wv, J, sd.nt);     // its place, or the mirror of it
  T* up = base + tile_off(J, kb0 + wv, sd.nt);
  mm.visit([&](int row, int col, T v) {
    if (!after) {
      Ws[wv * TT + in_tile(row, col)] = v;
      up[in_tile(col, row)] = v;
    }
    if (after || last) lo[in_tile(row, col)] = v;
  });
}

// A_IJ <- A_IJ - C_I W_J (I <= J, both outside the pivot block): one wave per
// tile, four row tiles I of a column J per work-group.  Per pivot tile u the
// four waves stage W_J,u in LDS together (two buffers, one barrier per u; in
// FP32 already split for the products) and each reads its C_I,u from memory;
// both of the next u are fetched while the current one feeds the products.
// Work-group ids are mapped so that all tiles of one subdomain run on the same
// XCD and read the panels from its L2.  The last pivot block of a plane also
// writes the mirror tile.
// On 512 subdomains of 576-row planes in FP32 a call takes 398 us (429 with one
// wave per work-group that staged and split W for itself), of which the tiles'
// own traffic is 170 and the matrix unit 134; on 64 of 800-row planes in FP64
// 171, of which either is about 100.  The tile itself is fetched into the
// registers that the last products free, and nothing is fetched past the last
// pivot tile: with two halves of the subdomains side by side, 32 of 800 rows in
// FP64 take 82 us a call (89 with a fetch in every step and the tile read after
// the products), a factorisation of 96^3 in FP64 90 ms (96), of 160^3 in FP32
// 113 (118).  Four columns per work-group, to amortise
// its start, changed nothing in FP32 and spilled in FP64 (206).
constexpr int NXCD = 8;
constexpr int UW = 4;      // waves, row tiles, of an update work-group
// Work-groups of nt tile columns: column J has J / UW + 1 groups of row tiles,
// column a UW + b starts at (a + 1) (a UW / 2 + b).
__host__ __device__ inline int update_items(int nt) {
  const int a = nt / UW, b = nt % UW;
  return (a + 1) * (a * UW / 2 + b);
}
template <typename R>
__global__ void __launch_bounds__(64 * UW) __attribute__((amdgpu_waves_per_eu(sizeof(R) == 4 ? 3 : 2)))
gj_update_kernel(const SubDesc* subs, int nsub, int max_nt, int k, int kb0, C<R>* fac,
                 const C<R>* tbuf) {
  using T = C<R>;
  using M = TileMma<R>;
  constexpr int NBT = GjBlock<R>::NBT, TT = TILE * TILE;
  __shared__ __align__(16) unsigned char lds[2][M::OPERAND_BYTES];
  const int bid = blockIdx.x, r = bid / NXCD, items = update_items(max_nt);
  const int sub = (r / items) * NXCD + bid % NXCD, item = r % items;
  if (sub >= nsub) return;
  const SubDesc sd = subs[sub];
  // item -> column J = UW a + b and row group g
  int a = (int)((sqrtf(1.f + 8.f * item / UW) - 1.f) * 0.5f);
  a += update_items((a + 1) * UW) <= item;
  a -= update_items(a * UW) > item;
  const int rest = item - update_items(a * UW), J = UW * a + rest / (a + 1), g = rest % (a + 1);
  if (k >= sd.sz || kb0 >= sd.nt || J >= sd.nt) return;
  const int nb = min(NBT, sd.nt - kb0);
  if (J >= kb0 && J < kb0 + nb) return;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), I = UW * g + wv;
  const bool live = I <= J && !(I >= kb0 && I < kb0 + nb), last = kb0 + nb == sd.nt;
  T* base = fac + sd.fac_off + (long long)k * sd.P * sd.P;
  T* Aij = base + tile_off(I, J, sd.nt);
  T* Aji = base + tile_off(J, I, sd.nt);
  const T* Cs = tbuf + sd.t_off + (long long)(I > kb0 ? I - nb : I) * nb * TT;
  // W_J: in its place after the pivot block, in the scratch before it
  const T* Ws = J > kb0 ? base + tile_off(kb0, J, sd.nt)
                        : tbuf + sd.t_off + (long long)(sd.nt - nb + J) * nb * TT;
  const long long wstep = J > kb0 ? (long long)sd.nt * TT : TT;
  M mm;
  mm.zero();
  mm.fetch_y(Ws);
  if (live) mm.fetch_x(Cs);
  int u = 0;
  for (; u < nb - 1; ++u) {
    mm.stage_y(lds[u & 1]);
    __syncthreads();
    mm.fetch_y(Ws + (u + 1) * wstep);
    const T* next = Cs + (u + 1) * TT;
    if (live) mm.mac(lds[u & 1], [&](int i0, int i1) { mm.fetch_x(next, i0, i1); });
    asm volatile("" ::: "memory");      // keeps the fetches in this iteration
  }
  mm.stage_y(lds[u & 1]);
  __syncthreads();
  if (!live) return;
  // the last products: the tile itself comes into the registers they free
  T cv[16];
  mm.mac(lds[u & 1], [&](int i0, int i1) {
    int n = 0;
    mm.visit([&](int row, int col, T) {
      if (n >= i0 * 16 / M::NX && n < i1 * 16 / M::NX) cv[n] = Aij[in_tile(row, col)];
      ++n;
    });
  });
  int n = 0;
  mm.visit([&](int row, int col, T v) {
    const T w = csub(cv[n], v);
    Aij[in_tile(row, col)] = w;
    if (last && I != J) Aji[in_tile(col, row)] = w;
    ++n;
  });
}

}  // namespace

template <typename R>
void launch_factor_plane(const SubDesc* subs_dev, int nsub, int k, int max_nt, int max_sz,
                         C<R>* fac, C<R>* tbuf, const C<R>* lca, int* status,
                         unsigned long long* stats, hipStream_t st) {
  const dim3 g2(max_nt, max_nt, nsub);
  const int nsub8 = (nsub + NXCD - 1) / NXCD * NXCD;
  constexpr int NBT = GjBlock<R>::NBT;
  if (k > 0)
    hipLaunchKernelGGL((schur_T_kernel<R>), g2, dim3(256), 0, st, subs_dev, k, fac, tbuf, lca);
  hipLaunchKernelGGL((build_S_kernel<R>), g2, dim3(256), 0, st, subs_dev, k, fac, tbuf, lca, stats,
                     max_sz);
  for (int kb0 = 0; kb0 < max_nt; kb0 += NBT) {
    hipLaunchKernelGGL((gj_diag_kernel<R>), dim3(nsub), dim3(64 * GjBlock<R>::WAVES),
                       0, st, subs_dev, k, kb0, fac, status, stats, max_sz);
    hipLaunchKernelGGL((gj_panel_kernel<R>), dim3(max_nt, nsub), dim3(64 * NBT), 0, st,
                       subs_dev, k, kb0, fac, tbuf);
    hipLaunchKernelGGL((gj_update_kernel<R>),
                       dim3((unsigned)(nsub8 * update_items(max_nt))), dim3(64 * UW), 0, st,
                       subs_dev, nsub, max_nt, k, kb0, fac, tbuf);
  }
}

template void launch_factor_plane<float>(const SubDesc*, int, int, int, int, float2*, float2*,
                                         const float2*, int*, unsigned long long*, hipStream_t);
template void launch_factor_plane<double>(const SubDesc*, int, int, int, int, double2*, double2*,
                                          const double2*, int*, unsigned long long*, hipStream_t);

}  // namespace oras

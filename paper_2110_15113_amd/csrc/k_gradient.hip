// Misfit gradient with respect to the squared slowness m from forward fields u
// and adjoint fields mu (paper sec. 1, sec. 4), with the stencil weights frozen
// or following the model (sec. 2.3: each node's weights are picked from its
// local G = lambda / h, so they move with m).
//
// Frozen weights:
//   g_i = -Re omega^2 q_i sum_c [ wm0_i S_i conj(mu_i) u_i
//        + sum_{j~i} 1/2 mhat_ij (conj(mu_i) u_j + conj(mu_j) u_i) ],
//   mhat_ij = 1/2 (wm_t,i + wm_t,j) 1/2 (S_i + S_j).
// Following weights add -Re sum_k H_k,i dw_k/dm_i, with
// H_k,i = sum_c d(mu_c^H A u_c)/dw_k,i and dw_k/dm_i = (table slope at G_i)
// dG/dm_i, dG/dm = -G / (2 m), over the four mass weights: the table keeps the
// three stiffness weights constant over G (weights_fit.cpp), so their slope is
// zero.
//
// Both need, per node, the 27 sums over the right-hand sides of the products
// of u and mu with their neighbours, and nothing else of u and mu.  A
// work-group owns a 16 x 4 x 4 tile of nodes (4 x 8 x 8 where the grid has few
// along x), keeps its 27 sums in registers and streams the right-hand sides
// through LDS (tile and halo, two buffers, the next one's loads in flight), so u
// and mu are read once from memory and the halo's share (1.5 times the tile)
// again from the caches.  Bound by its LDS reads, 54 of 16 bytes per node and
// right-hand side: 0.31 of the 0.58 ms that 96^3 nodes with 32 right-hand sides
// take, at 128 bytes per CU and clock (its 53 complex multiply-adds are 0.15 ms
// of the FP64 vector unit; 14.1 ms with one thread per node gathering every
// product from memory, a pass for each of the two parts and seven for the
// stiffness weights).
#include <algorithm>

#include "oras_internal.h"

namespace oras {

namespace {

constexpr int GT = 256;      // threads of a work-group, nodes of its GX x GY x GZ tile

template <bool WEIGHTS, int GX, int GY, int GZ>
__global__ void __launch_bounds__(GT) __attribute__((amdgpu_waves_per_eu(3)))
gradient_kernel(OpView V, const double2* __restrict__ qfac, const double* __restrict__ wtab,
                int tab_count, double g0, double dg, const double2* __restrict__ u,
                const double2* __restrict__ mu, int nrhs, unsigned first,
                double* __restrict__ gout) {
  static_assert(GX * GY * GZ == GT, "one node per thread");
  constexpr int GHX = GX + 2, GHY = GY + 2, GHZ = GZ + 2, GN = GHX * GHY * GHZ;
  constexpr int GL = (GN + GT - 1) / GT;      // halo nodes per thread
  __shared__ double2 su[2][GN], sm[2][GN];
  const int tid = threadIdx.x;
  const long long n = (long long)V.nx * V.ny * V.nz;
  // tiles in one grid dimension, x fastest
  const unsigned tx = (V.nx + GX - 1) / GX, ty = (V.ny + GY - 1) / GY, tile = first + blockIdx.x;
  const int i0 = tile % tx * GX, j0 = tile / tx % ty * GY, k0 = tile / (tx * ty) * GZ;
  // the halo nodes this thread fetches (-1: outside the grid, zero)
  long long src[GL];
#pragma unroll
  for (int l = 0; l < GL; ++l) {
    const int h = tid + l * GT;
    const int hi = i0 - 1 + h % GHX, hj = j0 - 1 + (h / GHX) % GHY, hk = k0 - 1 + h / (GHX * GHY);
    const bool in = h < GN && hi >= 0 && hi < V.nx && hj >= 0 && hj < V.ny && hk >= 0 && hk < V.nz;
    src[l] = in ? ((long long)hk * V.ny + hj) * V.nx + hi : -1;
  }
  double2 ru[GL], rm[GL];
  auto fetch = [&](int c) {
#pragma unroll
    for (int l = 0; l < GL; ++l) {
      ru[l] = rm[l] = make_double2(0.0, 0.0);
      if (src[l] >= 0) {
        ru[l] = u[c * n + src[l]];
        rm[l] = mu[c * n + src[l]];
      }
    }
  };
  auto stash = [&](int buf) {
#pragma unroll
    for (int l = 0; l < GL; ++l)
      if (tid + l * GT < GN) {
        su[buf][tid + l * GT] = ru[l];
        sm[buf][tid + l * GT] = rm[l];
      }
  };
  const int lx = tid % GX, ly = (tid / GX) % GY, lz = tid / (GX * GY);
  const int ctr = ((lz + 1) * GHY + ly + 1) * GHX + lx + 1;
  // sum over c of conj(mu_i) u_j + conj(mu_j) u_i per offset (13: conj(mu_i) u_i)
  double2 s2[27];
#pragma unroll
  for (int e = 0; e < 27; ++e) s2[e] = make_double2(0.0, 0.0);
  fetch(0);
  stash(0);
  __syncthreads();
  for (int c = 0; c < nrhs; ++c) {
    const int buf = c & 1;
    if (c + 1 < nrhs) fetch(c + 1);
    const double2 ui = su[buf][ctr], mi = sm[buf][ctr];
#pragma unroll
    for (int e = 0; e < 27; ++e) {
      const int at = ctr + ((e / 9 - 1) * GHY + (e / 3) % 3 - 1) * GHX + e % 3 - 1;
      cfmaconj(s2[e], mi, e == 13 ? ui : su[buf][at]);
      if (e != 13) cfmaconj(s2[e], sm[buf][at], ui);
      // one neighbour at a time: left free, the compiler reads them all first
      // and sinks the products behind the stores to LDS (368 registers)
      asm volatile("" : "+v"(s2[e].x), "+v"(s2[e].y));
      if (e % 3 == 2) __builtin_amdgcn_sched_barrier(0);
    }
    if (c + 1 < nrhs) stash(buf ^ 1);
    __syncthreads();
  }

  const int i = i0 + lx, j = j0 + ly, k = k0 + lz;
  if (i >= V.nx || j >= V.ny || k >= V.nz) return;
  const long long node = ((long long)k * V.ny + j) * V.nx + i;
  const double om2 = V.omega * V.omega;
  const double2 Si = cmul(cmul(V.px[2 * i + 1], V.py[2 * j + 1]), V.pz[2 * k + 1]);
  const double2 mti = V.mt[node];
  double2 acc = cscale(cmul(Si, s2[13]), V.w7[node * 7 + 3]);
  double H[4] = {0, 0, 0, 0};      // mass weights: centre, face, edge, corner
  if (WEIGHTS) H[0] = om2 * cmul(cmul(mti, Si), s2[13]).x;
#pragma unroll
  for (int e = 0; e < 27; ++e) {
    const int ex = e % 3 - 1, ey = (e / 3) % 3 - 1, ez = e / 9 - 1;
    const int qi = i + ex, qj = j + ey, qk = k + ez;
    if (e == 13 || qi < 0 || qi >= V.nx || qj < 0 || qj >= V.ny || qk < 0 || qk >= V.nz) continue;
    const long long nb = ((long long)qk * V.ny + qj) * V.nx + qi;
    const int t = (ex != 0) + (ey != 0) + (ez != 0);
    const double2 Sj = cmul(cmul(V.px[2 * qi + 1], V.py[2 * qj + 1]), V.pz[2 * qk + 1]);
    const double2 mh =
        cscale(cadd(Si, Sj), 0.25 * (V.w7[node * 7 + 3 + t] + V.w7[nb * 7 + 3 + t]));
    acc = cadd(acc, cscale(cmul(mh, s2[e]), 0.5));
    if (WEIGHTS) {
      const double2 coup = cmul(cscale(cadd(mti, V.mt[nb]), 0.5), cscale(cadd(Si, Sj), 0.5));
      H[t] += 0.5 * om2 * cmul(coup, s2[e]).x;
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  const double2 r = cmul(qfac[node], acc);
  double g = -V.omega * V.omega * r.x;
  if (WEIGHTS) {
    // dw/dm from the piecewise-linear table at G = 2 pi / (omega h sqrt(m));
    // where the lookup clamps the weights do not move
    const double m = cdiv(mti, qfac[node]).x;
    const double G = 2.0 * M_PI / (V.omega * V.h * sqrt(m));
    const double tt = (G - g0) / dg;
    if (tt > 0.0 && tt < tab_count - 1.0) {
      const int r0 = min((int)floor(tt), tab_count - 2);
      const double dGdm = -G / (2.0 * m);
      double dw = 0.0;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        dw += (wtab[(r0 + 1) * 7 + 3 + q] - wtab[r0 * 7 + 3 + q]) / dg * dGdm * H[q];
      g -= dw;
    }
  }
  gout[node] = g;
}

}  // namespace

void launch_gradient(const OpView& op, const double2* qfac, const double* wtab, int tab_count,
                     double g0, double dg, bool weights, const double2* u, const double2* mu,
                     int nrhs, double* g, hipStream_t st) {
  auto launch = [&](auto kernel, int gx, int gy, int gz) {
    const long long tiles = (long long)((op.nx + gx - 1) / gx) * ((op.ny + gy - 1) / gy) *
                            ((op.nz + gz - 1) / gz);
    // A launch holds fewer than 2^32 threads, which badly filled tiles can exceed
    // (5 x 3 x 2^26 nodes, half of what a grid may have, take 2^24 tiles and
    // more): 2^20 tiles, over a millisecond's work, per launch.
    constexpr long long MAX_TILES = 1LL << 20;
    for (long long first = 0; first < tiles; first += MAX_TILES)
      hipLaunchKernelGGL(kernel, dim3((unsigned)std::min(MAX_TILES, tiles - first)), dim3(GT), 0,
                         st, op, qfac, wtab, tab_count, g0, dg, u, mu, nrhs, (unsigned)first, g);
  };
  // Rows of 16 nodes are what the loads want; with a few nodes along x most of a
  // tile is empty, and one right-hand side took longer than without tiles (400 x
  // 400 x 3 nodes 222 us against 157).
  if (op.nx <= 8) {
    if (weights) launch(gradient_kernel<true, 4, 8, 8>, 4, 8, 8);
    else launch(gradient_kernel<false, 4, 8, 8>, 4, 8, 8);
  } else {
    if (weights) launch(gradient_kernel<true, 16, 4, 4>, 16, 4, 4);
    else launch(gradient_kernel<false, 16, 4, 4>, 16, 4, 4);
  }
}

}  // namespace oras

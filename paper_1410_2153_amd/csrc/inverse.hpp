// Dense inverses of the bottom matrices A_lc (Algorithm 2, B_0) on the device, for one mesh or a batch.
//
// Block Gauss-Jordan elimination in place, without pivoting (the matrices are symmetric positive
// definite): for every block of 32 unknowns, one launch inverts the diagonal block D (each thread block for
// itself, in LDS) and stores R = D^-1 A_k and C = A_k^T, a second one updates A_ij -= C_i R_j, with
// A_ik = -C_i D^-1 and A_kj = R_j. 2 n^3 operations where the Cholesky factor and its triangular solves
// take n^3, but 31 dependent steps instead of 961: 961 unknowns take about 0.6 ms, against 50-100 ms for
// the factor on the host's threads (the Cholesky factor alone is a serial chain of 961 columns).
#pragma once

#include <cstdint>
#include <vector>

#include "common.hpp"

namespace asmg {

static constexpr int kInvB = 32;    // unknowns per elimination step
static constexpr int kInvT = 64;    // rows and columns of a tile

struct InvBatch {  // device arrays of the matrices: size, offset in M, offset in the scratch (64 n values each)
  const int *n;
  const int64_t *moff, *soff;
};

static __global__ __launch_bounds__(BS) void k_inv_panel(int k0, InvBatch B, const double *__restrict__ M,
                                                         double *__restrict__ scratch, int *__restrict__ bad) {
  __shared__ double D[kInvB][kInvB + 1];
  __shared__ double A[kInvB][kInvT + 1];
  const int n = B.n[blockIdx.y], t0 = blockIdx.x * kInvT, tid = threadIdx.x;
  if (k0 >= n || t0 >= n) return;
  const int kb = min(kInvB, n - k0);
  const double *m = M + B.moff[blockIdx.y];
  double *R = scratch + B.soff[blockIdx.y], *C = R + (int64_t)kInvB * n;
  for (int e = tid; e < kInvB * kInvB; e += BS) {
    const int r = e / kInvB, c = e % kInvB;
    D[r][c] = r < kb && c < kb ? m[(int64_t)(k0 + r) * n + k0 + c] : r == c ? 1.0 : 0.0;
  }
  for (int e = tid; e < kInvB * kInvT; e += BS) {
    const int r = e / kInvT, c = e % kInvT;
    A[r][c] = r < kb && t0 + c < n ? m[(int64_t)(k0 + r) * n + t0 + c] : 0.0;
  }
  for (int e = tid; e < kInvT * kInvB; e += BS) {
    const int r = e / kInvB, c = e % kInvB;
    if (t0 + r < n) C[(int64_t)(t0 + r) * kInvB + c] = c < kb ? m[(int64_t)(t0 + r) * n + k0 + c] : 0.0;
  }
  __syncthreads();
  constexpr int per = kInvB * kInvB / BS;
  for (int s = 0; s < kb; ++s) {
    const double p = D[s][s];
    if (!(p > 0.0) && tid == 0) bad[blockIdx.y] = 1;
    const double pi = 1.0 / p;
    double v[per];
#pragma unroll
    for (int q = 0; q < per; ++q) {
      const int e = tid + q * BS, r = e / kInvB, c = e % kInvB;
      const double row = D[s][c], col = D[r][s];
      v[q] = r == s ? (c == s ? pi : row * pi) : c == s ? -col * pi : D[r][c] - col * row * pi;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < per; ++q) {
      const int e = tid + q * BS;
      D[e / kInvB][e % kInvB] = v[q];
    }
    __syncthreads();
  }
  for (int e = tid; e < kInvB * kInvT; e += BS) {
    const int r = e / kInvT, c = e % kInvT, j = t0 + c;
    if (r >= kb || j >= n) continue;
    double s = 0.0;
    if (j >= k0 && j < k0 + kb)
      s = D[r][j - k0];
    else
      for (int t = 0; t < kb; ++t) s += D[r][t] * A[t][c];
    R[(int64_t)r * n + j] = s;
  }
}

static __global__ __launch_bounds__(BS) void k_inv_update(int k0, InvBatch B, double *__restrict__ M,
                                                          const double *__restrict__ scratch) {
  __shared__ double Ct[kInvT][kInvB + 1];
  __shared__ double Rt[kInvB][kInvT + 1];
  const int n = B.n[blockIdx.z], i0 = blockIdx.y * kInvT, j0 = blockIdx.x * kInvT, tid = threadIdx.x;
  if (k0 >= n || i0 >= n || j0 >= n) return;
  const int kb = min(kInvB, n - k0);
  double *m = M + B.moff[blockIdx.z];
  const double *R = scratch + B.soff[blockIdx.z], *C = R + (int64_t)kInvB * n;
  for (int e = tid; e < kInvT * kInvB; e += BS) {
    const int r = e / kInvB, c = e % kInvB;
    Ct[r][c] = i0 + r < n ? C[(int64_t)(i0 + r) * kInvB + c] : 0.0;
    const int rr = e / kInvT, cc = e % kInvT;
    Rt[rr][cc] = rr < kb && j0 + cc < n ? R[(int64_t)rr * n + j0 + cc] : 0.0;
  }
  __syncthreads();
  const int tx = tid & 15, ty = tid >> 4;
  double acc[4][4] = {};
  for (int s = 0; s < kb; ++s) {
    double a[4], b[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      a[q] = Ct[ty + 16 * q][s];
      b[q] = Rt[s][tx + 16 * q];
    }
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[p][q] += a[p] * b[q];
  }
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = i0 + ty + 16 * p, j = j0 + tx + 16 * q;
      if (i >= n || j >= n) continue;
      double *at = m + (int64_t)i * n + j;
      if (i >= k0 && i < k0 + kb)
        *at = Rt[i - k0][j - j0];
      else
        *at = (j >= k0 && j < k0 + kb ? 0.0 : *at) - acc[p][q];
    }
}

// M = A (CSR), with gamma of the row's component added to every entry inside a component that has one
static __global__ __launch_bounds__(BS) void k_inv_fill(int n, const int *__restrict__ rp, const int *__restrict__ ci,
                                                        const double *__restrict__ v, const int *__restrict__ comp,
                                                        const double *__restrict__ gamma, double *__restrict__ M) {
  const int i = blockIdx.x;
  double *row = M + (int64_t)i * n;
  const double g = gamma[comp[i]];
  for (int j = threadIdx.x; j < n; j += BS) row[j] = g != 0.0 && comp[j] == comp[i] ? g : 0.0;
  __syncthreads();
  for (int p = rp[i] + threadIdx.x; p < rp[i + 1]; p += BS) row[ci[p]] += v[p];
}

static constexpr const char *kNotSpd = "matrix of an exact subsystem solve is not positive definite";

// One matrix to invert: A_lc with the rank-one terms of its singular components (coarse_components).
struct InvInput {
  const Csr *A;
  std::vector<int> comp;
  std::vector<double> gamma;
};

// M + moff[i] = inverse of matrix i, FP64 on the device; returns the first matrix with a pivot that is not
// positive, -1 = none
static int device_inverses(const std::vector<InvInput> &in, const std::vector<int64_t> &moff, double *M) {
  std::vector<int> ns;
  std::vector<int64_t> soff;
  int64_t scratch = 0;
  int most = 0;
  // one upload for all inputs: integers (row pointers, columns, components), then doubles
  std::vector<int> iv;
  std::vector<double> dv;
  struct At {
    size_t rp, ci, comp, v, gamma;
  };
  std::vector<At> at;
  for (const InvInput &x : in) {
    const int n = (int)x.A->nrows;
    ns.push_back(n);
    soff.push_back(scratch);
    scratch += 2 * (int64_t)kInvB * n;
    most = std::max(most, n);
    At a;
    a.rp = iv.size();
    iv.insert(iv.end(), x.A->rp.begin(), x.A->rp.end());
    a.ci = iv.size();
    iv.insert(iv.end(), x.A->ci.begin(), x.A->ci.end());
    a.comp = iv.size();
    iv.insert(iv.end(), x.comp.begin(), x.comp.end());
    a.v = dv.size();
    dv.insert(dv.end(), x.A->v.begin(), x.A->v.end());
    a.gamma = dv.size();
    dv.insert(dv.end(), x.gamma.begin(), x.gamma.end());
    at.push_back(a);
  }
  if (most == 0) return -1;
  const size_t m = in.size(), nsat = iv.size();
  iv.insert(iv.end(), ns.begin(), ns.end());
  iv.resize(iv.size() + m, 0);  // flags of a pivot that is not positive
  struct Bufs {
    std::vector<void *> p;
    void *get(size_t bytes) {
      void *x = nullptr;
      HIPCHECK(hipMalloc(&x, std::max<size_t>(bytes, 8)));
      p.push_back(x);
      return x;
    }
    ~Bufs() {
      for (void *x : p) (void)hipFree(x);
    }
  } bufs;
  int *di = (int *)bufs.get(iv.size() * 4);
  double *dd = (double *)bufs.get(dv.size() * 8);
  int64_t *off = (int64_t *)bufs.get(2 * m * 8);
  double *sc = (double *)bufs.get((size_t)scratch * 8);
  HIPCHECK(hipMemcpy(di, iv.data(), iv.size() * 4, hipMemcpyHostToDevice));
  HIPCHECK(hipMemcpy(dd, dv.data(), dv.size() * 8, hipMemcpyHostToDevice));
  HIPCHECK(hipMemcpy(off, moff.data(), m * 8, hipMemcpyHostToDevice));
  HIPCHECK(hipMemcpy(off + m, soff.data(), m * 8, hipMemcpyHostToDevice));
  for (size_t i = 0; i < m; ++i)
    if (ns[i] > 0)
      hipLaunchKernelGGL(k_inv_fill, dim3(ns[i]), dim3(BS), 0, nullptr, ns[i], di + at[i].rp, di + at[i].ci,
                         dd + at[i].v, di + at[i].comp, dd + at[i].gamma, M + moff[i]);
  int *bad = di + nsat + m;
  const int tiles = (most + kInvT - 1) / kInvT;
  constexpr size_t kMost = 32768;  // matrices per launch (a grid dimension holds 65535)
  for (size_t i0 = 0; i0 < m; i0 += kMost) {
    const InvBatch B{di + nsat + i0, off + i0, off + m + i0};
    const unsigned c = (unsigned)std::min(kMost, m - i0);
    for (int k0 = 0; k0 < most; k0 += kInvB) {
      hipLaunchKernelGGL(k_inv_panel, dim3(tiles, c), dim3(BS), 0, nullptr, k0, B, M, sc, bad + i0);
      hipLaunchKernelGGL(k_inv_update, dim3(tiles, tiles, c), dim3(BS), 0, nullptr, k0, B, M, sc);
    }
  }
  HIPCHECK(hipGetLastError());
  std::vector<int> flag(m);
  HIPCHECK(hipMemcpy(flag.data(), bad, m * 4, hipMemcpyDeviceToHost));
  for (size_t i = 0; i < m; ++i)
    if (flag[i]) return (int)i;
  return -1;
}

}  // namespace asmg

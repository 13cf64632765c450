// Host check of the patch layout (csrc/patch.hpp): builds a level's patches and runs both patch kernels' steps on
// the CPU, one patch after the other, on an LDS image that starts as NaN. Usage: patch_check <in> <out>.
// in:  int32 n, C, nu, ncoarse, own rows per patch, shape (0 small, 1 big); A (CSR without the diagonal), diagonal,
//      colour and spatial order of each row, P (CSR); then b, e (coarse) and the number of patches wanted is n / own.
// out: x (after the forward sweeps), bc (restricted residual), xo (after the backward sweeps), int32 patches,
//      int32 cells that a slice of rows without neighbours reads (its width, summed)
#include <cstdio>
#include <cstdlib>
#include <limits>

#include "patch.hpp"

using namespace asmg;

struct Mat {
  std::vector<int> rp, ci;
  std::vector<double> v;
};

static FILE *in;

template <class T>
static std::vector<T> get(size_t n) {
  std::vector<T> v(n);
  if (n && fread(v.data(), sizeof(T), n, in) != n) exit(2);
  return v;
}

static Mat matrix(int rows) {
  Mat m;
  m.rp = get<int>(rows + 1);
  m.ci = get<int>(m.rp[rows]);
  m.v = get<double>(m.rp[rows]);
  return m;
}

int main(int, char **argv) {
  in = fopen(argv[1], "rb");
  if (!in) return 2;
  const std::vector<int> h = get<int>(6);
  const int n = h[0], C = h[1], nu = h[2], nc = h[3], own = h[4];
  const Mat A = matrix(n);
  const std::vector<double> diag = get<double>(n);
  std::vector<PatchJob<Mat>> jobs(1);
  PatchSource<Mat> &S = jobs[0].src;
  S.A = &A;
  S.n = n;
  S.C = C;
  S.nu = nu;
  S.ncoarse = nc;
  for (int c : get<int>(n)) S.col.push_back((uint8_t)c);
  S.order = get<int>(n);
  const Mat P = matrix(n);
  const std::vector<double> b = get<double>(n), e = get<double>(nc);
  Mat R;  // P^T
  R.rp.assign(nc + 1, 0);
  for (int c : P.ci) ++R.rp[c + 1];
  for (int i = 0; i < nc; ++i) R.rp[i + 1] += R.rp[i];
  R.ci.resize(P.ci.size());
  R.v.resize(P.ci.size());
  std::vector<int> at(R.rp.begin(), R.rp.end() - 1);
  for (int i = 0; i < n; ++i)
    for (int p = P.rp[i]; p < P.rp[i + 1]; ++p) {
      R.ci[at[P.ci[p]]] = i;
      R.v[at[P.ci[p]]++] = P.v[p];
    }
  S.P = &P;
  S.R = &R;
  S.shape = h[5] ? kPatchBig : kPatchSmall;
  S.prepare();
  const int np0 = std::max(1, n / own);
  for (int p = 0; p <= np0; ++p) jobs[0].cuts.push_back((int)((int64_t)p * n / np0));
  jobs[0].code_matrix = false;
  patch_build(1, jobs);
  if (jobs[0].cuts.empty()) return 3;
  const PatchHost &H = jobs[0].all;
  const PatchCodes &K = jobs[0].codes;
  const int bits = S.shape.bits;
  const uint32_t mask = (1u << bits) - 1;
  auto weight = [&](uint32_t code) { return code == 0 ? 1.0 : code == 1 ? 0.5 : 0.0; };
  const double nan = std::numeric_limits<double>::quiet_NaN();
  std::vector<double> x(n, nan), bc(nc, nan), xo(n, nan);
  std::vector<double> xs, bs;
  int alone = 0;
  for (int up = 0; up < 2; ++up)
    for (size_t p = 0; p < H.head.size(); ++p) {
      const PatchHead &d = H.head[p];
      const int *g = &H.gidx[p * S.shape.slices * 64];
      xs.assign(64 * d.ncs, nan);
      bs.assign(64 * d.ns, nan);
      auto row = [&](int i) { return g[i] < 0 ? 0 : g[i] & (kPatchHalo - 1); };
      auto owns = [&](int i) { return g[i] >= 0 && !(g[i] & kPatchHalo); };
      auto turn = [&](int k) { return (int)(d.sc[k / S.shape.waves] >> 4 * (k % S.shape.waves) & 15); };
      auto dot = [&](int k, int l, int above) {
        double a0 = 0, a1 = 0;
        for (int q = d.poff[k]; q < d.poff[k + 1]; ++q) {
          const size_t t = (size_t)q * 64 + l;
          const int c0 = H.pidx[t] & mask, c1 = H.pidx[t] >> 16 & mask;
          a0 += (c0 > above ? H.pval[2 * t] : 0.0) * xs[c0];
          a1 += (c1 > above ? H.pval[2 * t + 1] : 0.0) * xs[c1];
        }
        return a0 + a1;
      };
      auto pass = [&](int c) {
        std::vector<std::pair<int, double>> w;
        for (int k = 0; k < d.ns; ++k)
          if (turn(k) == c)
            for (int l = 0; l < 64; ++l) {
              const int i = 64 * k + l;
              w.push_back({i, (bs[i] - dot(k, l, -1)) / diag[row(i)]});
            }
        for (auto &v : w) xs[v.first] = v.second;
      };
      for (int i = 0; i < 64 * d.ns; ++i) bs[i] = b[row(i)];
      if (!up) {
        for (int i = 0; i < 64 * d.ncs; ++i)
          xs[i] = i < 64 * d.ns && turn(i / 64) == 0 ? bs[i] / diag[row(i)] : 0.0;
        for (int s = 0; s < nu; ++s)
          for (int c = s == 0 ? 1 : 0; c < C; ++c) pass(c);
        for (int k = 0; k < d.ns; ++k)
          for (int l = 0; l < 64; ++l) {
            const int i = 64 * k + l;
            if (owns(i)) {
              x[g[i]] = xs[i];
              if (A.rp[g[i] + 1] == A.rp[g[i]]) alone += d.poff[k + 1] - d.poff[k];
            }
          }
        std::vector<double> r(64 * d.ns);
        for (int k = 0; k < d.ns; ++k)
          for (int l = 0; l < 64; ++l) {
            const int i = 64 * k + l;
            r[i] = turn(k) == C - 1 ? 0.0
                   : nu == 1        ? -dot(k, l, i)
                                    : bs[i] - diag[row(i)] * xs[i] - dot(k, l, -1);
          }
        for (int k = 0; k < d.nco; ++k)
          for (int l = 0; l < 64; ++l) {
            const int c = H.rrow[(size_t)(d.coarse0 + k) * 64 + l];
            if (c < 0) continue;
            double a0 = 0, a1 = 0;
            for (int q = H.roff[d.coarse0 + k]; q < H.roff[d.coarse0 + k + 1]; ++q) {
              const size_t t = (size_t)q * 64 + l;
              const uint32_t id = H.ridx[t];
              const double v0 = K.transfer ? weight(id >> bits & (65535u >> bits)) : H.rval[2 * t];
              const double v1 = K.transfer ? weight(id >> (16 + bits)) : H.rval[2 * t + 1];
              a0 += v0 * r[id & mask];
              a1 += v1 * r[id >> 16 & mask];
            }
            bc[c] = a0 + a1;
          }
      } else {
        for (int k = 0; k < d.nst; ++k)
          for (int l = 0; l < 64; ++l) {
            const size_t t = (size_t)(d.start0 + k) * 64 + l;
            if (H.ugidx[t] < 0) continue;
            double a = x[H.ugidx[t]];
            for (int q = d.uoff[k]; q < d.uoff[k + 1]; ++q) {
              const size_t u = (size_t)q * 64 + l;
              const int c = K.transfer ? H.ucol[u] & 0xfffffff : H.ucol[u];
              a += (K.transfer ? weight((uint32_t)H.ucol[u] >> 28) : H.uval[u]) * e[c];
            }
            xs[H.ucell[t]] = a;
          }
        for (int s = 0; s < nu; ++s)
          for (int c = C - 1; c >= 0; --c) pass(c);
        for (int i = 0; i < 64 * d.ns; ++i)
          if (owns(i)) xo[g[i]] = xs[i];
      }
    }
  FILE *out = fopen(argv[2], "wb");
  fwrite(x.data(), 8, n, out);
  fwrite(bc.data(), 8, nc, out);
  fwrite(xo.data(), 8, n, out);
  const int np = (int)H.head.size();
  fwrite(&np, 4, 1, out);
  fwrite(&alone, 4, 1, out);
  fclose(out);
  return 0;
}

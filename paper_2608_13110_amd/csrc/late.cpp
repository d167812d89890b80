// Late-phase launch construction (see late.hpp).
#include "late.hpp"

#include <algorithm>

namespace tnc {

namespace {

// A 2x2 on bit `bit`, or a 4x4 on bits (bit, bit + 1), of `rows` states of
// 2^sb entries each (FP64, real and imaginary parts spelled out: the library's
// complex product checks for NaN).
void apply_u1(cd* st, size_t rows, int sb, int bit, const cd* m) {
  const size_t total = rows << sb, h = size_t(1) << bit;
  double k[8];
  for (int e = 0; e < 4; ++e) k[2 * e] = m[e].real(), k[2 * e + 1] = m[e].imag();
  double* v = reinterpret_cast<double*>(st);
  for (size_t i0 = 0; i0 < total; i0 += 2 * h)
    for (size_t i = i0; i < i0 + h; ++i) {
      double* a = v + 2 * i;
      double* b = v + 2 * (i + h);
      const double ax = a[0], ay = a[1], bx = b[0], by = b[1];
      a[0] = k[0] * ax - k[1] * ay + k[2] * bx - k[3] * by;
      a[1] = k[0] * ay + k[1] * ax + k[2] * by + k[3] * bx;
      b[0] = k[4] * ax - k[5] * ay + k[6] * bx - k[7] * by;
      b[1] = k[4] * ay + k[5] * ax + k[6] * by + k[7] * bx;
    }
}

void apply_g4(cd* st, size_t rows, int sb, int bit, const cd* g) {
  const size_t total = rows << sb, h = size_t(1) << bit;
  double* v = reinterpret_cast<double*>(st);
  for (size_t i0 = 0; i0 < total; i0 += 4 * h)
    for (size_t i = i0; i < i0 + h; ++i) {
      // basis 2 bit_a + bit_{a+1}
      double* p[4] = {v + 2 * i, v + 2 * (i + 2 * h), v + 2 * (i + h), v + 2 * (i + 3 * h)};
      double x[4], y[4];
      for (int u = 0; u < 4; ++u) x[u] = p[u][0], y[u] = p[u][1];
      for (int o = 0; o < 4; ++o) {
        double re = 0, im = 0;
        for (int u = 0; u < 4; ++u) {
          const double kr = g[4 * o + u].real(), ki = g[4 * o + u].imag();
          re += kr * x[u] - ki * y[u];
          im += kr * y[u] + ki * x[u];
        }
        p[o][0] = re;
        p[o][1] = im;
      }
    }
}

int bitrev(int b, int k) {
  int t = 0;
  for (int j = 0; j < k; ++j) t |= ((b >> (k - 1 - j)) & 1) << j;
  return t;
}

}  // namespace

int build_late(const Plan& p, const Schedule& s, LatePlan* out, std::string* err, int fold, bool host_join) {
  const auto& L = s.late;
  if (L.empty()) {
    if (err) *err = "empty late program";
    return -1;
  }
  const int sb = s.s_bits;
  const int dim = 1 << sb;
  const int k = s.k;
  out->s = sb;
  const LateOp& fin = L.back();
  out->final_kind = fin.kind;
  out->final_xrow = fin.xrow;
  if (fin.kind == L_DOT) out->dot = fin.m;
  const int nbody = int(L.size()) - 1;
  // removals and the slots they consume: slots_to[i] = slots removed by
  // removals 0..i-1
  std::vector<int> rpos, slots_to(1, 0);
  for (int i = 0; i < nbody; ++i)
    if (L[i].kind == L_REMOVE || L[i].kind == L_REMOVE2) {
      rpos.push_back(i);
      slots_to.push_back(slots_to.back() + (L[i].kind == L_REMOVE2 ? 2 : 1));
    }
  const int nrem = int(rpos.size());
  // k = 0: fold removals of up to 12 slots (the state is one qubit), but not
  // a removal with an output-bit variant (the first launch has one variant
  // row, the final one's).  k >= 1: folding j removals costs O(k 2^(2k+j)) on
  // the host and shrinks the first launch's FP64 output to 2^(m-j) rows;
  // worth it for large tensors only.  With no removal folded, the join
  // matrix is Z_early itself and every late op runs on the device.
  int j1;  // removals folded
  if (k == 0) {
    j1 = 0;
    while (j1 < nrem && slots_to[j1 + 1] <= 12 && L[rpos[j1]].xrow < 0) ++j1;
  } else {
    // 2^35-entry tensors (256 GiB of complex64) leave room for a join output
    // of 2^(h-j) x 16 B only with j = 7 (4 GiB).  From 2^30 entries on, j = 5
    // shrinks the late launches' input 32-fold; the join's flops do not depend on j.
    const int want = fold != -2 ? std::max(0, fold)
                     : p.opt.late_fold == 0 ? (s.m_fix >= 35 ? 7 : s.m_fix >= 30 ? 5 : s.m_fix >= 26 ? 3 : 0)
                                          : std::max(0, p.opt.late_fold);
    j1 = std::min(nrem, std::min(want, k <= 8 ? 8 : 1));
  }
  const bool first_final = j1 == nrem;
  const int first_end = first_final ? nbody : (j1 == 0 ? 0 : rpos[j1 - 1] + 1);

  // The rows of J: the states that enter the late program (Z_early's rows, or
  // the start vector) taken through the folded ops, doubled at each removal
  // (row u * 2^ub + ue: bit l of u the value of the l-th folded slot).
  const int js = slots_to[j1];
  const int ub = s.join_u_bits;
  const size_t de = size_t(1) << ub;
  const bool on_device = !host_join && k >= 1 && js > 0 && !first_final;
  std::vector<cd> Ju;
  if (!on_device) Ju.assign(s.join.begin(), s.join.begin() + de * dim);
  for (int i = 0; i < first_end && !on_device; ++i) {
    const LateOp& o = L[i];
    const size_t rows = Ju.size() >> sb;
    if (o.kind == L_U1) apply_u1(Ju.data(), rows, sb, o.a, o.m.data());
    else if (o.kind == L_G4) apply_g4(Ju.data(), rows, sb, o.a, o.m.data());
    else {
      const int nu = o.kind == L_REMOVE2 ? 4 : 2;
      const size_t part = Ju.size();
      Ju.resize(part * nu);
      for (int u = nu - 1; u >= 0; --u) {
        if (u > 0) std::copy(Ju.begin(), Ju.begin() + part, Ju.begin() + part * u);
        apply_u1(Ju.data() + part * u, rows, sb, 0, o.m.data() + 4 * u);
      }
    }
  }
  LateFirst& F = out->first;
  F.j = js;
  F.final = first_final;
  F.fold_ops = first_end;
  F.K = 1 << (ub + js);
  F.M = 1LL << (s.m_fix - ub - js);
  if (!first_final) {
    F.N = dim;
    F.nvar = 1;
    F.xrow = -1;
    F.J.swap(Ju);
  } else if (fin.kind == L_OUT) {
    F.N = 1 << k;
    F.nvar = 1;
    F.J.assign((size_t)F.K * F.N, cd(0));
    for (int kk = 0; kk < F.K; ++kk)
      for (int b = 0; b < F.N; ++b) F.J[(size_t)kk * F.N + b] = Ju[(size_t)kk * dim + bitrev(b, k)];
  } else {
    F.N = 1;
    F.nvar = 2;
    F.xrow = fin.xrow;
    F.J.assign((size_t)2 * F.K, cd(0));
    for (int var = 0; var < 2; ++var)
      for (int kk = 0; kk < F.K; ++kk) {
        cd acc = 0;
        for (int t = 0; t < dim; ++t) acc += fin.m[2 * var + t] * Ju[(size_t)kk * dim + t];
        F.J[(size_t)var * F.K + kk] = acc;
      }
  }
  // remaining launches
  if (!first_final) {
    // each launch takes whole removals of at most jmax slots
    const int jmax = std::max(2, 12 - sb);
    int done = j1;
    int pos = first_end;
    long long rows = F.M;
    while (done < nrem) {
      int e = done + 1;
      while (e < nrem && slots_to[e + 1] - slots_to[done] <= jmax) ++e;
      const int j = slots_to[e] - slots_to[done];
      const bool last = e == nrem;
      const int end = last ? nbody : rpos[e - 1] + 1;
      LateOpsLaunch ln;
      ln.op_begin = pos;
      ln.op_end = end;
      ln.j = j;
      ln.rows_in = rows;
      ln.final = last;
      out->ops.push_back(ln);
      rows >>= j;
      done = e;
      pos = end;
    }
  }
  return 0;
}

}  // namespace tnc

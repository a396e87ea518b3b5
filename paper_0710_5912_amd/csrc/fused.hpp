// fused.hpp -- the four-pass step: the inverse row transforms run inside the
// stencil kernels, so a step is two row kernels and two column kernels.
//
//   k_flow_adv   stages 0 and 1: omega, psi row spectra -> real rows in LDS,
//                stage 1a with phi, forward row transforms
//   k_phi_mu     stages 3 and 4: phi' row spectrum -> real phi (stored: the
//                state) and its halo rows in LDS, stage 2a, forward row
//                transform of g
//
// A block owns NR rows and inverse-transforms its halo rows again (2 for the
// advection, 4 for mu and g): more transform work, but neither omega, psi nor
// phi goes through memory as a real field between the passes (168 -> 128
// bytes per site and step in FP64) and a step has four launches instead of
// six.  LDS holds the block's rows, so it applies to rows of up to 16 KB (see
// FuseCfg).
#pragma once

#include <type_traits>

#include "common.hpp"
#include "fft.hpp"
#include "ops.hpp"
#include "stages.hpp"

namespace le {

// Half spectrum staged in lds[0 .. L] (DC and Nyquist with zero imaginary
// parts) to the real row, row_c2r's arithmetic without its branch at m = 0
// (X[0] and X[L] give it by the general formula), left in lds[0 .. L) as pairs
// and in v.  w0: the table entry t.
template <typename T, int L, int E, typename TW>
__device__ __forceinline__ void rows_c2r(c2<T>* v, c2<T>* lds, const TW& tw, c2<double> w0,
                                         int t) {
  constexpr int P = L / E;
#pragma unroll
  for (int q = 0; q < E; ++q) {
    const int m = t + q * P;
    const c2<T> X = lds[m], Xc = lds[L - m];
    const c2<T> a = {X.x + Xc.x, X.y - Xc.y};
    const c2<T> d = {X.x - Xc.x, X.y + Xc.y};
    const c2<double> wd = q == 0 ? w0 : cmul(w0, root_step<E>(q));
    const c2<T> b = cmulc(d, c2<T>{static_cast<T>(wd.x), static_cast<T>(wd.y)});
    v[q] = {a.x - b.y, a.y + b.x};
  }
  group_sync<true>();
  fft_regs<T, L, E, +1, true>(v, lds, 1, tw, t);
  const T sc = static_cast<T>(1.0 / (2.0 * L));
  group_sync<true>();
#pragma unroll
  for (int q = 0; q < E; ++q) {
    v[q] = {v[q].x * sc, v[q].y * sc};
    lds[t + q * P] = v[q];
  }
}

// Real row pairs v[q] = pair t + q P to the complex transform z of the packed
// row in lds[0 .. L), and z[0] again in lds[L] (rows_out reads the mirror of
// m = 0 there).
template <typename T, int L, int E, typename TW>
__device__ __forceinline__ void rows_r2c_z(c2<T>* v, c2<T>* lds, const TW& tw, int t) {
  constexpr int P = L / E;
  fft_regs<T, L, E, -1, true>(v, lds, 1, tw, t);
  group_sync<true>();
#pragma unroll
  for (int q = 0; q < E; ++q) lds[t + q * P] = v[q];
  if (t == 0) lds[L] = v[0];
}

// Shapes.  E values per thread, P = L/E threads per transform, within one
// wavefront (its passes need no block barrier, and groups beyond the rows sit
// them out).  LS: row stride in LDS, L + 1
// modes, two mod 8 (FP64) and mod 16 (FP32), so the tile runs of consecutive
// rows fall on distinct banks.
template <typename T, int L_, int NR_, int NF_, int E_>
struct FuseCfg {
  static constexpr int L = L_, NR = NR_, NF = NF_, E = E_;
  static constexpr int P = L / E;
  static_assert(P <= 64, "a transform lies within one wavefront");
  static constexpr int LS = L + 2;
  // advection: inverse rows, forward rows, transform groups
  static constexpr int AI = (NF == 3 ? 2 : 1) * (NR + 2), AO = NF * NR;
  static constexpr int AG = AI > AO ? AI : AO;
  static constexpr int AR = 2 * (NR + 2) > AG ? 2 * (NR + 2) : AG;  // rows in LDS
  static constexpr int ATPB = AG * P > 64 ? AG * P : 64;
  static constexpr long ALDS = (long)AR * LS * (long)sizeof(c2<T>);
  // waves per SIMD to compile for: blocks of eight waves that LDS holds twice on a
  // CU keep to 128 registers (1024-point rows, two to a block)
  static constexpr int AWPE = E <= 8 && ATPB == 512 && 2 * ALDS + 8192 <= 160L * 1024 ? 4 : 1;
  // mu and g
  static constexpr int MI = NR + 4;
  static constexpr int MG = E >= 8 && MI < 8 ? 8 : MI;  // (E >= 8: at most two pairs per thread)
  static constexpr int MTPB = MG * P > 64 ? MG * P : 64;
  static constexpr long MLDS = (long)MG * LS * (long)sizeof(c2<T>);
  typedef PassSet<T, L, E, 0, kFolded<T, E>, true, (L >= 128)> Tw;
  static constexpr long TAB = (long)(TwTab<L>::N + Tw::NLDS) * 16;
  static constexpr long LIMIT = 160L * 1024;
  static constexpr bool AOK = ALDS + TAB <= LIMIT && ATPB <= 1024;
  static constexpr bool MOK = MLDS + TAB <= LIMIT && MTPB <= 1024;
};

__device__ __forceinline__ int wrap_row(int j, int ny) {
  return j < 0 ? j + ny : (j >= ny ? j - ny : j);
}

// NROW rows ja .. (periodic) of a row spectrum into LDS rows, tile run by tile
// run (a run: the NROW rows' kTW modes of a tile).  A thread keeps one place of
// the run, so a step to its next tile is one constant offset.
template <typename T, int L, int NROW, int NT>
struct RowsIn {
  static constexpr int RUN = kTW * NROW, GR = NT / RUN;  // runs per step
  static constexpr int K = L / kTW + 1, N = (K + GR - 1) / GR;
  static_assert(GR >= 1, "a block holds at least one run");
  c2<T> v[N];
  __device__ __forceinline__ void get(gp<const c2<T>> X, int ny, int ja) {
    const int w = (int)threadIdx.x % RUN, k0 = (int)threadIdx.x / RUN;
    auto x = X + ((size_t)k0 * ny + wrap_row(ja + w / kTW, ny)) * kTW + w % kTW;
    const size_t step = (size_t)GR * ny * kTW;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int k = k0 + i * GR;
      if (k0 < GR && (k < K - 1 || (k == K - 1 && w % kTW == 0))) v[i] = ldg<T>(x + i * step);
    }
  }
  __device__ __forceinline__ void put(c2<T>* lds, int LS) {
    const int w = (int)threadIdx.x % RUN, k0 = (int)threadIdx.x / RUN;
    c2<T>* o = lds + (w / kTW) * LS + k0 * kTW + w % kTW;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int k = k0 + i * GR;
      // DC and Nyquist are real
      const bool real = w % kTW == 0 && (k == 0 || k == K - 1);
      if (k0 < GR && (k < K - 1 || (k == K - 1 && w % kTW == 0)))
        o[i * GR * kTW] = {v[i].x, real ? T(0) : v[i].y};
    }
  }
};

// The NF NR transformed rows in LDS (row f NR + r at stride LS) as half
// spectra, r2c_mode's arithmetic with the twiddle and the place formed once for
// the NF fields, stored tile run by tile run.
template <typename T, int L, int NR, int NF, int NT>
__device__ __forceinline__ void rows_out(gp<c2<T>> const (&X)[NF], const c2<T>* rows, int LS,
                                         const c2<double>* wtab, int ny, int j0) {
  constexpr int RUN = kTW * NR, GR = NT / RUN, K = L / kTW + 1;
  static_assert(GR >= 1, "a block holds at least one run");
  const int w = (int)threadIdx.x % RUN, k0 = (int)threadIdx.x / RUN;
  const int r = w / kTW;
  if (k0 >= GR) return;
  size_t at = ((size_t)k0 * ny + j0 + r) * kTW + w % kTW;
  const size_t step = (size_t)GR * ny * kTW;
  for (int m = k0 * kTW + w % kTW; m <= L; m += GR * kTW, at += step) {
    const c2<double> wd = tw_tab<L>(wtab, m);
    const c2<T> wm = {static_cast<T>(wd.x), static_cast<T>(wd.y)};
    const T h = static_cast<T>(0.5);
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const c2<T>* z_ = rows + (f * NR + r) * LS;
      const c2<T> z = z_[m], zc = z_[L - m];
      const c2<T> e = {h * (z.x + zc.x), h * (z.y - zc.y)};
      const c2<T> o = {h * (z.y + zc.y), -h * (z.x - zc.x)};
      c2<T> x = cadd(e, cmul(o, wm));
      if (m == L) x.y = T(0);
      stg<T>(X[f] + at, x);
    }
  }
}

// Pair p of the thread and where its x neighbours come from: the adjacent lanes
// (DPP), or, for the first and last pair of a wavefront's run, one halo value
// read from the row (every lane reads it: two addresses per wavefront).
template <typename T, int L>
struct Pair {
  int p, at;  // pair; the halo's place in the row
  bool first, last;
  __device__ __forceinline__ explicit Pair(int p_) : p(p_) {
    const int lane = threadIdx.x & 63;
    first = lane == 0;
    last = lane == 63 || p == L - 1;
    at = last ? 2 * ((p + 1) & (L - 1)) : 2 * ((p - lane - 1) & (L - 1)) + 1;
  }
};
// Quad of a real row in LDS (periodic).  Every lane with a pair executes this.
template <typename T, int L>
__device__ __forceinline__ Quad<T> lds_quad(const c2<T>* row, const Pair<T, L>& pr) {
  const c2<T> a = row[pr.p];
  const T h = reinterpret_cast<const T*>(row)[pr.at];
  const T nl = dpp_mov<kDppWaveShr1>(a.y), nr = dpp_mov<kDppWaveShl1>(a.x);
  return {pr.first ? h : nl, a.x, a.y, pr.last ? h : nr};
}
// quad_dys with the diagonal values from LDS rows.  DIAG: +1 and -1 for an
// offset of one cell (r = 1: the quads' own neighbours), 0 for an even one
// (aligned pairs, hp = off / 2).
template <typename T, int L, int DIAG>
__device__ __forceinline__ void lds_dys(const Quad<T> up, const Quad<T> dn, const c2<T>* rowu,
                                        const c2<T>* rowd, int p, int hp, const Stencil<T>& st,
                                        T& d0, T& d1) {
  T u0, u1, m0, m1;
  if constexpr (DIAG > 0) {
    u0 = up.l; u1 = up.a0; m0 = dn.a1; m1 = dn.r;
  } else if constexpr (DIAG < 0) {
    u0 = up.a1; u1 = up.r; m0 = dn.l; m1 = dn.a0;
  } else {
    const c2<T> pu = rowu[(p - hp) & (L - 1)];
    const c2<T> pd = rowd[(p + hp) & (L - 1)];
    u0 = pu.x; u1 = pu.y; m0 = pd.x; m1 = pd.y;
  }
  d0 = (st.wm * (up.a0 - dn.a0) + st.w * (u0 - m0)) * st.inv2dy;
  d1 = (st.wm * (up.a1 - dn.a1) + st.w * (u1 - m1)) * st.inv2dy;
}
// f(integral constant DIAG) for the block's offset.
template <typename F>
__device__ __forceinline__ void by_diag(int r, int off, F&& f) {
  if (r != 1)
    f(std::integral_constant<int, 0>{});
  else if (off > 0)
    f(std::integral_constant<int, 1>{});
  else
    f(std::integral_constant<int, -1>{});
}

// Stages 0 and 1 of NR rows per block (file header).  Inverse groups: psi
// rows j0-1 .. j0+NR, then omega's (inertial); forward groups: field-major.
template <typename T, int NX, int NR, int NF, int E_>
__global__ __launch_bounds__((FuseCfg<T, NX / 2, NR, NF, E_>::ATPB),
                             (FuseCfg<T, NX / 2, NR, NF, E_>::AWPE)) void k_flow_adv(
    const Run* __restrict__ runs, const StepArgs* __restrict__ sa) {
  using C = FuseCfg<T, NX / 2, NR, NF, E_>;
  constexpr int L = C::L, E = C::E, P = C::P, LS = C::LS, NT = C::ATPB;
  constexpr int SEG = (L + NT - 1) / NT;
  __shared__ c2<T> rows[C::AR * LS];
  __shared__ c2<double> wtab[TwTab<L>::N];
  __shared__ c2<double> wpass[C::Tw::NLDS];
  const BPos bp = block_pos();
  const Run& R = runs[bp.z];
  const Geo& geo = R.g;
  const int ny = geo.ny;
  const int j0 = bp.x * NR;
  const int grp = threadIdx.x / P, t = threadIdx.x % P;
  auto tw = to_global<const c2<double>>(R.twx);
  auto phi = reinterpret_cast<gp<const c2<T>>>(bufp<const T>(R, B_PHI));
  RowsIn<T, L, NR + 2, NT> ps, om;
  ps.get(bufp<const c2<T>>(R, B_PS_S), ny, j0 - 1);
  if constexpr (NF == 3) om.get(bufp<const c2<T>>(R, B_OM_S), ny, j0 - 1);
  c2<T> pv[SEG][NR + 2];
#pragma unroll
  for (int g = 0; g < SEG; ++g) {
    const int p = (int)threadIdx.x + g * NT;
    if (SEG * NT > L && p >= L) break;
#pragma unroll
    for (int r = 0; r < NR + 2; ++r)
      pv[g][r] = ldg<T>(phi + (size_t)wrap_row(j0 - 1 + r, ny) * L + p);
  }
  typename C::Tw ptw;
  ptw.load(tw, t, wpass);
  const c2<double> w0 = ldg<double>(tw + t);
  tw_tab_fill<L, NT>(wtab, tw);
  const Stencil<T> st = make_stencil<T>(geo, sa[bp.z]);
  const T dt = T(geo.dt);
  const bool fh = geo.f_half != 0;
  const int hp = st.off / 2;
  // rows NR + 2 on: omega's, and after it phi's (Stokes: phi's from the start)
  c2<T>* const second = rows + (NR + 2) * LS;
  auto put_phi = [&](c2<T>* dst) {
#pragma unroll
    for (int g = 0; g < SEG; ++g) {
      const int p = (int)threadIdx.x + g * NT;
      if (SEG * NT > L && p >= L) break;
#pragma unroll
      for (int r = 0; r < NR + 2; ++r) dst[r * LS + p] = pv[g][r];
    }
  };
  ps.put(rows, LS);
  if constexpr (NF == 3)
    om.put(second, LS);
  else
    put_phi(second);
  __syncthreads();
  ptw.form();
  if (grp < C::AI) {
    c2<T> v[E];
    rows_c2r<T, L, E>(v, rows + grp * LS, ptw, w0, t);
  }
  __syncthreads();
  by_diag(geo.r, st.off, [&](auto diag) {
    constexpr int D = decltype(diag)::value;
    // psi's differences of the thread's pairs
    T bx0[SEG][NR], bx1[SEG][NR], by0[SEG][NR], by1[SEG][NR];
#pragma unroll
    for (int g = 0; g < SEG; ++g) {
      const int p = (int)threadIdx.x + g * NT;
      if (SEG * NT > L && p >= L) break;
      const Pair<T, L> pr(p);
      Quad<T> m = lds_quad<T, L>(rows, pr), c = lds_quad<T, L>(rows + LS, pr);
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const Quad<T> u = lds_quad<T, L>(rows + (r + 2) * LS, pr);
        quad_dx(c, st.inv2dx, bx0[g][r], bx1[g][r]);
        lds_dys<T, L, D>(u, m, rows + (r + 2) * LS, rows + r * LS, p, hp, st, by0[g][r],
                         by1[g][r]);
        m = c;
        c = u;
        LE_SCHED_FENCE();
      }
    }
    // the advected rows of the field in `second`: emit(g, p, r, value, centre)
    auto adv = [&](auto&& emit) {
#pragma unroll
      for (int g = 0; g < SEG; ++g) {
        const int p = (int)threadIdx.x + g * NT;
        if (SEG * NT > L && p >= L) break;
        const Pair<T, L> pr(p);
        Quad<T> m = lds_quad<T, L>(second, pr), c = lds_quad<T, L>(second + LS, pr);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          const Quad<T> u = lds_quad<T, L>(second + (r + 2) * LS, pr);
          T ax0, ax1, ay0, ay1;
          quad_dx(c, st.inv2dx, ax0, ax1);
          lds_dys<T, L, D>(u, m, second + (r + 2) * LS, second + r * LS, p, hp, st, ay0, ay1);
          emit(g, p, r, c2<T>{c.a0 - dt * (ax0 * by0[g][r] - ay0 * bx0[g][r]),
                              c.a1 - dt * (ax1 * by1[g][r] - ay1 * bx1[g][r])},
               c2<T>{c.a0, c.a1});
          m = c;
          c = u;
          LE_SCHED_FENCE();
        }
      }
    };
    // omega_h and f wait in registers for the rows they overwrite
    c2<T> oh[NF == 3 ? SEG : 1][NR], fv[SEG][NR];
    if constexpr (NF == 3) {
      adv([&](int g, int, int r, c2<T> h, c2<T>) { oh[g][r] = h; });
      __syncthreads();
      put_phi(second);
    }
    __syncthreads();
    adv([&](int g, int p, int r, c2<T> h, c2<T> c) {
      rows[r * LS + p] = h;  // psi's rows are free
      if (fh) c = h;
      fv[g][r] = {c.x * c.x * c.x, c.y * c.y * c.y};
    });
    __syncthreads();
#pragma unroll
    for (int g = 0; g < SEG; ++g) {
      const int p = (int)threadIdx.x + g * NT;
      if (SEG * NT > L && p >= L) break;
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        rows[(NR + r) * LS + p] = fv[g][r];
        if constexpr (NF == 3) rows[(2 * NR + r) * LS + p] = oh[g][r];
      }
    }
  });
  __syncthreads();
  // forward transforms, group f NR + r: phi_h, f, omega_h
  if (grp < C::AO) {
    c2<T> v[E];
#pragma unroll
    for (int q = 0; q < E; ++q) v[q] = rows[grp * LS + t + q * P];
    group_sync<true>();
    rows_r2c_z<T, L, E>(v, rows + grp * LS, ptw, t);
  }
  __syncthreads();
  if constexpr (NF == 3) {
    gp<c2<T>> const X[3] = {bufp<c2<T>>(R, B_PHIH), bufp<c2<T>>(R, B_FH), bufp<c2<T>>(R, B_OMH)};
    rows_out<T, L, NR, 3, NT>(X, rows, LS, wtab, ny, j0);
  } else {
    gp<c2<T>> const X[2] = {bufp<c2<T>>(R, B_PHIH), bufp<c2<T>>(R, B_FH)};
    rows_out<T, L, NR, 2, NT>(X, rows, LS, wtab, ny, j0);
  }
}

// Stages 3 and 4 of NR rows per block: phi rows j0-2 .. j0+NR+1 from the
// spectrum (group g row j0-2+g), the block's own NR rows stored, mu on rows
// j0-1 .. j0+NR over the phi rows' LDS (phi's differences kept in registers),
// g over mu's.
template <typename T, int NX, int NR, int E_>
__global__ __launch_bounds__((FuseCfg<T, NX / 2, NR, 2, E_>::MTPB)) void k_phi_mu(
    const Run* __restrict__ runs, const StepArgs* __restrict__ sa) {
  using C = FuseCfg<T, NX / 2, NR, 2, E_>;
  constexpr int L = C::L, E = C::E, P = C::P, LS = C::LS, NT = C::MTPB;
  constexpr int SEG = (L + NT - 1) / NT;
  __shared__ c2<T> rows[C::MG * LS];
  __shared__ c2<double> wtab[TwTab<L>::N];
  __shared__ c2<double> wpass[C::Tw::NLDS];
  const BPos bp = block_pos();
  const Run& R = runs[bp.z];
  const Geo& geo = R.g;
  const int ny = geo.ny;
  const int j0 = bp.x * NR;
  const int grp = threadIdx.x / P, t = threadIdx.x % P;
  auto tw = to_global<const c2<double>>(R.twx);
  RowsIn<T, L, NR + 4, NT> in;
  in.get(bufp<const c2<T>>(R, B_PHIN), ny, j0 - 2);
  typename C::Tw ptw;
  ptw.load(tw, t, wpass);
  const c2<double> w0 = ldg<double>(tw + t);
  tw_tab_fill<L, NT>(wtab, tw);
  const MuCoef<T> k = make_mu<T>(geo, sa[bp.z].s);
  const Stencil<T> st = make_stencil<T>(geo, sa[bp.z]);
  const T neg_inv = T(geo.ninv);
  const int hp = st.off / 2;
  in.put(rows, LS);
  __syncthreads();
  ptw.form();
  if (grp < C::MI) {
    c2<T> v[E];
    rows_c2r<T, L, E>(v, rows + grp * LS, ptw, w0, t);
    if (grp >= 2 && grp < NR + 2) {
      auto phi = reinterpret_cast<gp<c2<T>>>(bufp<T>(R, B_PHI)) + (size_t)(j0 - 2 + grp) * L;
#pragma unroll
      for (int q = 0; q < E; ++q) stg<T>(phi + t + q * P, v[q]);
    }
  }
  __syncthreads();
  by_diag(geo.r, st.off, [&](auto diag) {
    constexpr int D = decltype(diag)::value;
    T px0[SEG][NR], px1[SEG][NR], py0[SEG][NR], py1[SEG][NR];
    c2<T> mu[SEG][NR + 2];
#pragma unroll
    for (int g = 0; g < SEG; ++g) {
      const int p = (int)threadIdx.x + g * NT;
      if (SEG * NT > L && p >= L) break;
      const Pair<T, L> pr(p);
      Quad<T> d = lds_quad<T, L>(rows, pr), c = lds_quad<T, L>(rows + LS, pr);
#pragma unroll
      for (int r = 0; r < NR + 2; ++r) {
        const c2<T>* ru = rows + (r + 2) * LS;
        const Quad<T> u = lds_quad<T, L>(ru, pr);
        mu[g][r] = {mu_at(k, d.l, d.a0, d.a1, c.l, c.a0, c.a1, u.l, u.a0, u.a1),
                    mu_at(k, d.a0, d.a1, d.r, c.a0, c.a1, c.r, u.a0, u.a1, u.r)};
        if (r >= 1 && r <= NR) {
          quad_dx(c, st.inv2dx, px0[g][r - 1], px1[g][r - 1]);
          lds_dys<T, L, D>(u, d, ru, rows + r * LS, p, hp, st, py0[g][r - 1], py1[g][r - 1]);
        }
        d = c;
        c = u;
        LE_SCHED_FENCE();
      }
    }
    __syncthreads();
#pragma unroll
    for (int g = 0; g < SEG; ++g) {
      const int p = (int)threadIdx.x + g * NT;
      if (SEG * NT > L && p >= L) break;
#pragma unroll
      for (int r = 0; r < NR + 2; ++r) rows[r * LS + p] = mu[g][r];
    }
    __syncthreads();
    c2<T> gv[SEG][NR];
#pragma unroll
    for (int g = 0; g < SEG; ++g) {
      const int p = (int)threadIdx.x + g * NT;
      if (SEG * NT > L && p >= L) break;
      const Pair<T, L> pr(p);
      Quad<T> d = lds_quad<T, L>(rows, pr), c = lds_quad<T, L>(rows + LS, pr);
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const c2<T>* ru = rows + (r + 2) * LS;
        const Quad<T> u = lds_quad<T, L>(ru, pr);
        T mx0, mx1, my0, my1;
        quad_dx(c, st.inv2dx, mx0, mx1);
        lds_dys<T, L, D>(u, d, ru, rows + r * LS, p, hp, st, my0, my1);
        gv[g][r] = {neg_inv * (px0[g][r] * my0 - py0[g][r] * mx0),
                    neg_inv * (px1[g][r] * my1 - py1[g][r] * mx1)};
        d = c;
        c = u;
        LE_SCHED_FENCE();
      }
    }
    __syncthreads();
#pragma unroll
    for (int g = 0; g < SEG; ++g) {
      const int p = (int)threadIdx.x + g * NT;
      if (SEG * NT > L && p >= L) break;
#pragma unroll
      for (int r = 0; r < NR; ++r) rows[r * LS + p] = gv[g][r];
    }
  });
  __syncthreads();
  if (grp < NR) {
    c2<T> v[E];
#pragma unroll
    for (int q = 0; q < E; ++q) v[q] = rows[grp * LS + t + q * P];
    group_sync<true>();
    rows_r2c_z<T, L, E>(v, rows + grp * LS, ptw, t);
  }
  __syncthreads();
  gp<c2<T>> const X[1] = {bufp<c2<T>>(R, B_GH)};
  rows_out<T, L, NR, 1, NT>(X, rows, LS, wtab, ny, j0);
}

}  // namespace le

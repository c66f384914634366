// me_qew_pol.h -- the quark-line + lepton-pair processes summed over spins with
// real polarisation vectors: 2^NG lanes per event, lane l the gluon
// polarisations l.
//
// With real polarisations every gluon current and every propagator of the
// massless line is real, so the line of the other chirality is the complex
// conjugate of this one (with eps conj in place of a two-spinor): only one
// chirality is evaluated, as two-spinors, and the line enters through
//   T^mu = sum over cuts of L(first gluons) sigma^mu R(the rest),
// one complex vector per ordering that does not know the leptons.  The four
// spin states of quark and lepton line are then products with the vectors E_R
// and conj E_L of each lepton spin (qew_externals' insertion).  Colour-ordered
// rules, signs and currents as in me_wave.h.
//
// Against one helicity per pass over the diagram program (k_me_qew) this is
// about a tenth of the arithmetic: 2^20 events of g ubar -> tau+ tau- g g ubar
// take 0.88 ms (0.96 to 1.1 when the clock has come down under a longer load) against
// 8.73 ms.  3,430 vector instructions per wave of eight
// events, the VALU active 91 % of the time: bound by VALU issue.  Eight lanes
// share the externals in LDS; each lane forms its own currents and rows, since
// sharing those too would save less than a fifth and cost a barrier per stage.
#pragma once
#include "me_qew.h"
#include "me_wave.h"

namespace qp {

using namespace wv;

struct two {  // two-spinor
    c2 a, b;
};
// f (W.sigma) of a row: (f0, f1) to the other chirality, and back
MEV two row1(const two& f, const vec& W) {
    const double p = W.v[0] + W.v[3], m = W.v[0] - W.v[3];
    const c2 c{W.v[1], W.v[2]}, d{W.v[1], -W.v[2]};
    return {axpy(m, f.a, f.b * -c), axpy(p, f.b, f.a * -d)};
}
MEV two row2(const two& f, const vec& W) {
    const double p = W.v[0] + W.v[3], m = W.v[0] - W.v[3];
    const c2 c{W.v[1], W.v[2]}, d{W.v[1], -W.v[2]};
    return {axpy(p, f.a, f.b * c), axpy(m, f.b, f.a * d)};
}
// (W.sigma) of a column, one way and back
MEV two col1(const vec& W, const two& r) {
    const double p = W.v[0] + W.v[3], m = W.v[0] - W.v[3];
    const c2 c{W.v[1], W.v[2]}, d{W.v[1], -W.v[2]};
    return {axpy(m, r.a, r.b * -d), axpy(p, r.b, r.a * -c)};
}
MEV two col2(const vec& W, const two& r) {
    const double p = W.v[0] + W.v[3], m = W.v[0] - W.v[3];
    const c2 c{W.v[1], W.v[2]}, d{W.v[1], -W.v[2]};
    return {axpy(p, r.a, r.b * d), axpy(m, r.b, r.a * c)};
}
MEV two operator+(const two& x, const two& y) { return {x.a + y.a, x.b + y.b}; }
MEV two operator-(const two& x, const two& y) { return {x.a - y.a, x.b - y.b}; }

// T: coefficients of (E0 + E3, E0 - E3, -(E1 + i E2), -(E1 - i E2))
struct line {
    c2 t[4];
};
MEV void cut(line& T, const two& f, const two& r) {
    T.t[0] = cfma(f.b, r.b, T.t[0]);
    T.t[1] = cfma(f.a, r.a, T.t[1]);
    T.t[2] = cfma(f.b, r.a, T.t[2]);
    T.t[3] = cfma(f.a, r.b, T.t[3]);
}

// One event's block in LDS, in doubles.
template <int NG>
struct layout {
    enum {
        SUBS = (1 << NG) - 1,
        Q = 0,                    // gluons, incoming flow [NG][4]
        SLOT = Q + 4 * NG,        // row end, column end, insertion, l-, l+ [5][4]
        PL = SLOT + 20,           // -P/P^2 after the gluons of a subset from the row end [SUBS][4]
        PR = PL + 4 * SUBS,       // the same from the column end
        IQ = PR + 4 * SUBS,       // 1/Q_S^2 by subset [SUBS + 1]
        EPS = IQ + SUBS + 1,      // g e [NG][2][4]
        F = EPS + 8 * NG,         // row end, two complex
        R = F + 4,                // column end
        E = R + 4,                // [4][4 complex], as line
        SIZE = E + 32,
        // odd multiples of 16 bytes: events on different banks
        STRIDE = SIZE % 4 == 2 ? SIZE : (SIZE + 3) / 4 * 4 + 2
    };
};

MEV vec ld4(const double* p) {
    const double2* q = reinterpret_cast<const double2*>(p);
    const double2 a = q[0], b = q[1];
    return {{a.x, a.y, b.x, b.y}};
}
MEV void st4(double* p, const vec& w) {
    double2* q = reinterpret_cast<double2*>(p);
    q[0] = double2{w.v[0], w.v[1]};
    q[1] = double2{w.v[2], w.v[3]};
}
MEV two ld2(const double* p) {
    const vec w = ld4(p);
    return {{w.v[0], w.v[1]}, {w.v[2], w.v[3]}};
}

// Whether the line momentum after subset S is taken from the row end (p3 - Q_S)
// rather than the column end (Q_rest - p4): the form with fewer beam momenta.
template <class P>
MEV bool from_row(int S) {
    int in = P::row_in, out = P::col_in;
#pragma unroll
    for (int a = 0; a < P::ngluon; ++a) (((S >> a) & 1) ? in : out) += P::gluon_in[a];
    return in <= out;
}

}  // namespace qp

// idx and count as for k_me_ee; first0: the launch's first event (or entry of idx).
template <class P>
__global__ __launch_bounds__(64, 2) void k_me_qew_pol(const double* __restrict__ mom, int64_t nevt,
                                                      double* __restrict__ out, me_params prm,
                                                      const int* __restrict__ idx, const int* __restrict__ count,
                                                      int64_t first0) {
    using namespace qp;
    constexpr int NG = P::ngluon, G = 1 << NG, FULL = G - 1;
    using Y = layout<NG>;
    __shared__ double2 mem[(64 >> NG) * (Y::STRIDE / 2)];
    const int lane = threadIdx.x, l = lane & (G - 1), e = lane >> NG;
    const int64_t n = count ? (int64_t)*count : nevt;
    const int64_t first = first0 + (int64_t)blockIdx.x * (64 >> NG);
    if (first >= n) return;
    int64_t i = first + e;
    const bool valid = i < n;
    if (!valid) i = n - 1;
    const int64_t ev = count ? (int64_t)idx[i] : i;
    double* const D = reinterpret_cast<double*>(mem) + e * Y::STRIDE;
    const double* pe = mom + ev * (P::npart * 4);

    // ---- externals, handed out over the event's lanes ----
#pragma unroll
    for (int k0 = 0; k0 < NG + 4; k0 += G) {  // gluons, row, column, l-, l+
        const int k = k0 + l;
        if (k < NG + 4) {
            int part = P::lp_part;
            double sg = 1.0;
#pragma unroll
            for (int a = 0; a < NG; ++a)
                if (k == a) part = P::gluon_part[a], sg = P::gluon_in[a] ? 1.0 : -1.0;
            if (k == NG) part = P::row_part, sg = P::row_in ? -1.0 : 1.0;
            if (k == NG + 1) part = P::col_part, sg = P::col_in ? -1.0 : 1.0;
            if (k == NG + 2) part = P::lm_part;
            const double* p = pe + 4 * part;
            st4(D + (k < NG ? Y::Q + 4 * k : Y::SLOT + 4 * (k - NG + (k >= NG + 2))), vec{{sg * p[0], sg * p[1], sg * p[2], sg * p[3]}});
        }
    }
    __syncthreads();
    const vec qE = mul(-1.0, add(ld4(D + Y::SLOT + 12), ld4(D + Y::SLOT + 16)));
    for (int k = l; k < 3 * FULL; k += G) {  // propagators: from the row, from the column, of gluon sets
        const int kind = k / FULL, S = k % FULL + 1;
        // the line momentum after U from the row end, or U's momentum
        const int U = kind == 1 ? FULL & ~S : S;
        const bool row = kind == 2 || from_row<P>(U);
        vec K{{0.0, 0.0, 0.0, 0.0}};
#pragma unroll
        for (int a = 0; a < NG; ++a) {
            const double w = ((row ? U : FULL & ~U) >> a) & 1 ? 1.0 : 0.0;
            const vec q = ld4(D + Y::Q + 4 * a);
#pragma unroll
            for (int c = 0; c < 4; ++c) K.v[c] = fma(w, q.v[c], K.v[c]);
        }
        if (kind != 2) {
            const double w = row == (kind == 1) ? 1.0 : 0.0;  // the insertion is on the summed side
            const vec end = ld4(D + Y::SLOT + (row ? 0 : 4));
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const double s = fma(w, qE.v[c], K.v[c]);
                K.v[c] = row ? end.v[c] - s : s - end.v[c];
            }
        }
        const double r = 1.0 / (K.v[0] * K.v[0] - K.v[1] * K.v[1] - K.v[2] * K.v[2] - K.v[3] * K.v[3]);
        if (kind == 2)
            D[Y::IQ + S] = r;
        else
            st4(D + (kind ? Y::PR : Y::PL) + 4 * (S - 1), mul(-r, K));
    }
    for (int k = l; k < 2 * NG; k += G) {  // polarisation vectors
        const int a = k >> 1;
        bool in = false;
#pragma unroll
        for (int b = 0; b < NG; ++b) in = (a == b) ? (bool)P::gluon_in[b] : in;
        const vec q = ld4(D + Y::Q + 4 * a);
        st4(D + Y::EPS + 4 * k, mul(prm.gs, polarisation(in ? q : mul(-1.0, q), k & 1)));
    }
    if (l < 2) {  // ends of the line: sqrt(2E) (conj chi_+, chi_+)
        const vec q = ld4(D + Y::SLOT + 4 * l);
        const double sg = (l ? P::col_in : P::row_in) ? -1.0 : 1.0;
        const mom4<double> p{sg * q.v[0], sg * q.v[1], sg * q.v[2], sg * q.v[3]};
        double pabs, wm, wp;
        spinor_weights(p, 0.0, pabs, wm, wp);
        c2 h0, h1;
        helicity_chi(p, pabs, 1, h0, h1);
        const double s = l ? 1.0 : -1.0;
        st4(D + (l ? Y::R : Y::F), vec{{wp * h0.r, s * wp * h0.i, wp * h1.r, s * wp * h1.i}});
    }
    for (int k = l; k < 4; k += G) {  // insertion: (lepton spin, E_R or conj E_L)
        const vec pm = ld4(D + Y::SLOT + 12), pp = ld4(D + Y::SLOT + 16);
        const int s = (k & 1) ? 1 : -1;
        const spinor<double> ub = bar(u_spinor(mom4<double>{pm.v[0], pm.v[1], pm.v[2], pm.v[3]}, 0.0, s));
        const spinor<double> v = v_spinor(mom4<double>{pp.v[0], pp.v[1], pp.v[2], pp.v[3]}, 0.0, -s);
        vec4<double> jl, jr;
        fbar_gamma_f_lr(ub, v, jl, jr);
        const double k2 = mdot(qE, qE), sw2 = prm.sw2, gz2 = prm.gz * prm.gz;
        const double g_q = (k & 2) ? P::q_t3 - P::q_charge * sw2 : -P::q_charge * sw2;
        const double gl = P::l_t3 - P::l_charge * sw2, gr = -P::l_charge * sw2;
        const c2 iz = (gz2 * g_q) * crecip(k2 - prm.mz * prm.mz, prm.mz * prm.wz);
        const double ga = prm.e * prm.e * P::q_charge * P::l_charge / k2;
        c2 E[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            E[c] = ga * (jl.v[c] + jr.v[c]) + iz * (gl * jl.v[c] + gr * jr.v[c]);
            if (k & 2) E[c] = conj(E[c]);
        }
        const c2 lc[4] = {E[0] + E[3], E[0] - E[3], -(E[1] + times_i(E[2])), -(E[1] - times_i(E[2]))};
#pragma unroll
        for (int c = 0; c < 4; ++c)
            reinterpret_cast<double2*>(D + Y::E)[4 * k + c] = double2{lc[c].r, lc[c].i};
    }
    __syncthreads();

    // ---- the line at this lane's polarisations ----
    const two L0 = ld2(D + Y::F), R0 = ld2(D + Y::R);
    auto eps = [&](int a) __attribute__((always_inline)) { return ld4(D + Y::EPS + 8 * a + 4 * bit(l, a)); };
    auto pl = [&](int S) __attribute__((always_inline)) { return ld4(D + Y::PL + 4 * (S - 1)); };
    auto pr = [&](int S) __attribute__((always_inline)) { return ld4(D + Y::PR + 4 * (S - 1)); };
    auto mg = [&](int a) __attribute__((always_inline)) { return ld4(D + Y::Q + 4 * a); };
    line T[P::ncol];
    each<P::ncol>([&](auto K) __attribute__((always_inline)) {
        each<4>([&](auto C) __attribute__((always_inline)) { T[K].t[C] = c2{0.0, 0.0}; });
    });
    if constexpr (NG == 1) {
        const vec e0 = eps(0);
        cut(T[0], L0, col2(pr(1), col1(e0, R0)));
        cut(T[0], row2(row1(L0, e0), pl(1)), R0);
    } else {
        // pair currents (sorted) and R(d)
        constexpr int NP2 = NG * (NG - 1) / 2;
        vec W[NP2], W3[3];
        auto pidx = [](int a, int b) constexpr { return a + b - 1; };  // (0,1) 0, (0,2) 1, (1,2) 2
        each<NG>([&](auto B) __attribute__((always_inline)) {
            each<B>([&](auto A) __attribute__((always_inline)) {
                vec w{{0.0, 0.0, 0.0, 0.0}};
                sub_vvv(w, eps(A), mg(A), eps(B), mg(B));
                W[pidx(A, B)] = mul(D[Y::IQ + (1 << A) + (1 << B)], w);
            });
        });
        if constexpr (NG == 3) {
            // middle 1: (0, 1, 2); middle 0: (1, 0, 2); middle 2: minus their sum
            const vec q0 = mg(0), q1 = mg(1), q2 = mg(2);
            const double iq = D[Y::IQ + 7];
            vec a{{0.0, 0.0, 0.0, 0.0}}, b{{0.0, 0.0, 0.0, 0.0}};
            const vec q01 = add(q0, q1);
            sub_vvv(a, W[0], q01, eps(2), q2);
            sub_vvv(b, mul(-1.0, W[0]), q01, eps(2), q2);
            sub_vvv(a, eps(0), q0, W[2], add(q1, q2));
            sub_vvv(b, eps(1), q1, W[1], add(q0, q2));
            add_vvvv(a, eps(0), eps(1), eps(2));
            add_vvvv(b, eps(1), eps(0), eps(2));
            W3[1] = mul(iq, a);
            W3[0] = mul(iq, b);
            W3[2] = mul(-1.0, add(W3[0], W3[1]));
        }
        two R1[NG];
        each<NG>([&](auto A) __attribute__((always_inline)) { R1[A] = col2(pr(1 << A), col1(eps(A), R0)); });
        // one ordered pair current
        auto row_w = [&](const two& f, auto A, auto B) __attribute__((always_inline)) {
            const two r = row1(f, W[pidx(A, B)]);
            return A < B ? r : two{-r.a, -r.b};
        };
        auto col_w = [&](auto A, auto B, const two& f) __attribute__((always_inline)) {
            const two r = col1(W[pidx(A, B)], f);
            return A < B ? r : two{-r.a, -r.b};
        };
        each<NG>([&](auto A) __attribute__((always_inline)) {
            const vec eA = eps(A);
            const two l1 = row2(row1(L0, eA), pl(1 << A));
            each<NG>([&](auto B) __attribute__((always_inline)) {
                if constexpr (A != B) {
                    const vec eB = eps(B);
                    const two l2 = row2(row1(l1, eB) + row_w(L0, A, B), pl((1 << A) + (1 << B)));
                    if constexpr (NG == 2) {
                        const two r2 = col2(pr(3), col1(eA, R1[B]) + col_w(A, B, R0));
                        constexpr int k = A;
                        cut(T[k], L0, r2);
                        cut(T[k], l1, R1[B]);
                        cut(T[k], l2, R0);
                    } else {
                        constexpr int C = 3 - A - B, k = 2 * A + (B > C);
                        using IC = std::integral_constant<int, C>;
                        const vec eC = eps(C);
                        const two r2 = col2(pr((1 << B) + (1 << C)), col1(eB, R1[C]) + col_w(B, IC{}, R0));
                        const two l3 = row2(row1(l2, eC) + row_w(l1, B, IC{}) + row1(L0, W3[B]), pl(7));
                        const two r3 = col2(pr(7), col1(eA, r2) + col_w(A, B, R1[C]) + col1(W3[B], R0));
                        cut(T[k], L0, r3);
                        cut(T[k], l1, r2);
                        cut(T[k], l2, R1[C]);
                        cut(T[k], l3, R0);
                        settle(T[k].t);
                    }
                }
            });
        });
    }
    // ---- the four spin states of the lines, and the colour sum ----
    double acc = 0.0;
#pragma unroll 1
    for (int k = 0; k < 4; ++k) {
        const double2* Ep = reinterpret_cast<const double2*>(D + Y::E) + 4 * k;
        const double2 x0 = Ep[0], x1 = Ep[1], x2 = Ep[2], x3 = Ep[3];
        const c2 E[4] = {{x0.x, x0.y}, {x1.x, x1.y}, {x2.x, x2.y}, {x3.x, x3.y}};
        c2 J[P::ncol];
        each<P::ncol>([&](auto F) __attribute__((always_inline)) {
            J[F] = cfma(T[F].t[3], E[3], cfma(T[F].t[2], E[2], cfma(T[F].t[1], E[1], T[F].t[0] * E[0])));
        });
        acc += P::template colour_blocks<double>(J);
    }
    const double tot = group_sum(acc, NG);
    if (valid && l == 0) out[ev] = tot * (1.0 / (P::avg * P::lcd));
}

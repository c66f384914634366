// me_gg_pol.h -- g g -> t tbar and g g -> t tbar g summed over spins with real
// polarisation vectors.  Rules, signs and the row form of columns as in
// me_wave.h.
//
// Two gluons: one event per lane (small calls: four lanes), everything in registers.  The configurations
// share four one-gluon rows per ordering and spin.
//   J_ab = L(a) W(b) v + ubar W(ab) v.
// Three gluons: eight lanes per event (small calls: 32), lane l the gluon polarisations l; the
// externals, one-gluon rows, pair currents and the current of the line's ends
// are computed once per event and shared in LDS, the rest by each lane for its
// polarisations and the four spin pairs.
//   J_abc = L(a) [W(b) R(c) + W(bc) v] + ubar W(ab) R(c) + ubar W(abc) v.
//
// Both are bound by VALU issue (2,600 vector instructions per wave of 64 events
// and of eight).  Against one helicity per pass over the diagram program
// (k_me_gg): 2^20 events of g g -> t tbar take 92 us against 521 us, 2^18
// events of g g -> t tbar g 0.30 ms against 2.7 ms; with the weights of the
// events' channels 2^19 events of g g -> t tbar 65 us against 316 us, 2^17 events
// of g g -> t tbar g 0.24 ms against 0.55 ms (k_me_gg_mc).
#pragma once
#include "me_qew_pol.h"

namespace g2 {

using namespace wv;

// f (gamma.e) for a polarisation vector: no time component, e2 none along z.
template <bool E2>
MEV row slash_e(const row& f, const vec& e) {
    const c2 c{e.v[1], e.v[2]}, d{e.v[1], -e.v[2]};
    if constexpr (E2) return {{f.s[3] * c, f.s[2] * d, f.s[1] * -c, f.s[0] * -d}};
    const double z = e.v[3];
    return {{axpy(z, f.s[2], f.s[3] * c), axpy(-z, f.s[3], f.s[2] * d), axpy(-z, f.s[0], f.s[1] * -c),
             axpy(z, f.s[1], f.s[0] * -d)}};
}
// f gamma_mu R for mu = 1, 2, 3, R held as the row r, dotted with e1 and e2
MEV void currents_e(const row& f, const row& r, const vec& e1, const vec& e2, c2& d1, c2& d2) {
    const c2 u = cfma(f.s[2], r.s[0], f.s[0] * r.s[2]), v = cfma(f.s[3], r.s[1], f.s[1] * r.s[3]);
    const c2 x = u - v, y = times_mi(u + v);
    const c2 z = cfma(f.s[3], r.s[0], cfma(f.s[2], r.s[1], cfma(f.s[1], r.s[2], f.s[0] * r.s[3])));
    d1 = axpy(-e1.v[3], z, axpy(e1.v[2], y, rmul(e1.v[1], x)));
    d2 = axpy(e2.v[2], y, rmul(e2.v[1], x));
}

}  // namespace g2

// idx, count and spins as for k_me_gg4_wave; first0: the launch's first event (or
// entry of idx).  With IDS (the channel numbers of
// the diagrams) also the single-diagram weight of each event's channel, as k_me_gg4_chan.
// LANES: lanes per event, one for all spin pairs or four with one each, for calls
// that leave most of the chip idle (2,049 events 4.9 us instead of 7.8; one helicity per
// lane 5.7).  The pairs are added in the same order either way.
template <class P, class IDS = void, int LANES = 1>
__global__ __launch_bounds__(64, 2) void k_me_gg2_pol(const double* __restrict__ mom, int64_t nevt,
                                                      double* __restrict__ out, unsigned spins, me_params prm,
                                                      const int* __restrict__ idx, const int* __restrict__ count,
                                                      int64_t first0,
                                                      const int* __restrict__ chan = nullptr,
                                                      double* __restrict__ alpha = nullptr) {
    using namespace g2;
    static_assert(P::ngluon == 2 && P::ncol == 2, "two gluons");
    const int64_t at = (int64_t)blockIdx.x * 64 + threadIdx.x;
    int64_t ev = first0 + at / LANES;
    if (count) {
        if (ev >= *count) return;
        ev = idx[ev];
    } else if (ev >= nevt) {
        return;
    }
    constexpr bool MC = !std::is_void_v<IDS>;
    static_assert(LANES == 1 || (LANES == 4 && !MC), "the weights are summed by one lane");
    const double m = prm.mt;
    const int ch = MC ? chan[ev] : 0;
    double num = 0.0, den = 0.0;
    auto found = [&](auto id, c2 a) __attribute__((always_inline)) {
        const double a2 = fma(a.r, a.r, a.i * a.i);
        den += a2;
        num += id == ch ? a2 : 0.0;
        asm volatile("" : "+v"(den), "+v"(num));
    };
    vec q[2], p3, p4;
    {
        const double* pe = mom + ev * 16;
        auto ld = [&](int k) __attribute__((always_inline)) {
            return vec{{pe[4 * k], pe[4 * k + 1], pe[4 * k + 2], pe[4 * k + 3]}};
        };
        q[0] = ld(0), q[1] = ld(1), p3 = ld(2), p4 = ld(3);
    }
    // end rows by spin, or of this lane's spins
    const int l = (int)threadIdx.x & (LANES - 1);
    row n3[2], n4[2];
    if constexpr (LANES == 1) {
        each<2>([&](auto S) __attribute__((always_inline)) {
            n3[S] = end_row(p3, m, 0, S ? 1 : -1);
            n4[S] = end_row(p4, m, 1, S ? 1 : -1);
        });
    } else {
        n3[0] = end_row(p3, m, 0, (l & 2) ? 1 : -1);
        n4[0] = end_row(p4, m, 1, (l & 1) ? 1 : -1);
    }
    vec e[2][2], K[2];
    c2 f[2];
    each<2>([&](auto A) __attribute__((always_inline)) {
        e[A][0] = mul(prm.gs, polarisation(q[A], false));
        e[A][1] = mul(prm.gs, polarisation(q[A], true));
        K[A] = add(p3, mul(-1.0, q[A]));
        f[A] = crecip(mdot(K[A], K[A]) - m * m, m * prm.wt);
    });
    vec w[4];  // W(01) by polarisations
    {
        const vec Q = add(q[0], q[1]);
        const double iq = 1.0 / mdot(Q, Q);
        each<4>([&](auto PP) __attribute__((always_inline)) {
            vec t{{0.0, 0.0, 0.0, 0.0}};
            sub_vvv(t, e[0][PP % 2], q[0], e[1][PP / 2], q[1]);
            w[PP] = mul(iq, t);
        });
    }
    // L(a) up to the sign, by gluon and polarisation, at one spin of t
    auto lines = [&](const row& u, row(&L)[2][2]) __attribute__((always_inline)) {
        each<4>([&](auto I) __attribute__((always_inline)) {
            L[I / 2][I % 2] = scale(f[I / 2], slash_m(slash_e<I % 2>(u, e[I / 2][I % 2]), K[I / 2], m));
        });
    };
    // colour sum over the polarisations at one spin pair
    auto spin_pair = [&](const row& u, const row& v, const row(&L)[2][2]) __attribute__((always_inline)) {
        c2 t[4], J01[4], J10[4];  // by polarisations
        {
            const row V = current(u, v);
            each<4>([&](auto PP) __attribute__((always_inline)) { t[PP] = cdot(V, w[PP]); });
            settle(t);
        }
        each<2>([&](auto A) __attribute__((always_inline)) {
            currents_e(L[0][A], v, e[1][0], e[1][1], J01[A], J01[A + 2]);
            currents_e(L[1][A], v, e[0][0], e[0][1], J10[2 * A], J10[1 + 2 * A]);
        });
        settle(J01), settle(J10);
        double part = 0.0;
        each<4>([&](auto PP) __attribute__((always_inline)) {
            if constexpr (MC) found(IDS::tree[0], t[PP]), found(IDS::order[0], J01[PP]), found(IDS::order[1], J10[PP]);
            c2 J[2] = {J01[PP] - t[PP], J10[PP] + t[PP]};  // (both with the sign of L)
            part += P::colour_blocks(J);
        });
        return part;
    };
    double acc = 0.0;
    if constexpr (LANES == 1) {
        // Spin by spin: the rows L of all sixteen at once do not fit in registers (2^20
        // events took 126 us).  The other end enters through the current of L with it,
        // which both polarisations of the second gluon share (92 us; 110 with the
        // end's rows slashed by each of them).
        each<2>([&](auto S3) __attribute__((always_inline)) {
            settle(n4[0].s), settle(n4[1].s);  // what is formed from them is not kept for the other spin
            row L[2][2];
            lines(n3[S3], L);
            each<2>([&](auto S4) __attribute__((always_inline)) {
                const double part = spin_pair(n3[S3], n4[S4], L);
                acc += ((spins >> (S3 + 2 * S4)) & 1) ? part : 0.0;
                asm volatile("" : "+v"(acc));  // or the sums sink below the next ones, their operands held
            });
        });
    } else {
        row L[2][2];
        lines(n3[0], L);
        double part = spin_pair(n3[0], n4[0], L);
        part = ((spins >> ((l >> 1) + 2 * (l & 1))) & 1) ? part : 0.0;
        each<4>([&](auto S) __attribute__((always_inline)) { acc += __shfl(part, S, 4); });
    }
    if (l == 0) out[ev] = acc * (1.0 / (256.0 * P::identical * P::lcd));
    if constexpr (MC) alpha[ev] = num / den;
}

namespace g3 {

using namespace qp;

// One event's block in LDS, in doubles.
enum {
    Q = 0,             // gluons in incoming flow, p3, p4 [5][4]
    K = Q + 20,        // p3 - q_a, p4 - q_a [6][4]
    F = K + 24,        // their propagators, complex [6]
    IQ = F + 12,       // 1/Q^2 of pairs (01), (02), (12), of all three, 1/(p3 + p4)^2, (pad) [6]
    EPS = IQ + 6,      // g e [3][2][4]
    N0 = EPS + 24,     // end rows [end][spin][8]
    N1 = N0 + 32,      // one-gluon rows [end][gluon][pol][spin][8]
    W2 = N1 + 192,     // pair currents [pair][pols][4]
    C0 = W2 + 48,      // current of the ends [spins][8], with the gluon propagator
    SIZE = C0 + 32,
    STRIDE = SIZE % 4 == 2 ? SIZE : (SIZE + 3) / 4 * 4 + 2
};

MEV row ld8(const double* p) {
    const vec a = ld4(p), b = ld4(p + 4);
    return {{{a.v[0], a.v[1]}, {a.v[2], a.v[3]}, {b.v[0], b.v[1]}, {b.v[2], b.v[3]}}};
}
MEV void st8(double* p, const row& f) {
    st4(p, vec{{f.s[0].r, f.s[0].i, f.s[1].r, f.s[1].i}});
    st4(p + 4, vec{{f.s[2].r, f.s[2].i, f.s[3].r, f.s[3].i}});
}

}  // namespace g3

// LANES: lanes per event, eight for its polarisations, which take the spin pairs in
// turn, or 32 with a spin pair each, for calls that leave most of the chip idle (511 events
// 6.8 us instead of 10.0; one helicity per lane 9.8).  The pairs are added in the same
// order either way.
template <class P, class IDS = void, int LANES = 8>
__global__ __launch_bounds__(64, 2) void k_me_gg3_pol(const double* __restrict__ mom, int64_t nevt,
                                                      double* __restrict__ out, unsigned spins, me_params prm,
                                                      const int* __restrict__ idx, const int* __restrict__ count,
                                                      int64_t first0,
                                                      const int* __restrict__ chan = nullptr,
                                                      double* __restrict__ alpha = nullptr) {
    using namespace g3;
    static_assert(P::ngluon == 3 && P::ncol == 6, "three gluons");
    constexpr bool MC = !std::is_void_v<IDS>;
    static_assert(LANES == 8 || (LANES == 32 && !MC), "the weights are summed by eight lanes");
    constexpr int EV = 64 / LANES;  // events per wave
    __shared__ double2 mem[EV * (STRIDE / 2)];
    const int lane = threadIdx.x, ln = lane & (LANES - 1), l = lane & 7, e = lane / LANES;
    const double m = prm.mt;
    const int64_t n = count ? (int64_t)*count : nevt;
    const int64_t first = first0 + (int64_t)blockIdx.x * EV;
    if (first >= n) return;
    int64_t i = first + e;
    const bool valid = i < n;
    if (!valid) i = n - 1;
    const int64_t ev = count ? (int64_t)idx[i] : i;
    const int ch = MC ? chan[ev] : 0;
    double num = 0.0, den = 0.0;
    auto found = [&](auto id, c2 a) __attribute__((always_inline)) {
        const double a2 = fma(a.r, a.r, a.i * a.i);
        den += a2;
        num += id == ch ? a2 : 0.0;
        asm volatile("" : "+v"(den), "+v"(num));
    };
    double* const D = reinterpret_cast<double*>(mem) + e * STRIDE;
    if (ln < 5) {  // slots: gluons 0, 1, 2 (particle 4), p3, p4
        const double* p = mom + ev * 20 + 4 * (ln < 2 ? ln : ln == 2 ? 4 : ln - 1);
        const double sg = ln == 2 ? -1.0 : 1.0;
        st4(D + Q + 4 * ln, vec{{sg * p[0], sg * p[1], sg * p[2], sg * p[3]}});
    }
    __syncthreads();
    for (int k = ln; k < 11; k += LANES) {  // summed momenta and propagators
        const vec q0 = ld4(D + Q), q1 = ld4(D + Q + 4), q2 = ld4(D + Q + 8);
        const vec end = ld4(D + Q + (k < 3 || k == 10 ? 12 : 16));
        const int a = k < 3 ? k : k - 3;
        const vec qa = ld4(D + Q + 4 * (a < 3 ? a : 0)), p4 = ld4(D + Q + 16);
        vec s;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const double x = k == 8 ? q1.v[c] : q0.v[c];
            const double y = k == 6 ? q1.v[c] : q2.v[c];
            s.v[c] = k < 6 ? end.v[c] - qa.v[c] : k < 9 ? x + y : k == 9 ? q0.v[c] + q1.v[c] + q2.v[c] : end.v[c] + p4.v[c];
        }
        const double d = s.v[0] * s.v[0] - s.v[1] * s.v[1] - s.v[2] * s.v[2] - s.v[3] * s.v[3];
        const c2 f = crecip(k < 6 ? d - m * m : d, k < 6 ? m * prm.wt : 0.0);
        if (k < 6) {
            st4(D + K + 4 * k, s);
            D[F + 2 * k] = f.r;
            D[F + 2 * k + 1] = f.i;
        } else {
            D[IQ + k - 6] = f.r;
        }
    }
    if (ln < 6) {  // polarisation vectors (gluon, which)
        const vec q = ld4(D + Q + 4 * (ln >> 1));
        st4(D + EPS + 4 * ln, mul(prm.gs, polarisation(ln < 4 ? q : mul(-1.0, q), ln & 1)));
    }
    if (ln < 4)  // end rows (end, spin)
        st8(D + N0 + 8 * ln, end_row(ld4(D + Q + 12 + 4 * (ln >> 1)), m, ln >> 1, (ln & 1) ? 1 : -1));
    __syncthreads();
#pragma unroll
    for (int r = 0; r < (LANES == 8 ? 3 : 1); ++r) {  // one-gluon rows (end, gluon, pol, spin); L(a) up to the sign
        if (LANES > 24 && ln >= 24) break;
        const int k = 8 * r + ln, en = k >= 12, a = (k >> 2) - 3 * en, pol = (k >> 1) & 1, s = k & 1;
        const row f = slash_m(slash(ld8(D + N0 + 16 * en + 8 * s), ld4(D + EPS + 8 * a + 4 * pol)),
                              ld4(D + K + 4 * (3 * en + a)), m);
        st8(D + N1 + 8 * k, scale(c2{D[F + 2 * (3 * en + a)], D[F + 2 * (3 * en + a) + 1]}, f));
    }
#pragma unroll
    for (int r = 0; r < (LANES == 8 ? 2 : 1); ++r) {  // pair currents (pair, pols), current of the ends (spins)
        const int k = 8 * r + ln;
        if (LANES > 16 && k >= 16) break;
        if (k < 12) {
            const int p = k >> 2, a = p == 2, b = p == 0 ? 1 : 2;
            vec w{{0.0, 0.0, 0.0, 0.0}};
            sub_vvv(w, ld4(D + EPS + 8 * a + 4 * (k & 1)), ld4(D + Q + 4 * a), ld4(D + EPS + 8 * b + 2 * (k & 2)),
                    ld4(D + Q + 4 * b));
            st4(D + W2 + 4 * k, mul(D[IQ + p], w));
        } else {
            st8(D + C0 + 8 * (k - 12),
                scale(c2{D[IQ + 4], 0.0}, current(ld8(D + N0 + 8 * (k & 1)), ld8(D + N0 + 16 + 4 * (k & 2)))));
        }
    }
    __syncthreads();

    // ---- this lane's polarisations ----
    const int b0 = bit(l, 0), b1 = bit(l, 1), b2 = bit(l, 2);
    const int pol[3] = {b0, b1, b2};
    const vec W[3] = {ld4(D + W2 + 4 * (b0 + 2 * b1)), ld4(D + W2 + 16 + 4 * (b0 + 2 * b2)),
                      ld4(D + W2 + 32 + 4 * (b1 + 2 * b2))};
    vec eps[3];
    each<3>([&](auto A) __attribute__((always_inline)) { eps[A] = ld4(D + EPS + 8 * A + 4 * pol[A]); });
    vec W3[2];  // middle 0: (1, 0, 2); middle 1: (0, 1, 2); without their propagator
    vec X3[3];  // the trees that join a pair and the third gluon
    if constexpr (MC) {
        each<3>([&](auto K) __attribute__((always_inline)) {
            constexpr int c = 2 - K, a = c == 0 ? 1 : 0, b = c == 2 ? 1 : 2;
            X3[K] = vec{{0.0, 0.0, 0.0, 0.0}};
            sub_vvv(X3[K], W[K], add(ld4(D + Q + 4 * a), ld4(D + Q + 4 * b)), eps[c], ld4(D + Q + 4 * c));
        });
    }
    {
        const vec q0 = ld4(D + Q), q1 = ld4(D + Q + 4), q2 = ld4(D + Q + 8), q01 = add(q0, q1);
        vec a{{0.0, 0.0, 0.0, 0.0}}, b{{0.0, 0.0, 0.0, 0.0}};
        sub_vvv(a, W[0], q01, eps[2], q2);
        sub_vvv(b, mul(-1.0, W[0]), q01, eps[2], q2);
        sub_vvv(a, eps[0], q0, W[2], add(q1, q2));
        sub_vvv(b, eps[1], q1, W[1], add(q0, q2));
        add_vvvv(a, eps[0], eps[1], eps[2]);
        add_vvvv(b, eps[1], eps[0], eps[2]);
        W3[1] = a;
        W3[0] = b;
    }
    // With the weights also in registers these are read again where they are used.
    auto pair = [&](auto K, int at) __attribute__((always_inline)) {
        constexpr int a = K == 2, b = K == 0 ? 1 : 2;
        return MC ? ld4(D + W2 + 16 * K + 4 * (bit(at, a) + 2 * bit(at, b))) : W[K];
    };
    double acc = 0.0;
    const int pair_first = LANES == 8 ? 0 : ln >> 3;  // spin pair s3 + 2 s4: all in turn, or this lane's
#pragma unroll 1
    for (int s4 = pair_first >> 1; s4 < (LANES == 8 ? 2 : (pair_first >> 1) + 1); ++s4) {
        int l4 = l;
        asm volatile("" : "+v"(l4));
        // rows from p4: R(c), and W(b) R(c) + W(bc) v as r(c) slash(b) + r0 slash W(bc)
        const row r0 = ld8(D + N0 + 16 + 8 * s4);
        row r1[3], r2[3][2], rw[3];
        each<3>([&](auto C) __attribute__((always_inline)) {
            r1[C] = ld8(D + N1 + 96 + 32 * C + 16 * pol[C] + 8 * s4);
            if constexpr (!MC) rw[C] = slash(r0, W[C]);
        });
        each<3>([&](auto C) __attribute__((always_inline)) {
            each<2>([&](auto H) __attribute__((always_inline)) {  // b: the H-th gluon other than C
                constexpr int b = H < C ? H : H + 1, p = b + C - 1;
                const row t = slash(r1[C], ld4(D + EPS + 8 * b + 4 * bit(l4, b)));
                const double sg = b < C ? 1.0 : -1.0;
                if constexpr (MC)
                    r2[C][H] = t;
                else
                    r2[C][H] = row{{axpy(sg, rw[p].s[0], t.s[0]), axpy(sg, rw[p].s[1], t.s[1]),
                                    axpy(sg, rw[p].s[2], t.s[2]), axpy(sg, rw[p].s[3], t.s[3])}};
            });
        });
#pragma unroll 1
        for (int s3 = pair_first & 1; s3 < (LANES == 8 ? 2 : (pair_first & 1) + 1); ++s3) {
            int l3 = l;
            if constexpr (MC) asm volatile("" : "+v"(l3));
            const row f0 = ld8(D + N0 + 8 * s3), V = ld8(D + C0 + 8 * (s3 + 2 * s4));
            c2 J[6];
            {
                const c2 t0 = cdot(V, W3[0]), t1 = cdot(V, W3[1]), t2 = -(t0 + t1);
                J[0] = t1, J[5] = t1;  // 012, 210
                J[1] = t2, J[3] = t2;  // 021, 120
                J[2] = t0, J[4] = t0;  // 102, 201
            }
            if constexpr (MC) each<3>([&](auto K) __attribute__((always_inline)) { found(IDS::tree[K], cdot(V, X3[K])); });
            each<3>([&](auto C) __attribute__((always_inline)) {  // ubar W(ab) R(c)
                constexpr int a = C == 0 ? 1 : 0, b = C == 2 ? 1 : 2, p = a + b - 1;
                const c2 t = wedge(slash(f0, pair(std::integral_constant<int, p>{}, l3)), r1[C], c2{0.0, 0.0});
                if constexpr (MC) found(IDS::last[p], t);
                constexpr int kab = 2 * a + (b > C), kba = 2 * b + (a > C);
                J[kab] += t;
                J[kba] -= t;
            });
            each<3>([&](auto A) __attribute__((always_inline)) {  // L(a) [...]
                const row f = ld8(D + N1 + 32 * A + 16 * pol[A] + 8 * s3);
                each<2>([&](auto H) __attribute__((always_inline)) {  // c: the H-th gluon other than a
                    constexpr int c = H < A ? H : H + 1, b = 3 - A - c, k = 2 * A + (b > c);
                    if constexpr (MC) {
                        const c2 t = wedge(f, r2[c][b < c ? b : b - 1], c2{0.0, 0.0});
                        found(IDS::order[k], t);
                        J[k] += t;
                    } else {
                        J[k] = wedge(f, r2[c][b < c ? b : b - 1], J[k]);
                    }
                });
                if constexpr (MC) {  // and the pair of the others
                    constexpr int p = 2 - A;
                    const c2 t = cdot(current(f, r0), pair(std::integral_constant<int, p>{}, l3));
                    found(IDS::first[p], t);
                    J[2 * A] -= t;  // a row takes the vertex with the other sign
                    J[2 * A + 1] += t;
                    settle(J);
                }
            });
            const double q = P::colour_blocks(J);
            acc += ((spins >> (s3 + 2 * s4)) & 1) ? q : 0.0;
        }
    }
    if constexpr (LANES == 32) {
        const double part = acc;
        acc = 0.0;
        each<4>([&](auto S) __attribute__((always_inline)) { acc += __shfl(part, l + 8 * S, 32); });
    }
    const double tot = group_sum(acc, 3);
    if (valid && ln == 0) out[ev] = tot * (1.0 / (256.0 * P::identical * P::lcd));
    if constexpr (MC) {
        num = group_sum(num, 3);
        den = group_sum(den, 3);
        if (valid && l == 0) alpha[ev] = num / den;
    }
}

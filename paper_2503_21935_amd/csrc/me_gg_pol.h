// me_gg_pol.h -- g g -> t tbar and g g -> t tbar g summed over spins with real
// polarisation vectors.  Rules, signs and the row form of columns as in
// me_wave.h.
//
// Two gluons: one event per lane, everything in registers.  All sixteen
// configurations share four one-gluon rows per ordering and end.
//   J_ab = L(a) W(b) v + ubar W(ab) v.
// Three gluons: eight lanes per event, lane l the gluon polarisations l; the
// externals, one-gluon rows, pair currents and the current of the line's ends
// are computed once per event and shared in LDS, the rest by each lane for its
// polarisations and the four spin pairs.
//   J_abc = L(a) [W(b) R(c) + W(bc) v] + ubar W(ab) R(c) + ubar W(abc) v.
//
// Both are bound by VALU issue (2,600 vector instructions per wave of 64 events
// and of eight events).  Against one helicity per pass over the diagram program
// (k_me_gg): 2^20 events of g g -> t tbar take 127 us against 521 us, 2^18
// events of g g -> t tbar g 0.30 ms against 2.7 ms.
#pragma once
#include "me_qew_pol.h"

// idx, count and spins as for k_me_gg4_wave.
template <class P>
__global__ __launch_bounds__(64, 2) void k_me_gg2_pol(const double* __restrict__ mom, int64_t nevt,
                                                      double* __restrict__ out, unsigned spins, me_params prm,
                                                      const int* __restrict__ idx, const int* __restrict__ count) {
    using namespace wv;
    static_assert(P::ngluon == 2 && P::ncol == 2, "two gluons");
    int64_t ev = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (count) {
        if (ev >= *count) return;
        ev = idx[ev];
    } else if (ev >= nevt) {
        return;
    }
    const double m = prm.mt;
    vec q[2], p3, p4;
    {
        const double* pe = mom + ev * 16;
        auto ld = [&](int k) __attribute__((always_inline)) {
            return vec{{pe[4 * k], pe[4 * k + 1], pe[4 * k + 2], pe[4 * k + 3]}};
        };
        q[0] = ld(0), q[1] = ld(1), p3 = ld(2), p4 = ld(3);
    }
    row n3[2], n4[2];  // end rows by spin
    each<2>([&](auto S) __attribute__((always_inline)) {
        n3[S] = end_row(p3, m, 0, S ? 1 : -1);
        n4[S] = end_row(p4, m, 1, S ? 1 : -1);
    });
    vec e[2][2];
    each<4>([&](auto K) __attribute__((always_inline)) {
        e[K / 2][K % 2] = mul(prm.gs, polarisation(q[K / 2], K % 2));
    });
    auto line = [&](auto A) __attribute__((always_inline)) {  // L(a) up to the sign, by polarisation and spin
        const vec K = add(p3, mul(-1.0, q[A]));
        const c2 f = crecip(K.v[0] * K.v[0] - K.v[1] * K.v[1] - K.v[2] * K.v[2] - K.v[3] * K.v[3] - m * m, m * prm.wt);
        return [=, &n3, &e](auto PS) __attribute__((always_inline)) {
            return scale(f, slash_m(slash(n3[PS / 2], e[A][PS % 2]), K, m));
        };
    };
    // J_01 without the tree: [L of gluon 0 (pol, spin of t)][gluon 1's pol, spin of tbar]
    c2 J[4][4];
    {
        const auto L = line(std::integral_constant<int, 0>{});
        row x[4];
        each<4>([&](auto K) __attribute__((always_inline)) { x[K] = slash(n4[K / 2], e[1][K % 2]); });
        each<4>([&](auto A) __attribute__((always_inline)) {
            const row l = L(A);
            each<4>([&](auto B) __attribute__((always_inline)) { J[A][B] = wedge(l, x[B], c2{0.0, 0.0}); });
            settle(J[A]);
        });
    }
    double acc = 0.0;
    const vec Q = add(q[0], q[1]);
    const double iq = 1.0 / (Q.v[0] * Q.v[0] - Q.v[1] * Q.v[1] - Q.v[2] * Q.v[2] - Q.v[3] * Q.v[3]);
    const auto L = line(std::integral_constant<int, 1>{});
    vec w[4];  // W(01) by polarisations
    each<4>([&](auto K) __attribute__((always_inline)) {
        vec t{{0.0, 0.0, 0.0, 0.0}};
        sub_vvv(t, e[0][K % 2], q[0], e[1][K / 2], q[1]);
        w[K] = mul(iq, t);
    });
    row x[4];
    each<4>([&](auto K) __attribute__((always_inline)) { x[K] = slash(n4[K / 2], e[0][K % 2]); });
    each<2>([&](auto S3) __attribute__((always_inline)) {
        const row l[2] = {L(std::integral_constant<int, 2 * S3>{}), L(std::integral_constant<int, 2 * S3 + 1>{})};
        each<2>([&](auto S4) __attribute__((always_inline)) {
            const row V = current(n3[S3], n4[S4]);
            double part = 0.0;
            each<4>([&](auto PP) __attribute__((always_inline)) {
                constexpr int P0 = PP % 2, P1 = PP / 2;
                const c2 t = cdot(V, w[PP]);
                c2 f[2] = {J[P0 + 2 * S3][P1 + 2 * S4] + t, wedge(l[P1], x[P0 + 2 * S4], -t)};
                part += P::colour_blocks(f);
            });
            acc += ((spins >> (S3 + 2 * S4)) & 1) ? part : 0.0;
        });
    });
    out[ev] = acc * (1.0 / (256.0 * P::identical * P::lcd));
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

template <class P>
__global__ __launch_bounds__(64, 2) void k_me_gg3_pol(const double* __restrict__ mom, int64_t nevt,
                                                      double* __restrict__ out, unsigned spins, me_params prm,
                                                      const int* __restrict__ idx, const int* __restrict__ count) {
    using namespace g3;
    static_assert(P::ngluon == 3 && P::ncol == 6, "three gluons");
    __shared__ double2 mem[8 * (STRIDE / 2)];
    const int lane = threadIdx.x, l = lane & 7, e = lane >> 3;
    const double m = prm.mt;
    const int64_t n = count ? (int64_t)*count : nevt;
    const int64_t first = (int64_t)blockIdx.x * 8;
    if (first >= n) return;
    int64_t i = first + e;
    const bool valid = i < n;
    if (!valid) i = n - 1;
    const int64_t ev = count ? (int64_t)idx[i] : i;
    double* const D = reinterpret_cast<double*>(mem) + e * STRIDE;
    if (l < 5) {  // slots: gluons 0, 1, 2 (particle 4), p3, p4
        const double* p = mom + ev * 20 + 4 * (l < 2 ? l : l == 2 ? 4 : l - 1);
        const double sg = l == 2 ? -1.0 : 1.0;
        st4(D + Q + 4 * l, vec{{sg * p[0], sg * p[1], sg * p[2], sg * p[3]}});
    }
    __syncthreads();
    for (int k = l; k < 11; k += 8) {  // summed momenta and propagators
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
    if (l < 6) {  // polarisation vectors (gluon, which)
        const vec q = ld4(D + Q + 4 * (l >> 1));
        st4(D + EPS + 4 * l, mul(prm.gs, polarisation(l < 4 ? q : mul(-1.0, q), l & 1)));
    }
    if (l < 4)  // end rows (end, spin)
        st8(D + N0 + 8 * l, end_row(ld4(D + Q + 12 + 4 * (l >> 1)), m, l >> 1, (l & 1) ? 1 : -1));
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 3; ++r) {  // one-gluon rows (end, gluon, pol, spin); L(a) up to the sign
        const int k = 8 * r + l, en = k >= 12, a = (k >> 2) - 3 * en, pol = (k >> 1) & 1, s = k & 1;
        const row f = slash_m(slash(ld8(D + N0 + 16 * en + 8 * s), ld4(D + EPS + 8 * a + 4 * pol)),
                              ld4(D + K + 4 * (3 * en + a)), m);
        st8(D + N1 + 8 * k, scale(c2{D[F + 2 * (3 * en + a)], D[F + 2 * (3 * en + a) + 1]}, f));
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) {  // pair currents (pair, pols), current of the ends (spins)
        const int k = 8 * r + l;
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
    double acc = 0.0;
#pragma unroll 1
    for (int s4 = 0; s4 < 2; ++s4) {
        // rows from p4: R(c), and W(b) R(c) + W(bc) v as r(c) slash(b) + r0 slash W(bc)
        const row r0 = ld8(D + N0 + 16 + 8 * s4);
        row r1[3], r2[3][2], rw[3];
        each<3>([&](auto C) __attribute__((always_inline)) {
            r1[C] = ld8(D + N1 + 96 + 32 * C + 16 * pol[C] + 8 * s4);
            rw[C] = slash(r0, W[C]);
        });
        each<3>([&](auto C) __attribute__((always_inline)) {
            each<2>([&](auto H) __attribute__((always_inline)) {  // b: the H-th gluon other than C
                constexpr int b = H < C ? H : H + 1, p = b + C - 1;
                const row t = slash(r1[C], eps[b]);
                const double sg = b < C ? 1.0 : -1.0;
                r2[C][H] = row{{axpy(sg, rw[p].s[0], t.s[0]), axpy(sg, rw[p].s[1], t.s[1]),
                                axpy(sg, rw[p].s[2], t.s[2]), axpy(sg, rw[p].s[3], t.s[3])}};
            });
        });
#pragma unroll 1
        for (int s3 = 0; s3 < 2; ++s3) {
            const row f0 = ld8(D + N0 + 8 * s3), V = ld8(D + C0 + 8 * (s3 + 2 * s4));
            c2 J[6];
            {
                const c2 t0 = cdot(V, W3[0]), t1 = cdot(V, W3[1]), t2 = -(t0 + t1);
                J[0] = t1, J[5] = t1;  // 012, 210
                J[1] = t2, J[3] = t2;  // 021, 120
                J[2] = t0, J[4] = t0;  // 102, 201
            }
            each<3>([&](auto C) __attribute__((always_inline)) {  // ubar W(ab) R(c)
                constexpr int a = C == 0 ? 1 : 0, b = C == 2 ? 1 : 2, p = a + b - 1;
                const c2 t = wedge(slash(f0, W[p]), r1[C], c2{0.0, 0.0});
                constexpr int kab = 2 * a + (b > C), kba = 2 * b + (a > C);
                J[kab] += t;
                J[kba] -= t;
            });
            each<3>([&](auto A) __attribute__((always_inline)) {  // L(a) [...]
                const row f = ld8(D + N1 + 32 * A + 16 * pol[A] + 8 * s3);
                each<2>([&](auto H) __attribute__((always_inline)) {  // c: the H-th gluon other than a
                    constexpr int c = H < A ? H : H + 1, b = 3 - A - c, k = 2 * A + (b > c);
                    J[k] = wedge(f, r2[c][b < c ? b : b - 1], J[k]);
                });
            });
            const double q = P::colour_blocks(J);
            acc += ((spins >> (s3 + 2 * s4)) & 1) ? q : 0.0;
        }
    }
    const double tot = group_sum(acc, 3);
    if (valid && l == 0) out[ev] = tot * (1.0 / (256.0 * P::identical * P::lcd));
}

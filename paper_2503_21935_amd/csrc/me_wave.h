// me_wave.h -- one event per wave: g g -> t tbar g g summed over spins with
// real polarisation vectors and wavefunctions shared across the wave.
//
// The helicity sum of |M|^2 does not depend on the basis of the gluons'
// polarisation space, so the kernel sums over the two real transverse vectors
// e1, e2 of each gluon (those of which the helicity vectors are made, in the
// same frame) instead of the circular ones.  With them every gluon current is a
// real vector, and with the colour-ordered rules (Berends, Giele 1988) the
// couplings and propagator phases drop out of it:
//   W(A) = g e_A,
//   W(S) = (1/Q_S^2) [ - sum vvv(W(S'), W(S'')) + sum vvvv(W(S'), W(S''), W(S''')) ],
//   vvvv(X, Y, Z) = 2 (X.Z) Y - (Y.Z) X - (X.Y) Z,
// with W reflection-symmetric up to a sign and subject to the shuffle
// identities, so that 6, 8 and 6 currents of two, three and four gluons suffice.
//
// The top line is cut after two gluons.  With L(a..) the row from ubar(p3) and
// R(..d) the column from v(p4), each with its propagators,
//   J_abcd = L(ab) [W(c) R(d) + W(cd) v] + L(a) W(bc) R(d)
//          + L(a) W(bcd) v + ubar W(abc) R(d) + ubar W(abcd) v
// (up to a phase common to all orderings).  Every factor depends on the
// polarisations and spins of its own gluons and line end only: a wave
// computes each of them once, the lanes taking different nodes of one kind
// (192 of the two-gluon rows, say), and keeps them in LDS; then lane l sums J
// over the products for configuration l (bits 0..3 the polarisations, 4 and 5
// the spins of t and tbar) and takes the colour sum.  Against one helicity per
// lane with every wavefunction computed per helicity (k_me_gg) this is about a
// sixth of the arithmetic: 2^18 events take 1.59 ms against 11.3 ms, 48 events
// (one wave's time) 12 us against 45 us.  Bound by VALU issue: 2,690 vector
// instructions per event and wave, the VALU active 76 % of the time with two
// waves per SIMD (LDS capacity and registers allow no third).
//
// Columns are held as rows: with B = diag(eps, -eps) one has
// B gamma^mu B^-1 = -gamma^mu^T, so r = (R1, -R0, -R3, R2) turns (W R) into
// -(r W) and (Pslash + m) R into r (-Pslash + m), and both line ends run the
// same code; f R = f1 r0 - f0 r1 + f2 r3 - f3 r2.
#pragma once
#include <type_traits>

#include "me_kernels.h"

namespace wv {

typedef cx<double> c2;

struct vec {  // real 4-vector, contravariant
    double v[4];
};
struct row {
    c2 s[4];
};

MEV double mdot(const vec& a, const vec& b) {
    return fma(a.v[0], b.v[0], -fma(a.v[1], b.v[1], fma(a.v[2], b.v[2], a.v[3] * b.v[3])));
}
MEV vec add(const vec& a, const vec& b) { return {{a.v[0] + b.v[0], a.v[1] + b.v[1], a.v[2] + b.v[2], a.v[3] + b.v[3]}}; }
MEV vec mul(double s, const vec& a) { return {{s * a.v[0], s * a.v[1], s * a.v[2], s * a.v[3]}}; }

// acc - V(X, QX, Y, QY): (X.Y)(QX - QY) + Y ((QX + 2 QY).X) - X ((2 QX + QY).Y)
MEV void sub_vvv(vec& acc, const vec& X, const vec& QX, const vec& Y, const vec& QY) {
    vec a, b, d;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        a.v[k] = fma(2.0, QY.v[k], QX.v[k]);
        b.v[k] = fma(2.0, QX.v[k], QY.v[k]);
        d.v[k] = QX.v[k] - QY.v[k];
    }
    const double xy = -mdot(X, Y), ax = -mdot(a, X), by = mdot(b, Y);
#pragma unroll
    for (int k = 0; k < 4; ++k) acc.v[k] = fma(Y.v[k], ax, fma(d.v[k], xy, fma(X.v[k], by, acc.v[k])));
}
// acc + 2 (X.Z) Y - (Y.Z) X - (X.Y) Z
MEV void add_vvvv(vec& acc, const vec& X, const vec& Y, const vec& Z) {
    const double xz = 2.0 * mdot(X, Z), yz = -mdot(Y, Z), xy = -mdot(X, Y);
#pragma unroll
    for (int k = 0; k < 4; ++k) acc.v[k] = fma(xz, Y.v[k], fma(yz, X.v[k], fma(xy, Z.v[k], acc.v[k])));
}

MEV c2 rmul(double s, c2 a) { return {s * a.r, s * a.i}; }

// o + f (gamma.W), real W
MEV row add_slash(const row& o, const row& f, const vec& W) {
    const double a = W.v[0] + W.v[3], b = W.v[0] - W.v[3];
    const c2 c{W.v[1], W.v[2]}, d{W.v[1], -W.v[2]};
    return {{axpy(a, f.s[2], cfma(f.s[3], c, o.s[0])), axpy(b, f.s[3], cfma(f.s[2], d, o.s[1])),
             axpy(b, f.s[0], cfma(f.s[1], -c, o.s[2])), axpy(a, f.s[1], cfma(f.s[0], -d, o.s[3]))}};
}
// f (gamma.W), real W
MEV row slash(const row& f, const vec& W) {
    const double a = W.v[0] + W.v[3], b = W.v[0] - W.v[3];
    const c2 c{W.v[1], W.v[2]}, d{W.v[1], -W.v[2]};
    return {{axpy(a, f.s[2], f.s[3] * c), axpy(b, f.s[3], f.s[2] * d), axpy(b, f.s[0], f.s[1] * -c),
             axpy(a, f.s[1], f.s[0] * -d)}};
}
MEV row scale(c2 s, const row& f) { return {{s * f.s[0], s * f.s[1], s * f.s[2], s * f.s[3]}}; }
// f (gamma.P + m)
MEV row slash_m(const row& f, const vec& P, double m) {
    return add_slash(row{{rmul(m, f.s[0]), rmul(m, f.s[1]), rmul(m, f.s[2]), rmul(m, f.s[3])}}, f, P);
}
// f R with R held as the row r
MEV c2 wedge(const row& f, const row& r, c2 acc) {
    acc = cfma(f.s[1], r.s[0], acc);
    acc = cfma(-f.s[0], r.s[1], acc);
    acc = cfma(f.s[2], r.s[3], acc);
    return cfma(-f.s[3], r.s[2], acc);
}
// f gamma_mu R (covariant index), R held as the row r
MEV row current(const row& f, const row& r) {
    const c2 a = f.s[0] * r.s[3], b = f.s[1] * r.s[2], c = f.s[0] * r.s[2], d = f.s[1] * r.s[3];
    const c2 e = f.s[2] * r.s[1], g = f.s[3] * r.s[0], h = f.s[2] * r.s[0], k = f.s[3] * r.s[1];
    return {{(a - b) + (g - e), (c - d) + (h - k), times_mi((d + c) + (h + k)), -((b + a) + (e + g))}};
}
// acc + sum over mu of V_mu W^mu
MEV c2 cdot_acc(const row& V, const vec& W, c2 acc) {
    acc = axpy(W.v[0], V.s[0], acc);
    acc = axpy(W.v[1], V.s[1], acc);
    acc = axpy(W.v[2], V.s[2], acc);
    return axpy(W.v[3], V.s[3], acc);
}
MEV c2 cdot(const row& V, const vec& W) {
    c2 r = rmul(W.v[0], V.s[0]);
    r = axpy(W.v[1], V.s[1], r);
    r = axpy(W.v[2], V.s[2], r);
    return axpy(W.v[3], V.s[3], r);
}

// Real transverse vectors of a gluon of momentum k (those that gluon_eps
// combines): e1 = (cos th cos ph, cos th sin ph, -sin th), e2 = (-sin ph, cos ph, 0);
// along the z axis the azimuth is taken as 0.
MEV vec polarisation(const vec& k, bool e2) {
    const double kx = k.v[1], ky = k.v[2], kz = k.v[3];
    const double kt2 = kx * kx + ky * ky, kk = sqrt(kt2 + kz * kz), kt = sqrt(kt2);
    const bool axis = !(kt > 0.0);
    const double ikt = 1.0 / kt, ikk = 1.0 / kk, c = kz * ikk;
    vec e;
    e.v[0] = 0.0;
    e.v[1] = axis ? (e2 ? 0.0 : (kz >= 0.0) ? 1.0 : -1.0) : e2 ? -ky * ikt : c * kx * ikt;
    e.v[2] = axis ? (e2 ? 1.0 : 0.0) : e2 ? kx * ikt : c * ky * ikt;
    e.v[3] = (axis || e2) ? 0.0 : -kt * ikk;
    return e;
}
// ubar(p3) (e = 0) and v(p4) as a row (e = 1) at helicity lam.
MEV row end_row(const vec& q, double m, int e, int lam) {
    const mom4<double> p{q.v[0], q.v[1], q.v[2], q.v[3]};
    double pabs, wm, wp;
    spinor_weights(p, m, pabs, wm, wp);
    c2 h0, h1;
    helicity_chi(p, pabs, e ? -lam : lam, h0, h1);
    // ubar = (conj of the right, conj of the left half); v as the row (v1, -v0, -v3, v2)
    const double a = ((lam > 0) != (e == 1)) ? wm : wp;
    const double b = e ? ((lam > 0) ? wm : wp) : ((lam > 0) ? wp : wm);
    return e ? row{{rmul(a, h1), rmul(-a, h0), rmul(b, h1), rmul(-b, h0)}}
             : row{{conj(rmul(b, h0)), conj(rmul(b, h1)), conj(rmul(a, h0)), conj(rmul(a, h1))}};
}

// f(0), f(1), ... f(N - 1) with constant arguments, so that registers can be indexed.
template <int N, int K = 0, class F>
MEV void each(F&& f) {
    if constexpr (K < N) {
        f(std::integral_constant<int, K>{});
        each<N, K + 1>(f);
    }
}

// Sum over the 64 lanes, valid in lane 63 (a fixed tree).
template <int CTRL, int ROWMASK>
MEV double dpp_add(double v) {
    const long long x = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWMASK, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(x >> 32), CTRL, ROWMASK, 0xf, false);
    return v + __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
MEV double wave_sum(double v) {
    v = dpp_add<0xB1, 0xf>(v);   // quad_perm [1,0,3,2]
    v = dpp_add<0x4E, 0xf>(v);   // quad_perm [2,3,0,1]
    v = dpp_add<0x141, 0xf>(v);  // row_half_mirror
    v = dpp_add<0x140, 0xf>(v);  // row_mirror
    v = dpp_add<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
    return dpp_add<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
}

// --------------------------------------------------------------------------
// Index tables (four gluons)
// --------------------------------------------------------------------------
__host__ __device__ constexpr int pair_of(int a, int b) {
    const int lo = a < b ? a : b, hi = a < b ? b : a;
    return lo * (7 - lo) / 2 + hi - lo - 1;
}
__host__ __device__ constexpr int pair_lo(int p) { return p < 3 ? 0 : p < 5 ? 1 : 2; }
__host__ __device__ constexpr int pair_hi(int p) { return p < 3 ? p + 1 : p < 5 ? p - 1 : 3; }
// k-th gluon other than m
__host__ __device__ constexpr int other(int m, int k) { return k < m ? k : k + 1; }
// position of gluon x among those other than m
__host__ __device__ constexpr int rank_without(int m, int x) { return x < m ? x : x - 1; }
// lexicographic index of the ordering (a, b, c, d)
__host__ __device__ constexpr int flow(int a, int b, int c, int d) {
    const int ib = b - (b > a), ic = c - (c > a) - (c > b);
    return 6 * a + 2 * ib + ic;
}

// index of the ordering (0, b, c, rest) among those that start with gluon 0
__host__ __device__ constexpr int tree(int b, int c) { return 2 * (b - 1) + (c > b ? c - 2 : c - 1); }

// LDS of one wave, in double2 units.  The first block belongs to one event
// and is filled for two at a time (a second copy at S_B), since its phases have
// work for 32 lanes at most per event; what follows is used by one event
// after the other.  20,384 bytes: eight waves per CU.
enum {
    S_Q = 0,               // gluon momenta, incoming flow [gluon][2]
    S_K = S_Q + 8,         // top-line momenta [14][2]: entries 10..23 of k_of
    S_F = S_K + 28,        // propagators [25], numbered as k_of
    S_EPS = S_F + 25,      // g e [gluon][2][pol 2]
    S_N0 = S_EPS + 16,     // end rows [end][component][spin]
    S_C0 = S_N0 + 16,      // current of the ends [mu][spins 4], with the gluon propagator
    S_N1 = S_C0 + 16,      // one-gluon rows [end][gluon][component][pol, spin: 4]
    S_W2 = S_N1 + 128,     // pair currents [pair][2][pols 4]
    S_W3 = S_W2 + 48,      // triple currents [missing gluon][middle 3][2][pols 8]
    S_T = S_W3 + 192,      // stage, one of the following at a time
    S_P = S_T,             // (setup) momenta of both events [event][slot 6][2]
    S_C1 = S_T,            // line currents [end][gluon][mu][pol, spins: 8]
    S_W4 = S_C1 + 256,     // four-gluon currents [order of gluons 1..3: 6][2][pols 16]
    S_N2 = S_T,            // two-gluon rows [split 4][end][order][component][pols, spin: 8]
    S_C2 = S_T,            // line currents [pair 4][order][mu][pols 4, spins 4]
    S_C2B = S_T + 256,     // those of pairs 4 and 5, beside the rows of splits 4 and 5
    S_B = S_T + 512,       // the second event's copy of S_Q .. S_W2
    S_SMALL = S_W3,        // its size
    S_END = S_B + S_SMALL
};

// Entries of S_K / S_F: 0..5 pairs, 6..9 triples (by missing gluon), 10..13
// p3 - q_a, 14..19 the top line after a pair, 20..23 p4 - q_d, 24 p3 + p4.
// Coefficients of (q0, q1, q2, q3, p3, p4): two bits each, 1 plus, 2 minus.
// The line after pair S is p3 - Q_S or Q_rest - p4, whichever has fewer of
// the two beam momenta (which rounds less).
MEV unsigned k_of(int i) {
    unsigned c = 0;
    if (i < 6) {
        c = (1u << 2 * pair_lo(i)) | (1u << 2 * pair_hi(i));
    } else if (i < 10) {
        c = 0x55u & ~(3u << 2 * (i - 6));
    } else if (i < 14) {
        c = (2u << 2 * (i - 10)) | (1u << 8);
    } else if (i < 20) {
        const int p = i - 14;
        const unsigned s = (1u << 2 * pair_lo(p)) | (1u << 2 * pair_hi(p));
        c = (p == 0) ? ((0x55u & ~s) | (2u << 10)) : ((s << 1) | (1u << 8));
    } else if (i < 24) {
        c = (2u << 2 * (i - 20)) | (1u << 10);
    } else {
        c = (1u << 8) | (1u << 10);
    }
    return c;
}

// Accesses at byte offset `at`; components `stride` double2 apart.
MEV const double2* lds_at(const double2* T, int at) {
    return reinterpret_cast<const double2*>(reinterpret_cast<const char*>(T) + at);
}
MEV double2* lds_at(double2* T, int at) { return reinterpret_cast<double2*>(reinterpret_cast<char*>(T) + at); }
MEV vec ld_vec(const double2* T, int at, int stride) {
    const double2 *p = lds_at(T, at), a = p[0], b = p[stride];
    return {{a.x, a.y, b.x, b.y}};
}
MEV void st_vec(double2* T, int at, int stride, const vec& w) {
    double2* p = lds_at(T, at);
    p[0] = double2{w.v[0], w.v[1]};
    p[stride] = double2{w.v[2], w.v[3]};
}
MEV row ld_row(const double2* T, int at, int stride) {
    const double2* p = lds_at(T, at);
    const double2 a = p[0], b = p[stride], c = p[2 * stride], d = p[3 * stride];
    return {{{a.x, a.y}, {b.x, b.y}, {c.x, c.y}, {d.x, d.y}}};
}
MEV void st_row(double2* T, int at, int stride, const row& f) {
    double2* p = lds_at(T, at);
#pragma unroll
    for (int k = 0; k < 4; ++k) p[k * stride] = double2{f.s[k].r, f.s[k].i};
}

MEV int bit(int x, int k) { return (x >> k) & 1; }

// v with its sign flipped where the top bit of s is set
MEV double flip_sign(double v, int s) {
    const long long x = __double_as_longlong(v) ^ ((long long)(s & 0x80000000) << 32);
    return __longlong_as_double(x);
}
MEV vec flip_sign(const vec& w, int s) {
    return {{flip_sign(w.v[0], s), flip_sign(w.v[1], s), flip_sign(w.v[2], s), flip_sign(w.v[3], s)}};
}

// Two LDS byte offsets (below 2^15) in one register, the sign bit free.
MEV int pack(int lo, int hi) { return lo | (hi << 16); }
MEV int lo16(int p) { return p & 0xffff; }
MEV int hi16(int p) { return (p >> 16) & 0x7fff; }
// k-th byte
template <int K>
MEV int byte_of(int p) { return (p >> (8 * K)) & 0xff; }
// The packed offsets stay packed: what is taken out of them in one pass over
// the events is not kept for the next.
template <int N>
MEV void keep(int (&p)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+v"(p[i]));
}

// Sums so far are formed here: without it the products of one stage are put off
// until the end, with all their operands held.
template <int N>
MEV void settle(c2 (&J)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+v"(J[i].r), "+v"(J[i].i));
}

// Byte offset of the pair current of a and b at polarisations pa, pb (sorted
// pair), with the sign bit set if W(a, b) is minus that.
MEV int w2_at(int a, int b, int pa, int pb) {
    const int lo = a < b ? pa : pb, hi = a < b ? pb : pa;
    return 16 * (S_W2 + 8 * pair_of(a, b) + lo + 2 * hi);
}
MEV int minus(int a, int b) { return a > b ? (int)0x80000000 : 0; }
MEV int eps_at(int a, int pol) { return 16 * (S_EPS + 4 * a + pol); }
MEV int q_at(int a) { return 16 * (S_Q + 2 * a); }

// The blocks of one or two events (ne): lanes 0..31 the first, 32..63 the second
// (or the first again).
MEV void gg4_setup(double2* T, const double* __restrict__ mom, int64_t base, int ne, const int* __restrict__ idx,
                   const int* __restrict__ count, const me_params& prm, int lane) {
    constexpr int NP = 6;
    const double m = prm.mt;
    int ln = lane;
    asm volatile("" : "+v"(ln));  // addresses are formed here, not kept across the events
    const int j = ln >> 5, hl = ln & 31;
    const int64_t i = base + (j < ne ? j : 0);
    const int64_t ev = count ? (int64_t)idx[i] : i;
    const int B = 16 * (j ? (int)S_B : 0);  // this event's block
    // momenta: lane (slot, component); slots the gluons in incoming flow, p3, p4
    if (hl < 24) {
        const int slot = hl >> 2, part = slot < 2 ? slot : slot < 4 ? slot + 2 : slot - 2;
        const double v = mom[ev * (NP * 4) + 4 * part + (hl & 3)];
        const double q = (slot == 2 || slot == 3) ? -v : v;
        reinterpret_cast<double*>(T + S_P + 12 * j)[hl] = q;
        if (slot < 4) reinterpret_cast<double*>(lds_at(T, B + 16 * S_Q))[hl] = q;
    }
    __syncthreads();
    // summed momenta and propagators
    if (hl < 25) {
        const unsigned c = k_of(hl);
        vec K{{0.0, 0.0, 0.0, 0.0}};
#pragma unroll
        for (int s = 0; s < 6; ++s) {
            const double w = (double)((int)((c >> 2 * s) & 1) - (int)((c >> (2 * s + 1)) & 1));
            const vec q = ld_vec(T, 16 * (S_P + 12 * j + 2 * s), 1);
#pragma unroll
            for (int k = 0; k < 4; ++k) K.v[k] = fma(w, q.v[k], K.v[k]);
        }
        const bool top = hl >= 10 && hl < 24;
        const double d = K.v[0] * K.v[0] - K.v[1] * K.v[1] - K.v[2] * K.v[2] - K.v[3] * K.v[3];
        const c2 f = crecip(top ? d - m * m : d, top ? m * prm.wt : 0.0);
        if (top) st_vec(T, B + 16 * (S_K + 2 * (hl - 10)), 1, K);
        *lds_at(T, B + 16 * (S_F + hl)) = double2{f.r, f.i};
    }
    // polarisation vectors: lane (gluon, pol)
    if (hl < 8) {
        const int a = hl >> 1;
        const vec q = ld_vec(T, B + q_at(a), 1);
        st_vec(T, B + 16 * (S_EPS + 4 * a + (hl & 1)), 2,
               mul(prm.gs, polarisation(a < 2 ? q : mul(-1.0, q), hl & 1)));
    }
    // end rows: lane (end, spin)
    if (hl < 4) {
        const int e = hl >> 1;
        const row f = end_row(ld_vec(T, 16 * (S_P + 12 * j + 2 * (4 + e)), 1), m, e, (hl & 1) ? 1 : -1);
        st_row(T, B + 16 * (S_N0 + 8 * e + (hl & 1)), 2, f);
    }
    __syncthreads();
    // pair currents: lane (pair, pols); the other lanes: current of the ends (spins)
    if (hl < 24) {
        const int p = hl >> 2, a = pair_lo(p), b = pair_hi(p);
        vec w{{0.0, 0.0, 0.0, 0.0}};
        sub_vvv(w, ld_vec(T, B + eps_at(a, bit(hl, 0)), 2), ld_vec(T, B + q_at(a), 1),
                ld_vec(T, B + eps_at(b, bit(hl, 1)), 2), ld_vec(T, B + q_at(b), 1));
        st_vec(T, B + 16 * (S_W2 + 8 * p + (hl & 3)), 4, mul(lds_at(T, B + 16 * (S_F + p))->x, w));
    } else if (hl < 28) {
        const double iq = lds_at(T, B + 16 * (S_F + 24))->x;
        const row V = current(ld_row(T, B + 16 * (S_N0 + bit(hl, 0)), 2),
                              ld_row(T, B + 16 * (S_N0 + 8 + bit(hl, 1)), 2));
        st_row(T, B + 16 * (S_C0 + (hl & 3)), 4, scale(c2{iq, 0.0}, V));
    }
    // one-gluon rows: lane (end, gluon, pol, spin)
    {
        const int e = hl >> 4, a = (hl >> 2) & 3, k = 10 * e + a;
        const row f = slash_m(slash(ld_row(T, B + 16 * (S_N0 + 8 * e + bit(hl, 1)), 2),
                                    ld_vec(T, B + eps_at(a, bit(hl, 0)), 2)),
                              ld_vec(T, B + 16 * (S_K + 2 * k), 1), m);
        const double2 d = *lds_at(T, B + 16 * (S_F + 10 + k));
        st_row(T, B + 16 * (S_N1 + 16 * (4 * e + a) + (hl & 3)), 4, scale(e ? c2{d.x, d.y} : c2{-d.x, -d.y}, f));
    }
}

}  // namespace wv

// idx, count as for k_me_ee.  spins: bit s3 + 2 s4 set for the spin pairs of t
// and tbar that the helicity filter kept.  Blocks of one wave stride over the
// events, eb (1 or 2) at a time.  CM: colour sum on the matrix cores from J
// staged in LDS.
template <class P, bool CM>
__global__ __launch_bounds__(64, CM ? 1 : 2) void k_me_gg4_wave(const double* __restrict__ mom, int64_t nevt,
                                                               double* __restrict__ out, unsigned spins,
                                                               me_params prm, const int* __restrict__ idx,
                                                               const int* __restrict__ count, int eb) {
    using namespace wv;
    static_assert(P::ngluon == 4 && P::ncol == 24, "four gluons");
    __shared__ double2 T[S_END];
    const int lane = threadIdx.x;
    const int64_t n = count ? (int64_t)*count : nevt;
    const double m = prm.mt;

    // ---- where this lane's nodes and configuration read and write ----
    // triple currents: lane (missing gluon, which of two orderings, pols)
    int w3[5];
    {
        const int mg = lane >> 4, k = bit(lane, 3);
        const int lo = other(mg, 0), mi = other(mg, 1), hi = other(mg, 2);
        const int A = k ? mi : lo, B = k ? lo : mi, C = hi;
        const int pA = bit(lane, k), pB = bit(lane, 1 - k), pC = bit(lane, 2);
        w3[0] = pack(eps_at(A, pA), eps_at(B, pB));
        w3[1] = pack(eps_at(C, pC), q_at(A));
        w3[2] = pack(q_at(B), q_at(C));
        w3[3] = pack(16 * (S_F + 6 + mg), w2_at(A, B, pA, pB)) | minus(A, B);
        // stored as [middle 1] for (lo, mi, hi), [middle 0] for (mi, lo, hi)
        w3[4] = pack(16 * (S_W3 + 48 * mg + 16 * (1 - k) + (lane & 7)), w2_at(B, C, pB, pC)) | minus(B, C);
    }
    // four-gluon currents: node 64 pass + lane = (order of 1..3, pols)
    int w4[2][6];
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        const int node = (64 * pass + lane) % 96, o = node >> 4;
        const int B = 1 + (o >> 1), C = (o == 2 || o == 4) ? 1 : (o == 0 || o == 5) ? 2 : 3, D = 6 - B - C;
        const int pA = bit(node, 0), pB = bit(node, B), pC = bit(node, C), pD = bit(node, D);
        // polarisations of the gluons other than 0, and other than D, in label order
        const int i0 = (node >> 1) & 7, below = (1 << D) - 1;
        const int iD = (node & below) | (i0 & ~below);
        w4[pass][0] = pack(eps_at(B, pB), q_at(B));
        w4[pass][1] = pack(eps_at(C, pC), q_at(C));
        w4[pass][2] = pack(eps_at(D, pD), q_at(D));
        w4[pass][3] = pack(w2_at(0, B, pA, pB), w2_at(B, C, pB, pC)) | minus(B, C);
        w4[pass][4] = pack(16 * (S_W3 + 16 * (C - 1) + i0), w2_at(C, D, pC, pD)) | minus(C, D);
        w4[pass][5] = pack(16 * (S_W3 + 48 * D + 16 * rank_without(D, B) + iD), 16 * (S_W4 + 32 * o + (node & 15)));
    }
    // line currents with one gluon: lane (end, gluon, pol, spins)
    int c1[2];
    {
        const int e = lane >> 5, a = (lane >> 3) & 3, pol = bit(lane, 0), s3 = bit(lane, 1), s4 = bit(lane, 2);
        const int o1 = 16 * (S_N1 + 16 * (4 * e + a) + pol + 2 * (e ? s4 : s3));
        const int o0 = 16 * (e ? S_N0 + s3 : S_N0 + 8 + s4);
        c1[0] = e ? pack(o0, o1) : pack(o1, o0);
        c1[1] = 16 * (S_C1 + 32 * (4 * e + a) + (lane & 7));
    }
    // two-gluon rows.  Pass 0: rows from p3 of pairs 0..3; pass 1: rows from p4
    // of the complementary pairs 5..2; pass 2: both for pairs 4, 5 and 1, 0.
    // Lane (split, (end in pass 2), order, pols and spin); the rows from p3
    // get the propagator.
    int n2[3][3];
#pragma unroll
    for (int pass = 0; pass < 3; ++pass) {
        const int e = pass < 2 ? pass : bit(lane, 4), split = pass < 2 ? lane >> 4 : 4 + (lane >> 5);
        const int p = e ? 5 - split : split, lo = pair_lo(p), hi = pair_hi(p), flip = bit(lane, 3);
        const int x = flip ? hi : lo, y = flip ? lo : hi;
        const int px = bit(lane, flip), py = bit(lane, 1 - flip), sp = bit(lane, 2);
        n2[pass][0] = pack(16 * (S_N1 + 16 * (4 * e + x) + px + 2 * sp), eps_at(y, py));
        // the pair current enters as W(x, y) from p3 and W(y, x) from p4
        n2[pass][1] = pack(16 * (S_N0 + 8 * e + sp), 16 * (S_W2 + 8 * p + (lane & 3))) | ((flip ^ e) << 31);
        n2[pass][2] = pack(16 * (S_K + 2 * (4 + p)), 16 * (S_N2 + 128 * (split & 3) + 64 * e + 32 * flip + (lane & 7)));
    }
    // line currents with two gluons: pass 0, 1 pairs 0..3, pass 2 pairs 4, 5;
    // lane (pair, order, pols, spins)
    int k2[3];
#pragma unroll
    for (int pass = 0; pass < 3; ++pass) {
        const int op = 4 * pass + (lane >> 4), p = op >> 1, flip = op & 1;
        const int a = flip ? pair_hi(p) : pair_lo(p), d = flip ? pair_lo(p) : pair_hi(p);
        k2[pass] = pack(16 * (S_N1 + 16 * a + bit(lane, flip) + 2 * bit(lane, 2)),
                        16 * (S_N1 + 16 * (4 + d) + bit(lane, 1 - flip) + 2 * bit(lane, 3)));
    }
    // configuration `lane`: byte offsets inside the tables, four to a register
    const int s3 = bit(lane, 4), s4 = bit(lane, 5);
    int cfg[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int p = 0; p < 6; ++p) {
        const int pp = bit(lane, pair_lo(p)) + 2 * bit(lane, pair_hi(p));
        cfg[p] = 16 * ((pp + 4 * s3) | (pp + 4 * s4) << 8 | (pp + 4 * s3 + 8 * s4) << 16 | pp << 24);
    }
#pragma unroll
    for (int mg = 0; mg < 4; ++mg) {
        const int x = other(mg, 0), y = other(mg, 1), z = other(mg, 2);
        cfg[6] |= (16 * (bit(lane, x) + 2 * bit(lane, y) + 4 * bit(lane, z))) << (8 * mg);
        cfg[7] |= (16 * (bit(lane, mg) + 2 * s3 + 4 * s4)) << (8 * mg);
    }

    for (int64_t base = (int64_t)blockIdx.x * eb; base < n; base += (int64_t)gridDim.x * eb) {
        const int ne = (eb == 2 && base + 1 < n) ? 2 : 1;
        __syncthreads();  // the previous event's reads are done
        // Issue priority falls from the setup (long chains) over J (operands from LDS) to the colour sum
        // (registers only), so that of two waves on a SIMD the one that has to wait most asks first:
        // 2^20 events 6.46 -> 6.35 ms, 2^14 108 -> 105.6 us.  Raised for the setup alone: 6.45 ms.
        __builtin_amdgcn_s_setprio(2);
        gg4_setup(T, mom, base, ne, idx, count, prm, lane);
#pragma unroll 1
        for (int j = 0; j < ne; ++j) {
            int ln = lane;
            asm volatile("" : "+v"(ln));
            keep(w3), keep(w4[0]), keep(w4[1]), keep(c1), keep(n2[0]), keep(n2[1]), keep(n2[2]), keep(k2), keep(cfg);
            __syncthreads();
            if (j == 1) {  // the second event's block takes the first one's place
                for (int k = ln; k < S_SMALL; k += 64) T[k] = T[S_B + k];
                __syncthreads();
            }
            {  // triple currents
                const int sAB = w3[3], sBC = w3[4];
                const vec X = ld_vec(T, lo16(w3[0]), 2), Y = ld_vec(T, hi16(w3[0]), 2), Z = ld_vec(T, lo16(w3[1]), 2);
                const vec QA = ld_vec(T, hi16(w3[1]), 1), QB = ld_vec(T, lo16(w3[2]), 1), QC = ld_vec(T, hi16(w3[2]), 1);
                vec w{{0.0, 0.0, 0.0, 0.0}};
                sub_vvv(w, flip_sign(ld_vec(T, hi16(sAB), 4), sAB), add(QA, QB), Z, QC);
                sub_vvv(w, X, QA, flip_sign(ld_vec(T, hi16(sBC), 4), sBC), add(QB, QC));
                add_vvvv(w, X, Y, Z);
                st_vec(T, lo16(sBC), 8, mul(lds_at(T, lo16(sAB))->x, w));
            }
            {  // line currents with one gluon: strides of N0 and N1 differ
                const int t = (ln & 32) ? 16 : 0;
                const int of = lo16(c1[0]), orr = hi16(c1[0]);
                const int df = 64 - 2 * t, dr = 32 + 2 * t;
                const double2 f0 = *lds_at(T, of), f1 = *lds_at(T, of + df), f2 = *lds_at(T, of + 2 * df),
                              f3 = *lds_at(T, of + 3 * df);
                const double2 r0 = *lds_at(T, orr), r1 = *lds_at(T, orr + dr), r2 = *lds_at(T, orr + 2 * dr),
                              r3 = *lds_at(T, orr + 3 * dr);
                st_row(T, c1[1], 8, current(row{{{f0.x, f0.y}, {f1.x, f1.y}, {f2.x, f2.y}, {f3.x, f3.y}}},
                                            row{{{r0.x, r0.y}, {r1.x, r1.y}, {r2.x, r2.y}, {r3.x, r3.y}}}));
            }
            __syncthreads();
            if (ln < 32) {  // [middle 2] = - [middle 0] - [middle 1]
                const int o = 16 * (S_W3 + 48 * (ln >> 3) + (ln & 7));
                const vec w = add(ld_vec(T, o, 8), ld_vec(T, o + 256, 8));
                st_vec(T, o + 512, 8, mul(-1.0, w));
            }
            __syncthreads();
            // four-gluon currents without their propagator
            auto four = [&](const int(&o)[6]) __attribute__((always_inline)) {
                const vec eA = ld_vec(T, 16 * S_EPS + 16 * bit(ln, 0), 2), eB = ld_vec(T, lo16(o[0]), 2),
                          eC = ld_vec(T, lo16(o[1]), 2), eD = ld_vec(T, lo16(o[2]), 2);
                const vec QA = ld_vec(T, 16 * S_Q, 1), QB = ld_vec(T, hi16(o[0]), 1), QC = ld_vec(T, hi16(o[1]), 1),
                          QD = ld_vec(T, hi16(o[2]), 1);
                const vec AB = ld_vec(T, lo16(o[3]), 4), BC = flip_sign(ld_vec(T, hi16(o[3]), 4), o[3]),
                          CD = flip_sign(ld_vec(T, hi16(o[4]), 4), o[4]);
                const vec BCD = ld_vec(T, lo16(o[4]), 8), ABC = ld_vec(T, lo16(o[5]), 8);
                const vec QAB = add(QA, QB), QCD = add(QC, QD);
                vec w{{0.0, 0.0, 0.0, 0.0}};
                sub_vvv(w, eA, QA, BCD, add(QB, QCD));
                sub_vvv(w, AB, QAB, CD, QCD);
                sub_vvv(w, ABC, add(QAB, QC), eD, QD);
                add_vvvv(w, eA, eB, CD);
                add_vvvv(w, eA, BC, eD);
                add_vvvv(w, AB, eC, eD);
                st_vec(T, hi16(o[5]), 16, w);
            };
            four(w4[0]);
            __builtin_amdgcn_sched_barrier(0);
            if (ln < 32) four(w4[1]);
            __syncthreads();

            __builtin_amdgcn_s_setprio(1);
            // ---- J of configuration `lane` ----
            c2 J[24];
            {  // all four gluons in one tree
                const row V = ld_row(T, 16 * S_C0 + ((ln >> 4) << 4), 4);
                c2 t[6];
                each<6>([&](auto O) __attribute__((always_inline)) {
                    t[O] = cdot(V, ld_vec(T, 16 * (S_W4 + 32 * O) + ((ln & 15) << 4), 16));
                });
                each<9>([&](auto I) __attribute__((always_inline)) {
                    constexpr int b = 1 + I / 3, c = 1 + I % 3, d = 6 - b - c;
                    if constexpr (b != c) {
                        J[flow(0, b, c, d)] = t[tree(b, c)];
                        J[flow(b, c, d, 0)] = -t[tree(d, c)];
                        J[flow(b, 0, c, d)] = -(t[tree(b, c)] + t[tree(c, b)] + t[tree(c, d)]);
                        J[flow(b, c, 0, d)] = t[tree(c, b)] + t[tree(c, d)] + t[tree(d, c)];
                    }
                });
            }
            {  // three gluons in one tree
                each<4>([&](auto MG) __attribute__((always_inline)) {
                    constexpr int mg = MG;
                    constexpr int x = other(mg, 0), y = other(mg, 1), z = other(mg, 2);
                    const int ip = 16 * (S_W3 + 48 * mg) + byte_of<mg>(cfg[6]);
                    const vec w0 = ld_vec(T, ip, 8), w1 = ld_vec(T, ip + 256, 8);
                    const int iv = 16 * (S_C1 + 32 * mg) + byte_of<mg>(cfg[7]);
                    {
                        const row V = ld_row(T, iv, 8);
                        // the middle gluon is x (t0), y (t1) or z (t2)
                        const c2 t0 = cdot(V, w0), t1 = cdot(V, w1), t2 = t0 + t1;
                        J[flow(mg, y, x, z)] += t0;
                        J[flow(mg, z, x, y)] += t0;
                        J[flow(mg, x, y, z)] += t1;
                        J[flow(mg, z, y, x)] += t1;
                        J[flow(mg, x, z, y)] -= t2;
                        J[flow(mg, y, z, x)] -= t2;
                    }
                    {
                        const row V = ld_row(T, iv + 16 * 128, 8);
                        const c2 t0 = cdot(V, w0), t1 = cdot(V, w1), t2 = t0 + t1;
                        J[flow(y, x, z, mg)] += t0;
                        J[flow(z, x, y, mg)] += t0;
                        J[flow(x, y, z, mg)] += t1;
                        J[flow(z, y, x, mg)] += t1;
                        J[flow(x, z, y, mg)] -= t2;
                        J[flow(y, z, x, mg)] -= t2;
                    }
                });
            }
            // two-gluon row of one lane
            auto rows = [&](const int(&o)[3], bool prop, bool mine) __attribute__((always_inline)) {
                row f = slash(ld_row(T, lo16(o[0]), 4), ld_vec(T, hi16(o[0]), 2));
                f = add_slash(f, ld_row(T, lo16(o[1]), 2), flip_sign(ld_vec(T, hi16(o[1]), 4), o[1]));
                if (prop) {
                    const int k = lo16(o[2]);
                    const double2 d = *lds_at(T, (k >> 1) + 16 * S_F + 160 - 8 * S_K);
                    const row g = scale(c2{d.x, d.y}, slash_m(f, ld_vec(T, k, 1), m));
                    if (mine) f = g;
                }
                st_row(T, hi16(o[2]), 8, f);
            };
            // L(ab) [W(c) R(d) + W(cd) v] for the split of pair p from its rows in slot s
            auto split = [&](auto PR) __attribute__((always_inline)) {
                constexpr int p = PR, s = p & 3, a = pair_lo(p), b = pair_hi(p), q = 5 - p, c = pair_lo(q), d = pair_hi(q);
                const int ol = 16 * (S_N2 + 128 * s) + byte_of<0>(cfg[p]);
                const int orr = 16 * (S_N2 + 128 * s + 64) + byte_of<1>(cfg[q]);
                const row l0 = ld_row(T, ol, 8), l1 = ld_row(T, ol + 512, 8);    // (a, b), (b, a)
                const row r0 = ld_row(T, orr, 8), r1 = ld_row(T, orr + 512, 8);  // absorbing c then d, d then c
                J[flow(a, b, c, d)] = wedge(l0, r1, J[flow(a, b, c, d)]);
                J[flow(a, b, d, c)] = wedge(l0, r0, J[flow(a, b, d, c)]);
                J[flow(b, a, c, d)] = wedge(l1, r1, J[flow(b, a, c, d)]);
                J[flow(b, a, d, c)] = wedge(l1, r0, J[flow(b, a, d, c)]);
            };
            // currents L(a) gamma R(d) of one lane, and L(a) W(bc) R(d) for pair p = {a, d}
            auto currents = [&](int o, int to) __attribute__((always_inline)) {
                st_row(T, to, 16, current(ld_row(T, lo16(o), 4), ld_row(T, hi16(o), 4)));
            };
            const int c2at = ((ln >> 4) << 10) + ((ln & 15) << 4);
            auto middle = [&](auto PR) __attribute__((always_inline)) {
                constexpr int p = PR, lo = pair_lo(p), hi = pair_hi(p), q = 5 - p, b = pair_lo(q), c = pair_hi(q);
                const vec w = ld_vec(T, 16 * (S_W2 + 8 * q) + byte_of<3>(cfg[q]), 4);
                const int o = 16 * (p < 4 ? S_C2 + 128 * p : S_C2B + 128 * (p - 4)) + byte_of<2>(cfg[p]);
                c2 t = cdot(ld_row(T, o, 16), w);
                J[flow(lo, b, c, hi)] += t;
                J[flow(lo, c, b, hi)] -= t;
                t = cdot(ld_row(T, o + 1024, 16), w);
                J[flow(hi, b, c, lo)] += t;
                J[flow(hi, c, b, lo)] -= t;
            };
            settle(J);
            __syncthreads();
            rows(n2[0], true, true);
            __builtin_amdgcn_sched_barrier(0);
            rows(n2[1], false, false);
            __syncthreads();
            each<4>(split);
            settle(J);
            __syncthreads();
            currents(k2[0], 16 * S_C2 + c2at);
            currents(k2[1], 16 * (S_C2 + 256) + c2at);
            __syncthreads();
            each<4>(middle);
            settle(J);
            __syncthreads();
            rows(n2[2], true, !(ln & 16));
            __builtin_amdgcn_sched_barrier(0);
            currents(k2[2], 16 * S_C2B + c2at);
            __syncthreads();
            each<6, 4>(split);
            settle(J);
            each<6, 4>(middle);
            __builtin_amdgcn_s_setprio(0);
            double q;
            if constexpr (CM) {
                __shared__ double Jt[P::ncol * 2 * 64];
                each<P::ncol>([&](auto K) __attribute__((always_inline)) {
                    Jt[(2 * K) * 64 + lane] = J[K].r;
                    Jt[(2 * K + 1) * 64 + lane] = J[K].i;
                });
                __syncthreads();
                q = 0.0;
#pragma unroll
                for (int eb16 = 0; eb16 < 4; ++eb16) {
                    const double s = colour_mfma_group_sum(
                        colour_mfma16<P::ncol>(Jt, 16 * eb16, colour_table<P>::mfma_frag(), lane));
                    if (eb16 == (lane >> 4)) q = s;  // this lane's own column
                }
            } else {
                q = P::colour_blocks(J);
            }
            q = ((spins >> (lane >> 4)) & 1) ? q : 0.0;
            const double tot = wave_sum(q);
            if (lane == 63) {
                const int64_t i = base + j;
                out[count ? (int64_t)idx[i] : i] = tot * (1.0 / (256.0 * P::identical * P::lcd));
            }
            __builtin_amdgcn_s_setprio(2);
        }
    }
}

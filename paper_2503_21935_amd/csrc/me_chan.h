// me_chan.h -- single-diagram weights of the multi-channel form, g g -> t tbar g g:
// alpha = sum |A_chan|^2 / sum over the channels d of sum |A_d|^2, both sums over
// polarisations and spins.  Rules and signs as in me_wave.h.
//
// A_d is linear in every polarisation vector, so its sum of squares, like that
// of the whole amplitude, may run over the real vectors, and diagrams share
// their factors: one event per wave, its currents and rows in LDS, the rows of
// the different diagrams kept apart (no tree is merged with another, and there
// are no four-gluon vertices).  Of the 105 diagrams 54 are products of a row
// with two gluons from either end: for each of the six ways to part the
// gluons lane (i, j) holds three rows of the left end at configuration i and
// three of the right end at j and forms all nine products.  Elsewhere a lane keeps a
// current and runs over the vectors it meets.  |A_d|^2 is formed from A_d, not
// from spin density matrices, which would take fewer operations but square
// the cancellations between the components of a row.
// The channel only selects which sums enter the numerator.
//
// Bound by VALU issue (about 3,000 vector instructions per event): 2^16 events
// take 0.44 ms, 0.86 ms with their |M|^2 (k_me_gg4_wave), against 4.45 ms with
// one amplitude program per helicity, one event per lane (k_me_gg_mc).
#pragma once
#include "me_wave.h"

// C: the channel numbers of the diagrams (chan_ids_*).  Blocks of one wave
// stride over the events, eb (1 or 2) at a time.
template <class C>
__global__ __launch_bounds__(64, 2) void k_me_gg4_chan(const double* __restrict__ mom, int64_t nevt,
                                                       const int* __restrict__ chan, double* __restrict__ alpha,
                                                       me_params prm, int eb) {
    using namespace wv;
    // From S_W3 on, one event at a time: the trees of three gluons [missing
    // gluon][which of the others joins last][2][pols 8], then the rows of three
    // splits [split][end][kind 3][component][config 8].
    constexpr int S_ROWS = S_W3;
    static_assert(S_ROWS + 3 * 192 <= S_B, "rows fit below the second event");
    __shared__ double2 T[S_END];
    const int lane = threadIdx.x;
    const double m = prm.mt;

    // ---- where this lane's nodes read and write ----
    // trees of three gluons: node 64 pass + lane = (missing gluon, k, pols)
    int t3[2][3];
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        const int node = (64 * pass + lane) % 96, mg = node / 24, k = (node >> 3) % 3;
        const int l = k, a = k == 0 ? 1 : 0, b = k == 2 ? 1 : 2;  // of the three, l joins a and b
        const int A = other(mg, a), B = other(mg, b), L = other(mg, l);
        t3[pass][0] = pack(w2_at(A, B, bit(node, a), bit(node, b)), eps_at(L, bit(node, l)));
        t3[pass][1] = pack(q_at(A), q_at(B));
        t3[pass][2] = pack(16 * (S_W3 + 48 * mg + 16 * k + (node & 7)), q_at(L));
    }
    // four gluons in one tree: lane (gluon mg that joins the others last, or pair (0, mg + 1), pols)
    const int g4 = lane >> 4;
    int t4[4];
    {
        const int x = other(g4, 0), y = other(g4, 1), z = other(g4, 2);
        t4[0] = pack(16 * (S_W3 + 48 * g4 + bit(lane, x) + 2 * bit(lane, y) + 4 * bit(lane, z)),
                     eps_at(g4, bit(lane, g4)));
        const int p = g4 % 3, q = 5 - p;  // pair (0, p + 1) and the rest
        t4[1] = pack(16 * (S_W2 + 8 * p + bit(lane, pair_lo(p)) + 2 * bit(lane, pair_hi(p))),
                     16 * (S_W2 + 8 * q + bit(lane, pair_lo(q)) + 2 * bit(lane, pair_hi(q))));
        t4[2] = pack(q_at(pair_hi(p)), q_at(pair_lo(q)));
        t4[3] = pack(q_at(pair_hi(q)), 0);
    }
    // one gluon on the line, three in a tree: lane (end, gluon, pol, spins)
    int c1[2];
    {
        const int e = lane >> 5, a = (lane >> 3) & 3, pol = bit(lane, 0), s3 = bit(lane, 1), s4 = bit(lane, 2);
        const int o1 = 16 * (S_N1 + 16 * (4 * e + a) + pol + 2 * (e ? s4 : s3));
        const int o0 = 16 * (e ? S_N0 + s3 : S_N0 + 8 + s4);
        c1[0] = e ? pack(o0, o1) : pack(o1, o0);
        c1[1] = 16 * (S_W3 + 48 * a);
    }
    // a pair between two gluons: lane (outer pair 2 of 6, order, pols, spins) in three passes
    int c2m[3][2];
#pragma unroll
    for (int pass = 0; pass < 3; ++pass) {
        const int op = 4 * pass + (lane >> 4), p = op >> 1, flip = op & 1;
        const int a = flip ? pair_hi(p) : pair_lo(p), d = flip ? pair_lo(p) : pair_hi(p);
        c2m[pass][0] = pack(16 * (S_N1 + 16 * a + bit(lane, 0) + 2 * bit(lane, 2)),
                            16 * (S_N1 + 16 * (4 + d) + bit(lane, 1) + 2 * bit(lane, 3)));
        c2m[pass][1] = 16 * (S_W2 + 8 * (5 - p));
    }
    // rows of splits 0..2 or 3..5: lane (split, first gluon, pols, spin) at either end,
    // and with the pair current: lane (split, end, pols, spin)
    int rw[2][5];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const int s = (lane >> 4) % 3, p = 3 * half + s, q = 5 - p, flip = bit(lane, 3), sp = bit(lane, 2);
        auto one = [&](int e, int r) {
            const int x = flip ? pair_hi(r) : pair_lo(r), y = flip ? pair_lo(r) : pair_hi(r);
            return pack(16 * (S_N1 + 16 * (4 * e + x) + bit(lane, flip) + 2 * sp), eps_at(y, bit(lane, 1 - flip)));
        };
        rw[half][0] = one(0, p);
        rw[half][1] = one(1, q);
        rw[half][2] = pack(16 * (S_N0 + 8 * flip + sp), 16 * (S_W2 + 8 * (flip ? q : p) + (lane & 3)));
        rw[half][3] = pack(16 * (S_K + 2 * (4 + p)), 16 * (S_ROWS + 192 * s + 32 * flip + (lane & 7)));
        // from p4 the gluon absorbed first stands last
        rw[half][4] = pack(16 * (S_ROWS + 192 * s + 96 + 32 * (1 - flip) + (lane & 7)),
                           16 * (S_ROWS + 192 * s + 96 * flip + 64 + (lane & 7)));
    }
    // channels of this lane's diagrams, a byte each
    int id[3] = {0, 0, 0};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int op = 4 * k + (lane >> 4);
        id[0] |= C::middle[op] << (8 * k);
        id[1] |= C::three[12 * (lane >> 5) + 3 * ((lane >> 3) & 3) + k] << (8 * k);
        id[2] |= C::four[3 * g4 + k] << (8 * k);
    }
    id[0] |= C::four[12 + g4 % 3] << 24;

    for (int64_t base = (int64_t)blockIdx.x * eb; base < nevt; base += (int64_t)gridDim.x * eb) {
        const int ne = (eb == 2 && base + 1 < nevt) ? 2 : 1;
        __syncthreads();  // the previous event's reads are done
        gg4_setup(T, mom, base, ne, nullptr, nullptr, prm, lane);
#pragma unroll 1
        for (int j = 0; j < ne; ++j) {
            int ln = lane;
            asm volatile("" : "+v"(ln));
            keep(t3[0]), keep(t3[1]), keep(t4), keep(c1), keep(c2m[0]), keep(c2m[1]), keep(c2m[2]);
            keep(rw[0]), keep(rw[1]), keep(id);
            const int ch = chan[base + j];
            __syncthreads();
            if (j == 1) {  // the second event's block takes the first one's place
                for (int k = ln; k < S_SMALL; k += 64) T[k] = T[S_B + k];
                __syncthreads();
            }
            double num = 0.0, den = 0.0;
            auto found = [&](int c, double a2) __attribute__((always_inline)) {
                den += a2;
                num += c == ch ? a2 : 0.0;
                asm volatile("" : "+v"(den), "+v"(num));  // formed here, or the operands are held until the end
            };
            auto square = [](c2 a, double acc) __attribute__((always_inline)) { return fma(a.r, a.r, fma(a.i, a.i, acc)); };
            // trees of three gluons, with their propagator
            auto three = [&](const int(&o)[3]) __attribute__((always_inline)) {
                const vec X = ld_vec(T, lo16(o[0]), 4), Y = ld_vec(T, hi16(o[0]), 2);
                const vec QX = add(ld_vec(T, lo16(o[1]), 1), ld_vec(T, hi16(o[1]), 1)), QY = ld_vec(T, hi16(o[2]), 1);
                const vec Q = add(QX, QY);
                vec w{{0.0, 0.0, 0.0, 0.0}};
                sub_vvv(w, X, QX, Y, QY);
                st_vec(T, lo16(o[2]), 8, mul(1.0 / mdot(Q, Q), w));
            };
            three(t3[0]);
            __builtin_amdgcn_sched_barrier(0);
            if (ln < 32) three(t3[1]);
            __syncthreads();
            {  // four gluons in one tree: every spin pair of the ends
                row V[4];
                each<4>([&](auto S) __attribute__((always_inline)) { V[S] = ld_row(T, 16 * (S_C0 + S), 4); });
                auto sum = [&](const vec& w) __attribute__((always_inline)) {
                    double a2 = 0.0;
                    each<4>([&](auto S) __attribute__((always_inline)) { a2 = square(cdot(V[S], w), a2); });
                    return a2;
                };
                {
                    const vec Y = ld_vec(T, hi16(t4[0]), 2), QY = ld_vec(T, 16 * S_Q + 2 * (ln & 48), 1);
                    vec QX = mul(-1.0, QY);
                    each<4>([&](auto A) __attribute__((always_inline)) { QX = add(QX, ld_vec(T, q_at(A), 1)); });
                    each<3>([&](auto K) __attribute__((always_inline)) {
                        vec w{{0.0, 0.0, 0.0, 0.0}};
                        sub_vvv(w, ld_vec(T, lo16(t4[0]) + 256 * K, 8), QX, Y, QY);
                        found(byte_of<K>(id[2]), sum(w));
                    });
                }
                {
                    vec w{{0.0, 0.0, 0.0, 0.0}};
                    sub_vvv(w, ld_vec(T, lo16(t4[1]), 4), add(ld_vec(T, q_at(0), 1), ld_vec(T, lo16(t4[2]), 1)),
                            ld_vec(T, hi16(t4[1]), 4), add(ld_vec(T, hi16(t4[2]), 1), ld_vec(T, lo16(t4[3]), 1)));
                    found(byte_of<3>(id[0]), ln < 48 ? sum(w) : 0.0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            {  // three gluons in a tree, one on the line: strides of N0 and N1 differ
                const int t = (ln & 32) ? 16 : 0;
                const int of = lo16(c1[0]), orr = hi16(c1[0]);
                const int df = 64 - 2 * t, dr = 32 + 2 * t;
                const double2 f0 = *lds_at(T, of), f1 = *lds_at(T, of + df), f2 = *lds_at(T, of + 2 * df),
                              f3 = *lds_at(T, of + 3 * df);
                const double2 r0 = *lds_at(T, orr), r1 = *lds_at(T, orr + dr), r2 = *lds_at(T, orr + 2 * dr),
                              r3 = *lds_at(T, orr + 3 * dr);
                const row V = current(row{{{f0.x, f0.y}, {f1.x, f1.y}, {f2.x, f2.y}, {f3.x, f3.y}}},
                                      row{{{r0.x, r0.y}, {r1.x, r1.y}, {r2.x, r2.y}, {r3.x, r3.y}}});
                each<3>([&](auto K) __attribute__((always_inline)) {
                    double a2 = 0.0;
                    each<8>([&](auto P) __attribute__((always_inline)) {
                        a2 = square(cdot(V, ld_vec(T, c1[1] + 16 * (16 * K + P), 8)), a2);
                        asm volatile("" : "+v"(a2));
                    });
                    found(byte_of<K>(id[1]), a2);
                });
            }
            __builtin_amdgcn_sched_barrier(0);
            each<3>([&](auto K) __attribute__((always_inline)) {  // a pair between two gluons
                const row V = current(ld_row(T, lo16(c2m[K][0]), 4), ld_row(T, hi16(c2m[K][0]), 4));
                double a2 = 0.0;
                each<4>([&](auto P) __attribute__((always_inline)) {
                    a2 = square(cdot(V, ld_vec(T, c2m[K][1] + 16 * P, 4)), a2);
                });
                found(byte_of<K>(id[0]), a2);
                __builtin_amdgcn_sched_barrier(0);
            });
            // two gluons from either end
            each<2>([&](auto H) __attribute__((always_inline)) {
                const int(&o)[5] = rw[H];
                __syncthreads();  // the trees, or the previous rows, have been read
                if (ln < 48) {
                    const vec P = ld_vec(T, lo16(o[3]), 1);
                    st_row(T, hi16(o[3]), 8, slash_m(slash(ld_row(T, lo16(o[0]), 4), ld_vec(T, hi16(o[0]), 2)), P, m));
                    st_row(T, lo16(o[4]), 8, slash(ld_row(T, lo16(o[1]), 4), ld_vec(T, hi16(o[1]), 2)));
                    row f = slash(ld_row(T, lo16(o[2]), 2), ld_vec(T, hi16(o[2]), 4));
                    const row g = slash_m(f, P, m);
                    if (!(ln & 8)) f = g;
                    st_row(T, hi16(o[4]), 8, f);
                }
                __syncthreads();
                const int ol = 16 * S_ROWS + ((ln & 7) << 4), orr = 16 * (S_ROWS + 96) + ((ln >> 3) << 4);
                each<3>([&](auto S) __attribute__((always_inline)) {
                    constexpr int p = 3 * H + S;
                    row l[3], r[3];
                    each<3>([&](auto K) __attribute__((always_inline)) {
                        l[K] = ld_row(T, ol + 16 * (192 * S + 32 * K), 8);
                        r[K] = ld_row(T, orr + 16 * (192 * S + 32 * K), 8);
                    });
                    // the propagator between them belongs to all nine
                    const double2 d = *lds_at(T, 16 * (S_F + 14 + p));
                    const double f2 = fma(d.x, d.x, d.y * d.y);
                    double dn = 0.0, nm = 0.0;
                    each<9>([&](auto K) __attribute__((always_inline)) {
                        constexpr int c = C::split[9 * p + K];
                        const double a2 = square(wedge(l[K / 3], r[K % 3], c2{0.0, 0.0}), 0.0);
                        dn += a2;
                        nm += c == ch ? a2 : 0.0;
                        asm volatile("" : "+v"(dn), "+v"(nm));
                    });
                    den = fma(f2, dn, den);
                    num = fma(f2, nm, num);
                    asm volatile("" : "+v"(den), "+v"(num));
                    __builtin_amdgcn_sched_barrier(0);
                });
            });
            num = wave_sum(num);
            den = wave_sum(den);
            if (lane == 63) alpha[base + j] = num / den;
        }
    }
}

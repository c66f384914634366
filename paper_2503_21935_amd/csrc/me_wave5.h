// me_wave5.h -- g g -> t tbar g g g summed over spins with real polarisation
// vectors: one event per workgroup, every wavefunction computed once and kept
// in LDS.  Rules, signs and the row form of columns as in me_wave.h; the top
// line is cut after two gluons,
//   J_abcde = L(ab) [W(c) R(de) + W(cd) R(e) + W(cde) v]
//           + [L(a) W(bc) + ubar W(abc)] R(de)
//           + L(a) W(bcd) R(e) + L(a) W(bcde) v + ubar W(abcd) R(e) + ubar W(abcde) v.
//
// Twelve waves.  The nodes of one kind (pair currents, three-gluon rows, ...)
// are handed out over all lanes, operands and destinations from generated
// tables.  Then the waves sum J, in twenty units of twelve orderings (those
// that begin with the two gluons of one pair, at one spin of tbar) by 64
// configurations (the polarisations and the top's spin): of the three waves
// on a SIMD two take two units and one takes one, so that the SIMDs are even;
// the latter (waves 8 to 11) also prepare the next event's externals.  Every
// ordering is summed directly from full tables of currents (no shuffle
// identities there), so a contribution is a chain of fma on J.  The colour sum
// goes through LDS one part (real, imaginary) at a time: signed sums over the
// Klein four-group and the reversal split the 120 x 120 form into eight blocks.
// 159 kB of LDS: one workgroup per CU, three waves per SIMD.
//
// Measured: 2^15 events in 3.45 ms (9.5e6 per second) where the kernel with one
// event per lane and a diagram program split over four waves (k_me_gg_coop)
// takes 37 ms, 64 events in 31 us against 280 us.  An event takes a CU about 65,000
// cycles: 38,000 vector instructions, the VALU active 60 % of the time; the rest
// is barriers between some twenty stages and the latency of LDS and tables
// that three waves per SIMD leave open.  168 registers per lane are what three
// waves leave; what was kept from phase to phase (lane indices, 64-bit table
// addresses, the second unit's sums while the next event is prepared) spilled
// 136 bytes per lane, now 100: 50,021 events write 1.0 GB of it instead of 2.7
// and took 5.33 ms instead of 5.56 (now 5.26, with the priority of the preparing waves).
#pragma once
#include "gen/proc_gg_ttggg_wave.h"
#include "me_wave.h"

namespace w5 {

using namespace wv;

// Byte offsets packed in a table word: bits 4..17 and 18..31.
MEV int lo_at(int w) { return w & 0x3fff0; }
MEV int hi_at(int w) { return (int)((unsigned)w >> 14) & 0x3fff0; }

template <int Q>
struct words {
    int4 q[Q];
    template <int I>
    MEV int at() const {  // I-th offset
        constexpr int k = I / 2;
        const int4 v = q[k / 4];
        const int w = k % 4 == 0 ? v.x : k % 4 == 1 ? v.y : k % 4 == 2 ? v.z : v.w;
        return I & 1 ? hi_at(w) : lo_at(w);
    }
};
// The loads of w have to have arrived here.
template <int Q>
MEV void arrived(words<Q>& w) {
#pragma unroll
    for (int k = 0; k < Q; ++k) asm volatile("" : "+v"(w.q[k].x), "+v"(w.q[k].y), "+v"(w.q[k].z), "+v"(w.q[k].w));
}
// Entry `node` of a table of [Q][n] int4.
template <int Q>
MEV words<Q> ld_words(const int4* __restrict__ tab, int n, int node) {
    words<Q> w;
    const unsigned off = 16u * (unsigned)node;  // scalar base plus this: no 64-bit addresses to keep
#pragma unroll
    for (int k = 0; k < Q; ++k)
        w.q[k] = *reinterpret_cast<const int4*>(reinterpret_cast<const char*>(tab + k * n) + off);
    return w;
}

enum { THREADS = 768 };

// The small tables of the event whose momenta (component `lane`, 28 of them) the
// lanes hold, into the block at byte offset B, in two rounds; the parts of a
// round may run on different waves.  Round 0, part 0: summed momenta and
// propagators; part 1: polarisation vectors; part 2: end rows.
MEV void prepare0(double2* T, int B, int part, double q, int lane, const me_params& prm) {
    const double m = prm.mt;
    if (lane < 28) reinterpret_cast<double*>(lds_at(T, B + 16 * w5::S_Q))[lane] = q;  // every part: the same values
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (part == 0) {
        if (lane < 56) {
            const int c = tab_K[lane];
            vec K{{0.0, 0.0, 0.0, 0.0}};
#pragma unroll
            for (int s = 0; s < 7; ++s) {
                const double w = (double)(bit(c, 2 * s) - bit(c, 2 * s + 1));
                const vec p = ld_vec(T, B + 16 * (w5::S_Q + 2 * s), 1);
#pragma unroll
                for (int k = 0; k < 4; ++k) K.v[k] = fma(w, p.v[k], K.v[k]);
            }
            const bool top = lane >= 26;
            const double d = K.v[0] * K.v[0] - K.v[1] * K.v[1] - K.v[2] * K.v[2] - K.v[3] * K.v[3];
            c2 f = crecip(top ? d - m * m : d, top ? m * prm.wt : 0.0);
            // the row after one gluon from p3 carries -1/D
            if (lane >= 26 && lane < 31) f = -f;
            if (top) st_vec(T, B + 16 * (w5::S_K + 2 * (lane - 26)), 1, K);
            *lds_at(T, B + 16 * (w5::S_F + lane)) = double2{f.r, f.i};
        }
    } else if (part == 1) {
        if (lane < 10) {  // (gluon, which)
            const int a = lane >> 1;
            const vec p = ld_vec(T, B + 16 * (w5::S_Q + 2 * a), 1);
            st_vec(T, B + 16 * (w5::S_EPS + 4 * a + (lane & 1)), 2,
                   mul(prm.gs, polarisation(a < 2 ? p : mul(-1.0, p), lane & 1)));
        }
    } else if (lane < 4) {  // (end, spin)
        const int e = lane >> 1;
        st_row(T, B + 16 * (w5::S_N0 + 8 * e + (lane & 1)), 2,
               end_row(ld_vec(T, B + 16 * (w5::S_Q + 2 * (5 + e)), 1), m, e, (lane & 1) ? 1 : -1));
    }
}
// Round 1, part 0: pair currents and the current of the ends; part 1: one-gluon rows.
MEV void prepare1(double2* T, int B, int part, int lane, const me_params& prm) {
    if (part == 0) {
        if (lane < N_W2) {
            const auto w = ld_words<1>(tab_W2, N_W2, lane);
            vec x{{0.0, 0.0, 0.0, 0.0}};
            sub_vvv(x, ld_vec(T, B + w.at<0>(), 2), ld_vec(T, B + w.at<2>(), 1), ld_vec(T, B + w.at<1>(), 2),
                    ld_vec(T, B + w.at<3>(), 1));
            x = mul(lds_at(T, B + w.at<4>())->x, x);
            st_vec(T, B + w.at<5>(), 4, x);
            st_vec(T, B + w.at<6>(), 4, mul(-1.0, x));
        } else if (lane < N_W2 + 4) {  // with the gluon propagator
            const int l = lane - N_W2;
            const double iq = lds_at(T, B + 16 * (w5::S_F + 25))->x;
            const row V = current(ld_row(T, B + 16 * (w5::S_N0 + bit(l, 0)), 2),
                                  ld_row(T, B + 16 * (w5::S_N0 + 8 + bit(l, 1)), 2));
            st_row(T, B + 16 * (w5::S_C0 + l), 4, scale(c2{iq, 0.0}, V));
        }
    } else if (lane < N_N1) {
        const auto w = ld_words<1>(tab_N1, N_N1, lane);
        const row f = slash_m(slash(ld_row(T, B + w.at<0>(), 2), ld_vec(T, B + w.at<1>(), 2)),
                              ld_vec(T, B + w.at<2>(), 1), prm.mt);
        const double2 d = *lds_at(T, B + w.at<3>());
        st_row(T, B + w.at<4>(), 4, scale(c2{d.x, d.y}, f));
    }
}

}  // namespace w5

// Arguments as for k_me_gg4_wave; blocks of 768 threads stride over the events.
// The tables of a phase are asked for before the barrier in front of it: they
// come from the L2, and one workgroup per CU has nothing else to hide that.
template <class P, bool CM>
__global__ __launch_bounds__(w5::THREADS) void k_me_gg5_wave(const double* __restrict__ mom, int64_t nevt,
                                                             double* __restrict__ out, unsigned spins,
                                                             me_params prm, const int* __restrict__ idx,
                                                             const int* __restrict__ count) {
    using namespace wv;
    using namespace w5;
    static_assert(P::ngluon == 5 && P::ncol == 120, "five gluons");
    constexpr int NP = 7;
    __shared__ double2 T[w5::S_END];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // Lane and thread index, made anew in every phase: kept, they and what is
    // formed from them spill.
    int lane, tid;
    auto here = [&]() __attribute__((always_inline)) {
        lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        asm volatile("" : "+v"(lane));
        tid = 64 * wave + lane;
    };
    here();
    const int64_t n = count ? (int64_t)*count : nevt;
    const double m = prm.mt;
    double* const D = reinterpret_cast<double*>(T);
    constexpr int NEXT = 16 * w5::S_WINDOW;
    // this wave's units and their spin of tbar
    const int unit[2] = {wave < 8 ? 2 * wave : 8 + wave, wave < 8 ? 2 * wave + 1 : 0};
    const int s4[2] = {unit[0] / 10, unit[1] / 10};
    const bool both = wave < 8;
    // waves 8, 9 and 10 prepare the next event: lane l holds component l of (gluons in incoming flow, p3, p4)
    const bool ahead = wave >= 8 && wave < 11;
    double q28 = 0.0;
    auto fetch = [&](int64_t i, int l) __attribute__((always_inline)) {
        const int slot = l >> 2;
        if (ahead && l < 28 && i < n) {
            const int part = slot < 2 ? slot : slot < 5 ? slot + 2 : slot - 3;
            q28 = mom[(count ? (int64_t)idx[i] : i) * (NP * 4) + 4 * part + (l & 3)];
        }
    };
    auto incoming = [&](int l) __attribute__((always_inline)) {  // with the sign of the incoming flow
        return (l >> 2) >= 2 && (l >> 2) < 5 ? -q28 : q28;
    };
    fetch(blockIdx.x, lane);
    if (ahead) prepare0(T, NEXT, wave - 8, incoming(lane), lane, prm);
    __syncthreads();
    if (ahead && wave < 10) prepare1(T, NEXT, wave - 8, lane, prm);
    // the waves' shares of the colour sum of event i, added up once every wave has passed a barrier
    double* const part = D + 2 * (w5::S_END - 8);
    auto finish = [&](int64_t i, int lane) __attribute__((always_inline)) {
        const double s = wave_sum(lane < THREADS / 64 ? part[lane] : 0.0);
        if (lane == 63) out[count ? (int64_t)idx[i] : i] = s * (1.0 / (256.0 * P::identical * P::lcd));
    };
    int64_t done = -1;
    for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
        here();
        static_assert(N_N2 == 320 && N_W3 == 240, "five waves and the next four");
        words<2> w23;
        if (wave < 5) {
            w23.q[0] = tab_N2[tid];
        } else {
            const int k = tid - 320 < N_W3 ? tid - 320 : N_W3 - 1;
            w23 = ld_words<2>(tab_W3, N_W3, k);
        }
        __syncthreads();
        here();
        if (wave == 11 && done >= 0) finish(done, lane);
        if (tid < w5::S_SMALL) T[tid] = T[w5::S_WINDOW + tid];
        auto w4 = ld_words<2>(tab_W4, N_W4, tid < N_W4 ? tid : N_W4 - 1);
        arrived(w23);
        __syncthreads();
        here();
        // ---- two-gluon rows and triple currents ----
        if (wave < 5) {
            const auto& w = w23;
            row f = slash(ld_row(T, w.template at<0>(), 4), ld_vec(T, w.template at<1>(), 2));
            f = add_slash(f, ld_row(T, w.template at<2>(), 2), ld_vec(T, w.template at<3>(), 4));
            const double2 d = *lds_at(T, w.template at<5>());
            st_row(T, w.template at<6>(), 8, scale(c2{d.x, d.y}, slash_m(f, ld_vec(T, w.template at<4>(), 1), m)));
        } else if (tid < 320 + N_W3) {
            const auto& w = w23;
            const vec X = ld_vec(T, w.template at<0>(), 2), Y = ld_vec(T, w.template at<1>(), 2),
                      Z = ld_vec(T, w.template at<2>(), 2);
            const vec QA = ld_vec(T, w.template at<3>(), 1), QB = ld_vec(T, w.template at<4>(), 1),
                      QC = ld_vec(T, w.template at<5>(), 1);
            vec x{{0.0, 0.0, 0.0, 0.0}};
            sub_vvv(x, ld_vec(T, w.template at<6>(), 4), add(QA, QB), Z, QC);
            sub_vvv(x, X, QA, ld_vec(T, w.template at<7>(), 4), add(QB, QC));
            add_vvvv(x, X, Y, Z);
            st_vec(T, w.template at<9>(), 8, mul(lds_at(T, w.template at<8>())->x, x));
        }
        arrived(w4);
        auto w4s = ld_words<1>(tab_W4S, N_W4S, tid < N_W4S ? tid : N_W4S - 1);
        auto w5d = ld_words<3>(tab_W5, N_W5, tid);
        __syncthreads();
        here();
        // ---- four-gluon currents: those that begin with the first gluon, then the rest ----
        if (tid < N_W4) {
            const auto& w = w4;
            const vec eA = ld_vec(T, w.template at<0>(), 2), eB = ld_vec(T, w.template at<1>(), 2),
                      eC = ld_vec(T, w.template at<2>(), 2), eD = ld_vec(T, w.template at<3>(), 2);
            const vec QA = ld_vec(T, w.template at<4>(), 1), QB = ld_vec(T, w.template at<5>(), 1),
                      QC = ld_vec(T, w.template at<6>(), 1), QD = ld_vec(T, w.template at<7>(), 1);
            const vec AB = ld_vec(T, w.template at<8>(), 4), BC = ld_vec(T, w.template at<9>(), 4),
                      CD = ld_vec(T, w.template at<10>(), 4);
            const vec QAB = add(QA, QB), QCD = add(QC, QD);
            vec x{{0.0, 0.0, 0.0, 0.0}};
            sub_vvv(x, eA, QA, ld_vec(T, w.template at<12>(), 8), add(QB, QCD));
            sub_vvv(x, AB, QAB, CD, QCD);
            sub_vvv(x, ld_vec(T, w.template at<11>(), 8), add(QAB, QC), eD, QD);
            add_vvvv(x, eA, eB, CD);
            add_vvvv(x, eA, BC, eD);
            add_vvvv(x, AB, eC, eD);
            x = mul(lds_at(T, w.template at<13>())->x, x);
            st_vec(T, w.template at<14>(), 16, x);
            st_vec(T, w.template at<15>(), 16, mul(-1.0, x));
        }
        static_assert(N_W5 == THREADS && N_W5A == THREADS && N_W5B <= THREADS, "one node per thread");
        arrived(w4s);
        arrived(w5d);
        __syncthreads();
        here();
        if (tid < N_W4S) {
            const auto& w = w4s;
            const vec x = add(add(ld_vec(T, w.template at<0>(), 16), ld_vec(T, w.template at<1>(), 16)),
                              ld_vec(T, w.template at<2>(), 16));
            st_vec(T, w.template at<3>(), 16, mul(-1.0, x));
            st_vec(T, w.template at<4>(), 16, x);
        }
        __syncthreads();
        here();
        // ---- five-gluon currents, without their propagator ----
        auto w5a = ld_words<1>(tab_W5A, N_W5A, tid);
        auto w5b = ld_words<1>(tab_W5B, N_W5B, tid < N_W5B ? tid : N_W5B - 1);
        {
            const auto& w = w5d;
            vec x{{0.0, 0.0, 0.0, 0.0}};
            const vec eA = ld_vec(T, w.template at<0>(), 2), eE = ld_vec(T, w.template at<4>(), 2);
            const vec QA = ld_vec(T, w.template at<5>(), 1), QB = ld_vec(T, w.template at<6>(), 1),
                      QC = ld_vec(T, w.template at<7>(), 1), QD = ld_vec(T, w.template at<8>(), 1),
                      QE = ld_vec(T, w.template at<9>(), 1);
            const vec QAB = add(QA, QB), QDE = add(QD, QE), QCDE = add(QC, QDE), QABC = add(QAB, QC);
            {
                const vec BCDE = ld_vec(T, w.template at<18>(), 16), ABCD = ld_vec(T, w.template at<17>(), 16);
                sub_vvv(x, eA, QA, BCDE, add(QB, QCDE));
                sub_vvv(x, ABCD, add(QABC, QD), eE, QE);
            }
            const vec AB = ld_vec(T, w.template at<10>(), 4), DE = ld_vec(T, w.template at<13>(), 4);
            const vec ABC = ld_vec(T, w.template at<14>(), 8), CDE = ld_vec(T, w.template at<16>(), 8);
            sub_vvv(x, AB, QAB, CDE, QCDE);
            sub_vvv(x, ABC, QABC, DE, QDE);
            const vec eB = ld_vec(T, w.template at<1>(), 2), eD = ld_vec(T, w.template at<3>(), 2);
            add_vvvv(x, eA, eB, CDE);
            add_vvvv(x, ABC, eD, eE);
            add_vvvv(x, eA, ld_vec(T, w.template at<15>(), 8), eE);
            add_vvvv(x, AB, ld_vec(T, w.template at<2>(), 2), DE);
            add_vvvv(x, eA, ld_vec(T, w.template at<11>(), 4), DE);
            add_vvvv(x, AB, ld_vec(T, w.template at<12>(), 4), eE);
            st_vec(T, w.template at<19>(), 32, x);
        }
        // entries of this wave's orderings at configuration `lane`, per slot and stage
        const int4* const cfg[2] = {tab_cfg + unit[0] * CFG_UNIT, tab_cfg + unit[1] * CFG_UNIT};
        words<Q_TREE> tree[2] = {ld_words<Q_TREE>(cfg[0] + AT_TREE, 64, lane), ld_words<Q_TREE>(cfg[1] + AT_TREE, 64, lane)};
        arrived(w5a);
        arrived(w5b);
        __syncthreads();
        here();
        {
            const vec x = add(add(ld_vec(T, w5a.template at<0>(), 32), ld_vec(T, w5a.template at<1>(), 32)),
                              add(ld_vec(T, w5a.template at<2>(), 32), ld_vec(T, w5a.template at<3>(), 32)));
            st_vec(T, w5a.template at<4>(), 32, mul(-1.0, x));
            if (tid < N_W5B) {
                const vec y = add(add(ld_vec(T, w5b.template at<0>(), 32), ld_vec(T, w5b.template at<1>(), 32)),
                                  add(ld_vec(T, w5b.template at<2>(), 32), ld_vec(T, w5b.template at<3>(), 32)));
                st_vec(T, w5b.template at<6>(), 32,
                       add(y, add(ld_vec(T, w5b.template at<4>(), 32), ld_vec(T, w5b.template at<5>(), 32))));
            }
        }
        static_assert(N_CAE == 320 && N_C1L == 40 && N_C1R == 40, "waves 0-4, 5, 6");
        const int lane40 = lane < 40 ? lane : 39;
        words<1> wc = wave < 5    ? ld_words<1>(tab_CAE, N_CAE, tid)
                      : wave == 5 ? ld_words<1>(tab_C1L, N_C1L, lane40)
                                  : ld_words<1>(tab_C1R, N_C1R, lane40);
        arrived(tree[0]);
        arrived(tree[1]);
        __syncthreads();
        here();

        // ---- J of 24 (or 12) orderings at configuration `lane` ----
        c2 J[2][12];
        // The waves that prepare the next event have one unit: the second is not live while they do.
        auto one_unit = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < 12; ++k) J[1][k] = c2{0.0, 0.0};
        };
        each<12>([&](auto K) __attribute__((always_inline)) { J[0][K] = J[1][K] = c2{0.0, 0.0}; });
        each<2>([&](auto S) __attribute__((always_inline)) {  // ubar W(abcde) v
            if (S == 1 && !both) return;
            const row V = ld_row(T, 16 * (w5::S_C0 + (lane >> 5) + 2 * s4[S]), 4);
            each<12>([&](auto K) __attribute__((always_inline)) {
                J[S][K] = cdot(V, ld_vec(T, tree[S].template at<K>(), 32));
                if constexpr (K % 4 == 3) settle(J[S]);
            });
        });
        arrived(wc);
        __syncthreads();
        here();
        // currents of the line with one gluon on each side, and with one at an end
        words<Q_ENDS> ends = ld_words<Q_ENDS>(cfg[0] + AT_ENDS, 64, lane);
        if (wave < 7) {
            // component strides: end rows 2, one-gluon rows 4
            const int sf = wave == 6 ? 2 : 4, sr = wave == 5 ? 2 : 4;
            const row V = current(ld_row(T, wc.template at<0>(), sf), ld_row(T, wc.template at<1>(), sr));
            st_row(T, wc.template at<2>(), wave < 5 ? 16 : 8, V);
        }
        static_assert(N_N3 > THREADS && N_N3 <= 2 * THREADS && N_X3 == N_N3, "one or two per thread");
        auto tid2 = [&]() __attribute__((always_inline)) { return tid + THREADS < N_N3 ? tid + THREADS : N_N3 - 1; };
        arrived(ends);
        __syncthreads();
        here();
        words<1> wn[2];
        each<2>([&](auto S) __attribute__((always_inline)) {
            if (S == 1 && !both) return;
            words<Q_MID> mid = ld_words<Q_MID>(cfg[S] + AT_MID, 64, lane);
            each<2>([&](auto O) __attribute__((always_inline)) {  // L(a) W(bcde) v
                const row V = ld_row(T, ends.template at<O>(), 8);
                each<6>([&](auto K) __attribute__((always_inline)) {
                    c2& j = J[S][6 * O + K];
                    j = cdot_acc(V, ld_vec(T, ends.template at<2 + 6 * O + K>(), 16), j);
                });
                settle(J[S]);
            });
            each<3>([&](auto Z) __attribute__((always_inline)) {  // ubar W(abcd) R(e)
                const row V = ld_row(T, ends.template at<14 + Z>(), 8);
                each<4>([&](auto OK) __attribute__((always_inline)) {
                    // the orders of the last three that end with their Z-th gluon
                    constexpr int O = OK / 2, K = Z == 0 ? (OK % 2 ? 5 : 3) : Z == 1 ? (OK % 2 ? 4 : 1) : (OK % 2 ? 2 : 0);
                    c2& j = J[S][6 * O + K];
                    j = cdot_acc(V, ld_vec(T, ends.template at<17 + 6 * O + K>(), 16), j);
                });
                settle(J[S]);
            });
            if (S == 0 && both) ends = ld_words<Q_ENDS>(cfg[1] + AT_ENDS, 64, lane);
            each<6>([&](auto OZ) __attribute__((always_inline)) {  // L(a) W(bcd) R(e)
                constexpr int O = OZ / 3, Z = OZ % 3;
                const row V = ld_row(T, mid.template at<3 * O + Z>(), 16);
                each<2>([&](auto H) __attribute__((always_inline)) {
                    constexpr int K = Z == 0 ? (H ? 5 : 3) : Z == 1 ? (H ? 4 : 1) : (H ? 2 : 0);
                    c2& j = J[S][6 * O + K];
                    j = cdot_acc(V, ld_vec(T, mid.template at<6 + 6 * O + K>(), 8), j);
                });
                settle(J[S]);
            });
        });
        fetch(i + gridDim.x, lane);  // used a phase later
        wn[0] = ld_words<1>(tab_N3, N_N3, tid);
        wn[1] = ld_words<1>(tab_N3, N_N3, tid2());
        __syncthreads();
        here();
        // three-gluon rows from p4 without the propagator at the cut
        words<1> rows[2] = {ld_words<1>(cfg[0] + AT_ROWS, 64, lane), ld_words<1>(cfg[1] + AT_ROWS, 64, lane)};
        {
            auto node = [&](const words<1>& w) __attribute__((always_inline)) {
                row f = slash(ld_row(T, w.template at<0>(), 8), ld_vec(T, w.template at<1>(), 2));
                f = add_slash(f, ld_row(T, w.template at<2>(), 4), ld_vec(T, w.template at<3>(), 4));
                f = add_slash(f, ld_row(T, w.template at<4>(), 2), ld_vec(T, w.template at<5>(), 8));
                st_row(T, w.template at<6>(), 16, f);
            };
            node(wn[0]);
            if (tid + THREADS < N_N3) node(wn[1]);
        }
        arrived(rows[0]);
        arrived(rows[1]);
        __syncthreads();
        here();
        words<1> wx[2] = {ld_words<1>(tab_X3, N_X3, tid), ld_words<1>(tab_X3, N_X3, tid2())};
        // A chain of divisions and roots on few lanes: the wave issues it first, or the others wait for
        // it at the barrier (50,021 events 5.31 -> 5.26 ms; any other wave or phase so raised is slower).
        if (ahead) {
            __builtin_amdgcn_s_setprio(2);
            prepare0(T, NEXT, wave - 8, incoming(lane), lane, prm);
            one_unit();
            __builtin_amdgcn_s_setprio(0);
        }
        each<2>([&](auto S) __attribute__((always_inline)) {  // L(ab) [...]
            if (S == 1 && !both) return;
            const auto& w = rows[S];
            const row l0 = ld_row(T, w.template at<0>(), 8), l1 = ld_row(T, w.template at<1>(), 8);
            each<6>([&](auto K) __attribute__((always_inline)) {
                const row r = ld_row(T, w.template at<2 + K>(), 16);
                J[S][K] = wedge(l0, r, J[S][K]);
                J[S][6 + K] = wedge(l1, r, J[S][6 + K]);
                settle(J[S]);
            });
        });
        arrived(wx[0]);
        arrived(wx[1]);
        __syncthreads();
        here();
        // [L(a) W(bc) + ubar W(abc)] R(de)
        words<Q_TWO> two[2] = {ld_words<Q_TWO>(cfg[0] + AT_TWO, 64, lane), ld_words<Q_TWO>(cfg[1] + AT_TWO, 64, lane)};
        {
            auto node = [&](const words<1>& w) __attribute__((always_inline)) {
                row f = slash(ld_row(T, w.template at<0>(), 4), ld_vec(T, w.template at<1>(), 4));
                f = add_slash(f, ld_row(T, w.template at<2>(), 2), ld_vec(T, w.template at<3>(), 8));
                st_row(T, w.template at<4>(), 16, f);
            };
            node(wx[0]);
            if (tid + THREADS < N_N3) node(wx[1]);
        }
        arrived(two[0]);
        arrived(two[1]);
        __syncthreads();
        here();
        if (ahead && wave < 10) {
            __builtin_amdgcn_s_setprio(2);
            prepare1(T, NEXT, wave - 8, lane, prm);
            one_unit();
            __builtin_amdgcn_s_setprio(0);
        }
        each<2>([&](auto S) __attribute__((always_inline)) {
            if (S == 1 && !both) return;
            const auto& w = two[S];
            each<3>([&](auto C) __attribute__((always_inline)) {
                const row x0 = ld_row(T, w.template at<C>(), 16), x1 = ld_row(T, w.template at<3 + C>(), 16);
                each<2>([&](auto H) __attribute__((always_inline)) {
                    constexpr int K = 2 * C + H;
                    const row r = ld_row(T, w.template at<6 + K>(), 8);
                    J[S][K] = wedge(x0, r, J[S][K]);
                    J[S][6 + K] = wedge(x1, r, J[S][6 + K]);
                    settle(J[S]);
                });
            });
        });
        __syncthreads();
        here();
        // ---- colour sum ----
        double q = 0.0;
        double* const DJ = D + 2 * w5::S_J;
        auto exchange = [&](auto&& put) __attribute__((always_inline)) {
            each<2>([&](auto S) __attribute__((always_inline)) {
                if (S == 1 && !both) return;
                const int* fl = tab_flow + 12 * (unit[S] - 10 * s4[S]);
                each<12>([&](auto K) __attribute__((always_inline)) { put(fl[K], s4[S], J[S][K]); });
            });
        };
        if constexpr (CM) {
            for (int h = 0; h < 2; ++h) {
                exchange([&](int f, int s, c2 j) __attribute__((always_inline)) {
                    if (s != h) return;
                    DJ[(2 * f) * 64 + lane] = j.r;
                    DJ[(2 * f + 1) * 64 + lane] = j.i;
                });
                __syncthreads();
                if (wave < 4) {
                    const double s = colour_mfma_group_sum(
                        colour_mfma16<P::ncol>(DJ, 16 * wave, colour_table<P>::mfma_frag(), lane));
                    const int s3 = wave >> 1;  // of the columns 16 wave .. + 15
                    if (lane < 16 && ((spins >> (s3 + 2 * h)) & 1)) q += s;
                }
                __syncthreads();
            }
        } else {
            // wave w: share w % 6 of the configurations with spin w / 6 of tbar
            const int g = wave % 6, h4 = wave / 6;
            double* const Dl = DJ + 64 * h4 + lane;
            each<2>([&](auto PART) __attribute__((always_inline)) {
                exchange([&](int f, int s, c2 j) __attribute__((always_inline)) {
                    DJ[128 * f + 64 * s + lane] = PART ? j.i : j.r;
                });
                __syncthreads();
                each<6>([&](auto W) __attribute__((always_inline)) {
                    if (g == W) colour_orbits<W>(Dl);
                });
                __syncthreads();
                each<6>([&](auto W) __attribute__((always_inline)) {
                    if (g == W) q += colour_quads<W>(Dl);
                });
                if constexpr (PART == 0) __syncthreads();
            });
            q = ((spins >> ((lane >> 5) + 2 * h4)) & 1) ? q : 0.0;
        }
        const double tot = wave_sum(q);
        if (lane == 63) part[wave] = tot;
        done = i;
    }
    __syncthreads();
    if (wave == 11 && done >= 0) finish(done, lane);
}

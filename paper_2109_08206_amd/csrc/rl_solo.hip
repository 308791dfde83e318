// BBPGD in one workgroup: the whole solve of a small problem (start phases,
// every iteration, the stop) in one launch.
//
// Up to a few thousand constraints the two-kernel loop is bound by its
// launches: about 8 us per iteration whatever the size (k_rod 4.2 and k_con
// 3.5 us in a trace of 460 constraints, and the gaps).  One workgroup keeps
// the iterate in registers (thread t owns constraints t, t + T, ...: gamma,
// g, q) and exchanges the two directions of the product through LDS: the
// owners write gamma', the rods sum their records, apply the mobility and
// write the contact velocities of their records, and the owners read w back.
// Three workgroup barriers per iteration (two around the rods' turn, one for
// the dot products), no launch, and nothing written to memory before the end.
//
// What bounds it: the instruction issue of one compute unit and the dependent
// chain between the barriers, not memory.  Hence few waves (every wave runs
// the reduction and the step rule itself: at 1,024 threads these took 3,400
// clocks of an iteration, whatever the size), the records of a rod in its
// thread's registers, and the rods dealt to the threads in descending order
// of their number of records (a wave takes as long as its longest list, and a
// random 64 rods nearly always hold one two or three times the average).
//
// Per iteration (solve_lcp, everything before and after the loop included as
// one fixed part): 452 constraints on 400 rods 8.0 -> 1.8 us, 1,280 on 1,000
// 7.7 -> 2.7 us, 1,876 on 1,200 (the four-rods-a-thread form) 8.0 -> 5.6 us.
// Beyond 3,000 constraints or 2,048 rods one compute unit is no faster than
// the two kernels (3,100 constraints streamed from the caches: 13 us).
#include <algorithm>
#include <cmath>

#include "rl_device.hpp"

namespace rl {

// Sums of four numbers over a workgroup of NW waves, the same bits in every
// thread.  Two exchanges inside each quad leave lane i with the quad's sum of
// number i, two rotations add the quads of a row, and the row sums (red[i]
// holds 4 NW of them for number i) meet in LDS.  red is double-buffered by
// the caller, so one barrier suffices.
template <int NW>
__device__ __forceinline__ void solo_sum4(double p[4], double (*red)[4 * NW])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const bool b0 = lane & 1, b1 = lane & 2;
    const double a = (b0 ? p[1] : p[0]) + dpp_f64<0xb1>(b0 ? p[0] : p[1]);
    const double b = (b0 ? p[3] : p[2]) + dpp_f64<0xb1>(b0 ? p[2] : p[3]);
    double c = (b1 ? b : a) + dpp_f64<0x4e>(b1 ? a : b);
    c += dpp_f64<0x124>(c);  // row_ror:4
    c += dpp_f64<0x128>(c);  // row_ror:8
    if ((lane & 12) == 0) red[lane & 3][4 * wave + (lane >> 4)] = c;
    __syncthreads();
    // every row of lanes: lane 4 g + i sums NW row sums of number i
    const double2 *s = reinterpret_cast<const double2 *>(&red[lane & 3][NW * ((lane >> 2) & 3)]);
    double v = 0.0;
#pragma unroll
    for (int k = 0; k < NW / 2; ++k) {
        const double2 x = s[k];
        v += x.x + x.y;
    }
    v += dpp_f64<0x124>(v);
    v += dpp_f64<0x128>(v);
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i] = lane_f64(v, i);
}

// largest value over the workgroup (only where a stop reports its residual)
template <int NW>
__device__ __forceinline__ double solo_max(double v, double *red)
{
    v = wave_total<true>(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    for (int w = 0; w < NW; ++w) v = fmax(v, red[w]);
    return v;
}

// A lane's share of one rod: records sub, sub + ln, ... of its P list
// followed by its Q list.  The first R are held: the arclength s, the
// constraint c, and with HELD the normal, its sign turned on the Q side so
// that both sides add.  Longer lists look the rest up.
template <int R, bool HELD>
struct SoloRod {
    int rod, pb, np, qb, cnt;
    int wmax;  // longest list of the wave, at most R
    double d[3], s[R], e[HELD ? R : 1][3];
    int c[R];
};

struct SoloLds {
    const double *ex, *ey, *ez;  // the normals
    const double *sP, *sQ;       // with HELD: arclengths in P order and Q-list order
    const unsigned short *qi;    // with HELD: the Q lists
    const double *G;             // what the product takes
    double *U;                   // u of the P side, then -u of the Q side, NC slots each
};

// record t of a rod's list: its constraint, its arclength, its side
template <int R, bool HELD>
__device__ __forceinline__ bool solo_record(const SolveArgs &a, const SoloLds &l, const SoloRod<R, HELD> &r, int t,
                                            int &c, double &s)
{
    const bool pside = t < r.np;
    const int k = pside ? r.pb + t : r.qb + t - r.np;
    if (HELD) {
        c = pside ? k : (int)l.qi[k];
        s = (pside ? l.sP : l.sQ)[k];
    } else {
        c = pside ? k : a.qidx[k];
        s = (pside ? a.geo : a.qgeo)[4 * (int64_t)k + 3];
    }
    return pside;
}

template <int NC, int R, bool HELD>
__device__ __forceinline__ void solo_rod_setup(const SolveArgs &a, const SoloLds &l, int rod, int sub, int ln,
                                               SoloRod<R, HELD> &r)
{
    r.rod = rod < 0 ? 0 : rod;
    r.pb = r.np = r.qb = r.cnt = 0;
    r.d[0] = r.d[1] = r.d[2] = 0.0;
    if (rod >= 0) {
        r.pb = a.pptr[rod];
        r.np = a.pptr[rod + 1] - r.pb;
        r.qb = a.qptr[rod];
        const int tot = r.np + a.qptr[rod + 1] - r.qb;
        r.cnt = tot > sub ? (tot - sub + ln - 1) / ln : 0;
        for (int d = 0; d < 3; ++d) r.d[d] = a.dir[3 * rod + d];
    }
#pragma unroll
    for (int i = 0; i < R; ++i) {
        r.c[i] = NC - 1;  // past the list: the zero slot
        r.s[i] = 0.0;
        bool pside = true;
        if (i < r.cnt) pside = solo_record(a, l, r, sub + i * ln, r.c[i], r.s[i]);
        if (HELD) {
            const double e[3] = {l.ex[r.c[i]], l.ey[r.c[i]], l.ez[r.c[i]]};
            for (int d = 0; d < 3; ++d) r.e[i][d] = pside ? e[d] : -e[d];
        }
    }
    int m = min(r.cnt, R);
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) m = max(m, __shfl_xor(m, o, 64));
    r.wmax = __builtin_amdgcn_readfirstlane(m);
}

// G of the held records, all in flight before the first is used
template <int R, bool HELD>
__device__ __forceinline__ void solo_rod_load(const SoloLds &l, const SoloRod<R, HELD> &r, double gv[R])
{
#pragma unroll
    for (int i = 0; i < R; ++i) gv[i] = i < r.wmax ? l.G[r.c[i]] : 0.0;
}

// D v summed over the rod's records, the mobility, and u of every record
template <int NC, int R, bool HELD>
__device__ __forceinline__ void solo_rod(const SolveArgs &a, const SoloLds &l, int sub, int ln,
                                         const SoloRod<R, HELD> &r, const double gv[R])
{
    if (r.wmax == 0) return;  // none in the wave
    double f[3] = {0.0, 0.0, 0.0}, m[3] = {0.0, 0.0, 0.0};
    auto add = [&](double v, double s, const double e[3]) {
        const double vs = v * s;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            f[d] += v * e[d];
            m[d] += vs * e[d];
        }
    };
    auto normal = [&](int c, bool pside, double e[3]) {
        e[0] = l.ex[c];
        e[1] = l.ey[c];
        e[2] = l.ez[c];
        for (int d = 0; d < 3; ++d) e[d] = pside ? e[d] : -e[d];
    };
    // records past the held ones, looked up kTail at a time
    constexpr int kTail = 4;
    auto tail = [&](int i, auto &&use) {
        int c[kTail];
        double s[kTail];
        bool pside[kTail];
#pragma unroll
        for (int k = 0; k < kTail; ++k)
            pside[k] = solo_record(a, l, r, sub + min(i + k, r.cnt - 1) * ln, c[k], s[k]);
#pragma unroll
        for (int k = 0; k < kTail; ++k)
            if (i + k < r.cnt) use(c[k], pside[k], s[k]);
    };
    double apar, aperp, rperp;
    rod_mob(a, r.rod, a.coef == nullptr, apar, aperp, rperp);
#pragma unroll
    for (int i = 0; i < R; ++i)
        if (i < r.wmax) {
            if (HELD) {
                add(gv[i], r.s[i], r.e[i]);
            } else {
                double e[3];
                normal(r.c[i], sub + i * ln < r.np, e);
                add(gv[i], r.s[i], e);
            }
        }
    for (int i = R; i < r.cnt; i += kTail)
        tail(i, [&](int c, bool pside, double s) {
            double e[3];
            normal(c, pside, e);
            add(l.G[c], s, e);
        });
    if (ln >= 2) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            f[d] += dpp_f64<0xb1>(f[d]);
            m[d] += dpp_f64<0xb1>(m[d]);
        }
    }
    if (ln >= 4) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            f[d] += dpp_f64<0x4e>(f[d]);
            m[d] += dpp_f64<0x4e>(m[d]);
        }
    }
    const double fd = (apar - aperp) * (r.d[0] * f[0] + r.d[1] * f[1] + r.d[2] * f[2]);
    const double md = r.d[0] * m[0] + r.d[1] * m[1] + r.d[2] * m[2];
    double V[3], W[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        V[d] = aperp * f[d] + fd * r.d[d];
        W[d] = rperp * (m[d] - md * r.d[d]);
    }
    auto along = [&](double s, const double e[3]) {
        return e[0] * (V[0] + s * W[0]) + e[1] * (V[1] + s * W[1]) + e[2] * (V[2] + s * W[2]);
    };
    // the normals come from LDS again: kept from the sums they would spill
    if (!HELD) __asm__ volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < R; ++i)
        if (i < r.wmax) {
            // past the list: +-0 on the P side of the zero slot, which nobody reads
            const bool pside = sub + i * ln < r.np || i >= r.cnt;
            double e[3];
            if (!HELD) normal(r.c[i], pside, e);
            l.U[pside ? r.c[i] : NC + r.c[i]] = along(r.s[i], HELD ? r.e[i] : e);
        }
    for (int i = R; i < r.cnt; i += kTail)
        tail(i, [&](int c, bool pside, double s) {
            double e[3];
            normal(c, pside, e);
            l.U[pside ? c : NC + c] = along(s, e);
        });
}

// T threads; NC constraint slots, the last one a zero that no constraint
// takes; J = NC / T constraints per thread; K rods per thread (2 or 4); HELD:
// the rods hold the normals of their records in registers; BIL: general set.  ln: lanes per
// rod.  The launch runs iterations k0 .. kend - 1 at most (k0 = 0: the start
// phases first); a stop is latched in the state, else the iterate and the
// step length are left for the next launch.
template <int T, int NC, int K, bool HELD, bool BIL>
__global__ void __launch_bounds__(T) k_solo(SolveArgs a, int ln, long long k0, long long kend)
{
    constexpr int NW = T / 64, J = NC / T, kBins = 64;
    static_assert(NC % T == 0 && (K == 2 || K == 4), "");
    __shared__ double E[3][NC], G[NC], U[2 * NC];
    __shared__ double sP[HELD ? NC : 1], sQ[HELD ? NC : 1];
    __shared__ unsigned short qi[HELD ? NC : 1];
    __shared__ __align__(16) double red[2][4][4 * NW];
    const int tid = threadIdx.x;
    const int n = (int)a.n, nc = (int)a.nc;
    SolverState *S = a.state;
    if (k0 > 0 && S->done) return;
    const SoloLds l{E[0], E[1], E[2], sP, sQ, qi, G, U};
    const int lsh = ln == 4 ? 2 : (ln == 2 ? 1 : 0), sub = tid & (ln - 1);

    double gam[J], g[J], q[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int c = tid + j * T;
        const bool ok = c < nc;
        gam[j] = g[j] = q[j] = 0.0;
        if (ok) {
            const double2 s = a.st[c];
            gam[j] = s.x;
            g[j] = s.y;
            q[j] = a.qv[c];
        }
        const double2 *gd = reinterpret_cast<const double2 *>(a.geo + 4 * (int64_t)(ok ? c : 0));
        const double2 g0 = gd[0], g1 = gd[1];
        E[0][c] = ok ? g0.x : 0.0;
        E[1][c] = ok ? g0.y : 0.0;
        E[2][c] = ok ? g1.x : 0.0;
        if (HELD) {
            sP[c] = ok ? g1.y : 0.0;
            if (c < a.qptr[n]) {
                sQ[c] = a.qgeo[4 * (int64_t)c + 3];
                qi[c] = (unsigned short)a.qidx[c];
            }
        }
        G[c] = 0.0;
    }
    // the rods in descending order of their number of records: slot t of the
    // order goes to lanes ln t ... of the workgroup (which rod a thread holds
    // does not enter any sum).  Later slots hold shorter lists.
    constexpr int R1 = HELD ? 9 : 8, R2 = HELD ? 3 : 4, R3 = 3, R4 = 2;
    SoloRod<R1, HELD> rod1;
    SoloRod<R2, HELD> rod2;
    SoloRod<R3, HELD> rod3;
    SoloRod<R4, HELD> rod4;
    {
        int *hist = reinterpret_cast<int *>(&red[0][0][0]);  // [kBins]
        int *ord = reinterpret_cast<int *>(U);               // [n], n <= K T <= 4 NC
        static_assert(K * T <= 4 * NC, "");
        if (tid < kBins) hist[tid] = 0;
        __syncthreads();
        int key[K], slot[K];
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const int r = tid + i * T;
            if (r < n) {
                key[i] = kBins - 1 - min(a.pptr[r + 1] - a.pptr[r] + a.qptr[r + 1] - a.qptr[r], kBins - 1);
                slot[i] = atomicAdd(&hist[key[i]], 1);
            }
        }
        __syncthreads();
        if (tid < 64) {
            const int v = hist[tid];
            int incl = v;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int t = __shfl_up(incl, d, 64);
                if (tid >= d) incl += t;
            }
            hist[tid] = incl - v;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const int r = tid + i * T;
            if (r < n) ord[hist[key[i]] + slot[i]] = r;
        }
        __syncthreads();
        const int t = tid >> lsh, st = T >> lsh;
        solo_rod_setup<NC>(a, l, t < n ? ord[t] : -1, sub, ln, rod1);
        // every other slot backwards, so that no wave has the longest of all
        const int t2 = 2 * st - 1 - t, t3 = 2 * st + t, t4 = 4 * st - 1 - t;
        solo_rod_setup<NC>(a, l, t2 < n ? ord[t2] : -1, sub, ln, rod2);
        if (K == 4) {
            solo_rod_setup<NC>(a, l, t3 < n ? ord[t3] : -1, sub, ln, rod3);
            solo_rod_setup<NC>(a, l, t4 < n ? ord[t4] : -1, sub, ln, rod4);
        }
        __syncthreads();
        // a constraint without a Q side keeps u_Q = 0
#pragma unroll
        for (int j = 0; j < J; ++j) U[NC + tid + j * T] = 0.0;
    }
    // the rods' turn: G holds v, U receives the two halves of D^T M D v
    auto turn = [&]() {
        __syncthreads();
        double g1[R1], g2[R2];
        solo_rod_load(l, rod1, g1);
        solo_rod_load(l, rod2, g2);
        solo_rod<NC>(a, l, sub, ln, rod1, g1);
        solo_rod<NC>(a, l, sub, ln, rod2, g2);
        if (K == 4) {
            double g3[R3], g4[R4];
            solo_rod_load(l, rod3, g3);
            solo_rod_load(l, rod4, g4);
            solo_rod<NC>(a, l, sub, ln, rod3, g3);
            solo_rod<NC>(a, l, sub, ln, rod4, g4);
        }
        __syncthreads();
    };
    auto cmp_of = [&](int c) { return BIL ? a.cmpv[c] : -1.0; };

    const double tol = S->tol;
    const long long max_iter = S->max_iter;
    double alpha = 0.0, alpha0 = 0.0, amin = 0.0, amax = 0.0;
    double p[4], res = 0.0;
    int status = RL_OK;
    bool done = false;
    long long iter = 0;
    if (k0 == 0) {
        // g0 = Mc gamma0 + q on the projected start
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int c = tid + j * T;
            if (c < nc) {
                if (!(BIL && cmp_of(c) >= 0.0)) gam[j] = gamma_prime<kModeInit>(gam[j], 0.0, 0.0);
                G[c] = gam[j];
            }
        }
        turn();
        p[0] = p[1] = p[2] = p[3] = 0.0;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int c = tid + j * T;
            if (c < nc) {
                const double cm = cmp_of(c);
                const bool bil = BIL && cm >= 0.0;
                g[j] = (U[c] + U[NC + c]) + (q[j] + (bil ? cm * gam[j] : 0.0));
                p[2] += g[j] * g[j];
                p[3] = fmax(p[3], fabs(!bil && gam[j] < g[j] ? gam[j] : g[j]));
            }
        }
        res = solo_max<NW>(p[3], &red[1][0][0]);
        solo_sum4<NW>(p, red[0]);
        if (!isfinite(p[2]) || !isfinite(res)) {
            status = RL_ERR_NONFINITE;
            done = true;
        } else if (res <= tol) {
            done = true;
        }
        if (!done) {
            // the Cauchy step on the projected gradient
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const int c = tid + j * T;
                if (c < nc) G[c] = BIL && cmp_of(c) >= 0.0 ? g[j] : gamma_prime<kModeAlpha0>(gam[j], g[j], 0.0);
            }
            turn();
            p[0] = p[1] = p[2] = p[3] = 0.0;
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const int c = tid + j * T;
                if (c < nc) {
                    const double cm = cmp_of(c);
                    const bool bil = BIL && cm >= 0.0;
                    const double gh = bil ? g[j] : gamma_prime<kModeAlpha0>(gam[j], g[j], 0.0);
                    p[0] += gh * gh;
                    p[1] += gh * ((U[c] + U[NC + c]) + (bil ? cm * gh : 0.0));
                }
            }
            solo_sum4<NW>(p, red[1]);
            if (!isfinite(p[0]) || !isfinite(p[1])) {
                status = RL_ERR_NONFINITE;
                done = true;
            } else if (p[0] == 0.0) {
                done = true;
            } else {
                alpha0 = p[1] > 0.0 ? p[0] / p[1] : 1.0;
                alpha = alpha0;
                amin = 1e-12 * alpha0;
                amax = 1e12 * alpha0;
                if (max_iter <= 0) {
                    status = RL_NOT_CONVERGED;
                    done = true;
                }
            }
        }
    } else {
        alpha = S->alpha;
        alpha0 = S->alpha0;
        amin = S->amin;
        amax = S->amax;
    }
    // the same in every thread: scalar registers
    alpha = lane_f64(alpha, 0);
    amin = lane_f64(amin, 0);
    amax = lane_f64(amax, 0);
    for (long long k = k0; !done && k < kend; ++k) {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int c = tid + j * T;
            if (c < nc)
                G[c] = BIL && cmp_of(c) >= 0.0 ? gamma_free<kModeLoop>(gam[j], g[j], alpha)
                                               : gamma_prime<kModeLoop>(gam[j], g[j], alpha);
        }
        turn();
        // (s.s, s.y, y.y, constraints above the tolerance)
        p[0] = p[1] = p[2] = p[3] = 0.0;
        double rmax = 0.0;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int c = tid + j * T;
            if (c < nc) {
                const double cm = cmp_of(c);
                const bool bil = BIL && cm >= 0.0;
                // gamma' again (cheaper than registers held across the rods' turn)
                const double v = bil ? gamma_free<kModeLoop>(gam[j], g[j], alpha)
                                     : gamma_prime<kModeLoop>(gam[j], g[j], alpha);
                const double gn = (U[c] + U[NC + c]) + (q[j] + (bil ? cm * v : 0.0));
                const double sc = v - gam[j], yc = gn - g[j];
                p[0] += sc * sc;
                p[1] += sc * yc;
                p[2] += yc * yc;
                rmax = fmax(rmax, fabs(!bil && v < gn ? v : gn));
                gam[j] = v;
                g[j] = gn;
            }
        }
        p[3] = rmax > tol ? 1.0 : 0.0;
        solo_sum4<NW>(p, red[k & 1]);
        // the step rule's residual only has to be on the right side of the
        // tolerance here; the stop takes the true one below
        const double t[4] = {p[0], p[1], p[2], p[3] > 0.0 ? 2.0 * tol + 1.0 : 0.0};
        const Decision d = decide_from(DecideIn{tol, amin, amax, alpha, max_iter}, k + 1, t);
        done = d.stop;
        status = d.status;
        alpha = lane_f64(d.alpha, 0);
        if (done) {
            iter = k + 1;
            res = solo_max<NW>(rmax, &red[(k + 1) & 1][0][0]);
            if (status != RL_ERR_NONFINITE && !isfinite(res)) status = RL_ERR_NONFINITE;
        }
    }
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int c = tid + j * T;
        if (c < nc) {
            const double2 s = make_double2(gam[j], g[j]);
            a.st[c] = s;
            const int k = a.qpos[c];
            if (!BIL || k >= 0) a.stq[k] = s;
        }
    }
    if (tid == 0) {
        S->alpha = alpha;
        S->alpha0 = alpha0;
        S->amin = amin;
        S->amax = amax;
        S->res = res;
        S->iter = iter;
        S->status = status;
        S->done = done ? 1 : 0;
    }
}

template <int T, int NC, int K, bool HELD>
static void launch_solo_t(hipStream_t st, const SolveArgs &a, long long k0, long long kend)
{
    // several lanes per rod while that leaves one rod per thread (at most K
    // are there to take), or while the lists are long
    int ln = 1;
    while (ln < 4 && (2 * ln * a.n <= T || (2 * ln * a.n <= K * T && 2 * a.nc > 6 * ln * a.n))) ln *= 2;
    if (a.gen)
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_solo<T, NC, K, HELD, true>), dim3(1), dim3(T), 0, st, a, ln, k0, kend);
    else
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_solo<T, NC, K, HELD, false>), dim3(1), dim3(T), 0, st, a, ln, k0, kend);
}

bool solo_takes(int64_t n, int64_t nc) { return n <= 2048 && nc < kSoloSlots; }

hipError_t launch_solo(hipStream_t st, const SolveArgs &a, long long k0, long long kend)
{
    if (a.n <= 512 && a.nc < 1024) launch_solo_t<256, 1024, 2, true>(st, a, k0, kend);
    else if (a.n <= 1024 && a.nc < 2048) launch_solo_t<512, 2048, 2, true>(st, a, k0, kend);
    else launch_solo_t<512, kSoloSlots, 4, false>(st, a, k0, kend);
    return hipGetLastError();
}

}  // namespace rl

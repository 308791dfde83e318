// BBPGD with the whole problem on chip: one launch runs the start phases,
// every iteration and the stop, in one workgroup (small problems) or in up to
// one per compute unit that exchange what crosses between them.
//
// The two-kernel loop costs about 8 us per iteration in launches whatever the
// size, and beyond that streams 188 bytes per constraint and iteration.  Here
// a workgroup owns a contiguous range of rods and keeps, for the whole solve,
// the iterate of its constraints in registers (thread t: slots t, t + T, ...:
// gamma, g, q) and the records of its rods in its threads' registers and LDS.
// Nothing is read from or written to memory per iteration but the exchange.
//
// One product: the slots' gamma' goes to LDS, the rods sum their records,
// apply the mobility and leave the contact velocities of their records in
// LDS, and the slots read w = u_P - u_Q back (three workgroup barriers per
// iteration with the one of the dot products).
//
// Across workgroups: a constraint belongs to the workgroup of its P rod.  One
// whose Q rod lives elsewhere has a second slot there that follows the same
// iterate bit for bit, so only the two contact velocities travel, and then
// the four sums of every workgroup, which all of them add in the same order.
// Both exchanges are 64-bit words of 32 data bits and a 32-bit sequence
// number, written and polled with relaxed device-scope accesses: a word is
// its own flag, so there is no barrier, no fence (an L2 write-back on this
// part) and no clearing between iterations.  A workgroup sends its sums after
// it has read the velocities of the same product and writes the next
// velocities after it has read everybody's sums, so no word is overwritten
// unread; the sums alternate between two buffers for the same reason.  Every
// wait is bounded: past the bound (or where the problem turns out not to fit)
// all workgroups leave without a result, and the caller runs the two kernels.
// (A grid barrier with device-scope fences took 17 us and more.)
//
// What bounds it: the exchanges, and the instruction issue of a compute unit
// and the dependent chain between the barriers, not memory.  Hence few waves
// (every wave runs the reduction and the step rule itself: at 1,024 threads
// these took 3,400 clocks of an iteration whatever the size), and rods dealt
// to the threads in descending order of their number of records (a wave takes
// as long as its longest list, and a random 64 rods nearly always hold one
// two or three times the average).  Where an iteration of a whole step goes, us,
// by a clock in one wave of each workgroup (mean over the workgroups; the
// waits hold the others' delay as well):
//   rods, constraints, workgroups   gamma'  rods  velocities  sums inside, between
//     2,000    3,108   13   4.0      0.5    0.6      1.2         0.3   1.5
//    10,000   31,026   64   5.0      0.5    0.7      1.6         0.2   1.9
//    20,000   62,479  128   5.3      0.5    0.7      1.7         0.2   2.2
//    50,000  155,397  256   6.7      0.5    0.7      2.4         0.3   2.9
//   100,000  311,923  256  10.7      0.5    2.8      4.2         0.3   2.9
//   100,000  470,657  256  15.3      0.6    6.0      4.2         0.8   3.8
#include <algorithm>
#include <climits>
#include <cmath>

#include "rl_device.hpp"

namespace rl {

typedef unsigned long long u64;

// Where the workgroups of one solve meet.  Words carry (data << 32 | number).
struct Exchange {
    u64 *u;         // [2][workgroups][NC] low and high halves of the velocities a workgroup
                    // sends, in its own order (consecutive lanes, consecutive words)
    u64 *at;        // [nc][2] where in it u_P and -u_Q of a constraint are found
    u64 *tot;       // [2][2][kResMost][kSlot] the four sums, by parity of the number: of
                    // the workgroups, and of the groups of kTeam workgroups; behind it
                    // [kResMost] the number at which a workgroup left its results
    unsigned base;  // numbers base + 1, ... belong to this launch
    int *fail;      // set when a wait ran out (1) or the problem does not fit (2)
    unsigned until;  // waits for numbers above it run out at the first poll
};

constexpr int kSlot = 32;      // words from one workgroup's sums to the next (256 bytes)
constexpr int kLeft = 4 * kResMost * kSlot;
// iterations of one launch of a solve (8 ms at 4 us each, 31 ms at the 15 of
// 100,000 rods and 469,000 constraints, more with long lists), and the numbers
// that its exchanges may take
constexpr long long kResChunk = 2048, kResNumbers = kResChunk + 8;
// Above 128 workgroups their sums meet in two steps, teams of 16 and then the
// teams.  Up to 128 a thread of each workgroup polls one word pair of the
// others' sums, with 256 two after each other.  Whole iterations flat and in
// two steps: 128 workgroups 5.2 and 5.6 us (16,000 rods, 49,000 constraints),
// 5.5 and 5.9 (20,000, 62,000), 6.5 and 7.1 (30,000 nematic, 57,000), 6.0 and
// 6.7 (40,000, 62,000); 256 workgroups 6.75 and 6.9 (40,000, 124,000), 6.8 and
// 6.4 (50,000, 155,000), 10.2 and 10.4 (100,000, 312,000), 14.9 and 15.2
// (100,000 nematic, 471,000): no difference in the mean.
constexpr int kTeam = 16, kFlat = 128;

// polls of one word before the wait is given up (about 0.3 s)
constexpr int kSpin = 1 << 18;

__device__ __forceinline__ void word_put(u64 *p, u64 v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ u64 word_get(const u64 *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ u64 half_word(int half, unsigned num) { return ((u64)(unsigned)half << 32) | num; }

__device__ __forceinline__ void pair_put(u64 *p, double v, unsigned num)
{
    word_put(p, half_word(__double2loint(v), num));
    word_put(p + 1, half_word(__double2hiint(v), num));
}

__device__ __forceinline__ double pair_value(u64 lo, u64 hi)
{
    return __hiloint2double((int)(hi >> 32), (int)(lo >> 32));
}

// whether poll number `spin` was one too many, or somebody else gave up
__device__ __forceinline__ bool give_up(int spin, int *fail, int *bad)
{
    if (spin < kSpin && ((spin & 1023) != 1023 ||
                         __hip_atomic_load(fail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0))
        return false;
    __hip_atomic_store(fail, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *bad = 1;
    return true;
}

// the count of polls of a wait for number `num` before the first
__device__ __forceinline__ int spent(const Exchange &x, unsigned num) { return num > x.until ? kSpin : 0; }

// the two words of a number, polled until both carry `num`
__device__ __forceinline__ double pair_wait(const u64 *p, const Exchange &x, unsigned num, int *bad)
{
    for (int spin = spent(x, num);; ++spin) {
        const u64 lo = word_get(p), hi = word_get(p + 1);
        if (((unsigned)lo == num && (unsigned)hi == num) || give_up(spin, x.fail, bad)) return pair_value(lo, hi);
    }
}

// The second half of it: lane l of every wave holds a part of number l & 3.
template <int NW>
__device__ __forceinline__ void res_sum4_lanes(double c, double p[4], double (*red)[4 * NW])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
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

// Sums of four numbers over a workgroup of NW waves, the same bits in every
// thread.  Two exchanges inside each quad leave lane i with the quad's sum of
// number i, two rotations add the quads of a row, and the row sums (red[i]
// holds 4 NW of them for number i) meet in LDS.  One barrier: the caller has
// another one, or another red, between two of these.
template <int NW>
__device__ __forceinline__ void res_sum4(double p[4], double (*red)[4 * NW])
{
    const int lane = threadIdx.x & 63;
    const bool b0 = lane & 1, b1 = lane & 2;
    const double a = (b0 ? p[1] : p[0]) + dpp_f64<0xb1>(b0 ? p[0] : p[1]);
    const double b = (b0 ? p[3] : p[2]) + dpp_f64<0xb1>(b0 ? p[2] : p[3]);
    double c = (b1 ? b : a) + dpp_f64<0x4e>(b1 ? a : b);
    res_sum4_lanes<NW>(c, p, red);
}

// largest value over the workgroup (only where a stop reports its residual)
template <int NW>
__device__ __forceinline__ double res_max(double v, double *red)
{
    v = wave_total<true>(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    for (int w = 0; w < NW; ++w) v = fmax(v, red[w]);
    return v;
}

// A lane's share of one rod: records sub, sub + ln, ... of its P list
// followed by its Q list.  The first R are held: the arclength s, the slot,
// and with HELD the normal, its sign turned on the Q side so that both sides
// add.  Longer lists look the rest up.
template <int R, bool HELD>
struct ResRod {
    int rod, pb, np, qb, cnt;
    int wmax;  // longest list of the wave, at most R
    double d[3], s[R], e[HELD ? R : 1][3], mob[HELD ? 3 : 1];
    int c[R];
};

constexpr int kGroup = 4;  // records handled together; R is a multiple

struct ResLds {
    const double *ex, *ey, *ez;    // the normals by slot
    const double *sP, *sQ;         // with HELD: arclengths by slot (P side) and Q-list position
    const unsigned short *qslot;   // slots of the Q lists
    const double *G;               // what the product takes, by slot
    double *U;                     // u of the P side, then -u of the Q side, NC each, by slot
    int c0, q0;                    // the workgroup's first constraint and Q-list position
};

// record t of a rod's list: slot, arclength and side
template <int R, bool HELD>
__device__ __forceinline__ bool res_record(const SolveArgs &a, const ResLds &l, const ResRod<R, HELD> &r, int t,
                                           int &c, double &s)
{
    const bool pside = t < r.np;
    const int k = pside ? r.pb + t : r.qb + t - r.np;
    c = pside ? k - l.c0 : (int)l.qslot[k - l.q0];
    if (HELD) s = pside ? l.sP[k - l.c0] : l.sQ[k - l.q0];
    else s = (pside ? a.geo : a.qgeo)[4 * (int64_t)k + 3];
    return pside;
}

template <int NC, int R, bool HELD>
__device__ __forceinline__ void res_rod_setup(const SolveArgs &a, const ResLds &l, int rod, int sub, int ln,
                                              ResRod<R, HELD> &r)
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
        for (int d = 0; d < 3; ++d) r.d[d] = a.dir[3 * (int64_t)rod + d];
    }
    if (HELD) rod_mob(a, r.rod, a.coef == nullptr, r.mob[0], r.mob[HELD ? 1 : 0], r.mob[HELD ? 2 : 0]);
#pragma unroll
    for (int i = 0; i < R; ++i) {
        r.c[i] = NC - 1;  // past the list: the zero slot
        r.s[i] = 0.0;
        bool pside = true;
        if (i < r.cnt) pside = res_record(a, l, r, sub + i * ln, r.c[i], r.s[i]);
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

// D v summed over the rod's records, the mobility, and u of every record
template <int NC, int R, bool HELD>
__device__ __forceinline__ void res_rod(const SolveArgs &a, const ResLds &l, int sub, int ln,
                                        const ResRod<R, HELD> &r)
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
            pside[k] = res_record(a, l, r, sub + min(i + k, r.cnt - 1) * ln, c[k], s[k]);
#pragma unroll
        for (int k = 0; k < kTail; ++k)
            if (i + k < r.cnt) use(c[k], pside[k], s[k]);
    };
    double apar = r.mob[0], aperp = r.mob[HELD ? 1 : 0], rperp = r.mob[HELD ? 2 : 0];
    if (!HELD) rod_mob(a, r.rod, a.coef == nullptr, apar, aperp, rperp);
    // kGroup records at a time without a branch between them: their loads go
    // out together and their chains overlap (past the list: the zero slot)
#pragma unroll
    for (int b = 0; b < R; b += kGroup)
        if (b < r.wmax) {
            double gv[kGroup], e[kGroup][3];
#pragma unroll
            for (int i = 0; i < kGroup; ++i) {
                gv[i] = l.G[r.c[b + i]];
                if (!HELD) normal(r.c[b + i], sub + (b + i) * ln < r.np, e[i]);
            }
#pragma unroll
            for (int i = 0; i < kGroup; ++i) add(gv[i], r.s[b + i], HELD ? r.e[b + i] : e[i]);
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
    for (int b = 0; b < R; b += kGroup)
        if (b < r.wmax) {
            double e[kGroup][3];
            int at[kGroup];
#pragma unroll
            for (int i = 0; i < kGroup; ++i) {
                // past the list: +-0 on the P side of the zero slot, which nobody reads
                const int k = b + i;
                const bool pside = sub + k * ln < r.np || k >= r.cnt;
                at[i] = pside ? r.c[k] : NC + r.c[k];
                if (!HELD) normal(r.c[k], pside, e[i]);
            }
#pragma unroll
            for (int i = 0; i < kGroup; ++i) l.U[at[i]] = along(r.s[b + i], HELD ? r.e[b + i] : e[i]);
        }
    for (int i = R; i < r.cnt; i += kTail)
        tail(i, [&](int c, bool pside, double s) {
            double e[3];
            normal(c, pside, e);
            l.U[pside ? c : NC + c] = along(s, e);
        });
}

// First rod r with pptr[r] + qptr[r] + 2 r >= target (W(0) = 0, W(n) the
// total), by a wave: 64 probes a round.
__device__ __forceinline__ int res_boundary(const SolveArgs &a, int n, int64_t target)
{
    const int lane = threadIdx.x & 63;
    int lo = 0, hi = n;  // W(hi) >= target; everything before lo is below it
    while (lo < hi) {
        const int step = (hi - lo + 63) / 64;
        const int r = min(lo + lane * step, hi);
        const bool ge = (int64_t)a.pptr[r] + a.qptr[r] + 2 * (int64_t)r >= target;
        const unsigned long long m = __ballot(ge);
        if (m == 0) {
            lo = min(lo + 63 * step + 1, hi);
            continue;
        }
        const int f = __ffsll(m) - 1;
        const int rf = min(lo + f * step, hi);
        lo = f == 0 ? lo : lo + (f - 1) * step + 1;
        hi = rf;
        if (f == 0) lo = hi;
    }
    return __builtin_amdgcn_readfirstlane(lo);
}

// T threads; NC slots, the last one a zero that no constraint takes; J = NC /
// T slots per thread; K rods per thread (1 or 2); HELD: the rods hold the
// normals of their records in registers; KIND: a contact set, a general set,
// or the conjugate gradients of a contact set's adjoint; MANY: several
// workgroups.  ln: lanes per rod; a rod with more than `longest` records is
// refused.  The launch runs iterations k0 .. kend - 1
// at most (k0 = 0: the start phases first); a stop is latched in the state,
// else the iterate and the step length are left for the next launch.
enum ResKind { kResContacts, kResGeneral, kResCg };

template <int T, int NC, int R1, int R2, bool HELD, ResKind KIND, bool MANY>
__global__ void __launch_bounds__(T, 2)
    k_resident(SolveArgs a, Exchange x, ResCg io, int ln, int longest, double tol, long long max_iter, long long k0,
               long long kend)
{
    constexpr bool BIL = KIND == kResGeneral, CG = KIND == kResCg;
    constexpr int NW = T / 64, J = NC / T, kBins = 64;
    static_assert(NC % T == 0 && J <= 16 && NC <= 0xffff && R1 % kGroup == 0 && R2 % kGroup == 0, "");
    __shared__ __align__(16) double E[3][NC], G[NC], U[2 * NC];
    __shared__ double sP[HELD ? NC : 1], sQ[HELD ? NC : 1];
    __shared__ unsigned short qslot[NC];
    __shared__ __align__(16) double red[MANY ? 2 : 1][4][4 * NW];
    __shared__ int hist[kBins], share[4], bad, slow;
    const int tid = threadIdx.x;
    const int n = (int)a.n, nc = (int)a.nc;
    SolverState *S = a.state;
    if (k0 > 0 && S->done) return;
    const int lsh = ln == 4 ? 2 : (ln == 2 ? 1 : 0), sub = tid & (ln - 1);

    // the workgroup's rods
    int r0 = 0, r1 = n;
    if (MANY) {
        const int64_t total = (int64_t)a.pptr[n] + a.qptr[n] + 2 * (int64_t)n;
        if (tid < 128) {
            const int g = (int)blockIdx.x + (tid >> 6);
            const int r = g >= (int)gridDim.x ? n : res_boundary(a, n, total * g / (int)gridDim.x);
            if ((tid & 63) == 0) share[tid >> 6] = r;
        }
        __syncthreads();
        r0 = share[0];
        r1 = share[1];
    }
    const int c0 = a.pptr[r0], q0 = a.qptr[r0], own = a.pptr[r1] - c0, nq = a.qptr[r1] - q0;
    if (tid == 0) {
        share[2] = own;  // slots in use
        share[3] = 0;    // rods with records
        bad = slow = 0;
    }
    if (tid < kBins) hist[tid] = 0;
    __syncthreads();
    // slots of the Q lists: the owner's, or a second one for a constraint
    // whose P rod is elsewhere (its constraint left in `away` for now)
    int *ord = reinterpret_cast<int *>(U), *away = reinterpret_cast<int *>(U + NC);
    for (int k = tid; k < nq; k += T) {
        const int c = a.qidx[q0 + k];
        int s = c - c0;
        if (s < 0 || s >= own) {
            s = atomicAdd(&share[2], 1);
            if (s < NC) away[s] = c;
        }
        if (k < NC) qslot[k] = (unsigned short)min(s, NC - 1);
    }
    // the rods with records, by descending number of them: slot t of the
    // order goes to lanes ln t ... of the workgroup (which rod a thread holds
    // does not enter any sum)
    auto records_of = [&](int r) { return a.pptr[r + 1] - a.pptr[r] + a.qptr[r + 1] - a.qptr[r]; };
    auto key_of = [&](int r) { return kBins - 1 - min(records_of(r), kBins - 1); };
    for (int r = r0 + tid; r < r1; r += T) {
        const int m = records_of(r);
        atomicAdd(&hist[kBins - 1 - min(m, kBins - 1)], 1);
        if (m > longest) slow = 1;
    }
    __syncthreads();
    const int slots = share[2], cap = (R2 ? 2 : 1) * (T >> lsh);
    if (tid < 64) {
        const int v = hist[tid];
        int incl = v;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int t = __shfl_up(incl, d, 64);
            if (tid >= d) incl += t;
        }
        hist[tid] = incl - v;
        if (tid == kBins - 2) share[3] = incl;  // the last key holds the rods without records
    }
    __syncthreads();
    const int nrod = share[3];  // share[3] counts the velocities to send from here on
    const bool fits = slots < NC && nrod <= cap && !slow;  // (slots: of own constraints and of every Q record)
    if (!fits && tid == 0) {
        atomicMax(&S->need_slots, slots);
        atomicMax(&S->need_rods, slow ? INT_MAX : nrod);
    }
    static_assert((R2 ? 2 : 1) * T <= 2 * NC, "the order fits in half of U");
    if (fits)
        for (int r = r0 + tid; r < r1; r += T) {
            const int key = key_of(r);
            if (key < kBins - 1) ord[atomicAdd(&hist[key], 1)] = r;
        }
    __syncthreads();
    if (tid == 0) share[3] = 0;

    unsigned num = x.base;  // number of the last exchange
    // sums over the workgroups of what every thread holds the same, p[0..3]
    const int groups = (int)gridDim.x;
    auto publish = [&](u64 *slot, const double p[4]) {
        if (tid < 4) pair_put(slot + 2 * tid, tid == 0 ? p[0] : (tid == 1 ? p[1] : (tid == 2 ? p[2] : p[3])), num);
    };
    // number tid & 3 of the slots tid >> 2, ... of cnt at buf, summed
    auto collect = [&](const u64 *buf, int cnt) {
        double c = 0.0;
        for (int i = tid; i < 4 * cnt; i += T) {
            const u64 *u = buf + (i >> 2) * kSlot + 2 * (i & 3);
            c += pair_wait(u, x, num, &bad);
        }
        return c;
    };
    auto gather4 = [&](double p[4]) {
        if (!MANY) return;
        u64 *buf = x.tot + (num & 1) * 2 * kResMost * kSlot;
        publish(buf + (int)blockIdx.x * kSlot, p);
        int cnt = groups;
        if (groups > kFlat) {
            const int team = (int)blockIdx.x / kTeam;
            cnt = (groups + kTeam - 1) / kTeam;
            if (blockIdx.x % kTeam == 0) {
                const int first = team * kTeam;
                res_sum4_lanes<NW>(collect(buf + first * kSlot, min(kTeam, groups - first)), p, red[MANY]);
                publish(buf + (kResMost + team) * kSlot, p);
                res_sum4_lanes<NW>(collect(buf + kResMost * kSlot, cnt), p, red[0]);
                return;
            }
            buf += kResMost * kSlot;
        }
        res_sum4_lanes<NW>(collect(buf, cnt), p, red[MANY]);
    };
    auto max_all = [&](double v) {
        v = res_max<NW>(v, &red[0][0][0]);
        if (MANY) {
            ++num;
            u64 *buf = x.tot + (num & 1) * 2 * kResMost * kSlot;
            if (tid == 0) pair_put(buf + (int)blockIdx.x * kSlot, v, num);
            double c = 0.0;
            for (int i = tid; i < groups; i += T) {
                const u64 *u = buf + i * kSlot;
                c = fmax(c, pair_wait(u, x, num, &bad));
            }
            v = res_max<NW>(c, &red[0][0][0]);
        }
        return v;
    };
    if (MANY) {
        // everybody is here, and everybody's share fits
        double p[4] = {fits ? 0.0 : 1.0, 0.0, 0.0, 0.0};
        ++num;
        gather4(p);
        if (bad || p[0] > 0.0) {
            if (tid == 0) __hip_atomic_store(x.fail, bad ? 1 : 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
    } else if (!fits) {
        if (tid == 0) *x.fail = 2;
        return;
    }

    if (MANY) {
        // the second slots in the order of their constraints (by rank), so
        // that neighbouring lanes send and receive neighbouring words
        // (four of them a read: at 250 second slots one by one took 13 us)
        int *moved = reinterpret_cast<int *>(U) + (R2 ? 2 : 1) * T;
        static_assert(!MANY || (R2 ? 2 : 1) * T + NC <= 2 * NC, "order and moved slots fit in half of U");
        const int first = own & ~3, last = (slots + 3) & ~3;
        if (tid < 4) {
            if (first + tid < own) away[first + tid] = INT_MAX;
            if (slots + tid < last) away[slots + tid] = INT_MAX;
        }
        __syncthreads();
        int c[J], rank[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int s = own + tid + j * T;
            c[j] = s < slots ? away[s] : 0;
            rank[j] = 0;
        }
        for (int k = first; k < last; k += 4) {
            const int4 v = *reinterpret_cast<const int4 *>(away + k);
#pragma unroll
            for (int j = 0; j < J; ++j)
                rank[j] += (v.x < c[j]) + (v.y < c[j]) + (v.z < c[j]) + (v.w < c[j]);
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int s = own + tid + j * T;
            if (s < slots) {
                moved[s - own] = own + rank[j];
                away[own + rank[j]] = c[j];
            }
        }
        __syncthreads();
        for (int k = tid; k < nq; k += T)
            if (qslot[k] >= own) qslot[k] = (unsigned short)moved[qslot[k] - own];
        __syncthreads();
    }
    const ResLds l{E[0], E[1], E[2], sP, sQ, qslot, G, U, c0, q0};
    // Slot state.  A slot past the last one is a constraint without rods that
    // stays at zero, so the iteration needs no test.  cross: bit j set where
    // the other rod is in another workgroup; out, in: byte offsets in x.u of
    // our velocity and of the other (their high halves `high` further).
    // Conjugate gradients: lambda, r and s in the place of gamma, g and q, the
    // direction in pv, and the active constraints in act.
    double gam[J], g[J], q[J], cm[BIL ? J : 1], pv[CG ? J : 1];
    unsigned act = 0;
    unsigned out[MANY ? J : 1], in[MANY ? J : 1];
    unsigned cross = 0;
    const unsigned high = 8u * (unsigned)(MANY ? gridDim.x : 0) * NC;
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int s = tid + j * T;
        const bool ok = s < slots;
        const int c = !ok ? 0 : (s < own ? c0 + s : away[s]);
        gam[j] = g[j] = q[j] = 0.0;
        if (BIL) cm[j] = -1.0;
        if (MANY) out[j] = in[j] = 0;
        if (CG) pv[CG ? j : 0] = 0.0;
        if (ok) {
            if (CG) {
                const double2 *cs = reinterpret_cast<const double2 *>(io.cs + 4 * (int64_t)c);
                const double2 lp = cs[0], rs = *reinterpret_cast<const double2 *>(io.cr + 4 * (int64_t)c);
                gam[j] = lp.x;
                pv[CG ? j : 0] = lp.y;
                g[j] = rs.x;
                q[j] = rs.y;
                if (cs[1].x > 0.0) act |= 1u << j;
            } else {
                const double2 st = a.st[c];
                gam[j] = st.x;
                g[j] = st.y;
                q[j] = a.qv[c];
                if (BIL) cm[j] = a.cmpv[c];
            }
            if (MANY) {
                const int r = a.pp[c].y;  // the Q rod (below 0: a fixed body)
                if (s >= own || (r >= 0 && (r < r0 || r >= r1))) {
                    cross |= 1u << j;
                    const unsigned k = (unsigned)blockIdx.x * NC + (unsigned)atomicAdd(&share[3], 1);
                    out[j] = 8u * k;
                    in[j] = 2u * (unsigned)c + (s < own ? 1u : 0u);
                    word_put(x.at + 2 * (int64_t)c + (s < own ? 0 : 1), ((u64)k << 32) | num);
                }
            }
        }
        const double2 *gd = reinterpret_cast<const double2 *>(a.geo + 4 * (int64_t)c);
        const double2 g0 = gd[0], g1 = gd[1];
        E[0][s] = ok ? g0.x : 0.0;
        E[1][s] = ok ? g0.y : 0.0;
        E[2][s] = ok ? g1.x : 0.0;
        if (HELD) {
            sP[s] = ok ? g1.y : 0.0;
            if (s < nq) sQ[s] = a.qgeo[4 * (int64_t)(q0 + s) + 3];
        }
        G[s] = 0.0;
    }
    // the start, for when a wait runs out after somebody's results are out (the
    // two kernels' product is not in use here)
    if (MANY && !CG && k0 == 0)
#pragma unroll
        for (int j = 0; j < J; ++j)
            if (tid + j * T < own) a.uP[c0 + tid + j * T] = gam[j];
    ResRod<R1, HELD> rod1;
    ResRod<R2 ? R2 : kGroup, HELD> rod2;
    __syncthreads();
    {
        const int t = tid >> lsh, st = T >> lsh;
        res_rod_setup<NC>(a, l, t < nrod ? ord[t] : -1, sub, ln, rod1);
        // the second rods backwards, so that no wave has the longest of both
        const int t2 = 2 * st - 1 - t;
        if (R2) res_rod_setup<NC>(a, l, t2 < nrod ? ord[t2] : -1, sub, ln, rod2);
    }
    __syncthreads();
    if (MANY) {
        // where the other velocities will be
#pragma unroll
        for (int j = 0; j < J; ++j)
            if ((cross >> j) & 1u) {
                u64 v = 0;
                for (int spin = spent(x, num);; ++spin) {
                    v = word_get(x.at + in[j]);
                    if ((unsigned)v == num || give_up(spin, x.fail, &bad)) break;
                }
                in[j] = (unsigned)v == num ? 8u * (unsigned)(v >> 32) : 0u;
            }
    }
    // a constraint without a Q side keeps u_Q = 0, an empty slot both
#pragma unroll
    for (int j = 0; j < J; ++j) U[tid + j * T] = U[NC + tid + j * T] = 0.0;

    // one product: G holds v, w[j] receives D^T M D v of the thread's slots
    auto product = [&](double w[J]) {
        if (MANY) ++num;
        __syncthreads();
        res_rod<NC>(a, l, sub, ln, rod1);
        if (R2) res_rod<NC>(a, l, sub, ln, rod2);
        __syncthreads();
        double up[J], uq[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            up[j] = U[tid + j * T];
            uq[j] = U[NC + tid + j * T];
        }
        if (MANY) {
            // our halves out, then all of the others polled together (a round
            // trip is most of the wait: one slot after the other would take
            // one each)
            unsigned char *base = reinterpret_cast<unsigned char *>(x.u);
            auto word = [&](unsigned o) { return reinterpret_cast<u64 *>(base + o); };
#pragma unroll
            for (int j = 0; j < J; ++j)
                if ((cross >> j) & 1u) {
                    const double v = tid + j * T < own ? up[j] : uq[j];
                    word_put(word(out[j]), half_word(__double2loint(v), num));
                    word_put(word(out[j] + high), half_word(__double2hiint(v), num));
                }
            unsigned left = cross;
            for (int spin = spent(x, num); left; ++spin) {
                u64 lo[J], hi[J];
#pragma unroll
                for (int j = 0; j < J; ++j)
                    if ((left >> j) & 1u) {
                        lo[j] = word_get(word(in[j]));
                        hi[j] = word_get(word(in[j] + high));
                    }
#pragma unroll
                for (int j = 0; j < J; ++j)
                    if (((left >> j) & 1u) && (unsigned)lo[j] == num && (unsigned)hi[j] == num) {
                        const double v = pair_value(lo[j], hi[j]);
                        if (tid + j * T < own) uq[j] = v;
                        else up[j] = v;
                        left &= ~(1u << j);
                    }
                if (left && give_up(spin, x.fail, &bad)) break;
            }
        }
#pragma unroll
        for (int j = 0; j < J; ++j) w[j] = up[j] + uq[j];
    };
    auto bil = [&](int j) { return BIL && cm[BIL ? j : 0] >= 0.0; };
    auto diag = [&](int j, double v) { return bil(j) ? cm[BIL ? j : 0] * v : 0.0; };
    // its sums are over the constraints: a second slot does not enter them
    auto ours = [&](int j) { return !MANY || tid + j * T < own; };

    double alpha = 0.0, alpha0 = 0.0, amin = 0.0, amax = 0.0, rmax = 0.0;
    if (k0 > 0) {
        alpha = S->alpha;
        alpha0 = S->alpha0;
        amin = S->amin;
        amax = S->amax;
    }
    int status = RL_OK;
    bool done = false;
    long long iter = 0;
    double p[4], w[J];
    auto sum_all = [&]() {
        res_sum4<NW>(p, red[0]);
        gather4(p);
    };
    if constexpr (CG) {
        double rho = 0.0, bb = 0.0, nact = 0.0, res = 0.0;
        if (k0 == 0) {
            p[0] = p[1] = p[2] = p[3] = 0.0;
#pragma unroll
            for (int j = 0; j < J; ++j) {
                p[0] += ours(j) ? g[j] * g[j] : 0.0;
                p[2] += ours(j) ? (double)((act >> j) & 1u) : 0.0;
            }
            if (MANY) ++num;
            sum_all();
            bb = p[0];
            nact = p[2];
            if (!(bb > 0.0)) {
                status = isfinite(bb) ? RL_OK : RL_ERR_NONFINITE;
                done = true;
            }
        } else {
            bb = S->alpha0;
            nact = S->ss;
            rho = S->amin;
        }
        if (!done && !(MANY && bad))
            for (long long k = k0; k < kend; ++k) {
#pragma unroll
                for (int j = 0; j < J; ++j) G[tid + j * T] = g[j];
                product(w);
                p[0] = p[1] = p[2] = p[3] = 0.0;
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    if (!((act >> j) & 1u)) w[j] = 0.0;
                    const double rv = ours(j) ? g[j] : 0.0;
                    p[0] += rv * rv;
                    p[1] += rv * w[j];
                }
                sum_all();
                // the rules of the two-kernel loop (alpha: of the iteration before)
                double beta = 0.0, den = p[1];
                if (k > 0) {
                    beta = p[0] / rho;
                    den = p[1] - beta * p[0] / alpha;
                }
                rho = p[0];
                const double a1 = rho / den;
                status = 1000;
                if (!isfinite(rho) || !isfinite(p[1])) status = RL_ERR_NONFINITE;
                else if (rho <= tol * tol * bb) status = RL_OK;
                else if (k >= max_iter) status = RL_NOT_CONVERGED;
                else if (!(a1 > 0.0) || !isfinite(a1)) status = RL_STAGNATED;
                if (__builtin_expect(status != 1000 || (MANY && bad), 0)) {
                    done = !(MANY && bad);
                    iter = k;
                    res = sqrt(rho / bb);
                    break;
                }
                alpha = a1;
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    q[j] = fma(beta, q[j], w[j]);
                    pv[CG ? j : 0] = fma(beta, pv[CG ? j : 0], g[j]);
                    gam[j] = fma(alpha, pv[CG ? j : 0], gam[j]);
                    g[j] = fma(-alpha, q[j], g[j]);
                }
            }
        if (MANY) {
            __syncthreads();
            if (bad) return;  // the flag is set
        }
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int s = tid + j * T;
            if (s < own) {
                const int c = c0 + s;
                *reinterpret_cast<double2 *>(io.cs + 4 * (int64_t)c) = make_double2(gam[j], pv[CG ? j : 0]);
                *reinterpret_cast<double2 *>(io.cr + 4 * (int64_t)c) = make_double2(g[j], q[j]);
                io.cq[4 * (int64_t)a.qpos[c] + 3] = gam[j];
            }
        }
        if (blockIdx.x == 0 && tid == 0) {
            S->alpha = alpha;
            S->alpha0 = bb;
            S->amin = rho;
            S->ss = nact;
            S->res = res;
            S->iter = iter;
            S->status = done ? status : RL_OK;
            S->done = done ? 1 : 0;
        }
        return;
    }
    if (k0 == 0) {
        // g0 = Mc gamma0 + q on the projected start
#pragma unroll
        for (int j = 0; j < J; ++j) {
            if (!bil(j)) gam[j] = gamma_prime<kModeInit>(gam[j], 0.0, 0.0);
            G[tid + j * T] = gam[j];
        }
        product(w);
        p[0] = p[1] = p[2] = p[3] = 0.0;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            g[j] = w[j] + (q[j] + diag(j, gam[j]));
            const double gn = ours(j) ? g[j] : 0.0;
            p[2] += gn * gn;
            rmax = fmax(rmax, ours(j) ? fabs(!bil(j) && gam[j] < g[j] ? gam[j] : g[j]) : 0.0);
        }
        p[3] = rmax > tol ? 1.0 : 0.0;
        sum_all();
        if (!isfinite(p[2])) {
            status = RL_ERR_NONFINITE;
            done = true;
        } else if (!(p[3] > 0.0)) {
            done = true;
        }
        if (!done && !(MANY && bad)) {
            // the Cauchy step on the projected gradient
#pragma unroll
            for (int j = 0; j < J; ++j)
                G[tid + j * T] = bil(j) ? g[j] : gamma_prime<kModeAlpha0>(gam[j], g[j], 0.0);
            product(w);
            p[0] = p[1] = p[2] = p[3] = 0.0;
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const double gh = !ours(j) ? 0.0 : (bil(j) ? g[j] : gamma_prime<kModeAlpha0>(gam[j], g[j], 0.0));
                p[0] += gh * gh;
                p[1] += gh * (w[j] + diag(j, gh));
            }
            sum_all();
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
    }
    // The iterations, written to fall through: a taken branch costs about as
    // much as ten instructions here.
    if (!done && !(MANY && bad))
        for (long long k = k0; k < kend; ++k) {
#pragma unroll
            for (int j = 0; j < J; ++j)
                G[tid + j * T] = bil(j) ? gamma_free<kModeLoop>(gam[j], g[j], alpha)
                                        : gamma_prime<kModeLoop>(gam[j], g[j], alpha);
            product(w);
            // (s.s, s.y, y.y, whether a residual is above the tolerance)
            p[0] = p[1] = p[2] = rmax = 0.0;
#pragma unroll
            for (int j = 0; j < J; ++j) {
                // gamma' again (cheaper than registers held across the rods' turn)
                const double v = bil(j) ? gamma_free<kModeLoop>(gam[j], g[j], alpha)
                                        : gamma_prime<kModeLoop>(gam[j], g[j], alpha);
                const double gn = w[j] + (q[j] + diag(j, v));
                const double sc = ours(j) ? v - gam[j] : 0.0, yc = ours(j) ? gn - g[j] : 0.0;
                const double r = fabs(!bil(j) && v < gn ? v : gn);
                p[0] += sc * sc;
                p[1] += sc * yc;
                p[2] += yc * yc;
                rmax = fmax(rmax, ours(j) ? r : 0.0);
                gam[j] = v;
                g[j] = gn;
            }
            p[3] = rmax > tol ? 1.0 : 0.0;
            sum_all();
            // the step rule's residual only has to be on the right side of
            // the tolerance here; the stop takes the true one below
            const double t[4] = {p[0], p[1], p[2], p[3] > 0.0 ? 2.0 * tol + 1.0 : 0.0};
            const Decision d = decide_from(DecideIn{tol, amin, amax, alpha, max_iter}, k + 1, t);
            alpha = d.alpha;
            if (__builtin_expect(d.stop || (MANY && bad), 0)) {
                done = !(MANY && bad);
                status = d.status;
                iter = k + 1;
                break;
            }
        }
    double res = 0.0;
    if (done) {
        res = max_all(rmax);
        if (!isfinite(res)) status = RL_ERR_NONFINITE;
    }
    if (MANY) {
        __syncthreads();
        if (bad) return;  // the flag is set
        if (tid == 0) x.tot[kLeft + blockIdx.x] = num;  // (all on one word took 10 us)
    }
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int s = tid + j * T;
        if (s < own) {
            const int c = c0 + s, k = a.qpos[c];
            const double2 v = make_double2(gam[j], g[j]);
            a.st[c] = v;
            if (!BIL || k >= 0) a.stq[k] = v;
        }
    }
    if (blockIdx.x == 0 && tid == 0) {
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

// The start of a solve of contacts or a general set back from where the first
// launch left it, if results are out: always after a second launch (left
// null), else if a workgroup says so.
__global__ void __launch_bounds__(kResMost) k_resident_start(SolveArgs a, const u64 *left, unsigned base)
{
    if (left && !__syncthreads_or(left[threadIdx.x] - base - 1 < (u64)kResNumbers)) return;
    const int64_t c = blockIdx.x * (int64_t)kResMost + threadIdx.x;
    if (c >= a.nc) return;
    const double2 v = make_double2(a.uP[c], 0.0);
    const int k = a.qpos[c];
    a.st[c] = v;
    if (k >= 0) a.stq[k] = v;
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// form, workgroups (0: no form takes the problem) and lanes per rod
struct ResPlan {
    int form, groups, ln;
    int longest;  // list of a rod that it takes
    int forms;    // the first form that it does not go up to
};
constexpr int kResSolo = 1536;  // constraints up to which one workgroup is as fast as several
constexpr int kResFew = 64;     // workgroups up to which a problem takes only as many as it needs,
constexpr int kResPer = 256;    // of so many constraints

// The forms: threads, slots, records held by a thread's first and second rod,
// whether with their normals.
constexpr int kResSlots[kResForms] = {1024, 1536, 2048, 2560, 3072};
constexpr int kResThreads = 512;  // threads of all but the smallest

template <int T, int NC, int R1, int R2, bool HELD, bool MANY>
static hipError_t launch_form(hipStream_t st, const SolveArgs &a, Exchange x, const ResCg *cg, const ResPlan &p,
                              double tol, long long max_iter, long long k0, long long kend)
{
    SolveArgs aa = a;
    ResCg io = cg ? *cg : ResCg{nullptr, nullptr, nullptr};
    int ln = p.ln, longest = p.longest;
    void *args[] = {&aa, &x, &io, &ln, &longest, &tol, &max_iter, &k0, &kend};
    const void *f = cg ? (const void *)k_resident<T, NC, R1, R2, HELD, kResCg, MANY>
                    : a.gen ? (const void *)k_resident<T, NC, R1, R2, HELD, kResGeneral, MANY>
                            : (const void *)k_resident<T, NC, R1, R2, HELD, kResContacts, MANY>;
    // cooperative: all workgroups are resident before any waits for another
    if (MANY) return hipLaunchCooperativeKernel(f, dim3(p.groups), dim3(T), args, 0, st);
    return hipLaunchKernel(f, dim3(1), dim3(T), args, 0, st);
}

// The longest list of a rod that a plan takes.  The lanes of one rod walk its
// records alone while everybody waits: past the held ones 0.27 us a lane and
// record, 0.40 where the normals come from LDS, and only 0.066 a record of all
// in the loop over memory, where eight lanes of several rods share a wave.  So
// lists decide against the chip where the first costs more than the chip
// gains: 32 records on one lane of one workgroup 8.2 us per iteration (memory
// 9.1), 48 12.6 (10.0); of 16 workgroups 16 6.2 (8.3), 32 10.6 (9.4); on two
// lanes 64 10.7 (11.6), 96 15.0 (13.6), of 128 workgroups 96 17.5 (17.6);
// with the normals from LDS 48 13.8 (14.9), 64 17.2 (16.3); on four lanes 256
// 19.5 (24.6) and 25.9 (24.6).  (901 rods, 900 contacts of one: 243 and 81.)
// Suspensions of up to 100,000 rods have lists of 25 to 35, at 30,000 rods and
// phi 0.08 49 on two lanes: there the chip gains 5 to 7 us.
static int resident_longest(const ResPlan &p)
{
    const bool few = p.groups > 1 && p.groups <= kResFew, held = p.groups == 1 || p.form < 3;
    if (p.ln == 1) return few ? 26 : (p.groups == 1 ? 36 : 40);
    if (p.ln == 2) return held ? (few ? 76 : 96) : 64;
    return held ? INT_MAX : 240;
}

// Form, workgroups and lanes per rod of a problem; groups = 0: none takes it.
static ResPlan resident_plan(const rl_ctx *h, int64_t n, int64_t nc, bool ordered, bool cg)
{
    ResPlan p{0, 0, 1, INT_MAX, kResForms};
    if (nc <= 0 || nc >= (1 << 29)) return p;
    if (h->onchip.groups > 0) return ResPlan{h->onchip.form, h->onchip.groups, h->onchip.lanes, INT_MAX, kResForms};
    if (n <= 512 && nc < 1024) {
        p.groups = 1;
    } else if (n <= 1024 && nc < kResSolo) {
        p.form = 1;
        p.groups = 1;
    } else {
        // slots of a workgroup: its own constraints and those that reach in
        // from outside, nearly all of them when the rods are in no spatial
        // order.  In a step's order the fullest workgroup of suspensions asks
        // for 1.33 (100,000 nematic rods, phi 0.03) to 1.45 times the mean of
        // its own at 390 rods a workgroup, 1.5 to 1.6 at 200, 1.8 at 80.  The
        // estimate is the lower end: a refused launch costs 65 to 80 us of the
        // solve, a form larger than needed 0.4 to 1.3 us of each iteration
        // (100,000 nematic, 281,000 constraints: 8.5 with 1,536 slots, 9.5 with
        // 2,048).  In no order the larger forms lose (60,000
        // rods and 180,000 constraints 15.2 us per iteration, two kernels 17.5;
        // 200,000 18.0 and 17.5, 240,000 20.2 and 17.9; general sets 180,000
        // 14.9 and 17.6, 240,000 20.3 and 18.4), the conjugate gradients later
        // (200,000 17.9 and 22.2, 240,000 20.1 and 24.0).  A problem that does
        // not fit after all is tried again with as many slots as it asks for.
        const double reach = ordered ? 1.30 : 2.05;
        const int forms = p.forms = ordered ? kResForms : (cg ? 3 : 2);
        const int most = std::min(h->cus, kResMost);
        auto fits = [&](int g, int form) {
            return (double)nc * reach / g <= 0.96 * kResSlots[form] && 1.15 * (double)n / g + 8.0 <= 512.0;
        };
        int g = (int)std::min<int64_t>((nc + kResPer - 1) / kResPer, kResFew);
        g = std::max(g, 2);
        if (!fits(g, 0)) g = 2 * kResFew;
        // past 550 a workgroup 256 cost less, about (50,000 rods, 77,000
        // constraints: 6.3 us per iteration with 128, 5.9; 20,000 and 62,000:
        // 5.2 and 5.6; but 24,000 and 82,000, where 128 leave room for two
        // lanes a rod: 5.4 and 6.0)
        if (!fits(g, 0) || (ordered && nc > 550 * 2 * kResFew)) g = most;
        if (g > most) return p;
        while (p.form < forms && !fits(g, p.form)) ++p.form;
        if (p.form == forms) return p;
        p.groups = g;
    }
    // several lanes per rod while that leaves one rod per thread (the single
    // workgroup has two, and takes them for long lists)
    const bool two = p.groups == 1;
    const int T = two && p.form == 0 ? 256 : kResThreads;
    const double rods = two ? (double)n : 1.15 * (double)n / p.groups + 8.0;
    while (p.ln < 4 && (2 * p.ln * rods <= T || (two && 2 * p.ln * rods <= 2 * T && 2.0 * nc > 6.0 * p.ln * n)))
        p.ln *= 2;
    p.longest = resident_longest(p);
    return p;
}

// The form that holds what the refused one did not; false: there is none.  (All
// several-workgroup forms have the same threads.)
static bool resident_larger(ResPlan &p, int slots, int rods)
{
    while (p.form < p.forms && kResSlots[p.form] <= slots) ++p.form;
    if (p.longest < INT_MAX) p.longest = resident_longest(p);
    return p.groups > 1 && p.form < p.forms && rods <= kResThreads / p.ln;
}

static int64_t resident_words(const ResPlan &p, int64_t nc)
{
    return p.groups > 1 ? 2 * (int64_t)p.groups * kResSlots[kResForms - 1] + 2 * nc + kLeft + kResMost : 0;
}

size_t resident_bytes(const rl_ctx *h, int64_t n, int64_t nc)
{
    const ResPlan most{kResForms - 1, std::min(h->cus, kResMost), 1, INT_MAX, kResForms};
    return n <= 1024 && nc < kResSolo ? 0 : sizeof(u64) * (size_t)resident_words(most, nc);
}

static hipError_t launch_resident(hipStream_t st, const SolveArgs &a, const ResPlan &p, const ResCg *cg,
                                  const rl_onchip &ctl, unsigned long long *words, unsigned base, double tol,
                                  long long max_iter, long long k0, long long kend)
{
    // (of this launch's exchanges)
    const long long patient = std::max<long long>(0, ctl.patient - k0 / kResChunk * kResNumbers);
    if (ctl.refuse == RL_ONCHIP_NO_ROOM) return hipErrorCooperativeLaunchTooLarge;
    u64 *at = words ? words + 2 * (int64_t)p.groups * kResSlots[p.form] : nullptr;
    const Exchange x{words, at, words ? at + 2 * a.nc : nullptr, base, &a.state->fail,
                     ctl.patient < 0 ? UINT_MAX : (unsigned)std::min<long long>(base + patient, UINT_MAX)};
    if (p.groups == 1) {
        if (p.form == 0) return launch_form<256, 1024, 8, 4, true, false>(st, a, x, cg, p, tol, max_iter, k0, kend);
        return launch_form<512, 2048, 8, 4, true, false>(st, a, x, cg, p, tol, max_iter, k0, kend);
    }
    switch (p.form) {
    case 0: return launch_form<512, 1024, 8, 0, true, true>(st, a, x, cg, p, tol, max_iter, k0, kend);
    case 1: return launch_form<512, 1536, 12, 0, true, true>(st, a, x, cg, p, tol, max_iter, k0, kend);
    case 2: return launch_form<512, 2048, 8, 0, true, true>(st, a, x, cg, p, tol, max_iter, k0, kend);
    case 3: return launch_form<512, 2560, 16, 0, false, true>(st, a, x, cg, p, tol, max_iter, k0, kend);
    default: return launch_form<512, 3072, 12, 0, false, true>(st, a, x, cg, p, tol, max_iter, k0, kend);
    }
}

// The form of a solve on chip, and its exchange words cleared of any number
// it could take for one of its own.  groups = 0: the two kernels take it
// (sampled timing of the loop kernels needs them too, and
// the allocation-free solve, which takes no samples, has the same bits).
static int resident_prepare(rl_ctx *h, const SolveArgs &a, bool cg, ResPlan *plan, unsigned long long **words)
{
    *words = nullptr;
    plan->groups = 0;
    if (h->prm.precision != RL_FP64 || h->prof_every > 0) return RL_OK;
    *plan = resident_plan(h, a.n, a.nc, a.ordered, cg);
    if (plan->groups <= 1) return RL_OK;
    if (h->xchg_skip > 0) {
        --h->xchg_skip;
        plan->groups = 0;
        return RL_OK;
    }
    const size_t bytes = sizeof(unsigned long long) * (size_t)resident_words(*plan, a.nc);
    if (h->arena_on && h->arena_used + bytes + 512 > kScratchBytes) {
        plan->groups = 0;  // the list itself fits, the exchange does not
        return RL_OK;
    }
    int err = h->onchip.refuse == RL_ONCHIP_NO_MEMORY ? RL_ERR_NOMEM : 0;
    if (!err) *words = (unsigned long long *)ws_get(h, kWsXchg, bytes, &err);
    if (err) {
        // no memory for the exchange: the two kernels have all they need
        h->xchg_buf = nullptr;
        plan->groups = 0;
        ++h->onchip_out[3];
        return RL_OK;
    }
    // a new buffer, the scratch array (anybody's) or numbers about to run out
    const bool arena = h->arena_on;
    if (arena || h->xchg_buf != *words || h->xchg_cap != h->cap[kWsXchg] || h->xchg_num > 0xf0000000u) {
        RL_HIP(hipMemsetAsync(*words, 0, arena ? bytes : h->cap[kWsXchg], h->stream));
        h->xchg_buf = arena ? nullptr : *words;
        h->xchg_cap = arena ? 0 : h->cap[kWsXchg];
        h->xchg_num = 0;
    }
    return RL_OK;
}

int resident_run(rl_ctx *h, const SolveArgs &a, const ResCg *cg, double tol, const std::function<hipError_t()> &queue,
                 bool copies, bool *solved)
{
    hipStream_t st = h->stream;
    *solved = false;
    ResPlan plan{0, 0, 1, INT_MAX, kResForms};
    unsigned long long *words = nullptr;
    const int rc = resident_prepare(h, a, cg != nullptr, &plan, &words);
    if (rc) return rc;
    h->onchip_out[5] = 0;
    // the launches start from a state without a failure, which they leave so
    if (plan.groups > 0 && !h->state_ready) {
        hipLaunchKernelGGL(k_state_init, dim3(1), dim3(64), 0, st, h->state, tol, (long long)h->prm.max_iter);
        RL_HIP(hipGetLastError());
        h->state_ready = true;
    }
    // a long solve is cut into launches so that each ends soon
    for (long long k0 = 0; plan.groups > 0 && !*solved;) {
        if (words && h->xchg_num > 0xf8000000u) {
            RL_HIP(hipMemsetAsync(words, 0, sizeof(*words) * (size_t)resident_words(plan, a.nc), st));
            h->xchg_num = 0;
        }
        const unsigned base = h->xchg_num;
        h->xchg_num += (unsigned)kResNumbers;
        int64_t *out = h->onchip_out;
        out[4] = plan.form;
        out[5] = plan.groups;
        out[6] = plan.ln;
        if (launch_resident(st, a, plan, cg, h->onchip, words, base, tol, (long long)h->prm.max_iter, k0,
                            k0 + kResChunk) != hipSuccess) {
            // no room for its workgroups on this device (a part of its compute
            // units, say): the two kernels need none
            (void)hipGetLastError();
            ++out[3];
            break;
        }
        if (!copies)
            RL_HIP(hipMemcpyAsync(h->state_host, h->state, sizeof(SolverState), hipMemcpyDeviceToHost, st));
        RL_HIP(queue());
        RL_HIP(hipStreamSynchronize(st));
        *solved = h->state_host->done != 0;
        const int fail = h->state_host->fail;
        if (!fail) {
            k0 += kResChunk;
            out[0] += *solved;
            continue;
        }
        ++out[fail == 2 ? 1 : 2];
        // left without a result: more slots, or the two kernels from the start.
        // What does not fit is found again by each solve that does not (a
        // launch of 20 to 30 us), so that the loop a problem takes, and with it
        // the last bits of its solution, depends on the problem alone.
        *solved = false;
        const int slots = h->state_host->need_slots, rods = h->state_host->need_rods;
        // (no workgroup's results are out before all have put their start away)
        if (fail == 1 && !cg) {
            const u64 *left = words + 2 * (int64_t)plan.groups * kResSlots[plan.form] + 2 * a.nc + kLeft;
            hipLaunchKernelGGL(k_resident_start, dim3((unsigned)((a.nc + kResMost - 1) / kResMost)), dim3(kResMost), 0,
                               st, a, k0 > 0 ? nullptr : left, base);
            RL_HIP(hipGetLastError());
        }
        hipLaunchKernelGGL(k_state_init, dim3(1), dim3(64), 0, st, h->state, tol, (long long)h->prm.max_iter);
        RL_HIP(hipGetLastError());  // (clears the failure)
        if (fail == 2 && k0 == 0 && resident_larger(plan, slots, rods)) continue;
        if (fail != 2) h->xchg_skip = 64;
        break;
    }
    if (!*solved) h->onchip_out[5] = 0;
    return RL_OK;
}

}  // namespace rl

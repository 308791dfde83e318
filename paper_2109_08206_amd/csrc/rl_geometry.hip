// Rod geometry on gfx950: directors, per-rod mobility, closest points of rod
// axes, the uniform-grid pair search and the constraint geometry.
//
// Method: Yan et al., arXiv 2109.08206.  Directors come from the unit
// quaternion of each rod (Appendix "Filament dynamics"); pairs are the rods
// whose surface gap is below the threshold (Appendix "Implementation");
// the constraint column of a pair uses the closest points and the unit
// normal between them (Appendix "Symmetry of the geometrically constrained
// optimization problem", D_PQ and r = x_P + y_P - x_Q - y_Q); q follows
// eq. (blockdef), block A.
#include <cmath>
#include <cstdarg>
#include <cstring>
#include <type_traits>

#include "rl_device.hpp"
#include "rl_vec.hpp"

namespace rl {


// ---------------------------------------------------------------------------
// directors: third column of R(theta) = (s^2 - p.p) I + 2 p p^T + 2 s [p]x
// ---------------------------------------------------------------------------
__global__ void k_directors(int64_t n, const double *__restrict__ quat, double *__restrict__ dir)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double2 a = *reinterpret_cast<const double2 *>(quat + 4 * i);
    const double2 b = *reinterpret_cast<const double2 *>(quat + 4 * i + 2);
    const double s = a.x, px = a.y, py = b.x, pz = b.y;
    dir[3 * i + 0] = 2.0 * (px * pz + s * py);
    dir[3 * i + 1] = 2.0 * (py * pz - s * px);
    dir[3 * i + 2] = s * s - px * px - py * py + pz * pz;
}

hipError_t launch_directors(hipStream_t st, int64_t n, const double *quat, double *dir)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_directors, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, n, quat, dir);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// slender-body mobility of a rod of length L (perpendicular drag
// 4 pi eta L / log(2L/d) as in Section 3; parallel drag half of it;
// rotational drag pi eta L^3 / (3 log(2L/d)))
// ---------------------------------------------------------------------------
__host__ __device__ inline Mob mobility_of(double L, double diam, double eta)
{
    const double lg = log(2.0 * L / diam);
    Mob m;
    m.aperp = lg / (4.0 * M_PI * eta * L);
    m.apar = 2.0 * m.aperp;
    m.rperp = 3.0 * lg / (M_PI * eta * L * L * L);
    return m;
}

Mob mobility_host(double L, double diam, double eta) { return mobility_of(L, diam, eta); }

__global__ void k_mobility_coeffs(int64_t n, const double *__restrict__ len, double diam, double eta,
                                  double *__restrict__ coef)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const Mob m = mobility_of(len[i], diam, eta);
    coef[3 * i + 0] = m.apar;
    coef[3 * i + 1] = m.aperp;
    coef[3 * i + 2] = m.rperp;
}

hipError_t launch_mobility_coeffs(hipStream_t st, int64_t n, const double *len, double diam, double eta, double *coef)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mobility_coeffs, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, n, len,
                       diam, eta, coef);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Closest points of two rod axes xi + s di (|s| <= hi) and xj + t dj
// (|t| <= hj), xj already imaged.  The squared distance is a convex
// quadratic in (s, t): take the stationary s with t free and clamp it, the
// best t for that s, and if t leaves its range clamp it and take the best s
// again (clamped normal equations for segment pairs, Lumelsky 1985).  For
// parallel axes (1 - b^2 <= 1e-14) the contact is the midpoint of the
// overlap of the two parameter ranges, else the best end-point candidate.
// ---------------------------------------------------------------------------
struct Contact {
    double s, t, dist;
    V3 e;
    unsigned flags;
};

__device__ Contact closest_point(V3 xi, V3 di, double hi, V3 xj, V3 dj, double hj)
{
    const V3 r0 = xi - xj;
    const double b = dot(di, dj);
    const double c = dot(di, r0);
    const double f = dot(dj, r0);
    const double den = 1.0 - b * b;
    Contact out;
    out.flags = den <= kBandPar ? 2u : 0u;
    double s, t;
    if (den > kEpsPar) {
        s = clampd((b * f - c) / den, -hi, hi);
        t = b * s + f;
        if (t < -hj) {
            t = -hj;
            s = clampd(b * t - c, -hi, hi);
        } else if (t > hj) {
            t = hj;
            s = clampd(b * t - c, -hi, hi);
        }
    } else {
        const double sg = b >= 0.0 ? 1.0 : -1.0;
        double lo = (-hj - f) * sg, up = (hj - f) * sg;
        if (lo > up) {
            const double tmp = lo;
            lo = up;
            up = tmp;
        }
        lo = lo > -hi ? lo : -hi;
        up = up < hi ? up : hi;
        if (lo <= up) {
            s = 0.5 * (lo + up);
            t = clampd(b * s + f, -hj, hj);
        } else {
            double best = INFINITY;
            s = 0.0;
            t = 0.0;
            for (int k = 0; k < 4; ++k) {
                double sk, tk;
                if (k < 2) {
                    sk = k == 0 ? -hi : hi;
                    tk = clampd(b * sk + f, -hj, hj);
                } else {
                    tk = k == 2 ? -hj : hj;
                    sk = clampd(b * tk - c, -hi, hi);
                }
                const V3 rk = r0 + sk * di - tk * dj;
                const double d2 = dot(rk, rk);
                if (d2 < best) {
                    best = d2;
                    s = sk;
                    t = tk;
                }
            }
        }
    }
    const V3 r = r0 + s * di - t * dj;
    const double dist = sqrt(dot(r, r));
    out.s = s;
    out.t = t;
    out.dist = dist;
    if (dist >= kDegenDist) {
        out.e = v3(r.x / dist, r.y / dist, r.z / dist);
    } else {
        out.flags |= 4u;
        V3 nrm = cross(di, dj);
        double nn = sqrt(dot(nrm, nrm));
        if (nn < 1e-12) {
            // collinear axes: normal to di and the coordinate axis least aligned with it
            const double ax = fabs(di.x), ay = fabs(di.y), az = fabs(di.z);
            int k = 0;
            double best = ax;
            if (ay < best) {
                k = 1;
                best = ay;
            }
            if (az < best) k = 2;
            const V3 ek = v3(k == 0 ? 1.0 : 0.0, k == 1 ? 1.0 : 0.0, k == 2 ? 1.0 : 0.0);
            nrm = cross(di, ek);
            nn = sqrt(dot(nrm, nrm));
        }
        const double sg = dot(nrm, r0) >= 0.0 ? 1.0 : -1.0;
        out.e = v3(sg * nrm.x / nn, sg * nrm.y / nn, sg * nrm.z / nn);
    }
    return out;
}

// ---------------------------------------------------------------------------
// Pair search.  Cells of edge >= reach (max length + diam + cutoff) on a
// periodic grid; rods are binned by centre and copied in cell order so that
// the lanes of a wave, which hold rods of the same cell, read the same
// neighbour-cell entries together.  The stencil offset u of a cell maps to
// the wrapped cell u mod nc and the shift floor(u / nc) of the neighbour.
// ---------------------------------------------------------------------------
struct GridDev {
    int nc[3];
    int S[3];
    double cell[3];
    double box[3];
};

__device__ __forceinline__ int cell_coord(double x, double cell, int nc)
{
    int k = (int)floor(x / cell);
    return k < 0 ? 0 : (k >= nc ? nc - 1 : k);
}

// Spread the low three bits of v to bits 0, 3 and 6.
__device__ __forceinline__ unsigned spread3(unsigned v)
{
    return (v & 1u) | ((v & 2u) << 2) | ((v & 4u) << 4);
}

// The rod's cell (in id) and the same followed by `fb` bits (0, 3, 6 or 9) of
// the Morton code of its sub-cell (fb / 3 bits per direction) for rods that
// are to be ordered by position inside their cells as well.  A rod that is not
// finite goes to cell 0, so that the cell counts stay consistent.
__device__ __forceinline__ unsigned rod_bin(const V3 &xi, const V3 &di, const GridDev &g, int fb, int &id, int &err)
{
    const double xs[3] = {xi.x, xi.y, xi.z};
    id = 0;
    if (!(isfinite(xi.x) && isfinite(xi.y) && isfinite(xi.z) && isfinite(di.x) && isfinite(di.y) && isfinite(di.z))) {
        err = 1;
        return 0;
    }
    int kc[3];
    unsigned sub = 0;
    const int per = fb / 3, side = 1 << per;
    bool inside = true;
    for (int a = 0; a < 3; ++a) {
        inside = inside && xs[a] >= 0.0 && xs[a] < g.box[a];
        kc[a] = cell_coord(xs[a], g.cell[a], g.nc[a]);
        if (per > 0) {
            int f = (int)floor((xs[a] / g.cell[a] - kc[a]) * side);
            f = f < 0 ? 0 : (f >= side ? side - 1 : f);
            sub |= spread3((unsigned)f << (3 - per)) << a;
        }
    }
    err = inside ? 0 : 2;
    id = (kc[0] * g.nc[1] + kc[1]) * g.nc[2] + kc[2];
    return ((unsigned)id << fb) | (sub >> (9 - fb));
}

// bins, counts by bin without its last `drop` bits, and (rank may be null) the
// rod's place among those it is counted with
__global__ void k_bin(int64_t n, const double *__restrict__ x, const double *__restrict__ dir, GridDev g, int fb,
                      int drop, int *__restrict__ cell_of, int *__restrict__ cell_cnt, int *__restrict__ rank,
                      int *__restrict__ err)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    int id, e;
    const unsigned code = rod_bin(load3(x + 3 * i), load3(dir + 3 * i), g, fb, id, e);
    if (e) atomicOr(err, e);
    cell_of[i] = (int)code;
    const int r = atomicAdd(cell_cnt + (code >> drop), 1);
    if (rank) rank[i] = r;
}

// counts of a search, zero when it starts: pairs by rod on either side,
// pairs emitted, errors
struct PairCounts {
    int *p, *q;
    unsigned long long *emitted;
    int *err;
};

// Small systems in cell order by one workgroup: bins, cell offsets and the
// order (by bin, then index) in one launch, with the counts of the search
// cleared on the way.  Bound by latency: of 12 launches (bins, scan, radix
// sort, clears) each takes 1.2 to 5.5 us however little it does.  Up to 4,096
// rods and cells, the LDS of one workgroup; the library's radix sort takes
// over above.  Rods go to buckets (a bin's leading 12 bits), then each to its
// rank in its bucket: 4.6 us at 1,000 rods (a bitonic
// network over the keys took 22).
constexpr int kCellsOne = 4096, kCellsBlock = 1024, kCellsPer = kCellsOne / kCellsBlock;

__global__ void __launch_bounds__(kCellsBlock)
    k_cells_one(int n, const double *__restrict__ x, const double *__restrict__ dir, GridDev g, int fb, int drop,
                int ncell, int *__restrict__ cell_start, int *__restrict__ sorted, PairCounts c)
{
    __shared__ unsigned long long key[kCellsOne];
    __shared__ int off[kCellsOne + 1], part[kCellsBlock / 64], bad;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int u = 0; u < kCellsPer; ++u) off[kCellsPer * tid + u] = 0;
    if (tid == 0) bad = 0;
    __syncthreads();
    int err = 0, place[kCellsPer];
    unsigned code[kCellsPer];
#pragma unroll
    for (int u = 0; u < kCellsPer; ++u) {
        const int i = tid + u * kCellsBlock;
        if (i < n) {
            int id, e;
            code[u] = rod_bin(load3(x + 3 * i), load3(dir + 3 * i), g, fb, id, e);
            err |= e;
            place[u] = atomicAdd(off + (code[u] >> drop), 1);
            c.p[i] = 0;
            c.q[i] = 0;
        }
    }
    if (err) atomicOr(&bad, err);
    __syncthreads();
    int v[kCellsPer], incl = 0;
    for (int u = 0; u < kCellsPer; ++u) incl += v[u] = off[kCellsPer * tid + u];
    const int own = incl;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int t = __shfl_up(incl, d, 64);
        if (lane >= d) incl += t;
    }
    if (lane == 63) part[wave] = incl;
    __syncthreads();
    int run = incl - own;
    for (int w = 0; w < wave; ++w) run += part[w];
    for (int u = 0; u < kCellsPer; ++u) {
        off[kCellsPer * tid + u] = run;
        run += v[u];
    }
    if (tid == kCellsBlock - 1) off[kCellsOne] = run;
    if (tid == 0) {
        *c.emitted = 0;
        *c.err = bad;
    }
    __syncthreads();
    for (int k = tid; k <= ncell; k += kCellsBlock) cell_start[k] = off[k == ncell ? kCellsOne : k << (fb - drop)];
#pragma unroll
    for (int u = 0; u < kCellsPer; ++u) {
        const int i = tid + u * kCellsBlock;
        if (i < n) key[off[code[u] >> drop] + place[u]] = ((unsigned long long)code[u] << 32) | (unsigned)i;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kCellsPer; ++u) {
        const int i = tid + u * kCellsBlock;
        if (i >= n) continue;
        const unsigned long long k = ((unsigned long long)code[u] << 32) | (unsigned)i;
        const int b = off[code[u] >> drop], e = off[(code[u] >> drop) + 1];
        int r = b;
        for (int w = b; w < e; ++w) r += key[w] < k;
        sorted[r] = i;
    }
}

__global__ void k_scatter(int64_t n, const double *__restrict__ x, const double *__restrict__ dir,
                          const double *__restrict__ len, double len0, const int *__restrict__ cell_of,
                          const int *__restrict__ cell_start, const int *__restrict__ rank, int *__restrict__ sorted,
                          double *__restrict__ xs, double *__restrict__ ds, double *__restrict__ ls)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int c = cell_of[i];
    const int slot = cell_start[c] + rank[i];
    sorted[slot] = (int)i;
    store3(xs + 3 * (int64_t)slot, load3(x + 3 * i));
    store3(ds + 3 * (int64_t)slot, load3(dir + 3 * i));
    ls[slot] = len ? len[i] : len0;
}

__device__ __forceinline__ bool lex_positive(int a, int b, int c)
{
    return a > 0 || (a == 0 && (b > 0 || (b == 0 && c > 0)));
}

// The counting and filling passes (rod numbers too large for the 64-bit keys
// of the emitting search below).  INTERNAL: rods are numbered by their
// cell-order slot; otherwise by the caller's index sorted[t].  A pair is
// listed by its smaller rod number (self-images: positive shifts only).
// One workgroup per home cell.  The home cell's rods and then, one stencil
// cell at a time, the neighbour cell's rods (shifted by the periodic image)
// are staged in LDS; every (home, neighbour) combination is tested from LDS in
// parallel with the cheap necessary conditions (centre distance within reach;
// axis lines closer than the threshold).  Survivors go to an LDS queue and get
// the exact closest-point test together.  Counting pass: per-rod counts.
// Filling pass: each pair takes the next slot of its rod (LDS atomic); the
// order within a rod is then fixed by the per-rod sort that follows.
constexpr int kPairBlock = 256;
constexpr int kCellChunk = 256;  // rods of one cell staged at a time
constexpr int kQueue = 4096;     // candidate (home, neighbour) pairs per flush

// The staged copies are FP32, with the centres relative to the home cell's
// corner (so they stay within a few cells of 0 and round finely): the cheap
// tests run on them with margins that cover FP32 rounding, so that they
// never drop a pair the FP64 tests would keep; the exact test of a survivor
// reads the FP64 values from the cell-order arrays.
struct CellStage {
    float p[7][kCellChunk];  // x, y, z (shifted by image - corner), dx, dy, dz, length
    int idx[kCellChunk];     // rod index (the caller's or the cell order's)
};

template <bool INTERNAL>
__device__ __forceinline__ void stage_cell(CellStage &S, int q0, int m, V3 shift, const int *sorted,
                                           const double *xs, const double *ds, const double *ls)
{
    for (int u = threadIdx.x; u < m; u += kPairBlock) {
        const int64_t q = q0 + u;
        S.p[0][u] = (float)(xs[3 * q] + shift.x);
        S.p[1][u] = (float)(xs[3 * q + 1] + shift.y);
        S.p[2][u] = (float)(xs[3 * q + 2] + shift.z);
        S.p[3][u] = (float)ds[3 * q];
        S.p[4][u] = (float)ds[3 * q + 1];
        S.p[5][u] = (float)ds[3 * q + 2];
        S.p[6][u] = (float)ls[q];
        S.idx[u] = INTERNAL ? (int)q : sorted[q];
    }
}

enum PairPass : int { kPairCount = 0, kPairFill = 1 };

template <int PASS, bool INTERNAL>
__global__ void __launch_bounds__(kPairBlock) k_pairs(GridDev g, double diam, double cutoff,
                                                      const int *__restrict__ sorted, const double *__restrict__ xs,
                                                      const double *__restrict__ ds, const double *__restrict__ ls,
                                                      const int *__restrict__ cell_start, int *__restrict__ pcnt,
                                                      const int *__restrict__ poff, int32_t *__restrict__ pi,
                                                      int32_t *__restrict__ pj, int32_t *__restrict__ img,
                                                      uint8_t *__restrict__ flags)
{
    constexpr bool FILL = PASS == kPairFill;
    __shared__ CellStage H, Nb;
    __shared__ int hcnt[kCellChunk], hoff[kCellChunk];
    __shared__ int queue[kQueue];
    __shared__ int qn;
    const int h = blockIdx.x;
    const int hz = h % g.nc[2], hy = (h / g.nc[2]) % g.nc[1], hx = h / (g.nc[2] * g.nc[1]);
    const int hb = cell_start[h], he = cell_start[h + 1];
    const float greach = (float)(diam + cutoff), fgap0 = (float)(diam + cutoff) + 1e-2f;
    const V3 corner = v3(hx * g.cell[0], hy * g.cell[1], hz * g.cell[2]);
    const int NY = 2 * g.S[1] + 1, NZ = 2 * g.S[2] + 1, NS = (2 * g.S[0] + 1) * NY * NZ;
    for (int a0 = hb; a0 < he; a0 += kCellChunk) {
        const int na = he - a0 < kCellChunk ? he - a0 : kCellChunk;
        stage_cell<INTERNAL>(H, a0, na, v3(-corner.x, -corner.y, -corner.z), sorted, xs, ds, ls);
        for (int u = threadIdx.x; u < na; u += kPairBlock) {
            hcnt[u] = 0;
            if (PASS == kPairFill) hoff[u] = poff[INTERNAL ? a0 + u : sorted[a0 + u]];
        }
        __syncthreads();
        for (int sc = 0; sc < NS; ++sc) {
            const int ux = hx + sc / (NY * NZ) - g.S[0];
            const int uy = hy + (sc / NZ) % NY - g.S[1];
            const int uz = hz + sc % NZ - g.S[2];
            const int wx = ((ux % g.nc[0]) + g.nc[0]) % g.nc[0];
            const int wy = ((uy % g.nc[1]) + g.nc[1]) % g.nc[1];
            const int wz = ((uz % g.nc[2]) + g.nc[2]) % g.nc[2];
            const int sx = (ux - wx) / g.nc[0], sy = (uy - wy) / g.nc[1], sz = (uz - wz) / g.nc[2];
            const bool selfok = lex_positive(sx, sy, sz);
            const int packed = ((sx + 8) << 8) | ((sy + 8) << 4) | (sz + 8);
            const V3 shift = v3(sx * g.box[0], sy * g.box[1], sz * g.box[2]);
            const int w = (wx * g.nc[1] + wy) * g.nc[2] + wz;
            const int nb = cell_start[w], ne = cell_start[w + 1];
            for (int b0 = nb; b0 < ne; b0 += kCellChunk) {
                const int nn = ne - b0 < kCellChunk ? ne - b0 : kCellChunk;
                // rods in cell order: a neighbour chunk entirely below the home
                // chunk holds no j >= i
                if (INTERNAL && b0 + nn <= a0) continue;
                __syncthreads();
                stage_cell<INTERNAL>(Nb, b0, nn, v3(shift.x - corner.x, shift.y - corner.y, shift.z - corner.z),
                                     sorted, xs, ds, ls);
                __syncthreads();
                const int total = na * nn;
                // (a, b) of entry e = a nn + b, advanced by kPairBlock entries
                // per step without a division
                const int step_a = kPairBlock / nn, step_b = kPairBlock % nn;
                for (int base = 0; base < total; base += kQueue) {
                    if (threadIdx.x == 0) qn = 0;
                    __syncthreads();
                    const int lim = total - base < kQueue ? total - base : kQueue;
                    int a = (base + (int)threadIdx.x) / nn, b = (base + (int)threadIdx.x) - a * nn;
                    for (int e = threadIdx.x; e < lim; e += kPairBlock) {
                        const int ca = a, cb = b;
                        a += step_a;
                        b += step_b;
                        if (b >= nn) {
                            b -= nn;
                            ++a;
                        }
                        const int i = H.idx[ca], j = Nb.idx[cb];
                        if (j < i || (j == i && !selfok)) continue;
                        const float rx = H.p[0][ca] - Nb.p[0][cb], ry = H.p[1][ca] - Nb.p[1][cb],
                                    rz = H.p[2][ca] - Nb.p[2][cb];
                        const float reach0 = 0.5f * (H.p[6][ca] + Nb.p[6][cb]) + greach;
                        const float reach = reach0 * (1.0f + 1e-5f) + 1e-3f;
                        if (rx * rx + ry * ry + rz * rz >= reach * reach) continue;
                        // two segments are never closer than their axis lines
                        // (near-parallel lines go through)
                        const float ax = H.p[3][ca], ay = H.p[4][ca], az = H.p[5][ca];
                        const float bx = Nb.p[3][cb], by = Nb.p[4][cb], bz = Nb.p[5][cb];
                        const float nx = ay * bz - az * by, ny = az * bx - ax * bz, nz = ax * by - ay * bx;
                        const float nn2 = nx * nx + ny * ny + nz * nz, rn = rx * nx + ry * ny + rz * nz;
                        const float fgap = fgap0 + 1e-2f * reach0;
                        if (nn2 > 1e-5f && rn * rn > fgap * fgap * nn2) continue;
                        queue[atomicAdd(&qn, 1)] = (ca << 16) | cb;
                    }
                    __syncthreads();
                    const int nq = qn;
                    for (int u = threadIdx.x; u < nq; u += kPairBlock) {
                        const int a = (queue[u] >> 16) & 0xff, b = queue[u] & 0xff;
                        const int64_t qa = a0 + a, qb = b0 + b;
                        const V3 xi = load3(xs + 3 * qa), di = load3(ds + 3 * qa);
                        const V3 xq = load3(xs + 3 * qb), dj = load3(ds + 3 * qb);
                        const V3 xj = v3(xq.x + shift.x, xq.y + shift.y, xq.z + shift.z);
                        const Contact c = closest_point(xi, di, 0.5 * ls[qa], xj, dj, 0.5 * ls[qb]);
                        const double phi = c.dist - diam;
                        if (!(phi < cutoff)) continue;
                        const unsigned fl = c.flags | (fabs(phi - cutoff) <= kCutoffBand ? 1u : 0u);
                        const int slot = atomicAdd(&hcnt[a], 1);
                        if (FILL) {
                            const int o = hoff[a] + slot;
                            pi[o] = H.idx[a];
                            pj[o] = Nb.idx[b];
                            img[o] = packed;
                            if (flags) flags[o] = (uint8_t)fl;
                        }
                    }
                    __syncthreads();
                }
            }
        }
        if (PASS == kPairCount)
            for (int u = threadIdx.x; u < na; u += kPairBlock) pcnt[H.idx[u]] = hcnt[u];
        __syncthreads();
    }
}

// The emitting search: every pair once as a key (pi, pj, shift) with its flags,
// counted on both rods; the list is put in canonical order afterwards.  A
// workgroup stages the rods of a home cell; a wave takes a cell of the half of
// the stencil that meets every pair and image once (its jobs: these cells, by
// parts of the home rods), holds 64 of its rods in registers, a lane each, and
// runs through the home rods in reach of each 16 of them.  Where the numbers
// run the other way the pair is turned round before the exact test.  Survivors
// of the cheap tests go to the wave's queue and get the exact test 64 at a
// time, so the waves never wait for each other and the exact test has full
// waves.  Bound by the issue of the cheap tests (33 vector instructions a row
// of 64) and the imbalance of the jobs.  100,000 rods of the paper's
// suspension, 469,000 pairs: 265 us in the caller's order, 239 in cell order;
// 701 and 263 when workgroups staged both cells, queued and tested together,
// and the caller's order met every pair from both sides.  1,000 rods: 11.8 us
// (18.9).
// The staged values are FP32, with the centres relative to the home cell's
// corner (so they stay within a few cells of 0 and round finely): the cheap
// tests have margins that cover FP32 rounding, so that they never drop a pair
// the FP64 tests would keep; the exact test reads the FP64 values.
constexpr int kEmitWaves = kPairBlock / 64, kEmitHold = 512, kRows = 4;

__device__ __forceinline__ float lane_f32(float v, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// hmax: half length of the longest rod
template <bool INTERNAL>
__global__ void __launch_bounds__(kPairBlock)
    k_pairs_emit(GridDev g, int cshift, double diam, double cutoff, const int *__restrict__ sorted,
                 const double *__restrict__ xs, const double *__restrict__ ds, const double *__restrict__ ls,
                 const int *__restrict__ cell_start, PairCounts ec, unsigned long long *__restrict__ ekeys,
                 uint8_t *__restrict__ eflags, int2 *__restrict__ erank, int64_t ecap, int kshift, int split,
                 int rparts, float hmax)
{
    __shared__ float4 Hp[kCellChunk + 1], Hd[kCellChunk + 1];  // centre and half length; director (last: far away)
    __shared__ int2 queue[kEmitWaves][64 * (kRows + 1)];  // (home rod << 12 | image, neighbour's slot)
    // home rods in reach of each 16 of a wave's rods, to a multiple of kRows
    __shared__ __align__(8) unsigned short list[kEmitWaves][4][kCellChunk + kRows];
    // pairs found, so that a workgroup reserves its place in the list once
    // (atomics on one word take about 20 ns each, whoever issues them)
    __shared__ unsigned long long okey[kEmitHold];
    __shared__ unsigned long long obase;
    __shared__ uint8_t oflag[kEmitHold];
    __shared__ int on, ofull;  // places taken; the first one of those without room
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int h = blockIdx.x / split, part = blockIdx.x % split;
    const int hz = h % g.nc[2], hy = (h / g.nc[2]) % g.nc[1], hx = h / (g.nc[2] * g.nc[1]);
    const int hb = cell_start[h << cshift], he = cell_start[(h + 1) << cshift];
    // FP32 margins.  Staged centres lie within S + 1 cells of the corner (S <=
    // 7), so a component of r0 carries at most 1e-6 x cell of rounding, and
    // directions 6e-8 per component.  The reach test gets 1e-3 + 1e-5 x reach
    // more.  The axis-line test runs only where |d_i x d_j|^2 > 1e-5 (|n| >
    // 3.1e-3) and gets 1e-2 x (1 + reach) on the gap: the rounding of r0 . n,
    // below 2.2e-6 x reach (cell <= reach), is then under a tenth of
    // margin x |n|.
    const float greach = (float)(diam + cutoff), fgap0 = (float)(diam + cutoff) + 1e-2f;
    const V3 corner = v3(hx * g.cell[0], hy * g.cell[1], hz * g.cell[2]);
    const int NY = 2 * g.S[1] + 1, NZ = 2 * g.S[2] + 1, NS = (2 * g.S[0] + 1) * NY * NZ;
    const int NJ = NS / 2 + 1;  // the home cell itself and the half of the stencil after it
    if (threadIdx.x == 0) {
        on = 0;
        ofull = kEmitHold;
        Hp[kCellChunk] = make_float4(-1e18f, 0.0f, 0.0f, 0.0f);  // (a lane without a rod is at +1e18)
        Hd[kCellChunk] = make_float4(0.0f, 0.0f, 1.0f, 0.0f);
    }
    auto emit = [&](unsigned long long o, unsigned long long key, unsigned fl) {
        if (o >= (unsigned long long)ecap) return;
        const int i = (int)(key >> kshift), j = (int)((key >> 12) & ((1ull << (kshift - 12)) - 1ull));
        erank[o] = make_int2(atomicAdd(ec.p + i, 1), ec.q ? atomicAdd(ec.q + j, 1) : 0);
        ekeys[o] = key;
        eflags[o] = (uint8_t)fl;
    };
    for (int a0 = hb; a0 < he; a0 += kCellChunk) {
        const int na = min(he - a0, kCellChunk);
        __syncthreads();
        for (int u = threadIdx.x; u < na; u += kPairBlock) {
            const int64_t q = a0 + u;
            Hp[u] = make_float4((float)(xs[3 * q] - corner.x), (float)(xs[3 * q + 1] - corner.y),
                                (float)(xs[3 * q + 2] - corner.z), 0.5f * (float)ls[q] * (1.0f + 1e-5f));
            Hd[u] = make_float4((float)ds[3 * q], (float)ds[3 * q + 1], (float)ds[3 * q + 2], 0.0f);
        }
        __syncthreads();
        int qn = 0;  // entries in the wave's queue
        auto flush = [&](int cnt) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            qn -= cnt;
            bool hit = false;
            int i = 0, j = 0, image = 0;
            unsigned fl = 0;
            if (lane < cnt) {
                const int2 v = queue[wave][qn + lane];
                const int ha = a0 + (v.x >> 12), hq = v.y;
                image = v.x & 0xfff;
                i = INTERNAL ? ha : sorted[ha];
                j = INTERNAL ? hq : sorted[hq];
                const bool turn = j < i;
                if (turn) {
                    const int k = i;
                    i = j;
                    j = k;
                    image = 0x1110 - image;  // each shift s + 8 becomes 16 - (s + 8)
                }
                const int64_t qa = turn ? hq : ha, qb = turn ? ha : hq;
                const V3 xi = load3(xs + 3 * qa), di = load3(ds + 3 * qa);
                const V3 xj = load3(xs + 3 * qb) + v3((((image >> 8) & 15) - 8) * g.box[0],
                                                      (((image >> 4) & 15) - 8) * g.box[1],
                                                      ((image & 15) - 8) * g.box[2]);
                const Contact c = closest_point(xi, di, 0.5 * ls[qa], xj, load3(ds + 3 * qb), 0.5 * ls[qb]);
                const double phi = c.dist - diam;
                hit = phi < cutoff;
                fl = c.flags | (fabs(phi - cutoff) <= kCutoffBand ? 1u : 0u);
            }
            const unsigned long long m = __ballot(hit);
            if (m == 0) return;
            const unsigned long long key = ((unsigned long long)(unsigned)i << kshift) |
                                           ((unsigned long long)(unsigned)j << 12) | (unsigned long long)image;
            const int mine = __popcll(m & ((1ull << lane) - 1ull));
            int at = 0;
            if (lane == 0) at = atomicAdd(&on, __popcll(m));
            at = __builtin_amdgcn_readfirstlane(at);
            if (at + __popcll(m) <= kEmitHold) {
                if (hit) {
                    okey[at + mine] = key;
                    oflag[at + mine] = (uint8_t)fl;
                }
                return;
            }
            // no room: straight to the list
            unsigned long long base = 0;
            if (lane == 0) atomicMin(&ofull, at);
            if (lane == 0) base = atomicAdd(ec.emitted, (unsigned long long)__popcll(m));
            base = (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(base >> 32)) << 32 |
                   (unsigned)__builtin_amdgcn_readfirstlane((int)base);
            if (hit) emit(base + mine, key, fl);
        };
        for (int job = part * kEmitWaves + wave; job < NJ * rparts; job += split * kEmitWaves) {
            const int sc = NS / 2 + job % NJ, rp = job / NJ;
            const int ux = hx + sc / (NY * NZ) - g.S[0];
            const int uy = hy + (sc / NZ) % NY - g.S[1];
            const int uz = hz + sc % NZ - g.S[2];
            const int wx = ((ux % g.nc[0]) + g.nc[0]) % g.nc[0];
            const int wy = ((uy % g.nc[1]) + g.nc[1]) % g.nc[1];
            const int wz = ((uz % g.nc[2]) + g.nc[2]) % g.nc[2];
            const int w = (wx * g.nc[1] + wy) * g.nc[2] + wz;
            const int sx = (ux - wx) / g.nc[0], sy = (uy - wy) / g.nc[1], sz = (uz - wz) / g.nc[2];
            const int packed = ((sx + 8) << 8) | ((sy + 8) << 4) | (sz + 8);
            const V3 shift = v3(sx * g.box[0] - corner.x, sy * g.box[1] - corner.y, sz * g.box[2] - corner.z);
            const int nb = cell_start[w << cshift], ne = cell_start[(w + 1) << cshift];
            const int r0 = (int)((int64_t)na * rp / rparts), r1 = (int)((int64_t)na * (rp + 1) / rparts);
            for (int b0 = nb; b0 < ne; b0 += 64) {
                const int64_t q = min(b0 + lane, ne - 1);
                const bool mine = b0 + lane < ne;
                const float bx = mine ? (float)(xs[3 * q] + shift.x) : 1e18f, by = (float)(xs[3 * q + 1] + shift.y),
                            bz = (float)(xs[3 * q + 2] + shift.z);
                const float breach = (0.5f * (float)ls[q] + greach) * (1.0f + 1e-5f) + 1e-3f;
                const float ex = (float)ds[3 * q], ey = (float)ds[3 * q + 1], ez = (float)ds[3 * q + 2];
                // a ball around each 16 of the rods, and the home rods in reach
                // of it; in the home cell itself those before the lane's own
                const bool same = sc == NS / 2;
                const int last = same ? b0 + lane - a0 - 1 : kCellChunk;
                const int g0 = lane & 48, l1 = min(15, ne - 1 - b0 - g0);
                auto mid = [&](float v) {
                    return 0.5f * (__shfl(v, g0 + max(0, l1 / 4), 64) + __shfl(v, g0 + max(0, (3 * l1 + 3) / 4), 64));
                };
                const float cx = mid(bx), cy = mid(by), cz = mid(bz);
                float far2 = 0.0f;
                if (mine) far2 = (bx - cx) * (bx - cx) + (by - cy) * (by - cy) + (bz - cz) * (bz - cz);
#pragma unroll
                for (int o = 1; o < 16; o <<= 1) far2 = fmaxf(far2, __shfl_xor(far2, o, 64));
                const float cover = (sqrtf(far2) + (hmax + greach) * (1.0f + 1e-5f)) * (1.0f + 1e-5f) + 2e-3f;
                int longest = 0, held[4];
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    int cnt = 0;
                    const float ux = lane_f32(cx, 16 * q4), uy = lane_f32(cy, 16 * q4), uz = lane_f32(cz, 16 * q4),
                                uc = lane_f32(cover, 16 * q4);
                    const int rend = b0 + 16 * q4 >= ne ? r0 : (same ? min(r1, b0 + 16 * q4 + 15 - a0) : r1);
                    for (int s0 = r0; s0 < rend; s0 += 64) {
                        const float4 p = Hp[min(s0 + lane, na - 1)];
                        const float rx = p.x - ux, ry = p.y - uy, rz = p.z - uz, r = p.w + uc;
                        const bool in = (s0 + lane < rend) & (rx * rx + ry * ry + rz * rz < r * r);
                        const unsigned long long m = __ballot(in);
                        if (in)
                            list[wave][q4][cnt + __popcll(m & ((1ull << lane) - 1ull))] = (unsigned short)(s0 + lane);
                        cnt += __popcll(m);
                    }
                    longest = max(longest, cnt);
                    held[q4] = cnt;
                }
                longest = (longest + kRows - 1) / kRows * kRows;
                for (int q4 = 0; q4 < 4; ++q4)
                    for (int u = held[q4] + lane; u < longest; u += 64) list[wave][q4][u] = kCellChunk;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                // kRows of them at a time, without a branch between: a row is a
                // chain of about 400 clocks
                for (int it = 0; it < longest; it += kRows) {
                    int a[kRows];
                    float4 p[kRows], d[kRows];
                    unsigned long long m[kRows], any = 0;
                    const ushort4 rows = *reinterpret_cast<const ushort4 *>(&list[wave][lane >> 4][it]);
                    a[0] = rows.x;
                    a[1] = rows.y;
                    a[2] = rows.z;
                    a[3] = rows.w;
#pragma unroll
                    for (int k = 0; k < kRows; ++k) {
                        p[k] = Hp[a[k]];
                        d[k] = Hd[a[k]];
                    }
#pragma unroll
                    for (int k = 0; k < kRows; ++k) {
                        const float rx = p[k].x - bx, ry = p[k].y - by, rz = p[k].z - bz;
                        const float reach = p[k].w + breach;
                        const bool near = (a[k] <= last) & (rx * rx + ry * ry + rz * rz < reach * reach);
                        // two segments are never closer than their axis
                        // lines (near-parallel lines go through)
                        const float nx = d[k].y * ez - d[k].z * ey, ny = d[k].z * ex - d[k].x * ez,
                                    nz = d[k].x * ey - d[k].y * ex;
                        const float nn2 = nx * nx + ny * ny + nz * nz, rn = rx * nx + ry * ny + rz * nz;
                        const float fgap = fgap0 + 1e-2f * reach;
                        m[k] = __ballot(near & !((nn2 > 1e-5f) & (rn * rn > fgap * fgap * nn2)));
                        any |= m[k];
                    }
                    if (any == 0) continue;
#pragma unroll
                    for (int k = 0; k < kRows; ++k) {
                        if ((m[k] >> lane) & 1ull)
                            queue[wave][qn + __popcll(m[k] & ((1ull << lane) - 1ull))] =
                                make_int2((a[k] << 12) | packed, b0 + lane);
                        qn += __popcll(m[k]);
                    }
                    while (qn >= 64) flush(64);
                }
            }
        }
        if (qn > 0) flush(qn);
    }
    __syncthreads();
    const int n_out = min(on, ofull);
    if (n_out == 0) return;
    if (threadIdx.x == 0) obase = atomicAdd(ec.emitted, (unsigned long long)n_out);
    __syncthreads();
    for (int u = threadIdx.x; u < n_out; u += kPairBlock) emit(obase + u, okey[u], oflag[u]);
}

// Emitted pair keys (pi, pj, shift) into the canonical order: bucketed by pi
// with the ranks that the counting gave, then each pair to the place of its
// key among its bucket's (a lane per pair reads the bucket: 4.7 pairs on
// average at 100,000 rods, 468,000 pairs).  The keys are distinct, so the
// result is the order of the keys whatever order the counting took.  qtmp
// (may be null): the pairs of each second rod, at the offsets qoff.
__global__ void k_pair_bucket(int64_t m, const unsigned long long *__restrict__ keys, const int2 *__restrict__ rank,
                              int kshift, const int *__restrict__ off, int *__restrict__ slot)
{
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= m) return;
    slot[off[keys[t] >> kshift] + rank[t].x] = (int)t;
}

__global__ void k_pair_place(int64_t m, const unsigned long long *__restrict__ keys,
                             const uint8_t *__restrict__ kflags, const int2 *__restrict__ rank, int kshift,
                             const int *__restrict__ off, const int *__restrict__ slot, int32_t *__restrict__ pi,
                             int32_t *__restrict__ pj, int32_t *__restrict__ img, uint8_t *__restrict__ flags,
                             const int *__restrict__ qoff, int32_t *__restrict__ qtmp)
{
    const int64_t s = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (s >= m) return;
    const int t = slot[s];
    const unsigned long long k = keys[t];
    const int a = (int)(k >> kshift), b = off[a], e = off[a + 1];
    int c = b;
    for (int u = b; u < e; ++u) c += keys[slot[u]] < k;
    pi[c] = a;
    const int j = (int)((k >> 12) & ((1ull << (kshift - 12)) - 1ull));
    pj[c] = j;
    img[c] = (int32_t)(k & 0xfffull);
    if (flags) flags[c] = kflags[t];
    if (qtmp) qtmp[qoff[j] + rank[t].y] = c;
}

// velocity of a rod under its external force and torque alone
__device__ __forceinline__ void rod_unc(const Mob &m, const V3 &d, const V3 &f, const V3 &tq, double *out)
{
    // (fused by hand, so that every kernel rounds alike)
    const double k = (m.apar - m.aperp) * fma(d.z, f.z, fma(d.x, f.x, d.y * f.y));
    store3(out, v3(fma(m.aperp, f.x, k * d.x), fma(m.aperp, f.y, k * d.y), fma(m.aperp, f.z, k * d.z)));
    store3(out + 3, m.rperp * tq);  // axial rotational mobility equals the normal one
}

// copies of centres, directors and lengths in cell order, and the velocities
// of the forces (Unc null: not asked for)
__global__ void k_gather_rods(int64_t n, const int *__restrict__ perm, const double *__restrict__ x,
                              const double *__restrict__ dir, const double *__restrict__ len, double len0,
                              double *__restrict__ xs, double *__restrict__ ds, double *__restrict__ ls, Mob mob,
                              double diam, double eta, const double *__restrict__ F, double *__restrict__ Unc)
{
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= n) return;
    const int64_t i = perm[t];
    const V3 d = load3(dir + 3 * i);
    store3(xs + 3 * t, load3(x + 3 * i));
    store3(ds + 3 * t, d);
    ls[t] = len ? len[i] : len0;
    if (!Unc) return;
    V3 f = v3(0, 0, 0), tq = v3(0, 0, 0);
    if (F) {
        f = load3(F + 6 * i);
        tq = load3(F + 6 * i + 3);
    }
    rod_unc(len ? mobility_of(len[i], diam, eta) : mob, d, f, tq, Unc + 6 * t);
}

// order each rod's pairs by (pj, img) (lists from the counting and filling
// passes).  Up to 32 pairs (every rod at the paper's densities)
// are sorted in registers by an odd-even transposition network over keys
// (pj, img, flags) packed into 64 bits, so the loads go out together and the
// stores once; longer lists take an insertion sort in memory.
constexpr int kSortRegs = 32;

// (256-thread groups, so that the 32 keys stay in registers)
__global__ void __launch_bounds__(256)
    k_sort_pairs(int64_t n, const int *__restrict__ poff, int32_t *__restrict__ pj, int32_t *__restrict__ img,
                 uint8_t *__restrict__ flags)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int b = poff[i], e = poff[i + 1];
    const int cnt = e - b;
    if (cnt <= 1) return;
    if (cnt <= kSortRegs) {
        unsigned long long key[kSortRegs];
#pragma unroll
        for (int k = 0; k < kSortRegs; ++k)
            key[k] = k < cnt ? ((unsigned long long)(unsigned)pj[b + k] << 16) |
                                   ((unsigned long long)(unsigned)img[b + k] << 4) |
                                   (unsigned long long)(flags ? flags[b + k] : 0)
                             : ~0ull;
#pragma unroll
        for (int r = 0; r < kSortRegs; ++r)
#pragma unroll
            for (int k = r & 1; k + 1 < kSortRegs; k += 2) {
                const unsigned long long lo = key[k] < key[k + 1] ? key[k] : key[k + 1];
                const unsigned long long hi = key[k] < key[k + 1] ? key[k + 1] : key[k];
                key[k] = lo;
                key[k + 1] = hi;
            }
#pragma unroll
        for (int k = 0; k < kSortRegs; ++k)
            if (k < cnt) {
                pj[b + k] = (int32_t)(key[k] >> 16);
                img[b + k] = (int32_t)((key[k] >> 4) & 0xfffull);
                if (flags) flags[b + k] = (uint8_t)(key[k] & 15ull);
            }
        return;
    }
    for (int k = b + 1; k < e; ++k) {
        const int32_t kj = pj[k], ki = img[k];
        const uint8_t kf = flags ? flags[k] : 0;
        const long long key = ((long long)kj << 12) | ki;
        int m = k - 1;
        while (m >= b && (((long long)pj[m] << 12) | img[m]) > key) {
            pj[m + 1] = pj[m];
            img[m + 1] = img[m];
            if (flags) flags[m + 1] = flags[m];
            --m;
        }
        pj[m + 1] = kj;
        img[m + 1] = ki;
        if (flags) flags[m + 1] = kf;
    }
}

__global__ void k_len_max(int64_t n, const double *__restrict__ len, unsigned long long *__restrict__ out,
                          int *__restrict__ err)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double L = len[i];
    if (!(L > 0.0) || !isfinite(L)) {
        atomicOr(err, 4);
        return;
    }
    // positive doubles order like their bit patterns
    atomicMax(out, (unsigned long long)__double_as_longlong(L));
}

static inline unsigned grid_of(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

// Shared body of the two pair searches.  internal = false: canonical list
// in the caller's rod numbering; internal = true: rods renumbered in cell
// order (stable by caller index), h's workspace keeps the order and copies,
// Unc the velocities of the forces F, and ix where the constraints of each rod
// are.
static int pairs_core(rl_ctx *h, int64_t n, const double *x, const double *dir, const double *len, double len0,
                      bool internal, const double *F, double *Unc, int64_t capacity, int32_t *pi, int32_t *pj,
                      int32_t *img, uint8_t *flags, int64_t *n_pairs, PairIndex *ix)
{
    hipStream_t st = h->stream;
    const rl_params &p = h->prm;
    int werr = 0;
    if (n_pairs) *n_pairs = 0;
    if (n == 0) return RL_OK;
    // longest rod
    double Lmax = len0;
    if (len) {
        RL_HIP(hipMemsetAsync(h->flag_dev, 0, sizeof(int) * 4, st));
        auto *lm = (unsigned long long *)ws_get(h, kWsLenMax, sizeof(unsigned long long), &werr);
        if (werr) return werr;
        RL_HIP(hipMemsetAsync(lm, 0, sizeof(unsigned long long), st));
        hipLaunchKernelGGL(k_len_max, dim3(grid_of(n)), dim3(kBlock), 0, st, n, len, lm, h->flag_dev);
        RL_HIP(hipGetLastError());
        RL_HIP(hipMemcpyAsync(h->host_scratch, lm, sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
        RL_HIP(hipMemcpyAsync(h->host_scratch + 1, h->flag_dev, sizeof(int), hipMemcpyDeviceToHost, st));
        RL_HIP(hipStreamSynchronize(st));
        if (((int *)(h->host_scratch + 1))[0] & 4) {
            set_error("pair search: rod lengths must be finite and > 0");
            return RL_ERR_ARG;
        }
        unsigned long long bits = (unsigned long long)h->host_scratch[0];
        std::memcpy(&Lmax, &bits, sizeof(double));
    } else if (!(len0 > 0.0)) {
        set_error("pair search: len0 must be > 0");
        return RL_ERR_ARG;
    }
    const double reach = Lmax + p.diam + p.cutoff;
    GridDev g;
    int64_t ncell = 1;
    for (int a = 0; a < 3; ++a) {
        int nca = (int)floor(p.box[a] / reach);
        if (nca < 1) nca = 1;
        if (nca > 1024) nca = 1024;
        g.nc[a] = nca;
        g.cell[a] = p.box[a] / nca;
        g.S[a] = (int)ceil(reach / g.cell[a]);
        g.box[a] = p.box[a];
        if (g.S[a] > 7) {
            set_error("pair search: box edge %g too small for rod reach %g (needs box >= reach/7)", p.box[a], reach);
            return RL_ERR_ARG;
        }
        ncell *= nca;
    }
    if (ncell > (1 << 26)) {
        set_error("pair search: too many cells (%lld)", (long long)ncell);
        return RL_ERR_ARG;
    }
    // internal order: by cell, then along a Morton curve of 8^3 sub-cells
    // inside the cell (fewer when the cell ids leave no room in 31 bits), so
    // that rods with consecutive numbers are close in space and so are their
    // partners' records in the solver's Q-side arrays.  The caller's order
    // needs none inside the cells, but the emitting search is faster when 64
    // rods in a row are neighbours: there the bins are octants of the cells.
    int cbits = 1, ibits = 1;
    while ((1LL << cbits) < ncell) ++cbits;
    while ((1LL << ibits) < n) ++ibits;
    const bool emit = 2 * ibits + 12 <= 64;
    const int cshift = !internal && emit && ncell <= (1 << 20) ? 3 : 0;
    const int fb = internal ? std::min(9, (31 - cbits) / 3 * 3) : cshift;
    const int64_t nbin = ncell << cshift;
    int *cell_of = (int *)ws_get(h, kWsCellOf, sizeof(int) * n, &werr);
    // emitted (8 bytes), errors, then the counts by cell and by rod
    int *counts = (int *)ws_get(h, kWsPairCnt, sizeof(int) * (4 + nbin + 2 * n), &werr);
    int *cell_start = (int *)ws_get(h, kWsCellStart, sizeof(int) * (nbin + 1), &werr);
    int *cell_rank = internal ? nullptr : (int *)ws_get(h, kWsCellCur, sizeof(int) * n, &werr);
    int *sorted = (int *)ws_get(h, kWsSorted, sizeof(int) * n, &werr);
    int *cell_key = internal ? (int *)ws_get(h, kWsCellKey, sizeof(int) * n, &werr) : nullptr;
    double *xs = (double *)ws_get(h, kWsXs, sizeof(double) * 3 * n, &werr);
    double *ds = (double *)ws_get(h, kWsDs, sizeof(double) * 3 * n, &werr);
    double *ls = (double *)ws_get(h, kWsLs, sizeof(double) * n, &werr);
    int *poff = (int *)ws_get(h, kWsPoff, sizeof(int) * (n + 1), &werr);
    int *qoff = internal ? (int *)ws_get(h, kWsQptr, sizeof(int) * (n + 1), &werr) : nullptr;
    int64_t *tot = (int64_t *)ws_get(h, kWsScan, sizeof(int64_t) * 2, &werr);
    if (werr) return werr;
    int *cell_cnt = counts + 4, *pcnt = cell_cnt + nbin;
    const PairCounts ec{pcnt, internal ? pcnt + n : nullptr, (unsigned long long *)counts, counts + 2};

    if (internal && n <= kCellsOne && ncell <= kCellsOne) {
        hipLaunchKernelGGL(k_cells_one, dim3(1), dim3(kCellsBlock), 0, st, (int)n, x, dir, g, fb,
                           std::max(0, cbits + fb - 12), (int)ncell, cell_start, sorted, ec);
        RL_HIP(hipGetLastError());
    } else {
        RL_HIP(hipMemsetAsync(counts, 0, sizeof(int) * (4 + nbin + 2 * n), st));
        hipLaunchKernelGGL(k_bin, dim3(grid_of(n)), dim3(kBlock), 0, st, n, x, dir, g, fb, fb - cshift, cell_of,
                           cell_cnt, cell_rank, ec.err);
        RL_HIP(hipGetLastError());
        int rc = device_scan(h, cell_cnt, nbin, cell_start, nullptr);
        if (!rc && internal) rc = stable_sort_by_key(h, n, cell_of, cbits + fb, cell_key, sorted);
        if (rc) return rc;
    }
    if (internal)
        hipLaunchKernelGGL(k_gather_rods, dim3(grid_of(n)), dim3(kBlock), 0, st, n, (const int *)sorted, x, dir, len,
                           len0, xs, ds, ls, mobility_of(len ? 1.0 : len0, p.diam, p.eta), p.diam, p.eta, F, Unc);
    else
        hipLaunchKernelGGL(k_scatter, dim3(grid_of(n)), dim3(kBlock), 0, st, n, x, dir, len, len0, cell_of,
                           cell_start, (const int *)cell_rank, sorted, xs, ds, ls);
    RL_HIP(hipGetLastError());
    // one pass emitting keys (pi, pj, shift), then buckets by pi and ranks in
    // them for the canonical order; rod counts above 2^26 do not fit the
    // 64-bit key and take the counting and filling passes instead
    const dim3 pgrid((unsigned)ncell), pblock(kPairBlock);
    const bool one = n <= kScanOne;
    const int kshift = ibits + 12;
    unsigned long long *ekeys = nullptr;
    uint8_t *eflags = nullptr;
    int2 *erank = nullptr;
    int *pslot = nullptr;
    auto search = [&](auto pass) {
        constexpr int PASS = decltype(pass)::value;
        if (internal)
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_pairs<PASS, true>), pgrid, pblock, 0, st, g, p.diam, p.cutoff, sorted,
                               xs, ds, ls, cell_start, pcnt, (const int *)poff, pi, pj, img, flags);
        else
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_pairs<PASS, false>), pgrid, pblock, 0, st, g, p.diam, p.cutoff,
                               sorted, xs, ds, ls, cell_start, pcnt, (const int *)poff, pi, pj, img, flags);
        return hipGetLastError();
    };
    bool reported = false;
    int64_t total = 0;
    if (emit) {
        // two waves per neighbour cell, each on a part of the home rods, up to
        // about 1,500 cells (100,000 rods, 729 cells: 422 us for the whole
        // search with one, 352 with two, 359 with three, 390 with four), four
        // where there are few
        const int64_t ns = (int64_t)(2 * g.S[0] + 1) * (2 * g.S[1] + 1) * (2 * g.S[2] + 1);
        const int rparts = (int)std::max<int64_t>(1, std::min<int64_t>(4, 40000 / (ncell * ns)));
        const int split = (int)std::max<int64_t>(
            1, std::min<int64_t>(((ns / 2 + 1) * rparts + kEmitWaves - 1) / kEmitWaves, 8192 / ncell));
        // The workspace follows the pairs there are, not the room that the
        // caller has for them: at first as many as it holds, in a new handle 32
        // per rod (the densest suspensions have 12); a search that finds more
        // runs again.
        const int64_t room = std::max<int64_t>(capacity, 0), holds = (int64_t)(h->cap[kWsEmit] / kEmitBytes);
        int64_t ecap = internal ? room : std::min(room, holds > 0 ? holds : 32 * n + 4096);
        for (;; ecap = total) {
            const int64_t eb = std::max<int64_t>(ecap, 1);
            ekeys = (unsigned long long *)ws_get(h, kWsEmit, (size_t)kEmitBytes * eb, &werr);
            if (werr) return werr;
            erank = (int2 *)(ekeys + eb);
            pslot = (int *)(erank + eb);
            eflags = (uint8_t *)(pslot + eb);
            auto go = [&](auto order) {
                hipLaunchKernelGGL(HIP_KERNEL_NAME(k_pairs_emit<decltype(order)::value>),
                                   dim3((unsigned)(ncell * split)), pblock, 0, st, g, cshift, p.diam, p.cutoff,
                                   (const int *)sorted, (const double *)xs, (const double *)ds, (const double *)ls,
                                   (const int *)cell_start, ec, ekeys, eflags, erank, ecap, kshift, split, rparts,
                                   0.5f * (float)Lmax * (1.0f + 1e-6f));
                return hipGetLastError();
            };
            RL_HIP(internal ? go(std::true_type{}) : go(std::false_type{}));
            if (one) {
                // the offsets while the host learns the number of pairs
                RL_HIP(launch_scan_one(st, n, pcnt, poff, ec.q, qoff, nullptr,
                                       ScanReport{ec.emitted, ec.err, h->host_scratch}));
                reported = true;
            } else {
                RL_HIP(hipMemcpyAsync(h->host_scratch, counts, 2 * sizeof(int64_t), hipMemcpyDeviceToHost, st));
            }
            RL_HIP(hipStreamSynchronize(st));
            total = h->host_scratch[0];
            if (total <= ecap || total > capacity || ((int *)(h->host_scratch + 1))[0]) break;
            RL_HIP(hipMemsetAsync(ec.emitted, 0, sizeof(*ec.emitted), st));
            RL_HIP(hipMemsetAsync(pcnt, 0, sizeof(int) * n, st));
        }
    } else {
        RL_HIP(search(std::integral_constant<int, kPairCount>{}));
        const int rc = device_scan(h, pcnt, n, poff, tot);
        if (rc) return rc;
        RL_HIP(hipMemcpyAsync(h->host_scratch, tot, sizeof(int64_t), hipMemcpyDeviceToHost, st));
        RL_HIP(hipMemcpyAsync(h->host_scratch + 1, ec.err, sizeof(int), hipMemcpyDeviceToHost, st));
        RL_HIP(hipStreamSynchronize(st));
        total = h->host_scratch[0];
    }
    const int ferr = ((int *)(h->host_scratch + 1))[0];
    if (ferr & 1) {
        set_error("pair search: non-finite centre or director");
        return RL_ERR_NONFINITE;
    }
    if (ferr & 2) {
        set_error("pair search: a centre lies outside [0, box)");
        return RL_ERR_ARG;
    }
    if (n_pairs) *n_pairs = total;
    if (total > capacity) {
        set_error("pair search: %lld pairs exceed capacity %lld", (long long)total, (long long)capacity);
        return RL_ERR_CAPACITY;
    }
    if (total > 0x7fffffffLL) {
        set_error("pair search: pair count overflows int32");
        return RL_ERR_CAPACITY;
    }
    if (total == 0) return RL_OK;
    if (emit) {
        if (!reported) {
            int rc = device_scan(h, pcnt, n, poff, nullptr);
            if (!rc && internal) rc = device_scan(h, ec.q, n, qoff, nullptr);
            if (rc) return rc;
        }
        int32_t *qtmp = internal ? (int32_t *)ws_get(h, kWsQtmp, sizeof(int32_t) * total, &werr) : nullptr;
        if (werr) return werr;
        hipLaunchKernelGGL(k_pair_bucket, dim3(grid_of(total)), dim3(kBlock), 0, st, total,
                           (const unsigned long long *)ekeys, (const int2 *)erank, kshift, (const int *)poff, pslot);
        RL_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_pair_place, dim3(grid_of(total)), dim3(kBlock), 0, st, total,
                           (const unsigned long long *)ekeys, (const uint8_t *)eflags, (const int2 *)erank, kshift,
                           (const int *)poff, (const int *)pslot, pi, pj, img, flags, (const int *)qoff, qtmp);
        RL_HIP(hipGetLastError());
        if (ix) *ix = PairIndex{poff, qoff, qtmp};
        return RL_OK;
    }
    RL_HIP(search(std::integral_constant<int, kPairFill>{}));
    hipLaunchKernelGGL(k_sort_pairs, dim3(grid_of(n)), dim3(kBlock), 0, st, n, (const int *)poff, pj, img, flags);
    RL_HIP(hipGetLastError());
    return RL_OK;
}

int rod_cells(rl_ctx *h, int64_t n, const double *x, const double *dir, const double *len, double len0,
              double radius, RodCells *out)
{
    hipStream_t st = h->stream;
    const rl_params &p = h->prm;
    int werr = 0;
    double Lmax = len0;
    RL_HIP(hipMemsetAsync(h->flag_dev, 0, sizeof(int) * 4, st));
    if (len && n > 0) {
        auto *lm = (unsigned long long *)ws_get(h, kWsLenMax, sizeof(unsigned long long), &werr);
        if (werr) return werr;
        RL_HIP(hipMemsetAsync(lm, 0, sizeof(unsigned long long), st));
        hipLaunchKernelGGL(k_len_max, dim3(grid_of(n)), dim3(kBlock), 0, st, n, len, lm, h->flag_dev);
        RL_HIP(hipGetLastError());
        RL_HIP(hipMemcpyAsync(h->host_scratch, lm, sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
        RL_HIP(hipMemcpyAsync(h->host_scratch + 1, h->flag_dev, sizeof(int), hipMemcpyDeviceToHost, st));
        RL_HIP(hipStreamSynchronize(st));
        if (((int *)(h->host_scratch + 1))[0] & 4) {
            set_error("rod cells: rod lengths must be finite and > 0");
            return RL_ERR_ARG;
        }
        unsigned long long bits = (unsigned long long)h->host_scratch[0];
        std::memcpy(&Lmax, &bits, sizeof(double));
    } else if (!(len0 > 0.0)) {
        set_error("rod cells: len0 must be > 0");
        return RL_ERR_ARG;
    }
    const double reach = 0.5 * Lmax + radius;
    GridDev g;
    int64_t ncell = 1;
    for (int a = 0; a < 3; ++a) {
        if (!(2.0 * reach <= p.box[a])) {
            set_error("rod cells: half the longest rod plus the radius %g exceeds half the box edge %g", reach,
                      0.5 * p.box[a]);
            return RL_ERR_ARG;
        }
        int nca = (int)floor(p.box[a] / reach);
        if (nca < 1) nca = 1;
        if (nca > 1024) nca = 1024;
        g.nc[a] = nca;
        g.cell[a] = p.box[a] / nca;
        g.S[a] = 1;
        g.box[a] = p.box[a];
        ncell *= nca;
    }
    if (ncell > (1 << 26)) {
        set_error("rod cells: too many cells (%lld)", (long long)ncell);
        return RL_ERR_ARG;
    }
    const int64_t nb = n > 0 ? n : 1;
    int *cell_of = (int *)ws_get(h, kWsCellOf, sizeof(int) * nb, &werr);
    int *cell_cnt = (int *)ws_get(h, kWsCellCnt, sizeof(int) * ncell, &werr);
    int *cell_start = (int *)ws_get(h, kWsCellStart, sizeof(int) * (ncell + 1), &werr);
    int *sorted = (int *)ws_get(h, kWsSorted, sizeof(int) * nb, &werr);
    int *cell_rank = (int *)ws_get(h, kWsCellCur, sizeof(int) * nb, &werr);
    double *xs = (double *)ws_get(h, kWsXs, sizeof(double) * 3 * nb, &werr);
    double *ds = (double *)ws_get(h, kWsDs, sizeof(double) * 3 * nb, &werr);
    double *ls = (double *)ws_get(h, kWsLs, sizeof(double) * nb, &werr);
    if (werr) return werr;
    RL_HIP(hipMemsetAsync(cell_cnt, 0, sizeof(int) * ncell, st));
    if (n > 0) {
        hipLaunchKernelGGL(k_bin, dim3(grid_of(n)), dim3(kBlock), 0, st, n, x, dir, g, 0, 0, cell_of, cell_cnt,
                           cell_rank, h->flag_dev);
        RL_HIP(hipGetLastError());
    }
    {
        const int rc = device_scan(h, cell_cnt, ncell, cell_start, nullptr);
        if (rc) return rc;
    }
    if (n > 0) {
        hipLaunchKernelGGL(k_scatter, dim3(grid_of(n)), dim3(kBlock), 0, st, n, x, dir, len, len0, cell_of,
                           cell_start, (const int *)cell_rank, sorted, xs, ds, ls);
        RL_HIP(hipGetLastError());
    }
    RL_HIP(hipMemcpyAsync(h->host_scratch + 1, h->flag_dev, sizeof(int), hipMemcpyDeviceToHost, st));
    RL_HIP(hipStreamSynchronize(st));
    const int ferr = ((int *)(h->host_scratch + 1))[0];
    if (ferr & 1) {
        set_error("rod cells: non-finite centre or director");
        return RL_ERR_NONFINITE;
    }
    if (ferr & 2) {
        set_error("rod cells: a centre lies outside [0, box)");
        return RL_ERR_ARG;
    }
    for (int a = 0; a < 3; ++a) {
        out->nc[a] = g.nc[a];
        out->cell[a] = g.cell[a];
        out->box[a] = g.box[a];
    }
    out->start = cell_start;
    out->order = sorted;
    out->xs = xs;
    out->ds = ds;
    out->ls = ls;
    return RL_OK;
}

int build_pairs_impl(rl_ctx *h, int64_t n, const double *x, const double *dir, const double *len, double len0,
                     int64_t capacity, int32_t *pi, int32_t *pj, int32_t *img, uint8_t *flags, int64_t *n_pairs)
{
    return pairs_core(h, n, x, dir, len, len0, false, nullptr, nullptr, capacity, pi, pj, img, flags, n_pairs,
                      nullptr);
}

int build_pairs_sorted(rl_ctx *h, int64_t n, const double *x, const double *dir, const double *len, double len0,
                       const double *F, double *Unc, int64_t *n_pairs, const int **perm, const double **xs,
                       const double **ds, const double **ls, PairIndex *ix)
{
    int err = 0;
    // pairs that all three lists hold
    auto held = [&]() {
        return (int64_t)(std::min(h->cap[kWsStepPi], std::min(h->cap[kWsStepPj], h->cap[kWsStepImg])) /
                         sizeof(int32_t));
    };
    int64_t np = 0;
    int rc = RL_ERR_CAPACITY;
    *ix = PairIndex{nullptr, nullptr, nullptr};
    for (int attempt = 0; attempt < 2 && rc == RL_ERR_CAPACITY; ++attempt) {
        rc = pairs_core(h, n, x, dir, len, len0, true, F, Unc, held(), (int32_t *)h->buf[kWsStepPi],
                        (int32_t *)h->buf[kWsStepPj], (int32_t *)h->buf[kWsStepImg], nullptr, &np, ix);
        if (rc == RL_ERR_CAPACITY && np <= 0x7fffffffLL) {
            const int64_t cap = np + np / 4 + 64;
            ws_get(h, kWsStepPi, sizeof(int32_t) * cap, &err);
            ws_get(h, kWsStepPj, sizeof(int32_t) * cap, &err);
            ws_get(h, kWsStepImg, sizeof(int32_t) * cap, &err);
            if (err) return err;
        }
    }
    if (rc) return rc;
    *n_pairs = np;
    *perm = (const int *)h->buf[kWsSorted];
    *xs = (const double *)h->buf[kWsXs];
    *ds = (const double *)h->buf[kWsDs];
    *ls = (const double *)h->buf[kWsLs];
    return RL_OK;
}

// ---------------------------------------------------------------------------
// Constraint geometry: phi, e, arm and q = phi/h + D^T M F per pair.
// ---------------------------------------------------------------------------
template <bool UNI>
__global__ void k_unc(int64_t n, const double *__restrict__ dir, const double *__restrict__ len, Mob mob, double diam,
                      double eta, const double *__restrict__ F, double *__restrict__ Unc)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const Mob m = UNI ? mob : mobility_of(len[i], diam, eta);
    const V3 d = load3(dir + 3 * i);
    V3 f = v3(0, 0, 0), tq = v3(0, 0, 0);
    if (F) {
        f = load3(F + 6 * i);
        tq = load3(F + 6 * i + 3);
    }
    rod_unc(m, d, f, tq, Unc + 6 * i);
}

template <bool PACK>
__global__ void k_assemble(int64_t nc, const double *__restrict__ x, const double *__restrict__ dir,
                           const double *__restrict__ len, double len0, GridDev g, double diam, double dt,
                           const int32_t *__restrict__ pi, const int32_t *__restrict__ pj,
                           const int32_t *__restrict__ img, const double *__restrict__ Unc, double *__restrict__ phi,
                           double *__restrict__ e, double *__restrict__ arm, double *__restrict__ q, int64_t n,
                           int *__restrict__ err, PackOut pk)
{
    const int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (c >= nc) return;
    const int i = pi[c], j = pj[c], im = img[c];
    if (!PACK && (i < 0 || j < 0 || i >= n || j >= n)) {
        atomicOr(err, 8);
        phi[c] = q[c] = arm[2 * c] = arm[2 * c + 1] = NAN;
        store3(e + 3 * c, v3(NAN, NAN, NAN));
        return;
    }
    const double sx = ((im >> 8) & 15) - 8, sy = ((im >> 4) & 15) - 8, sz = (im & 15) - 8;
    const V3 xi = load3(x + 3 * (int64_t)i), di = load3(dir + 3 * (int64_t)i);
    const V3 xj = load3(x + 3 * (int64_t)j) + v3(sx * g.box[0], sy * g.box[1], sz * g.box[2]);
    const V3 dj = load3(dir + 3 * (int64_t)j);
    const double Li = len ? len[i] : len0, Lj = len ? len[j] : len0;
    const Contact ct = closest_point(xi, di, 0.5 * Li, xj, dj, 0.5 * Lj);
    const double ph = ct.dist - diam;
    if (!PACK || phi) {
        phi[c] = ph;
        store3(e + 3 * c, ct.e);
        arm[2 * c] = ct.s;
        arm[2 * c + 1] = ct.t;
    }
    // D^T U_nc: e.U_i + (s_i d_i x e).Omega_i - e.U_j - (t d_j x e).Omega_j
    const V3 ui = load3(Unc + 6 * (int64_t)i), wi = load3(Unc + 6 * (int64_t)i + 3);
    const V3 uj = load3(Unc + 6 * (int64_t)j), wj = load3(Unc + 6 * (int64_t)j + 3);
    const double rate = dot(ct.e, ui) + dot(cross(ct.s * di, ct.e), wi) - dot(ct.e, uj) -
                        dot(cross(ct.t * dj, ct.e), wj);
    if (!PACK) {
        q[c] = ph / dt + rate;
        return;
    }
    const double qc = ph / dt + rate;
    pack_record(pk, c, i, j, ct.e.x, ct.e.y, ct.e.z, ct.s, ct.t, qc);
}

hipError_t launch_assemble(hipStream_t st, const rl_params &p, int64_t n, const double *x, const double *dir,
                           const double *len, double len0, int64_t nc, const int32_t *pi, const int32_t *pj,
                           const int32_t *img, const double *Unc, double *phi, double *e, double *arm, double *q,
                           int *err, const PackOut *pk)
{
    if (nc <= 0) return hipSuccess;
    GridDev g{};
    for (int a = 0; a < 3; ++a) g.box[a] = p.box[a];
    if (pk)
        hipLaunchKernelGGL(k_assemble<true>, dim3(grid_of(nc)), dim3(kBlock), 0, st, nc, x, dir, len, len0, g, p.diam,
                           p.dt, pi, pj, img, Unc, phi, e, arm, q, n, err, *pk);
    else
        hipLaunchKernelGGL(k_assemble<false>, dim3(grid_of(nc)), dim3(kBlock), 0, st, nc, x, dir, len, len0, g,
                           p.diam, p.dt, pi, pj, img, Unc, phi, e, arm, q, n, err, PackOut{});
    return hipGetLastError();
}

hipError_t launch_unc(hipStream_t st, int64_t n, const double *dir, const double *len, double len0, double diam,
                      double eta, const double *F, double *Unc)
{
    if (n <= 0) return hipSuccess;
    const Mob mob = mobility_of(len ? 1.0 : len0, diam, eta);
    if (len)
        hipLaunchKernelGGL(k_unc<false>, dim3(grid_of(n)), dim3(kBlock), 0, st, n, dir, len, mob, diam, eta, F, Unc);
    else
        hipLaunchKernelGGL(k_unc<true>, dim3(grid_of(n)), dim3(kBlock), 0, st, n, dir, len, mob, diam, eta, F, Unc);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Bilateral links (eq. linearconstraints b): a Hookean link between the point
// at arclength sP on rod P's axis and the point at sQ on rod Q's axis, or a
// fixed point (Q < 0).  r = (x_P + sP d_P) - (x_Q + sQ d_Q) with each
// component of the difference taken to its nearest periodic image; the
// link's length is |r|, its direction e = r/|r| (from Q to P), its column of
// D is that of a contact with lever arms sP d_P and sQ d_Q (Appendix
// "Symmetry ...": the two points are arbitrary for bilateral constraints).
// Row (eq. blockdef D and F): q = (|r| - rest)/h + D^T M F, compliance
// 1/(kappa h), 0 for kappa = +inf.  A link of zero length takes e normal to
// both axes (d_P x d_Q, or d_P x the coordinate axis least aligned with d_P
// for parallel axes, d_Q = e_z for a fixed point) and flag bit 2.
// inv (may be null) maps the caller's rod index to the rods' order in x.
// ---------------------------------------------------------------------------
__device__ V3 normal_to(V3 dp, V3 dq)
{
    V3 c = cross(dp, dq);
    double nn = sqrt(dot(c, c));
    if (nn < 1e-12) {
        const double ax = fabs(dp.x), ay = fabs(dp.y), az = fabs(dp.z);
        int k = 0;
        double best = ax;
        if (ay < best) {
            k = 1;
            best = ay;
        }
        if (az < best) k = 2;
        c = cross(dp, v3(k == 0 ? 1.0 : 0.0, k == 1 ? 1.0 : 0.0, k == 2 ? 1.0 : 0.0));
        nn = sqrt(dot(c, c));
    }
    return v3(c.x / nn, c.y / nn, c.z / nn);
}

__global__ void k_links(int64_t nl, int64_t n, const double *__restrict__ x, const double *__restrict__ dir,
                        const int *__restrict__ inv, const int32_t *__restrict__ lp, const int32_t *__restrict__ lq,
                        const double *__restrict__ larm, const double *__restrict__ kappa,
                        const double *__restrict__ rest, const double *__restrict__ anchor, GridDev g, double dt,
                        const double *__restrict__ Unc, int32_t *__restrict__ pi_out, int32_t *__restrict__ pj_out,
                        double *__restrict__ len_out, double *__restrict__ e_out, double *__restrict__ arm_out,
                        double *__restrict__ q_out, double *__restrict__ cmp_out, uint8_t *__restrict__ fl_out,
                        int *__restrict__ err)
{
    const int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (k >= nl) return;
    const int32_t P0 = lp[k], Q0 = lq[k];
    const double kap = kappa[k], r0 = rest[k];
    if (P0 < 0 || P0 >= n || Q0 >= n || Q0 < -1 || P0 == Q0 || (Q0 < 0 && !anchor) || !(kap > 0.0) ||
        !(r0 >= 0.0) || !isfinite(r0)) {
        atomicOr(err, 16);
        return;
    }
    const int P = inv ? inv[P0] : P0, Q = Q0 < 0 ? -1 : (inv ? inv[Q0] : Q0);
    const double sP = larm[2 * k], sQ = larm[2 * k + 1];
    const V3 xP = load3(x + 3 * (int64_t)P), dP = load3(dir + 3 * (int64_t)P);
    const V3 aP = xP + sP * dP;
    V3 dQ = v3(0.0, 0.0, 1.0), aQ;
    if (Q >= 0) {
        dQ = load3(dir + 3 * (int64_t)Q);
        aQ = load3(x + 3 * (int64_t)Q) + sQ * dQ;
    } else {
        aQ = load3(anchor + 3 * k);
    }
    double r[3] = {aP.x - aQ.x, aP.y - aQ.y, aP.z - aQ.z};
    for (int a = 0; a < 3; ++a) r[a] -= g.box[a] * floor(r[a] / g.box[a] + 0.5);
    const V3 rv = v3(r[0], r[1], r[2]);
    const double L = sqrt(dot(rv, rv));
    V3 e;
    uint8_t fl = 0;
    if (L < kDegenDist) {
        e = normal_to(dP, dQ);
        fl = 4;
    } else {
        e = v3(rv.x / L, rv.y / L, rv.z / L);
    }
    // D^T U_nc: e.U_P + (sP d_P x e).W_P - e.U_Q - (sQ d_Q x e).W_Q
    double rate = dot(e, load3(Unc + 6 * (int64_t)P)) + dot(cross(sP * dP, e), load3(Unc + 6 * (int64_t)P + 3));
    if (Q >= 0)
        rate -= dot(e, load3(Unc + 6 * (int64_t)Q)) + dot(cross(sQ * dQ, e), load3(Unc + 6 * (int64_t)Q + 3));
    pi_out[k] = P;
    pj_out[k] = Q;
    len_out[k] = L;
    store3(e_out + 3 * k, e);
    arm_out[2 * k] = sP;
    arm_out[2 * k + 1] = Q >= 0 ? sQ : 0.0;
    q_out[k] = (L - r0) / dt + rate;
    cmp_out[k] = isinf(kap) ? 0.0 : 1.0 / (kap * dt);
    if (fl_out) fl_out[k] = fl;
}

hipError_t launch_links(hipStream_t st, int64_t nl, int64_t n, const double *x, const double *dir, const int *inv,
                        const rl_links *lk, const double box[3], double dt, const double *Unc, int32_t *pi,
                        int32_t *pj, double *len, double *e, double *arm, double *q, double *cmp, uint8_t *flags,
                        int *err)
{
    if (nl <= 0) return hipSuccess;
    GridDev g{};
    for (int a = 0; a < 3; ++a) g.box[a] = box[a];
    hipLaunchKernelGGL(k_links, dim3(grid_of(nl)), dim3(kBlock), 0, st, nl, n, x, dir, inv, lk->p, lk->q, lk->arm,
                       lk->kappa, lk->rest, lk->anchor, g, dt, Unc, pi, pj, len, e, arm, q, cmp, flags, err);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Walls (confinement): constraints between a rod and a fixed body, only the
// rod's side in D (Appendix "Equation of motion with geometric constraints",
// last paragraph).  The allowed regions are convex (a half-space, the inside
// of a sphere or of a cylinder), so each end of a rod is a candidate contact
// point: for ends s = -L/2, +L/2 and each wall in order, phi = (distance of
// the end to the wall) - diam/2, and an end with phi < cutoff gives a
// unilateral constraint with e the wall's inward unit normal at its nearest
// point, lever arm s and q = phi/h + D^T M F.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double wall_gap(const WallSet &W, int w, V3 pt, double diam, V3 &e)
{
    const int kind = W.kind[w];
    const V3 p0 = v3(W.p[w][0], W.p[w][1], W.p[w][2]), a = v3(W.a[w][0], W.a[w][1], W.a[w][2]);
    V3 v = pt - p0;
    if (kind == RL_WALL_PLANE) {
        e = a;
        return dot(a, v) - 0.5 * diam;
    }
    if (kind == RL_WALL_CYLINDER_IN) v = v - dot(v, a) * a;
    const double dist = sqrt(dot(v, v));
    e = dist > 0.0 ? v3(-v.x / dist, -v.y / dist, -v.z / dist) : v3(0.0, 0.0, 0.0);
    return W.r[w] - dist - 0.5 * diam;
}

// FILL = false: per-rod counts; FILL = true: the list at the rod's offset
template <bool FILL>
__global__ void k_walls(int64_t n, const double *__restrict__ x, const double *__restrict__ dir,
                        const double *__restrict__ len, double len0, double diam, double cutoff, double dt, WallSet W,
                        const double *__restrict__ Unc, int *__restrict__ cnt, const int *__restrict__ off,
                        int32_t *__restrict__ rod, double *__restrict__ e_out, double *__restrict__ arm,
                        double *__restrict__ phi, double *__restrict__ q, uint8_t *__restrict__ flags)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const V3 xi = load3(x + 3 * i), di = load3(dir + 3 * i);
    const double L = len ? len[i] : len0;
    int m = FILL ? off[i] : 0;
    for (int end = 0; end < 2; ++end) {
        const double s = end == 0 ? -0.5 * L : 0.5 * L;
        const V3 pt = xi + s * di;
        for (int w = 0; w < W.n; ++w) {
            V3 e;
            const double ph = wall_gap(W, w, pt, diam, e);
            if (!(ph < cutoff)) continue;
            if (FILL) {
                const double rate = dot(e, load3(Unc + 6 * i)) + dot(cross(s * di, e), load3(Unc + 6 * i + 3));
                rod[m] = (int32_t)i;
                store3(e_out + 3 * (int64_t)m, e);
                arm[2 * (int64_t)m] = s;
                arm[2 * (int64_t)m + 1] = 0.0;
                if (phi) phi[m] = ph;
                q[m] = ph / dt + rate;
                if (flags) flags[m] = fabs(ph - cutoff) <= kCutoffBand ? 1u : 0u;
            }
            ++m;
        }
    }
    if (!FILL) cnt[i] = m;
}

int walls_impl(rl_ctx *h, int64_t n, const double *x, const double *dir, const double *len, double len0,
               const double *Unc, const WallSet &W, int64_t capacity, int32_t *rod, double *e, double *arm,
               double *phi, double *q, uint8_t *flags, int64_t *count)
{
    hipStream_t st = h->stream;
    const rl_params &p = h->prm;
    int werr = 0;
    *count = 0;
    if (n <= 0 || W.n <= 0) return RL_OK;
    int *cnt = (int *)ws_get(h, kWsWallCnt, sizeof(int) * n, &werr);
    int *off = (int *)ws_get(h, kWsWallOff, sizeof(int) * (n + 1), &werr);
    int64_t *tot = (int64_t *)ws_get(h, kWsScan, sizeof(int64_t) * 2, &werr);
    if (werr) return werr;
    hipLaunchKernelGGL(k_walls<false>, dim3(grid_of(n)), dim3(kBlock), 0, st, n, x, dir, len, len0, p.diam, p.cutoff,
                       p.dt, W, Unc, cnt, (const int *)nullptr, (int32_t *)nullptr, (double *)nullptr,
                       (double *)nullptr, (double *)nullptr, (double *)nullptr, (uint8_t *)nullptr);
    RL_HIP(hipGetLastError());
    int rc = device_scan(h, cnt, n, off, tot);
    if (rc) return rc;
    RL_HIP(hipMemcpyAsync(h->host_scratch, tot, sizeof(int64_t), hipMemcpyDeviceToHost, st));
    RL_HIP(hipStreamSynchronize(st));
    const int64_t total = h->host_scratch[0];
    *count = total;
    if (total > capacity) {
        set_error("walls: %lld contacts exceed capacity %lld", (long long)total, (long long)capacity);
        return RL_ERR_CAPACITY;
    }
    if (total == 0) return RL_OK;
    hipLaunchKernelGGL(k_walls<true>, dim3(grid_of(n)), dim3(kBlock), 0, st, n, x, dir, len, len0, p.diam, p.cutoff,
                       p.dt, W, Unc, cnt, (const int *)off, rod, e, arm, phi, q, flags);
    RL_HIP(hipGetLastError());
    return RL_OK;
}

int assemble_impl(rl_ctx *h, int64_t n, const double *x, const double *dir, const double *len, double len0,
                  int64_t nc, const int32_t *pi, const int32_t *pj, const int32_t *img, const double *F,
                  double *phi, double *e, double *arm, double *q)
{
    hipStream_t st = h->stream;
    const rl_params &p = h->prm;
    int werr = 0;
    if (nc == 0) return RL_OK;
    double *Unc = (double *)ws_get(h, kWsUnc, sizeof(double) * 6 * (n > 0 ? n : 1), &werr);
    if (werr) return werr;
    RL_HIP(launch_unc(st, n, dir, len, len0, p.diam, p.eta, F, Unc));
    RL_HIP(hipMemsetAsync(h->flag_dev, 0, sizeof(int), st));
    RL_HIP(launch_assemble(st, p, n, x, dir, len, len0, nc, pi, pj, img, Unc, phi, e, arm, q, h->flag_dev, nullptr));
    RL_HIP(hipMemcpyAsync(h->host_scratch, h->flag_dev, sizeof(int), hipMemcpyDeviceToHost, st));
    RL_HIP(hipStreamSynchronize(st));
    if (((int *)h->host_scratch)[0] & 8) {
        set_error("rl_assemble_D: a pair index is outside [0, n)");
        return RL_ERR_ARG;
    }
    return RL_OK;
}

// ---------------------------------------------------------------------------
// adjoint of the constraint geometry (differentiation form)
// ---------------------------------------------------------------------------
// Per constraint, from phi_bar = q_bar / h, e_bar and the arclength
// adjoints (s_bar, t_bar), the adjoints of r0 = x_i - x_j' and of the two
// directors; d_bar (the lever-arm parts) is added to the director terms.
// r = r0 + s di - t dj, phi = |r| - diam, e = r / |r|.  The arclengths are
// stationary points of |r|^2 over the free ones: r.di = 0 when s is inside
// (-L_i/2, L_i/2), r.dj = 0 when t is inside (-L_j/2, L_j/2); an arclength
// on a rod end stays there.  Their derivatives follow from differentiating
// those conditions (implicit function; unit directors, so the 2x2 system
// has the matrix [[1, -b], [b, -1]], b = di.dj).  Parallel axes keep their
// closest points fixed and intersecting axes their normal (the midpoint and
// cross-product rules have no derivative that the step uses).
__global__ void k_geo_adjoint(int64_t nc, const double *__restrict__ x, const double *__restrict__ dir,
                              const double *__restrict__ len, double len0, GridDev g,
                              const int32_t *__restrict__ pi, const int32_t *__restrict__ pj,
                              const int32_t *__restrict__ img, double dt, const double *__restrict__ qbar,
                              const double *__restrict__ ebar, const double *__restrict__ armbar,
                              const double *__restrict__ dbar, double *__restrict__ gbar)
{
    const int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (c >= nc) return;
    const int i = pi[c], j = pj[c], im = img[c];
    const double sx = ((im >> 8) & 15) - 8, sy = ((im >> 4) & 15) - 8, sz = (im & 15) - 8;
    const V3 xi = load3(x + 3 * (int64_t)i), di = load3(dir + 3 * (int64_t)i);
    const V3 xj = load3(x + 3 * (int64_t)j) + v3(sx * g.box[0], sy * g.box[1], sz * g.box[2]);
    const V3 dj = load3(dir + 3 * (int64_t)j);
    const double hi = 0.5 * (len ? len[i] : len0), hj = 0.5 * (len ? len[j] : len0);
    const Contact ct = closest_point(xi, di, hi, xj, dj, hj);
    const double b = dot(di, dj), den = 1.0 - b * b;
    const V3 r = (xi - xj) + ct.s * di - ct.t * dj;
    const double phib = qbar[c] / dt;
    const V3 eb = load3(ebar + 3 * c);
    V3 rb = phib * ct.e;
    if (!(ct.flags & 4u)) rb = rb + (1.0 / ct.dist) * (eb - dot(ct.e, eb) * ct.e);
    const double sb = armbar[2 * c] + dot(rb, di);
    const double tb = armbar[2 * c + 1] - dot(rb, dj);
    V3 r0b = rb;
    V3 dib = ct.s * rb + load3(dbar + 6 * c);
    V3 djb = (-ct.t) * rb + load3(dbar + 6 * c + 3);
    if (den > kEpsPar) {
        const bool s_in = fabs(ct.s) < hi, t_in = fabs(ct.t) < hj;
        // dF1 = dr0.di + (r + s di).ddi - t di.ddj (+ ds - b dt)
        // dF2 = dr0.dj + s dj.ddi + (r - t dj).ddj (+ b ds - dt)
        if (s_in && t_in) {
            const double mu2 = -(tb + b * sb) / den, mu1 = sb - b * mu2;
            r0b = r0b - (mu1 * di + mu2 * dj);
            dib = dib - (mu1 * (r + ct.s * di) + (mu2 * ct.s) * dj);
            djb = djb - ((-mu1 * ct.t) * di + mu2 * (r - ct.t * dj));
        } else if (t_in) {
            r0b = r0b + tb * dj;
            dib = dib + (tb * ct.s) * dj;
            djb = djb + tb * (r - ct.t * dj);
        } else if (s_in) {
            r0b = r0b - sb * di;
            dib = dib - sb * (r + ct.s * di);
            djb = djb + (sb * ct.t) * di;
        }
    }
    store3(gbar + 9 * c, r0b);
    store3(gbar + 9 * c + 3, dib);
    store3(gbar + 9 * c + 6, djb);
}

hipError_t launch_geo_adjoint(hipStream_t st, int64_t nc, const double *x, const double *dir, const double *len,
                              double len0, const double box[3], const int32_t *pi, const int32_t *pj,
                              const int32_t *img, double dt, const double *q_bar, const double *e_bar,
                              const double *arm_bar, const double *d_bar, double *gbar)
{
    if (nc <= 0) return hipSuccess;
    GridDev g{};
    for (int a = 0; a < 3; ++a) g.box[a] = box[a];
    hipLaunchKernelGGL(k_geo_adjoint, dim3(grid_of(nc)), dim3(kBlock), 0, st, nc, x, dir, len, len0, g, pi, pj, img,
                       dt, q_bar, e_bar, arm_bar, d_bar, gbar);
    return hipGetLastError();
}

}  // namespace rl

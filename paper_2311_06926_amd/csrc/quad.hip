// Quadrature-based (matrix-free) forward operator: the forward problem
// evaluated by sum factorisation with p+1 Gauss-Legendre points per element in
// each direction (Sec. 5.3), on the weak form of Sec. 3.1 with the symmetric
// Nitsche terms of Sec. 3.3 on the faces.
//
// With G = grad u and P the pressure at a point of the tensor grid, the
// volume flux for the test function v_c is
//     coefficient of d_d v_c :  S_cd = w nu (G_cd + G_dc) + w P delta_cd,
// and for the pressure test function q it is F_q = w (G_11 + G_22 + G_33):
// 2 nu eps(u):eps(v) = nu (grad u + grad u^T):grad v, b(v,p) = (p, div v).
// On a face with outward normal s e_d (s = -1 at x_d = 0, +1 at x_d = 1)
// the tangential components c != d carry
//     nu (2 alpha u_c v_c - v_c d_n u_c - u_c d_n v_c),  alpha = C_pen / h:
//     F_c = w nu (2 alpha u_c - s G_cd) for v_c and S_cd = -w nu s u_c for d_d v_c;
// the normal component vanishes there (strongly imposed v.n = 0), and so
// does d_c u_d on that face, which is why only d_n u_c enters.
//
// The points of one direction are [x = 0, the E (p+1) Gauss points, x = 1];
// the weight of an end point is 1, so that a point with one end-point
// coordinate carries the weight of the two-dimensional Gauss rule of its
// face.  Points with two or more end-point coordinates (edges) carry nothing.
//
// Values at the points never leave the CU: a workgroup owns EX x EY elements
// of the (1, 2) plane and streams a chunk of element layers of direction 3,
// one thread per point column.  Per coefficient plane the modes 1 and 2 give
// ten values per column (per component the value and the two in-plane
// derivatives, the pressure), kept in registers for the p or p+1 planes an
// element layer sees; mode 3, the flux and the transposed mode 3 are register
// arithmetic with the direction's tables in scalar registers; a finished
// plane goes through LDS for the transposed modes 2 and 1.  The layer loop has
// two barriers: the forward modes of the next plane share them with the
// transposed modes of the last.  A tile's coefficients overlap its neighbours',
// so the partial sums go to a scratch block per tile and k_quad_gather adds
// the blocks in a fixed order.
// Bound: latency of LDS and barriers with one or two workgroups per CU (32^3,
// degree 3: LDS busy 35 %, FP64 issue 32 % of the time).  Six launches that
// kept the flux fields of all points in HBM, with 560 MB through them at 32^3
// degree 3, took (us): 32^3 degree 2 / 3 / 4 96 / 212 / 474, 64^3 degree 3
// 1911, 96^3 6666, 24^3 degree 6 691, 16^3 degree 8 563; this form takes 36 /
// 68 / 172, 332, 874, 222, 312.
#include <algorithm>
#include <climits>
#include <new>
#include <stdexcept>

#include "hp_internal.h"

namespace hp {

namespace {

constexpr int QT = 256;

// Elements per tile in directions 1 and 2: (EX (p+1) + 2) (EY (p+1) + 2)
// points, the end points of a mesh of one tile among them, fit QT threads.
template <int P>
struct Tile2 {
    static constexpr int EX = P == 2 ? 4 : P == 3 ? 4 : P == 4 ? 3 : 2;
    static constexpr int EY = P == 2 ? 5 : P == 3 ? 3 : P <= 6 ? 2 : 1;
};

// Workgroups (four waves) per CU: the windows and accumulators of degrees 2
// and 3 leave room for two (degree 4 spills: 32^3 189 -> 249 us).
constexpr int quad_per_cu(int p) { return p <= 3 ? 2 : 1; }

struct QuadArgs {
    const double* x[4];   // u1, u2, u3, p of the first right-hand side
    long long sx[4];
    const double* tab;    // per point: values and derivatives of the degree p-1, then the degree p functions
    const double* wq;
    double* scratch;
    int E, nN, nM, nq;
    int L, nch, nt1, nt2;  // layers per chunk, chunks, tiles
    double nu, alpha;
};

// a row of the point tables, uniform over the workgroup: scalar loads
__device__ __forceinline__ double sload(const double* base, int i) {
    return reinterpret_cast<const __attribute__((address_space(4))) double*>(
        reinterpret_cast<uintptr_t>(base))[i];
}

// The points of one direction inside a tile of ne elements: `off` = 1 if the
// first is x = 0; n points in all (x = 1 the last one of the last tile).
struct Points {
    int ne, off, n;
};

struct FaceWeights {
    double d1, d2, d3;          // w nu at points of the faces normal to 1, 2, 3
    double s1, s2, s3, alpha2;  // outward signs, 2 alpha
};

// One point of a column: mode 3, the flux and the transposed mode 3.  tb: the
// point's table row in direction 3 (scalar registers), w: the weight at volume
// points.  FACE: the point may lie on a face; the terms of every kind of point
// are formed with their weights, so that no branch stands between updates of
// the accumulators (branches made the compiler copy all of them).
template <int P, bool FACE>
__device__ __forceinline__ void quad_point(const double* tb, double w, double nu,
                                           const FaceWeights& fw, const double (&WM)[7][P],
                                           const double (&WN)[3][P + 1], double (&AM)[6][P],
                                           double (&AN)[3][P + 1]) {
    constexpr int W = P + 1;
    auto dotM = [&](int k, const double (&w)[P]) {
        double v = 0.0;
#pragma unroll
        for (int t = 0; t < P; ++t) v += sload(tb, k * W + t) * w[t];
        return v;
    };
    auto dotN = [&](int k, const double (&w)[W]) {
        double v = 0.0;
#pragma unroll
        for (int t = 0; t < W; ++t) v += sload(tb, k * W + t) * w[t];
        return v;
    };
    auto addM = [&](double (&acc)[P], int k, double v) {
#pragma unroll
        for (int t = 0; t < P; ++t) acc[t] += sload(tb, k * W + t) * v;
    };
    auto addN = [&](double (&acc)[W], int k, double v) {
#pragma unroll
        for (int t = 0; t < W; ++t) acc[t] += sload(tb, k * W + t) * v;
    };
    constexpr int VM = 0, DM = 1, VN = 2, DN = 3;  // rows of the table
    const double g13 = dotM(DM, WM[0]), g12 = dotM(VM, WM[1]), g11 = dotM(VM, WM[2]);
    const double g23 = dotM(DM, WM[3]), g22 = dotM(VM, WM[4]), g21 = dotM(VM, WM[5]);
    const double g33 = dotN(DN, WN[0]), g32 = dotN(VN, WN[1]), g31 = dotN(VN, WN[2]);
    const double wn = w * nu, wp = w * dotM(VM, WM[6]);
    double s12 = wn * (g12 + g21), s13 = wn * (g13 + g31), s23 = wn * (g23 + g32);
    if constexpr (FACE) {
        const double v1 = dotM(VM, WM[0]), v2 = dotM(VM, WM[3]), v3 = dotN(VN, WN[0]);
        s12 -= fw.d1 * fw.s1 * v2 + fw.d2 * fw.s2 * v1;
        s13 -= fw.d1 * fw.s1 * v3 + fw.d3 * fw.s3 * v1;
        s23 -= fw.d2 * fw.s2 * v3 + fw.d3 * fw.s3 * v2;
        addM(AM[0], VM, fw.d2 * (fw.alpha2 * v1 - fw.s2 * g12) + fw.d3 * (fw.alpha2 * v1 - fw.s3 * g13));
        addM(AM[3], VM, fw.d1 * (fw.alpha2 * v2 - fw.s1 * g21) + fw.d3 * (fw.alpha2 * v2 - fw.s3 * g23));
        addN(AN[0], VN, fw.d1 * (fw.alpha2 * v3 - fw.s1 * g31) + fw.d2 * (fw.alpha2 * v3 - fw.s2 * g32));
    }
    addM(AM[0], DM, s13);
    addM(AM[1], VM, s12);
    addM(AM[2], VM, wn * (g11 + g11) + wp);
    addM(AM[3], DM, s23);
    addM(AM[4], VM, wn * (g22 + g22) + wp);
    addM(AM[5], VM, w * (g11 + g22 + g33));
    addN(AN[0], DN, wn * (g33 + g33) + wp);
    addN(AN[1], VN, s23);
    addN(AN[2], VN, s13);
}

template <int P>
__global__ __launch_bounds__(QT) __attribute__((amdgpu_waves_per_eu(quad_per_cu(P)))) void k_quad(QuadArgs a) {
    constexpr int W = P + 1, EX = Tile2<P>::EX, EY = Tile2<P>::EY;
    constexpr int NQ1 = EX * W + 2, NQ2 = EY * W + 2;
    constexpr int PQ1 = (NQ1 + 1) & ~1, PQ2 = (NQ2 + 1) & ~1;  // 16-byte rows of the dense tables
    constexpr int S1 = EX + P, S2 = EY + P;
    static_assert(NQ1 * NQ2 <= QT, "one thread per point column");
    // rows of the components in direction 2 (degree p: one more)
    constexpr int RM = S2 - 1, RN = S2;
    // (component, RG rows, point q1): one task per thread for modes 1 and
    // transposed 2, so that a table or flux value read serves RG rows
    constexpr int RG = P <= 6 ? 2 : 3;
    constexpr int GM = (RM + RG - 1) / RG, GN = (RN + RG - 1) / RG;
    static_assert((3 * GM + GN) * NQ1 <= QT, "one row group per thread");
    // outputs of a plane: S1 x RM, (S1-1) x RN, (S1-1) x RM twice
    constexpr int O1 = S1 * RM, O2 = O1 + (S1 - 1) * RN, O3 = O2 + (S1 - 1) * RM, OT = O3 + (S1 - 1) * RM;
    constexpr int NC = (OT + QT - 1) / QT;  // coefficients a thread stages per plane
    constexpr int UN = P <= 6 ? W : 2;      // taps of modes 1 and 2 loaded together
    // point tables: per point (forward modes), and per function over the
    // tile's points, zero outside its support (transposed modes)
    __shared__ __align__(16) double tab1[NQ1][4][W], tab2[NQ2][4][W];
    __shared__ __align__(16) double dt1[4][S1][PQ1], dt2[4][S2][PQ2];
    __shared__ __align__(16) double C[4][S2 * S1], A[7][S2 * NQ1], F[9][PQ2 * NQ1], G[7][S2 * PQ1];
    const int tid = threadIdx.x;
    const int t1 = blockIdx.x % a.nt1, t2 = blockIdx.x / a.nt1, ch = blockIdx.y, r = blockIdx.z;
    const int ea = t1 * EX, eb = t2 * EY, e0 = ch * a.L, nl = min(a.L, a.E - e0);
    auto points = [&](int e, int size, int& r0) {
        Points p;
        p.ne = min(size, a.E - e);
        p.off = e == 0 ? 1 : 0;
        r0 = e == 0 ? 0 : 1 + e * W;
        p.n = (e + p.ne == a.E ? a.nq : 1 + (e + p.ne) * W) - r0;
        return p;
    };
    int ra, rb;
    const Points pa = points(ea, EX, ra), pb = points(eb, EY, rb);
    auto element = [&](const Points& p, int q) { return min(max(q - p.off, 0) / W, p.ne - 1); };
    for (int i = tid; i < 4 * S1 * PQ1; i += QT) (&dt1[0][0][0])[i] = 0.0;
    for (int i = tid; i < 4 * S2 * PQ2; i += QT) (&dt2[0][0][0])[i] = 0.0;
    for (int i = tid; i < 9 * PQ2 * NQ1; i += QT) (&F[0][0])[i] = 0.0;  // points a tile lacks
    for (int i = tid; i < 7 * S2 * PQ1; i += QT) (&G[0][0])[i] = 0.0;
    __syncthreads();
    for (int i = tid; i < NQ1 * 4 * W; i += QT) {
        const int q = i / (4 * W), k = (i / W) % 4, t = i % W;
        const double v = q < pa.n ? a.tab[(long long)ra * 4 * W + i] : 0.0;
        tab1[q][k][t] = v;
        if (q < pa.n && (k >= 2 || t < P)) dt1[k][element(pa, q) + t][q] = v;
    }
    for (int i = tid; i < NQ2 * 4 * W; i += QT) {
        const int q = i / (4 * W), k = (i / W) % 4, t = i % W;
        const double v = q < pb.n ? a.tab[(long long)rb * 4 * W + i] : 0.0;
        tab2[q][k][t] = v;
        if (q < pb.n && (k >= 2 || t < P)) dt2[k][element(pb, q) + t][q] = v;
    }
    // this thread's point column
    // (threads past the last one repeat it with weight 0)
    const int q2r = tid / pa.n, q1 = tid - q2r * pa.n, q2 = min(q2r, pb.n - 1);
    const bool act = q2r < pb.n;
    // this thread's row group: component tf, rows tr .. tr + RG - 1 of tn, point tq
    const int tg = tid / NQ1, tq = tid - tg * NQ1;
    const int tf = tg < GM ? 0 : tg < GM + GN ? 1 : tg < 2 * GM + GN ? 2 : 3;
    const bool task = tg < 3 * GM + GN;
    const int tr = RG * (tg - (tf == 0 ? 0 : tf == 1 ? GM : tf == 2 ? GM + GN : 2 * GM + GN));
    const int tn = tf == 1 ? RN : RM;
    const int tl = element(pa, tq);
    const int l2 = element(pb, q2);
    const bool f1 = ra + q1 == 0 || ra + q1 == a.nq - 1;
    const bool f2 = rb + q2 == 0 || rb + q2 == a.nq - 1;
    // uniform: whether the tile has face points in direction 1 or 2
    const bool edge_tile = ea == 0 || eb == 0 || ea + pa.ne == a.E || eb + pb.ne == a.E;
    const double s1 = ra + q1 == 0 ? -1.0 : 1.0, s2 = rb + q2 == 0 ? -1.0 : 1.0;
    const double w12 = act ? a.wq[ra + q1] * a.wq[rb + q2] : 0.0;
    // coefficients of plane k: entry e of [u1 | u2 | u3 | p], local (i, j);
    // local index t is function el0 + t (degree p-1) or interior function
    // el0 - 1 + t (degree p); zero outside the mesh
    double cr[NC];
    const double* src[NC];   // of plane 0
    long long pitch[NC];     // planes
    int depth[NC], dst[NC];  // planes of the component (0: no such coefficient), entry of C
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int e = min(tid + c * QT, OT - 1);
        const int f = e < O1 ? 0 : e < O2 ? 1 : e < O3 ? 2 : 3;
        const int le = e - (f == 0 ? 0 : f == 1 ? O1 : f == 2 ? O2 : O3);
        const int w = f == 0 ? S1 : S1 - 1, j = le / w, i = le - j * w;
        const int n1 = f == 0 ? a.nN : a.nM, n2 = f == 1 ? a.nN : a.nM, n3 = f == 2 ? a.nN : a.nM;
        const int gi = ea + i - (f == 0), gj = eb + j - (f == 1);
        const bool in = gi >= 0 && gi < n1 && gj >= 0 && gj < n2;
        pitch[c] = (long long)n1 * n2;
        depth[c] = in ? n3 : 0;
        src[c] = a.x[f] + r * a.sx[f] + (in ? gi + (long long)n1 * gj : 0);
        dst[c] = f * (S2 * S1) + j * S1 + i;
    }
    auto fetch = [&](int k) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const bool in = k >= 0 && k < depth[c];
            const double v = src[c][in ? pitch[c] * k : 0];
            cr[c] = in ? v : 0.0;
        }
    };
    // windows of the mode-1/2 values and accumulators of the transposed mode 3
    // over the planes of a layer; M: degree p-1 in direction 3 (u1: value,
    // d_2, d_1; u2 the same; p), N: degree p (u3)
    double WM[7][P], WN[3][W], AM[6][P], AN[3][W];
#pragma unroll
    for (int t = 0; t < W; ++t) {
#pragma unroll
        for (int q = 0; q < 3; ++q) WN[q][t] = AN[q][t] = 0.0;
        if (t < P) {
#pragma unroll
            for (int q = 0; q < 7; ++q) WM[q][t] = 0.0;
#pragma unroll
            for (int q = 0; q < 6; ++q) AM[q][t] = 0.0;
        }
    }
    double* blk = a.scratch + ((((long long)r * a.nch + ch) * a.nt2 + t2) * a.nt1 + t1) *
                                  (4LL * (a.L + P) * S2 * S1);
    fetch(e0 - 1);
    // step s: push plane e0 - 1 + s (interior index for u3), process layer
    // e0 + s - p, retire plane s - p - 1 of the block
#pragma unroll 1
    for (int s = 0; s <= 2 * P + nl; ++s) {
        const bool push = s < P + nl, retire = s > P;
        if (push) {
#pragma unroll
            for (int c = 0; c < NC; ++c) (&C[0][0])[dst[c]] = cr[c];  // repeated entries agree
        }
        if (retire) {
            const int o = q2 * NQ1 + q1;
            if (act) {
#pragma unroll
                for (int q = 0; q < 6; ++q) F[q][o] = AM[q][0];
#pragma unroll
                for (int q = 0; q < 3; ++q) F[6 + q][o] = AN[q][0];
            }
#pragma unroll
            for (int q = 0; q < 6; ++q) {
#pragma unroll
                for (int t = 0; t + 1 < P; ++t) AM[q][t] = AM[q][t + 1];
                AM[q][P - 1] = 0.0;
            }
#pragma unroll
            for (int q = 0; q < 3; ++q) {
#pragma unroll
                for (int t = 0; t + 1 < W; ++t) AN[q][t] = AN[q][t + 1];
                AN[q][W - 1] = 0.0;
            }
        }
        __syncthreads();
        if (s + 1 < P + nl) fetch(e0 + s);
        if (push) {
            // mode 1: V and D of the row group at tq
            if (task) {
                const double(*tb)[W] = tab1[tq] + (tf == 0 ? 2 : 0);
                double v[RG], d[RG];
#pragma unroll
                for (int g = 0; g < RG; ++g) v[g] = d[g] = 0.0;
#pragma unroll(UN)
                for (int t = 0; t < W; ++t) {
                    const double cv = tb[0][t], cd = tb[1][t];
#pragma unroll
                    for (int g = 0; g < RG; ++g) {
                        // the degree p-1 tables are zero at t = p; rows past the last repeat it
                        const int tt = t < P || tf == 0 ? t : 0;
                        const double x = C[tf][min(tr + g, tn - 1) * S1 + tl + tt];
                        v[g] += cv * x;
                        d[g] += cd * x;
                    }
                }
#pragma unroll
                for (int g = 0; g < RG; ++g)
                    if (tr + g < tn) {
                        A[2 * tf][(tr + g) * NQ1 + tq] = v[g];
                        if (tf < 3) A[2 * tf + 1][(tr + g) * NQ1 + tq] = d[g];
                    }
            }
        }
        if (retire && task) {
            // transposed mode 2 of the row group at tq.  u1: value and d_2 (F0, F1),
            // d_1 (F2); u2: F3, F4, and F1, which serves both S_12; u3: F6..F8;
            // p: F5 (its other sums are not used)
            const double* fv = F[tf == 0 ? 0 : tf == 1 ? 3 : tf == 2 ? 6 : 5] + tq;
            const double* fd = F[tf == 0 ? 1 : tf == 1 ? 4 : 7] + tq;
            const double* fb = F[tf == 0 ? 2 : tf == 1 ? 1 : 8] + tq;
            const int k = tf == 1 ? 2 : 0;
            const double *tv[RG], *td[RG];
            double ga[RG], gb[RG];
#pragma unroll
            for (int g = 0; g < RG; ++g) {
                const int row = min(tr + g, tn - 1);
                tv[g] = dt2[k][row];
                td[g] = dt2[k + 1][row];
                ga[g] = gb[g] = 0.0;
            }
// (a loop: fully unrolled, its loads took 150 registers)
#pragma unroll 2
            for (int m = 0; m < PQ2; m += 2) {
                double xv[2], xd[2], xb[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    xv[h] = fv[(m + h) * NQ1];
                    xd[h] = fd[(m + h) * NQ1];
                    xb[h] = fb[(m + h) * NQ1];
                }
                if (tf == 3) xd[0] = xd[1] = 0.0;
#pragma unroll
                for (int g = 0; g < RG; ++g) {
                    const double2 cv = *reinterpret_cast<const double2*>(tv[g] + m);
                    const double2 cd = *reinterpret_cast<const double2*>(td[g] + m);
                    ga[g] += cv.x * xv[0];
                    ga[g] += cd.x * xd[0];
                    gb[g] += cv.x * xb[0];
                    ga[g] += cv.y * xv[1];
                    ga[g] += cd.y * xd[1];
                    gb[g] += cv.y * xb[1];
                }
            }
            // Where a zero of the tables outside a function's support met an infinity
            // or a NaN, which may reach no other function, the sums are taken again
            // without the zeros: together before they are stored, or row by row after
            // (RG = 3: together, degree 8 spills, 16^3 298 -> 366 us).
            double zero = 0.0;
#pragma unroll
            for (int g = 0; g < RG; ++g) zero += 0.0 * ga[g] + 0.0 * gb[g];
            if (RG == 2 && zero != 0.0) {
#pragma unroll
                for (int g = 0; g < RG; ++g) ga[g] = gb[g] = 0.0;
#pragma unroll 1
                for (int m = 0; m < PQ2; ++m)
#pragma unroll
                    for (int g = 0; g < RG; ++g) {
                        const double cv = tv[g][m], cd = td[g][m];
                        if (cv != 0.0) ga[g] += cv * fv[m * NQ1];
                        if (cd != 0.0 && tf < 3) ga[g] += cd * fd[m * NQ1];
                        if (cv != 0.0) gb[g] += cv * fb[m * NQ1];
                    }
            }
#pragma unroll
            for (int g = 0; g < RG; ++g)
                if (tr + g < tn) {
                    G[2 * tf][(tr + g) * PQ1 + tq] = ga[g];
                    if (tf < 3) G[2 * tf + 1][(tr + g) * PQ1 + tq] = gb[g];
                }
            if (RG > 2 && zero != 0.0)
#pragma unroll 1
                for (int row = tr; row < min(tr + RG, tn); ++row) {
                    double va = 0.0, vb = 0.0;
#pragma unroll 1
                    for (int m = 0; m < PQ2; ++m) {
                        const double cv = dt2[k][row][m], cd = dt2[k + 1][row][m];
                        if (cv != 0.0) va += cv * fv[m * NQ1];
                        if (cd != 0.0 && tf < 3) va += cd * fd[m * NQ1];
                        if (cv != 0.0) vb += cv * fb[m * NQ1];
                    }
                    G[2 * tf][row * PQ1 + tq] = va;
                    if (tf < 3) G[2 * tf + 1][row * PQ1 + tq] = vb;
                }
        }
        __syncthreads();
        if (retire) {
            // transposed mode 1: the plane's partial sums to the block
            const int kl = s - P - 1;
            for (int e = tid; e < OT; e += QT) {
                const int f = e < O1 ? 0 : e < O2 ? 1 : e < O3 ? 2 : 3;
                const int le = e - (f == 0 ? 0 : f == 1 ? O1 : f == 2 ? O2 : O3);
                const int w = f == 0 ? S1 : S1 - 1, j = le / w, i = le - j * w;
                const double* ga = &G[2 * f][j * PQ1];
                const double* gb = &G[f < 3 ? 2 * f + 1 : 6][j * PQ1];
                const double* cv = dt1[f == 0 ? 2 : 0][i];
                const double* cd = dt1[f == 0 ? 3 : 1][i];
                double y = 0.0, z = 0.0;
#pragma unroll 3
                for (int m = 0; m < PQ1; m += 2) {
                    const double2 v = *reinterpret_cast<const double2*>(cv + m);
                    const double2 d = *reinterpret_cast<const double2*>(cd + m);
                    const double2 x = *reinterpret_cast<const double2*>(ga + m);
                    const double2 u = *reinterpret_cast<const double2*>(gb + m);
                    y += v.x * x.x;
                    z += d.x * u.x;
                    y += v.y * x.y;
                    z += d.y * u.y;
                }
                if (f < 3) y += z;
                if (0.0 * y != 0.0) {  // as for the transposed mode 2
                    y = z = 0.0;
#pragma unroll 1
                    for (int m = 0; m < PQ1; ++m) {
                        if (cv[m] != 0.0) y += cv[m] * ga[m];
                        if (cd[m] != 0.0 && f < 3) z += cd[m] * gb[m];
                    }
                    y += z;
                }
                blk[(((long long)f * (a.L + P) + kl) * S2 + j) * S1 + i] = y;
            }
        }
        if (push) {
            // mode 2 at this thread's column, into the windows
#pragma unroll
            for (int q = 0; q < 7; ++q)
#pragma unroll
                for (int t = 0; t + 1 < P; ++t) WM[q][t] = WM[q][t + 1];
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int t = 0; t + 1 < W; ++t) WN[q][t] = WN[q][t + 1];
            double z[10];
#pragma unroll
            for (int q = 0; q < 10; ++q) z[q] = 0.0;
#pragma unroll(UN)
            for (int t = 0; t < W; ++t) {
                const int o = (l2 + t) * NQ1 + q1;
                const double vn = tab2[q2][2][t], dn = tab2[q2][3][t];
                const double bv = A[2][o], bd = A[3][o];
                z[3] += vn * bv;
                z[4] += dn * bv;
                z[5] += vn * bd;
                if (t < P) {
                    const double vm = tab2[q2][0][t], dm = tab2[q2][1][t];
                    const double av = A[0][o], ad = A[1][o], cv = A[4][o], cd = A[5][o];
                    z[0] += vm * av;
                    z[1] += dm * av;
                    z[2] += vm * ad;
                    z[7] += vm * cv;
                    z[8] += dm * cv;
                    z[9] += vm * cd;
                    z[6] += vm * A[6][o];
                }
            }
#pragma unroll
            for (int q = 0; q < 7; ++q) WM[q][P - 1] = z[q];
#pragma unroll
            for (int q = 0; q < 3; ++q) WN[q][W - 1] = z[7 + q];
        }
        if (s < P || !push) continue;
        // the points of layer e, the end points with the first and last layer
        const int e = e0 + s - P;
        const int g0 = e == 0 ? 0 : 1 + e * W, g1 = e == a.E - 1 ? a.nq : 1 + (e + 1) * W;
        if (edge_tile || e == 0 || e == a.E - 1) {
#pragma unroll 1
            for (int g = g0; g < g1; ++g) {
                const bool f3 = g == 0 || g == a.nq - 1;
                const double w = w12 * sload(a.wq, g), wn = w * a.nu;
                const int faces = (int)f1 + (int)f2 + (int)f3;
                // the weight for each kind of point, zero for the others
                const FaceWeights fw{faces == 1 && f1 ? wn : 0.0, faces == 1 && f2 ? wn : 0.0,
                                     faces == 1 && f3 ? wn : 0.0, s1, s2, g == 0 ? -1.0 : 1.0,
                                     2.0 * a.alpha};
                quad_point<P, true>(a.tab + (long long)g * 4 * W, faces == 0 ? w : 0.0, a.nu, fw, WM,
                                    WN, AM, AN);
            }
        } else {
#pragma unroll 1
            for (int g = g0; g < g1; ++g)
                quad_point<P, false>(a.tab + (long long)g * 4 * W, w12 * sload(a.wq, g), a.nu, FaceWeights{},
                                     WM, WN, AM, AN);
        }
    }
}

// y = the sum of the tiles' partial sums, tiles in ascending order.
struct GatherArgs {
    const double* scratch;
    double* y[4];
    long long sy[4];
    int E, P, nN, nM, EX, EY, L, nt1, nt2, nch;
};
__global__ __launch_bounds__(QT) void k_quad_gather(GatherArgs a) {
    const int f = blockIdx.y, r = blockIdx.z;
    const int n1 = f == 0 ? a.nN : a.nM, n2 = f == 1 ? a.nN : a.nM, n3 = f == 2 ? a.nN : a.nM;
    const int S1 = a.EX + a.P, S2 = a.EY + a.P, S3 = a.L + a.P;
    const long long o = (long long)blockIdx.x * QT + threadIdx.x;
    if (o >= (long long)n1 * n2 * n3) return;
    const int i = (int)(o % n1), j = (int)((o / n1) % n2), k = (int)(o / ((long long)n1 * n2));
    // tiles of size e (the last one shorter) that hold function i: local index
    // i + n - e t (n = 1 for interior degree-p functions) in [0, size + P - 1 + n)
    auto range = [&](int idx, int n, int e, int nt, int& lo, int& hi) {
        hi = min(nt - 1, (idx + n) / e);
        lo = max(0, (idx + n - (e + a.P - 1 + n) + e) / e);
        if (idx + n < e + a.P - 1 + n) lo = 0;
    };
    int a0, a1, b0, b1, c0, c1;
    const int m1 = f == 0, m2 = f == 1, m3 = f == 2;
    range(i, m1, a.EX, a.nt1, a0, a1);
    range(j, m2, a.EY, a.nt2, b0, b1);
    range(k, m3, a.L, a.nch, c0, c1);
    double s = 0.0;
    for (int c = c0; c <= c1; ++c)
        for (int b = b0; b <= b1; ++b)
            for (int t = a0; t <= a1; ++t) {
                const long long blk = (((long long)r * a.nch + c) * a.nt2 + b) * a.nt1 + t;
                s += a.scratch[(((blk * 4 + f) * S3 + (k + m3 - a.L * c)) * S2 + (j + m2 - a.EY * b)) * S1 +
                               (i + m1 - a.EX * t)];
            }
    a.y[f][r * a.sy[f] + o] = s;
}

void tile_size(int p, int& ex, int& ey) {
    switch (p) {
        case 2: ex = Tile2<2>::EX; ey = Tile2<2>::EY; break;
        case 3: ex = Tile2<3>::EX; ey = Tile2<3>::EY; break;
        case 4: ex = Tile2<4>::EX; ey = Tile2<4>::EY; break;
        case 5: ex = Tile2<5>::EX; ey = Tile2<5>::EY; break;
        case 6: ex = Tile2<6>::EX; ey = Tile2<6>::EY; break;
        case 7: ex = Tile2<7>::EX; ey = Tile2<7>::EY; break;
        default: ex = Tile2<8>::EX; ey = Tile2<8>::EY; break;
    }
}

// Right-hand sides per launch: the scratch holds this many.
constexpr int QUAD_RHS = 8;

}  // namespace

static hipError_t make_quad(hp_ctx* c, QuadOp* q) {
    const QuadTables1D Q = build_quad_tables(c->tab);
    const int p = c->p, W = p + 1, E = c->E, nq = Q.nq, nN = c->nN, nM = c->nM;
    q->nq = nq;
    tile_size(p, q->ex, q->ey);
    q->nt1 = (E + q->ex - 1) / q->ex;
    q->nt2 = (E + q->ey - 1) / q->ey;
    // layers per chunk: fewest rounds of resident workgroups x (layers + the
    // lighter steps before and after them, about half a layer each) for one
    // right-hand side (a batch takes the same chunks, hence the same sums)
    const long long slots = 256LL * quad_per_cu(p), tiles = (long long)q->nt1 * q->nt2;
    long long best = LLONG_MAX;
    for (int L = 1; L <= E; ++L) {
        const long long rounds = (tiles * ((E + L - 1) / L) + slots - 1) / slots;
        if (rounds * (2 * L + 2 * p + 1) < best) {
            best = rounds * (2 * L + 2 * p + 1);
            q->L = L;
        }
    }
    q->nch = (E + q->L - 1) / q->L;
    q->block_doubles = 4LL * (q->L + p) * (q->ey + p) * (q->ex + p);
    const size_t nr = (size_t)std::min(c->opts.max_rhs, QUAD_RHS);
    q->scratch_doubles = (size_t)q->nt1 * q->nt2 * q->nch * q->block_doubles * nr;
    // point tables: per point values and derivatives of the degree p-1
    // functions el .. el + p - 1 and of the interior degree-p functions
    // el - 1 .. el + p - 1 of its element el (zero where there is none)
    std::vector<double> h((size_t)nq * 4 * W, 0.0);
    for (int r = 0; r < nq; ++r) {
        const int el = r == 0 ? 0 : r == nq - 1 ? E - 1 : (r - 1) / W;
        double* t = h.data() + (size_t)r * 4 * W;
        for (int k = 0; k < W; ++k) {
            const int m = el + k, n = el - 1 + k;
            if (k < p && m < nM) {
                t[k] = Q.MV[(size_t)r * nM + m];
                t[W + k] = Q.MD[(size_t)r * nM + m];
            }
            if (n >= 0 && n < nN) {
                t[2 * W + k] = Q.NV[(size_t)r * nN + n];
                t[3 * W + k] = Q.ND[(size_t)r * nN + n];
            }
        }
    }
    const size_t wo = h.size();
    h.insert(h.end(), Q.w.begin(), Q.w.end());
    // an early error return releases what was allocated so far, so that a
    // later call starts again from an empty QuadOp
    auto fail = [q](hipError_t err) {
        quad_free(q);
        return err;
    };
    hipError_t e;
    if ((e = hipMalloc(&q->tables, sizeof(double) * h.size())) != hipSuccess) return fail(e);
    if ((e = hipMalloc(&q->scratch, sizeof(double) * q->scratch_doubles)) != hipSuccess)
        return fail(e);
    q->wq = q->tables + wo;
    if ((e = hipMemcpy(q->tables, h.data(), sizeof(double) * h.size(), hipMemcpyHostToDevice)) !=
        hipSuccess)
        return fail(e);
    q->ready = true;
    return hipSuccess;
}

// (no exception of the host tables may cross the C interface)
hipError_t quad_setup(hp_ctx* c, QuadOp* q) {
    if (q->ready) return hipSuccess;
    try {
        return make_quad(c, q);
    } catch (const std::bad_alloc&) {
        quad_free(q);
        return hipErrorOutOfMemory;
    } catch (const std::exception&) {
        quad_free(q);
        return hipErrorInvalidValue;
    }
}

void quad_free(QuadOp* q) {
    if (q->tables) (void)hipFree(q->tables);
    if (q->scratch) (void)hipFree(q->scratch);
    *q = QuadOp{};
}

hipError_t launch_quad_K(hp_ctx* c, const QuadOp* q, const Fields& in, const Fields& out,
                         int nrhs) {
    if (!q->ready) return hipErrorNotInitialized;
    const int cap = std::min(c->opts.max_rhs, QUAD_RHS);
    for (int r0 = 0; r0 < nrhs; r0 += cap) {
        const int nr = std::min(cap, nrhs - r0);
        QuadArgs a{};
        GatherArgs g{};
        for (int f = 0; f < 4; ++f) {
            a.x[f] = in.f[f] + (long long)r0 * in.stride[f];
            a.sx[f] = in.stride[f];
            g.y[f] = out.f[f] + (long long)r0 * out.stride[f];
            g.sy[f] = out.stride[f];
        }
        a.tab = q->tables;
        a.wq = q->wq;
        a.scratch = q->scratch;
        a.E = g.E = c->E;
        a.nN = g.nN = c->nN;
        a.nM = g.nM = c->nM;
        a.nq = q->nq;
        a.L = g.L = q->L;
        a.nch = g.nch = q->nch;
        a.nt1 = g.nt1 = q->nt1;
        a.nt2 = g.nt2 = q->nt2;
        a.nu = c->nu;
        a.alpha = c->tab.alpha;
        const dim3 grid(q->nt1 * q->nt2, q->nch, nr), b(QT);
        switch (c->p) {
            case 2: hipLaunchKernelGGL(k_quad<2>, grid, b, 0, c->stream, a); break;
            case 3: hipLaunchKernelGGL(k_quad<3>, grid, b, 0, c->stream, a); break;
            case 4: hipLaunchKernelGGL(k_quad<4>, grid, b, 0, c->stream, a); break;
            case 5: hipLaunchKernelGGL(k_quad<5>, grid, b, 0, c->stream, a); break;
            case 6: hipLaunchKernelGGL(k_quad<6>, grid, b, 0, c->stream, a); break;
            case 7: hipLaunchKernelGGL(k_quad<7>, grid, b, 0, c->stream, a); break;
            case 8: hipLaunchKernelGGL(k_quad<8>, grid, b, 0, c->stream, a); break;
            default: return hipErrorInvalidValue;
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        g.scratch = q->scratch;
        g.P = c->p;
        g.EX = q->ex;
        g.EY = q->ey;
        const long long n = (long long)c->nM * c->nM * c->nM;
        hipLaunchKernelGGL(k_quad_gather, dim3((unsigned)((n + QT - 1) / QT), 4, nr), b, 0, c->stream, g);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace hp

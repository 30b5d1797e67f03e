// Base preconditioner P_0^{-1} (Sec. 4, eq. blockdiagprecond) on MFMA.
//
// Velocity block c: the diagonal block A_cc is a generalised Kronecker sum
// (Sec. 3.3, App. A.3) of (K_int, M_int) in direction c and (T^, M^) in the
// other two.  With the generalised eigenpairs U^T M U = I, U^T K U = Lambda,
// fast diagonalisation (App. A.4) gives
//     A_cc^{-1} = (U3 (x) U2 (x) U1) diag(1 / (2 nu (l1 + l2 + l3))) (U3 (x) U2 (x) U1)^T.
// Pressure: P_{Q,0}^{-1} = 2 nu (M^^{-1})^{(x)3} (dense 1D inverses).
//
// Parity split.  On the uniform mesh every 1D matrix commutes with the
// reversal i -> n-1-i, so its eigenvectors are even or odd (setup1d.cpp
// computes them in the two subspaces).  With the folds e_i = x_i + x_{n-1-i}
// (the middle entry of an odd n once) and o_i = x_i - x_{n-1-i}, a transform
// of length n is two products of half the length, U^T x = [F_e e | F_o o],
// and back y_i = E_i + O_i, y_{n-1-i} = E_i - O_i with E = V_e c_e,
// O = V_o c_o: half the products of the dense form.  M^^{-1} splits the same
// way (fold, two half products, unfold).  Spectral vectors keep the order
// [even modes | odd modes].
//
// The products run as 16x16x4 MFMA tiles (FP64 or FP32 operands, or split
// BF16, see mm4).  The 1D matrices are stored as MFMA fragments: tile (u, t)
// of a matrix is 64 x 4 values, lane l holding its four contraction values
// contiguously, so a fragment is one fully coalesced 16- or 32-byte load per
// lane from L2.  The contraction index of step i and lane group lk is
// kmap(lk, i), which is also the row of element i of an MFMA result: a result
// tile can therefore be the other operand of a following product as it lies
// in registers.
//   plane (n <= 128): one i3-plane per workgroup, modes 1 and 2: the plane is
//     folded into LDS, a wave takes 16 outputs of direction 1 and one parity
//     through both products without a further barrier or LDS pass;
//   line: 16 CT columns x the whole direction 2 or 3: mode 3 forward, scaling
//     and inverse in one pass, or one product;
//   row: 16 CT lines of direction 1, one product.
// P_0 is plane, line (mode 3), plane, or, one direction per pass, row, line,
// line (mode 3), line, row.  Measured, FP64 (us; before: dense products, the
// whole plane by 16 waves, from 129 per direction six batched GEMMs per
// component): 32^3 degree 3 20.8 -> 19.7, 61^3 44 -> 30, 96^3 228 -> 124,
// 192^3 2155 -> 1143, 256^3 degree 2 4930 -> 2756; FP32, 32 right-hand sides
// at 48^3 degree 2: 676 -> 190.
#include <algorithm>
#include <climits>
#include <type_traits>

#include "fd_layout.h"
#include "hp_internal.h"
#include "vec.h"

namespace hp {

namespace {

constexpr int FD_PLANE_MAX = 128;     // longest direction of the plane kernel
constexpr size_t FD_LDS = 160 * 1024;

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf4 __attribute__((ext_vector_type(4)));

// Operand layout of both 16x16x4 forms: lane l holds A[l%16][l/16] and
// B[l/16][l%16].  Result element i of lane l is D[kmap(l/16, i)][l%16]; the
// row map differs between the FP64 and FP32 instructions (measured).
template <typename T>
struct Mfma;
template <>
struct Mfma<double> {
    using V = d4;
    static __device__ __forceinline__ V mma(double a, double b, V c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __host__ __device__ constexpr int kmap(int lk, int i) { return mfma_row<double>(lk, i); }
    static __device__ __forceinline__ int steps(int rem) { return mfma_steps<double>(rem); }
};
template <>
struct Mfma<float> {
    using V = f4;
    static __device__ __forceinline__ V mma(float a, float b, V c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __host__ __device__ constexpr int kmap(int lk, int i) { return mfma_row<float>(lk, i); }
    static __device__ __forceinline__ int steps(int rem) { return mfma_steps<float>(rem); }
};

// Split-BF16 ("bf16x3") products for FP32 data: each operand is written as
// hi + lo with hi = bf16(x), lo = bf16(x - hi) (round to nearest even), and
// A B ~= A_hi B_hi + A_hi B_lo + A_lo B_hi, three 16x16x16 BF16 MFMAs per
// 16-wide k step accumulated in FP32.  hi + lo keeps 16 significant bits of
// each operand (relative error up to 2^-17), so a product is good to about
// 1e-5 relative, not to FP32 rounding; the dropped lo*lo term is of the
// same order.  A lane supplies the four values k = 16c + 4 lk + j, which is
// kmap for FP32.
struct Bf2 {
    bf4 hi, lo;
};
__device__ __forceinline__ Bf2 split_bf16(f4 x) {
    Bf2 r;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const __bf16 h = (__bf16)x[j];
        r.hi[j] = h;
        r.lo[j] = (__bf16)(x[j] - (float)h);
    }
    return r;
}

// acc += A B over the first N (of four) steps of a 16-wide contraction tile, a
// and b the lane's four values of the two operands.
template <typename T, bool SPLIT, int N>
__device__ __forceinline__ void mm(typename Mfma<T>::V& acc, typename Mfma<T>::V a,
                                   typename Mfma<T>::V b) {
    if constexpr (SPLIT) {
        const Bf2 x = split_bf16(a), y = split_bf16(b);
        acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(x.hi, y.hi, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(x.hi, y.lo, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(x.lo, y.hi, acc, 0, 0, 0);
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) acc = Mfma<T>::mma(a[i], b[i], acc);
    }
}

// Of the nt contraction tiles of a half all but the last are full (he and ho of
// nN and nM differ by at most one); fn gets the last one's step count as a
// constant, so that no branch stands between the MFMAs (branches there made
// the compiler copy the accumulators around: 112 spilled registers).
template <typename F>
__device__ __forceinline__ void tail_steps(int st, F fn) {
    if (st == 4) fn(std::integral_constant<int, 4>{});
    else if (st == 2) fn(std::integral_constant<int, 2>{});
    else if (st == 1) fn(std::integral_constant<int, 1>{});
}

// One direction of one field: its length, the sizes of the even and odd
// halves and the fragment table (forward F, inverse V; for the pressure both
// are M^^{-1}): nt x nt tiles of the even half, then of the odd half, with
// nt = half_tiles(nM) for every table.
template <typename T>
struct Dir {
    int n, he, ho;
    const T* tab;
};
template <typename T>
__device__ __forceinline__ Dir<T> dir_of(const FDTables<T>& t, int f, int d, bool inverse) {
    const int fam = f == 3 ? 2 : (d == f ? 0 : 1);
    Dir<T> r;
    r.n = fam == 0 ? t.nN : t.nM;
    r.he = (r.n + 1) >> 1;
    r.ho = r.n >> 1;
    r.tab = fam == 2 ? t.Mi : (inverse ? t.V[fam] : t.F[fam]);
    return r;
}
template <typename T>
__device__ __forceinline__ typename Mfma<T>::V frag(const T* tab, int tile, int lane) {
    return *reinterpret_cast<const typename Mfma<T>::V*>(tab + (tile * 64 + lane) * 4);
}

// Memory access through buffer resources: a base in scalar registers and a
// 32-bit byte offset per lane.  Lanes without an element take the offset OOB,
// beyond every buffer: their loads return zero and their stores are dropped.
constexpr uint32_t OOB = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_at(const void* base) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, 0x7ffffff8,
                                             0x00020000);
}
template <typename T>
__device__ __forceinline__ T bload(const T* base, uint32_t off) {
    if constexpr (sizeof(T) == 8)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(buffer_at(base), (int)off, 0, 0));
    else
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(buffer_at(base), (int)off, 0, 0));
}
// Two neighbours of an array of `bytes` bytes; what lies beyond reads as zero.
template <typename T>
__device__ __forceinline__ void bload2(const T* base, uint32_t bytes, uint32_t off, T (&v)[2]) {
    const auto r = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(base), (short)0, (int)bytes,
                                                     0x00020000);
    if constexpr (sizeof(T) == 8) {
        typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
        const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0);
        v[0] = __builtin_bit_cast(T, (uint64_t)w.x | ((uint64_t)w.y << 32));
        v[1] = __builtin_bit_cast(T, (uint64_t)w.z | ((uint64_t)w.w << 32));
    } else {
        typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
        const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0);
        const unsigned int lo = w.x, hi = w.y;  // (a cast of w.y itself reads w.x)
        v[0] = __builtin_bit_cast(T, lo);
        v[1] = __builtin_bit_cast(T, hi);
    }
}
template <typename T>
__device__ __forceinline__ void bstore(T* base, uint32_t off, T v) {
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    if constexpr (sizeof(T) == 8)
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), buffer_at(base), (int)off, 0, 0);
    else
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), buffer_at(base), (int)off, 0, 0);
}

// Sum over the workgroup in a fixed order (wave trees, then the waves in
// order); valid in thread 0.  red: one value per wave.
__device__ __forceinline__ double wg_sum(double s, double* red) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += red[w];
    return t;
}

// One field of one set of right-hand sides; a launch takes one or two sets of
// nr each (P_k: the V block's residual beside the Q block's B P_{Q,0}^{-1} s).
// All that a workgroup reads of it is one cache line of the kernel arguments
// (spread over arrays per member, P_0 at 32^3 took 20.1 us instead of 19.7).
struct alignas(64) FieldIO {
    const void* in;
    void* out;
    long long sin, sout;  // per-rhs strides
    const double* dw;     // the dot's other vector (dpart set), rhs stride sout
    int dims[3];
    int add;              // the result is added to the output
};

// ---- modes 1 and 2 of one i3-plane -----------------------------------------------------
struct PlaneArgs {
    int nr;
    int fields_lo, nf;
    int inverse;                // velocity: 0 forward (fold, F), 1 inverse (V, unfold)
    int comb;                   // the pressure's input is a combination (below)
    FieldIO io[2][4];
    // FP64 output only: partial sums of (stored output) . dw per (field,
    // plane) to dpart[r * dp_stride + f * dp_planes + k] (dpart null: none)
    double* dpart;
    long long dp_stride;
    int dp_planes;
    // FP64 input only, comb: the pressure's input is ca in + cb inb + cc inc
    // (the same layout as in, rhs strides sinb, sinc), formed in the operation
    // order of the vector kernel k_axpbypcz
    const double* inb;
    const double* inc;
    long long sinb, sinc;
    double ca, cb, cc;
};

// NT: tiles per half direction (nM's).  Wave (a, u1): D1 = X^T L^T for the 16
// outputs i' of parity a and tile u1 of direction 1 and every j (contraction
// over i, operands LDS and fragments held in registers), then D2 = R^T D1 per
// parity of direction 2 (contraction over j = the rows of D1, which lie in
// the registers as the B operand).  Up to two tiles per half (n <= 64) the
// two parities of direction 2 go to two waves, for shorter chains.
// The fragments of the second product are loaded RING - 1 tiles ahead, the
// first ones before the plane.
// What bounds it: MFMA issue (64 cycles per FP64 instruction), and at small
// meshes the latency of launch, staging and write-out.
template <typename T, typename TI, typename TO, bool SPLIT, int NT>
__global__ __launch_bounds__(NT <= 2 ? 256 * NT : 128 * NT)
__attribute__((amdgpu_waves_per_eu(4))) void k_fd_plane(PlaneArgs a,
                                                                             FDTables<T> t) {
    using M = Mfma<T>;
    using V = typename M::V;
    constexpr int NB = NT <= 2 ? 1 : 2;   // parities of direction 2 per wave
    constexpr int NTH = (NB == 1 ? 256 : 128) * NT;
    constexpr int RING = 4, NF = NB * NT * NT;
    extern __shared__ unsigned char smem_raw[];
    T* S = reinterpret_cast<T*>(smem_raw);
    const int f = a.fields_lo + (int)blockIdx.y;
    const int set = (int)blockIdx.z >= a.nr, r = (int)blockIdx.z - set * a.nr;
    const FieldIO& io = a.io[set][f];
    const int k = blockIdx.x;
    const int n1 = io.dims[0], n2 = io.dims[1];
    if (k >= io.dims[2]) return;
    const bool pres = f == 3;
    const bool fold = !a.inverse, unfold = a.inverse || pres;
    const Dir<T> d1 = dir_of(t, f, 0, a.inverse), d2 = dir_of(t, f, 1, a.inverse);
    const int he1 = d1.he, ho1 = d1.ho, he2 = d2.he, ho2 = d2.ho;
    const int ld = plane_pitch<T>(n1);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lr = lane & 15, lk = lane >> 4;
    const int pa = wave & 1, u1 = (wave >> 1) % NT, b0 = NB == 1 ? wave / (2 * NT) : 0;
    const int ha = pa ? ho1 : he1, offa = pa ? he1 : 0;
    const bool mine = 16 * u1 < ha;
    // this wave's fragments of L, and the first of R^T (tile w: parity
    // b0 + w / NT^2, output tile (w / NT) % NT, contraction tile w % NT)
    V bl[NT], fr[RING];
    const T* tl = d1.tab + (pa * NT + u1) * NT * 256;
    const T* tr = d2.tab + b0 * NT * NT * 256;
    if (mine) {
#pragma unroll
        for (int q = 0; q < NT; ++q) bl[q] = frag(tl, q, lane);
#pragma unroll
        for (int w = 0; w < RING - 1; ++w)
            if (w < NF) fr[w] = frag(tr, w, lane);
    }
    const long long kofs = (long long)k * n1 * n2;
    const TI* x = reinterpret_cast<const TI*>(io.in) + (long long)r * io.sin + kofs;
    // a thread's groups (i, j): i, j of the first, advanced by NTH groups
    const int ng = he1 * he2, dj = NTH / he1, di = NTH - dj * he1;
    const int j00 = (int)threadIdx.x / he1, i00 = (int)threadIdx.x - j00 * he1;
    // the offsets of the four mirror images of (i, j)
    auto mirror = [&](int i, int j, int (&o)[4]) {
        const int p0 = j * n1, p1 = (n2 - 1 - j) * n1, i1 = n1 - 1 - i;
        o[0] = p0 + i;
        o[1] = p0 + i1;
        o[2] = p1 + i;
        o[3] = p1 + i1;
    };
    auto next = [&](int& i, int& j) {
        i += di;
        j += dj;
        if (i >= he1) {
            i -= he1;
            ++j;
        }
    };
    if (fold) {
        const double* xb = nullptr;
        const double* xc = nullptr;
        bool comb = false;
        if constexpr (std::is_same<TI, double>::value) {
            if (f == 3 && a.comb) {
                comb = true;
                if (a.cb != 0.0) xb = a.inb + (long long)r * a.sinb + kofs;
                if (a.cc != 0.0) xc = a.inc + (long long)r * a.sinc + kofs;
            }
        }
        int i0 = i00, j0 = j00;
        for (int base = threadIdx.x; base < ng; base += 2 * NTH) {
            TI v[2][4];
            double vb[2][4], vc[2][4];
            int gi[2], gj[2];
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                const bool on = base + g * NTH < ng;
                gi[g] = on ? i0 : 0;
                gj[g] = on ? j0 : 0;
                next(i0, j0);
                int o[4];
                mirror(gi[g], gj[g], o);
#pragma unroll
                for (int q = 0; q < 4; ++q) v[g][q] = x[o[q]];
                if (xb)
#pragma unroll
                    for (int q = 0; q < 4; ++q) vb[g][q] = xb[o[q]];
                if (xc)
#pragma unroll
                    for (int q = 0; q < 4; ++q) vc[g][q] = xc[o[q]];
            }
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                if (base + g * NTH >= ng) break;
                if (comb) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        double c = a.ca * (double)v[g][q];
                        if (xb) c += a.cb * vb[g][q];
                        if (xc) c += a.cc * vc[g][q];
                        v[g][q] = (TI)c;
                    }
                }
                const int i = gi[g], j = gj[g];
                const bool im = i >= ho1, jm = j >= ho2;  // the middle of an odd length
                const TI ep = im ? v[g][0] : v[g][0] + v[g][1], op = v[g][0] - v[g][1];
                const TI eq = im ? v[g][2] : v[g][2] + v[g][3], oq = v[g][2] - v[g][3];
                S[j * ld + i] = (T)(jm ? ep : ep + eq);
                if (!im) S[j * ld + he1 + i] = (T)(jm ? op : op + oq);
                if (!jm) S[(he2 + j) * ld + i] = (T)(ep - eq);
                if (!im && !jm) S[(he2 + j) * ld + he1 + i] = (T)(op - oq);
            }
        }
    } else {
        // Pairs, four in flight: lanes past the plane repeat its last pair, so
        // that no load stands in a branch (the compiler moved each there, behind
        // the wait for the one before: P_0 at 64^3 53.7 -> 52.6 us, FP32 42.6 ->
        // 41.3).  The row of entry i is exact in FP32:
        // the quotient's distance from an integer is 1/256 or more.
        const int n = n1 * n2, np = (n + 1) >> 1;
        const float rn = 1.0f / (float)n1;
        for (int base = threadIdx.x; base < np; base += 4 * NTH) {
            TI v[4][2];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int i = 2 * min(base + g * NTH, np - 1);
                bload2(x, (uint32_t)sizeof(TI) * n, (uint32_t)sizeof(TI) * i, v[g]);
            }
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int i = 2 * min(base + g * NTH, np - 1);
                const int j = (int)(((float)i + 0.5f) * rn), c = i - j * n1;
                const int o0 = j * ld + c, o1 = o0 + (c + 1 < n1 ? 1 : ld - c);
                const bool two = i + 1 < n;
                S[o0] = (T)v[g][0];
                S[two ? o1 : o0] = (T)(two ? v[g][1] : v[g][0]);
            }
        }
    }
    {
        // the columns past n1 that a last MFMA step reads (times zeros)
        const int pw = ld - n1;
        for (int idx = threadIdx.x; idx < pw * n2; idx += NTH) {
            const int j = idx / pw;
            S[j * ld + n1 + (idx - j * pw)] = T(0);
        }
    }
    __syncthreads();
    V D1[NB][NT];
    if (mine) {
        int row[NB][NT];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int q = 0; q < NT; ++q) {
                // rows past the half multiply zeros in the second product
                row[b][q] = min((b0 + b ? he2 : 0) + 16 * q + lr, n2 - 1) * ld + offa;
                D1[b][q] = V{0, 0, 0, 0};
            }
        auto tile = [&](int c, auto steps) {
            constexpr int N = decltype(steps)::value;
            V av[NB][NT];
#pragma unroll
            for (int i = 0; i < (SPLIT ? 4 : N); ++i)
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int q = 0; q < NT; ++q)
                        av[b][q][i] = S[row[b][q] + 16 * c + M::kmap(lk, i)];
            if constexpr (SPLIT) {
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int q = 0; q < NT; ++q) mm<T, true, 4>(D1[b][q], av[b][q], bl[c]);
            } else {
#pragma unroll
                for (int i = 0; i < N; ++i)
#pragma unroll
                    for (int b = 0; b < NB; ++b)
#pragma unroll
                        for (int q = 0; q < NT; ++q)
                            D1[b][q] = M::mma(av[b][q][i], bl[c][i], D1[b][q]);
            }
        };
#pragma unroll
        for (int c = 0; c + 1 < NT; ++c) tile(c, std::integral_constant<int, 4>{});
        tail_steps(M::steps(ha - 16 * (NT - 1)), [&](auto st) { tile(NT - 1, st); });
    }
    TO* y = reinterpret_cast<TO*>(io.out) + (long long)r * io.sout + kofs;
    if (unfold) __syncthreads();  // every wave is done with the input plane
    if (mine) {
        const int col = 16 * u1 + lr;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int hb = b0 + b ? ho2 : he2, offb = b0 + b ? he2 : 0;
#pragma unroll
            for (int u = 0; u < NT; ++u) {
                V acc = {0, 0, 0, 0};
#pragma unroll
                for (int q = 0; q < NT; ++q) {
                    const int w = (b * NT + u) * NT + q;
                    if (w + RING - 1 < NF) fr[(w + RING - 1) % RING] = frag(tr, w + RING - 1, lane);
                    if (q + 1 < NT)
                        mm<T, SPLIT, 4>(acc, fr[w % RING], D1[b][q]);
                    else
                        tail_steps(M::steps(hb - 16 * q), [&](auto st) {
                            mm<T, SPLIT, decltype(st)::value>(acc, fr[w % RING], D1[b][q]);
                        });
                }
                if (col < ha)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int j = 16 * u + M::kmap(lk, i);
                        if (j < hb) {
                            if (unfold) S[(offb + j) * ld + offa + col] = acc[i];
                            else y[(offb + j) * n1 + offa + col] = (TO)acc[i];
                        }
                    }
            }
        }
    }
    if (!unfold) return;
    __syncthreads();
    // y = unfold(S), or y += unfold(S): the four mirror images of (i, j)
    const bool add = io.add;
    const bool dot = std::is_same<TO, double>::value && a.dpart != nullptr;
    const double* w = dot ? io.dw + (long long)r * io.sout + kofs : nullptr;
    double sum = 0.0;
    int i0 = i00, j0 = j00;
    for (int base = threadIdx.x; base < ng; base += 2 * NTH) {
        TO yv[2][4];
        double wv[2][4];
        int o[2][4], gi[2], gj[2];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const bool on = base + g * NTH < ng;
            gi[g] = on ? i0 : 0;
            gj[g] = on ? j0 : 0;
            next(i0, j0);
            mirror(gi[g], gj[g], o[g]);
            if (add)
#pragma unroll
                for (int q = 0; q < 4; ++q) yv[g][q] = y[o[g][q]];
            if (dot)
#pragma unroll
                for (int q = 0; q < 4; ++q) wv[g][q] = w[o[g][q]];
        }
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            if (base + g * NTH >= ng) break;
            const int i = gi[g], j = gj[g];
            const bool im = i >= ho1, jm = j >= ho2;
            const T ee = S[j * ld + i], oe = im ? T(0) : S[j * ld + he1 + i];
            const T eo = jm ? T(0) : S[(he2 + j) * ld + i];
            const T oo = (im || jm) ? T(0) : S[(he2 + j) * ld + he1 + i];
            const T pe = ee + oe, po = eo + oo, me = ee - oe, mo = eo - oo;
            const T v[4] = {pe + po, me + mo, pe - po, me - mo};
            const bool on[4] = {true, !im, !jm, !im && !jm};
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (on[q]) {
                    TO s = (TO)v[q];
                    if (add) s += yv[g][q];
                    y[o[g][q]] = s;
                    if (dot) sum += (double)s * wv[g][q];
                }
        }
    }
    if (dot) {
        __syncthreads();
        const double s = wg_sum(sum, reinterpret_cast<double*>(smem_raw));
        if (threadIdx.x == 0)
            a.dpart[(long long)r * a.dp_stride + (long long)f * a.dp_planes + k] = s;
    }
}

// ---- one direction per pass ----------------------------------------------------------------
// A workgroup takes a tile: 16 CT columns or lines of one field, right-hand
// side and, for direction 2, i3-plane; each XCD a contiguous range of the
// tiles.  Wave w takes output tile u = w of both parities, so that the unfold
// y = E +- O happens in registers; beyond one tile per wave the further ones
// are dealt round-robin from a start that changes with the workgroup, so that
// a short last round does not always load the same SIMD.  Eight waves from
// nt = 8 on: two per SIMD (nine, one per tile at 257 per direction, left room
// for one workgroup per CU only).  Several workgroups per CU overlap one's loads and stores with
// another's products; looking ahead to the next tile in registers instead
// (one resident workgroup walking several tiles) spilled and was slower.
struct LineArgs {
    int nr;
    int fields_lo, nf;
    int dir;          // 0: row kernel, 1: direction 2, 2: direction 3
    int inverse;      // one product: 0 forward (fold, F), 1 inverse (V, unfold)
    int fused;        // direction 3: the velocity's forward product, scaling and inverse product
    int ctiles, nbatch, ntiles;  // tiles per (field, rhs, plane), planes, tiles in all
    double two_nu;
    double omega;     // damping factor of P_0^{-1} (1: the plain base preconditioner)
    double pscale;    // the pressure's product is multiplied by this
    FieldIO io[2][4];
    // FP64 output: partial sums of (stored pressure) . dw per tile, or per 16
    // columns (dp_cols: the same sums for tiles of 16 and of 32), to
    // dpart[r * dp_stride + index]
    int dp_cols;
    double* dpart;
    long long dp_stride;
};

template <typename T, int CT>
constexpr int line_pitch() {
    // FP32 operands read rows 4 apart: 4 more words put them in other banks
    return 16 * CT + (std::is_same<T, double>::value ? 0 : 4);
}

// Workgroups are dealt round-robin to the 8 XCDs in launch order: workgroup i
// to the tile, so that an XCD's tiles are one contiguous range.
__device__ __forceinline__ int xcd_tile(int i, int total) {
    const int per = total / 8, rem = total % 8, x = i % 8;
    return x * per + min(x, rem) + i / 8;
}

struct Tile {
    int c, b, f, set, r;  // column tile, plane, field, set, right-hand side
};
__device__ __forceinline__ Tile tile_of(const LineArgs& a, int id) {
    Tile w;
    w.c = id % a.ctiles;
    id /= a.ctiles;
    w.b = id % a.nbatch;
    id /= a.nbatch;
    w.f = a.fields_lo + id % a.nf;
    id /= a.nf;
    w.set = id >= a.nr;
    w.r = id - w.set * a.nr;
    return w;
}

// Both parities of one product with the fragments of tab, output tile u:
// acc[h][c] += table tile . operand, operand value i of lane (lr, lk) from
// opnd(h, c, 16 s, i), i.e. contraction index 16 s + kmap(lk, i).  TA: the
// table is the A operand.
// Fragments are loaded ahead: a contraction tile of both parities (two tiles
// in registers) or, LEAN, one parity's fragment (the directions beyond 128,
// where the registers saved give a second workgroup per CU).
template <typename T, bool SPLIT, bool TA, int CT, bool LEAN>
struct HalfProduct {
    using M = Mfma<T>;
    using V = typename M::V;
    const T* tab;
    int u, nt, he, ho, lane;
    V g0[2], g1[2];  // LEAN: g0[0] and g1[0] only
    __device__ __forceinline__ V load(int s, int h) const {
        return frag(tab, (h * nt + u) * nt + min(s, nt - 1), lane);
    }
    // the first fragments, to be in flight before the operand is ready
    __device__ __forceinline__ void prime(const T* table) {
        tab = table;
        g0[0] = load(0, 0);
        if constexpr (LEAN) {
            g1[0] = 16 * u < ho ? load(0, 1) : load(1, 0);
        } else {
            g0[1] = load(0, 1);
            g1[0] = load(1, 0);
            g1[1] = load(1, 1);
        }
    }
    // N steps of tile s of parity h with the fragment g
    template <int N, typename F>
    __device__ __forceinline__ void step(const V& g, int s, int h, V (&acc)[CT], F opnd) const {
        V b[CT];
#pragma unroll
        for (int i = 0; i < (SPLIT ? 4 : N); ++i)
#pragma unroll
            for (int c = 0; c < CT; ++c) b[c][i] = opnd(h, c, 16 * s, i);
        if constexpr (SPLIT) {
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                if (TA) mm<T, true, 4>(acc[c], g, b[c]);
                else mm<T, true, 4>(acc[c], b[c], g);
            }
        } else {
#pragma unroll
            for (int i = 0; i < N; ++i)
#pragma unroll
                for (int c = 0; c < CT; ++c)
                    acc[c] = TA ? M::mma(g[i], b[c][i], acc[c]) : M::mma(b[c][i], g[i], acc[c]);
        }
    }
    // NH parities (1: there is no odd output tile u)
    template <int NH, typename F>
    __device__ __forceinline__ void loop(V (&acc)[2][CT], F opnd) {
#pragma unroll 1
        for (int s = 0; s + 1 < nt; ++s) {
#pragma unroll
            for (int h = 0; h < NH; ++h) {
                if constexpr (LEAN) {
                    step<4>(g0[0], s, h, acc[h], opnd);
                    g0[0] = g1[0];
                    g1[0] = NH == 2 ? load(s + 1, h) : load(s + 2, 0);
                } else {
                    step<4>(g0[h], s, h, acc[h], opnd);
                    g0[h] = g1[h];
                    g1[h] = load(s + 2, h);
                }
            }
        }
        // the even half's steps serve the odd half too (no more than one fewer)
        tail_steps(M::steps(he - 16 * (nt - 1)), [&](auto st) {
            constexpr int N = decltype(st)::value;
            step<N>(g0[0], nt - 1, 0, acc[0], opnd);
            if (NH == 2) step<N>(LEAN ? g1[0] : g0[1], nt - 1, 1, acc[1], opnd);
        });
    }
    template <typename F>
    __device__ __forceinline__ void run(V (&acc)[2][CT], F opnd) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int c = 0; c < CT; ++c) acc[h][c] = V{0, 0, 0, 0};
        if (16 * u < ho) loop<2>(acc, opnd);
        else loop<1>(acc, opnd);
    }
};

// Direction 2 or 3 of 16 CT columns: the columns are contiguous (the B
// operand, [k][column] in LDS), the table is the A operand.  Mode 3 forward,
// scaling by omega / (2 nu (l1 + l2 + l3)) and inverse run in one pass: the
// scaled tiles of the first product replace its operand in LDS.  The division
// is the correctly rounded one, over the whole range of nu (an estimate with two
// Newton steps: P_0 at 32^3 19.3 us instead of 19.6, but an ulp more and NaN
// where the sum overflows).
template <typename T, typename TI, typename TO, bool SPLIT, int CT, int NW>
__global__ __launch_bounds__(64 * NW)
__attribute__((amdgpu_waves_per_eu(4))) void k_fd_line(LineArgs a, FDTables<T> t) {
    using M = Mfma<T>;
    using V = typename M::V;
    constexpr int W = 16 * CT, P = line_pitch<T, CT>();
    constexpr int U = NW == 4 ? 1 : (NW == 8 ? 2 : 3);
    // pairs (k, n-1-k) a thread has in flight: the whole tile to 320 per direction
    constexpr int NG = NW == 4 ? 4 * CT : (NW == 8 ? 10 : 4);
    extern __shared__ unsigned char smem_raw[];
    const int nt = t.nt;
    T* X[2];
    X[0] = reinterpret_cast<T*>(smem_raw);
    X[1] = X[0] + 16 * nt * P;
    const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lr = lane & 15, lk = lane >> 4;
    const bool d3 = a.dir == 2;
    const int sc = threadIdx.x % W, sk = threadIdx.x / W, ks = blockDim.x / W;
    const int turn = (wave + (int)blockIdx.x) % nw;
    auto tile_u = [&](int q) { return q == 0 ? wave : q * nw + turn; };
    const Tile w = tile_of(a, xcd_tile(blockIdx.x, a.ntiles));
    const int f = w.f, r = w.r;
    const FieldIO& io = a.io[w.set][f];
    const int n1 = io.dims[0];
    const unsigned plane = (unsigned)n1 * io.dims[1];
    const unsigned ncol = d3 ? plane : (unsigned)n1;  // columns, and the direction's stride
    const unsigned c0 = (unsigned)w.c * W;
    if (c0 >= ncol || (!d3 && w.b >= io.dims[2])) return;
    const long long ofs = (d3 ? 0 : (long long)w.b * plane) + c0;
    const bool pres = f == 3, second = a.fused && !pres;
    const bool fold = !a.inverse, unfold = a.inverse || a.fused || pres;
    const Dir<T> d = dir_of(t, f, a.dir, a.inverse);
    const int n = d.n, he = d.he, ho = d.ho;
    HalfProduct<T, SPLIT, true, CT, NW == 8> hp;
    hp.u = min(wave, nt - 1);
    hp.nt = nt;
    hp.he = he;
    hp.ho = ho;
    hp.lane = lane;
    hp.prime(d.tab);
    {
        // the pairs (k, n-1-k) (or (k, he + k)), k = kb + sk + g ks
        const TI* x = reinterpret_cast<const TI*>(io.in) + (long long)r * io.sin + ofs;
        const bool in = c0 + sc < ncol;
        const uint32_t o0 = (uint32_t)sizeof(TI) * (sk * ncol + sc);
        const uint32_t o1 = (uint32_t)sizeof(TI) * ((ks - 1 - sk) * ncol + sc);
#pragma unroll 1
        for (int kb = 0; kb < 16 * nt; kb += NG * ks) {
            TI v[NG][2];
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const int k = kb + g * ks;  // of the lanes with sk = 0
                const bool on = in && k + sk < he;
                v[g][0] = bload(x + (long long)k * ncol, on ? o0 : OOB);
                v[g][1] = fold ? bload(x + (long long)(n - k - ks) * ncol, on ? o1 : OOB)
                               : bload(x + (long long)(he + k) * ncol, in && k + sk < ho ? o0 : OOB);
            }
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const int k = kb + sk + g * ks;
                if (k >= 16 * nt) break;
                TI e = v[g][0], o = v[g][1];
                if (fold) {
                    o = v[g][0] - v[g][1];
                    e = k < ho ? v[g][0] + v[g][1] : v[g][0];
                }
                X[0][k * P + sc] = (T)e;
                X[1][k * P + sc] = k < ho ? (T)o : T(0);
            }
        }
    }
    __syncthreads();
    V acc[U][2][CT];
    auto opnd = [&](int h, int c, int k, int i) {
        return X[h][(k + M::kmap(lk, i)) * P + 16 * c + lr];
    };
    auto product = [&](const T* tab) {
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int u = tile_u(q);
            if (u >= nt) break;
            if (q > 0) {
                hp.u = u;
                hp.prime(tab);
            }
            hp.run(acc[q], opnd);
        }
    };
    product(d.tab);
    if (second) {
        const T* tab2 = dir_of(t, f, a.dir, true).tab;
        hp.u = min(wave, nt - 1);
        hp.prime(tab2);
        const double* t1 = t.lam[f == 0 ? 0 : 1];
        const double* t2 = t.lam[f == 1 ? 0 : 1];
        const double* t3 = t.lam[f == 2 ? 0 : 1];
        double l12[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const unsigned rr = min(c0 + 16 * c + lr, ncol - 1);
            const unsigned i2 = rr / (unsigned)n1;
            l12[c] = t1[rr - i2 * n1] + t2[i2];
        }
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int u = tile_u(q);
            if (u >= nt) break;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int m = 16 * u + M::kmap(lk, i);
                    const bool ok = m < (h ? ho : he);
                    const double l3 = t3[min(h * he + m, n - 1)];
#pragma unroll
                    for (int c = 0; c < CT; ++c)
                        acc[q][h][c][i] = ok ? (T)(a.omega / (a.two_nu * (l12[c] + l3)) *
                                                   (double)acc[q][h][c][i])
                                             : T(0);
                }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int u = tile_u(q);
            if (u >= nt) break;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int c = 0; c < CT; ++c)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        X[h][(16 * u + M::kmap(lk, i)) * P + 16 * c + lr] = acc[q][h][c][i];
        }
        __syncthreads();
        product(tab2);
    }
    TO* y = reinterpret_cast<TO*>(io.out) + (long long)r * io.sout + ofs;
    const bool add = io.add;
    const bool dot = std::is_same<TO, double>::value && pres && a.dpart != nullptr;
    const double* dw = dot ? io.dw + (long long)r * io.sout + ofs : nullptr;
    const double ps = pres ? a.pscale : 1.0;
    double sum[CT] = {};
#pragma unroll
    for (int q = 0; q < U; ++q) {
        const int u = tile_u(q);
        if (u >= nt) break;
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const unsigned col = 16 * c + lr;
            const bool in = c0 + col < ncol;
            // rows 16 u + kmap(lk, i) (and their mirror images), from the
            // row of lk = 0 (of the last lk)
            constexpr int S = M::kmap(1, 0), E3 = 3 * S;
            const uint32_t o0 = (uint32_t)sizeof(TO) * (lk * S * ncol + col);
            const uint32_t o1 = (uint32_t)sizeof(TO) * ((E3 - lk * S) * ncol + col);
            TO yv[4][2];
            double wv[4][2];
            uint32_t o[4][2];
            long long ro[4][2];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int m0 = 16 * u + M::kmap(0, i), m = m0 + lk * S;
                ro[i][0] = (long long)m0 * ncol;
                ro[i][1] = (long long)(unfold ? n - 1 - m0 - E3 : he + m0) * ncol;
                o[i][0] = in && m < he ? o0 : OOB;
                o[i][1] = in && m < ho ? (unfold ? o1 : o0) : OOB;
                if (add)
#pragma unroll
                    for (int h = 0; h < 2; ++h) yv[i][h] = bload(y + ro[i][h], o[i][h]);
                if (dot)
#pragma unroll
                    for (int h = 0; h < 2; ++h) wv[i][h] = bload(dw + ro[i][h], o[i][h]);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const T E = acc[q][0][c][i], O = acc[q][1][c][i];
                T z[2] = {E, O};
                if (unfold) {
                    z[0] = o[i][1] != OOB ? E + O : E;
                    z[1] = E - O;
                }
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    TO s = pres ? (TO)(ps * (double)z[h]) : (TO)z[h];
                    if (add) s += yv[i][h];
                    bstore(y + ro[i][h], o[i][h], s);
                    if (dot) sum[c] += o[i][h] != OOB ? (double)s * wv[i][h] : 0.0;
                }
            }
        }
    }
    if (dot) {
        double* red = reinterpret_cast<double*>(smem_raw);
        double* part = a.dpart + (long long)r * a.dp_stride;
        if (!a.dp_cols) {
            for (int c = 1; c < CT; ++c) sum[0] += sum[c];
            __syncthreads();
            const double s = wg_sum(sum[0], red);
            if (threadIdx.x == 0) part[w.c] = s;
            return;
        }
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            __syncthreads();
            const double s = wg_sum(sum[c], red);
            const int o = CT * w.c + c;
            if (threadIdx.x == 0 && o < a.dp_stride) part[o] = s;
        }
    }
}

// Direction 1 of 16 CT lines.  The lines are contiguous: rows of the products
// are lines (the A operand, [line][even | odd] in LDS with an odd pitch),
// columns the outputs (the table is the B operand), so that a store covers 16
// consecutive entries of four lines.
template <typename T, typename TI, typename TO, int CT, int NW>
__global__ __launch_bounds__(64 * NW)
__attribute__((amdgpu_waves_per_eu(4))) void k_fd_row(LineArgs a, FDTables<T> t) {
    using M = Mfma<T>;
    using V = typename M::V;
    constexpr int W = 16 * CT;
    constexpr int U = NW == 4 ? 1 : (NW == 8 ? 2 : 3);
    // pairs (k, n-1-k) a thread has in flight: the whole tile to 320 per direction
    constexpr int NG = NW == 4 ? 4 * CT : (NW == 8 ? 10 : 4);
    extern __shared__ unsigned char smem_raw[];
    T* S = reinterpret_cast<T*>(smem_raw);
    const int nt = t.nt, K16 = 16 * nt, P = 2 * K16 + 1, nth = blockDim.x;
    const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lr = lane & 15, lk = lane >> 4;
    const int turn = (wave + (int)blockIdx.x) % nw;
    auto tile_u = [&](int q) { return q == 0 ? wave : q * nw + turn; };
    const Tile w = tile_of(a, xcd_tile(blockIdx.x, a.ntiles));
    const int f = w.f;
    const FieldIO& io = a.io[w.set][f];
    const long long left = (long long)io.dims[1] * io.dims[2] - (long long)w.c * W;
    if (left <= 0) return;
    const int nl = (int)min((long long)W, left);
    const bool fold = !a.inverse, unfold = a.inverse || f == 3;
    const Dir<T> d = dir_of(t, f, 0, a.inverse);
    const int n = d.n, he = d.he, ho = d.ho;
    HalfProduct<T, false, false, CT, NW == 8> hp;
    hp.u = min(wave, nt - 1);
    hp.nt = nt;
    hp.he = he;
    hp.ho = ho;
    hp.lane = lane;
    hp.prime(d.tab);
    {
        // entries k and n-1-k (or he + k) of line l; a thread's (l, k) advance
        // by nth entries of the 16 CT x K16 tile
        const TI* x = reinterpret_cast<const TI*>(io.in) + (long long)w.r * io.sin +
                      (long long)w.c * W * n;
        const int dl = nth / K16, dk = nth - dl * K16;
        int l0 = threadIdx.x / K16, k0 = threadIdx.x - l0 * K16;
#pragma unroll 1
        for (int base = 0; base < W * K16; base += NG * nth) {
            TI v[NG][2];
            int l = l0, k = k0;
            auto next = [&]() {
                l += dl;
                k += dk;
                if (k >= K16) {
                    k -= K16;
                    ++l;
                }
            };
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const uint32_t lo = (uint32_t)sizeof(TI) * l * n;
                const int k2 = fold ? n - 1 - k : he + k;
                const bool in = l < nl;
                v[g][0] = bload(x, in && k < he ? lo + (uint32_t)sizeof(TI) * k : OOB);
                v[g][1] = bload(x, in && k < (fold ? he : ho) ? lo + (uint32_t)sizeof(TI) * k2 : OOB);
                next();
            }
            l = l0;
            k = k0;
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                if (l < W) {
                    TI e = v[g][0], o = v[g][1];
                    if (fold) {
                        o = v[g][0] - v[g][1];
                        e = k < ho ? v[g][0] + v[g][1] : v[g][0];
                    }
                    S[l * P + k] = (T)e;
                    S[l * P + K16 + k] = k < ho ? (T)o : T(0);
                }
                next();
            }
            l0 = l;
            k0 = k;
        }
    }
    __syncthreads();
    TO* y = reinterpret_cast<TO*>(io.out) + (long long)w.r * io.sout +
            (long long)w.c * W * n;
    const bool add = io.add;
#pragma unroll
    for (int q = 0; q < U; ++q) {
        const int u = tile_u(q);
        if (u >= nt) break;
        if (q > 0) {
            hp.u = u;
            hp.prime(d.tab);
        }
        const int m = 16 * u + lr;
        const bool one = m < he, two = m < ho;
        const int m2 = unfold ? n - 1 - m : he + m;
        // line 16 c + kmap(lk, i), from the line of lk = 0
        constexpr int ST = M::kmap(1, 0);
        const uint32_t o0 = (uint32_t)sizeof(TO) * (lk * ST * n + m);
        const uint32_t o1 = (uint32_t)sizeof(TO) * (lk * ST * n + m2);
        auto offset = [&](int c, int i, int h) -> uint32_t {
            if (!(h ? two : one) || 16 * c + M::kmap(lk, i) >= nl) return OOB;
            return h ? o1 : o0;
        };
        auto line0 = [&](int c, int i) { return y + (16 * c + M::kmap(0, i)) * n; };
        V acc[2][CT];
        hp.run(acc, [&](int h, int c, int k, int i) {
            return S[(16 * c + lr) * P + h * K16 + k + M::kmap(lk, i)];
        });
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            TO yv[4][2];
            if (add)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int h = 0; h < 2; ++h) yv[i][h] = bload(line0(c, i), offset(c, i, h));
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const T E = acc[0][c][i], O = acc[1][c][i];
                T z[2] = {E, O};
                if (unfold) {
                    z[0] = two ? E + O : E;
                    z[1] = E - O;
                }
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    TO s = (TO)z[h];
                    if (add) s += yv[i][h];
                    bstore(line0(c, i), offset(c, i, h), s);
                }
            }
        }
    }
}

// Partial sums of y . w for the Krylov dot of launch_P0 where the last launch
// is a direction-1 pass: one per (field, i3-plane) at f nM + k, as the plane
// kernel writes them.  Fixed-order block sums.
struct DotArgs {
    const double* y[3];
    const double* w[3];
    long long stride[3];  // per rhs, of y and w
    long long plane[3];
    int planes[3];
    double* part;
    long long dp_stride;
    int nM;
};
__global__ __launch_bounds__(256) void k_fd_dot_vel(DotArgs a) {
    __shared__ double red[4];
    const int k = blockIdx.x, f = blockIdx.y, r = blockIdx.z;
    if (k >= a.planes[f]) return;
    const long long plane = a.plane[f], ofs = (long long)r * a.stride[f] + k * plane;
    const double* y = a.y[f] + ofs;
    const double* w = a.w[f] + ofs;
    double s = 0.0;
    for (long long i = threadIdx.x; i < plane; i += 256) s += y[i] * w[i];
    s = wg_sum(s, red);
    if (threadIdx.x == 0) a.part[(long long)r * a.dp_stride + f * a.nM + k] = s;
}

// ---- launches -----------------------------------------------------------------------------
int half_tiles(int n) { return ((n + 1) / 2 + 15) / 16; }

// Waves per line / row workgroup: one per tile up to 8, with up to two tiles
// each to 512 per direction, then 16 with up to three; and its columns per tile
// in 16s: two share each fragment load, one gives FD_PLAN_SMALL twice the
// workgroups and the longest directions their LDS.
int line_waves(int n) { return half_tiles(n) <= 4 ? 4 : (half_tiles(n) <= 16 ? 8 : 16); }
int line_ct(int plan, int n) { return plan == FD_PLAN_SMALL || line_waves(n) == 16 ? 1 : 2; }

template <typename T>
size_t line_lds(int n, int ct) {
    const size_t p = 16 * ct + (std::is_same<T, double>::value ? 0 : 4);
    return 2 * 16 * (size_t)half_tiles(n) * p * sizeof(T);
}
template <typename T>
size_t row_lds(int n, int ct) {
    return (size_t)16 * ct * (32 * half_tiles(n) + 1) * sizeof(T);
}
template <typename T>
size_t plane_lds(int n1, int n2) {
    // at least the partial sums of the dot
    return std::max<size_t>((size_t)n2 * plane_pitch<T>(n1) * sizeof(T), 256);
}

template <typename T, typename TI, typename TO, bool SPLIT>
hipError_t launch_plane(hipStream_t st, const PlaneArgs& a, const FDTables<T>& t, int nsets) {
    const int nt = t.nt;
    const dim3 g(t.nM, a.nf, a.nr * nsets), b(nt <= 2 ? 256 * nt : 128 * nt);
    size_t lds = plane_lds<T>(t.nM, t.nM);
    if (t.nN < t.nM) {
        lds = std::max(lds, plane_lds<T>(t.nN, t.nM));
        lds = std::max(lds, plane_lds<T>(t.nM, t.nN));
    }
    if (lds > FD_LDS) return hipErrorInvalidConfiguration;
    switch (nt) {
        case 1: hipLaunchKernelGGL((k_fd_plane<T, TI, TO, SPLIT, 1>), g, b, lds, st, a, t); break;
        case 2: hipLaunchKernelGGL((k_fd_plane<T, TI, TO, SPLIT, 2>), g, b, lds, st, a, t); break;
        case 3: hipLaunchKernelGGL((k_fd_plane<T, TI, TO, SPLIT, 3>), g, b, lds, st, a, t); break;
        case 4: hipLaunchKernelGGL((k_fd_plane<T, TI, TO, SPLIT, 4>), g, b, lds, st, a, t); break;
        default: return hipErrorInvalidConfiguration;
    }
    return hipGetLastError();
}

// LINE: the line kernel (directions 2 and 3), else the row kernel (direction 1).
template <typename T, typename TI, typename TO, bool SPLIT, bool LINE>
hipError_t launch_lines(hipStream_t st, const LineArgs& arg, const FDTables<T>& t, int ct, int nsets) {
    const int nM = t.nM, nt = t.nt;
    const size_t lds = std::max<size_t>(LINE ? line_lds<T>(nM, ct) : row_lds<T>(nM, ct), 256);
    if (lds > FD_LDS || nt > 48) return hipErrorInvalidConfiguration;
    const bool planes = LINE && arg.dir == 1;
    const long long cols = planes ? nM : (long long)nM * nM;
    LineArgs a = arg;
    a.ctiles = (int)((cols + 16 * ct - 1) / (16 * ct));
    a.nbatch = planes ? nM : 1;
    const long long tiles = (long long)a.ctiles * a.nbatch * a.nf * a.nr * nsets;
    if (tiles > INT_MAX) return hipErrorInvalidConfiguration;
    a.ntiles = (int)tiles;
    const dim3 g((unsigned)tiles);
    const dim3 b(64 * std::min(nt, line_waves(nM)));
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, g, b, lds, st, a, t); };
    const int nw = line_waves(nM);
    if constexpr (SPLIT) {  // with the plane kernel only: up to 128 per direction
        if (ct == 2) go(k_fd_line<T, TI, TO, true, 2, 4>);
        else go(k_fd_line<T, TI, TO, true, 1, 4>);
    } else if constexpr (LINE) {
        if (nw == 16) go(k_fd_line<T, TI, TO, false, 1, 16>);
        else if (nw == 8) go(k_fd_line<T, TI, TO, false, 2, 8>);
        else if (ct == 2) go(k_fd_line<T, TI, TO, false, 2, 4>);
        else go(k_fd_line<T, TI, TO, false, 1, 4>);
    } else {
        if (nw == 16) go(k_fd_row<T, TI, TO, 1, 16>);
        else if (nw == 8) go(k_fd_row<T, TI, TO, 2, 8>);
        else go(k_fd_row<T, TI, TO, 2, 4>);
    }
    return hipGetLastError();
}

// P_0^{-1} of the fields [vel ? 0 : 3, pres ? 4 : 3) of one or two sets: modes
// 1 and 2 (one plane launch, or two passes with FD_PLAN_PASSES / LINES), mode
// 3 with the scaling and the inverse mode 3, and the velocity's inverse modes
// 2 and 1.  In FP64 the four fields share the mode-3 launch; otherwise the
// pressure's writes its FP64 output from a launch of its own.  Intermediates
// of precision T ping-pong between the two scratch vectors of each set's
// workspace.
template <typename T, bool SPLIT = false>
hipError_t run_P0(hp_ctx* c, const FDTables<T>& t, const P0Set* sets, int nsets, bool vel,
                  bool pres, int plan, int nrhs, const FdDot* vdot, const FdDot* qdot,
                  const FdComb* comb) {
    const long long N = c->N;
    const int lo = vel ? 0 : 3, hi = pres ? 4 : 3;
    if (lo >= hi) return hipSuccess;
    const bool lines = !SPLIT && fd_plan_lines(plan);
    const int ct = line_ct(plan, c->nM);
    hipStream_t st = c->stream;
    hipError_t e;
    LineArgs la{};
    PlaneArgs pa{};
    T* tmp[2][2];
    for (int i = 0; i < nsets; ++i) {
        tmp[i][0] = reinterpret_cast<T*>(sets[i].ws + ops_ws_stride(c) * (long long)c->opts.max_rhs);
        tmp[i][1] = tmp[i][0] + N * (long long)c->opts.max_rhs;
    }
    la.nr = pa.nr = nrhs;
    la.fields_lo = pa.fields_lo = lo;
    la.nf = pa.nf = hi - lo;
    la.two_nu = 2.0 * c->nu;
    la.omega = c->opts.p0_scale;
    la.pscale = 1.0;
    // the sets' vectors: scratch 0 or 1, or the caller's (-1)
    auto bind = [&](FieldIO (&io)[2][4], int src, int dst) {
        for (int i = 0; i < nsets; ++i)
            for (int f = 0; f < 4; ++f) {
                const Fields &in = sets[i].in, &out = sets[i].out;
                FieldIO& w = io[i][f];
                w.in = src < 0 ? (const void*)in.f[f] : tmp[i][src] + c->off[f];
                w.sin = src < 0 ? in.stride[f] : N;
                w.out = dst < 0 ? (void*)out.f[f] : tmp[i][dst] + c->off[f];
                w.sout = dst < 0 ? out.stride[f] : N;
                w.dw = nullptr;
                for (int d = 0; d < 3; ++d) w.dims[d] = (int)c->dims[f][d];
                w.add = dst < 0 && sets[i].acc_vel;
            }
    };
    int cur = 0;  // the scratch that holds the forward modes 1 and 2
    if (lines) {
        bind(la.io, -1, 0);
        if (comb && pres) {
            // the operator workspace holds n_Q per right-hand side
            const Fields &in = sets[0].in, &cb = comb->b, &cc = comb->c;
            e = vec_axpbypcz(st, c->nQ, nrhs, comb->ca, in.f[3], in.stride[3], comb->cb, cb.f[3],
                             cb.stride[3], comb->cc, cc.f[3], cc.stride[3], sets[0].ws,
                             ops_ws_stride(c));
            if (e != hipSuccess) return e;
            la.io[0][3].in = sets[0].ws;
            la.io[0][3].sin = ops_ws_stride(c);
        }
        if ((e = launch_lines<T, double, T, false, false>(st, la, t, ct, nsets)) != hipSuccess) return e;
        bind(la.io, 0, 1);
        la.dir = 1;
        if ((e = launch_lines<T, T, T, false, true>(st, la, t, ct, nsets)) != hipSuccess) return e;
        cur = 1;
    } else {
        bind(pa.io, -1, 0);
        if (comb) {
            pa.comb = 1;
            pa.inb = comb->b.f[3];
            pa.inc = comb->c.f[3];
            pa.sinb = comb->b.stride[3];
            pa.sinc = comb->c.stride[3];
            pa.ca = comb->ca;
            pa.cb = comb->cb;
            pa.cc = comb->cc;
        }
        if ((e = launch_plane<T, double, T, SPLIT>(st, pa, t, nsets)) != hipSuccess) return e;
    }
    bind(la.io, cur, cur ^ 1);
    la.dir = 2;
    la.fused = 1;
    la.pscale = la.omega * la.two_nu;
    // the pressure's mode-3 step writes the final output; the velocity's
    // feeds the inverse modes 2 and 1
    for (int i = 0; i < nsets; ++i) {
        FieldIO& w = la.io[i][3];
        w.out = sets[i].out.f[3];
        w.sout = sets[i].out.stride[3];
        w.add = sets[i].acc_pres;
    }
    if (qdot) {
        la.io[0][3].dw = qdot->with + c->off[3];
        la.dpart = qdot->part;
        la.dp_stride = fd_dot_count(c, false);
        la.dp_cols = !fd_plan_lines(plan);
    }
    if (vel && pres && std::is_same<T, double>::value) {
        if ((e = launch_lines<T, T, double, SPLIT, true>(st, la, t, ct, nsets)) != hipSuccess) return e;
    } else {
        if (vel) {
            la.fields_lo = 0;
            la.nf = 3;
            if ((e = launch_lines<T, T, T, SPLIT, true>(st, la, t, ct, nsets)) != hipSuccess) return e;
        }
        if (pres) {
            LineArgs lp = la;
            lp.fields_lo = 3;
            lp.nf = 1;
            if ((e = launch_lines<T, T, double, SPLIT, true>(st, lp, t, ct, nsets)) != hipSuccess) return e;
        }
    }
    if (!vel) return hipSuccess;
    const Fields& out = sets[0].out;
    if (lines) {
        la.fields_lo = 0;
        la.nf = 3;
        la.inverse = 1;
        la.fused = 0;
        la.dpart = nullptr;
        bind(la.io, cur ^ 1, cur);
        la.dir = 1;
        if ((e = launch_lines<T, T, T, false, true>(st, la, t, ct, nsets)) != hipSuccess) return e;
        bind(la.io, cur, -1);
        la.dir = 0;
        if ((e = launch_lines<T, T, double, false, false>(st, la, t, ct, nsets)) != hipSuccess) return e;
        if (vdot) {
            DotArgs da{};
            for (int f = 0; f < 3; ++f) {
                da.y[f] = out.f[f];
                da.w[f] = vdot->with + c->off[f];
                da.stride[f] = out.stride[f];
                da.plane[f] = c->dims[f][0] * c->dims[f][1];
                da.planes[f] = (int)c->dims[f][2];
            }
            da.part = vdot->part;
            da.dp_stride = fd_dot_count(c, true);
            da.nM = c->nM;
            hipLaunchKernelGGL(k_fd_dot_vel, dim3(c->nM, 3, nrhs), dim3(256), 0, st, da);
        }
        return hipGetLastError();
    }
    PlaneArgs pi{};
    bind(pi.io, cur ^ 1, -1);
    pi.nr = nrhs;
    pi.nf = 3;
    pi.inverse = 1;
    if (vdot) {
        for (int f = 0; f < 3; ++f) pi.io[0][f].dw = vdot->with + c->off[f];
        pi.dpart = vdot->part;
        pi.dp_stride = fd_dot_count(c, true);
        pi.dp_planes = c->nM;
    }
    return launch_plane<T, T, double, SPLIT>(st, pi, t, nsets);
}

// dynamic LDS up to the CU's 160 KiB for every instantiation
template <size_t N>
hipError_t set_lds(const void* const (&ks)[N]) {
    for (const void* k : ks) {
        const hipError_t e =
            hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)FD_LDS);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
template <typename F>
const void* fptr(F* f) {
    return reinterpret_cast<const void*>(f);
}
template <typename T, typename TI, typename TO, bool SPLIT>
hipError_t set_plane_attrs() {
    return set_lds({fptr(&k_fd_plane<T, TI, TO, SPLIT, 1>), fptr(&k_fd_plane<T, TI, TO, SPLIT, 2>),
                    fptr(&k_fd_plane<T, TI, TO, SPLIT, 3>), fptr(&k_fd_plane<T, TI, TO, SPLIT, 4>)});
}
template <typename T, typename TI, typename TO>
hipError_t set_row_attrs() {
    return set_lds({fptr(&k_fd_row<T, TI, TO, 2, 4>), fptr(&k_fd_row<T, TI, TO, 2, 8>),
                    fptr(&k_fd_row<T, TI, TO, 1, 16>)});
}
template <typename T, typename TO>
hipError_t set_line_attrs() {
    return set_lds({fptr(&k_fd_line<T, T, TO, false, 1, 4>), fptr(&k_fd_line<T, T, TO, false, 2, 4>),
                    fptr(&k_fd_line<T, T, TO, false, 2, 8>), fptr(&k_fd_line<T, T, TO, false, 1, 16>)});
}

}  // namespace

hipError_t fd_init_attributes() {
    const hipError_t es[] = {
        set_plane_attrs<double, double, double, false>(), set_plane_attrs<float, double, float, false>(),
        set_plane_attrs<float, float, double, false>(),   set_plane_attrs<float, double, float, true>(),
        set_plane_attrs<float, float, double, true>(),    set_row_attrs<double, double, double>(),
        set_row_attrs<float, double, float>(),            set_row_attrs<float, float, double>(),
        set_line_attrs<double, double>(),                 set_line_attrs<float, float>(),
        set_line_attrs<float, double>(),
        set_lds({fptr(&k_fd_line<float, float, float, true, 1, 4>),
                 fptr(&k_fd_line<float, float, float, true, 2, 4>),
                 fptr(&k_fd_line<float, float, double, true, 1, 4>),
                 fptr(&k_fd_line<float, float, double, true, 2, 4>)})};
    for (hipError_t e : es)
        if (e != hipSuccess) return e;
    return hipSuccess;
}

int fd_half_tiles(int n) { return half_tiles(n); }

// Fragments of the half-size matrices of one parity: tile (u, t), lane l,
// value i holds A(16u + l%16, 16t + kmap(l/16, i)), zero outside.
template <typename T, typename F>
static void pack_half(std::vector<T>& out, int h, int nt, F A) {
    for (int u = 0; u < nt; ++u)
        for (int t = 0; t < nt; ++t)
            for (int l = 0; l < 64; ++l)
                for (int i = 0; i < 4; ++i) {
                    const int lk = l / 16;
                    const int k = 16 * t + mfma_row<T>(lk, i);
                    const int m = 16 * u + l % 16;
                    out.push_back(m < h && k < h ? (T)A(m, k) : (T)0);
                }
}

template <typename T>
void fd_pack(const std::vector<double>& A, int n, int nt, FdPack kind, std::vector<T>& out) {
    const int he = (n + 1) / 2, ho = n / 2;
    auto at = [&](int i, int j) { return A[(size_t)i * n + j]; };
    for (int par = 0; par < 2; ++par) {
        const int h = par ? ho : he, m0 = par ? he : 0;
        if (kind == FdPack::forward) {          // rows: modes, columns: points
            pack_half(out, h, nt, [&](int m, int k) { return at(k, m0 + m); });
        } else if (kind == FdPack::inverse) {   // rows: points, columns: modes
            pack_half(out, h, nt, [&](int m, int k) { return at(m, m0 + k); });
        } else {
            // symmetric matrix on the folded vectors: the middle column once
            pack_half(out, h, nt, [&](int m, int k) {
                return k >= ho ? at(m, k) : 0.5 * (at(m, k) + (par ? -1.0 : 1.0) * at(m, n - 1 - k));
            });
        }
    }
}
template void fd_pack<double>(const std::vector<double>&, int, int, FdPack, std::vector<double>&);
template void fd_pack<float>(const std::vector<double>&, int, int, FdPack, std::vector<float>&);

// Whether plan `plan` exists for this mesh and precision (see hp_internal.h).
bool fd_plan_valid(const hp_ctx* c, int precision, int plan) {
    const bool planes = c->nM <= FD_PLANE_MAX;
    if (plan == FD_PLAN_LINES) return precision != HP_PREC_BF16X3 || !planes;
    return planes && (plan == FD_PLAN_PASSES || plan == FD_PLAN_PLANE || plan == FD_PLAN_SMALL);
}

int fd_plan_in_use(const hp_ctx* c, int precision) {
    if (c->fd_force >= 0) return c->fd_force;
    // codes 0 and 2 promise FP32 products to split BF16 (1e-7, the plane plans' 1e-5)
    const int want = precision == HP_PREC_BF16X3 && c->opts.fd_plan == 2 ? FD_PLAN_PASSES : c->opts.fd_plan;
    if (want >= 0 && fd_plan_valid(c, precision, want)) return want;
    if (c->nM > FD_PLANE_MAX) return FD_PLAN_LINES;
    return c->fd_tuned[precision] >= 0 ? c->fd_tuned[precision] : FD_PLAN_PLANE;
}

long long fd_dot_count(const hp_ctx* c, bool vel) {
    const long long nM = c->nM;
    if (vel) return 3 * nM;
    // 16 columns each for the plane plans, so that a solve does not depend on
    // which of them the tuner took; otherwise the mode-3 launch's workgroups
    const int plan = fd_plan_in_use(c, HP_PREC_FP64);
    const int ct = fd_plan_lines(plan) ? line_ct(plan, c->nM) : 1;
    return (nM * nM + 16 * ct - 1) / (16 * ct);
}

long long fd_dot_capacity(const hp_ctx* c, bool vel) {
    const long long nM = c->nM;
    return vel ? 3 * nM : (nM * nM + 15) / 16;
}

hipError_t launch_P0_sets(hp_ctx* c, const P0Set* sets, int nsets, bool vel, bool pres,
                          int precision, int nrhs, const FdDot* vdot, const FdDot* qdot,
                          const FdComb* comb) {
    if ((vdot || qdot) && (precision != HP_PREC_FP64 || nsets != 1)) return hipErrorInvalidValue;
    if (nsets < 1 || nsets > 2 || (comb && nsets != 1)) return hipErrorInvalidValue;
    const int plan = fd_plan_in_use(c, precision);
    if (precision == HP_PREC_FP64)
        return run_P0<double>(c, c->fd64, sets, nsets, vel, pres, plan, nrhs, vdot, qdot, comb);
    // split BF16 takes FP32 products in the direction passes
    if (precision == HP_PREC_BF16X3 && !fd_plan_lines(plan))
        return run_P0<float, true>(c, c->fd32, sets, nsets, vel, pres, plan, nrhs, nullptr, nullptr, comb);
    return run_P0<float>(c, c->fd32, sets, nsets, vel, pres, plan, nrhs, nullptr, nullptr, comb);
}

hipError_t launch_P0(hp_ctx* c, const Fields& in, const Fields& out, bool vel, bool pres,
                     bool accumulate, int precision, int nrhs, const FdDot* dot,
                     const FdComb* comb) {
    if (dot && vel && pres) return hipErrorInvalidValue;
    const P0Set set{in, out, c->ws, accumulate, accumulate};
    return launch_P0_sets(c, &set, 1, vel, pres, precision, nrhs, vel ? dot : nullptr,
                          vel ? nullptr : dot, comb);
}

}  // namespace hp

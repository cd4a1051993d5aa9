// Pencil passes with the transform length fixed at compile time.
//
// A length N = A B (A >= B, both at most 18) takes two register DFTs around one
// LDS exchange: the first DFT works on elements as they arrive from memory, the
// second on what the exchange brings, and its results go to memory as they are
// (x forward: once more through LDS, to split the two packed components).  The
// generic passes (rpm_kernels.h) fill LDS, run every stage through it with the
// length as a run-time plan and drain it again: three LDS round trips and five
// barriers per transform instead of one and one, integer divisions per
// butterfly, and 30-80 KB of code per kernel that a small grid waits for
// (13 us per x pass of a 32 x 32 grid).  They serve every other length.
//
// n = j + R2 q, k = k1 + R1 k2:  X[k] = sum_j w_N^(j k1) w_R2^(j k2)
// sum_q w_R1^(q k1) x[j + R2 q].  First butterfly j: radix R1 over q, twiddles
// w_N^(j k1); second butterfly k1: radix R2 over j.
//
// What a pass does not depend on is loaded up front (the stop flag is looked at
// once the data are on their way): a step of a small grid is a chain of such
// kernels, each a few memory latencies long.
//
// The x passes run one block per tile and packed component pair (three pairs):
// three times the blocks and a third of the serial chain of a block that loops
// over the pairs.
#pragma once

#include "rpm_kernels.h"

namespace rpm {

template <int N>
struct Fac;
#define RPM_FAC(N_, A_, B_)                  \
    template <>                              \
    struct Fac<N_> {                         \
        static constexpr int A = A_, B = B_; \
        static_assert(A_ * B_ == N_, "");    \
    };
RPM_FAC(16, 4, 4)
RPM_FAC(18, 6, 3)
RPM_FAC(24, 6, 4)
RPM_FAC(27, 9, 3)
RPM_FAC(32, 8, 4)
RPM_FAC(36, 6, 6)
RPM_FAC(48, 8, 6)
RPM_FAC(54, 9, 6)
RPM_FAC(64, 8, 8)
RPM_FAC(72, 9, 8)
RPM_FAC(81, 9, 9)
RPM_FAC(96, 12, 8)
RPM_FAC(108, 12, 9)
RPM_FAC(128, 16, 8)
RPM_FAC(144, 12, 12)
RPM_FAC(162, 18, 9)
RPM_FAC(192, 16, 12)
RPM_FAC(256, 16, 16)
#undef RPM_FAC
// The lengths that are built: the extents from 16 points on that the benchmark and the
// timed workloads run.  The scheme would reach others, which stay with the run-time
// passes although these are faster there, measured with the same kernels (a map
// application, run-time / fixed): 216^3 FP32 1343 / 787 us, FP64 2761 / 1351; 288x288x64
// 603 / 458; 324x324x64 813 / 563; 12^3 101 / 75; 8^3 90 / 66; each length takes 250 KB of
// library and 5 s of the build.  Out of reach: 2, 3 (one factor) and 243, 384, 432, 486,
// 512 (a factor above 18).
#define RPM_PENCIL_LENGTHS(X) \
    X(16) X(18) X(24) X(27) X(32) X(36) X(48) X(54) X(64) X(72) X(81) X(96) X(108) X(128) X(144) X(162) X(192) X(256)

// cos(m 10 degrees)
__device__ __forceinline__ constexpr double cos10(int m)
{
    m %= 36;
    if (m < 0) m += 36;
    if (m > 18) m = 36 - m;
    const double s = m > 9 ? -1.0 : 1.0;
    if (m > 9) m = 18 - m;
    switch (m) {
        case 0: return s;
        case 1: return s * 0.98480775301220805937;
        case 2: return s * 0.93969262078590838405;
        case 3: return s * 0.86602540378443864676;
        case 4: return s * 0.76604444311897803520;
        case 5: return s * 0.64278760968653932632;
        case 6: return s * 0.5;
        case 7: return s * 0.34202014332566873304;
        case 8: return s * 0.17364817766693034885;
        default: return 0.0;
    }
}

// a exp(D 2 pi i m / R) for constant m, R a divisor of 36
template <typename T, int R, int D>
__device__ __forceinline__ cx<T> mul_root(cx<T> a, int m)
{
    m %= R;
    if (m == 0) return a;
    if (4 * m == R) return cmul_si<T, D>(a);
    if (2 * m == R) return cx<T>{-a.x, -a.y};
    if (4 * m == 3 * R) return cmul_si<T, -D>(a);
    const T c = (T)cos10(m * (36 / R)), s = (T)(D * cos10(m * (36 / R) - 9));
    return cx<T>{a.x * c - a.y * s, a.x * s + a.y * c};
}

// In-register DFT of length R = P Q, n = b + Q a, k = ka + P kb
template <typename T, int P, int Q, int D>
__device__ __forceinline__ void dft_pq(cx<T>* v)
{
    cx<T> y[Q][P];
#pragma unroll
    for (int b = 0; b < Q; ++b) {
#pragma unroll
        for (int a = 0; a < P; ++a) y[b][a] = v[b + Q * a];
        dftR<T, P, D>(y[b]);
#pragma unroll
        for (int k = 0; k < P; ++k) y[b][k] = mul_root<T, P * Q, D>(y[b][k], b * k);
    }
#pragma unroll
    for (int k = 0; k < P; ++k) {
        cx<T> t[Q];
#pragma unroll
        for (int b = 0; b < Q; ++b) t[b] = y[b][k];
        dftR<T, Q, D>(t);
#pragma unroll
        for (int b = 0; b < Q; ++b) v[k + P * b] = t[b];
    }
}

// Length 6 as 2 x 3 without twiddles (the factors are coprime: n = 3 a + 2 b,
// k = 3 ka + 4 kb mod 6).  With a twiddle between them, maps on 24^3 and 36^3 were
// 18 and 13 % further off the exact ones than the run-time-length passes.
template <typename T, int D>
__device__ __forceinline__ void dft6(cx<T>* v)
{
    cx<T> e[3] = {v[0], v[2], v[4]}, o[3] = {v[3], v[5], v[1]};
    dftR<T, 3, D>(e);
    dftR<T, 3, D>(o);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        v[4 * k % 6] = cadd(e[k], o[k]);
        v[(4 * k + 3) % 6] = csub(e[k], o[k]);
    }
}

template <typename T, int R, int D>
__device__ __forceinline__ void dft(cx<T>* v)
{
    if constexpr (R == 6) dft6<T, D>(v);
    else if constexpr (R == 9) dft_pq<T, 3, 3, D>(v);
    else if constexpr (R == 12) dft_pq<T, 4, 3, D>(v);
    else if constexpr (R == 18) {
        // 18 = 9 x 2
        cx<T> e[9], o[9];
#pragma unroll
        for (int a = 0; a < 9; ++a) {
            e[a] = v[2 * a];
            o[a] = v[2 * a + 1];
        }
        dft_pq<T, 3, 3, D>(e);
        dft_pq<T, 3, 3, D>(o);
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            const cx<T> w = mul_root<T, 18, D>(o[k], k);
            v[k] = cadd(e[k], w);
            v[k + 9] = csub(e[k], w);
        }
    } else dftR<T, R, D>(v);
}

// v[k1] *= w_N^(D' j k1) with the forward table tw (conjugate for D > 0)
template <typename T, int R, int D>
__device__ __forceinline__ void twiddle(cx<T>* v, const cx<T>* __restrict__ tw, int j)
{
#pragma unroll
    for (int k = 1; k < R; ++k) {
        cx<T> w = tw[j * k];
        if (D > 0) w.y = -w.y;
        v[k] = cmul(v[k], w);
    }
}
// The same with the table entries loaded ahead, beside the data they belong to
// (a kernel's first access to the table misses the caches).
template <typename T, int R>
__device__ __forceinline__ void load_twiddles(cx<T> (&w)[R], const cx<T>* __restrict__ tw, int j)
{
#pragma unroll
    for (int k = 1; k < R; ++k) w[k] = tw[j * k];
}
template <typename T, int R, int D>
__device__ __forceinline__ void apply_twiddles(cx<T>* v, const cx<T> (&w)[R])
{
#pragma unroll
    for (int k = 1; k < R; ++k) v[k] = cmul(v[k], D > 0 ? cconj(w[k]) : w[k]);
}

// The grid as these passes take it (Geo is more than their arguments have room for).
struct PGeo {
    int ny, nz, nh;
    long long N, nspec;
    __device__ __forceinline__ PGeo(int nx, int ny_, int nz_, int nh_)
        : ny(ny_), nz(nz_), nh(nh_), N((long long)nx * ny_ * nz_), nspec((long long)nh_ * ny_ * nz_)
    {
    }
};

// Rows per x- or y-pass tile: the transposed side moves in segments of this
// many complex numbers (128 bytes; FP64 lengths whose smaller factor would leave
// half a wave idle take 16 rows).
template <typename T, int N>
constexpr int tile_rows() { return sizeof(T) == 8 && Fac<N>::B >= 8 ? 8 : 16; }
// One first-stage butterfly of radix A per thread, in whole waves.
template <typename T, int N>
constexpr int tile_threads() { return (tile_rows<T, N>() * Fac<N>::B + 63) / 64 * 64; }

// ---------------------------------------------------------------------------
// y passes: S1[c][kx][z][y] -> S2[c][ky][kx][z] (D = -1) and back (D = +1).  A
// block transforms one tile of rows (z) of one (c, kx).  Lanes run along the
// contiguous side of each access: forward the first butterflies along y (radix
// B, A of them side by side) and the second along z, inverse the other way.
// ---------------------------------------------------------------------------
template <typename T, int N, int D>
__device__ __forceinline__ void py_body(const cx<T>* __restrict__ Sin, cx<T>* __restrict__ Sout, const PGeo& g,
                                        int nzt, const cx<T>* __restrict__ tw, const int* __restrict__ done)
{
    const int stop = done ? *done : 0;
    constexpr int TZ = tile_rows<T, N>(), NT = tile_threads<T, N>(), LS = TZ + 1;
    constexpr int R1 = D < 0 ? Fac<N>::B : Fac<N>::A, R2 = N / R1;
    constexpr int I1 = (R2 * TZ + NT - 1) / NT, I2 = (R1 * TZ + NT - 1) / NT;
    __shared__ cx<T> X[N * LS];
    int b = blockIdx.x;
    const int zt = b % nzt;
    b /= nzt;
    const int kx = b % g.nh, c = b / g.nh;
    const int z0 = zt * TZ;
    const cx<T>* src = Sin + (long long)c * g.nspec;
    cx<T>* dst = Sout + (long long)c * g.nspec;
    const long long row = ((long long)kx * g.nz + z0) * N;               // first row of the tile in S1
    const long long seg = (long long)kx * g.nz + z0, ks = (long long)g.nh * g.nz;  // its segment of a ky plane in S2
    cx<T> v[I1][R1], w[I1][R1];
#pragma unroll
    for (int i = 0; i < I1; ++i) {
        const int e = threadIdx.x + i * NT;
        const int j = D < 0 ? e % R2 : e / TZ, r = D < 0 ? e / R2 : e % TZ;
        const bool in = e < R2 * TZ && z0 + r < g.nz;
#pragma unroll
        for (int q = 0; q < R1; ++q) {
            const long long o = D < 0 ? row + r * N + j + R2 * q : (j + R2 * q) * ks + seg + r;
            v[i][q] = in ? src[o] : cx<T>{T(0), T(0)};
        }
        load_twiddles<T, R1>(w[i], tw, e < R2 * TZ ? j : 0);
    }
    if (stop) return;
    // element (j, k1) of row r: neighbouring lanes of both sides on different banks
    auto at = [](int j, int k1, int r) { return (D < 0 ? k1 * R2 + j : j * R1 + k1) * LS + r; };
#pragma unroll
    for (int i = 0; i < I1; ++i) {
        const int e = threadIdx.x + i * NT;
        const int j = D < 0 ? e % R2 : e / TZ, r = D < 0 ? e / R2 : e % TZ;
        if (R2 * TZ % NT == 0 || e < R2 * TZ) {
            dft<T, R1, D>(v[i]);
            apply_twiddles<T, R1, D>(v[i], w[i]);
#pragma unroll
            for (int k1 = 0; k1 < R1; ++k1) X[at(j, k1, r)] = v[i][k1];
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < I2; ++i) {
        const int e = threadIdx.x + i * NT;
        const int k1 = D < 0 ? e / TZ : e % R1, r = D < 0 ? e % TZ : e / R1;
        if (e < R1 * TZ && z0 + r < g.nz) {
            cx<T> u[R2];
#pragma unroll
            for (int j = 0; j < R2; ++j) u[j] = X[at(j, k1, r)];
            dft<T, R2, D>(u);
#pragma unroll
            for (int k2 = 0; k2 < R2; ++k2) {
                const int k = k1 + R1 * k2;
                dst[D < 0 ? k * ks + seg + r : row + r * N + k] = u[k2];
            }
        }
    }
}

template <typename T>
struct PyArgs {
    const cx<T>* Sin;
    cx<T>* Sout;
    const cx<T>* tw;
    const int* done;
    int nh, nz, nzt;
};
static_assert(sizeof(PyArgs<double>) <= 112, "one cheap launch");

template <typename T, int N, int D>
__global__ __launch_bounds__((tile_threads<T, N>())) void k_py(PyArgs<T> a)
{
    const PGeo g(0, N, a.nz, a.nh);
    py_body<T, N, D>(a.Sin, a.Sout, g, a.nzt, a.tw, a.done);
}

// Blocks of the x passes: tile and component pair of block id b.  The pairs of a
// tile go to the same XCD (blocks are dealt to the eight in turn), whose L2 then
// serves the strains they share.  Returns false past the last tile.
__device__ __forceinline__ bool x_block(int b, int ntiles, int np, int& tile, int& pair)
{
    const int x = b & 7, i = b >> 3;
    tile = (i / np) * 8 + x;
    pair = i % np;
    return tile < ntiles;
}
inline int x_grid(int ntiles, int np) { return (ntiles + 7) / 8 * 8 * np; }

// Sums of M values over a block of NT threads, thread 0 writes dst[m].
template <int M, int NT>
__device__ __forceinline__ void block_sum(double (&v)[M], double* __restrict__ dst)
{
    __shared__ double red[NT / 64][M];
#pragma unroll
    for (int m = 0; m < M; ++m) v[m] = wave_sum(v[m]);
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int m = 0; m < M; ++m) red[threadIdx.x >> 6][m] = v[m];
    __syncthreads();
    if (threadIdx.x < M) {
        double s = red[0][threadIdx.x];
#pragma unroll
        for (int w = 1; w < NT / 64; ++w) s += red[w][threadIdx.x];
        dst[threadIdx.x] = s;
    }
}

// ---------------------------------------------------------------------------
// x-forward: constitutive law + transform along x of one packed pair of
// components (pairs 0..2 of sigma; 3..5 of eps for the polarization map), half
// spectrum to S1[c][kx][z][y], <eps> partial sums of the pair's components.
// ---------------------------------------------------------------------------
template <typename T, int N, int NP>
__device__ __forceinline__ void pxf_body(const T* __restrict__ xin, const uint8_t* __restrict__ phase,
                                         const double* __restrict__ lame, int nph, int use_ref, double lam0, double mu0,
                                         cx<T>* __restrict__ S1, double* __restrict__ part_mean, const PGeo& g,
                                         int ntiles, int nyt, const cx<T>* __restrict__ tw,
                                         const int* __restrict__ done)
{
    const int stop = done ? *done : 0;
    constexpr int TY = tile_rows<T, N>(), NT = tile_threads<T, N>(), LS = TY + 1;
    constexpr int R1 = Fac<N>::B, R2 = Fac<N>::A, NH = N / 2 + 1;
    constexpr int I1 = (R2 * TY + NT - 1) / NT, I2 = (R1 * TY + NT - 1) / NT;
    __shared__ cx<T> X[N * LS];
    __shared__ T lt[2 * 256];  // phase table
    int tile, pair;
    if (!x_block(blockIdx.x, ntiles, NP, tile, pair)) return;
    const int z = tile / nyt, y0 = (tile - z * nyt) * TY;
    const T* src = xin + ((long long)z * g.ny + y0) * N;
    const uint8_t* ph = phase + ((long long)z * g.ny + y0) * N;
    double ms[2] = {0.0, 0.0};
    cx<T> v[I1][R1];
    auto each = [&](auto f) {
#pragma unroll
        for (int i = 0; i < I1; ++i) {
            const int e = threadIdx.x + i * NT;
            const int j = e % R2, r = e / R2;
            const bool in = e < R2 * TY && y0 + r < g.ny;
#pragma unroll
            for (int q = 0; q < R1; ++q) f(i, q, in ? r * N + j + R2 * q : 0, in);
        }
    };
    // phase labels; the table comes from LDS once both have arrived.  Labels past the
    // table are voids, as in the passes that read it in memory, where zeros follow it: a
    // wave that meets one writes those zeros here.  (In every block the zeros took 0.17 us
    // of 5.1 on 32^2 grids; a bound on each label, 115 us instead of 107 at 192^3.)
    const bool tab = pair < 3 && !use_ref;
    int lab[I1][R1];
    auto table_ready = [&]() {
        if (!tab) return;
        int top = 0;
        each([&](int i, int q, int, bool) { top = max(top, lab[i][q]); });
        if (__any(top >= nph))
            for (int i = 2 * nph + (threadIdx.x & 63); i < 512; i += 64) lt[i] = T(0);
        __syncthreads();
    };
    if (tab) {
        for (int i = threadIdx.x; i < 2 * nph; i += NT) lt[i] = (T)lame[i];
        each([&](int i, int q, int o, bool) { lab[i][q] = (int)ph[o]; });
    }
    cx<T> w[I1][R1];
#pragma unroll
    for (int i = 0; i < I1; ++i) load_twiddles<T, R1>(w[i], tw, (threadIdx.x + i * NT) % R2);
    auto lam_mu = [&](int i, int q, T& l, T& m) {
        l = use_ref ? (T)lam0 : lt[2 * lab[i][q]];
        m = use_ref ? (T)mu0 : lt[2 * lab[i][q] + 1];
    };
    const long long M = g.N;
    if (pair == 0 || pair == 1) {
        T e0[I1][R1], e1[I1][R1], e2[I1][R1], e3[I1][R1];
        each([&](int i, int q, int o, bool) {
            e0[i][q] = src[o];
            e1[i][q] = src[M + o];
            e2[i][q] = src[2 * M + o];
            if (pair == 1) e3[i][q] = src[3 * M + o];
        });
        if (stop) return;
        table_ready();
        each([&](int i, int q, int, bool in) {
            T lam, mu;
            lam_mu(i, q, lam, mu);
            const T l = lam * (e0[i][q] + e1[i][q] + e2[i][q]), m2 = mu + mu;
            const T a = pair == 0 ? e0[i][q] : e2[i][q], b = pair == 0 ? e1[i][q] : e3[i][q];
            v[i][q] = in ? cx<T>{m2 * a + l, pair == 0 ? m2 * b + l : m2 * b} : cx<T>{T(0), T(0)};
            ms[0] += in ? (double)a : 0.0;
            ms[1] += in ? (double)b : 0.0;
        });
    } else {
        const int c = pair == 2 ? 4 : 2 * (pair - 3);
        T a[I1][R1], b[I1][R1];
        each([&](int i, int q, int o, bool) {
            a[i][q] = src[c * M + o];
            b[i][q] = src[(c + 1) * M + o];
        });
        if (stop) return;
        table_ready();
        each([&](int i, int q, int, bool in) {
            T lam = T(0), mu = T(0.5);
            if (pair == 2) lam_mu(i, q, lam, mu);
            const T m2 = mu + mu;
            v[i][q] = in ? cx<T>{m2 * a[i][q], m2 * b[i][q]} : cx<T>{T(0), T(0)};
            ms[0] += in ? (double)a[i][q] : 0.0;
            ms[1] += in ? (double)b[i][q] : 0.0;
        });
    }
#pragma unroll
    for (int i = 0; i < I1; ++i) {
        const int e = threadIdx.x + i * NT;
        const int j = e % R2, r = e / R2;
        if (R2 * TY % NT == 0 || e < R2 * TY) {
            dft<T, R1, -1>(v[i]);
            apply_twiddles<T, R1, -1>(v[i], w[i]);
#pragma unroll
            for (int k1 = 0; k1 < R1; ++k1) X[(k1 * R2 + j) * LS + r] = v[i][k1];
        }
    }
    __syncthreads();
    cx<T> u[I2][R2];
#pragma unroll
    for (int i = 0; i < I2; ++i) {
        const int e = threadIdx.x + i * NT;
        if (R1 * TY % NT == 0 || e < R1 * TY) {
            const int k1 = e / TY, r = e % TY;
#pragma unroll
            for (int j = 0; j < R2; ++j) u[i][j] = X[(k1 * R2 + j) * LS + r];
            dft<T, R2, -1>(u[i]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < I2; ++i) {
        const int e = threadIdx.x + i * NT;
        if (R1 * TY % NT == 0 || e < R1 * TY) {
            const int k1 = e / TY, r = e % TY;
#pragma unroll
            for (int k2 = 0; k2 < R2; ++k2) X[(k1 + R1 * k2) * LS + r] = u[i][k2];
        }
    }
    __syncthreads();
    // split the packed transform into the two real-input spectra
    cx<T>* outa = S1 + (long long)(2 * pair) * g.nspec;
    cx<T>* outb = outa + g.nspec;
#pragma unroll 4
    for (int t = threadIdx.x; t < NH * TY; t += NT) {
        const int k = t / TY, r = t % TY;
        if (y0 + r < g.ny) {
            const cx<T> p = X[k * LS + r], n = cconj(X[(k == 0 ? 0 : N - k) * LS + r]);
            const cx<T> s = cadd(p, n), d = csub(p, n);
            const long long o = ((long long)k * g.nz + z) * g.ny + y0 + r;
            outa[o] = cx<T>{T(0.5) * s.x, T(0.5) * s.y};
            outb[o] = cx<T>{T(0.5) * d.y, T(-0.5) * d.x};
        }
    }
    if (part_mean && pair < 3) block_sum<2, NT>(ms, part_mean + (long long)tile * 6 + 2 * pair);
}

template <typename T>
struct PxfArgs {
    const T* xin;
    const uint8_t* phase;
    const double* lame;
    cx<T>* S1;
    double* part_mean;
    const cx<T>* tw;
    const int* done;
    double lam0, mu0;
    int use_ref, nph, ny, nz, ntiles, nyt;
};
static_assert(sizeof(PxfArgs<double>) <= 112, "one cheap launch");

template <typename T, int N, int NP>
__global__ __launch_bounds__((tile_threads<T, N>())) void k_pxf(PxfArgs<T> a)
{
    const PGeo g(N, a.ny, a.nz, N / 2 + 1);
    pxf_body<T, N, NP>(a.xin, a.phase, a.lame, a.nph, a.use_ref, a.lam0, a.mu0, a.S1, a.part_mean, g, a.ntiles, a.nyt,
                       a.tw, a.done);
}

// ---------------------------------------------------------------------------
// x-inverse: S1 -> complex-to-real transform along x, out = eps - t (OUT_XI) or
// t (OUT_T), for one packed pair.  Entries k > N/2 of the packed pair are
// conjugates of loaded ones (read twice, the second time from cache).
// ---------------------------------------------------------------------------
// First butterflies of component pair q of a tile into the exchange X (threads
// t of tile_threads).
template <typename T, int N>
__device__ __forceinline__ void xinv_first(const cx<T>* __restrict__ S1, cx<T>* X, int q_, int t, int z, int y0,
                                           const PGeo& g, const cx<T>* __restrict__ tw, int stop)
{
    constexpr int TY = tile_rows<T, N>(), NT = tile_threads<T, N>(), LS = TY + 1;
    constexpr int R1 = Fac<N>::A, R2 = Fac<N>::B, I1 = (R2 * TY + NT - 1) / NT;
    const cx<T>* ina = S1 + (long long)(2 * q_) * g.nspec + (long long)z * g.ny + y0;
    const long long ks = (long long)g.nz * g.ny;
    cx<T> v[I1][R1], w[I1][R1], f[I1][R1];
#pragma unroll
    for (int i = 0; i < I1; ++i) {
        const int e = t + i * NT;
        const int j = e / TY, r = e % TY;
        const bool in = e < R2 * TY && y0 + r < g.ny;
#pragma unroll
        for (int q = 0; q < R1; ++q) {
            const int k = j + R2 * q, h = 2 * k <= N ? k : N - k;
            const long long o = in ? h * ks + r : 0;
            v[i][q] = ina[o];
            w[i][q] = ina[g.nspec + o];
        }
        load_twiddles<T, R1>(f[i], tw, e < R2 * TY ? j : 0);
    }
    if (stop) return;
#pragma unroll
    for (int i = 0; i < I1; ++i) {
        const int e = t + i * NT;
        const int j = e / TY, r = e % TY;
        if (R2 * TY % NT == 0 || e < R2 * TY) {
#pragma unroll
            for (int q = 0; q < R1; ++q) {
                const int k = j + R2 * q;
                cx<T> a = v[i][q], b = w[i][q];
                if (k == 0 || 2 * k == N) a.y = b.y = T(0);
                v[i][q] = 2 * k <= N ? cx<T>{a.x - b.y, a.y + b.x} : cx<T>{a.x + b.y, b.x - a.y};
            }
            dft<T, R1, +1>(v[i]);
            apply_twiddles<T, R1, +1>(v[i], f[i]);
#pragma unroll
            for (int k1 = 0; k1 < R1; ++k1) X[(j * R1 + k1) * LS + r] = v[i][k1];
        }
    }
}

template <typename T, int N>
__device__ __forceinline__ void pxi_body(const cx<T>* __restrict__ S1, const T* __restrict__ eps,
                                         T* __restrict__ out, int out_mode, const T* __restrict__ shift,
                                         double* __restrict__ part_inc, const PGeo& g, int ntiles, int nyt,
                                         const cx<T>* __restrict__ tw, const int* __restrict__ done)
{
    const int stop = done ? *done : 0;
    constexpr int TY = tile_rows<T, N>(), NT = tile_threads<T, N>(), LS = TY + 1;
    constexpr int R1 = Fac<N>::A, R2 = Fac<N>::B, I2 = (R1 * TY + NT - 1) / NT;
    __shared__ cx<T> X[N * LS];
    int tile, pair;
    if (!x_block(blockIdx.x, ntiles, 3, tile, pair)) return;
    const int z = tile / nyt, y0 = (tile - z * nyt) * TY;
    const long long base = ((long long)z * g.ny + y0) * N, M = g.N;
    const T invN = T(1.0 / (double)M);
    const int ca = 2 * pair, cb = ca + 1;
    double inc[1] = {0.0};
    xinv_first<T, N>(S1, X, pair, threadIdx.x, z, y0, g, tw, stop);
    if (stop) return;
    T ea[I2][R2], eb[I2][R2];
    if (out_mode == OUT_XI)
#pragma unroll
        for (int i = 0; i < I2; ++i) {
            const int e = threadIdx.x + i * NT;
            const int k1 = e % R1, r = e / R1;
            const bool in = e < R1 * TY && y0 + r < g.ny;
#pragma unroll
            for (int k2 = 0; k2 < R2; ++k2) {
                const long long o = base + (in ? r * N + k1 + R1 * k2 : 0);
                ea[i][k2] = eps[ca * M + o];
                eb[i][k2] = eps[cb * M + o];
            }
        }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < I2; ++i) {
        const int e = threadIdx.x + i * NT;
        const int k1 = e % R1, r = e / R1;
        if (e < R1 * TY && y0 + r < g.ny) {
            cx<T> u[R2];
#pragma unroll
            for (int j = 0; j < R2; ++j) u[j] = X[(j * R1 + k1) * LS + r];
            dft<T, R2, +1>(u);
#pragma unroll
            for (int k2 = 0; k2 < R2; ++k2) {
                const long long o = base + r * N + k1 + R1 * k2;
                const T ta = u[k2].x * invN, tb = u[k2].y * invN;
                if (out_mode == OUT_XI) {
                    T oa = ea[i][k2] - ta, ob = eb[i][k2] - tb;
                    if (shift) {
                        oa += shift[ca * M + o];
                        ob += shift[cb * M + o];
                    }
                    out[ca * M + o] = oa;
                    out[cb * M + o] = ob;
                    if (part_inc) {
                        const double da = (double)oa - (double)ea[i][k2], db = (double)ob - (double)eb[i][k2];
                        inc[0] += frob_w(ca) * da * da + frob_w(cb) * db * db;
                    }
                } else {
                    out[ca * M + o] = ta;
                    out[cb * M + o] = tb;
                }
            }
        }
    }
    if (part_inc) block_sum<1, NT>(inc, part_inc + (tile * 3 + pair));
}

template <typename T>
struct PxiArgs {
    const cx<T>* S1;
    const T* eps;
    T* out;
    const T* shift;
    double* part_inc;
    const cx<T>* tw;
    const int* done;
    int out_mode, ny, nz, ntiles, nyt;
};
static_assert(sizeof(PxiArgs<double>) <= 112, "one cheap launch");

template <typename T, int N>
__global__ __launch_bounds__((tile_threads<T, N>())) void k_pxi(PxiArgs<T> a)
{
    const PGeo g(N, a.ny, a.nz, N / 2 + 1);
    pxi_body<T, N>(a.S1, a.eps, a.out, a.out_mode, a.shift, a.part_inc, g, a.ntiles, a.nyt, a.tw, a.done);
}

// The polarization map's x-inverse (OUT_XI): t is Gamma0 s_b - beta E, and out =
// (C + C0)^-1 (sigma + (1 - beta) C0 eps - C0 t) voxel by voxel, so a block takes
// all three pairs of its tile: side by side in three groups of waves where the
// exchanges fit LDS (a 128 x 128 plane: 15.6 us in turn), else in turn.
template <typename T, int N>
constexpr int pol_groups()
{
    return (size_t)3 * N * (tile_rows<T, N>() + 1) * 2 * sizeof(T) <= 60 * 1024 ? 3 : 1;
}

template <typename T>
__device__ __forceinline__ double pol_voxel(const T* __restrict__ eps, T* __restrict__ out, long long M, long long o,
                                            const T (&t)[6], const uint8_t* __restrict__ phase,
                                            const double* __restrict__ lame, double lam0, double mu0, double beta,
                                            const T* __restrict__ shift)
{
    const T l0 = (T)lam0, m0 = (T)mu0, omb = (T)(1.0 - beta);
    T e[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) e[c] = eps[c * M + o];
    const int ph = phase[o];
    const T lam = (T)lame[2 * ph], mu = (T)lame[2 * ph + 1];
    const T tre = e[0] + e[1] + e[2], tru = t[0] + t[1] + t[2];
    // X = sigma + (1 - beta) C0 eps - C0 t
    T x[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) {
        x[c] = T(2) * (mu + omb * m0) * e[c] - T(2) * m0 * t[c];
        if (c < 3) x[c] += (lam + omb * l0) * tre - l0 * tru;
    }
    // (C + C0)^-1 X for the isotropic sum (lam + lam0, mu + mu0)
    const T lp = lam + l0, mp = mu + m0;
    const T kap = lp / (T(3) * lp + T(2) * mp), trx = x[0] + x[1] + x[2];
    const T inv2m = T(1) / (T(2) * mp);
    double inc = 0.0;
#pragma unroll
    for (int c = 0; c < 6; ++c) {
        T f = (c < 3 ? x[c] - kap * trx : x[c]) * inv2m;
        if (shift) f += shift[c * M + o];
        out[c * M + o] = f;
        const double dd = (double)f - (double)e[c];
        inc += frob_w(c) * dd * dd;
    }
    return inc;
}

template <typename T, int N>
__device__ __forceinline__ void pxi_pol_body(const cx<T>* __restrict__ S1, const T* __restrict__ eps,
                                             T* __restrict__ out, const T* __restrict__ shift,
                                             double* __restrict__ part_inc, const PGeo& g, int nyt,
                                             const cx<T>* __restrict__ tw, const uint8_t* __restrict__ phase,
                                             const double* __restrict__ lame, double lam0, double mu0,
                                             double beta, const int* __restrict__ done)
{
    const int stop = done ? *done : 0;
    constexpr int TY = tile_rows<T, N>(), NT = tile_threads<T, N>(), LS = TY + 1, NG = pol_groups<T, N>();
    constexpr int R1 = Fac<N>::A, R2 = Fac<N>::B, I2 = (R1 * TY + NT - 1) / NT;
    __shared__ cx<T> X_[NG * N * LS];
    const int tile = blockIdx.x, t = threadIdx.x % NT, grp = threadIdx.x / NT;
    const int z = tile / nyt, y0 = (tile - z * nyt) * TY;
    const long long base = ((long long)z * g.ny + y0) * N, M = g.N;
    const T invN = T(1.0 / (double)M);
    cx<T>* X = X_ + grp * N * LS;
    double inc[1] = {0.0};
    cx<T> u[NG == 1 ? 3 : 1][I2][R2];
#pragma unroll
    for (int pp = 0; pp < (NG == 1 ? 3 : 1); ++pp) {
        if (pp > 0) __syncthreads();  // the previous pair's exchange has been read
        xinv_first<T, N>(S1, X, NG == 1 ? pp : grp, t, z, y0, g, tw, stop);
        if (stop) return;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < I2; ++i) {
            const int e = t + i * NT;
            if (R1 * TY % NT == 0 || e < R1 * TY) {
                const int k1 = e % R1, r = e / R1;
#pragma unroll
                for (int j = 0; j < R2; ++j) u[pp][i][j] = X[(j * R1 + k1) * LS + r];
                dft<T, R2, +1>(u[pp][i]);
            }
        }
    }
    if constexpr (NG == 3) {
        // t of all components to LDS, [component][voxel of the tile]
        T* tl = reinterpret_cast<T*>(X_);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < I2; ++i) {
            const int e = t + i * NT;
            if (R1 * TY % NT == 0 || e < R1 * TY) {
                const int k1 = e % R1, r = e / R1;
#pragma unroll
                for (int k2 = 0; k2 < R2; ++k2) {
                    const int v = r * N + k1 + R1 * k2;
                    tl[(2 * grp) * N * TY + v] = u[0][i][k2].x * invN;
                    tl[(2 * grp + 1) * N * TY + v] = u[0][i][k2].y * invN;
                }
            }
        }
        __syncthreads();
        const int nv = min(TY, g.ny - y0) * N;
        for (int v = threadIdx.x; v < nv; v += NG * NT) {
            T tv[6];
#pragma unroll
            for (int c = 0; c < 6; ++c) tv[c] = tl[c * N * TY + v];
            inc[0] += pol_voxel<T>(eps, out, M, base + v, tv, phase, lame, lam0, mu0, beta, shift);
        }
    } else {
#pragma unroll
        for (int i = 0; i < I2; ++i) {
            const int e = t + i * NT;
            const int k1 = e % R1, r = e / R1;
            if (e < R1 * TY && y0 + r < g.ny) {
#pragma unroll
                for (int k2 = 0; k2 < R2; ++k2) {
                    T tv[6];
#pragma unroll
                    for (int c = 0; c < 6; ++c)
                        tv[c] = (c & 1 ? u[NG == 1 ? c / 2 : 0][i][k2].y : u[NG == 1 ? c / 2 : 0][i][k2].x) * invN;
                    inc[0] += pol_voxel<T>(eps, out, M, base + r * N + k1 + R1 * k2, tv, phase, lame, lam0, mu0,
                                           beta, shift);
                }
            }
        }
    }
    if (part_inc) block_sum<1, NG * NT>(inc, part_inc + tile);
}

template <typename T>
struct PxpArgs {
    const cx<T>* S1;
    const T* eps;
    T* out;
    const T* shift;
    double* part_inc;
    const cx<T>* tw;
    const uint8_t* phase;
    const double* lame;
    const int* done;
    double lam0, mu0, beta;
    int ny, nz, nyt;
};
static_assert(sizeof(PxpArgs<double>) <= 112, "one cheap launch");

template <typename T, int N>
__global__ __launch_bounds__((pol_groups<T, N>() * tile_threads<T, N>())) void k_pxi_pol(PxpArgs<T> a)
{
    const PGeo g(N, a.ny, a.nz, N / 2 + 1);
    pxi_pol_body<T, N>(a.S1, a.eps, a.out, a.shift, a.part_inc, g, a.nyt, a.tw, a.phase, a.lame, a.lam0, a.mu0, a.beta,
                       a.done);
}

// ---------------------------------------------------------------------------
// gamma: transform along the last axis, Green operator, inverse transform, in
// place (see k_gamma for the operator and the k = 0 term).  A block owns P
// pencils with all their components: first butterflies from memory, second ones
// in place in LDS, the filter frequency by frequency, and back.
// Wide blocks: one pencil and a thread for every butterfly and frequency of it, so
// that no stage is a loop and the filter's direction (a square root and three
// divisions) is computed while the data are on their way.  Narrow blocks: P pencils
// that fill the waves with radix-A butterflies of the six components (6 B P of
// them), the other stages looping.  Small grids are bound by the chain of stages,
// large ones by memory if enough blocks are in flight.  Narrow / wide, us:
//   FP64 32^2 6.8 / 5.3, 128^2 9.5 / 6.6, 32^3 7.1 / 5.7, 64^3 13.3 / 11.7, 128^3 54
//   / 44.8, 96x96x256 61 / 53; FP32 48^3 7.7 / 6.4, 64^3 8.3 / 7.5, 128^3 29.4 / 29.8
//   polarization: FP64 128^2 10.8 / 6.9, 64^3 17.9 / 14.0, 128^3 100 / 67
// Narrow ones are better where a pencil leaves many of a wide block's lanes idle and
// there are pencils enough to hide the stages: FP32 192x192x96 40.2 / 44.8, 192^3 77 /
// 97; FP64 192x192x32 25.7 / 29.0, 256x256x48 62 / 68, 144^3 63 / 73; at 144, 544
// pencils take 11.5 / 10.3, 2112 take 18.8 / 20.6.
// ---------------------------------------------------------------------------
template <typename T, int N>
__host__ __device__ constexpr bool always_wide(bool pol)
{
    return pol || (sizeof(T) == 8 && ((N >= 64 && N <= 128) || N == 256));
}
// The polarization map's FP64 grids end at 128 points along the last axis (the run-time
// pass's LDS, which decides what a call takes), so its pass is not there beyond.
template <typename T, int N>
constexpr bool pol_gamma() { return sizeof(T) == 4 || N <= 128; }
template <typename T, int N>
constexpr bool gamma_wide(bool pol, int npen)
{
    return always_wide<T, N>(pol) || npen <= (N > 128 && N < 256 ? 1024 : 4096);
}
template <typename T, int N, bool POL, bool WIDE>
struct GCfg {
    static constexpr int A = Fac<N>::A, B = Fac<N>::B;
    static constexpr int NC = POL ? 12 : 6;
    static constexpr int LS = A + 1;                               // LDS row (j, k2): A elements
    static constexpr size_t pencil = (size_t)NC * B * LS * 2 * sizeof(T);
    static constexpr size_t cap = 56 * 1024;
    // pencils whose butterflies fill whole waves best, for B of 3, 4, 6, 8, 9, 12, 16
    static constexpr int want = B == 3 ? 7 : B == 4 ? 8 : B == 6 ? 7 : B == 8 ? 4 : B == 9 ? 4 : B == 12 ? 3 : 2;
    static constexpr int fit = (int)((cap - N * 2 * sizeof(T)) / pencil);
    static constexpr int P = WIDE ? 1 : fit < 1 ? 1 : fit < want ? fit : want;
    static constexpr int NT = ((WIDE ? (NC * A > N ? NC * A : N) : 6 * B * P) + 63) / 64 * 64;
    static constexpr int SLOTS = NC * P * B * LS;
};

template <typename T, int N, bool POL, bool WIDE>
__device__ __forceinline__ void pg_body(cx<T>* __restrict__ S, const Geo& g, const cx<T>* __restrict__ tw,
                                        double lam0, double mu0, double alpha, double beta, int dc_mode,
                                        const double* __restrict__ E, const double* __restrict__ part_mean,
                                        int n_mean, double* __restrict__ part_err, DevState* __restrict__ st,
                                        const int* __restrict__ done)
{
    const int stop = done ? *done : 0;
    using G = GCfg<T, N, POL, WIDE>;
    constexpr int A = G::A, B = G::B, P = G::P, NT = G::NT, LS = G::LS, NC = G::NC;
    __shared__ cx<T> X[G::SLOTS];
    __shared__ cx<T> W[N];
    __shared__ double dcm[6], Es[6];
    const int t = threadIdx.x;
    const int npen = g.two_d ? g.nh : g.ny * g.nh;
    const int p0 = blockIdx.x * P;
    // (component, pencil, j or k2, k1)
    auto slot = [](int c, int p, int j, int k) { return ((c * P + p) * B + j) * LS + k; };
    auto freq = [&](int pen, int i, int& kx, int& ky, int& kz) {
        const int q = g.two_d ? 0 : (int)((unsigned)pen / (unsigned)g.nh);
        kx = pen - q * g.nh;
        ky = g.two_d ? i : q;
        kz = g.two_d ? 0 : i;
    };
    // <eps> from the x-pass partial sums (block 0 holds k = 0)
    double acc[6] = {0, 0, 0, 0, 0, 0};
    if (blockIdx.x == 0 && dc_mode == DC_MEAN) {
        if (t < 6) Es[t] = E[t];
#pragma unroll 4
        for (int b = t; b < n_mean; b += NT)
#pragma unroll
            for (int c = 0; c < 6; ++c) acc[c] += part_mean[(long long)b * 6 + c];
    }
    GreenAt<T> at;  // WIDE: of the thread's only frequency, while the data are on their way
    // first butterflies, from memory: column j fastest
    constexpr int NF = NC * B * P, IF = (NF + NT - 1) / NT;
#pragma unroll
    for (int i = 0; i < IF; ++i) {
        const int e = t + NT * i;
        const int j = e % B, p = (e / B) % P, c = e / (B * P);
        cx<T> v[A];
        const bool in = e < NF && p0 + p < npen;
        const cx<T>* s = S + (in ? (long long)c * g.nspec + (long long)(p0 + p) * N + j : 0);
#pragma unroll
        for (int q = 0; q < A; ++q) v[q] = s[in ? B * q : 0];
        if (i == 0) {
            for (int m = t; m < N; m += NT) W[m] = tw[m];
            if constexpr (WIDE) {
                int kx, ky, kz;
                freq(p0, t % A + A * (t / A % B), kx, ky, kz);
                at = green_at<T>(kx, ky, kz, g, lam0, mu0);
            }
            if (stop) return;
            __syncthreads();
        }
        if (NF % NT == 0 || e < NF) {
            dft<T, A, -1>(v);
            twiddle<T, A, -1>(v, W, j);
#pragma unroll
            for (int k = 0; k < A; ++k) X[slot(c, p, j, k)] = v[k];
        }
    }
    if (blockIdx.x == 0) block_sum<6, NT>(acc, dcm);
    __syncthreads();
    // second butterflies in place: column k1 fastest
    constexpr int NS = NC * A * P, NI = 6 * A * P;
#pragma unroll 1
    for (int e = t; e < NS; e += NT) {
        const int k = e % A, p = (e / A) % P, c = e / (A * P);
        cx<T> u[B];
#pragma unroll
        for (int j = 0; j < B; ++j) u[j] = X[slot(c, p, j, k)];
        dft<T, B, -1>(u);
#pragma unroll
        for (int j = 0; j < B; ++j) X[slot(c, p, j, k)] = u[j];
    }
    __syncthreads();
    double esum[1] = {0.0};
#pragma unroll 1
    for (int e = t; e < N * P; e += NT) {
        const int k1 = e % A, k2 = (e / A) % B, p = e / N;
        const int pen = p0 + p;
        if (pen < npen) {
            int kx, ky, kz;
            freq(pen, k1 + A * k2, kx, ky, kz);
            if constexpr (!WIDE) at = green_at<T>(kx, ky, kz, g, lam0, mu0);
            esum[0] += gamma_point_at<T, POL>(X + slot(0, p, k2, k1), P * B * LS, kx, ky, kz, at, g, lam0, mu0, alpha,
                                              beta, dc_mode, Es, dcm, st);
        }
    }
    __syncthreads();
#pragma unroll 1
    for (int e = t; e < NI; e += NT) {
        const int k = e % A, p = (e / A) % P, c = e / (A * P);
        cx<T> u[B];
#pragma unroll
        for (int j = 0; j < B; ++j) u[j] = X[slot(c, p, j, k)];
        dft<T, B, +1>(u);
        twiddle<T, B, +1>(u, W, k);
#pragma unroll
        for (int j = 0; j < B; ++j) X[slot(c, p, j, k)] = u[j];
    }
    __syncthreads();
    {
        const int j = t % B, p = (t / B) % P, c = t / (B * P);
        if (t < 6 * B * P && p0 + p < npen) {
            cx<T> w[A];
#pragma unroll
            for (int k = 0; k < A; ++k) w[k] = X[slot(c, p, j, k)];
            dft<T, A, +1>(w);
            cx<T>* o = S + (long long)c * g.nspec + (long long)(p0 + p) * N + j;
#pragma unroll
            for (int q = 0; q < A; ++q) o[B * q] = w[q];
        }
    }
    if (part_err) block_sum<1, NT>(esum, part_err + blockIdx.x);
}

template <typename T>
struct PgArgs {
    cx<T>* S;
    const cx<T>* tw;
    const double* E;
    const double* part_mean;
    double* part_err;
    DevState* st;
    const int* done;
    double lam0, mu0;
    double c[3];  // 2 pi / n per axis; polarization: alpha, beta
    int nx, ny, nz;
    int n_mean;  // partial sums of the mean, 0: no mean (DC_ZERO)
};
static_assert(sizeof(PgArgs<double>) <= 112, "one cheap launch");

template <typename T, int N, bool POL, bool WIDE>
__global__ __launch_bounds__((GCfg<T, N, POL, WIDE>::NT)) void k_pg(PgArgs<T> a)
{
    Geo g;
    g.nx = a.nx;
    g.ny = a.ny;
    g.nz = a.nz;
    g.nh = a.nx / 2 + 1;
    g.two_d = a.nz == 1;
    g.N = (long long)a.nx * a.ny * a.nz;
    g.nspec = (long long)g.nh * a.ny * a.nz;
    for (int i = 0; i < 3; ++i)
        g.kh[i] = POL ? 2.0 * 3.14159265358979323846 / (double)(i == 0 ? a.nx : i == 1 ? a.ny : a.nz) : a.c[i];
    pg_body<T, N, POL, WIDE>(a.S, g, a.tw, a.lam0, a.mu0, POL ? a.c[0] : 0.0, POL ? a.c[1] : 0.0,
                             a.n_mean > 0 ? DC_MEAN : DC_ZERO, a.E, a.part_mean, a.n_mean, a.part_err, a.st, a.done);
}

// ---------------------------------------------------------------------------
// Launchers, instantiated in rpm_pencil.hip
// ---------------------------------------------------------------------------
template <typename T, int N>
struct Pencil {
    static void y_pass(int dir, int comps, const cx<T>* in, cx<T>* out, const Geo& g, const cx<T>* tw,
                       const int* done, hipStream_t s);
    static int rows() { return tile_rows<T, N>(); }
    static bool has_gamma(bool pol) { return !pol || pol_gamma<T, N>(); }
    static void x_forward(bool pol, const T* xin, const uint8_t* phase, const double* lame, int use_ref, double lam0,
                          double mu0, cx<T>* S1, double* part_mean, const Geo& g, const cx<T>* tw, const int* done,
                          hipStream_t s);
    static void x_inverse(bool pol, const cx<T>* S1, const T* eps, T* out, int out_mode, const T* shift,
                          double* part_inc, const Geo& g, const cx<T>* tw, const uint8_t* phase, const double* lame,
                          double lam0, double mu0, double beta, const int* done, hipStream_t s);
    static int gamma_blocks(bool pol, int npen)
    {
        const int p = gamma_wide<T, N>(pol, npen) ? 1 : GCfg<T, N, false, false>::P;
        return (npen + p - 1) / p;
    }
    static void gamma(bool pol, cx<T>* S, const Geo& g, const cx<T>* tw, double lam0, double mu0, double alpha,
                      double beta, int dc_mode, const double* E, const double* part_mean, int n_mean,
                      double* part_err, DevState* st, const int* done, hipStream_t s);
};

}  // namespace rpm

// Fused passes of the warm-start network (rpm_fno.hip) for up to 64 channels
// and 16 modes per axis.
//
// A spectral layer is five launches: k_dft_xy and k_dft_z (the truncated DFT),
// k_mix (per-frequency channel mixing), k_idft_z, and k_layer_out (inverse DFT
// along y and x, pointwise channel map, bias and GELU).  Each h is read twice
// and written once per layer; as separate batched GEMMs the same layer was 26
// launches that read h five times and moved every partial sum of a complex
// product through memory.  Warm start of a 64^3 cell (width 32, 4 layers, 12
// modes): 1990 -> 305 us; training step on four 32^3 cells: 44.2 -> 0.75 ms, of
// which the weight gradients (k_wgrad) were most.
//
// The arithmetic is that of the batched GEMM (k_gemm_bf16), bit for bit:
// operands in FP32, rounded to bfloat16 where an MFMA reads them, one FP32
// accumulator per real product, k ascending in steps of 16, the partial sums of
// a complex product added in FP32 afterwards.  A layer's result feeds the next
// layer's bfloat16 operands, so a different order would flip roundings there.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fno {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// round to nearest even (v_cvt_pk_bf16_f32)
__device__ __forceinline__ short to_bf16(float f) { return __builtin_bit_cast(short, (__bf16)f); }
__device__ __forceinline__ bf16x4 to_bf16(const float (&f)[4])
{
    typedef __bf16 h4 __attribute__((ext_vector_type(4)));
    return __builtin_bit_cast(bf16x4, __builtin_convertvector((f32x4{f[0], f[1], f[2], f[3]}), h4));
}
// v_mfma_f32_16x16x16_bf16: lane l holds A(l % 16, 4 (l / 16) + q) and
// B(4 (l / 16) + q, l % 16), and receives C(4 (l / 16) + q, l % 16), q < 4
__device__ __forceinline__ f32x4 mfma(bf16x4 a, bf16x4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ bf16x4 ld4(const short* p) { return *reinterpret_cast<const bf16x4*>(p); }

__device__ __forceinline__ float gelu(float x)
{
    return 0.5f * x * (1.f + erff(x * 0.70710678118654752f));
}
__device__ __forceinline__ float gelu_grad(float x)
{
    const float cdf = 0.5f * (1.f + erff(x * 0.70710678118654752f));
    const float pdf = 0.39894228040143268f * expf(-0.5f * x * x);
    return cdf + x * pdf;
}

constexpr int kModeSlots = 16;  // modes per axis, padded to one MFMA tile

// Twiddles of one axis in bfloat16, cos and sin of 2 pi k x / n with k the
// signed frequency kk - m/2, zero where kk >= m or x >= n (np: n padded to 16).
// Forward tables [kk][x], inverse tables [x][kk]: an MFMA operand is one 8-byte
// load from either.  q: cos at a quarter, sin at a half and cos at three quarters
// of a turn as the host's long double functions give them (about 1e-20, not 0:
// the MFMA's sums see the difference).
struct AxTab {
    short *fc, *fs, *ic, *is;
    int n, np;
    float q[3];
};

__global__ __launch_bounds__(256) void k_tables(AxTab a0, AxTab a1, AxTab a2, int m)
{
    const AxTab a = blockIdx.y == 0 ? a0 : blockIdx.y == 1 ? a1 : a2;
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= kModeSlots * a.np) return;
    const int kk = e / a.np, x = e - kk * a.np;
    short c = 0, s = 0;
    if (kk < m && x < a.n) {
        const int r = (((kk - m / 2) * x) % a.n + a.n) % a.n;
        double sd, cd;
        sincospi(2.0 * r / a.n, &sd, &cd);
        c = to_bf16(4 * r == a.n ? a.q[0] : 4 * r == 3 * a.n ? a.q[2] : (float)cd);
        s = to_bf16(2 * r == a.n ? a.q[1] : (float)sd);
    }
    a.fc[kk * a.np + x] = c;
    a.fs[kk * a.np + x] = s;
    a.ic[x * kModeSlots + kk] = c;
    a.is[x * kModeSlots + kk] = s;
}

// Truncated DFT of one (y, x) plane per block: x, then y.  The waves transform
// 16 rows each along x (K = n0) and leave the rounded operands of the y
// transform in LDS as [kx][y]; waves 0 and 1 then form the real and imaginary
// part of T2[plane][ky][kx].  One read of v; 16-byte loads (VEC: rows of a
// multiple of four elements, aligned).
template <bool VEC>
__global__ __launch_bounds__(256) void k_dft_xy(const float* __restrict__ v, float* __restrict__ T2, long long plane,
                                                int m, AxTab ax, AxTab ay)
{
    extern __shared__ __align__(16) short T1[];  // [re, im][kx][y], rows of ld
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int li = lane & 15, lk = 4 * (lane >> 4);
    const int n0 = ax.n, n1 = ay.n, ld = ay.np + 4;
    short* Tre = T1;
    short* Tim = T1 + kModeSlots * ld;
    const float* src = v + (long long)blockIdx.x * n0 * n1;
    for (int yt = 16 * wave; yt < ay.np; yt += 16 * nw) {
        f32x4 re = {0.f, 0.f, 0.f, 0.f}, im = re;
        const bool yin = yt + li < n1;
        const float* row = src + (long long)(yin ? yt + li : 0) * n0;
#pragma unroll 4
        for (int x0 = 0; x0 < ax.np; x0 += 16) {
            const int x = x0 + lk;
            float a[4];
            if constexpr (VEC) {
                const float4 t = *reinterpret_cast<const float4*>(row + (x < n0 ? x : 0));
                const bool in = yin && x < n0;
                a[0] = in ? t.x : 0.f;
                a[1] = in ? t.y : 0.f;
                a[2] = in ? t.z : 0.f;
                a[3] = in ? t.w : 0.f;
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) a[q] = yin && x + q < n0 ? row[x + q] : 0.f;
            }
            const bf16x4 ab = to_bf16(a);
            re = mfma(ab, ld4(ax.fc + li * ax.np + x), re);
            im = mfma(ab, ld4(ax.fs + li * ax.np + x), im);
        }
        bf16x4 tr, ti;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            tr[q] = to_bf16(re[q]);
            ti[q] = to_bf16(-im[q]);
        }
        *reinterpret_cast<bf16x4*>(Tre + li * ld + yt + lk) = tr;
        *reinterpret_cast<bf16x4*>(Tim + li * ld + yt + lk) = ti;
    }
    __syncthreads();
    if (wave < 2) {
        // re = C Tre + S Tim, im = C Tim - S Tre
        const short* Tc = wave == 0 ? Tre : Tim;
        const short* Ts = wave == 0 ? Tim : Tre;
        f32x4 c = {0.f, 0.f, 0.f, 0.f}, s = c;
        for (int y0 = 0; y0 < ay.np; y0 += 16) {
            const int o = li * ld + y0 + lk, t = li * ay.np + y0 + lk;
            c = mfma(ld4(ay.fc + t), ld4(Tc + o), c);
            s = mfma(ld4(ay.fs + t), ld4(Ts + o), s);
        }
        float* out = T2 + wave * plane + (long long)blockIdx.x * m * m;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (lk + q < m && li < m) out[(lk + q) * m + li] = wave == 0 ? s[q] + c[q] : c[q] - s[q];
    }
}

// X[p][kz][(ky, kx)] = sum_z F[kz][z] T2[p][z][(ky, kx)]: one block of two
// waves (real, imaginary) per field and 16 columns.
__global__ __launch_bounds__(128) void k_dft_z(const float* __restrict__ T2, long long plane2, float* __restrict__ X,
                                               long long planeX, int m, int ctiles, AxTab az)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 15, lk = 4 * (lane >> 4);
    const int mm = m * m;
    const long long p = blockIdx.x / ctiles;
    const int col = (int)(blockIdx.x - p * ctiles) * 16 + li;
    const float* base = T2 + p * az.n * mm + (col < mm ? col : 0);
    const float* tc = base + (wave == 0 ? 0 : plane2);
    const float* ts = base + (wave == 0 ? plane2 : 0);
    f32x4 c = {0.f, 0.f, 0.f, 0.f}, s = c;
#pragma unroll 4
    for (int z0 = 0; z0 < az.np; z0 += 16) {
        float fc[4], fs[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int z = z0 + lk + q;
            const bool in = z < az.n && col < mm;
            const long long o = (long long)(z < az.n ? z : 0) * mm;
            const float u = tc[o], w = ts[o];
            fc[q] = in ? u : 0.f;
            fs[q] = in ? w : 0.f;
        }
        const int t = li * az.np + z0 + lk;
        c = mfma(ld4(az.fc + t), to_bf16(fc), c);
        s = mfma(ld4(az.fs + t), to_bf16(fs), s);
    }
    float* out = X + wave * planeX + p * m * mm + col;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (lk + q < m && col < mm) out[(lk + q) * mm] = wave == 0 ? s[q] + c[q] : c[q] - s[q];
}

// U[p][z][(ky, kx)] = sum_kz G[z][kz] Y[p][kz][(ky, kx)], G = cos + i sin: one
// block per field and 16 columns, waves (part, every other tile of 16 z).
__global__ __launch_bounds__(256) void k_idft_z(const float* __restrict__ Y, long long planeY, float* __restrict__ U,
                                                long long planeU, int m, int ctiles, AxTab az)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 15, lk = 4 * (lane >> 4);
    const int mm = m * m, part = wave & 1;
    const long long p = blockIdx.x / ctiles;
    const int col = (int)(blockIdx.x - p * ctiles) * 16 + li;
    float fr[4], fi[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const bool in = lk + q < m && col < mm;
        const float* y = Y + (p * m + (in ? lk + q : 0)) * mm + (in ? col : 0);
        const float a = y[0], b = y[planeY];
        fr[q] = in ? a : 0.f;
        fi[q] = in ? b : 0.f;
    }
    // re = C Yre - S Yim, im = C Yim + S Yre
    const bf16x4 yc = to_bf16(part == 0 ? fr : fi), ys = to_bf16(part == 0 ? fi : fr);
    float* out = U + part * planeU + p * az.n * mm + col;
    for (int zt = 16 * (wave >> 1); zt < az.np; zt += 32) {
        const int t = (zt + li) * kModeSlots + lk;
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        const f32x4 c = mfma(ld4(az.ic + t), yc, zero), s = mfma(ld4(az.is + t), ys, zero);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int z = zt + lk + q;
            if (z < az.n && col < mm) out[(long long)z * mm] = part == 0 ? c[q] - s[q] : s[q] + c[q];
        }
    }
}

// Y[b][o][k] = sum_i R(k)[o][i] X[b][i][k], or with CONJ sum_i conj(R(k)[i][o])
// X[b][i][k]; one wave per frequency, every weight read once (16-byte loads:
// VEC).  The pass is bound by the weights: 8 C^2 bytes per frequency.
template <int CT, bool CONJ, bool VEC>
__global__ __launch_bounds__(256) void k_mix(const float* __restrict__ Rre, const float* __restrict__ Rim,
                                             const float* __restrict__ X, long long planeX, float* __restrict__ Y,
                                             long long planeY, int C, int B, int m3)
{
    const int lane = threadIdx.x & 63;
    const int li = lane & 15, lk = 4 * (lane >> 4);
    const long long k = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (k >= m3) return;
    const float* R[2] = {Rre + k * C * C, Rim + k * C * C};
    for (int b0 = 0; b0 < B; b0 += 16) {
        bf16x4 xr[CT], xi[CT];
#pragma unroll
        for (int ks = 0; ks < CT; ++ks) {
            float fr[4], fi[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = 16 * ks + lk + q, b = b0 + li;
                const bool in = i < C && b < B;
                const float* x = X + ((long long)(in ? b : 0) * C + (in ? i : 0)) * m3 + k;
                const float u = x[0], w = x[planeX];
                fr[q] = in ? u : 0.f;
                fi[q] = in ? w : 0.f;
            }
            xr[ks] = to_bf16(fr);
            xi[ks] = to_bf16(fi);
        }
#pragma unroll
        for (int ot = 0; ot < CT; ++ot) {
            f32x4 rr = {0.f, 0.f, 0.f, 0.f}, ii = rr, ri = rr, ir = rr;
#pragma unroll
            for (int ks = 0; ks < CT; ++ks) {
                const int o = 16 * ot + li, i = 16 * ks + lk;
                bf16x4 a[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    float f[4];
                    if constexpr (VEC && !CONJ) {
                        const bool in = o < C && i < C;
                        const float4 t = *reinterpret_cast<const float4*>(R[h] + (in ? o * C + i : 0));
                        f[0] = in ? t.x : 0.f;
                        f[1] = in ? t.y : 0.f;
                        f[2] = in ? t.z : 0.f;
                        f[3] = in ? t.w : 0.f;
                    } else {
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const bool in = o < C && i + q < C;
                            const float t = R[h][in ? (CONJ ? (i + q) * C + o : o * C + i + q) : 0];
                            f[q] = in ? t : 0.f;
                        }
                    }
                    a[h] = to_bf16(f);
                }
                rr = mfma(a[0], xr[ks], rr);
                ii = mfma(a[1], xi[ks], ii);
                ri = mfma(a[0], xi[ks], ri);
                ir = mfma(a[1], xr[ks], ir);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int o = 16 * ot + lk + q, b = b0 + li;
                if (o < C && b < B) {
                    float* y = Y + ((long long)b * C + o) * m3 + k;
                    y[0] = CONJ ? ii[q] + rr[q] : rr[q] - ii[q];
                    y[planeY] = CONJ ? ri[q] - ir[q] : ir[q] + ri[q];
                }
            }
        }
    }
}

// Gradient of the spectral weights, dR(k) = (1/N) sum_b D[b][.][k] X[b][.][k]^H:
// one wave per frequency, the gradient written once in whole rows.
template <int CT>
__global__ __launch_bounds__(256) void k_spec_wgrad(const float* __restrict__ D, const float* __restrict__ X,
                                                    long long plane, float* __restrict__ gre,
                                                    float* __restrict__ gim, int C, int B, int m3, float invN)
{
#pragma clang fp contract(off)
    const int lane = threadIdx.x & 63;
    const int li = lane & 15, lk = 4 * (lane >> 4);
    const long long k = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (k >= m3) return;
    auto frag = [&](const float* S, int t, int b0) {
        float f[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int c = 16 * t + li, b = b0 + lk + q;
            const bool in = c < C && b < B;
            const float u = S[((long long)(in ? b : 0) * C + (in ? c : 0)) * m3 + k];
            f[q] = in ? u : 0.f;
        }
        return to_bf16(f);
    };
#pragma unroll
    for (int ot = 0; ot < CT; ++ot) {
        f32x4 a[4][CT];
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int it = 0; it < CT; ++it) a[e][it] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int b0 = 0; b0 < B; b0 += 16) {
            const bf16x4 dr = frag(D, ot, b0), di = frag(D + plane, ot, b0);
#pragma unroll
            for (int it = 0; it < CT; ++it) {
                const bf16x4 xr = frag(X, it, b0), xi = frag(X + plane, it, b0);
                a[0][it] = mfma(dr, xr, a[0][it]);
                a[1][it] = mfma(di, xi, a[1][it]);
                a[2][it] = mfma(di, xr, a[2][it]);
                a[3][it] = mfma(dr, xi, a[3][it]);
            }
        }
#pragma unroll
        for (int it = 0; it < CT; ++it)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int o = 16 * ot + lk + q, i = 16 * it + li;
                if (o < C && i < C) {
                    const long long e = (k * C + o) * C + i;
                    gre[e] = invN * a[1][it][q] + invN * a[0][it][q];
                    gim[e] = invN * a[2][it][q] - invN * a[3][it][q];
                }
            }
    }
}

// End of a layer.  A block owns 16 rows y of one (batch, z) and all channels:
// it forms V = sum_ky G[y][ky] U[c][z][ky][kx] (rounded operands in LDS), then
// each of its 16 waves takes one row and, 16 voxels at a time,
//   val = (1/N) Re sum_kx V exp(2 pi i kx x / n) + W h        (W^T h with trans)
// FWD: pre = val + bias (kept when pre_out is given), out = gelu(pre).
// BWD: out = val gelu'(aux) (aux: pre-activations of the layer below), the
// gradient the next lower layer starts from, possibly in aux's place; PLAIN: out = val.
enum { LAYER_FWD = 0, LAYER_BWD = 1, LAYER_PLAIN = 2 };
__host__ __device__ constexpr int layer_vs(int CT) { return CT * 256 + (CT < 4 ? 4 : 0); }  // row of V, per y

template <int CT, int MODE>
__global__ __launch_bounds__(1024) void k_layer_out(const float* __restrict__ U, long long planeU,
                                                    const float* __restrict__ h, const float* __restrict__ W,
                                                    int trans, const float* __restrict__ bias,
                                                    const float* aux, float* __restrict__ pre_out, float* out, int C,
                                                    int n2, int m, float alpha, AxTab ax, AxTab ay)
{
#pragma clang fp contract(off)
    extern __shared__ __align__(16) short V[];  // [re, im][y][c][kx]
    constexpr int vs = layer_vs(CT);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 15, lk = 4 * (lane >> 4);
    const int n0 = ax.n, n1 = ay.n, mm = m * m, nyt = ay.np / 16;
    const int yt = blockIdx.x % nyt;
    const long long bz = blockIdx.x / nyt;
    const int z = (int)(bz % n2);
    const long long b = bz / n2;
    const long long N = (long long)n0 * n1 * n2;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    {
        const int t = (16 * yt + li) * kModeSlots + lk;
        const bf16x4 gc = ld4(ay.ic + t), gs = ld4(ay.is + t);
#pragma unroll
        for (int cc = 0; cc < CT; ++cc) {
            const int c = wave + 16 * cc;
            float fr[4], fi[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const bool in = c < C && li < m && lk + q < m;
                const float* u = U + ((b * C + (in ? c : 0)) * n2 + z) * mm + (in ? (lk + q) * m + li : 0);
                const float r = u[0], i = u[planeU];
                fr[q] = in ? r : 0.f;
                fi[q] = in ? i : 0.f;
            }
            const bf16x4 ur = to_bf16(fr), ui = to_bf16(fi);
            const f32x4 rc = mfma(ur, gc, zero), is = mfma(ui, gs, zero), ic = mfma(ui, gc, zero),
                        rs = mfma(ur, gs, zero);
            bf16x4 vr, vi;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                vr[q] = to_bf16(rc[q] - is[q]);
                vi[q] = to_bf16(rs[q] + ic[q]);
            }
            *reinterpret_cast<bf16x4*>(V + li * vs + c * 16 + lk) = vr;
            *reinterpret_cast<bf16x4*>(V + (16 + li) * vs + c * 16 + lk) = vi;
        }
    }
    __syncthreads();
    const int y = 16 * yt + wave;
    if (y >= n1) return;
    bf16x4 wf[CT][CT], vr[CT], vi[CT];
    float bv[CT][4];
#pragma unroll
    for (int ot = 0; ot < CT; ++ot) {
        vr[ot] = ld4(V + wave * vs + (16 * ot + li) * 16 + lk);
        vi[ot] = ld4(V + (16 + wave) * vs + (16 * ot + li) * 16 + lk);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int c = 16 * ot + lk + q;
            bv[ot][q] = MODE == LAYER_FWD && c < C ? bias[c] : 0.f;
        }
#pragma unroll
        for (int ks = 0; ks < CT; ++ks) {
            float f[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int o = 16 * ot + li, i = 16 * ks + lk + q;
                f[q] = o < C && i < C ? W[trans ? i * C + o : o * C + i] : 0.f;
            }
            wf[ot][ks] = to_bf16(f);
        }
    }
    const long long row = b * C * N + ((long long)z * n1 + y) * n0;
    float hn[CT][4], an[CT][4];
    auto load = [&](int x0) {
        const int x = x0 + li;
#pragma unroll
        for (int ks = 0; ks < CT; ++ks)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int c = 16 * ks + lk + q;
                const bool in = c < C && x < n0;
                const long long o = row + (in ? c * N + x : 0);
                const float t = h[o];
                hn[ks][q] = in ? t : 0.f;
                if constexpr (MODE == LAYER_BWD) an[ks][q] = aux[o];  // same (c, x) as this lane's outputs
            }
    };
    load(0);
    for (int x0 = 0; x0 < ax.np; x0 += 16) {
        bf16x4 hb[CT];
        float ac[CT][4];
#pragma unroll
        for (int ks = 0; ks < CT; ++ks) {
            hb[ks] = to_bf16(hn[ks]);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if constexpr (MODE == LAYER_BWD) ac[ks][q] = an[ks][q];
        }
        if (x0 + 16 < ax.np) load(x0 + 16);  // the next voxels in flight meanwhile
        const int t = (x0 + li) * kModeSlots + lk;
        const bf16x4 gc = ld4(ax.ic + t), gs = ld4(ax.is + t);
        const int x = x0 + li;
#pragma unroll
        for (int ot = 0; ot < CT; ++ot) {
            const f32x4 re = mfma(vr[ot], gc, zero), im = mfma(vi[ot], gs, zero);
            f32x4 w = zero;
#pragma unroll
            for (int ks = 0; ks < CT; ++ks) w = mfma(wf[ot][ks], hb[ks], w);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int c = 16 * ot + lk + q;
                if (c < C && x < n0) {
                    const float t0 = alpha * re[q];
                    const float t1 = -alpha * im[q] + t0;
                    const float val = w[q] + t1;
                    const long long o = row + c * N + x;
                    if constexpr (MODE == LAYER_FWD) {
                        const float p = val + bv[ot][q];
                        if (pre_out) pre_out[o] = p;
                        out[o] = gelu(p);
                    } else if constexpr (MODE == LAYER_BWD) {
                        out[o] = val * gelu_grad(ac[ot][q]);
                    } else {
                        out[o] = val;
                    }
                }
            }
        }
    }
}

// out[b][o][v] = sum_i W(o, i) in[b][i][v] (W row-major [M][K], or [K][M] with
// trans) for K <= 16 KT, M <= 64: + bias[o], or * gelu'(aux[b][o][v]) (out may be
// aux).  A wave takes 32 voxels and all rows at a time.
template <int KT>
__global__ __launch_bounds__(256) void k_pointwise(const float* __restrict__ W, int trans,
                                                   const float* __restrict__ in, float* out,
                                                   const float* __restrict__ bias, const float* aux,
                                                   int M, int K, long long N, long long ntiles, long long tpb)
{
    constexpr int KS = 16 * KT + 4;
    __shared__ __align__(16) short Ws[64 * KS];
    const int Mp = (M + 15) / 16 * 16;
    for (int e = threadIdx.x; e < Mp * 16 * KT; e += 256) {
        const int o = e / (16 * KT), i = e - o * (16 * KT);
        Ws[o * KS + i] = to_bf16(o < M && i < K ? W[trans ? i * M + o : o * K + i] : 0.f);
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int li = lane & 15, lk = 4 * (lane >> 4);
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    for (long long t = (long long)blockIdx.x * 4 + (threadIdx.x >> 6); t < ntiles; t += (long long)gridDim.x * 4) {
        const long long b = t / tpb, v0 = (t - b * tpb) * 32;
        bf16x4 xb[2][KT];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int ks = 0; ks < KT; ++ks) {
                float f[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int i = 16 * ks + lk + q;
                    const long long v = v0 + 16 * u + li;
                    const bool ok = i < K && v < N;
                    const float x = in[ok ? (b * K + i) * N + v : 0];
                    f[q] = ok ? x : 0.f;
                }
                xb[u][ks] = to_bf16(f);
            }
        for (int m0 = 0; m0 < Mp; m0 += 16) {
            f32x4 acc[2] = {zero, zero};
            float z[2][4];  // aux, before the first store
            if (aux)
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int o = m0 + lk + q;
                        const long long v = v0 + 16 * u + li;
                        z[u][q] = aux[o < M && v < N ? (b * M + o) * N + v : 0];
                    }
#pragma unroll
            for (int ks = 0; ks < KT; ++ks) {
                const bf16x4 a = ld4(Ws + (m0 + li) * KS + 16 * ks + lk);
#pragma unroll
                for (int u = 0; u < 2; ++u) acc[u] = mfma(a, xb[u][ks], acc[u]);
            }
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int o = m0 + lk + q;
                    const long long v = v0 + 16 * u + li;
                    if (o < M && v < N) {
                        float r = acc[u][q];
                        if (bias) r += bias[o];
                        if (aux) r *= gelu_grad(z[u][q]);
                        out[(b * M + o) * N + v] = r;
                    }
                }
        }
    }
}

// Weight and bias gradients of the pointwise maps (lift, layers, projection),
// dW[o][i] = sum_b sum_v d[b][o][v] in[b][i][v] and db[o] = sum_b sum_v d, all of
// a backward pass at once.  The sums keep the order of the batched GEMM (voxels
// ascending in one chain of MFMAs per item, batch and 16 x 16 tile, batches
// added afterwards): Adam divides by the gradient's own scale, so a gradient
// changed in its last bits moves weights across bfloat16 roundings and the next
// step's gradients by 1e-3 in places.  A chain of N / 16 dependent MFMAs is short
// (32^3: 2048 of them); what bounded the GEMM was the latency of its loads in the
// same chain, 1.2 ms per contraction.  Here four waves stream both operands
// through LDS while a fifth runs the chain, and the chains of all maps run side
// by side.
struct WItem {
    const float *d, *in;  // [B][M][N], [B][K][N]
    float *dW, *db;       // [M][K], [M]
    int M, K;
};
constexpr int kMaxItems = 18;  // 16 layers, lift, projection
struct WItems {
    WItem it[kMaxItems];
    int n;
};
constexpr int kChunk = 256, kChunkLd = kChunk + 16;  // voxels per LDS stage, its row

constexpr int kWgradThreads = 320;
template <bool VEC>
__global__ __launch_bounds__(kWgradThreads) void k_wgrad(WItems items, float* __restrict__ part, int B, long long N)
{
    __shared__ __align__(16) short S[2][32][kChunkLd];  // 16 rows of d, 16 of in
    const int ib = blockIdx.x;
    if (ib >= items.n * B) return;
    const WItem w = items.it[ib / B];
    const int b = ib % B, nt = (w.K + 15) / 16;
    const int tile = blockIdx.y;
    if (tile >= (w.M + 15) / 16 * nt) return;
    const int o0 = tile / nt * 16, i0 = tile % nt * 16;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 15, lk = 4 * (lane >> 4);
    // wave 0 runs the chain; wave w > 0 stages rows w - 1, w + 3, ... (0..15 of d,
    // 16..31 of in)
    const float* row[8];
    bool rin[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const int q = max(wave - 1, 0) + 4 * r;
        const int c = q < 16 ? o0 + q : i0 + q - 16, C = q < 16 ? w.M : w.K;
        rin[r] = c < C;
        row[r] = (q < 16 ? w.d : w.in) + ((long long)b * C + (rin[r] ? c : 0)) * N;
    }
    // loads of the next D stages in flight: one stage ahead, the loop waited on
    // memory latency (2.1 us per stage of 0.2 us of work)
    constexpr int D = 4;
    float f[D][8][4];
    auto load = [&](float (&g)[8][4], long long v0) {
        const long long v = v0 + 4 * lane;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            if constexpr (VEC) {
                const bool in = rin[r] && v < N;
                const float4 t = *reinterpret_cast<const float4*>(row[r] + (v < N ? v : 0));
                g[r][0] = in ? t.x : 0.f;
                g[r][1] = in ? t.y : 0.f;
                g[r][2] = in ? t.z : 0.f;
                g[r][3] = in ? t.w : 0.f;
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) g[r][q] = rin[r] && v + q < N ? row[r][v + q] : 0.f;
            }
        }
    };
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < D; ++u)
        if (wave > 0 && u * kChunk < N) load(f[u], u * kChunk);
    for (long long base = 0; base < N; base += D * kChunk) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const long long v0 = base + u * kChunk;
            if (v0 >= N) break;
            const int buf = u & 1;
            if (wave > 0)
#pragma unroll
                for (int r = 0; r < 8; ++r)
                    *reinterpret_cast<bf16x4*>(&S[buf][wave - 1 + 4 * r][4 * lane]) = to_bf16(f[u][r]);
            __syncthreads();  // also: the chain has left the other buffer
            if (wave > 0) {
                if (v0 + D * kChunk < N) load(f[u], v0 + D * kChunk);
            } else {
                const short* da = &S[buf][li][lk];
                const short* db = &S[buf][16 + li][lk];
                if (v0 + kChunk <= N) {
                    // all operands first, then the chain
                    bf16x4 a[kChunk / 16], c[kChunk / 16];
#pragma unroll
                    for (int s = 0; s < kChunk / 16; ++s) {
                        a[s] = ld4(da + 16 * s);
                        c[s] = ld4(db + 16 * s);
                    }
#pragma unroll
                    for (int s = 0; s < kChunk / 16; ++s) acc = mfma(a[s], c[s], acc);
                } else {
                    for (int s = 0; s < (int)(N - v0 + 15) / 16; ++s)
                        acc = mfma(ld4(da + 16 * s), ld4(db + 16 * s), acc);
                }
            }
        }
    }
    if (wave == 0) {
        float* dst = part + ((long long)tile * gridDim.x + ib) * 256;
#pragma unroll
        for (int q = 0; q < 4; ++q) dst[(lk + q) * 16 + li] = acc[q];
    }
}

// dW from the chains' results, batches in order; one thread per weight
__global__ __launch_bounds__(256) void k_wgrad_sum(WItems items, const float* __restrict__ part, int B, int stride)
{
    const WItem w = items.it[blockIdx.y];
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= w.M * w.K) return;
    const int o = e / w.K, i = e - o * w.K, nt = (w.K + 15) / 16;
    const int tile = o / 16 * nt + i / 16;
    const float* p = part + ((long long)tile * stride + blockIdx.y * B) * 256 + (o % 16) * 16 + i % 16;
    float s = p[0];
    for (int b = 1; b < B; ++b) s += p[(long long)b * 256];
    w.dW[e] = s;
}

// db[o] of every item: one block per channel, thread t the voxels t, t + 256, ...
// of every batch, then a tree
__global__ __launch_bounds__(256) void k_bias_grads(WItems items, int B, long long N)
{
    __shared__ float red[256];
    const WItem w = items.it[blockIdx.y];
    const int c = blockIdx.x;
    if (c >= w.M) return;
    float s = 0.f;
    for (int b = 0; b < B; ++b) {
        const float* p = w.d + ((long long)b * w.M + c) * N;
#pragma unroll 8
        for (long long v = threadIdx.x; v < N; v += 256) s += p[v];
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) w.db[c] = red[0];
}

}  // namespace fno

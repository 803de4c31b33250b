// JTFS forward and backward on gfx950: FFT passes in LDS, the fused scalogram
// and second-order kernels, the frequential contraction on FP32 MFMA with the
// modulus and time lowpass fused into its epilogue, and every stage's adjoint.
//
// Scaling conventions: all FFTs are unnormalised; every 1/M of an inverse DFT is
// applied explicitly where the stage's definition puts it.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "fft_lds.hpp"
#include "plan.hpp"
#include "timing.hpp"
#include "split.hpp"
#include "regk.hpp"

namespace jtfs {

typedef float floatx16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ floatx16 mfma32(float a, float b, floatx16 c) {
    // D[i][j] += sum_k A[i][k] B[k][j], 32x32x2: lane (i + 32k) holds A[i][k] and
    // B[k][i]; D element (i, j) sits in lane j + 32*((i/4)%2), register (i%4) + 4*(i/8).
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ floatx16 zero16() {
    floatx16 z;
#pragma unroll
    for (int r = 0; r < 16; ++r) z[r] = 0.f;
    return z;
}
// row (within a 32x32 tile) held by register r of a lane in half h
__device__ __forceinline__ int crow(int r, int h) { return 8 * (r >> 2) + 4 * h + (r & 3); }

// Inverse of the real-spectrum post-pass: Z'[k] = (X[k] + conj X[H-k]) + i w_n^{-k} (X[k] - conj X[H-k]),
// whose unnormalised inverse FFT is n times the interleaved real signal.
__device__ __forceinline__ float2 irfft_bin(float2 p, float2 q, float2 w) {
    const float2 S = make_float2(p.x + q.x, p.y - q.y);          // p + conj q
    const float2 D = make_float2(p.x - q.x, p.y + q.y);          // p - conj q
    const float2 wD = cmulc(D, w);                               // w^{-k} D
    return make_float2(S.x - wD.y, S.y + wD.x);                  // S + i wD
}

// ---------------------------------------------------------------------------
// One step of a four-step transform over LDS: transform c of batch b has element e at
// in[b*ib + c + e*ies]; the output X_c[k] (times w_n^{c k} when twl > 0, the four-step
// twist, and times scale) goes to out[b*ob + c*ocs + k*oes].  2^logC adjacent
// transforms per workgroup, loaded with adjacent columns on adjacent threads.
// PACK: the input rows are half spectra, packed on the way in (element i of the row's
// 2^twl from its bins i and 2^twl - i) instead of by a pass of its own.
// ---------------------------------------------------------------------------
template <typename CI, typename C>
__device__ __forceinline__ C to_cplx(CI v) {
    using R = typename cplx<C>::real;
    return cplx<C>::make((R)v.x, (R)v.y);
}

template <typename CI, typename C, bool PACK = false>
__global__ void __launch_bounds__(1024) k_fft_cols_t(const CI* in, C* out, int loglen, int ncols, int logC,
                                                    int64_t ib, int64_t ies, int64_t ob, int64_t ocs,
                                                    int64_t oes, int twl, const C* __restrict__ tw, int tw_log, int inv,
                                                    typename cplx<C>::real scale) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    C* s = (C*)lds_raw;
    const int len = 1 << loglen, st = lpad_len(len) + 1;     // odd stride: columns in distinct banks
    const int Cn = 1 << logC;
    const int c0 = blockIdx.x * Cn;
    const int nc = min(Cn, ncols - c0);
    const int tot = nc * len;
    const int64_t b = blockIdx.y;
    in += b * ib;
    out += b * ob;
    // all of a thread's loads (at most 16: tot <= 16 blockDim, as the transform
    // requires) are issued before any LDS store, so that their latencies overlap
    // instead of following one another
    constexpr int kMaxPerThread = 16;
    C v[kMaxPerThread];
#pragma unroll
    for (int q = 0; q < kMaxPerThread; ++q) {
        const int e = threadIdx.x + q * blockDim.x;
        if (e < tot) {
            const int64_t i = c0 + (e & (Cn - 1)) + (int64_t)(e >> logC) * ies;
            if constexpr (PACK) v[q] = irfft_bin(in[i], in[((int64_t)1 << twl) - i], tw[i << (tw_log - twl - 1)]);
            else v[q] = to_cplx<CI, C>(in[i]);
        }
    }
#pragma unroll
    for (int q = 0; q < kMaxPerThread; ++q) {
        const int e = threadIdx.x + q * blockDim.x;
        if (e < tot) {
            const int c = e & (Cn - 1), k = e >> logC;
            s[c * st + lpad(k)] = v[q];
        }
    }
    __syncthreads();
    lds_fft<16>(s, loglen, nc, st, tw, tw_log, inv != 0);
    const int tws = tw_log - twl;
    if (ocs == 1) {
        for (int e = threadIdx.x; e < tot; e += blockDim.x) {
            const int c = e & (Cn - 1), k = e >> logC;
            C v = s[lpad(k) + c * st];
            if (twl) v = cmul(v, twiddle(tw, ((c0 + c) * k) << tws, inv != 0));
            out[(int64_t)(c0 + c) + (int64_t)k * oes] = cplx<C>::make(v.x * scale, v.y * scale);
        }
    } else {
        for (int e = threadIdx.x; e < tot; e += blockDim.x) {
            const int c = e >> loglen, k = e & (len - 1);
            C v = s[lpad(k) + c * st];
            if (twl) v = cmul(v, twiddle(tw, ((c0 + c) * k) << tws, inv != 0));
            out[(int64_t)(c0 + c) * ocs + (int64_t)k * oes] = cplx<C>::make(v.x * scale, v.y * scale);
        }
    }
}

// Real-input spectrum in FP64 from the half-length complex FFT of
// z[k] = x[2k] + i x[2k+1]: X[m] = E[m] + w_n^m O[m], E/O the spectra of the
// even/odd samples; bins m and H - m (H = n/2) from z's bins a and b at them, rounded
// once to FP32.  w: the twiddle of bin m; m = 0 gives bins 0 and H.
__device__ __forceinline__ float2 rfft_bin64(double2 p, double2 q, double2 w) {
    const double2 E = make_double2(0.5 * (p.x + q.x), 0.5 * (p.y - q.y));
    const double2 D = make_double2(p.x - q.x, p.y + q.y);          // p - conj(q)
    const double2 O = make_double2(0.5 * D.y, -0.5 * D.x);      // D / (2i)
    const double2 X = cadd(E, cmul(O, w));
    return make_float2((float)X.x, (float)X.y);
}

// The input transform of rows of up to 2^12 samples in one launch: the FP64 FFT of
// the sample pairs in LDS and the spectrum's bins 0..H straight from there (two
// launches and a round trip of the FP64 row: with the output transform below one signal
// of 2^11 samples took 49.4 us in all, 46.5 now).  2^logH pairs a row, 2^logC rows a
// workgroup.
__global__ void __launch_bounds__(1024) k_rfft64_rows(const float2* __restrict__ x, int rows, int logH, int logC,
                                                     float2* __restrict__ xh, int64_t pitch,
                                                     const double2* __restrict__ tw, int tw_log) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    double2* s = (double2*)lds_raw;
    const int H = 1 << logH, st = lpad_len(H) + 1;
    const int c0 = blockIdx.x << logC, nc = min(1 << logC, rows - c0);
    const int tot = nc << logH;
    constexpr int kMaxPerThread = 4;                 // tot <= 2^12
    float2 v[kMaxPerThread];
#pragma unroll
    for (int q = 0; q < kMaxPerThread; ++q) {
        const int e = threadIdx.x + q * blockDim.x;
        if (e < tot) v[q] = x[((int64_t)c0 << logH) + e];
    }
#pragma unroll
    for (int q = 0; q < kMaxPerThread; ++q) {
        const int e = threadIdx.x + q * blockDim.x;
        if (e < tot) s[(e >> logH) * st + lpad(e & (H - 1))] = make_double2((double)v[q].x, (double)v[q].y);
    }
    __syncthreads();
    lds_fft<16>(s, logH, nc, st, tw, tw_log, false);
    const int tws = tw_log - logH - 1, nm = H / 2 + 1;
    for (int e = threadIdx.x; e < nc * nm; e += blockDim.x) {
        const int c = e / nm, m = e - c * nm;
        float2* row = xh + (c0 + c) * pitch;
        const double2 a = s[c * st + lpad(m)];
        if (m == 0) {
            row[0] = make_float2((float)(a.x + a.y), 0.f);
            row[H] = make_float2((float)(a.x - a.y), 0.f);
            continue;
        }
        const double2 b = s[c * st + lpad(H - m)];
        row[m] = rfft_bin64(a, b, tw[m << tws]);
        row[H - m] = rfft_bin64(b, a, tw[(H - m) << tws]);
    }
}

// The same bins from the FP64 transform in memory (z rows of pitch zp), for longer rows.
__global__ void k_rfft_post64(const double2* __restrict__ z, int64_t zp, float2* __restrict__ xh, int64_t pitch,
                              int logn, const double2* __restrict__ tw, int tw_log) {
    const int H = 1 << (logn - 1);
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m > H / 2) return;
    const double2* zr = z + (int64_t)blockIdx.y * zp;
    float2* row = xh + (int64_t)blockIdx.y * pitch;
    const int tws = tw_log - logn;
    if (m == 0) {
        const double2 q = zr[0];
        row[0] = make_float2((float)(q.x + q.y), 0.f);
        row[H] = make_float2((float)(q.x - q.y), 0.f);
        return;
    }
    const double2 a = zr[m], b = zr[H - m];
    row[m] = rfft_bin64(a, b, tw[m << tws]);
    row[H - m] = rfft_bin64(b, a, tw[(H - m) << tws]);
}

// The output transform of rows of up to 2^12 samples in one launch: packing into LDS,
// inverse FFT, scaled samples out (2^11 samples with gradient 147 -> 141 us, the input
// transform included).  2^logH pairs a row, 2^logC rows a workgroup.
__global__ void __launch_bounds__(1024) k_irfft_rows(const float2* __restrict__ xh, int64_t pitch, int rows, int logH,
                                                    int logC, float2* __restrict__ out, float scale,
                                                    const float2* __restrict__ tw, int tw_log) {
    extern __shared__ float2 s[];
    const int H = 1 << logH, st = lpad_len(H) + 1;
    const int c0 = blockIdx.x << logC, nc = min(1 << logC, rows - c0);
    const int tws = tw_log - logH - 1, nm = H / 2 + 1;
    for (int e = threadIdx.x; e < nc * nm; e += blockDim.x) {
        const int c = e / nm, k = e - c * nm;
        const float2* row = xh + (c0 + c) * pitch;
        const float2 a = row[k], b = row[H - k];
        s[c * st + lpad(k)] = irfft_bin(a, b, tw[k << tws]);
        if (k > 0 && H - k != k) s[c * st + lpad(H - k)] = irfft_bin(b, a, tw[(H - k) << tws]);
    }
    __syncthreads();
    lds_fft<16>(s, logH, nc, st, tw, tw_log, true);
    for (int e = threadIdx.x; e < nc << logH; e += blockDim.x)
        out[((int64_t)c0 << logH) + e] = cscale(s[(e >> logH) * st + lpad(e & (H - 1))], scale);
}

// ---------------------------------------------------------------------------
// First order (fused): fold x_hat * psi_hat_lambda over the band into NX bins,
// inverse FFT (the filtered signal at the scalogram rate), modulus, real FFT of
// the scalogram row; writes X_hat[b][lambda][0..NX/2].
// ---------------------------------------------------------------------------
__device__ __forceinline__ void fold_band(float2* s, const float2* __restrict__ src, const float* __restrict__ ps, int lo,
                                          int hi, int logM) {
    const int M = 1 << logM;
    if (hi - lo < M && M <= 16 * (int)blockDim.x) {
        // every bin receives at most one band sample: all of a thread's loads are
        // issued before any product is formed
        // (two rounds of eight keep the kernels within 64 VGPRs)
#pragma unroll
        for (int q0 = 0; q0 < 16; q0 += 8) {
            float2 v[8];
            float g[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int p = threadIdx.x + (q0 + q) * blockDim.x;
                const int m = lo + ((p - lo) & (M - 1));
                const bool ok = p < M && m <= hi;
                v[q] = ok ? src[m] : make_float2(0.f, 0.f);
                g[q] = ok ? ps[m - lo] : 0.f;
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int p = threadIdx.x + (q0 + q) * blockDim.x;
                if (p < M) s[lpad(p)] = make_float2(v[q].x * g[q], v[q].y * g[q]);
            }
        }
        return;
    }
    for (int p = threadIdx.x; p < M; p += blockDim.x) {
        float2 acc = make_float2(0.f, 0.f);
        for (int m = lo + ((p - lo) & (M - 1)); m <= hi; m += M) {
            const float2 v = src[m];
            const float g = ps[m - lo];
            acc.x += v.x * g;
            acc.y += v.y * g;
        }
        s[lpad(p)] = acc;
    }
}

__global__ void __launch_bounds__(1024, 8) k_scalogram(const float2* __restrict__ xh, int64_t xh_pitch,
                                                   const float* __restrict__ psi1, const int* __restrict__ band1,
                                                   const int64_t* __restrict__ off1, float2* __restrict__ Xh,
                                                   int64_t Xh_pitch, int logNX, float invN,
                                                   const float2* __restrict__ tw, int tw_log) {
    extern __shared__ float2 s[];
    const int lam = blockIdx.x, n1 = gridDim.x;
    const int64_t b = blockIdx.y;
    const int NX = 1 << logNX, H = NX >> 1;
    fold_band(s, xh + b * xh_pitch, psi1 + off1[lam], band1[2 * lam], band1[2 * lam + 1], logNX);
    __syncthreads();
    lds_fft<16>(s, logNX, 1, NX, tw, tw_log, true);
    // modulus of the scalogram-rate samples, packed as z[k] = X[2k] + i X[2k+1]
    {
        float2 v[8];   // H <= 8192 = 8 * blockDim
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int k = threadIdx.x + q * blockDim.x;
            if (k < H) {
                const float2 a = s[lpad(2 * k)], c = s[lpad(2 * k + 1)];
                v[q] = make_float2(__builtin_amdgcn_sqrtf(a.x * a.x + a.y * a.y) * invN,
                                   __builtin_amdgcn_sqrtf(c.x * c.x + c.y * c.y) * invN);
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int k = threadIdx.x + q * blockDim.x;
            if (k < H) s[lpad(k)] = v[q];
        }
        __syncthreads();
    }
    if (logNX > 1) lds_fft<16>(s, logNX - 1, 1, H, tw, tw_log, false);
    float2* out = Xh + (b * n1 + lam) * Xh_pitch;
    const int tws = tw_log - logNX;
    for (int m = threadIdx.x; m <= H / 2; m += blockDim.x) {
        if (m == 0) {
            const float2 z = s[0];
            out[0] = make_float2(z.x + z.y, 0.f);
            out[H] = make_float2(z.x - z.y, 0.f);
            continue;
        }
        const float2 a = s[lpad(m)], c = s[lpad(H - m)];
        auto spec = [&](float2 p, float2 q, int k) {
            const float2 E = make_float2(0.5f * (p.x + q.x), 0.5f * (p.y - q.y));
            const float2 D = make_float2(p.x - q.x, p.y + q.y);
            const float2 O = make_float2(0.5f * D.y, -0.5f * D.x);
            return cadd(E, cmul(O, tw[k << tws]));
        };
        out[m] = spec(a, c, m);
        if (H - m != m) out[H - m] = spec(c, a, H - m);
    }
}

// Zeroth order: S0[b][tau] = (x (*) phi_T)[tau T] as the direct circular sum over the
// offsets where phi_T is stored, h[k] = phi_T[(k - H) mod N]:
//   S0[tau] = sum_{k < len} h[k] x[(tau T + H - k) mod N].
// grid (N/T, B), 1024 threads; each sums a strided share of k with its loads eight at
// once, then the workgroup reduces.  N is a power of two: the circular index is a
// mask (with a 64-bit remainder per term, on 256 threads, this took 92 us for 8
// signals of 2^16 samples and 32 frames, now 9.7).
__global__ void __launch_bounds__(1024) k_s0(const float* __restrict__ x, int64_t N, int64_t T,
                                            const float* __restrict__ h, int64_t len, int64_t H,
                                            float* __restrict__ s0) {
    __shared__ float red[16];
    const int tau = blockIdx.x, NT = gridDim.x;
    const int64_t b = blockIdx.y;
    const float* xb = x + b * N;
    const int64_t base = (int64_t)tau * T + H;       // x index = (base - k) mod N
    float acc = 0.f;
#pragma unroll 8
    for (int64_t k = threadIdx.x; k < len; k += 1024) acc += h[k] * xb[(base - k) & (N - 1)];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        float a = 0.f;
#pragma unroll
        for (int w = 0; w < 16; ++w) a += red[w];
        s0[b * NT + tau] = a;
    }
}

// Its adjoint, added to gx: gx[n] += sum_tau gS0[tau] h[(tau T - n + H) mod N] where
// that index is below len.  grid (ceil(N / 256), B).
__global__ void __launch_bounds__(256) k_s0_bwd(const float* __restrict__ gs0, int64_t N, int64_t T, int NT,
                                                const float* __restrict__ h, int64_t len, int64_t H,
                                                float* __restrict__ gx) {
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t b = blockIdx.y;
    if (n >= N) return;
    const float* g = gs0 + b * NT;
    float acc = 0.f;
    for (int tau = 0; tau < NT; ++tau) {
        const int64_t k = ((int64_t)tau * T - n + H) & (N - 1);
        if (k < len) acc += g[tau] * h[k];
    }
    gx[b * N + n] += acc;
}

// The temporal rates whose rows are transformed in LDS, as one launch covers them:
// blocks blk0[q] .. blk0[q + 1] - 1 of the grid take rate q, `rows` rows each.  A
// launch per rate left most of the GPU idle for several microseconds each, in the
// second order and again in the row FFTs of its adjoint: one signal of 2^11 samples
// (6 such rates) forward 86 -> 58 us, fwd+bwd 200 -> 162 us; 2^18 (14) forward 2469
// -> 2360 us.
struct ShortRate {
    int64_t yoff, psoff;             // its Y2 block and its spectrum in psi2
    int lo, hi, logTa, Tp, rows, alpha;
};
constexpr int kMaxShort = 32;        // rates per launch (1.7 KB of kernel arguments)
struct ShortRates {
    int n;
    int blk0[kMaxShort];
    ShortRate r[kMaxShort];
};
// the rate of this block: the last one that starts at or before it
__device__ __forceinline__ int short_rate(const ShortRates& sr) {
    int q = 0;
    for (int k = 1; k < sr.n; ++k) q += (int)blockIdx.x >= sr.blk0[k] ? 1 : 0;
    return q;
}

// The first-order lowpass as the last blocks (from blk0 on) of a second-order launch.
struct S1Rows {
    int blk0, rows, Mphi, logNX, logNT, Tp, alpha;   // rows per block; Tp, alpha of phi_T's second-order rows
    float eps;
    const float *phiX, *mu1;
    float* S1;
    float2* Yphi;
};

// S1[tau] = (X (*) phi_T)[tau T/2^kX] of sa.rows scalogram rows: fold X_hat * phi_hat over
// the N/T-bin grid (bins -Mneg..Mphi of the NX grid), inverse FFT, real part / NX.  S1
// may be null.  With the lowpass pairs, the same rows are also the second-order rows
// of alpha = phi_T: written to Yphi (real, zero beyond N/T frames and for the padding
// rows n1 <= lambda < Kp) with their row maxima for the operand split.
// It reads the same rows as the second order and waits for the same few loads: in a
// launch of its own one signal of 2^11 samples took 54.7 us in all, now 49.4, and 8 of 2^16
// (as features) 2047, now 2000.
__device__ __forceinline__ void s1_rows(float2* s, unsigned int* rmx, const S1Rows& sa, const float2* __restrict__ Xh,
                                        int64_t Xh_pitch, int n1, int Kp, int64_t y_bstride, float invNX,
                                        const float2* __restrict__ tw, int tw_log, float* __restrict__ rowmax,
                                        int n_alpha) {
    const int64_t b = blockIdx.y;
    const int NX = 1 << sa.logNX, NT = 1 << sa.logNT, rs = lpad_len(NT);
    const int r0 = ((int)blockIdx.x - sa.blk0) * sa.rows, nr = min(sa.rows, (sa.Yphi ? Kp : n1) - r0);
    const int Mneg = (sa.Mphi == NX / 2) ? sa.Mphi - 1 : sa.Mphi;
    if (threadIdx.x < 64) rmx[threadIdx.x] = 0u;
    for (int e = threadIdx.x; e < nr << sa.logNT; e += blockDim.x) {
        const int c = e >> sa.logNT, p = e & (NT - 1);
        float2 acc = make_float2(0.f, 0.f);
        if (r0 + c < n1) {
            const float2* row = Xh + (b * n1 + r0 + c) * Xh_pitch;
#pragma unroll 4
            for (int mt = -Mneg + ((p + Mneg) & (NT - 1)); mt <= sa.Mphi; mt += NT) {
                const int m = mt >= 0 ? mt : -mt;
                const float2 v = row[m];
                const float g = sa.phiX[m];
                acc.x += v.x * g;
                acc.y += (mt >= 0 ? v.y : -v.y) * g;
            }
        }
        s[c * rs + lpad(p)] = acc;
    }
    __syncthreads();
    lds_fft<16>(s, sa.logNT, nr, rs, tw, tw_log, true);
    if (sa.S1) {
        const float inv = mulog_inv(sa.mu1, 0, sa.eps);
        float* o = sa.S1 + (b * n1 + r0) * NT;
        for (int e = threadIdx.x; e < min(nr, n1 - r0) << sa.logNT; e += blockDim.x)
            o[e] = mulog_out(s[(e >> sa.logNT) * rs + lpad(e & (NT - 1))].x * invNX, sa.mu1, inv);
    }
    if (sa.Yphi) {
        float2* y = sa.Yphi + b * y_bstride + (int64_t)r0 * sa.Tp;
        for (int c = 0; c < nr; ++c) {
            float mx = 0.f;
            for (int t = threadIdx.x; t < sa.Tp; t += blockDim.x) {
                const float v = t < NT && r0 + c < n1 ? s[c * rs + lpad(t)].x * invNX : 0.f;
                y[(int64_t)c * sa.Tp + t] = make_float2(v, 0.f);
                mx = fmaxf(mx, fabsf(v));
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
            if ((threadIdx.x & 63) == 0) atomicMax(&rmx[c], __float_as_uint(mx));
        }
        __syncthreads();
        if ((int)threadIdx.x < nr)
            rowmax[(b * n_alpha + sa.alpha) * Kp + r0 + threadIdx.x] = __uint_as_float(rmx[threadIdx.x]);
    }
}

// Second order: Y2[b][alpha][lambda][t] = (X_lambda (*) psi_alpha)[t 2^k2] for t < Ta,
// zero for Ta <= t < Tp and for lambda >= n1 (the K padding of the contraction).
__global__ void __launch_bounds__(1024) k_second_order(const float2* __restrict__ Xh, int64_t Xh_pitch, int n1,
                                                      const float* __restrict__ psi2, const ShortRates sr,
                                                      const S1Rows sa, int Kp, float2* __restrict__ Y, int64_t y_bstride,
                                                      float invNX, const float2* __restrict__ tw, int tw_log,
                                                      float* __restrict__ rowmax, int n_alpha) {
    extern __shared__ float2 s[];
    __shared__ unsigned int rmx[64];
    if ((int)blockIdx.x >= sa.blk0) {
        s1_rows(s, rmx, sa, Xh, Xh_pitch, n1, Kp, y_bstride, invNX, tw, tw_log, rowmax, n_alpha);
        return;
    }
    const int64_t b = blockIdx.y;
    const int q_ = short_rate(sr);
    const ShortRate rt = sr.r[q_];
    const int rows = rt.rows, lo = rt.lo, hi = rt.hi, logTa = rt.logTa, Tp = rt.Tp, alpha = rt.alpha;
    const float* __restrict__ ps = psi2 + rt.psoff;
    Y += rt.yoff;
    const int r0 = ((int)blockIdx.x - sr.blk0[q_]) * rows;
    const int Ta = 1 << logTa, rs = lpad_len(Ta);    // row stride in LDS
    const int nr = min(rows, Kp - r0);
    if (r0 >= n1) {
        // padding rows lambda >= n1 only: zero rows (the contraction reads them), maxima 0
        float2* out = Y + b * y_bstride + (int64_t)r0 * Tp;
        for (int64_t e = threadIdx.x; e < (int64_t)nr * Tp; e += blockDim.x) out[e] = make_float2(0.f, 0.f);
        if ((int)threadIdx.x < nr) rowmax[(b * n_alpha + alpha) * Kp + r0 + threadIdx.x] = 0.f;
        return;
    }
    if (threadIdx.x < 64) rmx[threadIdx.x] = 0u;
    if (hi - lo < Ta && nr * Ta <= 16 * (int)blockDim.x) {
        // every bin receives at most one band sample: all of a thread's loads are
        // issued before any product is formed
#pragma unroll
        for (int q0 = 0; q0 < 16; q0 += 8) {
            float2 v[8];
            float g[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int e = threadIdx.x + (q0 + q) * blockDim.x;
                const int c = e >> logTa, p = e & (Ta - 1);
                const int lam = r0 + c;
                const int m = lo + ((p - lo) & (Ta - 1));
                const bool ok = e < nr * Ta && lam < n1 && m <= hi;
                v[q] = ok ? Xh[(b * n1 + lam) * Xh_pitch + m] : make_float2(0.f, 0.f);
                g[q] = ok ? ps[m - lo] : 0.f;
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int e = threadIdx.x + (q0 + q) * blockDim.x;
                if (e < nr * Ta) s[(e >> logTa) * rs + lpad(e & (Ta - 1))] = make_float2(v[q].x * g[q], v[q].y * g[q]);
            }
        }
    } else {
        for (int e = threadIdx.x; e < nr * Ta; e += blockDim.x) {
            const int c = e >> logTa, p = e & (Ta - 1);
            const int lam = r0 + c;
            float2 acc = make_float2(0.f, 0.f);
            if (lam < n1) {
                const float2* row = Xh + (b * n1 + lam) * Xh_pitch;
                for (int m = lo + ((p - lo) & (Ta - 1)); m <= hi; m += Ta) {
                    const float2 v = row[m];
                    const float g = ps[m - lo];
                    acc.x += v.x * g;
                    acc.y += v.y * g;
                }
            }
            s[c * rs + lpad(p)] = acc;
        }
    }
    __syncthreads();
    lds_fft<16>(s, logTa, nr, rs, tw, tw_log, true);
    float2* out = Y + b * y_bstride + (int64_t)r0 * Tp;
    for (int c = 0; c < nr; ++c) {
        float m = 0.f;
        for (int t = threadIdx.x; t < Tp; t += blockDim.x) {
            const float2 v = t < Ta ? cscale(s[c * rs + lpad(t)], invNX) : make_float2(0.f, 0.f);
            out[(int64_t)c * Tp + t] = v;
            m = fmaxf(m, fmaxf(fabsf(v.x), fabsf(v.y)));
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
        if ((threadIdx.x & 63) == 0) atomicMax(&rmx[c], __float_as_uint(m));
    }
    __syncthreads();
    if ((int)threadIdx.x < nr) rowmax[(b * n_alpha + alpha) * Kp + r0 + threadIdx.x] = __uint_as_float(rmx[threadIdx.x]);
}

// Forward FFT of the gY2 rows lambda < n1 of the rates in sr, in place: `rows` rows
// of 2^logTa points per block.
__global__ void __launch_bounds__(1024) k_rowfft_short(float2* __restrict__ Y, int64_t y_bstride, int n1,
                                                      const ShortRates sr, const float2* __restrict__ tw,
                                                      int tw_log) {
    extern __shared__ float2 s[];
    const int q_ = short_rate(sr);
    const ShortRate rt = sr.r[q_];
    const int logTa = rt.logTa, Ta = 1 << logTa, rs = lpad_len(Ta) + 1;   // odd stride: rows in distinct banks
    const int r0 = ((int)blockIdx.x - sr.blk0[q_]) * rt.rows;
    const int tot = min(rt.rows, n1 - r0) << logTa;
    float2* row = Y + blockIdx.y * y_bstride + rt.yoff + (int64_t)r0 * rt.Tp;
    // all of a thread's loads (at most 16) before any LDS store
    float2 v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int e = threadIdx.x + q * blockDim.x;
        if (e < tot) v[q] = row[(int64_t)(e >> logTa) * rt.Tp + (e & (Ta - 1))];
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int e = threadIdx.x + q * blockDim.x;
        if (e < tot) s[(e >> logTa) * rs + lpad(e & (Ta - 1))] = v[q];
    }
    __syncthreads();
    lds_fft<16>(s, logTa, tot >> logTa, rs, tw, tw_log, false);
    for (int e = threadIdx.x; e < tot; e += blockDim.x)
        row[(int64_t)(e >> logTa) * rt.Tp + (e & (Ta - 1))] = s[(e >> logTa) * rs + lpad(e & (Ta - 1))];
}

// ---------------------------------------------------------------------------
// Frequential contraction (eq. 3 along lambda, both spins) on FP32 MFMA, fused
// with the modulus and the time lowpass:
//   Z_up^T[t][l]   = sum_k Y[k][t] W[l][k]        (theta = -1)
//   Z_down^T[t][l] = sum_k Y[k][t] conj W[l][k]   (theta = +1, the mirrored wavelet)
// from the four real products of (Yr, Yi) x (Wr, Wi); then
//   V^T[tau][l] += sum_t Phi[t][tau] |Z^T[t][l]|   (second MFMA, the C registers of
// the first serve directly as its B operand).  One workgroup: 64 l x one t-chunk,
// four waves on 32x32 sub-tiles; partial V per (t-chunk, t-half) slot.
// ---------------------------------------------------------------------------
template <int NTB>
__global__ void __launch_bounds__(256) k_freq_fwd(const float2* __restrict__ Y, int64_t y_bstride, int Tp, int chunk,
                                                  const float2* __restrict__ Wt, int Mp, int Kp,
                                                  const float* __restrict__ Phi, float* __restrict__ Vp,
                                                  int64_t vp_bstride, int slot0, int nlt) {
    constexpr int NTp = 32 * NTB;
    __shared__ float2 Ys[kKStep][kTileT];
    __shared__ float2 Ws[kKStep][kTileL];
    const int lt = blockIdx.x, ch = blockIdx.y;
    const int64_t b = blockIdx.z;
    const int l0 = lt * kTileL;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int h = lane >> 5, i32 = lane & 31;
    const int lw = (wave >> 1) * 32, twv = (wave & 1) * 32;
    const float2* Yb = Y + b * y_bstride;
    floatx16 vu[NTB], vd[NTB];
#pragma unroll
    for (int n = 0; n < NTB; ++n) { vu[n] = zero16(); vd[n] = zero16(); }

    for (int t0 = ch * chunk; t0 < (ch + 1) * chunk; t0 += kTileT) {
        floatx16 rr = zero16(), ir = zero16(), ri = zero16(), ii = zero16();
        for (int k0 = 0; k0 < Kp; k0 += kKStep) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int f = tid + q * 256, row = f >> 5, c = (f & 31) * 2;
                *(float4*)&Ys[row][c] = *(const float4*)(Yb + (int64_t)(k0 + row) * Tp + t0 + c);
                *(float4*)&Ws[row][c] = *(const float4*)(Wt + (int64_t)(k0 + row) * Mp + l0 + c);
            }
            __syncthreads();
#pragma unroll
            for (int ks = 0; ks < kKStep / 2; ++ks) {
                const float2 a = Ys[2 * ks + h][twv + i32];
                const float2 w = Ws[2 * ks + h][lw + i32];
                rr = mfma32(a.x, w.x, rr);
                ir = mfma32(a.y, w.x, ir);
                ri = mfma32(a.x, w.y, ri);
                ii = mfma32(a.y, w.y, ii);
            }
            __syncthreads();
        }
        floatx16 uu, ud;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float ur = rr[r] - ii[r], ui = ir[r] + ri[r];
            const float dr = rr[r] + ii[r], di = ir[r] - ri[r];
            uu[r] = sqrtf(ur * ur + ui * ui);
            ud[r] = sqrtf(dr * dr + di * di);
        }
        const float* ph = Phi + (int64_t)(t0 + twv) * NTp;
#pragma unroll
        for (int n = 0; n < NTB; ++n) {
#pragma unroll
            for (int sidx = 0; sidx < 16; ++sidx) {
                const float p = ph[crow(sidx, h) * NTp + n * 32 + i32];
                vu[n] = mfma32(p, uu[sidx], vu[n]);
                vd[n] = mfma32(p, ud[sidx], vd[n]);
            }
        }
    }
    // partial V: [slot][lt][spin][tau][64 l]
    const int slot = slot0 + ch * 2 + (wave & 1);
    float* out = Vp + b * vp_bstride + ((int64_t)slot * nlt + lt) * 2 * NTp * kTileL;
#pragma unroll
    for (int n = 0; n < NTB; ++n) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int tau = n * 32 + crow(r, h);
            out[(int64_t)tau * kTileL + lw + i32] = vu[n][r];
            out[(int64_t)(NTp + tau) * kTileL + lw + i32] = vd[n][r];
        }
    }
}

// Frequency lowpass (eq. (3)): S2[b][alpha][beta][theta][m][tau] =
// sum_l PF_beta[m][l] V[theta][rowoff + l][tau], V summed over the partial slots
// of the contraction's t-chunks.  grid (n_beta ceil(NT / TT), 2 n_alpha, B), every
// temporal rate in one launch.  The l axis runs in chunks of 64: the chunk's V (64 x
// TT columns tau, its partial slots summed on the way in) and its rows of PF^T (64 x
// 32 rows m, from the transposed table PFt) are staged in LDS and multiplied by FP32
// matrix operations, 16 rows l to each of the four waves, whose sums are added at
// the end; rows m beyond 32 take further passes.  What bounded it was the chain of
// loads (row, slots, then the next element) and after that the LDS reads of vector
// multiply-adds: 84 -> 48 us for 8 signals of 2^16 samples, 141 -> 86 for 16, 453 ->
// 194 for 32 of 2^18, 5.6 -> 3.8 for one of 2^11.  The launch takes 8 or 16 columns
// a workgroup where 32 would leave under 1024 workgroups, each summing many slots one
// after the other (a whole call on one signal of 2^16 samples 428 -> 403 us); an
// output's terms keep their order.
template <int TT>
__global__ void __launch_bounds__(256) k_s2_out(const float* __restrict__ Vp, int64_t vp_bstride,
                                                const int64_t* __restrict__ vchoff, const int* __restrict__ nch,
                                                int slot_mult, int nlt, int NTp, int NT, const float* __restrict__ PFt,
                                                const int64_t* __restrict__ pfoff, const int* __restrict__ Lbv,
                                                const int* __restrict__ rowoffv, const int* __restrict__ rowpos,
                                                int NL, int NLo, int n_alpha,
                                                float* __restrict__ S2, const float* __restrict__ mu2, float eps,
                                                int n_beta) {
    // NLo <= NL output rows (the unpadded lambda axis keeps the first NLo)
    constexpr int LC = 64, MB = 32, VS = TT + 1, kUn = 64 / TT;    // kUn: 16 loads of V in flight
    __shared__ float buf[LC * VS + LC * MB > 4096 ? LC * VS + LC * MB : 4096];
    float *Vs = buf, *Ps = buf + LC * VS, *red = buf;    // red: the four waves' sums
    const int beta = blockIdx.x % n_beta, tb = (int)(blockIdx.x / n_beta) * TT;
    const int th = blockIdx.y & 1, alpha = blockIdx.y >> 1;
    const int slot0 = (int)vchoff[alpha] * slot_mult, nslots = nch[alpha] * slot_mult;
    const int64_t b = blockIdx.z;
    const int Lb = Lbv[beta], ro = rowoffv[beta];
    const float* PT = PFt + pfoff[beta];                 // Lb x NL
    const float* Vb = Vp + b * vp_bstride;
    float* o = S2 + ((((b * n_alpha + alpha) * n_beta + beta) * 2 + th) * NLo) * (int64_t)NT;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i32 = lane & 31, h = lane >> 5;
    const float inv = mulog_inv(mu2, (alpha * n_beta + beta) * 2 + th, eps);
    for (int mb = 0; mb < NLo; mb += MB) {
        floatx16 acc = zero16();
        for (int l0 = 0; l0 < Lb; l0 += LC) {
            const int lc = Lb - l0 < LC ? Lb - l0 : LC;
            // a thread's row l is the same for all its columns; every load of a slot
            // (and of PF) issues before the first is used
            const int l = threadIdx.x & 63, t4 = threadIdx.x >> 6;
            float v[TT / 4], p[LC * MB / 256];
#pragma unroll
            for (int q = 0; q < LC * MB / 256; ++q) {
                const int e = threadIdx.x + 256 * q, ll = min(e / MB, lc - 1), mm = min(mb + e % MB, NLo - 1);
                p[q] = PT[(int64_t)(l0 + ll) * NL + mm];
            }
            const int row = rowpos[ro + l0 + min(l, lc - 1)], lt = row / kTileL, lr = row % kTileL;
            const float* vs = Vb + (((int64_t)slot0 * nlt + lt) * 2 + th) * NTp * kTileL + (int64_t)(tb + t4) * kTileL + lr;
#pragma unroll
            for (int q = 0; q < TT / 4; ++q) v[q] = 0.f;
#pragma unroll kUn
            for (int sl = 0; sl < nslots; ++sl, vs += (int64_t)nlt * 2 * NTp * kTileL)
#pragma unroll
                for (int q = 0; q < TT / 4; ++q) v[q] += vs[4 * q * kTileL];
            __syncthreads();                         // the previous chunk (or pass) is read
#pragma unroll
            for (int q = 0; q < LC * MB / 256; ++q) {
                const int e = threadIdx.x + 256 * q;
                Ps[e] = e / MB < lc && mb + e % MB < NLo ? p[q] : 0.f;
            }
#pragma unroll
            for (int q = 0; q < TT / 4; ++q) Vs[l * VS + t4 + 4 * q] = l < lc && tb + t4 + 4 * q < NT ? v[q] : 0.f;
            __syncthreads();
#pragma unroll
            for (int k = 0; k < LC / 8; ++k) {
                const int l = wave * (LC / 4) + 2 * k + h;
                acc = mfma32(Ps[l * MB + i32], i32 < TT ? Vs[l * VS + i32] : 0.f, acc);
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 16; ++r) red[(wave * 16 + r) * 64 + lane] = acc[r];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = wave * 4 + q, m = mb + crow(r, h);
            const float* p = red + r * 64 + lane;
            const float a = (p[0] + p[1024]) + (p[2048] + p[3072]);
            if (m < NLo && i32 < TT && tb + i32 < NT) o[(int64_t)m * NT + tb + i32] = mulog_out(a, mu2, inv);
        }
    }
}

// Eq. (4) (no frequential lowpass): V summed over its partial slots and stored per
// (beta, theta) at rows 2 rowoff(beta) + theta Lb + l of S2[b][alpha][2 Mh][NT].
// grid (n_beta nlc ceil(NT / TT), 2 n_alpha, B), every temporal rate in one launch: 64 rows l
// (chunk of nlc) and TT frames a workgroup, the sums through LDS so that the stores
// run along the frames.  (A workgroup per scale, a load after the other and stores NT
// floats apart: one call on 3 signals of 2^15 samples with gradient 851 us, 837 now.)
template <int TT>
__global__ void __launch_bounds__(256) k_v_out(const float* __restrict__ Vp, int64_t vp_bstride,
                                               const int64_t* __restrict__ vchoff, const int* __restrict__ nch,
                                               int slot_mult, int nlt, int NTp, int NT, const int* __restrict__ Lbv,
                                               const int* __restrict__ rowoffv, const int* __restrict__ rowpos,
                                               int Mh, int n_alpha,
                                               float* __restrict__ S2, const float* __restrict__ mu2, float eps,
                                               int n_beta, int nlc) {
    constexpr int LC = 64, VS = TT + 1, kUn = 64 / TT;             // kUn: 16 loads of V in flight
    __shared__ float Vs[LC * VS];
    const int beta = blockIdx.x % n_beta, bx = (int)(blockIdx.x / n_beta);
    const int l0 = bx % nlc * LC, tb = bx / nlc * TT;
    const int th = blockIdx.y & 1, alpha = blockIdx.y >> 1;
    const int slot0 = (int)vchoff[alpha] * slot_mult, nslots = nch[alpha] * slot_mult;
    const int64_t b = blockIdx.z;
    const int Lb = Lbv[beta], ro = rowoffv[beta], lc = min(LC, Lb - l0);
    if (lc <= 0) return;
    const int l = threadIdx.x & 63, t4 = threadIdx.x >> 6;
    const int row = rowpos[ro + l0 + min(l, lc - 1)], lt = row / kTileL, lr = row % kTileL;
    const float* vs = Vp + b * vp_bstride + (((int64_t)slot0 * nlt + lt) * 2 + th) * NTp * kTileL +
                      (int64_t)(tb + t4) * kTileL + lr;
    float v[TT / 4];
#pragma unroll
    for (int q = 0; q < TT / 4; ++q) v[q] = 0.f;
#pragma unroll kUn
    for (int sl = 0; sl < nslots; ++sl, vs += (int64_t)nlt * 2 * NTp * kTileL)
#pragma unroll
        for (int q = 0; q < TT / 4; ++q) v[q] += vs[4 * q * kTileL];
#pragma unroll
    for (int q = 0; q < TT / 4; ++q) Vs[l * VS + t4 + 4 * q] = v[q];
    __syncthreads();
    float* o = S2 + ((b * n_alpha + alpha) * 2 * (int64_t)Mh + 2 * ro + th * Lb + l0) * NT + tb;
    const float inv = mulog_inv(mu2, (alpha * n_beta + beta) * 2 + th, eps);
    const int nt = min(TT, NT - tb);
    for (int e = threadIdx.x; e < lc * nt; e += 256) {
        const int ll = e / nt, tau = e - ll * nt;
        o[(int64_t)ll * NT + tau] = mulog_out(Vs[ll * VS + tau], mu2, inv);
    }
}

// Time scattering (sec. 4): S2[b][alpha][lambda][tau] = sum_t |Y2[b][alpha][lambda][t]| Phi_alpha[t][tau]
// (modulus of the second-order row, then the time lowpass on the N/T frames) as a
// product on the FP32 matrix cores: 32 rows lambda by 32 NTB frames a workgroup,
// sixteen waves sharing the columns t, their partial sums added in wave order at
// the end.  Every rate in one launch, grid (ceil(n1 / 32), B, n_alpha), the longest
// rates first.  A workgroup reads Phi_alpha once for its 32 rows (a workgroup per
// row had read it from L2 for each: 8 x 2^16 2.36 -> 0.25 ms, whose bytes take 0.11).
template <int NTB>
__global__ void __launch_bounds__(1024) k_ts_out(const float2* __restrict__ Y, int64_t y_bstride,
                                                 const FreqRate* __restrict__ rates, const float* __restrict__ Phi,
                                                 int n1, int NT, int n_alpha, float* __restrict__ S2,
                                                 const float* __restrict__ mu2, float eps) {
    constexpr int NTp = 32 * NTB;
    __shared__ float red[16 * 1024];
    const int alpha = blockIdx.z, r0 = 32 * (int)blockIdx.x;
    const int64_t b = blockIdx.y;
    const FreqRate rate = rates[alpha];
    const int Tp = rate.Tp;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, h = lane >> 5, i32 = lane & 31;
    const float4* row = (const float4*)(Y + b * y_bstride + rate.yoff + (int64_t)min(r0 + i32, n1 - 1) * Tp);
    const float* ph = Phi + rate.phioff + i32;
    floatx16 acc[NTB];
#pragma unroll
    for (int n = 0; n < NTB; ++n) acc[n] = zero16();
    // per wave eight columns t of each 128; lane half h holds columns 2 h, 2 h + 1 of every four
#pragma unroll 4
    for (int t0 = 8 * wave; t0 < Tp; t0 += 128) {
        float4 y[2];
        float p[2][2][NTB];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int t = t0 + 4 * q + 2 * h;
            y[q] = row[t >> 1];
#pragma unroll
            for (int n = 0; n < NTB; ++n) {
                p[q][0][n] = ph[(int64_t)t * NTp + 32 * n];
                p[q][1][n] = ph[(int64_t)(t + 1) * NTp + 32 * n];
            }
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const float u0 = sqrtf(y[q].x * y[q].x + y[q].y * y[q].y), u1 = sqrtf(y[q].z * y[q].z + y[q].w * y[q].w);
#pragma unroll
            for (int n = 0; n < NTB; ++n) {
                acc[n] = mfma32(u0, p[q][0][n], acc[n]);
                acc[n] = mfma32(u1, p[q][1][n], acc[n]);
            }
        }
    }
#pragma unroll
    for (int n = 0; n < NTB; ++n) {
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 16; ++r) red[wave * 1024 + r * 64 + lane] = acc[n][r];
        __syncthreads();
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < 16; ++w) sum += red[w * 1024 + tid];
        const int lam = r0 + crow(tid >> 6, h), tau = 32 * n + i32;      // register tid / 64 of lane tid % 64
        if (lam < n1 && tau < NT)
            S2[((b * n_alpha + alpha) * n1 + lam) * (int64_t)NT + tau] =
                mulog_out(sum, mu2, mulog_inv(mu2, alpha * n1 + lam, eps));
    }
}

// ---------------------------------------------------------------------------
// Backward.
// ---------------------------------------------------------------------------

// Time scattering adjoint: gY2[t] = (sum_tau gS2[tau] Phi_alpha[t][tau]) y_t / max(|y_t|, eps),
// zero for Ta <= t < Tp where Phi and y are (rows lambda < n1).  The sum runs on the
// FP32 matrix cores: 32 rows by 128 columns t a workgroup, a wave 32 columns, whose
// Phi rows it reads once for the 32 rows.  Every rate in one launch, grid (tiles of
// 128 columns, ceil(n1 / 32), B).  8 x 2^16: 1.67 -> 0.34 ms, whose bytes take 0.22.
template <int NTB>
__global__ void __launch_bounds__(256) k_ts_bwd(const float2* __restrict__ Y, int64_t y_bstride,
                                                const FreqRate* __restrict__ rates, const FreqUnit* __restrict__ tiles,
                                                const float* __restrict__ Phi, int n1, int NT, int n_alpha,
                                                const float* __restrict__ gS2, float2* __restrict__ gY, MuLogArg ml) {
    constexpr int NTp = 32 * NTB;
    const FreqUnit un = tiles[blockIdx.x];
    const FreqRate rate = rates[un.alpha];
    const int alpha = un.alpha, r0 = 32 * (int)blockIdx.y;
    const int64_t b = blockIdx.z;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, h = lane >> 5, i32 = lane & 31;
    const int t = un.t0 + 32 * wave + i32;
    const int lam = r0 + i32;                        // this lane's row of the cotangent
    const int64_t so = ((b * n_alpha + alpha) * n1 + lam) * (int64_t)NT;
    const float em = ml.mu2 && lam < n1 ? ml.eps * ml.mu2[alpha * n1 + lam] : 0.f;
    const float4* ph = (const float4*)(Phi + rate.phioff + (int64_t)t * NTp);
    floatx16 gu = zero16();
#pragma unroll
    for (int q = 0; q < 4 * NTB; ++q) {              // lane half h holds frames 8 q + 4 h .. + 3
        const float4 p4 = ph[2 * q + h];
        const float p[4] = {p4.x, p4.y, p4.z, p4.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int tau = 8 * q + 4 * h + j;
            const bool in = gS2 && lam < n1 && tau < NT;
            const float g = in ? mulog_cot(gS2[so + tau], ml.mu2, em, ml.mu2 ? ml.o2[so + tau] : 0.f) : 0.f;
            gu = mfma32(g, p[j], gu);
        }
    }
    const float2* y_ = Y + b * y_bstride + rate.yoff + t;
    float2* out = gY + b * y_bstride + rate.yoff + t;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int row = r0 + crow(r, h);
        if (row >= n1) continue;
        const float2 y = y_[(int64_t)row * rate.Tp];
        const float sc = gu[r] / fmaxf(sqrtf(y.x * y.x + y.y * y.y), kEpsMod);
        out[(int64_t)row * rate.Tp] = make_float2(y.x * sc, y.y * sc);
    }
}

// Sum over each aligned group of `width` lanes (32 or 64), returned to every lane of
// the group: rotations within rows of 16 lanes (DPP), then swaps between rows, all
// in registers (a butterfly of shuffles takes five round trips through LDS).
__device__ __forceinline__ float group_sum(float a, int width) {
    a += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(a), 0x128, 0xF, 0xF, false));   // row_ror:8
    a += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(a), 0x124, 0xF, 0xF, false));   // row_ror:4
    a += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(a), 0x122, 0xF, 0xF, false));   // row_ror:2
    a += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(a), 0x121, 0xF, 0xF, false));   // row_ror:1
    const unsigned u = __float_as_uint(a);
    const auto r16 = __builtin_amdgcn_permlane16_swap(u, u, false, false);   // rows 0+1, 2+3
    a = __uint_as_float(r16[0]) + __uint_as_float(r16[1]);
    if (width > 32) {
        const unsigned v = __float_as_uint(a);
        const auto r32 = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        a = __uint_as_float(r32[0]) + __uint_as_float(r32[1]);
    }
    return a;
}

// Eq. (4), whose gV is the gS2 row itself: gV[b][alpha][theta][slot of row l][tau] =
// gS2[b][alpha][2 rowoff + theta Lb + l][tau] (after the mu-log adjoint when set), zero
// for tau >= N/T; block n_beta of the grid (n_beta + 1, 2 n_alpha, B) zeroes the padding
// rows.  Also writes, per (signal, alpha, spin, beta), the largest row sum over tau of
// |gV| (a bound used to scale the split backward contraction): the sums of a row's
// lanes are reduced by a cross-lane sum before one LDS atomic per row segment.  LDS
// holds the Lb row sums alone.
__global__ void __launch_bounds__(256) k_s2_bwd(const float* __restrict__ gS2, const int* __restrict__ Lbv,
                                                const int* __restrict__ rowoffv, const int* __restrict__ rowpos,
                                                const int* __restrict__ pad, int n_beta, int NT, int NTp,
                                                int Mh, int Mp, int n_alpha,
                                                float* __restrict__ gV, float* __restrict__ gvmax, MuLogArg ml) {
    extern __shared__ float rowsum[];
    const int beta = blockIdx.x, th = blockIdx.y & 1, alpha = blockIdx.y >> 1;
    const int64_t b = blockIdx.z;
    float* g = gV + (((b * n_alpha + alpha) * 2 + th) * (int64_t)Mp) * NTp;
    if (beta == n_beta) {
        for (int e = threadIdx.x; e < (Mp - Mh) * NTp; e += blockDim.x) g[(int64_t)pad[e / NTp] * NTp + e % NTp] = 0.f;
        return;
    }
    const int Lb = Lbv[beta], ro = rowoffv[beta];
    const int64_t so = ((b * n_alpha + alpha) * 2 * (int64_t)Mh + 2 * ro + th * Lb) * NT;
    const float* src = gS2 ? gS2 + so : nullptr;
    const float* osrc = ml.mu2 ? ml.o2 + so : nullptr;
    const float em = ml.mu2 ? ml.eps * ml.mu2[(alpha * n_beta + beta) * 2 + th] : 0.f;
    for (int l = threadIdx.x; l < Lb; l += blockDim.x) rowsum[l] = 0.f;
    __syncthreads();
    const int width = NTp < 64 ? NTp : 64;           // lanes of one row segment within a wave
    for (int e0 = 0; e0 < Lb * NTp; e0 += blockDim.x) {
        const int e = e0 + (int)threadIdx.x;
        const bool valid = e < Lb * NTp;
        const int l = e / NTp, tau = e - l * NTp;
        float acc = 0.f;
        if (valid && src && tau < NT)
            acc = mulog_cot(src[(int64_t)l * NT + tau], ml.mu2, em, osrc ? osrc[(int64_t)l * NT + tau] : 0.f);
        if (valid) g[(int64_t)rowpos[ro + l] * NTp + tau] = acc;
        float a = fabsf(acc);
        a = group_sum(a, width);
        if (valid && (tau & (width - 1)) == 0) atomicAdd(&rowsum[l], a);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        float m = 0.f;
        for (int l = 0; l < Lb; ++l) m = fmaxf(m, rowsum[l]);
        gvmax[((b * n_alpha + alpha) * 2 + th) * n_beta + beta] = m;
    }
}

// Adjoint of the frequency lowpass of eq. (3): gV[rowoff + l][tau] =
// sum_m PF_beta[m][l] gS2[m][tau] over the NLo output rows m, with the row sums
// over tau of |gV| whose maximum sets the split scale of the backward
// contraction.  One lane per row l: the gS2 tile (after the mu-log adjoint when
// set) sits in LDS and every lane reads the same element of it at a time (a
// broadcast), PF[m][l] comes from global memory with consecutive lanes on
// consecutive l, and each lane keeps TT outputs of its row in registers, stores
// them as 16-byte writes and sums their moduli itself.  The tile holds all N/T frames
// where they fit the LDS limit, else TT of them at a time (cols), with the rows' sums
// so far in LDS behind it.  grid (n_beta + 1, 2 n_alpha, B); block n_beta zeroes the
// padding rows.
template <int TT>
__global__ void __launch_bounds__(256) k_s2_bwd_avg(const float* __restrict__ gS2, const float* __restrict__ PFall,
                                                    const int64_t* __restrict__ pfoff, const int* __restrict__ Lbv,
                                                    const int* __restrict__ rowoffv, const int* __restrict__ rowpos,
                                                    const int* __restrict__ pad, int n_beta, int NLo, int NT,
                                                    int NTp, int cols, int Mh, int Mp, int n_alpha,
                                                    float* __restrict__ gV, float* __restrict__ gvmax, MuLogArg ml) {
    extern __shared__ __align__(16) float st[];      // gS2 tile [NLo][cols] | (cols < NT) sums [Lb]
    __shared__ float red[256];
    const int beta = blockIdx.x, th = blockIdx.y & 1, alpha = blockIdx.y >> 1;
    const int64_t b = blockIdx.z;
    float* g = gV + (((b * n_alpha + alpha) * 2 + th) * (int64_t)Mp) * NTp;
    if (beta == n_beta) {
        for (int e = threadIdx.x; e < (Mp - Mh) * NTp; e += blockDim.x) g[(int64_t)pad[e / NTp] * NTp + e % NTp] = 0.f;
        return;
    }
    const int Lb = Lbv[beta], ro = rowoffv[beta];
    const float* PF = PFall + pfoff[beta];           // [NL][Lb]
    const int64_t so = ((((b * n_alpha + alpha) * n_beta + beta) * 2 + th) * NLo) * (int64_t)NT;
    const float* src = gS2 ? gS2 + so : nullptr;
    const float* osrc = ml.mu2 ? ml.o2 + so : nullptr;
    const float em = ml.mu2 ? ml.eps * ml.mu2[(alpha * n_beta + beta) * 2 + th] : 0.f;
    float* sums = st + NLo * cols;
    float mx = 0.f;
    for (int c0 = 0; c0 < NT; c0 += cols) {
        const bool last = c0 + cols >= NT;
        if (c0) __syncthreads();                     // the tile before is read
        for (int e = threadIdx.x; e < NLo * cols; e += blockDim.x) {
            const int i = cols == NT ? e : e / cols * NT + c0 + e % cols;
            st[e] = src ? mulog_cot(src[i], ml.mu2, em, osrc ? osrc[i] : 0.f) : 0.f;
        }
        __syncthreads();
        for (int l = threadIdx.x; l < Lb; l += blockDim.x) {
            float* grow = g + (int64_t)rowpos[ro + l] * NTp;
            float rs = c0 ? sums[l] : 0.f;
            for (int t0 = c0; t0 < (last ? NTp : c0 + cols); t0 += TT) {
                float acc[TT];
#pragma unroll
                for (int j = 0; j < TT; ++j) acc[j] = 0.f;
                if (t0 < NT) {
                    if (NT - t0 >= TT) {
                        for (int m = 0; m < NLo; ++m) {
                            const float p = PF[(int64_t)m * Lb + l];
                            const float4* s4 = (const float4*)(st + m * cols + t0 - c0);
#pragma unroll
                            for (int q = 0; q < TT / 4; ++q) {
                                const float4 v = s4[q];
                                acc[4 * q] += p * v.x;
                                acc[4 * q + 1] += p * v.y;
                                acc[4 * q + 2] += p * v.z;
                                acc[4 * q + 3] += p * v.w;
                            }
                        }
                    } else {
                        for (int m = 0; m < NLo; ++m) {
                            const float p = PF[(int64_t)m * Lb + l];
#pragma unroll
                            for (int j = 0; j < TT; ++j)
                                if (t0 + j < NT) acc[j] += p * st[m * cols + t0 - c0 + j];
                        }
                    }
                }
                float4* o4 = (float4*)(grow + t0);
#pragma unroll
                for (int q = 0; q < TT / 4; ++q) {
                    o4[q] = make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
                    rs += fabsf(acc[4 * q]) + fabsf(acc[4 * q + 1]) + fabsf(acc[4 * q + 2]) + fabsf(acc[4 * q + 3]);
                }
            }
            if (last) mx = fmaxf(mx, rs);
            else sums[l] = rs;                       // (this thread's row in every pass)
        }
    }
    red[threadIdx.x] = mx;
    __syncthreads();
    for (int w = blockDim.x / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0) gvmax[((b * n_alpha + alpha) * 2 + th) * n_beta + beta] = red[0];
}

// Recompute Z = W Y (both spins) on a 64 l x 64 t tile, gU = gV Phi^T (adjoint of
// the time lowpass), gZ = gU Z / max(|Z|, eps) (modulus adjoint), and store
// P = gZ_up + gZ_down and Q' = i (gZ_down - gZ_up), so that the adjoint of the
// contraction is gY = Wr^T P + Wi^T Q'.  Non-transposed orientation: C rows = l.
template <int NTB>
__global__ void __launch_bounds__(256) k_bwd_pq(const float2* __restrict__ Y, int64_t y_bstride, int Tp,
                                                const float2* __restrict__ Wt, int Mp, int Kp,
                                                const float* __restrict__ Phi, const float* __restrict__ gV,
                                                int64_t gv_bstride, float2* __restrict__ PQ) {
    constexpr int NTp = 32 * NTB;
    constexpr int LDG = NTp + 1;
    __shared__ float2 Ys[kKStep][kTileT];
    __shared__ float2 Ws[kKStep][kTileL];
    __shared__ float gVs[2][kTileL][LDG];
    __shared__ float Phs[kTileT][LDG];
    const int lt = blockIdx.x, tt = blockIdx.y;
    const int64_t b = blockIdx.z;
    const int l0 = lt * kTileL, t0 = tt * kTileT;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int h = lane >> 5, i32 = lane & 31;
    const int lw = (wave >> 1) * 32, twv = (wave & 1) * 32;
    const float2* Yb = Y + b * y_bstride;
    const float* gvb = gV + b * gv_bstride;
    for (int e = tid; e < kTileL * NTp; e += 256) {
        const int l = e / NTp, tau = e - l * NTp;
        gVs[0][l][tau] = gvb[(int64_t)(l0 + l) * NTp + tau];
        gVs[1][l][tau] = gvb[(int64_t)(Mp + l0 + l) * NTp + tau];
        Phs[l][tau] = Phi[(int64_t)(t0 + l) * NTp + tau];
    }
    floatx16 rr = zero16(), ri = zero16(), ir = zero16(), ii = zero16();
    for (int k0 = 0; k0 < Kp; k0 += kKStep) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int f = tid + q * 256, row = f >> 5, c = (f & 31) * 2;
            *(float4*)&Ys[row][c] = *(const float4*)(Yb + (int64_t)(k0 + row) * Tp + t0 + c);
            *(float4*)&Ws[row][c] = *(const float4*)(Wt + (int64_t)(k0 + row) * Mp + l0 + c);
        }
        __syncthreads();
#pragma unroll
        for (int ks = 0; ks < kKStep / 2; ++ks) {
            const float2 w = Ws[2 * ks + h][lw + i32];   // A: rows l
            const float2 y = Ys[2 * ks + h][twv + i32];  // B: columns t
            rr = mfma32(w.x, y.x, rr);
            ri = mfma32(w.x, y.y, ri);
            ir = mfma32(w.y, y.x, ir);
            ii = mfma32(w.y, y.y, ii);
        }
        __syncthreads();
    }
    floatx16 gu = zero16(), gd = zero16();
#pragma unroll
    for (int n = 0; n < NTB; ++n) {
#pragma unroll
        for (int sidx = 0; sidx < 16; ++sidx) {
            const int tau = n * 32 + 2 * sidx + h;
            const float p = Phs[twv + i32][tau];
            gu = mfma32(gVs[0][lw + i32][tau], p, gu);
            gd = mfma32(gVs[1][lw + i32][tau], p, gd);
        }
    }
    float2* Pp = PQ + b * (2 * (int64_t)Mp * Tp);
    float2* Qp = Pp + (int64_t)Mp * Tp;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const float ur = rr[r] - ii[r], ui = ri[r] + ir[r];
        const float dr = rr[r] + ii[r], di = ri[r] - ir[r];
        const float su = gu[r] / fmaxf(sqrtf(ur * ur + ui * ui), kEpsMod);
        const float sd = gd[r] / fmaxf(sqrtf(dr * dr + di * di), kEpsMod);
        const float gur = su * ur, gui = su * ui, gdr = sd * dr, gdi = sd * di;
        const int l = l0 + lw + crow(r, h), t = t0 + twv + i32;
        Pp[(int64_t)l * Tp + t] = make_float2(gur + gdr, gui + gdi);
        Qp[(int64_t)l * Tp + t] = make_float2(-(gdi - gui), gdr - gur);
    }
}

// gY[i][t] = sum_l Wr[l][i] P[l][t] + Wi[l][i] Q'[l][t]  (adjoint of the contraction)
__global__ void __launch_bounds__(256) k_bwd_gy(const float2* __restrict__ PQ, int Tp, const float2* __restrict__ Wl,
                                                int Mp, int Kp, float2* __restrict__ gY, int64_t gy_bstride) {
    __shared__ float As[kKStep][kTileL];
    __shared__ float2 Bs[kKStep][kTileT];
    const int it = blockIdx.x, tt = blockIdx.y;
    const int64_t b = blockIdx.z;
    const int i0 = it * 64, t0 = tt * kTileT;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int h = lane >> 5, i32 = lane & 31;
    const int iw = (wave >> 1) * 32, twv = (wave & 1) * 32;
    const float2* PQb = PQ + b * (2 * (int64_t)Mp * Tp);
    floatx16 are = zero16(), aim = zero16();
    for (int plane = 0; plane < 2; ++plane) {
        const float2* Bsrc = PQb + (int64_t)plane * Mp * Tp;
        for (int k0 = 0; k0 < Mp; k0 += kKStep) {
            for (int e = tid; e < kKStep * 64; e += 256) {
                const int row = e >> 6, c = e & 63;
                float v = 0.f;
                if (i0 + c < Kp) {
                    const float2 w = Wl[(int64_t)(k0 + row) * Kp + i0 + c];
                    v = plane ? w.y : w.x;
                }
                As[row][c] = v;
            }
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int f = tid + q * 256, row = f >> 5, c = (f & 31) * 2;
                *(float4*)&Bs[row][c] = *(const float4*)(Bsrc + (int64_t)(k0 + row) * Tp + t0 + c);
            }
            __syncthreads();
#pragma unroll
            for (int ks = 0; ks < kKStep / 2; ++ks) {
                const float a = As[2 * ks + h][iw + i32];
                const float2 v = Bs[2 * ks + h][twv + i32];
                are = mfma32(a, v.x, are);
                aim = mfma32(a, v.y, aim);
            }
            __syncthreads();
        }
    }
    float2* o = gY + b * gy_bstride;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int i = i0 + iw + crow(r, h), t = t0 + twv + i32;
        if (i < Kp) o[(int64_t)i * Tp + t] = make_float2(are[r], aim[r]);
    }
}

// Adjoint of the second order and of S1 for one scalogram row: accumulates the
// Hermitian half-spectrum of gX,
//   H[m] = 1/2 sum_alpha psi_hat_alpha[m] G_alpha[m mod Ta] (real part at m = 0, NX/2)
//        + phi_hat[m] G1[m mod NT],
// G_alpha = FFT of gY2 rows (done beforehand), G1 = FFT of gS1 row, then the
// real inverse FFT gives gX[b][lambda][0..NX) (scaled 1/NX).
__global__ void __launch_bounds__(1024, 8) k_scal_bwd_a(const float2* __restrict__ G, int64_t y_bstride,
                                                    const int64_t* __restrict__ yoff, const int* __restrict__ Tpv,
                                                    const int* __restrict__ Tav, const float* __restrict__ psi2,
                                                    const int* __restrict__ band2, const int64_t* __restrict__ off2,
                                                    int n_alpha, const float* __restrict__ gS1,
                                                    const float* __restrict__ phiX, int Mphi, int logNT, int logNX,
                                                    float* __restrict__ gX, const float2* __restrict__ tw, int tw_log,
                                                    MuLogArg ml, const float2* __restrict__ gYphi, int Tphi) {
    extern __shared__ float2 s[];
    const int lam = blockIdx.x, n1 = gridDim.x;
    const int64_t b = blockIdx.y;
    const int NX = 1 << logNX, H = NX >> 1, NT = 1 << logNT;
    float2* g1 = s + lpad(H) + 1;
    const float em = ml.mu1 ? ml.eps * ml.mu1[0] : 0.f;
    for (int t = threadIdx.x; t < NT; t += blockDim.x) {
        const int64_t i = (b * n1 + lam) * NT + t;
        float g = gS1 ? mulog_cot(gS1[i], ml.mu1, em, ml.mu1 ? ml.o1[i] : 0.f) : 0.f;
        if (gYphi) g += gYphi[b * y_bstride + (int64_t)lam * Tphi + t].x;   // Re of phi_T's second-order rows
        g1[lpad(t)] = make_float2(g, 0.f);
    }
    __syncthreads();
    lds_fft<16>(g1, logNT, 1, NT, tw, tw_log, false);
    // bins m = m0 + tid + q blockDim, q < 5: the temporal rates in the outer loop,
    // so that a rate's loads for all of a thread's bins issue together
    for (int m0 = 0; m0 <= H; m0 += 5 * (int)blockDim.x) {
        float2 c[5];
#pragma unroll
        for (int q = 0; q < 5; ++q) c[q] = make_float2(0.f, 0.f);
        for (int a = 0; a < n_alpha; ++a) {
            const int lo = band2[2 * a], hi = band2[2 * a + 1];
            const float* pa = psi2 + off2[a] - lo;
            const float2* ga = G + b * y_bstride + yoff[a] + (int64_t)lam * Tpv[a];
            const int tmask = Tav[a] - 1;
#pragma unroll
            for (int q = 0; q < 5; ++q) {
                const int m = m0 + threadIdx.x + q * blockDim.x;
                if (m >= lo && m <= hi) {
                    const float g = pa[m];
                    const float2 v = ga[m & tmask];
                    c[q].x += g * v.x;
                    c[q].y += g * v.y;
                }
            }
        }
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            const int m = m0 + threadIdx.x + q * blockDim.x;
            if (m > H) continue;
            float2 hm = (m == 0 || m == H) ? make_float2(c[q].x, 0.f) : cscale(c[q], 0.5f);
            if (m <= Mphi) {
                const float2 v = g1[lpad(m & (NT - 1))];
                hm.x += phiX[m] * v.x;
                hm.y += phiX[m] * v.y;
            }
            s[lpad(m)] = hm;
        }
    }
    __syncthreads();
    const int tws = tw_log - logNX;
    for (int k = threadIdx.x; k <= H / 2; k += blockDim.x) {
        const float2 p = s[lpad(k)], q = s[lpad(H - k)];
        auto pk = [&](float2 pp, float2 qq, int kk) {
            const float2 S = make_float2(pp.x + qq.x, pp.y - qq.y);
            const float2 D = make_float2(pp.x - qq.x, pp.y + qq.y);
            const float2 wD = cmulc(D, tw[kk << tws]);
            return make_float2(S.x - wD.y, S.y + wD.x);
        };
        const float2 zk = pk(p, q, k);
        float2 zn = make_float2(0.f, 0.f);
        const bool two = k > 0 && H - k != k;
        if (two) zn = pk(q, p, H - k);
        s[lpad(k)] = zk;
        if (two) s[lpad(H - k)] = zn;
    }
    __syncthreads();
    if (logNX > 1) lds_fft<16>(s, logNX - 1, 1, H, tw, tw_log, true);
    float2* o = (float2*)(gX + (b * n1 + lam) * (int64_t)NX);
    const float sc = 1.f / (float)NX;
    for (int k = threadIdx.x; k < H; k += blockDim.x) o[k] = cscale(s[lpad(k)], sc);
}

// Adjoint of the modulus and of the first-order filter for one row: recompute the
// scalogram-rate filtered signal y, gY1 = gX y / max(|y|, eps), and its FFT
// (the spectrum that the decimation adjoint replicates): g1[b][lambda][0..NX).
__global__ void __launch_bounds__(1024, 8) k_scal_bwd_b(const float2* __restrict__ xh, int64_t xh_pitch,
                                                    const float* __restrict__ psi1, const int* __restrict__ band1,
                                                    const int64_t* __restrict__ off1, const float* __restrict__ gX,
                                                    float2* __restrict__ g1, int logNX, float invN,
                                                    const float2* __restrict__ tw, int tw_log) {
    extern __shared__ float2 s[];
    const int lam = blockIdx.x, n1 = gridDim.x;
    const int64_t b = blockIdx.y;
    const int NX = 1 << logNX;
    fold_band(s, xh + b * xh_pitch, psi1 + off1[lam], band1[2 * lam], band1[2 * lam + 1], logNX);
    __syncthreads();
    lds_fft<16>(s, logNX, 1, NX, tw, tw_log, true);
    const float* gx = gX + (b * n1 + lam) * (int64_t)NX;
    for (int n = threadIdx.x; n < NX; n += blockDim.x) {
        const float2 y = cscale(s[lpad(n)], invN);
        const float sc = gx[n] * __builtin_amdgcn_rcpf(fmaxf(__builtin_amdgcn_sqrtf(y.x * y.x + y.y * y.y), kEpsMod));
        s[lpad(n)] = cscale(y, sc);
    }
    __syncthreads();
    lds_fft<16>(s, logNX, 1, NX, tw, tw_log, false);
    float2* o = g1 + (b * n1 + lam) * (int64_t)NX;
    for (int n = threadIdx.x; n < NX; n += blockDim.x) o[n] = s[lpad(n)];
}

// Band-owned accumulation of the first-order adjoint over lambda for bins
// 0..N/2: K[m] = sum_lambda psi_hat_lambda[m] g1_lambda[m mod NX]; writes the
// Hermitian half-spectrum of gx (K/2, real part at m = 0 and N/2).
__global__ void __launch_bounds__(256) k_band_accum(const float2* __restrict__ g1, int n1, int logNX,
                                                    const float* __restrict__ psi1, const int* __restrict__ band1,
                                                    const int64_t* __restrict__ off1,
                                                    const int* __restrict__ lam_range, int Hn,
                                                    float2* __restrict__ gxh, int64_t pitch) {
    const int r = blockIdx.x;
    const int64_t b = blockIdx.y;
    const int m = r * 256 + threadIdx.x;
    if (m > Hn) return;
    const int la = lam_range[2 * r], lb = lam_range[2 * r + 1];
    const int mask = (1 << logNX) - 1;
    float2 k = make_float2(0.f, 0.f);
    for (int lam = la; lam <= lb; ++lam) {
        const int lo = band1[2 * lam], hi = band1[2 * lam + 1];
        if (m < lo || m > hi) continue;
        const float g = psi1[off1[lam] + m - lo];
        const float2 v = g1[(b * n1 + lam) * (int64_t)(mask + 1) + (m & mask)];
        k.x += g * v.x;
        k.y += g * v.y;
    }
    gxh[b * pitch + m] = (m == 0 || m == Hn) ? make_float2(k.x, 0.f) : cscale(k, 0.5f);
}

// ---------------------------------------------------------------------------
// Launch helpers
// ---------------------------------------------------------------------------
static bool g_attr_done = false;

int setup_kernel_attributes() {
    if (g_attr_done) return JTFS_OK;
    const int lds = kMaxDynLds;
    const void* ks[] = {(const void*)k_fft_cols_t<float2, float2>, (const void*)k_fft_cols_t<float2, float2, true>, (const void*)k_fft_cols_t<float2, double2>,
                        (const void*)k_fft_cols_t<double2, double2>, (const void*)k_scalogram, (const void*)k_rfft64_rows, (const void*)k_irfft_rows,
                        (const void*)k_s2_bwd_avg<16>, (const void*)k_s2_bwd_avg<32>,
                        (const void*)k_second_order, (const void*)k_rowfft_short, (const void*)k_scal_bwd_a, (const void*)k_scal_bwd_b};
    for (const void* k : ks) {
        hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) {
            set_error(std::string("hipFuncSetAttribute: ") + hipGetErrorString(e));
            return JTFS_EHIP;
        }
    }
    int rs = split_attributes();
    if (rs != JTFS_OK) return rs;
    rs = reg_attributes();
    if (rs != JTFS_OK) return rs;
    g_attr_done = true;
    return JTFS_OK;
}

// Rows of more than 2^kOneRowLog complex points are transformed in four steps: in one
// launch, a workgroup per row, the output of 3 signals of 2^15 samples kept 3 of the 256
// CUs busy for 26 us (844 us in all, 824 now).  By the length alone, so that a signal's
// bits do not depend on its batch: up to 64 rows the steps are the faster ones (input and
// output transform of 2^14 samples, one launch and four steps, us: 1 signal 47 and 31, 16
// 51 and 38, 64 53 and 53), and a batch with a row for every CU loses by them what is
// little beside the rest (256: 70 and 110, of 15.7 ms forward and gradient).
constexpr int kOneRowLog = 11;

// Columns (log2) a workgroup of the four-step takes of 2^logcols transforms of 2^loglen
// points, B times: 4096 points, but down to four columns (runs of 32 bytes, 64 in FP64)
// while the launch holds under 256 workgroups (one signal of 2^16 samples had 8: 364 us
// in all, 355 now).
static int step_cols(int loglen, int logcols, int64_t B) {
    int logC = std::min(std::max(0, 12 - loglen), logcols);
    while (logC > 2 && ((int64_t)1 << (logcols - logC)) * B < 256) --logC;
    return logC;
}
static dim3 step_threads(int logpoints) { return dim3((unsigned)std::min(1024, std::max(256, 1 << logpoints >> 2))); }

// Real rows of 2 H = 2^(logn+1) samples, H beyond one LDS transform, from their half
// spectra (pitch ip): the packed spectrum's inverse FFT, four-step through scratch
// (pitch H).
static void irfft_four_step(const float2* in, int64_t ip, float2* out, float2* scratch, int logn, int64_t B, float scale,
                            const jtfs_plan* P, hipStream_t st) {
    // n = P Q: input index a + P*bq (a < P columns, bq < Q), output k_b + Q*k_a
    const int lq = (logn + 1) / 2, lp = logn - lq;
    const int64_t Pn = (int64_t)1 << lp, Qn = (int64_t)1 << lq, n = (int64_t)1 << logn;
    int logC = step_cols(lq, lp, B);
    size_t lds = (size_t)(1 << logC) * (lpad_len(Qn) + 1) * sizeof(float2);
    hipLaunchKernelGGL((k_fft_cols_t<float2, float2, true>), dim3((unsigned)(Pn >> logC), (unsigned)B),
                       step_threads(lq + logC), lds, st, in, scratch, lq, (int)Pn, logC, ip, Pn, n, Qn,
                       (int64_t)1, logn, P->tw, P->tw_log, 1, 1.0f);
    logC = step_cols(lp, lq, B);
    lds = (size_t)(1 << logC) * (lpad_len(Pn) + 1) * sizeof(float2);
    hipLaunchKernelGGL((k_fft_cols_t<float2, float2>), dim3((unsigned)(Qn >> logC), (unsigned)B), step_threads(lp + logC), lds, st, scratch,
                       out, lp, (int)Qn, logC, n, Qn, n, (int64_t)1, Qn, 0, P->tw, P->tw_log, 1, scale);
}

// Real FFT of the B input rows (N samples) in FP64: the complex FFT of the N/2
// interleaved pairs (one LDS transform up to 2^kOneRowLog points, four-step above),
// then the real-spectrum post-pass, which rounds each bin once to FP32.  Every later stage works on
// bands of x_hat, so the only transform that mixes all bands keeps its error
// below FP32 rounding of each bin (not of the whole spectrum).
static void input_fft64(const float* x, int64_t B, float2* xh, int64_t xh_pitch, double2* scratch, double2* z,
                        const jtfs_plan* P, hipStream_t st) {
    const int logn = P->s.logN - 1;
    const int64_t H = (int64_t)1 << logn;
    const float2* in = (const float2*)x;
    if (logn <= kOneRowLog) {
        const int logC = 12 - logn;
        const size_t lds = (size_t)(1 << logC) * (lpad_len(H) + 1) * sizeof(double2);
        hipLaunchKernelGGL(k_rfft64_rows, dim3((unsigned)((B + (1 << logC) - 1) >> logC)), dim3(1024), lds, st, in, (int)B,
                           logn, logC, xh, xh_pitch, P->tw64, P->tw_log);
        return;
    }
    const int lq = (logn + 1) / 2, lp = logn - lq;
    const int64_t Pn = (int64_t)1 << lp, Qn = (int64_t)1 << lq;
    int logC = step_cols(lq, lp, B);
    size_t lds = (size_t)(1 << logC) * (lpad_len(Qn) + 1) * sizeof(double2);
    hipLaunchKernelGGL((k_fft_cols_t<float2, double2>), dim3((unsigned)(Pn >> logC), (unsigned)B), step_threads(lq + logC),
                       lds, st, in, scratch, lq, (int)Pn, logC, H, Pn, H, Qn, (int64_t)1, logn, P->tw64,
                       P->tw_log, 0, 1.0);
    logC = step_cols(lp, lq, B);
    lds = (size_t)(1 << logC) * (lpad_len(Pn) + 1) * sizeof(double2);
    hipLaunchKernelGGL((k_fft_cols_t<double2, double2>), dim3((unsigned)(Qn >> logC), (unsigned)B), step_threads(lp + logC),
                       lds, st, scratch, z, lp, (int)Qn, logC, H, Qn, H, (int64_t)1, Qn, 0, P->tw64,
                       P->tw_log, 0, 1.0);
    hipLaunchKernelGGL(k_rfft_post64, dim3((unsigned)((H / 2 + 1 + 255) / 256), (unsigned)B), dim3(256), 0, st, z, H,
                       xh, xh_pitch, P->s.logN, P->tw64, P->tw_log);
}

}  // namespace jtfs

using namespace jtfs;

#define LAUNCHCHK(what)                                                                  \
    do {                                                                                 \
        hipError_t e_ = hipGetLastError();                                               \
        if (e_ != hipSuccess) {                                                          \
            set_error(std::string(what) + ": " + hipGetErrorString(e_));                 \
            return JTFS_EHIP;                                                            \
        }                                                                                \
    } while (0)

// Whether the backward of the plan's contraction mode runs on the split kernels
// (else the FP32 pair, which keeps P and Q' in the workspace).
static bool split_backward(const jtfs_plan* P) {
    if (P->contraction == JTFS_CONTRACTION_FP32 || P->s.tscat) return false;
    return P->contraction == JTFS_CONTRACTION_SPLIT_F16_PHASE ? P->split_bwdp_ok : P->split_bwd_ok;
}

// Workspace of a plan in its current contraction mode.
static Workspace plan_layout(const jtfs_plan* P, int64_t B) {
    const bool split = P->contraction != JTFS_CONTRACTION_FP32;          // SPLIT_F16 or SPLIT_F16_PHASE
    const bool phase = P->contraction == JTFS_CONTRACTION_SPLIT_F16_PHASE && !P->s.tscat;
    return layout(P->s, B, split, !(split && split_backward(P)), phase, split ? split_chunks(P).sumch : 2 * P->s.sumch);
}

// forward_only: a forward needs the leading part of the layout only
static int check_common(const jtfs_plan* P, int64_t B, void* ws, size_t ws_bytes, bool forward_only) {
    if (!P) { set_error("null plan"); return JTFS_EINVAL; }
    if (B < 1 || B > 65535) { set_error("B must lie in [1, 65535]"); return JTFS_ESHAPE; }   // grid y / z
    if (!ws) { set_error("null workspace"); return JTFS_EINVAL; }
    const Workspace w = plan_layout(P, B);
    if (ws_bytes < (forward_only ? w.fwd_total : w.total)) { set_error("workspace too small"); return JTFS_EWORKSPACE; }
    return JTFS_OK;
}

extern "C" int jtfs_workspace_size(const jtfs_plan* P, int64_t B, size_t* bytes) {
    if (!P || !bytes) { set_error("null pointer"); return JTFS_EINVAL; }
    if (B < 1) { set_error("B must be >= 1"); return JTFS_ESHAPE; }
    *bytes = plan_layout(P, B).total;
    return JTFS_OK;
}

extern "C" int jtfs_forward_workspace_size(const jtfs_plan* P, int64_t B, size_t* bytes) {
    if (!P || !bytes) { set_error("null pointer"); return JTFS_EINVAL; }
    if (B < 1) { set_error("B must be >= 1"); return JTFS_ESHAPE; }
    *bytes = plan_layout(P, B).fwd_total;
    return JTFS_OK;
}

namespace {

// whether rows of 2^logn points take the register-resident transform (2^11 to 2^13 with the choice of 2^14)
bool reg_row(int logn, bool knob) {
    return use_reg_rows(logn, knob) || (logn >= kRegMinLogRows - 3 && logn < kRegMinLogRows && knob);
}

// The next launch over `nrows` rows of each rate from *a on that is transformed in
// LDS (false where none is left).  Rows per workgroup: what fills its LDS (4096 or
// 8192 points), at most max_rows, and fewer where the launch would hold under about
// 1024 workgroups.  A launch's workgroups all ask for the LDS of its longest rate (147 KB
// for rows of 2^14 points); with launches of their own for such rates, 8 x 2^16 with all
// rows in LDS took 465 us for the second order instead of 483, but 555 for the row FFTs
// instead of 490.
bool short_rates(const jtfs_plan* P, bool knob, int* a, int nrows, int max_rows, int64_t B, ShortRates* sr,
                 unsigned* blocks, size_t* lds) {
    const Shapes& s = P->s;
    sr->n = 0;
    for (; *a < s.n_alpha_psi && sr->n < kMaxShort; ++*a)
        if (!reg_row(s.logNX - s.k2[*a], knob)) sr->r[sr->n++].alpha = *a;
    if (!sr->n) return false;
    const int fill = (int)std::min<int64_t>(1 << 20, std::max<int64_t>(1, ((int64_t)nrows * sr->n * B + 1023) / 1024));
    unsigned blk = 0;
    *lds = 0;
    for (int q = 0; q < sr->n; ++q) {
        const int al = sr->r[q].alpha, logTa = s.logNX - s.k2[al];
        const int rows = std::min({max_rows, std::max(1, (1 << lds_batch_log(P->tune)) >> logTa), fill});
        sr->blk0[q] = (int)blk;
        sr->r[q] = ShortRate{s.yoff[al], s.f2.off[al], s.f2.lo[al], s.f2.hi[al], logTa, s.Tp[al], rows, al};
        blk += (unsigned)((nrows + rows - 1) / rows);
        *lds = std::max(*lds, sizeof(float2) * rows * (lpad_len(s.Ta[al]) + 1));
    }
    *blocks = blk;
    return true;
}

// x -> x_hat -> X_hat -> S1, Y2
int forward_front(const jtfs_plan* P, const float* x, int64_t B, float* s1, char* base, const Workspace& w,
                  const MuLogArg& ml, hipStream_t st) {
    const Shapes& s = P->s;
    float2* xh = (float2*)(base + w.xh);
    float2* Xh = (float2*)(base + w.Xh);
    float2* Y2 = (float2*)(base + w.Y2);
    JTFS_TIMED(JTFS_STAGE_INPUT_FFT, st, input_fft64(x, B, xh, w.xh_pitch, (double2*)(base + w.tmp64),
                                                     (double2*)(base + w.z64), P, st));
    LAUNCHCHK("input FFT");
    if (use_reg_rows(s.logNX, P->tune.reg_scalogram)) {
        JTFS_TIMED(JTFS_STAGE_SCALOGRAM, st, launch_scalogram_r(P, xh, w.xh_pitch, Xh, w.Xh_pitch, B, st));
    } else {
        JTFS_TIMED(JTFS_STAGE_SCALOGRAM, st, hipLaunchKernelGGL(k_scalogram, dim3(s.n1, (unsigned)B), dim3(1024), sizeof(float2) * lpad_len(s.NX), st, xh, w.xh_pitch,
                       P->psi1, P->band1, P->off1, Xh, w.Xh_pitch, s.logNX, 1.0f / (float)s.N, P->tw, P->tw_log));
    }
    LAUNCHCHK("scalogram");
    for (int a = 0; a < s.n_alpha_psi; ++a) {
        if (!reg_row(s.logNX - s.k2[a], P->tune.reg_second)) continue;
        JTFS_TIMED(JTFS_STAGE_SECOND_ORDER, st,
                   launch_second_order_r(P, a, Xh, w.Xh_pitch, Y2, (float*)(base + w.rowmax), B, st));
        LAUNCHCHK("second order");
    }
    // the rates transformed in LDS, and S1 with the first of their launches
    const int aphi = s.n_alpha_psi, nrow1 = s.complete ? s.Kp : s.n1;
    S1Rows sa = {};
    if (s1 || s.complete) {
        sa.rows = std::max(1, std::min(32, 1024 / s.NT));
        sa.Mphi = s.Mphi;
        sa.logNX = s.logNX;
        sa.logNT = s.logN - s.logT;
        sa.Tp = s.complete ? s.Tp[aphi] : 0;
        sa.alpha = aphi;
        sa.eps = ml.eps;
        sa.phiX = P->phiX;
        sa.mu1 = ml.mu1;
        sa.S1 = s1;
        sa.Yphi = s.complete ? Y2 + s.yoff[aphi] : nullptr;
    }
    ShortRates sr;
    size_t lds = 0;
    unsigned blocks = 0;
    for (int a = 0;;) {
        if (!short_rates(P, P->tune.reg_second, &a, s.Kp, 64, B, &sr, &blocks, &lds)) blocks = 0, lds = 0;
        sa.blk0 = (int)blocks;
        if (sa.rows) {
            blocks += (unsigned)((nrow1 + sa.rows - 1) / sa.rows);
            lds = std::max(lds, sizeof(float2) * sa.rows * lpad_len(s.NT));
        }
        if (!blocks) break;
        JTFS_TIMED(JTFS_STAGE_SECOND_ORDER, st, hipLaunchKernelGGL(k_second_order, dim3(blocks, (unsigned)B), dim3(1024), lds, st,
                           Xh, w.Xh_pitch, s.n1, P->psi2, sr, sa, s.Kp, Y2, (int64_t)s.Kp * s.sumTp, 1.0f / (float)s.NX,
                           P->tw, P->tw_log, (float*)(base + w.rowmax), s.n_alpha));
        LAUNCHCHK("second order and first-order lowpass");
        sa.rows = 0;
    }
    return JTFS_OK;
}

int forward_impl(const jtfs_plan* P, const float* x, int64_t B, float* s1, float* s2, void* ws, size_t ws_bytes,
                 const MuLogArg& ml, hipStream_t st) {
    int rc = check_common(P, B, ws, ws_bytes, true);
    if (rc != JTFS_OK) return rc;
    if (!x || !s1 || !s2) { set_error("null pointer"); return JTFS_EINVAL; }
    const Shapes& s = P->s;
    const Workspace w = plan_layout(P, B);
    char* base = (char*)ws;
    rc = forward_front(P, x, B, s1, base, w, ml, st);
    if (rc != JTFS_OK) return rc;
    float2* Y2 = (float2*)(base + w.Y2);
    float* Vp = (float*)(base + w.Vp);
    const int nlt = s.Mp / kTileL;
    if (s.tscat) {
        // every temporal rate in one launch (N/T <= 128: one, two or four blocks of 32 frames)
        auto k = s.NTp == 32 ? k_ts_out<1> : s.NTp == 64 ? k_ts_out<2> : k_ts_out<4>;
        JTFS_TIMED(JTFS_STAGE_FREQ_FWD, st, hipLaunchKernelGGL(k, dim3((unsigned)((s.n1 + 31) / 32), (unsigned)B, (unsigned)s.n_alpha), dim3(1024), 0, st,
                           Y2, (int64_t)s.Kp * s.sumTp, P->d_rates, P->Phi, s.n1, s.NT, s.n_alpha, s2, ml.mu2, ml.eps));
        LAUNCHCHK("time-scattering lowpass");
    }
    const bool split = P->contraction != JTFS_CONTRACTION_FP32 && !s.tscat;
    unsigned* phase = P->contraction == JTFS_CONTRACTION_SPLIT_F16_PHASE && !s.tscat ? (unsigned*)(base + w.phase) : nullptr;
    if (split) {
        unsigned short* Yh = (unsigned short*)(base + w.Yh);
        float* ysc = (float*)(base + w.yscale);
        JTFS_TIMED(JTFS_STAGE_OPERAND_SPLIT, st,
                   rc = launch_ysplit(P, Y2, (const float*)(base + w.rowmax), Yh, ysc, B, st));
        if (rc != JTFS_OK) { set_error("operand split kernel failed"); return rc; }
        JTFS_TIMED(JTFS_STAGE_FREQ_FWD, st,
                   rc = launch_freq_fwd_split(P, Yh, ysc, Vp, w.vp_bstride, phase, w.ph_bstride, B, st));
        if (rc != JTFS_OK) { if (rc == JTFS_EHIP) set_error("split contraction launch failed"); return rc; }
    }
    for (int a = 0; a < s.n_alpha && !split && !s.tscat; ++a) {
        dim3 grid(nlt, s.nch[a], (unsigned)B);
        const int slot0 = (int)s.vchoff[a] * 2;
        const float2* Ya = Y2 + s.yoff[a];
        const float* Ph = P->Phi + s.phioff[a];
        const int64_t yb = (int64_t)s.Kp * s.sumTp;
        {
        TimedLaunch tl_fwd(JTFS_STAGE_FREQ_FWD, st);
        switch (s.NTp / 32) {
            case 1: hipLaunchKernelGGL(k_freq_fwd<1>, grid, dim3(256), 0, st, Ya, yb, s.Tp[a], s.chunk[a], P->Wt, s.Mp, s.Kp, Ph, Vp, w.vp_bstride, slot0, nlt); break;
            case 2: hipLaunchKernelGGL(k_freq_fwd<2>, grid, dim3(256), 0, st, Ya, yb, s.Tp[a], s.chunk[a], P->Wt, s.Mp, s.Kp, Ph, Vp, w.vp_bstride, slot0, nlt); break;
            case 4: hipLaunchKernelGGL(k_freq_fwd<4>, grid, dim3(256), 0, st, Ya, yb, s.Tp[a], s.chunk[a], P->Wt, s.Mp, s.Kp, Ph, Vp, w.vp_bstride, slot0, nlt); break;
            default: set_error("unsupported N/T"); return JTFS_ENOTSUP;
        }
        LAUNCHCHK("frequential contraction");
        }
    }
    if (!s.tscat) {
        // every temporal rate in one launch; the FP32 contraction writes two partial
        // slots per t-chunk (both halves of its row tile), the split one one
        const int mult = split ? 1 : 2;
        const ChunkSet& cs = split ? split_chunks(P) : fp32_chunks(P);
        if (s.avg_fr) {
            int tt = s.NT <= 8 ? 8 : s.NT <= 16 ? 16 : 32;
            while (tt > 8 && (int64_t)s.n_beta * ((s.NT + tt - 1) / tt) * 2 * s.n_alpha * B < 1024) tt /= 2;
            auto k = tt == 8 ? k_s2_out<8> : tt == 16 ? k_s2_out<16> : k_s2_out<32>;
            const dim3 g2((unsigned)(s.n_beta * ((s.NT + tt - 1) / tt)), (unsigned)(2 * s.n_alpha), (unsigned)B);
            JTFS_TIMED(JTFS_STAGE_FREQ_LOWPASS, st, hipLaunchKernelGGL(k, g2, dim3(256), 0, st, Vp, w.vp_bstride, cs.d_vchoff,
                               cs.d_nch, mult, nlt, s.NTp, s.NT, P->PFt, P->d_pfoff, P->d_Lb, P->d_rowoff, P->d_rowpos, s.NL, s.NLo, s.n_alpha, s2,
                               ml.mu2, ml.eps, s.n_beta));
        } else {
            const int tt = s.NT <= 8 ? 8 : s.NT <= 16 ? 16 : 32, nlc = (s.L + 63) / 64;
            auto k = tt == 8 ? k_v_out<8> : tt == 16 ? k_v_out<16> : k_v_out<32>;
            const dim3 g4((unsigned)(s.n_beta * nlc * ((s.NT + tt - 1) / tt)), (unsigned)(2 * s.n_alpha), (unsigned)B);
            JTFS_TIMED(JTFS_STAGE_FREQ_LOWPASS, st, hipLaunchKernelGGL(k, g4, dim3(256), 0, st, Vp, w.vp_bstride, cs.d_vchoff,
                               cs.d_nch, mult, nlt, s.NTp, s.NT, P->d_Lb, P->d_rowoff, P->d_rowpos, s.Mh, s.n_alpha, s2,
                               ml.mu2, ml.eps, s.n_beta, nlc));
        }
        LAUNCHCHK("frequency lowpass");
    }
    return JTFS_OK;
}

}  // namespace

extern "C" int jtfs_forward(const jtfs_plan* P, const float* x, int64_t B, float* s1, float* s2, void* ws,
                            size_t ws_bytes, hipStream_t st) {
    return forward_impl(P, x, B, s1, s2, ws, ws_bytes, MuLogArg{}, st);
}

namespace {

// forward FFT of every gY2 row lambda < n1 (length T_alpha), in place; phi_T's rows go
// back through the S1 adjoint untransformed
// the FFTs of the gY2 rows under 2^logmax points
int gy2_row_ffts(const jtfs_plan* P, float2* gY2, int64_t yb, int logmax, int64_t B, hipStream_t st) {
    const Shapes& s = P->s;
    for (int a = 0; a < s.n_alpha_psi; ++a) {
        const int logTa = s.logNX - s.k2[a];
        if (logTa >= logmax) continue;
        if (!reg_row(logTa, P->tune.reg_rowfft)) continue;
        JTFS_TIMED(JTFS_STAGE_SECOND_ADJ_FFT, st,
                   launch_rowfft_r(P, gY2 + s.yoff[a], yb, (int64_t)s.Tp[a], s.n1, logTa, B, st));
        LAUNCHCHK("second-order adjoint FFT");
    }
    ShortRates sr;
    size_t lds = 0;
    unsigned blocks = 0;
    for (int a = 0; short_rates(P, P->tune.reg_rowfft, &a, s.n1, s.n1, B, &sr, &blocks, &lds);) {
        JTFS_TIMED(JTFS_STAGE_SECOND_ADJ_FFT, st, hipLaunchKernelGGL(k_rowfft_short, dim3(blocks, (unsigned)B), dim3(1024), lds, st,
                           gY2, yb, s.n1, sr, P->tw, P->tw_log));
        LAUNCHCHK("second-order adjoint FFT");
    }
    return JTFS_OK;
}

int backward_impl(const jtfs_plan* P, const float* x, const float* gs1, const float* gs2, float* gx, int64_t B,
                  void* ws, size_t ws_bytes, uint32_t flags, const MuLogArg& ml, hipStream_t st) {
    int rc = check_common(P, B, ws, ws_bytes, false);
    if (rc != JTFS_OK) return rc;
    if (!x || !gx) { set_error("null pointer"); return JTFS_EINVAL; }
    const Shapes& s = P->s;
    const Workspace w = plan_layout(P, B);
    char* base = (char*)ws;
    if (!(flags & JTFS_BWD_REUSE_FORWARD)) {
        rc = forward_front(P, x, B, nullptr, base, w, MuLogArg{}, st);
        if (rc != JTFS_OK) return rc;
    }
    float2* xh = (float2*)(base + w.xh);
    float2* tmp = (float2*)(base + w.tmp);
    float2* Y2 = (float2*)(base + w.Y2);
    float* gV = (float*)(base + w.gV);
    float2* PQ = (float2*)(base + w.PQ);
    float2* gY2 = (float2*)(base + w.gY2);
    float* gX = (float*)(base + w.gX);
    float2* g1 = (float2*)(base + w.g1);
    float2* gxh = (float2*)(base + w.gxh);
    const int64_t yb = (int64_t)s.Kp * s.sumTp;
    const int nlt = s.Mp / kTileL;
    // time scattering: the lowpass and modulus adjoints give gY2 directly
    if (s.tscat) {
        auto k = s.NTp == 32 ? k_ts_bwd<1> : s.NTp == 64 ? k_ts_bwd<2> : k_ts_bwd<4>;
        JTFS_TIMED(JTFS_STAGE_LOWPASS_ADJ, st, hipLaunchKernelGGL(k, dim3((unsigned)(s.sumTp / kTileTh), (unsigned)((s.n1 + 31) / 32), (unsigned)B), dim3(256), 0, st,
                           Y2, yb, P->d_rates, P->d_tiles, P->Phi, s.n1, s.NT, s.n_alpha, gs2, gY2, ml));
        LAUNCHCHK("time-scattering adjoint");
    }
    if (!s.tscat) {
        // every temporal rate in one launch
        const dim3 grid(s.n_beta + 1, 2 * s.n_alpha, (unsigned)B);
        if (s.avg_fr) {
            auto k = s.NTp % 32 == 0 && s.NT >= 32 ? k_s2_bwd_avg<32> : k_s2_bwd_avg<16>;
            const size_t whole = sizeof(float) * s.NLo * s.NT;
            const int cols = whole <= (size_t)kMaxDynLds ? s.NT : 32;
            const size_t lds = cols == s.NT ? whole : sizeof(float) * (s.NLo * 32 + s.L);
            JTFS_TIMED(JTFS_STAGE_LOWPASS_ADJ, st, hipLaunchKernelGGL(k, grid, dim3(256), lds, st, gs2,
                               P->PF, P->d_pfoff, P->d_Lb, P->d_rowoff, P->d_rowpos, P->d_pad, s.n_beta, s.NLo, s.NT, s.NTp, cols, s.Mh, s.Mp,
                               s.n_alpha, gV, (float*)(base + w.gvmax), ml));
        } else {
            JTFS_TIMED(JTFS_STAGE_LOWPASS_ADJ, st, hipLaunchKernelGGL(k_s2_bwd, grid, dim3(256), sizeof(float) * s.L, st, gs2, P->d_Lb,
                               P->d_rowoff, P->d_rowpos, P->d_pad, s.n_beta, s.NT, s.NTp, s.Mh, s.Mp, s.n_alpha,
                               gV, (float*)(base + w.gvmax), ml));
        }
        LAUNCHCHK("frequency lowpass adjoint");
    }
    const bool split = split_backward(P);
    const bool phase_mode = split && P->contraction == JTFS_CONTRACTION_SPLIT_F16_PHASE;
    // the phase the forward stored, when this backward follows it on the same
    // workspace; without that forward, the phase is taken again by the forward
    // contraction where the recomputing kernel cannot hold the shapes
    const bool reuse = flags & JTFS_BWD_REUSE_FORWARD;
    const bool regen_phase = phase_mode && !reuse && !P->split_bwd_ok;
    const bool from_phase = phase_mode && (reuse || regen_phase);
    unsigned short* Yh = (unsigned short*)(base + w.Yh);
    float* ysc = (float*)(base + w.yscale);
    if (split && !reuse) {
        JTFS_TIMED(JTFS_STAGE_OPERAND_SPLIT, st,
                   rc = launch_ysplit(P, Y2, (const float*)(base + w.rowmax), Yh, ysc, B, st));
        if (rc != JTFS_OK) { set_error("operand split kernel failed"); return rc; }
        if (regen_phase) {
            JTFS_TIMED(JTFS_STAGE_FREQ_FWD, st,
                       rc = launch_freq_fwd_split(P, Yh, ysc, (float*)(base + w.Vp), w.vp_bstride,
                                                  (unsigned*)(base + w.phase), w.ph_bstride, B, st));
            if (rc != JTFS_OK) { if (rc == JTFS_EHIP) set_error("split contraction launch failed"); return rc; }
        }
    }
    if (from_phase) {
        JTFS_TIMED(JTFS_STAGE_OPERAND_SPLIT, st, rc = launch_gv_split(P, gV, (uint4*)(base + w.gvs), B, st));
        if (rc != JTFS_OK) { if (rc == JTFS_EHIP) set_error("gV split launch failed"); return rc; }
    }
    if (split) {
        // every temporal rate in one launch
        if (from_phase) {
            JTFS_TIMED(JTFS_STAGE_FREQ_ADJ_PQ, st,
                       rc = launch_freq_bwd_phase(P, (const unsigned*)(base + w.phase), w.ph_bstride,
                                                  (const uint4*)(base + w.gvs), w.gvs_bstride,
                                                  (const float*)(base + w.gvmax), gY2, B, st));
        } else {
            JTFS_TIMED(JTFS_STAGE_FREQ_ADJ_PQ, st,
                       rc = launch_freq_bwd_split(P, Yh, ysc, gV, (const float*)(base + w.gvmax), gY2, B, st));
        }
        if (rc != JTFS_OK) { if (rc == JTFS_EHIP) set_error("split backward contraction launch failed"); return rc; }
    }
    for (int a = 0; a < s.n_alpha && !split && !s.tscat; ++a) {
        dim3 grid(nlt, s.Tp[a] / kTileT, (unsigned)B);
        const float2* Ya = Y2 + s.yoff[a];
        const float* Ph = P->Phi + s.phioff[a];
        const float* gVa = gV + (int64_t)a * 2 * s.Mp * s.NTp;
        const int64_t gvb = (int64_t)s.n_alpha * 2 * s.Mp * s.NTp;
        {
        TimedLaunch tl_pq(JTFS_STAGE_FREQ_ADJ_PQ, st);
        switch (s.NTp / 32) {
            case 1: hipLaunchKernelGGL(k_bwd_pq<1>, grid, dim3(256), 0, st, Ya, yb, s.Tp[a], P->Wt, s.Mp, s.Kp, Ph, gVa, gvb, PQ); break;
            case 2: hipLaunchKernelGGL(k_bwd_pq<2>, grid, dim3(256), 0, st, Ya, yb, s.Tp[a], P->Wt, s.Mp, s.Kp, Ph, gVa, gvb, PQ); break;
            case 4: hipLaunchKernelGGL(k_bwd_pq<4>, grid, dim3(256), 0, st, Ya, yb, s.Tp[a], P->Wt, s.Mp, s.Kp, Ph, gVa, gvb, PQ); break;
            default: set_error("unsupported N/T"); return JTFS_ENOTSUP;
        }
        LAUNCHCHK("contraction adjoint (recompute, modulus)");
        }
        JTFS_TIMED(JTFS_STAGE_FREQ_ADJ_WH, st, hipLaunchKernelGGL(k_bwd_gy, dim3((s.Kp + 63) / 64, s.Tp[a] / kTileT, (unsigned)B), dim3(256), 0, st, PQ,
                           s.Tp[a], P->Wl, s.Mp, s.Kp, gY2 + s.yoff[a], yb));
        LAUNCHCHK("contraction adjoint (W^H)");
    }
    // with both in registers, the scalogram adjoint transforms the long gY2 rows itself
    const bool rows_in_a = rows_in_adjoint(P);
    rc = gy2_row_ffts(P, gY2, yb, rows_in_a ? kRegMinLogRows - 1 : 31, B, st);
    if (rc != JTFS_OK) return rc;
    const int logNT = s.logN - s.logT;
    const size_t lds_a = sizeof(float2) * (lpad_len(s.NX / 2) + 1 + lpad_len(s.NT));   // g1 at lpad(H) + 1
    const float2* gYphi = s.complete ? gY2 + s.yoff[s.n_alpha_psi] : nullptr;
    const int Tphi = s.complete ? s.Tp[s.n_alpha_psi] : 0;
    if (use_reg_rows(s.logNX, P->tune.reg_first_adj)) {
        JTFS_TIMED(JTFS_STAGE_SECOND_ADJ, st, launch_scal_bwd_a_r(P, gY2, yb, gs1, ml, gYphi, Tphi, gX, rows_in_a, B, st));
    } else {
        JTFS_TIMED(JTFS_STAGE_SECOND_ADJ, st, hipLaunchKernelGGL(k_scal_bwd_a, dim3(s.n1, (unsigned)B), dim3(1024), lds_a, st, gY2, yb, P->d_yoff, P->d_Tp, P->d_Ta, P->psi2,
                           P->band2, P->off2, s.n_alpha_psi, gs1, P->phiX, s.Mphi, logNT, s.logNX, gX, P->tw, P->tw_log, ml,
                           gYphi, Tphi));
    }
    LAUNCHCHK("scalogram adjoint");
    if (use_reg_rows(s.logNX, P->tune.reg_first_adj)) {
        JTFS_TIMED(JTFS_STAGE_FIRST_ADJ, st, launch_scal_bwd_b_r(P, xh, w.xh_pitch, gX, g1, B, st));
    } else {
        JTFS_TIMED(JTFS_STAGE_FIRST_ADJ, st, hipLaunchKernelGGL(k_scal_bwd_b, dim3(s.n1, (unsigned)B), dim3(1024), sizeof(float2) * lpad_len(s.NX), st, xh, w.xh_pitch,
                       P->psi1, P->band1, P->off1, gX, g1, s.logNX, 1.0f / (float)s.N, P->tw, P->tw_log));
    }
    LAUNCHCHK("modulus and first-order adjoint");
    const int Hn = (int)(s.N / 2);
    JTFS_TIMED(JTFS_STAGE_BAND_ACCUM, st, hipLaunchKernelGGL(k_band_accum, dim3((unsigned)((Hn + 1 + 255) / 256), (unsigned)B), dim3(256), 0, st, g1, s.n1,
                       s.logNX, P->psi1, P->band1, P->off1, P->lam_range, Hn, gxh, w.xh_pitch));
    LAUNCHCHK("band accumulation");
    const int logH = s.logN - 1;
    if (logH <= kOneRowLog) {
        const int logC = 12 - logH;
        const size_t lds = (size_t)(1 << logC) * (lpad_len(Hn) + 1) * sizeof(float2);
        JTFS_TIMED(JTFS_STAGE_OUTPUT_FFT, st, hipLaunchKernelGGL(k_irfft_rows, dim3((unsigned)((B + (1 << logC) - 1) >> logC)), dim3(1024), lds, st,
                           gxh, w.xh_pitch, (int)B, logH, logC, (float2*)gx, 1.0f / (float)s.N, P->tw, P->tw_log));
    } else {
        JTFS_TIMED(JTFS_STAGE_OUTPUT_FFT, st, irfft_four_step(gxh, w.xh_pitch, (float2*)gx, tmp, logH, B, 1.0f / (float)s.N, P, st));
    }
    LAUNCHCHK("output inverse FFT");
    return JTFS_OK;
}

int mulog_check(const jtfs_plan* P, const float* mu1, const float* mu2, float eps) {
    if (!P || !mu1 || !mu2) { set_error("null pointer"); return JTFS_EINVAL; }
    if (!(eps > 0.f)) { set_error("eps must be positive"); return JTFS_EINVAL; }
    return JTFS_OK;
}

}  // namespace

extern "C" int jtfs_backward(const jtfs_plan* P, const float* x, const float* gs1, const float* gs2, float* gx,
                             int64_t B, void* ws, size_t ws_bytes, uint32_t flags, hipStream_t st) {
    return backward_impl(P, x, gs1, gs2, gx, B, ws, ws_bytes, flags, MuLogArg{}, st);
}

extern "C" int jtfs_zeroth_order(const jtfs_plan* P, const float* x, int64_t B, float* s0, hipStream_t st) {
    if (!P || !x || !s0) { set_error("null pointer"); return JTFS_EINVAL; }
    if (B < 1 || B > 65535) { set_error("B must lie in [1, 65535]"); return JTFS_ESHAPE; }
    const Shapes& s = P->s;
    hipLaunchKernelGGL(k_s0, dim3((unsigned)s.NT, (unsigned)B), dim3(1024), 0, st, x, s.N, s.T, P->phiN, P->phiN_len,
                       P->phiN_half, s0);
    LAUNCHCHK("zeroth order");
    return JTFS_OK;
}

extern "C" int jtfs_zeroth_order_backward(const jtfs_plan* P, const float* gs0, int64_t B, float* gx, hipStream_t st) {
    if (!P || !gs0 || !gx) { set_error("null pointer"); return JTFS_EINVAL; }
    if (B < 1 || B > 65535) { set_error("B must lie in [1, 65535]"); return JTFS_ESHAPE; }
    const Shapes& s = P->s;
    hipLaunchKernelGGL(k_s0_bwd, dim3((unsigned)((s.N + 255) / 256), (unsigned)B), dim3(256), 0, st, gs0, s.N, s.T, s.NT,
                       P->phiN, P->phiN_len, P->phiN_half, gx);
    LAUNCHCHK("zeroth-order adjoint");
    return JTFS_OK;
}

extern "C" int jtfs_forward_mulog(const jtfs_plan* P, const float* x, int64_t B, const float* mu1, const float* mu2,
                                  float eps, float* o1, float* o2, void* ws, size_t ws_bytes, hipStream_t st) {
    const int rc = mulog_check(P, mu1, mu2, eps);
    if (rc != JTFS_OK) return rc;
    return forward_impl(P, x, B, o1, o2, ws, ws_bytes, MuLogArg{mu1, mu2, eps, nullptr, nullptr}, st);
}

extern "C" int jtfs_backward_mulog(const jtfs_plan* P, const float* x, const float* o1, const float* o2,
                                   const float* mu1, const float* mu2, float eps, const float* go1, const float* go2,
                                   float* gx, int64_t B, void* ws, size_t ws_bytes, uint32_t flags, hipStream_t st) {
    const int rc = mulog_check(P, mu1, mu2, eps);
    if (rc != JTFS_OK) return rc;
    if ((go1 && !o1) || (go2 && !o2)) { set_error("null pointer"); return JTFS_EINVAL; }
    return backward_impl(P, x, go1, go2, gx, B, ws, ws_bytes, flags, MuLogArg{mu1, mu2, eps, o1, o2}, st);
}


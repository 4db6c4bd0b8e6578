// K2 in double, old history by transforms: the far field of kFftRows rows at
// once.
//
// The direct products of far.hip cost 2L rows x K per column and block, which
// for long histories is the whole solve (65536 steps, 1024 oscillators: 245 of
// 262 ms at the fp64 matrix peak).  The weights are Toeplitz, so the part of
// those sums whose history is older than the current superblock is a
// convolution: with superblock Q = rows n = QS .. QS + S - 1 (S = kFftRows)
// and history block p = the S rows k = pS - L + 1 .. (p+1)S - L,
//   sum over p < Q, j < S of w[(Q-p)S + L - 1 + r - j] F[pS - L + 1 + j]
// is, for every column, elements S-1 .. 2S-2 of
//   IFFT( sum over p of FFT(F_p) FFT(v_{Q-p}) ),  v_s[i] = w[(s-1)S + L + i],
// transforms of length 2S = 4096 (the wrapped-around elements are the others).
// History up to QS - L is complete one block before row QS is stepped, so this
// runs beside the chain of the block between; the direct products are left
// with the history since QS - L, at most S - L rows.
//
// Every history block is transformed once and its spectrum kept (the half
// that a real sequence needs); a superblock reads the spectra before it once,
// adds them up against the spectra of the weights and takes one inverse
// transform, with the predictor's sums as real and the corrector's as
// imaginary part.  A column never meets another one, so a trajectory's bits do
// not depend on its batch and a non-finite member stays alone.
//
// What bounds it: reading the spectra, S + 1 complex values per history block
// and column -- in the sweep of 1024 oscillators over 65536 steps 1.15 GB a
// launch on average, 328 us, 3.5 TB/s (a large copy: 5.5); of it about 50 us
// are bank conflicts where the sums leave through LDS.  One column per
// workgroup of 256 threads, 16 points per thread, three radix-16 passes
// exchanged through 35 KB of LDS, four workgroups to a CU.  S = 2048: of 4096
// points a pass is 16 per thread and 4096 = 16^3; half of it doubles the
// spectra read, twice of it leaves one workgroup per CU and doubles the direct
// part.
#include "abm_dev.h"
#include "abm_kernels.h"

namespace abm {

namespace {

constexpr int S = kFftRows, NF = 2 * S;      // transform length
constexpr int kThreads = 256, kPts = NF / kThreads;
constexpr int kRow1 = 272, kRow2 = 17;       // padded rows of the two exchanges (doubles)
constexpr int kLds = 16 * kRow1;             // 4352 doubles; 256 * kRow2 = 4352
static_assert(kPts == 16 && NF == 16 * 16 * 16, "three radix-16 passes");
// 1 / NF, taken at the front so that no value between exceeds what the direct
// products would form: 2^-11 from the history (a sum of S values), the rest
// from the weights.  Powers of two: nothing else changes.
constexpr double kScaleF = 1.0 / S, kScaleW = (double)S / NF;

struct cplx {
    double re, im;
};
__device__ __forceinline__ cplx operator+(cplx a, cplx b) { return {a.re + b.re, a.im + b.im}; }
__device__ __forceinline__ cplx operator-(cplx a, cplx b) { return {a.re - b.re, a.im - b.im}; }
__device__ __forceinline__ cplx mul(cplx a, cplx b)
{
    return {fma(a.re, b.re, -(a.im * b.im)), fma(a.re, b.im, a.im * b.re)};
}
__device__ __forceinline__ cplx mul_mi(cplx a) { return {a.im, -a.re}; }   // -i a

// 4-point transform (forward)
__device__ __forceinline__ void dft4(cplx& a, cplx& b, cplx& c, cplx& d)
{
    const cplx s = a + c, t = a - c, u = b + d, v = mul_mi(b - d);
    a = s + u;
    b = t + v;
    c = s - u;
    d = t - v;
}

// 16-point forward transform in place: x[e], e = 4 e1 + e0 -> x[k]
__device__ __forceinline__ void dft16(cplx (&x)[16])
{
    constexpr double c1 = 0.92387953251128675613, s1 = 0.38268343236508977173, h = 0.70710678118654752440;
    // e = e0 + 4 e1: transforms over e1, then over e0; k = 4 k0 + k1
#pragma unroll
    for (int e0 = 0; e0 < 4; ++e0) dft4(x[e0], x[e0 + 4], x[e0 + 8], x[e0 + 12]);
    // x[e0 + 4 k1] times w16^(e0 k1)
    x[5] = mul(x[5], {c1, -s1});
    x[9] = mul(x[9], {h, -h});
    x[13] = mul(x[13], {s1, -c1});
    x[6] = mul(x[6], {h, -h});
    x[10] = mul_mi(x[10]);
    x[14] = mul(x[14], {-h, -h});
    x[7] = mul(x[7], {s1, -c1});
    x[11] = mul(x[11], {-h, -h});
    x[15] = mul(x[15], {-c1, s1});
    cplx y[16];
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1) {
        cplx a = x[4 * k1], b = x[4 * k1 + 1], c = x[4 * k1 + 2], d = x[4 * k1 + 3];
        dft4(a, b, c, d);
        y[k1] = a;
        y[k1 + 4] = b;
        y[k1 + 8] = c;
        y[k1 + 12] = d;
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) x[k] = y[k];
}

// x[j] of the 256 threads through LDS, one part after the other: thread
// values written at w(j), read at r(j).
template <class W, class R>
__device__ __forceinline__ void exchange(cplx (&x)[16], double* lds, W w, R r)
{
#pragma unroll
    for (int j = 0; j < 16; ++j) lds[w(j)] = x[j].re;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 16; ++j) x[j].re = lds[r(j)];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 16; ++j) lds[w(j)] = x[j].im;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 16; ++j) x[j].im = lds[r(j)];
    __syncthreads();
}

// Thread v's place in the result: it holds elements low(v) + 256 j.
__device__ __forceinline__ int low(int v) { return (v >> 4) + 16 * (v & 15); }

// Forward transform of NF points: in, x[e] = element t + 256 e (t: any
// numbering of the threads); out, thread v's x[j] = element low(v) + 256 j.
// tw[i] = exp(-2 pi i / NF).
__device__ __forceinline__ void fft(cplx (&x)[16], int t, int v, double* lds, gptr<const cplx> tw)
{
    auto twiddle = [&](int i) {
        const gptr<const cplx> p = tw + i;
        return cplx{p->re, p->im};
    };
    dft16(x);                                           // k of element 16 q + k
#pragma unroll
    for (int k = 1; k < 16; ++k) x[k] = mul(x[k], twiddle(t * k));
    const int k = v >> 4, t1 = v & 15;
    exchange(x, lds, [&](int j) { return j * kRow1 + t; }, [&](int j) { return k * kRow1 + t1 + 16 * j; });
    dft16(x);                                           // k' of q = 16 q' + k'
#pragma unroll
    for (int j = 1; j < 16; ++j) x[j] = mul(x[j], twiddle(16 * t1 * j));
    exchange(x, lds, [&](int j) { return (16 * k + j) * kRow2 + t1; }, [&](int j) { return v * kRow2 + j; });
    dft16(x);
}

// Half spectrum of a real sequence, stored as the threads hold it: value j of
// thread v (element low(v) + 256 j, j < 8) at 256 j + v, element S at S.
__device__ __forceinline__ void store_half(const cplx (&x)[16], int v, gptr<cplx> out)
{
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const gptr<cplx> o = out + 256 * j + v;
        o->re = x[j].re;
        o->im = x[j].im;
    }
    if (v == 0) {
        const gptr<cplx> o = out + S;
        o->re = x[8].re;
        o->im = x[8].im;
    }
}

// Column of workgroup x of n: neighbours in memory on one XCD (workgroups go
// to the 8 XCDs in turn), which then reads each line of the history once.
__device__ __forceinline__ int column_of(int x, int n)
{
    const int each = (n + 7) / 8;
    return (x & 7) * each + (x >> 3);
}

__global__ __launch_bounds__(kThreads) void k_fft_twiddles(cplx* tw)
{
    const int i = blockIdx.x * kThreads + threadIdx.x;
    double sn, cs;
    sincospi(-2.0 * i / NF, &sn, &cs);
    tw[i] = {cs, sn};
}

// spectra of v_s: blockIdx.x = s - 1, blockIdx.y = 0 (b) or 1 (a); n: table length
__global__ __launch_bounds__(kThreads) void k_fft_weights(const double* b, const double* a, int64_t n, int L,
                                                          const cplx* tw, cplx* out)
{
    __shared__ double lds[kLds];
    const int v = threadIdx.x;
    const gptr<const double> w = as_global(blockIdx.y ? a : b);
    const int64_t at = (int64_t)blockIdx.x * S + L;
    cplx x[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int i = v + 256 * e;
        x[e] = {i < NF - 1 && at + i < n ? kScaleW * w[at + i] : 0.0, 0.0};
    }
    fft(x, v, v, lds, as_global(tw));
    store_half(x, v, as_global(out) + ((size_t)blockIdx.x * 2 + blockIdx.y) * kFftStride);
}

// spectrum of history block Q - 1 of every column of an item
__global__ __launch_bounds__(kThreads) void k_fft_history(const GroupDev* groups, const FftItem* items, int L,
                                                          const cplx* tw)
{
    __shared__ double lds[kLds];
    const FftItem it = items[blockIdx.y];
    const int c = column_of(blockIdx.x, it.ncols);
    if ((int)(blockIdx.x >> 3) >= (it.ncols + 7) / 8 || c >= it.ncols) return;
    const GroupDev& G = groups[it.group];
    const int v = threadIdx.x, col = it.coff + c;
    const gptr<const double> F = as_global((const double*)G.F) + col;
    const int64_t k0 = (int64_t)(it.Q - 1) * S - L + 1;
    cplx x[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int64_t k = k0 + v + 256 * e;
        x[e] = {e < 8 && k >= 1 ? kScaleF * F[k * G.ldF] : 0.0, 0.0};
    }
    fft(x, v, v, lds, as_global(tw));
    store_half(x, v, as_global((cplx*)G.spec) + ((size_t)(it.Q - 1) * G.ldF + col) * kFftStride);
}

// far-field sums of superblock Q from every history block before it
__global__ __launch_bounds__(kThreads) void k_fft_sums(const GroupDev* groups, const FftItem* items, int L,
                                                       const cplx* tw)
{
    __shared__ double lds[kLds];
    const FftItem it = items[blockIdx.y];
    const int c = column_of(blockIdx.x, it.ncols);
    if ((int)(blockIdx.x >> 3) >= (it.ncols + 7) / 8 || c >= it.ncols) return;
    const GroupDev& G = groups[it.group];
    const int v = threadIdx.x, col = it.coff + c;
    const size_t step = (size_t)G.ldF * kFftStride;
    gptr<const cplx> f = as_global((const cplx*)G.spec) + (size_t)col * kFftStride + v;
    // lag Q - p of history block p: its weights' spectra, b then a
    gptr<const cplx> w = as_global((const cplx*)G.wspec[it.comp]) + (size_t)(it.Q - 1) * 2 * kFftStride + v;
    cplx yb[8], ya[8], mb{0.0, 0.0}, ma{0.0, 0.0};
#pragma unroll
    for (int j = 0; j < 8; ++j) yb[j] = ya[j] = {0.0, 0.0};
    auto add = [](cplx& y, cplx a, cplx b) {
        y.re = fma(a.re, b.re, fma(-a.im, b.im, y.re));
        y.im = fma(a.re, b.im, fma(a.im, b.re, y.im));
    };
    auto get = [](gptr<const cplx> p) { return cplx{p->re, p->im}; };
    for (int p = 0; p < it.Q; ++p, f += step, w -= 2 * kFftStride) {
        cplx a[8], b[8], d[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            a[j] = get(f + 256 * j);
            b[j] = get(w + 256 * j);
            d[j] = get(w + kFftStride + 256 * j);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            add(yb[j], a[j], b[j]);
            add(ya[j], a[j], d[j]);
        }
        if (v == 0) {
            const cplx m = get(f + S);
            add(mb, m, get(w + S));
            add(ma, m, get(w + kFftStride + S));
        }
    }
    // Y = Yb + i Ya, the upper half by the symmetry of Yb and Ya; conjugated,
    // so that a forward transform gives the conjugate of the inverse's result.
    // conj(Y)[NF - e] = Yb[e] - i Ya[e] for e = low + 256 j goes to the thread
    // that holds element NF - e = (256 - low) + 256 (15 - j)
    // (256 (16 - j) for low = 0).
    const int lo = low(v);
    const int lo2 = (256 - lo) & 255;
    const int v2 = 16 * (lo2 & 15) + (lo2 >> 4);
    cplx x[16];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = {yb[j].re - ya[j].im, -(yb[j].im + ya[j].re)};
    const int up = lo == 0 ? 1 : 0;                     // element 8 + 7 - j + up of thread v2
#pragma unroll
    for (int part = 0; part < 2; ++part) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (!(up && j == 0))
                lds[(7 - j + up) * 256 + v2] = part == 0 ? yb[j].re + ya[j].im : yb[j].im - ya[j].re;
        if (up) lds[v2] = part == 0 ? mb.re - ma.im : -(mb.im + ma.re);   // element S
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 8; ++j) (part == 0 ? x[8 + j].re : x[8 + j].im) = lds[j * 256 + v];
        __syncthreads();
    }
    fft(x, lo, v, lds, as_global(tw));
    // element n = low + 256 j of conj(result); rows r = n - (S - 1)
    const gptr<double> out = as_global(G.fpart) + (size_t)(it.Q & 1) * (S / L) * G.ldF * (2 * L);
#pragma unroll
    for (int part = 0; part < 2; ++part) {
#pragma unroll
        for (int j = 0; j < 16; ++j) lds[lo + 256 * j] = part == 0 ? x[j].re : -x[j].im;
        __syncthreads();
#pragma unroll
        for (int e = 0; e < S / kThreads; ++e) {
            const int r = v + kThreads * e;
            const int blk = r / L;
            out[((size_t)blk * G.ldF + col) * (2 * L) + part * L + (r - blk * L)] = lds[r + S - 1];
        }
        __syncthreads();
    }
}

}  // namespace

hipError_t launch_fft_weights(const double* b, const double* a, int64_t n, int L, int lags, const double* tw,
                              double* out, hipStream_t st)
{
    if (lags < 1) return hipSuccess;
    hipLaunchKernelGGL(k_fft_weights, dim3((unsigned)lags, 2), dim3(kThreads), 0, st, b, a, n, L,
                       (const cplx*)tw, (cplx*)out);
    return hipGetLastError();
}

hipError_t launch_fft_twiddles(double* tw, hipStream_t st)
{
    hipLaunchKernelGGL(k_fft_twiddles, dim3(NF / kThreads), dim3(kThreads), 0, st, (cplx*)tw);
    return hipGetLastError();
}

hipError_t launch_far_fft(const GroupDev* groups, const FftItem* items, int n, int max_cols, int L,
                          const double* tw, hipStream_t st)
{
    if (n < 1 || max_cols < 1) return hipSuccess;
    const dim3 grid((unsigned)((max_cols + 7) / 8 * 8), (unsigned)n);
    hipLaunchKernelGGL(k_fft_history, grid, dim3(kThreads), 0, st, groups, items, L, (const cplx*)tw);
    hipLaunchKernelGGL(k_fft_sums, grid, dim3(kThreads), 0, st, groups, items, L, (const cplx*)tw);
    return hipGetLastError();
}

}  // namespace abm

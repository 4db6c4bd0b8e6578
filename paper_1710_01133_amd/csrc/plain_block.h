// K1: one trajectory, blocks of 64 steps -- the kernel of abm_solve and
// abm_solve_noalloc in double (plain.hip) and double-double (plain_dd.hip).
//
// The paper's parallel scheme (Algorithm 1: every process sums its slice of
// the history, one all-reduce, the update) asks for one grid-wide reduction
// per step, which costs about 3 us on this GPU however little is summed.  Here
// the reduction is taken once per block of kB = 64 steps:
//   * workgroup 0 steps.  Its wave 0 (the sequencer) owns the 64 rows of the
//     current block, one per lane, scatters every new f_s into the later rows
//     of this block and the rows of the next one, and reads the sums of row
//     r + 1, complete but for the newest term, while row r is updated, so only
//     that term (b_0 f, a_0 f), the predictor, the corrector and their two
//     right-hand sides are on a step's dependent path.  No global memory
//     operation and no barrier is inside a block;
//   * what block q needs from chunk c (the 64 rows f that block c produced):
//     c = q and q - 1 the sequencer's scatter; c = q - 2 one other wave of
//     workgroup 0 while block q - 1 runs (from LDS); c <= q - 3 the workers;
//   * a worker (workgroup 1 .. W) owns the chunks c with c mod W = its index,
//     kept in LDS, and sums them against the 64 rows of every block q, at
//     most kSlots blocks ahead of the sequencer; a worker waits only for its
//     own newest chunk, so all but one of them run ahead;
//   * with more than kFan workers, groups of kFan of them are summed by a
//     reducer workgroup each; workgroup 0 sums the at most kFan results.
// What bounds it: the sequencer's instructions (one wave; an f64 operation
// issues every 4.2 cycles whether or not it depends on the one before, and so
// does every other instruction), 0.053 us per step for the linear equation
// (0.065 with every state written), 0.098 for the oscillator, 0.138 for Lorenz,
// 0.169 for the circuit, from a few thousand steps on (double-double: 0.43,
// 1.02, 1.41, 1.23).  Beyond about 5e5 steps the workers' weights come from
// beyond L2 (10^6 steps of the oscillator: 0.139).  One reduction per step took
// 0.91 (8192 steps of the linear equation, one workgroup) and 2.9 (200000 steps
// of the oscillator; double-double 2.4 and 5.0).  Hence the 64 rows unrolled
// (a lane index in an SGPR costs a readlane twice the time: 0.135 us per step
// of the oscillator with a rolled loop) and the weights read one group of rows
// ahead.
// Every sum is taken in an order fixed by (N, W) alone.  Short histories run
// in workgroup 0 alone (W = 0): the waves beside the sequencer then sum the
// chunks c <= q - 2 from LDS while block q - 1 runs.
//
// A chunk against 64 rows is a 64 x 64 Toeplitz product per weight table: lane
// (lr, g) of a wave takes the rows lr + LR j and the indices kr + LR i of the
// chunk, so that 2 RP - 1 weights serve RP x RP pairs (LR RP = 64) and a
// chunk costs (2 RP - 1 + RP) LDS reads per 4 D RP RP operations (16-byte reads: the
// LDS block is 16-byte aligned; 8 bytes off, every read is taken as unaligned
// and a chunk costs about four times as much).
#pragma once
#include "abm_dev.h"
#include "abm_kernels.h"

namespace abm {

// Of each pair of lanes l, l ^ mask the upper one's a and the lower one's b
// change places (mask 32, 16 or 8): vector moves, where a shuffle goes through
// the LDS unit twice per double.
__device__ __forceinline__ void exchange_halves(uint32_t& a, uint32_t& b, int mask)
{
    if (mask == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
        a = r[0];
        b = r[1];
    } else if (mask == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
        a = r[0];
        b = r[1];
    } else {
        // rows of 16 lanes rotated by 8, into their upper (banks 2, 3) and lower half
        const uint32_t up = (uint32_t)__builtin_amdgcn_update_dpp((int)a, (int)b, 0x128, 0xf, 0xc, false);
        b = (uint32_t)__builtin_amdgcn_update_dpp((int)b, (int)a, 0x128, 0xf, 0x3, false);
        a = up;
    }
}
__device__ __forceinline__ void exchange_halves(double& a, double& b, int mask)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, a), v = __builtin_bit_cast(uint64_t, b);
    uint32_t al = (uint32_t)u, ah = (uint32_t)(u >> 32), bl = (uint32_t)v, bh = (uint32_t)(v >> 32);
    exchange_halves(al, bl, mask);
    exchange_halves(ah, bh, mask);
    a = __builtin_bit_cast(double, ((uint64_t)ah << 32) | al);
    b = __builtin_bit_cast(double, ((uint64_t)bh << 32) | bl);
}

// Arithmetic of the path in the type T (double here; double-double in
// plain_dd.hip).  LR: lanes along the rows in a chunk product (64 / LR rows
// per lane: as many as the registers hold).
template <class T>
struct Num;

template <>
struct Num<double> {
    static constexpr int LR = 8;
    static constexpr bool kUnroll = true;    // the sequencer's 64 rows unrolled
    static __device__ __forceinline__ double zero() { return 0.0; }
    static __device__ __forceinline__ double mac(double w, double f, double acc) { return fma(w, f, acc); }   // acc + w f
    // the same for the newest block's terms, and for the state's update
    static __device__ __forceinline__ double mac_near(double w, double f, double acc) { return fma(w, f, acc); }
    static __device__ __forceinline__ double mac_state(double w, double f, double acc) { return fma(w, f, acc); }
    static __device__ __forceinline__ double mul_add(double a, double b, double c) { return fma(a, b, c); }
    // mac for a step's newest term, w = newest_weight(weight): as a
    // multiply-add of -f it takes acc from scalar registers
    static __device__ __forceinline__ double newest_weight(double w) { return -w; }
    static __device__ __forceinline__ double newest(double w, double f, double acc) { return fma(w, -f, acc); }
    static __device__ __forceinline__ double newest_predictor(double w, double f, double acc) { return fma(w, -f, acc); }
    static __device__ __forceinline__ double add(double a, double b) { return a + b; }
    static __device__ __forceinline__ double mul(double a, double b) { return a * b; }
    static __device__ __forceinline__ double of(double x) { return x; }
    static __device__ __forceinline__ double recip(double x) { return 1.0 / x; }
    static __device__ __forceinline__ double power(double h, double al) { return pow(h, al); }
    static __device__ __forceinline__ double time(int64_t s, double h) { return (double)s * h; }
    static __device__ __forceinline__ bool finite(double x) { return isfinite(x); }
    static __device__ __forceinline__ double nan() { return __builtin_nan(""); }
    static __device__ __forceinline__ double lane(double v, int l)
    {
        const uint64_t u = __builtin_bit_cast(uint64_t, v);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, l);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l);
        return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
    }
    static __device__ __forceinline__ double swap(double v, int mask) { return __shfl_xor(v, mask, kWave); }
    static __device__ __forceinline__ void exchange(double& a, double& b, int mask) { exchange_halves(a, b, mask); }
    static __device__ __forceinline__ double get(const double* p) { return *as_global(p); }
    static __device__ __forceinline__ void put(double* p, double v) { *as_global(p) = v; }
    static __device__ __forceinline__ double ld_agent(const double* p) { return ld_relaxed(p); }
    static __device__ __forceinline__ void st_agent(double* p, double v)
    {
        __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    template <int R>
    static __device__ __forceinline__ double force(const double* p, int64_t s, double h)
    {
        return forcing<R>(p, (double)s * h);
    }
    template <int R, int D>
    static __device__ __forceinline__ void rhs(const double* p, const double* y, double frc, double* f)
    {
        if constexpr (R == ABM_RHS_LCR) {
            // the three pieces of g as one selected line: no branch in the
            // unrolled rows
            const bool in = fabs(y[0]) < 1.0;
            const double c = p[3] - p[2];
            const double g = fma(in ? p[2] : p[3], y[0], in ? 0.0 : y[0] < 0.0 ? c : -c);
            f[0] = y[1] - g;
            f[1] = -p[0] * y[1] - y[0] + frc;
        } else {
            rhs_eval_forced<R, D>(p, y, frc, f);
        }
    }
    template <int R, int D>
    static __device__ __forceinline__ void rhs0(const double* p, const double* y, double* f)
    {
        rhs_eval<R, D>(p, 0.0, y, f);
    }
};

namespace plainblk {

constexpr int kB = kPlainBlock;          // steps per block, rows per chunk
constexpr int kThreads = 512;
constexpr int kWaves = kThreads / kWave;
constexpr int kLag = 3;                  // the workers' newest chunk for block q is q - kLag
constexpr int kSlots = kPlainSlots;      // partial slots, by block mod kSlots
constexpr int kFan = kPlainFan;          // partials summed by one workgroup
constexpr int kRing = kPlainRing;        // chunks in the ring that publishes them
constexpr int kNear = 256;               // near table: weights -64 .. 191 (zero below 0)
constexpr int kDump = kWave + 4;         // rows that only take the sequencer's spare stores
constexpr int kAlone = 5;                // waves that sum chunks when workgroup 0 is alone
constexpr int kPartsAlone = 1 + kAlone, kPartsGrid = 2;

template <class T>
struct alignas(16) Weight {
    T b, a;
};
// one row of a chunk, or of the states
template <class T, int D>
struct alignas(sizeof(T) * D % 16 == 0 ? 16 : 8) Row {
    T v[D];
};

// LDS of workgroup 0, in T
template <int D, bool PC>
constexpr size_t chain_units(int64_t chunks, bool alone)
{
    constexpr int NW = PC ? D : 1;
    return (size_t)NW * kNear * 2 + kDump * D + 2 * (alone ? kPartsAlone : kPartsGrid) * 2 * D * kB + 2 * kB +
           2 * kB * D + (size_t)(alone ? chunks : 2) * kB * D + (alone ? kAlone * 2 * kB * 2 : 0);
}
// ... of a worker: its chunks, and per wave a weight window, the sums and
// (spilled chunks) one chunk
template <int D>
constexpr size_t worker_units(int nloc, bool spill)
{
    return (size_t)nloc * kB * D + (size_t)kWaves * kB * (4 + 2 * D + (spill ? D : 0));
}

// Poll *flag until it reaches want; false if the bound on polls ran out.
__device__ __forceinline__ bool await(const uint32_t* flag, uint32_t want, uint32_t limit)
{
    for (uint32_t spins = 0; ld_relaxed(flag) < want; ++spins) {
        if (spins >= limit) return false;
        spin_pause();
    }
    return true;
}

// acc += chunk Fc against 64 rows for the components I0 .. I1 - 1; win[x]:
// weights of row - index = x - 63.
template <class T, int D, int I0, int I1>
__device__ __forceinline__ void chunk_mac(const Weight<T>* win, const T* Fc, int lane,
                                          T (&acc)[kB / Num<T>::LR][2][D])
{
    constexpr int LR = Num<T>::LR, RP = kB / LR, GR = kWave / LR;
    const int lr = lane % LR, g = lane / LR;
#pragma unroll 1
    for (int kr = g; kr < LR; kr += GR) {
        Weight<T> w[2 * RP - 1];
#pragma unroll
        for (int x = 0; x < 2 * RP - 1; ++x) w[x] = win[63 + lr - kr + LR * (x - (RP - 1))];
#pragma unroll
        for (int i = I0; i < I1; ++i)
#pragma unroll
            for (int kq = 0; kq < RP; ++kq) {
                const T f = Fc[(kr + LR * kq) * D + i];
#pragma unroll
                for (int j = 0; j < RP; ++j) {
                    acc[j][0][i] = Num<T>::mac(w[j - kq + RP - 1].b, f, acc[j][0][i]);
                    acc[j][1][i] = Num<T>::mac(w[j - kq + RP - 1].a, f, acc[j][1][i]);
                }
            }
    }
}

// Sums of the lane groups: lane l ends with row l's sums in out.  Every wave
// of a block pays this once per target block; exchanging lanes with vector
// moves instead of shuffles (two trips through the LDS unit per double, and
// four selects) took the linear system of 8192 steps from 536 to 528 us, the
// oscillator of 200000 from 20.1 to 19.8 ms and of 10^6 from 145.9 to 140.0;
// in double-double 3.91 to 3.48 ms for one component.  Two and three
// components there shuffle: no slower for two (1.017 us per step either way)
// and faster for three (Lorenz 1.407 against 1.420).
template <class T, int D>
__device__ __forceinline__ void group_sum(T (&acc)[kB / Num<T>::LR][2][D], int lane, T* out)
{
    using M = Num<T>;
    constexpr int RP = kB / Num<T>::LR;
#pragma unroll
    for (int half = RP / 2, mask = 32; half >= 1; half >>= 1, mask >>= 1) {
#pragma unroll
        for (int j = 0; j < half; ++j)
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int i = 0; i < D; ++i) {
                    if constexpr (M::kUnroll || D == 1) {
                        M::exchange(acc[j][u][i], acc[j + half][u][i], mask);
                        acc[j][u][i] = M::add(acc[j][u][i], acc[j + half][u][i]);
                    } else {
                        const bool up = (lane & mask) != 0;
                        const T keep = up ? acc[j + half][u][i] : acc[j][u][i];
                        const T give = up ? acc[j][u][i] : acc[j + half][u][i];
                        acc[j][u][i] = M::add(keep, M::swap(give, mask));
                    }
                }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int i = 0; i < D; ++i) out[u * D + i] = acc[0][u][i];
}

// The chunks c0, c0 + dc, .. <= cmax against the rows of block q: their
// weight windows pass through the wave's window buffer, loaded one ahead.
// chunk(c, n): chunk c (the n-th) in LDS.
template <class T, int D, bool PC, class Chunk>
__device__ __forceinline__ void sum_chunks(const PlainArgs& A, int q, int c0, int dc, int cmax, int lane,
                                           Weight<T>* win, Chunk chunk, T* out)
{
    constexpr int RP = kB / Num<T>::LR, NW = PC ? D : 1;
    T acc[RP][2][D];
#pragma unroll
    for (int j = 0; j < RP; ++j)
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int i = 0; i < D; ++i) acc[j][u][i] = Num<T>::zero();
    T nb[2], na[2];
    auto fetch = [&](int c, int w) {
        const T *tb = (const T*)A.b[w], *ta = (const T*)A.a[w];
        const int64_t at = (int64_t)kB * (q - c - 1) + lane;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            nb[e] = Num<T>::get(tb + at + kWave * e);
            na[e] = Num<T>::get(ta + at + kWave * e);
        }
    };
    auto stage = [&]() {
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            win[lane + kWave * e].b = nb[e];
            win[lane + kWave * e].a = na[e];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    if (c0 <= cmax) fetch(c0, 0);
    for (int c = c0, n = 0; c <= cmax; c += dc, ++n) {
        const T* Fc = chunk(c, n);
        if constexpr (NW == 1) {
            stage();
            if (c + dc <= cmax) fetch(c + dc, 0);
            chunk_mac<T, D, 0, D>(win, Fc, lane, acc);
        } else {
            stage();
            fetch(c, 1);
            chunk_mac<T, D, 0, 1>(win, Fc, lane, acc);
            stage();
            if constexpr (NW == 3) {
                fetch(c, 2);
                chunk_mac<T, D, 1, 2>(win, Fc, lane, acc);
                stage();
            }
            if (c + dc <= cmax) fetch(c + dc, 0);
            chunk_mac<T, D, NW - 1, NW>(win, Fc, lane, acc);
        }
    }
    group_sum<T, D>(acc, lane, out);
}

// Index of the state written after step s (stride 0: the final state only), or -1.
__device__ __forceinline__ int64_t out_index(int64_t s, int64_t N, int64_t stride)
{
    if (stride == 0) return s == N ? 0 : -1;
    if (s % stride == 0) return s / stride;
    return s == N ? s / stride + 1 : -1;
}

// ---------------------------------------------------------------- workgroup 0
template <class T, int R, int D, bool PC>
__device__ __forceinline__ void chain(const PlainArgs& A, T* sm, uint32_t* s_abort)
{
    using M = Num<T>;
    constexpr int NW = PC ? D : 1;
    const bool alone = A.W == 0;
    const int np = alone ? kPartsAlone : kPartsGrid;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int mlast = (int)((A.N - 1) / kB);
    Weight<T>* near = reinterpret_cast<Weight<T>*>(sm);              // [NW][kNear], weight x at x + 64
    Row<T, D>* dump = reinterpret_cast<Row<T, D>*>(sm + (size_t)NW * kNear * 2);
    T* parts = sm + (size_t)NW * kNear * 2 + kDump * D;              // [2][np][2D][64]
    T* frc = parts + (size_t)2 * np * 2 * D * kB;                    // [2][64]
    T* Y = frc + 2 * kB;                                             // [2][64][D]
    T* F = Y + 2 * kB * D;                                           // chunks [64][D]: all, or the last two
    Weight<T>* wins = reinterpret_cast<Weight<T>*>(F + (alone ? (size_t)(mlast + 1) : 2) * kB * D);
    auto chunk_at = [&](int c) { return F + (size_t)(alone ? c : c & 1) * kB * D; };
    auto part_at = [&](int q, int slot) { return parts + ((size_t)(q & 1) * np + slot) * 2 * D * kB; };

    T x0[D], F0[D];
#pragma unroll
    for (int i = 0; i < D; ++i) x0[i] = M::of(A.x0[i]);
    M::template rhs0<R, D>(A.p, x0, F0);

#pragma unroll
    for (int w = 0; w < NW; ++w)
        for (int x = threadIdx.x; x < kNear; x += kThreads) {
            const bool in = x >= 64;
            near[w * kNear + x].b = in ? ((const T*)A.b[w])[x - 64] : M::zero();
            near[w * kNear + x].a = in ? ((const T*)A.a[w])[x - 64] : M::zero();
        }

    // the sums of item j (predictor components, then corrector) of block q
    // that no other wave forms: the k = 0 terms, and the workers' results
    const int gw = wave == 3 ? 0 : wave >= 5 ? wave - 4 : -1;      // waves 3, 5, 6, 7
    auto init = [&](int q) {
        const int src = A.nred ? A.nred : A.W;
        const bool far = !alone && q >= kLag;
        const int64_t n = (int64_t)q * kB + lane;
#pragma unroll
        for (int jj = 0; jj < (2 * D + 3) / 4; ++jj) {
            const int j = gw + 4 * jj;
            if (j < 2 * D) {
                const int i = j < D ? j : j - D;
                const int w = PC ? i : 0;
                const T* tab = (const T*)(j < D ? A.b[w] : A.c[w]);
                T v = M::zero();
#pragma unroll
                for (int e = 0; e < D; ++e)
                    if (e == i) v = M::mul(M::get(tab + n), F0[e]);
                if (far) {
                    if (jj == 0) {
                        // the flags of the sources reach q once their slots hold block q
                        const uint32_t* fl = A.flags + kPlainFlagPad + (A.nred ? A.W : 0);
                        bool ok = true;
                        if (lane < src) ok = await(fl + lane, (uint32_t)q + A.wait_bias, A.spin_limit);
                        if (!__all(ok)) {
                            *s_abort = 1;
                            if (lane == 0) raise_status(A.status, kStatusTimeout);
                            return;
                        }
                    }
                    const T* from = (const T*)(A.nred ? A.rpart : A.part) +
                                    ((size_t)(q % kSlots) * src * 2 * D + j) * kB + lane;
                    T t[kFan];
#pragma unroll
                    for (int e = 0; e < kFan; ++e)
                        t[e] = e < src ? M::ld_agent(from + (size_t)e * 2 * D * kB) : M::zero();
#pragma unroll
                    for (int e = 0; e < kFan; ++e)
                        if (e < src) v = M::add(v, t[e]);
                }
                part_at(q, 0)[j * kB + lane] = v;
            }
        }
    };
    auto force = [&](int q) { frc[(q & 1) * kB + lane] = M::template force<R>(A.p, (int64_t)q * kB + lane + 1, A.h); };
    auto outputs = [&](int m) {
        const int64_t s = (int64_t)m * kB + lane + 1;
        if (s <= A.N) {
            const T* y = Y + ((m & 1) * kB + lane) * D;
            bool ok = true;
#pragma unroll
            for (int i = 0; i < D; ++i) ok = ok && M::finite(y[i]);
            if (!ok) raise_status(A.status, kStatusNonFinite);
            const int64_t w = out_index(s, A.N, A.out_stride);
            if (w >= 0) {
#pragma unroll
                for (int i = 0; i < D; ++i) M::put((T*)A.y_out + w * D + i, y[i]);
            }
        }
    };
    auto give_up = [&]() {
        // the run is incomplete: its final state reads NaN
        if (threadIdx.x < D) {
            const int64_t last = out_index(A.N, A.N, A.out_stride);
            ((T*)A.y_out)[last * D + threadIdx.x] = M::nan();
        }
    };

    if (wave == 0) {
        constexpr int GS = !M::kUnroll ? 1 : NW == 1 ? 4 : NW == 2 ? 2 : 1;
        __builtin_amdgcn_s_setprio(3);
        double p[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) p[i] = A.p[i];
        // h^alpha, and times 1 / Gamma(alpha + 2), b_0, a_0 (as newest takes them)
        T ha[D], gi[D], b0[D], a0[D], x1[D];
        bool deriv = false;
#pragma unroll
        for (int i = 0; i < D; ++i) {
            const int w = PC ? i : 0;
            ha[i] = M::power(A.h, A.alpha[w]);
            gi[i] = M::mul(ha[i], M::recip(((const T*)A.gam[w])[1]));
            b0[i] = M::newest_weight(M::mul(ha[i], ((const T*)A.b[w])[0]));
            a0[i] = M::newest_weight(M::mul(ha[i], ((const T*)A.a[w])[0]));
            x1[i] = M::of(A.alpha[w] > 1.0 ? A.x1[i] : 0.0);
            deriv = deriv || A.alpha[w] > 1.0;
        }
        if (lane == 0 && A.out_stride > 0) {
#pragma unroll
            for (int i = 0; i < D; ++i) ((T*)A.y_out)[i] = x0[i];
        }
        // f and y are stored by all lanes at once, lane 0 into its row and the
        // others beside it, so that no step changes the execution mask
        Row<T, D>* const spare = dump + lane;
        T P[2 * D], nxt[2 * D];
#pragma unroll
        for (int j = 0; j < 2 * D; ++j) nxt[j] = M::zero();
        for (int m = 0; m <= mlast; ++m) {
            __syncthreads();
            if (*s_abort) {
                give_up();
                return;
            }
            const int rows = (int)(A.N - (int64_t)m * kB < kB ? A.N - (int64_t)m * kB : kB);
            const T fr = frc[(m & 1) * kB + lane];
            // this lane's row: start term and h^alpha times the sums over the
            // older chunks (base), which are large beside the sums over the
            // newest two (P): kept apart, so that the 64 to 127 terms added
            // one by one round at the size of P
            T base[2 * D];
#pragma unroll
            for (int i = 0; i < D; ++i) base[i] = x0[i];
            if (deriv) {
                const T t = M::time((int64_t)m * kB + lane + 1, A.h);
#pragma unroll
                for (int i = 0; i < D; ++i) base[i] = M::mul_add(t, x1[i], x0[i]);
            }
#pragma unroll
            for (int i = 0; i < D; ++i) base[D + i] = base[i];
#pragma unroll
            for (int j = 0; j < 2 * D; ++j) {
                T v = part_at(m, 0)[j * kB + lane];
                for (int e = 1; e < np; ++e) v = M::add(v, part_at(m, e)[j * kB + lane]);
                base[j] = M::mul_add(ha[j % D], v, base[j]);
                P[j] = nxt[j];
                nxt[j] = M::zero();
            }
            Row<T, D>* Fm = lane == 0 ? reinterpret_cast<Row<T, D>*>(chunk_at(m)) : spare;
            Row<T, D>* Ym = lane == 0 ? reinterpret_cast<Row<T, D>*>(Y + (m & 1) * kB * D) : spare;
            Row<T, D> Fp;                     // f of the row before, not yet scattered
#pragma unroll
            for (int i = 0; i < D; ++i) Fp.v[i] = M::zero();
            // weights of the row before against this lane's rows of this
            // block and the next, GS rows at a time, one group ahead
            const Weight<T>* wl = near + 64 + lane;
            Weight<T> wc[GS][NW], wn[GS][NW];
            auto weights = [&](int r0, int e) {
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    wc[e][w] = wl[w * kNear - r0 - e];
                    wn[e][w] = wl[w * kNear + 64 - r0 - e];
                }
            };
#pragma unroll
            for (int e = 0; e < GS; ++e) weights(0, e);
            auto group = [&](int r0, int at) {         // rows r0 .. r0 + GS - 1
                Weight<T> vc[GS][NW], vn[GS][NW];
#pragma unroll
                for (int e = 0; e < GS; ++e)
#pragma unroll
                    for (int w = 0; w < NW; ++w) {
                        vc[e][w] = wc[e][w];
                        vn[e][w] = wn[e][w];
                    }
#pragma unroll
                for (int e = 0; e < GS; ++e)
                    if (r0 + GS < kB) weights(r0 + GS, e);
#pragma unroll
                for (int e = 0; e < GS; ++e) {
                    const int r = r0 + e;
                    T yP[D], fP[D], C[D];
                    Row<T, D> y;
                    const T f_t = M::lane(fr, r);
                    // lane r's value broadcast, the newest term added to it
#pragma unroll
                    for (int i = 0; i < D; ++i) {
                        yP[i] = M::newest_predictor(b0[i], Fp.v[i], M::lane(M::mul_add(ha[i], P[i], base[i]), r));
                        C[i] = M::newest(a0[i], Fp.v[i], M::lane(M::mul_add(ha[i], P[D + i], base[D + i]), r));
                    }
                    M::template rhs<R, D>(p, yP, f_t, fP);
#pragma unroll
                    for (int i = 0; i < D; ++i) y.v[i] = M::mac_state(gi[i], fP[i], C[i]);
                    // the row before's f into the later rows (row l of this
                    // block: weight l - r, of the next one: 64 + l - r; rows
                    // already done receive what is never read)
#pragma unroll
                    for (int i = 0; i < D; ++i) {
                        const int w = PC ? i : 0;
                        P[i] = M::mac_near(vc[e][w].b, Fp.v[i], P[i]);
                        P[D + i] = M::mac_near(vc[e][w].a, Fp.v[i], P[D + i]);
                        nxt[i] = M::mac_near(vn[e][w].b, Fp.v[i], nxt[i]);
                        nxt[D + i] = M::mac_near(vn[e][w].a, Fp.v[i], nxt[D + i]);
                    }
                    M::template rhs<R, D>(p, y.v, f_t, Fp.v);
                    Fm[at + e] = Fp;
                    Ym[at + e] = y;
                }
            };
            // rows past the last step are computed and not used
            if constexpr (M::kUnroll) {
                // every lane index a constant
#pragma unroll
                for (int r0 = 0; r0 < kB; r0 += GS) {
                    if (r0 % 16 == 0 && r0 >= rows) break;
                    group(r0, lane == 0 ? r0 : 0);
                }
            } else {
                for (int r0 = 0; r0 < rows; r0 += GS) {
                    // Nearly all of the loop's instructions take 8 bytes, and
                    // those that straddle an 8-byte boundary are fetched late:
                    // its first one is put where most of them do not (us per
                    // step on and 4 bytes off a boundary: linear 0.429 and
                    // 0.475, oscillator 1.145 and 1.015, Lorenz 1.53 and 1.42)
                    if constexpr (D == 1)
                        asm volatile(".p2align 3");
                    else
                        asm volatile(".p2align 3\n\ts_nop 0");
                    __builtin_amdgcn_sched_barrier(0);
                    group(r0, lane == 0 ? r0 : 0);
                }
            }
            // the block's last f into the next block's rows: weight l
#pragma unroll
            for (int i = 0; i < D; ++i) {
                const Weight<T> w = near[(PC ? i : 0) * kNear + 64 + lane];
                nxt[i] = M::mac_near(w.b, Fp.v[i], nxt[i]);
                nxt[D + i] = M::mac_near(w.a, Fp.v[i], nxt[D + i]);
            }
        }
        __syncthreads();
        return;
    }

    // the other waves: block 0's sums, then block m + 1's while block m runs
    if (gw >= 0) init(0);
    if (wave == 1) force(0);
    const int fw = wave == 2 ? 0 : wave == 3 ? 1 : wave >= 5 ? wave - 3 : -1;   // waves 2, 3, 5, 6, 7
    const int slot = alone ? 1 + fw : wave == 2 ? 1 : 0;           // of the chunk sums; 0: none
    if (fw >= 0 && slot > 0) {
#pragma unroll
        for (int j = 0; j < 2 * D; ++j) part_at(0, slot)[j * kB + lane] = M::zero();
    }
    for (int m = 0; m <= mlast; ++m) {
        __syncthreads();
        if (*s_abort) return;
        const int q = m + 1;
        if (wave == 1 && m >= 1) {
            if (!alone) {
                // chunk m - 1 to the workers, then the progress flag: m chunks published
                const T* Fc = chunk_at(m - 1);
                T* ring = (T*)A.ring + (size_t)((m - 1) % kRing) * kB * D;
#pragma unroll
                for (int i = 0; i < D; ++i) M::st_agent(ring + i * kB + lane, Fc[i * kB + lane]);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                if (lane == 0) st_release(A.flags, (uint32_t)m);
            }
            outputs(m - 1);
        }
        if (q <= mlast) {
            if (wave == 1) force(q);
            if (gw >= 0) init(q);
            if (fw >= 0 && slot > 0) {
                T s[2 * D];
                if (alone) {
                    sum_chunks<T, D, PC>(A, q, fw, kAlone, q - 2, lane, wins + fw * 2 * kB,
                                         [&](int c, int) { return (const T*)chunk_at(c); }, s);
                } else {
                    constexpr int RP = kB / M::LR;
                    T acc[RP][2][D];
#pragma unroll
                    for (int j = 0; j < RP; ++j)
#pragma unroll
                        for (int u = 0; u < 2; ++u)
#pragma unroll
                            for (int i = 0; i < D; ++i) acc[j][u][i] = M::zero();
                    if (q >= 2) {
                        const T* Fc = chunk_at(q - 2);
                        if constexpr (NW == 1) {
                            chunk_mac<T, D, 0, D>(near + 128, Fc, lane, acc);
                        } else {
                            chunk_mac<T, D, 0, 1>(near + 128, Fc, lane, acc);
                            chunk_mac<T, D, 1, 2>(near + kNear + 128, Fc, lane, acc);
                            if constexpr (NW == 3)
                                chunk_mac<T, D, NW - 1, NW>(near + (NW - 1) * kNear + 128, Fc, lane, acc);
                        }
                    }
                    group_sum<T, D>(acc, lane, s);
                }
#pragma unroll
                for (int j = 0; j < 2 * D; ++j) part_at(q, slot)[j * kB + lane] = s[j];
            }
        }
    }
    __syncthreads();
    if (wave == 1) outputs(mlast);
}

// -------------------------------------------------------------------- workers
template <class T, int R, int D, bool PC>
__device__ __forceinline__ void worker(const PlainArgs& A, int w, T* sm, uint32_t* s_abort)
{
    using M = Num<T>;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int mlast = (int)((A.N - 1) / kB);
    const int W = A.W, nloc = A.nloc;
    T* hist = sm;                                                    // [nloc][64][D]
    Weight<T>* win = reinterpret_cast<Weight<T>*>(sm + (size_t)nloc * kB * D) + wave * 2 * kB;
    T* red = sm + (size_t)nloc * kB * D + (size_t)kWaves * 2 * kB * 2;   // [waves][2D][64]
    T* spill = (T*)A.spill + (size_t)w * A.nspill * kB * D;         // chunks beyond nloc
    T* back = red + (size_t)kWaves * 2 * D * kB + wave * kB * D;     // this wave's copy of one of them
    for (int q = kLag; q <= mlast; ++q) {
        const int cnew = q - kLag;                                   // newest chunk of block q
        const bool mine = cnew % W == w;
        // progress: chunk cnew published (its owner), and slot q mod kSlots
        // read for block q - kSlots, which workgroup 0 did while block
        // q - kSlots - 1 ran; chunk q - kSlots - 1 is published after that
        const int need = mine ? cnew + 1 : q - kSlots;
        if (tid == 0 && need > 0 && !await(A.flags, (uint32_t)need + A.wait_bias, A.spin_limit)) {
            raise_status(A.status, kStatusTimeout);
            *s_abort = 1;
        }
        __syncthreads();
        if (*s_abort) return;
        if (mine) {
            const T* ring = (const T*)A.ring + (size_t)(cnew % kRing) * kB * D;
            const int l = cnew / W;
            if (tid < kB * D) {
                const T v = M::ld_agent(ring + tid);
                if (l < nloc)
                    hist[(size_t)l * kB * D + tid] = v;
                else
                    spill[(size_t)(l - nloc) * kB * D + tid] = v;
            }
            __threadfence_block();
            __syncthreads();
        }
        T s[2 * D];
        // this wave's local chunks wave, wave + 8, ..: chunk l is c = w + W l
        sum_chunks<T, D, PC>(A, q, w + W * wave, W * kWaves, cnew, lane, win,
                             [&](int, int n) -> const T* {
                                 const int l = wave + kWaves * n;
                                 if (l < nloc) return hist + (size_t)l * kB * D;
                                 __builtin_amdgcn_wave_barrier();
#pragma unroll
                                 for (int i = 0; i < D; ++i)
                                     back[i * kB + lane] = spill[(size_t)(l - nloc) * kB * D + i * kB + lane];
                                 __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                                 __builtin_amdgcn_wave_barrier();
                                 return back;
                             },
                             s);
#pragma unroll
        for (int j = 0; j < 2 * D; ++j) red[((size_t)wave * 2 * D + j) * kB + lane] = s[j];
        __syncthreads();
        if (tid < 2 * D * kB) {
            T v = red[tid];
#pragma unroll
            for (int e = 1; e < kWaves; ++e) v = M::add(v, red[(size_t)e * 2 * D * kB + tid]);
            M::st_agent((T*)A.part + ((size_t)(q % kSlots) * W + w) * 2 * D * kB + tid, v);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) st_release(A.flags + kPlainFlagPad + w, (uint32_t)q);
    }
}

// ------------------------------------------------------------------- reducers
template <class T, int D>
__device__ __forceinline__ void reducer(const PlainArgs& A, int j, uint32_t* s_abort)
{
    using M = Num<T>;
    const int tid = threadIdx.x;
    const int mlast = (int)((A.N - 1) / kB);
    const int w0 = j * kFan, nw = A.W - w0 < kFan ? A.W - w0 : kFan;
    for (int q = kLag; q <= mlast; ++q) {
        bool ok = true;
        if (tid < nw) ok = await(A.flags + kPlainFlagPad + w0 + tid, (uint32_t)q + A.wait_bias, A.spin_limit);
        if (tid == kWave && q > kSlots) ok = await(A.flags, (uint32_t)(q - kSlots) + A.wait_bias, A.spin_limit);
        if (!ok) {
            raise_status(A.status, kStatusTimeout);
            *s_abort = 1;
        }
        __syncthreads();
        if (*s_abort) return;
        if (tid < 2 * D * kB) {
            const T* from = (const T*)A.part + ((size_t)(q % kSlots) * A.W + w0) * 2 * D * kB + tid;
            T t[kFan];
#pragma unroll
            for (int e = 0; e < kFan; ++e)
                t[e] = e < nw ? M::ld_agent(from + (size_t)e * 2 * D * kB) : M::zero();
            T v = t[0];
#pragma unroll
            for (int e = 1; e < kFan; ++e)
                if (e < nw) v = M::add(v, t[e]);
            M::st_agent((T*)A.rpart + ((size_t)(q % kSlots) * A.nred + j) * 2 * D * kB + tid, v);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) st_release(A.flags + kPlainFlagPad + A.W + j, (uint32_t)q);
    }
}

template <class T, int R, int D, bool PC>
__global__ __launch_bounds__(kThreads) void k_plain(PlainArgs A)
{
    extern __shared__ __align__(16) double lds[];
    __shared__ uint32_t s_abort;
    T* sm = reinterpret_cast<T*>(lds);
    if (A.gate) {
        const uint32_t bits = ld_relaxed(A.gate);
        if (!(bits & kStatusTimeout)) {
            if (bits && blockIdx.x == 0 && threadIdx.x == 0) raise_status(A.status, bits);
            return;
        }
    }
    if (threadIdx.x == 0) s_abort = 0;
    __syncthreads();
    const int g = blockIdx.x;
    if (g == 0)
        chain<T, R, D, PC>(A, sm, &s_abort);
    else if (g <= A.W)
        worker<T, R, D, PC>(A, g - 1, sm, &s_abort);
    else
        reducer<T, D>(A, g - 1 - A.W, &s_abort);
}

// LDS of a launch.  Several workgroups: more than half a CU's, so that no two
// of them share a CU.
template <class T, int D, bool PC>
size_t lds_bytes(const PlainArgs& A)
{
    const int64_t chunks = (A.N + kB - 1) / kB;
    size_t n = chain_units<D, PC>(chunks, A.W == 0);
    if (A.W > 0 && worker_units<D>(A.nloc, A.nspill > 0) > n)
        n = worker_units<D>(A.nloc, A.nspill > 0);
    n *= sizeof(T);
    return A.W > 0 && n < (size_t)84 * 1024 ? (size_t)84 * 1024 : n;
}

template <class T, int R, int D, bool PC>
hipError_t launch(const PlainArgs& A, hipStream_t st)
{
    const size_t shmem = lds_bytes<T, D, PC>(A);
    const void* fn = reinterpret_cast<const void*>(&k_plain<T, R, D, PC>);
    hipError_t e = allow_lds(fn, shmem);
    if (e != hipSuccess) return e;
    if (A.W == 0 || A.gate) {
        hipLaunchKernelGGL((k_plain<T, R, D, PC>), dim3(1 + A.W + A.nred), dim3(kThreads), shmem, st, A);
        return hipGetLastError();
    }
    PlainArgs a = A;
    void* args[] = {&a};
    return hipLaunchCooperativeKernel(fn, dim3(1 + A.W + A.nred), dim3(kThreads), args, (unsigned)shmem, st);
}

template <class T>
hipError_t launch_kind(const PlainArgs& A, int kind, hipStream_t st)
{
    switch (kind) {
    case ABM_RHS_LINEAR: return launch<T, ABM_RHS_LINEAR, 1, false>(A, st);
    case ABM_RHS_DUFFING: return launch<T, ABM_RHS_DUFFING, 2, false>(A, st);
    case ABM_RHS_LORENZ: return launch<T, ABM_RHS_LORENZ, 3, false>(A, st);
    case ABM_RHS_POLY: return launch<T, ABM_RHS_POLY, 1, false>(A, st);
    case ABM_RHS_LCR: return launch<T, ABM_RHS_LCR, 2, false>(A, st);
    case ABM_RHS_DIAG: return launch<T, ABM_RHS_DIAG, 2, false>(A, st);
    case kRhsCount + ABM_RHS_DUFFING: return launch<T, ABM_RHS_DUFFING, 2, true>(A, st);
    case kRhsCount + ABM_RHS_LORENZ: return launch<T, ABM_RHS_LORENZ, 3, true>(A, st);
    case kRhsCount + ABM_RHS_LCR: return launch<T, ABM_RHS_LCR, 2, true>(A, st);
    case kRhsCount + ABM_RHS_DIAG: return launch<T, ABM_RHS_DIAG, 2, true>(A, st);
    default: return hipErrorInvalidValue;
    }
}

template <class T>
size_t chain_lds(int d, bool pc, int64_t chunks, bool alone)
{
    size_t n = 0;
    switch (d * 2 + (pc ? 1 : 0)) {
    case 2: n = chain_units<1, false>(chunks, alone); break;
    case 4: n = chain_units<2, false>(chunks, alone); break;
    case 5: n = chain_units<2, true>(chunks, alone); break;
    case 6: n = chain_units<3, false>(chunks, alone); break;
    case 7: n = chain_units<3, true>(chunks, alone); break;
    default: return ~(size_t)0;
    }
    return n * sizeof(T);
}

// local chunks a worker's LDS holds
template <class T>
int worker_chunks(int d)
{
    const size_t fixed = d == 1   ? worker_units<1>(0, true)
                         : d == 2 ? worker_units<2>(0, true)
                                  : worker_units<3>(0, true);
    return (int)((kPlainLds / sizeof(T) - fixed) / ((size_t)kB * d));
}

}  // namespace plainblk
}  // namespace abm

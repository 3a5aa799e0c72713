// In-place mixed-radix FFT on LDS for any even length L = 2 n <= 512 with
// factors 2, 3, 5, 7, in two or three stages.
//
// The forward transform is decimation in frequency: stage i splits the
// sequence into groups of M = L / (r_0 .. r_{i-1}) slots and transforms the
// r_i slots j + r M / r_i of a group in place, each result q times
// w_M^(j q).  The result of frequency q_0 + r_0 q_1 + r_0 r_1 q_2 ends in slot
// q_0 s_0 + q_1 s_1 + q_2 (s_i = the slot stride of stage i, the last one 1).
// The inverse runs the stages backwards (decimation in time) and returns to
// natural order.  A butterfly reads and writes the same slots, so a stage
// needs one barrier, no second buffer and no register array sized for the
// longest length, and the digit order is free: the Fourier-domain product and
// the passes' global reads and writes only need each slot's frequency.
//
// The first radix r_0 is even, so the zero half of the padded input is
// exactly its inputs r >= r_0 / 2, and the discarded half of the inverse its
// outputs r >= r_0 / 2: the first stage reads n values straight from global
// memory and the last one writes n values straight back.
#pragma once
#include "dev_common.h"
#include "fft_device.h"

namespace vie {

// Stage plan: L = r0 * r1 * rl (r1 = 1: two stages).  rl = 1 leaves the last
// stage a pointwise one.
struct MixPlan {
    int L;
    int r0, r1, rl;
    int s0;             // slot stride of the first stage, L / r0
    unsigned m_s0;      // quotients by s0, rl and r1 (mix_div)
    unsigned m_rl;
    unsigned m_r1;
};

// Plan of an even length (false: no plan with these radices).  max_rl bounds
// the last radix of a z pass, which holds three sequences' butterflies in
// registers at once.
bool mix_plan(int L, int max_rl, MixPlan& p);

// i / d for 0 <= i < 2^16, m = ceil(2^32 / d) (0 stands for d = 1)
__device__ __forceinline__ int mix_div(int i, unsigned m)
{
    return m ? (int)__umulhi((unsigned)i, m) : i;
}

// ---- short transforms beyond fft_device.h's 2, 3, 4, 5, 7, 8

// cos and sin of 2 pi num / den, 0 <= num / den <= 1/8 (Taylor series, below
// the rounding of the last bit)
constexpr double cx_cos(double x)
{
    double s = 1.0, t = 1.0;
    for (int k = 1; k < 14; ++k) {
        t *= -x * x / ((2 * k - 1) * (2 * k));
        s += t;
    }
    return s;
}
constexpr double cx_sin(double x)
{
    double s = x, t = x;
    for (int k = 1; k < 14; ++k) {
        t *= -x * x / ((2 * k) * (2 * k + 1));
        s += t;
    }
    return s;
}
constexpr double kTwoPi = 6.283185307179586476925;
// cos(2 pi r / R): reduced to an eighth of a turn
constexpr double root_cos(int r, int R)
{
    r %= R;
    if (r < 0) r += R;
    if (2 * r > R) r = R - r;                                     // even in the angle
    if (4 * r > R) return -root_cos(R - 2 * r, 2 * R);             // cos(pi - a) = -cos a
    if (8 * r > R) return cx_sin(kTwoPi * (R - 4 * r) / (4.0 * R));   // cos a = sin(pi/2 - a)
    return cx_cos(kTwoPi * r / R);
}
constexpr double root_sin(int r, int R) { return root_cos(4 * r - R, 4 * R); }   // sin a = cos(a - pi/2)

// spacing of the floats around |x| < 1, x != 0
constexpr double float_spacing(double x)
{
    double u = 1.0 / (1 << 24);
    for (x = x < 0 ? -x : x; x < 0.5; x *= 2) u /= 2;
    return u;
}

// exp(2 pi i r / R) as constants of type T.  In FP32 not the nearest floats but,
// within two spacings, the pair whose modulus is nearest to one (a tenth of the
// weight on the phase): a modulus error is a gain, the same in the forward and
// the inverse transform and along every axis, and adds up, while the phase
// errors of the two directions cancel.  Mean gain of a forward and inverse
// transform of 240 = 16 x 15 -2.4e-8 with the nearest floats, -1.4e-8 so.
template <typename T, int R>
struct RootTab {
    T c[R] = {}, s[R] = {};
    constexpr RootTab()
    {
        for (int r = 0; r < R; ++r) {
            const double cr = root_cos(r, R), sr = root_sin(r, R);
            c[r] = (T)cr;
            s[r] = (T)sr;
            if (sizeof(T) == 8 || 8 * r % R == 0) continue;   // (quarters are exact, eighths symmetric)
            double best = 1.0;
            for (int i = -2; i <= 2; ++i)
                for (int j = -2; j <= 2; ++j) {
                    const T ct = (T)((double)(T)cr + i * float_spacing(cr));
                    const T st = (T)((double)(T)sr + j * float_spacing(sr));
                    const double ec = (double)ct - cr, es = (double)st - sr;
                    const double radial = ec * cr + es * sr, tangential = es * cr - ec * sr;
                    const double v = radial * radial + 0.1 * tangential * tangential;
                    if (v < best) {
                        best = v;
                        c[r] = ct;
                        s[r] = st;
                    }
                }
        }
    }
};

// a * exp(DIR 2 pi i r / R), r a compile-time constant after unrolling
template <int R, int DIR, typename T>
__device__ __forceinline__ c2<T> mul_root(c2<T> a, int r)
{
    constexpr RootTab<T, R> tab;
    if (r == 0) return a;
    if (4 * r == R) return mul_i<DIR>(a);
    if (2 * r == R) return mk<T>(-a.x, -a.y);
    const T c = tab.c[r], s = (T)DIR * tab.s[r];
    return mk<T>(a.x * c - a.y * s, a.x * s + a.y * c);
}

template <int R, int DIR, typename T>
__device__ __forceinline__ void dft_mix(c2<T>* a);

// length A B with A, B coprime (the prime-factor map needs no twiddles)
template <int A, int B, int DIR, typename T>
__device__ __forceinline__ void dft_pfa(c2<T>* a)
{
    constexpr int R = A * B;
    c2<T> t[B][A];
#pragma unroll
    for (int j = 0; j < B; ++j) {
#pragma unroll
        for (int i = 0; i < A; ++i) t[j][i] = a[(B * i + A * j) % R];
        dft_mix<A, DIR>(t[j]);
    }
#pragma unroll
    for (int i = 0; i < A; ++i) {
        c2<T> u[B];
#pragma unroll
        for (int j = 0; j < B; ++j) u[j] = t[j][i];
        dft_mix<B, DIR>(u);
        // the frequency k with k = i (mod A) and k = j (mod B)
#pragma unroll
        for (int j = 0; j < B; ++j)
#pragma unroll
            for (int k = 0; k < R; ++k)
                if (k % A == i && k % B == j) a[k] = u[j];
    }
}

// length A B, any A, B (decimation in frequency with constant twiddles)
template <int A, int B, int DIR, typename T>
__device__ __forceinline__ void dft_ct(c2<T>* a)
{
    constexpr int R = A * B;
    c2<T> t[B][A];
#pragma unroll
    for (int j = 0; j < B; ++j) {
#pragma unroll
        for (int i = 0; i < A; ++i) t[j][i] = a[j + B * i];
        dft_mix<A, DIR>(t[j]);
#pragma unroll
        for (int q = 0; q < A; ++q) t[j][q] = mul_root<R, DIR>(t[j][q], j * q);
    }
#pragma unroll
    for (int q = 0; q < A; ++q) {
        c2<T> u[B];
#pragma unroll
        for (int j = 0; j < B; ++j) u[j] = t[j][q];
        dft_mix<B, DIR>(u);
#pragma unroll
        for (int j = 0; j < B; ++j) a[q + A * j] = u[j];
    }
}

template <int R, int DIR, typename T>
__device__ __forceinline__ void dft_mix(c2<T>* a)
{
    if constexpr (R == 1) return;
    else if constexpr (R == 6) dft_pfa<2, 3, DIR>(a);
    else if constexpr (R == 9) dft_ct<3, 3, DIR>(a);
    else if constexpr (R == 10) dft_pfa<2, 5, DIR>(a);
    else if constexpr (R == 12) dft_pfa<4, 3, DIR>(a);
    else if constexpr (R == 15) dft_pfa<3, 5, DIR>(a);
    else if constexpr (R == 16) dft_ct<4, 4, DIR>(a);
    else dftR<R, DIR>(a);
}

// first stage, forward: the R outputs (before their twiddles) of inputs
// a[0 .. R/2), the other half zero: even outputs are the transform of a,
// odd ones that of a_r w_R^r
template <int R, typename T>
__device__ __forceinline__ void dft_half_in(const c2<T>* a, c2<T>* y)
{
    constexpr int H = R / 2;
    c2<T> e[H], o[H];
#pragma unroll
    for (int r = 0; r < H; ++r) {
        e[r] = a[r];
        o[r] = mul_root<R, -1>(a[r], r);
    }
    dft_mix<H, -1>(e);
    dft_mix<H, -1>(o);
#pragma unroll
    for (int q = 0; q < H; ++q) {
        y[2 * q] = e[q];
        y[2 * q + 1] = o[q];
    }
}

// first stage, inverse: the outputs r < R/2 of all R inputs
template <int R, typename T>
__device__ __forceinline__ void dft_half_out(const c2<T>* y, c2<T>* a)
{
    constexpr int H = R / 2;
    c2<T> e[H], o[H];
#pragma unroll
    for (int q = 0; q < H; ++q) {
        e[q] = y[2 * q];
        o[q] = y[2 * q + 1];
    }
    dft_mix<H, 1>(e);
    dft_mix<H, 1>(o);
#pragma unroll
    for (int r = 0; r < H; ++r) a[r] = e[r] + mul_root<R, 1>(o[r], r);
}

// twiddle w_L^m (forward) or its conjugate (inverse) times a
template <int DIR, typename T>
__device__ __forceinline__ c2<T> mix_tw(c2<T> a, const c2<T>* tws, int m)
{
    const c2<T> w = tws[m];
    return DIR < 0 ? a * w : mulc(a, w);
}

// the middle stage of `nseq` sequences, slot p of sequence s at
// buf[p * S + s], consecutive threads on consecutive sequences
template <int R, int DIR, int NSEQ, int S, typename T>
__device__ __forceinline__ void mix_middle(c2<T>* buf, const MixPlan& p, const c2<T>* tws, int tid, int nt)
{
    const int total = NSEQ * p.r0 * p.rl;
#pragma unroll 1
    for (int e = tid; e < total; e += nt) {
        const int s = e % NSEQ, t = e / NSEQ;
        const int b = mix_div(t, p.m_rl), j = t - b * p.rl;
        c2<T>* q = buf + (b * p.s0 + j) * S + s;
        c2<T> a[R];
        const int st = p.rl * S;
#pragma unroll
        for (int r = 0; r < R; ++r) a[r] = q[r * st];
        const int step = j * p.r0;
        if (DIR > 0) {
#pragma unroll
            for (int r = 1; r < R; ++r) a[r] = mix_tw<DIR>(a[r], tws, r * step);
        }
        dft_mix<R, DIR>(a);
        if (DIR < 0) {
#pragma unroll
            for (int r = 1; r < R; ++r) a[r] = mix_tw<DIR>(a[r], tws, r * step);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) q[r * st] = a[r];
    }
}

template <int DIR, int NSEQ, int S, typename T>
__device__ __forceinline__ void mix_middle_any(c2<T>* buf, const MixPlan& p, const c2<T>* tws, int tid, int nt)
{
    switch (p.r1) {
    case 4: mix_middle<4, DIR, NSEQ, S>(buf, p, tws, tid, nt); break;
    case 5: mix_middle<5, DIR, NSEQ, S>(buf, p, tws, tid, nt); break;
    case 6: mix_middle<6, DIR, NSEQ, S>(buf, p, tws, tid, nt); break;
    case 7: mix_middle<7, DIR, NSEQ, S>(buf, p, tws, tid, nt); break;
    case 8: mix_middle<8, DIR, NSEQ, S>(buf, p, tws, tid, nt); break;
    case 9: mix_middle<9, DIR, NSEQ, S>(buf, p, tws, tid, nt); break;
    case 10: mix_middle<10, DIR, NSEQ, S>(buf, p, tws, tid, nt); break;
    default: break;
    }
}

// frequency of the first slot of last-stage group b (the others follow at
// steps of L / rl): q_0 + r_0 q_1 with b = q_0 r_1 + q_1
__device__ __forceinline__ int mix_freq(const MixPlan& p, int b)
{
    if (p.r1 == 1) return b;
    const int q0 = mix_div(b, p.m_r1);
    return q0 + p.r0 * (b - q0 * p.r1);
}

}  // namespace vie

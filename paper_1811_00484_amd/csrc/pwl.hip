// Piecewise-linear (PWL) basis, eq. 7a-7b: twelve unknowns per voxel (the
// pulse and three linear functions per current component) and the sixty
// unique defining tensors of Sec. II-B (ten basis pairs l <= l' of six
// dyadic components each), every one held in Tucker form.
//
// The matvec is the five-pass scheme of the pulse basis with the twelve
// components as four groups of three:
//   X+, Y+   the pulse kernels on (l, q) = 4 right-hand sides of 3 components
//   Z        this file: per pencil group, the forward z FFT of all twelve
//            components, the Fourier-domain sum over the sixteen (l, l')
//            blocks, the inverse z FFT
//   Y-, X-   the pulse kernels, X- with the contrast epilogue
//            y = eps_c x - chi (N x)
// The operator acts on coefficients of the mass-normalised basis (linear
// functions scaled by sqrt 12, unit self products), in which that epilogue is
// exact; the blocks carry the factor sqrt 12 per linear function in their
// cores.
//
// The Fourier-domain sum.  Block (l, l') of the Galerkin sum is a convolution
// with K_ll'(E) = Nt^(l,l')(-E).  For a stored pair (a, b), a <= b, with
// T = the transform of the parity-embedded Nt^(a,b) (eq. 13-14 per pencil):
//   K^_ab = sigma T,   K^_ba = T,   sigma = -1 iff exactly one of a, b is 0,
// because reflecting every axis multiplies Nt^(a,b) by sigma and
// Nt^(a,b)(-E) = Nt^(b,a)(E).  The adjoint takes conj(T) with sigma moved to
// the (b, a) block.  T is symmetric over the dyadic pair (p, q), so each
// block is the 3 x 3 product of the pulse basis.
//
// The magnetic operator K (eq. 5) in the same basis runs through the same
// kernels with the operator family as a template argument: thirty stored
// tensors (ten pairs x xy, xz, yz, the block views' slots 3..5), the
// antisymmetric 3 x 3 product Kt_qp = -Kt_pq, and, since K's sum is a
// convolution over m - m' (test function at the observation voxel),
//   K^_ab = T,   K^_ba = sigma T.
// The coupled JM operator of eq. 4 takes [J; M] as two right-hand sides of
// the N and of the K product and combines them per voxel.
//
// Kernel layout: the V rows of every stored tensor, V_c(k1, k2, :) =
// U1_c(k1, :) (G_c x2 U2_c(k2, :)), come from a kernel that runs first.  A
// workgroup of the z pass takes one mirror group of pencils (four; two or one
// where they do not fit), builds the group's N^ tables from V and the z
// factors and keeps all ten pairs' (or as many as the LDS holds) while the
// right-hand sides go by.  The twelve pencils of each of the group's (k1, k2)
// are transformed in place in LDS (mix_fft.h) and every thread then owns one
// Fourier position: twelve values in, the sixteen blocks accumulated in
// registers, twelve values out.
//
// Signs: N^_(l,p),(l',q) at a mirrored position is the octant's value times
// d_(l,p) d_(l',q), d_(l,p) = (-1)^(f_p + f_(l-1)) with f_a = 1 on a mirrored
// axis (K: times (-1)^(f1 + f2 + f3) too), so twelve values change sign on
// the way in and on the way out instead of sixty table entries.
//
// What bounds it: at 120^3 complex64 a group issues about 38 k cycles of vector
// instructions per SIMD set (0.9 ms in all) in phases that alternate with LDS
// traffic behind barriers, one 960-thread workgroup per CU (vector units 62 %
// busy, LDS 26 %, of which a third bank conflicts); leaving phases out
// of a copy, the tables take 0.5 ms, the product 0.3, the transforms and the
// rest 0.6.  The previous kernel (V contracted in every group, a table entry
// read per sign, stages through two barriers) took 3.6 ms for the pass, 1.36
// now; whole products, MI355X: 120^3 4.63 -> 2.14 ms, 36 x 45 x 50 complex128
// adjoint 0.90 -> 0.28 ms, the coupled product at 60^3 1.95 -> 0.87 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <iterator>
#include <string>
#include <utility>

#include "krylov.h"
#include "mix_fft.h"
#include "v_rows.h"

#include "vie.h"
#include "vie_internal.h"

namespace vie {
vie_status fail(vie_status st, const std::string& msg);
vie_status hip_fail(hipError_t e, const char* where);
}  // namespace vie

namespace {

using namespace vie;

size_t al256(size_t b) { return (b + 255) & ~(size_t)255; }

// components per stored pair and the first slot of the block views: N keeps
// all six, K the three off-diagonal ones (slots 3..5)
template <int FAM>
constexpr int pwl_nc()
{
    return FAM ? 3 : 6;
}

// ---------------------------------------------------------------------------
// One slab of canonical (k1, k2): k1 in [k10, k10 + k1n), k2 likewise.
struct PwlSlab {
    int k10, k1n;
    int k20, k2n;
};

// V[(((k2 - k20) 10 nc + nc b + c) k1n + k1 - k10) rs + g] for every stored
// tensor, zero for g beyond its z rank (rs: pwl_v_stride): one workgroup per
// (k2, tensor).
template <typename T, int FAM>
__global__ void __launch_bounds__(kVNT) k_pwl_v(const PwlBlock<T>* __restrict__ blk, int rmax, int rs, PwlSlab sl,
                                                c2<T>* __restrict__ V)
{
    constexpr int NC = pwl_nc<FAM>();
    const int k2 = sl.k20 + blockIdx.x, bc = blockIdx.y;
    const int b = bc / NC, c = 6 - NC + bc % NC;
    const OpView& v = blk[b].v;
    const int r1 = v.r[c][0], r2 = v.r[c][1], r3 = v.r[c][2];
    v_rows<T>(blk[b].core + v.core_off[c], blk[b].fac + v.fac_off[c][0] + (long)sl.k10 * r1,
              blk[b].fac + v.fac_off[c][1] + (long)k2 * r2, r1, r2, r3, r2 * r3, r3, 1, sl.k1n, rmax, rs, false,
              V + ((long)blockIdx.x * 10 * NC + bc) * sl.k1n * rs);
}

// ---------------------------------------------------------------------------
// table tasks (64 k3 of one tensor) a wavefront can hold for a second group
constexpr int kPwlHold = 8;

// elements that the batched reads of V run past its last row (batches of
// sixteen at most, of which a row has its whole fours)
constexpr int kPwlPast = 12;

struct PwlZArgs {
    int n[3];
    int nq;      // neighbouring groups (k1, k1 + 1) per workgroup, 1 or 2
    int L1, L2;
    int nrhs;    // right-hand sides, walked from blockIdx.y in steps of gridDim.y
    int rs;      // V stride per tensor
    PwlSlab sl;  // of this launch
};

// threads per workgroup at most: one Fourier position each
template <typename T>
constexpr int pwl_max_nt()
{
    return sizeof(T) == 4 ? 1024 : 512;
}

// acc += a b, acc -= a b
template <bool NEG, typename T>
__device__ __forceinline__ void cmac(c2<T>& acc, c2<T> a, c2<T> b)
{
    fma_c(acc, NEG ? mk<T>(-a.x, -a.y) : a, b);
}

// The N^ tables lie in LDS position by position, a row per k3 of the PB pairs'
// tensors: with compile-time offsets a thread reads its row from one address
// register.  Rows of an odd number of 16-byte units spread eight consecutive
// rows over all banks.
template <typename T, int FAM, int PB>
constexpr int pwl_row()
{
    constexpr int t = PB * pwl_nc<FAM>();
    constexpr int u = (t + 1) / 2;
    return sizeof(T) == 4 ? 2 * (u | 1) : (t | 1);
}

// acc +- (a0 x0 + a1 x1 (+ a2 x2)): the products of one row of a block, summed
// by themselves.  Added one by one to acc, the twelve products of an output
// make a chain of 24 roundings of the growing sum; four sums of three round
// 0.77 times as much (random blocks, FP32).
template <bool NEG, typename T>
__device__ __forceinline__ void row3(c2<T>& acc, c2<T> a0, c2<T> x0, c2<T> a1, c2<T> x1, c2<T> a2, c2<T> x2)
{
    c2<T> s = a0 * x0;
    fma_c(s, a1, x1);
    fma_c(s, a2, x2);
    acc = NEG ? acc - s : acc + s;
}
template <bool NEG, bool DIFF, typename T>
__device__ __forceinline__ void row2(c2<T>& acc, c2<T> a0, c2<T> x0, c2<T> a1, c2<T> x1)
{
    c2<T> s = a0 * x0;
    cmac<DIFF>(s, a1, x1);
    acc = NEG ? acc - s : acc + s;
}

// the (a, b) and (b, a) blocks of stored pair B on one Fourier position.
// N (FAM 0): K^_ab = sigma T, K^_ba = T (the sum runs over m' - m), the
// adjoint moves sigma to the (b, a) block; K (FAM 1): K^_ab = T,
// K^_ba = sigma T (the sum runs over m - m'); no adjoint
template <int B, int FAM, bool CONJ, typename T>
__device__ __forceinline__ void pwl_pair(c2<T> (&acc)[12], const c2<T> (&x)[12], const c2<T>* row)
{
    constexpr int la = 3 * kPwlPairs[B][0], lb = 3 * kPwlPairs[B][1];
    constexpr bool sig = (la == 0) != (lb == 0);
    constexpr int NC = pwl_nc<FAM>();
    constexpr bool nab = FAM == 0 && sig && !CONJ, nba = sig && (FAM == 1 || CONJ);
    c2<T> N[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) N[c] = row[c];
    if constexpr (FAM == 0) {
        constexpr int at[3][3] = {{0, 3, 4}, {3, 1, 5}, {4, 5, 2}};
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            const c2<T> n0 = N[at[p][0]], n1 = N[at[p][1]], n2 = N[at[p][2]];
            row3<nab>(acc[la + p], n0, x[lb], n1, x[lb + 1], n2, x[lb + 2]);
            if constexpr (la != lb) row3<nba>(acc[lb + p], n0, x[la], n1, x[la + 1], n2, x[la + 2]);
        }
    } else {
        // Kt_qp = -Kt_pq, zero diagonal (eq. 5: Kt_pq = eps_psq F_s)
        row2<false, false>(acc[la], N[0], x[lb + 1], N[1], x[lb + 2]);
        row2<false, true>(acc[la + 1], N[2], x[lb + 2], N[0], x[lb]);
        row2<true, false>(acc[la + 2], N[1], x[lb], N[2], x[lb + 1]);
        if constexpr (la != lb) {
            row2<nba, false>(acc[lb], N[0], x[la + 1], N[1], x[la + 2]);
            row2<nba, true>(acc[lb + 1], N[2], x[la + 2], N[0], x[la]);
            row2<!nba, false>(acc[lb + 2], N[1], x[la], N[2], x[la + 1]);
        }
    }
}

// PB: pairs whose tables are in LDS together
template <typename T, int G, int FAM, bool CONJ, int PB>
struct PwlZ {
    static constexpr int NC = pwl_nc<FAM>(), ROW = pwl_row<T, FAM, PB>();
    static constexpr int NSEQ = 12 * G, S = NSEQ + 1;
    const PwlZArgs& a;
    const MixPlan& p;
    const PwlBlock<T>* blk;
    const c2<T>* V;     // this group's row of the first tensor
    c2<T>* buf;
    c2<T>* tab;
    const c2<T>* tws;
    int tid, nt;
    int k1, k2;         // canonical
    int i0, j0;         // first pencil (kx, ky) of the group
    bool m1, m2;        // whether the group holds the mirror along x, y

    // pencil pe = s1 | s2 << 1 of the group (G = 2: along x only)
    __device__ __forceinline__ bool exists(int pe) const { return (!(pe & 1) || m1) && (!(pe & 2) || m2); }
    __device__ __forceinline__ long base(int s, long rhs) const
    {
        const int comp = s / G, pe = s % G;
        const int i = (pe & 1) ? a.L1 - i0 : i0, j = (pe & 2) ? a.L2 - j0 : j0;
        return (((rhs * 12 + comp) * a.L2 + j) * a.L1 + i) * a.n[2];
    }

    // inputs of butterfly e of the first stage
    __device__ __forceinline__ void load(c2<T> (&v)[8], const c2<T>* __restrict__ S2, int e, long rhs) const
    {
        const int s = mix_div(e, p.m_s0), j = e - s * p.s0;
        const bool ex = e < NSEQ * p.s0 && exists(s % G);
        const c2<T>* src = S2 + (ex ? base(s, rhs) + j : 0);
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = ex && 2 * r < p.r0 ? src[r * p.s0] : mk<T>(0, 0);
    }

    template <int R>
    __device__ __forceinline__ void first_fwd(c2<T> (&v)[8], const c2<T>* __restrict__ S2, long rhs) const
    {
        const int total = NSEQ * p.s0;
#pragma unroll 1
        for (int e = tid; e < total; e += nt) {
            if (e != tid) load(v, S2, e, rhs);
            const int s = mix_div(e, p.m_s0), j = e - s * p.s0;
            c2<T> o[R];
            dft_half_in<R>(v, o);
            c2<T>* q = buf + j * S + s;
            q[0] = o[0];
#pragma unroll
            for (int r = 1; r < R; ++r) q[r * p.s0 * S] = mix_tw<-1>(o[r], tws, r * j);
        }
    }

    template <int R>
    __device__ __forceinline__ void last_inv(c2<T>* __restrict__ S2, long rhs) const
    {
        constexpr int H = R / 2;
        const int total = NSEQ * p.s0;
#pragma unroll 1
        for (int e = tid; e < total; e += nt) {
            const int s = mix_div(e, p.m_s0), j = e - s * p.s0;
            if (!exists(s % G)) continue;
            c2<T> v[R], o[H];
            const c2<T>* q = buf + j * S + s;
            v[0] = q[0];
#pragma unroll
            for (int r = 1; r < R; ++r) v[r] = mix_tw<1>(q[r * p.s0 * S], tws, r * j);
            dft_half_out<R>(v, o);
            c2<T>* dst = S2 + base(s, rhs) + j;
#pragma unroll
            for (int r = 0; r < H; ++r) dst[r * p.s0] = o[r];
        }
    }

    // the last forward / first inverse stage in place (no twiddles)
    template <int R, int DIR>
    __device__ __forceinline__ void inner() const
    {
        const int total = NSEQ * (p.L / R);
#pragma unroll 1
        for (int e = tid; e < total; e += nt) {
            const int s = e % NSEQ, b = e / NSEQ;
            c2<T>* q = buf + b * R * S + s;
            c2<T> v[R];
#pragma unroll
            for (int r = 0; r < R; ++r) v[r] = q[r * S];
            dft_mix<R, DIR>(v);
#pragma unroll
            for (int r = 0; r < R; ++r) q[r * S] = v[r];
        }
    }
    template <int DIR>
    __device__ __forceinline__ void inner_any() const
    {
        switch (p.rl) {
        case 2: inner<2, DIR>(); break;
        case 3: inner<3, DIR>(); break;
        case 4: inner<4, DIR>(); break;
        case 5: inner<5, DIR>(); break;
        case 6: inner<6, DIR>(); break;
        case 7: inner<7, DIR>(); break;
        case 8: inner<8, DIR>(); break;
        case 9: inner<9, DIR>(); break;
        case 10: inner<10, DIR>(); break;
        case 12: inner<12, DIR>(); break;
        case 15: inner<15, DIR>(); break;
        case 16: inner<16, DIR>(); break;
        default: return;
        }
        __syncthreads();
    }

    // sA, sB = sum over g of V rows (this group's, and with TWO its neighbour's
    // at k1 + 1) times the z factors of one tensor at k3: sixteen factors in
    // flight, skipped in fours beyond the rank (within four the V rows are
    // zero there and the last factor stands in)
    template <bool TWO>
    __device__ __forceinline__ void contract(int t, int b0, int k3, c2<T>& sA, c2<T>& sB) const
    {
        const int b = b0 + t / NC, c = 6 - NC + t % NC;
        const int r3 = blk[b].v.r[c][2];
        const c2<T>* U3 = blk[b].fac + blk[b].v.fac3t_off[c] + min(k3, a.n[2]);
        const c2<T>* va = V + (long)(NC * b0 + t) * a.sl.k1n * a.rs;
        c2<T> eA = mk<T>(0, 0), eB = mk<T>(0, 0);   // even g (odd ones in sA, sB): shorter sums round less
        sA = mk<T>(0, 0);
        sB = mk<T>(0, 0);
        constexpr int CH = sizeof(T) == 4 ? 16 : 8;
        for (int g0 = 0; g0 < r3; g0 += CH) {
            c2<T> u[CH], wA[CH], wB[CH];
#pragma unroll
            for (int h = 0; h < CH; h += 4) {
                if (g0 + h < r3) {
#pragma unroll
                    for (int q = h; q < h + 4; ++q) u[q] = ldg(U3 + (long)min(g0 + q, r3 - 1) * (a.n[2] + 1));
                }
            }
            // V a whole batch at once (scalar loads beside the factors'), into
            // the next row or, from the last one, into kPwlPast elements
#pragma unroll
            for (int q = 0; q < CH; ++q) {
                wA[q] = va[g0 + q];
                if (TWO) wB[q] = va[a.rs + g0 + q];
            }
#pragma unroll
            for (int h = 0; h < CH; h += 4) {
                if (g0 + h < r3) {
#pragma unroll
                    for (int q = h; q < h + 4; ++q) {
                        fma_c(q & 1 ? sA : eA, wA[q], u[q]);
                        if (TWO) fma_c(q & 1 ? sB : eB, wB[q], u[q]);
                    }
                }
            }
        }
        sA = sA + eA;
        sB = sB + eB;
        if (CONJ) {
            sA.y = -sA.y;
            sB.y = -sB.y;
        }
    }

    // N^ tables of pairs b0 .. b0 + nb: a wavefront takes 64 k3 of one tensor
    // at a time (uniform V row, coalesced z factors)
    __device__ __forceinline__ void tables(int b0, int nb) const
    {
        const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), nw = nt >> 6, lane = tid & 63;
        const int tensors = nb * NC, total = tensors * ((a.n[2] + 64) >> 6);
        for (int task = wv; task < total; task += nw) {
            const int t = task % tensors, k3 = (task / tensors) * 64 + lane;
            c2<T> sA, sB;
            contract<false>(t, b0, k3, sA, sB);
            if (k3 <= a.n[2]) tab[k3 * ROW + t] = sA;
        }
    }

    // all ten pairs' tables of two neighbouring groups with one pass over the
    // z factors: the second group's wait in registers (at most kPwlHold tasks
    // a wavefront) until the first group is done
    __device__ __forceinline__ void tables_two(c2<T> (&hold)[kPwlHold]) const
    {
        const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), nw = nt >> 6, lane = tid & 63;
        const int total = 10 * NC * ((a.n[2] + 64) >> 6);
#pragma unroll
        for (int i = 0; i < kPwlHold; ++i) {
            const int task = wv + i * nw;
            if (task < total) {
                const int t = task % (10 * NC), k3 = (task / (10 * NC)) * 64 + lane;
                c2<T> sA;
                contract<true>(t, 0, k3, sA, hold[i]);
                if (k3 <= a.n[2]) tab[k3 * ROW + t] = sA;
            }
        }
    }
    __device__ __forceinline__ void tables_held(const c2<T> (&hold)[kPwlHold]) const
    {
        const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), nw = nt >> 6, lane = tid & 63;
        const int total = 10 * NC * ((a.n[2] + 64) >> 6);
#pragma unroll
        for (int i = 0; i < kPwlHold; ++i) {
            const int task = wv + i * nw;
            if (task < total) {
                const int t = task % (10 * NC), k3 = (task / (10 * NC)) * 64 + lane;
                if (k3 <= a.n[2]) tab[k3 * ROW + t] = hold[i];
            }
        }
    }

    __device__ __forceinline__ void read(c2<T> (&x)[12], const c2<T>* cell, const T (&d)[12]) const
    {
#pragma unroll
        for (int c = 0; c < 12; ++c) x[c] = d[c] * cell[c * G];
    }

    template <int B>
    __device__ __forceinline__ void pair(c2<T> (&acc)[12], c2<T> (&x)[12], const c2<T>* cell, const T (&d)[12],
                                         const c2<T>* row) const
    {
        if constexpr (PB < 10 && B % PB == 0) {   // the next batch of tables
            if (B > 0) __syncthreads();
            tables(B, PB < 10 - B ? PB : 10 - B);
            __syncthreads();
            read(x, cell, d);
        }
        pwl_pair<B, FAM, CONJ>(acc, x, row + NC * (B % PB));
        // finish this pair before the next one's table reads: otherwise all
        // sixty entries are read first and spilled
#pragma unroll
        for (int c = 0; c < 12; ++c) asm volatile("" : "+v"(acc[c].x), "+v"(acc[c].y));
    }
    template <int... B>
    __device__ __forceinline__ void pairs(c2<T> (&acc)[12], const c2<T>* cell, const T (&d)[12], const c2<T>* row,
                                          std::integer_sequence<int, B...>) const
    {
        c2<T> x[12];
        if constexpr (PB == 10) read(x, cell, d);
        (pair<B>(acc, x, cell, d, row), ...);
    }

    __device__ __forceinline__ void product() const
    {
        const int n3 = a.n[2], groups = p.L / p.rl, total = G * p.L;
        // slot and pencil of this thread: along the groups for an odd last
        // radix (LDS stride 2 x odd), along the pencils first for an even one
        const int e = min(tid, total - 1);
        int pe, b, q;
        if (p.rl & 1) {
            q = e / groups;
            b = e - q * groups;
            pe = q / p.rl;
            q -= pe * p.rl;
        } else {
            pe = e % G;
            const int t = e / G;
            q = t / groups;
            b = t - q * groups;
        }
        const int k = mix_freq(p, b) + q * groups;
        const bool f3 = k > n3;
        const int kk = f3 ? p.L - k : k;
        // signs of the mirrored axes (a group of one or two pencils may lie
        // beyond the octant as a whole)
        const T sx = ((pe & 1) != 0) != (i0 != k1) ? (T)-1 : (T)1;
        const T sy = ((pe & 2) != 0) != (j0 != k2) ? (T)-1 : (T)1;
        const T sz = f3 ? (T)-1 : (T)1;
        const T d[12] = {sx, sy, sz, (T)1, sx * sy, sx * sz, sx * sy, (T)1, sy * sz, sx * sz, sy * sz, (T)1};
        c2<T>* cell = buf + (b * p.rl + q) * S + pe;
        c2<T> acc[12];
#pragma unroll
        for (int c = 0; c < 12; ++c) acc[c] = mk<T>(0, 0);
        pairs(acc, cell, d, tab + kk * ROW, std::make_integer_sequence<int, 10>{});
        const T o = FAM ? sx * sy * sz : (T)1;
        if (tid < total) {
#pragma unroll
            for (int c = 0; c < 12; ++c) cell[c * G] = (FAM ? o * d[c] : d[c]) * acc[c];
        }
    }
};

template <typename T, int G, int FAM, bool CONJ, int PB>
__global__ void __launch_bounds__(pwl_max_nt<T>())
    k_pwl_z(c2<T>* __restrict__ S2, const c2<T>* __restrict__ tw, PwlZArgs a, MixPlan p,
            const PwlBlock<T>* __restrict__ blk, const c2<T>* __restrict__ V)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    using Z = PwlZ<T, G, FAM, CONJ, PB>;
    const int n1 = a.n[0], n2 = a.n[1];
    // XCD-wise runs of neighbouring groups (workgroups go round robin over
    // the eight XCDs): their pencils share cache lines
    const int nk1 = (G >= 2 ? 1 : 2) * a.sl.k1n, nx = (nk1 + a.nq - 1) / a.nq, ny = (G == 4 ? 1 : 2) * a.sl.k2n;
    const int per = (nx * ny + 7) / 8;
    const int g = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per || g >= nx * ny) return;
    c2<T>* buf = reinterpret_cast<c2<T>*>(smem_raw);                            // [L][12 G + 1]
    c2<T>* tws = buf + (((size_t)p.L * Z::S + 1) & ~(size_t)1);                  // [L]
    c2<T>* tab = tws + p.L;                                                     // [n3 + 1][ROW], 16-byte aligned
    // the slab's positions, and after them (groups of one pencil along x, of
    // one or two along y) their mirrors, where they have one
    const int ix = (g % nx) * a.nq, jy = g / nx;
    const bool mx = ix >= a.sl.k1n && G == 1, my = jy >= a.sl.k2n;
    const int k1 = a.sl.k10 + (mx ? ix - a.sl.k1n : ix), k2 = a.sl.k20 + (my ? jy - a.sl.k2n : jy);
    if ((mx && (k1 == 0 || k1 == n1)) || (my && (k2 == 0 || k2 == n2))) return;
    const int i0 = mx ? a.L1 - k1 : k1, j0 = my ? a.L2 - k2 : k2;
    const int nq = min(a.nq, nk1 - ix);
    Z z{a,    p,  blk, V + ((long)(k2 - a.sl.k20) * 10 * Z::NC * a.sl.k1n + k1 - a.sl.k10) * a.rs,
        buf,  tab, tws, (int)threadIdx.x, (int)blockDim.x,
        k1,   k2, i0,  j0, G >= 2 && k1 > 0 && k1 < n1, G == 4 && k2 > 0 && k2 < n2};
    c2<T> v[8], hold[kPwlHold];
    z.load(v, S2, z.tid, blockIdx.y);   // in flight while the tables are built
    for (int m = z.tid; m < p.L; m += z.nt) tws[m] = tw[m];
    if constexpr (PB == 10) {
        if (nq == 2) z.tables_two(hold);
        else z.tables(0, 10);
    }
    __syncthreads();
    for (int i = 0; i < nq; ++i) {
        if (i > 0) {
            if constexpr (PB == 10) z.tables_held(hold);   // its first use is barriers away
        }
        for (int rhs = blockIdx.y; rhs < a.nrhs; rhs += gridDim.y) {
            // the stages' addresses are cheap to form again and too many to
            // keep in registers from one pass of this loop to the next
            asm volatile("" : "+v"(z.tid));
            switch (p.r0) {
            case 2: z.template first_fwd<2>(v, S2, rhs); break;
            case 4: z.template first_fwd<4>(v, S2, rhs); break;
            case 6: z.template first_fwd<6>(v, S2, rhs); break;
            case 8: z.template first_fwd<8>(v, S2, rhs); break;
            case 10: z.template first_fwd<10>(v, S2, rhs); break;
            case 12: z.template first_fwd<12>(v, S2, rhs); break;
            case 14: z.template first_fwd<14>(v, S2, rhs); break;
            default: z.template first_fwd<16>(v, S2, rhs); break;
            }
            __syncthreads();
            if (p.r1 > 1) {
                mix_middle_any<-1, Z::NSEQ, Z::S>(buf, p, tws, z.tid, z.nt);
                __syncthreads();
            }
            z.template inner_any<-1>();
            z.product();
            __syncthreads();
            z.template inner_any<1>();
            if (p.r1 > 1) {
                mix_middle_any<1, Z::NSEQ, Z::S>(buf, p, tws, z.tid, z.nt);
                __syncthreads();
            }
            switch (p.r0) {
            case 2: z.template last_inv<2>(S2, rhs); break;
            case 4: z.template last_inv<4>(S2, rhs); break;
            case 6: z.template last_inv<6>(S2, rhs); break;
            case 8: z.template last_inv<8>(S2, rhs); break;
            case 10: z.template last_inv<10>(S2, rhs); break;
            case 12: z.template last_inv<12>(S2, rhs); break;
            case 14: z.template last_inv<14>(S2, rhs); break;
            default: z.template last_inv<16>(S2, rhs); break;
            }
            // the next right-hand side's, or the next group's first
            if (rhs + (int)gridDim.y < a.nrhs) z.load(v, S2, z.tid, rhs + gridDim.y);
            else if (i + 1 < nq) {
                z.k1 = ++z.i0;
                z.m1 = G >= 2 && z.k1 > 0 && z.k1 < n1;
                z.load(v, S2, z.tid, blockIdx.y);
            }
            __syncthreads();   // the slots are reused
        }
    }
}

// The shapes of the z pass, best first: the largest mirror group (it shares
// its tables) whose positions have a thread each, with as many pairs' tables
// in LDS as fit beside the group's pencils.  The last ones of each type fit
// every z length up to 512.
struct PwlShape {
    int G, PB;
};
template <typename T>
constexpr PwlShape kPwlShapes[] = {{4, 10}, {4, 5}, {2, 10}, {2, 5}, {2, 2}};
template <>
constexpr PwlShape kPwlShapes<double>[] = {{4, 10}, {4, 5}, {2, 10}, {2, 5}, {2, 2}, {1, 5}, {1, 2}, {1, 1}};

template <typename T, int FAM, int G, int PB>
size_t pwl_z_lds(const OpView& v)
{
    const size_t pencils = ((size_t)v.L[2] * (12 * G + 1) + 1) & ~(size_t)1;
    return sizeof(c2<T>) * (pencils + v.L[2] + (size_t)(v.n[2] + 1) * pwl_row<T, FAM, PB>());
}

int pwl_op_nc(const vie_pwl_op& P)
{
    return P.fam ? pwl_nc<1>() : pwl_nc<0>();
}

// V's row length: the largest z rank of the stored tensors, in whole fours, so
// that the z pass reads and sums four at a time without a branch
int pwl_v_stride(const vie_pwl_op& P)
{
    int rs = 1;
    for (int b = 0; b < 10; ++b)
        for (int c = P.fam ? 3 : 0; c < 6; ++c) rs = std::max(rs, P.blk[b]->d.view.r[c][2]);
    return (rs + 3) & ~3;
}

// complex elements of the V rows of k1n k1 and k2n k2
size_t pwl_v_elems(const vie_pwl_op& P, int k1n, int k2n)
{
    return (size_t)k1n * k2n * 10 * pwl_op_nc(P) * pwl_v_stride(P) + kPwlPast;
}

size_t pwl_s2_elems(const OpView& v, int nrhs) { return (size_t)12 * v.L[1] * v.L[0] * v.n[2] * nrhs; }
size_t pwl_s1_elems(const OpView& v, int nrhs) { return (size_t)12 * v.n[2] * v.L[0] * v.n[1] * nrhs; }

// S2, then S1, in whose place the V rows live while S1 is dead (between Y+ and
// Y-).  They exceed it where the z ranks come near 0.4 n3 (ranks of n3 take 2.5
// (n1 + 1) (n2 + 1) / n1 n2 times S1, rows padded to fours on a grid of one
// voxel along z ten times that); S1 then grows to hold them in one piece, since
// a slab of a small grid takes as long as its whole pass: complex64 products,
// MI355X, 18 x 24 x 6 149 us in two slabs, 84 in one, 128 x 126 x 1 503 and 443.
size_t pwl_ws_elems(const vie_pwl_op& P, int nrhs)
{
    const OpView& v = P.blk[0]->d.view;
    return pwl_s2_elems(v, nrhs) + std::max(pwl_s1_elems(v, nrhs), pwl_v_elems(P, v.n[0] + 1, v.n[1] + 1));
}

// the least that a product runs in: S1 as it is (and room for one row of every
// tensor), with the z pass in slabs of (k1, k2)
size_t pwl_ws_least(const vie_pwl_op& P, int nrhs)
{
    const OpView& v = P.blk[0]->d.view;
    return pwl_s2_elems(v, nrhs) + std::max(pwl_s1_elems(v, nrhs), pwl_v_elems(P, 1, 1));
}

template <typename T, int FAM, bool CONJ, int G, int PB>
bool try_pwl_z(const DeviceOp& op, int max_pb, PwlZArgs za, const MixPlan& p, c2<T>* S2, const c2<T>* tw,
               const PwlBlock<T>* blk, const c2<T>* V, hipStream_t s)
{
    const OpView& v = op.view;
    const size_t lds = pwl_z_lds<T, FAM, G, PB>(v);
    if (PB > max_pb || G * v.L[2] > pwl_max_nt<T>() || lds > op.max_lds) return false;
    // two neighbouring groups a workgroup halve the z factor reads, which set
    // the pace of a single one; not where the table tasks exceed what the
    // wavefronts can hold, or where the grid would drop below two workgroups
    // per CU
    const int nk1 = (G >= 2 ? 1 : 2) * za.sl.k1n, ny = (G == 4 ? 1 : 2) * za.sl.k2n;
    const int tasks = 10 * pwl_nc<FAM>() * ((v.n[2] + 64) / 64);
    int waves = (G * v.L[2] + 63) / 64;
    za.nq = 1;
    if (G == 4 && PB == 10 && (long)nk1 * ny >= 1024 && tasks <= kPwlHold * (pwl_max_nt<T>() / 64)) {
        za.nq = 2;
        waves = std::max(waves, (tasks + kPwlHold - 1) / kPwlHold);
    }
    const int nblk = 8 * (((nk1 + za.nq - 1) / za.nq * ny + 7) / 8);
    // right-hand sides share a workgroup's tables where all ten pairs stay in
    // LDS and the grid still holds four workgroups per CU
    int gy = za.nrhs;
    if (PB == 10)
        for (gy = 1; gy < za.nrhs && (long)nblk * gy < 1024;) ++gy;
    auto kern = k_pwl_z<T, G, FAM, CONJ, PB>;
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kern, dim3(nblk, gy), dim3(64 * waves), lds, s, S2, tw, za, p, blk, V);
    return true;
}

template <typename T, int FAM, bool CONJ, int... I>
bool try_pwl_shapes(const DeviceOp& op, int max_pb, const PwlZArgs& za, const MixPlan& p, c2<T>* S2,
                    const c2<T>* tw, const PwlBlock<T>* blk, const c2<T>* V, hipStream_t s,
                    std::integer_sequence<int, I...>)
{
    return (try_pwl_z<T, FAM, CONJ, kPwlShapes<T>[I].G, kPwlShapes<T>[I].PB>(op, max_pb, za, p, S2, tw, blk, V, s) ||
            ...);
}

template <typename T>
hipError_t launch_pwl_z(const vie_pwl_op& P, int conj, c2<T>* S2, c2<T>* V, size_t vcap, int nrhs, hipStream_t s,
                        std::string& err)
{
    const DeviceOp& op = P.blk[0]->d;
    const OpView& v = op.view;
    const int nc = pwl_op_nc(P);
    int max_pb = 10;
    // tuning override: at most this many pairs per table batch where a shape has so few
    if (const char* e = getenv("VIE_PWL_PAIRS_PER_BATCH")) max_pb = std::max(1, std::min(max_pb, atoi(e)));
    MixPlan p;
    if (!mix_plan(v.L[2], 16, p)) {
        err = "the piecewise-linear z pass has no plan for this z length";
        return hipErrorInvalidValue;
    }
    PwlZArgs za;
    for (int a = 0; a < 3; ++a) za.n[a] = v.n[a];
    za.L1 = v.L[0];
    za.L2 = v.L[1];
    za.nrhs = nrhs;
    za.rs = pwl_v_stride(P);
    const c2<T>* tw;
    const PwlBlock<T>* blk;
    if constexpr (sizeof(T) == 8) {
        tw = op.tw64[2];
        blk = P.dev64;
    } else {
        tw = op.tw32[2];
        blk = P.dev32;
    }
    const size_t vlds = v_rows_lds<T>(P.rmax, za.rs);
    auto kv = P.fam ? k_pwl_v<T, 1> : k_pwl_v<T, 0>;
    (void)hipFuncSetAttribute((const void*)kv, hipFuncAttributeMaxDynamicSharedMemorySize, (int)vlds);
    // slabs: all k1 of as many k2 as V has room for, or part of one k2's k1
    const int n1p1 = v.n[0] + 1, n2p1 = v.n[1] + 1;
    const size_t rows = vcap < kPwlPast ? 0 : (vcap - kPwlPast) / ((size_t)10 * nc * za.rs);
    if (rows < 1) {
        err = "the workspace has no room for a row of V";
        return hipErrorInvalidValue;
    }
    const int k1n = (int)std::min<size_t>(rows, n1p1), k2n = (int)std::min<size_t>(rows / k1n, n2p1);
    constexpr auto shapes = std::make_integer_sequence<int, (int)std::size(kPwlShapes<T>)>{};
    auto slab = [&]() {
        hipLaunchKernelGGL(kv, dim3(za.sl.k2n, 10 * nc), dim3(kVNT), vlds, s, blk, P.rmax, za.rs, za.sl, V);
        for (int m : {max_pb, 10}) {   // an override that no shape serves is left out
            const bool ok = P.fam  ? try_pwl_shapes<T, 1, false>(op, m, za, p, S2, tw, blk, V, s, shapes)
                            : conj ? try_pwl_shapes<T, 0, true>(op, m, za, p, S2, tw, blk, V, s, shapes)
                                   : try_pwl_shapes<T, 0, false>(op, m, za, p, S2, tw, blk, V, s, shapes);
            if (ok) return hipGetLastError();
        }
        err = "the piecewise-linear z pass does not fit in LDS (z length too large)";
        return hipErrorInvalidValue;
    };
    for (int k20 = 0; k20 < n2p1; k20 += k2n)
        for (int k10 = 0; k10 < n1p1; k10 += k1n) {
            za.sl = {k10, std::min(k1n, n1p1 - k10), k20, std::min(k2n, n2p1 - k20)};
            const hipError_t e = slab();
            if (e != hipSuccess) return e;
        }
    return hipSuccess;
}

// TV: vector element type, T: compute type (T = float with TV = double: the
// FP32 products on FP64 vectors of a refined solve)
template <typename TV, typename T>
hipError_t pwl_matvec(const vie_pwl_op& P, int mode, const c2<TV>* eps, const c2<TV>* x, c2<TV>* y, c2<T>* ws,
                      size_t ws_elems, int nrhs, hipStream_t s, std::string& err)
{
    const DeviceOp& op = P.blk[0]->d;
    const OpView& v = op.view;
    const int nb = 4 * nrhs;   // groups of three components through the pulse passes
    const size_t s2 = pwl_s2_elems(v, nrhs);
    c2<T>* S2 = ws;
    c2<T>* S1 = ws + s2;
    const bool conj = (mode == MODE_AH || mode == MODE_NH);
    // X+ : x -> S1, Y+ : S1 -> S2, Z : S2 in place, Y- : S2 -> S1, X- : S1 -> y
    hipError_t e = run_pass<TV, T>(op, 0, mode, 0, eps, x, nullptr, S1, nb, s, nullptr, err, false, nullptr, 0);
    if (e == hipSuccess) e = run_pass<TV, T>(op, 1, mode, 0, eps, x, S1, S2, nb, s, nullptr, err, false, nullptr, 0);
    if (e == hipSuccess) e = launch_pwl_z<T>(P, conj ? 1 : 0, S2, S1, ws_elems - s2, nrhs, s, err);
    if (e == hipSuccess) e = run_pass<TV, T>(op, 3, mode, 0, eps, x, S2, S1, nb, s, nullptr, err, false, nullptr, 0);
    if (e == hipSuccess) e = run_pass<TV, T>(op, 4, mode, 0, eps, x, S1, y, nb, s, nullptr, err, false, nullptr, 0);
    return e;
}

}  // namespace

namespace vie {
size_t pwl_workspace_least(const vie_pwl_op* op, int dtype, int nrhs)
{
    if (!op || !op->blk[0] || nrhs < 1) return 0;
    return pwl_ws_least(*op, nrhs) * (dtype == VIE_C128 ? sizeof(c2<double>) : sizeof(c2<float>));
}

// FP32 products on complex128 vectors (refined solves)
vie_status pwl_apply_mixed(const vie_pwl_op* op, int mode, const void* eps, const void* x, void* y, void* ws,
                           size_t ws_bytes, hipStream_t s)
{
    std::string err;
    hipError_t e = pwl_matvec<double, float>(*op, mode, (const c2<double>*)eps, (const c2<double>*)x, (c2<double>*)y,
                                             (c2<float>*)ws, ws_bytes / sizeof(c2<float>), 1, s, err);
    if (e != hipSuccess) {
        if (!err.empty()) return fail(VIE_E_UNSUPPORTED, "vie_solve_pwl: " + err);
        return hip_fail(e, "vie_solve_pwl launch");
    }
    return VIE_OK;
}

static size_t jm_pwl_ws_bytes(const vie_pwl_op* op_n, const vie_pwl_op* op_k, int dtype,
                              size_t (*of)(const vie_pwl_op*, int, int))
{
    if (!op_n || !op_k || !op_n->blk[0] || !op_k->blk[0] || (dtype != VIE_C64 && dtype != VIE_C128)) return 0;
    const OpView& v = op_n->blk[0]->d.view;
    const size_t vec = (size_t)2 * 12 * v.n[0] * v.n[1] * v.n[2] * (dtype == VIE_C128 ? 16 : 8);
    return 2 * al256(vec) + std::max(of(op_n, dtype, 2), of(op_k, dtype, 2));
}

size_t jm_pwl_workspace_least(const vie_pwl_op* op_n, const vie_pwl_op* op_k, int dtype)
{
    return jm_pwl_ws_bytes(op_n, op_k, dtype, pwl_workspace_least);
}
}  // namespace vie

extern "C" {

size_t vie_pwl_workspace_bytes(const vie_pwl_op* op, int dtype, int nrhs)
{
    if (!op || !op->blk[0] || nrhs < 1) return 0;
    const size_t el = dtype == VIE_C128 ? sizeof(c2<double>) : sizeof(c2<float>);
    return pwl_ws_elems(*op, nrhs) * el;
}

vie_status vie_pwl_op_query(const vie_pwl_op* op, int n[3], int ranks[10][6][3])
{
    if (!op || !op->blk[0]) return fail(VIE_E_ARG, "vie_pwl_op_query: null operator");
    const OpView& v0 = op->blk[0]->d.view;
    if (n)
        for (int a = 0; a < 3; ++a) n[a] = v0.n[a];
    if (ranks)
        for (int b = 0; b < 10; ++b)
            for (int c = 0; c < 6; ++c)
                for (int a = 0; a < 3; ++a) ranks[b][c][a] = op->blk[b]->d.view.r[c][a];
    return VIE_OK;
}

vie_status vie_matvec_pwl(const vie_pwl_op* op, int kind, int adjoint, int dtype, const void* eps_c, const void* x,
                          void* y, int nrhs, void* ws, size_t ws_bytes, void* stream)
{
    if (!op || !op->blk[0] || !x || !y || !ws) return fail(VIE_E_ARG, "vie_matvec_pwl: null argument");
    if (nrhs < 1 || nrhs > 4096) return fail(VIE_E_ARG, "vie_matvec_pwl: nrhs must be in [1, 4096]");
    if (kind != VIE_OP_A && kind != VIE_OP_N) return fail(VIE_E_ARG, "vie_matvec_pwl: bad kind");
    if (adjoint != 0 && adjoint != 1) return fail(VIE_E_ARG, "vie_matvec_pwl: adjoint must be 0 or 1");
    if (dtype != VIE_C64 && dtype != VIE_C128) return fail(VIE_E_ARG, "vie_matvec_pwl: bad dtype");
    if (op->fam != 0 && (kind != VIE_OP_N || adjoint != 0))
        return fail(VIE_E_UNSUPPORTED, "vie_matvec_pwl: a K operator has the bare forward product (VIE_OP_N) only");
    if (kind == VIE_OP_A && !eps_c) return fail(VIE_E_ARG, "vie_matvec_pwl: eps_c is required for VIE_OP_A");
    if (ws_bytes < pwl_workspace_least(op, dtype, nrhs))
        return fail(VIE_E_ARG, "vie_matvec_pwl: workspace too small");
    const OpView& v = op->blk[0]->d.view;
    const size_t vbytes = (size_t)nrhs * 12 * v.n[0] * v.n[1] * v.n[2] * (dtype == VIE_C128 ? 16 : 8);
    const char* xb = (const char*)x;
    const char* yb = (const char*)y;
    if (!(xb + vbytes <= yb || yb + vbytes <= xb)) return fail(VIE_E_ARG, "vie_matvec_pwl: x and y overlap");
    const int mode = kind == VIE_OP_A ? (adjoint ? MODE_AH : MODE_A) : (adjoint ? MODE_NH : MODE_N);
    hipStream_t s = (hipStream_t)stream;
    std::string err;
    hipError_t e = dtype == VIE_C128
                       ? pwl_matvec<double, double>(*op, mode, (const c2<double>*)eps_c, (const c2<double>*)x,
                                                    (c2<double>*)y, (c2<double>*)ws, ws_bytes / sizeof(c2<double>),
                                                    nrhs, s, err)
                       : pwl_matvec<float, float>(*op, mode, (const c2<float>*)eps_c, (const c2<float>*)x,
                                                  (c2<float>*)y, (c2<float>*)ws, ws_bytes / sizeof(c2<float>), nrhs,
                                                  s, err);
    if (e != hipSuccess) {
        if (!err.empty()) return fail(VIE_E_UNSUPPORTED, "vie_matvec_pwl: " + err);
        return hip_fail(e, "vie_matvec_pwl launch");
    }
    return VIE_OK;
}

size_t vie_jm_pwl_workspace_bytes(const vie_pwl_op* op_n, const vie_pwl_op* op_k, int dtype)
{
    return jm_pwl_ws_bytes(op_n, op_k, dtype, vie_pwl_workspace_bytes);
}

vie_status vie_matvec_jm_pwl(const vie_pwl_op* op_n, const vie_pwl_op* op_k, int dtype, double h, double omega,
                             const void* eps_c, const void* mu_c, const void* x, void* y, void* ws, size_t ws_bytes,
                             void* stream)
{
    if (!op_n || !op_k || !op_n->blk[0] || !op_k->blk[0] || !eps_c || !mu_c || !x || !y || !ws || !(h > 0) ||
        !(omega > 0))
        return fail(VIE_E_ARG, "vie_matvec_jm_pwl: bad argument");
    if (op_n->fam != 0 || op_k->fam != 1)
        return fail(VIE_E_ARG, "vie_matvec_jm_pwl: needs an N operator and a K operator");
    const OpView& v = op_n->blk[0]->d.view;
    for (int a = 0; a < 3; ++a)
        if (op_k->blk[0]->d.view.n[a] != v.n[a]) return fail(VIE_E_ARG, "vie_matvec_jm_pwl: N and K grids differ");
    if (dtype != VIE_C64 && dtype != VIE_C128) return fail(VIE_E_ARG, "vie_matvec_jm_pwl: bad dtype");
    if (ws_bytes < jm_pwl_workspace_least(op_n, op_k, dtype))
        return fail(VIE_E_ARG, "vie_matvec_jm_pwl: workspace too small");
    const long nv = (long)v.n[0] * v.n[1] * v.n[2];
    const size_t vec = (size_t)2 * 12 * nv * (dtype == VIE_C128 ? 16 : 8);
    const char* xb = (const char*)x;
    const char* yb = (const char*)y;
    if (!(xb + vec <= yb || yb + vec <= xb)) return fail(VIE_E_ARG, "vie_matvec_jm_pwl: x and y overlap");
    char* w = (char*)ws;
    void* NX = w;
    void* KX = w + al256(vec);
    void* mw = w + 2 * al256(vec);
    const size_t mb = ws_bytes - 2 * al256(vec);
    hipStream_t s = (hipStream_t)stream;
    // [J; M] as two right-hand sides of each operator
    if (jm_mixed_products && dtype == VIE_C128) {
        // FP64 vectors, products in FP32 (the inner operator of a refined solve)
        std::string err;
        hipError_t he = pwl_matvec<double, float>(*op_n, MODE_N, nullptr, (const c2<double>*)x, (c2<double>*)NX,
                                                  (c2<float>*)mw, mb / sizeof(c2<float>), 2, s, err);
        if (he == hipSuccess)
            he = pwl_matvec<double, float>(*op_k, MODE_N, nullptr, (const c2<double>*)x, (c2<double>*)KX,
                                           (c2<float>*)mw, mb / sizeof(c2<float>), 2, s, err);
        if (he != hipSuccess)
            return err.empty() ? hip_fail(he, "vie_matvec_jm_pwl") : fail(VIE_E_UNSUPPORTED, "vie_matvec_jm_pwl: " + err);
    } else {
        vie_status st = vie_matvec_pwl(op_n, VIE_OP_N, 0, dtype, nullptr, x, NX, 2, mw, mb, stream);
        if (st != VIE_OK) return st;
        st = vie_matvec_pwl(op_k, VIE_OP_N, 0, dtype, nullptr, x, KX, 2, mw, mb, stream);
        if (st != VIE_OK) return st;
    }
    const double EPS0 = 8.8541878128e-12, C0 = 299792458.0;
    const double MU0 = 1.0 / (EPS0 * C0 * C0);
    hipError_t e;
    if (dtype == VIE_C128)
        e = kr_jm_combine<double>((const c2<double>*)eps_c, (const c2<double>*)mu_c, (const c2<double>*)x,
                                  (const c2<double>*)NX, (const c2<double>*)KX, omega * EPS0 * h, omega * MU0 * h,
                                  (c2<double>*)y, nv, 12, s);
    else
        e = kr_jm_combine<float>((const c2<float>*)eps_c, (const c2<float>*)mu_c, (const c2<float>*)x,
                                 (const c2<float>*)NX, (const c2<float>*)KX, omega * EPS0 * h, omega * MU0 * h,
                                 (c2<float>*)y, nv, 12, s);
    if (e != hipSuccess) return hip_fail(e, "vie_matvec_jm_pwl");
    return VIE_OK;
}

}  // extern "C"

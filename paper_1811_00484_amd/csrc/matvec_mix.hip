// The matvec passes for every FFT length without a register-FFT kernel
// (matvec_fast.hip), on the in-place LDS transforms of mix_fft.h, and the
// V tables of the z pass.
//
// X/Y passes: one workgroup per tile of W pencils, slot p of pencil w at
// buf[p * (W + 1) + w].  The first stage reads the rows (contiguous along the
// transform axis) straight into its butterflies, the last one writes its
// frequencies straight to the transposed output, W contiguous elements a
// row; a length up to 144 passes through LDS once.  The inverse passes run
// the same stages backwards.
//
// Z pass: V_c(k1, k2, :) = U1_c(k1, :) G_c x2 U2_c(k2, :) comes from a kernel
// that runs first (k_zv): built inside the z workgroups, as before, its core
// contraction cost more than all of their transforms.  A z workgroup takes
// the mirror quads of two neighbouring k1 (one on small grids), builds their
// N^ tables together, so that every z factor is read once for both, and then
// transforms each right-hand side's pencils against them: first stage from
// global memory, last forward stage + 3 x 3 product + first inverse stage
// fused in registers (a thread holds the three components of one group of
// slots), last inverse stage to global memory.
//
// Against the kernels these replace (stages through two barriers each with
// every length's worst-case register array, 164 VGPRs and scratch; cores
// contracted per quad), whole products, MI355X: 75 x 54 x 35 complex64
// adjoint with four right-hand sides 2.60 -> 0.172 ms, 90^3 complex128
// 1.68 -> 0.395 ms, the coupled product at 96^3 5.66 -> 0.765 ms, 16^3
// 69 -> 34 us.  What bounds them now, by counters: the z pass the issue of
// vector instructions (busy 81 % of the cycles at 96^3 complex64, 53 % on the
// ragged grid, whose 2096 workgroups are two wavefronts a SIMD, 38 % at 90^3
// complex128, where LDS access waits for a third of its cycles on bank
// conflicts); the X/Y passes their traffic: 3.8 to 5.4 TB/s at 120^3 complex64
// and 90^3 complex128 (X- 3.9 and 2.8), where copies reach 4.9 to 6.1, with the
// vector units 12 to 57 % busy.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "mix_fft.h"
#include "v_rows.h"
#include "vie_internal.h"

namespace vie {

// ---------------------------------------------------------------------------
// plans

// Relative cost of a short transform per element (measured order; the
// constant per stage below stands for its LDS round trip and barrier)
static double radix_cost(int r)
{
    switch (r) {
    case 1: return 0;
    case 2: return 2;
    case 3: return 5.5;
    case 4: return 4;
    case 5: return 9;
    case 6: return 9;
    case 7: return 16;
    case 8: return 6.5;
    case 9: return 13;
    case 10: return 12;
    case 12: return 10;
    case 14: return 18;
    case 15: return 16;
    default: return 9.5;
    }
}

bool mix_plan(int L, int max_rl, MixPlan& p)
{
    static const int first[] = {2, 4, 6, 8, 10, 12, 14, 16};
    static const int last[] = {1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 12, 15, 16};
    static const int middle[] = {1, 4, 5, 6, 7, 8, 9, 10};
    double best = 1e30;
    for (int a : first)
        for (int b : middle)
            for (int c : last) {
                if (a * b * c != L || c > max_rl || (b > 1 && c == 1)) continue;
                // (of equal ones not the first radix 10, whose FP32 constants have
                // the largest gain: 120 = 10 x 12 2.1e-8 a round trip, 12 x 10 0.2e-8)
                const double cost =
                    radix_cost(a) + radix_cost(b) + radix_cost(c) + (b > 1 ? 14.0 : 0.0) + (a == 10 ? 0.01 : 0.0);
                if (cost >= best) continue;
                best = cost;
                p.r0 = a;
                p.r1 = b;
                p.rl = c;
            }
    if (best > 1e29) return false;
    auto magic = [](int d) { return d == 1 ? 0u : (unsigned)(((1ull << 32) + d - 1) / d); };
    p.L = L;
    p.s0 = p.r1 * p.rl;
    p.m_s0 = magic(p.s0);
    p.m_rl = magic(p.rl);
    p.m_r1 = magic(p.r1);
    return true;
}

// ---------------------------------------------------------------------------
// X/Y passes.  KIND: 0 = X+, 1 = Y+, 2 = Y-, 3 = X-.  IDENT: the identity in
// place of the transform (debug entry points), leaving the index maps.
constexpr int kMixNT = 256;

template <typename TV, typename T, int W, int KIND>
struct MixXY {
    const c2<T>* in;
    c2<T>* out;
    const c2<TV>* x;
    const c2<TV>* eps;
    c2<TV>* y;
    XYArgs a;
    MixPlan p;
    int row;      // row of the tile (z plane for the x passes, kx for the y passes)
    int p0;       // first pencil
    int npen;     // pencils there are
    long bqc;     // workspace and vector component indices
    long bqv;
    c2<T>* buf;
    const c2<T>* tws;
    int tid;
    static constexpr int S = W + 1;

    // element m of pencil pw on the side that is contiguous along the axis
    __device__ __forceinline__ long row_index(int pw, int m) const
    {
        if (KIND == 0 || KIND == 3) return ((bqv * a.n3 + row) * a.n2 + pw) * a.n1 + m;
        return ((bqc * a.n3 + pw) * a.L1 + row) * a.n2 + m;
    }
    // frequency k of pencil pw on the transposed side
    __device__ __forceinline__ long col_index(int pw, int k) const
    {
        if (KIND == 0 || KIND == 3) return ((bqc * a.n3 + row) * a.L1 + k) * a.n2 + pw;
        return ((bqc * a.L2 + k) * a.L1 + row) * a.n3 + pw;
    }

    template <int R>
    __device__ __forceinline__ void first_fwd() const
    {
        constexpr int H = R / 2;
        const int total = W * p.s0;
#pragma unroll 1
        for (int e = tid; e < total; e += kMixNT) {
            const int w = mix_div(e, p.m_s0), j = e - w * p.s0;
            const int pw = p0 + w;
            c2<T> v[H], o[R];
#pragma unroll
            for (int r = 0; r < H; ++r) {
                v[r] = mk<T>(0, 0);
                if (pw < npen) {
                    const long idx = row_index(pw, j + r * p.s0);
                    if (KIND == 0) {
                        v[r] = cvt<T>(x[idx]);
                        if (a.mode == MODE_AH) {   // pre-scale by conj(chi) = conj(eps) - 1
                            const c2<T> ep = cvt<T>(eps[((long)row * a.n2 + pw) * a.n1 + j + r * p.s0]);
                            v[r] = mk<T>(ep.x - (T)1, -ep.y) * v[r];
                        }
                    } else {
                        v[r] = in[idx];
                    }
                }
            }
            dft_half_in<R>(v, o);
            c2<T>* q = buf + j * S + w;
            q[0] = o[0];
#pragma unroll
            for (int r = 1; r < R; ++r) q[r * p.s0 * S] = mix_tw<-1>(o[r], tws, r * j);
        }
    }

    template <int R>
    __device__ __forceinline__ void last_fwd() const
    {
        const int total = W * (p.L / R), step = p.L / R;
#pragma unroll 1
        for (int e = tid; e < total; e += kMixNT) {
            const int w = e % W, b = e / W;
            const int pw = p0 + w;
            c2<T> v[R];
            const c2<T>* q = buf + b * R * S + w;
#pragma unroll
            for (int r = 0; r < R; ++r) v[r] = q[r * S];
            dft_mix<R, -1>(v);
            if (pw < npen) {
                const int k = mix_freq(p, b);
#pragma unroll
                for (int r = 0; r < R; ++r) out[col_index(pw, k + r * step)] = v[r];
            }
        }
    }

    template <int R>
    __device__ __forceinline__ void first_inv() const
    {
        const int total = W * (p.L / R), step = p.L / R;
#pragma unroll 1
        for (int e = tid; e < total; e += kMixNT) {
            const int w = e % W, b = e / W;
            const int pw = p0 + w;
            c2<T> v[R];
            const int k = mix_freq(p, b);
#pragma unroll
            for (int r = 0; r < R; ++r) v[r] = pw < npen ? in[col_index(pw, k + r * step)] : mk<T>(0, 0);
            dft_mix<R, 1>(v);
            c2<T>* q = buf + b * R * S + w;
#pragma unroll
            for (int r = 0; r < R; ++r) q[r * S] = v[r];
        }
    }

    // one kept element of the output row
    __device__ __forceinline__ void store(int pw, int m, c2<T> v) const
    {
        const long idx = row_index(pw, m);
        if (KIND == 2) {
            out[idx] = v;
            return;
        }
        if (a.mode == MODE_A || a.mode == MODE_AH) {
            const c2<T> u = cvt<T>(x[idx]);
            const c2<T> ep = cvt<T>(eps[((long)row * a.n2 + pw) * a.n1 + m]);
            if (a.mode == MODE_A) v = ep * u - mk<T>(ep.x - (T)1, ep.y) * v;   // eps u - chi (N u)
            else v = conj(ep) * u - v;
        }
        y[idx] = cvt<TV>(v);
    }

    template <int R>
    __device__ __forceinline__ void last_inv() const
    {
        constexpr int H = R / 2;
        const int total = W * p.s0;
#pragma unroll 1
        for (int e = tid; e < total; e += kMixNT) {
            const int w = mix_div(e, p.m_s0), j = e - w * p.s0;
            const int pw = p0 + w;
            if (pw >= npen) continue;
            c2<T> v[R], o[H];
            const c2<T>* q = buf + j * S + w;
            v[0] = q[0];
#pragma unroll
            for (int r = 1; r < R; ++r) v[r] = mix_tw<1>(q[r * p.s0 * S], tws, r * j);
            dft_half_out<R>(v, o);
#pragma unroll
            for (int r = 0; r < H; ++r) store(pw, j + r * p.s0, o[r]);
        }
    }

    __device__ __forceinline__ void ident() const
    {
        if (KIND == 0 || KIND == 1) {
            for (int e = tid; e < W * p.L; e += kMixNT) {
                const int w = e / p.L, m = e - w * p.L;
                const int pw = p0 + w;
                c2<T> v = mk<T>(0, 0);
                if (pw < npen && m < p.L / 2) v = KIND == 0 ? cvt<T>(x[row_index(pw, m)]) : in[row_index(pw, m)];
                buf[m * S + w] = v;
            }
            __syncthreads();
            for (int e = tid; e < W * p.L; e += kMixNT) {
                const int w = e % W, k = e / W;
                if (p0 + w < npen) out[col_index(p0 + w, k)] = buf[k * S + w];
            }
        } else {
            for (int e = tid; e < W * p.L; e += kMixNT) {
                const int w = e % W, k = e / W;
                if (p0 + w < npen) buf[k * S + w] = in[col_index(p0 + w, k)];
            }
            __syncthreads();
            const int n = p.L / 2;
            for (int e = tid; e < W * n; e += kMixNT) {
                const int w = e / n, m = e - w * n;
                if (p0 + w < npen) store(p0 + w, m, buf[m * S + w]);
            }
        }
    }
};

#define VIE_MIX_FIRST(call)                  \
    switch (X.p.r0) {                        \
    case 2: X.template call<2>(); break;     \
    case 4: X.template call<4>(); break;     \
    case 6: X.template call<6>(); break;     \
    case 8: X.template call<8>(); break;     \
    case 10: X.template call<10>(); break;   \
    case 12: X.template call<12>(); break;   \
    case 14: X.template call<14>(); break;   \
    default: X.template call<16>(); break;   \
    }
#define VIE_MIX_LAST(call)                   \
    switch (X.p.rl) {                        \
    case 1: X.template call<1>(); break;     \
    case 2: X.template call<2>(); break;     \
    case 3: X.template call<3>(); break;     \
    case 4: X.template call<4>(); break;     \
    case 5: X.template call<5>(); break;     \
    case 6: X.template call<6>(); break;     \
    case 7: X.template call<7>(); break;     \
    case 8: X.template call<8>(); break;     \
    case 9: X.template call<9>(); break;     \
    case 10: X.template call<10>(); break;   \
    case 12: X.template call<12>(); break;   \
    case 15: X.template call<15>(); break;   \
    default: X.template call<16>(); break;   \
    }

template <typename TV, typename T, int W, int KIND, bool IDENT>
__global__ void __launch_bounds__(kMixNT) k_mix_xy(const c2<T>* __restrict__ in, c2<T>* __restrict__ out,
                                                   const c2<TV>* __restrict__ x, const c2<TV>* __restrict__ eps,
                                                   c2<TV>* __restrict__ y, const c2<T>* __restrict__ tw, XYArgs a,
                                                   MixPlan p, const int* __restrict__ rhs_map)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    MixXY<TV, T, W, KIND> X;
    X.in = in;
    X.out = out;
    X.x = x;
    X.eps = eps;
    X.y = y;
    X.a = a;
    X.p = p;
    X.tid = threadIdx.x;
    X.row = blockIdx.y;
    X.p0 = blockIdx.x * W;
    X.npen = (KIND == 0 || KIND == 3) ? a.n2 : a.n3;
    const int q = blockIdx.z % 3, bl = blockIdx.z / 3;
    X.bqc = (long)bl * 3 + q;
    X.bqv = (long)(rhs_map ? rhs_map[bl] : bl) * 3 + q;
    X.buf = reinterpret_cast<c2<T>*>(smem_raw);
    c2<T>* tws = X.buf + (size_t)p.L * (W + 1);
    X.tws = tws;
    if constexpr (IDENT) {
        X.ident();
        return;
    }
    for (int m = X.tid; m < p.L; m += kMixNT) tws[m] = tw[m];
    if constexpr (KIND == 0 || KIND == 1) {
        __syncthreads();
        VIE_MIX_FIRST(first_fwd)
        __syncthreads();
        if (p.r1 > 1) {
            mix_middle_any<-1, W, W + 1>(X.buf, p, tws, X.tid, kMixNT);
            __syncthreads();
        }
        VIE_MIX_LAST(last_fwd)
    } else {
        VIE_MIX_LAST(first_inv)
        __syncthreads();
        if (p.r1 > 1) {
            mix_middle_any<1, W, W + 1>(X.buf, p, tws, X.tid, kMixNT);
            __syncthreads();
        }
        VIE_MIX_FIRST(last_inv)
    }
}

template <typename TV, typename T, int KIND, bool IDENT>
static bool launch_mix_xy(const DeviceOp& op, const c2<T>* in, c2<T>* out, const c2<TV>* x, const c2<TV>* eps,
                          c2<TV>* y, int mode, int nrhs, const int* rhs_map, hipStream_t s)
{
    constexpr int W = sizeof(T) == 4 ? 16 : 8;   // 128 contiguous bytes a row of the transposed side
    const OpView& v = op.view;
    const int axis = (KIND == 0 || KIND == 3) ? 0 : 1;
    MixPlan p;
    if (!mix_plan(v.L[axis], 16, p)) return false;
    const size_t lds = sizeof(c2<T>) * ((size_t)p.L * (W + 1) + p.L);
    if (lds > op.max_lds) return false;
    const c2<T>* tw;
    if constexpr (sizeof(T) == 8) tw = op.tw64[axis];
    else tw = op.tw32[axis];
    const XYArgs a{v.n[0], v.n[1], v.n[2], v.L[0], v.L[1], mode};
    const int npen = axis == 0 ? v.n[1] : v.n[2];
    const int rows = axis == 0 ? v.n[2] : v.L[0];
    auto kern = k_mix_xy<TV, T, W, KIND, IDENT>;
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kern, dim3((npen + W - 1) / W, rows, nrhs * 3), dim3(kMixNT), lds, s, in, out, x, eps, y, tw,
                       a, p, rhs_map);
    return true;
}

template <typename TV, typename T>
bool xy_pass_mix(const DeviceOp& op, int kind, const void* in, void* out, const c2<TV>* x, const c2<TV>* eps,
                 int mode, int nrhs, const int* rhs_map, bool ident, hipStream_t s)
{
    const c2<T>* i = reinterpret_cast<const c2<T>*>(in);
    c2<T>* o = reinterpret_cast<c2<T>*>(out);
    c2<TV>* y = reinterpret_cast<c2<TV>*>(out);
    switch (kind) {
    case 0:
        if (ident) return launch_mix_xy<TV, T, 0, true>(op, nullptr, o, x, eps, nullptr, MODE_N, nrhs, rhs_map, s);
        return launch_mix_xy<TV, T, 0, false>(op, nullptr, o, x, eps, nullptr, mode, nrhs, rhs_map, s);
    case 1: return launch_mix_xy<TV, T, 1, false>(op, i, o, x, eps, nullptr, mode, nrhs, rhs_map, s);
    case 2: return launch_mix_xy<TV, T, 2, false>(op, i, o, x, eps, nullptr, mode, nrhs, rhs_map, s);
    default:
        if (ident) return launch_mix_xy<TV, T, 3, true>(op, i, nullptr, x, eps, y, MODE_N, nrhs, rhs_map, s);
        return launch_mix_xy<TV, T, 3, false>(op, i, nullptr, x, eps, y, mode, nrhs, rhs_map, s);
    }
}

// ---------------------------------------------------------------------------
// V tables: V[((k2 nc + c) (n1 + 1) + k1) rs + g], c the stored components (six,
// or K's three), zero for g beyond the component's z rank (rs: the largest one
// in whole fours, so that the z pass reads and sums four at a time without a
// branch).  One workgroup per (k2, c).
template <typename T>
__global__ void __launch_bounds__(kVNT) k_zv(OpView v, const c2<T>* __restrict__ core, const c2<T>* __restrict__ fac,
                                             int rs, int k20, c2<T>* __restrict__ V)
{
    const int k2 = k20 + blockIdx.x, nc = gridDim.y, ci = blockIdx.y, c = 6 - nc + ci;
    const int r2 = v.r[c][1], n1p1 = v.n[0] + 1;
    v_rows<T>(core + v.core_off[c], fac + v.fac_off[c][0], fac + v.fac_off[c][1] + (long)k2 * r2, v.r[c][0], r2,
              v.r[c][2], r2 * v.r[c][2], v.r[c][2], 1, n1p1, v.rmax, rs, v.cp, V + ((long)blockIdx.x * nc + ci) * n1p1 * rs);
}

int zv_stride(const OpView& v)
{
    int rs = 1;
    for (int c = v.fam ? 3 : 0; c < 6; ++c) rs = rs > v.r[c][2] ? rs : v.r[c][2];
    return (rs + 3) & ~3;
}

size_t zv_elems(const OpView& v)
{
    return (size_t)(v.n[0] + 1) * (v.n[1] + 1) * (v.fam ? 3 : 6) * zv_stride(v);
}

int zv_slab(const OpView& v, size_t cap)
{
    const size_t per = (size_t)(v.n[0] + 1) * (v.fam ? 3 : 6) * zv_stride(v);
    return (int)std::min<size_t>(cap / per, v.n[1] + 1);
}

template <typename T>
void launch_zv(const DeviceOp& op, c2<T>* V, int k20, int k2n, hipStream_t s)
{
    const OpView& v = op.view;
    const c2<T>*core, *fac;
    if constexpr (sizeof(T) == 8) {
        core = op.d64.core;
        fac = op.d64.fac;
    } else {
        core = op.d32.core;
        fac = op.d32.fac;
    }
    const int rs = zv_stride(v);
    const size_t lds = v_rows_lds<T>(v.rmax, rs);
    (void)hipFuncSetAttribute((const void*)k_zv<T>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(k_zv<T>, dim3(k2n, v.fam ? 3 : 6), dim3(kVNT), lds, s, v, core, fac, rs, k20, V);
}

// ---------------------------------------------------------------------------
// Z pass
struct MixZArgs {
    int n[3];
    int L1, L2;
    int nq;         // k1 quads per workgroup (1 or 2)
    int nrhs;       // right-hand sides, walked by every workgroup from blockIdx.y in steps of gridDim.y
    int conj;
    int dense;
    int rs;         // V stride per component
    int k20, k2n;   // canonical k2 of this launch: [k20, k20 + k2n)
    int r3[6];
    int fac3t_off[6];
};

// sequences of a quad: component q of pencil pe = s1 | s2 << 1 at slot
// stride S, index 4 q + pe
constexpr int kZSeq = 12, kZS = 13;

template <typename T, int FAM>
struct MixZ {
    const MixZArgs& a;
    const MixPlan& p;
    c2<T>* buf;
    const c2<T>* tws;
    int tid, nt;
    int k2;
    bool m2;      // k2 has a mirror

    __device__ __forceinline__ bool exists(int pe, bool m1) const { return (!(pe & 1) || m1) && (!(pe & 2) || m2); }
    // first element of sequence s of the quad at k1
    __device__ __forceinline__ long base(int s, int k1, long rhs) const
    {
        const int q = s >> 2, f1 = s & 1, f2 = (s >> 1) & 1;
        const int i = f1 ? a.L1 - k1 : k1, j = f2 ? a.L2 - k2 : k2;
        return (((rhs * 3 + q) * a.L2 + j) * a.L1 + i) * a.n[2];
    }

    template <int R>
    __device__ __forceinline__ void first_fwd(const c2<T>* __restrict__ S2, int k1, bool m1, long rhs) const
    {
        constexpr int H = R / 2;
        const int total = kZSeq * p.s0;
#pragma unroll 1
        for (int e = tid; e < total; e += nt) {
            const int s = mix_div(e, p.m_s0), j = e - s * p.s0;
            c2<T> v[H], o[R];
            const bool ex = exists(s & 3, m1);
            const c2<T>* src = S2 + base(s, k1, rhs) + j;
#pragma unroll
            for (int r = 0; r < H; ++r) v[r] = ex ? src[r * p.s0] : mk<T>(0, 0);
            dft_half_in<R>(v, o);
            c2<T>* q = buf + j * kZS + s;
            q[0] = o[0];
#pragma unroll
            for (int r = 1; r < R; ++r) q[r * p.s0 * kZS] = mix_tw<-1>(o[r], tws, r * j);
        }
    }

    template <int R>
    __device__ __forceinline__ void last_inv(c2<T>* __restrict__ S2, int k1, bool m1, long rhs) const
    {
        constexpr int H = R / 2;
        const int total = kZSeq * p.s0;
#pragma unroll 1
        for (int e = tid; e < total; e += nt) {
            const int s = mix_div(e, p.m_s0), j = e - s * p.s0;
            if (!exists(s & 3, m1)) continue;
            c2<T> v[R], o[H];
            const c2<T>* q = buf + j * kZS + s;
            v[0] = q[0];
#pragma unroll
            for (int r = 1; r < R; ++r) v[r] = mix_tw<1>(q[r * p.s0 * kZS], tws, r * j);
            dft_half_out<R>(v, o);
            c2<T>* dst = S2 + base(s, k1, rhs) + j;
#pragma unroll
            for (int r = 0; r < H; ++r) dst[r * p.s0] = o[r];
        }
    }

    // last forward stage, 3 x 3 product with the quad's tables, first inverse
    // stage.  N^ of a mirrored position is the table's value with the sign of
    // the component's parities along the mirrored axes.
    template <int R>
    __device__ __forceinline__ void product(const c2<T>* tab) const
    {
        const int n3 = a.n[2], n3p1 = n3 + 1;
        const int groups = p.L / R;
#pragma unroll 1
        for (int e = tid; e < 4 * groups; e += nt) {
            // the walk whose LDS rows spread over the banks: for odd R along
            // the groups (stride 13 R), for even R along the four pencils
            int pe, b;
            if (R & 1) {
                pe = (e >= groups) + (e >= 2 * groups) + (e >= 3 * groups);
                b = e - pe * groups;
            } else {
                pe = e & 3;
                b = e >> 2;
            }
            c2<T>* q = buf + b * R * kZS + pe;
            c2<T> x[3][R];
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int r = 0; r < R; ++r) x[c][r] = q[r * kZS + 4 * c];
#pragma unroll
            for (int c = 0; c < 3; ++c) dft_mix<R, -1>(x[c]);
            const int k0 = mix_freq(p, b);
            const bool f1 = pe & 1, f2 = pe & 2;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int k = k0 + r * groups;
                const bool f3 = k > n3;
                const c2<T>* t = tab + (f3 ? p.L - k : k);
                const c2<T> x0 = x[0][r], x1 = x[1][r], x2 = x[2][r];
                if constexpr (FAM == 0) {
                    const T s3 = f1 != f2 ? (T)-1 : (T)1, s4 = f1 != f3 ? (T)-1 : (T)1, s5 = f2 != f3 ? (T)-1 : (T)1;
                    const c2<T> N3 = s3 * t[3 * n3p1], N4 = s4 * t[4 * n3p1], N5 = s5 * t[5 * n3p1];
                    x[0][r] = t[0] * x0 + N3 * x1 + N4 * x2;
                    x[1][r] = N3 * x0 + t[n3p1] * x1 + N5 * x2;
                    x[2][r] = N4 * x0 + N5 * x1 + t[2 * n3p1] * x2;
                } else {
                    // K: xy odd along z, xz along y, yz along x
                    const T s3 = f3 ? (T)-1 : (T)1, s4 = f2 ? (T)-1 : (T)1, s5 = f1 ? (T)-1 : (T)1;
                    const c2<T> N3 = s3 * t[0], N4 = s4 * t[n3p1], N5 = s5 * t[2 * n3p1];
                    x[0][r] = N3 * x1 + N4 * x2;
                    x[1][r] = N5 * x2 - N3 * x0;
                    x[2][r] = mk<T>(0, 0) - (N4 * x0 + N5 * x1);
                }
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) dft_mix<R, 1>(x[c]);
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int r = 0; r < R; ++r) q[r * kZS + 4 * c] = x[c][r];
        }
    }
};

template <typename T, int FAM>
__global__ void __launch_bounds__(512) k_mix_z(c2<T>* __restrict__ S2, const c2<T>* __restrict__ tw, MixZArgs a,
                                               MixPlan p, const c2<T>* __restrict__ V, const c2<T>* __restrict__ fac,
                                               const c2<T>* __restrict__ dense)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    constexpr int NC = FAM ? 3 : 6;
    const int n1 = a.n[0], n2 = a.n[1], n3 = a.n[2], n3p1 = n3 + 1;
    const int tid = threadIdx.x, nt = blockDim.x;
    c2<T>* buf = reinterpret_cast<c2<T>*>(smem_raw);   // [L][13]
    c2<T>* tab = buf + (size_t)p.L * kZS;               // [nq][NC][n3 + 1]
    c2<T>* tws = tab + (size_t)a.nq * NC * n3p1;        // [L]
    // workgroups go round robin over the eight XCDs: give each XCD a run of
    // neighbouring quads, whose pencils share cache lines and z factors
    const int nx = (n1 + 1 + a.nq - 1) / a.nq;
    const int per = (nx * a.k2n + 7) / 8;
    const int g = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per || g >= nx * a.k2n) return;
    const int kA = (g % nx) * a.nq, k2l = g / nx, k2 = a.k20 + k2l;
    const int nq = min(a.nq, n1 + 1 - kA);
    for (int m = tid; m < p.L; m += nt) tws[m] = tw[m];

    // ---- N^ tables of the workgroup's quads, k3 in [0, n3]: a wavefront
    // takes 64 k3 of one component (uniform V, coalesced z factors)
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), nw = nt >> 6, lane = tid & 63;
    const int chunks = (n3p1 + 63) >> 6;
    const T cs = a.conj ? (T)-1 : (T)1;
    for (int task = wv; task < NC * chunks; task += nw) {
        const int c = task % NC, k3 = (task / NC) * 64 + lane;
        const int cc = 6 - NC + c, r3 = a.r3[cc];
        if (k3 > n3) continue;
        if (a.dense) {
            const long per3 = (long)(n1 + 1) * (n2 + 1) * n3p1;
            for (int i = 0; i < nq; ++i) {
                const c2<T> t = dense[cc * per3 + ((long)k2 * (n1 + 1) + kA + i) * n3p1 + k3];
                tab[(i * NC + c) * n3p1 + k3] = mk<T>(t.x, cs * t.y);
            }
            continue;
        }
        const c2<T>* U3 = fac + a.fac3t_off[cc] + k3;
        const c2<T>* va = V + (((long)k2l * NC + c) * (n1 + 1) + kA) * a.rs;
        const c2<T>* vb = nq > 1 ? va + a.rs : va;
        c2<T> s0 = mk<T>(0, 0), s1 = mk<T>(0, 0), u[8], w[8];
        // sixteen z factors in flight; rows beyond the rank meet zeros of V
        auto factors = [&](c2<T>(&d)[8], int g0) {
#pragma unroll
            for (int q = 0; q < 8; ++q) d[q] = U3[(long)min(g0 + q, r3 - 1) * n3p1];
        };
        auto sum = [&](const c2<T>(&d)[8], int g0) {
#pragma unroll
            for (int h = 0; h < 8; h += 4)
                if (g0 + h < r3) {
#pragma unroll
                    for (int q = h; q < h + 4; ++q) {
                        fma_c(s0, va[g0 + q], d[q]);
                        fma_c(s1, vb[g0 + q], d[q]);
                    }
                }
        };
        factors(u, 0);
        for (int g0 = 0; g0 < r3; g0 += 16) {
            if (g0 + 8 < r3) factors(w, g0 + 8);
            sum(u, g0);
            if (g0 + 16 < r3) factors(u, g0 + 16);
            if (g0 + 8 < r3) sum(w, g0 + 8);
        }
        tab[c * n3p1 + k3] = mk<T>(s0.x, cs * s0.y);
        if (nq > 1) tab[(NC + c) * n3p1 + k3] = mk<T>(s1.x, cs * s1.y);
    }
    __syncthreads();   // twiddles (the tables have further barriers before their use)

    MixZ<T, FAM> Z{a, p, buf, tws, tid, nt, k2, k2 > 0 && k2 < n2};
    for (int rhs = blockIdx.y; rhs < a.nrhs; rhs += gridDim.y)
        for (int i = 0; i < nq; ++i) {
            const int k1 = kA + i;
            const bool m1 = k1 > 0 && k1 < n1;
            switch (p.r0) {
            case 2: Z.template first_fwd<2>(S2, k1, m1, rhs); break;
            case 4: Z.template first_fwd<4>(S2, k1, m1, rhs); break;
            case 6: Z.template first_fwd<6>(S2, k1, m1, rhs); break;
            case 8: Z.template first_fwd<8>(S2, k1, m1, rhs); break;
            case 10: Z.template first_fwd<10>(S2, k1, m1, rhs); break;
            case 12: Z.template first_fwd<12>(S2, k1, m1, rhs); break;
            case 14: Z.template first_fwd<14>(S2, k1, m1, rhs); break;
            default: Z.template first_fwd<16>(S2, k1, m1, rhs); break;
            }
            __syncthreads();
            if (p.r1 > 1) {
                mix_middle_any<-1, kZSeq, kZS>(buf, p, tws, tid, nt);
                __syncthreads();
            }
            const c2<T>* t = tab + (size_t)i * NC * n3p1;
            switch (p.rl) {
            case 1: Z.template product<1>(t); break;
            case 2: Z.template product<2>(t); break;
            case 3: Z.template product<3>(t); break;
            case 4: Z.template product<4>(t); break;
            case 5: Z.template product<5>(t); break;
            case 6: Z.template product<6>(t); break;
            case 7: Z.template product<7>(t); break;
            case 8: Z.template product<8>(t); break;
            default: Z.template product<9>(t); break;
            }
            __syncthreads();
            if (p.r1 > 1) {
                mix_middle_any<1, kZSeq, kZS>(buf, p, tws, tid, nt);
                __syncthreads();
            }
            switch (p.r0) {
            case 2: Z.template last_inv<2>(S2, k1, m1, rhs); break;
            case 4: Z.template last_inv<4>(S2, k1, m1, rhs); break;
            case 6: Z.template last_inv<6>(S2, k1, m1, rhs); break;
            case 8: Z.template last_inv<8>(S2, k1, m1, rhs); break;
            case 10: Z.template last_inv<10>(S2, k1, m1, rhs); break;
            case 12: Z.template last_inv<12>(S2, k1, m1, rhs); break;
            case 14: Z.template last_inv<14>(S2, k1, m1, rhs); break;
            default: Z.template last_inv<16>(S2, k1, m1, rhs); break;
            }
            __syncthreads();   // the slots are reused by the next quad
        }
}

template <typename T>
bool z_pass_mix(const DeviceOp& op, int mode, int nrhs, c2<T>* S2, c2<T>* V, size_t vcap, hipStream_t s)
{
    const OpView& v = op.view;
    const c2<T>*tw, *fac, *dense;
    if constexpr (sizeof(T) == 8) {
        tw = op.tw64[2];
        fac = op.d64.fac;
        dense = op.dense64;
    } else {
        tw = op.tw32[2];
        fac = op.d32.fac;
        dense = op.dense32;
    }
    MixPlan p;
    if (!mix_plan(v.L[2], 9, p)) return false;
    const int nc = v.fam ? 3 : 6;
    MixZArgs a;
    for (int i = 0; i < 3; ++i) a.n[i] = v.n[i];
    a.L1 = v.L[0];
    a.L2 = v.L[1];
    a.nrhs = nrhs;
    a.conj = mode == MODE_AH || mode == MODE_NH;
    a.dense = op.nhat_source == 1;
    a.rs = zv_stride(v);
    for (int c = 0; c < 6; ++c) {
        a.r3[c] = v.r[c][2];
        a.fac3t_off[c] = v.fac3t_off[c];
    }
    // two quads a workgroup share every z factor read; one where that would
    // leave fewer than two workgroups per CU, or where the tables do not fit
    auto lds_of = [&](int nq) {
        return sizeof(c2<T>) * ((size_t)p.L * kZS + (size_t)nq * nc * (v.n[2] + 1) + p.L);
    };
    a.nq = (long)(v.n[0] + 1) * (v.n[1] + 1) >= 1024 && lds_of(2) <= op.max_lds / 2 ? 2 : 1;
    const size_t lds = lds_of(a.nq);
    if (lds > op.max_lds) return false;
    const int n2p1 = v.n[1] + 1, slab = a.dense ? n2p1 : zv_slab(v, vcap);
    if (slab < 1) return false;
    const int groups = 4 * (p.L / p.rl);
    int nt = 64 * ((groups + 63) / 64);
    nt = nt < 64 ? 64 : (nt > 512 ? 512 : nt);
    auto kern = v.fam ? k_mix_z<T, 1> : k_mix_z<T, 0>;
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    for (a.k20 = 0; a.k20 < n2p1; a.k20 += slab) {
        a.k2n = std::min(slab, n2p1 - a.k20);
        if (!a.dense) launch_zv<T>(op, V, a.k20, a.k2n, s);
        const int nblk = 8 * (((v.n[0] + a.nq) / a.nq * a.k2n + 7) / 8);
        // right-hand sides share the tables of a workgroup as far as the grid
        // still holds eight workgroups per CU
        int gy = 1;
        while (gy < nrhs && (long)nblk * gy < 2048) ++gy;
        hipLaunchKernelGGL(kern, dim3(nblk, gy), dim3(nt), lds, s, S2, tw, a, p, (const c2<T>*)V, fac, dense);
    }
    return true;
}

#define VIE_MIX_INST(TV, T)                                                                                    \
    template bool xy_pass_mix<TV, T>(const DeviceOp&, int, const void*, void*, const c2<TV>*, const c2<TV>*, int, \
                                     int, const int*, bool, hipStream_t);
VIE_MIX_INST(float, float)
VIE_MIX_INST(double, double)
VIE_MIX_INST(double, float)
template void launch_zv<float>(const DeviceOp&, c2<float>*, int, int, hipStream_t);
template void launch_zv<double>(const DeviceOp&, c2<double>*, int, int, hipStream_t);
template bool z_pass_mix<float>(const DeviceOp&, int, int, c2<float>*, c2<float>*, size_t, hipStream_t);
template bool z_pass_mix<double>(const DeviceOp&, int, int, c2<double>*, c2<double>*, size_t, hipStream_t);

}  // namespace vie

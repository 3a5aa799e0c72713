// One Tucker (eq. 14) or Tucker+CP (eq. 17) component applied element-wise
// to a vector on its own n1 x n2 x n3 grid, y = D .* x with
// D = G x1 U1 x2 U2 x3 U3: the "decompression and element-wise product" of
// Sec. V-B (Table II, timed in Table IV), done in one pass over x and y with
// no buffer for D.
//
//   Tucker: W(k)   = G x3 U3(k, :)           (r1 x r2, in LDS)
//           V(j,k) = W(k) U2(j, :)^T          (r1 per (j, k); one workgroup per k)
//   CP:     V_l(j,k) = lambda_l U2(j, l) U3(k, l) (the 4-D loop of Sec. V-B)
//   then    D(i,j,k) = U1(i, :) . V(j, k), y = D .* x   (last kernel)
// V of fewer than four columns and rows of few i have kernels of their own
// (k_vk_few, k_apply_flat).
// The last kernel gives a workgroup a tile of i and a run of (j, k) rows: a
// thread keeps U1(i, :) of its i in registers for the whole run, and the rows
// V(j, k), the same for every lane, come by scalar loads, so that the inner
// product costs its multiply-adds and nothing else.  HBM traffic: x in, y out,
// and V (r1 complex per (j, k)).
//
// 300^3, rank 25, complex128, MI355X: 0.94 ms with V read through the vector
// memory unit by every lane (16 rows of k per thread) and W through HBM;
// 0.32 ms now, of which 0.27 apply: 3.2 TB/s of x and y, the vector units 30 %
// busy, three quarters of the wavefronts' time spent waiting (25 complex128
// factors leave three wavefronts a SIMD to hide the loads of x and V).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>

#include "vie.h"
#include "v_rows.h"
#include "vie_internal.h"

namespace vie {
vie_status fail(vie_status st, const std::string& msg);
vie_status hip_fail(hipError_t e, const char* where);
}  // namespace vie

namespace {

using namespace vie;

constexpr int kRMax = 32;    // largest rank per mode
constexpr int kNT = 64;      // threads per workgroup of the apply kernel, one i each
constexpr int kRun = 32;     // (j, k) rows per workgroup of the apply kernel
// A lane per i wastes 64 - n1 lanes of short rows: below kShort the flat walk
// of the (i, j) plane wins at every rank (8 M elements, rank 8 and 25:
// complex64 n1 = 4 200 -> 94 and 291 -> 187 us, 8 117 -> 66 and 170 -> 119, 15
// 77 -> 55 and 153 -> 125; complex128 12 154 -> 135 and 317 -> 314, but 15 116
// -> 117 and 264 -> 288).
template <typename T>
constexpr int kShort = sizeof(T) == 4 ? 17 : 13;
constexpr int kFlatNT = 256; // threads per workgroup of the flat kernel, an (i, j) each
constexpr int kKT = 16;      // k per thread of it
// workgroups that the V kernel may reach by splitting each k's rows of U2: two
// per CU (complex128, rank 25: 64 x 20000 x 1 2207 -> 53 us, 64 x 8000 x 8 922 ->
// 77; 290^3, which keeps one per k, 306, with two 308, with four 316)
constexpr int kVkFill = 512;
constexpr int kFew = 4;      // columns of V below which it has a kernel of its own
constexpr int kFewK = 8;     // k per workgroup of that one

// V(j, k) of a Tucker form: a workgroup contracts the core with U3(k, :) of its
// k and applies it to nj rows of U2.
template <typename T>
__global__ void __launch_bounds__(kVNT) k_vk(const c2<T>* __restrict__ G, const c2<T>* __restrict__ U2,
                                             const c2<T>* __restrict__ U3, c2<T>* __restrict__ V, int n2, int nj, int r1,
                                             int r2, int r3, int rmax)
{
    const long k = blockIdx.x;
    const int j0 = blockIdx.y * nj;
    v_rows<T>(G, U2 + (long)j0 * r2, U3 + k * r3, r2, r3, r1, r3, 1, r2 * r3, min(nj, n2 - j0), rmax, r1, false,
              V + (k * n2 + j0) * r1);
}

// V(j, k) of fewer columns than k_vk has wavefronts (n1, and so r1, of a plane
// or two): a thread holds its row of U2 for kFewK values of k, whose
// contracted cores come by broadcast.  What bounds k_vk there is U2, read again
// for every k by one wavefront of four.
template <typename T>
__global__ void __launch_bounds__(256) k_vk_few(const c2<T>* __restrict__ G, const c2<T>* __restrict__ U2,
                                                const c2<T>* __restrict__ U3, c2<T>* __restrict__ V, int n2, int n3,
                                                int r1, int r2, int r3)
{
    __shared__ c2<T> W[kFewK * (kFew - 1) * kRMax];   // [k][r1][kRMax], zero beyond r2
    const int k0 = blockIdx.y * kFewK, nk = min(kFewK, n3 - k0);
    for (int e = threadIdx.x; e < nk * r1 * kRMax; e += 256) {
        const int b = e % kRMax, t = e / kRMax, a = t % r1;
        const c2<T>* u = U3 + (long)(k0 + t / r1) * r3;
        c2<T> acc = mk<T>(0, 0);
        if (b < r2)
            for (int c = 0; c < r3; ++c) fma_c(acc, G[((long)a * r2 + b) * r3 + c], u[c]);
        W[e] = acc;
    }
    const int j = blockIdx.x * 256 + threadIdx.x;
    const c2<T>* row = U2 + (long)min(j, n2 - 1) * r2;
    c2<T> u[kRMax];
#pragma unroll
    for (int b = 0; b < kRMax; ++b) u[b] = b < r2 ? row[b] : mk<T>(0, 0);
    __syncthreads();
    for (int t = 0; t < nk * r1; ++t) {
        c2<T> even = mk<T>(0, 0), odd = mk<T>(0, 0);
#pragma unroll
        for (int h = 0; h < kRMax; h += 4)
            if (h < r2) {
#pragma unroll
                for (int b = h; b < h + 4; ++b) fma_c(b & 1 ? odd : even, u[b], W[t * kRMax + b]);
            }
        if (j < n2) V[((long)(k0 + t / r1) * n2 + j) * r1 + t % r1] = even + odd;
    }
}

template <typename T>
__global__ void __launch_bounds__(256) k_vjk_cp(const c2<T>* __restrict__ lam, const c2<T>* __restrict__ U2,
                                                const c2<T>* __restrict__ U3, c2<T>* __restrict__ V, int n2, int r)
{
    const int e = blockIdx.x * 256 + threadIdx.x, k = blockIdx.y;   // a column of one k's rows
    if (e >= n2 * r) return;
    V[(long)k * n2 * r + e] = lam[e % r] * (U2[e] * U3[(long)k * r + e % r]);
}

// U1 (n1 x r1) into U1T (r1 x n1), so that the apply kernel's lanes read
// consecutive i of one column
template <typename T>
__global__ void __launch_bounds__(256) k_transpose(const c2<T>* __restrict__ U1, c2<T>* __restrict__ U1T, int n1,
                                                   int r1)
{
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (long)n1 * r1) return;
    const int a = (int)(e / n1), i = (int)(e - (long)a * n1);
    U1T[e] = U1[(long)i * r1 + a];
}

template <typename T, int R>
__global__ void __launch_bounds__(kNT) k_apply(const c2<T>* __restrict__ V, const c2<T>* __restrict__ U1T,
                                               const c2<T>* __restrict__ x, c2<T>* __restrict__ y, int n1, long rows)
{
    const int i = blockIdx.y * kNT + threadIdx.x;
    const int il = min(i, n1 - 1);   // lanes beyond the row compute and do not store
    c2<T> u[R];
#pragma unroll
    for (int a = 0; a < R; ++a) u[a] = U1T[(long)a * n1 + il];
    const long r0 = (long)blockIdx.x * kRun;
    const int nr = (int)min((long)kRun, rows - r0);
    const c2<T>* v = V + r0 * R;
    const c2<T>* xr = x + r0 * n1 + il;
    c2<T>* yr = y + r0 * n1 + il;
    // four rows of x in flight while the four before them are worked on
    c2<T> next[4], cur[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) next[q] = xr[(long)min(q, nr - 1) * n1];
    for (int q0 = 0; q0 < nr; q0 += 4) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            cur[q] = next[q];
            next[q] = xr[(long)min(q0 + 4 + q, nr - 1) * n1];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (q0 + q >= nr) break;
            c2<T> d = mk<T>(0, 0);
#pragma unroll
            for (int a = 0; a < R; ++a) fma_c(d, u[a], v[(q0 + q) * R + a]);
            if (i < n1) yr[(long)(q0 + q) * n1] = d * cur[q];
        }
    }
}

// Rows of fewer than kShort<T> elements: consecutive threads take consecutive
// (i, j), wrapping into the next j, for kKT consecutive k, and read V(j, k)
// through the cache.
template <typename T, int R>
__global__ void __launch_bounds__(kFlatNT) k_apply_flat(const c2<T>* __restrict__ V, const c2<T>* __restrict__ U1T,
                                                        const c2<T>* __restrict__ x, c2<T>* __restrict__ y, int n1,
                                                        int n2, int n3)
{
    const int plane = n1 * n2;   // at most 16 x 65535
    const int p = blockIdx.x * kFlatNT + threadIdx.x;
    if (p >= plane) return;
    const int j = p / n1, i = p - j * n1;
    c2<T> u[R];
#pragma unroll
    for (int a = 0; a < R; ++a) u[a] = U1T[(long)a * n1 + i];
    const int k0 = blockIdx.y * kKT, kend = min(n3, k0 + kKT);
    for (int k = k0; k < kend; ++k) {
        const c2<T>* v = V + ((long)k * n2 + j) * R;
        c2<T> d = mk<T>(0, 0);
#pragma unroll
        for (int a = 0; a < R; ++a) fma_c(d, u[a], v[a]);
        const long o = (long)k * plane + p;
        y[o] = d * x[o];
    }
}

template <typename T, int R>
void launch_apply(int r, const c2<T>* V, const c2<T>* U1T, const c2<T>* x, c2<T>* y, const int n[3], hipStream_t s)
{
    if constexpr (R > 1) {
        if (r < R) return launch_apply<T, R - 1>(r, V, U1T, x, y, n, s);
    }
    if (n[0] < kShort<T>) {
        hipLaunchKernelGGL((k_apply_flat<T, R>), dim3((n[0] * n[1] + kFlatNT - 1) / kFlatNT, (n[2] + kKT - 1) / kKT),
                           dim3(kFlatNT), 0, s, V, U1T, x, y, n[0], n[1], n[2]);
        return;
    }
    const long rows = (long)n[1] * n[2];   // below 2^31: with rows this long, more exceed the memory
    hipLaunchKernelGGL((k_apply<T, R>), dim3((unsigned)((rows + kRun - 1) / kRun), (n[0] + kNT - 1) / kNT), dim3(kNT), 0,
                       s, V, U1T, x, y, n[0], rows);
}

template <typename T>
hipError_t run(const int n[3], const int r[3], int cp, const void* core, const void* u1, const void* u2,
               const void* u3, const void* x, void* y, void* ws, hipStream_t s)
{
    const c2<T>* G = (const c2<T>*)core;
    c2<T>* U1T = (c2<T>*)ws;
    c2<T>* V = U1T + (size_t)n[0] * r[0];
    hipLaunchKernelGGL((k_transpose<T>), dim3((unsigned)(((long)n[0] * r[0] + 255) / 256)), dim3(256), 0, s,
                       (const c2<T>*)u1, U1T, n[0], r[0]);
    if (cp) {
        hipLaunchKernelGGL((k_vjk_cp<T>), dim3((n[1] * r[0] + 255) / 256, n[2]), dim3(256), 0, s, G,
                           (const c2<T>*)u2, (const c2<T>*)u3, V, n[1], r[0]);
    } else if (r[0] < kFew) {
        hipLaunchKernelGGL((k_vk_few<T>), dim3((n[1] + 255) / 256, (n[2] + kFewK - 1) / kFewK), dim3(256), 0, s, G,
                           (const c2<T>*)u2, (const c2<T>*)u3, V, n[1], n[2], r[0], r[1], r[2]);
    } else {
        // rows of U2 in tiles of 64: all of them to one workgroup per k, which
        // contracts the core once, or split over as many as kVkFill allows
        const int rmax = std::max(r[0], std::max(r[1], r[2]));
        const int tiles = (n[1] + 63) / 64, split = std::min(tiles, std::max(1, kVkFill / n[2]));
        const int nj = 64 * ((tiles + split - 1) / split);
        const size_t lds = v_rows_lds<T>(rmax, r[0]);
        (void)hipFuncSetAttribute((const void*)k_vk<T>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        hipLaunchKernelGGL((k_vk<T>), dim3(n[2], (n[1] + nj - 1) / nj), dim3(kVNT), lds, s, G, (const c2<T>*)u2,
                           (const c2<T>*)u3, V, n[1], nj, r[0], r[1], r[2], rmax);
    }
    launch_apply<T, kRMax>(r[0], V, U1T, (const c2<T>*)x, (c2<T>*)y, n, s);
    return hipGetLastError();
}

}  // namespace

extern "C" {

size_t vie_tucker_hadamard_ws_bytes(const int n[3], const int r[3], int, int dtype)
{
    if (!n || !r) return 0;
    const size_t el = dtype == VIE_C128 ? 16 : 8;
    return ((size_t)n[0] * r[0] + (size_t)n[2] * n[1] * r[0]) * el;
}

vie_status vie_tucker_hadamard(const int n[3], const int r[3], int cp, int dtype, const void* core, const void* u1,
                               const void* u2, const void* u3, const void* x, void* y, void* ws, size_t ws_bytes,
                               void* stream)
{
    using namespace vie;
    if (!n || !r || !core || !u1 || !u2 || !u3 || !x || !y)
        return fail(VIE_E_ARG, "vie_tucker_hadamard: null argument");
    if (dtype != VIE_C64 && dtype != VIE_C128) return fail(VIE_E_ARG, "vie_tucker_hadamard: bad dtype");
    if (cp != 0 && cp != 1) return fail(VIE_E_ARG, "vie_tucker_hadamard: cp must be 0 or 1");
    for (int a = 0; a < 3; ++a) {
        if (n[a] < 1 || n[a] > 65535) return fail(VIE_E_ARG, "vie_tucker_hadamard: n_i must be in [1, 65535]");
        if (r[a] < 1 || r[a] > kRMax) return fail(VIE_E_UNSUPPORTED, "vie_tucker_hadamard: ranks must be in [1, 32]");
    }
    if (cp && (r[1] != r[0] || r[2] != r[0]))
        return fail(VIE_E_ARG, "vie_tucker_hadamard: a CP form has r1 = r2 = r3");
    const size_t need = vie_tucker_hadamard_ws_bytes(n, r, cp, dtype);
    if (!ws || ws_bytes < need) return fail(VIE_E_ARG, "vie_tucker_hadamard: workspace too small");
    const size_t el = dtype == VIE_C128 ? 16 : 8;
    const size_t vb = (size_t)n[0] * n[1] * n[2] * el;
    const char* xb = (const char*)x;
    const char* yb = (const char*)y;
    if (xb != yb && !(xb + vb <= yb || yb + vb <= xb))
        return fail(VIE_E_ARG, "vie_tucker_hadamard: x and y overlap without being equal");
    hipStream_t s = (hipStream_t)stream;
    hipError_t e = dtype == VIE_C128 ? run<double>(n, r, cp, core, u1, u2, u3, x, y, ws, s)
                                     : run<float>(n, r, cp, core, u1, u2, u3, x, y, ws, s);
    if (e != hipSuccess) return hip_fail(e, "vie_tucker_hadamard launch");
    return VIE_OK;
}

}  // extern "C"

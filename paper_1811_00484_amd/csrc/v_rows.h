// V rows of one Tucker tensor at one k2, V(k1, :) = U1(k1, :) (G x2 U2(k2, :)):
// the x and y factors of the on-the-fly reconstruction contracted with the
// core before the z pass (eq. 14 without its last factor).
//
// One workgroup: W = G x2 U2(k2, :) into LDS, then a lane per k1 with its row
// of U1 in registers and W read by broadcast, the sums transposed through LDS
// into one contiguous run.  With lanes on the columns instead, every factor
// read served eight lanes only and the vector memory unit set the pace
// (60 tensors on 121 x 121 (k1, k2): 137 us, 65 now).
#pragma once
#include "dev_common.h"

namespace vie {

constexpr int kVNT = 256;     // threads per workgroup: 64 k1 at a time, four shares of the columns

// W rows in batches of eight, whole sixteens wherever more than eight are left
__host__ __device__ inline int v_rows_pad(int r) { return r % 16 > 8 ? (r + 15) / 16 * 16 : (r + 7) / 8 * 8; }
__host__ __device__ inline int v_rows_row(int rmax, int rs) { return (rmax > rs ? rmax : rs) | 1; }

template <typename T>
inline size_t v_rows_lds(int rmax, int rs)
{
    return sizeof(c2<T>) * ((size_t)rmax * ((rmax + 15) / 16 * 16) + (size_t)64 * v_rows_row(rmax, rs));
}

// sums of x ranks a0 .. a0 + CH for this lane's row, columns share, share + 4, ..
template <int CH, typename T>
__device__ __forceinline__ void v_rows_sums(const c2<T> (&u)[16], const c2<T>* Wt, int wrow, int a0, int share, int r3,
                                            int rs, c2<T>* mine)
{
#pragma unroll 2
    for (int ga = share; ga < rs; ga += kVNT / 64) {
        c2<T> acc = a0 ? mine[ga] : mk<T>(0, 0), odd = mk<T>(0, 0);
        if (ga < r3) {
            const c2<T>* w = Wt + ga * wrow + a0;
#pragma unroll
            for (int q = 0; q < CH; ++q) fma_c(q & 1 ? odd : acc, u[q], w[q]);
        }
        mine[ga] = acc + odd;
    }
}

// out[k1 rs + g] for k1 in [0, n1p1), zero for g in [r3, rs); cp: a
// superdiagonal core.  rmax: as given to v_rows_lds.  g1, g2, g3: strides of
// the core along the contracted x rank, the contracted y rank and g.
template <typename T>
__device__ __forceinline__ void v_rows(const c2<T>* G, const c2<T>* U1, const c2<T>* U2, int r1, int r2, int r3,
                                       int g1, int g2, int g3, int n1p1, int rmax,
                                       int rs, bool cp, c2<T>* __restrict__ out)
{
    extern __shared__ __align__(16) unsigned char v_smem[];
    const int row = v_rows_row(rmax, rs), wrow = v_rows_pad(r1);
    c2<T>* Wt = reinterpret_cast<c2<T>*>(v_smem);                // [r3][wrow], zero beyond r1
    c2<T>* tile = Wt + (size_t)rmax * ((rmax + 15) / 16 * 16);   // [64][row]
    const int tid = threadIdx.x;
    constexpr int nt = kVNT;
    if (cp) {
        for (int l = tid; l < r3; l += nt) Wt[l] = ldg(G + (long)l * (r3 * r3 + r3 + 1)) * ldg(U2 + l);
        __syncthreads();
        for (int e = tid; e < n1p1 * rs; e += nt) {
            const int k1 = e / rs, l = e - k1 * rs;
            out[e] = l < r3 ? ldg(U1 + (long)k1 * r3 + l) * Wt[l] : mk<T>(0, 0);
        }
        return;
    }
    for (int e = tid; e < wrow * r3; e += nt) {
        const int al = e / r3, ga = e - al * r3;
        c2<T> acc = mk<T>(0, 0);
        if (al < r1) {
            const c2<T>* g = G + (long)al * g1 + (long)ga * g3;
            for (int b0 = 0; b0 < r2; b0 += 16) {
                c2<T> gv[16], uv[16];
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    const int b = min(b0 + q, r2 - 1);
                    gv[q] = ldg(g + (long)b * g2);
                    uv[q] = ldg(U2 + b);
                }
#pragma unroll
                for (int q = 0; q < 16; ++q)
                    if (b0 + q < r2) fma_c(acc, gv[q], uv[q]);
            }
        }
        Wt[ga * wrow + al] = acc;
    }
    const int lane = tid % 64, share = tid / 64;
    for (int k0 = 0; k0 < n1p1; k0 += 64) {
        const int rows = min(64, n1p1 - k0);
        for (int e = tid; e < rows * r1; e += nt) {
            const int k = e / r1;
            tile[k * row + e - k * r1] = ldg(U1 + (long)k0 * r1 + e);
        }
        __syncthreads();   // W and the tile's rows of U1
        c2<T>* mine = tile + lane * row;
        c2<T> u[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) u[q] = q < r1 && lane < rows ? mine[q] : mk<T>(0, 0);
        __syncthreads();   // the rows are replaced by the sums
        for (int a0 = 0; a0 < r1; a0 += 16) {
            if (a0 > 0) {
#pragma unroll
                for (int q = 0; q < 16; ++q)
                    u[q] = a0 + q < r1 && lane < rows ? ldg(U1 + (long)(k0 + lane) * r1 + a0 + q) : mk<T>(0, 0);
            }
            if (r1 - a0 <= 8) v_rows_sums<8>(u, Wt, wrow, a0, share, r3, rs, mine);
            else v_rows_sums<16>(u, Wt, wrow, a0, share, r3, rs, mine);
        }
        __syncthreads();
        for (int e = tid; e < rows * rs; e += nt) {
            const int k = e / rs;
            out[(long)k0 * rs + e] = tile[k * row + e - k * rs];
        }
        __syncthreads();   // the tile is reused
    }
}

}  // namespace vie

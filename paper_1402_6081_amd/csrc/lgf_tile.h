// The passes of one tile's zero-padded forward and truncated inverse transform (Eq. alg_upfft /
// alg_dwfft) inside a workgroup, for the kernels that transform a tile and for those that
// interpolate and transform it in one go.
//
// Data: an m^3 real tile [z][y][x] <-> its padded M^3 real-to-complex spectrum
// [kz][ky][kx], M = 2m, kx in [0, M/2], stored chunk-major (spec_at) across the batch.
// The tile lives in a [z < m][ky < M][kx <= M/2] LDS array (the largest intermediate of either
// direction); the real input / output is staged in the not-yet-used upper ky half of each z
// plane.  The staged rows are padded to m + 1 values: the x pass reads (and the inverse writes)
// one row per lane, and rows m apart would share LDS banks.  Passes: x (real rows), y (complex
// columns of the z < m planes), z (complex columns, straight to / from HBM).
#pragma once
#include "lgf_device.h"

namespace lgfdev {

template <int m>
constexpr int tile_values() { return m * 2 * m * (m + 1); }  // complex values of the LDS array

// Staged real value (z, y, x) of a tile.
template <typename T, int m>
__device__ __forceinline__ T& staged(cplx<T>* buf, int z, int y, int x) {
    constexpr int H = m + 1, PLANE = 2 * m * H;
    return reinterpret_cast<T*>(buf + z * PLANE + m * H)[y * (m + 1) + x];
}

// Forward passes of the staged tile (visible to the workgroup) into item b of out (nout items).
// The workgroup may reuse buf after its next barrier.
template <typename T, int m, int NT>
__device__ __forceinline__ void tile_forward(cplx<T>* buf, int tid, cplx<T>* __restrict__ out, size_t b,
                                             int64_t nout) {
    constexpr int M = 2 * m, H = m + 1, PLANE = M * H;
    // x pass: real rows (z, y) -> kx in [0, M/2]
    for (int row = tid; row < m * m; row += NT) {
        const int z = row / m, y = row - z * m;
        const T* s = &staged<T, m>(buf, z, y, 0);
        cplx<T>* d = buf + z * PLANE + y * H;
        T xr[m];
#pragma unroll
        for (int j = 0; j < m; ++j) xr[j] = s[j];
        if constexpr (is_pow2(M)) {
            T xi[m], Xr[M], Xi[M];
#pragma unroll
            for (int j = 0; j < m; ++j) xi[j] = T(0);
            pencil_fwd<T, m, M>(xr, xi, Xr, Xi);
#pragma unroll
            for (int k = 0; k < H; ++k) d[k] = cplx<T>{Xr[k], Xi[k]};
        } else {
            T Xr[H], Xi[H];
            pencil_r2c<T, m, M>(xr, Xr, Xi);
#pragma unroll
            for (int k = 0; k < H; ++k) d[k] = cplx<T>{Xr[k], Xi[k]};
        }
    }
    __syncthreads();
    // y pass: columns (z, kx), y < m -> ky < M
    for (int col = tid; col < m * H; col += NT) {
        const int z = col / H, kx = col - z * H;
        cplx<T>* base = buf + z * PLANE + kx;
        T xr[m], xi[m];
#pragma unroll
        for (int j = 0; j < m; ++j) {
            const cplx<T> v = base[j * H];
            xr[j] = v.x;
            xi[j] = v.y;
        }
        T Xr[M], Xi[M];
        pencil_fwd<T, m, M>(xr, xi, Xr, Xi);
#pragma unroll
        for (int k = 0; k < M; ++k) base[k * H] = cplx<T>{Xr[k], Xi[k]};
    }
    __syncthreads();
    // z pass: columns (ky, kx), z < m -> kz < M, written to HBM (chunk-major spectrum)
    for (int col = tid; col < PLANE; col += NT) {
        T xr[m], xi[m];
#pragma unroll
        for (int j = 0; j < m; ++j) {
            const cplx<T> v = buf[j * PLANE + col];
            xr[j] = v.x;
            xi[j] = v.y;
        }
        T Xr[M], Xi[M];
        pencil_fwd<T, m, M>(xr, xi, Xr, Xi);
#pragma unroll
        for (int k = 0; k < M; ++k) out[spec_at(b, k * PLANE + col, nout)] = cplx<T>{Xr[k], Xi[k]};
    }
}

// Inverse passes of item b of in (nbatch items; elements Tin, arithmetic A), the m^3 results
// staged in buf (not yet visible to the workgroup).
template <typename Tin, typename A, int m, int NT>
__device__ __forceinline__ void tile_inverse(const cplx<Tin>* __restrict__ in, size_t b, int64_t nbatch, cplx<A>* buf,
                                             int tid) {
    constexpr int M = 2 * m, H = m + 1, PLANE = M * H;
    // z pass: HBM columns (ky, kx), kz < M -> z < m
    for (int col = tid; col < PLANE; col += NT) {
        A Xr[M], Xi[M];
#pragma unroll
        for (int k = 0; k < M; ++k) {
            const cplx<Tin> v = in[spec_at(b, k * PLANE + col, nbatch)];
            Xr[k] = A(v.x);
            Xi[k] = A(v.y);
        }
        A xr[m], xi[m];
        pencil_inv<A, m, M>(Xr, Xi, xr, xi);
#pragma unroll
        for (int j = 0; j < m; ++j) buf[j * PLANE + col] = cplx<A>{xr[j], xi[j]};
    }
    __syncthreads();
    // y pass: columns (z, kx), ky < M -> y < m
    for (int col = tid; col < m * H; col += NT) {
        const int z = col / H, kx = col - z * H;
        cplx<A>* base = buf + z * PLANE + kx;
        A Xr[M], Xi[M];
#pragma unroll
        for (int k = 0; k < M; ++k) {
            const cplx<A> v = base[k * H];
            Xr[k] = v.x;
            Xi[k] = v.y;
        }
        A xr[m], xi[m];
        pencil_inv<A, m, M>(Xr, Xi, xr, xi);
#pragma unroll
        for (int j = 0; j < m; ++j) base[j * H] = cplx<A>{xr[j], xi[j]};
    }
    __syncthreads();
    // x pass: Hermitian rows (z, y) -> real x < m, staged in the upper ky half
    for (int row = tid; row < m * m; row += NT) {
        const int z = row / m, y = row - z * m;
        const cplx<A>* s = buf + z * PLANE + y * H;
        A Yr[H], Yi[H];
#pragma unroll
        for (int k = 0; k < H; ++k) {
            const cplx<A> v = s[k];
            Yr[k] = v.x;
            Yi[k] = v.y;
        }
        A x[m];
        pencil_c2r<A, m, M>(Yr, Yi, x);
        A* d = &staged<A, m>(buf, z, y, 0);
#pragma unroll
        for (int j = 0; j < m; ++j) d[j] = x[j];
    }
}

}  // namespace lgfdev

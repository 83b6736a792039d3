// Zero-padded forward FFT (Pad + FFT, Eq. alg_upfft) and truncated inverse FFT
// (FFT^-1 + Trunc, Eq. alg_dwfft) of one block or interval per workgroup: level 0, and the
// levels >= 1 of the lattice scheme (13 and 17 nodes).  The passes are in lgf_tile.h; the other
// levels >= 1 are transformed by the kernels that interpolate them (lgf_interp.hip).
#include <algorithm>
#include <map>
#include <mutex>
#include <type_traits>
#include <utility>

#include "lgf_device.h"
#include "lgf_internal.h"
#include "lgf_tile.h"

namespace lgfdev {

// Persistent: a workgroup transforms tiles blockIdx.x, blockIdx.x + gridDim.x, ... of the
// launch; while it transforms one, the next tile's input is already on its way into
// registers (a tile occupies so much LDS that at most one or two workgroups share a CU, so
// the input reads would otherwise stall the CU).
template <typename T, int m, int NT>
__global__ void __launch_bounds__(NT)
    k_pad_fft(const T* __restrict__ in, cplx<T>* __restrict__ out, int64_t nbatch, int64_t nout) {
    constexpr int NPRE = (m * m * m + NT - 1) / NT;
    __shared__ cplx<T> buf[tile_values<m>()];
    const int tid = threadIdx.x;
    auto fetch = [&](int64_t b, T(&pre)[NPRE]) {
        const T* src = in + (size_t)b * (m * m * m);
#pragma unroll
        for (int k = 0; k < NPRE; ++k) {
            const int i = tid + k * NT;
            pre[k] = i < m * m * m ? src[i] : T(0);
        }
    };
    int64_t b = blockIdx.x;
    if (b >= nbatch) return;
    T pre[NPRE];
    fetch(b, pre);
    for (; b < nbatch; b += gridDim.x) {
#pragma unroll
        for (int k = 0; k < NPRE; ++k) {
            const int i = tid + k * NT;
            if (i < m * m * m) staged<T, m>(buf, i / (m * m), i / m % m, i % m) = pre[k];
        }
        __syncthreads();
        if (b + gridDim.x < nbatch) fetch(b + gridDim.x, pre);  // the next tile's input
        tile_forward<T, m, NT>(buf, tid, out, (size_t)b, nout);
        __syncthreads();  // the next tile is staged into buf
    }
}

// Inverse: spectrum elements of type Tin, arithmetic in A, real output of type Tout.
// (FP64 path: all double.  FP32 path: float at level 0 and at level 1 of the lattice
// scheme; at the other levels >= 1 the float spectra are inverted in double arithmetic to
// double node values: the Lebesgue constant of equispaced interpolation would amplify FP32
// rounding of the node values above 1e-6, and gfx950 issues FP64 FMAs at the non-packed FP32
// rate.)
template <typename Tin, typename A, typename Tout, int m, int NT>
__global__ void __launch_bounds__(NT)
    k_ifft_trunc(const cplx<Tin>* __restrict__ in, Tout* __restrict__ out, int64_t nbatch,
                 const int32_t* __restrict__ out_map, int opitch) {
    __shared__ cplx<A> buf[tile_values<m>()];
    const int tid = threadIdx.x;
    const size_t b = blockIdx.x;
    tile_inverse<Tin, A, m, NT>(in, b, nbatch, buf, tid);
    __syncthreads();
    // output tiles of opitch^3 values: the m^3 results, zeros in the planes beyond them
    Tout* dst = out + (out_map ? (size_t)out_map[b] : b) * (size_t)(opitch * opitch * opitch);
    if (opitch == m) {
        for (int i = tid; i < m * m * m; i += NT) dst[i] = (Tout)staged<A, m>(buf, i / (m * m), i / m % m, i % m);
    } else {
        for (int i = tid; i < opitch * opitch * opitch; i += NT) {
            const int x = i % opitch, y = (i / opitch) % opitch, z = i / (opitch * opitch);
            dst[i] = (z < m && y < m && x < m) ? (Tout)staged<A, m>(buf, z, y, x) : Tout(0);
        }
    }
}

// ------------------------------------------------------------------ two-phase transforms
constexpr int kShare = 3;  // threads sharing one pencil (each forms every third output)
// For tiles whose one-workgroup LDS tile [m][M][M/2+1] exceeds the 160 KB of a workgroup
// (m = 17: 166 KB of complex doubles), the transforms run in two kernels through an HBM
// intermediate [z < m][ky < M][kx <= M/2] per item (`scratch`, complex of 16 bytes):
//   forward  k_fft2_xy (per z plane: x pass, y pass -> scratch), k_fft2_z (z pass -> spectrum);
//   inverse  k_ifft2_z (z pass -> scratch), k_ifft2_yx (per z plane: y pass, x pass -> tile).
template <typename T, int m, int M, int NT>
__global__ void __launch_bounds__(NT) k_fft2_xy(const T* __restrict__ in, cplx<T>* __restrict__ scratch) {
    // one workgroup per z plane of an item: the x and y passes do not mix planes
    constexpr int H = M / 2 + 1;
    __shared__ T tile[m * m];
    __shared__ cplx<T> buf[m * H];  // [y][kx]
    __shared__ double2 tw[M];
    const int tid = threadIdx.x;
    const size_t b = blockIdx.x / m;
    const int z = blockIdx.x - (int)b * m;
    const T* src = in + b * (m * m * m) + z * (m * m);
    stage_roots<M>(tw, tid, NT);
    for (int i = tid; i < m * m; i += NT) tile[i] = src[i];
    __syncthreads();
    for (int t = tid; t < kShare * m; t += NT) {  // x pass: real rows, kShare threads per row
        const int y = t / kShare, k0 = t - y * kShare;
        T xr[m], xi[m];
#pragma unroll
        for (int j = 0; j < m; ++j) {
            xr[j] = tile[y * m + j];
            xi[j] = T(0);
        }
        cplx<T>* d = buf + y * H;
        dft_each<T, m, M, -1, H>(xr, xi, tw, [&](int k, T re, T im) { d[k] = cplx<T>{re, im}; }, k0, kShare);
    }
    __syncthreads();
    cplx<T>* dst = scratch + b * (m * M * H) + z * (M * H);
    for (int t = tid; t < kShare * H; t += NT) {  // y pass: columns kx -> [ky][kx] of plane z
        const int kx = t / kShare, k0 = t - kx * kShare;
        T xr[m], xi[m];
#pragma unroll
        for (int j = 0; j < m; ++j) {
            const cplx<T> v = buf[j * H + kx];
            xr[j] = v.x;
            xi[j] = v.y;
        }
        cplx<T>* d = dst + kx;
        dft_each<T, m, M, -1, M>(xr, xi, tw, [&](int k, T re, T im) { d[k * H] = cplx<T>{re, im}; }, k0, kShare);
    }
}

// z pass of the forward two-phase transform: one thread per column (ky, kx) of one item
template <typename T, int m, int M, int NT>
__global__ void __launch_bounds__(NT) k_fft2_z(const cplx<T>* __restrict__ scratch, cplx<T>* __restrict__ out,
                                               int64_t nout) {
    constexpr int H = M / 2 + 1;
    constexpr int PLANE = M * H;
    __shared__ double2 tw[M];
    stage_roots<M>(tw, threadIdx.x, NT);
    __syncthreads();
    const size_t b = blockIdx.y;
    const int t = blockIdx.x * NT + threadIdx.x;
    if (t >= kShare * PLANE) return;
    const int col = t / kShare, k0 = t - col * kShare;
    const cplx<T>* s = scratch + b * (m * PLANE) + col;
    T xr[m], xi[m];
#pragma unroll
    for (int j = 0; j < m; ++j) {
        const cplx<T> v = s[j * PLANE];
        xr[j] = v.x;
        xi[j] = v.y;
    }
    dft_each<T, m, M, -1, M>(
        xr, xi, tw, [&](int k, T re, T im) { out[spec_at(b, k * PLANE + col, nout)] = cplx<T>{re, im}; }, k0,
        kShare);
}

// z pass of the inverse two-phase transform: spectrum (Tin) -> scratch (arithmetic type A)
template <typename Tin, typename A, int m, int M, int NT>
__global__ void __launch_bounds__(NT) k_ifft2_z(const cplx<Tin>* __restrict__ in, cplx<A>* __restrict__ scratch,
                                                int64_t nbatch) {
    constexpr int H = M / 2 + 1;
    constexpr int PLANE = M * H;
    __shared__ double2 tw[M];
    stage_roots<M>(tw, threadIdx.x, NT);
    __syncthreads();
    const size_t b = blockIdx.y;
    const int t = blockIdx.x * NT + threadIdx.x;
    if (t >= kShare * PLANE) return;
    const int col = t / kShare, j0 = t - col * kShare;
    A Xr[M], Xi[M];
#pragma unroll
    for (int k = 0; k < M; ++k) {
        const cplx<Tin> v = in[spec_at(b, k * PLANE + col, nbatch)];
        Xr[k] = A(v.x);
        Xi[k] = A(v.y);
    }
    cplx<A>* d = scratch + b * (m * PLANE) + col;
    dft_each<A, M, M, +1, m>(Xr, Xi, tw, [&](int j, A re, A im) { d[j * PLANE] = cplx<A>{re, im}; }, j0, kShare);
}

// y and x passes of the inverse two-phase transform: scratch -> real tile (Tout); one
// workgroup per z plane of an item
template <typename A, typename Tout, int m, int M, int NT>
__global__ void __launch_bounds__(NT) k_ifft2_yx(const cplx<A>* __restrict__ scratch, Tout* __restrict__ out,
                                                 const int32_t* __restrict__ out_map) {
    constexpr int H = M / 2 + 1;
    __shared__ cplx<A> buf[m * H];  // [y][kx]
    __shared__ A tile[m * m];
    __shared__ double2 tw[M];
    const int tid = threadIdx.x;
    const size_t b = blockIdx.x / m;
    const int z = blockIdx.x - (int)b * m;
    const cplx<A>* s = scratch + b * (m * M * H) + z * (M * H);
    stage_roots<M>(tw, tid, NT);
    __syncthreads();
    for (int t = tid; t < kShare * H; t += NT) {  // y pass: ky < M -> y < m, kShare threads per column
        const int kx = t / kShare, j0 = t - kx * kShare;
        A Xr[M], Xi[M];
#pragma unroll
        for (int k = 0; k < M; ++k) {
            const cplx<A> v = s[k * H + kx];
            Xr[k] = v.x;
            Xi[k] = v.y;
        }
        cplx<A>* d = buf + kx;
        dft_each<A, M, M, +1, m>(Xr, Xi, tw, [&](int j, A re, A im) { d[j * H] = cplx<A>{re, im}; }, j0, kShare);
    }
    __syncthreads();
    for (int t = tid; t < kShare * m; t += NT) {  // x pass: Hermitian rows -> real x < m
        const int y = t / kShare, j0 = t - y * kShare;
        A Yr[H], Yi[H];
#pragma unroll
        for (int k = 0; k < H; ++k) {
            const cplx<A> v = buf[y * H + k];
            Yr[k] = v.x;
            Yi[k] = v.y;
        }
        A* d = tile + y * m;
        c2r_each<A, m, M>(Yr, Yi, tw, [&](int j, A v) { d[j] = v; }, j0, kShare);
    }
    __syncthreads();
    Tout* dst = out + (out_map ? (size_t)out_map[b] : b) * (m * m * m) + z * (m * m);
    for (int i = tid; i < m * m; i += NT) dst[i] = (Tout)tile[i];
}

template <typename T, int m>
static hipError_t fwd_two_phase(const T* in, cplx<T>* out, int64_t nbatch, int64_t nout, void* scratch,
                                hipStream_t s) {
    constexpr int M = 2 * m, PLANE = M * (M / 2 + 1), NT = 256;
    if (!scratch) return hipErrorInvalidValue;
    hipError_t e = lgf_launch(k_fft2_xy<T, m, M, 64>, dim3((unsigned)(nbatch * m)), dim3(64), 0, s, in,
                              (cplx<T>*)scratch);
    if (e != hipSuccess) return e;
    const dim3 grid((kShare * PLANE + NT - 1) / NT, (unsigned)nbatch);
    return lgf_launch(k_fft2_z<T, m, M, NT>, grid, dim3(NT), 0, s, (const cplx<T>*)scratch, out, nout);
}

template <typename Tin, typename A, typename Tout, int m>
static hipError_t inv_two_phase(const cplx<Tin>* in, Tout* out, int64_t nbatch, const int32_t* out_map,
                                void* scratch, hipStream_t s) {
    constexpr int M = 2 * m, PLANE = M * (M / 2 + 1), NT = 256;
    if (!scratch) return hipErrorInvalidValue;
    const dim3 grid((kShare * PLANE + NT - 1) / NT, (unsigned)nbatch);
    hipError_t e = lgf_launch(k_ifft2_z<Tin, A, m, M, NT>, grid, dim3(NT), 0, s, in, (cplx<A>*)scratch, nbatch);
    if (e != hipSuccess) return e;
    return lgf_launch(k_ifft2_yx<A, Tout, m, M, 64>, dim3((unsigned)(nbatch * m)), dim3(64), 0, s,
                      (const cplx<A>*)scratch, out, out_map);
}

// nt: threads per workgroup (0 = default: 256, measured faster than 128 for the small
// tiles of levels >= 1 as well); the autotuner picks among {128, 256, 512} for the level-0
// tiles (m = 8, 16).  The forward FP64 16^3 tile is not offered 512 threads: its 32-point
// pencils would then spill (the inverse's fit, 219 registers, and are its default).

// Tiles whose LDS allows at most two workgroups per CU (the level-0 tiles) get a
// persistent grid (measured: the 256^3 level-0 FP64 transform 375 -> 248 us, FP32 143 ->
// 108 us; small tiles were 5% slower persistent, so they keep one workgroup per tile).
template <typename T, int m, int NT>
static hipError_t fwd_mnt(const T* in, cplx<T>* out, int64_t nbatch, int64_t nout, hipStream_t s) {
    auto kernel = k_pad_fft<T, m, NT>;
    return lgf_launch(kernel, dim3((unsigned)persistent_grid(kernel, NT, nbatch, 2)), dim3(NT), 0, s, in, out, nbatch,
                      nout);
}

template <typename T, int m>
static hipError_t launch_fwd_m(const T* in, cplx<T>* out, int64_t nbatch, int64_t nout, hipStream_t s,
                               int nt = 0) {
    if constexpr (m == 8 || m == 16) {
        if constexpr (!(m == 16 && sizeof(T) == 8))
            if (nt == 512) return fwd_mnt<T, m, 512>(in, out, nbatch, nout, s);
        if (nt == 128) return fwd_mnt<T, m, 128>(in, out, nbatch, nout, s);
    }
    return fwd_mnt<T, m, 256>(in, out, nbatch, nout, s);
}

template <typename Tin, typename A, typename Tout, int m, int NT>
static hipError_t inv_mnt(const cplx<Tin>* in, Tout* out, int64_t nbatch, int64_t nin, const int32_t* out_map,
                          int opitch, hipStream_t s) {
    return lgf_launch(k_ifft_trunc<Tin, A, Tout, m, NT>, dim3((unsigned)nbatch), dim3(NT), 0, s, in, out, nin,
                      out_map, opitch);
}

template <typename Tin, typename A, typename Tout, int m>
static hipError_t launch_inv_m(const cplx<Tin>* in, Tout* out, int64_t nbatch, int64_t nin, const int32_t* out_map,
                               int opitch, hipStream_t s, int nt = 0) {
    if (opitch <= 0) opitch = m;
    // FP64 16^3 tiles default to 512 threads: one workgroup fills a CU's LDS, and 8 waves
    // keep twice the column loads in flight (256^3: 331 -> 299 us; 128^3: 51 -> 47 us)
    if (nt == 0 && m == 16 && sizeof(A) == 8) nt = 512;
    if constexpr (m == 8 || m == 16) {
        if (nt == 512) return inv_mnt<Tin, A, Tout, m, 512>(in, out, nbatch, nin, out_map, opitch, s);
        if (nt == 128) return inv_mnt<Tin, A, Tout, m, 128>(in, out, nbatch, nin, out_map, opitch, s);
    }
    return inv_mnt<Tin, A, Tout, m, 256>(in, out, nbatch, nin, out_map, opitch, s);
}

template <typename T>
hipError_t launch_pad_fft(int m, const T* in, cplx<T>* out, int64_t nbatch, hipStream_t s, int nt, int64_t nout,
                          void* scratch) {
    if (nbatch <= 0) return hipSuccess;
    if (nout <= 0) nout = nbatch + 1;
    switch (m) {
        case 17: return fwd_two_phase<T, 17>(in, out, nbatch, nout, scratch, s);
        case 4: return launch_fwd_m<T, 4>(in, out, nbatch, nout, s);
        case 6: return launch_fwd_m<T, 6>(in, out, nbatch, nout, s);
        case 8: return launch_fwd_m<T, 8>(in, out, nbatch, nout, s, nt);
        case 12: return launch_fwd_m<T, 12>(in, out, nbatch, nout, s);
        case 13: return launch_fwd_m<T, 13>(in, out, nbatch, nout, s);
        case 16: return launch_fwd_m<T, 16>(in, out, nbatch, nout, s, nt);
        default: return hipErrorInvalidValue;
    }
}

template <typename T>
hipError_t launch_ifft0(int n, const cplx<T>* in, T* out, int64_t nbatch, int64_t nin, hipStream_t s, int nt,
                        const int32_t* out_map) {
    if (nbatch <= 0) return hipSuccess;
    switch (n) {
        case 4: return launch_inv_m<T, T, T, 4>(in, out, nbatch, nin, out_map, 0, s);
        case 6: return launch_inv_m<T, T, T, 6>(in, out, nbatch, nin, out_map, 0, s);
        case 8: return launch_inv_m<T, T, T, 8>(in, out, nbatch, nin, out_map, 0, s, nt);
        case 12: return launch_inv_m<T, T, T, 12>(in, out, nbatch, nin, out_map, 0, s);
        case 16: return launch_inv_m<T, T, T, 16>(in, out, nbatch, nin, out_map, 0, s, nt);
        default: return hipErrorInvalidValue;
    }
}

template <typename T>
hipError_t launch_ifft_lattice(int m, const cplx<T>* in, double* out, int64_t nbatch, hipStream_t s, void* scratch,
                               int opitch) {
    if (nbatch <= 0) return hipSuccess;
    if (opitch > 0 && opitch < m) return hipErrorInvalidValue;  // output tiles hold the m^3 results
    switch (m) {
        // level 1: the blocks' spectra, in the path's own precision (these values are not
        // interpolated further)
        case 12: return launch_inv_m<T, T, double, 12>(in, out, nbatch, nbatch, nullptr, opitch, s);
        case 16: return launch_inv_m<T, T, double, 16>(in, out, nbatch, nbatch, nullptr, opitch, s);
        case 13: return launch_inv_m<T, double, double, 13>(in, out, nbatch, nbatch, nullptr, opitch, s);
        case 17: return inv_two_phase<T, double, double, 17>(in, out, nbatch, nullptr, scratch, s);
        default: return hipErrorInvalidValue;
    }
}

#define LGF_INST(T)                                                                                                  \
    template hipError_t launch_pad_fft<T>(int, const T*, cplx<T>*, int64_t, hipStream_t, int, int64_t, void*);       \
    template hipError_t launch_ifft0<T>(int, const cplx<T>*, T*, int64_t, int64_t, hipStream_t, int, const int32_t*);\
    template hipError_t launch_ifft_lattice<T>(int, const cplx<T>*, double*, int64_t, hipStream_t, void*, int);
LGF_INST(double)
LGF_INST(float)
#undef LGF_INST

}  // namespace lgfdev

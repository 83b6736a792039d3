// Regularization (Reg, Eq. alg_reg / kcprss1) and interpolation (Interp, Eq. alg_interp
// / kcprss3) between levels, as tensor products of 1D Lagrange matrices (Sec. 2.5):
//   block -> level-1 interval   ftilde = (A x A x A) f           A[k][j] = phi_k(j (p-1)/n)
//   children -> parent          ftilde_J = sum_c (C_c x C_c x C_c) ftilde_{2J+c}
//                                                                 C_c[m][k] = phi_m((c(p-1)+k)/2)
//   parent -> children (add)    utilde_{2J+c} += (C_c^T x C_c^T x C_c^T) utilde_J
//   level-1 interval -> block   u = vnear + (A^T x A^T x A^T) utilde    (FP64 add-back)
// Each 3D product is three 1D passes through LDS.  For p <= 10 a workgroup that has an interval's
// node values in LDS also transforms them: Reg goes on to the level's forward transform, the
// level's inverse transform to Interp from the parent, and at level 1 on to the block, so the node
// values of level 1 are not written to HBM on the way down, and each step is one launch less.
//
// A pass is a small matrix applied along one axis (contract below): a lane holds one column of
// inputs in registers and forms several outputs with the matrix values in scalar registers, so
// that a multiply-add needs no LDS read of its own (one thread per output, reading a value and a
// matrix entry from LDS for each multiply-add, made the passes LDS-bound).  On a 256^3 cube of
// 16^3 blocks, p = 8, from one output per thread to this, FP64 and FP32: Reg to level 1 with its
// transform 85 to 55 us (its 0.30 GB take 53 at a copy's rate) and 45 to 31, Reg up 25 to 17 and
// 14 to 11, the final pass with its transform and Interp 106 to 77 (0.42 GB: 74) and 85 to 66 (46
// since its reads go out ahead, node_values);
// at p = 17, FP64, 128^3: Reg up 63 to 36, Interp down 50 to 31, the final pass 30 to 22.
#include <type_traits>

#include "lgf_internal.h"
#include "lgf_tile.h"

namespace lgfdev {

// Reg up works on eight children per workgroup: more waves hide the latency of its few, long
// workgroups
constexpr int kRegUpThreads = 1024;
// block -> level 1
constexpr int kBlockThreads = 256;
// the lattice scheme's Reg up, Interp down and final pass: two waves per 64 of the 17^2 columns
constexpr int kLatThreads = 640;
constexpr int kSumThreads = 256;
// inverse transform, Interp and the final pass
constexpr int kInvThreads = 256;

constexpr int imax(int a, int b) { return a > b ? a : b; }

// Matrices of the plan, read at wave-uniform indices through scalar loads (constant address
// space: they do not change during a launch).
template <typename T>
using Uniform = const __attribute__((address_space(4))) T*;
template <typename T>
__device__ __forceinline__ Uniform<T> uniform_ptr(const T* p) {
    return (Uniform<T>)(uintptr_t)p;
}

// How W waves share the OUT outputs of C columns: a wave takes 64 columns, one per lane, and all
// their outputs, or, with fewer groups of columns than waves, a share of CH outputs.
template <int OUT, int C, int W>
struct Share {
    static constexpr int G = (C + 63) / 64, CH = W >= 2 * G ? (OUT + W / G - 1) / (W / G) : OUT;
    static constexpr int SPLIT = (OUT + CH - 1) / CH;  // shares, the last one with the rest
    static constexpr int TASKS = G * SPLIT;            // of which wave w takes w, w + W, ...
    static_assert(SPLIT * CH >= OUT && (SPLIT - 1) * CH < OUT && (SPLIT == 1 || TASKS <= W), "shares");
    static __device__ __forceinline__ int col(int task, int lane) { return task % G * 64 + lane; }
    static __device__ __forceinline__ int out0(int task) { return task / G * CH; }
};

// One pass: put(col, o, sum_k mat[o * IN + k] * load(col, k), base(col, o, i)) for o < OUT, the sum
// in increasing k; output o is the i-th of its share.  base, what the outputs are added to, is read
// for all of a share before the first is written.  mat is row-major [OUT][IN] and wave-uniform.
template <int IN, int OUT, int C, int W, typename T, typename Load, typename Base, typename Put>
__device__ __forceinline__ void contract_onto(int wave, int lane, Uniform<T> mat, Load load, Base base, Put put) {
    using Sh = Share<OUT, C, W>;
    for (int task = wave; task < Sh::TASKS; task += W) {
        const int col = Sh::col(task, lane), o0 = Sh::out0(task);
        const bool on = C % 64 == 0 || col < C;
        using B = std::remove_reference_t<decltype(base(0, 0, 0))>;
        B b[Sh::CH];
        T v[IN];
#pragma unroll
        for (int i = 0; i < Sh::CH; ++i)
            b[i] = on && (Sh::SPLIT * Sh::CH == OUT || o0 + i < OUT) ? base(col, o0 + i, i) : B(0);
#pragma unroll
        for (int k = 0; k < IN; ++k) v[k] = on ? load(col, k) : T(0);
#pragma unroll
        for (int i = 0; i < Sh::CH; ++i) {
            const int o = o0 + i;
            if (Sh::SPLIT * Sh::CH != OUT && o >= OUT) break;
            T acc = T(0);
#pragma unroll
            for (int k = 0; k < IN; ++k) acc += mat[o * IN + k] * v[k];
            if (on) put(col, o, acc, b[i]);
        }
    }
}
template <int IN, int OUT, int C, int W, typename T, typename Load, typename Put>
__device__ __forceinline__ void contract(int wave, int lane, Uniform<T> mat, Load load, Put put) {
    contract_onto<IN, OUT, C, W, T>(
        wave, lane, mat, load, [](int, int, int) { return 0; }, [&](int col, int o, T v, int) { put(col, o, v); });
}

// ------------------------------------------------------------------ block -> level 1
// One workgroup per block.  A: [P][N].
template <typename T, int N, int P>
__global__ void __launch_bounds__(kBlockThreads)
    k_reg_fft(const T* __restrict__ f, const T* __restrict__ A, T* __restrict__ ftil, cplx<T>* __restrict__ fhat,
              int64_t nout) {
    constexpr int N3 = N * N * N, P3 = P * P * P, W = kBlockThreads / 64;
    // t1[d][z][y] and t2[z][c][d], rows padded so that the lanes' columns fall into different banks
    constexpr int kZ = N + 1, kD = N * kZ + 1, kS = P * P + 4;
    constexpr int kFront = (imax(P * kD, 2 * tile_values<P>()) + 1) / 2 * 2;  // t1, then the transform
    __shared__ alignas(16) T lds[kFront + N * kS];
    T *t1 = lds, *t2 = lds + kFront;
    cplx<T>* buf = reinterpret_cast<cplx<T>*>(lds);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t b = blockIdx.x;
    const Uniform<T> m = uniform_ptr(A);
    const T* src = f + b * N3;
    contract<N, P, N * N, W, T>(
        wave, lane, m, [&](int zy, int x) { return src[zy * N + x]; },
        [&](int zy, int d, T v) { t1[d * kD + zy / N * kZ + zy % N] = v; });
    __syncthreads();
    contract<N, P, N * P, W, T>(
        wave, lane, m, [&](int zd, int y) { return t1[zd % P * kD + zd / P * kZ + y]; },
        [&](int zd, int c, T v) { t2[zd / P * kS + c * P + zd % P] = v; });
    __syncthreads();
    contract<N, P, P * P, W, T>(
        wave, lane, m, [&](int cd, int z) { return t2[z * kS + cd]; },
        [&](int cd, int a, T v) {
            if (ftil) ftil[b * P3 + a * (P * P) + cd] = v;
            staged<T, P>(buf, a, cd / P, cd % P) = v;
        });
    if (!fhat) return;
    __syncthreads();
    tile_forward<T, P, kBlockThreads>(buf, tid, fhat, (size_t)b, nout);
}

// ------------------------------------------------------------------ children -> parent
// C01: [2][P][P].
template <typename T, int P>
__global__ void __launch_bounds__(kRegUpThreads)
    k_regup_fft(const T* __restrict__ in, const int32_t* __restrict__ child8, const T* __restrict__ C01,
                T* __restrict__ ftil, cplx<T>* __restrict__ fhat, int64_t nout) {
    constexpr int P2 = P * P, P3 = P2 * P, NT = kRegUpThreads, W = NT / 64;
    constexpr int kD = P2 + 1, kC1 = P * kD;   // t1[c][d][z y]
    constexpr int kZ2 = P2 + 4, kC2 = P * kZ2;  // t2[c][z][b d]
    __shared__ alignas(16) T t1[imax(8 * kC1, 2 * tile_values<P>())], t2[8 * kC2];
    cplx<T>* buf = reinterpret_cast<cplx<T>*>(t1);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t J = blockIdx.x;
    const Uniform<T> m = uniform_ptr(C01);
    const Uniform<int32_t> ch = uniform_ptr(child8 + J * 8);
    // two waves per child
    constexpr int WC = W / 8;
    const int c = wave / WC, wc = wave % WC, q = ch[c];
    if (q >= 0) {  // x: t1[d][z y] = sum_x C_cx[d][x] in[z y][x]
        const T* src = in + (int64_t)q * P3;
        T* d1 = t1 + c * kC1;
        contract<P, P, P2, WC, T>(
            wc, lane, m + (c & 1) * P2, [&](int zy, int x) { return src[zy * P + x]; },
            [&](int zy, int d, T v) { d1[d * kD + zy] = v; });
    }
    __syncthreads();
    if (q >= 0) {  // y: t2[z][b d] = sum_y C_cy[b][y] t1[d][z y]
        const T* s1 = t1 + c * kC1;
        T* d2 = t2 + c * kC2;
        contract<P, P, P2, WC, T>(
            wc, lane, m + ((c >> 1) & 1) * P2, [&](int zd, int y) { return s1[zd % P * kD + zd / P * P + y]; },
            [&](int zd, int b, T v) { d2[zd / P * kZ2 + b * P + zd % P] = v; });
    }
    __syncthreads();
    // z and the sum over children: node values [a][b d] = sum_c sum_z C_cz[a][z] t2[c][z][b d]
    constexpr int G = (P2 + 63) / 64;
    for (int task = wave; task < G * P; task += W) {
        const int bd = task % G * 64 + lane, a = task / G;
        if (P2 % 64 != 0 && bd >= P2) continue;
        T s = T(0);
        for (int cc = 0; cc < 8; ++cc) {
            if (ch[cc] < 0) continue;
            const Uniform<T> row = m + ((cc >> 2) & 1) * P2 + a * P;
#pragma unroll
            for (int z = 0; z < P; ++z) s += row[z] * t2[cc * kC2 + z * kZ2 + bd];
        }
        if (ftil) ftil[J * P3 + a * P2 + bd] = s;
        staged<T, P>(buf, a, bd / P, bd % P) = s;
    }
    if (!fhat) return;
    __syncthreads();
    tile_forward<T, P, NT>(buf, tid, fhat, (size_t)J, nout);
}

// ------------------------------------------------------------------ inverse and parent -> child
// Interp of a parent's node values (in HBM) to its child c: at(yx, z) += its value for every node
// z, y x of the child (yx = y P + x).  rows: the parent's rows this lane's share of the x pass takes,
// read ahead (interp_rows).  Ct: [2][P][P], Ct_c[k][m] = C_c[m][k]; R: interp_values<P>() doubles.
template <int P>
constexpr int interp_values() { return P * (P * P + 1) + P * (P * P + 4); }
template <int P, int W>
__device__ __forceinline__ void interp_rows(const double* __restrict__ src, int wave, int lane, double (&rows)[P]) {
    using Sh = Share<P, P * P, W>;
    static_assert(Sh::TASKS <= W, "one share per wave");
    const int ab = Sh::col(wave, lane);
#pragma unroll
    for (int d = 0; d < P; ++d) rows[d] = wave < Sh::TASKS && ab < P * P ? src[ab * P + d] : 0.0;
}
template <int P, int W, typename At>
__device__ __forceinline__ void interp_child(const double (&rows)[P], int c, Uniform<double> Ct, double* R, int wave,
                                             int lane, At at) {
    constexpr int P2 = P * P, kX = P2 + 1, kA = P2 + 4;
    double *t1 = R, *t2 = R + P * kX;  // t1[x'][a b], t2[a][y' x']
    contract<P, P, P2, W, double>(
        wave, lane, Ct + (c & 1) * P2, [&](int, int d) { return rows[d]; },
        [&](int ab, int x, double v) { t1[x * kX + ab] = v; });
    __syncthreads();
    contract<P, P, P2, W, double>(
        wave, lane, Ct + ((c >> 1) & 1) * P2, [&](int ax, int bb) { return t1[ax % P * kX + ax / P * P + bb]; },
        [&](int ax, int y, double v) { t2[ax / P * kA + y * P + ax % P] = v; });
    __syncthreads();
    contract_onto<P, P, P2, W, double>(
        wave, lane, Ct + ((c >> 2) & 1) * P2, [&](int yx, int a) { return t2[a * kA + yx]; },
        [&](int yx, int z, int) { return at(yx, z); },
        [&](int yx, int z, double v, double before) { at(yx, z) = before + v; });
}

// The node values of interval q (rows of P values, VP apart) into V: the inverse transform of its
// field spectrum (uhat NULL: zeros) plus Interp from its parent (par[q] = 8 J + c, -1: none;
// up NULL: no level above).  The parent's rows, and what ahead() reads, are loaded as soon as the
// transform's registers are free, so that their latency passes behind its last results and Interp's
// passes: the final pass of 256^3 in FP32 66 -> 46 us (0.21 GB: 37), of 128^3 16 -> 12, FP64 within
// 1 us (loaded before the transform they cost it occupancy: 60 us, and spheres of 6^3 blocks 30 -> 33).
// R: max(2 tile_values, interp_values) doubles.
template <typename T, int P, int VP, int NT, typename Ahead>
__device__ __forceinline__ void node_values(const cplx<T>* __restrict__ uhat, int64_t nint,
                                            const double* __restrict__ up, const int32_t* __restrict__ par,
                                            Uniform<double> Ct, int64_t q, double* R, double* V, int tid,
                                            Ahead ahead) {
    constexpr int P3 = P * P * P, P2 = P * P;
    const int pc = up ? uniform_ptr(par)[q] : -1;  // uniform
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    double rows[P];
    auto load_ahead = [&] {
        if (pc >= 0) interp_rows<P, NT / 64>(up + (int64_t)(pc >> 3) * P3, wave, lane, rows);
        ahead();
    };
    if (uhat) {
        cplx<double>* buf = reinterpret_cast<cplx<double>*>(R);
        tile_inverse<T, double, P, NT>(uhat, (size_t)q, nint, buf, tid);
        __syncthreads();
        load_ahead();
        for (int i = tid; i < P3; i += NT) V[(i / P) * VP + i % P] = staged<double, P>(buf, i / P2, i / P % P, i % P);
    } else {
        load_ahead();
        for (int i = tid; i < P3; i += NT) V[(i / P) * VP + i % P] = 0.0;
    }
    __syncthreads();
    if (pc < 0) return;
    interp_child<P, NT / 64>(rows, pc & 7, Ct, R, wave, lane,
                             [&](int yx, int z) -> double& { return V[(z * P + yx / P) * VP + yx % P]; });
    __syncthreads();
}

template <typename T, int P>
__global__ void __launch_bounds__(kInvThreads)
    k_inv_interp(const cplx<T>* __restrict__ uhat, const double* __restrict__ up, const int32_t* __restrict__ par,
                 const double* __restrict__ Ct, double* __restrict__ out) {
    constexpr int P3 = P * P * P;
    __shared__ alignas(16) double R[imax(2 * tile_values<P>(), interp_values<P>())];
    __shared__ double V[P3];
    const int64_t q = blockIdx.x;
    node_values<T, P, P, kInvThreads>(uhat, gridDim.x, up, par, uniform_ptr(Ct), q, R, V, threadIdx.x,
                                   [] {});
    for (int i = threadIdx.x; i < P3; i += kInvThreads) out[q * P3 + i] = V[i];
}

// ------------------------------------------------------------------ one (parent, child) per workgroup
// (the lattice scheme, P = 13 and 17)
// The kernels above hold 8 children, or a tile and its transform, in LDS (629 KB at P = 17).
// Here one workgroup handles one (parent, child) pair:
//   Reg up:      k_reg_up_part writes each child's contribution to `part` (scratch), then
//                k_reg_up_sum adds them in child order c = 0..7 (as one workgroup would);
//   Interp down: each child accumulates its own values (no two workgroups write one child).
template <typename T, int P>
__global__ void __launch_bounds__(kLatThreads)
    k_reg_up_part(const T* __restrict__ in, const int32_t* __restrict__ child8, const T* __restrict__ C01,
                  T* __restrict__ part) {
    constexpr int P2 = P * P, P3 = P2 * P, W = kLatThreads / 64, kD = P2 + 1, kZ = P2 + 4;
    __shared__ T t1[P * kD], t2[P * kZ];  // t1[d][z y], t2[z][b d]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t J = blockIdx.x >> 3;
    const int c = blockIdx.x & 7;
    const int q = child8[J * 8 + c];  // uniform
    if (q < 0) return;
    const Uniform<T> m = uniform_ptr(C01);
    const T* src = in + (int64_t)q * P3;
    contract<P, P, P2, W, T>(
        wave, lane, m + (c & 1) * P2, [&](int zy, int x) { return src[zy * P + x]; },
        [&](int zy, int d, T v) { t1[d * kD + zy] = v; });
    __syncthreads();
    contract<P, P, P2, W, T>(
        wave, lane, m + ((c >> 1) & 1) * P2, [&](int zd, int y) { return t1[zd % P * kD + zd / P * P + y]; },
        [&](int zd, int b, T v) { t2[zd / P * kZ + b * P + zd % P] = v; });
    __syncthreads();
    T* o = part + (J * 8 + c) * P3;
    contract<P, P, P2, W, T>(
        wave, lane, m + ((c >> 2) & 1) * P2, [&](int bd, int z) { return t2[z * kZ + bd]; },
        [&](int bd, int a, T v) { o[a * P2 + bd] = v; });
}

template <typename T, int P>
__global__ void __launch_bounds__(kSumThreads)
    k_reg_up_sum(const T* __restrict__ part, const int32_t* __restrict__ child8, T* __restrict__ out, int64_t np) {
    constexpr int P3 = P * P * P;
    const int64_t g = (int64_t)blockIdx.x * kSumThreads + threadIdx.x;
    if (g >= np * P3) return;
    const int64_t J = g / P3;
    const int i = (int)(g - J * P3);
    T acc = T(0);
    for (int c = 0; c < 8; ++c)
        if (child8[J * 8 + c] >= 0) acc += part[(J * 8 + c) * P3 + i];
    out[g] = acc;
}

template <int P>
__global__ void __launch_bounds__(kLatThreads)
    k_interp_down_one(const double* __restrict__ par, const int32_t* __restrict__ child8,
                      const double* __restrict__ Ct, double* __restrict__ io) {
    constexpr int P2 = P * P, P3 = P2 * P;
    __shared__ double R[interp_values<P>()];
    const int64_t J = blockIdx.x >> 3;
    const int c = blockIdx.x & 7;
    const int q = child8[J * 8 + c];  // uniform
    if (q < 0) return;
    double* dst = io + (int64_t)q * P3;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double rows[P];
    interp_rows<P, kLatThreads / 64>(par + J * P3, wave, lane, rows);
    interp_child<P, kLatThreads / 64>(rows, c, uniform_ptr(Ct), R, wave, lane,
                                      [&](int yx, int z) -> double& { return dst[z * P2 + yx]; });
}

// Level-1 node values of the lattice scheme (p = n + 1 nodes on the grid points, Reg the
// identity on n^3 and a zero last plane): a padded copy, out[b] = [f[b]; 0] in each axis.
template <typename T>
__global__ void k_pad_copy(const T* __restrict__ f, T* __restrict__ out, int64_t nb, int n, int p) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t p3 = (int64_t)p * p * p;
    if (g >= nb * p3) return;
    const int64_t b = g / p3;
    const int r = (int)(g - b * p3);
    const int x = r % p, y = (r / p) % p, z = r / (p * p);
    out[g] = (x < n && y < n && z < n) ? f[((b * n + z) * n + y) * n + x] : T(0);
}

// ------------------------------------------------------------------ level 1 -> block, FP64 add-back
// The near-field values that this lane's share of the final z pass adds to (read ahead; zeros, and
// not read, without a near field).  Every thread reads the elements it writes, so u may alias vnear.
template <int N, int W>
using FinalShare = Share<N, N * N, W>;
template <typename T, int N, int W>
__device__ __forceinline__ void near_values(const T* vnear, int64_t b, bool has_near, int wave, int lane,
                                            T (&near)[FinalShare<N, W>::CH]) {
    using Sh = FinalShare<N, W>;
    static_assert(Sh::TASKS <= W, "one share per wave");
    const int yx = Sh::col(wave, lane), z0 = Sh::out0(wave);
    const T* v = vnear + b * (N * N * N);
    const bool on = has_near && wave < Sh::TASKS && yx < N * N;
#pragma unroll
    for (int i = 0; i < Sh::CH; ++i) near[i] = on && z0 + i < N ? v[(z0 + i) * (N * N) + yx] : T(0);
}

// u[b] from the level-1 node values V (LDS, rows of P values, P + 1 apart; visible to the
// workgroup) and near (near_values).  At: [N][P], the rows of A^T; R: final_values<N, P>() doubles.
template <int N, int P>
constexpr int final_values() { return P * P * (N + 1) + P * (N * N + 8); }
template <typename T, int N, int P, int W>
__device__ __forceinline__ void final_passes(const double* V, Uniform<double> At, double* R,
                                             const T (&near)[FinalShare<N, W>::CH], T* u, int64_t b, int wave,
                                             int lane) {
    constexpr int N2 = N * N, kX = N + 1, kA = N2 + 8;
    double *t1 = R, *t2 = R + P * P * kX;  // t1[a c][x], t2[a][y x]
    contract<P, N, P * P, W, double>(
        wave, lane, At, [&](int ac, int d) { return V[ac * (P + 1) + d]; },
        [&](int ac, int x, double v) { t1[ac * kX + x] = v; });
    __syncthreads();
    contract<P, N, P * N, W, double>(
        wave, lane, At, [&](int ax, int c) { return t1[(ax / N * P + c) * kX + ax % N]; },
        [&](int ax, int y, double v) { t2[ax / N * kA + y * N + ax % N] = v; });
    __syncthreads();
    T* o = u + b * (N2 * N);
    contract_onto<P, N, N2, W, double>(
        wave, lane, At, [&](int yx, int a) { return t2[a * kA + yx]; }, [&](int, int, int i) { return near[i]; },
        [&](int yx, int z, double acc, T v) { o[z * N2 + yx] = (T)((double)v + acc); });
}

// The level-1 inverse transform, Interp from level 2 and the interpolation to the block in one
// workgroup per evaluation block (p <= 10).
template <typename T, int N, int P>
__global__ void __launch_bounds__(kInvThreads)
    k_final_far(const T* vnear, const cplx<T>* __restrict__ uhat, int64_t nint, const double* __restrict__ up,
                const int32_t* __restrict__ par, const double* __restrict__ Ct, const double* __restrict__ At, T* u,
                const int32_t* __restrict__ l1map, const int32_t* __restrict__ near_flag) {
    __shared__ alignas(16)
        double R[imax(imax(2 * tile_values<P>(), interp_values<P>()), final_values<N, P>())];
    __shared__ double V[P * P * (P + 1)];
    const int tid = threadIdx.x;
    const int64_t b = blockIdx.x;
    const int64_t q = l1map ? (int64_t)uniform_ptr(l1map)[b] : b;  // level-1 interval of this block
    constexpr int W = kInvThreads / 64;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool has_near = !near_flag || near_flag[b];
    T near[FinalShare<N, W>::CH];
    node_values<T, P, P + 1, kInvThreads>(uhat, nint, up, par, uniform_ptr(Ct), q, R, V, tid, [&] {
        near_values<T, N, W>(vnear, b, has_near, wave, lane, near);
    });
    final_passes<T, N, P, W>(V, uniform_ptr(At), R, near, u, b, wave, lane);
}

// From node values in HBM (the lattice scheme).
template <typename T, int N, int P>
__global__ void __launch_bounds__(kLatThreads)
    k_final(const T* vnear, const double* __restrict__ ut, const double* __restrict__ At, T* u,
            const int32_t* __restrict__ l1map, const int32_t* __restrict__ near_flag) {
    constexpr int P3 = P * P * P, PR = P + 1;
    __shared__ double V[P * P * PR], R[final_values<N, P>()];
    const int tid = threadIdx.x;
    const int64_t b = blockIdx.x;
    const int64_t q = l1map ? (int64_t)uniform_ptr(l1map)[b] : b;  // level-1 interval of this block
    constexpr int W = kLatThreads / 64;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    T near[FinalShare<N, W>::CH];
    near_values<T, N, W>(vnear, b, !near_flag || near_flag[b], wave, lane, near);
    for (int i = tid; i < P3; i += kLatThreads) V[(i / P) * PR + i % P] = ut[q * P3 + i];
    __syncthreads();
    final_passes<T, N, P, W>(V, uniform_ptr(At), R, near, u, b, wave, lane);
}

// ------------------------------------------------------------------ launchers
// p <= 10 -> compile-time kernel
template <template <int> class K, typename... Args>
static hipError_t dispatch_p(int p, Args... args) {
    switch (p) {
        case 2: return K<2>::run(args...);
        case 3: return K<3>::run(args...);
        case 4: return K<4>::run(args...);
        case 5: return K<5>::run(args...);
        case 6: return K<6>::run(args...);
        case 7: return K<7>::run(args...);
        case 8: return K<8>::run(args...);
        case 9: return K<9>::run(args...);
        case 10: return K<10>::run(args...);
        default: return hipErrorInvalidValue;
    }
}

// n in {4, 6, 8, 12, 16} too
template <template <int> class K, typename... Args>
static hipError_t dispatch_np(int n, int p, Args... args) {
    switch (n) {
        case 4: return dispatch_p<K<4>::template At>(p, args...);
        case 6: return dispatch_p<K<6>::template At>(p, args...);
        case 8: return dispatch_p<K<8>::template At>(p, args...);
        case 12: return dispatch_p<K<12>::template At>(p, args...);
        case 16: return dispatch_p<K<16>::template At>(p, args...);
        default: return hipErrorInvalidValue;
    }
}

template <typename T>
struct RegFft {
    template <int N>
    struct K {
        template <int P>
        struct At {
            static hipError_t run(const T* f, const T* A, T* ftil, cplx<T>* fhat, int64_t nb, int64_t nout,
                                  hipStream_t s) {
                return lgf_launch(k_reg_fft<T, N, P>, dim3((unsigned)nb), dim3(kBlockThreads), 0, s, f, A, ftil, fhat,
                                  nout);
            }
        };
    };
};

template <typename T>
struct RegupFft {
    template <int P>
    struct K {
        static hipError_t run(const T* in, const int32_t* child8, const T* C01, T* ftil, cplx<T>* fhat,
                              int64_t np, int64_t nout, hipStream_t s) {
            return lgf_launch(k_regup_fft<T, P>, dim3((unsigned)np), dim3(kRegUpThreads), 0, s, in, child8, C01, ftil,
                              fhat, nout);
        }
    };
};

template <typename T>
struct InvInterp {
    template <int P>
    struct K {
        static hipError_t run(const cplx<T>* uhat, const double* up, const int32_t* par, const double* Ct,
                              double* out, int64_t nint, hipStream_t s) {
            return lgf_launch(k_inv_interp<T, P>, dim3((unsigned)nint), dim3(kInvThreads), 0, s, uhat, up, par, Ct,
                              out);
        }
    };
};

template <typename T>
struct FinalFar {
    template <int N>
    struct K {
        template <int P>
        struct At {
            static hipError_t run(const T* vnear, const cplx<T>* uhat, int64_t nint, const double* up,
                                  const int32_t* par, const double* Ct, const double* At, T* u, int64_t nb,
                                  hipStream_t s, const int32_t* l1map, const int32_t* near_flag) {
                return lgf_launch(k_final_far<T, N, P>, dim3((unsigned)nb), dim3(kInvThreads), 0, s, vnear, uhat,
                                  nint, up, par, Ct, At, u, l1map, near_flag);
            }
        };
    };
};

template <typename T>
hipError_t launch_reg_fft(const T* f, const T* A, T* ftil, cplx<T>* fhat, int64_t nb, int64_t nout, int n, int p,
                          hipStream_t s) {
    if (nb <= 0) return hipSuccess;
    return dispatch_np<RegFft<T>::template K>(n, p, f, A, ftil, fhat, nb, nout, s);
}

template <typename T>
hipError_t launch_regup_fft(const T* in, const int32_t* child8, const T* C01, T* ftil, cplx<T>* fhat, int64_t np,
                            int64_t nout, int p, hipStream_t s) {
    if (np <= 0) return hipSuccess;
    return dispatch_p<RegupFft<T>::template K>(p, in, child8, C01, ftil, fhat, np, nout, s);
}

template <typename T>
hipError_t launch_inv_interp(const cplx<T>* uhat, const double* up, const int32_t* par, const double* Ct,
                             double* out, int64_t nint, int p, hipStream_t s) {
    if (nint <= 0) return hipSuccess;
    return dispatch_p<InvInterp<T>::template K>(p, uhat, up, par, Ct, out, nint, s);
}

template <typename T>
hipError_t launch_final_far(const T* vnear, const cplx<T>* uhat, int64_t nint, const double* up, const int32_t* par,
                            const double* Ct, const double* At, T* u, int64_t nb, int n, int p, hipStream_t s,
                            const int32_t* l1map, const int32_t* near_flag) {
    if (nb <= 0) return hipSuccess;
    return dispatch_np<FinalFar<T>::template K>(n, p, vnear, uhat, nint, up, par, Ct, At, u, nb, s, l1map, near_flag);
}

// One workgroup per (parent, child) writes each child's contribution to scratch, a second
// kernel adds them in child order (eight children of 13^3 or 17^3 nodes do not fit one
// workgroup's LDS).
template <typename T, int P>
static hipError_t reg_up_parts(const T* in, const int32_t* child8, const T* C01, T* out, int64_t np,
                               hipStream_t s, void* scratch) {
    constexpr int P3 = P * P * P;
    if (!scratch) return hipErrorInvalidValue;
    const hipError_t e = lgf_launch(k_reg_up_part<T, P>, dim3((unsigned)(np * 8)), dim3(kLatThreads), 0, s, in,
                                    child8, C01, (T*)scratch);
    if (e != hipSuccess) return e;
    return lgf_launch(k_reg_up_sum<T, P>, dim3((unsigned)((np * P3 + kSumThreads - 1) / kSumThreads)),
                      dim3(kSumThreads), 0, s, (const T*)scratch, child8, out, np);
}

template <typename T>
hipError_t launch_reg_up(const T* in, const int32_t* child8, const T* C01, T* out, int64_t np, int p,
                         hipStream_t s, void* scratch) {
    if (np <= 0) return hipSuccess;
    switch (p) {
        case 13: return reg_up_parts<T, 13>(in, child8, C01, out, np, s, scratch);
        case 17: return reg_up_parts<T, 17>(in, child8, C01, out, np, s, scratch);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_interp_down(const double* par, const int32_t* child8, const double* Ct, double* io,
                              int64_t nparent, int p, hipStream_t s) {
    if (nparent <= 0) return hipSuccess;
    const dim3 grid((unsigned)(nparent * 8)), block(kLatThreads);
    switch (p) {
        case 13: return lgf_launch(k_interp_down_one<13>, grid, block, 0, s, par, child8, Ct, io);
        case 17: return lgf_launch(k_interp_down_one<17>, grid, block, 0, s, par, child8, Ct, io);
        default: return hipErrorInvalidValue;
    }
}

template <typename T>
hipError_t launch_pad_copy(const T* f, T* out, int64_t nb, int n, int p, hipStream_t s) {
    if (nb <= 0) return hipSuccess;
    const int64_t tot = nb * (int64_t)p * p * p;
    return lgf_launch(k_pad_copy<T>, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, f, out, nb, n, p);
}

template <typename T>
hipError_t launch_final(const T* vnear, const double* ut, const double* At, T* u, int64_t nb, int n, int p,
                        hipStream_t s, const int32_t* l1map, const int32_t* near_flag) {
    if (nb <= 0) return hipSuccess;
    const dim3 grid((unsigned)nb), block(kLatThreads);
    if (n == 12 && p == 13) return lgf_launch(k_final<T, 12, 13>, grid, block, 0, s, vnear, ut, At, u, l1map, near_flag);
    if (n == 16 && p == 17) return lgf_launch(k_final<T, 16, 17>, grid, block, 0, s, vnear, ut, At, u, l1map, near_flag);
    return hipErrorInvalidValue;
}

#define LGF_INST(T)                                                                                                 \
    template hipError_t launch_reg_fft<T>(const T*, const T*, T*, cplx<T>*, int64_t, int64_t, int, int,        \
                                          hipStream_t);                                                             \
    template hipError_t launch_regup_fft<T>(const T*, const int32_t*, const T*, T*, cplx<T>*, int64_t, int64_t, \
                                            int, hipStream_t);                                                      \
    template hipError_t launch_inv_interp<T>(const cplx<T>*, const double*, const int32_t*, const double*, double*, \
                                             int64_t, int, hipStream_t);                                            \
    template hipError_t launch_final_far<T>(const T*, const cplx<T>*, int64_t, const double*, const int32_t*,       \
                                            const double*, const double*, T*, int64_t, int, int, hipStream_t,       \
                                            const int32_t*, const int32_t*);                                        \
    template hipError_t launch_reg_up<T>(const T*, const int32_t*, const T*, T*, int64_t, int, hipStream_t,    \
                                         void*);                                                                    \
    template hipError_t launch_pad_copy<T>(const T*, T*, int64_t, int, int, hipStream_t);                           \
    template hipError_t launch_final<T>(const T*, const double*, const double*, T*, int64_t, int, int, hipStream_t, \
                                        const int32_t*, const int32_t*);
LGF_INST(double)
LGF_INST(float)
#undef LGF_INST

}  // namespace lgfdev

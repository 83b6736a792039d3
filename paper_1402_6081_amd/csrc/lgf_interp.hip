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
// The passes are latency-bound (a few barriers over little data).
#include <type_traits>

#include "lgf_internal.h"
#include "lgf_tile.h"

namespace lgfdev {

constexpr int kInterpThreads = 256;
// Reg up works on eight children per workgroup: more waves hide the latency of its few, long
// workgroups
constexpr int kRegUpThreads = 1024;
// block -> level 1
constexpr int kBlockThreads = 512;
// Interp down of the lattice scheme (one workgroup per (parent, child))
constexpr int kDownThreads = 512;
// inverse transform, Interp and the final pass
constexpr int kInvThreads = 256;

constexpr int imax(int a, int b) { return a > b ? a : b; }

// ------------------------------------------------------------------ block -> level 1
// One workgroup per block: the block is staged in LDS with coalesced loads, then the
// three passes run from LDS with compile-time extents, and the forward transform of the node
// values.  Rows that a wave reads at several indices at once (the block's x rows, the matrix
// rows) are padded to N + 1 values, so the reads fall into different LDS banks.
template <typename T, int N, int P>
__global__ void __launch_bounds__(kBlockThreads)
    k_reg_fft(const T* __restrict__ f, const double* __restrict__ A, T* __restrict__ ftil,
              cplx<T>* __restrict__ fhat, int64_t nout) {
    constexpr int N3 = N * N * N, P3 = P * P * P, NR = N + 1;
    constexpr int kX = N * N * NR, kT1 = N * N * P, kT2 = N * P * P;
    constexpr int kFront = (imax(kX + kT1, 2 * tile_values<P>()) + 1) / 2 * 2;  // X and t1, then the transform
    __shared__ alignas(16) T lds[kFront + kT2 + P * NR];
    T *X = lds, *t1 = lds + kX, *t2 = lds + kFront, *Am = t2 + kT2;
    cplx<T>* buf = reinterpret_cast<cplx<T>*>(lds);
    const int tid = threadIdx.x;
    const int64_t b = blockIdx.x;
    for (int i = tid; i < P * N; i += kBlockThreads) Am[(i / N) * NR + i % N] = (T)A[i];
    const T* src = f + b * N3;
    for (int i = tid; i < N3; i += kBlockThreads) X[(i / N) * NR + i % N] = src[i];
    __syncthreads();
    for (int i = tid; i < N * N * P; i += kBlockThreads) {  // x: t1[z][y][d]
        const int d = i % P, zy = i / P;
        const T* row = X + zy * NR;
        const T* m = Am + d * NR;
        T acc = T(0);
#pragma unroll
        for (int x = 0; x < N; ++x) acc += m[x] * row[x];
        t1[i] = acc;
    }
    __syncthreads();
    for (int i = tid; i < N * P * P; i += kBlockThreads) {  // y: t2[z][c][d]
        const int d = i % P, c = (i / P) % P, z = i / (P * P);
        const T* m = Am + c * NR;
        const T* col = t1 + z * N * P + d;
        T acc = T(0);
#pragma unroll
        for (int y = 0; y < N; ++y) acc += m[y] * col[y * P];
        t2[i] = acc;
    }
    __syncthreads();
    for (int i = tid; i < P3; i += kBlockThreads) {  // z: node values [a][c][d]
        const int cd = i % (P * P), a = i / (P * P);
        const T* m = Am + a * NR;
        T acc = T(0);
#pragma unroll
        for (int z = 0; z < N; ++z) acc += m[z] * t2[z * (P * P) + cd];
        if (ftil) ftil[b * P3 + i] = acc;
        staged<T, P>(buf, a, cd / P, cd % P) = acc;
    }
    if (!fhat) return;
    __syncthreads();
    tile_forward<T, P, kBlockThreads>(buf, tid, fhat, (size_t)b, nout);
}

// ------------------------------------------------------------------ children -> parent
template <typename T, int P>
__global__ void __launch_bounds__(kRegUpThreads)
    k_regup_fft(const T* __restrict__ in, const int32_t* __restrict__ child8, const double* __restrict__ C01,
                T* __restrict__ ftil, cplx<T>* __restrict__ fhat, int64_t nout) {
    constexpr int P3 = P * P * P, NT = kRegUpThreads;
    static_assert(8 * P3 >= 2 * tile_values<P>(), "the transform's tile fits in t1");
    __shared__ alignas(16) T X[8 * P3], t1[8 * P3];
    __shared__ T Cm[2 * P * P];
    __shared__ int32_t ch[8];
    cplx<T>* buf = reinterpret_cast<cplx<T>*>(t1);
    const int tid = threadIdx.x;
    const int64_t J = blockIdx.x;
    for (int i = tid; i < 2 * P * P; i += NT) Cm[i] = (T)C01[i];
    if (tid < 8) ch[tid] = child8[J * 8 + tid];
    __syncthreads();
    for (int i = tid; i < 8 * P3; i += NT) {
        const int c = i / P3, r = i - c * P3;
        const int q = ch[c];
        X[i] = q >= 0 ? in[(int64_t)q * P3 + r] : T(0);
    }
    __syncthreads();
    // x: t1[c][z][y][d] = sum_x C_cx[d][x] X[c][z][y][x]
    for (int i = tid; i < 8 * P3; i += NT) {
        const int d = i % P, rest = i / P, c = i / P3;
        const T* m = Cm + (c & 1) * P * P + d * P;
        const T* row = X + rest * P;
        T s = T(0);
#pragma unroll
        for (int x = 0; x < P; ++x) s += m[x] * row[x];
        t1[i] = s;
    }
    __syncthreads();
    // y: X[c][z][b][d] = sum_y C_cy[b][y] t1[c][z][y][d]
    for (int i = tid; i < 8 * P3; i += NT) {
        const int d = i % P, bb = (i / P) % P, cz = i / (P * P), c = i / P3;
        const T* m = Cm + ((c >> 1) & 1) * P * P + bb * P;
        T s = T(0);
#pragma unroll
        for (int y = 0; y < P; ++y) s += m[y] * t1[(cz * P + y) * P + d];
        X[i] = s;
    }
    __syncthreads();
    // z and the sum over children: node values [a][b][d] = sum_c sum_z C_cz[a][z] X[c][z][b][d]
    for (int i = tid; i < P3; i += NT) {
        const int bd = i % (P * P), a = i / (P * P);
        T s = T(0);
        for (int c = 0; c < 8; ++c) {
            if (ch[c] < 0) continue;
            const T* m = Cm + ((c >> 2) & 1) * P * P + a * P;
#pragma unroll
            for (int z = 0; z < P; ++z) s += m[z] * X[c * P3 + z * P * P + bd];
        }
        if (ftil) ftil[J * P3 + i] = s;
        staged<T, P>(buf, a, bd / P, bd % P) = s;
    }
    if (!fhat) return;
    __syncthreads();
    tile_forward<T, P, NT>(buf, tid, fhat, (size_t)J, nout);
}

// ------------------------------------------------------------------ inverse and parent -> child
// The node values of interval q (rows of P values, VP apart) into V: the inverse transform of its
// field spectrum (uhat NULL: zeros) plus Interp from its parent (par[q] = 8 J + c, -1: none;
// up NULL: no level above).  R: 2 tile_values<P>() doubles, Xp: P^3, Ct: 2 P^2, used on the way.
template <typename T, int P, int VP, int NT>
__device__ __forceinline__ void node_values(const cplx<T>* __restrict__ uhat, int64_t nint,
                                            const double* __restrict__ up, const int32_t* __restrict__ par,
                                            const double* __restrict__ C01, int64_t q, double* R, double* Xp,
                                            double* Ct, double* V, int tid) {
    constexpr int P3 = P * P * P, P2 = P * P;
    static_assert(tile_values<P>() >= P3, "the two passes' values fit in R");
    const int pc = up ? par[q] : -1;  // uniform
    if (pc >= 0) {
        for (int i = tid; i < P3; i += NT) Xp[i] = up[(int64_t)(pc >> 3) * P3 + i];
        for (int i = tid; i < 2 * P2; i += NT) {  // Ct_c[k][m] = C_c[m][k]
            const int cc = i / P2, r = i % P2, k = r / P, m = r % P;
            Ct[i] = C01[cc * P2 + m * P + k];
        }
    }
    if (uhat) {
        cplx<double>* buf = reinterpret_cast<cplx<double>*>(R);
        tile_inverse<T, double, P, NT>(uhat, (size_t)q, nint, buf, tid);
        __syncthreads();
        for (int i = tid; i < P3; i += NT) V[(i / P) * VP + i % P] = staged<double, P>(buf, i / P2, i / P % P, i % P);
    } else {
        for (int i = tid; i < P3; i += NT) V[(i / P) * VP + i % P] = 0.0;
    }
    __syncthreads();
    if (pc < 0) return;
    const int cx = pc & 1, cy = (pc >> 1) & 1, cz = (pc >> 2) & 1;
    double *t1 = R, *t2 = R + P3;
    for (int i = tid; i < P3; i += NT) {  // x: t1[a][b][x']
        const int xo = i % P, ab = i / P;
        const double* m = Ct + cx * P2 + xo * P;
        const double* row = Xp + ab * P;
        double sum = 0.0;
#pragma unroll
        for (int d = 0; d < P; ++d) sum += m[d] * row[d];
        t1[i] = sum;
    }
    __syncthreads();
    for (int i = tid; i < P3; i += NT) {  // y: t2[a][y'][x']
        const int xo = i % P, yo = (i / P) % P, a = i / P2;
        const double* m = Ct + cy * P2 + yo * P;
        const double* src = t1 + a * P2 + xo;
        double sum = 0.0;
#pragma unroll
        for (int bb = 0; bb < P; ++bb) sum += m[bb] * src[bb * P];
        t2[i] = sum;
    }
    __syncthreads();
    for (int i = tid; i < P3; i += NT) {  // z, added to the interval's own values
        const int yx = i % P2, zo = i / P2;
        const double* m = Ct + cz * P2 + zo * P;
        double sum = 0.0;
#pragma unroll
        for (int a = 0; a < P; ++a) sum += m[a] * t2[a * P2 + yx];
        double* v = V + (i / P) * VP + i % P;
        *v = *v + sum;
    }
    __syncthreads();
}

template <typename T, int P>
__global__ void __launch_bounds__(kInvThreads)
    k_inv_interp(const cplx<T>* __restrict__ uhat, const double* __restrict__ up, const int32_t* __restrict__ par,
                 const double* __restrict__ C01, double* __restrict__ out) {
    constexpr int P3 = P * P * P;
    __shared__ alignas(16) double R[2 * tile_values<P>()];
    __shared__ double Xp[P3], Ct[2 * P * P], V[P3];
    const int64_t q = blockIdx.x;
    node_values<T, P, P, kInvThreads>(uhat, gridDim.x, up, par, C01, q, R, Xp, Ct, V, threadIdx.x);
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
__global__ void __launch_bounds__(kInterpThreads)
    k_reg_up_part(const T* __restrict__ in, const int32_t* __restrict__ child8, const double* __restrict__ C01,
                  T* __restrict__ part) {
    constexpr int P3 = P * P * P;
    __shared__ T X[P3], t1[P3];
    __shared__ T Cm[2 * P * P];
    const int tid = threadIdx.x;
    const int64_t J = blockIdx.x >> 3;
    const int c = blockIdx.x & 7;
    const int q = child8[J * 8 + c];  // uniform
    if (q < 0) return;
    for (int i = tid; i < 2 * P * P; i += kInterpThreads) Cm[i] = (T)C01[i];
    for (int i = tid; i < P3; i += kInterpThreads) X[i] = in[(int64_t)q * P3 + i];
    __syncthreads();
    for (int i = tid; i < P3; i += kInterpThreads) {  // x: t1[z][y][d]
        const int d = i % P, rest = i / P;
        const T* m = Cm + (c & 1) * P * P + d * P;
        const T* row = X + rest * P;
        T sum = T(0);
#pragma unroll
        for (int x = 0; x < P; ++x) sum += m[x] * row[x];
        t1[i] = sum;
    }
    __syncthreads();
    for (int i = tid; i < P3; i += kInterpThreads) {  // y: X[z][b][d]
        const int d = i % P, bb = (i / P) % P, z = i / (P * P);
        const T* m = Cm + ((c >> 1) & 1) * P * P + bb * P;
        T sum = T(0);
#pragma unroll
        for (int y = 0; y < P; ++y) sum += m[y] * t1[(z * P + y) * P + d];
        X[i] = sum;
    }
    __syncthreads();
    T* o = part + (J * 8 + c) * P3;
    for (int i = tid; i < P3; i += kInterpThreads) {  // z
        const int bd = i % (P * P), a = i / (P * P);
        const T* m = Cm + ((c >> 2) & 1) * P * P + a * P;
        T sum = T(0);
#pragma unroll
        for (int z = 0; z < P; ++z) sum += m[z] * X[z * P * P + bd];
        o[i] = sum;
    }
}

template <typename T, int P>
__global__ void __launch_bounds__(kInterpThreads)
    k_reg_up_sum(const T* __restrict__ part, const int32_t* __restrict__ child8, T* __restrict__ out, int64_t np) {
    constexpr int P3 = P * P * P;
    const int64_t g = (int64_t)blockIdx.x * kInterpThreads + threadIdx.x;
    if (g >= np * P3) return;
    const int64_t J = g / P3;
    const int i = (int)(g - J * P3);
    T acc = T(0);
    for (int c = 0; c < 8; ++c)
        if (child8[J * 8 + c] >= 0) acc += part[(J * 8 + c) * P3 + i];
    out[g] = acc;
}

template <int P>
__global__ void __launch_bounds__(kDownThreads)
    k_interp_down_one(const double* __restrict__ par, const int32_t* __restrict__ child8, const double* __restrict__ C01,
                      double* __restrict__ io) {
    constexpr int P3 = P * P * P;
    __shared__ double X[P3], t1[P3], t2[P3];
    __shared__ double Ct[2 * P * P];  // Ct_c[k][m] = C_c[m][k]
    const int tid = threadIdx.x;
    const int64_t J = blockIdx.x >> 3;
    const int c = blockIdx.x & 7;
    const int q = child8[J * 8 + c];  // uniform
    if (q < 0) return;
    const int cx = c & 1, cy = (c >> 1) & 1, cz = (c >> 2) & 1;
    for (int i = tid; i < 2 * P * P; i += kDownThreads) {
        const int cc = i / (P * P), r = i % (P * P), k = r / P, m = r % P;
        Ct[i] = C01[cc * P * P + m * P + k];
    }
    for (int i = tid; i < P3; i += kDownThreads) X[i] = par[J * P3 + i];
    __syncthreads();
    for (int i = tid; i < P3; i += kDownThreads) {  // x: t1[a][b][x']
        const int xo = i % P, ab = i / P;
        const double* m = Ct + cx * P * P + xo * P;
        const double* row = X + ab * P;
        double sum = 0.0;
#pragma unroll
        for (int d = 0; d < P; ++d) sum += m[d] * row[d];
        t1[i] = sum;
    }
    __syncthreads();
    for (int i = tid; i < P3; i += kDownThreads) {  // y: t2[a][y'][x']
        const int xo = i % P, yo = (i / P) % P, a = i / (P * P);
        const double* m = Ct + cy * P * P + yo * P;
        const double* src = t1 + a * P * P + xo;
        double sum = 0.0;
#pragma unroll
        for (int bb = 0; bb < P; ++bb) sum += m[bb] * src[bb * P];
        t2[i] = sum;
    }
    __syncthreads();
    for (int i = tid; i < P3; i += kDownThreads) {  // z, accumulated into the child
        const int yx = i % (P * P), zo = i / (P * P);
        const double* m = Ct + cz * P * P + zo * P;
        double sum = 0.0;
#pragma unroll
        for (int a = 0; a < P; ++a) sum += m[a] * t2[a * P * P + yx];
        double* dst = io + (int64_t)q * P3 + i;
        *dst = *dst + sum;
    }
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
// u[b] from the level-1 node values X (rows of P values, P + 1 apart: rows that a wave reads at
// several indices at once fall into different LDS banks).  At: N (P + 1) values, the rows of A^T;
// t1: P^2 N, t2: P N^2.  At and X are visible to the workgroup.
template <typename T, int N, int P, int NT>
__device__ __forceinline__ void final_passes(const double* X, const double* At, double* t1, double* t2,
                                             const T* vnear, T* u, int64_t b, bool has_near, int tid) {
    constexpr int N3 = N * N * N, PR = P + 1;
    for (int i = tid; i < P * P * N; i += NT) {  // x: t1[a][c][x]
        const int x = i % N, ac = i / N;
        const double* m = At + x * PR;
        const double* row = X + ac * PR;
        double acc = 0.0;
#pragma unroll
        for (int d = 0; d < P; ++d) acc += m[d] * row[d];
        t1[i] = acc;
    }
    __syncthreads();
    for (int i = tid; i < P * N * N; i += NT) {  // y: t2[a][y][x]
        const int x = i % N, y = (i / N) % N, a = i / (N * N);
        const double* m = At + y * PR;
        const double* col = t1 + a * P * N + x;
        double acc = 0.0;
#pragma unroll
        for (int c = 0; c < P; ++c) acc += m[c] * col[c * N];
        t2[i] = acc;
    }
    __syncthreads();
    const T* v = vnear + b * N3;
    T* o = u + b * N3;
    for (int i = tid; i < N3; i += NT) {  // z: u[z][y][x]
        const int yx = i % (N * N), z = i / (N * N);
        const double* m = At + z * PR;
        double acc = 0.0;
#pragma unroll
        for (int a = 0; a < P; ++a) acc += m[a] * t2[a * N * N + yx];
        o[i] = (T)((has_near ? (double)v[i] : 0.0) + acc);  // no near field: v is not read
    }
}

// At[j][k] = A[k][j], rows P + 1 apart
template <int N, int P, int NT>
__device__ __forceinline__ void load_at(const double* __restrict__ A, double* At, int tid) {
    for (int i = tid; i < N * P; i += NT) At[(i / P) * (P + 1) + i % P] = A[(i % P) * N + i / P];
}

// The level-1 inverse transform, Interp from level 2 and the interpolation to the block in one
// workgroup per evaluation block (p <= 10).
template <typename T, int N, int P>
__global__ void __launch_bounds__(kInvThreads)
    k_final_far(const T* vnear, const cplx<T>* __restrict__ uhat, int64_t nint, const double* __restrict__ up,
                const int32_t* __restrict__ par, const double* __restrict__ C01, const double* __restrict__ A, T* u,
                const int32_t* __restrict__ l1map, const int32_t* __restrict__ near_flag) {
    constexpr int P3 = P * P * P, kT1 = P * P * N;
    __shared__ alignas(16) double R[imax(2 * tile_values<P>(), kT1 + P * N * N)];
    __shared__ double Xp[P3], Ct[2 * P * P], V[P * P * (P + 1)], At[N * (P + 1)];
    const int tid = threadIdx.x;
    const int64_t b = blockIdx.x;
    const int64_t q = l1map ? (int64_t)l1map[b] : b;  // level-1 interval of this block
    load_at<N, P, kInvThreads>(A, At, tid);
    node_values<T, P, P + 1, kInvThreads>(uhat, nint, up, par, C01, q, R, Xp, Ct, V, tid);
    final_passes<T, N, P, kInvThreads>(V, At, R, R + kT1, vnear, u, b, !near_flag || near_flag[b], tid);
}

// From node values in HBM (the lattice scheme).
template <typename T, int N, int P>
__global__ void __launch_bounds__(kBlockThreads)
    k_final(const T* vnear, const double* __restrict__ ut, const double* __restrict__ A, T* u,
            const int32_t* __restrict__ l1map, const int32_t* __restrict__ near_flag) {
    constexpr int P3 = P * P * P, PR = P + 1;
    __shared__ double X[P * P * PR], t1[P * P * N], t2[P * N * N];
    __shared__ double At[N * PR];
    const int tid = threadIdx.x;
    const int64_t b = blockIdx.x;
    load_at<N, P, kBlockThreads>(A, At, tid);
    const int64_t q = l1map ? (int64_t)l1map[b] : b;  // level-1 interval of this block
    for (int i = tid; i < P3; i += kBlockThreads) X[(i / P) * PR + i % P] = ut[q * P3 + i];
    __syncthreads();
    final_passes<T, N, P, kBlockThreads>(X, At, t1, t2, vnear, u, b, !near_flag || near_flag[b], tid);
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
            static hipError_t run(const T* f, const double* A, T* ftil, cplx<T>* fhat, int64_t nb, int64_t nout,
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
        static hipError_t run(const T* in, const int32_t* child8, const double* C01, T* ftil, cplx<T>* fhat,
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
        static hipError_t run(const cplx<T>* uhat, const double* up, const int32_t* par, const double* C01,
                              double* out, int64_t nint, hipStream_t s) {
            return lgf_launch(k_inv_interp<T, P>, dim3((unsigned)nint), dim3(kInvThreads), 0, s, uhat, up, par, C01,
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
                                  const int32_t* par, const double* C01, const double* A, T* u, int64_t nb,
                                  hipStream_t s, const int32_t* l1map, const int32_t* near_flag) {
                return lgf_launch(k_final_far<T, N, P>, dim3((unsigned)nb), dim3(kInvThreads), 0, s, vnear, uhat,
                                  nint, up, par, C01, A, u, l1map, near_flag);
            }
        };
    };
};

template <typename T>
hipError_t launch_reg_fft(const T* f, const double* A, T* ftil, cplx<T>* fhat, int64_t nb, int64_t nout, int n, int p,
                          hipStream_t s) {
    if (nb <= 0) return hipSuccess;
    return dispatch_np<RegFft<T>::template K>(n, p, f, A, ftil, fhat, nb, nout, s);
}

template <typename T>
hipError_t launch_regup_fft(const T* in, const int32_t* child8, const double* C01, T* ftil, cplx<T>* fhat, int64_t np,
                            int64_t nout, int p, hipStream_t s) {
    if (np <= 0) return hipSuccess;
    return dispatch_p<RegupFft<T>::template K>(p, in, child8, C01, ftil, fhat, np, nout, s);
}

template <typename T>
hipError_t launch_inv_interp(const cplx<T>* uhat, const double* up, const int32_t* par, const double* C01,
                             double* out, int64_t nint, int p, hipStream_t s) {
    if (nint <= 0) return hipSuccess;
    return dispatch_p<InvInterp<T>::template K>(p, uhat, up, par, C01, out, nint, s);
}

template <typename T>
hipError_t launch_final_far(const T* vnear, const cplx<T>* uhat, int64_t nint, const double* up, const int32_t* par,
                            const double* C01, const double* A, T* u, int64_t nb, int n, int p, hipStream_t s,
                            const int32_t* l1map, const int32_t* near_flag) {
    if (nb <= 0) return hipSuccess;
    return dispatch_np<FinalFar<T>::template K>(n, p, vnear, uhat, nint, up, par, C01, A, u, nb, s, l1map, near_flag);
}

// One workgroup per (parent, child) writes each child's contribution to scratch, a second
// kernel adds them in child order (eight children of 13^3 or 17^3 nodes do not fit one
// workgroup's LDS).
template <typename T, int P>
static hipError_t reg_up_parts(const T* in, const int32_t* child8, const double* C01, T* out, int64_t np,
                               hipStream_t s, void* scratch) {
    constexpr int P3 = P * P * P;
    if (!scratch) return hipErrorInvalidValue;
    const hipError_t e = lgf_launch(k_reg_up_part<T, P>, dim3((unsigned)(np * 8)), dim3(kInterpThreads), 0, s, in,
                                    child8, C01, (T*)scratch);
    if (e != hipSuccess) return e;
    return lgf_launch(k_reg_up_sum<T, P>, dim3((unsigned)((np * P3 + kInterpThreads - 1) / kInterpThreads)),
                      dim3(kInterpThreads), 0, s, (const T*)scratch, child8, out, np);
}

template <typename T>
hipError_t launch_reg_up(const T* in, const int32_t* child8, const double* C01, T* out, int64_t np, int p,
                         hipStream_t s, void* scratch) {
    if (np <= 0) return hipSuccess;
    switch (p) {
        case 13: return reg_up_parts<T, 13>(in, child8, C01, out, np, s, scratch);
        case 17: return reg_up_parts<T, 17>(in, child8, C01, out, np, s, scratch);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_interp_down(const double* par, const int32_t* child8, const double* C01, double* io,
                              int64_t nparent, int p, hipStream_t s) {
    if (nparent <= 0) return hipSuccess;
    const dim3 grid((unsigned)(nparent * 8)), block(kDownThreads);
    switch (p) {
        case 13: return lgf_launch(k_interp_down_one<13>, grid, block, 0, s, par, child8, C01, io);
        case 17: return lgf_launch(k_interp_down_one<17>, grid, block, 0, s, par, child8, C01, io);
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
hipError_t launch_final(const T* vnear, const double* ut, const double* A, T* u, int64_t nb, int n, int p,
                        hipStream_t s, const int32_t* l1map, const int32_t* near_flag) {
    if (nb <= 0) return hipSuccess;
    const dim3 grid((unsigned)nb), block(kBlockThreads);
    if (n == 12 && p == 13) return lgf_launch(k_final<T, 12, 13>, grid, block, 0, s, vnear, ut, A, u, l1map, near_flag);
    if (n == 16 && p == 17) return lgf_launch(k_final<T, 16, 17>, grid, block, 0, s, vnear, ut, A, u, l1map, near_flag);
    return hipErrorInvalidValue;
}

#define LGF_INST(T)                                                                                                 \
    template hipError_t launch_reg_fft<T>(const T*, const double*, T*, cplx<T>*, int64_t, int64_t, int, int,        \
                                          hipStream_t);                                                             \
    template hipError_t launch_regup_fft<T>(const T*, const int32_t*, const double*, T*, cplx<T>*, int64_t, int64_t, \
                                            int, hipStream_t);                                                      \
    template hipError_t launch_inv_interp<T>(const cplx<T>*, const double*, const int32_t*, const double*, double*, \
                                             int64_t, int, hipStream_t);                                            \
    template hipError_t launch_final_far<T>(const T*, const cplx<T>*, int64_t, const double*, const int32_t*,       \
                                            const double*, const double*, T*, int64_t, int, int, hipStream_t,       \
                                            const int32_t*, const int32_t*);                                        \
    template hipError_t launch_reg_up<T>(const T*, const int32_t*, const double*, T*, int64_t, int, hipStream_t,    \
                                         void*);                                                                    \
    template hipError_t launch_pad_copy<T>(const T*, T*, int64_t, int, int, hipStream_t);                           \
    template hipError_t launch_final<T>(const T*, const double*, const double*, T*, int64_t, int, int, hipStream_t, \
                                        const int32_t*, const int32_t*);
LGF_INST(double)
LGF_INST(float)
#undef LGF_INST

}  // namespace lgfdev

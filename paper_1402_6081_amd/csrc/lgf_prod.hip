// Level interactions (Step 2 of Sec. 3.1, Eq. alg_mult):
//   uhat^P = sum_{Q in InflList(P)} Prod(fhat^Q, khat^{P-Q}),
// independently for every DFT coefficient.
//
// Source spectra arrays hold one extra, all-zero item (index = item count) that stands in
// for inactive neighbours, so the inner loops load without branches or selects.
// Both blocked kernels exploit the lattice structure of the lists: the 8 targets that
// share a parent J see the same candidate sources (level 0: the 4^3 blocks 2J-1..2J+2;
// levels >= 1: the 6^3 children of the 27 neighbours of J) at offsets D = P - Q that
// depend only on the two child positions.  Each source spectrum is therefore read once per
// group instead of once per (target, source) pair, and the kernel spectra of a frequency
// chunk sit in an LDS tile shared by the workgroup (27 offsets at level 0, the 343 offsets
// of [-3, 3]^3 at levels >= 1).
// A plain CSR kernel covers the top level of a truncated tree, whose list is "every
// non-adjacent interval" and has no such structure.
#include <algorithm>
#include <cstdlib>

#include <type_traits>

#include "lgf_internal.h"

namespace lgfdev {

// Workgroups are dispatched round-robin over the 8 XCDs (each with its own L2).  Both
// blocked kernels map a 1D grid so that XCD x processes whole frequency chunks
// {c : c % 8 == x}, walking every group of such a chunk back to back: all reuse of a source
// spectrum within a chunk then stays in one L2.  Returns false for padding workgroups.
constexpr int kXcds = 8;
__device__ __forceinline__ bool xcd_tile_at(int L, int nchunks, int ngroupblocks, int& chunk, int& gblock) {
    const int xcd = L % kXcds, k = L / kXcds;
    chunk = (k / ngroupblocks) * kXcds + xcd;
    gblock = k % ngroupblocks;
    return chunk < nchunks;
}
__host__ __forceinline__ unsigned xcd_grid(int nchunks, int ngroupblocks) {
    const int padded = (nchunks + kXcds - 1) / kXcds * kXcds;
    return (unsigned)padded * (unsigned)ngroupblocks;
}

// complex multiply-accumulate as four FMAs
template <typename T>
__device__ __forceinline__ void cmac(T& ar, T& ai, const cplx<T>& f, const cplx<T>& k) {
    ar = fma(f.x, k.x, ar);
    ar = fma(-f.y, k.y, ar);
    ai = fma(f.x, k.y, ai);
    ai = fma(f.y, k.x, ai);
}

__device__ __forceinline__ int wave_uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Keeps the compiler from moving instructions across this point.  Placed after a batch of
// independent gathers, it keeps them issued together (all in flight at once) instead of
// each load being sunk to its first use, which left one or two loads in flight per wave.
__device__ __forceinline__ void issue_fence() { __builtin_amdgcn_sched_barrier(0); }

// Coefficient lane_off of item `item` in a frequency chunk whose items start at the
// wave-uniform `base` (64 coefficients per item).  A 32-bit byte offset from a uniform base
// lets the gather use a scalar base register plus one vector offset instead of 64-bit
// address arithmetic per load (the launchers check that a chunk spans less than 4 GiB).
template <typename T>
__device__ __forceinline__ cplx<T> load_item(const cplx<T>* base, int item, int lane_off) {
    const uint32_t off = ((uint32_t)item * 64u + (uint32_t)lane_off) * (uint32_t)sizeof(cplx<T>);
    return *reinterpret_cast<const cplx<T>*>(reinterpret_cast<const char*>(base) + off);
}
template <typename T>
__host__ __forceinline__ bool chunk_fits_u32(int64_t items) {
    return items * 64 * (int64_t)sizeof(cplx<T>) <= (int64_t)UINT32_MAX;
}

// A plan's list read at wave-uniform indices: lists do not change during a launch, so the reads
// may be scalar loads (constant address space).
typedef const __attribute__((address_space(4))) int32_t* ScalarList;
__device__ __forceinline__ ScalarList scalar_list(const int32_t* p) {
    return (ScalarList)(uintptr_t)p;
}

// 16 bytes per lane at p + off of a wave-uniform p, within [p, p + bytes): a lane out of range
// reads zeros or stores nothing (the buffer instructions' own range check), with no access to
// memory.  The address arithmetic stays in scalar registers.
template <typename T>
constexpr uint32_t kItemBytes = 64u * (uint32_t)sizeof(cplx<T>);  // an item's coefficients in one chunk
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr int kRawBuffer = 0x00020000;  // resource word 3: 32-bit elements, no swizzle
constexpr int kStream = 2;              // cache policy bit: nontemporal
template <typename V>
__device__ __forceinline__ V buffer_read(const char* p, uint32_t bytes, uint32_t off) {
    static_assert(sizeof(V) == 16, "one 16-byte access per lane");
    return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(
                                     __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, bytes, kRawBuffer), off, 0, 0));
}
template <typename V>
__device__ __forceinline__ void buffer_stream(char* p, uint32_t bytes, uint32_t off, const V& v) {
    static_assert(sizeof(V) == 16, "one 16-byte access per lane");
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v),
                                           __builtin_amdgcn_make_buffer_rsrc(p, 0, bytes, kRawBuffer), off, 0, kStream);
}
// The buffered loads have arrived: placed before a branch on their use, so that the wait is
// outside it and both ways leave the same loads in flight.
template <typename V, int N>
__device__ __forceinline__ void arrived(V (&x)[N]) {
    typedef unsigned int words __attribute__((ext_vector_type(sizeof(V) / 4)));
#pragma unroll
    for (int i = 0; i < N; ++i) {
        words r = __builtin_bit_cast(words, x[i]);
        asm volatile("" : "+v"(r));
        x[i] = __builtin_bit_cast(V, r);
    }
}

// ------------------------------------------------------------------ level 0
// Groups g: tgt8[g][c] = block 2J + c (c = cx | cy<<1 | cz<<2) or -1;
// src64[g][s] = source block 2J + (sx-1, sy-1, sz-1), s = sx + 4 sy + 16 sz, or the zero
// sentinel item (index nsrc) when that block is not a source.  fhat holds nsrc + 1 items
// (the last is 0), uhat ntgt items (targets and sources are numbered separately, so the
// evaluation blocks may differ from the source blocks).
// A lane owns FPL consecutive frequencies: FPL = 1, a wave covers one 64-frequency chunk;
// FPL = 2 (FP32), a wave covers two consecutive chunks, lanes 0-31 the first and 32-63 the
// second, each lane loading 16 bytes per item as the FP64 lanes do.  The waves of a
// workgroup are different groups of the same chunk(s) and share the kernel tile in LDS: the
// 27 near offsets, row (dx+1) + 3 (dy+1) + 9 (dz+1).  Every frequency is computed with the
// same arithmetic in the same order whatever FPL, the number of waves and the runs.
//
// A wave marches through a run, a stack of groups in z: source slab after source slab (16
// sources), each applied to the up to three target slabs it reaches, so a source slab inside
// the run is read once instead of once per group: 2R + 2 slabs for the 2R target slabs of R
// groups (4.5 reads per target at R = 8, 8 at R = 1).  Bound by those reads from L2, and now near
// the HBM rate: the 256^3 Prod went 612 -> 507 us in FP64 (3.7 -> 4.5 TB/s of its 2.3 GB, 78% of
// the 5.8 TB/s of a large elementwise copy) and 330 -> 286 us (4.0 TB/s) in FP32 with runs of 8,
// the 128^3 one 82 -> 71 us and 50 -> 45 us with runs of 4.
template <typename T, int FPL>
struct alignas(FPL * sizeof(cplx<T>)) LaneCoef {
    cplx<T> v[FPL];
};

template <typename T>
struct NearArgs {
    const cplx<T>* fhat;
    const cplx<T>* khat;
    const int32_t* tgt8;
    const int32_t* src64;
    const int32_t* runs;
    const int32_t* flags;
    cplx<T>* uhat;
    int S, nruns, nsrc, ntgt;
    SpecSym sym;
};

// Runs long enough for a workgroup's waves to march in lockstep.  Without and with it, us in FP64 /
// FP32 on 16^3 blocks: 256^3, runs of 8, 526 -> 498 / 300 -> 289; shorter runs in as large plans,
// 32 x 16 x 8 blocks (runs of 4) 515 -> 505 / 293 -> 284, 24 x 24 x 6 (of 3) 467 -> 455 / 263 -> 258;
// but 128^3 (of 4) 69 -> 72 / 42 -> 45, and where runs differ, the separate-set ring 253 -> 257 /
// 133 -> 137: 8 loses on none.
constexpr int kLockstepRun = 8;

template <typename T, int kNearWaves, int FPL>
__global__ void __launch_bounds__(64 * kNearWaves) k_prod_near_grouped(const NearArgs<T> a) {
    using V = LaneCoef<T, FPL>;
    __shared__ V tile[27 * 64];
    constexpr int NT = 64 * kNearWaves, NR = (27 * 64 + NT - 1) / NT;
    const cplx<T>* __restrict__ fhat = a.fhat;
    const cplx<T>* __restrict__ khat = a.khat;
    const ScalarList tgt8 = scalar_list(a.tgt8), src64 = scalar_list(a.src64), runs = scalar_list(a.runs),
                     flags = scalar_list(a.flags);
    cplx<T>* __restrict__ uhat = a.uhat;
    const int S = a.S, nruns = a.nruns, nsrc = a.nsrc, ntgt = a.ntgt;
    const SpecSym& sym = a.sym;
    const int lane = threadIdx.x & 63;
    const int nchunks = (S + 63) / 64;  // the last chunk may be partial (frequencies w >= S unused)
    int unit, gb;
    if (!xcd_tile_at((int)blockIdx.x, (nchunks + FPL - 1) / FPL, (nruns + kNearWaves - 1) / kNearWaves, unit, gb)) return;
    // this thread's chunk and first frequency in it; with FPL = 2 the second half of the
    // wave may fall past the last chunk, and then reads the first half's chunk and stores
    // nothing
    auto lane_pos = [&](int ln, int& ch, int& wl) {
        const int half = FPL == 2 ? (ln >> 5) : 0;
        ch = unit * FPL + half;
        wl = FPL == 2 ? 2 * (ln & 31) : ln;
    };
    int my_chunk, wl;
    lane_pos(lane, my_chunk, wl);
    const bool live = my_chunk < nchunks;
    if (!live) my_chunk = unit * FPL;
    const int w = my_chunk * 64 + wl;  // first frequency of this lane (S is even; it may end inside the last chunk)
    // this wave's run (waves past the last run only help to fill the tile)
    const int run = wave_uniform(gb * kNearWaves + (int)(threadIdx.x >> 6));
    const bool active = run < nruns;
    const int g0 = runs[active ? 2 * run : 0], len = active ? runs[2 * run + 1] : 0;
    // The kernel tile: every load of a thread is issued before the first is stored.
    V kv[NR];
    if (sym.info != nullptr) {
        // reduced spectra: each thread fills rows of its own frequencies (the loop steps by
        // whole waves), decoded once; the rows' descriptions first, then all the gathers
        Freq3 om[FPL];
#pragma unroll
        for (int q = 0; q < FPL; ++q) om[q] = freq_of(w + q, sym.M);
        uint32_t inf[NR];
        bool use[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const int i = (int)threadIdx.x + k * NT;
            use[k] = i < 27 * 64;
            inf[k] = use[k] ? sym.info[i >> 6] : 0u;
        }
#pragma unroll
        for (int k = 0; k < NR; ++k)
#pragma unroll
            for (int q = 0; q < FPL; ++q)
                kv[k].v[q] = use[k] && w + q < S ? sym_coef(khat, inf[k], om[q], sym.ncls, sym.M) : cplx<T>{T(0), T(0)};
    } else {
        const int wt = w < S ? w : 0;  // (S is even: a lane's two frequencies are both below it or not)
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const int row = (int)(threadIdx.x >> 6) + k * kNearWaves;
            kv[k] = *reinterpret_cast<const V*>(khat + spec_at(row < 27 ? row : 26, wt, 27));
        }
        if (w >= S) {
#pragma unroll
            for (int k = 0; k < NR; ++k) kv[k] = V{};
        }
    }
    // this lane's byte offset from an item's coefficients in the unit's first chunk: its chunk,
    // then its frequencies; dead lanes read as live ones do and store out of range (at ~15u, above
    // every range and with all 16 bytes below 2^32; dropped)
    const uint32_t lbytes = (uint32_t)(my_chunk - unit * FPL) * (uint32_t)(nsrc + 1) * kItemBytes<T> +
                            (uint32_t)wl * (uint32_t)sizeof(cplx<T>);
    const uint32_t sbytes = live ? (uint32_t)(my_chunk - unit * FPL) * (uint32_t)ntgt * kItemBytes<T> +
                                       (uint32_t)wl * (uint32_t)sizeof(cplx<T>)
                                 : ~15u;
    const char* const fbase = reinterpret_cast<const char*>(fhat + (int64_t)(unit * FPL) * (nsrc + 1) * 64);
    char* const ubase = reinterpret_cast<char*>(uhat + (int64_t)(unit * FPL) * ntgt * 64);
    // bytes from an item's first coefficient to the end of the lanes' last (0: reads as zeros,
    // stores nothing, without memory traffic)
    const uint32_t fspan = (FPL - 1) * (uint32_t)(nsrc + 1) * kItemBytes<T> + kItemBytes<T>;
    const uint32_t uspan = (FPL - 1) * (uint32_t)ntgt * kItemBytes<T> + kItemBytes<T>;
    auto load = [&](int item, bool on) -> V {
        return buffer_read<V>(fbase + (uint64_t)(uint32_t)item * kItemBytes<T>, on && item != nsrc ? fspan : 0u, lbytes);
    };
    // 4-wave workgroups whose runs all exist, equally long and long enough, step through the
    // source slabs together (a barrier before each half slab's loads): the waves' groups are
    // neighbours and share half their sources, which the lockstep serves from L1.  The
    // condition is uniform over the workgroup, so every wave meets the same barriers.
    bool lockstep = kNearWaves == 4 && len >= kLockstepRun && gb * kNearWaves + kNearWaves <= nruns;
    if (lockstep)
        for (int k = 0; k < kNearWaves; ++k) lockstep = lockstep && runs[2 * (gb * kNearWaves + k) + 1] == len;
    lockstep = wave_uniform(lockstep);
    // source slab s = 0 .. 2 len + 1 of the run: slabs 0 and 1 of the first group, then slabs
    // 2 and 3 of each group in turn (flags: bit 2 sz + h = half slab h of slab sz holds a
    // source, bit 8 + cz = target slab cz holds a target)
    ScalarList sg = nullptr;
    uint32_t have = 0;
    auto at = [&](int s) {
        const int g = s < 2 ? g0 : g0 + (s >> 1) - 1, sz = s < 2 ? s : 2 + (s & 1);
        sg = src64 + (int64_t)g * 64 + 16 * sz;
        have = (uint32_t)flags[g] >> (2 * sz);
    };
    auto target = [&](int t) {  // target slab t of the run exists and holds a target
        return t >= 0 && t < 2 * len && ((flags[g0 + (t >> 1)] >> (8 + (t & 1))) & 1);
    };
    // Every load and store from here on is issued whatever the layout (an absent item's with an
    // empty range), so the loads in flight are counted exactly: a wait for one half never waits
    // for the next one's loads or for the stores.
    V fa[8], fb[8];
    bool ha, hb;  // the buffered halves hold a source
    auto ld = [&](int h, bool on, V(&x)[8]) {
        if (lockstep) __builtin_amdgcn_s_barrier();
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = load(sg[8 * h + i], on);
        return (bool)((have >> h) & 1);
    };
    at(0);
    ha = ld(0, active, fa);
    hb = ld(1, active, fb);
#pragma unroll
    for (int k = 0; k < NR; ++k) {
        const int i = (int)threadIdx.x + k * NT;
        if (i < 27 * 64) tile[i] = kv[k];
    }
    __syncthreads();
    if (!active) return;
    // accumulators of the three target slabs a source slab reaches: [d] holds target slab
    // s - d, which meets source slab s (block plane s - 1 of the run) at dz = 1 - d;
    // targets c = cx | cy << 1
    T ar[3][FPL][4], ai[3][FPL][4];
    auto clear = [&](int d) {
#pragma unroll
        for (int q = 0; q < FPL; ++q)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                ar[d][q][c] = T(0);
                ai[d][q][c] = T(0);
            }
    };
    clear(0);
    clear(1);
    clear(2);
    // the half h of a source slab: source rows sy = 2h + j (j = 0, 1) in f[4 j + sx]; a target
    // row cy meets them through dy = cy - sy + 1, so half 0 uses dy = 1, 0 and half 1 dy = 0, -1.
    // (dy, dx) run from +1 down to -1, so every target adds its sources in increasing
    // (sz, sy, sx) order whatever the run.
    auto half = [&](auto hc, const V(&f)[8], const bool(&use)[3]) {
        constexpr int h = decltype(hc)::value;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            if (!use[d]) continue;  // wave-uniform: no such target slab, or none of its blocks
            const V* t = tile + 9 * (2 - d) * 64 + lane;
#pragma unroll
            for (int dy = 1 - h; dy >= -h; --dy) {
#pragma unroll
                for (int dx = 1; dx >= -1; --dx) {
                    const V k = t[((dx + 1) + 3 * (dy + 1)) * 64];
#pragma unroll
                    for (int cy = 0; cy < 2; ++cy) {
                        const int sy = cy - dy + 1;
                        if (sy < 2 * h || sy > 2 * h + 1) continue;
#pragma unroll
                        for (int cx = 0; cx < 2; ++cx) {
                            const int c = cx | (cy << 1);
                            const int sxy = (cx - dx + 1) + 4 * (sy - 2 * h);
#pragma unroll
                            for (int q = 0; q < FPL; ++q) cmac(ar[d][q][c], ai[d][q][c], f[sxy].v[q], k.v[q]);
                        }
                    }
                }
            }
        }
    };
    // target slab ar[2] / ai[2] to the items tg[0..3].  Streamed past the caches: the output is
    // read once, by the inverse transform, and must not evict the source spectra this kernel
    // re-reads (measured: this Prod 15% faster, the inverse 10% slower, the pair 7% faster at
    // 128^3 FP64)
    auto store = [&](bool on, ScalarList tg) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int t = tg[c];
            V o;
#pragma unroll
            for (int q = 0; q < FPL; ++q) o.v[q] = cplx<T>{ar[2][q][c], ai[2][q][c]};
            buffer_stream(ubase + (int64_t)(t < 0 ? 0 : t) * kItemBytes<T>, on && t >= 0 ? uspan : 0u, sbytes, o);
        }
    };
    store(false, tgt8);  // (as every pass through the loop does)
    issue_fence();
    using H0 = std::integral_constant<int, 0>;
    using H1 = std::integral_constant<int, 1>;
    const int nslab = 2 * len + 2;
    bool use[3] = {false, false, false};
#pragma unroll 1
    for (int s = 0; s < nslab; ++s) {
        use[2] = use[1];
        use[1] = use[0];
        use[0] = target(s);
        const bool more = s + 1 < nslab;
        const ScalarList tg = tgt8 + (int64_t)(g0 + ((s > 1 ? s - 2 : 0) >> 1)) * 8 + 4 * (s & 1);
        // half slabs through two buffers of 8 values: the next slab's first half is in flight
        // while this one's second half is consumed, and so on
        arrived(fa);
        if (ha) half(H0{}, fa, use);
        at(more ? s + 1 : s);
        ha = ld(0, more, fa);
        issue_fence();
        arrived(fb);
        if (hb) half(H1{}, fb, use);
        hb = ld(1, more, fb);
        issue_fence();
        store(use[2], tg);
#pragma unroll
        for (int q = 0; q < FPL; ++q)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                ar[2][q][c] = ar[1][q][c];
                ai[2][q][c] = ai[1][q][c];
                ar[1][q][c] = ar[0][q][c];
                ai[1][q][c] = ai[0][q][c];
            }
        clear(0);
    }
}

// ------------------------------------------------------------------ levels >= 1, sibling blocked
// Parents J (level l+1): src216[J][e * 8 + cs] = level-l interval 2(J + e') + cs with
// e' = (ex-1, ey-1, ez-1), e = ex + 3 ey + 9 ez, or the zero sentinel item (index nitems);
// child8[J][c] = target 2J + c (or -1); mask[J]: bit e set when neighbour e holds a source (never
// bit 13, the parent itself, all of whose pairs are near).  khat: 343 offsets, id
// (Dx+3) + 7 (Dy+3) + 49 (Dz+3).
//
// The target child c receives source child cs of neighbour e at offset D = c - cs - 2e'.
// Register blocking: a lane owns one frequency of one parent and accumulates CPL of its 8
// children (the subset Q of the children is fixed per wave, so all its index arithmetic is
// compile-time).  Per neighbour e the lane loads the 8 source coefficients once; its
// (child, source child) pairs need only the kernel values at delta = c - cs, each read once
// from LDS and applied to every pair with that delta.  The delta loop is unrolled and has
// no branch: the interaction-list condition |D|_inf >= 2 is met by zero kernel rows at the
// near offsets.  Every child sums its terms in the same order (its parent's neighbours by
// increasing e, then delta) whatever CPL, the number of waves and the order of the parents, so
// all variants give identical results; neighbours that hold no source would add exact zeros.
// Lanes: F consecutive frequencies (one 128-byte segment of a spectrum) x 64/F parents.
//
// Each parent steps through its own neighbours, not through all that a wave's parents have: on
// small levels, ragged layouts and batches the parents of a wave share few (a 2^3-parent level:
// 7 of 26 each, all 26 together), and the plan sorts the parents by their number of neighbours,
// so the lanes of a wave finish together.  The lanes' kernel rows then differ, so the tile holds
// all 343 rows (44 KB), and a neighbour step's rows are constant offsets from the lane's own
// base.  Bound by the vector units and, on small levels, by the longest parent's chain of steps.
// Against a wave stepping through every neighbour of its parents (and a half tile), us per step
// with its event: 256^3 FP64 350 -> 308, FP32 209 -> 175 (the n = 16, p = 8 cubes); 128^3 72 -> 50
// and 43 -> 33; 48 ragged layouts FP32 259 -> 134; separate-set ring FP64 287 -> 176; the n_I = 17
// scheme FP64 384 -> 272; 64 blocks of 8^3 FP64 18 -> 9.
template <typename T>
struct M2LShape {
    static constexpr int F = 128 / (int)sizeof(cplx<T>);  // frequencies per chunk: 8 FP64, 16 FP32
    static constexpr int PPW = 64 / F;                     // parents per wave
};

// child i of subset Q when a lane accumulates CPL children (subsets split z, then y, then x)
template <int CPL, int Q>
__device__ constexpr int m2l_child(int i) { return Q * CPL + i; }

// The contribution of one neighbour to this lane's children, with source values fa.  kb points
// at the tile row of delta (-1, -1, -1) for the lane's neighbour, so every delta's row is a
// constant offset away whatever the neighbour.  The deltas of one dz slab form one scheduling
// region, so the multiply-adds of several deltas interleave (deeper prefetches of the kernel
// values, 3 to 6 in flight, were 2-4% slower on large levels).
template <typename T, int CPL, int Q>
__device__ __forceinline__ void m2l_neighbour(const cplx<T>* kb, const cplx<T> (&fa)[8], T (&ar)[CPL], T (&ai)[CPL]) {
    constexpr int F = M2LShape<T>::F;
#pragma unroll
    for (int dz = -1; dz <= 1; ++dz) {
#pragma unroll
        for (int dd = 0; dd < 9; ++dd) {
            const int dx = dd % 3 - 1, dy = dd / 3 - 1;
            bool used = false;  // compile-time: does a child of this subset pair with delta d?
#pragma unroll
            for (int i = 0; i < CPL; ++i) {
                const int c = m2l_child<CPL, Q>(i);
                const int csx = (c & 1) - dx, csy = ((c >> 1) & 1) - dy, csz = (c >> 2) - dz;
                used |= csx >= 0 && csx <= 1 && csy >= 0 && csy <= 1 && csz >= 0 && csz <= 1;
            }
            if (!used) continue;
            const cplx<T> k = kb[((dx + 1) + 7 * (dy + 1) + 49 * (dz + 1)) * F];
#pragma unroll
            for (int i = 0; i < CPL; ++i) {
                const int c = m2l_child<CPL, Q>(i);
                const int csx = (c & 1) - dx, csy = ((c >> 1) & 1) - dy, csz = (c >> 2) - dz;
                if (csx < 0 || csx > 1 || csy < 0 || csy > 1 || csz < 0 || csz > 1) continue;  // compile-time
                cmac(ar[i], ai[i], fa[csx | (csy << 1) | (csz << 2)], k);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// This lane's neighbours, the set bits of mask in order; n: the most any lane of the wave has.
// Two source buffers, the next neighbour's sources in flight while one is consumed (a third
// buffer was 5-8% slower: registers).  A lane that has run out takes entry 13, whose list
// entries are the zero sentinel and whose kernel rows are zeros.
template <typename T, int CPL, int Q, typename IdxT>
__device__ __forceinline__ void m2l_lane(const cplx<T>* __restrict__ fb, int wl, const IdxT* si, const cplx<T>* tk,
                                         const int* rows, uint32_t mask, int n, T (&ar)[CPL], T (&ai)[CPL]) {
    cplx<T> fa[8], fbuf[8];
    const cplx<T>*ka, *kb;
    auto take = [&](cplx<T>(&f)[8], const cplx<T>*& k) {
        const int e = mask ? __builtin_ctz(mask) : 13;
        mask &= mask - 1;
#pragma unroll
        for (int cs = 0; cs < 8; ++cs) f[cs] = load_item(fb, (int)si[e * 8 + cs], wl);
        k = tk + rows[e];
    };
    take(fa, ka);
#pragma unroll 1
    for (int i = 0; i < n; i += 2) {
        take(fbuf, kb);
        issue_fence();
        m2l_neighbour<T, CPL, Q>(ka, fa, ar, ai);
        take(fa, ka);
        issue_fence();
        arrived(fbuf);
        if (i + 1 < n) m2l_neighbour<T, CPL, Q>(kb, fbuf, ar, ai);
    }
}

template <typename T, int CPL, int Q = 0, typename IdxT>
__device__ __forceinline__ void m2l_dispatch(int q, const cplx<T>* fb, int wl, const IdxT* si, const cplx<T>* tk,
                                             const int* rows, uint32_t mask, int n, T (&ar)[CPL], T (&ai)[CPL]) {
    if constexpr (Q + 1 < 8 / CPL) {
        if (q != Q) {
            m2l_dispatch<T, CPL, Q + 1, IdxT>(q, fb, wl, si, tk, rows, mask, n, ar, ai);
            return;
        }
    }
    m2l_lane<T, CPL, Q, IdxT>(fb, wl, si, tk, rows, mask, n, ar, ai);
}

// One launch may cover several levels (segments of the grid, each with its own spectra,
// lists, kernel spectra and spectrum size S): the coarse levels' small
// M2L then runs inside the level-1 launch instead of as latency-bound launches of their own.
// Segment k owns the workgroups [start_k, start_{k+1}); each start is a multiple of the
// XCD count, so every segment keeps the XCD-aware chunk mapping.
template <typename T>
struct FarSeg {
    const cplx<T>* fhat;
    const cplx<T>* khat;
    const int32_t* child8;
    const int32_t* src216;
    cplx<T>* uhat;
    const uint32_t* mask;
    int nparents, nitems, nsrc, ngroupblocks, start, S;
    bool heavy_first;
    SpecSym sym;  // reduced kernel spectra (sym.info == nullptr: one spectrum per offset)
};
template <typename T>
struct FarSegs {
    FarSeg<T> s[kMaxFarSegs];
    int n;
};

// table row r = (Dx+3) + 7 (Dy+3) + 49 (Dz+3) of a near offset (|D| <= 1 on every axis)
__device__ __forceinline__ bool m2l_near_row(int r) {
    const int dx = r % 7 - 3, dy = (r / 7) % 7 - 3, dz = r / 49 - 3;
    return dx >= -1 && dx <= 1 && dy >= -1 && dy <= 1 && dz >= -1 && dz <= 1;
}

// The kernel tile of one frequency chunk into LDS, zeros at the near offsets.  Only the 196
// rows with Dz >= 0 are read: the kernel spectra of opposite offsets are complex conjugates (the
// kernel is real and even, Sec. 2.1, and its padded tile is placed symmetrically about the
// origin: offset r at circulant index r mod M, zero at M/2; so the -D tile is the D tile
// reflected, and its DFT the conjugate).
template <typename T, int NT>
__device__ __forceinline__ void m2l_fill_tile(const FarSeg<T>& g, int w0, cplx<T>* tile) {
    constexpr int F = M2LShape<T>::F, kRows = 196, kRow0 = 147;  // first row read: D = (-3, -3, 0)
    const int S = g.S;
    auto put = [&](int i, const cplx<T>& v) {
        const int r = kRow0 + i / F, j = i % F;
        tile[r * F + j] = v;
        if (r >= kRow0 + 49) tile[(342 - r) * F + j] = cplx<T>{v.x, -v.y};
    };
    // reduced spectra: NT is a multiple of F, so every row a thread fills has the same
    // frequency, decoded once
    if (g.sym.info != nullptr) {
        // every row's description first, then all the (dependent) gathers, so the loads of
        // a thread's rows are in flight together
        constexpr int NR = (kRows * F + NT - 1) / NT;
        const int jj = (int)threadIdx.x % F;
        const bool wok = w0 + jj < S;
        const Freq3 om = wok ? freq_of(w0 + jj, g.sym.M) : Freq3{};
        uint32_t inf[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const int i = (int)threadIdx.x + k * NT;
            inf[k] = i < kRows * F ? g.sym.info[kRow0 + i / F] : 0u;
        }
        cplx<T> kv[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const int i = (int)threadIdx.x + k * NT;
            kv[k] = (i < kRows * F && wok && !m2l_near_row(kRow0 + i / F))
                        ? sym_coef(g.khat, inf[k], om, g.sym.ncls, g.sym.M)
                        : cplx<T>{T(0), T(0)};
        }
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const int i = (int)threadIdx.x + k * NT;
            if (i < kRows * F) put(i, kv[k]);
        }
    } else {
        // all of a thread's loads are issued before the first is stored (a loop of one load and
        // one store each waited for every load in turn)
        constexpr int NR = (kRows * F + NT - 1) / NT;
        cplx<T> kv[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const int i = (int)threadIdx.x + k * NT, r = kRow0 + (i < kRows * F ? i / F : 0), jj = i % F;
            kv[k] = g.khat[spec_at(r, w0 + jj < S ? w0 + jj : w0, 343)];
        }
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const int i = (int)threadIdx.x + k * NT;
            if (i < kRows * F) put(i, w0 + i % F < S && !m2l_near_row(kRow0 + i / F) ? kv[k] : cplx<T>{T(0), T(0)});
        }
    }
}

// The source lists of the workgroup's PPG parents into LDS.
template <typename IdxT, int PPG, int NT>
__device__ __forceinline__ void m2l_stage_lists(const int32_t* __restrict__ src216, int pb, int nparents, int nsrc,
                                                IdxT* sidx) {
    {
        // the parents' lists, four entries a load, in batches issued together
        constexpr int N4 = PPG * 54, NB = (N4 + NT - 1) / NT, B = NB < 7 ? NB : 7;
        const int have4 = (nparents - pb * PPG) * 54;  // padding parents read zeros
        const int4* src4 = reinterpret_cast<const int4*>(src216 + (int64_t)pb * PPG * 216);
#pragma unroll 1
        for (int k0 = 0; k0 < NB; k0 += B) {
            int4 v[B];
#pragma unroll
            for (int k = 0; k < B; ++k) {
                const int i = (int)threadIdx.x + (k0 + k) * NT;
                v[k] = src4[i < have4 ? i : 0];
            }
#pragma unroll
            for (int k = 0; k < B; ++k) {
                const int i = (int)threadIdx.x + (k0 + k) * NT;
                const int* e = reinterpret_cast<const int*>(&v[k]);
                if (i < N4)
#pragma unroll
                    for (int j = 0; j < 4; ++j) sidx[4 * i + j] = (IdxT)(i < have4 ? e[j] : nsrc);
            }
        }
    }
}

template <typename T, int kGroups, int CPL, typename IdxT>
__global__ void __launch_bounds__(64 * kGroups * (8 / CPL)) k_prod_far_sib(const FarSegs<T> segs) {
    constexpr int F = M2LShape<T>::F;
    constexpr int PPW = M2LShape<T>::PPW;
    constexpr int NQ = 8 / CPL;           // waves per group of parents (one per child subset)
    constexpr int PPG = PPW * kGroups;    // parents per workgroup
    constexpr int NT = 64 * kGroups * NQ;
    __shared__ cplx<T> tile[343 * F];
    __shared__ alignas(16) IdxT sidx[PPG * 216];  // 16-bit when every level's items fit (less LDS)
    __shared__ int rows[27];  // tile offset of delta (-1, -1, -1) for each neighbour
    // this workgroup's segment (uniform selects over the kernel arguments)
    FarSeg<T> g = segs.s[0];
#pragma unroll
    for (int k = 1; k < kMaxFarSegs; ++k)
        if (k < segs.n && (int)blockIdx.x >= segs.s[k].start) g = segs.s[k];
    const int nparents = g.nparents, nitems = g.nitems, nsrc = g.nsrc, S = g.S;
    const int L = (int)blockIdx.x - g.start, nchunks = (S + F - 1) / F;
    int chunk, pb;
    if (g.heavy_first) {
        // an XCD takes the first parents (those with the most neighbours) of all its chunks, then
        // the next ones: the short workgroups come last and fill the launch's tail
        const int per_xcd = (nchunks + kXcds - 1) / kXcds;
        chunk = (L / kXcds) % per_xcd * kXcds + L % kXcds;
        pb = (L / kXcds) / per_xcd;
        if (chunk >= nchunks) return;
    } else if (!xcd_tile_at(L, nchunks, g.ngroupblocks, chunk, pb)) {
        return;
    }
    const int w0 = chunk * F;
    const int lane = threadIdx.x & 63;
    const int wave = wave_uniform(threadIdx.x >> 6);
    const int q = wave % NQ, pw = wave / NQ;
    const int j = lane % F;
    const int Jl = pw * PPW + lane / F;
    const int J = pb * PPG + Jl;
    const uint32_t mask = J < nparents ? g.mask[J] : 0u;
    m2l_fill_tile<T, NT>(g, w0, tile);
    m2l_stage_lists<IdxT, PPG, NT>(g.src216, pb, nparents, nsrc, sidx);
    if (threadIdx.x < 27) {
        const int e = threadIdx.x;
        rows[e] = (228 - 2 * (e % 3 + 7 * (e / 3 % 3) + 49 * (e / 9))) * F;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < PPG * 8; i += NT) sidx[(i >> 3) * 216 + 13 * 8 + (i & 7)] = (IdxT)nsrc;
    __syncthreads();
    const int w = w0 + j;  // may exceed S in the last chunk: computed, never stored
    const cplx<T>* fb = g.fhat + (int64_t)(w0 >> 6) * (nsrc + 1) * 64;  // this chunk's items (uniform)
    T ar[CPL], ai[CPL];
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
        ar[i] = T(0);
        ai[i] = T(0);
    }
    // the wave's first parent has the most neighbours
    const int n = wave_uniform(__builtin_popcount(mask));
    m2l_dispatch<T, CPL, 0, IdxT>(q, fb, w & 63, sidx + Jl * 216, tile + j, rows, mask, n, ar, ai);
    if (J >= nparents || w >= S) return;
    const int32_t* c8 = g.child8 + (int64_t)J * 8 + q * CPL;
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
        const int t = c8[i];
        if (t >= 0) g.uhat[spec_at(t, w, nitems)] = cplx<T>{ar[i], ai[i]};
    }
}

// ------------------------------------------------------------------ generic CSR (top level)
constexpr int kProdThreads = 256;

// Targets tgt[i] (i = blockIdx.x) with list entries [ptr[i], ptr[i+1]).
template <typename T>
__global__ void __launch_bounds__(kProdThreads)
    k_prod_far(const cplx<T>* __restrict__ fhat, const cplx<T>* __restrict__ khat,
               const int32_t* __restrict__ ptr, const int32_t* __restrict__ src,
               const int32_t* __restrict__ off, const int32_t* __restrict__ tgt, cplx<T>* __restrict__ uhat, int S,
               int nitems, int noff, int nsrc, const SpecSym sym) {
    const int w = blockIdx.y * kProdThreads + threadIdx.x;
    const int64_t i = blockIdx.x;
    if (w >= S) return;
    const bool red = sym.info != nullptr;
    Freq3 om{};
    if (red) om = freq_of(w, sym.M);
    const int64_t P = tgt[i];
    const int e0 = ptr[i], e1 = ptr[i + 1];
    T ar = T(0), ai = T(0);
    for (int e = e0; e < e1; ++e) {
        const int q = src[e];
        const int o = off[e];
        const cplx<T> f = fhat[spec_at(q, w, nsrc + 1)];
        const cplx<T> k = red ? sym_coef(khat, sym.info[o], om, sym.ncls, sym.M) : khat[spec_at(o, w, noff)];
        cmac(ar, ai, f, k);
    }
    uhat[spec_at(P, w, nitems)] = cplx<T>{ar, ai};
}

// Frequencies per lane of the level-0 Prod: 2 in FP32, so that every lane moves 16 bytes
// per item as in FP64 (half the load and store instructions per byte).
template <typename T>
constexpr int kNearFpl = sizeof(T) == 4 ? 2 : 1;

// Grid and arguments of the level-0 Prod in workgroups of nw waves.
template <typename T>
static NearArgs<T> near_args(const NearLevel<T>& n, int nw, unsigned& grid) {
    const int nunits = ((n.S + 63) / 64 + kNearFpl<T> - 1) / kNearFpl<T>, nblocks = (int)((n.nruns + nw - 1) / nw);
    grid = xcd_grid(nunits, nblocks);
    return NearArgs<T>{n.fhat, n.khat, n.tgt8,       n.src64,     n.runs,      n.flags, n.uhat,
                       n.S,    (int)n.nruns, (int)n.nsrc, (int)n.ntgt, n.sym};
}

template <typename T, int NW>
static hipError_t near_nw(const NearLevel<T>& n, hipStream_t s) {
    unsigned grid;
    const NearArgs<T> a = near_args<T>(n, NW, grid);
    return lgf_launch(k_prod_near_grouped<T, NW, kNearFpl<T>>, dim3(grid), dim3(64 * NW), 0, s, a);
}

// a lane's 32-bit offsets span kNearFpl consecutive chunks of the source spectra, and reach one item
// in the last of as many chunks of the output
template <typename T>
static bool near_fits(const NearLevel<T>& n) {
    return n.S > 0 && n.S % 2 == 0 && chunk_fits_u32<T>((n.nsrc + 1) * kNearFpl<T>) &&
           near_fields_fit(n.ntgt, kNearFpl<T>, sizeof(cplx<T>)) && sym_fits(n.sym, n.S);
}

template <typename T>
hipError_t launch_prod_near(const NearLevel<T>& n, int waves, hipStream_t s) {
    if (n.nruns <= 0) return hipSuccess;
    if (!near_fits(n)) return hipErrorInvalidValue;
    switch (waves) {
        case 2: return near_nw<T, 2>(n, s);
        case 8: return near_nw<T, 8>(n, s);
        default: return near_nw<T, 4>(n, s);
    }
}

// LGF_M2L_WIDE_LISTS=1 in the environment keeps the 32-bit list entries at every level
// size, the form levels of 65535 or more items take (read at each launch; the same bits
// either way).
static bool m2l_wide_lists() {
    const char* v = std::getenv("LGF_M2L_WIDE_LISTS");
    return v && v[0] == '1';
}

// Segments of one launch for workgroups of PPG parents; returns the grid.
template <typename T>
static unsigned far_segments(const FarLevel<T>* lv, int nlev, int PPG, FarSegs<T>& segs) {
    constexpr int F = M2LShape<T>::F;
    unsigned grid = 0;
    for (int k = 0; k < nlev; ++k) {
        const int ngb = (int)((lv[k].nparents + PPG - 1) / PPG);
        const int nchunks = (lv[k].S + F - 1) / F;
        segs.s[k] = FarSeg<T>{lv[k].fhat,      lv[k].khat,         lv[k].child8,       lv[k].src216,
                              lv[k].uhat,      lv[k].mask,          (int)lv[k].nparents, (int)lv[k].nitems, (int)lv[k].nsrc,
                              ngb,             (int)grid,           lv[k].S,
                              lv[k].heavy_first,
                              lv[k].sym};
        grid += xcd_grid(nchunks, ngb);  // a multiple of the XCD count
    }
    segs.n = nlev;
    return grid;
}

// 16-bit list entries in LDS when every level's items (and the sentinel) fit: less LDS per
// workgroup, so more workgroups share a CU
template <typename T>
static bool far_idx16(const FarLevel<T>* lv, int nlev) {
    bool idx16 = !m2l_wide_lists();
    for (int k = 0; k < nlev; ++k) idx16 = idx16 && lv[k].nsrc < 65535;
    return idx16;
}

template <typename T, int NW, int CPL>
static hipError_t far_nw(const FarLevel<T>* lv, int nlev, hipStream_t s) {
    FarSegs<T> segs{};
    const unsigned grid = far_segments<T>(lv, nlev, M2LShape<T>::PPW * NW, segs);
    if (far_idx16<T>(lv, nlev))
        return lgf_launch(k_prod_far_sib<T, NW, CPL, uint16_t>, dim3(grid), dim3(64 * NW * (8 / CPL)), 0, s, segs);
    return lgf_launch(k_prod_far_sib<T, NW, CPL, int32_t>, dim3(grid), dim3(64 * NW * (8 / CPL)), 0, s, segs);
}

template <typename T, int CPL>
static hipError_t far_cpl(const FarLevel<T>* lv, int nlev, int waves, hipStream_t s) {
    // at most 16 waves (1024 threads) per workgroup, and at most 8 in FP64, whose pipeline
    // needs more registers.  Larger groups share one kernel tile among more parents (more waves
    // per CU for the same LDS).
    constexpr int kMaxWaves = sizeof(T) == 8 ? 8 : 16;
    constexpr int kMaxGroups = kMaxWaves / (8 / CPL);
    const int g = waves < kMaxGroups ? waves : kMaxGroups;
    if constexpr (kMaxGroups >= 16)
        if (g >= 16) return far_nw<T, 16, CPL>(lv, nlev, s);
    if constexpr (kMaxGroups >= 8)
        if (g >= 8) return far_nw<T, 8, CPL>(lv, nlev, s);
    if constexpr (kMaxGroups >= 4)
        if (g >= 4) return far_nw<T, 4, CPL>(lv, nlev, s);
    if constexpr (kMaxGroups >= 2)
        if (g >= 2) return far_nw<T, 2, CPL>(lv, nlev, s);
    return far_nw<T, 1, CPL>(lv, nlev, s);
}

// Number of levels with parents (empty levels only at the end), or -1 where a level does not
// fit what the kernels assume; most: the one with the most parents.
template <typename T>
static int far_check(const FarLevel<T>* lv, int nlev, const FarLevel<T>*& most) {
    int k = 0;
    most = lv;
    for (int i = 0; i < nlev; ++i) {
        if (lv[i].nparents <= 0) continue;
        if (k != i || !lv[i].mask || !chunk_fits_u32<T>(lv[i].nsrc + 1) || !sym_fits(lv[i].sym, lv[i].S)) return -1;
        if (lv[i].nparents > most->nparents) most = lv + i;
        ++k;
    }
    return k > kMaxFarSegs ? -1 : k;
}

template <typename T>
hipError_t launch_prod_far_sib_levels(const FarLevel<T>* lv, int nlev, int waves, int cpl, hipStream_t s) {
    const FarLevel<T>* most = nullptr;
    const int k = far_check<T>(lv, nlev, most);
    if (k < 0) return hipErrorInvalidValue;
    if (k == 0) return hipSuccess;
    const M2LVariant open = m2l_default(most->nparents, most->S, M2LShape<T>::F, most->n);
    if (cpl == 0) cpl = open.children;
    if (waves == 0) waves = open.parents / M2LShape<T>::PPW;
    switch (cpl) {
        case 8: return far_cpl<T, 8>(lv, k, waves, s);
        case 4: return far_cpl<T, 4>(lv, k, waves, s);
        case 2: return far_cpl<T, 2>(lv, k, waves, s);
        default: return far_cpl<T, 1>(lv, k, waves, s);
    }
}

template <typename T>
hipError_t launch_prod_far(const cplx<T>* fhat, const cplx<T>* khat, const int32_t* ptr, const int32_t* src,
                           const int32_t* off, const int32_t* tgt, cplx<T>* uhat, int64_t ntgt, int64_t nitems,
                           int noff, int S, hipStream_t s, int64_t nsrc, const SpecSym& sym) {
    if (ntgt <= 0) return hipSuccess;
    if (nsrc < 0) nsrc = nitems;
    if (!sym_fits(sym, S)) return hipErrorInvalidValue;
    dim3 grid((unsigned)ntgt, (unsigned)((S + kProdThreads - 1) / kProdThreads));
    return lgf_launch(k_prod_far<T>, grid, dim3(kProdThreads), 0, s, fhat, khat, ptr, src, off, tgt, uhat, S,
                      (int)nitems, noff, (int)nsrc, sym);
}

#define LGF_INST(T)                                                                                              \
    template hipError_t launch_prod_near<T>(const NearLevel<T>&, int, hipStream_t);                         \
    template hipError_t launch_prod_far_sib_levels<T>(const FarLevel<T>*, int, int, int, hipStream_t);           \
    template hipError_t launch_prod_far<T>(const cplx<T>*, const cplx<T>*, const int32_t*, const int32_t*,       \
                                           const int32_t*, const int32_t*, cplx<T>*, int64_t, int64_t, int, int, \
                                           hipStream_t, int64_t, const SpecSym&);
LGF_INST(double)
LGF_INST(float)
#undef LGF_INST

}  // namespace lgfdev

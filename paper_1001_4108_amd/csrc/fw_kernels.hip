// Blocked Floyd-Warshall kernels for CDNA4 (gfx950).
//
// The schedule is the blocked algorithm of section 3.2 (Fig. BFW-Alg): the
// matrix is cut into s x s tiles and, for each k-block b, three dependent
// phases run as three kernel launches (a kernel boundary is the global
// barrier between phases):
//
//   1. diag_kernel   -- the "independent block" (b, b): s dependent k-steps
//                       on one tile.
//   2. panels        -- the "singly dependent" row panel (b, j != b) and
//                       column panel (i != b, b).
//   3. bulk          -- the "doubly dependent" tiles (i != b, j != b), the
//                       phase that sets the speed of the whole algorithm.
//
// The panels and the bulk run tile64_kernel at tile 64 (modes of one kernel),
// panel_strip_kernel and bulk_dma_kernel at tile 128, and tile_kernel at tile
// 32 and with predecessors.  Both phases are the same tile update
//     C(i,j) <- min(C(i,j), min_{k in block b} A(i,k) + B(k,j))
// with A = tile (bi, b) and B = tile (b, bj) read at the moment the phase
// starts.  For the bulk this is the paper's order-free doubly dependent
// update (section 3.2: no dependencies inside the tile).  For a panel tile
// one operand is the finished diagonal tile D and the other is the panel tile
// itself, and the update is D (x) P in the min-plus sense: after phase 1, D
// holds the shortest paths inside block b, so every path from row-block b to
// column j that last leaves block b at vertex k splits into a D part and an
// unchanged P part.  In exact arithmetic this gives the same result as the
// figure's k-ordered panel loop while removing its k-to-k dependency, so the
// panel phase runs at the same register-tiled rate as the bulk.
//
// The workgroup-level bodies (closure_tile, product_tile) live in
// fw_tiles.h.  MFMA is not used: min-plus is not a multiply-add contraction.
#include <type_traits>

#include "fw_tiles.h"

// Build-time switches (variant builds override them with -D): keyed int32
// predecessor tiles, waves per SIMD of the bulk kernel.
#ifndef FW_PRED_KEYS
#define FW_PRED_KEYS 1
#endif
#ifndef FW_BULK_DMA_WAVES
#define FW_BULK_DMA_WAVES 4
#endif

namespace fw {
namespace {

// 64-wide launches of at most this many tiles take two halves of k per tile
// (512 threads): the launch lasts as long as its last round of workgroups, and a
// tile in halves ends sooner; with more tiles the joining of the halves costs
// more than that saves.  Solves in one launch a stage of k^2 tiles, one half a
// tile against two, n = 64 (k + 1) with aligned rows, then 37 vertices fewer with
// unaligned ones: k=23 fp32 564 / 440 and 635 / 607 us, int32 601 / 488 and 676 /
// 662; k=26 638 / 504 and 720 / 704, 680 / 563 and 765 / 763; k=27 670 / 592 and
// 753 / 756, 712 / 667 and 800 / 834; k=29 725 / 666 and 810 / 894, 768 / 747 and
// 859 / 977.  The line is where the unaligned ones cross.
constexpr int64_t kTile64SplitMax = 700;

// A gated launch (gate != NULL) does nothing unless *gate != 0: the 64-bit
// predecessor sweep queued behind a keyed one runs only when the keyed one
// gave up.  The gate is uniform, so the whole workgroup leaves at once.
__device__ __forceinline__ bool gated_off(const int32_t *gate) { return gate && *gate == 0; }

// A keyed launch whose solve has already given up (its flag set by an earlier
// launch or the packing) has nothing useful to do: the 64-bit sweep behind it
// starts over from the input.  A flag raised during the launch is only seen
// by later launches.
template <class A>
__device__ __forceinline__ bool given_up(const int32_t *flag) {
    if constexpr (A::kChecked)
        return *flag != 0;
    else
        return false;
}

// Phase 1: closure of the diagonal tile (b, b) -- one workgroup.
template <typename T, int S, bool PRED, class A>
__global__ void __launch_bounds__((closure_threads<T, S, PRED, A, true>()))
diag_kernel(T *__restrict__ d, int32_t *__restrict__ P, int n, int64_t ld, int64_t ldp,
            int b, int32_t *flag, const int32_t *gate) {
    __shared__ __align__(16) char smem[closure_smem_bytes<T, S, PRED, true>()];
    if (gated_off(gate) || given_up<A>(flag)) return;
    closure_tile_any<T, S, closure_tm<T, S, PRED, A, true>(), PRED, A,
                     closure_tn<T, S, PRED, A, true>(), true>(d, P, n, ld, ldp, b * S, smem, flag);
}

// Phases 2 and 3: one tile per workgroup.
//   mode 0: blockIdx.x enumerates the 2(nb-1) panel tiles of stage b;
//   mode 1: blockIdx.x enumerates the (nb-1)^2 bulk tiles.
// int32 with predecessors takes the keyed form (product_tile_key).
template <typename T, int S, int BK, bool PRED, class A>
constexpr bool keyed_tile() {
    return PRED && std::is_same<T, int32_t>::value && std::is_same<A, Ar<int32_t>>::value &&
           FW_PRED_KEYS;
}

// Forms whose geometry is the closure's (4 x 4 cells per thread: tile 64 over
// 256 threads, the 128-wide predecessor form over 1024) can also close the
// next stage's diagonal tile in mode 1, as bulk_dma_kernel does.  (Tile 32
// over 64 threads has it too, but one wave's 32-wide closure is slower than
// the separate four-wave diagonal launch.)
template <int S, int TM, int TN, bool PRED>
constexpr bool tile_can_close() {
    return TM == 4 && TN == 4 && (S == 64 || (PRED && S == 128));
}

template <typename T, int S, int BK, int TM, int TN, bool PRED, class A>
constexpr int tile_smem_bytes() {
    const int product = keyed_tile<T, S, BK, PRED, A>() ? product_key_smem_bytes<S, BK>()
                                                        : product_smem_bytes<T, S, BK, PRED>();
    const int closure = tile_can_close<S, TM, TN, PRED>() ? closure_smem_bytes<T, S, PRED>() : 0;
    return product > closure ? product : closure;
}

template <typename T, int S, int BK, int TM, int TN, bool VEC, bool PRED, class A>
__global__ void __launch_bounds__((S / TM) * (S / TN))
tile_kernel(T *__restrict__ d, int32_t *__restrict__ P, int n, int64_t ld, int64_t ldp, int b,
            int nb, int mode, int close_next, int32_t *flag, const int32_t *gate) {
    __shared__ __align__(16) char smem[tile_smem_bytes<T, S, BK, TM, TN, PRED, A>()];
    if (gated_off(gate) || given_up<A>(flag)) return;
    int idx = blockIdx.x, bi, bj;
    bool close = false;
    if constexpr (tile_can_close<S, TM, TN, PRED>()) {
        // the workgroup of tile (b+1, b+1) takes blockIdx 0 (see bulk_dma_kernel)
        const int dix = b * (nb - 1) + b;
        if (close_next && mode == 1) {
            idx = idx == 0 ? dix : idx == dix ? 0 : idx;
            close = idx == dix;
        }
    }
    if (mode == 0)
        panel_coords(idx, b, nb - 1, bi, bj);
    else
        bulk_coords(idx, b, nb - 1, bi, bj);
    if constexpr (keyed_tile<T, S, BK, PRED, A>())
        product_tile_key<S, BK, TM, TN, VEC>(d, P, n, ld, ldp, bi, bj, b, smem);
    else
        product_tile<T, S, BK, TM, TN, VEC, PRED, A>(d, P, n, ld, ldp, bi, bj, b, smem, flag);
    if constexpr (tile_can_close<S, TM, TN, PRED>()) {
        if (close) {
            __syncthreads();  // the tile's stores before its reloads
            closure_tile_any<T, S, TM, PRED, A>(d, P, n, ld, ldp, (b + 1) * S, smem, flag);
        }
    }
}


// Phases 2 and 3 at tile 64 without predecessors (product_tile_whole); mode
// and CLOSE as tile_kernel's mode and close_next.
// The closing form has the threads of the latency closure (closure_tm):
// 512, and the wave that closes ahead.
template <typename T, class A>
constexpr int tile64_threads(int halves, bool close) {
    const int closure = closure_threads<T, 64, false, A, true>();
    return halves == 2 && close && closure > 512 ? closure : halves * 256;
}
template <typename T, int HALVES, bool CLOSE, bool VEC, class A>
__global__ void __launch_bounds__((tile64_threads<T, A>(HALVES, CLOSE)))
__attribute__((amdgpu_waves_per_eu(HALVES == 2 ? 3 : 1, 5)))
tile64_kernel(T *__restrict__ d, int n, int64_t ld, int b, int nb, int mode, int32_t *flag,
              const int32_t *gate) {
    constexpr int S = 64;
    static_assert(product_whole_smem_bytes<T>() >= closure_smem_bytes<T, S, false, true>(),
                  "the closure runs in the product's LDS");
    __shared__ __align__(16) char smem[product_whole_smem_bytes<T>()];
    if (gated_off(gate) || given_up<A>(flag)) return;
    int idx = blockIdx.x, bi, bj;
    const int dix = b * (nb - 1) + b;  // tile (b+1, b+1), moved to blockIdx 0
    if (CLOSE) idx = idx == 0 ? dix : idx == dix ? 0 : idx;
    if (mode == 0)
        panel_coords(idx, b, nb - 1, bi, bj);
    else
        bulk_coords(idx, b, nb - 1, bi, bj);
    product_tile_whole<T, HALVES, VEC, A>(d, n, ld, bi, bj, b, smem, flag);
    if constexpr (CLOSE) {
        if (idx != dix) return;
        constexpr bool kAhead = HALVES == 2 && closure_in_blocks<T, S, false, A>();
        constexpr int TM = closure_tm<T, S, false, A, kAhead>();
        constexpr int TN = closure_tn<T, S, false, A, kAhead>();
        __syncthreads();  // the tile's stores before its reloads
        if (kAhead || threadIdx.x < 256)
            closure_tile_any<T, S, TM, false, A, TN, kAhead>(d, nullptr, n, ld, 0, (b + 1) * S,
                                                             smem, flag);
    }
}

template <typename T, int HALVES, class A>
hipError_t tile64_launch(T *d, int n, int64_t ld, bool vec, int b, int nb, int mode, bool close,
                         unsigned grid, hipStream_t st, int32_t *flag, const int32_t *gate) {
    const int nt = tile64_threads<T, A>(HALVES, close);
    if (close) {
        if (vec)
            tile64_kernel<T, HALVES, true, true, A><<<grid, nt, 0, st>>>(d, n, ld, b, nb, mode,
                                                                        flag, gate);
        else
            tile64_kernel<T, HALVES, true, false, A><<<grid, nt, 0, st>>>(d, n, ld, b, nb, mode,
                                                                         flag, gate);
    } else {
        if (vec)
            tile64_kernel<T, HALVES, false, true, A><<<grid, nt, 0, st>>>(d, n, ld, b, nb, mode,
                                                                         flag, gate);
        else
            tile64_kernel<T, HALVES, false, false, A><<<grid, nt, 0, st>>>(d, n, ld, b, nb, mode,
                                                                          flag, gate);
    }
    return hipGetLastError();
}

// Phase 3 for 128-wide tiles without predecessors: every bulk tile of the
// stage (blockIdx.x enumerates (nb-1)^2), slices copied into LDS directly
// (bulk_tile_dma): 16 bytes a lane where the rows are 16-byte aligned (VEC), 4
// otherwise and for the tiles of a partial last block; four waves per SIMD.
// Measured, fp32 n=6001 (unaligned, 46 full blocks and a partial one): 170 us
// a stage, 8.0 ms a solve; with the bulk staged through registers and a
// diagonal launch per stage 235 us, 11.1 ms.  n=8100 (aligned rows, a partial
// last block): 15.9 ms; with a launch of its own for the edge tiles 18.1.
//
// With close_next the workgroup of tile (b+1, b+1) -- the next stage's
// diagonal tile, whose stage-b value it alone computes -- also runs that
// tile's closure, which replaces the next stage's phase-1 launch.  It takes
// blockIdx 0 (swapped with the tile enumerated first) so that it is
// dispatched early and its longer run overlaps the rest of the bulk.
template <typename T, bool VEC, class A>
__global__ void __launch_bounds__(256, FW_BULK_DMA_WAVES)
bulk_dma_kernel(T *__restrict__ d, int n, int64_t ld, int b, int m, int close_next,
                int32_t *flag, const T *acol) {
    constexpr int S = 128, BK = 16;
    __shared__ __align__(16) T A0[S * BK];
    __shared__ __align__(16) T A1[S * BK];
    __shared__ __align__(16) T B0[BK * S];
    __shared__ __align__(16) T B1[BK * S];
    __shared__ __align__(16) T X[kCloseExtra];
    const BulkLds<T> lds = {A0, A1, B0, B1};
    if (given_up<A>(flag)) return;
    const int last = n / S;  // blocks below it are full
    // a partial last block's tiles take longer: from the last row upwards, so
    // that they are not the launch's tail
    const int dix = b * m + b, end = m * m - 1;  // dix: index of tile (b+1, b+1)
    const bool reverse = last <= m;
    int idx = blockIdx.x;
    if (close_next) {
        const int at = reverse ? end - dix : dix;  // where its turn would be
        idx = idx == 0 ? at : idx == at ? 0 : idx;
    }
    if (reverse) idx = end - idx;
    int bi, bj;
    bulk_coords(idx, b, m, bi, bj);
    const bool close = close_next && idx == dix;
    if (bi < last && bj < last && b < last && ld < (int64_t(1) << 25))
        bulk_tile_dma<T, VEC, false, A>(lds, d, n, ld, bi, bj, b, flag, acol);
    else
        bulk_tile_dma<T, VEC, true, A>(lds, d, n, ld, bi, bj, b, flag, acol);
    if (!close) return;
    // the next stage's diagonal tile: reread by the same workgroup (the
    // barrier orders its stores before the loads) and closed in place; the
    // product's LDS buffers are free by now
    __syncthreads();
    if constexpr (closure_in_blocks<T, S, false, A>())
        closure_blocks<T, S, 8, 8, A, false>(d, n, ld, bi * S,
                                             ClosureLds<T>{B0, B1, A0, A1, X, nullptr});
    else if constexpr (VEC)  // bulk_closes: a tile inside the matrix
        closure_tile<T, S, 8, false, A, true>(d, nullptr, n, ld, 0, bi * S,
                                              reinterpret_cast<char *>(A0), flag);
}

// Phase 2 for 128-wide tiles without predecessors: each panel tile as four
// strips (strip_tile), blockIdx.x = 4 * (panel tile number) + strip.  Row
// panel tiles (b, j) are cut into 32-column strips, column panel tiles
// (i, b) into 32-row strips.
template <typename T, bool VEC, class A>
__global__ void __launch_bounds__(kStripThreads)
panel_strip_kernel(T *__restrict__ d, int n, int64_t ld, int b, int nb, int32_t *flag,
                   T *acol) {
    constexpr int S = 128, W = kStripW;
    __shared__ __align__(16) char smem[strip_smem_bytes<T>()];
    if (given_up<A>(flag)) return;
    const int m = nb - 1;
    const int t = blockIdx.x >> 2, q = blockIdx.x & 3;
    int bi, bj;
    panel_coords(t, b, m, bi, bj);
    if (t < m)  // row panel: rows of block b, a 32-column strip of block bj
        strip_tile<T, S, W, VEC, A>(d, n, ld, b * S, bj * S + q * W, b * S, smem, flag);
    else        // column panel: a 32-row strip of block bi, columns of block b
        strip_tile<T, W, S, VEC, A>(d, n, ld, bi * S + q * W, b * S, b * S, smem, flag, acol);
}

// ---------------------------------------------------------------------------
// Predecessor initialisation and final fix-up, negative-cycle scan.
// ---------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(256)
pred_init_kernel(const T *__restrict__ d, int32_t *__restrict__ P, int n, int64_t ld,
                 int64_t ldp, const int32_t *gate) {
    if (gated_off(gate)) return;
    for (int i = blockIdx.y; i < n; i += gridDim.y)
        for (int j = blockIdx.x * 256 + threadIdx.x; j < n; j += gridDim.x * 256) {
            const T w = d[(int64_t)i * ld + j];
            P[(int64_t)i * ldp + j] = (i != j && !Ar<T>::absent(w)) ? i : kPredNone;
        }
}

// gated 64-bit sweeps that ran (one count per solve, from its fix-up)
__device__ unsigned long long g_pred_fallbacks;

template <typename T>
__global__ void __launch_bounds__(256)
pred_fix_kernel(const T *__restrict__ d, int32_t *__restrict__ P, int n, int64_t ld,
                int64_t ldp, const int32_t *gate) {
    if (gated_off(gate)) return;
    if (gate && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0)
        atomicAdd(&g_pred_fallbacks, 1ull);
    for (int i = blockIdx.y; i < n; i += gridDim.y)
        for (int j = blockIdx.x * 256 + threadIdx.x; j < n; j += gridDim.x * 256) {
            int32_t &p = P[(int64_t)i * ldp + j];
            p = final_pred<T>(i, j, d[(int64_t)i * ld + j], p);
        }
}

// ---------------------------------------------------------------------------
// The fp32 canonical path (fw_internal.h): the canonical last hops from the
// final distances and the original weights, as the oracle defines them.
// ---------------------------------------------------------------------------
// flag[4] is the canonical path's own word from here on (the row minima of a
// keyed sweep end with its key_finish, which comes before): see
// canon_strip_kernel.
__global__ void canon_gate_kernel(int32_t *__restrict__ flag, int direct) {
    if (threadIdx.x == 0) {
        flag[3] = ((direct || flag[0] != 0) && flag[2] == 0) ? 1 : 0;
        flag[4] = 0;
    }
}

// A gated save (behind a keyed sweep) counts one fallback.
__global__ void __launch_bounds__(256)
canon_save_kernel(const float *__restrict__ d, int32_t *__restrict__ P, int n, int64_t ld,
                  int64_t ldp, const int32_t *gate) {
    if (gated_off(gate)) return;
    if (gate && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0)
        atomicAdd(&g_pred_fallbacks, 1ull);
    for (int i = blockIdx.y; i < n; i += gridDim.y)
        for (int j = blockIdx.x * 256 + threadIdx.x; j < n; j += gridDim.x * 256)
            P[(int64_t)i * ldp + j] = __float_as_int(d[(int64_t)i * ld + j]);
}

__global__ void __launch_bounds__(256)
canon_restore_kernel(float *__restrict__ d, const int32_t *__restrict__ P, int n, int64_t ld,
                     int64_t ldp, const int32_t *gate) {
    if (gated_off(gate)) return;
    for (int i = blockIdx.y; i < n; i += gridDim.y)
        for (int j = blockIdx.x * 256 + threadIdx.x; j < n; j += gridDim.x * 256)
            d[(int64_t)i * ld + j] = __int_as_float(P[(int64_t)i * ldp + j]);
}

// The strip of weights, transposed: strip[c][q] = w[q][j0 + c], q padded to
// whole slices, so that the last hops' kernel reads both of its operands
// along q.  +INF at (j, j) (q = j is no last hop of j) and in the padding,
// whose sums match no finite distance.  *frac becomes the largest number of
// bits any weight has behind the binary point.
constexpr int kCanonTile = 64, kCanonDepth = 32, kCanonGroup = 8, kCanonThreads = 256;
constexpr int32_t kCanonAgain = -3;  // no last hop: the tile is left to the equality launch
static_assert(kCanonDepth == kCanonSlice, "the strip's rows are padded to whole slices");

__device__ __forceinline__ int fraction_bits(float v) {
    const uint32_t u = __float_as_uint(v), e = u >> 23 & 255;
    if ((u << 1) == 0 || (u << 1) == 0xff000000u) return 0;  // 0, infinite
    const uint32_t m = e ? (u & 0x7fffff) | 0x800000 : u & 0x7fffff;
    return max(0, 150 - (int)max(e, 1u) - (__ffs((int)m) - 1));
}

__global__ void __launch_bounds__(256)
canon_strip_kernel(const int32_t *__restrict__ P, int n, int64_t ldp, int j0, int w,
                   float *__restrict__ strip, int32_t *__restrict__ frac, const int32_t *gate) {
    if (gated_off(gate)) return;
    __shared__ float t[64][65];
    const int ldt = canon_ldt(n), tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const int c0 = blockIdx.x * 64;
    int bits = 0;
    for (int q0 = blockIdx.y * 64; q0 < ldt; q0 += gridDim.y * 64) {
        __syncthreads();  // the previous block's reads are done
        for (int q = ty; q < 64; q += 4) {
            float v = __builtin_inff();
            if (q0 + q < n && c0 + tx < w) v = __int_as_float(P[(int64_t)(q0 + q) * ldp + j0 + c0 + tx]);
            bits = max(bits, fraction_bits(v));
            t[q][tx] = q0 + q == j0 + c0 + tx ? __builtin_inff() : v;
        }
        __syncthreads();
        for (int c = ty; c < 64; c += 4)
            if (q0 + tx < ldt) strip[(int64_t)(c0 + c) * ldt + q0 + tx] = t[tx][c];
    }
    for (int o = 32; o; o >>= 1) bits = max(bits, __shfl_xor(bits, o));
    if (tx == 0 && bits > *frac) atomicMax(frac, bits);
}

// One 64 x 64 tile of P (rows i0.., strip columns c0..; global column j0 +
// c) per workgroup, 4 x 4 cells per thread.  A cell wants the smallest q
// whose sum equals its distance.  The scan only finds the group of 8
// candidates that q lies in: groups go downward, and a cell keeps the last
// one that hit.  The cell's one group is then searched for q itself, from
// memory.  Two forms of the hit:
// - kMin: the smallest sum of the group is at most the distance: one add and
//   half a minimum3 per candidate.  Where sums are exact none is below the
//   distance, and the hit holds a match.  Where they round, one may be below
//   it by an ulp and hide that the group has no match; the search then finds
//   none, and the tile is left to the other form.
// - equality: some sum of the group equals the distance (an add and a
//   compare per candidate; the lane masks are joined on the scalar unit).
// What bounds it: instruction issue.  One candidate at a time with its own
// compare and select (three instructions, two at the minimum's half rate, in
// strips of 1024 columns: 3 tiles a compute unit at n=3000) took 2.93 ms at
// n=3000 and 40.5 ms at n=8192; kMin takes 1.33 and 21.4 ms, equality 2.0 and
// 36 (its compare still issues once per candidate).  Groups of 16 compare less
// but search more scattered memory: 5 ms more at n=8192.  8 x 4 cells a thread
// (180 registers, 2 waves a SIMD): 15 ms more.
// Two launches, so that each form has its own registers: the first scans the
// tiles it may by kMin (102 registers, 48 bytes of scratch a lane) and marks the
// others in P, the second scans those by equality at six waves a SIMD (80
// registers, 7 spilled: 64 bytes of scratch; both forms in one kernel of four:
// reals 63.5 ms the solve at n=8192 against 58.1, at n=16400 486 against 445).  A
// tile begins with kMin when its distances lie below 2^(24 - *frac) in magnitude
// (*frac from canon_strip_kernel): sums of the weights are then exact where they
// could reach the distance.  Either form is right for any
// weights; beginning with kMin and going on to equality would cost both.
// A cell whose pair has no last hop (i == j, or d_ij = +INF) compares against
// NaN, which is neither equal to nor above anything.  The slice of d is
// staged with 0 at (i, i) (a path from i starts with the empty path).  Rows
// and columns beyond the matrix hold whatever the clamped row or the strip's
// padding does: their cells compare against NaN.  No order of the sums
// matters: each is one fp32 add, compared exactly.  fminf leaves out a NaN
// sum (of infinite weights), which equals nothing.
__device__ __forceinline__ uint64_t lanes_eq(float a, float b) {
    return __builtin_amdgcn_fcmpf(a, b, 1);  // ordered, equal
}

template <bool kMin>
__device__ __forceinline__ void canon_scan(const float *__restrict__ d, int n, int64_t ld,
                                           const float *__restrict__ strip, int i0, int c0,
                                           float (*As)[kCanonDepth + 4],
                                           float (*Bs)[kCanonDepth + 4], const float (&t)[4][4],
                                           int32_t (&grp)[4][4]) {
    constexpr int S = kCanonTile, KD = kCanonDepth, NT = kCanonThreads, NY = 16;
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    const int ldt = canon_ldt(n);
    using V4u = typename Vec4u<float>::type;
    constexpr int NL = S * KD / 4 / NT;  // 4-wide pieces of a slice per thread
    for (int q0 = ldt - KD; q0 >= 0; q0 -= KD) {
        float4 a[NL], b[NL];
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const int e = tid + l * NT, r = e / (KD / 4), q = q0 + e % (KD / 4) * 4;
            const int gi = min(i0 + r, n - 1);
            const float *src = d + (int64_t)gi * ld + q;
            if (q0 + KD <= n) {
                const V4u x = *reinterpret_cast<const V4u *>(src);
                a[l] = make_float4(x[0], x[1], x[2], x[3]);
            } else {
                a[l].x = q < n ? src[0] : __builtin_inff();
                a[l].y = q + 1 < n ? src[1] : __builtin_inff();
                a[l].z = q + 2 < n ? src[2] : __builtin_inff();
                a[l].w = q + 3 < n ? src[3] : __builtin_inff();
            }
            a[l].x = q == gi ? 0.0f : a[l].x;
            a[l].y = q + 1 == gi ? 0.0f : a[l].y;
            a[l].z = q + 2 == gi ? 0.0f : a[l].z;
            a[l].w = q + 3 == gi ? 0.0f : a[l].w;
            b[l] = *reinterpret_cast<const float4 *>(strip + (int64_t)(c0 + r) * ldt + q);
        }
        __syncthreads();  // the previous slice's reads are done
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const int e = tid + l * NT, r = e / (KD / 4), q = e % (KD / 4) * 4;
            *reinterpret_cast<float4 *>(&As[r][q]) = a[l];
            *reinterpret_cast<float4 *>(&Bs[r][q]) = b[l];
        }
        __syncthreads();
#pragma unroll 1
        for (int g = KD - kCanonGroup; g >= 0; g -= kCanonGroup) {
            float m[4][4];
            uint64_t eq[4][4];  // lane masks
#pragma unroll
            for (int k = 0; k < kCanonGroup; k += 4) {
                float4 bv[4];
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    bv[c] = *reinterpret_cast<const float4 *>(&Bs[tx + 16 * c][g + k]);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float4 av = *reinterpret_cast<const float4 *>(&As[ty + NY * r][g + k]);
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const float x0 = av.x + bv[c].x, x1 = av.y + bv[c].y;
                        const float x2 = av.z + bv[c].z, x3 = av.w + bv[c].w;
                        if constexpr (kMin) {
                            const float y = __builtin_fminf(x0, x1);
                            m[r][c] = k == 0 ? y : __builtin_fminf(__builtin_fminf(m[r][c], x0), x1);
                            m[r][c] = __builtin_fminf(__builtin_fminf(m[r][c], x2), x3);
                        } else {
                            const float v = t[r][c];
                            const uint64_t h = lanes_eq(x0, v) | lanes_eq(x1, v) |
                                               lanes_eq(x2, v) | lanes_eq(x3, v);
                            eq[r][c] = k == 0 ? h : (eq[r][c] | h);
                        }
                    }
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    bool hit;
                    if constexpr (kMin) hit = m[r][c] <= t[r][c];
                    else hit = __builtin_amdgcn_inverse_ballot_w64(eq[r][c]);
                    grp[r][c] = hit ? q0 + g : grp[r][c];
                }
        }
    }
}

template <bool kMin>
__global__ void __launch_bounds__(kCanonThreads, kMin ? 4 : 6)
canon_pred_kernel(const float *__restrict__ d, int n, int64_t ld, const float *__restrict__ strip,
                  int j0, int w, int32_t *__restrict__ P, int64_t ldp,
                  const int32_t *__restrict__ frac, const int32_t *gate) {
    if (gated_off(gate)) return;
    constexpr int S = kCanonTile, KD = kCanonDepth, NY = 16, NT = kCanonThreads;
    __shared__ __align__(16) float lds[2 * S * (KD + 4)];
    float(*As)[KD + 4] = reinterpret_cast<float(*)[KD + 4]>(lds);  // As[r][q] = d[i0+r][q0+q]
    float(*Bs)[KD + 4] = As + S;                                   // Bs[c][q] = w[q0+q][c0+c]
    static_assert(2 * (KD + 4) >= S, "the groups take the slices' place");
    const int i0 = blockIdx.y * S, c0 = blockIdx.x * S;
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int ldt = canon_ldt(n);
    int32_t *const mark = P + (int64_t)i0 * ldp + j0 + c0;
    if constexpr (!kMin)
        if (*mark != kCanonAgain) return;
    const float limit = __builtin_ldexpf(1.0f, 24 - *frac);
    bool inexact = false;
    float t[4][4];
    int32_t grp[4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int i = i0 + ty + NY * r, cc = c0 + tx + 16 * c, j = j0 + cc;
            float v = __builtin_nanf("");
            if (i < n && cc < w && i != j) {
                v = d[(int64_t)i * ld + j];
                if (v == __builtin_inff()) v = __builtin_nanf("");
            }
            inexact = inexact || __builtin_fabsf(v) >= limit;
            t[r][c] = v;
        }
    if constexpr (kMin)
        if (__syncthreads_or(inexact)) {
            if (threadIdx.x == 0) *mark = kCanonAgain;
            return;
        }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) grp[r][c] = -1;
    canon_scan<kMin>(d, n, ld, strip, i0, c0, As, Bs, t, grp);
    // The groups go through LDS, so that the search is a short loop whose
    // registers are not the scan's.
    int32_t *G = reinterpret_cast<int32_t *>(lds);
    __syncthreads();  // the last slice's reads are done
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) G[(ty + NY * r) * S + tx + 16 * c] = grp[r][c];
    __syncthreads();
    bool miss = false;
#pragma unroll 2
    for (int e = threadIdx.x; e < S * S; e += NT) {
        const int i = i0 + e / S, cc = c0 + e % S, q0 = G[e];
        int32_t best = -1;
        if (q0 >= 0) {
            const float v = d[(int64_t)i * ld + j0 + cc];
            const float *ra = d + (int64_t)i * ld + q0;
            const float *rb = strip + (int64_t)cc * ldt + q0;
#pragma unroll
            for (int q = kCanonGroup - 1; q >= 0; --q) {
                const float x = q0 + q < n ? ra[q] : __builtin_inff();
                best = (q0 + q == i ? 0.0f : x) + rb[q] == v ? q0 + q : best;
            }
            miss = miss || best < 0;
        }
        if (i < n && cc < w) P[(int64_t)i * ldp + j0 + cc] = best;
    }
    // (thread 0 wrote that cell itself)
    if constexpr (kMin)
        if (__syncthreads_or(miss) && threadIdx.x == 0) *mark = kCanonAgain;
}

// The same for small matrices: a wave for 64 cells of one row, each lane through
// every candidate of its column, one launch for any weights.  64 x 64 cells a
// workgroup leave most CUs idle here, and the groups and the second launch cost
// more than they save: a captured solve of reals n=64 79 -> 48 us, n=128 122 ->
// 77, n=512 414 -> 332; of halves n=512 361 -> 333, but n=700 528 -> 594, where
// the L2 has to feed every candidate of every cell.  Hence the line at 512.
constexpr int kCanonSmallMax = 512;
__global__ void __launch_bounds__(64)
canon_pred_small_kernel(const float *__restrict__ d, int n, int64_t ld,
                        const float *__restrict__ strip, int j0, int w, int32_t *__restrict__ P,
                        int64_t ldp, const int32_t *gate) {
    if (gated_off(gate)) return;
    const int ldt = canon_ldt(n), i = blockIdx.y, c = blockIdx.x * 64 + threadIdx.x, j = j0 + c;
    const float *row = d + (int64_t)i * ld, *col = strip + (int64_t)c * ldt;
    float v = row[min(j, n - 1)];
    if (i == j || v == __builtin_inff()) v = __builtin_nanf("");
    int32_t best = -1;
#pragma unroll 2
    for (int q0 = ldt - 8; q0 >= 0; q0 -= 8) {
        const float4 lo = *reinterpret_cast<const float4 *>(col + q0);
        const float4 hi = *reinterpret_cast<const float4 *>(col + q0 + 4);
        const float b[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
        for (int e = 7; e >= 0; --e) {
            const int q = q0 + e;  // past n: the strip's padding matches nothing
            const float a = q == i ? 0.0f : row[min(q, n - 1)];
            best = a + b[e] == v ? q : best;
        }
    }
    if (j < j0 + w) P[(int64_t)i * ldp + j] = best;
}

// ---------------------------------------------------------------------------
// The keyed int32 predecessor solve (keys as in fw_internal.h).
// ---------------------------------------------------------------------------
// Zero the head of the scratch: the flags, and the row and column minima,
// which start at 0 -- the empty path from a vertex to itself.  (The cleared
// column panel after them is written by each stage's panel launch before
// its bulk reads it.)
__global__ void __launch_bounds__(256)
key_zero_kernel(int32_t *__restrict__ scratch, int64_t words) {
    for (int64_t w = blockIdx.x * 256 + threadIdx.x; w < words; w += (int64_t)gridDim.x * 256)
        scratch[w] = 0;
}

// key_ij = d_ij * 2^kKeyBits + (last hop of the edge: i; none on the
// diagonal), kKeyInf for an absent pair -- the keyed form of the predecessor
// initialisation.  An entry that is not an integer with |d_ij| < 2^14 (fp32:
// also a fraction, a NaN or -INF) raises the flag; within that range fp32
// sums of integers are exact, so the int32 keys compute what the fp32
// compare form does.
template <typename T>
__global__ void __launch_bounds__(256)
key_pack_kernel(const T *__restrict__ d, int32_t *__restrict__ keys, int n, int64_t ld,
                int64_t ldk, int32_t *__restrict__ flag) {
    bool bad = false;
    for (int i = blockIdx.y; i < n; i += gridDim.y)
        for (int j = blockIdx.x * 256 + threadIdx.x; j < n; j += gridDim.x * 256) {
            const T w = d[(int64_t)i * ld + j];
            int32_t key = kKeyInf;
            if (!Ar<T>::absent(w)) {
                int32_t v;
                if constexpr (std::is_same<T, float>::value) {
                    bad |= !(w == __builtin_rintf(w)) || !(__builtin_fabsf(w) < (float)(1 << kKeyBits));
                    v = bad ? 0 : (int32_t)w;
                } else {
                    bad |= w <= -(1 << kKeyBits) || w >= (1 << kKeyBits);
                    v = w;
                }
                key = (int32_t)((uint32_t)v << kKeyBits) + (i == j ? kKeyHop : i);
            }
            keys[(int64_t)i * ldk + j] = key;
        }
    if (bad) *flag = 1;
}

// A negative diagonal entry after the keyed sweep (a negative cycle: the
// pair-form sweep then gives its documented result) raises the flag, and
// the negative-diagonal word beside it.
__global__ void __launch_bounds__(256)
key_diag_kernel(const int32_t *__restrict__ keys, int n, int64_t ldk, int32_t *__restrict__ flag) {
    bool bad = false;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
        const int32_t key = keys[(int64_t)i * ldk + i];
        bad |= key < kKeyInfFloor && (key >> kKeyBits) < 0;
    }
    if (bad) {
        flag[0] = 1;
        flag[2] = 1;
    }
}

__device__ __forceinline__ int32_t wave_min(int32_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const int32_t u = __shfl_xor(v, o, 64);
        v = u < v ? u : v;
    }
    return v;
}

// Unless the flag is set: every key becomes its distance in d and its last
// hop in the key matrix, now the predecessor matrix as pred_fix_kernel
// leaves it (-1 on the diagonal and for an infinite key).  fp32: an infinite
// key (j not reachable from i) is +INF, as in the fp32 sweep.  int32: it
// leaves FW_I32_INF in d, for key_inf_kernel, and raises the "some pair
// unreachable" word; on the way, the row and column minima of the finite
// distances (starting at 0): a workgroup covers 256 columns of kMinRows
// rows, a column's minimum kept per thread, a row's reduced over each wave
// and then over the four waves in LDS, both folded in with atomicMin.
constexpr int kMinRows = 64;

template <typename T>
__global__ void __launch_bounds__(256)
key_unpack_kernel(T *__restrict__ d, int32_t *__restrict__ keys, int n, int64_t ld, int64_t ldk,
                  int32_t *__restrict__ scratch) {
    constexpr bool I32 = std::is_same<T, int32_t>::value;
    __shared__ int32_t wmin[4][kMinRows];
    if (scratch[0] != 0) return;
    int32_t *rowmin = scratch + 4, *colmin = scratch + 4 + n;
    const int j = blockIdx.x * 256 + threadIdx.x, wave = threadIdx.x >> 6;
    const int r0 = blockIdx.y * kMinRows;
    const int rows = n - r0 < kMinRows ? n - r0 : kMinRows;
    int32_t cmin = 0;
    bool unreachable = false;
    for (int r = 0; r < rows; ++r) {
        const int i = r0 + r;
        int32_t v = 0;
        if (j < n) {
            int32_t &k = keys[(int64_t)i * ldk + j];
            const int32_t key = k;
            T dist = Ar<T>::inf();
            int32_t hop = -1;
            if (key < kKeyInfFloor) {
                v = key >> kKeyBits;
                dist = (T)v;
                const int32_t h = key & kKeyHop;
                if (i != j && h != kKeyHop) hop = h;
            } else {
                unreachable = true;
            }
            d[(int64_t)i * ld + j] = dist;
            k = hop;
        }
        if constexpr (I32) {
            cmin = v < cmin ? v : cmin;
            const int32_t rm = wave_min(v);
            if ((threadIdx.x & 63) == 0) wmin[wave][r] = rm;
        }
    }
    if constexpr (!I32) return;
    __syncthreads();
    if ((int)threadIdx.x < rows) {
        const int t = threadIdx.x;
        int32_t m = wmin[0][t];
        m = wmin[1][t] < m ? wmin[1][t] : m;
        m = wmin[2][t] < m ? wmin[2][t] : m;
        m = wmin[3][t] < m ? wmin[3][t] : m;
        if (m < 0) atomicMin(rowmin + r0 + t, m);
    }
    if (j < n && cmin < 0) atomicMin(colmin + j, cmin);
    if (unreachable) scratch[1] = 1;
}

// Where j is not reachable from i: the value the int32 sweep over the
// complete graph reaches, FW_I32_INF + (row i's minimum) + (column j's
// minimum) -- the cheapest path i ~> u -> v ~> j through one absent edge
// u -> v splits into independent best prefix and suffix, every such (u, v)
// pair being absent.  Runs only if the unpack found such a pair.
__global__ void __launch_bounds__(256)
key_inf_kernel(int32_t *__restrict__ d, int n, int64_t ld, const int32_t *__restrict__ scratch) {
    if (scratch[0] != 0 || scratch[1] == 0) return;
    const int32_t *rowmin = scratch + 4, *colmin = scratch + 4 + n;
    for (int i = blockIdx.y; i < n; i += gridDim.y) {
        const int32_t rm = rowmin[i];
        for (int j = blockIdx.x * 256 + threadIdx.x; j < n; j += gridDim.x * 256) {
            int32_t &v = d[(int64_t)i * ld + j];
            if (v == kI32Inf) v = kI32Inf + rm + colmin[j];
        }
    }
}

// The vertices i with d_ii < 0 after a solve, in ascending order, and their
// number; one workgroup of 1024 threads walks the diagonal in chunks of 1024,
// each chunk compacted by wave ballots and a scan of the 16 wave counts.
// Either output may be NULL (the flag-only call passes list = NULL).
template <typename T>
__global__ void __launch_bounds__(1024)
negcycle_kernel(const T *__restrict__ d, int n, int64_t ld, int32_t *__restrict__ list,
                int32_t *__restrict__ count) {
    __shared__ int wave_cnt[16];
    __shared__ int total;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x == 0) total = 0;
    __syncthreads();
    for (int base = 0; base < n; base += 1024) {
        const int i = base + (int)threadIdx.x;
        const bool neg = i < n && d[(int64_t)i * ld + i] < T(0);
        const uint64_t mask = __ballot(neg);
        if (lane == 0) wave_cnt[wave] = __popcll(mask);
        __syncthreads();
        int before = total;  // entries of earlier chunks and earlier waves
        for (int w = 0; w < wave; ++w) before += wave_cnt[w];
        const uint64_t below = lane ? (mask & (~0ull >> (64 - lane))) : 0ull;
        if (neg && list) list[before + __popcll(below)] = i;
        __syncthreads();
        if (threadIdx.x == 0)
            for (int w = 0; w < 16; ++w) total += wave_cnt[w];
        __syncthreads();
    }
    if (threadIdx.x == 0 && count) *count = total;
}

// About 8K workgroups whatever n: enough to stream the matrix, and cheap to
// dispatch when a gated launch finds its gate closed.
dim3 elementwise_grid(int n) {
    int gx = (n + 255) / 256 < 64 ? (n + 255) / 256 : 64;
    gx = gx > 0 ? gx : 1;
    int gy = 8192 / gx;
    gy = n < gy ? n : gy;
    return dim3(gx, gy > 0 ? gy : 1);
}

// ---------------------------------------------------------------------------
// Dispatch: compile-time tile configurations.  Cells per thread and threads:
//   tile  panels and bulk                        diagonal (with predecessors, or
//                                                 keys; closure_threads)
//   128   strips 4 x 4 (512), bulk 8 x 8 (256)   4 x 8, 512 + 64 (4 x 4, 1024)
//    64   4 x 4 (256, or 512 in two halves)      2 x 4, 512 + 64 (4 x 4, 256)
//    32   4 x 4 (64)                             2 x 2, 256 + 64 (2 x 2, 256)
// With predecessors panels and bulk are the register-staged tile_kernel: 4 x 4
// cells, 1024, 256 and 64 threads (keyed at 128: see tile_t).
// ---------------------------------------------------------------------------
template <typename T, bool PRED, class A>
hipError_t diag_t(int tile, T *d, int32_t *p, int n, int64_t ld, int64_t ldp, int b,
                  hipStream_t st, int32_t *flag, const int32_t *gate) {
    switch (tile) {
    case 128:
        diag_kernel<T, 128, PRED, A><<<1, closure_threads<T, 128, PRED, A, true>(), 0, st>>>(d, p, n, ld, ldp, b, flag, gate);
        break;
    case 64:
        diag_kernel<T, 64, PRED, A><<<1, closure_threads<T, 64, PRED, A, true>(), 0, st>>>(d, p, n, ld, ldp, b, flag, gate);
        break;
    case 32:
        diag_kernel<T, 32, PRED, A><<<1, closure_threads<T, 32, PRED, A, true>(), 0, st>>>(d, p, n, ld, ldp, b, flag, gate);
        break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}


#ifndef FW_PRED128_TM
#define FW_PRED128_TM 4
#define FW_PRED128_TN 4
#define FW_PRED128_BK 32
#endif

template <typename T, bool VEC, bool PRED, class A>
hipError_t tile_t(int tile, T *d, int32_t *p, int n, int64_t ld, int64_t ldp, int b, int nb,
                  int mode, unsigned grid, hipStream_t st, int close_next, int32_t *flag,
                  const int32_t *gate) {
    switch (tile) {
    case 128:
        if constexpr (PRED) {
            // the predecessor update keeps twice the state per cell; 4 x 4
            // sub-tiles over 1024 threads keep it at 4 waves per SIMD
            constexpr int TMP = FW_PRED128_TM, TNP = FW_PRED128_TN;
            tile_kernel<T, 128, FW_PRED128_BK, TMP, TNP, VEC, PRED, A>
                <<<grid, (128 / TMP) * (128 / TNP), 0, st>>>(d, p, n, ld, ldp, b, nb, mode,
                                                             close_next, flag, gate);
        } else {
            return hipErrorInvalidValue;  // panel_strip_kernel's, bulk_dma_kernel's
        }
        break;
    case 64:
        if constexpr (PRED)
            tile_kernel<T, 64, 16, 4, 4, VEC, PRED, A><<<grid, 256, 0, st>>>(
                d, p, n, ld, ldp, b, nb, mode, close_next, flag, gate);
        else
            return hipErrorInvalidValue;  // tile64_launch's
        break;
    case 32:
        tile_kernel<T, 32, 16, 4, 4, VEC, PRED, A><<<grid, 64, 0, st>>>(
            d, p, n, ld, ldp, b, nb, mode, 0, flag, gate);
        break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// The bulk launch of stage b also closes the next diagonal tile: at tile 64;
// at tile 128 with predecessors, and without them wherever the closure takes
// the bulk workgroup's registers: in sub-blocks, or, on keys, a whole tile in
// 16-byte pieces.
bool bulk_closes(int sr, int tile, bool pred, bool vec, int n, int b) {
    if (b + 1 >= (n + tile - 1) / tile) return false;
    if (tile == 64) return !pred || sr == kMinPlus;
    if (tile != 128) return false;
    if (pred) return sr == kMinPlus;
    return sr != kKey || (vec && b + 1 < n / 128);
}

template <typename T, class A, bool ALLOW_PRED>
hipError_t tile_dispatch(int tile, T *d, int32_t *p, int n, int64_t ld, int64_t ldp, int b,
                         int nb, int mode, bool close_next, hipStream_t st, int32_t *flag,
                         const int32_t *gate) {
    // gates: the predecessor forms (the pair-form sweep behind a keyed one),
    // and without predecessors tiles 64 and 32 (the distances of the fp32
    // canonical path)
    if (gate && !p && tile > 64) return hipErrorInvalidValue;
    const int64_t m = nb - 1;
    const int64_t grid = mode == 0 ? 2 * m : m * m;
    if (grid <= 0) return close_next ? hipErrorInvalidValue : hipSuccess;
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    const bool vec = vec_ok(d, ld) && (p == nullptr || vec_ok(p, ldp));
    constexpr int kSr = A::kChecked ? kKey : kMinPlus;
    if (close_next && (mode != 1 || !bulk_closes(kSr, tile, p != nullptr, vec, n, b)))
        return hipErrorInvalidValue;
    const int c = close_next ? 1 : 0;
    // the keyed 128-wide sweep's cleared column panel (in the solve's scratch)
    T *acol = nullptr;
    if constexpr (A::kChecked) acol = reinterpret_cast<T *>(flag + key_acol_offset(n));
    if constexpr (ALLOW_PRED) {
        if (p) {
            return vec ? tile_t<T, true, true, A>(tile, d, p, n, ld, ldp, b, nb, mode,
                                                  (unsigned)grid, st, c, flag, gate)
                       : tile_t<T, false, true, A>(tile, d, p, n, ld, ldp, b, nb, mode,
                                                   (unsigned)grid, st, c, flag, gate);
        }
    } else {
        if (p) return hipErrorInvalidValue;
    }
    if (tile == 64)
        return grid <= kTile64SplitMax
                   ? tile64_launch<T, 2, A>(d, n, ld, vec, b, nb, mode, close_next,
                                            (unsigned)grid, st, flag, gate)
                   : tile64_launch<T, 1, A>(d, n, ld, vec, b, nb, mode, close_next,
                                            (unsigned)grid, st, flag, gate);
    if (tile == 128) {
        if (mode == 0) {
            if (4 * grid > 0x7fffffffLL) return hipErrorInvalidValue;
            if (vec)
                panel_strip_kernel<T, true, A><<<(unsigned)(4 * grid), kStripThreads, 0, st>>>(
                    d, n, ld, b, nb, flag, acol);
            else
                panel_strip_kernel<T, false, A><<<(unsigned)(4 * grid), kStripThreads, 0, st>>>(
                    d, n, ld, b, nb, flag, acol);
        } else if (vec) {
            bulk_dma_kernel<T, true, A><<<(unsigned)grid, 256, 0, st>>>(d, n, ld, b, (int)m, c,
                                                                       flag, acol);
        } else {
            bulk_dma_kernel<T, false, A><<<(unsigned)grid, 256, 0, st>>>(d, n, ld, b, (int)m, c,
                                                                        flag, acol);
        }
        return hipGetLastError();
    }
    if (close_next) return hipErrorInvalidValue;  // every closing form is handled above
    return vec ? tile_t<T, true, false, A>(tile, d, p, n, ld, ldp, b, nb, mode, (unsigned)grid, st,
                                           0, flag, gate)
               : tile_t<T, false, false, A>(tile, d, p, n, ld, ldp, b, nb, mode, (unsigned)grid,
                                            st, 0, flag, gate);
}

template <typename T>
hipError_t tile_any(int sr, int tile, T *d, int32_t *p, int n, int64_t ld, int64_t ldp, int b,
                    int nb, int mode, bool close_next, hipStream_t st, int32_t *flag,
                    const int32_t *gate) {
    if (gate && sr != kMinPlus) return hipErrorInvalidValue;
    if (sr == kMaxMin)
        return tile_dispatch<T, ArMaxMin<T>, false>(tile, d, p, n, ld, ldp, b, nb, mode,
                                                     close_next, st, nullptr, gate);
    if (sr == kKey) {
        if constexpr (std::is_same<T, int32_t>::value) {
            if (!flag) return hipErrorInvalidValue;
            return tile_dispatch<int32_t, ArKey, false>(tile, d, p, n, ld, ldp, b, nb, mode,
                                                        close_next, st, flag, gate);
        }
        return hipErrorInvalidValue;
    }
    return tile_dispatch<T, Ar<T>, true>(tile, d, p, n, ld, ldp, b, nb, mode, close_next, st,
                                         nullptr, gate);
}

}  // namespace

hipError_t launch_diag(int dtype, int sr, int tile, void *d, int32_t *p, int n, int64_t ld,
                       int64_t ldp, int b, hipStream_t st, int32_t *flag, const int32_t *gate) {
    if (gate && (sr != kMinPlus || (!p && tile > 64))) return hipErrorInvalidValue;
    if (sr == kMaxMin) {
        if (p) return hipErrorInvalidValue;
        if (dtype == 0)
            return diag_t<float, false, ArMaxMin<float>>(tile, (float *)d, p, n, ld, ldp, b, st,
                                                         nullptr, nullptr);
        return diag_t<int32_t, false, ArMaxMin<int32_t>>(tile, (int32_t *)d, p, n, ld, ldp, b,
                                                         st, nullptr, nullptr);
    }
    if (sr == kKey) {
        if (p || dtype != 1 || !flag) return hipErrorInvalidValue;
        return diag_t<int32_t, false, ArKey>(tile, (int32_t *)d, p, n, ld, ldp, b, st, flag,
                                             nullptr);
    }
    if (dtype == 0)
        return p ? diag_t<float, true, Ar<float>>(tile, (float *)d, p, n, ld, ldp, b, st, nullptr,
                                                  gate)
                 : diag_t<float, false, Ar<float>>(tile, (float *)d, p, n, ld, ldp, b, st,
                                                   nullptr, gate);
    return p ? diag_t<int32_t, true, Ar<int32_t>>(tile, (int32_t *)d, p, n, ld, ldp, b, st,
                                                  nullptr, gate)
             : diag_t<int32_t, false, Ar<int32_t>>(tile, (int32_t *)d, p, n, ld, ldp, b, st,
                                                   nullptr, gate);
}

hipError_t launch_panels(int dtype, int sr, int tile, void *d, int32_t *p, int n, int64_t ld,
                         int64_t ldp, int b, int nb, hipStream_t st, int32_t *flag,
                         const int32_t *gate) {
    if (dtype == 0)
        return tile_any<float>(sr, tile, (float *)d, p, n, ld, ldp, b, nb, 0, false, st, flag,
                               gate);
    return tile_any<int32_t>(sr, tile, (int32_t *)d, p, n, ld, ldp, b, nb, 0, false, st, flag,
                             gate);
}

bool bulk_closes_next_diag(int sr, int tile, const void *d, const int32_t *p, int n, int64_t ld,
                           int b) {
    return bulk_closes(sr, tile, p != nullptr, vec_ok(d, ld), n, b);
}

hipError_t launch_bulk(int dtype, int sr, int tile, void *d, int32_t *p, int n, int64_t ld,
                       int64_t ldp, int b, int nb, bool close_next, hipStream_t st, int32_t *flag,
                       const int32_t *gate) {
    if (dtype == 0)
        return tile_any<float>(sr, tile, (float *)d, p, n, ld, ldp, b, nb, 1, close_next, st,
                               flag, gate);
    return tile_any<int32_t>(sr, tile, (int32_t *)d, p, n, ld, ldp, b, nb, 1, close_next, st,
                             flag, gate);
}

hipError_t launch_pred_init(int dtype, const void *d, int32_t *p, int n, int64_t ld,
                            int64_t ldp, hipStream_t st, const int32_t *gate) {
    const dim3 g = elementwise_grid(n);
    if (dtype == 0)
        pred_init_kernel<float><<<g, 256, 0, st>>>((const float *)d, p, n, ld, ldp, gate);
    else
        pred_init_kernel<int32_t><<<g, 256, 0, st>>>((const int32_t *)d, p, n, ld, ldp, gate);
    return hipGetLastError();
}

hipError_t launch_pred_fix(int dtype, const void *d, int32_t *p, int n, int64_t ld,
                           int64_t ldp, hipStream_t st, const int32_t *gate) {
    const dim3 g = elementwise_grid(n);
    if (dtype == 0)
        pred_fix_kernel<float><<<g, 256, 0, st>>>((const float *)d, p, n, ld, ldp, gate);
    else
        pred_fix_kernel<int32_t><<<g, 256, 0, st>>>((const int32_t *)d, p, n, ld, ldp, gate);
    return hipGetLastError();
}

hipError_t launch_key_prepare(int dtype, const void *d, int32_t *keys, int n, int64_t ld,
                              int64_t ldk, int32_t *scratch, hipStream_t st) {
    const int64_t words = key_acol_offset(n);
    key_zero_kernel<<<(unsigned)((words + 255) / 256), 256, 0, st>>>(scratch, words);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (dtype == 0)
        key_pack_kernel<float><<<elementwise_grid(n), 256, 0, st>>>((const float *)d, keys, n, ld,
                                                                   ldk, scratch);
    else
        key_pack_kernel<int32_t><<<elementwise_grid(n), 256, 0, st>>>((const int32_t *)d, keys,
                                                                     n, ld, ldk, scratch);
    return hipGetLastError();
}

hipError_t launch_key_finish(int dtype, void *d, int32_t *keys, int n, int64_t ld, int64_t ldk,
                             int32_t *scratch, hipStream_t st) {
    key_diag_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(keys, n, ldk, scratch);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 gu((unsigned)((n + 255) / 256), (unsigned)((n + kMinRows - 1) / kMinRows));
    if (dtype == 0) {
        key_unpack_kernel<float><<<gu, 256, 0, st>>>((float *)d, keys, n, ld, ldk, scratch);
        return hipGetLastError();
    }
    key_unpack_kernel<int32_t><<<gu, 256, 0, st>>>((int32_t *)d, keys, n, ld, ldk, scratch);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    key_inf_kernel<<<elementwise_grid(n), 256, 0, st>>>((int32_t *)d, n, ld, scratch);
    return hipGetLastError();
}

hipError_t launch_canon_gate(int32_t *scratch, bool direct, hipStream_t st) {
    canon_gate_kernel<<<1, 64, 0, st>>>(scratch, direct ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_canon_restore(float *d, const int32_t *p, int n, int64_t ld, int64_t ldp,
                                const int32_t *gate, hipStream_t st) {
    canon_restore_kernel<<<elementwise_grid(n), 256, 0, st>>>(d, p, n, ld, ldp, gate);
    return hipGetLastError();
}

hipError_t launch_canon_save(const float *d, int32_t *p, int n, int64_t ld, int64_t ldp,
                             const int32_t *gate, hipStream_t st) {
    canon_save_kernel<<<elementwise_grid(n), 256, 0, st>>>(d, p, n, ld, ldp, gate);
    return hipGetLastError();
}

hipError_t launch_canon_strip(const int32_t *p, int n, int64_t ldp, int j0, int w, float *strip,
                              int32_t *frac, const int32_t *gate, hipStream_t st) {
    if (n <= 0 || w <= 0 || j0 < 0 || j0 + w > n) return hipErrorInvalidValue;
    const int gx = (w + 63) / 64, gy = std::min((canon_ldt(n) + 63) / 64, std::max(1, 8192 / gx));
    canon_strip_kernel<<<dim3((unsigned)gx, (unsigned)gy), 256, 0, st>>>(p, n, ldp, j0, w, strip,
                                                                         frac, gate);
    return hipGetLastError();
}

hipError_t launch_canon_pred(const float *d, int n, int64_t ld, const float *strip, int j0, int w,
                             int32_t *p, int64_t ldp, const int32_t *frac, const int32_t *gate,
                             hipStream_t st) {
    if (n <= 0 || w <= 0 || j0 < 0 || j0 + w > n) return hipErrorInvalidValue;
    if (n <= kCanonSmallMax) {
        canon_pred_small_kernel<<<dim3((unsigned)((w + 63) / 64), (unsigned)n), 64, 0, st>>>(
            d, n, ld, strip, j0, w, p, ldp, gate);
        return hipGetLastError();
    }
    const dim3 g((unsigned)((w + kCanonTile - 1) / kCanonTile),
                 (unsigned)((n + kCanonTile - 1) / kCanonTile));
    canon_pred_kernel<true><<<g, kCanonThreads, 0, st>>>(d, n, ld, strip, j0, w, p, ldp, frac,
                                                         gate);
    canon_pred_kernel<false><<<g, kCanonThreads, 0, st>>>(d, n, ld, strip, j0, w, p, ldp, frac,
                                                          gate);
    return hipGetLastError();
}

int64_t pred_fallbacks() {
    unsigned long long v = 0;
    if (hipMemcpyFromSymbol(&v, HIP_SYMBOL(g_pred_fallbacks), sizeof(v), 0,
                            hipMemcpyDeviceToHost) != hipSuccess)
        return -1;
    return (int64_t)v;
}

hipError_t launch_negcycle(int dtype, const void *d, int n, int64_t ld, int32_t *list,
                           int32_t *count, hipStream_t st) {
    if (dtype == 0)
        negcycle_kernel<float><<<1, 1024, 0, st>>>((const float *)d, n, ld, list, count);
    else
        negcycle_kernel<int32_t><<<1, 1024, 0, st>>>((const int32_t *)d, n, ld, list, count);
    return hipGetLastError();
}

}  // namespace fw

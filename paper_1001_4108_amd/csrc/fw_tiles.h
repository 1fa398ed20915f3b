// Workgroup-level building blocks of blocked Floyd-Warshall on gfx950.
//
// Both are executed by one whole workgroup and shared by the per-phase
// kernels (one tile per workgroup, fw_kernels.hip) and by the persistent
// batched kernel (one graph per workgroup, fw_batched.hip), so a graph gets
// the same per-cell candidate sequence -- hence the same bits -- either way.
//
//   closure_tile_any -- Floyd-Warshall (section 3.1, Fig. FW-Alg) restricted to
//                    one s x s tile whose origin is on the diagonal: the
//                    paper's "independent block" (section 3.2).  With
//                    predecessors (closure_tile) step by step, so that a tile
//                    over the whole graph IS the plain algorithm; without them
//                    (closure_blocks) in 8-vertex sub-blocks, the same results
//                    in exact arithmetic from sums in another association.
//   product_tile  -- C <- min(C, A (x) B) over one k-block: the paper's
//                    "doubly dependent" update (section 3.2) with A = tile
//                    (bi, b), B = tile (b, bj), C = tile (bi, bj).
//
// Padding: cells outside the n x n matrix read as "infinity" and are never
// written, i.e. the padded vertices are isolated and change no distance.
#pragma once

#include <type_traits>
#include <utility>

#include "fw_internal.h"

namespace fw {

template <typename T> struct Ar;

// fp32 minimum and maximum.  With FW_MINIMUM the IEEE 754-2019 forms
// (gfx950's v_minimum3_f32 / v_maximum3_f32): IEEE-mode v_min_f32 needs its
// operands quieted first, and wherever the compiler cannot prove a value is
// already canonical (a load, a value pinned across a barrier) it spends a
// v_max_f32 x, x, x on it; the 2019 forms need none.  The two agree except
// on NaN (excluded by the contract) and on which zero of +0 / -0 is
// returned (left open by the contract).
#ifndef FW_MINIMUM
#define FW_MINIMUM 1
#endif
__device__ __forceinline__ float fmin32(float a, float b) {
#if FW_MINIMUM
    return __builtin_elementwise_minimum(a, b);
#else
    return __builtin_fminf(a, b);
#endif
}
__device__ __forceinline__ float fmax32(float a, float b) {
#if FW_MINIMUM
    return __builtin_elementwise_maximum(a, b);
#else
    return __builtin_fmaxf(a, b);
#endif
}

// Every policy says whether its values need settle() before they are stored
// or handed to other cells as operands (only the keyed policy does).  top()
// is the value that min2 and min3 leave out against any other.
template <> struct Ar<float> {
    static constexpr bool kChecked = false;
    __device__ __forceinline__ static float inf() { return __builtin_inff(); }
    __device__ __forceinline__ static float top() { return __builtin_inff(); }
    __device__ __forceinline__ static float add(float a, float b) { return a + b; }
    __device__ __forceinline__ static float min2(float a, float b) { return fmin32(a, b); }
    __device__ __forceinline__ static float min3(float a, float b, float c) {
        return fmin32(fmin32(a, b), c);
    }
    __device__ __forceinline__ static bool absent(float v) { return v == __builtin_inff(); }
    __device__ __forceinline__ static bool unreachable(float v) { return v == __builtin_inff(); }
};

template <> struct Ar<int32_t> {
    static constexpr bool kChecked = false;
    __device__ __forceinline__ static int32_t inf() { return kI32Inf; }
    __device__ __forceinline__ static int32_t top() { return 0x7fffffff; }
    __device__ __forceinline__ static int32_t add(int32_t a, int32_t b) {
        return (int32_t)((uint32_t)a + (uint32_t)b);
    }
    __device__ __forceinline__ static int32_t min2(int32_t a, int32_t b) { return a < b ? a : b; }
    __device__ __forceinline__ static int32_t min3(int32_t a, int32_t b, int32_t c) {
        return min2(min2(a, b), c);
    }
    __device__ __forceinline__ static bool absent(int32_t v) { return v == kI32Inf; }
    __device__ __forceinline__ static bool unreachable(int32_t v) { return v > kI32Inf / 2; }
};

// The (max, min) semiring through the same code: "add" is min (a path is as
// wide as its narrowest edge) and "min" is max (keep the widest path).  The
// padding value is the max-identity, so padded vertices stay isolated.  Over
// {0, 1} this is the transitive closure.  min and max are exact, so every
// order of the updates gives the same bits.
template <typename T> struct ArMaxMin;

template <> struct ArMaxMin<float> {
    static constexpr bool kChecked = false;
    __device__ __forceinline__ static float inf() { return -__builtin_inff(); }
    __device__ __forceinline__ static float top() { return -__builtin_inff(); }
    __device__ __forceinline__ static float add(float a, float b) { return fmin32(a, b); }
    __device__ __forceinline__ static float min2(float a, float b) { return fmax32(a, b); }
    __device__ __forceinline__ static float min3(float a, float b, float c) {
        return fmax32(fmax32(a, b), c);
    }
};

template <> struct ArMaxMin<int32_t> {
    static constexpr bool kChecked = false;
    __device__ __forceinline__ static int32_t inf() { return (int32_t)0x80000000; }
    __device__ __forceinline__ static int32_t top() { return (int32_t)0x80000000; }
    __device__ __forceinline__ static int32_t add(int32_t a, int32_t b) { return a < b ? a : b; }
    __device__ __forceinline__ static int32_t min2(int32_t a, int32_t b) { return a > b ? a : b; }
    __device__ __forceinline__ static int32_t min3(int32_t a, int32_t b, int32_t c) {
        return min2(min2(a, b), c);
    }
};

// Min-plus over the 32-bit (distance, last hop) keys of fw_internal.h: the
// int32 form of the lexicographic update below in one add and (for two
// k-steps) one three-input minimum, the arithmetic of the distances-only
// sweep.  "add" clears the hop field of its first operand -- always the
// (i, k) cell, whose last hop the candidate does not inherit -- and adds the
// (k, j) key.  settle() brings a value back to the key invariant before it is
// stored or published to other cells: an infinite-class value becomes exactly
// kKeyInf, and a real value outside [kKeyLow, kKeyReal) (|d| >= 2^14) is
// recorded in the KeyCheck (the solve is then redone by the 64-bit form).
//
// KeyCheck: two running minima instead of a flag, so the check costs a few
// vector instructions per value and no lane-mask state.  Values that reach
// settle() lie in (-2^29, 2^29) (real) or [kKeyInf - 2^28, kKeyInf] (infinite
// class, at or above 3 * 2^28 - 2^14), so a real value is too large exactly
// when v - kKeyReal, as unsigned, is below kKeyReal, and too small exactly
// when v < kKeyLow.
struct KeyCheck {
    uint32_t hi = 0xffffffffu;  // min over values of (uint32)(v - kKeyReal)
    int32_t lo = 0;             // min over values
    __device__ __forceinline__ bool bad() const {
        return hi < (uint32_t)kKeyReal || lo < kKeyLow;
    }
};

struct ArKey {
    static constexpr bool kChecked = true;
    __device__ __forceinline__ static int32_t inf() { return kKeyInf; }
    __device__ __forceinline__ static int32_t top() { return 0x7fffffff; }
    __device__ __forceinline__ static int32_t add(int32_t a, int32_t b) {
        return (int32_t)(((uint32_t)a & ~(uint32_t)kKeyHop) + (uint32_t)b);
    }
    // add for a first operand whose hop field is already clear
    __device__ __forceinline__ static int32_t add_cleared(int32_t a, int32_t b) {
        return (int32_t)((uint32_t)a + (uint32_t)b);
    }
    __device__ __forceinline__ static int32_t clear_hop(int32_t a) {
        return (int32_t)((uint32_t)a & ~(uint32_t)kKeyHop);
    }
    __device__ __forceinline__ static int32_t min2(int32_t a, int32_t b) { return a < b ? a : b; }
    __device__ __forceinline__ static int32_t min3(int32_t a, int32_t b, int32_t c) {
        return min2(min2(a, b), c);
    }
    __device__ __forceinline__ static int32_t settle(int32_t v, KeyCheck &c) {
        const uint32_t up = (uint32_t)v - (uint32_t)kKeyReal;
        c.hi = up < c.hi ? up : c.hi;
        c.lo = v < c.lo ? v : c.lo;
        return v >= kKeyInfFloor ? kKeyInf : v;
    }
};

template <class A, typename T>
__device__ __forceinline__ T settle(T v, KeyCheck &c) {
    if constexpr (A::kChecked)
        return A::settle(v, c);
    else
        return v;
}

// Raise the solve's flag from every lane whose check found a bad key.
template <class A>
__device__ __forceinline__ void raise_flag(int32_t *flag, const KeyCheck &c) {
    if constexpr (A::kChecked) {
        if (c.bad()) *flag = 1;
    }
}

// Lexicographic minimum of (distance, last hop): the candidate replaces the
// current pair when it is strictly shorter, or equally short with a smaller
// last hop.  This keeps, for every pair, the smallest last hop over all
// shortest paths, a quantity independent of the order of the updates.
template <typename T>
__device__ __forceinline__ void lex_update(T &c, int32_t &p, T cand, int32_t pc) {
    const bool take = (cand < c) || (cand == c && pc < p);
    c = take ? cand : c;
    p = take ? pc : p;
}

// The predecessor a cell keeps after the sweep: -1 where no last hop was
// found, for an unreachable pair, and on the diagonal -- except where d_ii < 0
// (a negative cycle through i, outside the problem statement), whose last hop
// is kept so that the cycle can be walked back from the matrix.
template <typename T>
__device__ __forceinline__ int32_t final_pred(int i, int j, T v, int32_t p) {
    if (p == kPredNone) return -1;
    if (i == j) return v < T(0) ? p : -1;
    return Ar<T>::unreachable(v) ? -1 : p;
}

template <typename T> struct Vec4 { typedef T type __attribute__((ext_vector_type(4))); };
// Four consecutive values at any 4-byte address: gfx950's 16-byte global loads
// and stores need no more.
template <typename T>
struct Vec4u {
    typedef T type __attribute__((ext_vector_type(4), aligned(4)));
};

// Load E consecutive elements of one matrix row starting at column `col`;
// out-of-range elements read as `fill`.
template <typename T, int E, bool VEC>
__device__ __forceinline__ void row_load(T (&v)[E], const T *__restrict__ base, int row, int col,
                                         int n, int64_t ld, bool full, T fill) {
    if (VEC && full) {
        const T *src = base + (int64_t)row * ld + col;
#pragma unroll
        for (int e = 0; e < E; e += 4) {
            const typename Vec4<T>::type x =
                *reinterpret_cast<const typename Vec4<T>::type *>(src + e);
            v[e] = x[0];
            v[e + 1] = x[1];
            v[e + 2] = x[2];
            v[e + 3] = x[3];
        }
    } else if (full) {
        const T *src = base + (int64_t)row * ld + col;
        if constexpr (E % 4 == 0) {
#pragma unroll
            for (int e = 0; e < E; e += 4) {
                const typename Vec4u<T>::type x =
                    *reinterpret_cast<const typename Vec4u<T>::type *>(src + e);
                v[e] = x[0];
                v[e + 1] = x[1];
                v[e + 2] = x[2];
                v[e + 3] = x[3];
            }
        } else {
#pragma unroll
            for (int e = 0; e < E; ++e) v[e] = src[e];
        }
    } else {
        const bool rok = row < n;
        const T *src = base + (rok ? (int64_t)row * ld : 0);
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] = (rok && col + e < n) ? src[col + e] : fill;
    }
}

template <typename T, int E, bool VEC>
__device__ __forceinline__ void row_store(const T (&v)[E], T *__restrict__ base, int row, int col,
                                          int n, int64_t ld, bool full) {
    if (VEC && full) {
        T *dst = base + (int64_t)row * ld + col;
#pragma unroll
        for (int e = 0; e < E; e += 4) {
            typename Vec4<T>::type x;
            x[0] = v[e];
            x[1] = v[e + 1];
            x[2] = v[e + 2];
            x[3] = v[e + 3];
            *reinterpret_cast<typename Vec4<T>::type *>(dst + e) = x;
        }
    } else if (full) {
        T *dst = base + (int64_t)row * ld + col;
        if constexpr (E % 4 == 0) {
#pragma unroll
            for (int e = 0; e < E; e += 4) {
                typename Vec4u<T>::type x;
                x[0] = v[e];
                x[1] = v[e + 1];
                x[2] = v[e + 2];
                x[3] = v[e + 3];
                *reinterpret_cast<typename Vec4u<T>::type *>(dst + e) = x;
            }
        } else {
#pragma unroll
            for (int e = 0; e < E; ++e) dst[e] = v[e];
        }
    } else if (row < n) {
        T *dst = base + (int64_t)row * ld;
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (col + e < n) dst[col + e] = v[e];
    }
}

// A policy's "add" for a first operand that first() has prepared: the keyed
// policy clears the hop field once per operand instead of once per sum.
template <class A, typename T>
__device__ __forceinline__ T first(T a) {
    if constexpr (A::kChecked)
        return A::clear_hop(a);
    else
        return a;
}
template <class A, typename T>
__device__ __forceinline__ T add_first(T a, T b) {
    if constexpr (A::kChecked)
        return A::add_cleared(a, b);
    else
        return A::add(a, b);
}

// Four cells of a product over a k-pair: c_e <- min3(c_e, a0 x b0_e, a1 x b1_e)
// (a0, a1 prepared by first()).
// Integer min-plus, written out: what bounds the int32 and keyed products is
// how the adds of one wave share the SIMD with the minima of the others, and
// that hangs on the order of issue.  Left to the compiler the two sums of every
// cell go through the same two registers, and the loop issues 56 lanes per
// clock per CU of a possible 107; with two registers of its own per cell and a
// one-cycle gap before each minimum it issues 69 (n=8192 int32: 24.4 -> 19.9
// ms, with predecessors 25.6 -> 21.1; without the gap 22.7, with the eight adds
// first 21.6, with a gap of three cycles 22.5).  A minimum is written before later
// cells read their operands, hence the early clobbers.  fp32 is fastest as the compiler
// orders it (n=16384 110 ms against 116-139 in these forms).
template <class A, typename T>
__device__ __forceinline__ void update4(T (&c)[4], T a0, T a1, const T *b0, const T *b1) {
    if constexpr (std::is_same<A, Ar<int32_t>>::value || A::kChecked) {
        int32_t s[4], t[4];
#define FW_CELL(i)                                                                   \
    "v_add_u32 %[s" #i "], %[p" #i "], %[a]\n\t"                                     \
    "v_add_u32 %[t" #i "], %[q" #i "], %[b]\n\t"                                     \
    "s_nop 0\n\t"                                                                    \
    "v_min3_i32 %[c" #i "], %[c" #i "], %[s" #i "], %[t" #i "]\n\t"
        asm(FW_CELL(0) FW_CELL(1) FW_CELL(2) FW_CELL(3)
            : [c0] "+&v"(c[0]), [c1] "+&v"(c[1]), [c2] "+&v"(c[2]), [c3] "+&v"(c[3]),
              [s0] "=&v"(s[0]), [s1] "=&v"(s[1]), [s2] "=&v"(s[2]), [s3] "=&v"(s[3]),
              [t0] "=&v"(t[0]), [t1] "=&v"(t[1]), [t2] "=&v"(t[2]), [t3] "=&v"(t[3])
            : [a] "v"(a0), [b] "v"(a1), [p0] "v"(b0[0]), [p1] "v"(b0[1]), [p2] "v"(b0[2]),
              [p3] "v"(b0[3]), [q0] "v"(b1[0]), [q1] "v"(b1[1]), [q2] "v"(b1[2]), [q3] "v"(b1[3]));
#undef FW_CELL
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) c[e] = A::min3(c[e], A::add(a0, b0[e]), A::add(a1, b1[e]));
    }
}

// ---------------------------------------------------------------------------
// closure_tile: s dependent k-steps on the tile with origin (base, base).
//
// (S/TM)^2 threads; thread (ty, tx) keeps the TM x TM cells rows ty*TM..,
// columns tx*TM.. in registers for all S steps.  Step k needs row k and
// column k as they are after step k-1; their owners publish them to a
// double-buffered LDS row/column before the step's barrier.  Row k and column
// k do not change during step k (d_kk >= 0), so one barrier per step
// suffices.  The TM steps of one register row are unrolled so the owner's
// register index is a compile-time constant.
// ---------------------------------------------------------------------------
// (without predecessors: closure_blocks' two buffers of 8 rows and of 8
// columns, its small ones, and ahead one more of 8 columns)
constexpr int kCloseExtra = 2 * 8 * 12 + 2 * 8 * 8;
template <typename T, int S, bool PRED, bool AHEAD = false>
constexpr int closure_smem_bytes() {
    return PRED ? 4 * S * (int)sizeof(T) + 2 * S * 4
                : ((AHEAD ? 40 : 32) * S + kCloseExtra) * (int)sizeof(T);
}

// FULL: the caller guarantees a tile inside the matrix with 16-byte aligned
// rows (no predecessors); cells move as 16-byte row pieces, no bounds tests.
template <typename T, int S, int TM, bool PRED, class A = Ar<T>, bool FULL = false>
__device__ __forceinline__ void closure_tile(T *__restrict__ d, int32_t *__restrict__ P, int n,
                                             int64_t ld, int64_t ldp, int base, char *smem,
                                             int32_t *flag = nullptr) {
    static_assert(!FULL || (!PRED && TM % 4 == 0), "full-tile form: no predecessors");
    constexpr int G = S / TM;
    T(*rowb)[S] = reinterpret_cast<T(*)[S]>(smem);
    T(*colb)[S] = reinterpret_cast<T(*)[S]>(smem + 2 * S * sizeof(T));
    int32_t(*rowp)[S] = reinterpret_cast<int32_t(*)[S]>(smem + 4 * S * sizeof(T));

    const int tx = threadIdx.x % G, ty = threadIdx.x / G;
    T c[TM][TM];
    int32_t pc[TM][TM];
    KeyCheck bad;
    if constexpr (FULL) {
#pragma unroll
        for (int r = 0; r < TM; ++r)
            row_load<T, TM, true>(c[r], d, base + ty * TM + r, base + tx * TM, n, ld, true,
                                  A::inf());
    } else {
#pragma unroll
        for (int r = 0; r < TM; ++r) {
            const int gi = base + ty * TM + r;
#pragma unroll
            for (int q = 0; q < TM; ++q) {
                const int gj = base + tx * TM + q;
                const bool ok = gi < n && gj < n;
                c[r][q] = ok ? d[(int64_t)gi * ld + gj] : A::inf();
                if constexpr (PRED) pc[r][q] = ok ? P[(int64_t)gi * ldp + gj] : kPredNone;
            }
        }
    }

    // steps k >= n only involve padded (isolated) vertices and change no real
    // cell, so the loop stops at the first register row past the last real k
    const int kreal = n - base < S ? n - base : S;
    const int kb_end = (kreal + TM - 1) / TM;
    for (int kb = 0; kb < kb_end; ++kb) {
#pragma unroll
        for (int r = 0; r < TM; ++r) {
            const int buf = (kb * TM + r) & 1;
            int oty = ty, otx = tx;
            if constexpr (FULL) {
                // opaque copies (no instruction is emitted): otherwise the
                // compiler threads the owner tests, equal across the TM
                // unrolled steps, and duplicates the step code per owner
                // class, which costs far more registers than the tile
                asm volatile("" : "+v"(oty), "+v"(otx));
            }
            if (oty == kb) {
#pragma unroll
                for (int q = 0; q < TM; ++q) {
                    rowb[buf][tx * TM + q] = settle<A>(c[r][q], bad);
                    if constexpr (PRED) rowp[buf][tx * TM + q] = pc[r][q];
                }
            }
            if (otx == kb) {
#pragma unroll
                for (int q = 0; q < TM; ++q) colb[buf][ty * TM + q] = settle<A>(c[q][r], bad);
            }
            __syncthreads();
            T rk[TM], ck[TM];
            int32_t pk[TM];
#pragma unroll
            for (int q = 0; q < TM; ++q) {
                rk[q] = rowb[buf][tx * TM + q];
                ck[q] = colb[buf][ty * TM + q];
                if constexpr (PRED) pk[q] = rowp[buf][tx * TM + q];
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TM; ++j) {
                    const T cand = A::add(ck[i], rk[j]);
                    if constexpr (PRED)
                        lex_update(c[i][j], pc[i][j], cand, pk[j]);
                    else
                        c[i][j] = A::min2(c[i][j], cand);
                }
            if constexpr (FULL) {
                // finish this step's updates here: left alone, the compiler
                // sinks them past later barriers and keeps every step's row
                // and column live
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TM; ++j) asm volatile("" : "+v"(c[i][j]));
            }
        }
    }

    if constexpr (A::kChecked) {
#pragma unroll
        for (int r = 0; r < TM; ++r)
#pragma unroll
            for (int q = 0; q < TM; ++q) c[r][q] = settle<A>(c[r][q], bad);
        raise_flag<A>(flag, bad);
    }
    if constexpr (FULL) {
        // addresses recomputed from opaque copies rather than kept live
        // through the k loop
        int sty = ty, stx = tx;
        asm volatile("" : "+v"(sty), "+v"(stx));
#pragma unroll
        for (int r = 0; r < TM; ++r)
            row_store<T, TM, true>(c[r], d, base + sty * TM + r, base + stx * TM, n, ld, true);
    } else {
#pragma unroll
        for (int r = 0; r < TM; ++r) {
            const int gi = base + ty * TM + r;
#pragma unroll
            for (int q = 0; q < TM; ++q) {
                const int gj = base + tx * TM + q;
                if (gi < n && gj < n) {
                    d[(int64_t)gi * ld + gj] = c[r][q];
                    if constexpr (PRED) P[(int64_t)gi * ldp + gj] = pc[r][q];
                }
            }
        }
    }
    // the LDS row/column buffers may be reused by the caller right away
    __syncthreads();
}

// Lane K (compile-time) of every 16-lane row, broadcast to that row.
template <int K, typename T>
__device__ __forceinline__ T row_lane(T v) {
    const int x = __builtin_bit_cast(int, v);
    return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(x, x, 0x150 + K, 0xf, 0xf, true));
}

// The 16-lane row Q (compile-time) of the wave, copied to all four rows: the
// halves exchanged, then the odd and even rows.
template <int Q, typename T>
__device__ __forceinline__ T wave_row(T v) {
    const unsigned x = __builtin_bit_cast(unsigned, v);
    const auto half = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    const unsigned u = half[Q >> 1];
    const auto row = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return __builtin_bit_cast(T, (unsigned)row[Q & 1]);
}

// Calls f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>).
template <class F, int... I>
__device__ __forceinline__ void static_for_seq(F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
    static_for_seq(f, std::make_integer_sequence<int, N>{});
}

// close8: the closure of an 8 x 8 block by one wave.  Lane 16 g + q holds D[r] =
// the block's entry (2 g + r, q % 8).  Rows are taken in pairs: rows 2 g and
// 2 g + 1 are spread to the whole wave by lane swaps (the two independent, so
// their latencies overlap), the second brought forward by the first, and then
// applied; column k is a row broadcast folded into the add.  The same sums as
// eight plain steps.
constexpr int kClosureK = 8;
template <class A, typename T>
__device__ __forceinline__ void close8(T (&D)[2]) {
    static_for<kClosureK / 2>([&](auto gc) {
        constexpr int g = decltype(gc)::value;
        const T r0 = wave_row<g>(D[0]);
        T r1 = wave_row<g>(D[1]);
        r1 = A::min2(r1, A::add(row_lane<2 * g>(r1), r0));
#pragma unroll
        for (int r = 0; r < 2; ++r) D[r] = A::min2(D[r], A::add(row_lane<2 * g>(D[r]), r0));
#pragma unroll
        for (int r = 0; r < 2; ++r) D[r] = A::min2(D[r], A::add(row_lane<2 * g + 1>(D[r]), r1));
    });
}

// x + sum over p < 8 of a_p x b_p in the semiring's (+, x), each of a and b
// given as two pieces of four.
template <class A, typename T, typename V4>
__device__ __forceinline__ T sum8(T x, V4 a0, V4 a1, V4 b0, V4 b1) {
    x = A::min3(x, A::add((T)a0[0], (T)b0[0]), A::add((T)a0[1], (T)b0[1]));
    x = A::min3(x, A::add((T)a0[2], (T)b0[2]), A::add((T)a0[3], (T)b0[3]));
    x = A::min3(x, A::add((T)a1[0], (T)b1[0]), A::add((T)a1[1], (T)b1[1]));
    return A::min3(x, A::add((T)a1[2], (T)b1[2]), A::add((T)a1[3], (T)b1[3]));
}

// closure_blocks: closure_tile in 8-vertex sub-blocks K instead of single
// steps (no predecessors, no range-checked keys).  For each K in turn, with
// D the closure of (K, K) and R the rows of K as they stand before it:
//   E_iq <- c_iq + sum over p in K of c_ip x D_pq  (the columns K of row i),
//   c_ij <- c_ij + sum over q in K of E_iq x R_qj  in the semiring's (+, x):
// a path through K enters it by one old entry, goes on inside K, and leaves
// it by one old entry (for i in K itself E is D).
// What bounds a closure is its serial chain, so the 8 steps of (K, K) run in
// one wave's registers, without LDS or barriers.
//   AHEAD false: the first wave closes (K, K) between two barriers.
//   AHEAD true: one more wave than the cells need does nothing else: while the
//     others update the cells by K, it forms the next sub-block's (K', K')
//     from E and R, the same sums as the owners of those cells, and closes
//     it.  One barrier per sub-block.
// Threads: (S / TM) x (S / TN) (+ 64), S / TN a multiple of 16.  A thread owns
// rows ty * TM .., and of every 4 (S / TN) columns the four at 4 tx (of all S
// the two at 2 tx where TN = 2).  A wave forms the E of its own rows, so no
// barrier lies between that and their use.  LDS, all but e in pairs used in
// turn (a buffer is written again only after a barrier that follows its last
// read): r, the rows of K (8 x S); c, the columns (S x 8); e, E (S x 8; over c
// where no wave reads ahead of its owner); dt, D by columns; t, the next
// (K', K') as its owners hold it.
// Every geometry and both forms take the same sums, so a tile's bits do not
// depend on them.
// Measured (one tile, launches back to back; in brackets two plain steps per
// barrier): 64-wide 8.1 us ahead (512 + 64 threads) and 12.4 us in 256 threads
// (14.7), 32-wide 3.7 us (5.2), 128-wide 29.1 us ahead (38.3).  16-vertex
// sub-blocks were slower (the closing wave's share grows with the square of
// their width): n=512 158 us the solve against 150.
constexpr int kCloseLd = kClosureK + 4;  // 16-byte pieces of D's columns in different banks
static_assert(kCloseExtra == 2 * kClosureK * kCloseLd + 2 * kClosureK * kClosureK, "dt, t");
template <typename T>
struct ClosureLds {
    T *r0, *r1, *c0, *c1;
    T *extra;  // kCloseExtra values: dt[2], t[2]
    T *e;      // 8 x S, AHEAD only
};

template <typename T, int S, int TM, int TN, class A, bool AHEAD>
__device__ __forceinline__ void closure_blocks(T *__restrict__ d, int n, int64_t ld, int base,
                                               const ClosureLds<T> &lds) {
    static_assert(!A::kChecked, "range-checked keys take closure_tile");
    constexpr int K = kClosureK, G = S / TN, NW = (S / TM) * (S / TN);
    constexpr int CW = TN < 4 ? TN : 4;           // piece of a row
    constexpr int WR = 64 / G * TM, M = WR / 8;   // rows of a wave; its E per lane
    constexpr int QS = AHEAD ? 4 : 2;             // of K per step of the update
    static_assert(G % 16 == 0 && TN % CW == 0 && K % TM == 0 && WR % 8 == 0, "geometry");
    typedef typename Vec4<T>::type V4;
    typedef T VW __attribute__((ext_vector_type(CW)));
    typedef T VP __attribute__((ext_vector_type(CW), aligned(4)));  // in the matrix
    typedef T VQ __attribute__((ext_vector_type(QS)));
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const bool ahead = AHEAD && wave == NW / 64;  // the wave that closes ahead
    const bool closer = AHEAD ? ahead : wave == 0;
    // its chain is the closure's: ahead of the waves it shares a SIMD with
    if (ahead) __builtin_amdgcn_s_setprio(3);
    int tx = threadIdx.x % G, ty = threadIdx.x / G;
    const int lane = threadIdx.x & 63, g = lane >> 4, cq = lane & 7;
    // a tile inside the matrix moves in 16-byte pieces (at any alignment)
    const bool full = base + S <= n;
    // elsewhere addresses are clamped into the matrix, so that every load is
    // issued before the first is waited for
    auto at = [&](int r, int q) {
        const T v = d[(int64_t)(r < n ? r : n - 1) * ld + (q < n ? q : n - 1)];
        return r < n && q < n ? v : A::inf();
    };
    T c[TM][TN], D[2];
    if (ahead) {
        // the first (K, K), straight from the matrix
#pragma unroll
        for (int r = 0; r < 2; ++r) D[r] = at(base + 2 * g + r, base + cq);
    } else if (full) {
#pragma unroll
        for (int r = 0; r < TM; ++r)
#pragma unroll
            for (int h = 0; h < TN / CW; ++h) {
                T v[CW];
                row_load<T, CW, false>(v, d, base + ty * TM + r, base + h * CW * G + tx * CW, n,
                                       ld, true, A::inf());
#pragma unroll
                for (int e = 0; e < CW; ++e) c[r][CW * h + e] = v[e];
            }
    } else if (n >= CW) {
        // whole pieces here too: one that reaches past the last column starts
        // earlier, and its values move up (element by element a 100-vertex
        // tile took 256 threads 4 us more)
#pragma unroll
        for (int r = 0; r < TM; ++r)
#pragma unroll
            for (int h = 0; h < TN / CW; ++h) {
                const int gi = base + ty * TM + r, gj = base + h * CW * G + tx * CW;
                const int from = gj < n - CW ? gj : n - CW;
                const T *src = d + (int64_t)(gi < n ? gi : n - 1) * ld + from;
                const VP x = *reinterpret_cast<const VP *>(src);
#pragma unroll
                for (int e = 0; e < CW; ++e) {
                    T v = x[e];
#pragma unroll
                    for (int m = e + 1; m < CW; ++m) v = gj - from == m - e ? (T)x[m] : v;
                    c[r][CW * h + e] = gi < n && gj + e < n ? v : A::inf();
                }
            }
    } else {
#pragma unroll
        for (int r = 0; r < TM; ++r)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                c[r][j] = at(base + ty * TM + r, base + j / CW * CW * G + tx * CW + j % CW);
    }
    auto put_closed = [&](T *dt) {
        close8<A>(D);
        dt[cq * kCloseLd + 2 * g] = D[0];
        dt[cq * kCloseLd + 2 * g + 1] = D[1];
    };
    if (ahead) put_closed(lds.extra);
    // sub-blocks past the last vertex hold padded (isolated) vertices only
    const int kreal = n - base < S ? n - base : S;
    const int blocks = (kreal + K - 1) / K;
#pragma unroll 1
    for (int s = 0; s < blocks; ++s) {
        T *R = s & 1 ? lds.r1 : lds.r0, *C = s & 1 ? lds.c1 : lds.c0;
        T *dt = lds.extra + (s & 1) * K * kCloseLd;
        T *next = lds.extra + 2 * K * kCloseLd + (s & 1) * K * K;
        if (!ahead) {
            // opaque (no instruction is emitted): LDS addresses are formed
            // anew in each sub-block instead of kept in registers
            asm volatile("" : "+v"(tx), "+v"(ty));
            const int rb = ty / (K / TM), row = (ty % (K / TM)) * TM;  // row block, row in it
            if (rb == s) {
#pragma unroll
                for (int r = 0; r < TM; ++r)
#pragma unroll
                    for (int h = 0; h < TN / CW; ++h) {
                        VW x;
#pragma unroll
                        for (int e = 0; e < CW; ++e) x[e] = c[r][CW * h + e];
                        *reinterpret_cast<VW *>(R + (row + r) * S + h * CW * G + tx * CW) = x;
                    }
            }
#pragma unroll
            for (int h = 0; h < TN / CW; ++h) {
                const int cb = h * (CW * G / K) + tx / (K / CW);  // column block
                const int col = CW * (tx % (K / CW));
                if (cb == s || (AHEAD && cb == s + 1 && rb == s + 1)) {
                    T *dst = cb == s ? C + ty * TM * K + col : next + row * K + col;
#pragma unroll
                    for (int r = 0; r < TM; ++r) {
                        VW x;
#pragma unroll
                        for (int e = 0; e < CW; ++e) x[e] = c[r][CW * h + e];
                        *reinterpret_cast<VW *>(dst + r * K) = x;
                    }
                }
            }
        }
        __syncthreads();
        if constexpr (!AHEAD) {
            if (closer) {
                D[0] = R[2 * g * S + s * K + cq];
                D[1] = R[(2 * g + 1) * S + s * K + cq];
                put_closed(dt);
            }
            __syncthreads();
        }
        if (ahead) {
            if (s + 1 < blocks) {
                const T *old = C + ((s + 1) * K + 2 * g) * K;  // rows 2 g, 2 g + 1 of K'
                const V4 d0 = *reinterpret_cast<const V4 *>(dt + cq * kCloseLd);
                const V4 d1 = *reinterpret_cast<const V4 *>(dt + cq * kCloseLd + 4);
                T E[2], b[K];
#pragma unroll
                for (int p = 0; p < K; ++p) b[p] = R[p * S + (s + 1) * K + cq];
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const V4 a0 = *reinterpret_cast<const V4 *>(old + r * K);
                    const V4 a1 = *reinterpret_cast<const V4 *>(old + r * K + 4);
                    E[r] = sum8<A, T>(old[r * K + cq], a0, a1, d0, d1);
                    D[r] = next[(2 * g + r) * K + cq];
                }
                static_for<K / 2>([&](auto pc) {
                    constexpr int p = 2 * decltype(pc)::value;
#pragma unroll
                    for (int r = 0; r < 2; ++r)
                        D[r] = A::min3(D[r], A::add(row_lane<p>(E[r]), b[p]),
                                       A::add(row_lane<p + 1>(E[r]), b[p + 1]));
                });
                put_closed(lds.extra + ((s + 1) & 1) * K * kCloseLd);
            }
        } else {
            // E of the wave's rows, a lane per column and eight rows at a time
            T *W = AHEAD ? lds.e : C;
            {
                const int row = wave * WR + (lane >> 3);
                const V4 d0 = *reinterpret_cast<const V4 *>(dt + cq * kCloseLd);
                const V4 d1 = *reinterpret_cast<const V4 *>(dt + cq * kCloseLd + 4);
                T E[M];
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    const T *old = C + (row + 8 * m) * K;
                    const V4 a0 = *reinterpret_cast<const V4 *>(old);
                    const V4 a1 = *reinterpret_cast<const V4 *>(old + 4);
                    E[m] = sum8<A, T>(old[cq], a0, a1, d0, d1);
                }
#pragma unroll
                for (int m = 0; m < M; ++m) W[(row + 8 * m) * K + cq] = E[m];
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            // QS of K a step; with AHEAD the next step's operands are read
            // before these are used (the scheduling barriers keep them there)
            T ea[2][QS][TM], rr[2][QS][TN];
            auto read = [&](int k, T(&x)[QS][TM], T(&y)[QS][TN]) {
#pragma unroll
                for (int r = 0; r < TM; ++r) {
                    const VQ v = *reinterpret_cast<const VQ *>(W + (ty * TM + r) * K + k);
#pragma unroll
                    for (int f = 0; f < QS; ++f) x[f][r] = v[f];
                }
#pragma unroll
                for (int f = 0; f < QS; ++f)
#pragma unroll
                    for (int h = 0; h < TN / CW; ++h) {
                        const VW v =
                            *reinterpret_cast<const VW *>(R + (k + f) * S + h * CW * G + tx * CW);
#pragma unroll
                        for (int e = 0; e < CW; ++e) y[f][CW * h + e] = v[e];
                    }
                __builtin_amdgcn_sched_barrier(0);
            };
            auto apply = [&](T(&x)[QS][TM], T(&y)[QS][TN]) {
#pragma unroll
                for (int f = 0; f < QS; f += 2)
#pragma unroll
                    for (int r = 0; r < TM; ++r)
#pragma unroll
                        for (int j = 0; j < TN; ++j)
                            c[r][j] = A::min3(c[r][j], A::add(x[f][r], y[f][j]),
                                              A::add(x[f + 1][r], y[f + 1][j]));
                __builtin_amdgcn_sched_barrier(0);
            };
            if constexpr (AHEAD) {
                static_assert(K == 2 * QS, "two steps");
                read(0, ea[0], rr[0]);
                read(QS, ea[1], rr[1]);
                apply(ea[0], rr[0]);
                apply(ea[1], rr[1]);
            } else {
#pragma unroll 1
                for (int k = 0; k < K; k += QS) {
                    read(k, ea[0], rr[0]);
                    apply(ea[0], rr[0]);
                }
            }
        }
    }
    // store addresses from opaque copies, not kept live through the steps
    int sty = ty, stx = tx;
    asm volatile("" : "+v"(sty), "+v"(stx));
    if (!ahead) {
#pragma unroll
        for (int r = 0; r < TM; ++r)
#pragma unroll
            for (int h = 0; h < TN / CW; ++h) {
                T v[CW];
#pragma unroll
                for (int e = 0; e < CW; ++e) v[e] = c[r][CW * h + e];
                const int gi = base + sty * TM + r, gj = base + h * CW * G + stx * CW;
                row_store<T, CW, false>(v, d, gi, gj, n, ld, full || (gi < n && gj + CW <= n));
            }
    }
    if (ahead) __builtin_amdgcn_s_setprio(0);
    // the LDS buffers may be reused by the caller right away
    __syncthreads();
}

// The diagonal closure in the form its arguments allow: in sub-blocks without
// predecessors or range-checked keys, else closure_tile.
template <typename T, int S, bool PRED, class A = Ar<T>>
constexpr bool closure_in_blocks() {
    return !PRED && !A::kChecked;
}
// Cells per thread (rows, columns) and threads of a diagonal launch's closure.
// AHEAD (one tile, latency): 512 threads and the wave that closes ahead, so
// that updating the cells takes no longer than its chain.  Many tiles
// (throughput): 256 threads.
#ifndef FW_CLOSURE64_TM
#define FW_CLOSURE64_TM 2
#define FW_CLOSURE64_TN 4
#endif
#ifndef FW_CLOSURE128_TM
#define FW_CLOSURE128_TM 4
#define FW_CLOSURE128_TN 8
#endif
template <typename T, int S, bool PRED, class A, bool AHEAD>
constexpr int closure_tm() {
    if (S == 32) return 2;
    if (!closure_in_blocks<T, S, PRED, A>()) return 4;
    return S == 64 ? (AHEAD ? FW_CLOSURE64_TM : 4) : (AHEAD ? FW_CLOSURE128_TM : 8);
}
template <typename T, int S, bool PRED, class A, bool AHEAD>
constexpr int closure_tn() {
    if (S == 32) return 2;
    if (!closure_in_blocks<T, S, PRED, A>()) return 4;
    return S == 64 ? (AHEAD ? FW_CLOSURE64_TN : 4) : (AHEAD ? FW_CLOSURE128_TN : 8);
}
template <typename T, int S, bool PRED, class A, bool AHEAD>
constexpr int closure_threads() {
    return (S / closure_tm<T, S, PRED, A, AHEAD>()) * (S / closure_tn<T, S, PRED, A, AHEAD>()) +
           (AHEAD && closure_in_blocks<T, S, PRED, A>() ? 64 : 0);
}
template <typename T, int S, int TM, bool PRED, class A = Ar<T>, int TN = TM, bool AHEAD = false>
__device__ __forceinline__ void closure_tile_any(T *__restrict__ d, int32_t *__restrict__ P, int n,
                                                 int64_t ld, int64_t ldp, int base, char *smem,
                                                 int32_t *flag = nullptr) {
    if constexpr (closure_in_blocks<T, S, PRED, A>()) {
        T *b = reinterpret_cast<T *>(smem);
        constexpr int W = kClosureK * S;
        const ClosureLds<T> lds = {b, b + W, b + 2 * W, b + 3 * W, b + 4 * W, b + 4 * W + kCloseExtra};
        closure_blocks<T, S, TM, TN, A, AHEAD>(d, n, ld, base, lds);
    } else {
        static_assert(TM == TN, "closure_tile has square sub-tiles");
        closure_tile<T, S, TM, PRED, A>(d, P, n, ld, ldp, base, smem, flag);
    }
}

// ---------------------------------------------------------------------------
// product_tile: register-tiled min-plus update of tile (bi, bj) over block b.
//
//   * each thread owns a TM x TN register sub-tile of C for the whole k-block
//     (section 4.1: the doubly dependent tile lives in registers);
//   * A and B are staged through LDS in k-slices of depth BK, double
//     buffered, the next slice prefetched from HBM into registers while the
//     current one is consumed (section 4.2's staged load);
//   * the A slice is stored k-major (transposed) so both operands are read
//     with 16-byte LDS loads;
//   * two k-steps are fused into one three-input minimum per cell,
//     c = min(c, a0 + b0, a1 + b1), legal because the tasks of a doubly
//     dependent tile may run in any order (section 3.2).
// ---------------------------------------------------------------------------
template <typename T, int S, int BK, bool PRED>
constexpr int product_smem_bytes() {
    return 4 * BK * S * (int)sizeof(T) + (PRED ? 2 * BK * S * 4 : 0);
}

template <typename T, int S, int BK, int TM, int TN, bool VEC, bool PRED, class A = Ar<T>>
__device__ __forceinline__ void product_tile(T *__restrict__ d, int32_t *__restrict__ P, int n,
                                             int64_t ld, int64_t ldp, int bi, int bj, int b,
                                             char *smem, int32_t *flag = nullptr) {
    constexpr int NT = (S / TM) * (S / TN);
    constexpr int GX = S / TN;       // threads along a tile row
    constexpr int EA = S * BK / NT;  // A-slice elements per thread
    constexpr int TPA = BK / EA;     // threads per A-slice row
    constexpr int EB = BK * S / NT;  // B-slice elements per thread
    constexpr int TPB = S / EB;      // threads per B-slice row
    constexpr int NS = S / BK;       // k-slices per block
    static_assert(EA * NT == S * BK && EB * NT == S * BK, "slice split");
    static_assert(TPA * EA == BK && TPB * EB == S, "slice rows");
    static_assert(!VEC || (EA % 4 == 0 && EB % 4 == 0 && TN % 4 == 0), "vector split");
    static_assert(BK % 2 == 0, "k-steps are fused in pairs");

    T(*As)[BK][S] = reinterpret_cast<T(*)[BK][S]>(smem);
    T(*Bs)[BK][S] = reinterpret_cast<T(*)[BK][S]>(smem + 2 * BK * S * sizeof(T));
    int32_t(*Bp)[BK][S] = reinterpret_cast<int32_t(*)[BK][S]>(smem + 4 * BK * S * sizeof(T));

    const int tid = threadIdx.x;
    const int tx = tid % GX, ty = tid / GX;
    const int row0 = bi * S, col0 = bj * S, k0 = b * S;
    const bool full = (row0 + S <= n) && (col0 + S <= n) && (k0 + S <= n);
    const T INF = A::inf();

    const int ia = tid / TPA, ka = (tid % TPA) * EA;
    const int kbr = tid / TPB, jb = (tid % TPB) * EB;

    T ra[EA], rb[EB];
    int32_t rp[PRED ? EB : 1];

    auto fetch = [&](int s) {
        row_load<T, EA, VEC>(ra, d, row0 + ia, k0 + s * BK + ka, n, ld, full, INF);
        row_load<T, EB, VEC>(rb, d, k0 + s * BK + kbr, col0 + jb, n, ld, full, INF);
        if constexpr (PRED)
            row_load<int32_t, EB, VEC>(rp, P, k0 + s * BK + kbr, col0 + jb, n, ldp, full,
                                       kPredNone);
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int e = 0; e < EA; ++e) As[buf][ka + e][ia] = ra[e];
#pragma unroll
        for (int e = 0; e < EB; ++e) Bs[buf][kbr][jb + e] = rb[e];
        if constexpr (PRED) {
#pragma unroll
            for (int e = 0; e < EB; ++e) Bp[buf][kbr][jb + e] = rp[e];
        }
    };

    // C first: the first slice's LDS store then waits for every load issued
    // so far, and the k loop never waits on a global load.
    T acc[TM][TN];
    int32_t accp[PRED ? TM : 1][PRED ? TN : 1];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        row_load<T, TN, VEC>(acc[i], d, row0 + ty * TM + i, col0 + tx * TN, n, ld, full, INF);
        if constexpr (PRED)
            row_load<int32_t, TN, VEC>(accp[i], P, row0 + ty * TM + i, col0 + tx * TN, n, ldp,
                                       full, kPredNone);
    }
    fetch(0);
    stash(0);
    __syncthreads();

    for (int s = 0; s < NS; ++s) {
        const int cur = s & 1;
        if (s + 1 < NS) fetch(s + 1);
        // one k-pair per iteration: unrolling further makes the compiler hoist
        // every LDS read of the slice and spill
#pragma unroll 1
        for (int kk = 0; kk < BK; kk += 2) {
            T a0[TM], a1[TM], b0[TN], b1[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                a0[i] = As[cur][kk][ty * TM + i];
                a1[i] = As[cur][kk + 1][ty * TM + i];
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                b0[j] = Bs[cur][kk][tx * TN + j];
                b1[j] = Bs[cur][kk + 1][tx * TN + j];
            }
            if constexpr (PRED) {
                int32_t p0[TN], p1[TN];
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    p0[j] = Bp[cur][kk][tx * TN + j];
                    p1[j] = Bp[cur][kk + 1][tx * TN + j];
                }
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        lex_update(acc[i][j], accp[i][j], A::add(a0[i], b0[j]), p0[j]);
                        lex_update(acc[i][j], accp[i][j], A::add(a1[i], b1[j]), p1[j]);
                    }
            } else {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = A::min3(acc[i][j], A::add(a0[i], b0[j]),
                                                A::add(a1[i], b1[j]));
            }
        }
        if (s + 1 < NS) stash(cur ^ 1);
        __syncthreads();
    }

    if constexpr (A::kChecked) {
        KeyCheck bad;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = settle<A>(acc[i][j], bad);
        raise_flag<A>(flag, bad);
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        row_store<T, TN, VEC>(acc[i], d, row0 + ty * TM + i, col0 + tx * TN, n, ld, full);
        if constexpr (PRED)
            row_store<int32_t, TN, VEC>(accp[i], P, row0 + ty * TM + i, col0 + tx * TN, n, ldp,
                                        full);
    }
}

// ---------------------------------------------------------------------------
// product_tile_whole: the 64 x 64 tile update of product_tile (no
// predecessors), bound by latency: the whole 64-deep k-block is staged at
// once, so one memory latency and one barrier replace four of each, and the k
// loop runs through with the next LDS reads in flight (88 registers, five
// waves per SIMD; product_tile's loop, made for six, waits on each).
// HALVES * 256 threads (any further ones only keep the barriers), 4 x 4 cells
// each; with two halves each takes 32 of the k, the second from top() on, and
// the first joins the two and stores.  LDS: A row-major, the 16-byte piece p
// of row r at p ^ (r / 4) (the 4 rows a wave reads at once fall in different
// banks), B as in memory.  Same candidates as product_tile, hence the same
// bits.  Measured (with the closure above): n=512 fp32 252 -> 144 us, n=1500
// 806 -> 607 us, and, at one half per tile and five workgroups per CU, n=4096
// 3.25 -> 2.62 ms: the read-ahead loop also beats product_tile's where the
// launch fills the GPU.
// ---------------------------------------------------------------------------
template <typename T>
constexpr int product_whole_smem_bytes() {
    return 2 * 64 * 64 * (int)sizeof(T);
}

template <typename T, int HALVES, bool VEC, class A = Ar<T>>
__device__ __forceinline__ void product_tile_whole(T *__restrict__ d, int n, int64_t ld, int bi,
                                                   int bj, int b, char *smem,
                                                   int32_t *flag = nullptr) {
    constexpr int S = 64, TM = 4, P = 4 / HALVES;  // P: 16-row groups a thread stages
    typedef typename Vec4<T>::type V4;
    using V4g = std::conditional_t<VEC, V4, typename Vec4u<T>::type>;  // in the matrix
    T *As = reinterpret_cast<T *>(smem), *Bs = As + S * S;
    const int half = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8);
    const int tid = threadIdx.x & 255, tx = tid & 15, ty = tid >> 4;
    const int64_t row0 = (int64_t)bi * S, col0 = (int64_t)bj * S, k0 = (int64_t)b * S;
    const bool full = (row0 + S <= n) && (col0 + S <= n) && (k0 + S <= n);
    V4 acc[TM];
    if (half < HALVES) {
        V4 ra[P], rb[P];
        const int sr = half * P * 16 + ty;  // first row staged
        if (full) {
#pragma unroll
            for (int i = 0; i < P; ++i) {
                ra[i] = *reinterpret_cast<const V4g *>(d + (row0 + sr + i * 16) * ld + k0 + tx * 4);
                rb[i] = *reinterpret_cast<const V4g *>(d + (k0 + sr + i * 16) * ld + col0 + tx * 4);
            }
            if (half == 0) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
                    acc[i] = *reinterpret_cast<const V4g *>(d + (row0 + ty * TM + i) * ld + col0 +
                                                            tx * 4);
            }
        } else {
            // addresses clamped into the matrix, so that every load is issued
            // before the first is waited for; what lies outside reads as absent
            auto at = [&](int64_t r, int64_t c) {
                const T v = d[(r < n ? r : n - 1) * ld + (c < n ? c : n - 1)];
                return r < n && c < n ? v : A::inf();
            };
#pragma unroll
            for (int i = 0; i < P; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    ra[i][e] = at(row0 + sr + i * 16, k0 + tx * 4 + e);
                    rb[i][e] = at(k0 + sr + i * 16, col0 + tx * 4 + e);
                }
            if (half == 0) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc[i][e] = at(row0 + ty * TM + i, col0 + tx * 4 + e);
            }
        }
        if (half != 0) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[i][e] = A::top();
        }
#pragma unroll
        for (int i = 0; i < P; ++i) {
            const int r = sr + i * 16;
            if constexpr (A::kChecked) {
#pragma unroll
                for (int e = 0; e < 4; ++e) ra[i][e] = first<A, T>(ra[i][e]);
            }
            *reinterpret_cast<V4 *>(As + r * S + (tx ^ (r >> 2)) * 4) = ra[i];
            *reinterpret_cast<V4 *>(Bs + r * S + tx * 4) = rb[i];
        }
    }
    __syncthreads();
    if (half < HALVES) {
        // four k a step, the next step's operands read before this one's use
        // (the scheduling barriers keep the reads there)
        constexpr int STEPS = S / HALVES / 4;
        const int s0 = half * STEPS;
        V4 a[2][TM], bb[2][4];
        auto read = [&](int s, V4(&x)[TM], V4(&y)[4]) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
                x[i] = *reinterpret_cast<const V4 *>(As + (ty * TM + i) * S + (s ^ ty) * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                y[e] = *reinterpret_cast<const V4 *>(Bs + (4 * s + e) * S + tx * 4);
            __builtin_amdgcn_sched_barrier(0);
        };
        auto apply = [&](V4(&x)[TM], V4(&y)[4]) {
#pragma unroll
            for (int e = 0; e < 4; e += 2) {
                const T b0[4] = {y[e][0], y[e][1], y[e][2], y[e][3]};
                const T b1[4] = {y[e + 1][0], y[e + 1][1], y[e + 1][2], y[e + 1][3]};
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    T c[4] = {acc[i][0], acc[i][1], acc[i][2], acc[i][3]};
                    update4<A>(c, (T)x[i][e], (T)x[i][e + 1], b0, b1);
#pragma unroll
                    for (int j = 0; j < TM; ++j) acc[i][j] = c[j];
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        read(s0, a[0], bb[0]);
#pragma unroll 1
        for (int t = 0; t < STEPS; t += 2) {
            read(s0 + t + 1, a[1], bb[1]);
            apply(a[0], bb[0]);
            // (the last step reads the block's first operands again)
            read(t + 2 < STEPS ? s0 + t + 2 : s0, a[0], bb[0]);
            apply(a[1], bb[1]);
        }
    }
    if constexpr (HALVES == 2) {
        __syncthreads();
        V4 *part = reinterpret_cast<V4 *>(smem);
        if (half == 1) {
#pragma unroll
            for (int i = 0; i < TM; ++i) part[i * 256 + tid] = acc[i];
        }
        __syncthreads();
        if (half == 0) {
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const V4 x = part[i * 256 + tid];
#pragma unroll
                for (int j = 0; j < TM; ++j) acc[i][j] = A::min2(acc[i][j], x[j]);
            }
        }
    }
    if (half != 0) return;
    if constexpr (A::kChecked) {
        KeyCheck bad;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j) acc[i][j] = settle<A>(acc[i][j], bad);
        raise_flag<A>(flag, bad);
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        T v[TM];
#pragma unroll
        for (int j = 0; j < TM; ++j) v[j] = acc[i][j];
        row_store<T, TM, VEC>(v, d, (int)row0 + ty * TM + i, (int)col0 + tx * TM, n, ld, full);
    }
}

// ---------------------------------------------------------------------------
// bulk_tile_dma: the 128 x 128 tile update of product_tile (no predecessors),
// the k-slices moved from global memory straight into LDS by gfx950's
// global->LDS loads instead of through registers.  A thread keeps only its
// 8 x 8 cells and one k-pair of operands, so four waves fit on a SIMD where the
// register-staged form fits three, and the copy costs no LDS store
// instructions.
//
// LDS layout (four separate arrays, so that the compiler's wait-count
// tracking can tell the buffer being filled from the one being read):
//   A slice: 128 rows x 16 k, row-major as in global memory; the four
//            16-byte chunks of row r are permuted, chunk c stored at
//            position c ^ ((r / 8) % 4), so that the 4 rows one wave reads
//            together fall in different banks;
//   B slice: 16 k x 128 columns, as in global memory.
// Three forms of the copy, the layout the same:
//   VEC, EDGE false: 16 bytes a lane (16-byte aligned rows), the tile and the
//            k-block inside the matrix;
//   VEC false:       4 bytes a lane, for rows of any alignment: 16 copies a
//            wave and slice instead of 4, which the slice's 1536 vector
//            instructions hide;
//   EDGE true:       4 bytes a lane, the tile or the k-block reaching past
//            the last vertex: every source is clamped to row and column
//            n - 1, the k loop stops at the last vertex, and cells outside
//            the matrix are neither loaded nor stored (they compute values
//            from clamped operands that go nowhere).
// Requirements on the caller: 256 threads; without EDGE ld < 2^25 (32-bit
// offsets within a tile).  Per cell the
// same candidates are formed, one add each, as in product_tile, hence the
// same bits.
// ---------------------------------------------------------------------------
typedef __attribute__((address_space(3))) void lds_void_t;

template <typename T>
struct Pair;
template <>
struct Pair<float> {
    using type = float2;
};
template <>
struct Pair<int32_t> {
    using type = int2;
};

// LDS of bulk_tile_dma (2048 values each), shared by the forms a kernel holds.
template <typename T>
struct BulkLds {
    T *A0, *A1, *B0, *B1;
};

// With the keyed policy the A slices come from `acol` (the stage's column
// panel with the hop fields cleared, 128 values per row, written by the
// panel launch), so the k loop adds without clearing.
template <typename T, bool VEC, bool EDGE, class A = Ar<T>>
__device__ __forceinline__ void bulk_tile_dma(const BulkLds<T> &lds, T *__restrict__ d, int n,
                                              int64_t ld, int bi, int bj, int b,
                                              int32_t *flag = nullptr,
                                              const T *__restrict__ acol = nullptr) {
    static_assert(sizeof(T) == 4, "32-bit values");
    constexpr int S = 128, BK = 16, TM = 8, NS = S / BK;
    static_assert(NS % 2 == 0, "slices alternate between two buffers");
    T *A0 = lds.A0, *A1 = lds.A1, *B0 = lds.B0, *B1 = lds.B1;
    using V4 = std::conditional_t<VEC, typename Vec4<T>::type, typename Vec4u<T>::type>;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tx = tid & 15, ty = tid >> 4;
    const int64_t row0 = (int64_t)bi * S, col0 = (int64_t)bj * S, k0 = (int64_t)b * S;

    // thread (tx, ty) owns rows 8*ty .. 8*ty + 7 and the two 4-column groups
    // starting at 4*tx and 64 + 4*tx: the 16 column groups a B read touches
    // are contiguous, so the read has no bank conflicts
    T acc[TM][2][4];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        T *row = d + (row0 + ty * TM + i) * ld + col0 + tx * 4;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if constexpr (EDGE) {
                const bool rok = row0 + ty * TM + i < n;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    acc[i][h][e] =
                        rok && col0 + tx * 4 + h * 64 + e < n ? row[h * 64 + e] : A::inf();
            } else {
                const V4 x = *reinterpret_cast<const V4 *>(row + h * 64);
                acc[i][h][0] = x[0];
                acc[i][h][1] = x[1];
                acc[i][h][2] = x[2];
                acc[i][h][3] = x[3];
            }
        }
    }

    // Copy sources: wave-uniform bases plus 32-bit per-lane offsets.  A wave
    // copies A rows 32*wave .. + 31 and B k-rows 4*wave .. + 3 of each slice.
    const int64_t lda = A::kChecked ? (int64_t)S : ld;
    const T *a_tile = A::kChecked ? acol + row0 * S : d + row0 * ld + k0;
    const T *b_tile = d + k0 * ld + col0;
    const T *a_base = a_tile + wave * 32 * lda, *b_base = b_tile + wave * 4 * ld;
    const int ar = wave * 32 + (lane >> 2);
    const uint32_t a_off0 = (uint32_t)((lane >> 2) * lda) + (((lane & 3) ^ ((ar >> 3) & 3)) << 2);
    const uint32_t a_off1 =
        (uint32_t)(((lane >> 2) + 16) * lda) + (((lane & 3) ^ (((ar + 16) >> 3) & 3)) << 2);
    const uint32_t b_off0 = (uint32_t)((lane >> 5) * ld) + ((lane & 31) << 2);
    const uint32_t b_off1 = b_off0 + (uint32_t)(2 * ld);
    const uint32_t a_lane = (uint32_t)((lane >> 4) * lda) + (lane & 3);
    const int last_r = (int)(n - 1 - row0), last_c = (int)(n - 1 - col0), last_k = (int)(n - 1 - k0);
    auto issue = [&](int s, T *Ad, T *Bd) {
        T *a = Ad + wave * 32 * BK;
        T *bb = Bd + wave * 4 * S;
        if constexpr (EDGE) {
            // addresses formed anew for each slice from an opaque copy of the
            // lane (no instruction is emitted), not kept through the k loop
            int el = lane;
            asm volatile("" : "+v"(el));
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                // lane: row el / 16 of four, position el % 16 of the row
                const int r = min(wave * 32 + 4 * i + (el >> 4), last_r);
                const int c = ((((el >> 2) & 3) ^ (i >> 1)) << 2) + (el & 3);
                __builtin_amdgcn_global_load_lds(a_tile + r * lda + min(s * BK + c, last_k),
                                                 (lds_void_t *)(a + i * 64), 4, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int k = min(s * BK + wave * 4 + (i >> 1), last_k);
                __builtin_amdgcn_global_load_lds(
                    b_tile + (int64_t)k * ld + min((i & 1) * 64 + el, last_c),
                    (lds_void_t *)(bb + i * 64), 4, 0, 0);
            }
        } else if constexpr (VEC) {
            const T *as = a_base + s * BK;
            const T *bs = b_base + (int64_t)s * BK * ld;
            __builtin_amdgcn_global_load_lds(as + a_off0, (lds_void_t *)a, 16, 0, 0);
            __builtin_amdgcn_global_load_lds(as + a_off1, (lds_void_t *)(a + 16 * BK), 16, 0, 0);
            __builtin_amdgcn_global_load_lds(bs + b_off0, (lds_void_t *)bb, 16, 0, 0);
            __builtin_amdgcn_global_load_lds(bs + b_off1, (lds_void_t *)(bb + 2 * S), 16, 0, 0);
        } else {
            const T *as = a_base + s * BK;
            const T *bs = b_base + (int64_t)s * BK * ld;
#pragma unroll
            for (int i = 0; i < 8; ++i)
                __builtin_amdgcn_global_load_lds(
                    as + 4 * i * lda + (a_lane + ((((lane >> 2) & 3) ^ (i >> 1)) << 2)),
                    (lds_void_t *)(a + i * 64), 4, 0, 0);
#pragma unroll
            for (int i = 0; i < 8; ++i)
                __builtin_amdgcn_global_load_lds(bs + (i >> 1) * ld + (i & 1) * 64 + lane,
                                                 (lds_void_t *)(bb + i * 64), 4, 0, 0);
        }
    };
    // EDGE: a wave whose 32 rows all lie beyond the matrix skips the
    // arithmetic (it still copies its share and meets every barrier)
    const bool idle = EDGE && wave * 32 > last_r;
    // kl: the slice's k inside the matrix
    auto compute = [&](const T *Ab, const T *Bb, int kl) {
        if (EDGE && idle) return;
        const int kpairs = EDGE ? kl & ~1 : BK;
        // one k-pair per iteration (see product_tile)
#pragma unroll 1
        for (int kk = 0; kk < kpairs; kk += 2) {
            const int aoff = ty * (TM * BK) + (((kk >> 2) ^ (ty & 3)) << 2) + (kk & 3);
            T a0[TM], a1[TM], b0[TM], b1[TM];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const typename Pair<T>::type v =
                    *reinterpret_cast<const typename Pair<T>::type *>(Ab + aoff + i * BK);
                a0[i] = v.x;
                a1[i] = v.y;
            }
#pragma unroll
            for (int j = 0; j < TM; ++j) {
                const int c = (j >> 2) * 64 + tx * 4 + (j & 3);
                b0[j] = Bb[kk * S + c];
                b1[j] = Bb[(kk + 1) * S + c];
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    update4<A>(acc[i][h], a0[i], a1[i], &b0[4 * h], &b1[4 * h]);
        }
        if (EDGE && (kl & 1)) {  // the last k alone
            const int kk = kl - 1;
            const int aoff = ty * (TM * BK) + (((kk >> 2) ^ (ty & 3)) << 2) + (kk & 3);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TM; ++j)
                    acc[i][j >> 2][j & 3] =
                        A::min2(acc[i][j >> 2][j & 3],
                                add_first<A>(Ab[aoff + i * BK],
                                             Bb[kk * S + (j >> 2) * 64 + tx * 4 + (j & 3)]));
        }
    };
    auto slice_k = [&](int s) { return EDGE ? max(0, min(BK, last_k + 1 - s * BK)) : BK; };

    // vmcnt(0): this wave's copies (and its C loads) have landed; the
    // barrier after it makes every wave's copies visible and guarantees that
    // every wave is done reading the buffer the next copy overwrites
    constexpr int kWaitVm0 = 0x0F70;
    issue(0, A0, B0);
#pragma unroll 1
    for (int s = 0; s < NS; s += 2) {
        __builtin_amdgcn_s_waitcnt(kWaitVm0);
        __syncthreads();
        issue(s + 1, A1, B1);
        compute(A0, B0, slice_k(s));
        __builtin_amdgcn_s_waitcnt(kWaitVm0);
        __syncthreads();
        if (s + 2 < NS) issue(s + 2, A0, B0);
        compute(A1, B1, slice_k(s + 1));
    }

    // store addresses recomputed from opaque copies of the thread ids (no
    // instruction is emitted): the load addresses would otherwise stay live
    // through the k loop, 16 VGPRs
    int stx = tx, sty = ty;
    asm volatile("" : "+v"(stx), "+v"(sty));
    if constexpr (A::kChecked) {
        KeyCheck bad;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j) {
                // a cell outside the matrix checks nothing
                T &c = acc[i][j >> 2][j & 3];
                if (EDGE && (row0 + sty * TM + i >= n ||
                             col0 + stx * 4 + (j >> 2) * 64 + (j & 3) >= n))
                    c = A::inf();
                c = settle<A>(c, bad);
            }
        raise_flag<A>(flag, bad);
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        T *row = d + (row0 + sty * TM + i) * ld + col0 + stx * 4;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if constexpr (EDGE) {
                const bool rok = row0 + sty * TM + i < n;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (rok && col0 + stx * 4 + h * 64 + e < n) row[h * 64 + e] = acc[i][h][e];
            } else {
                V4 x;
                x[0] = acc[i][h][0];
                x[1] = acc[i][h][1];
                x[2] = acc[i][h][2];
                x[3] = acc[i][h][3];
                *reinterpret_cast<V4 *>(row + h * 64) = x;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// product_tile_key: product_tile with predecessors for int32 matrices, the
// (distance, last hop) pair of a cell held as one 64-bit key, distance in the
// high word and last hop (>= 0) in the low word.  Compared as signed 64-bit
// integers, keys order exactly as lex_update orders pairs (shorter first,
// then smaller last hop), so one compare and two selects replace it.  The
// candidate through k is B's key plus the A distance shifted into the high
// word -- one 64-bit shift-and-add; the low word (B's last hop) is unchanged
// because the added value's low word is zero, and the high word is the int32
// sum the unkeyed form computes.  Same candidates, same order rule, hence
// the same distances and predecessors.  B is staged in LDS as keys.
// ---------------------------------------------------------------------------
template <int S, int BK>
constexpr int product_key_smem_bytes() {
    return 2 * BK * S * 4 + 2 * BK * S * 8;
}

__device__ __forceinline__ uint64_t make_key(int32_t d, int32_t p) {
    return ((uint64_t)(uint32_t)d << 32) | (uint32_t)p;
}

template <int S, int BK, int TM, int TN, bool VEC>
__device__ __forceinline__ void product_tile_key(int32_t *__restrict__ d, int32_t *__restrict__ P,
                                                 int n, int64_t ld, int64_t ldp, int bi, int bj,
                                                 int b, char *smem) {
    using T = int32_t;
    constexpr int NT = (S / TM) * (S / TN);
    constexpr int GX = S / TN;
    constexpr int EA = S * BK / NT, TPA = BK / EA;
    constexpr int EB = BK * S / NT, TPB = S / EB;
    constexpr int NS = S / BK;
    static_assert(EA * NT == S * BK && EB * NT == S * BK, "slice split");
    static_assert(TPA * EA == BK && TPB * EB == S, "slice rows");
    static_assert(!VEC || (EA % 4 == 0 && EB % 4 == 0 && TN % 4 == 0), "vector split");
    static_assert(BK % 2 == 0, "k-steps are taken in pairs");

    T(*As)[BK][S] = reinterpret_cast<T(*)[BK][S]>(smem);
    uint64_t(*Bk)[BK][S] = reinterpret_cast<uint64_t(*)[BK][S]>(smem + 2 * BK * S * sizeof(T));

    const int tid = threadIdx.x;
    const int tx = tid % GX, ty = tid / GX;
    const int row0 = bi * S, col0 = bj * S, k0 = b * S;
    const bool full = (row0 + S <= n) && (col0 + S <= n) && (k0 + S <= n);
    const int ia = tid / TPA, ka = (tid % TPA) * EA;
    const int kbr = tid / TPB, jb = (tid % TPB) * EB;

    T ra[EA], rb[EB];
    int32_t rp[EB];
    auto fetch = [&](int s) {
        row_load<T, EA, VEC>(ra, d, row0 + ia, k0 + s * BK + ka, n, ld, full, kI32Inf);
        row_load<T, EB, VEC>(rb, d, k0 + s * BK + kbr, col0 + jb, n, ld, full, kI32Inf);
        row_load<int32_t, EB, VEC>(rp, P, k0 + s * BK + kbr, col0 + jb, n, ldp, full, kPredNone);
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int e = 0; e < EA; ++e) As[buf][ka + e][ia] = ra[e];
#pragma unroll
        for (int e = 0; e < EB; ++e) Bk[buf][kbr][jb + e] = make_key(rb[e], rp[e]);
    };

    uint64_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        T cd[TN];
        int32_t cp[TN];
        row_load<T, TN, VEC>(cd, d, row0 + ty * TM + i, col0 + tx * TN, n, ld, full, kI32Inf);
        row_load<int32_t, TN, VEC>(cp, P, row0 + ty * TM + i, col0 + tx * TN, n, ldp, full,
                                   kPredNone);
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = make_key(cd[j], cp[j]);
    }
    fetch(0);
    stash(0);
    __syncthreads();

    for (int s = 0; s < NS; ++s) {
        const int cur = s & 1;
        if (s + 1 < NS) fetch(s + 1);
#pragma unroll 1
        for (int kk = 0; kk < BK; kk += 2) {
            T a0[TM], a1[TM];
            uint64_t b0[TN], b1[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                a0[i] = As[cur][kk][ty * TM + i];
                a1[i] = As[cur][kk + 1][ty * TM + i];
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                b0[j] = Bk[cur][kk][tx * TN + j];
                b1[j] = Bk[cur][kk + 1][tx * TN + j];
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const uint64_t c0 = ((uint64_t)(uint32_t)a0[i] << 32) + b0[j];
                    const uint64_t c1 = ((uint64_t)(uint32_t)a1[i] << 32) + b1[j];
                    uint64_t v = acc[i][j];
                    v = (int64_t)c0 < (int64_t)v ? c0 : v;
                    v = (int64_t)c1 < (int64_t)v ? c1 : v;
                    acc[i][j] = v;
                }
        }
        if (s + 1 < NS) stash(cur ^ 1);
        __syncthreads();
    }

#pragma unroll
    for (int i = 0; i < TM; ++i) {
        T cd[TN];
        int32_t cp[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            cd[j] = (int32_t)(uint32_t)(acc[i][j] >> 32);
            cp[j] = (int32_t)(uint32_t)acc[i][j];
        }
        row_store<T, TN, VEC>(cd, d, row0 + ty * TM + i, col0 + tx * TN, n, ld, full);
        row_store<int32_t, TN, VEC>(cp, P, row0 + ty * TM + i, col0 + tx * TN, n, ldp, full);
    }
}

// ---------------------------------------------------------------------------
// strip_tile: the panel update of product_tile on one strip of a 128-wide
// panel tile, R rows x CW columns (128 x 32 or 32 x 128) with the full k-block,
// so that a stage's 2(nb-1) panel tiles give four times as many workgroups
// (one 128 x 128 tile per workgroup leaves a CU with a single wave per SIMD).  A
// row-panel tile is cut into column strips and a column-panel tile into row
// strips: the panel operand a strip reads (its own columns of B, or its own
// rows of A) is then exactly the part it writes, and no two workgroups touch
// the same cell.
// A few hundred workgroups leave this launch bound by latency, so it goes as
// product_tile_whole: the whole k-block staged at once (80 KB, two workgroups
// per CU), 512 threads, each half taking 64 of the k for 4 x 4 cells a thread,
// LDS reads one step ahead.  Same per-cell candidates as product_tile, hence
// the same bits.  Measured, fp32: 14.8 us a launch at n=6001 and 21.8 at n=16384
// (16-deep slices in 256 threads: 19.3 and 27.1).
// ---------------------------------------------------------------------------
constexpr int kStripK = 128, kStripW = 32, kStripThreads = 512;
template <typename T>
constexpr int strip_smem_bytes() {
    return kStripK * (kStripK + kStripW) * (int)sizeof(T);
}

// With the keyed policy and `acol` non-NULL (a column-panel strip of a 128-
// wide sweep), the strip also writes its cells with the hop field cleared to
// acol (row r, column c - col0 at acol[r * CW + c - col0]): the bulk's A
// operand, ready to be added.
template <typename T, int R, int CW, bool VEC, class A = Ar<T>>
__device__ __forceinline__ void strip_tile(T *__restrict__ d, int n, int64_t ld, int row0,
                                           int col0, int k0, char *smem,
                                           int32_t *flag = nullptr, T *acol = nullptr) {
    constexpr int K = kStripK, TM = 4, GX = CW / 4, NT = kStripThreads;
    constexpr int PA = R * (K / 4) / NT, PB = K * GX / NT;  // 16-byte pieces a thread stages
    static_assert((R / TM) * GX * 2 == NT && PA >= 1 && PB >= 1, "geometry");
    typedef typename Vec4<T>::type V4;
    using V4g = std::conditional_t<VEC, V4, typename Vec4u<T>::type>;  // in the matrix
    T *As = reinterpret_cast<T *>(smem), *Bs = As + R * K;
    const int tid = threadIdx.x, half = __builtin_amdgcn_readfirstlane(tid >> 8);
    const int cell = tid & 255, tx = cell % GX, ty = cell / GX;
    const bool full = (row0 + R <= n) && (col0 + CW <= n) && (k0 + K <= n);
    auto at = [&](int64_t r, int64_t c) {
        const T v = d[(r < n ? r : n - 1) * ld + (c < n ? c : n - 1)];
        return r < n && c < n ? v : A::inf();
    };
    // piece p of A: k 4 (p % 32) .. of row p / 32, stored at piece ^ (row / 4);
    // of B: columns 4 (p % GX) .. of k-row p / GX
    V4 ra[PA], rb[PB], acc[TM];
    if (full) {
#pragma unroll
        for (int i = 0; i < PA; ++i) {
            const int p = tid + i * NT;
            ra[i] = *reinterpret_cast<const V4g *>(d + (int64_t)(row0 + p / (K / 4)) * ld + k0 +
                                                   p % (K / 4) * 4);
        }
#pragma unroll
        for (int i = 0; i < PB; ++i) {
            const int p = tid + i * NT;
            rb[i] = *reinterpret_cast<const V4g *>(d + (int64_t)(k0 + p / GX) * ld + col0 +
                                                   p % GX * 4);
        }
        if (half == 0) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
                acc[i] = *reinterpret_cast<const V4g *>(d + (int64_t)(row0 + ty * TM + i) * ld +
                                                        col0 + tx * 4);
        }
    } else {
        // clamped addresses: every load is issued before the first is used
#pragma unroll
        for (int i = 0; i < PA; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int p = tid + i * NT;
                ra[i][e] = at(row0 + p / (K / 4), k0 + p % (K / 4) * 4 + e);
            }
#pragma unroll
        for (int i = 0; i < PB; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int p = tid + i * NT;
                rb[i][e] = at(k0 + p / GX, col0 + p % GX * 4 + e);
            }
        if (half == 0) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[i][e] = at(row0 + ty * TM + i, col0 + tx * 4 + e);
        }
    }
    if (half != 0) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][e] = A::top();
    }
#pragma unroll
    for (int i = 0; i < PA; ++i) {
        const int p = tid + i * NT, r = p / (K / 4), q = p % (K / 4);
        V4 x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = first<A, T>(ra[i][e]);
        *reinterpret_cast<V4 *>(As + r * K + (q ^ ((r >> 2) & 31)) * 4) = x;
    }
#pragma unroll
    for (int i = 0; i < PB; ++i) *reinterpret_cast<V4 *>(Bs + (tid + i * NT) * 4) = rb[i];
    __syncthreads();
    {
        constexpr int STEPS = K / 2 / 4;
        const int s0 = half * STEPS;
        V4 a[2][TM], bb[2][4];
        auto read = [&](int s, V4(&x)[TM], V4(&y)[4]) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
                x[i] = *reinterpret_cast<const V4 *>(As + (ty * TM + i) * K + (s ^ ty) * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                y[e] = *reinterpret_cast<const V4 *>(Bs + (4 * s + e) * CW + tx * 4);
            __builtin_amdgcn_sched_barrier(0);
        };
        auto apply = [&](V4(&x)[TM], V4(&y)[4]) {
#pragma unroll
            for (int e = 0; e < 4; e += 2) {
                const T b0[4] = {y[e][0], y[e][1], y[e][2], y[e][3]};
                const T b1[4] = {y[e + 1][0], y[e + 1][1], y[e + 1][2], y[e + 1][3]};
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    T c[4] = {acc[i][0], acc[i][1], acc[i][2], acc[i][3]};
                    update4<A>(c, (T)x[i][e], (T)x[i][e + 1], b0, b1);
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc[i][j] = c[j];
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        read(s0, a[0], bb[0]);
#pragma unroll 1
        for (int t = 0; t < STEPS; t += 2) {
            read(s0 + t + 1, a[1], bb[1]);
            apply(a[0], bb[0]);
            // (the last step reads the half's first operands again)
            read(t + 2 < STEPS ? s0 + t + 2 : s0, a[0], bb[0]);
            apply(a[1], bb[1]);
        }
    }
    __syncthreads();
    V4 *part = reinterpret_cast<V4 *>(smem);
    if (half == 1) {
#pragma unroll
        for (int i = 0; i < TM; ++i) part[i * 256 + cell] = acc[i];
    }
    __syncthreads();
    if (half == 1) return;
    T c[TM][4];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const V4 x = part[i * 256 + cell];
#pragma unroll
        for (int j = 0; j < 4; ++j) c[i][j] = A::min2(acc[i][j], x[j]);
    }
    if constexpr (A::kChecked) {
        KeyCheck bad;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) c[i][j] = settle<A>(c[i][j], bad);
        raise_flag<A>(flag, bad);
        if (acol) {
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int r = row0 + ty * TM + i;
                T *dst = acol + (int64_t)r * CW + tx * 4;
                if (full) {
                    V4 x;
#pragma unroll
                    for (int j = 0; j < 4; ++j) x[j] = A::clear_hop(c[i][j]);
                    *reinterpret_cast<V4 *>(dst) = x;
                } else if (r < n) {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (col0 + tx * 4 + j < n) dst[j] = A::clear_hop(c[i][j]);
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
        row_store<T, 4, VEC>(c[i], d, row0 + ty * TM + i, col0 + tx * 4, n, ld, full);
}

// Tile coordinates of the stage-b panel tile number idx (0 <= idx < 2m,
// m = nb - 1): the row panel (b, j != b) first, then the column panel.
__device__ __forceinline__ void panel_coords(int idx, int b, int m, int &bi, int &bj) {
    if (idx < m) {
        bi = b;
        bj = idx < b ? idx : idx + 1;
    } else {
        idx -= m;
        bi = idx < b ? idx : idx + 1;
        bj = b;
    }
}

// Tile coordinates of the stage-b bulk tile number idx (0 <= idx < m^2).
__device__ __forceinline__ void bulk_coords(int idx, int b, int m, int &bi, int &bj) {
    const int q = idx / m, r = idx - q * m;
    bi = q < b ? q : q + 1;
    bj = r < b ? r : r + 1;
}

}  // namespace fw

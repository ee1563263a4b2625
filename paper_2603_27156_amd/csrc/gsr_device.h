// Device-side building blocks for gfx950 (wave64): storage conversion, sub-wave reductions,
// the exact top-k select of the GS operator, neighbour gathers and 16x16x4 float32 MFMA tiles.
//
// Three thread layouts appear.  "Row layout" (operators exposed on their own, first pass over split
// rows, head): a row of a group has DG = 32 or 64 columns and lane c of a (sub-)wave owns column
// c; with DG = 64 a wave holds one row, with DG = 32 two (lanes 0..31 and 32..63, `sub` = lane /
// DG).  "Tile register layout" (layer kernels: what the MFMA leaves in the accumulators for a
// 16-row tile; four rows per memory instruction) and "quarter layout" (GS of a 16-row tile: lane
// = (row, quarter of its columns)) are described where they are introduced below.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>
#include <utility>

namespace gsr {

struct bf16_t {
    uint16_t bits;
};

__device__ __forceinline__ float to_float(float v) { return v; }
__device__ __forceinline__ float to_float(bf16_t v) { return __uint_as_float((uint32_t)v.bits << 16); }

template <typename T>
__device__ __forceinline__ T from_float(float v);
template <>
__device__ __forceinline__ float from_float<float>(float v) { return v; }
template <>
__device__ __forceinline__ bf16_t from_float<bf16_t>(float v) {
    // round to nearest even; inputs are finite by contract
    uint32_t b = __float_as_uint(v);
    b = b + 0x7FFFu + ((b >> 16) & 1u);
    bf16_t r;
    r.bits = (uint16_t)(b >> 16);
    return r;
}

// value as it will read back after a store of type T
template <typename T>
__device__ __forceinline__ float stored(float v) { return to_float(from_float<T>(v)); }

template <int DG>
struct MaskOf;
template <>
struct MaskOf<32> { using type = uint32_t; };
template <>
struct MaskOf<64> { using type = uint64_t; };

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

// Orders this wave's LDS traffic for the compiler.  The hardware executes the LDS instructions of
// one wave in issue order, so a write followed by another lane's read needs no wait, only the
// guarantee that the compiler keeps the two in program order.
__device__ __forceinline__ void wave_sync() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// bits of a wave-wide ballot that belong to this lane's row
template <int DG>
__device__ __forceinline__ typename MaskOf<DG>::type sub_bits(uint64_t m, int sub) {
    if constexpr (DG == 64) return m;
    else return (uint32_t)(m >> (32 * sub));
}

template <int DG>
__device__ __forceinline__ int popc(typename MaskOf<DG>::type m) {
    if constexpr (DG == 64) return __popcll(m);
    else return __popc(m);
}

template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
    const int moved = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true);
    return v + __builtin_bit_cast(float, moved);
}

__device__ __forceinline__ float read_lane(float v, int l) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}

// Sum over the DG lanes of this lane's row, the same value (same association) in every lane:
// butterfly inside each group of 16 lanes with DPP (xor 1, xor 2, half-row mirror, row mirror),
// then the four group sums are combined as (g0 + g1) + (g2 + g3).
template <int DG>
__device__ __forceinline__ float sub_sum(float v) {
    v = dpp_add<0xB1>(v);    // quad_perm [1,0,3,2]
    v = dpp_add<0x4E>(v);    // quad_perm [2,3,0,1]
    v = dpp_add<0x141>(v);   // row_half_mirror
    v = dpp_add<0x140>(v);   // row_mirror
    const float lo = read_lane(v, 0) + read_lane(v, 16), hi = read_lane(v, 32) + read_lane(v, 48);
    if constexpr (DG == 64) return lo + hi;
    else return (threadIdx.x & 32) ? hi : lo;
}

// ---- "quarter layout": lane = (row r = lane % 16, quarter q = lane / 16) ------------------------
// The four lanes r, r+16, r+32, r+48 share a row of a 16-row tile, each holding a quarter of its
// columns.  v_permlane16_swap exchanges the odd 16-lane rows of its first operand with the even
// rows of its second, v_permlane32_swap the upper half of the first with the lower half of the
// second; fed the same register twice they hand every lane its partner quarters.

// q[i] = v of the lane of quarter i in this lane's row
__device__ __forceinline__ void quarter_all(uint32_t v, uint32_t (&q)[4]) {
    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);        // quarters {0|2}, {1|3} of my half
    const auto b = __builtin_amdgcn_permlane32_swap(a[0], a[0], false, false);  // quarter 0, quarter 2
    const auto d = __builtin_amdgcn_permlane32_swap(a[1], a[1], false, false);  // quarter 1, quarter 3
    q[0] = b[0]; q[1] = d[0]; q[2] = b[1]; q[3] = d[1];
}
__device__ __forceinline__ uint32_t quarter_sum(uint32_t v) {
    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    const uint32_t s = a[0] + a[1];
    const auto b = __builtin_amdgcn_permlane32_swap(s, s, false, false);
    return b[0] + b[1];
}
__device__ __forceinline__ uint32_t quarter_max(uint32_t v) {
    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    const uint32_t s = max(a[0], a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(s, s, false, false);
    return max(b[0], b[1]);
}
// (q0 + q1) + (q2 + q3), the same value in the four lanes
__device__ __forceinline__ float quarter_sum(float v) {
    const uint32_t u = __float_as_uint(v);
    const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const float s = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const uint32_t su = __float_as_uint(s);
    const auto b = __builtin_amdgcn_permlane32_swap(su, su, false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

__device__ __forceinline__ float quarter_fmax(float v) {
    const uint32_t u = __float_as_uint(v);
    const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const float s = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const uint32_t su = __float_as_uint(s);
    const auto b = __builtin_amdgcn_permlane32_swap(su, su, false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float quarter_fmin(float v) { return -quarter_fmax(-v); }

// ---- GS: exact top-k of a row ----------------------------------------------------------------
// The Group-Sparse operator of Section 4.1 of the paper keeps, per row, the k largest entries by
// signed value.  The row's k-th largest value is found by bisection on an order-preserving
// 32-bit image of the floats, one bit per round: count = popcount(ballot(key >= candidate)).
// As soon as a candidate splits off exactly k entries the search is over.  Ties at the
// threshold go to the lowest columns, -0 equals +0.  Row layout (lane c of a (sub-)wave owns
// column c), R rows at once: the independent bisections are interleaved so that their dependent
// ballot -> popcount -> compare chains overlap.  sel[r]: this lane's column of row r is kept;
// mask_out[r]: the row's column bit mask.  With one row per wave (DG = 64) every quantity of the
// search is wave-uniform and lives in scalar registers.  (The layer kernels select in the
// quarter layout instead, 16 rows at once in vector registers.)
template <int DG, int R>
__device__ __forceinline__ void topk_select_multi(const float (&x)[R], int k, int c, int sub, bool (&sel)[R],
                                                  typename MaskOf<DG>::type (&mask_out)[R]) {
    using M = typename MaskOf<DG>::type;
    uint32_t key[R], thr[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        uint32_t u = __float_as_uint(x[r]);
        if (u == 0x80000000u) u = 0u;
        key[r] = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
        thr[r] = 0u;
    }
    if constexpr (DG == 64) {
        // Interval bisection with a data-driven start.  Invariant per row: at least k keys are
        // >= lo and fewer than k are >= hi.  hi starts just above the row maximum; lo starts 4
        // binades below it (16x in value), which holds the k-th largest of almost every row, and
        // falls back to 0 when a count says it does not.  A row is closed as soon as a candidate
        // splits off exactly k keys.
        uint32_t lo[R], hi[R];
        uint32_t open = 0u;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            uint32_t m = key[r];
            m = max(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0xB1, 0xF, 0xF, true));
            m = max(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x4E, 0xF, 0xF, true));
            m = max(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x141, 0xF, 0xF, true));
            m = max(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x140, 0xF, 0xF, true));
            const uint32_t m01 = max((uint32_t)__builtin_amdgcn_readlane((int)m, 0), (uint32_t)__builtin_amdgcn_readlane((int)m, 16));
            const uint32_t m23 = max((uint32_t)__builtin_amdgcn_readlane((int)m, 32), (uint32_t)__builtin_amdgcn_readlane((int)m, 48));
            const uint32_t top = max(m01, m23);
            const uint32_t guess = top > (4u << 23) ? top - (4u << 23) : 0u;
            const int cnt = __popcll(ballot(key[r] >= guess));
            lo[r] = cnt >= k ? guess : 0u;
            hi[r] = top + 1u;
            if (cnt != k && k < DG) open |= 1u << r;
            if (k >= DG) lo[r] = 0u;
        }
        // 33 halvings bring any 32-bit interval down to one value (rows with a tie at the k-th
        // position never see an exact count and run the full course)
        for (int round = 0; round < 33 && open != 0u; ++round) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const uint32_t mid = lo[r] + ((hi[r] - lo[r]) >> 1);
                const int cnt = __popcll(ballot(key[r] >= mid));
                lo[r] = cnt >= k ? mid : lo[r];
                hi[r] = cnt >= k ? hi[r] : mid;
                open = cnt == k ? open & ~(1u << r) : open;
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) thr[r] = lo[r];
    } else {
        bool done[R];
#pragma unroll
        for (int r = 0; r < R; ++r) done[r] = (k >= DG);
        for (int bit = 31; bit >= 0; --bit) {
            bool all = true;
#pragma unroll
            for (int r = 0; r < R; ++r) all = all && done[r];
            if (ballot(!all) == 0ull) break;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const uint32_t cand = thr[r] | (1u << bit);
                const int cnt = popc<DG>(sub_bits<DG>(ballot(key[r] >= cand), sub));
                thr[r] = cnt >= k ? cand : thr[r];
                done[r] = done[r] || (cnt == k);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const bool ge = key[r] >= thr[r];
        const M ge_m = sub_bits<DG>(ballot(ge), sub);
        bool exact = popc<DG>(ge_m) == k;       // no tie at the threshold: the set is {key >= thr}
        if constexpr (DG != 64) exact = ballot(!exact) == 0ull;
        if (exact) {
            sel[r] = ge;
            mask_out[r] = ge_m;
        } else {
            const M below = ((M)1 << c) - 1;
            const M gt = sub_bits<DG>(ballot(key[r] > thr[r]), sub);
            const M eq = sub_bits<DG>(ballot(key[r] == thr[r]), sub);
            const int need = k - popc<DG>(gt);
            sel[r] = (key[r] > thr[r]) || (key[r] == thr[r] && popc<DG>(eq & below) < need);
            mask_out[r] = sub_bits<DG>(ballot(sel[r]), sub);
        }
    }
}

// ---- CSR views -------------------------------------------------------------------------------
struct CsrView {
    const int32_t* rp;
    const int32_t* ci;
    const float* av;
    const uint8_t* er;            // row of the entry modulo 16: its row in its 16-row tile
    // split plan of very long rows
    const int32_t* hub_rows;
    const int32_t* hub_cptr;
    const int32_t* hub_tile0;     // [tiles + 1]: split rows before row 16 t
    int32_t n_hub;
    int32_t hub_threshold;
    int32_t hub_chunk;            // a split row of at most this many entries is one chunk
    // tiles with more than heavy_edges stored entries, ascending (see TileDeal)
    const int32_t* heavy;
    int32_t n_heavy;
    int32_t heavy_edges;
    int32_t heavy_ptr[9];         // the entries of the list in every eighth of the tiles (an XCD's share of a sweep)
};

__device__ __forceinline__ int find_hub(const CsrView& g, int row) {
    int lo = 0, hi = g.n_hub - 1;
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (g.hub_rows[mid] < row) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// acc + partial rows q .. q1 - 1 of column c, added in chunk order, sixteen requested at a time.  The last batch is a
// whole one too, with zeros in the places past the end: one partial row after the other it was a round trip to memory
// each (30k nodes, eight nets of 5,000 sinks in one tile: 54 -> 38 us per launch of a tile kernel).
template <int DG, int NB = 16>
__device__ __forceinline__ float hub_chunks_sum(const float* __restrict__ part, int q, int q1, int c, float acc) {
    for (; q < q1; q += NB) {
        float v[NB];
#pragma unroll
        for (int u = 0; u < NB; ++u) v[u] = part[(size_t)(q + u < q1 ? q + u : q1 - 1) * DG + c];
#pragma unroll
        for (int u = 0; u < NB; ++u) acc += q + u < q1 ? v[u] : 0.f;
    }
    return acc;
}

// the same for two rows at once, thirty-two requested at a time (30k nodes, eight nets of 5,000 sinks: inverse kernel 18.2 -> 17.0 us; see
// hub_rows_fill)
template <int DG>
__device__ __forceinline__ void hub_chunks_sum2(const float* __restrict__ part, int qa, int qa1, int qb, int qb1, int c, float& a, float& b) {
    constexpr int NB = 16;
    for (; qa < qa1 || qb < qb1; qa += NB, qb += NB) {
        float va[NB], vb[NB];
#pragma unroll
        for (int u = 0; u < NB; ++u) va[u] = part[(size_t)(qa + u < qa1 ? qa + u : qa1 - 1) * DG + c];
#pragma unroll
        for (int u = 0; u < NB; ++u) vb[u] = part[(size_t)(qb + u < qb1 ? qb + u : qb1 - 1) * DG + c];
#pragma unroll
        for (int u = 0; u < NB; ++u) a += qa + u < qa1 ? va[u] : 0.f;
#pragma unroll
        for (int u = 0; u < NB; ++u) b += qb + u < qb1 ? vb[u] : 0.f;
    }
}

// sum of the first-pass partial rows of hub row `row`, in chunk order.  Few partial rows (on graphs of long rows nearly every
// row is one) are asked for four at a time: whole batches of sixteen took 352 us against 334 for a pass of Algorithm 1 there.
template <int DG>
__device__ __forceinline__ float hub_row_sum(const CsrView& g, const float* __restrict__ part, int row, int c) {
    const int h = find_hub(g, row), q = g.hub_cptr[h], q1 = g.hub_cptr[h + 1];
    return q1 - q <= 4 ? hub_chunks_sum<DG, 4>(part, q, q1, c, 0.f) : hub_chunks_sum<DG>(part, q, q1, c, 0.f);
}

// ---- 16-row tiles in LDS ---------------------------------------------------------------------------------
// Row stride of a tile of 16 x DG floats: a multiple of four words, so that adjacent columns move as 16-byte pieces, and
// four more than DG, which spreads the rows of a column over the banks.
template <int DG>
constexpr int tile_ld() { return DG + 4; }
typedef float f32v2 __attribute__((ext_vector_type(2)));
typedef float f32v4 __attribute__((ext_vector_type(4)));
// CPL adjacent columns (the first a multiple of CPL) between an LDS tile and registers
template <int CPL>
__device__ __forceinline__ void lds_load(const float* p, float (&v)[CPL]) {
    if constexpr (CPL == 1) {
        v[0] = *p;
    } else if constexpr (CPL == 2) {
        const f32v2 t = *reinterpret_cast<const f32v2*>(p);
        v[0] = t[0]; v[1] = t[1];
    } else {
#pragma unroll
        for (int c = 0; c < CPL; c += 4) {
            const f32v4 t = *reinterpret_cast<const f32v4*>(p + c);
            v[c] = t[0]; v[c + 1] = t[1]; v[c + 2] = t[2]; v[c + 3] = t[3];
        }
    }
}
template <int CPL>
__device__ __forceinline__ void lds_store(float* p, const float (&v)[CPL]) {
    if constexpr (CPL == 1) {
        *p = v[0];
    } else if constexpr (CPL == 2) {
        f32v2 t; t[0] = v[0]; t[1] = v[1];
        *reinterpret_cast<f32v2*>(p) = t;
    } else {
#pragma unroll
        for (int c = 0; c < CPL; c += 4) {
            f32v4 t; t[0] = v[c]; t[1] = v[c + 1]; t[2] = v[c + 2]; t[3] = v[c + 3];
            *reinterpret_cast<f32v4*>(p + c) = t;
        }
    }
}

// ---- tile gathers on the matrix cores ------------------------------------------------------------------
// A wave owns 16 consecutive rows.  Their neighbour lists are one contiguous edge range, so the
// dependent chain row pointer -> column index -> neighbour data is walked once per tile, 64 edges
// per step: lane l loads edge l, finds the tile row it belongs to, and parks (neighbour, a_ij, row)
// in LDS.  The aggregation itself is the product  H = P * X  of the tile's 16 x E selection
// matrix (P[r][e] = a_e if edge e belongs to row r, else 0) with the E x DG matrix of neighbour
// rows, taken four edges at a time by v_mfma_f32_16x16x4_f32:
//   A operand  lane (i = lane % 16, kk = lane / 16):  P[i][edge kk of the four]
//   B operand  lane (j = lane % 16, kk = lane / 16):  X[neighbour of edge kk][column of (j, cb)]
// One MFMA covers 16 columns; the DG / 16 column blocks cb are interleaved, column = CPL * j + cb
// with CPL = DG / 16, so that a lane's CPL columns are adjacent in memory and arrive in one load
// of CPL values.  One load instruction thus fetches the rows of four edges, nothing is predicated
// (edges past the end are staged with a_ij = 0 and neighbour 0) and the sum over a row's edges is
// taken in edge order inside the accumulators, which hold H as D[4 * (lane / 16) + reg][j].
using f32x4 = __attribute__((__vector_size__(4 * sizeof(float)))) float;
typedef uint32_t u32x2a __attribute__((ext_vector_type(2), aligned(4)));
typedef uint32_t u32x3a __attribute__((ext_vector_type(3), aligned(4)));
typedef uint32_t u32x4a __attribute__((ext_vector_type(4), aligned(4)));

template <int NW>
__device__ __forceinline__ void load_words(const void* p, uint32_t (&w)[NW]) {
    if constexpr (NW == 1) {
        w[0] = *reinterpret_cast<const uint32_t*>(p);
    } else if constexpr (NW == 2) {
        const u32x2a v = *reinterpret_cast<const u32x2a*>(p);
        w[0] = v[0]; w[1] = v[1];
    } else if constexpr (NW == 3) {
        const u32x3a v = *reinterpret_cast<const u32x3a*>(p);
        w[0] = v[0]; w[1] = v[1]; w[2] = v[2];
    } else {
        static_assert(NW == 4, "1 to 4 words");
        const u32x4a v = *reinterpret_cast<const u32x4a*>(p);
        w[0] = v[0]; w[1] = v[1]; w[2] = v[2]; w[3] = v[3];
    }
}

// column cb of a lane's adjacent columns as they were loaded
template <typename T, int NW>
__device__ __forceinline__ float word_col(const uint32_t (&w)[NW], int cb) {
    if constexpr (sizeof(T) == 4) return __uint_as_float(w[cb]);
    else return __uint_as_float((cb & 1) ? (w[cb >> 1] & 0xFFFF0000u) : (w[cb >> 1] << 16));
}

// ---- tile register layout ---------------------------------------------------------------------------
// What the MFMA leaves in a wave's accumulators for a 16 x DG tile when the A operand takes tile
// row 4 (i % 4) + i / 4 as its row i and the B operand takes column CPL j + cb as column j of
// block cb (CPL = DG / 16): lane (g = lane / 16, j = lane % 16) holds, in acc[cb][reg],
//     tile row 4 reg + g,  column CPL j + cb.
// For a fixed reg the 16 lanes of a group cover one whole row with CPL adjacent elements each, so
// a row moves between registers and memory with one fully coalesced access of CPL elements per
// lane, four rows per instruction.  Sums over a row are sums over the 16 lanes of a group.
template <int CPL, typename T>
__device__ __forceinline__ void load_cols(const T* p, float (&v)[CPL]) {       // non-temporal
    constexpr int NW = CPL * (int)sizeof(T) / 4;
    uint32_t w[NW];
    if constexpr (NW == 1) {
        w[0] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(p));
    } else if constexpr (NW == 2) {
        const u32x2a t = __builtin_nontemporal_load(reinterpret_cast<const u32x2a*>(p));
        w[0] = t[0]; w[1] = t[1];
    } else {
        const u32x4a t = __builtin_nontemporal_load(reinterpret_cast<const u32x4a*>(p));
        w[0] = t[0]; w[1] = t[1]; w[2] = t[2]; w[3] = t[3];
    }
#pragma unroll
    for (int c = 0; c < CPL; ++c) v[c] = word_col<T>(w, c);
}
// v must hold values representable in T (as stored<T>() returns them)
template <int CPL, typename T, bool CACHED = false>
__device__ __forceinline__ void store_cols(T* p, const float (&v)[CPL]) {      // non-temporal, or CACHED
    constexpr int NW = CPL * (int)sizeof(T) / 4;
    uint32_t w[NW];
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        if constexpr (sizeof(T) == 4) w[i] = __float_as_uint(v[i]);
        else w[i] = (__float_as_uint(v[2 * i]) >> 16) | (__float_as_uint(v[2 * i + 1]) & 0xFFFF0000u);
    }
    auto put = [](auto v, auto* q) {
        if constexpr (CACHED) *q = v;
        else __builtin_nontemporal_store(v, q);
    };
    if constexpr (NW == 1) {
        put(w[0], reinterpret_cast<uint32_t*>(p));
    } else if constexpr (NW == 2) {
        u32x2a t; t[0] = w[0]; t[1] = w[1];
        put(t, reinterpret_cast<u32x2a*>(p));
    } else {
        u32x4a t; t[0] = w[0]; t[1] = w[1]; t[2] = w[2]; t[3] = w[3];
        put(t, reinterpret_cast<u32x4a*>(p));
    }
}
// sum over the 16 lanes of this lane's group, the same value in all of them
__device__ __forceinline__ float group16_sum(float v) {
    v = dpp_add<0xB1>(v);    // quad_perm [1,0,3,2]
    v = dpp_add<0x4E>(v);    // quad_perm [2,3,0,1]
    v = dpp_add<0x141>(v);   // row_half_mirror
    v = dpp_add<0x140>(v);   // row_mirror
    return v;
}

// ---- bf16 operands for the gathers of the bf16-storage variant --------------------------------------
// With 16-bit stored values the product P * X runs on v_mfma_f32_16x16x16_bf16: sixteen edges per
// instruction instead of four.  The K index is permuted so that nothing has to move between
// lanes: K slot 4 kk + u of lane group kk is edge kk of staged group u (u = 0..3), which is what
// the lane already holds after four loads.  X is exact in bf16; a_ij is split into three bf16 terms
// (a = hi + mid + lo exactly), one MFMA each, float32 accumulation.
typedef short bf16x4 __attribute__((ext_vector_type(4)));

// upper halves of four float32 words as four bf16
__device__ __forceinline__ bf16x4 pack_upper4(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3) {
    const uint32_t lo = __builtin_amdgcn_perm(w1, w0, 0x07060302u), hi = __builtin_amdgcn_perm(w3, w2, 0x07060302u);
    return __builtin_bit_cast(bf16x4, (uint64_t)lo | ((uint64_t)hi << 32));
}
// lower halves of four words as four bf16
__device__ __forceinline__ bf16x4 pack_lower4(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3) {
    const uint32_t lo = __builtin_amdgcn_perm(w1, w0, 0x05040100u), hi = __builtin_amdgcn_perm(w3, w2, 0x05040100u);
    return __builtin_bit_cast(bf16x4, (uint64_t)lo | ((uint64_t)hi << 32));
}
// the selection operand of four groups as three bf16 terms: p = hi + mid + lo exactly
__device__ __forceinline__ void split_p4(const float* p, bf16x4& hi, bf16x4& mid, bf16x4& lo) {
    uint32_t h[4], m[4], l[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        h[u] = __float_as_uint(p[u]) & 0xFFFF0000u;
        const float r1 = p[u] - __uint_as_float(h[u]);
        m[u] = __float_as_uint(r1) & 0xFFFF0000u;
        l[u] = __float_as_uint(r1 - __uint_as_float(m[u]));
    }
    hi = pack_upper4(h[0], h[1], h[2], h[3]);
    mid = pack_upper4(m[0], m[1], m[2], m[3]);
    lo = pack_upper4(l[0], l[1], l[2], l[3]);
}

struct EdgeRec {
    int j;      // neighbour (column of A)
    float a;    // a_ij
    int r;      // row of the tile, 0..15
    int pad;
};

// Row pointer of row r0 + lane (clamped at n) for the 17 row boundaries of a tile, in lanes 0..16.
// Split from tile_begin so that a kernel can request its other per-tile data before it waits.
__device__ __forceinline__ int tile_rp_load(const CsrView& g, uint32_t r0, int n, int lane) {
    int rpv = 0;
    const uint32_t r = r0 + (uint32_t)lane;   // unsigned: a tile past the last may lie beyond 2^31
    if (lane < 17) rpv = g.rp[r < (uint32_t)n ? r : (uint32_t)n];
    return rpv;
}

// Publishes the tile's row pointers (rpv as tile_rp_load returned it) in s_rp.  Returns whether
// one of the rows is a split ("hub") row.
__device__ __forceinline__ bool tile_begin(const CsrView& g, int rpv, int* s_rp, int lane) {
    if (lane < 17) s_rp[lane] = rpv;
    wave_sync();
    const bool hub = lane < 16 && (s_rp[lane + 1] - rpv) > g.hub_threshold;
    return ballot(hub) != 0ull;
}

// tile row of edge e: the last row boundary at or below e
__device__ __forceinline__ int tile_row_of(const int* s_rp, int e) {
    int r = 0;
#pragma unroll
    for (int step = 8; step >= 1; step >>= 1)
        if (s_rp[r + step] <= e) r += step;
    return r;
}

// Runs `batch(GB, i0)` over the nit <= 16 groups of four staged edges in as few batches as
// possible: all sixteen at once if MAXB allows, else eight, then the rest as one batch of eight
// or four (a batch may overrun nit by up to three groups, which stay inside the 64 staged edges
// and contribute zero).
template <int MAXB, typename Batch>
__device__ __forceinline__ void edge_batches(int nit, Batch batch) {
    int i0 = 0;
    if constexpr (MAXB >= 16) {
        if (nit > 12) {
            batch(std::integral_constant<int, 16>{}, 0);
            return;
        }
    }
    if (nit > 8) {
        batch(std::integral_constant<int, 8>{}, 0);
        i0 = 8;
    }
    if (nit - i0 > 4) batch(std::integral_constant<int, 8>{}, i0);
    else if (nit - i0 > 0) batch(std::integral_constant<int, 4>{}, i0);
}

// acc += P * X over the edges [e_a, e_b) of ordinary rows; X is a dense plane, row stride ld.
// ONE_ROW: every edge belongs to tile row 0 (a chunk of a split row).  The matrix product would then spend
// fifteen of its sixteen rows on zeros; instead lane (kk, j) adds a_e * X[e][its columns] for the edges kk,
// kk + 4, .. in ordinary arithmetic into acc[cb][0], and the caller adds the four lane groups up.
template <int DG, typename T, int MAXB, bool ONE_ROW = false>
__device__ __forceinline__ void gather_dense_mfma(const CsrView& g, const T* __restrict__ x, int64_t ld, int e_a, int e_b,
                                                  const int* s_rp, EdgeRec* ebuf, int lane, f32x4 (&acc)[DG / 16]) {
    constexpr int CPL = DG / 16, NW = CPL * (int)sizeof(T) / 4;
    const int i16 = lane & 15, kk = lane >> 4;
    const T* xl = x + CPL * i16;
    const uint32_t ldu = (uint32_t)ld;
    for (int eb = e_a; eb < e_b; eb += 64) {
        const int e = eb + lane;
        const bool ok = e < e_b;
        EdgeRec me;
        if constexpr (ONE_ROW) me.j = __builtin_nontemporal_load(g.ci + (ok ? e : e_b - 1));   // a place past the end: 0 times a row of its own
        else me.j = ok ? __builtin_nontemporal_load(g.ci + e) : 0;
        me.a = ok ? __builtin_nontemporal_load(g.av + e) : 0.f;
        me.r = tile_row_of(s_rp, e);
        me.pad = 0;
        wave_sync();          // readers of the previous chunk are done
        ebuf[lane] = me;
        wave_sync();
        const int cnt = e_b - eb < 64 ? e_b - eb : 64;
        edge_batches<MAXB>((cnt + 3) >> 2, [&](auto gbc, int i0) {
            constexpr int GB = decltype(gbc)::value;
            uint32_t w[GB][NW];
            float p[GB];
#pragma unroll
            for (int u = 0; u < GB; ++u) {
                const EdgeRec er = ebuf[4 * (i0 + u) + kk];
                load_words<NW>(xl + (size_t)(uint32_t)er.j * ldu, w[u]);
                p[u] = (ONE_ROW || er.r == i16) ? er.a : 0.f;
            }
            if constexpr (ONE_ROW) {
#pragma unroll
                for (int u = 0; u < GB; ++u)
#pragma unroll
                    for (int cb = 0; cb < CPL; ++cb) {       // (through word_col: 10.6 us per launch against 9.5, 20k nodes, 16 bits)
                        uint32_t bits;
                        if constexpr (sizeof(T) == 4) bits = w[u][cb];
                        else bits = (cb & 1) ? (w[u][cb >> 1] & 0xFFFF0000u) : (w[u][cb >> 1] << 16);
                        acc[cb][0] = __builtin_fmaf(p[u], __uint_as_float(bits), acc[cb][0]);
                    }
            } else if constexpr (sizeof(T) == 4) {
#pragma unroll
                for (int u = 0; u < GB; ++u)
#pragma unroll
                    for (int cb = 0; cb < CPL; ++cb)
                        acc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(p[u], __uint_as_float(w[u][cb]), acc[cb], 0, 0, 0);
            } else {
#pragma unroll
                for (int u = 0; u < GB; u += 4) {
                    bf16x4 ph, pm, pl;
                    split_p4(p + u, ph, pm, pl);
#pragma unroll
                    for (int cb = 0; cb < CPL; ++cb) {
                        const int d = cb >> 1;
                        const bf16x4 b = (cb & 1) ? pack_upper4(w[u][d], w[u + 1][d], w[u + 2][d], w[u + 3][d])
                                                  : pack_lower4(w[u][d], w[u + 1][d], w[u + 2][d], w[u + 3][d]);
                        acc[cb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ph, b, acc[cb], 0, 0, 0);
                        acc[cb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(pm, b, acc[cb], 0, 0, 0);
                        acc[cb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(pl, b, acc[cb], 0, 0, 0);
                    }
                }
            }
        });
    }
}

// ---- gathers in ordinary arithmetic -------------------------------------------------------------------------
// acc += P * scatter(V, I) over the edges [e_a, e_b) of ordinary rows (Section 4.1, eq. (10)), a lane per kept value.  (On
// the matrix cores a 16-row product spends fifteen rows of every edge on zeros.)  Beside its k values a record
// holds the column of each as a byte; the value of slot t of a neighbour belongs to lane t of a group of sixteen, which
// adds a_ij * value to that column of the destination row's sums in LDS: read, fused multiply-add, written back.  (A lane
// that owns columns instead has to find the window of slots that may hold them from the neighbour's mask - a round trip to
// memory before the values can be requested -, load four times the record's bytes and deal them out: some 24 vector
// instructions per four edges and five round trips per 64 edges where this takes about eight and one: 1M nodes, D/C = 64,
// k = 16: forward kernel 280 -> 223 us, inverse 298 -> 246, vector instructions per tile 1,490 -> 950.  What is left is
// latency: a wave waits for two thirds of its time, and LDS holds no more waves.)
// The staged edges of a round are cut into four equal runs, one per lane group; a run's edges add straight into the rows
// of the tile, except those of the run's first row, which the run before may share: they add into a row of the group's
// own (the four rows of st behind the tile), and those four rows join the tile at the end of the round, the rows that end inside
// their run before the rows that fill one.  So no two groups touch one row in the same step, the values of one record
// are in different columns, and the order of the additions is fixed by the edge list alone.
// Lane s of a group holds edge s of the group's run, and a step takes its edge from there by a row broadcast of the
// lanes (through LDS it took as much of the LDS pipe as the additions themselves).
// st: TR + 4 rows, zeroed by the caller (the last four are left zero), and 64 words behind them where lanes without a value
// add.  A run is a whole number of ROUND steps; the places past the last edge hold that edge once more with a_ij = 0.
// k above 16 takes ceil(k / 16) passes over the edges of a round.  FEW: four steps' loads in flight instead of a whole
// run's (for kernels without registers to spare).
// The tile has TR rows (16, or 8 where a group is wider than 64 columns and LDS would hold too few waves).
template <int DG, int TR = 16>
constexpr int gather_floats() { return (TR + 4) * tile_ld<DG>() + 64; }
typedef __attribute__((address_space(3))) float lds_float;

// v of lane S of this lane's row of sixteen
template <int S>
__device__ __forceinline__ uint32_t row_lane(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x150 + S, 0xF, 0xF, true);
}

// steps S0 .. S0 + NB - 1 of a run, value t of every record: all loads first, then the additions in edge order
template <int S0, int NB, typename T, int... U>
__device__ __forceinline__ void values_run(const T* __restrict__ vals, const uint8_t* __restrict__ cols, uint32_t off0, float a,
                                           uint32_t row, uint32_t t, bool has, uint32_t dump, std::integer_sequence<int, U...>) {
    T v[NB];
    uint32_t col[NB];
    ((v[U] = vals[(size_t)(row_lane<S0 + U>(off0) + t)], col[U] = cols[(size_t)(row_lane<S0 + U>(off0) + t)]), ...);
    wave_sync();
    (([&] {
         const uint32_t at = row_lane<S0 + U>(row) + 4u * col[U];
         lds_float* s = (lds_float*)(uintptr_t)(has ? at : dump);
         *s = __builtin_fmaf(__uint_as_float(row_lane<S0 + U>(__float_as_uint(a))), to_float(v[U]), *s);
         wave_sync();
     }()),
     ...);
}

// The edges of one round as the lanes hold them: lane s of group kk the s-th edge of the kk-th of four equal runs of the
// (up to 64) edges from eb on.
struct RunEdges {
    int j, r;        // neighbour, row of the tile
    float a;         // a_ij (of the last edge in the places past it)
    int steps;       // edges per run, at most 16 (wave-uniform)
};
// Edges per run of a round over the edges [eb, e_b): at least one step's worth.
template <int ROUND>
__host__ __device__ constexpr int run_steps(int eb, int e_b) {
    const int cnt = e_b - eb < 1 ? 1 : e_b - eb < 64 ? e_b - eb : 64;
    return (((cnt + 3) >> 2) + ROUND - 1) / ROUND * ROUND;
}
// The entry a lane loads in that round: its edge, or the last one in the places past it.  The first round is asked for before
// anyone knows that there is one, so the range may be empty (a tile without entries), also at the front of the arrays: the entry
// is then one nobody uses, and one that exists (the arrays have room for an entry on a graph without any).
__host__ __device__ constexpr int run_entry(int eb, int e_b, int steps, int lane) {
    const int slot = lane & 15, last = e_b > 0 ? e_b - 1 : 0;
    const int e = eb + (lane >> 4) * steps + (slot < steps ? slot : steps - 1);
    return e < last ? e : last;
}
template <int ROUND>
__device__ __forceinline__ RunEdges run_edges(const CsrView& g, int eb, int e_b, int lane) {
    RunEdges d;
    d.steps = run_steps<ROUND>(eb, e_b);
    const int ec = run_entry(eb, e_b, d.steps, lane);
    d.j = __builtin_nontemporal_load(g.ci + ec);
    d.a = __builtin_nontemporal_load(g.av + ec);
    d.r = __builtin_nontemporal_load(g.er + ec);
    return d;
}

template <int DG, int ROUND, bool FEW, int TR = 16, typename T>
__device__ __forceinline__ void gather_values_rows(const CsrView& g, const T* __restrict__ vals, const uint8_t* __restrict__ cols,
                                                   int k, int e_a, int e_b, int lane, float* st) {
    constexpr int LR = tile_ld<DG>();
    static_assert(ROUND == 4 || ROUND == 8, "a run must fit the sixteen lanes of a group");
    const int slot = lane & 15, kk = lane >> 4;
    const uint32_t base = (uint32_t)(uintptr_t)(lds_float*)st, dump = base + 4u * (uint32_t)((TR + 4) * LR + lane);
    RunEdges next = run_edges<ROUND>(g, e_a, e_b, lane);
    for (int eb = e_a; eb < e_b; eb += 64) {
        const int steps = next.steps, j = next.j, r = next.r & (TR - 1);
        const float a = eb + kk * steps + slot < e_b ? next.a : 0.f;      // (lanes past the run: not used)
        int head[4], tail[4];                              // first and last row of every run
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            head[q] = __builtin_amdgcn_readlane(r, 16 * q);
            tail[q] = __builtin_amdgcn_readlane(r, 16 * q + steps - 1);
        }
        const uint32_t off0 = (uint32_t)j * (uint32_t)k;
        const uint32_t row = base + 4u * (uint32_t)((r == (int)row_lane<0>((uint32_t)r) ? TR + kk : r) * LR);
        if (eb + 64 < e_b) next = run_edges<ROUND>(g, eb + 64, e_b, lane);     // arrives while this round is added
        for (int t0 = 0; t0 < k; t0 += 16) {
            const bool has = t0 + slot < k;
            const uint32_t t = (uint32_t)(has ? t0 + slot : t0);
            auto run = [&](auto nbc, auto s0c) {
                constexpr int NB = decltype(nbc)::value;
                // (keeps the variants apart: folded together, every load is waited for before the next)
                asm volatile("; %0 steps" ::"n"(NB));
                values_run<decltype(s0c)::value, NB>(vals, cols, off0, a, row, t, has, dump, std::make_integer_sequence<int, NB>{});
            };
            constexpr std::integral_constant<int, 0> s0{};
            if constexpr (FEW) {
                run(std::integral_constant<int, 4>{}, s0);
                if (steps > 4) run(std::integral_constant<int, 4>{}, std::integral_constant<int, 4>{});
                if (steps > 8) run(std::integral_constant<int, 4>{}, std::integral_constant<int, 8>{});
                if (steps > 12) run(std::integral_constant<int, 4>{}, std::integral_constant<int, 12>{});
            } else if constexpr (ROUND == 4) {
                if (steps == 4) run(std::integral_constant<int, 4>{}, s0);
                else if (steps == 8) run(std::integral_constant<int, 8>{}, s0);
                else if (steps == 12) run(std::integral_constant<int, 12>{}, s0);
                else run(std::integral_constant<int, 16>{}, s0);
            } else {
                if (steps == 8) run(std::integral_constant<int, 8>{}, s0);
                else run(std::integral_constant<int, 16>{}, s0);
            }
        }
        // the groups' own rows join the tile
#pragma unroll
        for (int c = lane; c < DG; c += 64) {
            float sum[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) sum[q] = st[(TR + q) * LR + c];
#pragma unroll
            for (int q = 0; q < 4; ++q) st[(TR + q) * LR + c] = 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (head[q] != tail[q]) st[head[q] * LR + c] += sum[q];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (head[q] == tail[q]) st[head[q] * LR + c] += sum[q];
        }
        wave_sync();
    }
}

// The same for a dense plane X (row stride ld): st += P * X over the edges [e_a, e_b) of ordinary rows, lane j of
// a group keeping a running sum of its CPL columns for the run's present row in registers and adding it to the row of the
// tile when the row changes and at the end of the round.  Two groups never add to one row in the same instruction: inside
// a round only the last run that holds a row sees it end; the sums left at the end of the round are added group by group.
// Lane s of a group holds edge s of the run (row_lane hands it to the others).
template <int DG, int S0, typename T, int... U>
__device__ __forceinline__ void dense_run(const T* __restrict__ xl, uint32_t ldu, uint32_t j, uint32_t a, uint32_t r, float* mine,
                                          uint32_t& cur, float (&run)[DG / 16], std::integer_sequence<int, U...>) {
    constexpr int CPL = DG / 16, LR = tile_ld<DG>(), NW = CPL * (int)sizeof(T) / 4;
    uint32_t w[sizeof...(U)][NW];
    (load_words<NW>(xl + (size_t)row_lane<S0 + U>(j) * ldu, w[U]), ...);
    (([&] {
         const uint32_t row = row_lane<S0 + U>(r);
         if (row != cur) {
             float was[CPL];
             lds_load<CPL>(mine + cur * LR, was);
#pragma unroll
             for (int cb = 0; cb < CPL; ++cb) {
                 was[cb] += run[cb];
                 run[cb] = 0.f;
             }
             lds_store<CPL>(mine + cur * LR, was);
             cur = row;
         }
         const float p = __uint_as_float(row_lane<S0 + U>(a));
#pragma unroll
         for (int cb = 0; cb < CPL; ++cb) run[cb] = __builtin_fmaf(p, word_col<T>(w[U], cb), run[cb]);
     }()),
     ...);
}

template <int DG, int GB, typename T>
__device__ __forceinline__ void gather_dense_rows(const CsrView& g, const T* __restrict__ x, int64_t ld, int e_a, int e_b,
                                                  int lane, float* st) {
    constexpr int CPL = DG / 16, LR = tile_ld<DG>();
    static_assert(GB == 8, "a run is one or two batches");
    const int i16 = lane & 15, kk = lane >> 4;
    const T* xl = x + CPL * i16;
    const uint32_t ldu = (uint32_t)ld;
    float* mine = st + CPL * i16;
    for (int eb = e_a; eb < e_b; eb += 64) {
        const int cnt = e_b - eb < 64 ? e_b - eb : 64;     // wave-uniform
        const int steps = (((cnt + 3) >> 2) + GB - 1) / GB * GB;      // edges per run: 8 or 16
        const int e = eb + kk * steps + (i16 < steps ? i16 : steps - 1);
        const int ec = e < e_b ? e : e_b - 1;              // (places past the last edge: the last edge once more with a_ij = 0)
        const uint32_t j = (uint32_t)__builtin_nontemporal_load(g.ci + ec);
        const float av = __builtin_nontemporal_load(g.av + ec);
        const uint32_t r = __builtin_nontemporal_load(g.er + ec);
        const uint32_t a = __float_as_uint(e < e_b ? av : 0.f);
        uint32_t cur = row_lane<0>(r);
        float run[CPL];
#pragma unroll
        for (int cb = 0; cb < CPL; ++cb) run[cb] = 0.f;
        dense_run<DG, 0>(xl, ldu, j, a, r, mine, cur, run, std::make_integer_sequence<int, GB>{});
        if (steps > GB) dense_run<DG, GB>(xl, ldu, j, a, r, mine, cur, run, std::make_integer_sequence<int, GB>{});
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
            wave_sync();
            if (kk == gq) {
                float was[CPL];
                lds_load<CPL>(mine + cur * LR, was);
#pragma unroll
                for (int cb = 0; cb < CPL; ++cb) was[cb] += run[cb];
                lds_store<CPL>(mine + cur * LR, was);
            }
        }
        wave_sync();
    }
}

template <int DG, bool FAST, bool PAIRS = true>
__device__ __forceinline__ void hub_rows_fill(const CsrView& g, const float* __restrict__ hub_part, int r0, const int* s_rp,
                                              float* st, int lane);

// H of the tile into st through a row-wise gather: st (ROWS rows of it) is cleared, the runs of ordinary rows are added into it,
// split rows receive the sum of their first-pass partial rows afterwards.
template <int DG, bool FAST = true, int ROWS = 16, bool PAIRS = true, typename Range>
__device__ __forceinline__ void tile_gather_rows(const CsrView& g, const float* __restrict__ hub_part, bool has_hub, int r0,
                                                 const int* s_rp, float* st, int lane, Range range) {
    static_assert(ROWS * tile_ld<DG>() % 4 == 0, "cleared in pieces of 16 bytes");
    for (int i = 4 * lane; i < ROWS * tile_ld<DG>(); i += 256) *reinterpret_cast<f32v4*>(st + i) = f32v4{0.f, 0.f, 0.f, 0.f};
    wave_sync();
    tile_ranges(g, has_hub, s_rp, range);
    wave_sync();
    if (has_hub) hub_rows_fill<DG, FAST, PAIRS>(g, hub_part, r0, s_rp, st, lane);
}

// sum of the first-pass partial rows of every split row of the tile into st, each row's in chunk order.  On a graph of
// long rows every row of every tile is split, into one or two chunks, and a tile is all a wave has to do in a launch:
// what counts is the number of memory round trips in a row.  So the sixteen rows find their places in the list of
// split rows from one number per tile (split rows before the tile) and a count over the lanes before them, not by a
// search each; the first partial rows of all sixteen are requested together, then the second ones, up to the fourth;
// and only rows of more than four chunks go on one by one, sixteen loads in flight (Table-1-shaped graph: forward
// kernel 43 -> 38 us per launch, fused inverse + dW 51 -> 46 us).  The additions of a row are 0 + p_0 + p_1 + .. in this
// order whatever the batching.
constexpr int HUB_FILL_ROWS = 16;     // rows whose partial rows are requested together
constexpr int HUB_FILL_DEPTH = 4;     // partial rows per row taken that way (the launch of a long-row graph ends with the
                                      // tile whose rows go on one by one: 26 us against a median of 6)
// PAIRS: rows of more chunks than that go on two at a time, else one by one.  Two at a time shorten
// the tile of the longest rows, which a launch of few tiles per wave ends with; a kernel that only gathers pays for it in its sweep (93
// registers for 65, k_spmm_tile of 32 columns: 750k rows 106 us against 98), so the operators take it by their number of tiles.
template <int DG, bool FAST, bool PAIRS>
__device__ __forceinline__ void hub_rows_fill(const CsrView& g, const float* __restrict__ hub_part, int r0, const int* s_rp,
                                              float* st, int lane) {
    // (FAST = false: a search per row and the rows one by one - for kernels that have no register to spare; same
    // additions)
    if constexpr (!FAST) {
        int q0s = 0, q1s = 0;
        if (lane < 16 && (s_rp[lane + 1] - s_rp[lane]) > g.hub_threshold) {
            const int h = find_hub(g, r0 + lane);
            q0s = g.hub_cptr[h];
            q1s = g.hub_cptr[h + 1];
        }
        for (int r = 0; r < 16; ++r) {
            const int q = __builtin_amdgcn_readlane(q0s, r), q1 = __builtin_amdgcn_readlane(q1s, r);
            if (q1 <= q) continue;                 // not a split row
            const float acc = hub_chunks_sum<DG>(hub_part, q, q1, lane < DG ? lane : 0, 0.f);
            if (lane < DG) st[r * tile_ld<DG>() + lane] = acc;
        }
        return;
    }
    const bool split = lane < 16 && (s_rp[lane + 1] - s_rp[lane]) > g.hub_threshold;
    const uint64_t splits = __builtin_amdgcn_ballot_w64(split);
    int q0v = 0, q1v = 0;
    if (split) {
        const int h = g.hub_tile0[r0 >> 4] + __popcll(splits & (((uint64_t)1 << lane) - 1));
        q0v = g.hub_cptr[h];
        q1v = g.hub_cptr[h + 1];
    }
    const int c = lane < DG ? lane : 0;
    // partial row j of every row that has one, j = 0 .. HUB_FILL_DEPTH - 1, while any row has one
    for (int j = 0; j < HUB_FILL_DEPTH; ++j) {
        if (__builtin_amdgcn_ballot_w64(q1v - q0v > j) == 0) break;
#pragma unroll
        for (int rb = 0; rb < 16; rb += HUB_FILL_ROWS) {
            float v[HUB_FILL_ROWS];
#pragma unroll
            for (int u = 0; u < HUB_FILL_ROWS; ++u) {
                const int q = __builtin_amdgcn_readlane(q0v, rb + u) + j, q1 = __builtin_amdgcn_readlane(q1v, rb + u);
                v[u] = hub_part[(size_t)(q < q1 ? q : 0) * DG + c];        // (no chunk j: any row, not used)
            }
#pragma unroll
            for (int u = 0; u < HUB_FILL_ROWS; ++u) {
                const int r = rb + u;
                const int q = __builtin_amdgcn_readlane(q0v, r) + j, q1 = __builtin_amdgcn_readlane(q1v, r);
                if (q < q1 && lane < DG) st[r * tile_ld<DG>() + lane] = (j == 0 ? 0.f : st[r * tile_ld<DG>() + lane]) + v[u];
            }
        }
    }
    if constexpr (!PAIRS) {
        for (int r = 0; r < 16; ++r) {          // sixteen loads in flight
            const int q = __builtin_amdgcn_readlane(q0v, r) + HUB_FILL_DEPTH, q1 = __builtin_amdgcn_readlane(q1v, r);
            if (q1 <= q) continue;
            const float acc = hub_chunks_sum<DG>(hub_part, q, q1, c, st[r * tile_ld<DG>() + c]);
            if (lane < DG) st[r * tile_ld<DG>() + lane] = acc;
        }
        return;
    }
    // in pairs, thirty-two loads in flight (an odd one with itself)
    uint64_t more = __builtin_amdgcn_ballot_w64(q1v - q0v > HUB_FILL_DEPTH);
    while (more != 0ull) {
        const int ra = __builtin_ctzll(more);
        more &= more - 1;
        const int rb = more != 0ull ? __builtin_ctzll(more) : ra;
        more &= more - 1;          // (of nothing: nothing)
        float a = st[ra * tile_ld<DG>() + c], b = st[rb * tile_ld<DG>() + c];
        hub_chunks_sum2<DG>(hub_part, __builtin_amdgcn_readlane(q0v, ra) + HUB_FILL_DEPTH, __builtin_amdgcn_readlane(q1v, ra),
                            __builtin_amdgcn_readlane(q0v, rb) + HUB_FILL_DEPTH, __builtin_amdgcn_readlane(q1v, rb), c, a, b);
        if (lane < DG) {
            st[ra * tile_ld<DG>() + lane] = a;
            st[rb * tile_ld<DG>() + lane] = b;
        }
    }
}

// Calls `range(e_a, e_b)` for every maximal run of ordinary (not split) rows of the tile.
template <typename Range>
__device__ __forceinline__ void tile_ranges(const CsrView& g, bool has_hub, const int* s_rp, Range range) {
    if (!has_hub) {
        range(s_rp[0], s_rp[16]);
        return;
    }
    int run = 0;
    for (int r = 0; r <= 16; ++r) {
        const bool hub = r < 16 && (s_rp[r + 1] - s_rp[r]) > g.hub_threshold;
        if (r == 16 || hub) {
            if (s_rp[r] > s_rp[run]) range(s_rp[run], s_rp[r]);
            run = r + 1;
        }
    }
}

// H of the tile into st (16 rows, row stride tile_ld): the runs of ordinary rows go through
// `range(e_a, e_b)`, which accumulates into acc (D[4 (lane / 16) + reg][j] of column block cb,
// column = CPL j + cb); split rows receive the sum of their first-pass partial rows afterwards.
template <int DG, bool FAST = true, typename Range>
__device__ __forceinline__ void tile_gather(const CsrView& g, const float* __restrict__ hub_part, bool has_hub, int r0,
                                            const int* s_rp, float* st, int lane, f32x4 (&acc)[DG / 16], Range range) {
    constexpr int CPL = DG / 16, LR = tile_ld<DG>();
#pragma unroll
    for (int cb = 0; cb < CPL; ++cb) acc[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
    tile_ranges(g, has_hub, s_rp, range);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        float v[CPL];
#pragma unroll
        for (int cb = 0; cb < CPL; ++cb) v[cb] = acc[cb][r];
        lds_store<CPL>(st + (4 * (lane >> 4) + r) * LR + CPL * (lane & 15), v);
    }
    if (has_hub) hub_rows_fill<DG, FAST>(g, hub_part, r0, s_rp, st, lane);
}

// ---- 16-row MFMA tiles -------------------------------------------------------------------------
// A wave multiplies its 16 x DG tile (staged in LDS, row stride tile_ld) by a DG x DG matrix with
// v_mfma_f32_16x16x4_f32:
//   A[i][kk]: lane = kk*16 + i;  B[kk][j]: lane = kk*16 + j;  D[4*(lane/16)+r][lane%16] in reg r.
// The DG x DG weight matrix sits in LDS (odd row stride DG + 1, which spreads the four k-rows of a
// B operand over different banks), loaded once per workgroup; transposed = true stores W^T.
template <int DG>
struct WLds {
    static constexpr int WP = DG + 1;
    float w[DG * WP];
};

template <int DG>
__device__ __forceinline__ void load_w_lds(const float* __restrict__ w, bool transposed, WLds<DG>& l) {
    // eight loads of a thread in flight at a time: on a graph where a launch is one short tile per wave this
    // prologue is a good part of the launch, and one load after the other is a round trip to memory each
    // (the transposed form, whose loads touch a cache line per lane, was a tenth slower that way and keeps the plain loop)
    constexpr int NL = 8;
    const int nt = blockDim.x;
    if (transposed) {
        for (int i = threadIdx.x; i < DG * DG; i += nt) {
            const int r = i / DG, cc = i % DG;
            l.w[r * WLds<DG>::WP + cc] = w[cc * DG + r];
        }
    } else {
        for (int i0 = threadIdx.x; i0 < DG * DG; i0 += NL * nt) {
            float v[NL];
#pragma unroll
            for (int u = 0; u < NL; ++u) {
                v[u] = w[i0 + u * nt < DG * DG ? i0 + u * nt : 0];
            }
#pragma unroll
            for (int u = 0; u < NL; ++u) {
                const int i = i0 + u * nt;
                if (i < DG * DG) l.w[(i / DG) * WLds<DG>::WP + i % DG] = v[u];
            }
        }
    }
    __syncthreads();
}

// acc = tile (16 x DG, LDS, row stride tile_ld) * B (DG x DG, LDS), left in the tile register
// layout: acc[cb][reg] = product[row 4 reg + lane / 16][column CPL (lane % 16) + cb].
template <int DG>
__device__ __forceinline__ void mfma_tile(const float* st, const WLds<DG>& wl, f32x4 (&acc)[DG / 16]) {
    constexpr int CPL = DG / 16;
    const int lane = lane_id(), i = lane & 15, kk = lane >> 4;
    const int arow = 4 * (i & 3) + (i >> 2);
#pragma unroll
    for (int cb = 0; cb < CPL; ++cb) acc[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < DG / 4; ++s) {
        const float a = st[arow * tile_ld<DG>() + 4 * s + kk];
#pragma unroll
        for (int cb = 0; cb < CPL; ++cb) {
            const float b = wl.w[(4 * s + kk) * WLds<DG>::WP + CPL * i + cb];
            acc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc[cb], 0, 0, 0);
        }
    }
}

// ---- the same products on the bf16 matrix pipe, exact to float32 rounding --------------------------------
// A float32 value is the exact sum of three bf16 terms (8 + 8 + 8 significant bits: hi = the value truncated to bf16,
// mid = the remainder truncated, lo = what is left).  A product a b is then the sum of nine exact bf16 products, of
// which the six with the largest weights (hi hi, hi mid, mid hi, hi lo, mid mid, lo hi) are taken.  What the other three
// would add is 2^-24.5 of the product on average and 2^-21.1 at most (normally distributed factors; a float32 multiply:
// 2^-25.5 and 2^-24); over a row of H W_i the sum's own rounding covers it: Y's error against 64 bits is the float32
// instructions' or a little less (50k nodes of mean degree 236, groups of 192: 5.5e-8 against 5.6e-8; ten more draws of
// such graphs and widths: 1 - 5 % less each).  (A long sum over rows, dW, is another matter: see mfma_outer.)
// v_mfma_f32_16x16x32_bf16 takes 32 K-slots per instruction and, unlike the float32 matrix instructions of this chip, runs beside
// the vector pipe, so the six products of a 32-deep step cost less than the float32 instruction sequence they replace and hide
// under the vector work of the other waves.  (The 16-deep form takes the same 16 cycles of the pipe for half of the slots; a tile
// kernel waits for much of a product's chain.  1M nodes, D/C = 64: forward kernel 228 -> 213 us, 100k nodes inverse + dW 45.9 ->
// 43.3; 200k nodes, groups of 128, X_i - H W_i 98 -> 88 us, 50k long rows, groups of 192, back through W_i^T 57 -> 45.  Its sums lose
// less: error of layer outputs and gradients against 64 bits with every column kept 5 - 8 % lower, dW up to 64 columns 8 - 9 %.)
// With 16-bit storage the products stay 16-deep (DEEP = false).  The 32-deep form adds in another order, which is below any rounding of
// the sum itself, but one stored value in thirty thousand then rounds to the neighbouring 16-bit number, a step of 2^-8, and where that value
// is at the k-th place of its row GS keeps another column: a few rows per pass over 8 planes of 1M nodes (their k-th and next
// value are one such step apart), whose gradients differ by up to twice the plane's root mean square from what the 16-deep form gives.
// W is kept in LDS already split and laid out as B operands: entry [term][s][cb][lane] holds, for lane (kk = lane / 16,
// j = lane % 16), the eight bf16 of a 32-deep step s in column CPL j + cb (of W, or of W^T).
// A lane's eight K-slots of a 32-deep step are two times four rows: with h = 0, 1 and u = 0 .. 3, slot 4 h + u of lane group kk is
// row 32 s + 16 h + 4 kk + u.  v_mfma_f32_16x16x32_bf16 takes as long as its 16-deep form (16 cycles of the pipe): see mfma_tile_b3.
// 16-deep steps (DEEP = false) read one of the two at a time and have each in a piece of its own.
template <int DG, bool DEEP>
struct WLdsB3 {
    alignas(16) uint64_t w[3][DEEP ? DG / 32 : DG / 16][DG / 16][64][DEEP ? 2 : 1];
    // rows 16 s + 4 kk .. + 3
    __device__ __forceinline__ uint64_t& at(int term, int s, int cb, int lane) {
        if constexpr (DEEP) return w[term][s >> 1][cb][lane][s & 1];
        else return w[term][s][cb][lane][0];
    }
};
// whether the products of a layer in storage type T take 32 K-slots per instruction
template <typename T>
constexpr bool deep_products() { return sizeof(T) == 4; }
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ uint64_t as_u64(bf16x4 v) { return __builtin_bit_cast(uint64_t, v); }
__device__ __forceinline__ bf16x4 as_bf16x4(uint64_t v) { return __builtin_bit_cast(bf16x4, v); }
// two times four bf16 as the operand of a 32-deep step
__device__ __forceinline__ bf16x8 join8(bf16x4 h0, bf16x4 h1) {
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(h0, h1, 0, 1, 2, 3, 4, 5, 6, 7));
}
__device__ __forceinline__ f32x4 mfma_k32(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }

template <int DG, bool DEEP>
__device__ __forceinline__ void load_w_lds_b3(const float* __restrict__ w, int ldw, bool transposed, WLdsB3<DG, DEEP>& l) {
    constexpr int CPL = DG / 16, NB = DG / 16;
    // (the loads of two of a thread's items in flight at a time, as in load_w_lds; not for the transposed form)
    constexpr int NI = 2, ITEMS = NB * NB * 64;
    const int nt = blockDim.x;
    if (transposed) {
        for (int e = threadIdx.x; e < ITEMS; e += nt) {
            const int lane = e & 63, cb = (e >> 6) % NB, s = (e >> 6) / NB;
            const int kk = lane >> 4, j = lane & 15, col = CPL * j + cb;
            float v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = w[col * ldw + 16 * s + 4 * kk + u];
            bf16x4 hi, mid, lo;
            split_p4(v, hi, mid, lo);
            l.at(0, s, cb, lane) = as_u64(hi);
            l.at(1, s, cb, lane) = as_u64(mid);
            l.at(2, s, cb, lane) = as_u64(lo);
        }
        __syncthreads();
        return;
    }
    for (int e0 = threadIdx.x; e0 < ITEMS; e0 += NI * nt) {
        float v[NI][4];
#pragma unroll
        for (int t = 0; t < NI; ++t) {
            const int e = e0 + t * nt < ITEMS ? e0 + t * nt : 0;
            const int lane = e & 63, cb = (e >> 6) % NB, s = (e >> 6) / NB;
            const int kk = lane >> 4, j = lane & 15, col = CPL * j + cb;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int row = 16 * s + 4 * kk + u;
                v[t][u] = w[row * ldw + col];
            }
        }
#pragma unroll
        for (int t = 0; t < NI; ++t) {
            const int e = e0 + t * nt;
            if (e < ITEMS) {
                const int lane = e & 63, cb = (e >> 6) % NB, s = (e >> 6) / NB;
                bf16x4 hi, mid, lo;
                split_p4(v[t], hi, mid, lo);
                l.at(0, s, cb, lane) = as_u64(hi);
                l.at(1, s, cb, lane) = as_u64(mid);
                l.at(2, s, cb, lane) = as_u64(lo);
            }
        }
    }
    __syncthreads();
}

__device__ __forceinline__ bf16x4 half8(bf16x8 v, int h) {
    return __builtin_bit_cast(bf16x4, h == 0 ? __builtin_shufflevector(v, v, 0, 1, 2, 3) : __builtin_shufflevector(v, v, 4, 5, 6, 7));
}

// acc[cb] += the six products of one 32-deep step with W's blocks cb, smallest terms first; two column blocks in turn, so that no
// instruction waits for the one before it.  Not DEEP: as two 16-deep steps.
template <int DG, bool DEEP>
__device__ __forceinline__ void mfma_b3(bf16x8 ah, bf16x8 am, bf16x8 al, const WLdsB3<DG, DEEP>& wl, int s, int lane, f32x4 (&acc)[DG / 16]) {
    if constexpr (DEEP) {
#pragma unroll
        for (int c0 = 0; c0 < DG / 16; c0 += 2) {
            bf16x8 bh[2], bm[2], bl[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                bh[c] = *reinterpret_cast<const bf16x8*>(wl.w[0][s][c0 + c][lane]);
                bm[c] = *reinterpret_cast<const bf16x8*>(wl.w[1][s][c0 + c][lane]);
                bl[c] = *reinterpret_cast<const bf16x8*>(wl.w[2][s][c0 + c][lane]);
            }
            auto both = [&](bf16x8 a, const bf16x8 (&b)[2]) {
#pragma unroll
                for (int c = 0; c < 2; ++c) acc[c0 + c] = mfma_k32(a, b[c], acc[c0 + c]);
            };
            both(al, bh); both(ah, bl); both(am, bm); both(am, bh); both(ah, bm); both(ah, bh);
        }
    } else {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int cb = 0; cb < DG / 16; ++cb) {
                const bf16x4 bh = as_bf16x4(wl.w[0][2 * s + h][cb][lane][0]), bm = as_bf16x4(wl.w[1][2 * s + h][cb][lane][0]),
                             bl = as_bf16x4(wl.w[2][2 * s + h][cb][lane][0]);
                auto add = [&](bf16x8 a, bf16x4 b) { acc[cb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(half8(a, h), b, acc[cb], 0, 0, 0); };
                add(al, bh); add(am, bm); add(ah, bl); add(am, bh); add(ah, bm); add(ah, bh);
            }
    }
}

// acc = tile (16 x DG float32, LDS, row stride tile_ld) * W, in the tile register layout of mfma_tile.
template <int DG, bool DEEP>
__device__ __forceinline__ void mfma_tile_b3(const float* st, const WLdsB3<DG, DEEP>& wl, f32x4 (&acc)[DG / 16]) {
    constexpr int CPL = DG / 16;
    const int lane = lane_id(), i = lane & 15, kk = lane >> 4;
    const int arow = 4 * (i & 3) + (i >> 2);
#pragma unroll
    for (int cb = 0; cb < CPL; ++cb) acc[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < DG / 32; ++s) {
        float a[8];
        lds_load<4>(st + arow * tile_ld<DG>() + 32 * s + 4 * kk, *reinterpret_cast<float(*)[4]>(&a[0]));
        lds_load<4>(st + arow * tile_ld<DG>() + 32 * s + 16 + 4 * kk, *reinterpret_cast<float(*)[4]>(&a[4]));
        bf16x4 ah[2], am[2], al[2];
        split_p4(a, ah[0], am[0], al[0]);
        split_p4(a + 4, ah[1], am[1], al[1]);
        mfma_b3<DG, DEEP>(join8(ah[0], ah[1]), join8(am[0], am[1]), join8(al[0], al[1]), wl, s, lane, acc);
        if constexpr (DEEP) __builtin_amdgcn_sched_barrier(0);      // (the next step's operands requested beside this one's: a register spilled in three variants)
    }
}

// dW += H^T dY over the 16 rows of the tile, as mfma_outer, on the bf16 pipe.  The 16 rows are half of the 32 K-slots of one
// instruction, so an instruction takes two of the six products at once: slot 4 kk + u of either half stands for tile row 4 u + kk, so
// that the B operand of lane (kk, j) is what the lane already holds of dY (gy[u][ob], rows 4 u + kk) and the A operand is
// H[4 u + kk][16 mb + j] from the LDS tile.  Pairs: (lo hi, mid mid), (mid hi, hi mid), (hi lo, hi hi).  Rows of dY held in 16 bits
// (T) are their own first term and have no others: lo hi, mid hi and hi hi one by one, the rows 16 deep (see mfma_tile_b3).
template <int DG, typename T>
__device__ __forceinline__ void mfma_outer_b3(const float* st_h, const float (&gy)[4][DG / 16], f32x4 (&acc)[DG / 16][DG / 16]) {
    const int lane = lane_id(), kk = lane >> 4, j = lane & 15;
    constexpr bool EXACT = sizeof(T) == 2;
    bf16x4 bh[DG / 16], bm[DG / 16], bl[DG / 16];
#pragma unroll
    for (int ob = 0; ob < DG / 16; ++ob) {
        const float b[4] = {gy[0][ob], gy[1][ob], gy[2][ob], gy[3][ob]};
        if constexpr (EXACT) bh[ob] = pack_upper4(__float_as_uint(b[0]), __float_as_uint(b[1]), __float_as_uint(b[2]), __float_as_uint(b[3]));
        else split_p4(b, bh[ob], bm[ob], bl[ob]);
    }
#pragma unroll
    for (int mb = 0; mb < DG / 16; ++mb) {
        float a[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] = st_h[(4 * u + kk) * tile_ld<DG>() + 16 * mb + j];
        bf16x4 ah, am, al;
        split_p4(a, ah, am, al);
        if constexpr (EXACT) {
#pragma unroll
            for (int ob = 0; ob < DG / 16; ++ob) acc[mb][ob] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(al, bh[ob], acc[mb][ob], 0, 0, 0);
#pragma unroll
            for (int ob = 0; ob < DG / 16; ++ob) acc[mb][ob] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(am, bh[ob], acc[mb][ob], 0, 0, 0);
#pragma unroll
            for (int ob = 0; ob < DG / 16; ++ob) acc[mb][ob] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ah, bh[ob], acc[mb][ob], 0, 0, 0);
        } else {
#pragma unroll
            for (int ob = 0; ob < DG / 16; ++ob) acc[mb][ob] = mfma_k32(join8(al, am), join8(bh[ob], bm[ob]), acc[mb][ob]);
#pragma unroll
            for (int ob = 0; ob < DG / 16; ++ob) acc[mb][ob] = mfma_k32(join8(am, ah), join8(bh[ob], bm[ob]), acc[mb][ob]);
#pragma unroll
            for (int ob = 0; ob < DG / 16; ++ob) acc[mb][ob] = mfma_k32(join8(ah, ah), join8(bl[ob], bh[ob]), acc[mb][ob]);
        }
    }
}

// dW += H^T dY over the 16 rows of the tile: D[m][o] += sum_n H[n][m] dY[n][o], on the float32 matrix instructions.  H comes
// from the LDS tile; dY is held in the tile register layout (gy[reg][cb] = dY[row 4 reg + lane / 16]
// [column CPL (lane % 16) + cb]), which is the B operand as it stands.  The result has its
// columns interleaved the same way: acc[mb][ob][r] = dW[16 mb + 4 (lane / 16) + r][CPL (lane % 16) + ob].
// The sixteen rows are summed from zero and join the accumulators in one vector addition: the matrix instructions of this
// chip leave more error in a long sum than additions rounded to nearest do, the 16-bit ones most.  Error of dW against
// 64 bits, 200k rows, groups of 128: 6.3e-7 as mfma_outer_b3 over the same tiles, 3.4e-7 with the accumulators as the
// instructions' own, 2.8e-7 this way.
template <int DG>
__device__ __forceinline__ void mfma_outer(const float* st_h, const float (&gy)[4][DG / 16], f32x4 (&acc)[DG / 16][DG / 16]) {
    const int lane = lane_id();
#pragma unroll
    for (int mb = 0; mb < DG / 16; ++mb) {
        float a[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) a[ks] = st_h[(4 * ks + (lane >> 4)) * tile_ld<DG>() + 16 * mb + (lane & 15)];
#pragma unroll
        for (int ob = 0; ob < DG / 16; ++ob) {
            f32x4 t = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) t = __builtin_amdgcn_mfma_f32_16x16x4f32(a[ks], gy[ks][ob], t, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[mb][ob][r] += t[r];
        }
    }
}

// ---- GS of a 16-row tile --------------------------------------------------------------------------
// Compressed record of a row ("CBSR" of Section 4.3): the k kept values in ascending column
// order (already RMS-scaled) and the row's column bit mask.  Where more than half of the columns are kept a record is held as
// the row itself, zeros in the dropped columns (cols == NULL; see records_as_rows).
template <int DG, typename T>
struct Record {
    using M = typename MaskOf<DG>::type;
    T* vals;        // [n][k], or [n][DG] as rows
    M* mask;        // [n]
    uint8_t* cols;  // [n][k]: column of every value
};

// ---- the k-th largest key of a row when k is a quarter of its width -------------------------------
// (k = 16 of 64 columns, k = 8 of 32: the shapes of the benchmark configurations.)  A selection network of fixed
// cost instead of a search whose length depends on the data (Section 4.1: the k largest entries of a row).
// Lane (r, q) holds QW = k keys of row r.
//   1. every lane sorts its keys (Batcher's odd-even merge sort): even quarters descending, odd quarters ascending
//      in register order;
//   2. quarters (0,1) and (2,3): u[i] = max(even[i], odd[i]) pairs the i-th largest of one with the i-th smallest of
//      the other, so u is the set of the k largest of the two quarters, and a bitonic sequence; the even lane keeps
//      u[0 .. k/2), the odd lane the rest;
//   3. a bitonic merge sorts u over the two lanes: quarters (0,1) descending, quarters (2,3) ascending;
//   4. the same pairing over the halves leaves the k largest of the whole row; their minimum is the answer.
// A compare-exchange whose direction depends on the lane is two v_med3_u32 with a third operand of all ones
// (the median is then the larger of the two) or zero (the smaller).
constexpr int SORT8[19][2] = {{0, 1}, {2, 3}, {4, 5}, {6, 7}, {0, 2}, {1, 3}, {4, 6}, {5, 7}, {1, 2}, {5, 6},
                              {0, 4}, {1, 5}, {2, 6}, {3, 7}, {2, 4}, {3, 5}, {1, 2}, {3, 4}, {5, 6}};
constexpr int SORT16[63][2] = {
    {0, 1}, {2, 3}, {4, 5}, {6, 7}, {8, 9}, {10, 11}, {12, 13}, {14, 15}, {0, 2}, {1, 3}, {4, 6}, {5, 7}, {8, 10},
    {9, 11}, {12, 14}, {13, 15}, {1, 2}, {5, 6}, {9, 10}, {13, 14}, {0, 4}, {1, 5}, {2, 6}, {3, 7}, {8, 12}, {9, 13},
    {10, 14}, {11, 15}, {2, 4}, {3, 5}, {10, 12}, {11, 13}, {1, 2}, {3, 4}, {5, 6}, {9, 10}, {11, 12}, {13, 14}, {0, 8},
    {1, 9}, {2, 10}, {3, 11}, {4, 12}, {5, 13}, {6, 14}, {7, 15}, {4, 8}, {5, 9}, {6, 10}, {7, 11}, {2, 4}, {3, 5},
    {6, 8}, {7, 9}, {10, 12}, {11, 13}, {1, 2}, {3, 4}, {5, 6}, {7, 8}, {9, 10}, {11, 12}, {13, 14}};

__device__ __forceinline__ uint32_t med3_u32(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t d;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}
// a <- the larger of (a, b) where up is all ones, the smaller where it is zero; b <- the other one
__device__ __forceinline__ void compare_exchange(uint32_t& a, uint32_t& b, uint32_t up) {
    const uint32_t hi = med3_u32(a, b, up), lo = med3_u32(a, b, ~up);
    a = hi; b = lo;
}

template <int QW>
__device__ __forceinline__ uint32_t kth_largest_quarter(const uint32_t (&key)[QW], int q) {
    static_assert(QW == 8 || QW == 16, "selection network for 8 or 16 keys per lane");
    constexpr int H = QW / 2, NCE = QW == 16 ? 63 : 19;
    uint32_t s[QW];
#pragma unroll
    for (int j = 0; j < QW; ++j) s[j] = key[j];
    const uint32_t up1 = (q & 1) ? 0u : 0xFFFFFFFFu;
#pragma unroll
    for (int c = 0; c < NCE; ++c) {
        if constexpr (QW == 16) compare_exchange(s[SORT16[c][0]], s[SORT16[c][1]], up1);
        else compare_exchange(s[SORT8[c][0]], s[SORT8[c][1]], up1);
    }
    uint32_t t[H];
#pragma unroll
    for (int i = 0; i < H; ++i) {
        const auto a = __builtin_amdgcn_permlane16_swap(s[i], s[i + H], false, false);
        t[i] = max(a[0], a[1]);
    }
    const uint32_t up3 = (q == 0 || q == 3) ? 0xFFFFFFFFu : 0u, upl = q < 2 ? 0xFFFFFFFFu : 0u;
#pragma unroll
    for (int i = 0; i < H; ++i) {
        const auto a = __builtin_amdgcn_permlane16_swap(t[i], t[i], false, false);
        t[i] = med3_u32(a[0], a[1], up3);
    }
#pragma unroll
    for (int d = H / 2; d >= 1; d >>= 1) {
#pragma unroll
        for (int i = 0; i < H; ++i)
            if ((i & d) == 0) compare_exchange(t[i], t[i + d], upl);
    }
    uint32_t m = 0xFFFFFFFFu;
#pragma unroll
    for (int i = 0; i < H / 2; ++i) {
        const auto a = __builtin_amdgcn_permlane32_swap(t[i], t[i + H / 2], false, false);
        m = min(m, max(a[0], a[1]));
    }
    const auto a = __builtin_amdgcn_permlane16_swap(m, m, false, false);
    const uint32_t m2 = min(a[0], a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(m2, m2, false, false);
    return min(b[0], b[1]);
}

// Bits of the quarter's columns that belong to the row's k largest entries (x: the quarter's QW
// values; valid: the row exists; q: the quarter).  All four lanes of a row must call it together.
template <int DG, int KS>
__device__ __forceinline__ uint32_t select_quarter(const float (&x)[DG / 4], int k, bool valid, int q) {
    constexpr int QW = DG / 4;
    uint32_t key[QW];
#pragma unroll
    for (int j = 0; j < QW; ++j) {
        const uint32_t u = __float_as_uint(x[j] + 0.0f);    // -0 -> +0, every other value as it is
        const uint32_t kk = u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
        key[j] = kk >> KS;
    }
    uint32_t lo;
    if (k == QW) {
        lo = kth_largest_quarter<QW>(key, q);          // the k-th largest key itself
    } else {
        uint32_t top = 0u;
#pragma unroll
        for (int j = 0; j < QW; ++j) top = max(top, key[j]);
        top = quarter_max(top);
        auto count_ge = [&](uint32_t t) {
            uint32_t cnt = 0u;
#pragma unroll
            for (int j = 0; j < QW; ++j) cnt += key[j] >= t ? 1u : 0u;
            return quarter_sum(cnt);
        };
        constexpr uint32_t span = (4u << 23) >> KS;
        const uint32_t uk = (uint32_t)k;
        uint32_t hi = top + 1u;
        lo = top > span ? top - span : 0u;
        const uint32_t cnt = count_ge(lo);
        lo = (cnt >= uk && k < DG) ? lo : 0u;
        uint32_t open = (cnt != uk && k < DG && valid) ? 1u : 0u;
        for (int round = 0; round < 33 && ballot(open != 0u) != 0ull; ++round) {
            const uint32_t mid = lo + ((hi - lo) >> 1);
            const uint32_t c2 = count_ge(mid);
            lo = c2 >= uk ? mid : lo;
            hi = c2 >= uk ? hi : mid;
            open = (c2 == uk || hi - lo <= 1u) ? 0u : open;
        }
    }
    // Column set of this quarter at or above the threshold, built as a shift register (a compare and an add with
    // carry per key).  It is the answer unless the row has more than k keys there: then several keys equal the
    // threshold (which is a key of the row in that case) and the lowest columns among them win.
    uint32_t mge = 0u;
#pragma unroll
    for (int j = QW - 1; j >= 0; --j) mge = mge + mge + (key[j] >= lo ? 1u : 0u);
    uint32_t msel = mge;
    if (ballot(quarter_sum((uint32_t)__popc(mge)) != (uint32_t)k) != 0ull) {
        uint32_t mgt = 0u;
#pragma unroll
        for (int j = QW - 1; j >= 0; --j) mgt = mgt + mgt + (key[j] > lo ? 1u : 0u);
        const uint32_t meq = mge & ~mgt;
        const uint32_t cg = __popc(mgt), ce = __popc(meq);
        uint32_t all[4];
        quarter_all(cg | ce << 8, all);
        const int need = k - (int)((all[0] & 255u) + (all[1] & 255u) + (all[2] & 255u) + (all[3] & 255u));
        int before = 0;   // ties in lower quarters
#pragma unroll
        for (int i = 0; i < 3; ++i) before += i < q ? (int)(all[i] >> 8) : 0;
        int take = min(max(need - before, 0), (int)ce);
        msel = mgt;
#pragma unroll
        for (int j = 0; j < QW; ++j) {
            const uint32_t s1 = ((meq >> j) & 1u) & (take > 0 ? 1u : 0u);
            msel |= s1 << j;
            take -= (int)s1;
        }
    }
    return msel;
}

// Rows whose column set is kept because they selected at a near-tie (a selective form of the save of Section 4.2):
// one segment per application of GS in the forward sweep.  A row is listed iff k < DG and, with v_k the smallest
// kept and v_(k+1) the largest dropped value, v_k - v_(k+1) <= tol * max|row| in float32 (exact ties always are).
// The inverse sweep selects again on the rebuilt rows and then gives the listed rows their kept sets back.
// The list of a segment is kept as TIE_SUB sub-lists, each with its own counter on its own cache line: a tile appends
// to sub-list (tile number mod TIE_SUB).  (All appends of a launch on one counter - 15 thousand at 1M rows - are served
// one after the other by the memory side: 36 us on a 172 us kernel.)
constexpr int TIE_SUB = 16, TIE_COUNTER_STRIDE = 32;
template <int DG>
struct TieSeg {
    using M = typename MaskOf<DG>::type;
    int* count;        // [TIE_SUB] counters, TIE_COUNTER_STRIDE ints apart: rows listed so far in each sub-list (may run
                       // past cap: the excess is not kept); NULL: nothing is listed
    uint32_t* rows;    // [TIE_SUB][cap]
    M* masks;          // [TIE_SUB][cap]
    int cap;           // places per sub-list
    float tol;
};

// The rows of a tile that a list names get the column sets kept with them instead of what the search found (see TieSeg), where the
// record is taken: the tile's sub-list has few rows on a graph with few tiles per wave (a few dozen on 100k nodes), and its first 64 are
// requested ahead with its length.  (As a launch after the record's, 4 us on 2,000 nodes and 6 us on 100k.)  Every tile walks its whole
// sub-list, so with room for more than TIE_FIX_MOST rows there the launch stays.  Steps of four layers, two groups of 64, every row at a near-tie
// so that the lists are full, launch / here, us: 30k nodes, 491 places per sub-list 648 / 625, 1,875 places 662 / 672; 60k, 182 places 871 / 854,
// 725 places 872 / 888; 100k, 260 places 1,216 / 1,209, 1,038 places 1,225 / 1,286, 6,250 places 1,298 / 1,759.
constexpr int TIE_FIX_MOST = 320;
template <int DG, bool ON>
struct TieFix {
    TieSeg<DG> seg;
    int sub, tile, lane, listed;
    uint32_t first;
    __device__ __forceinline__ TieFix(const TieSeg<DG>& s, int t, int l) : seg(s), sub(t & (TIE_SUB - 1)), tile(t), lane(l), listed(0), first(0u) {
        if constexpr (ON) {
            if (seg.count) {
                listed = seg.count[sub * TIE_COUNTER_STRIDE];
                first = seg.rows[(size_t)sub * seg.cap + (lane < seg.cap ? lane : seg.cap - 1)];
            }
        }
    }
    // msel: the bits of this lane's quarter q of row r
    __device__ __forceinline__ void apply(uint32_t& msel, int r, int q) const {
        if constexpr (ON) {
            if (!seg.count) return;
            constexpr int QW = DG / 4;
            const int n = min(__builtin_amdgcn_readfirstlane(listed), seg.cap);
            for (int e0 = 0; e0 < n; e0 += 64) {
                const int e = e0 + lane;
                const uint32_t row = e0 == 0 ? first : seg.rows[(size_t)sub * seg.cap + (e < n ? e : n - 1)];
                uint64_t hits = ballot(e < n && (int)(row >> 4) == tile);
                while (hits != 0ull) {
                    const int l = __builtin_ctzll(hits);
                    hits &= hits - 1;
                    const typename MaskOf<DG>::type m = seg.masks[(size_t)sub * seg.cap + e0 + l];
                    if (r == (int)(__builtin_amdgcn_readlane(row, l) & 15u)) msel = (uint32_t)(m >> (QW * q)) & ((1u << QW) - 1u);
                }
            }
        }
    }
};

// The factor GS applies to the kept values of a row held in the quarter layout (x: this lane's quarter); the same
// value in the four lanes of the row.
template <int DG>
__device__ __forceinline__ float record_scale(const float (&x)[DG / 4], int norm, float eps) {
    float scale = 1.f;
    if (norm == GSR_NORM_RMS) {
        float ss = 0.f;
#pragma unroll
        for (int j = 0; j < DG / 4; ++j) ss += x[j] * x[j];
        ss = quarter_sum(ss);
        scale = __builtin_amdgcn_rsqf(ss * (1.0f / (float)DG) + eps);
    }
    return scale;
}

// GS of the 16 rows of an LDS tile and their records (Section 4.1; record layout of Section 4.3).
// st holds the rows as they read back from memory (16 x tile_ld floats, rows past the end zero).
// Lane (r, q) takes the quarter q of row r into registers, so the 16 searches for the k-th largest
// key run side by side in vector registers on an order-preserving integer image of the values
// (select_quarter): a selection network when k is a quarter of the width, else interval bisection,
// count = own compares + the three partner quarters.  Invariant per row of the bisection: at
// least k keys are >= lo and fewer than k are >= hi; hi starts just above the row maximum, lo four
// binades below it (0 when a count says that is too high).  A row closes when a candidate splits
// off exactly k keys or the interval is down to one value (a tie at the k-th position); ties go
// to the lowest columns, -0 equals +0.  The kept values (RMS-scaled) are compacted in LDS in
// column order and leave as one contiguous block, since rows r0..r0+15 are adjacent in [n][k].
// With `given` the column set is not searched for: out.mask already holds the set an earlier
// application selected (Section 4.2 keeps the indices of the forward pass) and only the values
// are taken, from the present rows.  st is overwritten.  With idx_out (and ist, 16 * DG words of
// LDS scratch) the kept column numbers are written as well, [n][k] in ascending order, and
// out.mask may be NULL.  FORM says what leaves: the values, the values and their columns as bytes ([n][k] like the values),
// or the row with zeros in the dropped columns.
// Floats of LDS emit_tile works with: the tile, 64 dump words, and with columns a byte for every one of those.
enum RecordForm { REC_VALUES, REC_COLUMNS, REC_ROWS };
template <int DG, RecordForm FORM>
constexpr int emit_floats() { return (16 * tile_ld<DG>() + 64) + (FORM == REC_COLUMNS ? (16 * tile_ld<DG>() + 64) / 4 : 0); }

template <int DG, typename T, RecordForm FORM = REC_VALUES, typename Fix = TieFix<DG, false>>
__device__ __forceinline__ void emit_tile(float* st, int r0, int n, int k, int norm, float eps, const Record<DG, T>& out,
                                          bool given, int lane, int32_t* idx_out = nullptr, int* ist = nullptr,
                                          TieSeg<DG> tie = TieSeg<DG>{nullptr, nullptr, nullptr, 0, 0.f},
                                          const Fix& fix = Fix(TieSeg<DG>{nullptr, nullptr, nullptr, 0, 0.f}, 0, 0)) {
    using M = typename MaskOf<DG>::type;
    constexpr int QW = DG / 4, LR = tile_ld<DG>();
    constexpr int KS = sizeof(T) == 2 ? 16 : 0;   // bf16 values: the low 16 key bits are zero
    const int r = lane & 15, q = lane >> 4;
    float x[QW];
    lds_load<QW>(st + r * LR + q * QW, x);
    uint32_t msel;
    if (given) {
        const M m = out.mask[r0 + r < n ? r0 + r : n - 1];
        msel = (uint32_t)(m >> (QW * q)) & ((1u << QW) - 1u);
    } else {
        msel = select_quarter<DG, KS>(x, k, r0 + r < n, q);
        fix.apply(msel, r, q);
    }
    uint32_t all[4];
    quarter_all(msel | (uint32_t)__popc(msel) << 16, all);
    int slot = r * k;
#pragma unroll
    for (int i = 0; i < 3; ++i) slot += i < q ? (int)(all[i] >> 16) : 0;
    M mask;
    if constexpr (DG == 64)
        mask = (M)(all[0] & 0xFFFFu) | (M)(all[1] & 0xFFFFu) << 16 | (M)(all[2] & 0xFFFFu) << 32 | (M)(all[3] & 0xFFFFu) << 48;
    else
        mask = (all[0] & 0xFFu) | (all[1] & 0xFFu) << 8 | (all[2] & 0xFFu) << 16 | (all[3] & 0xFFu) << 24;
    if (tie.count && !given) {
        // near-tie test on the row's values: smallest kept, largest dropped, largest magnitude
        float vk = __builtin_huge_valf(), vr = -__builtin_huge_valf(), am = 0.f;
#pragma unroll
        for (int j = 0; j < QW; ++j) {
            const bool bit = (msel >> j) & 1u;
            vk = bit ? fminf(vk, x[j]) : vk;
            vr = bit ? vr : fmaxf(vr, x[j]);
            am = fmaxf(am, fabsf(x[j]));
        }
        vk = quarter_fmin(vk); vr = quarter_fmax(vr); am = quarter_fmax(am);
        const float gap = vk - vr, bar = tie.tol * am;
        if (q == 0 && r0 + r < n && k < DG && gap <= bar) {
            const int sub = (r0 >> 4) & (TIE_SUB - 1);
            const int pos = atomicAdd(tie.count + sub * TIE_COUNTER_STRIDE, 1);
            if (pos < tie.cap) { tie.rows[sub * tie.cap + pos] = (uint32_t)(r0 + r); tie.masks[sub * tie.cap + pos] = mask; }
        }
    }
    const float scale = record_scale<DG>(x, norm, eps);
    const int rows = min(16, n - r0);
    if constexpr (FORM == REC_ROWS) {
        constexpr int CPL = DG / 16;
#pragma unroll
        for (int j = 0; j < QW; ++j) x[j] = (msel >> j) & 1u ? x[j] * scale : 0.f;
        lds_store<QW>(st + r * LR + q * QW, x);       // (the lane's own quarter)
        wave_sync();
#pragma unroll
        for (int reg = 0; reg < 4; ++reg) {           // four rows per store instruction
            const int rr = 4 * reg + q;
            float v[CPL];
            lds_load<CPL>(st + rr * LR + CPL * r, v);
#pragma unroll
            for (int cb = 0; cb < CPL; ++cb) v[cb] = stored<T>(v[cb]);
            if (rr < rows) store_cols<CPL, T, true>(out.vals + (size_t)(r0 + rr) * DG + CPL * r, v);
        }
        if (!given && out.mask && q == 0 && r < rows) out.mask[r0 + r] = mask;
        return;
    }
    wave_sync();   // every lane holds its quarter: the tile can be reused for the compacted values
    // a kept value goes to its slot, a dropped one to the lane's dump word: word number = dump + bit * (slot - dump)
    const int dump = 16 * LR + lane;
    uint8_t* cst = reinterpret_cast<uint8_t*>(st + 16 * LR + 64);      // (REC_COLUMNS: the column beside every word)
    int ahead = slot - dump;
#pragma unroll
    for (int j = 0; j < QW; ++j) {
        const int bit = (int)((msel >> j) & 1u);
        const int at = dump + __mul24(bit, ahead);
        st[at] = x[j] * scale;
        if constexpr (FORM == REC_COLUMNS) cst[at] = (uint8_t)(q * QW + j);
        if (idx_out && bit) ist[dump + ahead] = q * QW + j;
        ahead += bit;
    }
    wave_sync();
    const int total = rows * k;
    T* dst = out.vals + (size_t)r0 * k;
    for (int i = lane; i < total; i += 64) dst[i] = from_float<T>(st[i]);
    if constexpr (FORM == REC_COLUMNS) {        // whole words: the array is padded, and 16 k bytes per tile keep r0 * k a multiple of four
        uint32_t* dc = reinterpret_cast<uint32_t*>(out.cols + (size_t)r0 * k);
        for (int i = lane; 4 * i < total; i += 64) dc[i] = reinterpret_cast<const uint32_t*>(cst)[i];
    }
    if (idx_out)
        for (int i = lane; i < total; i += 64) idx_out[(size_t)r0 * k + i] = ist[i];
    if (!given && out.mask && q == 0 && r < rows) out.mask[r0 + r] = mask;
}

// ---- persistent row-tile schedule ---------------------------------------------------------------
// Workgroups are dealt to the 8 XCDs round-robin by the hardware; each XCD has its own L2.  Every
// XCD therefore sweeps one contiguous eighth of the row tiles, its resident waves working on
// adjacent tiles, so that neighbour records (circuit graphs connect nearby levels) stay in that L2.
struct TileSweep {
    int first, end, step;
};
__device__ __forceinline__ TileSweep tile_sweep(int tiles) {
    const int xcd = blockIdx.x & 7, local_wg = blockIdx.x >> 3, wg_per_xcd = gridDim.x >> 3;
    const int waves_per_wg = blockDim.x >> 6;
    // the wave index through readfirstlane: everything derived from the tile number then lives in scalar registers
    const int slot = local_wg * waves_per_wg + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    TileSweep t;
    const int t0 = (int)((int64_t)tiles * xcd / 8), t1 = (int)((int64_t)tiles * (xcd + 1) / 8);
    t.first = t0 + slot;
    t.end = t1;
    t.step = wg_per_xcd * waves_per_wg;
    return t;
}

// Dynamic form of the sweep.  Tiles differ a lot in cost (a few rows have hundreds of neighbours),
// and with a fixed assignment the kernel ends when the unluckiest wave does.  Here the tiles of an
// XCD's eighth are dealt to nq = TILE_NQ queues (queue q owns tiles t0 + q + nq v); a wave serves
// queue (its slot mod nq): its first tile is the one of its place among the queue's waves, every further one it draws
// from the queue's counter, so a wave that drew long rows draws fewer tiles.  (The first tile drawn as well, every
// launch began with a round trip to the counters; and where no XCD has more tiles than waves nothing is drawn at all
// and no wave signs off.)  The active window still moves through the rows in order.  Many
// queues rather than one keep the atomics on different addresses: one counter for the 512 waves
// of an XCD serialises and costs more than the balance gains.  The next draw is requested at
// the start of a tile and read at its end.  A launch leaves the counters as it found them (all
// zero): every wave signs off when it has drawn its last tile, and the wave that signs off last
// clears them (tile_finish), so launches need no clearing step and may be replayed from a
// captured graph in any number.  Which wave processes which tile varies between runs; kernels
// that sum over the tiles a wave has seen must keep the fixed sweep.
constexpr int TILE_NQ = 64, TILE_QSTRIDE = 32;              // counters sit 128 bytes apart
constexpr int TILE_COUNTERS = 8 * TILE_NQ * TILE_QSTRIDE;   // ints of the counter set (the host allocates kTileCounters)
struct TileDraws {
    int* ctr;      // this wave's queue counter
    int base;      // first tile of the queue
    int nq;        // queues in use: TILE_NQ, or the number of waves of the XCD if that is smaller
    int end;       // one past the XCD's last tile
    int* set;      // the whole counter set
    int* done;     // waves that have signed off
    int first;     // this wave's first tile
    int waves;     // waves of the queue: draw v is the queue's tile waves + v
    bool draws;    // some XCD has more tiles than waves (the same in the whole grid)
};
__device__ __forceinline__ TileDraws tile_draws(int tiles, int* set, int* done) {
    const int xcd = blockIdx.x & 7;
    const int slot = (blockIdx.x >> 3) * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = (gridDim.x >> 3) * (blockDim.x >> 6);
    TileDraws d;
    d.nq = waves < TILE_NQ ? waves : TILE_NQ;
    const int q = slot % d.nq;
    d.ctr = set + (xcd * TILE_NQ + q) * TILE_QSTRIDE;
    d.base = (int)((int64_t)tiles * xcd / 8) + q;
    d.end = (int)((int64_t)tiles * (xcd + 1) / 8);
    d.set = set;
    d.done = done;
    d.first = d.base + d.nq * (slot / d.nq);
    d.waves = (waves - q + d.nq - 1) / d.nq;
    d.draws = (tiles + 7) / 8 > waves;
    return d;
}
// requests a draw; the value is valid in lane 0 once the wave waits for it (tile_drawn)
__device__ __forceinline__ int tile_request(const TileDraws& d) {
    int v = 0;
    if (d.draws && lane_id() == 0) v = atomicAdd(d.ctr, 1);
    return v;
}
__device__ __forceinline__ int tile_drawn(const TileDraws& d, int requested) {
    return d.draws ? d.base + d.nq * (d.waves + __builtin_amdgcn_readfirstlane(requested)) : d.end;
}
// Every wave of the grid calls this once, after its last tile_drawn (all its draws have returned).
// Sign-off in two levels, an XCD's waves on the XCD's counter and the last wave of each XCD on a
// common one, keeps the atomics on one address few.  d.done: 9 counters, 128 bytes apart.
__device__ __forceinline__ void tile_finish(const TileDraws& d) {
    if (!d.draws) return;
    int last = 0;
    if (lane_id() == 0) {
        // no fence: this wave's own draws have returned, and nothing but the counters is handed over
        const int waves = (int)((gridDim.x >> 3) * (blockDim.x >> 6));
        if (atomicAdd(d.done + (blockIdx.x & 7) * TILE_QSTRIDE, 1) == waves - 1)
            last = atomicAdd(d.done + 8 * TILE_QSTRIDE, 1) == 7 ? 1 : 0;
    }
    if (__builtin_amdgcn_readfirstlane(last)) {
        for (int i = lane_id(); i < 8 * TILE_NQ; i += 64) d.set[i * TILE_QSTRIDE] = 0;
        if (lane_id() < 9) d.done[lane_id() * TILE_QSTRIDE] = 0;
    }
}

// ---- the long tiles first -----------------------------------------------------------------------------
// A tile with many stored entries takes many times longer than a median one.  Met late in a sweep it makes
// the kernel's tail; met twice by one wave of a fixed sweep it makes that wave the last.  The layer kernels
// therefore deal such tiles out first, an XCD's waves taking the listed tiles of the XCD's own eighth in turn, and
// pass them over in the sweep that follows (a tile is heavy by its row pointers alone, so the sweep
// needs no flag; the check sits after the tile's own rows have been requested, which costs a few wasted loads).
// The assignment is the same on every run.
struct TileDeal {
    int at;        // this wave's next entry of the list
    int step;      // waves of the XCD
    int end;       // one past the XCD's last entry
    bool on;       // still dealing
};
__device__ __forceinline__ TileDeal tile_deal(const CsrView& g) {
    const int xcd = blockIdx.x & 7, wpw = (int)(blockDim.x >> 6);
    TileDeal d;
    d.step = (int)(gridDim.x >> 3) * wpw;
    d.at = g.heavy_ptr[xcd] + (int)(blockIdx.x >> 3) * wpw + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    d.end = g.heavy_ptr[xcd + 1];
    d.on = d.at < d.end;
    return d;
}
__device__ __forceinline__ void tile_deal_next(TileDeal& d) {
    d.at += d.step;
    d.on = d.at < d.end;
}
// s_rp: the tile's row pointers as tile_begin published them.  Rows that are split do not count: their
// neighbours are summed by the first pass.
__device__ __forceinline__ bool tile_is_heavy(const CsrView& g, int rpv, const int* s_rp, bool has_hub) {
    int e = __builtin_amdgcn_readlane(rpv, 16) - __builtin_amdgcn_readlane(rpv, 0);   // rpv: as tile_rp_load returned it
    if (e <= g.heavy_edges) return false;
    if (has_hub)
        for (int r = 0; r < 16; ++r) {
            const int d = s_rp[r + 1] - s_rp[r];
            e -= d > g.hub_threshold ? d : 0;
        }
    return e > g.heavy_edges;
}

// Per-wave LDS of the tile operators: staged edges, the tile's row pointers.
struct TileLds {
    EdgeRec ebuf[64];
    int rp[20];
};

// The order in which a wave of these kernels visits tiles: its share of the listed heavy tiles first (DEAL, see
// TileDeal), then tiles drawn from the counters, with the next draw requested a tile ahead.  (Walking one tile
// further ahead, so that the next tile's row pointers and first edges arrive during the present tile, was
// measured on the dense product: 233 us against 224, so it is not done.)
template <bool DEAL>
struct TileWalk {
    TileDraws td;
    TileDeal deal;
    int requested, t, t_end;
    __device__ __forceinline__ TileWalk(const CsrView& g, int tiles, int* set, int* done) {
        td = tile_draws(tiles, set, done);
        deal = TileDeal{0, 0, 0, false};
        if constexpr (DEAL) deal = tile_deal(g);
        requested = 0;
        if (DEAL && deal.on) { t = g.heavy[deal.at]; t_end = tiles; }
        else { t = td.first; t_end = td.end; }
    }
    __device__ __forceinline__ bool more() const { return t < t_end; }
    // at the top of a tile: ask for the next draw (not while dealing: the sweep begins with the wave's first tile)
    __device__ __forceinline__ void ahead() { if (!DEAL || !deal.on) requested = tile_request(td); }
    // in the sweep, a heavy tile has been dealt out already
    __device__ __forceinline__ bool dealt(const CsrView& g, int rpv, const int* s_rp, bool has_hub) const {
        if constexpr (DEAL) return !deal.on && tile_is_heavy(g, rpv, s_rp, has_hub);
        return false;
    }
    __device__ __forceinline__ void next(const CsrView& g) {
        if (DEAL && deal.on) {
            tile_deal_next(deal);
            if (deal.on) { t = g.heavy[deal.at]; return; }
            t = td.first;
            t_end = td.end;
            return;
        }
        t = tile_drawn(td, requested);
    }
    __device__ __forceinline__ void finish() { tile_finish(td); }
};

// ---- first pass over the chunks of split rows ------------------------------------------------
// One wave per chunk, ordinary arithmetic.  Dense rows (hub_dense_pass: dY, the operand of gsr_spmm, records held as rows) go
// through the staging and the wide loads of the tile gathers, the chunk treated as a tile whose row 0 owns every edge
// (ONE_ROW): lane (kk, j) adds the edges kk, kk + 4, .. for its columns, and the four lane groups are added at the end.
// Records of values go a lane per value into rows of sums in LDS, four edges at a time (hub_value_rows_pass), or as many as
// their values leave lanes for (hub_values_pass).  part[chunk][DG] receives the un-scaled partial row.
struct HubChunks {
    const int32_t* ce0;
    const int32_t* ce1;
    int32_t n_chunks;
    int32_t banded = 0;      // every XCD takes a contiguous eighth of the list (hub_sweep)
    const int32_t* row = nullptr;    // the row that is all this chunk, or -1 (hub_out)
};

// Which chunks a wave takes; what a chunk's partial row holds does not depend on the wave that sums it.  The chunks
// are listed in row order and the hardware deals workgroups to the XCDs round-robin.  On a graph of long rows (nearly
// every row split, chunks alike in cost, neighbours within a few thousand rows) the sweep is banded: XCD x takes the
// x-th eighth of the list and its waves walk that eighth side by side, so the rows its L2 has to hold are the
// neighbourhood of a narrow band of rows and not that of every row in flight on the chip.  Elsewhere the split rows are
// few and unlike (a handful of rows with tens of thousands of neighbours from all over the graph, listed first, then
// rows of a few hundred): there the chunks go to the waves of the whole grid in turn, which shares the costly ones out
// (banded, the 8M-node workload's first passes took 117 us against 88).  Any grid is covered (banded with fewer than
// eight workgroups: one part each).
struct HubSweep {
    int q, end, step;
};
__device__ __forceinline__ HubSweep hub_sweep(const HubChunks& h) {
    const int wpw = (int)blockDim.x >> 6;
    HubSweep w;
    if (!h.banded) {
        w.q = (int)blockIdx.x * wpw + ((int)threadIdx.x >> 6);
        w.end = h.n_chunks;
        w.step = (int)gridDim.x * wpw;
        return w;
    }
    const int parts = gridDim.x < 8 ? (int)gridDim.x : 8;
    const int part = (int)blockIdx.x % parts, wg = (int)blockIdx.x / parts;
    const int wgs = ((int)gridDim.x - part + parts - 1) / parts;
    w.q = (int)((int64_t)h.n_chunks * part / parts) + wg * wpw + ((int)threadIdx.x >> 6);
    w.end = (int)((int64_t)h.n_chunks * (part + 1) / parts);
    w.step = wgs * wpw;
    return w;
}

struct HubLds {
    EdgeRec ebuf[64];
    int rp[20];
};
// row pointers of the pretended tile: row 0 spans [e0, e1), rows 1..15 are empty
__device__ __forceinline__ void hub_chunk_begin(HubLds& L, int e0, int e1, int lane) {
    wave_sync();
    if (lane < 17) L.rp[lane] = lane == 0 ? e0 : e1;
    wave_sync();
}
template <int DG>
__device__ __forceinline__ void hub_chunk_store(const f32x4 (&acc)[DG / 16], float* __restrict__ part, int lane) {
    constexpr int CPL = DG / 16;
    if (lane < 16) {
#pragma unroll
        for (int cb = 0; cb < CPL; ++cb) part[CPL * lane + cb] = acc[cb][0];
    }
}

// Where the sums of chunk q go: its partial row, or, with `rows`, straight to the row itself if that is all one chunk
// (h.row).  Arrays of sums are [blocks of 64 columns][chunks or n][64].
__device__ __forceinline__ float* hub_out(const HubChunks& h, float* part, float* rows, int n, int q, int block, int cols) {
    if (rows) {
        const int r = h.row[q];
        if (r >= 0) return rows + ((size_t)block * n + r) * cols;
    }
    return part + ((size_t)block * h.n_chunks + q) * cols;
}

// Records with the column of every value, any k and any width: a lane per value (gather_values_rows), lane group kk taking
// the edges kk, kk + 4, .. of the chunk into a row of sums of its own; the four rows are added at the end of the chunk.
template <int DG>
struct HubRowsLds {
    float rows[4][DG];
    float dump[64];
};
template <int DG, typename T>
__device__ __forceinline__ void hub_value_rows_pass(const CsrView& g, const HubChunks& h, const T* __restrict__ vals,
                                                    const uint8_t* __restrict__ cols, int k, int n, float* __restrict__ part,
                                                    float* __restrict__ rows, HubRowsLds<DG>& L, const HubSweep w) {
    constexpr int BC = DG < 64 ? DG : 64;
    const int lane = lane_id(), slot = lane & 15, kk = lane >> 4;
    const uint32_t row = (uint32_t)(uintptr_t)(lds_float*)&L.rows[kk][0], dump = (uint32_t)(uintptr_t)(lds_float*)&L.dump[lane];
    for (int i = lane; i < 4 * DG; i += 64) (&L.rows[0][0])[i] = 0.f;
    wave_sync();
    for (int q = w.q; q < w.end; q += w.step) {
        const int e0 = __builtin_amdgcn_readfirstlane(h.ce0[q]), e1 = __builtin_amdgcn_readfirstlane(h.ce1[q]);
        int j_next = 0;
        float a_next = 0.f;
        auto request = [&](int eb) {
            const int e = eb + 4 * slot + kk, ec = e < e1 ? e : e1 - 1;
            j_next = __builtin_nontemporal_load(g.ci + ec);
            a_next = __builtin_nontemporal_load(g.av + ec);
        };
        request(e0);
        for (int eb = e0; eb < e1; eb += 64) {
            const uint32_t off0 = (uint32_t)j_next * (uint32_t)k;
            const float a = eb + 4 * slot + kk < e1 ? a_next : 0.f;
            if (eb + 64 < e1) request(eb + 64);        // the next round's edges arrive while this one is added
            const int steps = (min(e1 - eb, 64) + 3) >> 2;
            for (int t0 = 0; t0 < k; t0 += 16) {
                const bool has = t0 + slot < k;
                const uint32_t t = (uint32_t)(has ? t0 + slot : t0);
                if (steps > 8) {
                    asm volatile("; 16 steps");       // (keeps the two apart, see gather_values_rows)
                    values_run<0, 16>(vals, cols, off0, a, row, t, has, dump, std::make_integer_sequence<int, 16>{});
                } else {
                    asm volatile("; 8 steps");
                    values_run<0, 8>(vals, cols, off0, a, row, t, has, dump, std::make_integer_sequence<int, 8>{});
                }
            }
        }
        wave_sync();
#pragma unroll
        for (int c0 = 0; c0 < DG; c0 += 64) {
            if (lane < BC) {
                const int c = c0 + lane;
                const float s = (L.rows[0][c] + L.rows[1][c]) + (L.rows[2][c] + L.rows[3][c]);
#pragma unroll
                for (int p = 0; p < 4; ++p) L.rows[p][c] = 0.f;
                hub_out(h, part, rows, n, q, c0 >> 6, BC)[lane] = s;
            }
        }
        wave_sync();
    }
}
template <int DG, typename T>
__device__ __forceinline__ void hub_dense_pass(const CsrView& g, const HubChunks& h, const T* __restrict__ x, int64_t ld,
                                               float* __restrict__ part, HubLds& L, const HubSweep w, float* __restrict__ rows = nullptr) {
    const int lane = lane_id();
    for (int q = w.q; q < w.end; q += w.step) {
        const int e0 = __builtin_amdgcn_readfirstlane(h.ce0[q]), e1 = __builtin_amdgcn_readfirstlane(h.ce1[q]);
        hub_chunk_begin(L, e0, e1, lane);
        f32x4 acc[DG / 16];
#pragma unroll
        for (int cb = 0; cb < DG / 16; ++cb) acc[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
        gather_dense_mfma<DG, T, 16, true>(g, x, ld, e0, e1, L.rp, L.ebuf, lane, acc);
#pragma unroll
        for (int cb = 0; cb < DG / 16; ++cb) acc[cb][0] = quarter_sum(acc[cb][0]);
        hub_chunk_store<DG>(acc, hub_out(h, part, rows, 0, q, 0, DG), lane);
    }
}

template <int DG, typename T>
__global__ __launch_bounds__(256) void k_hub_records(CsrView g, HubChunks h, Record<DG, T> in, int k, float* __restrict__ part) {
    __shared__ HubRowsLds<DG> lds[4];
    hub_value_rows_pass<DG, T>(g, h, in.vals, in.cols, k, 0, part, nullptr, lds[threadIdx.x >> 6], hub_sweep(h));
}

template <int DG, typename T>
__global__ __launch_bounds__(256) void k_hub_dense(CsrView g, HubChunks h, const T* __restrict__ x, int64_t ld,
                                                   float* __restrict__ part, float* __restrict__ rows = nullptr) {
    __shared__ HubLds lds[4];
    hub_dense_pass<DG, T>(g, h, x, ld, part, lds[threadIdx.x >> 6], hub_sweep(h), rows);
}

// Both first passes of one block's backward in one launch: blockIdx.y = 0 takes the records over A (for the
// inverse), blockIdx.y = 1 the dense gradient rows over A^T (for the data gradient).
template <int DG, typename T>
__global__ __launch_bounds__(256) void k_hub_both(CsrView ga, HubChunks ha, Record<DG, T> in, int k, float* __restrict__ part_a,
                                                  CsrView gt, HubChunks ht, const T* __restrict__ x, int64_t ld,
                                                  float* __restrict__ part_t) {
    union Lds { HubLds dense; HubRowsLds<DG> rows; };
    __shared__ Lds lds[4];
    Lds& L = lds[threadIdx.x >> 6];
    const bool rec = blockIdx.y == 0;
    if (rec && in.cols) hub_value_rows_pass<DG, T>(ga, ha, in.vals, in.cols, k, 0, part_a, nullptr, L.rows, hub_sweep(ha));
    else                                              // (or records held as rows)
        hub_dense_pass<DG, T>(rec ? ga : gt, rec ? ha : ht, rec ? in.vals : x, rec ? DG : ld, rec ? part_a : part_t, L.dense,
                              hub_sweep(rec ? ha : ht));
}

// The records of a group of S column blocks
template <int S, typename T>
__global__ __launch_bounds__(256) void k_hub_records_wide(CsrView g, HubChunks h, const T* __restrict__ vals, const uint8_t* __restrict__ cols,
                                                          int k, int n, float* __restrict__ part, float* __restrict__ rows) {
    __shared__ HubRowsLds<64 * S> lds[4];
    hub_value_rows_pass<64 * S, T>(g, h, vals, cols, k, n, part, rows, lds[threadIdx.x >> 6], hub_sweep(h));
}

// ---- first pass over the chunks of a graph of long rows, value by value (float32 records) -----------------
// There nearly every row is split and the first pass is the step.  As hub_value_rows_pass, but with as many lanes per edge
// as the record has values, LPE = 2^LG: lane t of them loads value t (+ LPE, + 2 LPE .. below k) and its column and adds
// a_ij * value to that column of its edge place's row in LDS (64 / LPE places, each a row of DG floats; the places of one
// instruction are different rows and the values of one record different columns, so no two lanes meet): the sum is read,
// added to and written back by the lane, and stays in the row for the whole chunk.  Even and odd instructions of a batch
// keep rows of their own, so two such chains are in flight.  At the end of a chunk the rows of the places are added in
// place order and cleared.  Scattering into zeroed rows, reading them back sixteen bytes wide into running sums and
// clearing them again was 3 % slower; LDS float atomics were four times slower (one such instruction takes some 140
// cycles).  The loads of a whole round of 64 edges are in flight together where k <= 16, and the next round's edges before
// them (50k nodes of mean degree 236, 192 columns: k = 16 170 -> 162 us per launch, k = 51 226 -> 210); what is left is the
// LDS pipe, where the sums of unrelated columns collide on banks.  The order of the additions is fixed by the edge list and
// the lane layout.
template <int DG, int LG>
struct HubValLds {
    uint2 ebuf[64];                   // (j * k, a_ij) of the staged edges
    float rows[2][(64 >> LG) * DG];   // two rows of sums per edge place (even and odd instructions of a batch)
    float spare[64];                  // where a lane without a value adds its zero
};

template <int DG, int LG, int KQ>
__device__ __forceinline__ void hub_values_pass(const CsrView& g, const HubChunks& h, const float* __restrict__ vals,
                                                const uint8_t* __restrict__ cols, int k, int n, float* __restrict__ part,
                                                float* __restrict__ rows, HubValLds<DG, LG>& L, const HubSweep w) {
    constexpr int LPE = 1 << LG, NE = 64 >> LG;          // lanes per edge, edges per instruction
    constexpr int MAXS = 64 / NE;                        // instructions per round of 64 staged edges
    constexpr int GB = KQ == 1 ? MAXS : MAXS / KQ;       // instructions whose loads are in flight together
    constexpr int TOT = NE * DG;
    static_assert(MAXS % GB == 0 && GB % 2 == 0, "a round is a whole number of batches, a batch of pairs");
    const int lane = lane_id();
    const int place = lane >> LG, t = lane & (LPE - 1);
    float* base = &L.rows[0][0];
    const int spare = (int)(&L.spare[lane] - base);
    for (int i = lane; i < 2 * TOT; i += 64) base[i] = 0.f;
    for (int q = w.q; q < w.end; q += w.step) {
        const int e0 = __builtin_amdgcn_readfirstlane(h.ce0[q]), e1 = __builtin_amdgcn_readfirstlane(h.ce1[q]);
        // places past the last edge: the last edge once more with a_ij = 0
        // (with sixteen lanes per edge a place is a row of sixteen lanes, and an instruction could take its edge
        // from a lane of the row by a DPP row broadcast instead of from LDS: measured 2.5 % slower)
        uint32_t j_next = 0;
        float a_next = 0.f;
        auto request = [&](int eb) {
            const int e = eb + lane, ec = e < e1 ? e : e1 - 1;
            j_next = (uint32_t)__builtin_nontemporal_load(g.ci + ec);
            const float av = __builtin_nontemporal_load(g.av + ec);
            a_next = e < e1 ? av : 0.f;
        };
        request(e0);
        for (int eb = e0; eb < e1; eb += 64) {
            wave_sync();          // readers of the previous round are done
            L.ebuf[lane] = make_uint2(j_next * (uint32_t)k, __float_as_uint(a_next));
            wave_sync();
            const int cnt = e1 - eb < 64 ? e1 - eb : 64;
            const int need = (cnt + NE - 1) / NE;
            if (eb + 64 < e1) request(eb + 64);        // the next round's edges arrive while this one is added
            // NB instructions from s0 on: all loads first
            auto batch = [&](auto nbc, int s0) {
                constexpr int NB = decltype(nbc)::value;
                asm volatile("; %0 steps" ::"n"(NB));        // (keeps the variants apart, see gather_values_rows)
                float v[NB][KQ], a[NB];
                uint32_t c[NB][KQ];
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    const uint2 er = L.ebuf[(s0 + u) * NE + place];
                    a[u] = __uint_as_float(er.y);
#pragma unroll
                    for (int w = 0; w < KQ; ++w) {
                        // (a lane past the record's last slot takes slot 0 again: with one value per lane it writes
                        // what slot 0's lane writes)
                        const int tt = t + w * LPE;
                        const uint32_t at = er.x + (uint32_t)(tt < k ? tt : 0);
                        v[u][w] = vals[at];
                        c[u][w] = cols[at];
                    }
                }
                // sum += value, read and written back: the lanes of an instruction hold different places or different
                // columns of one record, so no two of them meet; even and odd instructions keep rows of their own so
                // that two read - add - write chains are in flight
                wave_sync();
#pragma unroll
                for (int u = 0; u < NB; u += 2) {
#pragma unroll
                    for (int w = 0; w < KQ; ++w) {
                        const bool has = KQ == 1 || t + w * LPE < k;      // (else slot 0 once more: not added again)
                        const int i0 = has ? place * DG + (int)c[u][w] : spare;
                        const int i1 = has ? TOT + place * DG + (int)c[u + 1][w] : spare;
                        const float o0 = base[i0];
                        const float o1 = base[i1];
                        wave_sync();
                        base[i0] = o0 + (has ? v[u][w] * a[u] : 0.f);
                        base[i1] = o1 + (has ? v[u + 1][w] * a[u + 1] : 0.f);
                        wave_sync();
                    }
                }
            };
            if constexpr (GB >= 8) {
                for (int s0 = 0; s0 < need; s0 += GB) {
                    if (need - s0 > GB / 2) batch(std::integral_constant<int, GB>{}, s0);
                    else batch(std::integral_constant<int, GB / 2>{}, s0);
                }
            } else {
                for (int s0 = 0; s0 < need; s0 += GB) batch(std::integral_constant<int, GB>{}, s0);
            }
        }
        // the sums of the places are added in place order, even rows before odd rows, and the rows cleared
        wave_sync();
#pragma unroll
        for (int c0 = 0; c0 < DG; c0 += 64) {
            const int c = c0 + lane;
            if (c < DG) {
                float s = 0.f;
#pragma unroll
                for (int pl = 0; pl < 2 * NE; ++pl) {
                    s += base[pl * DG + c];
                    base[pl * DG + c] = 0.f;
                }
                hub_out(h, part, rows, n, q, c0 >> 6, DG < 64 ? DG : 64)[lane] = s;
            }
        }
        wave_sync();
    }
}

// Lanes per edge and values per lane for k kept values: (4, 1), (8, 1), (16, 1), (16, 2), (16, 4).
template <typename F>
inline void hub_values_variant(int k, F&& f) {
    if (k <= 4) f(std::integral_constant<int, 2>{}, std::integral_constant<int, 1>{});
    else if (k <= 8) f(std::integral_constant<int, 3>{}, std::integral_constant<int, 1>{});
    else if (k <= 16) f(std::integral_constant<int, 4>{}, std::integral_constant<int, 1>{});
    else if (k <= 32) f(std::integral_constant<int, 4>{}, std::integral_constant<int, 2>{});
    else f(std::integral_constant<int, 4>{}, std::integral_constant<int, 4>{});
}

// The same for a group of column blocks (rows of 128 or 192 sums per edge place in LDS): at least eight lanes per edge.
template <typename F>
inline void hub_values_variant_wide(int k, F&& f) {
    if (k <= 8) f(std::integral_constant<int, 3>{}, std::integral_constant<int, 1>{});
    else if (k <= 16) f(std::integral_constant<int, 4>{}, std::integral_constant<int, 1>{});
    else if (k <= 32) f(std::integral_constant<int, 4>{}, std::integral_constant<int, 2>{});
    else f(std::integral_constant<int, 4>{}, std::integral_constant<int, 4>{});
}

template <int DG, int LG, int KQ>
__global__ __launch_bounds__(256) void k_hub_values(CsrView g, HubChunks h, const float* __restrict__ vals,
                                                    const uint8_t* __restrict__ cols, int k, int n, float* __restrict__ part,
                                                    float* __restrict__ rows) {
    __shared__ HubValLds<DG, LG> lds[4];
    hub_values_pass<DG, LG, KQ>(g, h, vals, cols, k, n, part, rows, lds[threadIdx.x >> 6], hub_sweep(h));
}

}  // namespace gsr

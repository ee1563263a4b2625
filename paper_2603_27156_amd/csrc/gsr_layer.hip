// The grouped reversible layer (Section 3, eq. (6)/(7)), its backward fused with the inverse
// (Algorithm 2's structure; eq. (3), eq. (11)) and the whole training step.
//
// Kernels (persistent over 16-row tiles, one wave per tile, no cross-wave synchronisation inside
// the sweep):
//   k_block   H = A*scatter(V,I) of Y_{i-1} gathered from compressed records into an LDS tile;
//             O = H W_i on the matrix cores; Y_i = X_i + O (forward) or X_i = Y_i - O (inverse),
//             in place; the GS record of the row just written is emitted in the same pass.  With
//             WITH_DW it also accumulates dW_i += H^T dY_i, so the recomputed H is consumed
//             where it is rebuilt.
//   k_grad    (first: dW_i summed from the workgroup partials the kernel before left;) Q = A^T dY_i (dense-row gather); dH = Q W_i^T on the matrix cores; only the k
//             positions recorded by I are read; back through the RMS scale; dY_{i-1} += dZ.
//   k_sum     Y_0 = sum_{j>=2} X_j and/or the GS record of a plane.
//   k_head    scalar linear head, squared error, dX^L, partial sums for dw_out / db / loss.
#include "gsr_internal.h"
#include "gsr_device.h"

#include <algorithm>
#include <vector>

namespace gsr {

CsrView make_view(const gsr_graph_t* g, bool transpose);

// per-wave LDS: a tile of 16 x tile_ld floats, 64 staged edges, 17 row pointers
template <int DG, bool RECORDS = false>
struct WaveLds {
    // the tile, with what gather_values_rows and emit_tile need behind it (RECORDS)
    alignas(16) float st[!RECORDS ? 16 * tile_ld<DG>() : gather_floats<DG>() > emit_floats<DG, REC_COLUMNS>() ? gather_floats<DG>() : emit_floats<DG, REC_COLUMNS>()];
    EdgeRec ebuf[RECORDS ? 1 : 64];        // 64 staged edges (not with gather_values_rows)
    int rp[20];                            // row pointers of the tile's 17 row boundaries
};

// ---- block: forward / inverse (+ weight gradient) ------------------------------------------------
template <int DG, typename T>
struct BlockArgs {
    CsrView g;
    int n, tiles;
    Record<DG, T> in;       // record of Y_{i-1}
    int k;
    const float* hub_part;  // first-pass partial rows of split rows
    const float* w;         // W_i [DG][DG]
    T* plane;               // X_i on entry / Y_i on return (or the reverse), row stride ld
    int64_t ld;
    Record<DG, T> out;      // record of the row written (out.mask == NULL: none)
    bool out_given;         // out.mask holds the column sets to use (kept from the forward sweep)
    int norm;
    float eps;
    const T* dy;            // dY_i, row stride ldg            (WITH_DW)
    int64_t ldg;
    float* dw_partial;      // [gridDim.x][DG*DG]              (WITH_DW)
    int* draws;             // tile counters of the dynamic sweep and the sign-off counter (not WITH_DW)
    int* draws_done;
    TieSeg<DG> tie;         // where rows that select at a near-tie are listed (count == NULL: nowhere)
    float* h_out;           // [n][DG] float32: receives H = A scatter(V, I) of the block for k_dw (NULL: not kept)
    TieSeg<DG> fix;         // rows listed in the forward sweep get their kept column sets (WITH_DW; count == NULL: none, see TieFix)
};

// B3: the H W_i (and dW_i) products on the bf16 matrix pipe from three-term splits (mfma_tile_b3), with W_i kept
// split in LDS.  That copy is half as large again as the float32 one, so the kernels without dW accumulators run
// eight waves per workgroup on it to keep sixteen waves per compute unit resident.  Measured on the 1M-node workload:
// forward 345 -> 319 us, inverse + dW 516 -> 477 us per launch.  The forward kernel keeps a float32 variant (B3 =
// false, four waves per workgroup) for graphs whose rows nearly all go through the first pass, where a launch is a
// single short tile per wave and the variant with the larger workgroups took 121 us against 84.  Both inverse kernels
// always use the split form: the plain and the fused inverse must rebuild the same bits.
constexpr int block_waves(bool with_dw, bool b3) { return (!with_dw && b3) ? 8 : 4; }

template <int DG, typename T, int SIGN, bool WITH_DW, bool DEAL, bool B3, RecordForm FORM>
__global__ __launch_bounds__(64 * block_waves(WITH_DW, B3)) __attribute__((amdgpu_waves_per_eu(WITH_DW && DG == 64 ? 2 : 4))) void k_block(BlockArgs<DG, T> a) {
    static_assert(B3 || (SIGN > 0 && !WITH_DW), "only the forward kernel has a float32 variant");
    constexpr int LR = tile_ld<DG>(), CPL = DG / 16;
    __shared__ WaveLds<DG, true> lds[block_waves(WITH_DW, B3)];
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), tg = lane >> 4, tj = lane & 15;
    WaveLds<DG, true>& L = lds[wave];
    float* st_h = L.st;
    __shared__ typename std::conditional<B3, WLdsB3<DG, deep_products<T>()>, WLds<DG>>::type wl;
    if constexpr (B3) load_w_lds_b3(a.w, DG, false, wl);
    else load_w_lds<DG>(a.w, false, wl);
    f32x4 dw[WITH_DW ? DG / 16 : 1][WITH_DW ? DG / 16 : 1];
    if constexpr (WITH_DW) {
#pragma unroll
        for (int mb = 0; mb < DG / 16; ++mb)
#pragma unroll
            for (int ob = 0; ob < DG / 16; ++ob) dw[mb][ob] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // the weight gradient sums over the tiles a wave has seen: fixed sweep there, drawn tiles otherwise
    const TileSweep ts = tile_sweep(a.tiles);
    TileDraws td;
    TileDeal deal{0, 0, 0, false};      // DEAL: the heavy tiles first (a variant of its own: the bookkeeping costs
    if constexpr (DEAL) deal = tile_deal(a.g);   // 3 % on a graph with 120 short tiles per wave even when it never fires)
    int requested = 0;     // the draw that is outstanding (dynamic sweep)
    int t = ts.first, t_end = ts.end;
    if constexpr (!WITH_DW) {
        td = tile_draws(a.tiles, a.draws, a.draws_done);
        t_end = td.end;
        t = td.first;
    }
    if constexpr (DEAL) {
        if (deal.on) { t = a.g.heavy[deal.at]; t_end = a.tiles; }
    }
    // the tile after the present one: its row pointers are requested while the present one is finished (1M nodes: forward
    // 232 -> 223 us, inverse 257 -> 246; its first edges as well: slower, their registers live through the record)
    int t_next = 0, t_end_next = t_end;
    auto advance = [&]() {
        t_end_next = t_end;
        if (DEAL && deal.on) {
            tile_deal_next(deal);
            if (deal.on) {
                t_next = a.g.heavy[deal.at];
            } else if constexpr (WITH_DW) {
                t_next = ts.first; t_end_next = ts.end;
            } else {
                t_next = td.first; t_end_next = td.end;
            }
        } else {
            if constexpr (WITH_DW) t_next = t + ts.step;
            else t_next = tile_drawn(td, requested);
        }
    };
    int rpv = tile_rp_load(a.g, (uint32_t)t * 16u, a.n, lane);

    while (t < t_end) {
        if constexpr (!WITH_DW) {
            if (!DEAL || !deal.on) requested = tile_request(td);
        }
        const int r0 = t * 16;
        wave_sync();
        // The tile's own rows (X_i, and dY_i for the weight gradient), in the tile register layout.  Requested before
        // the gather they arrive while it runs, but hold sixteen registers through it; requested after it they arrive
        // during the weight product.  Measured per variant (1M-node workload, float32: forward 232 us early against 241
        // late, inverse 264 against 257; the fused inverse + dW kernel gains from late rows at D/C = 32 in float32 and loses
        // otherwise (1M nodes, 16 bits, D/C = 32: 152 us early, 159 late), the 16-bit forward kernel gains at 64).
        constexpr bool OWN_LATE = WITH_DW ? DG == 32 && sizeof(T) == 4 : (sizeof(T) == 4 ? SIGN < 0 : DG == 64);
        float xy[4][CPL], gy[WITH_DW ? 4 : 1][CPL];
        auto own_rows = [&]() {
#pragma unroll
            for (int reg = 0; reg < 4; ++reg) {
                const int row = r0 + 4 * reg + tg;
                const size_t rowc = (size_t)(row < a.n ? row : a.n - 1);
                load_cols<CPL, T>(a.plane + rowc * a.ld + CPL * tj, xy[reg]);
                if constexpr (WITH_DW) load_cols<CPL, T>(a.dy + rowc * a.ldg + CPL * tj, gy[reg]);
            }
        };
        if constexpr (!OWN_LATE) own_rows();
        const bool has_hub = tile_begin(a.g, rpv, L.rp, lane);
        if constexpr (DEAL) {
            if (!deal.on && tile_is_heavy(a.g, rpv, L.rp, has_hub)) {      // dealt out before the sweep
                advance();
                t = t_next;
                rpv = tile_rp_load(a.g, (uint32_t)t * 16u, a.n, lane);
                continue;
            }
        }
        // (in the forward and in both inverse kernels alike, so that f_i is recomputed by the instructions that computed it)
        tile_gather_rows<DG, true, 20>(a.g, a.hub_part, has_hub, r0, L.rp, st_h, lane, [&](int e_a, int e_b) {
            const int ea = __builtin_amdgcn_readfirstlane(e_a), eb = __builtin_amdgcn_readfirstlane(e_b);
            if constexpr (FORM == REC_ROWS) gather_dense_rows<DG, 8>(a.g, a.in.vals, DG, ea, eb, lane, st_h);
            else gather_values_rows<DG, 4, !B3>(a.g, a.in.vals, a.in.cols, a.k, ea, eb, lane, st_h);
        });
        advance();
        rpv = tile_rp_load(a.g, (uint32_t)t_next * 16u, a.n, lane);
        if constexpr (OWN_LATE) own_rows();
        if constexpr (WITH_DW) {
#pragma unroll
            for (int reg = 0; reg < 4; ++reg)
#pragma unroll
                for (int cb = 0; cb < CPL; ++cb) gy[reg][cb] = r0 + 4 * reg + tg < a.n ? gy[reg][cb] : 0.f;   // rows past the end
        }
        TieFix<DG, WITH_DW> fix{a.fix, t, lane};
        wave_sync();
        if constexpr (!WITH_DW) {
            if (a.h_out) {                                 // H leaves for the weight-gradient kernel, four rows per store
#pragma unroll
                for (int reg = 0; reg < 4; ++reg) {
                    const int rr = 4 * reg + tg, row = r0 + rr;
                    float hv[CPL];
                    lds_load<CPL>(st_h + rr * LR + CPL * tj, hv);
                    if (row < a.n) store_cols<CPL, float>(a.h_out + (size_t)row * DG + CPL * tj, hv);
                }
            }
        }
        f32x4 acc[CPL];
        if constexpr (B3) {
            mfma_tile_b3<DG>(st_h, wl, acc);               // O = H W_i in the tile register layout
            if constexpr (WITH_DW) mfma_outer_b3<DG, T>(st_h, gy, dw);
        } else {
            mfma_tile<DG>(st_h, wl, acc);
        }
        wave_sync();                                       // H has been read: the tile is free
        // residual: four rows per instruction, CPL adjacent elements per lane
#pragma unroll
        for (int reg = 0; reg < 4; ++reg) {
            const int rr = 4 * reg + tg, row = r0 + rr;
            const bool ok = row < a.n;
            T* p = a.plane + (size_t)(ok ? row : a.n - 1) * a.ld + CPL * tj;
            float y[CPL];
#pragma unroll
            for (int cb = 0; cb < CPL; ++cb) y[cb] = stored<T>(SIGN > 0 ? xy[reg][cb] + acc[cb][reg] : xy[reg][cb] - acc[cb][reg]);
            if (ok) store_cols<CPL, T>(p, y);
#pragma unroll
            for (int cb = 0; cb < CPL; ++cb) y[cb] = ok ? y[cb] : 0.f;
            lds_store<CPL>(st_h + rr * LR + CPL * tj, y);
        }
        if (a.out.mask) {
            wave_sync();
            emit_tile<DG, T, FORM>(st_h, r0, a.n, a.k, a.norm, a.eps, a.out, a.out_given, lane, nullptr, nullptr, a.tie, fix);
        }
        t = t_next;
        t_end = t_end_next;
    }
    if constexpr (!WITH_DW) tile_finish(td);
    if constexpr (WITH_DW) {
        // workgroup partial of dW_i: the four waves add their accumulators in wave order
        float* red = reinterpret_cast<float*>(lds);
        static_assert(sizeof(lds) >= DG * DG * sizeof(float), "LDS too small for the dW reduction");
        for (int w = 0; w < 4; ++w) {
            __syncthreads();
            if (wave == w) {
#pragma unroll
                for (int mb = 0; mb < DG / 16; ++mb)
#pragma unroll
                    for (int ob = 0; ob < DG / 16; ++ob)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int m = 16 * mb + 4 * (lane >> 4) + r, o = CPL * (lane & 15) + ob;
                            if (w == 0) red[m * DG + o] = dw[mb][ob][r];
                            else red[m * DG + o] += dw[mb][ob][r];
                        }
            }
        }
        __syncthreads();
        for (int i = threadIdx.x; i < DG * DG; i += 256) a.dw_partial[(size_t)blockIdx.x * DG * DG + i] = red[i];
    }
}

// The records of listed rows, written again with the column sets kept from the forward sweep: a wave takes sixteen
// list entries in the quarter layout of emit_tile (lane = (entry, quarter of the row)) and forms the values exactly
// as emit_tile does when the set is given.  plane: the rows the record was just taken from, row stride ld.  Called by
// every wave of a grid of `nwaves` waves (a multiple of TIE_SUB): wave w takes sub-list w mod TIE_SUB.
template <int DG, typename T>
__device__ __forceinline__ void tie_fixup_rows(const TieSeg<DG>& tie, const T* __restrict__ plane, int64_t ld, int k, int norm, float eps,
                                               const Record<DG, T>& out, int wave, int nwaves) {
    using M = typename MaskOf<DG>::type;
    constexpr int QW = DG / 4;
    const int lane = lane_id(), r = lane & 15, q = lane >> 4;
    const int sub = wave & (TIE_SUB - 1);
    const int listed = tie.count[sub * TIE_COUNTER_STRIDE], cnt = listed < tie.cap ? listed : tie.cap;
    for (int e0 = (wave / TIE_SUB) * 16; e0 < cnt; e0 += (nwaves / TIE_SUB) * 16) {
        const bool ok = e0 + r < cnt;
        const int e = sub * tie.cap + (ok ? e0 + r : cnt - 1);
        const size_t row = tie.rows[e];
        const M m = tie.masks[e];
        float x[QW];
#pragma unroll
        for (int j = 0; j < QW; ++j) x[j] = to_float(plane[row * ld + q * QW + j]);
        const uint32_t msel = (uint32_t)(m >> (QW * q)) & ((1u << QW) - 1u);
        uint32_t all[4];
        quarter_all((uint32_t)__popc(msel), all);
        const bool as_row = !out.cols;
        size_t slot = row * k;
#pragma unroll
        for (int i = 0; i < 3; ++i) slot += i < q ? all[i] : 0u;
        const float scale = record_scale<DG>(x, norm, eps);
#pragma unroll
        for (int j = 0; j < QW; ++j) {
            const bool bit = (msel >> j) & 1u;
            if (as_row) {
                if (ok) out.vals[row * DG + q * QW + j] = from_float<T>(bit ? x[j] * scale : 0.f);
            } else if (ok && bit) {
                out.vals[slot] = from_float<T>(x[j] * scale);
                out.cols[slot] = (uint8_t)(q * QW + j);
            }
            slot += bit ? 1 : 0;
        }
        if (ok && q == 0) out.mask[row] = m;
    }
}

// dW_i[e] = sum over workgroup partials, as a launch of its own (used when the gradient kernel that follows has too
// few tiles per wave to absorb the work, see layer_backward_impl).  A block of 256 threads owns 16 entries; its 16
// thread rows each sum a contiguous sixteenth of the partials in ascending order, then the 16 sums are added in order.
// (Blocks of 64 entries left three quarters of the compute units idle on a 64 x 64 matrix: 18 us per launch.)
constexpr int DW_REDUCE_ENTRIES = 16;
__device__ __forceinline__ void dw_reduce_block(int block, const float* __restrict__ partial, int nparts, int elems,
                                                float* __restrict__ out, int cols, int ld_out, float (&red)[16][DW_REDUCE_ENTRIES]) {
    const int j = threadIdx.x & (DW_REDUCE_ENTRIES - 1), seg = (threadIdx.x & 255) / DW_REDUCE_ENTRIES;
    const int e = block * DW_REDUCE_ENTRIES + j;
    const int per = (nparts + 15) / 16, p0 = seg * per, p1 = min(nparts, p0 + per);
    float acc = 0.f;
    if (e < elems) {
        int p = p0;
        for (; p + 8 <= p1; p += 8) {           // eight loads in flight, added in ascending order
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = partial[(size_t)(p + u) * elems + e];
#pragma unroll
            for (int u = 0; u < 8; ++u) acc += v[u];
        }
        for (; p < p1; ++p) acc += partial[(size_t)p * elems + e];
    }
    red[seg][j] = acc;
    __syncthreads();
    if (seg == 0 && e < elems) {
        float s = red[0][j];
#pragma unroll
        for (int q = 1; q < 16; ++q) s += red[q][j];
        out[(size_t)(e / cols) * ld_out + e % cols] = s;       // entry (e / cols, e % cols) of a matrix of row stride ld_out
    }
}

template <int DG, typename T>
__global__ __launch_bounds__(256) void k_tie_fixup(TieSeg<DG> tie, const T* __restrict__ plane, int64_t ld, int k, int norm,
                                                   float eps, Record<DG, T> out) {
    tie_fixup_rows<DG, T>(tie, plane, ld, k, norm, eps, out, (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6),
                          (int)((gridDim.x * blockDim.x) >> 6));
}

// dW_i = H^T dY_i as a pass of its own over H (left by the inverse kernel) and dY_i: a wave sums over the tiles of a
// fixed sweep (so the partial sums do not depend on timing), 64 x 64 accumulators in registers, products on the bf16
// pipe (mfma_outer_b3); workgroup partials as k_block writes them.  The inverse kernel then runs without the 64
// accumulator registers per lane, at sixteen waves per compute unit with the row-wise sums of the forward kernel.
template <int DG, typename T>
struct DwArgs {
    int n, tiles;
    const float* h;         // [n][DG]
    // groups of S column blocks: blockIdx.y = mb S + ob takes H_mb (planes of [n][64]) and dY's columns 64 ob on, into a set
    // of partials of its own, y_set floats on
    int S;
    size_t y_set;
    const T* dy;            // row stride ldg
    int64_t ldg;
    float* dw_partial;      // [gridDim.x][DG*DG]
    // mode 2 of the step: the record the inverse kernel has just taken again gets the kept column sets of its listed
    // rows back here (tie.count == NULL: nothing to do), which saves a launch per block
    TieSeg<DG> tie;
    const T* fix_plane;
    int64_t fix_ld;
    int k, norm;
    float eps;
    Record<DG, T> fix_out;
};

// WIDE: groups of S column blocks.  Their workgroups are shared out between S^2 sets, so a wave sums that many times more
// tiles than one of a plain group does (or of the kernels that took these products before, a set per input block).  With
// float32 rows, sums as mfma_outer takes them keep dW at least as close to 64 bits as it was (1.4e-7 against 2.4e-7 on 50k
// rows, groups of 192; 2.8e-7 against 6.1e-7 on 200k rows, groups of 128) at 1 % of the time of those layers' backward.  With
// 16-bit rows of dY half of the split products are zero and the sums hold (A = I, 150k - 400k rows, groups of 128 / 192 / 256:
// 1.7e-7 / 1.6e-7 / 1.8e-7 against 1.7e-7 / 1.6e-7 / 1.6e-7; 256 with twice the workgroups 1.5e-7), and float32 products
// would cost 4 %.
template <int DG, typename T, bool WIDE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_dw(DwArgs<DG, T> a) {
    if constexpr (WIDE) {
        a.h += (size_t)(blockIdx.y / a.S) * a.n * DG;
        a.dy += 64 * (blockIdx.y % a.S);
        a.dw_partial += (size_t)blockIdx.y * a.y_set;
    }
    if (a.tie.count)
        tie_fixup_rows<DG, T>(a.tie, a.fix_plane, a.fix_ld, a.k, a.norm, a.eps, a.fix_out, (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6),
                              (int)((gridDim.x * blockDim.x) >> 6));
    constexpr int LR = tile_ld<DG>(), CPL = DG / 16;
    __shared__ __attribute__((aligned(16))) float tile[4][16 * LR];
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), tg = lane >> 4, tj = lane & 15;
    float* st = tile[wave];
    f32x4 dw[DG / 16][DG / 16];
#pragma unroll
    for (int mb = 0; mb < DG / 16; ++mb)
#pragma unroll
        for (int ob = 0; ob < DG / 16; ++ob) dw[mb][ob] = f32x4{0.f, 0.f, 0.f, 0.f};
    const TileSweep ts = tile_sweep(a.tiles);
    // the next tile's rows are requested while the present tile is multiplied
    float hv[4][CPL], gy[4][CPL];
    auto request = [&](int t) {
#pragma unroll
        for (int reg = 0; reg < 4; ++reg) {
            const int row = t * 16 + 4 * reg + tg;
            const size_t rowc = (size_t)(row < a.n ? row : a.n - 1);
            load_cols<CPL, float>(a.h + rowc * DG + CPL * tj, hv[reg]);
            load_cols<CPL, T>(a.dy + rowc * a.ldg + CPL * tj, gy[reg]);
        }
    };
    int t = ts.first;
    if (t < ts.end) request(t);
    while (t < ts.end) {
        const int r0 = t * 16;
        float g[4][CPL];
        wave_sync();          // the tile before has been read
#pragma unroll
        for (int reg = 0; reg < 4; ++reg) {
            const bool ok = r0 + 4 * reg + tg < a.n;
            float h[CPL];
#pragma unroll
            for (int cb = 0; cb < CPL; ++cb) {
                h[cb] = ok ? hv[reg][cb] : 0.f;
                g[reg][cb] = ok ? gy[reg][cb] : 0.f;          // rows past the end
            }
            lds_store<CPL>(st + (4 * reg + tg) * LR + CPL * tj, h);
        }
        t += ts.step;
        if (t < ts.end) request(t);
        wave_sync();
        if constexpr (WIDE && sizeof(T) == 4) mfma_outer<DG>(st, g, dw);
        else mfma_outer_b3<DG, T>(st, g, dw);
    }
    // workgroup partial of dW_i: the four waves add their accumulators in wave order
    __shared__ float red[DG * DG];
    for (int w = 0; w < 4; ++w) {
        __syncthreads();
        if (wave == w) {
#pragma unroll
            for (int mb = 0; mb < DG / 16; ++mb)
#pragma unroll
                for (int ob = 0; ob < DG / 16; ++ob)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int m = 16 * mb + 4 * (lane >> 4) + r, o = CPL * (lane & 15) + ob;
                        if (w == 0) red[m * DG + o] = dw[mb][ob][r];
                        else red[m * DG + o] += dw[mb][ob][r];
                    }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < DG * DG; i += 256) a.dw_partial[(size_t)blockIdx.x * DG * DG + i] = red[i];
}

// blockIdx.y (groups wider than a tile: the S x S blocks of dW_i in one launch): set y of the partials starts
// y * set_stride floats on, and goes to block (y / sets_per_row, y % sets_per_row) of the output, 64 rows and 64 columns apart.
__global__ __launch_bounds__(256) void k_dw_reduce(const float* __restrict__ partial, int nparts, int elems,
                                                   float* __restrict__ out, int cols, int ld_out, size_t set_stride = 0,
                                                   int sets_per_row = 1) {
    partial += (size_t)blockIdx.y * set_stride;
    out += (size_t)(blockIdx.y / sets_per_row) * 64 * ld_out + (size_t)(blockIdx.y % sets_per_row) * 64;
    __shared__ float red[16][DW_REDUCE_ENTRIES];
    dw_reduce_block((int)blockIdx.x, partial, nparts, elems, out, cols, ld_out, red);
}

// ---- block: data gradient ---------------------------------------------------------------------------
template <int DG, typename T>
struct GradArgs {
    using M = typename MaskOf<DG>::type;
    CsrView gt;             // A^T
    int n, tiles;
    const T* dy;            // dY_i (complete), row stride ldg
    int64_t ldg;
    const float* hub_part;
    const float* w;         // W_i [DG][DG]
    const M* own_mask;      // columns recorded for Y_{i-1}
    const T* z;             // Y_{i-1} rows (RMS only), row stride ldz
    int64_t ldz;
    int norm;
    float eps;
    T* dst;                 // dY_{i-1} plane(s): ndst planes, dst_gs apart, row stride ldd
    int64_t ldd, dst_gs;
    int ndst;
    int* draws;             // tile counters of the dynamic sweep and the sign-off counter
    int* draws_done;
    // dW_i of the same block, left as workgroup partials by the inverse + dW kernel just before: summed here by
    // the first workgroups before they start on tiles, which saves a launch per block (dw_out == NULL: nothing to do)
    const float* dw_partial;
    int dw_parts;
    float* dw_out;
    // On small graphs a second row of workgroups (blockIdx.y = 1) sums them beside the tiles instead, as k_dw_reduce does (NULL: no
    // such row; not in the variants that deal heavy tiles out)
    float* beside_out;
};

// dW_i[e] = sum over the workgroup partials, in a fixed order: a workgroup takes 64 entries at a time; its four
// waves each sum a contiguous quarter of the partials in ascending order (sixteen loads in flight), then the four
// sums are added in order.
template <int ELEMS>
__device__ __forceinline__ void dw_reduce_slices(const float* __restrict__ partial, int nparts, float* __restrict__ out,
                                                 float* red /* 256 floats of LDS */) {
    const int col = threadIdx.x & 63, seg = threadIdx.x >> 6;
    const int per = (nparts + 3) / 4, p0 = seg * per, p1 = min(nparts, p0 + per);
    // the last workgroups take the slices: when there are fewer tiles than waves they are the ones without a tile
    for (int slice = gridDim.x - 1 - blockIdx.x; slice < ELEMS / 64; slice += gridDim.x) {
        const float* src = partial + slice * 64 + col;
        float acc = 0.f;
        int p = p0;
        for (; p + 16 <= p1; p += 16) {
            float v[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) v[u] = src[(size_t)(p + u) * ELEMS];
#pragma unroll
            for (int u = 0; u < 16; ++u) acc += v[u];
        }
        for (; p < p1; ++p) acc += src[(size_t)p * ELEMS];
        __syncthreads();
        if (seg < 4) red[seg * 64 + col] = acc;
        __syncthreads();
        if (seg == 0) out[slice * 64 + col] = ((red[col] + red[64 + col]) + red[128 + col]) + red[192 + col];
    }
    __syncthreads();
}

// Waves per workgroup of k_grad (they share one copy of W^T in LDS).  Measured at 1M rows, Dg = 64, float32 product:
// 4 and 8 waves (16 resident waves per compute unit either way) take the same time; 6 and 10
// waves, which would allow 18 and 20 resident waves, are 20 % and 10 % slower.
// B3 as in k_block: dH = Q W^T on the bf16 pipe with eight waves per workgroup (322 -> 309 us on the 1M-node
// workload), or the float32 product with four (graphs whose rows nearly all go through the first pass: 106 us
// against 132).
constexpr int grad_waves(bool b3) { return b3 ? 8 : 4; }

template <int DG, typename T, bool DEAL, bool B3>
__global__ __launch_bounds__(64 * grad_waves(B3)) __attribute__((amdgpu_waves_per_eu(4))) void k_grad(GradArgs<DG, T> a) {
    constexpr int CPL = DG / 16;
    constexpr int GRAD_WAVES = grad_waves(B3);
    // the partial rows of a tile's split rows requested together (hub_rows_fill) only where that spills no register:
    // these kernels sit at their 128 registers
    constexpr bool FILL_FAST = !DEAL && sizeof(T) == 4 && DG == 64;
    __shared__ WaveLds<DG> lds[GRAD_WAVES];
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), tg = lane >> 4, tj = lane & 15;
    WaveLds<DG>& L = lds[wave];
    float* st = L.st;
    __shared__ typename std::conditional<B3, WLdsB3<DG, deep_products<T>()>, WLds<DG>>::type wl;
    static_assert(GRAD_WAVES >= 4 && sizeof(lds) >= 64 * GRAD_WAVES * sizeof(float), "dw_reduce_slices works with the first 256 threads");
    if constexpr (!DEAL) {
        if (a.beside_out && blockIdx.y == 1) {
            constexpr int PER = GRAD_WAVES / 4, BLOCKS = DG * DG / DW_REDUCE_ENTRIES;
            for (int b0 = (int)blockIdx.x * PER; b0 < BLOCKS; b0 += (int)gridDim.x * PER) {       // (the same for every thread of the workgroup)
                const int half = (int)threadIdx.x >> 8;
                dw_reduce_block(b0 + half, a.dw_partial, a.dw_parts, DG * DG, a.beside_out, DG, DG,
                                reinterpret_cast<float(*)[16][DW_REDUCE_ENTRIES]>(lds)[half]);
                __syncthreads();
            }
            return;
        }
    }
    if (a.dw_out) dw_reduce_slices<DG * DG>(a.dw_partial, a.dw_parts, a.dw_out, reinterpret_cast<float*>(lds));
    if constexpr (B3) load_w_lds_b3(a.w, DG, true, wl);
    else load_w_lds<DG>(a.w, true, wl);
    TileDraws td = tile_draws(a.tiles, a.draws, a.draws_done);
    TileDeal deal{0, 0, 0, false};
    if constexpr (DEAL) deal = tile_deal(a.gt);
    int requested = 0;                     // the draw that is outstanding
    int t_end = td.end, t = td.first;
    if (DEAL && deal.on) { t = a.gt.heavy[deal.at]; t_end = a.tiles; }
    while (t < t_end) {
        if (!DEAL || !deal.on) requested = tile_request(td);
        const int r0 = t * 16;
        wave_sync();
        const int rpv = tile_rp_load(a.gt, r0, a.n, lane);
        // what the epilogue needs of the tile's own rows is requested first (but for the masks in the one variant that would
        // spill a register)
        constexpr bool OWN_LATE = DEAL && !B3 && sizeof(T) == 2 && DG == 64;
        typename MaskOf<DG>::type own[4];
        float z[4][CPL];
#pragma unroll
        for (int reg = 0; reg < 4; ++reg) {
            const int row = r0 + 4 * reg + tg;
            const size_t rowc = (size_t)(row < a.n ? row : a.n - 1);
            if constexpr (!OWN_LATE) own[reg] = a.own_mask[rowc];
            if (a.norm == GSR_NORM_RMS) load_cols<CPL, T>(a.z + rowc * a.ldz + CPL * tj, z[reg]);
        }
        const bool has_hub = tile_begin(a.gt, rpv, L.rp, lane);
        if constexpr (DEAL) {
            if (!deal.on && tile_is_heavy(a.gt, rpv, L.rp, has_hub)) {    // dealt out before the sweep
                t = tile_drawn(td, requested);
                continue;
            }
        }
        // float32: Q in ordinary arithmetic, a run of the staged edges per lane group (322 us against 378 through the
        // matrix cores on the 1M-node workload; sixteen steps in flight instead of eight spill)
        if constexpr (sizeof(T) == 4) {
            tile_gather_rows<DG, FILL_FAST>(a.gt, a.hub_part, has_hub, r0, L.rp, st, lane, [&](int e_a, int e_b) {
                gather_dense_rows<DG, 8>(a.gt, a.dy, a.ldg, __builtin_amdgcn_readfirstlane(e_a),
                                               __builtin_amdgcn_readfirstlane(e_b), lane, st);
            });
        } else {
            f32x4 qacc[DG / 16];
            tile_gather<DG, FILL_FAST>(a.gt, a.hub_part, has_hub, r0, L.rp, st, lane, qacc, [&](int e_a, int e_b) {
                gather_dense_mfma<DG, T, (sizeof(T) == 4 || DG == 32) ? 16 : 8>(a.gt, a.dy, a.ldg, __builtin_amdgcn_readfirstlane(e_a),
                                         __builtin_amdgcn_readfirstlane(e_b), L.rp, L.ebuf, lane, qacc);
            });
        }
        wave_sync();
        f32x4 acc[CPL];
        if constexpr (B3) mfma_tile_b3<DG>(st, wl, acc);          // dH = Q W^T in the tile register layout
        else mfma_tile<DG>(st, wl, acc);
        // epilogue on registers: row 4 reg + tg, columns CPL tj + cb
        float dz[4][CPL];
#pragma unroll
        for (int reg = 0; reg < 4; ++reg) {
            const int row = r0 + 4 * reg + tg;
            const bool ok = row < a.n;
            if constexpr (OWN_LATE) own[reg] = a.own_mask[ok ? row : a.n - 1];
            const uint32_t bits = ok ? (uint32_t)(own[reg] >> (CPL * tj)) & ((1u << CPL) - 1u) : 0u;
            if (a.norm == GSR_NORM_RMS) {
                // V = Z[I] * rinv, rinv = (mean Z^2 + eps)^-1/2:
                // dZ_c = [c in I] g_c rinv - Z_c (sum_t g_t Z_{I_t}) rinv^3 / DG
                float ss = 0.f, dot = 0.f;
#pragma unroll
                for (int cb = 0; cb < CPL; ++cb) {
                    ss += z[reg][cb] * z[reg][cb];
                    dot += ((bits >> cb) & 1u) ? acc[cb][reg] * z[reg][cb] : 0.f;
                }
                ss = group16_sum(ss);
                dot = group16_sum(dot);
                const float rinv = __builtin_amdgcn_rsqf(ss * (1.0f / (float)DG) + a.eps);
                const float coef = dot * (rinv * rinv * rinv) * (1.0f / (float)DG);
#pragma unroll
                for (int cb = 0; cb < CPL; ++cb) dz[reg][cb] = (((bits >> cb) & 1u) ? acc[cb][reg] * rinv : 0.f) - z[reg][cb] * coef;
            } else {
#pragma unroll
                for (int cb = 0; cb < CPL; ++cb) dz[reg][cb] = ((bits >> cb) & 1u) ? acc[cb][reg] : 0.f;
            }
        }
        // the planes that receive dZ: the four rows of a plane are requested together
        {
            // JC planes at a time: all their rows are requested before the first is written back (block 1 updates C - 1
            // planes; one plane after the other took 3.2 ms against 1.2 ms for a one-plane launch at 8M rows, C = 8, 16-bit
            // rows of 32 columns).  float32 at 64 columns: two planes spill registers, 285 us per launch against 273; at 32
            // columns four do.
            constexpr int JC = sizeof(T) == 4 ? (CPL <= 2 ? 2 : 1) : CPL <= 2 ? 4 : 2;
            if (a.ndst == 1) {          // the common case on its own, so that it requests nothing twice
                float g[4][CPL];
#pragma unroll
                for (int reg = 0; reg < 4; ++reg) {
                    const int row = r0 + 4 * reg + tg;
                    const int rowc = row < a.n ? row : a.n - 1;
                    load_cols<CPL, T>(a.dst + (size_t)rowc * a.ldd + CPL * tj, g[reg]);
                }
#pragma unroll
                for (int reg = 0; reg < 4; ++reg) {
                    const int row = r0 + 4 * reg + tg;
#pragma unroll
                    for (int cb = 0; cb < CPL; ++cb) g[reg][cb] = stored<T>(g[reg][cb] + dz[reg][cb]);
                    if (row < a.n) store_cols<CPL, T>(a.dst + (size_t)row * a.ldd + CPL * tj, g[reg]);
                }
            } else
            for (int j0 = 0; j0 < a.ndst; j0 += JC) {
                float g[JC][4][CPL];
#pragma unroll
                for (int jj = 0; jj < JC; ++jj) {
                    const int j = j0 + jj < a.ndst ? j0 + jj : a.ndst - 1;
#pragma unroll
                    for (int reg = 0; reg < 4; ++reg) {
                        const int row = r0 + 4 * reg + tg;
                        const int rowc = row < a.n ? row : a.n - 1;
                        load_cols<CPL, T>(a.dst + (size_t)j * a.dst_gs + (size_t)rowc * a.ldd + CPL * tj, g[jj][reg]);
                    }
                }
#pragma unroll
                for (int jj = 0; jj < JC; ++jj) {
                    const int j = j0 + jj;
#pragma unroll
                    for (int reg = 0; reg < 4; ++reg) {
                        const int row = r0 + 4 * reg + tg;
#pragma unroll
                        for (int cb = 0; cb < CPL; ++cb) g[jj][reg][cb] = stored<T>(g[jj][reg][cb] + dz[reg][cb]);
                        if (row < a.n && j < a.ndst) store_cols<CPL, T>(a.dst + (size_t)j * a.dst_gs + (size_t)row * a.ldd + CPL * tj, g[jj][reg]);
                    }
                }
            }
        }
        if (DEAL && deal.on) {
            tile_deal_next(deal);
            if (deal.on) t = a.gt.heavy[deal.at];
            else { t = td.first; t_end = td.end; }
        } else {
            t = tile_drawn(td, requested);
        }
    }
    tile_finish(td);
}

// ---- group sum / record of a plane --------------------------------------------------------------------
template <int DG, typename T>
struct SumArgs {
    int n;
    const T* src;           // nsrc planes, src_gs apart, row stride ld
    int64_t ld, src_gs;
    int nsrc;
    T* y0;                  // dense [n][DG] copy of the sum (NULL: not kept)
    int k, norm;
    float eps;
    Record<DG, T> out;
    bool out_given;         // out.mask holds the column sets to use
    TieSeg<DG> tie;         // where rows that select at a near-tie are listed (count == NULL: nowhere)
    TieSeg<DG> fix;         // as in BlockArgs
    size_t y_rec, y_mask;   // blockIdx.y: the records of that many planes in one launch, src_gs apart, their records these many bytes apart
};

__global__ void k_zero_ints(int* p, int count) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0;
}

template <int DG, typename T, RecordForm FORM, bool FIX>
__global__ __launch_bounds__(256) void k_sum(SumArgs<DG, T> a) {
    constexpr int LR = tile_ld<DG>(), CPL = DG / 16;
    __shared__ __attribute__((aligned(16))) float tile[4][emit_floats<DG, REC_COLUMNS>()];
    const int lane = lane_id(), tg = lane >> 4, tj = lane & 15;
    float* st = tile[threadIdx.x >> 6];
    if (blockIdx.y > 0) {
        a.src += blockIdx.y * a.src_gs;
        a.out.vals = reinterpret_cast<T*>(reinterpret_cast<char*>(a.out.vals) + blockIdx.y * a.y_rec);
        if (a.out.cols) a.out.cols += blockIdx.y * a.y_rec;
        a.out.mask = reinterpret_cast<typename MaskOf<DG>::type*>(reinterpret_cast<char*>(a.out.mask) + blockIdx.y * a.y_mask);
    }
    const int nwaves = (gridDim.x * blockDim.x) >> 6, tiles = (a.n + 15) / 16;
    for (int t = (blockIdx.x * blockDim.x + threadIdx.x) >> 6; t < tiles; t += nwaves) {
        const int r0 = t * 16;
        float y[4][CPL];
#pragma unroll
        for (int reg = 0; reg < 4; ++reg) {
            const int row = r0 + 4 * reg + tg;
            load_cols<CPL, T>(a.src + (size_t)(row < a.n ? row : a.n - 1) * a.ld + CPL * tj, y[reg]);
        }
        for (int j = 1; j < a.nsrc; ++j) {
            float v[4][CPL];
#pragma unroll
            for (int reg = 0; reg < 4; ++reg) {
                const int row = r0 + 4 * reg + tg;
                load_cols<CPL, T>(a.src + (size_t)j * a.src_gs + (size_t)(row < a.n ? row : a.n - 1) * a.ld + CPL * tj, v[reg]);
            }
#pragma unroll
            for (int reg = 0; reg < 4; ++reg)
#pragma unroll
                for (int cb = 0; cb < CPL; ++cb) y[reg][cb] += v[reg][cb];
        }
        TieFix<DG, FIX> fix{a.fix, t, lane};
        wave_sync();          // the previous tile's records have left the scratch
#pragma unroll
        for (int reg = 0; reg < 4; ++reg) {
            const int rr = 4 * reg + tg, row = r0 + rr;
            const bool ok = row < a.n;
#pragma unroll
            for (int cb = 0; cb < CPL; ++cb) y[reg][cb] = stored<T>(y[reg][cb]);
            if (ok && a.y0) store_cols<CPL, T>(a.y0 + (size_t)row * DG + CPL * tj, y[reg]);
#pragma unroll
            for (int cb = 0; cb < CPL; ++cb) y[reg][cb] = ok ? y[reg][cb] : 0.f;
            lds_store<CPL>(st + rr * LR + CPL * tj, y[reg]);
        }
        wave_sync();
        emit_tile<DG, T, FORM>(st, r0, a.n, a.k, a.norm, a.eps, a.out, a.out_given, lane, nullptr, nullptr, a.tie, fix);
    }
}

// ---- groups wider than one tile: D/C = 64 S, S = 2, 3 or 4 ---------------------------------------------------
// A block of such a group runs as separate passes over planes of 64 columns: H = A scatter(V, I) for the whole row at once
// (k_gather_wide; a row that is one first-pass chunk gets its sums straight from that pass), X_i +- H W_i
// (k_wide_product), GS over the whole row (k_gs_wide), and for the gradient Q = A^T dY_i (k_dense_planes), then dH = Q W_i^T
// and back through GS (k_wide_grad).  W_i, up to 256 x 256, does not fit the LDS beside the tiles of a gather, and a kernel
// per pair of 64-column blocks has to gather every input block S times and to read and write the plane S times (as it was
// before: 200k nodes, two groups of 128, backward 1,523 us; 50k nodes of mean degree 236, two groups of 192, forward 690).

template <int S, typename T>
struct WideGatherArgs {
    CsrView g;
    int n, tiles;           // tiles of eight rows
    const T* vals;          // the record: [n][k] values and columns of the whole row
    const uint8_t* cols;
    int k;
    const float* hub_part;  // [S][chunks][64]
    int n_chunks;
    float* h;               // [S][n][64]
    int* draws;
    int* draws_done;
};

// Eight rows per wave: their sums, twelve rows of 64 S floats, leave LDS for sixteen waves per compute unit at S = 3.
template <int S, typename T>
__global__ __launch_bounds__(256) void k_gather_wide(WideGatherArgs<S, T> a) {
    constexpr int DGW = 64 * S, LR = tile_ld<DGW>();
    struct Wave {
        alignas(16) float st[gather_floats<DGW, 8>()];
        int rp[20];
    };
    __shared__ Wave lds[4];
    Wave& L = lds[threadIdx.x >> 6];
    const int lane = lane_id();
    TileWalk<false> walk(a.g, a.tiles, a.draws, a.draws_done);
    while (walk.more()) {
        walk.ahead();
        const int r0 = walk.t * 8, up = r0 & 8;            // up: the second half of a 16-row tile
        wave_sync();
        const int rpv = tile_rp_load(a.g, r0 - up, a.n, lane);
        if (lane < 17) L.rp[lane] = rpv;
        for (int i = 4 * lane; i < 12 * LR; i += 256) *reinterpret_cast<f32v4*>(L.st + i) = f32v4{0.f, 0.f, 0.f, 0.f};
        wave_sync();
        const int len = lane < 16 ? L.rp[lane + 1] - rpv : 0;
        const uint64_t splits = ballot(len > a.g.hub_threshold);
        // rows the first pass has written already (h.row of HubChunks)
        const uint32_t done = (uint32_t)(ballot(len > a.g.hub_threshold && len <= a.g.hub_chunk) >> up) & 255u;
        const uint32_t split = (uint32_t)(splits >> up) & 255u;
        int run = 0;
        for (int r = 0; r <= 8; ++r) {
            const bool hub = r < 8 && ((split >> r) & 1u);
            if (r == 8 || hub) {
                const int e_a = __builtin_amdgcn_readfirstlane(L.rp[up + run]), e_b = __builtin_amdgcn_readfirstlane(L.rp[up + r]);
                if (e_b > e_a) gather_values_rows<DGW, 4, false, 8>(a.g, a.vals, a.cols, a.k, e_a, e_b, lane, L.st);
                run = r + 1;
            }
        }
        for (int r = 0; r < 8; ++r) {
            if (!((split & ~done) >> r & 1u)) continue;    // a row of several chunks
            const int hrow = a.g.hub_tile0[r0 >> 4] + __popcll(splits & (((uint64_t)1 << (up + r)) - 1));
            const int q = a.g.hub_cptr[hrow], q1 = a.g.hub_cptr[hrow + 1];
            for (int s = 0; s < S; ++s)
                L.st[r * LR + 64 * s + lane] = hub_chunks_sum<64>(a.hub_part + (size_t)s * a.n_chunks * 64, q, q1, lane, 0.f);
        }
        wave_sync();
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            if (r0 + r >= a.n || ((done >> r) & 1u)) continue;
#pragma unroll
            for (int s = 0; s < S; ++s)
                __builtin_nontemporal_store(L.st[r * LR + 64 * s + lane], a.h + ((size_t)s * a.n + r0 + r) * 64 + lane);
        }
        walk.next(a.g);
    }
    walk.finish();
}

// Q = A X of dense rows (dY over A^T, or records held as rows over A), blockIdx.y a block of 64 columns: planes q [S][n][64]
template <typename T>
struct DensePlanesArgs {
    CsrView g;
    int n, tiles;
    const T* x;             // row stride ld; block y 64 y columns on
    int64_t ld;
    const float* hub_part;  // [S][chunks][64]
    int n_chunks;
    float* q;
    int* draws;             // a counter set per block
    int* draws_done;
    int y_draws;
};
template <typename T, bool DEAL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_dense_planes(DensePlanesArgs<T> a) {
    constexpr int LR = tile_ld<64>();
    const int block = blockIdx.y;
    const T* x = a.x + 64 * block;
    const float* part = a.hub_part + (size_t)block * a.n_chunks * 64;
    float* q = a.q + (size_t)block * a.n * 64;
    __shared__ WaveLds<64> lds[4];
    WaveLds<64>& L = lds[threadIdx.x >> 6];
    const int lane = lane_id(), tg = lane >> 4, tj = lane & 15;
    TileWalk<DEAL> walk(a.g, a.tiles, a.draws + block * a.y_draws, a.draws_done + block * a.y_draws);
    while (walk.more()) {
        walk.ahead();
        const int r0 = walk.t * 16;
        wave_sync();
        const int rpv = tile_rp_load(a.g, r0, a.n, lane);
        const bool has_hub = tile_begin(a.g, rpv, L.rp, lane);
        if (walk.dealt(a.g, rpv, L.rp, has_hub)) { walk.next(a.g); continue; }
        if constexpr (sizeof(T) == 4) {
            // (rows of one chunk are in q already: nothing to fill where no row has more)
            const int len = lane < 16 ? L.rp[lane + 1] - rpv : 0;
            const bool many = has_hub && ballot(len > a.g.hub_threshold && len > a.g.hub_chunk) != 0ull;
            for (int i = 4 * lane; i < 16 * LR; i += 256) *reinterpret_cast<f32v4*>(L.st + i) = f32v4{0.f, 0.f, 0.f, 0.f};
            wave_sync();
            tile_ranges(a.g, has_hub, L.rp, [&](int e_a, int e_b) {
                gather_dense_rows<64, 8>(a.g, x, a.ld, __builtin_amdgcn_readfirstlane(e_a), __builtin_amdgcn_readfirstlane(e_b), lane, L.st);
            });
            wave_sync();
            if (many) hub_rows_fill<64, true>(a.g, part, r0, L.rp, L.st, lane);
        } else {
            f32x4 acc[4];
            tile_gather<64>(a.g, part, has_hub, r0, L.rp, L.st, lane, acc, [&](int e_a, int e_b) {
                gather_dense_mfma<64, T, 8>(a.g, x, a.ld, __builtin_amdgcn_readfirstlane(e_a), __builtin_amdgcn_readfirstlane(e_b), L.rp,
                                            L.ebuf, lane, acc);
            });
        }
        wave_sync();
#pragma unroll
        for (int reg = 0; reg < 4; ++reg) {
            const int rr = 4 * reg + tg, row = r0 + rr, len = L.rp[rr + 1] - L.rp[rr];
            float v[4];
            lds_load<4>(L.st + rr * LR + 4 * tj, v);
            if (row < a.n && !(len > a.g.hub_threshold && len <= a.g.hub_chunk)) store_cols<4, float>(q + (size_t)row * 64 + 4 * tj, v);
        }
        walk.next(a.g);
    }
    walk.finish();
}

// The A operands of a 16-row tile's product, straight from a plane of [n][64] floats: row arow, columns 16 s + 4 kk .. of
// step s, split in three terms (mfma_tile_b3).
struct PlaneOperand {
    bf16x8 hi[2], mid[2], lo[2];
};
__device__ __forceinline__ void plane_request(const float* __restrict__ plane, int r0, int n, float (&v)[4][4]) {
    const int lane = lane_id(), i = lane & 15, kk = lane >> 4;
    const int row = min(r0 + 4 * (i & 3) + (i >> 2), n - 1);
#pragma unroll
    for (int s = 0; s < 4; ++s) load_cols<4, float>(plane + (size_t)row * 64 + 16 * s + 4 * kk, v[s]);
}
template <bool DEEP>
__device__ __forceinline__ void plane_product(const PlaneOperand& p, const WLdsB3<64, DEEP>& wl, f32x4 (&acc)[4]) {
    const int lane = lane_id();
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) acc[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 2; ++s) mfma_b3<64>(p.hi[s], p.mid[s], p.lo[s], wl, s, lane, acc);
}
// the columns of v (steps s of plane_request) in three terms
__device__ __forceinline__ void plane_split(const float (&v)[4][4], PlaneOperand& p) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        bf16x4 h[2], m[2], l[2];
        split_p4(v[2 * s], h[0], m[0], l[0]);
        split_p4(v[2 * s + 1], h[1], m[1], l[1]);
        p.hi[s] = join8(h[0], h[1]);
        p.mid[s] = join8(m[0], m[1]);
        p.lo[s] = join8(l[0], l[1]);
    }
}

// Workgroups of eight waves, a 16-row tile each, sharing W_i's blocks: row mb of blocks (of the transpose: column ob) at a
// time, S x 24.6 KB of LDS.  The row is rounded to its storage type after every block mb of the sum.
template <int S, typename T>
struct WideProductArgs {
    int n, tiles;
    const float* h;         // [S][n][64]
    const float* w;         // W_i, row stride 64 S
    T* plane;               // X_i on entry / Y_i on return (or the reverse), row stride ld
    int64_t ld;
};
template <int S, typename T, int SIGN>
__global__ __launch_bounds__(512) void k_wide_product(WideProductArgs<S, T> a) {
    __shared__ WLdsB3<64, deep_products<T>()> wl[S];
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), tg = lane >> 4, tj = lane & 15;
    const int t = (int)blockIdx.x * 8 + wave, r0 = t * 16;
    float y[S][4][4];
#pragma unroll
    for (int ob = 0; ob < S; ++ob)
#pragma unroll
        for (int reg = 0; reg < 4; ++reg) load_cols<4, T>(a.plane + (size_t)min(r0 + 4 * reg + tg, a.n - 1) * a.ld + 64 * ob + 4 * tj, y[ob][reg]);
#pragma unroll 1
    for (int mb = 0; mb < S; ++mb) {
        float v[4][4];
        plane_request(a.h + (size_t)mb * a.n * 64, r0, a.n, v);
        __syncthreads();        // the blocks before have been read
#pragma unroll 1
        for (int ob = 0; ob < S; ++ob) load_w_lds_b3(a.w + (size_t)mb * 64 * (64 * S) + 64 * ob, 64 * S, false, wl[ob]);
        PlaneOperand p;
        plane_split(v, p);
#pragma unroll
        for (int ob = 0; ob < S; ++ob) {
            f32x4 acc[4];
            plane_product(p, wl[ob], acc);
#pragma unroll
            for (int reg = 0; reg < 4; ++reg)
#pragma unroll
                for (int cb = 0; cb < 4; ++cb) y[ob][reg][cb] = stored<T>(SIGN > 0 ? y[ob][reg][cb] + acc[cb][reg] : y[ob][reg][cb] - acc[cb][reg]);
        }
    }
#pragma unroll
    for (int ob = 0; ob < S; ++ob)
#pragma unroll
        for (int reg = 0; reg < 4; ++reg) {
            const int row = r0 + 4 * reg + tg;
            if (row < a.n) store_cols<4, T>(a.plane + (size_t)row * a.ld + 64 * ob + 4 * tj, y[ob][reg]);
        }
}

// Two column blocks: all four blocks of W_i stay in LDS (98 KB) and a workgroup per compute unit sweeps tiles with them, each wave's next tile
// on its way while the present one is multiplied.  (Loading and splitting W_i again for every eight tiles was a third of the time: 200k nodes,
// groups of 128, X_i - H W_i 88 -> 72 us, back through W_i^T 99 -> 84 us; three blocks' W_i does not fit.)
template <typename T, int SIGN>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) void k_wide_product2(WideProductArgs<2, T> a) {
    __shared__ WLdsB3<64, deep_products<T>()> wl[2][2];
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), tg = lane >> 4, tj = lane & 15;
    const int step = (int)gridDim.x * 8;
    int t = (int)blockIdx.x * 8 + wave;
    float v[2][4][4], y[2][4][4];
    auto request = [&](int tile) {
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) plane_request(a.h + (size_t)mb * a.n * 64, tile * 16, a.n, v[mb]);
#pragma unroll
        for (int ob = 0; ob < 2; ++ob)
#pragma unroll
            for (int reg = 0; reg < 4; ++reg) load_cols<4, T>(a.plane + (size_t)min(tile * 16 + 4 * reg + tg, a.n - 1) * a.ld + 64 * ob + 4 * tj, y[ob][reg]);
    };
    if (t < a.tiles) request(t);
#pragma unroll 1
    for (int b = 0; b < 4; ++b) load_w_lds_b3(a.w + (size_t)(b >> 1) * 64 * 128 + 64 * (b & 1), 128, false, wl[b >> 1][b & 1]);
    while (t < a.tiles) {
        const int r0 = t * 16;
        PlaneOperand p[2];
        float out[2][4][4];
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) plane_split(v[mb], p[mb]);
#pragma unroll
        for (int ob = 0; ob < 2; ++ob)
#pragma unroll
            for (int reg = 0; reg < 4; ++reg)
#pragma unroll
                for (int cb = 0; cb < 4; ++cb) out[ob][reg][cb] = y[ob][reg][cb];
        t += step;
        if (t < a.tiles) request(t);
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int ob = 0; ob < 2; ++ob) {
                f32x4 acc[4];
                wave_sync();          // (W_i's operands are read from LDS here, not kept in registers for the whole sweep)
                plane_product(p[mb], wl[mb][ob], acc);
#pragma unroll
                for (int reg = 0; reg < 4; ++reg)
#pragma unroll
                    for (int cb = 0; cb < 4; ++cb) out[ob][reg][cb] = stored<T>(SIGN > 0 ? out[ob][reg][cb] + acc[cb][reg] : out[ob][reg][cb] - acc[cb][reg]);
            }
#pragma unroll
        for (int ob = 0; ob < 2; ++ob)
#pragma unroll
            for (int reg = 0; reg < 4; ++reg) {
                const int row = r0 + 4 * reg + tg;
                if (row < a.n) store_cols<4, T>(a.plane + (size_t)row * a.ld + 64 * ob + 4 * tj, out[ob][reg]);
            }
    }
}

// dH = Q W_i^T, then back through GS and its scale: dZ_c = [c in I] g_c / r - Z_c (sum_t g_t Z_{I_t}) / (D/C r^3) with g = dH
// at the recorded positions (eq. (11): only those are read); dst planes += dZ.
template <int S, typename T>
struct WideGradArgs {
    int n, tiles;
    const float* q;                     // [S][n][64]
    const float* w;                     // W_i, row stride 64 S
    const uint64_t* mask[S];            // column sets recorded for the block's input
    const T* z;                         // rows of the block's input (RMS only): row stride ldz, sub-plane s at + s * z_sub
    int64_t ldz, z_sub;
    int norm;
    float eps;
    T* dst;                             // ndst groups, dst_gs apart, row stride ldd
    int64_t ldd, dst_gs;
    int ndst;
};
// What that takes of a 16-row tile beside dH: its own rows and column sets, and (one of them) the rows that receive dZ.
template <int S>
struct WideGradRows {
    float z[4][S][4];
    uint64_t mask[4][S];
    float d[4][S][4];
};
template <int S, typename T>
__device__ __forceinline__ void wide_grad_request(const WideGradArgs<S, T>& a, int r0, int reg, bool with_dst, WideGradRows<S>& w) {
    const int lane = lane_id(), tg = lane >> 4, tj = lane & 15, rowc = min(r0 + 4 * reg + tg, a.n - 1);
#pragma unroll
    for (int s = 0; s < S; ++s) {
        w.mask[reg][s] = a.mask[s][rowc];
        if (a.norm == GSR_NORM_RMS) load_cols<4, T>(a.z + (size_t)rowc * a.ldz + (size_t)s * a.z_sub + 4 * tj, w.z[reg][s]);
        if (with_dst) load_cols<4, T>(a.dst + (size_t)rowc * a.ldd + 64 * s + 4 * tj, w.d[reg][s]);
    }
}
// back through GS and its scale: g = dH of the tile -> dZ
template <int S, typename T>
__device__ __forceinline__ void wide_grad_back(const WideGradArgs<S, T>& a, float (&g)[S][4][4], int reg, const WideGradRows<S>& w) {
    constexpr int DGW = 64 * S;
    const int tj = lane_id() & 15;
    uint32_t bits[S];
#pragma unroll
    for (int s = 0; s < S; ++s) bits[s] = (uint32_t)(w.mask[reg][s] >> (4 * tj)) & 15u;
    if (a.norm == GSR_NORM_RMS) {
        float ss = 0.f, dot = 0.f;
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) {
                ss += w.z[reg][s][cb] * w.z[reg][s][cb];
                dot += ((bits[s] >> cb) & 1u) ? g[s][reg][cb] * w.z[reg][s][cb] : 0.f;
            }
        ss = group16_sum(ss);
        dot = group16_sum(dot);
        const float rinv = __builtin_amdgcn_rsqf(ss * (1.0f / (float)DGW) + a.eps);
        const float coef = dot * (rinv * rinv * rinv) * (1.0f / (float)DGW);
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) g[s][reg][cb] = (((bits[s] >> cb) & 1u) ? g[s][reg][cb] * rinv : 0.f) - w.z[reg][s][cb] * coef;
    } else {
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) g[s][reg][cb] = ((bits[s] >> cb) & 1u) ? g[s][reg][cb] : 0.f;
    }
}
// the planes j0 .. ndst - 1 that receive dZ
template <int S, typename T>
__device__ __forceinline__ void wide_grad_add(const WideGradArgs<S, T>& a, const float (&g)[S][4][4], int r0, int j0) {
    const int lane = lane_id(), tg = lane >> 4, tj = lane & 15;
    for (int j = j0; j < a.ndst; ++j)
#pragma unroll
        for (int s = 0; s < S; ++s) {
            float d[4][4];
            T* p = a.dst + (size_t)j * a.dst_gs + 64 * s + 4 * tj;
#pragma unroll
            for (int reg = 0; reg < 4; ++reg) load_cols<4, T>(p + (size_t)min(r0 + 4 * reg + tg, a.n - 1) * a.ldd, d[reg]);
#pragma unroll
            for (int reg = 0; reg < 4; ++reg) {
                const int row = r0 + 4 * reg + tg;
#pragma unroll
                for (int cb = 0; cb < 4; ++cb) d[reg][cb] = stored<T>(d[reg][cb] + g[s][reg][cb]);
                if (row < a.n) store_cols<4, T>(p + (size_t)row * a.ldd, d[reg]);
            }
        }
}

template <int S, typename T>
__global__ __launch_bounds__(512) void k_wide_grad(WideGradArgs<S, T> a) {
    constexpr int DGW = 64 * S;
    __shared__ WLdsB3<64, deep_products<T>()> wl[S];
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), tg = lane >> 4, tj = lane & 15;
    const int t = (int)blockIdx.x * 8 + wave, r0 = t * 16;
    float g[S][4][4];
#pragma unroll
    for (int mb = 0; mb < S; ++mb)
#pragma unroll
        for (int reg = 0; reg < 4; ++reg)
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) g[mb][reg][cb] = 0.f;
#pragma unroll 1
    for (int ob = 0; ob < S; ++ob) {
        float v[4][4];
        plane_request(a.q + (size_t)ob * a.n * 64, r0, a.n, v);
        __syncthreads();
#pragma unroll 1
        for (int mb = 0; mb < S; ++mb) load_w_lds_b3(a.w + (size_t)mb * 64 * DGW + 64 * ob, DGW, true, wl[mb]);
        PlaneOperand p;
        plane_split(v, p);
#pragma unroll
        for (int mb = 0; mb < S; ++mb) {
            f32x4 acc[4];
            plane_product(p, wl[mb], acc);
#pragma unroll
            for (int reg = 0; reg < 4; ++reg)
#pragma unroll
                for (int cb = 0; cb < 4; ++cb) g[mb][reg][cb] += acc[cb][reg];
        }
    }
    WideGradRows<S> w;
#pragma unroll
    for (int reg = 0; reg < 4; ++reg) {
        wide_grad_request<S, T>(a, r0, reg, false, w);
        wide_grad_back<S, T>(a, g, reg, w);
    }
    wide_grad_add<S, T>(a, g, r0, 0);
}

// Two column blocks, as k_wide_product2
template <typename T>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) void k_wide_grad2(WideGradArgs<2, T> a) {
    __shared__ WLdsB3<64, deep_products<T>()> wl[2][2];          // [ob][mb]
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int step = (int)gridDim.x * 8;
    int t = (int)blockIdx.x * 8 + wave;
    float v[2][4][4];
    auto request = [&](int tile) {
#pragma unroll
        for (int ob = 0; ob < 2; ++ob) plane_request(a.q + (size_t)ob * a.n * 64, tile * 16, a.n, v[ob]);
    };
    if (t < a.tiles) request(t);
#pragma unroll 1
    for (int b = 0; b < 4; ++b) load_w_lds_b3(a.w + (size_t)(b & 1) * 64 * 128 + 64 * (b >> 1), 128, true, wl[b >> 1][b & 1]);
    while (t < a.tiles) {
        const int r0 = t * 16;
        PlaneOperand p[2];
        float g[2][4][4];
#pragma unroll
        for (int ob = 0; ob < 2; ++ob) plane_split(v[ob], p[ob]);
        WideGradRows<2> w;
#pragma unroll
        for (int reg = 0; reg < 4; ++reg) wide_grad_request<2, T>(a, r0, reg, true, w);
        t += step;
        if (t < a.tiles) request(t);
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) {
            f32x4 acc[2][4];
#pragma unroll
            for (int ob = 0; ob < 2; ++ob) {
                wave_sync();          // (as in k_wide_product2)
                plane_product(p[ob], wl[ob][mb], acc[ob]);
            }
#pragma unroll
            for (int reg = 0; reg < 4; ++reg)
#pragma unroll
                for (int cb = 0; cb < 4; ++cb) g[mb][reg][cb] = acc[0][cb][reg] + acc[1][cb][reg];
        }
#pragma unroll
        for (int reg = 0; reg < 4; ++reg) {
            const int lane = lane_id(), row = r0 + 4 * reg + (lane >> 4);
            wide_grad_back<2, T>(a, g, reg, w);
#pragma unroll
            for (int s = 0; s < 2; ++s) {
#pragma unroll
                for (int cb = 0; cb < 4; ++cb) w.d[reg][s][cb] = stored<T>(w.d[reg][s][cb] + g[s][reg][cb]);
                if (row < a.n) store_cols<4, T>(a.dst + (size_t)row * a.ldd + 64 * s + 4 * (lane & 15), w.d[reg][s]);
            }
        }
        wide_grad_add<2, T>(a, g, r0, 1);
    }
}

// ---- gradient on graphs of long rows in a band --------------------------------------------------------------------
// dH_i = A^T dY_i W_i^T is read only at the k columns recorded for each row (eq. (11)).  A row that gathers its hundreds of
// neighbours' whole rows of dY_i moves D/C values per entry to use k of D/C sums: 50k nodes of mean degree 236, groups of 192: 3 GB
// per block of 64 columns from L2 to the compute units, three blocks of 172 us.  Here the product goes first, P = dY_i W_i^T
// (k_pre_product), and then the entries add a_ij P[j][c] for the recorded c alone (k_band_gather), from LDS: a workgroup takes
// B adjacent rows, whose neighbours lie in a band, and walks the band in windows of rows of P, every one staged once for all its
// rows (how many entries share a staged row decides whether that pays: band_rows_of).  k_band_back takes the sums back through GS.
// Per block of that graph, us: 516 of first passes, 18 of tiles and 45 of the product -> 33 + 178 + 27 (backward layer 1,770 ->
// 1,086; error of dX against 64 bits, median row, 11 - 14 % lower on five such graphs and widths, dW 0 - 8 %).
template <int DG, int S, typename T>
struct PreProductArgs {
    int n;
    const T* dy;            // row stride ld; block ob 64 ob columns on
    int64_t ld;
    const float* w;         // W_i, row stride DG S
    float* p;               // [n][DG S]
};
// Workgroups of eight waves, a 16-row tile each, sharing column ob of W_i's blocks at a time.  The sums of the matrix instructions
// are not rounded to nearest but to one side, and a few hundred rows of P are added up: odd rows are multiplied with their sign turned and
// turned back, so that what one row loses another gains (dW, which adds up the rows of dY: error against 64 bits 1.5e-7 with it,
// 3.0e-7 without; 30k nodes, groups of 128).
template <int DG, int S, typename T>
__global__ __launch_bounds__(512) void k_pre_product(PreProductArgs<DG, S, T> a) {
    constexpr int CPL = DG / 16, DGW = DG * S;
    __shared__ WLdsB3<DG, true> wl[S];
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), tg = lane >> 4, tj = lane & 15;
    const int r0 = ((int)blockIdx.x * 8 + wave) * 16;
    const int arow = min(r0 + 4 * (tj & 3) + (tj >> 2), a.n - 1);
    const uint32_t flip_in = (uint32_t)(tj >> 2 & 1) << 31, flip_out = (uint32_t)(tg & 1) << 31;      // of the odd rows
    f32x4 acc[S][CPL];
#pragma unroll
    for (int mb = 0; mb < S; ++mb)
#pragma unroll
        for (int cb = 0; cb < CPL; ++cb) acc[mb][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int ob = 0; ob < S; ++ob) {
        float v[DG / 16][4];
#pragma unroll
        for (int s = 0; s < DG / 16; ++s) load_cols<4, T>(a.dy + (size_t)arow * a.ld + 64 * ob + 16 * s + 4 * tg, v[s]);
#pragma unroll
        for (int s = 0; s < DG / 16; ++s)
#pragma unroll
            for (int u = 0; u < 4; ++u) v[s][u] = __uint_as_float(__float_as_uint(v[s][u]) ^ flip_in);
        __syncthreads();        // the blocks before have been read
#pragma unroll 1
        for (int mb = 0; mb < S; ++mb) load_w_lds_b3(a.w + (size_t)mb * 64 * DGW + 64 * ob, DGW, true, wl[mb]);
        bf16x8 hi[DG / 32], mid[DG / 32], lo[DG / 32];
#pragma unroll
        for (int s = 0; s < DG / 32; ++s) {
            bf16x4 h[2], m[2], l[2];
            split_p4(v[2 * s], h[0], m[0], l[0]);
            split_p4(v[2 * s + 1], h[1], m[1], l[1]);
            hi[s] = join8(h[0], h[1]); mid[s] = join8(m[0], m[1]); lo[s] = join8(l[0], l[1]);
        }
#pragma unroll
        for (int mb = 0; mb < S; ++mb) {
            f32x4 sum[CPL];          // (from zero for every block, as in k_wide_grad)
#pragma unroll
            for (int cb = 0; cb < CPL; ++cb) sum[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < DG / 32; ++s) mfma_b3<DG>(hi[s], mid[s], lo[s], wl[mb], s, lane, sum);
#pragma unroll
            for (int cb = 0; cb < CPL; ++cb)
#pragma unroll
                for (int reg = 0; reg < 4; ++reg) acc[mb][cb][reg] += sum[cb][reg];
        }
    }
    if constexpr (S == 1) {
        // The terms of an infinity (inf - inf is one of them) add up to a NaN.  The gather of whole rows multiplies groups of up to 64 columns
        // by the float32 instructions, which keep it, so what came out as no number is multiplied again in ordinary arithmetic.
        bool finite = true;
#pragma unroll
        for (int cb = 0; cb < CPL; ++cb)
#pragma unroll
            for (int reg = 0; reg < 4; ++reg) finite = finite && __builtin_isfinite(acc[0][cb][reg]);
        if (ballot(!finite) != 0) {
            float sum[4][CPL] = {};
#pragma unroll 1
            for (int o = 0; o < DG; ++o) {
                float d[4], w[CPL];
#pragma unroll
                for (int reg = 0; reg < 4; ++reg) d[reg] = to_float(a.dy[(size_t)min(r0 + 4 * reg + tg, a.n - 1) * a.ld + o]);
#pragma unroll
                for (int cb = 0; cb < CPL; ++cb) w[cb] = a.w[(size_t)(CPL * tj + cb) * DG + o];
#pragma unroll
                for (int reg = 0; reg < 4; ++reg)
#pragma unroll
                    for (int cb = 0; cb < CPL; ++cb) sum[reg][cb] = __builtin_fmaf(d[reg], w[cb], sum[reg][cb]);
            }
#pragma unroll
            for (int cb = 0; cb < CPL; ++cb)
#pragma unroll
                for (int reg = 0; reg < 4; ++reg)
                    if (!__builtin_isfinite(acc[0][cb][reg])) acc[0][cb][reg] = __uint_as_float(__float_as_uint(sum[reg][cb]) ^ flip_out);
        }
    }
#pragma unroll
    for (int mb = 0; mb < S; ++mb)
#pragma unroll
        for (int reg = 0; reg < 4; ++reg) {
            const int row = r0 + 4 * reg + tg;
            float v[CPL];
#pragma unroll
            for (int cb = 0; cb < CPL; ++cb) v[cb] = __uint_as_float(__float_as_uint(acc[mb][cb][reg]) ^ flip_out);
            if (row < a.n) store_cols<CPL, float, true>(a.p + (size_t)row * DGW + 64 * mb + CPL * tj, v);
        }
}

struct BandGatherArgs {
    CsrView gt;             // A^T
    int n, rows;            // rows per workgroup, at most 64 BAND_ROWS
    const float* p;         // [n][DGW]
    const uint8_t* cols;    // [n][k] recorded columns
    int k;
    float* out;             // [n][k]
};
constexpr int BAND_ROWS = 4;                    // rows per group of sixteen lanes
constexpr int BAND_FLOATS = 18432;              // of a window: 73,728 bytes, a whole number of rows of 32, 64, 128, 192 or 256 columns
// Sixteen waves; a group of sixteen lanes owns rows G, G + 64, .. of the workgroup's, lane l of it the sums of the recorded columns
// l, l + 16, .. (KQ of them).  Two windows of P in LDS: while the entries of one are added the next is on its way (loads straight
// into LDS).  The entries of a row are in ascending column order, so those of a window follow those of the one before; sixteen
// of them at a time sit in the lanes of the group (row_lane hands them out), the next sixteen are requested when it is known how many of these
// the window took.  A window's entries are summed from zero, eight windows' sums from zero again, which bounds the length of the
// chains of additions.  Places past the window's entries read a row of zeros.  50k nodes of mean degree 236, 192 columns: 173 us, 94 of them for
// the windows alone (1.2 GB into LDS) and 139 for the sums alone, which the LDS bounds: 6.1M reads counted, 16 cycles of a compute unit each over the
// launch, 4.5 of them bank conflicts of the 64 columns; 2.9M would do if the runs of four groups were equally long and whole fours (all rows' first eight
// places read before the first is added, a quarter more reads: 217).
template <int DGW, int KQ>
__global__ __launch_bounds__(1024) void k_band_gather(BandGatherArgs a) {
    constexpr int WROWS = BAND_FLOATS / DGW, ROWB = 4 * DGW;
    static_assert(BAND_FLOATS % DGW == 0 && ROWB % 128 == 0, "a window is a whole number of rows");
    struct Lds {
        alignas(16) float win[2][BAND_FLOATS];
        float zero[DGW];
        int lo, hi;
    };
    __shared__ Lds L;
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = lane & 15, gi = lane >> 4;
    // adjacent blocks of rows on one XCD: they share most of their bands
    const int per = (int)(gridDim.x + 7) / 8, block = ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);
    const int first = block * a.rows, last = min(first + a.rows, a.n);      // (first may lie past the end: no rows)
    if (threadIdx.x == 0) { L.lo = a.n; L.hi = 0; }
    if ((int)threadIdx.x < DGW) L.zero[threadIdx.x] = 0.f;
    __syncthreads();
    int ptr[BAND_ROWS], end[BAND_ROWS];
    uint32_t coff[BAND_ROWS][KQ];
    float acc[BAND_ROWS][KQ], total[BAND_ROWS][KQ];
#pragma unroll
    for (int q = 0; q < BAND_ROWS; ++q) {
        const int in = 4 * wave + gi + 64 * q, row = first + in;
        const bool ok = in < a.rows && row < last;
        ptr[q] = ok ? a.gt.rp[row] : 0;
        end[q] = ok ? a.gt.rp[row + 1] : 0;
        if (end[q] > ptr[q] && l == 0) {
            atomicMin(&L.lo, a.gt.ci[ptr[q]]);
            atomicMax(&L.hi, a.gt.ci[end[q] - 1] + 1);
        }
#pragma unroll
        for (int w = 0; w < KQ; ++w) {
            const int t = l + 16 * w;
            coff[q][w] = ok && t < a.k ? 4u * a.cols[(size_t)row * a.k + t] : 0u;
            acc[q][w] = total[q][w] = 0.f;
        }
    }
    int j[BAND_ROWS];
    float av[BAND_ROWS];
    auto request = [&](int q) {          // the next sixteen entries of row q (past the end: an entry that exists, not used)
        const int e = ptr[q] + l, ec = e < end[q] ? e : max(end[q] - 1, 0);
        j[q] = a.gt.ci[ec];
        av[q] = a.gt.av[ec];
    };
#pragma unroll
    for (int q = 0; q < BAND_ROWS; ++q) request(q);
    __syncthreads();
    const int lo = __builtin_amdgcn_readfirstlane(L.lo), hi = __builtin_amdgcn_readfirstlane(L.hi);
    // window at row w0 on into buffer b: a wave moves 64 pieces of 16 bytes per instruction
    auto stage = [&](int w0, int b) {
        const int pieces = min(WROWS, a.n - w0) * (DGW / 4);
        const char* src = reinterpret_cast<const char*>(a.p + (size_t)w0 * DGW);
        for (int i = wave; 64 * i < pieces; i += 16) {
            const int piece = min(64 * i + lane, pieces - 1);
            __builtin_amdgcn_global_load_lds(reinterpret_cast<const __attribute__((address_space(1))) void*>(reinterpret_cast<uintptr_t>(src + 16 * (size_t)piece)),
                                             (__attribute__((address_space(3))) void*)&L.win[b][256 * i], 16, 0, 0);
        }
    };
    const uint32_t zero = (uint32_t)(uintptr_t)(lds_float*)&L.zero[0];
    if (lo < hi) stage(lo, 0);
    for (int w0 = lo, step = 0; w0 < hi; w0 += WROWS, ++step) {
        const int b = step & 1;
        __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0): this wave's pieces of the window have arrived
        __syncthreads();                         // everyone's have, and nobody reads the other buffer any more
        if (w0 + WROWS < hi) stage(w0 + WROWS, b ^ 1);
        const uint32_t base = (uint32_t)(uintptr_t)(lds_float*)&L.win[b][0];
#pragma unroll
        for (int q = 0; q < BAND_ROWS; ++q) {
            float sum[KQ];
#pragma unroll
            for (int w = 0; w < KQ; ++w) sum[w] = 0.f;
            // the entries of the window among the sixteen in the lanes; whether there may be more of them
            auto pass = [&]() -> bool {
                const bool mine = ptr[q] + l < end[q] && j[q] < w0 + WROWS;
                const uint64_t m = ballot(mine);
                if (m == 0) return false;
                const uint32_t off = mine ? base + (uint32_t)(j[q] - w0) * ROWB : zero;
                const uint32_t f = __float_as_uint(mine ? av[q] : 0.f);
                uint32_t any = (uint32_t)m | (uint32_t)(m >> 32);
                any = (any | any >> 16) & 0xFFFFu;          // places any of the four groups has an entry in (each a run from place 0)
                ptr[q] += __popc((uint32_t)(m >> (16 * gi)) & 0xFFFFu);
                request(q);
                auto four = [&](auto sc) {
                    constexpr int S0 = decltype(sc)::value;
                    float v[4][KQ];
#pragma unroll
                    for (int w = 0; w < KQ; ++w) {
                        v[0][w] = *(lds_float*)(uintptr_t)(row_lane<S0>(off) + coff[q][w]);
                        v[1][w] = *(lds_float*)(uintptr_t)(row_lane<S0 + 1>(off) + coff[q][w]);
                        v[2][w] = *(lds_float*)(uintptr_t)(row_lane<S0 + 2>(off) + coff[q][w]);
                        v[3][w] = *(lds_float*)(uintptr_t)(row_lane<S0 + 3>(off) + coff[q][w]);
                    }
#pragma unroll
                    for (int w = 0; w < KQ; ++w) {
                        sum[w] = __builtin_fmaf(__uint_as_float(row_lane<S0>(f)), v[0][w], sum[w]);
                        sum[w] = __builtin_fmaf(__uint_as_float(row_lane<S0 + 1>(f)), v[1][w], sum[w]);
                        sum[w] = __builtin_fmaf(__uint_as_float(row_lane<S0 + 2>(f)), v[2][w], sum[w]);
                        sum[w] = __builtin_fmaf(__uint_as_float(row_lane<S0 + 3>(f)), v[3][w], sum[w]);
                    }
                };
                four(std::integral_constant<int, 0>{});
                if (any >> 4) four(std::integral_constant<int, 4>{});
                if (any >> 8) four(std::integral_constant<int, 8>{});
                if (any >> 12) four(std::integral_constant<int, 12>{});
                return any >> 15;                           // some group has seen sixteen
            };
            // (the first pass on its own: its entries arrived before the barrier, those of a further one are waited for, and with them
            // the window under way)
            if (pass())
                while (pass()) {}
#pragma unroll
            for (int w = 0; w < KQ; ++w) acc[q][w] += sum[w];
        }
        if ((step & 7) == 7 || w0 + WROWS >= hi) {
#pragma unroll
            for (int q = 0; q < BAND_ROWS; ++q)
#pragma unroll
                for (int w = 0; w < KQ; ++w) {
                    total[q][w] += acc[q][w];
                    acc[q][w] = 0.f;
                }
        }
    }
#pragma unroll
    for (int q = 0; q < BAND_ROWS; ++q) {
        const int in = 4 * wave + gi + 64 * q, row = first + in;
        if (in >= a.rows || row >= last) continue;
#pragma unroll
        for (int w = 0; w < KQ; ++w) {
            const int t = l + 16 * w;
            if (t < a.k) a.out[(size_t)row * a.k + t] = total[q][w];
        }
    }
}

// dst planes += dZ, with g = dH at the recorded positions as k_band_gather left them: dZ_c = [c in I] g_c / r - Z_c (sum_t g_t Z_{I_t}) /
// (D/C r^3).  A wave takes a 16-row tile; the slot of a recorded column is the number of recorded columns before it.
template <int DG, int S, typename T>
struct BandBackArgs {
    using M = typename MaskOf<DG>::type;
    int n, tiles;
    const float* g;                     // [n][k]
    int k;
    const M* mask[S];                   // column sets recorded for the block's input
    const T* z;                         // rows of the block's input (RMS only): row stride ldz, sub-plane s at + s * z_sub
    int64_t ldz, z_sub;
    int norm;
    float eps;
    T* dst;                             // ndst groups, dst_gs apart, row stride ldd
    int64_t ldd, dst_gs;
    int ndst;
};
template <int DG, int S, typename T>
__global__ __launch_bounds__(256) void k_band_back(BandBackArgs<DG, S, T> a) {
    using M = typename MaskOf<DG>::type;
    constexpr int CPL = DG / 16, DGW = DG * S;
    const int lane = lane_id(), tg = lane >> 4, tj = lane & 15;
    const int t = (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6), r0 = t * 16;
    if (t >= a.tiles) return;
#pragma unroll
    for (int reg = 0; reg < 4; ++reg) {
        const int row = r0 + 4 * reg + tg, rowc = min(row, a.n - 1);
        float g[S][CPL];
        bool bit[S][CPL];
        int slot = 0;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const M m = a.mask[s][rowc];
            int at = slot + popc<DG>(m & (((M)1 << (CPL * tj)) - 1));
            slot += popc<DG>(m);
#pragma unroll
            for (int cb = 0; cb < CPL; ++cb) {
                bit[s][cb] = (m >> (CPL * tj + cb)) & 1u;
                const float v = a.g[(size_t)rowc * a.k + (at < a.k ? at : a.k - 1)];
                g[s][cb] = bit[s][cb] ? v : 0.f;
                at += bit[s][cb] ? 1 : 0;
            }
        }
        if (a.norm == GSR_NORM_RMS) {
            float z[S][CPL], ss = 0.f, dot = 0.f;
#pragma unroll
            for (int s = 0; s < S; ++s) load_cols<CPL, T>(a.z + (size_t)rowc * a.ldz + (size_t)s * a.z_sub + CPL * tj, z[s]);
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int cb = 0; cb < CPL; ++cb) {
                    ss += z[s][cb] * z[s][cb];
                    dot += g[s][cb] * z[s][cb];
                }
            ss = group16_sum(ss);
            dot = group16_sum(dot);
            const float rinv = __builtin_amdgcn_rsqf(ss * (1.0f / (float)DGW) + a.eps);
            const float coef = dot * (rinv * rinv * rinv) * (1.0f / (float)DGW);
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int cb = 0; cb < CPL; ++cb) g[s][cb] = (bit[s][cb] ? g[s][cb] * rinv : 0.f) - z[s][cb] * coef;
        }
        for (int d = 0; d < a.ndst; ++d) {
            T* p = a.dst + (size_t)d * a.dst_gs + (size_t)rowc * a.ldd + CPL * tj;
            float v[S][CPL];
#pragma unroll
            for (int s = 0; s < S; ++s) load_cols<CPL, T>(p + 64 * s, v[s]);
#pragma unroll
            for (int s = 0; s < S; ++s) {
#pragma unroll
                for (int cb = 0; cb < CPL; ++cb) v[s][cb] = stored<T>(v[s][cb] + g[s][cb]);
                if (row < a.n) store_cols<CPL, T>(p + 64 * s, v[s]);
            }
        }
    }
}

template <int S, typename T>
struct WideGsArgs {
    int n;
    const T* src;           // nsrc groups, src_gs apart, row stride ld; sub-plane s of a row starts at + 64 s
    int64_t ld, src_gs;
    int nsrc;
    T* y0;                  // [S][n][64]: the sum, sub-plane by sub-plane (NULL: not kept)
    int k, norm;
    float eps;
    T* vals;                // the record: [n][k] values of the whole row in column order and their columns,
    uint8_t* cols;          // or (cols == NULL) rows [n][64 S] with zeros in the dropped columns
    uint64_t* mask[S];
    bool out_given;         // mask[s] hold the column sets to use
};

// GS of a 16-row tile of a wide group, lane (r, q) holding the q-th quarter (16 columns) of every sub-plane of row r:
// the same search as select_quarter over 16 S keys per lane; ties go to the lowest column of the whole row (sub-plane,
// then quarter, then column).
template <int S, typename T>
__global__ __launch_bounds__(256) void k_gs_wide(WideGsArgs<S, T> a) {
    constexpr int DGW = 64 * S, LRW = tile_ld<DGW>();
    constexpr int KS = sizeof(T) == 2 ? 16 : 0;
    __shared__ __attribute__((aligned(16))) float tile[4][16 * LRW + 64];
    const int lane = lane_id(), tg = lane >> 4, tj = lane & 15, r = lane & 15, q = lane >> 4;
    float* st = tile[threadIdx.x >> 6];
    const int nwaves = (gridDim.x * blockDim.x) >> 6, tiles = (a.n + 15) / 16;
    for (int t = (blockIdx.x * blockDim.x + threadIdx.x) >> 6; t < tiles; t += nwaves) {
        const int r0 = t * 16;
        wave_sync();          // the previous tile's records have left the scratch
        {
            float y[S][4][4];
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int reg = 0; reg < 4; ++reg)
                    load_cols<4, T>(a.src + (size_t)min(r0 + 4 * reg + tg, a.n - 1) * a.ld + 64 * s + 4 * tj, y[s][reg]);
            for (int j = 1; j < a.nsrc; ++j) {
                float v[S][4][4];
#pragma unroll
                for (int s = 0; s < S; ++s)
#pragma unroll
                    for (int reg = 0; reg < 4; ++reg)
                        load_cols<4, T>(a.src + (size_t)j * a.src_gs + (size_t)min(r0 + 4 * reg + tg, a.n - 1) * a.ld + 64 * s + 4 * tj, v[s][reg]);
#pragma unroll
                for (int s = 0; s < S; ++s)
#pragma unroll
                    for (int reg = 0; reg < 4; ++reg)
#pragma unroll
                        for (int cb = 0; cb < 4; ++cb) y[s][reg][cb] += v[s][reg][cb];
            }
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int reg = 0; reg < 4; ++reg) {
                    const int rr = 4 * reg + tg, row = r0 + rr;
                    const bool ok = row < a.n;
#pragma unroll
                    for (int cb = 0; cb < 4; ++cb) y[s][reg][cb] = stored<T>(y[s][reg][cb]);
                    if (ok && a.y0) store_cols<4, T>(a.y0 + ((size_t)s * a.n + row) * 64 + 4 * tj, y[s][reg]);
#pragma unroll
                    for (int cb = 0; cb < 4; ++cb) y[s][reg][cb] = ok ? y[s][reg][cb] : 0.f;
                    lds_store<4>(st + rr * LRW + 64 * s + 4 * tj, y[s][reg]);
                }
        }
        wave_sync();
        const bool valid = r0 + r < a.n;
        float x[S][16];
        float ss = 0.f;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            lds_load<16>(st + r * LRW + 64 * s + 16 * q, x[s]);
#pragma unroll
            for (int j = 0; j < 16; ++j) ss += x[s][j] * x[s][j];
        }
        uint32_t msel[S];
        if (a.out_given) {
#pragma unroll
            for (int s = 0; s < S; ++s) msel[s] = (uint32_t)(a.mask[s][valid ? r0 + r : a.n - 1] >> (16 * q)) & 0xFFFFu;
        } else {
            uint32_t key[S][16];
            uint32_t top = 0u;
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const uint32_t u = __float_as_uint(x[s][j] + 0.0f);          // -0 -> +0
                    key[s][j] = (u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u)) >> KS;
                    top = max(top, key[s][j]);
                }
            top = quarter_max(top);
            auto count_ge = [&](uint32_t th) {
                uint32_t cnt = 0u;
#pragma unroll
                for (int s = 0; s < S; ++s)
#pragma unroll
                    for (int j = 0; j < 16; ++j) cnt += key[s][j] >= th ? 1u : 0u;
                return quarter_sum(cnt);
            };
            constexpr uint32_t span = (4u << 23) >> KS;
            const uint32_t uk = (uint32_t)a.k;
            uint32_t lo = top > span ? top - span : 0u, hi = top + 1u;
            {
                const uint32_t cnt = count_ge(lo);
                lo = (cnt >= uk && a.k < DGW) ? lo : 0u;
                uint32_t open = (cnt != uk && a.k < DGW && valid) ? 1u : 0u;
                for (int round = 0; round < 33 && ballot(open != 0u) != 0ull; ++round) {
                    const uint32_t mid = lo + ((hi - lo) >> 1);
                    const uint32_t c2 = count_ge(mid);
                    lo = c2 >= uk ? mid : lo;
                    hi = c2 >= uk ? hi : mid;
                    open = (c2 == uk || hi - lo <= 1u) ? 0u : open;
                }
            }
            // kept: every key above the threshold, and of those at the threshold the lowest columns of the row
            uint32_t mgt[S], meq[S];
            int ngt = 0;
#pragma unroll
            for (int s = 0; s < S; ++s) {
                mgt[s] = meq[s] = 0u;
#pragma unroll
                for (int j = 15; j >= 0; --j) {
                    mgt[s] = mgt[s] + mgt[s] + (key[s][j] > lo ? 1u : 0u);
                    meq[s] = meq[s] + meq[s] + (key[s][j] == lo ? 1u : 0u);
                }
                ngt += __popc(mgt[s]);
            }
            int need = a.k - (int)quarter_sum((uint32_t)ngt);      // ties to take, in column order
#pragma unroll
            for (int s = 0; s < S; ++s) {
                uint32_t all[4];
                quarter_all((uint32_t)__popc(meq[s]), all);
                int before = 0;
#pragma unroll
                for (int i = 0; i < 3; ++i) before += i < q ? (int)all[i] : 0;
                int take = min(max(need - before, 0), (int)__popc(meq[s]));
                msel[s] = mgt[s];
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const uint32_t sbit = ((meq[s] >> j) & 1u) & (take > 0 ? 1u : 0u);
                    msel[s] |= sbit << j;
                    take -= (int)sbit;
                }
                need -= (int)(all[0] + all[1] + all[2] + all[3]);
            }
        }
        float scale = 1.f;
        if (a.norm == GSR_NORM_RMS) scale = __builtin_amdgcn_rsqf(quarter_sum(ss) * (1.0f / (float)DGW) + a.eps);
        const int rows = min(16, a.n - r0), total = rows * a.k;
        // first slot of this lane's quarter of every sub-plane, in column order over the whole row
        int slot[S], at = r * a.k;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            uint32_t all[4];
            quarter_all(msel[s] | (uint32_t)__popc(msel[s]) << 16, all);
            slot[s] = at;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                slot[s] += i < q ? (int)(all[i] >> 16) : 0;
                at += (int)(all[i] >> 16);
            }
            if (!a.out_given && q == 0 && r < rows)
                a.mask[s][r0 + r] = (uint64_t)(all[0] & 0xFFFFu) | (uint64_t)(all[1] & 0xFFFFu) << 16 |
                                    (uint64_t)(all[2] & 0xFFFFu) << 32 | (uint64_t)(all[3] & 0xFFFFu) << 48;
        }
        if (!a.cols) {
#pragma unroll
            for (int s = 0; s < S; ++s) {
#pragma unroll
                for (int j = 0; j < 16; ++j) x[s][j] = (msel[s] >> j) & 1u ? x[s][j] * scale : 0.f;
                lds_store<16>(st + r * LRW + 64 * s + 16 * q, x[s]);      // (the lane's own columns)
            }
            wave_sync();
#pragma unroll
            for (int reg = 0; reg < 4; ++reg)
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    const int rr = 4 * reg + tg;
                    float v[4];
                    lds_load<4>(st + rr * LRW + 64 * s + 4 * tj, v);
#pragma unroll
                    for (int cb = 0; cb < 4; ++cb) v[cb] = stored<T>(v[cb]);
                    if (rr < rows) store_cols<4, T, true>(a.vals + (size_t)(r0 + rr) * DGW + 64 * s + 4 * tj, v);
                }
            continue;
        }
        wave_sync();          // every lane holds its values: the tile can be reused
        const int dump = 16 * LRW + lane;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            int ahead = slot[s] - dump;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int bit = (int)((msel[s] >> j) & 1u);
                st[dump + __mul24(bit, ahead)] = x[s][j] * scale;      // dropped columns go to the dump words
                ahead += bit;
            }
        }
        wave_sync();
        T* dst = a.vals + (size_t)r0 * a.k;
        for (int i = lane; i < total; i += 64) dst[i] = from_float<T>(st[i]);
        wave_sync();
        uint8_t* cst = reinterpret_cast<uint8_t*>(st);
#pragma unroll
        for (int s = 0; s < S; ++s) {
            int ahead = slot[s] - 4 * dump;                            // (byte 4 dump: the lane's dump word)
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int bit = (int)((msel[s] >> j) & 1u);
                cst[4 * dump + __mul24(bit, ahead)] = (uint8_t)(64 * s + 16 * q + j);
                ahead += bit;
            }
        }
        wave_sync();
        uint32_t* dc = reinterpret_cast<uint32_t*>(a.cols + (size_t)r0 * a.k);      // whole words, see emit_tile
        for (int i = lane; 4 * i < total; i += 64) dc[i] = reinterpret_cast<const uint32_t*>(cst)[i];
    }
}

// ---- head: yhat = X w + b, loss = mean (yhat - t)^2 ----------------------------------------------------
template <typename T>
struct HeadArgs {
    int n, d, dg;
    const T* act;           // element (row, grp, c) at grp*gs + row*ld + c
    T* grad;                // same layout
    int64_t ld, gs;
    const float* w_out;
    const float* b_out;
    const float* target;
    float* yhat;            // may be NULL
    float* partial;         // [gridDim.x][d + 2]: dw (d), db, sum of squared errors
};

constexpr int HEAD_MAXQ = 8;  // d <= 512

// NQ: 64-column pieces of a row.  Four of a wave's rows are in flight at a time (one after the other, each a trip to memory and a sum over
// the lanes: 9.6 -> 5.4 us on 2,000 nodes of 64 columns, 33.6 -> 30.0 on 100k of 128), added in the same order as one by one.
template <typename T, int NQ>
__global__ __launch_bounds__(256) void k_head(HeadArgs<T> a) {
    constexpr int NR = NQ > 4 ? 2 : 4;
    __shared__ float red[4][NQ * 64 + 2];
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    float wv[NQ], dwacc[NQ];
    size_t off[NQ];
    bool in[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int cc = q * 64 + lane;
        in[q] = cc < a.d;
        wv[q] = in[q] ? a.w_out[cc] : 0.f;
        dwacc[q] = 0.f;
        off[q] = in[q] ? (size_t)(cc / a.dg) * a.gs + (cc % a.dg) : 0;      // (a column that is there, for the lanes past the last)
    }
    const float bias = a.b_out[0];
    float db = 0.f, sse = 0.f;
    const int64_t nwaves = (gridDim.x * blockDim.x) >> 6;
    for (int64_t row0 = (blockIdx.x * blockDim.x + threadIdx.x) >> 6; row0 < a.n; row0 += NR * nwaves) {
        float xv[NR][NQ], target[NR], dot[NR];
#pragma unroll
        for (int u = 0; u < NR; ++u) {
            const size_t row = (size_t)(row0 + u * nwaves < a.n ? row0 + u * nwaves : row0);
#pragma unroll
            for (int q = 0; q < NQ; ++q) xv[u][q] = to_float(a.act[off[q] + row * a.ld]);
            target[u] = a.target[row];
        }
#pragma unroll
        for (int u = 0; u < NR; ++u) {
            dot[u] = 0.f;
#pragma unroll
            for (int q = 0; q < NQ; ++q) dot[u] += (in[q] ? xv[u][q] : 0.f) * wv[q];
            dot[u] = sub_sum<64>(dot[u]);
        }
#pragma unroll
        for (int u = 0; u < NR; ++u) {
            if (row0 + u * nwaves >= a.n) break;
            const size_t row = (size_t)(row0 + u * nwaves);
            const float y = dot[u] + bias;
            const float e = y - target[u];
            const float gy = 2.0f * e / (float)a.n;
            if (lane == 0 && a.yhat) a.yhat[row] = y;
            db += gy;
            sse += e * e;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                dwacc[q] += (in[q] ? xv[u][q] : 0.f) * gy;
                if (in[q]) a.grad[off[q] + row * a.ld] = from_float<T>(gy * wv[q]);
            }
        }
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) red[wave][q * 64 + lane] = dwacc[q];
    if (lane == 0) { red[wave][NQ * 64] = db; red[wave][NQ * 64 + 1] = sse; }
    __syncthreads();
    for (int i = threadIdx.x; i < a.d + 2; i += 256) {
        const int src = i < a.d ? i : NQ * 64 + (i - a.d);
        a.partial[(size_t)blockIdx.x * (a.d + 2) + i] = ((red[0][src] + red[1][src]) + red[2][src]) + red[3][src];
    }
}

// One wave per output element: lane l adds partials l, l + 64, .. in that order, then the 64 lane sums are
// added in a fixed tree.  (One thread per element walking all partials in turn took 240 us whatever the size.)
__global__ __launch_bounds__(256) void k_head_reduce(const float* __restrict__ partial, int nparts, int d, int n,
                                                     float* __restrict__ dw_out, float* __restrict__ db_out,
                                                     float* __restrict__ loss_out) {
    const int i = (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6), lane = lane_id();
    if (i >= d + 2) return;
    float acc = 0.f;
    for (int p = lane; p < nparts; p += 64) acc += partial[(size_t)p * (d + 2) + i];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (lane != 0) return;
    if (i < d) dw_out[i] = acc;
    else if (i == d) db_out[0] = acc;
    else loss_out[0] = acc / (float)n;
}

// ---- layout copy: (row, grp, c) between two stride sets ---------------------------------------------------
// blockIdx.y: the group.  T: the element, or sixteen bytes of them where both sides' rows allow it (dg, strides in units of T; indices
// in 32 bits then: 100k nodes of 128 float32 columns 31.3 -> 16.0 us).
template <typename T, typename Index>
__global__ void k_copy_planes(Index n, int dg, const T* __restrict__ src, int64_t s_ld, int64_t s_gs, T* __restrict__ dst, int64_t d_ld, int64_t d_gs) {
    src += blockIdx.y * s_gs;
    dst += blockIdx.y * d_gs;
    const Index total = n * (Index)dg, step = (Index)gridDim.x * blockDim.x;
    for (Index i = (Index)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += step) {
        const Index row = i / (Index)dg, c = i - row * (Index)dg;
        dst[(int64_t)row * d_ld + c] = src[(int64_t)row * s_ld + c];
    }
}

// ======================================== host orchestration ===============================================

template <typename T>
struct Planes {
    T* base;
    int64_t ld, gs;
    T* grp(int i) const { return base + (size_t)i * gs; }
};

template <typename T>
static Planes<T> caller_planes(void* p, const gsr_config_t* cfg) {
    const int dg = cfg->d / cfg->c;
    if (cfg->layout == GSR_LAYOUT_ROW_MAJOR) return Planes<T>{(T*)p, (int64_t)cfg->d, (int64_t)dg};
    return Planes<T>{(T*)p, (int64_t)dg, (int64_t)cfg->n * dg};
}

template <int DG, typename T>
struct Ctx {
    using M = typename MaskOf<DG>::type;
    const gsr_graph_t* g;
    const gsr_config_t* cfg;
    hipStream_t s;
    char* ws;
    LayerWs lw;
    int tiles;
    int S;          // sub-planes of a group: 1, or D/C / 64 for groups wider than a tile (then DG = 64)
    bool rows;      // records are held as rows (records_as_rows)
    bool band;      // the gradient goes through a product before the gather (band_gradient)
    M* saved;       // [L+1][C][S][n] column masks kept from the forward sweep, or NULL
    // rows kept because they selected at a near-tie (cfg->save_indices == 2), per segment (layer, slot), or NULL
    int* tie_counts;
    uint32_t* tie_rows;
    M* tie_masks;
    int tie_cap;
    TieSeg<DG> tie_seg(int layer, int slot) const {
        if (!tie_counts || layer < 0) return TieSeg<DG>{nullptr, nullptr, nullptr, 0, 0.f};
        const size_t seg = (size_t)layer * cfg->c + slot;
        return TieSeg<DG>{tie_counts + seg * TIE_SUB * TIE_COUNTER_STRIDE, tie_rows + seg * TIE_SUB * tie_cap,
                          tie_masks + seg * TIE_SUB * tie_cap, tie_cap, cfg->tie_tol};
    }
    // Record slot `slot` of layer `layer`: the values always live in the slot (they are rebuilt),
    // the mask in the slot, or in the kept store when indices are saved.  (Groups of S column blocks: one list of values and
    // columns for the whole row, a mask per block.)
    Record<DG, T> rec(int slot, int layer = 0, int sub = 0) const {
        Record<DG, T> r;
        if (slot < 0) { r.vals = nullptr; r.mask = nullptr; r.cols = nullptr; return r; }
        r.vals = (T*)(ws + lw.rec_vals[slot]);
        r.cols = rows ? nullptr : (uint8_t*)(ws + lw.rec_cols[slot]);
        r.mask = saved ? saved + (((size_t)layer * cfg->c + slot) * S + sub) * (size_t)cfg->n : (M*)(ws + lw.rec_mask[slot * S + sub]);
        return r;
    }
    T* y0() const { return (T*)(ws + lw.y0); }
    float* dh() const { return (float*)(ws + lw.dh); }
    float* hplane() const { return (float*)(ws + lw.h); }
    float* dw_partial() const { return (float*)(ws + lw.dw_partial); }
    float* hub_part() const { return (float*)(ws + lw.hub_partial); }
    float* hub_part2() const { return (float*)(ws + lw.hub_partial2); }
    bool hub_by_value() const { return !rows && g->hub_values != 0; }
};

// Workgroups of 256 threads one CU keeps resident for a kernel, and the persistent grid that
// fills the chip with them: a multiple of 8 (one share per XCD), never above g->grid, which
// sizes the per-workgroup partial buffers, or g->gather_grid where the kernel has none.
static int resident_blocks(const void* kernel, int threads = 256) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kernel, threads, 0) != hipSuccess || nb < 1) nb = 1;
    return nb;
}
static unsigned persistent_grid(const gsr_graph_t* g, int per_cu, bool gather = false) {
    int grid = g->num_cus * per_cu / 8 * 8;
    const int most = gather ? g->gather_grid : g->grid;
    if (grid > most) grid = most;
    if (grid < 8) grid = 8;
    return (unsigned)grid;
}

template <int DG, typename T>
static void launch_sum(const Ctx<DG, T>& x, const T* src, int64_t ld, int64_t gs, int nsrc, T* y0,
                       const Record<DG, T>& out, bool out_given = false,
                       TieSeg<DG> tie = TieSeg<DG>{nullptr, nullptr, nullptr, 0, 0.f},
                       TieSeg<DG> fix = TieSeg<DG>{nullptr, nullptr, nullptr, 0, 0.f}, int planes = 1, size_t y_rec = 0, size_t y_mask = 0) {
    SumArgs<DG, T> a;
    a.tie = tie;
    a.fix = fix;
    a.y_rec = y_rec; a.y_mask = y_mask;
    a.n = (int)x.cfg->n; a.src = src; a.ld = ld; a.src_gs = gs; a.nsrc = nsrc; a.y0 = y0;
    a.k = x.cfg->k; a.norm = x.cfg->norm; a.eps = x.cfg->eps;
    a.out = out; a.out_given = out_given;
    ProfScope prof(KC_SUM, x.s);
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3((unsigned)x.g->grid * 2, (unsigned)planes), dim3(256), 0, x.s, a); };
    if (fix.count) x.rows ? launch(k_sum<DG, T, REC_ROWS, true>) : launch(k_sum<DG, T, REC_COLUMNS, true>);
    else x.rows ? launch(k_sum<DG, T, REC_ROWS, false>) : launch(k_sum<DG, T, REC_COLUMNS, false>);
}

// The records of Y_1 .. Y_{C-1} into slots 1 .. C - 1, in one launch (one each: two launches of 6.9 us on 30k nodes and three groups,
// so one of 9.6; 1M nodes, eight 16-bit groups, seven launches of 44 us, so one of 304).  A workspace holds the slots evenly spaced.
template <int DG, typename T>
static void launch_records(const Ctx<DG, T>& x, const Planes<T>& y, int layer, bool given) {
    const int C = x.cfg->c;
    const Record<DG, T> first = x.rec(1, layer), second = x.rec(C > 2 ? 2 : 1, layer);
    launch_sum<DG, T>(x, y.grp(0), y.ld, y.gs, 1, nullptr, first, given, x.tie_seg(-1, 0), x.tie_seg(-1, 0), C - 1,
                      (size_t)((char*)second.vals - (char*)first.vals), (size_t)((char*)second.mask - (char*)first.mask));
}

template <int DG, typename T>
static void launch_hub_records(const Ctx<DG, T>& x, const Record<DG, T>& in) {
    const HubPlan& h = x.g->a.hub;
    if (h.n_chunks == 0) return;
    HubChunks hc{h.ce0, h.ce1, h.n_chunks, x.g->long_rows};
    ProfScope prof(KC_HUB, x.s);
    if (!in.cols) {
        hipLaunchKernelGGL((k_hub_dense<DG, T>), dim3(hub_grid(h.n_chunks)), dim3(256), 0, x.s, make_view(x.g, false), hc,
                           (const T*)in.vals, (int64_t)DG, x.hub_part(), (float*)nullptr);
        return;
    }
    if constexpr (sizeof(T) == 4) {
        if (x.hub_by_value()) {
            hub_values_variant(x.cfg->k, [&](auto lg, auto kq) {
                hipLaunchKernelGGL((k_hub_values<DG, decltype(lg)::value, decltype(kq)::value>),
                                   dim3(hub_grid(h.n_chunks)), dim3(256), 0, x.s, make_view(x.g, false), hc,
                                   (const float*)in.vals, (const uint8_t*)in.cols, x.cfg->k, (int)x.cfg->n, x.hub_part(), (float*)nullptr);
            });
            return;
        }
    }
    hipLaunchKernelGGL((k_hub_records<DG, T>), dim3(hub_grid(h.n_chunks)), dim3(256), 0, x.s,
                       make_view(x.g, false), hc, in, x.cfg->k, x.hub_part());
}

template <int DG, typename T>
static void launch_hub_dense(const Ctx<DG, T>& x, const T* plane, int64_t ld) {
    const HubPlan& h = x.g->at.hub;
    if (h.n_chunks == 0) return;
    HubChunks hc{h.ce0, h.ce1, h.n_chunks, x.g->long_rows};
    ProfScope prof(KC_HUB, x.s);
    hipLaunchKernelGGL((k_hub_dense<DG, T>), dim3(hub_grid(h.n_chunks)), dim3(256), 0, x.s,
                       make_view(x.g, true), hc, plane, ld, x.hub_part(), (float*)nullptr);
}

// Both first passes of a block's backward (records over A into hub_part, dY rows over A^T into hub_part2).
// Returns false if there is nothing to do.
template <int DG, typename T>
static bool launch_hub_both(const Ctx<DG, T>& x, const Record<DG, T>& in, const T* dy, int64_t ldg) {
    const HubPlan &ha = x.g->a.hub, &ht = x.g->at.hub;
    if (ha.n_chunks == 0 && ht.n_chunks == 0) return false;
    HubChunks ca{ha.ce0, ha.ce1, ha.n_chunks, x.g->long_rows}, ct{ht.ce0, ht.ce1, ht.n_chunks, x.g->long_rows};
    ProfScope prof(KC_HUB, x.s);
    const unsigned gx = hub_grid(std::max(ha.n_chunks, ht.n_chunks));
    if constexpr (sizeof(T) == 4) {
        if (x.hub_by_value()) {
            // (two launches: as the two rows of one grid, as the dealing variant runs them, they took 50 us longer on the
            // Table-1-shaped graph than one after the other)
            if (ha.n_chunks > 0)
                hub_values_variant(x.cfg->k, [&](auto lg, auto kq) {
                    hipLaunchKernelGGL((k_hub_values<DG, decltype(lg)::value, decltype(kq)::value>),
                                       dim3(hub_grid(ha.n_chunks)), dim3(256), 0, x.s, make_view(x.g, false),
                                       ca, (const float*)in.vals, (const uint8_t*)in.cols, x.cfg->k, (int)x.cfg->n, x.hub_part(),
                                       (float*)nullptr);
                });
            if (ht.n_chunks > 0)
                hipLaunchKernelGGL((k_hub_dense<DG, T>), dim3(hub_grid(ht.n_chunks)), dim3(256), 0, x.s,
                                   make_view(x.g, true), ct, dy, ldg, x.hub_part2(), (float*)nullptr);
            return true;
        }
    }
    hipLaunchKernelGGL((k_hub_both<DG, T>), dim3(gx, 2), dim3(256), 0, x.s, make_view(x.g, false), ca, in, x.cfg->k, x.hub_part(),
                       make_view(x.g, true), ct, dy, ldg, x.hub_part2());
    return true;
}

// How the backward of a block takes dW_i.  float32, and 16-bit storage at D/C = 64: the inverse kernel (sixteen waves per
// compute unit) leaves H in memory and k_dw takes H^T dY_i in a pass of its own: 476 -> 320 + 112 us per block on the 1M-node
// workload when it was cut in two (246 + 88 us now) for 512 more bytes per row.  16-bit storage at D/C = 32: the fused kernel
// (inverse + dW accumulators): 1M nodes, 152 us fused against 143 + 32 us.
// Graphs with fewer than two tiles per resident wave (a launch there is one or two short tiles per wave, and two more launches
// per block cost more than the occupancy gains), or with all rows in the first pass, keep the fused kernel in float32 as well
// (figures where the rule is made, with the graph); it uses the same sums, so whichever way a block's backward runs
// it rebuilds the bits the plain inverse rebuilds.
template <int DG, typename T>
static bool split_dw(const gsr_graph_t* g) { return (sizeof(T) == 4 || DG == 64) && g->split_backward; }

// mode 0: forward (+), 1: inverse (-), 2: inverse (-) with dW
template <int DG, typename T>
static unsigned launch_block(const Ctx<DG, T>& x, int mode, const Record<DG, T>& in, const float* w, T* plane, int64_t ld,
                             const Record<DG, T>& out, bool out_given, const T* dy, int64_t ldg, bool first_pass_done = false,
                             TieSeg<DG> tie = TieSeg<DG>{nullptr, nullptr, nullptr, 0, 0.f}, float* h_out = nullptr,
                             TieSeg<DG> fix = TieSeg<DG>{nullptr, nullptr, nullptr, 0, 0.f}) {
    if (!first_pass_done) launch_hub_records<DG, T>(x, in);
    BlockArgs<DG, T> a;
    a.tie = tie;
    a.fix = fix;
    a.h_out = h_out;
    a.g = make_view(x.g, false);
    a.n = (int)x.cfg->n; a.tiles = x.tiles;
    a.in = in; a.k = x.cfg->k;
    a.hub_part = x.hub_part(); a.w = w; a.plane = plane; a.ld = ld;
    a.out = out; a.out_given = out_given;
    a.norm = x.cfg->norm; a.eps = x.cfg->eps; a.dy = dy; a.ldg = ldg; a.dw_partial = x.dw_partial();
    if (mode != 2) tile_counters(x.g, &a.draws, &a.draws_done);
    else a.draws = a.draws_done = nullptr;
    const bool b3 = mode != 0 || !x.g->long_rows;       // (see k_block)
    const dim3 block(64 * block_waves(mode == 2, b3));
    ProfScope prof(mode == 0 ? KC_BLOCK_FWD : mode == 1 ? KC_BLOCK_INV : KC_BLOCK_BWD, x.s);
    unsigned grid = 0;
    auto go = [&](auto plain, auto deal, int per_cu) {
        grid = persistent_grid(x.g, per_cu);
        if (heavy_first(a.g.n_heavy, x.tiles, grid * (block.x / 64) / 4)) hipLaunchKernelGGL(deal, dim3(grid), block, 0, x.s, a);
        else hipLaunchKernelGGL(plain, dim3(grid), block, 0, x.s, a);
    };
    auto launch = [&](auto form) {
        constexpr RecordForm F = decltype(form)::value;
        if (mode == 0 && b3) {
            static const int per_cu = resident_blocks((const void*)k_block<DG, T, +1, false, false, true, F>, 512);
            go(k_block<DG, T, +1, false, false, true, F>, k_block<DG, T, +1, false, true, true, F>, per_cu);
        } else if (mode == 0) {
            static const int per_cu = resident_blocks((const void*)k_block<DG, T, +1, false, false, false, F>, 256);
            go(k_block<DG, T, +1, false, false, false, F>, k_block<DG, T, +1, false, true, false, F>, per_cu);
        } else if (mode == 1) {
            static const int per_cu = resident_blocks((const void*)k_block<DG, T, -1, false, false, true, F>, 512);
            go(k_block<DG, T, -1, false, false, true, F>, k_block<DG, T, -1, false, true, true, F>, per_cu);
        } else {
            static const int per_cu = resident_blocks((const void*)k_block<DG, T, -1, true, false, true, F>, 256);
            go(k_block<DG, T, -1, true, false, true, F>, k_block<DG, T, -1, true, true, true, F>, per_cu);
        }
    };
    if (x.rows) launch(std::integral_constant<RecordForm, REC_ROWS>{});
    else launch(std::integral_constant<RecordForm, REC_COLUMNS>{});
    return grid;
}

template <int DG, typename T>
static void launch_dw_reduce(const Ctx<DG, T>& x, int parts, float* out) {
    ProfScope prof(KC_DW_REDUCE, x.s);
    hipLaunchKernelGGL(k_dw_reduce, dim3((DG * DG + DW_REDUCE_ENTRIES - 1) / DW_REDUCE_ENTRIES), dim3(256), 0, x.s, (const float*)x.dw_partial(),
                       parts, DG * DG, out, DG, DG);
}

template <int DG, typename T>
static void launch_grad(const Ctx<DG, T>& x, const T* dy, int64_t ldg, const float* w,
                        const typename MaskOf<DG>::type* own_mask, const T* z,
                        int64_t ldz, T* dst, int64_t ldd, int64_t dst_gs, int ndst, int dw_parts, float* dw_out,
                        bool first_pass_done = false, float* beside_out = nullptr) {
    if (!first_pass_done) launch_hub_dense<DG, T>(x, dy, ldg);
    GradArgs<DG, T> a;
    a.gt = make_view(x.g, true);
    a.n = (int)x.cfg->n; a.tiles = x.tiles; a.dy = dy; a.ldg = ldg; a.hub_part = first_pass_done ? x.hub_part2() : x.hub_part();
    a.w = w;
    a.own_mask = own_mask; a.z = z; a.ldz = ldz; a.norm = x.cfg->norm; a.eps = x.cfg->eps;
    a.dst = dst; a.ldd = ldd; a.dst_gs = dst_gs; a.ndst = ndst;
    a.dw_partial = x.dw_partial(); a.dw_parts = dw_parts; a.dw_out = dw_out; a.beside_out = beside_out;
    tile_counters(x.g, &a.draws, &a.draws_done);
    ProfScope prof(KC_GRAD, x.s);
    auto go = [&](auto plain, auto deal, int per_cu, unsigned threads) {
        const unsigned grid = persistent_grid(x.g, per_cu);
        if (heavy_first(a.gt.n_heavy, x.tiles, grid * (threads / 64) / 4)) {
            if (beside_out) launch_dw_reduce<DG, T>(x, dw_parts, beside_out);
            hipLaunchKernelGGL(deal, dim3(grid), dim3(threads), 0, x.s, a);
        } else {
            hipLaunchKernelGGL(plain, dim3(grid, beside_out ? 2 : 1), dim3(threads), 0, x.s, a);
        }
    };
    if (!x.g->long_rows) {
        static const int per_cu = resident_blocks((const void*)k_grad<DG, T, false, true>, 512);
        go(k_grad<DG, T, false, true>, k_grad<DG, T, true, true>, per_cu, 512u);
    } else {
        static const int per_cu = resident_blocks((const void*)k_grad<DG, T, false, false>, 256);
        go(k_grad<DG, T, false, false>, k_grad<DG, T, true, false>, per_cu, 256u);
    }
}

// After a record was taken again from rebuilt rows during the inverse sweep: the rows listed for that application of
// GS in the forward sweep get their kept column sets back (values from the same rebuilt rows).
template <int DG, typename T>
static void launch_tie_fixup(const Ctx<DG, T>& x, const TieSeg<DG>& tie, const T* plane, int64_t ld, const Record<DG, T>& out) {
    if (!tie.count) return;
    ProfScope prof(KC_TIE, x.s);
    const unsigned blocks = (unsigned)std::min((TIE_SUB * tie.cap + 63) / 64 / 4 * 4 + 4, 1024);     // 4 waves each: a multiple of TIE_SUB waves
    hipLaunchKernelGGL((k_tie_fixup<DG, T>), dim3(blocks), dim3(256), 0, x.s, tie, plane, ld, x.cfg->k, x.cfg->norm, x.cfg->eps, out);
}

// dW_i's workgroup partials from H (in x.hplane()) and dY_i; returns their number
template <int DG, typename T>
static unsigned launch_dw(const Ctx<DG, T>& x, const T* dy, int64_t ldg, const TieSeg<DG>& tie = TieSeg<DG>{nullptr, nullptr, nullptr, 0, 0.f},
                          const T* fix_plane = nullptr, int64_t fix_ld = 0, const Record<DG, T>* fix_out = nullptr) {
    DwArgs<DG, T> a;
    a.n = (int)x.cfg->n; a.tiles = x.tiles; a.h = x.hplane(); a.dy = dy; a.ldg = ldg;
    a.dw_partial = x.dw_partial();
    a.S = x.S;
    a.y_set = (size_t)x.g->grid * DG * DG;
    a.tie = fix_out ? tie : TieSeg<DG>{nullptr, nullptr, nullptr, 0, 0.f};
    a.fix_plane = fix_plane; a.fix_ld = fix_ld; a.k = x.cfg->k; a.norm = x.cfg->norm; a.eps = x.cfg->eps;
    a.fix_out = fix_out ? *fix_out : x.rec(-1);
    ProfScope prof(KC_DW, x.s);
    if constexpr (DG == 64) {
        if (x.S > 1) {       // the resident workgroups shared out between the sets (16-bit groups of 256: two rounds of them)
            static const int per_cu = resident_blocks((const void*)k_dw<DG, T, true>, 256);
            const unsigned rounds = sizeof(T) == 2 && x.S == 4 ? 2 : 1;
            const unsigned grid = std::max(8u, rounds * persistent_grid(x.g, per_cu) / (unsigned)(x.S * x.S) / 8 * 8);
            hipLaunchKernelGGL((k_dw<DG, T, true>), dim3(grid, (unsigned)(x.S * x.S)), dim3(256), 0, x.s, a);
            return grid;
        }
    }
    static const int per_cu = resident_blocks((const void*)k_dw<DG, T, false>, 256);
    const unsigned grid = persistent_grid(x.g, per_cu);
    hipLaunchKernelGGL((k_dw<DG, T, false>), dim3(grid), dim3(256), 0, x.s, a);
    return grid;
}

// ---- groups wider than one tile (see k_gather_wide): D/C = 64 S as S sub-planes of 64 columns -----------------------
// Sub-plane s of group i of a plane set p starts 64 s elements into the group's rows (both caller layouts and the
// step's arena keep a group's columns adjacent in a row).  W_i is D/C x D/C row-major.
template <typename F>
static void wide_blocks(int S, F&& f) {
    if (S == 2) f(std::integral_constant<int, 2>{});
    else if (S == 3) f(std::integral_constant<int, 3>{});
    else f(std::integral_constant<int, 4>{});
}

// GS over the whole rows of a wide group (sum of nsrc groups first when nsrc > 1), record of slot `slot`
template <typename T>
static void launch_gs_wide(const Ctx<64, T>& x, const T* src, int64_t ld, int64_t gs, int nsrc, T* y0, int slot, int layer,
                           bool given = false) {
    ProfScope prof(KC_SUM, x.s);
    wide_blocks(x.S, [&](auto sc) {
        constexpr int S = decltype(sc)::value;
        WideGsArgs<S, T> a;
        a.n = (int)x.cfg->n; a.src = src; a.ld = ld; a.src_gs = gs; a.nsrc = nsrc; a.y0 = y0;
        a.k = x.cfg->k; a.norm = x.cfg->norm; a.eps = x.cfg->eps;
        a.vals = x.rec(slot, layer).vals;
        a.cols = x.rec(slot, layer).cols;
        for (int s = 0; s < S; ++s) a.mask[s] = x.rec(slot, layer, s).mask;
        a.out_given = given;
        hipLaunchKernelGGL((k_gs_wide<S, T>), dim3((unsigned)x.g->grid * 2), dim3(256), 0, x.s, a);
    });
}

// A X (or A^T X) of dense rows X of 64 S columns into planes [S][n][64]
template <typename T>
static void launch_dense_planes(const Ctx<64, T>& x, bool transpose, const T* src, int64_t ld, float* planes, KernelClass kc) {
    const HubPlan& hp = transpose ? x.g->at.hub : x.g->a.hub;
    const size_t n = (size_t)x.cfg->n;
    if (hp.n_chunks > 0) {
        HubChunks hc{hp.ce0, hp.ce1, hp.n_chunks, x.g->long_rows, hp.single};
        ProfScope prof(KC_HUB, x.s);
        for (int s = 0; s < x.S; ++s)
            hipLaunchKernelGGL((k_hub_dense<64, T>), dim3(hub_grid(hp.n_chunks)), dim3(256), 0, x.s, make_view(x.g, transpose), hc, src + 64 * s, ld,
                               x.hub_part() + (size_t)s * hp.n_chunks * 64, planes + s * n * 64);
    }
    DensePlanesArgs<T> a;
    a.g = make_view(x.g, transpose);
    a.n = (int)n; a.tiles = x.tiles; a.x = src; a.ld = ld; a.hub_part = x.hub_part(); a.n_chunks = hp.n_chunks; a.q = planes;
    a.y_draws = kTileCounterSet;
    tile_counters(x.g, &a.draws, &a.draws_done);
    ProfScope prof(kc, x.s);
    static const int plain_per_cu = resident_blocks((const void*)k_dense_planes<T, false>), deal_per_cu = resident_blocks((const void*)k_dense_planes<T, true>);
    auto grid = [&](int per_cu) { return std::max(8u, persistent_grid(x.g, per_cu, true) / (unsigned)x.S / 8 * 8); };       // the resident workgroups shared out
    const unsigned dealt = grid(deal_per_cu), plain = grid(plain_per_cu);
    if (heavy_first(a.g.n_heavy, x.tiles, dealt)) hipLaunchKernelGGL((k_dense_planes<T, true>), dim3(dealt, (unsigned)x.S), dim3(256), 0, x.s, a);
    else hipLaunchKernelGGL((k_dense_planes<T, false>), dim3(plain, (unsigned)x.S), dim3(256), 0, x.s, a);
}

// H of block `slot` + 1 into x.hplane(): the first pass over split rows, then the tiles
template <typename T>
static void launch_gather_wide(const Ctx<64, T>& x, int slot, int layer) {
    const HubPlan& hp = x.g->a.hub;
    const Record<64, T> in = x.rec(slot, layer);
    const int n = (int)x.cfg->n, k = x.cfg->k;
    if (!in.cols) {
        launch_dense_planes<T>(x, false, in.vals, 64 * x.S, x.hplane(), KC_BLOCK_FWD);
        return;
    }
    wide_blocks(x.S, [&](auto sc) {
        constexpr int S = decltype(sc)::value;
        if (hp.n_chunks > 0) {
            HubChunks hc{hp.ce0, hp.ce1, hp.n_chunks, x.g->long_rows, hp.single};
            ProfScope prof(KC_HUB, x.s);
            bool by_value = false;
            if constexpr (sizeof(T) == 4 && S < 4) {
                by_value = x.hub_by_value() && k <= 64;
                if (by_value)
                    hub_values_variant_wide(k, [&](auto lg, auto kq) {
                        hipLaunchKernelGGL((k_hub_values<64 * S, decltype(lg)::value, decltype(kq)::value>), dim3(hub_grid(hp.n_chunks)),
                                           dim3(256), 0, x.s, make_view(x.g, false), hc, (const float*)in.vals, (const uint8_t*)in.cols, k, n,
                                           x.hub_part(), x.hplane());
                    });
            }
            if (!by_value)
                hipLaunchKernelGGL((k_hub_records_wide<S, T>), dim3(hub_grid(hp.n_chunks)), dim3(256), 0, x.s, make_view(x.g, false), hc,
                                   (const T*)in.vals, (const uint8_t*)in.cols, k, n, x.hub_part(), x.hplane());
        }
        ProfScope prof(KC_BLOCK_FWD, x.s);
        WideGatherArgs<S, T> a;
        a.g = make_view(x.g, false);
        a.n = n; a.tiles = (n + 7) / 8;
        a.vals = in.vals; a.cols = in.cols; a.k = k;
        a.hub_part = x.hub_part(); a.n_chunks = hp.n_chunks;
        a.h = x.hplane();
        tile_counters(x.g, &a.draws, &a.draws_done);
        static const int per_cu = resident_blocks((const void*)k_gather_wide<S, T>);
        hipLaunchKernelGGL((k_gather_wide<S, T>), dim3(persistent_grid(x.g, per_cu, true)), dim3(256), 0, x.s, a);
    });
}

// Two column blocks: workgroups of a sweep with all of W_i in LDS (k_wide_product2, k_wide_grad2), one per compute unit, or 0 where a workgroup
// per eight tiles (k_wide_product, k_wide_grad) is better.  The sweep leaves one workgroup resident per unit where the other form has two or three,
// so one round of eight tiles more than the other form needs costs a whole round: groups of 128, k = 32, forward / backward layer, sweep against
// other form, us: 16-bit 24k nodes (one round at most) 127.3 / 288.1, 125.3 / 288.6; 50k 188.6 / 401.2, 181.0 / 382.9; 64k (two rounds) 197.3 / 433.2,
// 190.1 / 416.3; 72k 217.8 / 481.7 against 228 / 499; float32 24k 129.4 / 300.3, 128.9 / 303.9; 50k 189.0 / 429.1, 185.9 / 412.4; 64k 202.7 / 478.3,
// 205.1 / 472.0.
template <typename T>
static unsigned sweep_workgroups(const Ctx<64, T>& x) {
    const int cus = std::min(x.g->num_cus, x.g->grid), groups = (x.tiles + 7) / 8;
    return groups > 2 * cus || (groups <= cus && sizeof(T) == 4) ? (unsigned)std::min(groups, cus) : 0u;
}

// plane (+/-)= H W_i with H in x.hplane()
template <typename T>
static void launch_wide_product(const Ctx<64, T>& x, int sign, const float* wi, T* plane, int64_t ld) {
    ProfScope prof(sign > 0 ? KC_BLOCK_FWD : KC_BLOCK_INV, x.s);
    wide_blocks(x.S, [&](auto sc) {
        constexpr int S = decltype(sc)::value;
        WideProductArgs<S, T> a;
        a.n = (int)x.cfg->n; a.tiles = x.tiles; a.h = x.hplane(); a.w = wi; a.plane = plane; a.ld = ld;
        const dim3 grid((unsigned)((x.tiles + 7) / 8));
        if constexpr (S == 2) {
            if (const unsigned cus = sweep_workgroups(x)) {
                if (sign > 0) hipLaunchKernelGGL((k_wide_product2<T, +1>), dim3(cus), dim3(512), 0, x.s, a);
                else hipLaunchKernelGGL((k_wide_product2<T, -1>), dim3(cus), dim3(512), 0, x.s, a);
                return;
            }
        }
        if (sign > 0) hipLaunchKernelGGL((k_wide_product<S, T, +1>), grid, dim3(512), 0, x.s, a);
        else hipLaunchKernelGGL((k_wide_product<S, T, -1>), grid, dim3(512), 0, x.s, a);
    });
}

// dst += back through GS of (Q W_i^T), Q in x.dh()
template <typename T>
static void launch_wide_grad(const Ctx<64, T>& x, const float* wi, int slot, int layer, const T* z, int64_t ldz, int64_t z_sub, T* dst,
                             int64_t ldd, int64_t dst_gs, int ndst) {
    ProfScope prof(KC_GRAD, x.s);
    wide_blocks(x.S, [&](auto sc) {
        constexpr int S = decltype(sc)::value;
        WideGradArgs<S, T> a;
        a.n = (int)x.cfg->n; a.tiles = x.tiles; a.q = x.dh(); a.w = wi;
        for (int s = 0; s < S; ++s) a.mask[s] = x.rec(slot, layer, s).mask;
        a.z = z; a.ldz = ldz; a.z_sub = z_sub; a.norm = x.cfg->norm; a.eps = x.cfg->eps;
        a.dst = dst; a.ldd = ldd; a.dst_gs = dst_gs; a.ndst = ndst;
        if constexpr (S == 2) {
            if (const unsigned cus = sweep_workgroups(x)) {
                hipLaunchKernelGGL((k_wide_grad2<T>), dim3(cus), dim3(512), 0, x.s, a);
                return;
            }
        }
        hipLaunchKernelGGL((k_wide_grad<S, T>), dim3((unsigned)((x.tiles + 7) / 8)), dim3(512), 0, x.s, a);
    });
}

// The gradient of block `slot` + 1 on a graph of long rows in a band (see k_pre_product): dst planes += dZ.  P in x.dh(), the sums at the
// recorded positions in x.hplane().
template <int DG, int S, typename T>
static void launch_band_grad(const Ctx<DG, T>& x, const T* dy, int64_t ldg, const float* wi, int slot, int layer, const T* z, int64_t ldz,
                             int64_t z_sub, T* dst, int64_t ldd, int64_t dst_gs, int ndst) {
    constexpr int DGW = DG * S;
    const int n = (int)x.cfg->n, k = x.cfg->k;
    ProfScope prof(KC_GRAD, x.s);
    PreProductArgs<DG, S, T> pa{n, dy, ldg, wi, x.dh()};
    hipLaunchKernelGGL((k_pre_product<DG, S, T>), dim3((unsigned)((x.tiles + 7) / 8)), dim3(512), 0, x.s, pa);
    BandGatherArgs ga{make_view(x.g, true), n, x.g->band_rows, x.dh(), x.rec(slot, layer).cols, k, x.hplane()};
    const int blocks = (n + ga.rows - 1) / ga.rows;
    const dim3 grid((unsigned)((blocks + 7) / 8 * 8));
    auto gather = [&](auto kq) { hipLaunchKernelGGL((k_band_gather<DGW, decltype(kq)::value>), grid, dim3(1024), 0, x.s, ga); };
    if (k <= 16) gather(std::integral_constant<int, 1>{});
    else if constexpr (DGW > 32) {
        if (k <= 32) gather(std::integral_constant<int, 2>{});
        else if constexpr (DGW > 64) gather(std::integral_constant<int, 4>{});
    }
    BandBackArgs<DG, S, T> ba;
    ba.n = n; ba.tiles = x.tiles; ba.g = x.hplane(); ba.k = k;
    for (int s = 0; s < S; ++s) ba.mask[s] = x.rec(slot, layer, s).mask;
    ba.z = z; ba.ldz = ldz; ba.z_sub = z_sub; ba.norm = x.cfg->norm; ba.eps = x.cfg->eps;
    ba.dst = dst; ba.ldd = ldd; ba.dst_gs = dst_gs; ba.ndst = ndst;
    hipLaunchKernelGGL((k_band_back<DG, S, T>), dim3((unsigned)((x.tiles + 3) / 4)), dim3(256), 0, x.s, ba);
}

template <typename T>
static void wide_forward(const Ctx<64, T>& x, const float* w, const Planes<T>& p, bool slot0_ready, int layer) {
    const int C = x.cfg->c, dgw = 64 * x.S;
    if (!slot0_ready) launch_gs_wide<T>(x, p.grp(1), p.ld, p.gs, C - 1, nullptr, 0, layer);
    for (int i = 1; i <= C; ++i) {
        launch_gather_wide<T>(x, i - 1, layer);
        launch_wide_product<T>(x, +1, w + (size_t)(i - 1) * dgw * dgw, p.grp(i - 1), p.ld);
        if (i < C) launch_gs_wide<T>(x, p.grp(i - 1), p.ld, p.gs, 1, nullptr, i, layer);
        else if (C == 2) launch_gs_wide<T>(x, p.grp(i - 1), p.ld, p.gs, 1, nullptr, 0, layer + 1);
    }
}

template <typename T>
static void wide_inverse(const Ctx<64, T>& x, const float* w, const Planes<T>& p) {
    const int C = x.cfg->c, dgw = 64 * x.S;
    for (int i = 1; i < C; ++i) launch_gs_wide<T>(x, p.grp(i - 1), p.ld, p.gs, 1, nullptr, i, 0);
    for (int i = C; i >= 1; --i) {
        if (i == 1 && C > 2) launch_gs_wide<T>(x, p.grp(1), p.ld, p.gs, C - 1, nullptr, 0, 0);
        launch_gather_wide<T>(x, i - 1, 0);
        launch_wide_product<T>(x, -1, w + (size_t)(i - 1) * dgw * dgw, p.grp(i - 1), p.ld);
        if (i == 2 && C == 2) launch_gs_wide<T>(x, p.grp(1), p.ld, p.gs, 1, nullptr, 0, 0);
    }
}

// as layer_backward_impl
template <typename T>
static void wide_backward(const Ctx<64, T>& x, const float* w, const Planes<T>& y, const Planes<T>& dy, float* dw_out, bool slots_ready,
                          int layer, bool in_step) {
    const int C = x.cfg->c, S = x.S, dgw = 64 * S;
    const int64_t n = x.cfg->n;
    const bool given = x.saved != nullptr;
    if (!slots_ready)
        for (int i = 1; i < C; ++i) launch_gs_wide<T>(x, y.grp(i - 1), y.ld, y.gs, 1, nullptr, i, layer, given);
    for (int i = C; i >= 1; --i) {
        const float* wi = w + (size_t)(i - 1) * dgw * dgw;
        const T* z;          // rows of Y_{i-1}: row stride ldz, sub-plane s at + s * z_sub
        int64_t ldz, z_sub;
        if (i >= 2) { z = y.grp(i - 2); ldz = y.ld; z_sub = 64; }
        else if (C == 2) { z = y.grp(1); ldz = y.ld; z_sub = 64; }      // Y_0 = X_2, rebuilt just before
        else {
            launch_gs_wide<T>(x, y.grp(1), y.ld, y.gs, C - 1, x.y0(), 0, layer, given);
            z = x.y0(); ldz = 64; z_sub = n * 64;
        }
        launch_gather_wide<T>(x, i - 1, layer);
        launch_wide_product<T>(x, -1, wi, y.grp(i - 1), y.ld);
        // dW_i = H^T dY_i: its S x S blocks from partial sets of their own, each in one launch
        const unsigned nparts = launch_dw<64, T>(x, dy.grp(i - 1), dy.ld);
        {
            ProfScope prof(KC_DW_REDUCE, x.s);
            hipLaunchKernelGGL(k_dw_reduce, dim3(64 * 64 / DW_REDUCE_ENTRIES, (unsigned)(S * S)), dim3(256), 0, x.s, (const float*)x.dw_partial(),
                               (int)nparts, 64 * 64, dw_out + (size_t)(i - 1) * dgw * dgw, 64, dgw, (size_t)x.g->grid * 64 * 64, S);
        }
        // the record of the rebuilt X_i, where the next block or the layer below needs it
        if (i < C) {
            if (!(in_step && layer == 0)) launch_gs_wide<T>(x, y.grp(i - 1), y.ld, y.gs, 1, nullptr, i, given ? layer - 1 : 0, given);
        } else if (C == 2) {
            launch_gs_wide<T>(x, y.grp(i - 1), y.ld, y.gs, 1, nullptr, 0, layer, given);      // X_2 = Y_0 of this layer
        }
        if (x.band) {
            wide_blocks(S, [&](auto sc) {
                launch_band_grad<64, decltype(sc)::value, T>(x, dy.grp(i - 1), dy.ld, wi, i - 1, layer, z, ldz, z_sub,
                                                             dy.grp(i >= 2 ? i - 2 : 1), dy.ld, dy.gs, i >= 2 ? 1 : C - 1);
            });
            continue;
        }
        launch_dense_planes<T>(x, true, dy.grp(i - 1), dy.ld, x.dh(), KC_GRAD);       // Q = A^T dY_i
        if (i >= 2) launch_wide_grad<T>(x, wi, i - 1, layer, z, ldz, z_sub, dy.grp(i - 2), dy.ld, dy.gs, 1);
        else launch_wide_grad<T>(x, wi, 0, layer, z, ldz, z_sub, dy.grp(1), dy.ld, dy.gs, C - 1);
    }
}

// eq. (6).  slot0_ready: the record of Y_0 is already in slot 0 (C = 2: it is the record of the
// previous layer's Y_2, emitted when that plane was written).  `layer`: index of the layer inside
// a step (selects the kept masks when indices are saved; 0 otherwise).
template <int DG, typename T>
static void layer_forward_impl(const Ctx<DG, T>& x, const float* w, const Planes<T>& p, bool slot0_ready, int layer = 0) {
    if constexpr (DG == 64) {
        if (x.S > 1) { wide_forward<T>(x, w, p, slot0_ready, layer); return; }
    }
    const int C = x.cfg->c;
    if (!slot0_ready) launch_sum<DG, T>(x, p.grp(1), p.ld, p.gs, C - 1, nullptr, x.rec(0, layer), false, x.tie_seg(layer, 0));
    for (int i = 1; i <= C; ++i) {
        const Record<DG, T> out = i < C ? x.rec(i, layer) : (C == 2 ? x.rec(0, layer + 1) : x.rec(-1));
        const TieSeg<DG> tie = i < C ? x.tie_seg(layer, i) : (C == 2 ? x.tie_seg(layer + 1, 0) : x.tie_seg(-1, 0));
        launch_block<DG, T>(x, 0, x.rec(i - 1, layer), w + (size_t)(i - 1) * DG * DG, p.grp(i - 1), p.ld, out, false, nullptr, 0,
                            false, out.mask ? tie : TieSeg<DG>{nullptr, nullptr, nullptr, 0, 0.f});
    }
}

// eq. (7)
template <int DG, typename T>
static void layer_inverse_impl(const Ctx<DG, T>& x, const float* w, const Planes<T>& p) {
    if constexpr (DG == 64) {
        if (x.S > 1) { wide_inverse<T>(x, w, p); return; }
    }
    const int C = x.cfg->c;
    launch_records<DG, T>(x, p, 0, false);
    for (int i = C; i >= 1; --i) {
        if (i == 1 && C > 2) launch_sum<DG, T>(x, p.grp(1), p.ld, p.gs, C - 1, nullptr, x.rec(0));
        const Record<DG, T> out = (i == 2 && C == 2) ? x.rec(0) : x.rec(-1);
        launch_block<DG, T>(x, 1, x.rec(i - 1), w + (size_t)(i - 1) * DG * DG, p.grp(i - 1), p.ld, out, false, nullptr, 0);
    }
}

// Backward fused with the inverse.  slots_ready: slots 1..C-1 already hold the records of
// Y_1..Y_{C-1} of this layer (left by the forward sweep, or by the layer above while it rebuilt
// its input).  On return slots 1..C-1 hold the records of X_1..X_{C-1}, i.e. of the layer below
// (not written for the lowest layer of a step, `layer` = 0 with `in_step`).  When indices are
// saved, every record written here takes its column set from the kept masks of the layer it
// belongs to instead of selecting again.
template <int DG, typename T>
static void layer_backward_impl(const Ctx<DG, T>& x, const float* w, const Planes<T>& y, const Planes<T>& dy, float* dw_out,
                                bool slots_ready, int layer = 0, bool in_step = false) {
    if constexpr (DG == 64) {
        if (x.S > 1) { wide_backward<T>(x, w, y, dy, dw_out, slots_ready, layer, in_step); return; }
    }
    const int C = x.cfg->c;
    const bool given = x.saved != nullptr;
    // With few tiles per wave a launch is worth more than the work it takes along: dW_i's partials are summed beside the gradient's tiles
    // (first they would delay them: a 49,600-node graph with 3,100 tiles, +80 us on a 405 us kernel), and the rows
    // listed in the forward sweep get their kept column sets back where the record is taken (TieFix, while the lists are short) instead of in
    // a launch after it.
    const bool few_tiles = x.tiles < 4 * 4 * x.g->grid, fix_here = few_tiles && x.tie_cap <= TIE_FIX_MOST;
    if (!slots_ready) launch_records<DG, T>(x, y, layer, given);
    for (int i = C; i >= 1; --i) {
        const float* wi = w + (size_t)(i - 1) * DG * DG;
        const T* z;      // rows of Y_{i-1}
        int64_t ldz;
        if (i >= 2) { z = y.grp(i - 2); ldz = y.ld; }
        else if (C == 2) { z = y.grp(1); ldz = y.ld; }      // Y_0 = X_2, rebuilt just before
        else {
            launch_sum<DG, T>(x, y.grp(1), y.ld, y.gs, C - 1, x.y0(), x.rec(0, layer), given, x.tie_seg(-1, 0),
                              x.tie_seg(fix_here ? layer : -1, 0));
            if (!fix_here) launch_tie_fixup<DG, T>(x, x.tie_seg(layer, 0), x.y0(), DG, x.rec(0, layer));
            z = x.y0(); ldz = DG;
        }
        Record<DG, T> out = x.rec(-1);
        TieSeg<DG> out_tie = x.tie_seg(-1, 0);       // the segment that listed rows of `out` in the forward sweep
        if (i < C) {
            if (!(in_step && layer == 0)) {
                out = x.rec(i, given ? layer - 1 : 0);                                 // record of Y_i of the layer below
                if (in_step) out_tie = x.tie_seg(layer - 1, i);
            }
        } else if (C == 2) {
            out = x.rec(0, layer);                                                     // X_2 = Y_0 of this layer
            if (in_step) out_tie = x.tie_seg(layer, 0);
        }
        if (x.band) launch_hub_records<DG, T>(x, x.rec(i - 1, layer));
        else launch_hub_both<DG, T>(x, x.rec(i - 1, layer), dy.grp(i - 1), dy.ld);
        unsigned nparts;
        float* dwi = dw_out + (size_t)(i - 1) * DG * DG;
        if (split_dw<DG, T>(x.g)) {
            // X_i = Y_i - f_i(Y_{i-1}) with H kept for the weight gradient, then dW_i = H^T dY_i
            launch_block<DG, T>(x, 1, x.rec(i - 1, layer), wi, y.grp(i - 1), y.ld, out, given, nullptr, 0, true,
                                TieSeg<DG>{nullptr, nullptr, nullptr, 0, 0.f}, x.hplane());
            nparts = launch_dw<DG, T>(x, dy.grp(i - 1), dy.ld, out_tie, y.grp(i - 1), y.ld, out.mask ? &out : nullptr);
        } else {
            const bool fix = fix_here && out.mask;
            nparts = launch_block<DG, T>(x, 2, x.rec(i - 1, layer), wi, y.grp(i - 1), y.ld, out, given, dy.grp(i - 1), dy.ld, true,
                                         TieSeg<DG>{nullptr, nullptr, nullptr, 0, 0.f}, nullptr, fix ? out_tie : x.tie_seg(-1, 0));
            if (out.mask && !fix) launch_tie_fixup<DG, T>(x, out_tie, y.grp(i - 1), y.ld, out);
        }
        if (x.band) launch_dw_reduce<DG, T>(x, (int)nparts, dwi);
        if (x.band) {
            launch_band_grad<DG, 1, T>(x, dy.grp(i - 1), dy.ld, wi, i - 1, layer, z, ldz, 0, dy.grp(i >= 2 ? i - 2 : 1), dy.ld, dy.gs,
                                       i >= 2 ? 1 : C - 1);
            continue;
        }
        const typename MaskOf<DG>::type* own = x.rec(i - 1, layer).mask;
        // (large graphs: the partials are the first job of the gradient kernel's workgroups)
        launch_grad<DG, T>(x, dy.grp(i - 1), dy.ld, wi, own, z, ldz, dy.grp(i >= 2 ? i - 2 : 1), dy.ld, dy.gs, i >= 2 ? 1 : C - 1, (int)nparts,
                           few_tiles ? nullptr : dwi, true, few_tiles ? dwi : nullptr);
    }
}

template <int DG, typename T>
static Ctx<DG, T> make_ctx(const gsr_graph_t* g, const gsr_config_t* cfg, void* ws, hipStream_t s) {
    Ctx<DG, T> x;
    x.g = g; x.cfg = cfg; x.s = s; x.ws = (char*)ws; x.lw = carve_layer(cfg, g);
    x.tiles = (int)((cfg->n + 15) / 16);
    x.S = sub_planes(cfg);
    x.rows = records_as_rows(cfg, g);
    x.band = band_gradient(cfg, g);
    x.saved = nullptr;
    x.tie_counts = nullptr; x.tie_rows = nullptr; x.tie_masks = nullptr; x.tie_cap = 0;
    return x;
}

enum LayerOp { OP_FWD, OP_INV, OP_BWD };

template <int DG, typename T>
static gsr_status_t layer_call(LayerOp op, const gsr_graph_t* g, const gsr_config_t* cfg, const float* w, void* y, void* dy,
                               float* dw, void* ws, hipStream_t s) {
    Ctx<DG, T> x = make_ctx<DG, T>(g, cfg, ws, s);
    Planes<T> py = caller_planes<T>(y, cfg);
    if (op == OP_FWD) layer_forward_impl<DG, T>(x, w, py, false);
    else if (op == OP_INV) layer_inverse_impl<DG, T>(x, w, py);
    else layer_backward_impl<DG, T>(x, w, py, caller_planes<T>(dy, cfg), dw, false);
    GSR_HIP_CHECK(hipGetLastError());
    return GSR_OK;
}

// rows are moved in pieces of up to 16 bytes
static bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

static gsr_status_t layer_dispatch(LayerOp op, const gsr_graph_t* g, const gsr_config_t* cfg, const float* w, void* y, void* dy,
                                   float* dw, void* ws, size_t ws_bytes, void* stream) {
    GSR_TRY(validate_config(cfg, g, false));
    if (cfg->n == 0) return GSR_OK;
    if (!w || !y || !ws || (op == OP_BWD && (!dy || !dw))) return fail(GSR_ERR_INVALID_ARG, "null pointer");
    if (op == OP_BWD && !g->has_transpose) return fail(GSR_ERR_UNSUPPORTED, "graph has no transpose");
    const size_t need = carve_layer(cfg, g).total;
    if (ws_bytes < need) return fail(GSR_ERR_WORKSPACE_TOO_SMALL, "workspace %zu < %zu bytes", ws_bytes, need);
    if (!aligned16(y) || !aligned16(dy) || ((uintptr_t)ws & 255))
        return fail(GSR_ERR_INVALID_ARG, "planes must be 16-byte aligned and the workspace 256-byte aligned");
    hipStream_t s = (hipStream_t)stream;
    const int dg = cfg->d / cfg->c;
    if (cfg->dtype == GSR_F32) {
        if (dg == 32) return layer_call<32, float>(op, g, cfg, w, y, dy, dw, ws, s);
        return layer_call<64, float>(op, g, cfg, w, y, dy, dw, ws, s);
    }
    if (dg == 32) return layer_call<32, bf16_t>(op, g, cfg, w, y, dy, dw, ws, s);
    return layer_call<64, bf16_t>(op, g, cfg, w, y, dy, dw, ws, s);
}

template <int DG, typename T>
static gsr_status_t step_impl(const gsr_graph_t* g, const gsr_config_t* cfg, const void* x0, const float* w_all,
                              const float* w_out, const float* b_out, const float* target, float* loss_out, float* yhat_out,
                              float* dw_all, float* dw_out, float* db_out, void* dx0_out, void* x0_rebuilt_out, void* xl_out,
                              void* ws, hipStream_t s) {
    const StepWs sw = carve_step(cfg, g);
    char* base = (char*)ws;
    Ctx<DG, T> x = make_ctx<DG, T>(g, cfg, base + sw.layer, s);
    if (cfg->save_indices == 1) x.saved = (typename MaskOf<DG>::type*)(base + sw.masks);
    const int C = cfg->c, L = cfg->l;
    if (cfg->save_indices == 2) {
        x.tie_counts = (int*)(base + sw.tie_counts);
        x.tie_rows = (uint32_t*)(base + sw.tie_rows);
        x.tie_masks = (typename MaskOf<DG>::type*)(base + sw.tie_masks);
        x.tie_cap = (int)sw.tie_cap;
        const int ints = (L + 1) * C * TIE_SUB * TIE_COUNTER_STRIDE;
        hipLaunchKernelGGL(k_zero_ints, dim3((ints + 255) / 256), dim3(256), 0, s, x.tie_counts, ints);
    }
    const int64_t n = cfg->n;
    const int dgw = DG * x.S;            // columns of a group (DG, or 64 S for the groups handled as sub-planes)
    const Planes<T> act{(T*)(base + sw.act), (int64_t)dgw, n * dgw};
    const Planes<T> grad{(T*)(base + sw.grad), (int64_t)dgw, n * dgw};
    const Planes<T> in = caller_planes<T>(const_cast<void*>(x0), cfg);
    const dim3 cgrid((unsigned)g->grid * 4, (unsigned)C), cblock(256);
    auto copy = [&](const Planes<T>& from, const Planes<T>& to) {
        ProfScope prof(KC_COPY, s);
        constexpr int64_t VE = 16 / sizeof(T);
        const bool pieces = aligned16(from.base) && aligned16(to.base) && (from.ld | from.gs | to.ld | to.gs | dgw) % VE == 0;
        if (pieces && n * (dgw / VE) < ((int64_t)1 << 30))
            hipLaunchKernelGGL((k_copy_planes<uint4, uint32_t>), cgrid, cblock, 0, s, (uint32_t)n, (int)(dgw / VE), (const uint4*)from.base, from.ld / VE,
                               from.gs / VE, (uint4*)to.base, to.ld / VE, to.gs / VE);
        else
            hipLaunchKernelGGL((k_copy_planes<T, int64_t>), cgrid, cblock, 0, s, n, dgw, (const T*)from.base, from.ld, from.gs, to.base, to.ld, to.gs);
    };
    copy(in, act);
    const size_t wl = (size_t)C * dgw * dgw;
    for (int l = 0; l < L; ++l) layer_forward_impl<DG, T>(x, w_all + l * wl, act, C == 2 && l > 0, l);
    if (xl_out) copy(act, caller_planes<T>(xl_out, cfg));
    HeadArgs<T> h;
    h.n = (int)n; h.d = cfg->d; h.dg = dgw; h.act = act.base; h.grad = grad.base; h.ld = act.ld; h.gs = act.gs;
    h.w_out = w_out; h.b_out = b_out; h.target = target; h.yhat = yhat_out; h.partial = (float*)(base + sw.head);
    {
        ProfScope prof(KC_HEAD, s);
        const dim3 grid((unsigned)g->grid), block(256);
        if (cfg->d <= 64) hipLaunchKernelGGL((k_head<T, 1>), grid, block, 0, s, h);
        else if (cfg->d <= 128) hipLaunchKernelGGL((k_head<T, 2>), grid, block, 0, s, h);
        else if (cfg->d <= 256) hipLaunchKernelGGL((k_head<T, 4>), grid, block, 0, s, h);
        else hipLaunchKernelGGL((k_head<T, HEAD_MAXQ>), grid, block, 0, s, h);
        hipLaunchKernelGGL(k_head_reduce, dim3((cfg->d + 2 + 3) / 4), dim3(256), 0, s, (const float*)h.partial, g->grid,
                           cfg->d, (int)n, dw_out, db_out, loss_out);
    }
    for (int l = L - 1; l >= 0; --l) layer_backward_impl<DG, T>(x, w_all + l * wl, act, grad, dw_all + l * wl, true, l, true);
    if (dx0_out) copy(grad, caller_planes<T>(dx0_out, cfg));
    if (x0_rebuilt_out) copy(act, caller_planes<T>(x0_rebuilt_out, cfg));
    GSR_HIP_CHECK(hipGetLastError());
    return GSR_OK;
}

}  // namespace gsr

using namespace gsr;

extern "C" {

gsr_status_t gsr_layer_forward(const gsr_graph_t* g, const gsr_config_t* cfg, const float* w, void* x_inout, void* workspace,
                               size_t workspace_bytes, void* stream) {
    return layer_dispatch(OP_FWD, g, cfg, w, x_inout, nullptr, nullptr, workspace, workspace_bytes, stream);
}

gsr_status_t gsr_layer_inverse(const gsr_graph_t* g, const gsr_config_t* cfg, const float* w, void* y_inout, void* workspace,
                               size_t workspace_bytes, void* stream) {
    return layer_dispatch(OP_INV, g, cfg, w, y_inout, nullptr, nullptr, workspace, workspace_bytes, stream);
}

gsr_status_t gsr_layer_backward(const gsr_graph_t* g, const gsr_config_t* cfg, const float* w, void* y_inout, void* dy_inout,
                                float* dw_out, void* workspace, size_t workspace_bytes, void* stream) {
    return layer_dispatch(OP_BWD, g, cfg, w, y_inout, dy_inout, dw_out, workspace, workspace_bytes, stream);
}

gsr_status_t gsr_step(const gsr_graph_t* g, const gsr_config_t* cfg, const void* x0, const float* w_all, const float* w_out,
                      const float* b_out, const float* target, float* loss_out, float* yhat_out, float* dw_all, float* dw_out,
                      float* db_out, void* dx0_out, void* x0_rebuilt_out, void* xl_out, void* workspace, size_t workspace_bytes,
                      void* stream) {
    GSR_TRY(validate_config(cfg, g, true));
    if (cfg->d > HEAD_MAXQ * 64) return fail(GSR_ERR_UNSUPPORTED, "D=%d above %d", cfg->d, HEAD_MAXQ * 64);
    if (!x0 || !w_all || !w_out || !b_out || !target || !loss_out || !dw_all || !dw_out || !db_out || !workspace)
        return fail(GSR_ERR_INVALID_ARG, "null pointer");
    if (!g->has_transpose) return fail(GSR_ERR_UNSUPPORTED, "graph has no transpose");
    const size_t need = carve_step(cfg, g).total;
    if (workspace_bytes < need) return fail(GSR_ERR_WORKSPACE_TOO_SMALL, "workspace %zu < %zu bytes", workspace_bytes, need);
    if (cfg->n == 0) return fail(GSR_ERR_INVALID_ARG, "empty graph");
    if ((uintptr_t)workspace & 255) return fail(GSR_ERR_INVALID_ARG, "the workspace must be 256-byte aligned");
    hipStream_t s = (hipStream_t)stream;
    const int dg = cfg->d / cfg->c;
#define GSR_STEP(DGV, TV)                                                                                            \
    return step_impl<DGV, TV>(g, cfg, x0, w_all, w_out, b_out, target, loss_out, yhat_out, dw_all, dw_out, db_out, \
                              dx0_out, x0_rebuilt_out, xl_out, workspace, s)
    if (cfg->dtype == GSR_F32) {
        if (dg == 32) GSR_STEP(32, float);
        GSR_STEP(64, float);
    }
    if (dg == 32) GSR_STEP(32, bf16_t);
    GSR_STEP(64, bf16_t);
#undef GSR_STEP
}

gsr_status_t gsr_step_tie_stats(const gsr_graph_t* g, const gsr_config_t* cfg, const void* workspace, int64_t* listed,
                                int64_t* max_per_block, int64_t* dropped, void* stream) {
    GSR_TRY(validate_config(cfg, g, true));
    if (!workspace) return fail(GSR_ERR_INVALID_ARG, "null pointer");
    if (cfg->save_indices != 2) return fail(GSR_ERR_INVALID_ARG, "cfg->save_indices is not 2: nothing was listed");
    const StepWs sw = carve_step(cfg, g);
    const int segs = cfg->l * cfg->c;      // (the set listed for a layer above the last is never used)
    std::vector<int> counts((size_t)segs * TIE_SUB * TIE_COUNTER_STRIDE);
    GSR_HIP_CHECK(hipStreamSynchronize((hipStream_t)stream));
    GSR_HIP_CHECK(hipMemcpy(counts.data(), (const char*)workspace + sw.tie_counts, counts.size() * sizeof(int), hipMemcpyDeviceToHost));
    int64_t total = 0, most = 0, lost = 0;
    for (int seg = 0; seg < segs; ++seg) {
        int64_t in_block = 0;
        for (int sub = 0; sub < TIE_SUB; ++sub) {
            const int64_t c = counts[((size_t)seg * TIE_SUB + sub) * TIE_COUNTER_STRIDE];
            in_block += c;
            total += std::min<int64_t>(c, sw.tie_cap);
            lost += std::max<int64_t>(0, c - sw.tie_cap);
        }
        most = std::max(most, in_block);
    }
    if (listed) *listed = total;
    if (max_per_block) *max_per_block = most;
    if (dropped) *dropped = lost;
    return GSR_OK;
}

gsr_status_t gsr_step_tie_export(const gsr_graph_t* g, const gsr_config_t* cfg, const void* workspace, int32_t layer,
                                 int32_t block, int32_t* rows_out, uint64_t* masks_out, int64_t* count_out, void* stream) {
    GSR_TRY(validate_config(cfg, g, true));
    if (!workspace || !rows_out || !masks_out || !count_out) return fail(GSR_ERR_INVALID_ARG, "null pointer");
    if (cfg->save_indices != 2) return fail(GSR_ERR_INVALID_ARG, "cfg->save_indices is not 2: nothing was listed");
    if (layer < 0 || layer >= cfg->l || block < 1 || block > cfg->c) return fail(GSR_ERR_INVALID_ARG, "layer %d / block %d out of range", layer, block);
    const StepWs sw = carve_step(cfg, g);
    const size_t seg = (size_t)layer * cfg->c + (block - 1);
    const char* base = (const char*)workspace;
    GSR_HIP_CHECK(hipStreamSynchronize((hipStream_t)stream));
    std::vector<int> counts((size_t)TIE_SUB * TIE_COUNTER_STRIDE);
    GSR_HIP_CHECK(hipMemcpy(counts.data(), base + sw.tie_counts + seg * counts.size() * sizeof(int), counts.size() * sizeof(int), hipMemcpyDeviceToHost));
    const int dg = std::min(cfg->d / cfg->c, 64);
    const size_t mbytes = dg == 64 ? 8 : 4;
    int64_t written = 0;
    for (int sub = 0; sub < TIE_SUB; ++sub) {
        const int64_t take = std::min<int64_t>(counts[(size_t)sub * TIE_COUNTER_STRIDE], sw.tie_cap);
        if (take == 0) continue;
        const size_t at = (seg * TIE_SUB + sub) * (size_t)sw.tie_cap;
        GSR_HIP_CHECK(hipMemcpy(rows_out + written, base + sw.tie_rows + at * sizeof(uint32_t), (size_t)take * sizeof(uint32_t), hipMemcpyDeviceToHost));
        if (mbytes == 8) {
            GSR_HIP_CHECK(hipMemcpy(masks_out + written, base + sw.tie_masks + at * 8, (size_t)take * 8, hipMemcpyDeviceToHost));
        } else {
            std::vector<uint32_t> m32((size_t)take);
            GSR_HIP_CHECK(hipMemcpy(m32.data(), base + sw.tie_masks + at * 4, (size_t)take * 4, hipMemcpyDeviceToHost));
            for (int64_t i = 0; i < take; ++i) masks_out[written + i] = m32[(size_t)i];
        }
        written += take;
    }
    *count_out = written;
    return GSR_OK;
}

}  // extern "C"

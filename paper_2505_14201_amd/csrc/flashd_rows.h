// Pieces shared by the prefill kernels whose wavefronts share out the keys of a row tile
// (flashd_short.hip, flashd_tile64.hip): the hand-out of row tiles to workgroups and the step of a
// 32-key block whose top score is looked at before it is exponentiated.
#pragma once

#include "flashd_common.h"
#include "flashd_mma.h"

namespace flashd {

// Row tiles of unequal length, longest first, of which the first `rounds` times 256 (32 to an XCD) are
// resident together, one of every 256 on each compute unit: in order, the longest of all would share
// its compute unit with the longest of the second half.  So every other round runs backwards.
// local: id of a workgroup (within its XCD where nx_log2 is 3), locals: how many there are.
__device__ __forceinline__ int back_and_forth(int local, int nx_log2, int rounds, int locals) {
    const int log2 = 8 - nx_log2;
    const int round = local >> log2;
    if (round >= rounds || (round & 1) == 0) return local;
    const int begin = round << log2;
    return begin + min(begin + (1 << log2), locals) - 1 - local;
}

// How workgroups map to work: id -> (rank of the row tile, split, unit), all units' longest row
// tiles first; unit u on XCD u % 8 where the units divide by 8, so that K and V of a head are
// read into one L2.  A unit is a (b, kv head) with the query heads of its group interleaved: row r
// is position r / heads of head r % heads.
struct RowSched {
    int rows;           // query rows of a unit: (Hq / Hkv) * Lq
    int tiles;          // row tiles of a unit
    int nx_log2;        // 3: units are dealt over the XCDs, 0: not
    int per_split;      // key blocks (or tiles) per split
    int locals;         // workgroups (of an XCD where nx_log2 is 3)
    int rounds;         // rounds of them that are resident together where row tiles differ in length
    FastDiv per_rank;   // splits * units per XCD
    FastDiv per_unit;   // units per XCD
    FastDiv heads;      // Hq / Hkv
};

// tile_rows: query rows per workgroup; keys: keys of a block; per_cu: workgroups resident on a
// compute unit
inline RowSched row_sched(const Problem& p, int tile_rows, int keys, int per_cu) {
    RowSched sc;
    const int g = p.Hq / p.Hkv;
    const long units = (long)p.B * p.Hkv;
    sc.rows = g * p.Lq;
    sc.tiles = (sc.rows + tile_rows - 1) / tile_rows;
    sc.nx_log2 = units % 8 == 0 ? 3 : 0;
    const int blocks = (p.Lk + keys - 1) / keys;
    sc.per_split = (blocks + p.splits - 1) / p.splits;
    sc.per_rank = make_fast_div((uint32_t)((units >> sc.nx_log2) * p.splits));
    sc.per_unit = make_fast_div((uint32_t)(units >> sc.nx_log2));
    sc.heads = make_fast_div((uint32_t)g);
    sc.locals = (int)((units * sc.tiles * p.splits) >> sc.nx_log2);
    sc.rounds = p.causal ? per_cu : 0;
    return sc;
}
inline long row_sched_total(const Problem& p, const RowSched& sc) {
    return (long)p.B * p.Hkv * sc.tiles * p.splits;
}

struct RowTile {
    int sp;             // key split
    size_t unit;
    int first, last;    // the rows of the unit that exist
};

__device__ __forceinline__ RowTile row_tile(const Problem& p, const RowSched& sc, int tile_rows) {
    const uint32_t id = blockIdx.x;
    const uint32_t local = back_and_forth((int)(id >> sc.nx_log2), sc.nx_log2, sc.rounds, sc.locals);
    const uint32_t rank = fast_div(local, sc.per_rank);
    const uint32_t rem = local - rank * sc.per_rank.d;
    RowTile t;
    t.sp = (int)fast_div(rem, sc.per_unit);
    t.unit = ((rem - (uint32_t)t.sp * sc.per_unit.d) << sc.nx_log2) + (id & ((1u << sc.nx_log2) - 1u));
    t.first = (p.causal ? sc.tiles - 1 - (int)rank : (int)rank) * tile_rows;
    t.last = min(t.first + tile_rows, sc.rows) - 1;
    return t;
}

__device__ __forceinline__ int position_of(const RowSched& sc, int r) {
    return (int)fast_div((uint32_t)r, sc.heads);
}
// row r of the unit -> row of [B][Hq][Lq]
__device__ __forceinline__ size_t row_of(const Problem& p, const RowSched& sc, const RowTile& t, int r) {
    const int pos = position_of(sc, r);
    return (t.unit * sc.heads.d + (r - pos * (int)sc.heads.d)) * (size_t)p.Lq + pos;
}

// A row's state beside U: the sums are each lane's own keys' (two lanes to a row).
struct RowState {
    float R;            // exponent reference, log2 units; -inf: the row has seen no key
    float l;            // sum of 2^{s - R}, of the rounded coefficients where those are summed
    float ltrue;        // TL: of the unrounded ones
};

// One 32-key block (acc: its dot products with Q, in the accumulator layout; overwritten): the
// lazy form of flashd_mma.h with the block's top score looked at first, as in lazy_checked_pack.
// The reference starts at the first block's top score and moves when a top lies more than
// LazyLimit::kMoveLog2 above it.  masked: keys may be hidden, those at offsets lim and beyond from
// the lane's first.  c_log2 >= 0.
template <typename T, int NDB, bool TL>
__device__ __forceinline__ void top_first_pack(f32x16& acc, u32x4 (&bfrag)[2], RowState& st, f32x16 (&U)[NDB],
                                               float c_log2, bool masked, int lim) {
    const float ninf = -__builtin_inff();
    // A hidden key's dot product becomes -inf, which a positive c_log2 leaves as it is: scores under a mask are
    // scaled and referred in one fma like the others.  (Any other c_log2, 0 or NaN, is applied here: it would
    // take a hidden key away from -inf.)
    const bool scaled = masked && !(c_log2 > 0.0f);
    const float scale = scaled ? 1.0f : c_log2;      // what is left to scale the scores by
    if (masked) {
        const float by = scaled ? c_log2 : 1.0f;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 8 * (r >> 2) + (r & 3) >= lim ? ninf : acc[r] * by;
    }
    float top = acc[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) top = fmaxf(top, acc[r]);
    top = pair_max(top) * scale;
    if (__builtin_amdgcn_ballot_w64(top > st.R + LazyLimit<T>::kMoveLog2) != 0) {
        const bool move = top > st.R + LazyLimit<T>::kMoveLog2;
        const float f = move ? exp2_fast(st.R - top) : 1.0f;        // 0 for a row without keys
        st.R = move ? top : st.R;
        st.l *= f;
        st.ltrue *= f;
#pragma unroll
        for (int i = 0; i < NDB; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) U[i][r] *= f;
    }
    // no key yet, or only keys of score -inf: weights of zero
    const float ref = st.R == ninf ? 0.0f : st.R;
    f32x4 ps = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        f32x8 pv;
#pragma unroll
        for (int e = 0; e < 8; ++e) pv[e] = exp2_fast(fmaf(acc[8 * g + e], scale, -ref));
        bfrag[g] = Mma<T>::pack8(pv);
        Mma<T>::sum8(pv, bfrag[g], ps);
        if (TL) st.ltrue += ((pv[0] + pv[1]) + (pv[2] + pv[3])) + ((pv[4] + pv[5]) + (pv[6] + pv[7]));
    }
    st.l += (ps[0] + ps[1]) + (ps[2] + ps[3]);
}

}  // namespace flashd

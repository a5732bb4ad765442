// Tiled FLASH-D prefill with 64 query rows per workgroup (variant TILE, f16/bf16), for calls whose
// 128-row tiles leave compute units idle or end on their longest row tiles.
//
// Same tile form of Alg. 3 as flashd_tile.hip, same LDS layout and copies of a 64-key tile.  There
// a wavefront owns 32 rows and all 64 keys of a tile; here the four wavefronts are two pairs: wavefront
// w owns rows 32 (w & 1) .. + 31 and keys 32 (w >> 1) .. + 31 of every tile, with a state of its
// own, and the two states of a row are folded at the end.  Twice the workgroups, each with half of
// the matrix and vector work per tile, and no partial states in memory or second launch as a
// split of the keys over workgroups needs.
#include "flashd_common.h"
#include "flashd_kernels.h"
#include "flashd_mma.h"
#include "flashd_rows.h"
#include "flashd_tile_parts.h"

namespace flashd {

constexpr int kT64Rows = 64;        // query rows per workgroup
constexpr int KW = 2;               // wavefronts that share out the keys of a row

// TL: the state is handed out and the coefficient sums are those of the rounded coefficients, so the
// unrounded sum is carried as well (the Lam handed out is then the true log-sum-exp).
template <typename T, int D, bool TL>
__global__ __launch_bounds__(kNW * 64, D == 64 ? 4 : 2)
void tile64_kernel(Problem p, RowSched sc) {
    constexpr bool kTL = TL && Mma<T>::kRoundedSum;
    using C = TileCfg<D>;
    constexpr int NKK = D / 16;
    constexpr int NDB = D / 32;
    constexpr int kSlots = 2;                 // tiles of K and V in LDS
    constexpr int kTile = kBC * D;
    constexpr int GR = 4 * NDB / KW;          // groups of four registers of U a wavefront finishes
    constexpr int kCols = D / KW;             // the columns they are
    constexpr int FROW = kCols + 4;           // floats per row of the staged output
    __shared__ __align__(1024) uint16_t lds[2 * kSlots * kTile];     // K tiles, V tiles
    __shared__ float fold_r[kNW][32], fold_l[kNW][32], fold_t[kTL ? kNW : 1][32], from_in[kNW][32];
    static_assert(4 * kNW * 32 * D <= (int)sizeof(lds) && FROW <= D, "the fold lies in the tiles' LDS");

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kw = wave >> 1;               // which 32 keys of every tile
    const int c = lane & 31;
    const int hh = lane >> 5;
    const float ninf = -__builtin_inff();

    const RowTile rt = row_tile(p, sc, kT64Rows);

    // key tiles of this row tile and split
    const int most = visible_at(p, position_of(sc, rt.last));
    const int t_begin = rt.sp * sc.per_split;
    const int n = max(min((most + kBC - 1) / kBC, t_begin + sc.per_split) - t_begin, 0);
    const int jbase = t_begin * kBC;
    const uint16_t* kg = static_cast<const uint16_t*>(p.k) + rt.unit * (size_t)p.Lk * D;
    const uint16_t* vg = static_cast<const uint16_t*>(p.v) + rt.unit * (size_t)p.Lk * D;
    const DmaLane<D> dl(wave, lane);
    auto copy = [&](int t) __attribute__((always_inline)) {
        uint16_t* dst = lds + (t % kSlots) * kTile;
        tile_copy<D>(kg, vg, jbase + t * kBC, p.Lk, dl, wave, lane, dst, dst + kSlots * kTile);
    };

    // the wavefront's rows; rows past the end stand in for the last one and are not stored
    const int wrow0 = rt.first + 32 * (wave & 1);
    const int row = min(wrow0 + c, rt.last);
    const uint16_t* qg = static_cast<const uint16_t*>(p.q) + row_of(p, sc, rt, row) * D;
    u32x4 qf[NKK];
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk)
        qf[kk] = *reinterpret_cast<const u32x4*>(qg + 16 * kk + 8 * hh);
    if (n > 0) copy(0);
    // a negative scale is taken into Q (exact), so that the largest dot product is the top score
    float c_log2 = p.scale * kLog2e;
    if (c_log2 < 0.0f) {
        c_log2 = -c_log2;
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk) qf[kk] ^= u32x4{0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u};
    }
    const int nvis = visible_at(p, position_of(sc, row));
    const int wmin = visible_at(p, position_of(sc, min(wrow0, rt.last)));
    const int wmax = visible_at(p, position_of(sc, min(wrow0 + 31, rt.last)));

    // operand addresses inside a tile (elements)
    int kaddr[NKK], vaddr[NDB];
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk)
        kaddr[kk] = (32 * kw + c) * D + 8 * ((2 * kk + hh) ^ C::swz_k(32 * kw + c));
    {
        const int t = lane & 15;
        const int tq = t >> 2;
        const int half = (lane >> 4) & 1;
#pragma unroll
        for (int i = 0; i < NDB; ++i)
            vaddr[i] = (32 * kw + 4 * hh + tq) * D +
                       8 * ((4 * i + 2 * half + ((t & 3) >> 1)) ^ C::swz_v(tq)) + 4 * (t & 1);
    }

    f32x16 U[NDB];
#pragma unroll
    for (int i = 0; i < NDB; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) U[i][r] = 0.0f;
    RowState st = {ninf, 0.0f, 0.0f};

    // Period t: start the copies of tile t + 1 into the other slot, which was last read in period
    // t - 1; do the math of tile t; wait for the copies; barrier.
    if (n > 0) {
        wait_copies();
        __syncthreads();
    }
    for (int t = 0; t < n; ++t) {
        if (t + 1 < n) copy(t + 1);
        const int j0 = jbase + t * kBC + 32 * kw;
        if (j0 < wmax) {
            const uint16_t* ks = lds + (t % kSlots) * kTile;
            const uint16_t* vs = ks + kSlots * kTile;
            u32x4 ka[NKK];
#pragma unroll
            for (int kk = 0; kk < NKK; ++kk) ka[kk] = *reinterpret_cast<const u32x4*>(&ks[kaddr[kk]]);
            f32x16 acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
            for (int kk = 0; kk < NKK; ++kk) acc = Mma<T>::mfma(ka[kk], qf[kk], acc);
            // V operands on their way while the coefficients are formed
            u32x4 va[2 * NDB];
#pragma unroll
            for (int m = 0; m < 2 * NDB; ++m) va[m] = tile_v_operand<D>(vs, vaddr[m % NDB], 16 * (m / NDB));

            u32x4 bfrag[2];
            top_first_pack<T, NDB, kTL>(acc, bfrag, st, U, c_log2, j0 + 32 > wmin, nvis - (j0 + 4 * hh));
#pragma unroll
            for (int m = 0; m < 2 * NDB; ++m) U[m % NDB] = Mma<T>::mfma(va[m], bfrag[m / NDB], U[m % NDB]);
        }
        wait_copies();
        __syncthreads();
    }

    // ---- fold the two states of a row, and the state handed in --------------------------
    st.l = pair_sum(st.l);
    if (kTL) st.ltrue = pair_sum(st.ltrue);
    if (hh == 0) {
        fold_r[wave][c] = st.R;
        fold_l[wave][c] = st.l;
        if (kTL) fold_t[wave][c] = st.ltrue;
    }
    __syncthreads();                     // also: nobody reads the tiles any more
    float lam_out, w_in = 0.0f;
    {
        float r_in = ninf;
        if (p.from_state) {
            const float* src = p.state_in + row_of(p, sc, rt, row) * (D + 2);
            r_in = (src[D] - src[D + 1]) * kLog2e;
        }
        float top = r_in;
#pragma unroll
        for (int w = 0; w < KW; ++w) top = fmaxf(top, fold_r[2 * w + (wave & 1)][c]);
        const float f_in = r_in == ninf ? 0.0f : exp2_fast(r_in - top);
        float lt = f_in;         // by the unrounded sums where they are at hand, see flashd_short.hip
#pragma unroll
        for (int w = 0; w < KW; ++w) {
            // A state without a key of the row is left out: its U holds 0 * V of keys that other
            // rows see, and that is NaN where such a V is infinite.  (l is 1 or more with a key,
            // NaN with a NaN score.)
            const float lw = fold_l[2 * w + (wave & 1)][c];
            const float fw = lw == 0.0f ? 0.0f : exp2_fast(fold_r[2 * w + (wave & 1)][c] - top);
            lt = fmaf(fw, kTL ? fold_t[2 * w + (wave & 1)][c] : lw, lt);
        }
        const float f = st.l == 0.0f ? 0.0f : exp2_fast(st.R - top);
        const bool empty = lt == 0.0f;
        lam_out = empty ? ninf : (top + log2_fast(lt)) * kLn2;
        const float fin = empty ? 0.0f : 1.0f / lt;
        w_in = f_in * fin;
        const float mul = (kTL && st.l != 0.0f ? f * st.ltrue * __builtin_amdgcn_rcpf(st.l) : f) * fin * p.oscale;
        const bool none = st.l == 0.0f;
#pragma unroll
        for (int i = 0; i < NDB; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) U[i][r] = none ? 0.0f : U[i][r] * mul;
    }
    // A wavefront finishes kCols columns of its rows: the states are handed over as they stand in the
    // registers, and each adds up its columns of all of them
    f32x4* xch = reinterpret_cast<f32x4*>(lds);
#pragma unroll
    for (int i = 0; i < NDB; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            xch[(wave * 4 * NDB + 4 * i + q) * 64 + lane] =
                f32x4{U[i][4 * q], U[i][4 * q + 1], U[i][4 * q + 2], U[i][4 * q + 3]};
    __syncthreads();
    f32x4 x[GR];
#pragma unroll
    for (int e = 0; e < GR; ++e) {
        x[e] = xch[((wave & 1) * 4 * NDB + kw * GR + e) * 64 + lane];
#pragma unroll
        for (int w = 1; w < KW; ++w) x[e] += xch[((2 * w + (wave & 1)) * 4 * NDB + kw * GR + e) * 64 + lane];
    }
    __syncthreads();
    // row by row through LDS, so that the stores are of whole pieces of rows
    float* stage = reinterpret_cast<float*>(lds) + wave * 32 * FROW;
#pragma unroll
    for (int e = 0; e < GR; ++e) *reinterpret_cast<f32x4*>(&stage[c * FROW + 8 * e + 4 * hh]) = x[e];
    if (hh == 0) from_in[wave][c] = w_in;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // rows of states are d + 2 floats long, so 8-byte aligned
    typedef float f4a8 __attribute__((ext_vector_type(4), aligned(8)));
    constexpr int LPR = kCols / 8;       // lanes of a row, 8 columns each
    constexpr int NST = 32 * LPR / 64;
#pragma unroll
    for (int s = 0; s < NST; ++s) {
        const int r = (s * 64 + lane) / LPR;
        const int t = 8 * (lane % LPR);
        if (wrow0 + r > rt.last) continue;
        const size_t orow = row_of(p, sc, rt, wrow0 + r);
        const int col = kw * kCols + t;
        f32x4 lo = *reinterpret_cast<const f32x4*>(&stage[r * FROW + t]);
        f32x4 hi = *reinterpret_cast<const f32x4*>(&stage[r * FROW + t + 4]);
        if (p.from_state) {
            const float w = from_in[wave][r];
            const float* src = p.state_in + orow * (D + 2) + col;
            const f4a8 a = *reinterpret_cast<const f4a8*>(src);
            const f4a8 b = *reinterpret_cast<const f4a8*>(src + 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                lo[e] = w != 0.0f ? fmaf(w, a[e], lo[e]) : lo[e];
                hi[e] = w != 0.0f ? fmaf(w, b[e], hi[e]) : hi[e];
            }
        }
        if (p.store_o)
            *reinterpret_cast<u32x4*>(static_cast<uint16_t*>(p.o) + orow * D + col) =
                Mma<T>::pack8(f32x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
        if (p.partial) {
            float* dst = p.ws + ((size_t)rt.sp * p.B * p.Hq * p.Lq + orow) * (D + 2) + col;
            *reinterpret_cast<f4a8*>(dst) = f4a8{lo[0], lo[1], lo[2], lo[3]};
            *reinterpret_cast<f4a8*>(dst + 4) = f4a8{hi[0], hi[1], hi[2], hi[3]};
        }
    }
    if (p.partial && kw == 0 && hh == 0 && wrow0 + c <= rt.last) {
        float* dst = p.ws + ((size_t)rt.sp * p.B * p.Hq * p.Lq + row_of(p, sc, rt, row)) * (D + 2);
        dst[D] = lam_out;
        dst[D + 1] = 0.0f;
    }
}

template <typename T, int D>
static hipError_t launch_tile64_t(const Problem& p, hipStream_t st) {
    const RowSched sc = row_sched(p, kT64Rows, kBC, D == 64 ? 4 : 2);
    const long total = row_sched_total(p, sc);
    if (total > 0x7fffffffL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)total), block(kNW * 64);
    if (p.partial) hipLaunchKernelGGL((tile64_kernel<T, D, true>), grid, block, 0, st, p, sc);
    else hipLaunchKernelGGL((tile64_kernel<T, D, false>), grid, block, 0, st, p, sc);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !p.merge) return e;
    return launch_merge_splits(p, st);
}

hipError_t launch_tile64(const Problem& p, hipStream_t st) {
    if (p.dtype == 1 && p.d == 64) return launch_tile64_t<F16, 64>(p, st);
    if (p.dtype == 1 && p.d == 128) return launch_tile64_t<F16, 128>(p, st);
    if (p.dtype == 2 && p.d == 64) return launch_tile64_t<BF16, 64>(p, st);
    if (p.dtype == 2 && p.d == 128) return launch_tile64_t<BF16, 128>(p, st);
    return hipErrorInvalidValue;
}

}  // namespace flashd

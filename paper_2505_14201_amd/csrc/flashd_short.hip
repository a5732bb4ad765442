// Prefill of small calls (f16/bf16, K and V of that type or fp8, variant TILE): 32 query rows per
// workgroup, whose keys are shared out over its four wavefronts.
//
// The 128-row kernel gives a wavefront 32 rows and all of their keys, 64 at a time, and a call with
// fewer row tiles than compute units leaves the chip idle while each walks its keys one after the
// other.  Here a workgroup owns 32 rows of a kv head (the heads of a kv group interleaved row by
// row) and wavefront w takes the 32-key blocks w, w + 4, ... with a state of its own; the four
// states are folded in LDS.  Four times the workgroups, each a quarter as long, and no partial
// states in memory and second launch as a split over workgroups needs.
//
// What bounds it: a block is one chain (K through LDS, scores, top score, exponentials, V through
// LDS, output product) of 0.8 us at d = 128 and 0.5 at 64 with one workgroup on a compute unit, whose LDS
// is then busy 27 % of the time (16 % at 64), its matrix cores 15 % and a wavefront's vector work 24 %: the chain.
// Two share it at 1.5 us a block; from fp8 LDS is busy 52 % of the time then, a third of that for bank conflicts
// of the widened rows.  Direct global->LDS copies in place of registers, with the scores
// of the next block formed before the coefficients of this one, ran at 0.9: no shorter.  Measured (bf16;
// 128-row kernel, then this): 1 x 8 heads, 1024 x 1024, d = 128 23.0 and 12.2 us (64 row tiles of 128),
// 5 x 12, 101 x 383 13.1 and 8.3, 1 x 16 of 576 causal, d = 64 13.8 and 7.4.
//
// Keys are fetched a block ahead into registers and staged through LDS, K and V in turn, as in
// flashd_decode16.hip; loads go through buffer descriptors that end with the split, so that the
// fetch of a next block that is not there needs neither a branch nor a clamped address.  A
// block's top score is looked at before it is exponentiated.
#include "flashd_common.h"
#include "flashd_kernels.h"
#include "flashd_mma.h"
#include "flashd_rows.h"

namespace flashd {

constexpr int kShortWaves = 4;
constexpr int kShortRows = 32;       // query rows per workgroup
constexpr int kShortBlock = 32;      // keys per wavefront step

template <int N> struct ShortInt { static constexpr int value = N; };

// TL: the state is handed out and the coefficient sums are those of the rounded coefficients, so
// the unrounded sum is carried as well (the Lam handed out is then the true log-sum-exp).
// FP8: K and V are stored as fp8.
template <typename T, int D, bool FP8, bool TL>
__global__ __launch_bounds__(kShortWaves * kWave, D == 64 ? 4 : 2)
void short_kernel(Problem p, RowSched sc) {
    constexpr bool kTL = TL && Mma<T>::kRoundedSum;
    constexpr int NKK = D / 16;                 // score products per block
    constexpr int NDB = D / 32;                 // 32-wide blocks of the output
    constexpr int ESZ = FP8 ? 1 : 2;
    constexpr int NV = kShortBlock * D * ESZ / 1024;   // 16-byte loads of K or V per lane and block
    constexpr int CPR = D * ESZ / 16;           // 16-byte chunks per key row
    constexpr int kBlockBytes = kShortBlock * D * ESZ;
    // LDS rows: 16 rows of a 16-byte read, 4 rows of a transposing read, land on all banks
    constexpr int KROW = D + 8;
    constexpr int VROW = D + 32;
    constexpr int STAGE = kShortBlock * VROW;   // elements per wavefront
    constexpr int FROW = D + 4;                 // floats per row of the fold buffer
    constexpr int kLds = 2 * kShortWaves * STAGE > 4 * kShortWaves * kShortRows * FROW
                             ? 2 * kShortWaves * STAGE : 4 * kShortWaves * kShortRows * FROW;
    __shared__ __align__(16) char lds[kLds];
    __shared__ float fold_r[kShortWaves][kShortRows], fold_l[kShortWaves][kShortRows],
        fold_t[kTL ? kShortWaves : 1][kShortRows];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 31;
    const int hh = lane >> 5;
    const float ninf = -__builtin_inff();
    const RowTile rt = row_tile(p, sc, kShortRows);

    // 32-key blocks of this row tile and split; wavefront w takes blk_begin + w, + 4, ...
    const int nvis_min = visible_at(p, position_of(sc, rt.first));
    const int nvis_max = visible_at(p, position_of(sc, rt.last));
    const int blk_begin = rt.sp * sc.per_split;
    const int blk_end = min((nvis_max + kShortBlock - 1) / kShortBlock, blk_begin + sc.per_split);
    const char* kg = static_cast<const char*>(p.k) + rt.unit * (size_t)p.Lk * (D * ESZ);
    const char* vg = static_cast<const char*>(p.v) + rt.unit * (size_t)p.Lk * (D * ESZ);
    const int64_t range = (int64_t)min(p.Lk, blk_end * kShortBlock) * (D * ESZ);

    u32x4 kreg[NV], vreg[NV];
    auto fetch = [&](const char* base, int blk_, u32x4 (&reg)[NV]) __attribute__((always_inline)) {
        const int64_t at = (int64_t)blk_ * kBlockBytes;
        const auto w = kv_window(base + at, range - at);
#pragma unroll
        for (int n = 0; n < NV; ++n) reg[n] = kv_load<0>(w, 1024 * n + 16 * lane);
    };
    int blk = blk_begin + wave;
    fetch(kg, blk, kreg);
    fetch(vg, blk, vreg);

    // Query row of this lane's column.  Columns past the last row stand in for it (output
    // discarded), so that they never leave the path it takes.
    const int row = min(rt.first + c, rt.last);
    const uint16_t* qg = static_cast<const uint16_t*>(p.q) + row_of(p, sc, rt, row) * D;
    u32x4 qf[NKK];
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk)
        qf[kk] = *reinterpret_cast<const u32x4*>(qg + 16 * kk + 8 * hh);
    // a negative scale is taken into Q (exact), so that the largest dot product is the top score
    float c_log2 = (FP8 ? p.scale * p.kscale : p.scale) * kLog2e;
    if (c_log2 < 0.0f) {
        c_log2 = -c_log2;
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk) qf[kk] ^= u32x4{0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u};
    }
    const int nvis = visible_at(p, position_of(sc, row));

    uint16_t* vs = reinterpret_cast<uint16_t*>(lds) + wave * STAGE;
    f32x16 U[NDB];
#pragma unroll
    for (int i = 0; i < NDB; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) U[i][r] = 0.0f;
    RowState st = {ninf, 0.0f, 0.0f};

    // K or V of a block -> this wavefront's LDS stage, which the two take in turn
    auto stage = [&](const u32x4 (&reg)[NV], auto row_elems) __attribute__((always_inline)) {
        constexpr int ROW = decltype(row_elems)::value;
#pragma unroll
        for (int n = 0; n < NV; ++n) {
            const int ch = n * kWave + lane;
            uint16_t* dst = &vs[(ch / CPR) * ROW + (FP8 ? 16 : 8) * (ch % CPR)];
            if constexpr (FP8) {
                *reinterpret_cast<u32x4*>(dst) = widen8<T>(reg[n][0], reg[n][1]);
                *reinterpret_cast<u32x4*>(dst + 8) = widen8<T>(reg[n][2], reg[n][3]);
            } else {
                *reinterpret_cast<u32x4*>(dst) = reg[n];
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    // the next write to the stage must not overtake the reads of it
    auto stage_done = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };

    for (; blk < blk_end; blk += kShortWaves) {
        const int j0 = blk * kShortBlock;
        // S^T = K Q^T
        stage(kreg, ShortInt<KROW>{});
        fetch(kg, blk + kShortWaves, kreg);
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk)
            acc = Mma<T>::mfma(*reinterpret_cast<const u32x4*>(&vs[c * KROW + 16 * kk + 8 * hh]), qf[kk], acc);
        stage_done();
        stage(vreg, ShortInt<VROW>{});
        fetch(vg, blk + kShortWaves, vreg);
        u32x4 bfrag[2];
        top_first_pack<T, NDB, kTL>(acc, bfrag, st, U, c_log2, j0 + kShortBlock > nvis_min, nvis - (j0 + 4 * hh));
#pragma unroll
        for (int g2 = 0; g2 < 2; ++g2)
#pragma unroll
            for (int i = 0; i < NDB; ++i)
                U[i] = Mma<T>::mfma(lds_read_v_operand(&vs[16 * g2 * VROW + 32 * i], VROW, lane),
                                    bfrag[g2], U[i]);
        stage_done();
    }

    // ---- fold the four wavefront states, and the state handed in ------------------------
    st.l = pair_sum(st.l);
    if (kTL) st.ltrue = pair_sum(st.ltrue);
    __syncthreads();                                   // stages are dead, reuse the LDS
    float* fold = reinterpret_cast<float*>(lds);       // [wave][row][FROW]
#pragma unroll
    for (int i = 0; i < NDB; ++i)
#pragma unroll
        for (int n = 0; n < 4; ++n)
            *reinterpret_cast<f32x4*>(&fold[(wave * kShortRows + c) * FROW + 32 * i + 8 * n + 4 * hh]) =
                f32x4{U[i][4 * n], U[i][4 * n + 1], U[i][4 * n + 2], U[i][4 * n + 3]};
    if (hh == 0) {
        fold_r[wave][c] = st.R;
        fold_l[wave][c] = st.l;
        if (kTL) fold_t[wave][c] = st.ltrue;
    }
    __syncthreads();
    // rows of states are d + 2 floats long, so 8-byte aligned
    typedef float f4a8 __attribute__((ext_vector_type(4), aligned(8)));
    const float oscale = FP8 ? p.vscale : p.oscale;
#pragma unroll
    for (int it = 0; it < kShortRows * (D / 4) / (kShortWaves * kWave); ++it) {
        const int idx = it * kShortWaves * kWave + tid;
        const int fr = idx / (D / 4);
        const int t = 4 * (idx % (D / 4));
        if (rt.first + fr > rt.last) break;
        const size_t orow = row_of(p, sc, rt, rt.first + fr);
        float top = fold_r[0][fr];
#pragma unroll
        for (int w = 1; w < kShortWaves; ++w) top = fmaxf(top, fold_r[w][fr]);
        // Where the unrounded sums are at hand a wavefront weighs by them, as a partial state does: u / l is
        // its output and l, the sum of rounded coefficients, is up to 2^-9 off.  (bf16 states,
        // scores of deviation 16, 270 calls: error of o against fp64 over that of the 128-row kernel in its
        // splits 0.83 on average and 1.14 at most; by l 0.96 and 2.15.)
        float lt = 0.0f;
        f32x4 o = {0.0f, 0.0f, 0.0f, 0.0f};
        if (p.from_state) {
            // the earlier keys are one key of score Lam and value o
            const float* src = p.state_in + orow * (D + 2);
            const float r_in = (src[D] - src[D + 1]) * kLog2e;
            const f4a8 oin = *reinterpret_cast<const f4a8*>(src + t);
            top = fmaxf(top, r_in);
            const float f = r_in == ninf ? 0.0f : exp2_fast(r_in - top);
            lt = f;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = f != 0.0f ? f * oin[e] : 0.0f;
        }
#pragma unroll
        for (int w = 0; w < kShortWaves; ++w) {
            // A wavefront without a key of the row is left out: its U holds 0 * V of keys that
            // other rows see, and that is NaN where such a V is infinite.  (l is 1 or more with a
            // key, NaN with a NaN score.)
            const bool none = fold_l[w][fr] == 0.0f;
            const float f = none ? 0.0f : exp2_fast(fold_r[w][fr] - top);
            const f32x4 u = *reinterpret_cast<const f32x4*>(&fold[(w * kShortRows + fr) * FROW + t]);
            lt = fmaf(f, kTL ? fold_t[w][fr] : fold_l[w][fr], lt);
            const float fu = kTL && !none ? f * fold_t[w][fr] * __builtin_amdgcn_rcpf(fold_l[w][fr]) : f;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = fmaf(fu, none ? 0.0f : u[e], o[e]);
        }
        const bool empty = lt == 0.0f;
        if (!empty) o *= 1.0f / lt * oscale;
        if (p.store_o)
            *reinterpret_cast<u32x2*>(static_cast<uint16_t*>(p.o) + orow * D + t) = Mma<T>::pack4(o);
        if (p.partial) {
            float* dst = p.ws + ((size_t)rt.sp * p.B * p.Hq * p.Lq + orow) * (D + 2);
            *reinterpret_cast<f4a8*>(dst + t) = f4a8{o[0], o[1], o[2], o[3]};
            if (t == 0) {
                dst[D] = empty ? ninf : (top + log2_fast(lt)) * kLn2;
                dst[D + 1] = 0.0f;
            }
        }
    }
}

template <typename T, int D>
static hipError_t launch_short_t(const Problem& p, hipStream_t st) {
    const RowSched sc = row_sched(p, kShortRows, kShortBlock, D == 64 ? 4 : 2);
    const long total = row_sched_total(p, sc);
    if (total > 0x7fffffffL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)total), block(kShortWaves * kWave);
    if (!p.kv8) {
        if (p.partial) hipLaunchKernelGGL((short_kernel<T, D, false, true>), grid, block, 0, st, p, sc);
        else hipLaunchKernelGGL((short_kernel<T, D, false, false>), grid, block, 0, st, p, sc);
    } else {
        if (p.partial) hipLaunchKernelGGL((short_kernel<T, D, true, true>), grid, block, 0, st, p, sc);
        else hipLaunchKernelGGL((short_kernel<T, D, true, false>), grid, block, 0, st, p, sc);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !p.merge) return e;
    return launch_merge_splits(p, st);
}

hipError_t launch_short(const Problem& p, hipStream_t st) {
    if (p.dtype == 1 && p.d == 64) return launch_short_t<F16, 64>(p, st);
    if (p.dtype == 1 && p.d == 128) return launch_short_t<F16, 128>(p, st);
    if (p.dtype == 2 && p.d == 64) return launch_short_t<BF16, 64>(p, st);
    if (p.dtype == 2 && p.d == 128) return launch_short_t<BF16, 128>(p, st);
    return hipErrorInvalidValue;
}

}  // namespace flashd

// Split-K decode for at most 16 query rows per kv head (variant TILE; f16/bf16 storage of Q, K and
// V of that type or fp8), with or without the saturation skip of Sec. III-C on the V fetch.  The
// kernels of flashd_decode.hip serve 17 to 32 rows and the other variants.
//
// A decode step of a grouped-query model has 4 or 8 query rows per kv head.  On the 32-column
// score tiles of flashd_decode.hip three quarters of the exponentials and matrix work are done for
// columns that hold no row: a 32-key block took a wavefront 1.1 us, which bounded short contexts
// (a launch has few blocks per wavefront and little else to run meanwhile) and the fp8 cache
// (half the bytes for the same instructions).  Here the tiles are 16 columns wide
// (v_mfma_f32_16x16x32): half the vector and half the matrix work per key.
//
// Mapping.  A workgroup of W wavefronts owns one (b, kv head, key split); wavefront w takes the
// 32-key blocks w, w + W, ... with a state of its own, the W are folded at the end.  W is 4; 8 for
// the whole calls that decode_on_eight in flashd_plan.h names, with its figures.  Lane
// (q, c) = (lane / 16, lane % 16): S^T = K Q^T comes as two 16-key tiles of which the lane holds,
// for query row c, the keys 4 q + r and 16 + 4 q + r (r = 0..3).  Rounded and packed, these are the
// eight B elements of the lane for O^T = V^T P^T over the whole block; V^T comes from the
// transposing LDS read in the same key order.  K and V are fetched in contiguous KBs into
// registers a block ahead and staged through the same LDS rows in turn.  What a compute unit
// streams is bounded by its requests in flight: K read as the A operand it is, 64 bytes per key
// and instruction, needs no LDS but half as many bytes per request, and took 1.7 us a block
// against 1.06 with one workgroup per compute unit (level at two, where HBM is the bound).
// Only the fp8 kernel with two workgroups per compute unit does that: it saves widening K into
// LDS (64 x 8 heads x 8192 keys: 154 us against 159; 64 x 8 x 2000: 41.5 against 43.6).
//
// Loads go through buffer descriptors whose size is what is left of the split: a block that sticks
// out past it, or lies past it, reads zeros without touching memory.  So the fetch of the next
// block needs neither a branch nor a clamped address, and the skip of a V fetch is a descriptor
// of size zero.
//
// State of a row: R, l = sum 2^{s - R} over the keys seen, each of the row's four lanes its own
// keys', and U; o = U / l, Lam = R + log2 l.  A block's top score is looked at first; the
// reference starts at the first block's and moves when a top lies more than kMoveLog2 above it
// (flashd_mma.h, lazy_checked_pack).
//
// Skip: the criterion and its margin are those of decode_vskip_kernel (flashd_decode.hip), with the
// largest score seen in place of Lam (a bound of it from below).  The scores decide, so V runs
// one block behind K, and is requested before the block's exponentials.
//
// Measured (bf16, d = 128, 32 / 8 heads, one position; before, on the 32-column kernels and their
// splits): 1 x 1000 keys 9.5 us (13.5), 4 x 3000 13.8 (18.0), 16 x 600 9.7 (15.6), 20 x 4000 51 (59),
// 64 x 8192 309 (312: 6.9 TB/s, HBM's rate).
#include "flashd_common.h"
#include "flashd_kernels.h"
#include "flashd_mma.h"

#include <type_traits>

namespace flashd {

constexpr int kD16Block = 32;      // keys per wavefront step

struct Dec16Sched {
    int nrows;         // query rows of a kv group, (Hq / Hkv) * Lq <= 16
    int per_split;     // 32-key blocks per split
    FastDiv lq;        // row of the group -> head of the group
};

template <int N> struct Set { static constexpr int value = N; };

template <typename T> struct Mma16;
template <> struct Mma16<BF16> {
    static __device__ __forceinline__ f32x4 mfma(u32x4 a, u32x4 b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
};
template <> struct Mma16<F16> {
    static __device__ __forceinline__ f32x4 mfma(u32x4 a, u32x4 b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a),
                                                      __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    }
};

// Reductions over the four lanes c, c + 16, c + 32, c + 48 of a query row
__device__ __forceinline__ float quad_max(float x) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return pair_max(fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1])));
}
__device__ __forceinline__ float quad_sum(float x) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return pair_sum(__uint_as_float(a[0]) + __uint_as_float(a[1]));
}

// TL: the state is handed out and the coefficient sums are those of the rounded coefficients, so
// the unrounded sum is carried as well (the Lam handed out is then the true log-sum-exp).
// FP8: 0 K and V in the storage type T, 1 and 2 in fp8; 2 reads K as the operand it is, straight
// from global memory (see launch_decode16_t).  SKIP: leave out the V fetch of blocks whose
// weights have all saturated at 0.
template <typename T, int D, int FP8, bool TL, bool SKIP, int W>
__global__ __launch_bounds__(W * kWave, D == 64 ? 4 : W == 8 ? 2 : 3)
void decode16_kernel(Problem p, Dec16Sched sc) {
    constexpr bool kTL = TL && Mma<T>::kRoundedSum;
    constexpr bool KV8 = FP8 != 0, KDIRECT = FP8 == 2;
    constexpr int NKK = D / 32;                 // score products per 16-key tile
    constexpr int NDB = D / 16;                 // 16-wide blocks of the output
    constexpr int ESZ = KV8 ? 1 : 2;
    constexpr int NV = kD16Block * D * ESZ / 1024;   // 16-byte loads of K or V per lane and block
    constexpr int CPR = D * ESZ / 16;           // 16-byte chunks per key row
    constexpr int kBlockBytes = kD16Block * D * ESZ;
    // LDS rows: 16 rows of a 16-byte read, 8 rows of a transposing read, land on all 64 banks
    constexpr int KROW = D + 8;
    constexpr int VROW = D + 16;
    constexpr int STAGE = kD16Block * VROW;     // elements per wavefront
    constexpr int FROW = D + 4;                 // floats per row of the fold buffer
    constexpr int kLds = 2 * W * STAGE > 4 * W * 16 * FROW
                             ? 2 * W * STAGE : 4 * W * 16 * FROW;
    __shared__ __align__(16) char lds[kLds];
    __shared__ float fold_r[W][16], fold_l[W][16], fold_t[W][16];
    // per row: the largest score any wavefront has seen, a bound of Lam from below (by atomics: the
    // other wavefronts' must be looked at on every block)
    __shared__ float top_seen[SKIP ? 16 : 1];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15;
    const int q = lane >> 4;
    const int sp = blockIdx.x;
    const size_t unit = (size_t)blockIdx.z * p.Hkv + blockIdx.y;        // (b, kv head)
    const float ninf = -__builtin_inff();

    // 32-key blocks of this split; wavefront w takes blk_begin + w, + W, ...  Position 0 sees the
    // fewest keys, position Lq - 1 the most.
    const int nvis_min = visible_at(p, 0);
    const int nvis_max = visible_at(p, p.Lq - 1);
    const int blk_begin = sp * sc.per_split;
    const int blk_end = min((nvis_max + kD16Block - 1) / kD16Block, blk_begin + sc.per_split);
    const char* kg = static_cast<const char*>(p.k) + unit * (size_t)p.Lk * (D * ESZ);
    const char* vg = static_cast<const char*>(p.v) + unit * (size_t)p.Lk * (D * ESZ);
    const int64_t range = (int64_t)min(p.Lk, blk_end * kD16Block) * (D * ESZ);

    u32x4 kreg[NV], vreg[NV];
    auto fetch_k = [&](int blk_) __attribute__((always_inline)) {
        const int64_t at = (int64_t)blk_ * kBlockBytes;
        const auto w = kv_window(kg + at, range - at);
#pragma unroll
        for (int n = 0; n < NV; ++n)
            kreg[n] = kv_load<2>(w, KDIRECT ? (c + 16 * (n & 1)) * (D * ESZ) + 64 * (n >> 1) + 16 * q
                                         : 1024 * n + 16 * lane);
    };
    auto fetch_v = [&](int blk_, bool wanted) __attribute__((always_inline)) {
        const int64_t at = (int64_t)blk_ * kBlockBytes;
        const auto w = kv_window(vg + at, wanted ? range - at : 0);
#pragma unroll
        for (int n = 0; n < NV; ++n) vreg[n] = kv_load<2>(w, 1024 * n + 16 * lane);
    };
    int blk = blk_begin + wave;
    fetch_k(blk);
    if (!SKIP) fetch_v(blk, true);

    // Query row of this lane's column.  Columns past the last row stand in for it (output
    // discarded), so that they never leave the path it takes.
    const bool row_ok = c < sc.nrows;
    const int row = min(c, sc.nrows - 1);
    const size_t row0 = unit * (size_t)sc.nrows;       // the group's rows follow one another
    const uint16_t* qg = static_cast<const uint16_t*>(p.q) + (row0 + row) * D;
    u32x4 qf[NKK];
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk)
        qf[kk] = *reinterpret_cast<const u32x4*>(
            qg + (KDIRECT ? 64 * (kk >> 1) + 16 * q + 8 * (kk & 1) : 32 * kk + 8 * q));
    // a negative scale is taken into Q (exact), so that the largest dot product is the top score
    float c_log2 = (KV8 ? p.scale * p.kscale : p.scale) * kLog2e;
    if (c_log2 < 0.0f) {
        c_log2 = -c_log2;
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk) qf[kk] ^= u32x4{0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u};
    }
    const int pos = row - (int)fast_div((uint32_t)row, sc.lq) * p.Lq;
    const int nvis = visible_at(p, pos);
    if (SKIP) {
        if (tid < 16) top_seen[tid] = ninf;
        __syncthreads();
    }

    uint16_t* vs = reinterpret_cast<uint16_t*>(lds) + wave * STAGE;
    f32x4 U[NDB];
#pragma unroll
    for (int i = 0; i < NDB; ++i) U[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    float R = ninf;                      // -inf: the row has seen no key
    float l = 0.0f, ltrue = 0.0f;        // this lane's keys
    float most = ninf;                   // SKIP: the row's largest score so far
    bool first = true;
    unsigned visited = 0, skipped = 0;   // wavefront-uniform

    // K or V of a block -> this wavefront's LDS stage, which the two take in turn
    auto stage = [&](const u32x4 (&reg)[NV], auto row_elems) __attribute__((always_inline)) {
        constexpr int ROW = decltype(row_elems)::value;
#pragma unroll
        for (int n = 0; n < NV; ++n) {
            const int ch = n * kWave + lane;
            uint16_t* dst = &vs[(ch / CPR) * ROW + (KV8 ? 16 : 8) * (ch % CPR)];
            if constexpr (KV8) {
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
    // U += V^T P^T over the staged block: lanes 4 r .. 4 r + 3 of a 16-lane group address the
    // 8-byte pieces of key row r, lane t receives column t of the four rows
    auto output_product = [&](u32x4 bfrag) __attribute__((always_inline)) {
        const uint16_t* base = &vs[(4 * q + (c >> 2)) * VROW + 4 * (c & 3)];
        typedef s16x4 __attribute__((address_space(3))) * lds_ptr;
#pragma unroll
        for (int i = 0; i < NDB; ++i) {
            const u32x2 lo = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (lds_ptr)(base + 16 * i)));
            const u32x2 hi = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (lds_ptr)(base + 16 * VROW + 16 * i)));
            U[i] = Mma16<T>::mfma(u32x4{lo[0], lo[1], hi[0], hi[1]}, bfrag, U[i]);
        }
        stage_done();
    };

    u32x4 pending_p = {0u, 0u, 0u, 0u};
    bool pending = false;                // SKIP, wavefront-uniform: a V fetch is under way
    for (; blk < blk_end; blk += W) {
        const int j0 = blk * kD16Block;
        // S^T = K Q^T, two 16-key tiles
        if (!KDIRECT) {
            stage(kreg, Set<KROW>{});
            fetch_k(blk + W);
        }
        f32x4 acc[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                u32x4 a;
                if constexpr (!KDIRECT) {
                    a = *reinterpret_cast<const u32x4*>(&vs[(16 * t + c) * KROW + 32 * kk + 8 * q]);
                } else {
                    const u32x4 w = kreg[2 * (kk >> 1) + t];
                    a = (kk & 1) == 0 ? widen8<T>(w[0], w[1]) : widen8<T>(w[2], w[3]);
                }
                acc[t] = Mma16<T>::mfma(a, qf[kk], acc[t]);
            }
        if (KDIRECT) fetch_k(blk + W);
        else stage_done();
        if (!SKIP) {
            stage(vreg, Set<VROW>{});
            fetch_v(blk + W, true);
        } else if (pending) {
            stage(vreg, Set<VROW>{});
            output_product(pending_p);
        }

        // the block's top score per row, then its coefficients
        const bool general = first || j0 + kD16Block > nvis_min;     // keys may be masked, rows empty
        first = false;
        float x[8];
        float top;
        if (general) {
            top = ninf;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                x[e] = acc[e >> 2][e & 3] * c_log2;
                if (j0 + 16 * (e >> 2) + 4 * q + (e & 3) >= nvis) x[e] = ninf;
                top = fmaxf(top, x[e]);
            }
            top = quad_max(top);
        } else {
            top = acc[0][0];
#pragma unroll
            for (int e = 1; e < 8; ++e) top = fmaxf(top, acc[e >> 2][e & 3]);
            top = quad_max(top) * c_log2;
        }
        if (SKIP) {
            // the skip decision, before the exponentials so that V is on its way early
            const float seen = __hip_atomic_load(&top_seen[c], __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_WORKGROUP);
            if (__builtin_amdgcn_ballot_w64(top > most) != 0) {
                most = fmaxf(most, top);
                if (q == 0)
                    __hip_atomic_fetch_max(&top_seen[c], most, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            const float bound = fmaxf(most, seen);
            pending = __builtin_amdgcn_ballot_w64(row_ok && !(top < bound - kSkipMarginLog2)) != 0;
            fetch_v(blk, pending);
            ++visited;
            skipped += pending ? 0u : 1u;
        }
        if (__builtin_amdgcn_ballot_w64(top > R + LazyLimit<T>::kMoveLog2) != 0) {
            const bool move = top > R + LazyLimit<T>::kMoveLog2;
            const float f = move ? exp2_fast(R - top) : 1.0f;        // 0 for a row without keys
            R = move ? top : R;
            l *= f;
            ltrue *= f;
#pragma unroll
            for (int i = 0; i < NDB; ++i) U[i] *= f;
        }
        f32x8 pv;
        // no key yet, or only keys of score -inf: weights of zero
        const float ref = R == ninf ? 0.0f : R;
        if (general) {
#pragma unroll
            for (int e = 0; e < 8; ++e) pv[e] = exp2_fast(x[e] - ref);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) pv[e] = exp2_fast(fmaf(acc[e >> 2][e & 3], c_log2, -ref));
        }
        const u32x4 bfrag = Mma<T>::pack8(pv);
        f32x4 ps = {0.0f, 0.0f, 0.0f, 0.0f};
        Mma<T>::sum8(pv, bfrag, ps);
        l += (ps[0] + ps[1]) + (ps[2] + ps[3]);
        if (kTL)
            ltrue += ((pv[0] + pv[1]) + (pv[2] + pv[3])) + ((pv[4] + pv[5]) + (pv[6] + pv[7]));

        if (SKIP) pending_p = bfrag;
        else output_product(bfrag);
    }
    if (SKIP) {
        if (pending) {
            stage(vreg, Set<VROW>{});
            output_product(pending_p);
        }
        if (p.vskip_counts != nullptr && lane == 0) {
            atomicAdd(p.vskip_counts, (unsigned long long)visited);
            atomicAdd(p.vskip_counts + 1, (unsigned long long)skipped);
        }
    }

    // ---- fold the wavefronts' states ----------------------------------------------------
    l = quad_sum(l);
    if (kTL) ltrue = quad_sum(ltrue);
    __syncthreads();                                   // stages are dead, reuse the LDS
    float* fold = reinterpret_cast<float*>(lds);       // [wave][row][FROW]
#pragma unroll
    for (int i = 0; i < NDB; ++i)
        *reinterpret_cast<f32x4*>(&fold[(wave * 16 + c) * FROW + 16 * i + 4 * q]) = U[i];
    if (q == 0) {
        fold_r[wave][c] = R;
        fold_l[wave][c] = l;
        fold_t[wave][c] = kTL ? ltrue : l;
    }
    __syncthreads();
    const float oscale = KV8 ? p.vscale : 1.0f;
    for (int idx = tid; idx < sc.nrows * (D / 4); idx += W * kWave) {
        const int fr = idx / (D / 4);
        const int t = 4 * (idx % (D / 4));
        float top = fold_r[0][fr];
#pragma unroll
        for (int w = 1; w < W; ++w) top = fmaxf(top, fold_r[w][fr]);
        float lt = 0.0f, tt = 0.0f;
        f32x4 o = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int w = 0; w < W; ++w) {
            // A wavefront without a key of the row is left out: its U holds 0 * V of keys that
            // other rows see, and that is NaN where such a V is infinite.  (l is 1 or more with a
            // key, NaN with a NaN score.  By selection: with a branch around it each wavefront's
            // state is read after the one before.)
            const bool none = fold_l[w][fr] == 0.0f;
            const float f = none ? 0.0f : exp2_fast(fold_r[w][fr] - top);
            const f32x4 u = *reinterpret_cast<const f32x4*>(&fold[(w * 16 + fr) * FROW + t]);
            lt = fmaf(f, fold_l[w][fr], lt);
            tt = fmaf(f, fold_t[w][fr], tt);
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = fmaf(f, none ? 0.0f : u[e], o[e]);
        }
        const bool empty = lt == 0.0f;
        if (!empty) o *= 1.0f / lt * oscale;
        if (!p.partial) {
            *reinterpret_cast<u32x2*>(static_cast<uint16_t*>(p.o) + (row0 + fr) * D + t) =
                Mma<T>::pack4(o);
        } else {
            float* dst = p.ws + ((size_t)sp * p.B * p.Hq * p.Lq + row0 + fr) * (D + 2);
            *reinterpret_cast<float2*>(dst + t) = float2{o[0], o[1]};
            *reinterpret_cast<float2*>(dst + t + 2) = float2{o[2], o[3]};
            if (t == 0) {
                dst[D] = empty ? ninf : (top + log2_fast(tt)) * kLn2;
                dst[D + 1] = 0.0f;
            }
        }
    }
}

template <typename T, int D>
static hipError_t launch_decode16_t(const Problem& p, int mode, hipStream_t st) {
    const dim3 grid((unsigned)p.splits, (unsigned)p.Hkv, (unsigned)p.B), block(4 * kWave);
    Dec16Sched sc;
    sc.nrows = p.Hq / p.Hkv * p.Lq;
    const int blocks = (p.Lk + kD16Block - 1) / kD16Block;
    sc.per_split = (blocks + p.splits - 1) / p.splits;
    sc.lq = make_fast_div((uint32_t)p.Lq);
    // the true log-sum-exp is wanted wherever the state leaves the kernel
    const bool tl = p.partial != 0;
    if (mode == kTileModeLazySkipV && p.kv8) return hipErrorInvalidValue;
    const dim3 eight(8 * kWave);
    if (p.many && p.kv8) {
        hipLaunchKernelGGL((decode16_kernel<T, D, 1, false, false, 8>), grid, eight, 0, st, p, sc);
    } else if (D == 64 && p.many) {
        if (mode == kTileModeLazySkipV) hipLaunchKernelGGL((decode16_kernel<T, 64, 0, false, true, 8>), grid, eight, 0, st, p, sc);
        else hipLaunchKernelGGL((decode16_kernel<T, 64, 0, false, false, 8>), grid, eight, 0, st, p, sc);
    } else if (mode == kTileModeLazySkipV) {
        if (tl) hipLaunchKernelGGL((decode16_kernel<T, D, 0, true, true, 4>), grid, block, 0, st, p, sc);
        else hipLaunchKernelGGL((decode16_kernel<T, D, 0, false, true, 4>), grid, block, 0, st, p, sc);
    } else if (!p.kv8) {
        if (tl) hipLaunchKernelGGL((decode16_kernel<T, D, 0, true, false, 4>), grid, block, 0, st, p, sc);
        else hipLaunchKernelGGL((decode16_kernel<T, D, 0, false, false, 4>), grid, block, 0, st, p, sc);
    } else if ((long)p.splits * p.B * p.Hkv >= 512) {
        if (tl) hipLaunchKernelGGL((decode16_kernel<T, D, 2, true, false, 4>), grid, block, 0, st, p, sc);
        else hipLaunchKernelGGL((decode16_kernel<T, D, 2, false, false, 4>), grid, block, 0, st, p, sc);
    } else {
        if (tl) hipLaunchKernelGGL((decode16_kernel<T, D, 1, true, false, 4>), grid, block, 0, st, p, sc);
        else hipLaunchKernelGGL((decode16_kernel<T, D, 1, false, false, 4>), grid, block, 0, st, p, sc);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !p.merge) return e;
    return launch_merge_splits(p, st);
}

bool decode16_applies(const Problem& p, int mode) {
    return (mode == kTileModeLazy || mode == kTileModeLazySkipV) &&
           (long)(p.Hq / p.Hkv) * p.Lq <= 16;
}

hipError_t launch_decode16(const Problem& p, int mode, hipStream_t st) {
    if (p.dtype == 1 && p.d == 64) return launch_decode16_t<F16, 64>(p, mode, st);
    if (p.dtype == 1 && p.d == 128) return launch_decode16_t<F16, 128>(p, mode, st);
    if (p.dtype == 2 && p.d == 64) return launch_decode16_t<BF16, 64>(p, mode, st);
    if (p.dtype == 2 && p.d == 128) return launch_decode16_t<BF16, 128>(p, mode, st);
    return hipErrorInvalidValue;
}

}  // namespace flashd

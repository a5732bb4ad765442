// Alg. 3 on key tiles for fp32 storage, on the matrix cores: scores in fp64
// (v_mfma_f64_16x16x4), output product in fp32 (v_mfma_f32_16x16x4).  This is what the automatic
// choice runs for fp32; the literal per-key kernel (variant PER_KEY) forms the same scores with
// fp64 fma on the vector ALUs, one key per lane, and was bound by them and by the 128 registers
// of output state that every lane carries (4.4 TFLOP/s).
//
// Precision is that of the per-key kernel: dot products and scaled scores in fp64, weights in
// fp32, l (hence s - ln w) and U in fp64 sums of short fp32 ones (kF32Chain).
//
// Tile form: U = sum_j 2^{s_j - R} v_j and l = sum_j 2^{s_j - R} against a reference R (fp64)
// that starts at the top score of the row's first block and moves only when a block's top score
// lies more than kMoveLog2 above it; o = U / l at the store, Lam = R + log2 l (the deferred
// blend of the f16/bf16 kernels, flashd_mma.h).
//
// Mapping.  A workgroup of 4 wavefronts owns 16 query rows of one kv head and one key range;
// the wavefronts take its 16-key blocks in turn, each with a state of its own, and the four
// states are folded at the end.  The query heads of a kv group are interleaved (row r is
// position r / g of head r % g), so K and V are read once for the group and the causal bounds of
// a row tile stay tight.  Lane (q, c) = (lane / 16, lane % 16) holds of S^T = K Q^T for query row
// c the keys 4 r + q (r = 0..3), which is the B operand of the r-th step of O^T = V^T P^T as it
// stands.  The contraction index of the scores and the column index of the output are permuted so
// that each lane reads K and V as float4 straight from global memory: every wavefront has keys of
// its own, so LDS would hold nothing that is used twice.  K of the next block is requested before
// the output product and V before the scores; the rest of the latency is covered by the other
// wavefronts of the SIMD.
//
// The score product runs as two chains, and for d = 64 Q stays in fp64 for the whole row tile: 3 %
// on causal calls (2 x 12 heads, 777 positions 36.9 -> 35.7 us), 1 % on others.
//
// What bounds it: the matrix cores.  A block of 16 keys x 16 rows x 64 columns takes 16 fp64
// instructions of 64 cycles (78.6 TFLOP/s peak) and 16 fp32 ones of 32 cycles.  On the causal call below they
// are busy 57 % of the time, three wavefronts to a SIMD wait 64 % of theirs to issue, and every compute unit has
// work to the end.  Measured
// against the per-key kernel: 2 x 12 heads, 777 causal positions, d = 64 36 us (425 us before; 52
// TFLOP/s of the 97 that the two kinds of instruction allow together), 4 heads of 1000 positions,
// d = 128 41 us (391), one head of 128 positions 5.5 us of kernel (26).
#include "flashd_common.h"
#include "flashd_kernels.h"
#include "flashd_mma.h"

namespace flashd {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kF32Waves = 4;
constexpr int kF32Rows = 16;       // query rows per workgroup
constexpr int kF32Block = 16;      // keys per wavefront step
constexpr double kMoveLog2 = 8.0;
// Blocks of a wavefront whose sums are formed in fp32; then they join sums in fp64, which lie in
// LDS, each lane's its own.  In fp32 throughout, U and l lose what the per-key kernel keeps, whose
// blend moves o by a part of itself.  Relative error against fp64 on N(0, 1) inputs (2-norm;
// per-key kernel, fp32 throughout, chains of 8, 6 and 4): 300 keys 1.8e-7, 1.8, 1.8, 1.8, 1.6;
// 777 keys 1.9e-7, 2.6, 2.1, 1.9, 1.7; 2048 keys 2.6e-7, 4.0, 2.3, 1.9, 1.7; 131072 keys 1.4e-6,
// 3.3e-6, 2.2e-7, 1.9e-7, 1.7e-7; 524288 equal keys, where every step rounds the same way, 1.8e-7
// and 5.4e-4 in fp32 throughout.  Time of 2 x 12 heads, 777 causal positions, d = 64: 34.8 us in
// fp32 throughout, 35.7, 36.2 and 36.8 in chains; 8 heads of 2048, d = 128: 234, 237, 238, 242.
constexpr int kF32Chain = 6;
// Weights of up to 2^kMoveLog2 per key can overflow the sum over large values (1e36 and up, some
// hundred keys), whose blend would not.  A row tile where that happened is done again with the
// reference this far above the top score: 1e9 keys of 2^(8 - 40) sum to less than a value.
constexpr double kHeadroomLog2 = 40.0;

// How workgroups map to work: id -> (rank of the row tile, split, unit), all units' longest row
// tiles first; unit u on XCD u % 8 where the units divide by 8, so that K and V of a head are
// read into one L2.
struct F32Sched {
    int heads;          // query heads interleaved in a unit: Hq / Hkv (1: not interleaved)
    int rows;           // query rows of a unit: heads * Lq
    int tiles;          // row tiles of a unit
    int nx_log2;        // 3: units are dealt over the XCDs, 0: not
    uint32_t total;     // workgroups of work
    FastDiv per_rank;   // splits * units per XCD
    FastDiv per_split;  // units per XCD
    FastDiv heads_div;
    FastDiv units_per_b;
    FastDiv kv_div;     // unit -> kv unit (Hq / Hkv where the heads are not interleaved, else 1)
};

// x over the four lanes c, c + 16, c + 32, c + 48 of a query row
template <typename S, typename F>
__device__ __forceinline__ S row_reduce(S x, F f) {
    x = f(x, __shfl_xor(x, 16, kWave));
    return f(x, __shfl_xor(x, 32, kWave));
}

template <int D>
__global__ __launch_bounds__(kF32Waves * kWave, D == 64 ? 3 : 2)
void tile_f32_kernel(Problem p, F32Sched sc) {
    constexpr int NM = D / 16;             // float4 of K per lane and block
    constexpr int NB = D / 64;             // 64-column groups of the output
    constexpr int FROW = D + 4;            // floats per row of the fold buffer (16-byte rows)
    constexpr int NV = D / 4;              // sums per lane
    static_assert(NV * kWave * 2 >= kF32Rows * FROW, "a wavefront's fold rows lie in its fp64 sums");
    // a wavefront's fp64 sums, [sum][lane], each lane its own: U, l and the reference they stand
    // at; for the fold its rows in fp32
    __shared__ __align__(16) double sums[kF32Waves][(NV + 2) * kWave];
    __shared__ double fold_r[kF32Waves][kF32Rows];
    __shared__ float fold_l[kF32Waves][kF32Rows];
    __shared__ int over[kF32Waves];        // a sum of the wavefront may overflow in the fold

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15;
    const int q = lane >> 4;
    double* mine = &sums[wave][lane];
    const double ninf = -__builtin_inf();
    const double c_log2 = (double)p.scale * 1.4426950408889634074;

    for (uint32_t id = blockIdx.x; id < sc.total; id += gridDim.x) {
        const uint32_t local = id >> sc.nx_log2;
        const uint32_t rank = fast_div(local, sc.per_rank);
        const uint32_t rem = local - rank * sc.per_rank.d;
        const int sp = (int)fast_div(rem, sc.per_split);
        const uint32_t unit = ((rem - (uint32_t)sp * sc.per_split.d) << sc.nx_log2) +
                              (id & ((1u << sc.nx_log2) - 1u));
        const int tile = p.causal ? sc.tiles - 1 - (int)rank : (int)rank;
        const uint32_t b = fast_div(unit, sc.units_per_b);
        const uint32_t hu = unit - b * sc.units_per_b.d;         // first head: hu * heads
        const size_t kv_unit = fast_div(unit, sc.kv_div);

        // row r of the unit -> row of [B][Hq][Lq], and its query position
        auto position = [&](int r) { return (int)fast_div((uint32_t)r, sc.heads_div); };
        auto q_row = [&](int r) {
            const int pos = position(r);
            const int head = (int)hu * sc.heads + (r - pos * sc.heads);
            return ((size_t)b * p.Hq + head) * (size_t)p.Lq + pos;
        };
        auto visible = [&](int pos) {
            return p.causal ? min(max(pos + p.shift + 1, 0), p.Lk) : p.Lk;
        };

        const int r0 = tile * kF32Rows;
        const int rlast = min(r0 + kF32Rows, sc.rows) - 1;
        // rows past the end stand in for the last one and are not stored
        const int row = min(r0 + c, rlast);
        const int nvis = visible(position(row));
        const int nvis_min = visible(position(r0));
        const int nvis_max = visible(position(rlast));
        const int nblk_all = (p.Lk + kF32Block - 1) / kF32Block;
        const int chunk = (nblk_all + p.splits - 1) / p.splits;
        const int blk_end = min((nvis_max + kF32Block - 1) / kF32Block, (sp + 1) * chunk);

        const float* kg = static_cast<const float*>(p.k) + kv_unit * (size_t)p.Lk * D + 4 * q;
        const float* vg = static_cast<const float*>(p.v) + kv_unit * (size_t)p.Lk * D + 4 * c;
        f32x4 qf[NM], kf[NM];
        // d = 64: Q in fp64 for the whole row tile (for d = 128 that would take 64 registers)
        double qd[D == 64 ? NM : 1][4];
        auto fetch_k = [&](int blk) __attribute__((always_inline)) {
            const float* src = kg + (size_t)min(blk * kF32Block + c, p.Lk - 1) * D;
#pragma unroll
            for (int m = 0; m < NM; ++m) kf[m] = *reinterpret_cast<const f32x4*>(src + 16 * m);
        };

        for (int pass = 0;; ++pass) {
            const double head = pass == 0 ? 0.0 : kHeadroomLog2;
            const double limit = pass == 0 ? kMoveLog2 : kMoveLog2 - kHeadroomLog2;
            f32x4 U[NB][4];                    // [column group][n]: columns 64 i + 16 q + 4 e + n
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int n = 0; n < 4; ++n) U[i][n] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            float l = 0.0f;                    // this lane's keys
            double R = ninf;
            int done = 0;                      // blocks of this wavefront
            // what brings the fp64 sums to the present reference
            auto to_reference = [&]() __attribute__((always_inline)) {
                const double R64 = mine[(NV + 1) * kWave];
                return R64 == R ? 1.0 : (double)exp2_fast((float)(R64 - R));
            };

            int blk = sp * chunk + wave;
            if (blk < blk_end) {
                fetch_k(blk);
                // (the address is formed anew for each pass: kept, it would cost two registers)
                int col = c;
                asm volatile("" : "+v"(col));
                const float* qg = static_cast<const float*>(p.q) +
                                  q_row(min(r0 + col, rlast)) * D + 4 * q;
#pragma unroll
                for (int m = 0; m < NM; ++m) qf[m] = *reinterpret_cast<const f32x4*>(qg + 16 * m);
                if constexpr (D == 64) {
#pragma unroll
                    for (int m = 0; m < NM; ++m)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            qd[m][e] = (double)qf[m][e];
                            asm volatile("" : "+v"(qd[m][e]));
                        }
                }
            }
            for (; blk < blk_end; blk += kF32Waves) {
                const int j0 = blk * kF32Block;
                f32x4 vf[NB][4];           // [column group][r]: key 4 r + q, columns 64 i + 4 c ..
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float* src = vg + (size_t)min(j0 + 4 * r + q, p.Lk - 1) * D;
#pragma unroll
                    for (int i = 0; i < NB; ++i)
                        vf[i][r] = *reinterpret_cast<const f32x4*>(src + 64 * i);
                }
                f64x4 acc2[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll
                for (int m = 0; m < NM; ++m) {
                    // d = 128: widen Q anew for every block
                    if (D == 128) asm volatile("" : "+v"(qf[m]));
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc2[e & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                            (double)kf[m][e], D == 64 ? qd[D == 64 ? m : 0][e] : (double)qf[m][e], acc2[e & 1], 0, 0, 0);
                }
                const f64x4 acc = acc2[0] + acc2[1];
                if (blk + kF32Waves < blk_end) fetch_k(blk + kF32Waves);

                const bool masked = j0 + kF32Block > nvis_min;
                double x[4];
                double top = ninf;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    x[r] = acc[r] * c_log2;
                    if (masked && j0 + 4 * r + q >= nvis) x[r] = ninf;
                    top = fmax(top, x[r]);
                }
                if (__builtin_amdgcn_ballot_w64(top > R + limit) != 0) {
                    top = row_reduce(top, [](double a, double bb) { return fmax(a, bb); });
                    if (top > R + limit) {
                        // 0 for a row without keys
                        const float f = exp2_fast((float)(R - head - top));
                        l *= f;
#pragma unroll
                        for (int i = 0; i < NB; ++i)
#pragma unroll
                            for (int n = 0; n < 4; ++n) U[i][n] *= f;
                        R = top + head;
                    }
                }
                float pw[4];
                // no key yet, or only keys of score -inf: weights of zero
                const double ref = R == ninf ? 0.0 : R;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    pw[r] = exp2_fast((float)(x[r] - ref));
                    l += pw[r];
                }
                bool plain = true;
                if (masked) {
                    // a weight of zero does not silence an infinite or NaN value of a hidden key
                    float bad = 0.0f;
#pragma unroll
                    for (int i = 0; i < NB; ++i)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
#pragma unroll
                            for (int e = 0; e < 4; ++e) bad = fmaf(vf[i][r][e], 0.0f, bad);
                    plain = __builtin_amdgcn_ballot_w64(bad != 0.0f) == 0;
                }
                if (plain) {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int i = 0; i < NB; ++i)
#pragma unroll
                            for (int n = 0; n < 4; ++n)
                                U[i][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[i][r][n], pw[r],
                                                                               U[i][n], 0, 0, 0);
                } else {
#pragma unroll 1
                    for (int kk = 0; kk < kF32Block; ++kk) {
                        const float own = (kk >> 2) == 0 ? pw[0] : (kk >> 2) == 1 ? pw[1]
                                          : (kk >> 2) == 2 ? pw[2] : pw[3];
                        const float w = __shfl(own, (kk & 3) * 16 + c, kWave);
                        if (j0 + kk < nvis) {
                            const float* src = vg - 4 * c + (size_t)(j0 + kk) * D + 16 * q;
#pragma unroll
                            for (int i = 0; i < NB; ++i)
#pragma unroll
                                for (int e = 0; e < 4; ++e)
#pragma unroll
                                    for (int n = 0; n < 4; ++n)
                                        U[i][n][e] = fmaf(w, src[64 * i + 4 * e + n], U[i][n][e]);
                        }
                    }
                }
                if (__builtin_expect(++done % kF32Chain == 0, 0)) {
                    if (done == kF32Chain) {
                        mine[NV * kWave] = (double)l;
#pragma unroll
                        for (int at = 0; at < NV; ++at)
                            mine[at * kWave] = (double)U[at / 16][(at / 4) % 4][at % 4];
                    } else {
                        const double f = to_reference();
                        mine[NV * kWave] = fma(mine[NV * kWave], f, (double)l);
#pragma unroll
                        for (int at = 0; at < NV; ++at)
                            mine[at * kWave] =
                                fma(mine[at * kWave], f, (double)U[at / 16][(at / 4) % 4][at % 4]);
                    }
                    mine[(NV + 1) * kWave] = R;
                    l = 0.0f;
#pragma unroll
                    for (int at = 0; at < NV; ++at) U[at / 16][(at / 4) % 4][at % 4] = 0.0f;
                }
            }
            double l64 = (double)l;
            if (done >= kF32Chain) {
                const double f = to_reference();
                l64 = fma(mine[NV * kWave], f, l64);
#pragma unroll
                for (int at = 0; at < NV; ++at) {
                    const double u = fma(mine[at * kWave], f, (double)U[at / 16][(at / 4) % 4][at % 4]);
                    U[at / 16][(at / 4) % 4][at % 4] = (float)u;
                }
            }

            // ---- fold the four wavefront states ----------------------------------------
            float bad = 0.0f;                  // NaN where four such sums might overflow
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int n = 0; n < 4; ++n)
#pragma unroll
                    for (int e = 0; e < 4; ++e) bad = fmaf(U[i][n][e] * 4.0f, 0.0f, bad);
            const bool big = __builtin_amdgcn_ballot_w64(bad != 0.0f) != 0;
            l = row_reduce((float)l64, [](float a, float bb) { return a + bb; });
            __syncthreads();                   // the previous fold has been read
            float* rows = reinterpret_cast<float*>(sums[wave]);
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    *reinterpret_cast<f32x4*>(&rows[c * FROW + 64 * i + 16 * q + 4 * e]) =
                        f32x4{U[i][0][e], U[i][1][e], U[i][2][e], U[i][3][e]};
            if (q == 0) {
                fold_r[wave][c] = R;
                fold_l[wave][c] = l;
            }
            if (lane == 0) over[wave] = big ? 1 : 0;
            __syncthreads();
            if (pass == 0 && (over[0] | over[1] | over[2] | over[3]) != 0) continue;
            for (int idx = tid; idx < kF32Rows * (D / 4); idx += kF32Waves * kWave) {
                const int fr = idx / (D / 4);
                const int t = 4 * (idx % (D / 4));
                if (r0 + fr > rlast) continue;
                double top = ninf;
#pragma unroll
                for (int w = 0; w < kF32Waves; ++w) top = fmax(top, fold_r[w][fr]);
                float lt = 0.0f;
                f32x4 o = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int w = 0; w < kF32Waves; ++w) {
                    const float lw = fold_l[w][fr];
                    // a wavefront that saw no key: weight 0 (NaN stays NaN)
                    const float f = fold_r[w][fr] == ninf ? lw * 0.0f
                                                          : exp2_fast((float)(fold_r[w][fr] - top));
                    lt = fmaf(f, lw, lt);
                    o += f * *reinterpret_cast<const f32x4*>(
                                 reinterpret_cast<const float*>(sums[w]) + fr * FROW + t);
                }
                const bool empty = lt == 0.0f;
                const float inv = empty ? 0.0f : 1.0f / lt;
                o *= inv;
                const size_t orow = q_row(r0 + fr);
                if (!p.partial) {
                    *reinterpret_cast<f32x4*>(static_cast<float*>(p.o) + orow * D + t) = o;
                } else {
                    float* dst = p.ws + ((size_t)sp * p.B * p.Hq * p.Lq + orow) * (D + 2);
                    *reinterpret_cast<float2*>(dst + t) = float2{o[0], o[1]};
                    *reinterpret_cast<float2*>(dst + t + 2) = float2{o[2], o[3]};
                    if (t == 0)
                        split_lam(empty ? ninf : (top + log2((double)lt)) * 0.69314718055994530942,
                                  dst[D], dst[D + 1]);
                }
            }
            break;
        }
        if (id + gridDim.x < sc.total) __syncthreads();   // the fold has been read, sums is free
    }
}

template <int D>
static hipError_t launch_tile_f32_t(const Problem& p, hipStream_t st) {
    F32Sched sc;
    const int g = p.Hq / p.Hkv;
    // rows of a unit are 32-bit; beyond that the heads run one by one
    sc.heads = (long)g * p.Lq < (1L << 30) ? g : 1;
    sc.rows = sc.heads * p.Lq;
    sc.tiles = (sc.rows + kF32Rows - 1) / kF32Rows;
    const long units = (long)p.B * (p.Hq / sc.heads);
    const long total = units * sc.tiles * p.splits;
    if (total > 0x7fffffffL) return hipErrorInvalidValue;
    sc.nx_log2 = units % 8 == 0 ? 3 : 0;
    sc.total = (uint32_t)total;
    sc.per_rank = make_fast_div((uint32_t)((units >> sc.nx_log2) * p.splits));
    sc.per_split = make_fast_div((uint32_t)(units >> sc.nx_log2));
    sc.heads_div = make_fast_div((uint32_t)sc.heads);
    sc.units_per_b = make_fast_div((uint32_t)(p.Hq / sc.heads));
    sc.kv_div = make_fast_div((uint32_t)(sc.heads == g ? 1 : g));
    const unsigned grid = (unsigned)(total < (1L << 22) ? total : (1L << 22));
    hipLaunchKernelGGL((tile_f32_kernel<D>), dim3(grid), dim3(kF32Waves * kWave), 0, st, p, sc);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !p.merge) return e;
    return launch_merge_splits(p, st);
}

hipError_t launch_tile_f32(const Problem& p, hipStream_t st) {
    if (p.dtype != 0) return hipErrorInvalidValue;
    if (p.d == 64) return launch_tile_f32_t<64>(p, st);
    if (p.d == 128) return launch_tile_f32_t<128>(p, st);
    return hipErrorInvalidValue;
}

}  // namespace flashd

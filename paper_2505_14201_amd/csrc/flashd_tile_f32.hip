// Alg. 3 on key tiles for fp32 storage, on the matrix cores: scores beyond fp32 precision, output
// product in fp32 (v_mfma_f32_16x16x4).  This is what the automatic choice runs for fp32; the
// literal per-key kernel (variant PER_KEY) forms its scores with fp64 fma on the vector ALUs, one
// key per lane, and was bound by them and by the 128 registers of output state that every lane
// carries (4.4 TFLOP/s).
//
// Weights are fp32, l (hence s - ln w) and U fp64 sums of short fp32 ones (kF32Chain); scores are fp64 or, up to a
// size (kSliceScore), sums of fp16 slices whose error is below that of an fp32 weight.  The output is then as far
// from fp64 as with fp64 scores throughout.
//
// Tile form: U = sum_j 2^{s_j - R} v_j and l = sum_j 2^{s_j - R} against a reference R (fp64)
// that starts at the top score of the row's first block and moves only when a block's top score
// lies more than kMoveLog2 above it; o = U / l at the store, Lam = R + log2 l (the deferred
// blend of the f16/bf16 kernels, flashd_mma.h).
//
// Mapping.  A workgroup of 4 wavefronts owns 16 query rows of one kv head and one key range;
// the wavefronts take its 16-key blocks in turn, each with a state of its own, and the four
// states are folded at the end.  The query heads of a kv group are interleaved (row r is position
// r / g of head r % g), so K and V are read once for the group and the causal bounds of a row tile
// stay tight.  Lane (q, c) = (lane / 16, lane % 16) holds of S^T = K Q^T for query row c the keys
// 4 q + r (r = 0..3), the r-th of which is the B operand of the r-th step of O^T = V^T P^T as it
// stands.  The contraction index of the scores and the column index of the output are permuted so
// that each lane reads K and V as float4 straight from global memory: every wavefront has keys of
// its own, so LDS would hold nothing that is used twice.  K of the next block is requested before
// the output product and V before the scores; the rest of the latency is covered by the other
// wavefronts of the SIMD.
//
// Scores, two ways (SLICED, sliced_scores()):
//   - fp64, v_mfma_f64_16x16x4: 16 instructions of 64 cycles for 16 keys x 16 rows x 64 columns, as
//     two chains, Q widened once for d = 64.
//   - sliced (the splitting of a product into short exact ones of Ozaki, Ogita, Oishi and Rump): a row of Q or K, scaled
//     by a power of two to at most 2^kSliceLog2, is the sum of three fp16 values per element (slice8), and six
//     products of slices, v_mfma_f32_16x16x32_f16, give the score.  The product of the leading slices is one of
//     integers and exact in fp32, 64 columns at a time; it and the sum of the others, 2^-10 of its size, are joined
//     in fp64.  12 instructions of 16 cycles and 110 vector instructions in place of 1024 cycles and 20.
//     What is left out of a column is at most 1.25 x 2^-31 of the product of the largest elements of both rows,
//     whatever the score: an element that meets a zero counts as well.  So a wavefront goes over to fp64, for the
//     rest of its keys, at the first block where |scale| log2(e) times the bound on that product exceeds
//     kSliceScore, or whose rows do not lend themselves to slices (infinities, exponents more than kSliceSpan
//     apart or beyond kSliceMin, kSliceMax).  Up to kSliceScore = 24 the error of a
//     score is 1.5e-8 (log2 units, rms; at most 9e-7 at d = 64), less than the rounding of a weight.  Error of the output against fp64, 2-norm, sliced and in fp64:
//     2 x 12 heads of 777 causal positions, d = 64 1.23e-7 both, at standard deviation 2 1.69e-7 both; 8 heads of
//     2048, d = 128 2.03e-7 both; 4 heads of 1000 1.93e-7 both.  Standard scale and N(0, 1) inputs reach 12 at
//     most; standard deviation 4 is beyond it.
//   The two are loops of their own, so that each keeps its operands in registers and no more.
//
// What bounds it: vector and matrix instructions, which hardly overlap.  Sliced, d = 64, a block takes a
// wavefront 250 vector instructions of 4 cycles and 704 cycles of the matrix pipe (512 of them the fp32 output
// product); 16 heads of 2048 causal positions run at the sum of the two.  Tried on it
// and not kept: two groups of 16 rows on the same sliced K (two wavefronts per SIMD and not three: 102 us against
// 98), V requested a block ahead (level), a raised wavefront priority for the longer row tiles (level), scores
// against R in pairs of fp32 in place of fp64 (level, and 2 % more error).
// Measured (us; in fp64, sliced, and where Q and K of standard deviation 4 send every block to fp64 from there): 2 x
// 12 heads, 777 causal positions, d = 64 34.9, 30.1, 41.7 (per-key kernel 425); 16 of 2048 125, 95.6, 135; 4 of 1000,
// d = 128, no mask 41.2, 34.5, 47.3; 8 of 2048 241, 174, 252; 16 of 1200, causal 97.0, 74.2, 107.
#include "flashd_common.h"
#include "flashd_kernels.h"
#include "flashd_mma.h"

#include <algorithm>

namespace flashd {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int kF32Waves = 4;
constexpr int kF32Rows = 16;       // query rows per workgroup
constexpr int kF32Block = 16;      // keys per wavefront step
constexpr double kMoveLog2 = 8.0;
// Rows of Q and K are scaled to below 2^kSliceLog2 in size before they are sliced (64 products of
// integers of that size add up to at most 2^24), K by one power of two for all rows of a block, whose
// largest elements lie within kSliceSpan powers of two of it.
constexpr int kSliceLog2 = 9, kSliceSpan = 8;
constexpr float kSliceMin = 0x1p-100f, kSliceMax = 0x1p100f;
// Largest |scale| log2(e) 2^(eq + ek) that is sliced, 2^eq and 2^ek the powers of two above the largest elements of
// the query row and of the K rows.  Without a limit the output is 0.5 % further from fp64 at standard deviation 4
// and 60 % at 16, and where one column of K is 2^10 and Q zero there the error is 12 times that of fp64 scores
// (one of 2^20 1300 times).
constexpr float kSliceScore = 24.0f;
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

// Eight fp32 values, scaled by sc to at most 2^kSliceLog2 in size, as the sum of three fp16 values
// each: the nearest integer, the rest rounded to 11 bits and what is left then; the remainder is at
// most 2^-25.  (The matrix instructions take fp16 values below 2^-14 as they are.)
struct Sliced {
    f16x8 s1, s2, s3;
};
__device__ __forceinline__ Sliced slice8(f32x4 lo, f32x4 hi, float sc) {
    uint32_t w1[4], w2[4], w3[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float ta = (i < 2 ? lo[2 * i] : hi[2 * i - 4]) * sc;
        const float tb = (i < 2 ? lo[2 * i + 1] : hi[2 * i - 3]) * sc;
        const float na = __builtin_rintf(ta), nb = __builtin_rintf(tb);
        const float ra = ta - na, rb = tb - nb;
        const f16x2 h2 = __builtin_convertvector(f32x2{ra, rb}, f16x2);
        w1[i] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(na, nb));
        w2[i] = __builtin_bit_cast(uint32_t, h2);
        w3[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(
                    f32x2{fmaf((float)h2[0], -1.0f, ra), fmaf((float)h2[1], -1.0f, rb)}, f16x2));
    }
    return {__builtin_bit_cast(f16x8, u32x4{w1[0], w1[1], w1[2], w1[3]}),
            __builtin_bit_cast(f16x8, u32x4{w2[0], w2[1], w2[2], w2[3]}),
            __builtin_bit_cast(f16x8, u32x4{w3[0], w3[1], w3[2], w3[3]})};
}

// The largest of a value over the four lanes c, c + 16, c + 32, c + 48, in all of them
__device__ __forceinline__ float quad_max(float x) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
// hi and lo joined with those of the lane N further round its row of 16
template <int N> __device__ __forceinline__ void turn16(float& hi, float& lo) {
    hi = fmaxf(hi, __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(hi), 0x120 + N, 0xf, 0xf, true)));
    lo = fminf(lo, __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(lo), 0x120 + N, 0xf, 0xf, true)));
}
template <int N> __device__ __forceinline__ float largest(const f32x4 (&x)[N]) {
    float m = 0.0f;
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) m = fmaxf(m, fabsf(x[i][e]));
    return quad_max(m);
}
__device__ __forceinline__ f32x4 mfma16(f16x8 a, f16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ bool sliceable(float a) { return a == 0.0f || (a >= kSliceMin && a < kSliceMax); }
// 2^n, n in -126 .. 127
__device__ __forceinline__ float power_of_two(int n) { return __uint_as_float((uint32_t)(127 + n) << 23); }

// x over the four lanes c, c + 16, c + 32, c + 48 of a query row
template <typename S, typename F>
__device__ __forceinline__ S row_reduce(S x, F f) {
    x = f(x, __shfl_xor(x, 16, kWave));
    return f(x, __shfl_xor(x, 32, kWave));
}

// log2.  CALLED: by a function call.  Inlined, the constants of the logarithm sit in registers from the
// start of the kernel on, also where no partial states are written; with slices that takes scratch
// memory, whose set-up costs every launch 0.7 us.  The call costs one that writes them 0.3 us.
__device__ __attribute__((noinline)) double log2_called(double x) { return log2(x); }
template <bool CALLED> __device__ __forceinline__ double log2_of(double x) {
    if constexpr (CALLED) return log2_called(x);
    return log2(x);
}

// SLICED: scores from fp16 slices, else in fp64.
template <int D, bool SLICED>
__global__ __launch_bounds__(kF32Waves * kWave, D == 64 ? 3 : 2)
void tile_f32_kernel(Problem p, F32Sched sc) {
    constexpr int NM = D / 16;             // float4 of K per lane and block
    constexpr int NK = D / 32;             // steps of the score product, sliced
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
    const float reach = (float)fabs(c_log2);

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

        const float* kg = static_cast<const float*>(p.k) + kv_unit * (size_t)p.Lk * D;
        const float* vg = static_cast<const float*>(p.v) + kv_unit * (size_t)p.Lk * D;
        f32x4 kf[NM], vf[NB][4];           // V: [column group][r], key 4 q + r, columns 64 i + 4 c ..
        // Operand row c of the score product.  In fp64 its output row 4 r + q lies in register r of the
        // lanes q, otherwise row 4 q + r: either way the scores of key 4 q + r end up there.
        int krow = 4 * (c & 3) + (c >> 2);
        // (a scalar base and a 32-bit offset per lane)
        auto fetch_k = [&](int blk) __attribute__((always_inline)) {
            const char* base = reinterpret_cast<const char*>(kg + (size_t)blk * kF32Block * D);
            const uint32_t off = (uint32_t)min(krow, p.Lk - 1 - blk * kF32Block) * (4 * D) + 16 * q;
#pragma unroll
            for (int m = 0; m < NM; ++m) kf[m] = *reinterpret_cast<const f32x4*>(base + off + 64 * m);
        };
        auto fetch_v = [&](int blk) __attribute__((always_inline)) {
            const char* base = reinterpret_cast<const char*>(vg + (size_t)blk * kF32Block * D);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t off = (uint32_t)min(4 * q + r, p.Lk - 1 - blk * kF32Block) * (4 * D) + 16 * c;
#pragma unroll
                for (int i = 0; i < NB; ++i) vf[i][r] = *reinterpret_cast<const f32x4*>(base + off + 256 * i);
            }
        };
        auto fetch_q = [&](f32x4 (&x)[NM]) __attribute__((always_inline)) {
            // (the address is formed anew each time: kept, it would cost two registers)
            int col = c, grp = q;
            asm volatile("" : "+v"(col), "+v"(grp));
            const float* qg = static_cast<const float*>(p.q) + q_row(min(r0 + col, rlast)) * D + 4 * grp;
#pragma unroll
            for (int m = 0; m < NM; ++m) x[m] = *reinterpret_cast<const f32x4*>(qg + 16 * m);
        };

        for (int pass = 0;; ++pass) {
            const double head = pass == 0 ? 0.0 : kHeadroomLog2;
            const double limit = pass == 0 ? kMoveLog2 : kMoveLog2 - kHeadroomLog2;
            f32x4 U[NB][4];                    // [column group][n]: columns 64 i + 16 q + 4 e + n
            float l = 0.0f;                    // this lane's keys
            double R = ninf;
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int n = 0; n < 4; ++n) U[i][n] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            int done = 0;                      // blocks of this wavefront
            // what brings the fp64 sums to the present reference
            auto to_reference = [&]() __attribute__((always_inline)) {
                const double R64 = mine[(NV + 1) * kWave];
                return R64 == R ? 1.0 : (double)exp2_fast((float)(R64 - R));
            };

            int blk = sp * chunk + wave;
            // What follows the scores of a block (log2 units; x[r]: key 4 q + r)
            auto take = [&](f64x4 x) __attribute__((always_inline)) {
                const int j0 = blk * kF32Block;
                if (blk + kF32Waves < blk_end) fetch_k(blk + kF32Waves);

                const bool masked = j0 + kF32Block > nvis_min;
                double top = ninf;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if (masked && j0 + 4 * q + r >= nvis) x[r] = ninf;
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
                        const float own = (kk & 3) == 0 ? pw[0] : (kk & 3) == 1 ? pw[1]
                                          : (kk & 3) == 2 ? pw[2] : pw[3];
                        const float w = __shfl(own, (kk >> 2) * 16 + c, kWave);
                        if (j0 + kk < nvis) {
                            const float* src = vg + (size_t)(j0 + kk) * D + 16 * q;
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
                        for (int at = 0; at < NV; ++at) {
                            mine[at * kWave] =
                                fma(mine[at * kWave], f, (double)U[at / 16][(at / 4) % 4][at % 4]);
                            if (SLICED && at % 4 == 3) __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                    mine[(NV + 1) * kWave] = R;
                    l = 0.0f;
#pragma unroll
                    for (int at = 0; at < NV; ++at) U[at / 16][(at / 4) % 4][at % 4] = 0.0f;
                }
            };
            if (SLICED) krow = c;
            if (blk < blk_end) fetch_k(blk);

            // ---- scores from slices, up to the first block that needs fp64
            if constexpr (SLICED) {
                if (blk < blk_end) {
                    // Q, each row scaled by the exponent of its largest element, and that exponent
                    f32x4 xq[NM];
                    fetch_q(xq);
                    const float qmax = largest(xq);
                    const int eq = __builtin_amdgcn_frexp_expf(qmax);
                    Sliced qs[NK];
#pragma unroll
                    for (int i = 0; i < NK; ++i)
                        qs[i] = slice8(xq[2 * i], xq[2 * i + 1], power_of_two(kSliceLog2 - eq));
                    bool far = __builtin_amdgcn_ballot_w64(!sliceable(qmax)) != 0;
                    int ek = 0;                        // exponent that K is sliced by (rows below 2^ek)
                    uint32_t klo = 0x80000000u;        // bits of 2^(ek - kSliceSpan); at first no row is in range
#pragma unroll 1
                    for (; !far && blk < blk_end; blk += far ? 0 : kF32Waves) {
                        fetch_v(blk);
                        const float kmax = largest(kf);
                        if (__builtin_amdgcn_ballot_w64(__float_as_uint(kmax) - klo >= (uint32_t)kSliceSpan << 23) != 0) {
                            // the first block, or rows outside the range that K is sliced by
                            float hi = kmax, lo = kmax == 0.0f ? kSliceMax : kmax;
                            turn16<8>(hi, lo); turn16<4>(hi, lo); turn16<2>(hi, lo); turn16<1>(hi, lo);
                            ek = __builtin_amdgcn_readfirstlane(__builtin_amdgcn_frexp_expf(hi));
                            klo = (uint32_t)(127 + ek - kSliceSpan) << 23;
                            const bool fits = hi == 0.0f || (sliceable(hi) && sliceable(lo) &&
                                                             __builtin_amdgcn_frexp_expf(lo) > ek - kSliceSpan);
                            const bool close = __builtin_amdgcn_ldexpf(reach, eq + ek) <= kSliceScore;
                            far = __builtin_amdgcn_ballot_w64(!fits || !close) != 0;
                        }
                        if (__builtin_expect(!far, 1)) {
                            const float s = power_of_two(kSliceLog2 - ek);
                            const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
                            f32x4 whole[NB], rest, rest2;      // whole: 64 columns each, exact
#pragma unroll
                            for (int i = 0; i < NK; ++i) {
                                const Sliced ks = slice8(kf[2 * i], kf[2 * i + 1], s);
                                whole[i / 2] = mfma16(ks.s1, qs[i].s1, i % 2 == 0 ? zero : whole[i / 2]);
                                rest = mfma16(ks.s1, qs[i].s2, i == 0 ? zero : rest);
                                rest2 = mfma16(ks.s2, qs[i].s1, i == 0 ? zero : rest2);
                                rest = mfma16(ks.s1, qs[i].s3, rest);
                                rest2 = mfma16(ks.s2, qs[i].s2, rest2);
                                rest = mfma16(ks.s3, qs[i].s1, rest);
                                __builtin_amdgcn_sched_barrier(0);
                            }
                            const double cs = __builtin_amdgcn_ldexp(c_log2, eq + ek - 2 * kSliceLog2);
                            f64x4 x;
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                x[r] = (double)whole[0][r] + (double)(rest[r] + rest2[r]);
                                if (NB == 2) x[r] += (double)whole[NB - 1][r];
                                x[r] *= cs;
                            }
                            take(x);
                        }
                    }
                    if (blk < blk_end) {
                        // (opaque, so that nothing of the loop above is kept for the one below)
                        int col = c;
                        asm volatile("" : "+v"(col), "+s"(blk));
                        krow = 4 * (col & 3) + (col >> 2);
                        fetch_k(blk);
                    }
                }
            }

            // ---- scores in fp64
            if (blk < blk_end) {
                // Q, for d = 64 widened once (for d = 128 that would take 64 registers)
                f32x4 qf[NM];
                double qd[D == 64 ? NM : 1][4];
                fetch_q(qf);
                if constexpr (D == 64) {
#pragma unroll
                    for (int m = 0; m < NM; ++m)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            qd[m][e] = (double)qf[m][e];
                            asm volatile("" : "+v"(qd[m][e]));
                        }
                }
                for (; blk < blk_end; blk += kF32Waves) {
                    fetch_v(blk);
                    f64x4 acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll
                    for (int m = 0; m < NM; ++m) {
                        // d = 128: widen Q anew for every block
                        if (D == 128) asm volatile("" : "+v"(qf[m]));
                        // (four registers in turn: one alone would be written only once the product before has read it)
                        double kd[4] = {(double)kf[m][0], (double)kf[m][1], (double)kf[m][2], (double)kf[m][3]};
                        asm volatile("" : "+v"(kd[0]), "+v"(kd[1]), "+v"(kd[2]), "+v"(kd[3]));
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            acc[e & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                                kd[e], D == 64 ? qd[D == 64 ? m : 0][e] : (double)qf[m][e], acc[e & 1], 0, 0, 0);
                    }
                    take((acc[0] + acc[1]) * c_log2);
                }
            }

            // ---- fold the four wavefront states ----------------------------------------
            float bad = 0.0f;                  // NaN where four such sums might overflow
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
#pragma unroll
            for (int at = 0; at < NV; ++at)
                bad = fmaf(U[at / 16][(at / 4) % 4][at % 4] * 4.0f, 0.0f, bad);
            l = row_reduce((float)l64, [](float a, float bb) { return a + bb; });
            const bool big = __builtin_amdgcn_ballot_w64(bad != 0.0f) != 0;
            __syncthreads();                   // the previous fold has been read
            float* rows = reinterpret_cast<float*>(sums[wave]);
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    *reinterpret_cast<f32x4*>(&rows[(c) * FROW + 64 * i + 16 * q + 4 * e]) =
                        f32x4{U[i][0][e], U[i][1][e], U[i][2][e], U[i][3][e]};
            if (q == 0) {
                fold_r[wave][c] = R;
                fold_l[wave][c] = l;
            }
            if (lane == 0) over[wave] = big ? 1 : 0;
            __syncthreads();
            if (pass == 0 && (over[0] | over[1] | over[2] | over[3]) != 0) continue;
            // (the thread's index afresh: the addresses below are formed here and not kept)
            int tid_now = tid;
            asm volatile("" : "+v"(tid_now));
            for (int idx = tid_now; idx < kF32Rows * (D / 4); idx += kF32Waves * kWave) {
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
                        split_lam(empty ? ninf : (top + log2_of<SLICED>((double)lt)) * 0.69314718055994530942,
                                  dst[D], dst[D + 1]);
                }
            }
            break;
        }
        if (id + gridDim.x < sc.total) __syncthreads();   // the fold has been read, sums is free
    }
}

// Where the scores are formed from slices (120 shapes of 4, 24 and 96 heads, 64 to 512 positions and short
// queries over 600 to 2000 keys; time sliced over time in fp64).  Slicing Q and the first block of K costs
// a wavefront some 0.4 us, a block then saves 0.2 at d = 64 and 0.45 at d = 128.
//   d = 128: from more than 128 keys per split on 0.80 to 0.97; 128 keys 0.95 to 1.01, 64 1.02 to 1.06.
//   d = 64: where compute units have more than one workgroup and more than 160 keys 0.82 to 0.99; with
//   a workgroup each at most, whose wavefronts wait for memory and not for the matrix cores, 0.95 to 1.015, not
//   worth the detour of a call whose scores end in fp64 after all; 160 keys 0.94 to 1.02, 64 1.05 to 1.07.
static bool sliced_scores(const Problem& p, long workgroups) {
    const long blocks = (p.Lk + kF32Block - 1L) / kF32Block;
    const long most = p.causal ? std::min((long)p.Lk, (long)p.Lq + p.shift) : (long)p.Lk;
    const long keys = std::min((blocks + p.splits - 1) / p.splits * kF32Block, most);
    return p.d == 128 ? keys > 128 : keys > 160 && workgroups > 256;
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
    const auto kernel = sliced_scores(p, total) ? tile_f32_kernel<D, true> : tile_f32_kernel<D, false>;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kF32Waves * kWave), 0, st, p, sc);
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

// Which kernel a small call runs on: the rules of the automatic choice that look at nothing but sizes
// (host code without HIP, so that a test can compile it by itself).
#pragma once

#include <algorithm>
#include <cmath>

namespace flashd {

struct Shape { int B, Hq, Hkv, Lq, Lk, d, dtype; };

inline int ceil_div(long a, long b) { return (int)((a + b - 1) / b); }

// Decode calls of up to 16 rows per kv head that the rule for splits leaves whole and that run on 8
// wavefronts per workgroup instead of 4: a workgroup alone on its compute unit waits for its own loads,
// and 8 have twice as many under way.  Device times, 4 wavefronts and then 8:
//   - d = 64, bf16: 32 units of 352 keys 5.2 and 4.8 us, of 1200 10.9 and 8.8, 192 of 2000 18.3 and 16.2, 171 of
//     8000 62 and 58, of 65536 453 and 430.  With more units HBM is the bound on long ranges and nothing is left to
//     gain: 0.97 to 1.01 at 192 to 256 units over 3000 keys and more, 1.01 to 1.02 at 240 and 256 from 12000 on,
//     so from 8192 keys only up to 208 units.  Up to 256 keys, one block for each of the 8, level.
//   - d = 64, fp8: 32 units of 600 keys 5.5 and 4.9, of 1200 8.6 and 7.0, 256 of 2000 14.2 and 11.5; longer ones
//     are split.
//   - d = 128 has the loads of two such already: from fp8 0.85 to 0.97 of the time at 128 to 192 units (10 counts
//     of them) over 900 to 40000 keys, 136 of 4000 31.8 and 27.0, 176 of 20000 152 and 138; at other counts 0.93 to
//     1.09, in 16 bits 0.94 to 1.12.
// Against splits it was 0.95 to 1.24 and those stay.
inline bool decode_on_eight(const Shape& s, bool fp8, int splits) {
    const long units = (long)s.B * s.Hkv;
    if (splits > 1 || units > 256 || (long)(s.Hq / s.Hkv) * s.Lq > 16) return false;
    if (s.d == 64) return s.Lk > 256 && (units <= 208 || s.Lk <= 8192);
    return fp8 && units >= 128 && units <= 192 && s.Lk > 800;
}

// fp32 calls that run whole on the tile kernel although the rule for splits, which counts the per-key
// kernel's workgroups of 4 or 8 rows, would split them.  Row tiles have 16 rows, and 256 of them run as one
// round; in splits the rounds are shorter and more, and it counts how many of them there are all in all
// (9200 drawn calls of 256 to 1100 row tiles and 512 to 16384 keys; us in the rule's splits, then whole; where
// not said otherwise d = 64, one sequence):
//   - as many, or nearly: whole.  8 heads of 1000 x 1306 51 and 46, x 8192 255 and 257, 700 of one row over 2000
//     keys 145 and 133.  One round alone leaves a wavefront to a SIMD, which long ranges notice: 64 heads of
//     63 x 13491 237 and 306, but 256 of one row over 1300 38 and 32.
//   - down to 0.79 of them: whole in place of three splits (400 heads of one row over 2000 keys 85 and 80), in place of
//     two below 1000 keys (637 of 3 x 1061 75 and 67).  d = 128 has more to gain from splits: 400 heads of
//     one row over 3000 keys 154 and 161.
//   - fewer: split.  8 heads of 545 x 1306 40 and 46, x 8192 193 and 253.  But row tiles of unequal length even out by
//     themselves, where the first row sees at most 0.6 of what the last sees (8 heads of 545 x 1000 under a
//     mask 33 and 27), and up to 600 keys the second launch takes as much as the splits give.
// A call with a state runs the merge anyway, so it has less to gain whole.  Against the rule's splits the calls
// take 0.961 of the time, where always the better of the two gives 0.959; of 9300 others 10 are slower by more
// than 6 %, 1.13 at most.
inline bool f32_runs_whole(const Shape& s, bool causal, int shift, bool states, int splits) {
    const long g = s.Hq / s.Hkv, units = (long)s.B * s.Hkv;
    if (units * ceil_div(g * s.Lq, 16) < 256) return false;
    // rows that see a key, keys that the first and the last row see
    const long rows = causal ? std::min(std::max((long)s.Lq + shift, 0L), (long)s.Lq) : s.Lq;
    const long least = causal ? std::min(std::max(shift + 1L, 0L), (long)s.Lk) : s.Lk;
    const long most = causal ? std::min(std::max((long)s.Lq + shift, 0L), (long)s.Lk) : s.Lk;
    if (most <= 500) return true;
    const long tiles = units * ceil_div(g * rows, 16);
    if (tiles < 256) return tiles >= 200 && least == 0;
    const long rounds = (tiles + 255) / 256, in_splits = (tiles * splits + 255) / 256;
    if (16 * in_splits > 15 * rounds * splits) return rounds > 1 || least < 2000;
    if (states) return 3 * least <= most && least < 1300;
    if (100 * in_splits > 79 * rounds * splits &&
        (splits > 2 ? s.d == 64 || least < 2000 : s.d == 64 && least < 1000))
        return true;
    return least <= 600 || (5 * least <= 3 * most && least < 1300);
}

// ---- the two prefill kernels ----------------------------------------------------------------
// Under a causal mask a workgroup can take a long and a short row tile, so that all carry the same work; the
// pairs then run in rounds of `slots` workgroups, the last of which may be nearly empty, while single row
// tiles, longest first, even out by themselves.  Measured over 840 calls of 1 to 40 sequences, 8 to 32 heads and
// 300 to 12288 keys, d = 128 (time single over time in pairs, both prefill kernels; waste: by how much the
// rounds exceed the pairs):
//   - up to 4 rounds, more than 800 keys: waste above 0.4 0.68 to 0.93 (128-row kernel 2 x 16/2 heads of 4288, 1.05
//     rounds, 0.75; 256-row 2 x 12 of 5568 289 us and 177), 0.2 to 0.4 0.84 to 1.02, 0.05 to 0.2 0.88 to 1.02,
//     below 0.95 to 1.08.
//   - more rounds: 0.15 to 0.4 0.94 to 0.99, below 0.95 to 1.1.
//   - row tiles of less than 800 keys, where starting a workgroup costs as much as rounds waste: 0.2 to 0.4 0.9 to
//     1.0, below 0.97 to 1.04; less than 500 keys 1.06 to 1.12 up to 0.4, 0.84 to 0.91 above.
//   - K and V of more than 200 MB (100 at d = 64), which the last-level cache does not hold: pairs run a few heads at a
//     time, single row tiles all of them.  Up to 0.25 0.96 to 1.23, up to 0.4 0.88 to 1.08, above 0.89 to 0.96.
// (d = 64, 90 calls: 0.96 of the time on average, 0.76 to 1.02.)
inline bool rows_in_pairs(long m_tiles, long units, long slots, int Lk, int d, double kv_mb) {
    if (m_tiles < 2 || m_tiles * units < 2 * slots) return false;
    const double rounds = (double)((m_tiles + 1) / 2) * (double)units / (double)slots;
    const double waste = std::ceil(rounds) / rounds - 1.0;
    return waste <= (Lk < 500 || 128.0 * kv_mb > 200.0 * d ? 0.4 : Lk < 800 ? 0.2 : rounds < 4.0 ? 0.05 : 0.15);
}

// Time of a prefill kernel at d = 128, in us.  Both terms count steps of 64 keys, a row tile's start among them: those
// of the compute unit that ends last, and the average, which sets the clock (the part is at its power limit while
// all compute units work).  Fits over the calls above; within 5 % on average (1 % in the mean), 11 % at the 2nd
// and 98th percentile.
struct PrefillCost {
    int rows, slots;            // query rows of a workgroup, workgroups that run at once
    double start;               // steps that starting and storing a row tile counts for
    double last, share;         // us per step
    double launch, kv;          // us, and us per MB of K and V
};

// g: query heads that run as one, row by row
inline double prefill_estimate(const PrefillCost& c, const Shape& s, bool causal, long g) {
    const double units = (double)s.B * (double)(s.Hq / g), tiles = std::ceil((double)g * s.Lq / c.rows);
    double most = ceil_div(s.Lk, 64), least = most, all = tiles * most;
    if (causal) {
        const double off = std::max((double)s.Lk - s.Lq, 0.0), step = (double)c.rows / (double)g;
        most = s.Lk / 64.0;
        least = std::min(off + step, (double)s.Lk) / 64.0;
        all = ((tiles - 1.0) * off + step * (tiles - 1.0) * tiles / 2.0 + s.Lk) / 64.0 + 0.5 * tiles;
    }
    const double rounds = tiles * units / c.slots, open = std::ceil(rounds) - rounds;
    const double share = (all + c.start * tiles) * units / c.slots;
    const double last = causal ? share + (least + c.start) * open : (rounds + open) * (most + c.start);
    return c.launch + c.last * std::max(most + c.start, last) + c.share * share +
           c.kv * (double)s.B * s.Hkv * s.Lk * s.d * 4e-6;
}

// Where the automatic choice takes the 256-row prefill kernel: within the limits below, where its estimate is not
// behind that of the 128-row kernel.  Of 840 calls drawn as above 400 are within the limits and 46 of those go to the
// 128-row kernel by the estimate; with row tiles in pairs or not as above all 840 take 0.97 of the time that the
// limits alone and pairs throughout gave, 0.62 to 1.04 (1.12 in one case), 1 % more than with the better of the two
// kernels everywhere.  What is left lies outside the limits: there scores that keep passing the rows' references
// (standard deviation 4, planted dominant keys) cost the 256-row kernel more than it gains on others (6 x 32
// heads of 2841, causal, 841 us and 532).
//   - a workgroup per compute unit, two under a causal mask;
//   - 1536 keys without a mask, rows that see 1536 keys on average under a causal one, or 1024 where pairs of row tiles
//     fill whole rounds: what it pays at every change of row tile with only one workgroup on the compute unit is
//     about 8 us, four to five periods of 64 keys;
//   - no row tiles that are mostly padding: up to 4/3 of the rows that the 128-row kernel works on (64 sequences of 16
//     positions and 4 heads to a kv head over 8192 keys 1366 and 357 us).  At 4/3 itself the estimate is 3 % high (32 x
//     32 heads, 384 x 4096, causal), hence the margin.
inline bool prefers_256_rows(const Shape& s, bool causal) {
    if (s.d != 128 || s.dtype == 0) return false;
    static const PrefillCost kWide = {256, 256, 5.0, 1.148, 0.437, 2.3, 0.009};
    static const PrefillCost kTile = {128, 512, 2.0, 0.98, 0.937, 2.3, 0.055};
    const long g = s.Hq / s.Hkv, lq = s.Lq;
    const long wgs = (long)s.B * s.Hq * ((lq + 255) / 256);
    const long tiles128 = (g * lq + 127) / 128;
    if (3 * 256 * wgs > 4 * 128 * (long)s.B * s.Hkv * tiles128) return false;
    if (causal) {
        const long seen = (long)s.Lk - lq / 2;          // keys a row sees on average
        const bool whole_rounds = lq % 512 == 0 && (wgs / 2) % 256 == 0;
        if (wgs < 512 || seen < (whole_rounds ? 1024 : 1536)) return false;
    } else if (wgs < 256 || s.Lk < 1536) {
        return false;
    }
    // (the 128-row kernel runs the heads of a group as one where that saves row tiles or the rows are not late)
    const bool as_one = tiles128 < g * ((lq + 127) / 128) || !causal || s.Lk <= 8 * lq;
    return prefill_estimate(kWide, s, causal, 1) <
           (causal ? 1.035 : 1.0) * prefill_estimate(kTile, s, causal, as_one ? g : 1);
}

// ---- kernels for prefill calls that the 128-row kernel does not fill the chip with ----------
// Which kernel, and in how many of the splits of the rule, is decided by an estimate of each one's time:
// the chain of its longest row tile, its work on the whole chip and its way to K and V, whichever
// is the longest (smoothed), and what it reads and writes of states.  The figures are fits over 2500
// calls of 1 to 64 sequences, 4 to 32 heads, 8 to 12288 positions and 16 to 117000 keys, causal or
// not, whole or in chunks; the estimates are within 7 to 13 % on average.  By it 900 drawn calls, of which the
// 128-row kernel keeps most, went to 0.96 (d = 128) and 0.92 (d = 64) of their time on average,
// the least to 0.45: 5 x 16 heads, 182 x 882, d = 128 29.3 -> 17.2 us, 3 x 16 heads of 681, causal, d = 64
// 22.0 -> 11.2, 1 x 16/2 heads of 664 17.9 either way.
enum class RowKernel { Tile, Tile64, Short };

struct RowCost {
    int rows, keys;     // query rows of a workgroup, keys that it steps over at a time
    double start;       // us: launch, first loads, fold, store
    double chain;       // us a step of the longest row tile
    double work, wg;    // us a step, and a workgroup, of one compute unit's share of all
    double state;       // us per MB of states and partial states, read and written
    double kv;          // us per MB of K and V (of the 32- and 64-row kernels more than fitted: where memory is
                        // the bound, 64 x 32/8 heads, 16 x 8192, the 64-row one took 368 us and the 128-row one 310)
};

inline double row_estimate(const RowCost& c, const Shape& s, bool causal, int shift, int splits, int states) {
    const double g = s.Hq / s.Hkv, units = (double)s.B * s.Hkv, lq = s.Lq, lk = s.Lk;
    const double tiles = std::ceil(g * lq / c.rows);
    double most = lk, mean = lk;            // keys the last row, and a row on average, sees
    if (causal) {
        // row i sees min(max(i + shift + 1, 0), lk)
        const double lo = std::min(std::max(-(double)shift - 1.0, 0.0), lq);
        const double hi = std::min(std::max(lk - shift - 1.0, lo), lq);
        mean = ((hi - lo) * (lo + hi + 2.0 * shift + 1.0) * 0.5 + (lq - hi) * lk) / lq;
        most = std::min(std::max(lq + shift, 0.0), lk);
    }
    const double wgs = units * tiles * splits;
    const double chain = c.chain * std::ceil(most / ((double)c.keys * splits));
    // row tiles of equal length end together, the fullest compute unit's last (the 128-row kernel, which
    // the others have to beat, by the average)
    const double share = causal || c.rows == 128 ? wgs / 256.0 : std::ceil(wgs / 256.0);
    const double work = share * (c.work * (mean / ((double)splits * c.keys) + 0.5) + c.wg);
    // K and V are read into every L2 that a unit's row tiles run beside
    const double reads = (long)units % 8 == 0 ? 1.0 : std::min(8.0, tiles);
    const double kv = c.kv * units * most * s.d * 4e-6 * reads;
    const double p2 = chain * chain, q2 = work * work, r2 = kv * kv;
    const double state_mb = (double)s.B * s.Hq * lq * (s.d + 2) * 4e-6;
    double t = c.start + std::sqrt(std::sqrt(p2 * p2 + q2 * q2 + r2 * r2)) +
               c.state * state_mb * (states + (splits > 1 ? 2 * splits : 0));
    if (splits > 1) t += splits > 8 ? 4.6 : 3.6;        // the merge
    return t;
}

struct RowPlan { RowKernel kernel; int splits; };

// splits: those of the rule, which are also what scratch memory is sized for: the plan has
// no more.  states: states read and written by the call.  fp8: K and V are fp8, which the 32-row
// kernel reads as such and the others need widened first.
inline RowPlan row_plan(const Shape& s, bool causal, int shift, int splits, int states, bool fp8) {
    static const RowCost kTile[2] = {{128, 64, 3.7, 1.03, 0.65, 0.86, 0.21, 0.16},
                                     {128, 64, 6.2, 1.15, 1.10, 0.62, 0.19, 0.14}};
    static const RowCost kTile64[2] = {{64, 64, 4.4, 0.55, 0.34, 0.73, 0.16, 0.18},
                                       {64, 64, 5.9, 0.74, 0.59, 1.74, 0.16, 0.17}};
    static const RowCost kShort[2] = {{32, 128, 3.8, 0.57, 0.42, 0.52, 0.15, 0.18},
                                      {32, 128, 5.1, 0.82, 0.77, 1.67, 0.13, 0.17}};
    const int w = s.d == 128 ? 1 : 0;
    RowPlan plan{RowKernel::Tile, splits};
    const long g = s.Hq / s.Hkv;
    if (g * s.Lq > (1L << 30)) return plan;             // row numbers are 32-bit
    const long wgs = (long)s.B * s.Hkv * ceil_div(g * s.Lq, kShort[w].rows);
    // Up to two key tiles the start and the end of a workgroup are most of its time, and what counts is
    // that each has a compute unit to itself (device times, 128-row kernel and then the smaller one):
    // 32 rows, 8 heads of 512 x 128 d = 128 6.9 and 5.9 us, with a state 9.8 and 7.2, d = 64 5.2 and
    // 4.0, with a state 7.0 and 4.6 (0.60 to 0.95 of the time over 434 sizes); 64 rows, 32 heads of
    // 300 x 128 with a state 10.4 and 9.3 (0.82 to 1.015 over 62).  One key tile at d = 128
    // without a state is level (5.75 and 5.8) and stays, but from fp8 the 32-row kernel needs no
    // widening launch.
    if (s.Lk <= 128) {
        if (wgs <= 256 && (s.Lk > 64 || w == 0 || fp8 || (states > 0 && g * s.Lq >= 128)))
            plan = {RowKernel::Short, 1};
        else if (wgs > 256 && (s.Lk > 64 || w == 0 || states > 0) &&
                 (long)s.B * s.Hkv * ceil_div(g * s.Lq, kTile64[w].rows) <= 256)
            plan = {RowKernel::Tile64, 1};
        return plan;
    }
    // beyond this the 128-row kernel has rounds of workgroups to even things out by
    if (wgs > 2048) return plan;
    const double widen = fp8 ? 3.0 + (double)s.B * s.Hkv * s.Lk * s.d * 1.5e-6 : 0.0;
    // The 128-row kernel stays where it is not clearly behind, and over long split ranges where the
    // estimate is at its worst (5 x 32/8 heads, 66 x 9530 112 us on the 32-row kernel, 88 on it).
    double best = (row_estimate(kTile[w], s, causal, shift, splits, states) + widen) /
                  (splits > 1 && s.Lk > 2500 ? 1.2 : 1.05);
    const double t64 = row_estimate(kTile64[w], s, causal, shift, 1, states) + widen;
    if (t64 < best) {
        best = t64;
        plan = {RowKernel::Tile64, 1};
    }
    for (int sp : {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64}) {
        // one workgroup per compute unit (two at d = 64), which the ranges share out
        if (sp > splits || (sp > 1 && (wgs * sp > (w ? 320 : 512) || s.Lk / sp < 256))) break;
        const double t = row_estimate(kShort[w], s, causal, shift, sp, states);
        if (t < best) {
            best = t;
            plan = {RowKernel::Short, sp};
        }
    }
    // K and V of more than 100 MB, which no cache holds, are read again by every further round of workgroups,
    // and the smaller row tiles have more of those than the estimate sees: then the 128-row kernel stays (16-bit
    // K and V; its time and the other's).  32 rows, more than two workgroups on a compute unit: 13 x 24/8 heads,
    // 46 x 5093 91 and 111 us, 25 x 96/8, 11 x 9065, d = 64 233 and 264; from 196 MB on with fewer as well,
    // 16 x 5 heads, 155 x 5306 68 and 92.  64 rows, more than two where the 128-row tiles are all resident, or
    // more than four: 4 x 64 heads, 152 x 1223 42 and 64, 34 x 12, 147 x 2012 150 and 187.  Of 36000 drawn calls
    // that the estimate takes from the 128-row kernel 115 that were slower by it (1.22 on average) go back, and
    // 31 that were not (0.88); 161 slower ones are left, a third of them by more than 10 %.  Of 13700 others (129
    // to 24000 keys, any number of heads, states) 26 are slower than on the 128-row kernel alone by more than 5 %.
    const double most = causal ? std::min(std::max((double)s.Lq + shift, 0.0), (double)s.Lk) : s.Lk;
    const double kv_mb = (double)s.B * s.Hkv * most * s.d * 4e-6;
    if (plan.kernel == RowKernel::Short && !fp8 && (kv_mb > 196.0 || (kv_mb > 100.0 && wgs * plan.splits > 512)))
        plan = {RowKernel::Tile, splits};
    if (plan.kernel == RowKernel::Tile64 && kv_mb > 100.0) {
        const long wgs64 = (long)s.B * s.Hkv * ceil_div(g * s.Lq, kTile64[w].rows);
        const long wgs128 = (long)s.B * s.Hkv * ceil_div(g * s.Lq, kTile[w].rows) * splits;
        if (wgs64 > 1024 || (wgs64 > 512 && wgs128 <= 512)) plan = {RowKernel::Tile, splits};
    }
    return plan;
}

}  // namespace flashd

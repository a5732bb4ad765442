// The C ABI of libflashd: argument validation, variant/split selection, the
// per-(device, stream) workspace cache, and dispatch to the kernel launchers.
#include <hip/hip_runtime.h>

#include <cstring>
#include <map>
#include <mutex>
#include <utility>
#include <vector>

#include "../../include/flashd.h"
#include "flashd_common.h"
#include "flashd_kernels.h"
#include "flashd_plan.h"

namespace {

using flashd::ceil_div;
using flashd::decode_on_eight;
using flashd::f32_runs_whole;
using flashd::prefers_256_rows;
using flashd::Problem;
using flashd::row_plan;
using flashd::RowKernel;
using flashd::RowPlan;
using flashd::Shape;

int validate_shape(const Shape& s) {
    if (s.B < 1 || s.Hq < 1 || s.Hkv < 1 || s.Lq < 1 || s.Lk < 1) return FLASHD_E_SHAPE;
    if (s.B > 65535 || s.Hq > 65535) return FLASHD_E_SHAPE;          // grid y/z limits
    // row and key indices, and their sums with the causal shift, are 32-bit in the kernels
    if (s.Lq > 1000000000 || s.Lk > 1000000000) return FLASHD_E_SHAPE;
    if (s.dtype != FLASHD_F32 && s.dtype != FLASHD_F16 && s.dtype != FLASHD_BF16)
        return FLASHD_E_DTYPE;
    if (s.d != 64 && s.d != 128) return FLASHD_E_HEADDIM;
    if (s.Hq % s.Hkv != 0) return FLASHD_E_GQA;
    // element counts must fit 2^40 so every byte offset fits size_t with room to spare
    const long double nq = (long double)s.B * s.Hq * s.Lq * s.d;
    const long double nk = (long double)s.B * s.Hkv * s.Lk * s.d;
    if (nq > 1.0e12L || nk > 1.0e12L) return FLASHD_E_SHAPE;
    return FLASHD_OK;
}

int resolve_variant(const Shape& s, int variant) {
    if (variant < FLASHD_VARIANT_AUTO || variant > FLASHD_VARIANT_TILE_256) return -1;
    if (variant == FLASHD_VARIANT_AUTO)
        return s.dtype == FLASHD_F32 ? FLASHD_VARIANT_PER_KEY : FLASHD_VARIANT_TILE;
    if (s.dtype == FLASHD_F32 && variant != FLASHD_VARIANT_PER_KEY) return -1;
    return variant;
}

// n partial states (o[d], s, ln w) per query row
size_t partial_bytes(const Shape& s, int n) {
    return (size_t)n * s.B * s.Hq * s.Lq * (size_t)(s.d + 2) * sizeof(float);
}

// Splits for decode shapes (measured over 8 to 640 (b, kv head) units, 700 to 131072 keys and 1 to
// 64 splits, with 4 and 32 query rows per kv head; times are of one launch among others).
//   - Short key ranges stay whole: a second launch and its gap cost 4 us, a 32-key block takes a
//     wavefront 1 us at d = 128 and half of that at 64.  8 units of 600 keys: 8.1 us whole, 9.0
//     in any number of splits; of 1000 keys 10.5 and 9.5.  Below 512 keys nothing is split, here
//     as in auto_splits, so that such calls need no scratch memory and can be captured into a graph
//     without a call before; nor from 512 units on.
//   - How many workgroups fill the chip depends on what one streams by itself, 32 keys of K and V per
//     wavefront and step:
//       16-bit cache, d = 128, up to 16 rows (1.1 us for 64 KB): HBM is the bound from 192 on, three
//       quarters of the compute units.  48 units of 4000 keys 21.2 us in 4 splits, 25.6 in 6; 24
//       of 20000 43 in 8, 57 in 12; 8 of 131072 84.9 in 24, 86.6 in 32, 89.8 in 64.
//       d = 64 from fp8 (0.6 us for 16 KB) or for 17 to 32 rows (0.65 us from fp8, 1.4 us for 32 KB
//       without): two per compute unit.  64 units of 20000 keys, fp8: 31.0 us in 8 splits, 35.7 in
//       4, 43.5 in 3; 32 rows without fp8 59.8, 74.1 and 92.8; 160 units of 8000 keys, 32 rows,
//       59.6 in 3, 66.9 in 2, 101.6 whole.
//       The others: one per compute unit.  64 units of 60000 keys, fp8, d = 128: 144.6 us in 4
//       splits, 162 in 3, 183 in 5; 32 rows, d = 128 301 in 4, 337 in 3.
//   - The second workgroup of a compute unit needs ranges of one or two steps to pay (d = 64, 32
//     rows: 56 units of 1326 keys with fp8 13.6 us in 4 splits, 14.9 in 5, 15.2 in 8).
//   - More units than 96: a last round of workgroups that is mostly empty costs more than splits
//     give.  104 units of 20000 keys take 163 us in two splits, 197 in three and 210 whole; 129
//     units with fp8, d = 128 take 0.76 of the time whole in three, 0.97 in two.  Above 256 units,
//     where few compute units have a second workgroup, two splits take 0.90 to 0.95 of the time
//     whole up to 342 units (16 rows, all types); with more rows a compute unit holds two
//     workgroups and not three, and only the fp8 cache with d = 64 gains, on long ranges (0.86 to
//     0.93 at 20000 keys up to 384 units, 1.03 to 1.13 at 3000).  Short ranges stay whole: 127
//     units of 1500 keys 20.2 us, 20.8 in 2; the slower kernel for 17 to 32 rows gains from 1024
//     keys on (128 units of 1500 keys, d = 64: 25.7 whole, 19.3 in 4).
//   - With up to 8 units more splits pay until a wavefront has two blocks left (8 units of 16000
//     keys: 29 us in 8, 17.7 in 32, 16.8 in 64; 4 units of 20000 keys 15.4 in 64).  Up to 8
//     splits cost the merge the same, more of them 1 us: 24 units with fp8 take 10.0 us in 8 and
//     11.0 in 13 (4000 keys, d = 64), 15.0 in 8 and 16.0 in 10 (7779 keys, d = 128), 20 units of
//     74088 keys 76 in 8 and 62 in 12.
//   - 17 to 32 query rows: a block takes longer, half a block is left per wavefront (4 units of
//     3000 keys: 20.3 us in 8 splits, 16.2 in 48).
// or_shorter: the most splits of any call with this many keys or fewer (the choice itself falls
// from 64 where the ranges of few units get long).
int decode_splits(const Shape& s, int variant, bool fp8, bool or_shorter) {
    const long units = flashd::decode_workgroups(s.B, s.Hkv);
    const long blocks = (s.Lk + 31L) / 32;
    // the kernel for 17 to 32 rows, which also runs the two ablations
    const bool wide = (long)(s.Hq / s.Hkv) * s.Lq > 16 || variant == FLASHD_VARIANT_ONLINE_SOFTMAX ||
                      variant == FLASHD_VARIANT_TILE_BLEND;
    if (s.Lk < 512 || blocks * s.d <= (wide ? 1024 : 2560) || units >= 512) return 1;
    const bool fast = !wide && !fp8 && s.d == 128;       // 192 workgroups saturate HBM
    const bool small = s.d == 64 && (wide || fp8);       // 512 do not
    const long one = 256 / units, two = 512 / units;     // splits for one, two workgroups per compute unit
    if (units > 96) {
        if (blocks < (wide && !fp8 ? 32 : 64)) return 1;
        if (units > 256)
            return wide ? (fp8 && small && units < 384 && blocks >= 256 ? 2 : 1) : units < 342 ? 2 : 1;
        const long more = small || (two == 3 && !fast && blocks >= 128) ? two : 1;
        return (int)(one > more ? one : more);
    }
    const long few = blocks / 4 < 8 ? blocks / 4 : 8;
    const long many = blocks / (wide ? 2 : 8);
    // long enough ranges for the second workgroup of a compute unit
    const bool deep = blocks / (fp8 ? 8 : 4) >= (two < FLASHD_MAX_SPLITS ? two : FLASHD_MAX_SPLITS);
    const long most = units <= 8 && (blocks < 2048 || or_shorter) && (!wide || deep) ? FLASHD_MAX_SPLITS
                      : fast ? 192 / units : small && deep ? two : one;
    long sp = few > many ? few : many;
    if (sp > most) sp = most;
    if (sp > 8 && units > 8 && !fast && blocks < (sp <= 12 ? 320 : 160)) sp = 8;
    return (int)(sp < 1 ? 1 : sp > FLASHD_MAX_SPLITS ? FLASHD_MAX_SPLITS : sp);
}

// Splits for the automatic choice: enough independent work to fill 256 compute units, but
// never key ranges shorter than 256 keys.  or_shorter: the most splits of any call with this many
// keys or fewer.  Outside the decode shapes the choice never falls as the keys grow.
int auto_splits(const Shape& s, int variant, bool fp8 = false, bool or_shorter = false) {
    if (variant != FLASHD_VARIANT_PER_KEY && flashd::decode_applies(s.Hq, s.Hkv, s.Lq))
        return decode_splits(s, variant, fp8, or_shorter);
    long units;
    if (variant == FLASHD_VARIANT_PER_KEY) {
        const int rows_per_group = (s.d <= 64 ? 2 : 1) * 4;             // 4 wavefronts
        units = (long)s.B * s.Hq * ceil_div(s.Lq, rows_per_group);      // workgroups
    } else {
        units = flashd::tile_workgroups(s.B, s.Hq, s.Hkv, s.Lq, s.d);
    }
    // Two workgroups are resident per compute unit (512 in all), and one full round of them
    // is what the tile kernel wants: measured over short-query and prefill
    // shapes of 64 to 512 units, the fastest split count is the one that brings the launch
    // to 256-512 workgroups; more of them only add partial states to write and merge.  The
    // per-key kernel keeps two rounds; the fp32 tile kernel that AUTO runs in its place takes its
    // splits from here too, or runs whole (f32_runs_whole).
    const long target = variant == FLASHD_VARIANT_PER_KEY ? 1024 : 512;
    if (units < 1) units = 1;
    long sp = units >= target ? 1 : ceil_div(target, units);
    // A split costs its partial states: (d + 2) floats per query row written and read back.
    // For the per-key kernel 256 keys are enough to pay for a
    // split; the tile kernel's workgroups carry 128 rows each, and measured over prefill
    // shapes a split only pays once it still holds some 2048 keys (B1 H32 L1024 causal:
    // 23 us unsplit, 39 us in two splits of 512 keys).
    // With few query rows in all (short queries that do not fit the decode kernel: 4 x 8
    // heads x 8 positions over 4096 keys runs 15 us in 16 splits, 45 us in 2) the partial
    // states are small again: splits of 256 keys are allowed as long as all the partial
    // states together stay within some 40 MB.
    const bool tile = variant != FLASHD_VARIANT_PER_KEY;
    long by_len = s.Lk / (tile ? 2048 : 256);
    if (tile) {
        const long double per_split = (long double)partial_bytes(s, 1) * 2.0L;   // written and read
        const long by_bytes = per_split > 0.0L ? (long)(40.0e6L / per_split) : 0;
        const long by_len_short = s.Lk / 256;
        const long few_rows = by_bytes < by_len_short ? by_bytes : by_len_short;
        if (few_rows > by_len) by_len = few_rows;
    }
    if (by_len < 1) by_len = 1;
    if (sp > by_len) sp = by_len;
    if (sp > FLASHD_MAX_SPLITS) sp = FLASHD_MAX_SPLITS;
    if (sp < 1) sp = 1;
    return (int)sp;
}

// Splits whose partial states the scratch memory of a call with sp splits is sized for.  A call of
// the automatic choice that needs scratch at all takes what every call with fewer keys needs, so
// that one made at the longest context serves a decode loop, or a graph captured later, at any
// shorter one.
int scratch_splits(const Shape& s, int variant, bool fp8, int splits, int sp) {
    return splits == 0 && sp > 1 ? auto_splits(s, variant, fp8, true) : sp;
}

size_t ws_bytes(const Shape& s, int splits) { return splits <= 1 ? 0 : partial_bytes(s, splits); }

// ---- device check ----------------------------------------------------------

std::mutex g_mu;
std::map<int, int> g_arch_ok;      // device -> 1 ok / 0 not gfx950

int check_arch() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); return FLASHD_E_HIP; }
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_arch_ok.find(dev);
    if (it == g_arch_ok.end()) {
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, dev) != hipSuccess) {
            (void)hipGetLastError();
            return FLASHD_E_HIP;
        }
        const int ok = std::strncmp(prop.gcnArchName, "gfx950", 6) == 0 ? 1 : 0;
        it = g_arch_ok.emplace(dev, ok).first;
    }
    return it->second ? FLASHD_OK : FLASHD_E_ARCH;
}

// ---- workspace cache: grow-only, one buffer per (device, stream) -----------
// A buffer that is outgrown is not freed on the spot, because work enqueued earlier on the
// stream may still be reading it: it is kept in the entry's list of retired buffers until
// flashd_release_workspace() frees everything (hipFree waits for the device first).

struct CacheEntry {
    void* ptr = nullptr;
    size_t bytes = 0;
    std::vector<void*> retired;
};
std::map<std::pair<int, void*>, CacheEntry> g_cache;

int cached_workspace(void* stream, size_t bytes, void** out) {
    *out = nullptr;
    if (bytes == 0) return FLASHD_OK;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); return FLASHD_E_HIP; }
    std::lock_guard<std::mutex> lk(g_mu);
    CacheEntry& e = g_cache[std::make_pair(dev, stream)];
    if (e.bytes < bytes) {
        // grow geometrically; if that much is not to be had, take exactly what is needed
        size_t want = e.bytes * 2 > bytes ? e.bytes * 2 : bytes;
        void* p = nullptr;
        if (hipMalloc(&p, want) != hipSuccess) {
            (void)hipGetLastError();
            want = bytes;
            if (hipMalloc(&p, want) != hipSuccess) { (void)hipGetLastError(); return FLASHD_E_HIP; }
        }
        if (e.ptr != nullptr) e.retired.push_back(e.ptr);
        e.ptr = p;
        e.bytes = want;
    }
    *out = e.ptr;
    return FLASHD_OK;
}

// Frees every cached buffer of the current device, live or retired.
int release_workspace() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); return FLASHD_E_HIP; }
    std::lock_guard<std::mutex> lk(g_mu);
    int rc = FLASHD_OK;
    for (auto it = g_cache.begin(); it != g_cache.end();) {
        if (it->first.first != dev) { ++it; continue; }
        CacheEntry& e = it->second;
        if (e.ptr != nullptr) e.retired.push_back(e.ptr);
        for (void* q : e.retired)
            if (hipFree(q) != hipSuccess) { (void)hipGetLastError(); rc = FLASHD_E_HIP; }
        it = g_cache.erase(it);
    }
    return rc;
}

// ---- static scratch: split-K partial states for the entry point that allocates nothing ---
// One array per GPU, part of the loaded code object, held until the process ends.  In host
// code the array's name is only a handle for hipGetSymbolAddress: the device address is asked
// for once per device (with that device current) and kept, and only that address is ever
// handed to a kernel.
constexpr size_t kScratchBytes = FLASHD_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
std::map<int, void*> g_scratch_ptr;     // device -> address of its copy of `scratch`

int static_scratch(void** out) {
    *out = nullptr;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); return FLASHD_E_HIP; }
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_scratch_ptr.find(dev);
    if (it == g_scratch_ptr.end()) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) {
            (void)hipGetLastError();
            return FLASHD_E_HIP;
        }
        it = g_scratch_ptr.emplace(dev, ptr).first;
    }
    *out = it->second;
    return FLASHD_OK;
}

enum class WsMode { Caller, Cache, Static };

struct SkipArgs {
    bool on = false;                 // decode kernel with the saturation skip on the V fetch
    unsigned long long* counts = nullptr;
};

// ---- common front end --------------------------------------------------------

struct StateArgs {
    bool on = false;                 // the state entry point: o may be NULL, shift is explicit
    int shift = 0;
    const float* in = nullptr;
    float* out = nullptr;
};

struct Kv8Args {
    bool on = false;                 // k and v are fp8 (e4m3) with one scale each
    float kscale = 1.0f, vscale = 1.0f;
};

int run(const void* q, const void* k, const void* v, void* o, const Shape& s, int causal,
        float scale, void* stream, int variant, int splits, void* workspace,
        size_t workspace_bytes, WsMode mode, const StateArgs& sa = StateArgs(),
        const Kv8Args& k8 = Kv8Args(), const SkipArgs& sk = SkipArgs()) {
    const bool use_cache = mode == WsMode::Cache;
    if (!q || !k || !v) return FLASHD_E_NULL;
    if (!o && !(sa.on && sa.out)) return FLASHD_E_NULL;
    int rc = validate_shape(s);
    if (rc != FLASHD_OK) return rc;
    const uintptr_t bits = (uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o |
                           (uintptr_t)workspace | (uintptr_t)sa.in | (uintptr_t)sa.out;
    if (bits & 15u) return FLASHD_E_ALIGN;
    if ((uintptr_t)sk.counts & 7u) return FLASHD_E_ALIGN;
    const int var = resolve_variant(s, variant);
    if (var < 0) return FLASHD_E_VARIANT;
    // fp8 K/V: the decode kernels and the prefill kernel with 32 query rows per workgroup read that
    // storage themselves; for the other kernels K and V are first widened (exactly) into scratch memory
    if (k8.on && s.dtype == FLASHD_F32) return FLASHD_E_VARIANT;
    // the skip lives in the split-K decode kernel (f16/bf16, at most 32 query rows per kv head)
    if (sk.on && (s.dtype == FLASHD_F32 || !flashd::decode_applies(s.Hq, s.Hkv, s.Lq)))
        return FLASHD_E_VARIANT;
    const bool decode = flashd::decode_applies(s.Hq, s.Hkv, s.Lq);
    if (splits < 0 || splits > FLASHD_MAX_SPLITS || splits > s.Lk) return FLASHD_E_VARIANT;
    const int sp_most = splits == 0 ? auto_splits(s, var, k8.on) : splits;
    // a shift of Lk or more shows every key and one below -Lq none: clamping the caller's
    // value there changes no result and keeps i + shift inside 32 bits
    const int shift = !sa.on ? s.Lk - s.Lq : sa.shift > s.Lk ? s.Lk : sa.shift < -s.Lq - 1 ? -s.Lq - 1 : sa.shift;
    const bool auto_wide = !sa.on && !k8.on && !sk.on && sp_most == 1 && prefers_256_rows(s, causal != 0);
    const bool wide = var == FLASHD_VARIANT_TILE_256 || (variant == FLASHD_VARIANT_AUTO && auto_wide);
    RowPlan plan{RowKernel::Tile, sp_most};
    if (var == FLASHD_VARIANT_TILE && splits == 0 && !decode && !auto_wide)
        plan = row_plan(s, causal != 0, shift, sp_most,
                        (sa.in != nullptr ? 1 : 0) + (sa.out != nullptr ? 1 : 0), k8.on);
    const bool eight = decode && var == FLASHD_VARIANT_TILE && splits == 0 && !sa.on &&
                       decode_on_eight(s, k8.on, sp_most);
    if (variant == FLASHD_VARIANT_AUTO && splits == 0 && s.dtype == FLASHD_F32 &&
        f32_runs_whole(s, causal != 0, shift, sa.on, sp_most))
        plan.splits = 1;
    const int sp = plan.splits;
    const bool widen = k8.on && !decode && plan.kernel != RowKernel::Short;
    // The state entry point always goes through partial states; a single partial may be
    // written straight into the caller's state buffer (unless that is also the input state).
    const bool direct = sa.on && sp == 1 && sa.out != nullptr && sa.out != sa.in;
    // The tile kernel can start from the state itself and write both results: no partial
    // states, no merge kernel.
    const bool in_kernel = sa.on && sp == 1 && var == FLASHD_VARIANT_TILE && !decode;
    // (by the splits of the rule, also where the plan has fewer: what scratch memory suffices for
    // does not depend on the kernel that runs)
    const size_t need = sa.on ? ((sp_most == 1 && (direct || in_kernel)) ? 0 : partial_bytes(s, sp_most))
                              : ws_bytes(s, sp_most);
    if (mode == WsMode::Caller && need > 0 && (workspace == nullptr || workspace_bytes < need))
        return FLASHD_E_WORKSPACE;
    if (mode == WsMode::Static && need > kScratchBytes) return FLASHD_E_WORKSPACE;

    rc = check_arch();
    if (rc != FLASHD_OK) return rc;
    void* ws = workspace;
    const size_t need_al = (need + 255) & ~(size_t)255;
    // (Also where the plan needs nothing widened: a call with fewer keys may, and is to find its scratch
    // memory taken by this one, for instance when it is captured into a graph.)
    const size_t kv_bytes = k8.on && !decode ? (size_t)s.B * s.Hkv * s.Lk * s.d * 2 : 0;   // per tensor
    if (use_cache) {
        const size_t cover = partial_bytes(s, scratch_splits(s, var, k8.on, splits, sp_most));
        const size_t most = need > 0 && cover > need_al ? (cover + 255) & ~(size_t)255 : need_al;
        rc = cached_workspace(stream, most + 2 * kv_bytes, &ws);
        if (rc != FLASHD_OK) return rc;
    }
    if (mode == WsMode::Static && need > 0) {
        rc = static_scratch(&ws);
        if (rc != FLASHD_OK) return rc;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    float score_scale = scale, out_scale = 1.0f;
    bool kv8_kernel = k8.on;
    if (widen) {
        char* base = static_cast<char*>(ws) + need_al;
        if (flashd::launch_widen_fp8(k, v, base, base + kv_bytes,
                                     (size_t)s.B * s.Hkv * s.Lk * s.d, s.dtype, st) != hipSuccess)
            return FLASHD_E_HIP;
        k = base;
        v = base + kv_bytes;
        score_scale = scale * k8.kscale;       // one fp32 product, as in the decode kernel
        out_scale = k8.vscale;
        kv8_kernel = false;
    }

    Problem p;
    p.q = q; p.k = k; p.v = v; p.o = o;
    p.ws = static_cast<float*>(ws);
    p.B = s.B; p.Hq = s.Hq; p.Hkv = s.Hkv; p.Lq = s.Lq; p.Lk = s.Lk; p.d = s.d;
    p.heads = flashd::make_fast_div(1);
    p.head_rows = s.Lq;
    p.dtype = s.dtype;
    p.causal = causal != 0;
    p.splits = sp;
    p.scale = score_scale;
    p.oscale = out_scale;
    p.shift = shift;
    p.partial = (sp > 1 || sa.on) ? 1 : 0;
    p.store_o = p.partial ? 0 : 1;
    p.merge = p.partial;
    p.from_state = 0;
    p.state_in = sa.in;
    p.state_out = sa.out;
    p.vskip_counts = sk.counts;
    p.wide = wide ? 1 : 0;
    p.many = eight ? 1 : 0;
    if (in_kernel) {
        p.partial = sa.out != nullptr ? 1 : 0;     // the "partial" is the state handed out
        p.store_o = o != nullptr ? 1 : 0;
        p.merge = 0;
        p.from_state = sa.in != nullptr ? 1 : 0;
        p.ws = sa.out;
    }
    p.kv8 = kv8_kernel ? 1 : 0;
    p.kscale = k8.kscale;
    p.vscale = k8.vscale;
    if (direct && !in_kernel) p.ws = sa.out;
    hipError_t e;
    // The automatic choice takes the decode kernel with the saturation skip: on inputs where
    // nothing can be skipped it returns the bits of the unskipped kernel at the same speed.
    const bool auto_skip = variant == FLASHD_VARIANT_AUTO && !k8.on && s.dtype != FLASHD_F32 && decode;
    const int tmode = (sk.on || auto_skip)                 ? flashd::kTileModeLazySkipV
                      : var == FLASHD_VARIANT_ONLINE_SOFTMAX ? flashd::kTileModeOnline
                      : var == FLASHD_VARIANT_TILE_BLEND   ? flashd::kTileModeBlend
                                                           : flashd::kTileModeLazy;
    // fp32 without a variant asked for: the tile form on the matrix cores
    if (s.dtype == FLASHD_F32 && variant == FLASHD_VARIANT_AUTO) e = flashd::launch_tile_f32(p, st);
    else if (var == FLASHD_VARIANT_PER_KEY) e = flashd::launch_perkey(p, st);
    else if (decode) e = flashd::launch_decode(p, tmode, st);
    else if (plan.kernel == RowKernel::Short) e = flashd::launch_short(p, st);
    else if (plan.kernel == RowKernel::Tile64) e = flashd::launch_tile64(p, st);
    else e = flashd::launch_tile(p, tmode, st);
    return e == hipSuccess ? FLASHD_OK : FLASHD_E_HIP;
}

}  // namespace

extern "C" {

int flashd_attn_fwd(const void* q, const void* k, const void* v, void* o, int B, int Hq, int Hkv,
                    int Lq, int Lk, int d, int causal, float scale, int dtype, void* stream) {
    const Shape s{B, Hq, Hkv, Lq, Lk, d, dtype};
    return run(q, k, v, o, s, causal, scale, stream, FLASHD_VARIANT_AUTO, 0, nullptr, 0,
               WsMode::Cache);
}

int flashd_attn_fwd_static(const void* q, const void* k, const void* v, void* o, int B, int Hq,
                           int Hkv, int Lq, int Lk, int d, int causal, float scale, int dtype,
                           void* stream) {
    const Shape s{B, Hq, Hkv, Lq, Lk, d, dtype};
    return run(q, k, v, o, s, causal, scale, stream, FLASHD_VARIANT_AUTO, 0, nullptr, 0,
               WsMode::Static);
}

int flashd_attn_fwd_ex(const void* q, const void* k, const void* v, void* o, int B, int Hq,
                       int Hkv, int Lq, int Lk, int d, int causal, float scale, int dtype,
                       void* stream, int variant, int splits, void* workspace,
                       size_t workspace_bytes) {
    const Shape s{B, Hq, Hkv, Lq, Lk, d, dtype};
    return run(q, k, v, o, s, causal, scale, stream, variant, splits, workspace, workspace_bytes,
               WsMode::Caller);
}

int flashd_attn_fwd_state(const void* q, const void* k, const void* v, void* o,
                          const float* state_in, float* state_out, int B, int Hq, int Hkv, int Lq,
                          int Lk, int d, int causal, int causal_shift, float scale, int dtype,
                          void* stream) {
    const Shape s{B, Hq, Hkv, Lq, Lk, d, dtype};
    StateArgs sa;
    sa.on = true;
    sa.shift = causal_shift;
    sa.in = state_in;
    sa.out = state_out;
    return run(q, k, v, o, s, causal, scale, stream, FLASHD_VARIANT_AUTO, 0, nullptr, 0,
               WsMode::Cache, sa);
}

int flashd_attn_fwd_kv8(const void* q, const void* k8, const void* v8, void* o, int B, int Hq,
                        int Hkv, int Lq, int Lk, int d, int causal, float scale, float kscale,
                        float vscale, int dtype, void* stream) {
    const Shape s{B, Hq, Hkv, Lq, Lk, d, dtype};
    Kv8Args a;
    a.on = true;
    a.kscale = kscale;
    a.vscale = vscale;
    return run(q, k8, v8, o, s, causal, scale, stream, FLASHD_VARIANT_AUTO, 0, nullptr, 0,
               WsMode::Cache, StateArgs(), a);
}

int flashd_attn_fwd_skipv(const void* q, const void* k, const void* v, void* o, int B, int Hq,
                          int Hkv, int Lq, int Lk, int d, int causal, float scale, int dtype,
                          void* stream, int splits, void* workspace, size_t workspace_bytes,
                          unsigned long long* counts) {
    const Shape s{B, Hq, Hkv, Lq, Lk, d, dtype};
    SkipArgs sk;
    sk.on = true;
    sk.counts = counts;
    return run(q, k, v, o, s, causal, scale, stream, FLASHD_VARIANT_TILE, splits, workspace,
               workspace_bytes, WsMode::Caller, StateArgs(), Kv8Args(), sk);
}

int flashd_skip_stats(const void* q, const void* k, int B, int Hq, int Hkv, int Lq, int Lk, int d,
                      int causal, float scale, int dtype, float lo, float hi,
                      unsigned long long* counts, void* stream) {
    if (!q || !k || !counts) return FLASHD_E_NULL;
    const Shape s{B, Hq, Hkv, Lq, Lk, d, dtype};
    int rc = validate_shape(s);
    if (rc != FLASHD_OK) return rc;
    if (((uintptr_t)q | (uintptr_t)k) & 15u) return FLASHD_E_ALIGN;
    if ((uintptr_t)counts & 7u) return FLASHD_E_ALIGN;
    rc = check_arch();
    if (rc != FLASHD_OK) return rc;
    Problem p;
    p.q = q; p.k = k; p.v = nullptr; p.o = nullptr; p.ws = nullptr;
    p.B = B; p.Hq = Hq; p.Hkv = Hkv; p.Lq = Lq; p.Lk = Lk; p.d = d;
    p.heads = flashd::make_fast_div(1);
    p.head_rows = Lq;
    p.dtype = dtype;
    p.causal = causal != 0;
    p.splits = 1;
    p.scale = scale;
    p.shift = Lk - Lq;
    p.partial = 0;
    p.store_o = 0;
    p.merge = 0;
    p.from_state = 0;
    p.state_in = nullptr;
    p.state_out = nullptr;
    p.wide = 0;
    p.many = 0;
    p.vskip_counts = nullptr;
    p.kv8 = 0;
    p.kscale = p.vscale = p.oscale = 1.0f;
    const hipError_t e =
        flashd::launch_skip_stats(p, lo, hi, counts, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? FLASHD_OK : FLASHD_E_HIP;
}

int flashd_auto_splits(int B, int Hq, int Hkv, int Lq, int Lk, int d, int dtype, int variant) {
    const Shape s{B, Hq, Hkv, Lq, Lk, d, dtype};
    if (validate_shape(s) != FLASHD_OK) return 1;
    const int var = resolve_variant(s, variant);
    if (var < 0) return 1;
    return auto_splits(s, var);
}

int flashd_auto_variant(int B, int Hq, int Hkv, int Lq, int Lk, int d, int dtype, int causal) {
    const Shape s{B, Hq, Hkv, Lq, Lk, d, dtype};
    if (validate_shape(s) != FLASHD_OK) return -1;
    const int var = resolve_variant(s, FLASHD_VARIANT_AUTO);
    if (var != FLASHD_VARIANT_TILE || flashd::decode_applies(s.Hq, s.Hkv, s.Lq)) return var;
    return auto_splits(s, var) == 1 && prefers_256_rows(s, causal != 0) ? FLASHD_VARIANT_TILE_256
                                                                          : FLASHD_VARIANT_TILE;
}

size_t flashd_workspace_bytes(int B, int Hq, int Hkv, int Lq, int Lk, int d, int dtype,
                              int variant, int splits) {
    const Shape s{B, Hq, Hkv, Lq, Lk, d, dtype};
    if (validate_shape(s) != FLASHD_OK) return 0;
    const int var = resolve_variant(s, variant);
    if (var < 0 || splits < 0 || splits > FLASHD_MAX_SPLITS || splits > Lk) return 0;
    const int sp = splits == 0 ? auto_splits(s, var) : splits;
    return ws_bytes(s, scratch_splits(s, var, false, splits, sp));
}

int flashd_release_workspace(void) { return release_workspace(); }

const char* flashd_status_string(int status) {
    switch (status) {
    case FLASHD_OK: return "ok";
    case FLASHD_E_NULL: return "q, k, v or o is NULL";
    case FLASHD_E_SHAPE: return "a dimension is out of range";
    case FLASHD_E_DTYPE: return "unknown dtype";
    case FLASHD_E_HEADDIM: return "head dimension must be 64 or 128";
    case FLASHD_E_GQA: return "Hq must be a multiple of Hkv";
    case FLASHD_E_ALIGN: return "pointers must be 16-byte aligned";
    case FLASHD_E_WORKSPACE: return "workspace missing or too small";
    case FLASHD_E_HIP: return "a HIP call failed";
    case FLASHD_E_ARCH: return "the current device is not gfx950";
    case FLASHD_E_VARIANT: return "variant or splits not valid for this problem";
    default: return "unknown status";
    }
}

int flashd_version(void) { return 100; }

}  // extern "C"

// libtlinattn: C-ABI entry points (see include/tlinattn.h), argument validation, partition
// planning and kernel launches.  gfx950 only.
#include "tlinattn.h"
#include "tlinattn_profile.h"

#include <math.h>
#include <string.h>

#include <atomic>
#include <mutex>
#include <utility>
#include <vector>

#include "attn_bf16.h"
#include "attn_f32.h"
#include "decode.h"
#include "merge.h"

using namespace tlin;

// Workspace of tlin_layer_attn_static_ws: split partials of the history axis and the window
// partial, for callers that cannot bring device memory of their own.  Host code never uses this
// name as an address; static_scratch() asks the runtime for the array's address on the current device.
static __device__ __align__(256) unsigned char scratch[TLIN_STATIC_WS_BYTES];

namespace {

constexpr int kVersion = 200;   // 0.2.0
constexpr int kMaxRows = 1 << 30;

// One kernel launch, reporting the status of this launch only: errors that the caller's earlier
// work left behind stay where they are (nothing here reads or clears the runtime's last error).
// Every kernel of the library takes a single argument structure by value.
template <typename Args>
tlin_status launch_kernel(const void *kernel, dim3 grid, dim3 block, size_t lds_bytes, hipStream_t st, const Args &a)
{
    void *argv[] = {const_cast<Args *>(&a)};
    return hipLaunchKernel(kernel, grid, block, argv, lds_bytes, st) == hipSuccess ? TLIN_OK : TLIN_ERR_HIP;
}

// The kernels and the partition planning are written for MI355X: gfx950, 256 compute units in 8
// XCDs (kNumCU, kNumXCD).  Checked once per device ordinal, after argument validation and before
// the first launch on that device.
tlin_status check_device()
{
    static std::atomic<uint64_t> good{0}, bad{0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return TLIN_ERR_HIP;
    if (dev < 0 || dev >= 64) return TLIN_ERR_UNSUPPORTED;
    const uint64_t bit = (uint64_t)1 << dev;
    if (good.load(std::memory_order_acquire) & bit) return TLIN_OK;
    if (bad.load(std::memory_order_acquire) & bit) return TLIN_ERR_UNSUPPORTED;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, dev) != hipSuccess) return TLIN_ERR_HIP;
    const bool ok = strncmp(prop.gcnArchName, "gfx950", 6) == 0 && prop.multiProcessorCount == kNumCU;
    (ok ? good : bad).fetch_or(bit, std::memory_order_release);
    return ok ? TLIN_OK : TLIN_ERR_UNSUPPORTED;
}

struct Strides { int64_t b, h, r; };

// Kernel shape chosen for a bf16 problem: NW waves, QB query blocks of 32 rows per wave.
struct Shape { int nw, qb; int bm() const { return nw * qb * 32; } };

Shape wave_shape(int W)
{
    if (W > 128) return {8, 1};
    if (W > 64) return {4, 1};
    return {2, 1};
}

// Head dimensions other than 64 and 128 run in the next of the two kernel sizes: the kernels
// treat the missing columns of Q as zeros and do not store the extra output columns.
int dpad(int D) { return D <= 64 ? 64 : 128; }

// Keys per tile: 32 KB of K and V per tile in both kernels.  Query rows per workgroup: the same
// shapes for both input types.
int key_tile(int in_dtype, int) { return in_dtype == TLIN_F32 ? 32 : 64; }
// At head dimension 64 and below long windows stay with four waves too.  bf16: the pipelined body takes 153
// registers, so three waves fit a SIMD, which is three four-wave workgroups per compute unit but only one
// of eight waves (12 heads x 36, 256 window rows over 131072 / 999754 history rows: 0.135 / 0.911 ms per step
// against 0.148 / 0.940 ms with eight-wave workgroups).  fp32, the same with 164 registers: long unmasked windows
// take equal times (32 heads x 64, 512 rows over 20000: 482 us, eight waves 483), causal and ragged ones gain (16
// heads, 4096 causal rows: 240 against 310; 300 rows over 20000: 330 against 415).
Shape kernel_shape(int in_dtype, int W, int D)
{
    const Shape s = wave_shape(W);
    if (dpad(D) == 64 && s.nw == 8) return {4, 1};
    return s;
}
// A causal launch of its own with fewer than four eight-wave workgroups per compute unit runs in
// four-wave ones: two of them share a compute unit, so that the start of one (queries and first tiles
// on the way), its diagonal tiles, where half of the waves have nothing to do, and its output are hidden
// by the other's products (8 heads x 128, 1024 rows: 26.4 -> 18.6 us; 32 heads, 4096 rows: 162 -> 145 us).
// Beyond that the starts no longer count and the larger workgroup's fewer tile loads are ahead (32 heads,
// 8192 rows: 472 against 487 us).  fp32 the same: 16 heads x 128, 4096 rows 558 -> 436 us; 32 heads, 8192 rows
// 2834 with eight waves, 2873 with four.
Shape causal_shape(const tlin_params *p)
{
    const Shape s = kernel_shape(p->in_dtype, p->W, p->D);
    const int64_t blocks = (int64_t)p->B * p->H * ((p->W + s.bm() - 1) / s.bm());
    return s.nw == 8 && blocks < 4 * kNumCU ? Shape{4, 1} : s;
}
int query_block(int in_dtype, int W, int D) { return kernel_shape(in_dtype, W, D).bm(); }

// Workgroups the chip holds at once for a given kernel shape (LDS- and register-limited).
int resident_wgs(int in_dtype, Shape s, int D)
{
    if (in_dtype == TLIN_F32) {
        // fp32: LDS, 160 KB (D = 128: 48 KB of planes and 8 KB per wave, half of that at 64), and the registers
        // (f32_waves_per_simd)
        if (dpad(D) == 128) return kNumCU * (s.nw == 8 ? 1 : 2);
        return kNumCU * (s.nw == 4 ? 3 : 4);
    }
    // head dimension 64: tiles and register sets are half as large, three workgroups share a
    // compute unit (measured best for few heads); 128: an eight-wave workgroup fills a compute unit
    // alone (registers), two of the smaller ones share it (two-tile LDS ring of 64 KB each)
    if (dpad(D) == 64) return kNumCU * 3;
    return kNumCU * (s.nw == 8 ? 1 : 2);
}

// ---- measurement aid: per-kernel timing with HIP events on the launch stream
enum KernelClass { KC_HISTORY = 0, KC_WINDOW = 1, KC_MERGE = 2, KC_COUNT = 3 };

struct Timed { int cls; hipEvent_t start, stop; };
struct Profiler {
    std::atomic<bool> on{false};
    std::vector<Timed> used;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> pool;
    std::mutex mu;
} g_prof;

// Brackets one launch with events when profiling is enabled.
struct LaunchTimer {
    bool active = false;
    Timed t{};
    hipStream_t st;
    LaunchTimer(int cls, hipStream_t s) : st(s)
    {
        if (!g_prof.on) return;
        std::lock_guard<std::mutex> lk(g_prof.mu);
        if (g_prof.pool.empty()) {
            hipEvent_t a, b;
            if (hipEventCreate(&a) != hipSuccess) return;
            if (hipEventCreate(&b) != hipSuccess) { (void)hipEventDestroy(a); return; }
            g_prof.pool.push_back({a, b});
        }
        t = {cls, g_prof.pool.back().first, g_prof.pool.back().second};
        g_prof.pool.pop_back();
        active = hipEventRecord(t.start, st) == hipSuccess;
        if (!active) g_prof.pool.push_back({t.start, t.stop});
    }
    ~LaunchTimer()
    {
        if (!active) return;
        const bool ok = hipEventRecord(t.stop, st) == hipSuccess;
        std::lock_guard<std::mutex> lk(g_prof.mu);
        if (ok) g_prof.used.push_back(t);
        else g_prof.pool.push_back({t.start, t.stop});
    }
};

bool dense(const int64_t s[3]) { return s[0] == 0 && s[1] == 0 && s[2] == 0; }

Strides resolve(const int64_t s[3], int H, int rows, int D)
{
    if (dense(s)) return {(int64_t)H * rows * D, (int64_t)rows * D, (int64_t)D};
    return {s[0], s[1], s[2]};
}

tlin_status check_strides(const int64_t s[3], int D, int elem_bytes)
{
    const int per16 = 16 / elem_bytes;
    // rows are read in 16-byte pieces: a row holds D elements rounded up to whole pieces
    const int row_elems = (D + per16 - 1) / per16 * per16;
    if (dense(s)) return TLIN_OK;   // whether a dense layout is possible is checked per call, for the tensors it uses
    if (s[2] < row_elems || s[0] < 0 || s[1] < 0) return TLIN_ERR_INVALID_ARG;
    // a tile of 64 rows is addressed with 32-bit byte offsets
    if (s[2] * elem_bytes >= (int64_t)1 << 25) return TLIN_ERR_INVALID_ARG;
    if (s[0] % per16 || s[1] % per16 || s[2] % per16) return TLIN_ERR_INVALID_ARG;
    return TLIN_OK;
}

bool aligned(const void *p, size_t a) { return ((uintptr_t)p % a) == 0; }

// A tensor given without strides is dense, which needs rows of whole 16-byte pieces.
enum Tensor { T_Q = 1, T_KH = 2, T_VH = 4, T_KW = 8, T_VW = 16, T_O = 32 };
tlin_status check_dense_rows(const tlin_params *p, int used)
{
    const int in16 = 16 / (p->in_dtype == TLIN_F32 ? 4 : 2), out16 = 16 / (p->out_dtype == TLIN_F32 ? 4 : 2);
    const struct { int bit; const int64_t *s; int per16; } t[] = {
        {T_Q, p->q_stride, in16}, {T_KH, p->kh_stride, in16}, {T_VH, p->vh_stride, in16},
        {T_KW, p->kw_stride, in16}, {T_VW, p->vw_stride, in16}, {T_O, p->o_stride, out16}};
    for (const auto &x : t)
        if ((used & x.bit) && dense(x.s) && p->D % x.per16) return TLIN_ERR_INVALID_ARG;
    return TLIN_OK;
}

tlin_status check_common(const tlin_params *p, bool need_history, bool allow_empty_history)
{
    if (!p) return TLIN_ERR_INVALID_ARG;
    if (p->B < 1 || p->H < 1 || p->W < 1) return TLIN_ERR_INVALID_ARG;
    if (p->W > kMaxRows || p->N > kMaxRows) return TLIN_ERR_INVALID_ARG;   // tile counts and row indices are 32-bit
    if ((int64_t)p->B * p->H > (1 << 24)) return TLIN_ERR_INVALID_ARG;
    if (need_history && (p->N < (allow_empty_history ? 0 : 1))) return TLIN_ERR_INVALID_ARG;
    if (p->in_dtype != TLIN_F32 && p->in_dtype != TLIN_BF16) return TLIN_ERR_INVALID_ARG;
    if (p->out_dtype != TLIN_F32 && p->out_dtype != TLIN_BF16) return TLIN_ERR_INVALID_ARG;
    if (p->D < 8 || p->D > 128 || p->D % 4) return TLIN_ERR_UNSUPPORTED;
    if (!(p->scale > 0.f) || !isfinite(p->scale)) return TLIN_ERR_INVALID_ARG;
    if (p->num_splits < 0) return TLIN_ERR_INVALID_ARG;
    const int eb = p->in_dtype == TLIN_F32 ? 4 : 2;
    const int ob = p->out_dtype == TLIN_F32 ? 4 : 2;
    tlin_status st;
    if ((st = check_strides(p->q_stride, p->D, eb))) return st;
    if ((st = check_strides(p->kh_stride, p->D, eb))) return st;
    if ((st = check_strides(p->vh_stride, p->D, eb))) return st;
    if ((st = check_strides(p->kw_stride, p->D, eb))) return st;
    if ((st = check_strides(p->vw_stride, p->D, eb))) return st;
    if ((st = check_strides(p->o_stride, p->D, ob))) return st;
    return TLIN_OK;
}

// Most query rows of a streaming call (use_decode).
constexpr int kDecodeRowsF32 = 8, kDecodeRowsBf16 = 2;

// Partition plan for the history axis.
struct Plan { int nsplit, tiles_per_split; };

size_t ws_bytes_for(const tlin_params *p, int nparts)
{
    const size_t rows = (size_t)p->B * p->H * nparts * p->W;
    return rows * dpad(p->D) * sizeof(float) + 2 * rows * sizeof(float);
}

// Work items along the query axis: (head, query block) pairs.
int64_t query_items(const tlin_params *p, Shape s) { return (int64_t)p->B * p->H * ((p->W + s.bm() - 1) / s.bm()); }

// target: workgroups to aim at; round_down: partitions per item from which on a shape that shares a compute unit
// has them rounded down.
Plan plan_for_shape(const tlin_params *p, Shape s, int64_t target, int round_down)
{
    if (p->N < 1) return {0, 0};
    const int bn = key_tile(p->in_dtype, dpad(p->D));
    const int ntiles = (p->N + bn - 1) / bn;
    int want;
    if (p->num_splits > 0) {
        want = p->num_splits;
    } else {
        // Enough workgroups to occupy every compute unit, but at least 8 tiles per partition: the
        // merge reads every partial, and with short partitions it would cost more than they save.
        const int64_t base = query_items(p, s);
        want = (int)((target + base - 1) / base);
        // Rounded up, a few workgroups more than the chip holds would start when the others end and run a
        // whole partition's time beside idle compute units (1/f of the history against 2/(f + 1)).  Where several
        // share a compute unit the last ones run faster alone, but rounding down is ahead there too (100 heads x
        // 128, 64 rows over 28867, 6 -> 5 partitions: 306 -> 233 us; fp32, 80 heads x 96, 40 rows over 14338, 7 -> 6:
        // 375 -> 257; 40 heads x 36, 260 rows over 64379, 7 -> 6: 263 -> 225; 100 heads x 36, 200 rows over 89222, 4 -> 3:
        // 651 -> 626), only not from three to two where three or four share one (100 heads x 64, 260 rows over
        // 7212: 86 -> 89; fp32, 100 heads x 36, 384 rows over 13767: 677 -> 719).
        const int64_t down = target / base;
        if (base * want > target && down >= (target == kNumCU ? 2 : round_down)) want = (int)down;
        // (a handful of (head, query block) items cannot fill the chip anyway: there the partials
        // are few in total and short partitions pay)
        const int min_tiles = base <= 4 ? 2 : 8;
        const int cap = ntiles / min_tiles > 1 ? ntiles / min_tiles : 1;
        if (want > cap) want = cap;
        // (fp32 in four-wave workgroups, three to a compute unit up to 64 columns and at any head dimension where
        // history_shape chooses them: many heads would be cut into more partitions than a layer call has room for in the
        // library's own array; they are cut into as many as fit, 664 heads x 64, 128 rows into one)
        const bool more_places = p->in_dtype == TLIN_F32 && s.nw == 4 && (dpad(p->D) == 64 || p->W > 128);
        while (more_places && want > 1 && ws_bytes_for(p, want + 1) > TLIN_STATIC_WS_BYTES) --want;
    }
    if (want < 1) want = 1;
    if (want > ntiles) want = ntiles;
    if (want > 1024) want = 1024;
    const int tps = (ntiles + want - 1) / want;
    return {(ntiles + tps - 1) / tps, tps};   // no partition is empty
}

Plan plan_for_shape(const tlin_params *p, Shape s)
{
    // (two-wave workgroups of at most 32 columns, half of whose tiles' places are not loaded: a fourth one per
    // compute unit; 12 heads x 16, 40 rows over 999754: 246 -> 206 us, 100 heads, 40 rows over 9000: 27.6 -> 24.8; 36 and
    // more columns lose up to 4 % with it)
    const bool narrow = p->in_dtype == TLIN_BF16 && s.nw == 2 && p->D <= 32;
    const int64_t target = narrow ? 4 * kNumCU : resident_wgs(p->in_dtype, s, p->D);
    // (one and two bf16 rows keep the plan by which the lines of use_decode were measured)
    if (p->in_dtype == TLIN_BF16 && p->W <= kDecodeRowsBf16) return plan_for_shape(p, s, resident_wgs(p->in_dtype, s, p->D), 8);
    return plan_for_shape(p, s, target, target > 2 * kNumCU ? 3 : 2);
}

// Workgroup shape of a history.  At head dimensions above 64, of a window of 257 to 384 rows the second eight-wave
// workgroup holds up to four waves' rows and still keeps a compute unit to itself; three four-wave workgroups, two to a
// compute unit, leave nothing idle and cut the history into more partitions.  A tile takes the two 1.12 of an
// eight-wave workgroup's time (each loads it for itself), one that has the compute unit to itself 0.8, and every
// partition its partials' way out and back in: a tile is some 1.75 us at 128 columns (fp32, half as many keys: 5.2),
// partials move at 5 TB/s.  Measured, eight waves -> four: 16 heads x 96, 300 rows over 50021: 147 -> 132 us; 48 heads x
// 128, 300 rows over 33996 405 -> 327, 32 heads, 260 rows over 131072 857 -> 743; fp32, 48 heads x 96, 300 rows over
// 17905: 907 -> 701; the other way round 64 heads x 128 (fp32), 300 rows over 2212: 143 against 150, 24 heads x 128, 384
// rows over 6280: 43.7 against 44.6, x 96 42.5 against 44.7.
Shape history_shape(const tlin_params *p)
{
    const Shape s = kernel_shape(p->in_dtype, p->W, p->D), four = {4, 1};
    if (s.nw != 8 || p->W <= 256 || p->W > 384 || p->N < 1) return s;
    const Plan p8 = plan_for_shape(p, s), p4 = plan_for_shape(p, four);
    if (ws_bytes_for(p, p4.nsplit + 1) > TLIN_STATIC_WS_BYTES) return s;
    const double tile = (p->in_dtype == TLIN_F32 ? 5.2e-6 : 1.75e-6) * p->D / 128;
    const double partial = p->B * p->H * (double)p->W * dpad(p->D) * 8 / 5e12;
    const double factor = query_items(p, four) * p4.nsplit <= kNumCU ? 0.8 : 1.12;
    const double t8 = p8.tiles_per_split * tile + p8.nsplit * partial, t4 = factor * p4.tiles_per_split * tile + p4.nsplit * partial;
    return t4 < 0.95 * t8 ? four : s;
}

Plan plan_history(const tlin_params *p) { return plan_for_shape(p, history_shape(p)); }

// The cache-hit shape (a few query rows over a long history) runs in the streaming kernel of
// decode.h when called through tlin_history_attn.
//   fp32 inputs: the matrix-core path pays for a whole 32-row tile of products, and for splitting every key and
// value, whatever W is (16 rows over 32768 rows of 32 heads x 128: 223 us; eight rows over four times as many take
// 655 us here, one row 610).
//   bf16: three and four rows are a little faster in the two-wave matrix-core shape at head dimension
// 128 (0.309 against 0.323 ms over 131072 rows of 32 heads; both read at the rate of a plain
// non-temporal read stream) and up to twice as fast at the narrow ones (four rows over 99991 rows of 12
// heads x 16: 24 against 46 us, x 36: 35 against 48, x 96: 75 against 87).
// bf16 calls below head dimension 128 take the matrix-core path wherever the streaming kernel is not ahead.
bool decode_optional(const tlin_params *p) { return p->in_dtype == TLIN_BF16 && p->D != 128; }
bool use_decode(const tlin_params *p)
{
    if (p->N < 1024 || p->W > (p->in_dtype == TLIN_F32 ? kDecodeRowsF32 : kDecodeRowsBf16)) return false;
    if (!decode_optional(p)) return true;
    // (the lines below were measured with partitions rounded up: which calls weigh in fp32 stays with them)
    const int64_t bh = (int64_t)p->B * p->H, places = resident_wgs(p->in_dtype, kernel_shape(p->in_dtype, p->W, p->D), p->D);
    const int64_t blocks = bh * plan_for_shape(p, kernel_shape(p->in_dtype, p->W, p->D), places, 8).nsplit;
    // A history of one partition is one launch on the matrix-core path, which writes O itself and needs no
    // workspace; here it would be partials and a merge.  That path is ahead where rows are short (one row, 800
    // heads x 36, 1100 rows: 25.4 against 28.3 us here, 2048 heads x 64, 1024 rows: 83.3 against 88.5) and
    // behind above 64 columns (800 heads x 96, 1100 rows: 59.7 against 55.6), where only the calls that ask for
    // a single partition take it, or bring no workspace.
    if (blocks == bh && (p->D <= 64 || p->num_splits == 1)) return false;
    // Where the heads do not divide the matrix-core path's places and it would run a second round, this
    // kernel's smaller workgroups are ahead (100 heads, one row, 0.5 GB: x 68 126 against 90 us, x 96 109
    // against 85, x 48 92 against 86), with two rows only above 32 columns (250 heads x 16, 3000 rows: 15.5
    // against 21.9; 100 heads x 68 126 against 94): a lane group of eight takes a row of few columns, whose
    // scores and weights cost the same for each query.
    if (blocks > places) return p->W == 1 || p->D > 32;
    // Otherwise two rows are up to 19 % faster on the matrix-core path (99991 rows of 12 heads x 36: 35 against
    // 39 us; 131072 rows of 32 heads x 80: 198 against 203).  One row: with up to 64 bytes of columns that
    // path moves its tiles in pieces of lines and is behind (131072 rows of 32 heads x 16: 76 against 61 us; x
    // 32 in 1.2 GB the same).  Wider rows are within 5 % either way as long as the last-level cache holds most
    // of the keys and values (99991 rows of 12 heads x 36: 36 against 37; x 96: 75 against 74; calls of some
    // 25 us up to 15 % behind, 128 heads x 64, 4096 rows: 25 against 28) and stay here, where weights are
    // fp32; beyond, where HBM alone is the limit, that path's loads, which leave the missing chunks out, are
    // up to 7 % ahead (1.6 GB of 32 heads x 48: 252 against 262, x 80: 251 against 263).
    const int64_t kv_bytes = 4 * bh * p->N * p->D;
    return p->W == 1 && (p->D <= 32 || kv_bytes < ((int64_t)384 << 20));
}

// One workgroup per partition; four per compute unit (they are small: four waves; more partitions
// only lengthen the merge), at least 256 rows each.
Plan plan_decode(const tlin_params *p)
{
    const int ntiles = (p->N + 63) / 64;
    int want;
    if (p->num_splits > 0) {
        want = p->num_splits;
    } else {
        const int64_t bh = (int64_t)p->B * p->H;
        // rounded down where there are many per head: a last workgroup more than the compute units hold
        // evenly would run beside four others that have finished
        const int64_t all = 4 * (int64_t)kNumCU;
        want = (int)(all >= 8 * bh ? all / bh : (all + bh - 1) / bh);
        const int cap = ntiles / 4 > 1 ? ntiles / 4 : 1;
        if (want > cap) want = cap;
    }
    if (want < 1) want = 1;
    if (want > ntiles) want = ntiles;
    if (want > 1024) want = 1024;
    const int tps = (ntiles + want - 1) / want;
    return {(ntiles + tps - 1) / tps, tps};
}

// Sliding schedule: chunks of W rows over a sequence of N rows; every chunk's history is cut into
// the same number of partitions (their length grows with the chunk index).
struct SlidePlan { int nchunks, nsplit, nparts; };

SlidePlan plan_slide(const tlin_params *p)
{
    const int nchunks = (p->N + p->W - 1) / p->W;
    const int bn = key_tile(p->in_dtype, dpad(p->D));
    const int qblk = query_block(p->in_dtype, p->W, p->D);
    const int nqb = (p->W + qblk - 1) / qblk;
    int want;
    if (p->num_splits > 0) {
        want = p->num_splits;
    } else {
        // With many chunks the work items (head, chunk, query block) already outnumber the compute
        // units several times and the long ones start first; split only short sequences.
        const int64_t items = (int64_t)p->B * p->H * nqb * (nchunks > 1 ? nchunks - 1 : 1);
        const int64_t target = 2 * (int64_t)resident_wgs(p->in_dtype, kernel_shape(p->in_dtype, p->W, p->D), p->D);
        want = (int)((target + items - 1) / items);
    }
    // at least 4 tiles per partition in the longest history
    const int max_tiles = (int)(((int64_t)(nchunks - 1) * p->W + bn - 1) / bn);
    const int cap = max_tiles / 4 > 1 ? max_tiles / 4 : 1;
    if (want > cap) want = cap;
    if (want > 64) want = 64;
    if (want < 1) want = 1;
    return {nchunks, want, want + 1};
}

size_t slide_ws_bytes(const tlin_params *p, const SlidePlan &pl)
{
    const size_t rows = (size_t)p->B * p->H * pl.nchunks * pl.nparts * p->W;
    return rows * dpad(p->D) * sizeof(float) + 2 * rows * sizeof(float);
}

struct Workspace { float *O, *M, *L; };

Workspace carve(void *ws, const tlin_params *p, int nparts)
{
    const size_t rows = (size_t)p->B * p->H * nparts * p->W;
    float *base = (float *)ws;
    return {base, base + rows * dpad(p->D), base + rows * dpad(p->D) + rows};
}

// More than 64 KB of dynamic LDS has to be allowed once per kernel and device.  `done` is the
// calling kernel's own record: one bit per device ordinal.
tlin_status allow_lds(const void *kernel, int lds_bytes, std::atomic<uint64_t> &done)
{
    if (lds_bytes <= 64 * 1024) return TLIN_OK;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return TLIN_ERR_HIP;
    const uint64_t bit = (uint64_t)1 << dev;
    if (done.load(std::memory_order_acquire) & bit) return TLIN_OK;
    // two threads may both get here: setting the attribute twice is harmless
    if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes) != hipSuccess) return TLIN_ERR_HIP;
    done.fetch_or(bit, std::memory_order_release);
    return TLIN_OK;
}

// Tensors with a head dimension below the kernel's D run in variants of their own (template argument
// DP: the columns that are computed), so that the exact sizes carry none of their code and the narrow
// ones none of the products of columns they do not have: contraction steps are 16 columns wide,
// output blocks 32.  The lines lie where a step or a block is saved.  Measured, all columns of the
// kernel's D -> those of the variant: 300 window rows over 50021 history rows, 16 heads of 96: 0.174 ->
// 0.138 ms (with the waves that own no rows no longer computing, see attn_bf16_pipe_body); 256 rows over
// 999754, 12 heads of 36 (bound by the softmax arithmetic, not by the products): 0.866 -> 0.840 ms.
// f(integral_constant<int, DP>), DP = 0 for the exact size.
template <int D, typename F>
tlin_status with_columns(int dim, F &&f)
{
    if (dim == D) return f(std::integral_constant<int, 0>{});
    if constexpr (D == 128) {
        if (dim <= 96) return f(std::integral_constant<int, 96>{});
    } else {
        if (dim <= 32) return f(std::integral_constant<int, 32>{});
        if (dim <= 48) return f(std::integral_constant<int, 48>{});
    }
    return f(std::integral_constant<int, D>{});
}

template <int D, int NW, int QB, bool CAUSAL, int NSTAGE, bool RESIDENT, int DP, bool NT, bool LSE = false>
tlin_status launch_bf16_kernel(const AttnArgs &a, int grid, hipStream_t st)
{
    constexpr int lds_bytes = 2 * NSTAGE * 64 * D * 2;
    static_assert(lds_bytes <= 160 * 1024, "LDS ring exceeds the 160 KB of a gfx950 compute unit");
    auto kernel = attn_bf16_kernel<D, NW, QB, CAUSAL, NSTAGE, RESIDENT, DP, NT, LSE>;
    static std::atomic<uint64_t> lds_allowed{0};
    if (allow_lds((const void *)kernel, lds_bytes, lds_allowed) != TLIN_OK) return TLIN_ERR_HIP;
    return launch_kernel((const void *)kernel, dim3(grid), dim3(NW * 64), lds_bytes, st, a);
}

// The non-temporal variant exists for the pipelined shapes of a history only: causal launches never
// stream (launch_attn).
template <int D, int NW, int QB, bool CAUSAL, int NSTAGE, bool RESIDENT = false>
tlin_status launch_bf16_shape(const AttnArgs &a, int grid, hipStream_t st)
{
    return with_columns<D>(a.D, [&](auto dp) {
        constexpr int DP = decltype(dp)::value;
        if constexpr (use_pipe_body<D, NW, QB, CAUSAL, NSTAGE, RESIDENT>()) {
            if constexpr (!CAUSAL) {
                if (a.stream_once) return launch_bf16_kernel<D, NW, QB, CAUSAL, NSTAGE, RESIDENT, DP, true>(a, grid, st);
            } else if constexpr (D == 64) {
                if (a.lse) return launch_bf16_kernel<D, NW, QB, CAUSAL, NSTAGE, RESIDENT, DP, false, true>(a, grid, st);
            }
        }
        return launch_bf16_kernel<D, NW, QB, CAUSAL, NSTAGE, RESIDENT, DP, false>(a, grid, st);
    });
}

template <int D, int T1, int TMAX>
tlin_status launch_resident_pipe(const AttnArgs &a, int grid, hipStream_t st)
{
    // the resident tiles and, behind them, 4 KB per wave for turning the output rows
    constexpr int lds_bytes = 2 * TMAX * 64 * D * 2 + 8 * 4096;
    static_assert(lds_bytes <= 160 * 1024, "resident tiles exceed the 160 KB of a gfx950 compute unit");
    return with_columns<D>(a.D, [&](auto dp) {
        constexpr int DP = decltype(dp)::value;
        if constexpr (DP == 0) {
            if (a.NK <= (T1 - 1) * 64) {
                static std::atomic<uint64_t> lds_allowed_odd{0};
                const void *kernel = (const void *)attn_bf16_resident_pipe_kernel<D, T1, TMAX, DP, true>;
                if (allow_lds(kernel, lds_bytes, lds_allowed_odd) != TLIN_OK) return TLIN_ERR_HIP;
                return launch_kernel(kernel, dim3(grid), dim3(512), lds_bytes, st, a);
            }
        }
        static std::atomic<uint64_t> lds_allowed{0};
        const void *kernel = (const void *)attn_bf16_resident_pipe_kernel<D, T1, TMAX, DP>;
        if (allow_lds(kernel, lds_bytes, lds_allowed) != TLIN_OK) return TLIN_ERR_HIP;
        return launch_kernel(kernel, dim3(grid), dim3(512), lds_bytes, st, a);
    });
}

// Ring depth per kernel shape (measured): a compute unit keeps little more than one tile of loads
// in flight, so a deep ring only makes waves wait at the issue of loads that cannot start yet.  Two
// stages also let two of the smaller workgroups share a compute unit.
template <int D, bool CAUSAL>
tlin_status launch_bf16(const AttnArgs &a, Shape s, int grid, hipStream_t st)
{
    if constexpr (D == 128) {
        if (s.nw == 8) return launch_bf16_shape<D, 8, 1, CAUSAL, 2>(a, grid, st);
    }
    if (s.nw == 4) return launch_bf16_shape<D, 4, 1, CAUSAL, 2>(a, grid, st);
    return launch_bf16_shape<D, 2, 1, CAUSAL, 2>(a, grid, st);
}

// fp32 kernel: three bf16 planes of a 32-key tile of K and of V, and part 2 of the waves' queries.
template <int D, int DP> constexpr int f32_lds_bytes(int nw) { return 2 * 3 * 32 * D * 2 + nw * ((DP ? DP : D) / 16) * 1024; }

template <int D, int NW, bool CAUSAL>
tlin_status launch_f32_shape(const AttnArgs &a, int grid, hipStream_t st)
{
    return with_columns<D>(a.D, [&](auto dp) {
        constexpr int DP = decltype(dp)::value, lds_bytes = f32_lds_bytes<D, DP>(NW);
        static_assert(lds_bytes <= 160 * 1024, "fp32 planes exceed the 160 KB of a gfx950 compute unit");
        static std::atomic<uint64_t> lds_allowed{0};
        const void *kernel = (const void *)attn_f32_kernel<D, NW, CAUSAL, DP>;
        if (allow_lds(kernel, lds_bytes, lds_allowed) != TLIN_OK) return TLIN_ERR_HIP;
        return launch_kernel(kernel, dim3(grid), dim3(NW * 64), lds_bytes, st, a);
    });
}
template <int D, bool CAUSAL>
tlin_status launch_f32(const AttnArgs &a, Shape s, int grid, hipStream_t st)
{
    if constexpr (D == 128) {
        if (s.nw == 8) return launch_f32_shape<D, 8, CAUSAL>(a, grid, st);
    }
    if (s.nw == 4) return launch_f32_shape<D, 4, CAUSAL>(a, grid, st);
    return launch_f32_shape<D, 2, CAUSAL>(a, grid, st);
}

// Window blocks launched behind the history blocks run when the compute units are already taken, as
// a tail of their own (1.5 to 5 % of the larger workloads' kernel time).  Where the partitions are
// long enough to absorb it, partition 0's workgroup computes the window block too and gets that
// much less history (partition_tiles): every partition stays non-empty when the tiles number at
// least nsplit^2 and a partition is longer than such a block.  Below four blocks' length that is worth it
// only where the chip does not hold the window blocks beside all of the history blocks anyway
// (layer calls, 300 rows over 20000, 8 heads x 128: fp32 427 -> 343 us, bf16 66 -> 51; 512 rows over 8192,
// 32 heads x 128: fp32 665 -> 585, bf16 95 -> 84).  BN, quarters: the kernel's
// keys per tile and cost ratio (window_block_cost).
bool fuses_window(int in_dtype, const PairArgs &f, Shape s, int BN, int quarters)
{
    const int tiles = (f.hist.NK + BN - 1) / BN, ns = f.hist.nsplit;
    const int cost = window_block_cost(f.hist.W, f.hist.nqb - 1, s.bm(), BN, quarters);
    if (f.hist.nchunks != 0 || f.n_win_blocks <= 0 || ns < 2 || tiles < ns * ns) return false;
    const bool full = f.n_hist_blocks + f.n_win_blocks > resident_wgs(in_dtype, s, f.hist.D);
    return tiles / ns >= (full ? cost + 2 : 4 * cost);
}

template <int D, int NW>
tlin_status launch_f32_pair_shape(const PairArgs &f, hipStream_t st)
{
    return with_columns<D>(f.hist.D, [&](auto dp) {
        constexpr int DP = decltype(dp)::value, lds_bytes = f32_lds_bytes<D, DP>(NW);
        static std::atomic<uint64_t> lds_allowed{0};
        const void *kernel = (const void *)attn_f32_pair_kernel<D, NW, DP>;
        if (allow_lds(kernel, lds_bytes, lds_allowed) != TLIN_OK) return TLIN_ERR_HIP;
        return launch_kernel(kernel, dim3(f.n_hist_blocks + f.n_win_blocks), dim3(NW * 64), lds_bytes, st, f);
    });
}
template <int D>
tlin_status launch_f32_pair(const PairArgs &f, Shape s, hipStream_t st)
{
    PairArgs g = f;
    if (fuses_window(TLIN_F32, f, s, 32, 4)) {
        g.hist.fuse_window = 1;
        g.n_win_blocks = 0;
    }
    if constexpr (D == 128) {
        if (s.nw == 8) return launch_f32_pair_shape<D, 8>(g, st);
    }
    if (s.nw == 4) return launch_f32_pair_shape<D, 4>(g, st);
    return launch_f32_pair_shape<D, 2>(g, st);
}

// The resident variant pays when the key/value side fits in LDS as a whole and every workgroup
// has several query blocks to walk over: long query side, short unsplit key side.
bool use_resident(const tlin_params *p, bool causal, const AttnArgs &a)
{
    if (causal || p->in_dtype != TLIN_BF16 || !a.direct || a.nsplit != 1) return false;
    if (p->W <= 128) return false;
    const int ntiles = (a.NK + 63) / 64;
    const int64_t blocks = (int64_t)p->B * p->H * ((p->W + 255) / 256);      // the resident kernels are eight-wave ones
    if (blocks < 4 * (int64_t)kNumCU) return false;
    if (dpad(p->D) == 128) return ntiles <= 4;
    // Head dimensions up to 64 run the unpipelined body here, which the pipelined ring passes where a block has more
    // than two tiles (four above 48 columns) to hide its start behind: 32 heads, 131072 rows over 400 keys, x 64 698
    // -> 629 us, x 36 649 -> 550, over 256 keys x 36 407 -> 375, but x 64 419 -> 439, and over 128 x 36 250 -> 286.
    // Three tiles of 40 to 48 columns only where a workgroup has few blocks to walk over: over 192 keys x 48, 32 heads,
    // 131072 rows (64 blocks) 305 against 358 us in the ring, 30000 rows (14) 71 against 74, 12 heads, 50000 rows
    // (9) 49.7 against 48.5.
    if (ntiles == 3 && p->D >= 40 && p->D <= 48) return blocks >= 14 * (int64_t)kNumCU;
    return ntiles <= (p->D > 48 ? 4 : 2);
}

// K/V rows of a history are read by exactly one workgroup when the window is a single query block,
// and stream through the caches without reuse when they exceed the last-level cache (256 MB)
// several times over: then the tile loads carry the non-temporal hint.  Not for the sliding
// schedule, whose chunks re-read each other's history.
bool streams_once(const tlin_params *p, const AttnArgs &a, int nqb)
{
    const int64_t kv_bytes = 2 * (int64_t)p->B * p->H * a.NK * p->D * 2;
    return p->in_dtype == TLIN_BF16 && nqb == 1 && a.nchunks == 0 && kv_bytes >= ((int64_t)192 << 20);
}

// Launch one partial-attention kernel over `nsplit` key partitions (or the causal window).
tlin_status launch_attn(const tlin_params *p, bool causal, AttnArgs a, hipStream_t st)
{
    const Shape s = causal ? causal_shape(p) : a.nchunks ? kernel_shape(p->in_dtype, p->W, p->D) : history_shape(p);
    a.nqb = (p->W + s.bm() - 1) / s.bm();
    a.stream_once = !causal && streams_once(p, a, a.nqb);
    if (use_resident(p, causal, a)) {
        // one workgroup per compute unit, spread evenly over the heads
        a.nqb = (p->W + 255) / 256;
        const int64_t bh = (int64_t)p->B * p->H;
        // (rounded down: twelve heads in 264 workgroups left eight for a second round; 50000 rows over 256 keys of 12
        // heads x 128: 129 -> 93 us)
        int64_t g = kNumCU / bh;
        if (g < 1) g = 1;
        if (g > a.nqb) g = a.nqb;
        a.q_groups = (int)g;
        const int64_t grid64 = bh * g;
        if (grid64 > 0x7fffffff) return TLIN_ERR_INVALID_ARG;
        LaunchTimer timer(KC_HISTORY, st);
        const int ntiles = (a.NK + 63) / 64;
        // (three tiles pay for the masked fourth one where a workgroup has a dozen blocks or more: 32 heads, 131072
        // rows over 180 keys 657 -> 632 us, 8200 rows 43 -> 46)
        const bool odd = p->D == 128 && (ntiles == 1 || a.nqb >= 12 * a.q_groups);
        if (dpad(p->D) == 128 && (ntiles % 2 == 0 || odd)) return ntiles > 2 ? launch_resident_pipe<128, 4, 4>(a, (int)grid64, st) : launch_resident_pipe<128, 2, 4>(a, (int)grid64, st);
        return dpad(p->D) == 128 ? launch_bf16_shape<128, 8, 1, false, 4, true>(a, (int)grid64, st) : launch_bf16_shape<64, 8, 1, false, 4, true>(a, (int)grid64, st);
    }
    const int64_t grid64 = (int64_t)p->B * p->H * a.nqb * a.nsplit * (a.nchunks ? a.nchunks : 1);
    if (grid64 > 0x7fffffff) return TLIN_ERR_INVALID_ARG;
    const int grid = (int)grid64;
    // every workgroup of a causal launch on the chip at once, up to two to a compute unit, whole heads to an
    // XCD: see decode_problem
    const int64_t heads = (int64_t)p->B * p->H;
    a.causal_flip = causal && s.nw == 4 && grid > kNumCU && grid <= 2 * kNumCU && heads % kNumXCD == 0 ? (int)(heads / kNumXCD) : 0;
    LaunchTimer timer(causal ? KC_WINDOW : KC_HISTORY, st);
    if (p->in_dtype == TLIN_BF16) {
        if (dpad(p->D) == 128) return causal ? launch_bf16<128, true>(a, s, grid, st) : launch_bf16<128, false>(a, s, grid, st);
        return causal ? launch_bf16<64, true>(a, s, grid, st) : launch_bf16<64, false>(a, s, grid, st);
    }
    if (dpad(p->D) == 128) return causal ? launch_f32<128, true>(a, s, grid, st) : launch_f32<128, false>(a, s, grid, st);
    return causal ? launch_f32<64, true>(a, s, grid, st) : launch_f32<64, false>(a, s, grid, st);
}

template <typename T, int DK, bool PAD>
const void *decode_kernel_for(int W)
{
    if constexpr (sizeof(T) == 4) {          // bf16 calls have at most two rows (kDecodeRowsBf16)
        if (W > 4) return (const void *)decode_kernel<T, DK, 8, PAD>;
        if (W > 2) return (const void *)decode_kernel<T, DK, 4, PAD>;
    }
    return W == 1 ? (const void *)decode_kernel<T, DK, 1, PAD> : (const void *)decode_kernel<T, DK, 2, PAD>;
}
template <typename T>
const void *decode_kernel_for(int W, int D)
{
    if (dpad(D) == 128) return D == 128 ? decode_kernel_for<T, 128, false>(W) : decode_kernel_for<T, 128, true>(W);
    return D == 64 ? decode_kernel_for<T, 64, false>(W) : decode_kernel_for<T, 64, true>(W);
}

tlin_status launch_decode(const tlin_params *p, const AttnArgs &a, hipStream_t st)
{
    const int64_t grid64 = (int64_t)p->B * p->H * a.nsplit;
    if (grid64 > 0x7fffffff) return TLIN_ERR_INVALID_ARG;
    LaunchTimer timer(KC_HISTORY, st);
    const void *kernel = p->in_dtype == TLIN_F32 ? decode_kernel_for<float>(p->W, p->D) : decode_kernel_for<__bf16>(p->W, p->D);
    return launch_kernel(kernel, dim3((unsigned)grid64), dim3(256), 0, st, a);
}

tlin_status launch_merge(const tlin_params *p, MergeArgs m, hipStream_t st)
{
    m.H = p->H;
    m.W = p->W;
    m.out_bf16 = p->out_dtype == TLIN_BF16;
    m.D = p->D;
    const int64_t total = (int64_t)p->B * p->H * (m.nchunks ? m.seq_rows : p->W);
    if (total > 0x7fffffff) return TLIN_ERR_INVALID_ARG;
    m.total_rows = (int)total;
    // threads per (row, 4 columns) item: more when a row has many partials to walk, and a block of 1024
    // threads to itself when there are too few rows to fill the chip otherwise
    const int joint = m.nhist + (m.has_window && m.joint ? 1 : 0);
    const int tpr = dpad(p->D) / 4;
    const int sl = joint <= 6 ? 1 : joint <= 16 ? 4 : joint > 32 && total <= 2 * kNumCU ? 1024 / tpr : 8;
    const int nt = tpr * sl > 256 ? tpr * sl : 256, rpb = nt / (tpr * sl);
    const int grid = (int)((total + rpb - 1) / rpb);
    LaunchTimer timer(KC_MERGE, st);
    const void *kernel;
    if (tpr == 32) kernel = sl == 32 ? (const void *)merge_kernel<128, 32> : sl == 8 ? (const void *)merge_kernel<128, 8> : sl == 4 ? (const void *)merge_kernel<128, 4> : (const void *)merge_kernel<128, 1>;
    else kernel = sl == 64 ? (const void *)merge_kernel<64, 64> : sl == 8 ? (const void *)merge_kernel<64, 8> : sl == 4 ? (const void *)merge_kernel<64, 4> : (const void *)merge_kernel<64, 1>;
    return launch_kernel(kernel, dim3(grid), dim3(nt), 0, st, m);
}

AttnArgs base_args(const tlin_params *p, const void *Q, const void *K, const void *V, const int64_t ks[3],
                   const int64_t vs[3], int nk)
{
    AttnArgs a = {};
    a.Q = Q; a.K = K; a.V = V;
    const Strides q = resolve(p->q_stride, p->H, p->W, p->D);
    const Strides k = resolve(ks, p->H, nk, p->D);
    const Strides v = resolve(vs, p->H, nk, p->D);
    a.q_sb = q.b; a.q_sh = q.h; a.q_sr = q.r;
    a.k_sb = k.b; a.k_sh = k.h; a.k_sr = k.r;
    a.v_sb = v.b; a.v_sh = v.h; a.v_sr = v.r;
    a.H = p->H; a.W = p->W; a.NK = nk;
    a.D = p->D;
    a.nsplit = 1; a.tiles_per_split = 0x3fffffff;
    a.scale = p->scale;
    a.c = p->scale * 1.4426950408889634f;
    return a;
}

void set_direct(AttnArgs &a, const tlin_params *p, void *O, float *lse)
{
    const Strides o = resolve(p->o_stride, p->H, p->W, p->D);
    a.direct = 1;
    a.O = O; a.o_sb = o.b; a.o_sh = o.h; a.o_sr = o.r;
    a.lse = lse;
    a.out_bf16 = p->out_dtype == TLIN_BF16;
}

void set_partial(AttnArgs &a, const Workspace &w, int nparts, int part0)
{
    a.direct = 0;
    a.Opart = w.O; a.Mpart = w.M; a.Lpart = w.L;
    a.nparts = nparts; a.part0 = part0;
}

MergeArgs merge_args(const tlin_params *p, const Workspace &w, int nparts, int nhist, bool has_window, bool joint,
                     void *O, float *lse)
{
    MergeArgs m = {};
    m.Opart = w.O; m.Mpart = w.M; m.Lpart = w.L;
    m.nparts = nparts; m.nhist = nhist; m.has_window = has_window; m.joint = joint;
    const Strides o = resolve(p->o_stride, p->H, p->W, p->D);
    m.O = O; m.o_sb = o.b; m.o_sh = o.h; m.o_sr = o.r;
    m.lse = lse;
    return m;
}

template <int D, int NW, int DP, bool NT>
tlin_status launch_pair_kernel(const PairArgs &f, hipStream_t st)
{
    constexpr int lds_bytes = 2 * 2 * 64 * D * 2;
    static_assert(lds_bytes <= 160 * 1024, "LDS ring exceeds the 160 KB of a gfx950 compute unit");
    auto kernel = attn_bf16_pair_kernel<D, NW, DP, NT>;
    static std::atomic<uint64_t> lds_allowed{0};
    if (allow_lds((const void *)kernel, lds_bytes, lds_allowed) != TLIN_OK) return TLIN_ERR_HIP;
    if (fuses_window(TLIN_BF16, f, Shape{NW, 1}, 64, 5)) {
        PairArgs g = f;
        g.hist.fuse_window = 1;
        g.n_win_blocks = 0;
        return launch_kernel((const void *)kernel, dim3(g.n_hist_blocks), dim3(NW * 64), lds_bytes, st, g);
    }
    return launch_kernel((const void *)kernel, dim3(f.n_hist_blocks + f.n_win_blocks), dim3(NW * 64), lds_bytes, st, f);
}

template <int D, int NW>
tlin_status launch_pair_shape(const PairArgs &f, hipStream_t st)
{
    return with_columns<D>(f.hist.D, [&](auto dp) {
        constexpr int DP = decltype(dp)::value;
        return f.hist.stream_once ? launch_pair_kernel<D, NW, DP, true>(f, st) : launch_pair_kernel<D, NW, DP, false>(f, st);
    });
}

// History partials and window partial of the same rows: one launch for both problem sets.
tlin_status launch_partials(const tlin_params *p, const AttnArgs &ah, const AttnArgs &aw, hipStream_t hs)
{
    const Shape s = ah.nchunks ? kernel_shape(p->in_dtype, p->W, p->D) : history_shape(p);
    const int nqb = (p->W + s.bm() - 1) / s.bm();
    const int64_t per_set = (int64_t)p->B * p->H * nqb * (ah.nchunks ? ah.nchunks : 1);
    const int64_t nh = per_set * ah.nsplit, nw = per_set;
    if (nh + nw <= 0x7fffffff) {
        PairArgs f = {};
        f.hist = ah;
        f.win = aw;
        f.hist.nqb = f.win.nqb = nqb;
        f.hist.stream_once = streams_once(p, ah, nqb);
        f.n_hist_blocks = (int)nh;
        f.n_win_blocks = (int)nw;
        LaunchTimer timer(KC_HISTORY, hs);
        if (p->in_dtype == TLIN_F32) return dpad(p->D) == 128 ? launch_f32_pair<128>(f, s, hs) : launch_f32_pair<64>(f, s, hs);
        if (dpad(p->D) == 128) {
            if (s.nw == 8) return launch_pair_shape<128, 8>(f, hs);
            if (s.nw == 4) return launch_pair_shape<128, 4>(f, hs);
            return launch_pair_shape<128, 2>(f, hs);
        }
        if (s.nw == 4) return launch_pair_shape<64, 4>(f, hs);
        // (ahead of the classic body with a ring of three tiles: 32 heads x 64, 64 rows over 60000: 103 -> 87 us, 12
        // heads x 36, 64 rows over 999754: 409 -> 334, sliding schedule of 8 heads x 64, 8000 rows in chunks of 64:
        // 135 -> 100)
        return launch_pair_shape<64, 2>(f, hs);
    }
    tlin_status st;
    if ((st = launch_attn(p, false, ah, hs))) return st;
    return launch_attn(p, true, aw, hs);
}

tlin_status check_ws(const void *ws, size_t have, size_t need)
{
    if (need == 0) return TLIN_OK;
    if (!ws || !aligned(ws, 256) || have < need) return TLIN_ERR_WORKSPACE;
    return TLIN_OK;
}

// Argument checks of the layer call (host only).
tlin_status check_layer_args(const tlin_params *p, const void *Q_win, const void *K_hist, const void *V_hist,
                             const void *K_win, const void *V_win, const void *O)
{
    tlin_status st = check_common(p, true, true);
    if (st) return st;
    if ((st = check_dense_rows(p, T_Q | T_KW | T_VW | T_O | (p->N > 0 ? T_KH | T_VH : 0)))) return st;
    if (p->combine != TLIN_COMBINE_SUM && p->combine != TLIN_COMBINE_JOINT) return TLIN_ERR_INVALID_ARG;
    if (!Q_win || !K_win || !V_win || !O) return TLIN_ERR_INVALID_ARG;
    if (p->N > 0 && (!K_hist || !V_hist)) return TLIN_ERR_INVALID_ARG;
    if (!aligned(Q_win, 16) || !aligned(K_win, 16) || !aligned(V_win, 16) || !aligned(O, 16)) return TLIN_ERR_INVALID_ARG;
    if (p->N > 0 && (!aligned(K_hist, 16) || !aligned(V_hist, 16))) return TLIN_ERR_INVALID_ARG;
    return TLIN_OK;
}

// The launches of a layer call; arguments and workspace have been checked.
tlin_status layer_attn(const tlin_params *p, const void *Q_win, const void *K_hist, const void *V_hist,
                       const void *K_win, const void *V_win, void *O, void *ws, hipStream_t hs)
{
    if (p->N == 0) {
        // Empty history: the layer is the window causal attention in both combine modes.
        AttnArgs a = base_args(p, Q_win, K_win, V_win, p->kw_stride, p->vw_stride, p->W);
        set_direct(a, p, O, nullptr);
        return launch_attn(p, true, a, hs);
    }
    const Plan pl = plan_history(p);
    const int nparts = pl.nsplit + 1;
    const Workspace w = carve(ws, p, nparts);

    AttnArgs ah = base_args(p, Q_win, K_hist, V_hist, p->kh_stride, p->vh_stride, p->N);
    ah.nsplit = pl.nsplit;
    ah.tiles_per_split = pl.tiles_per_split;
    set_partial(ah, w, nparts, 0);
    AttnArgs aw = base_args(p, Q_win, K_win, V_win, p->kw_stride, p->vw_stride, p->W);
    set_partial(aw, w, nparts, pl.nsplit);
    tlin_status st;
    if ((st = launch_partials(p, ah, aw, hs))) return st;
    return launch_merge(p, merge_args(p, w, nparts, pl.nsplit, true, p->combine == TLIN_COMBINE_JOINT, O, nullptr), hs);
}

// The launches of a history call in the streaming kernel; arguments and workspace have been checked.
tlin_status history_attn_streamed(const tlin_params *p, AttnArgs a, Plan pd, void *O, float *lse, void *ws, hipStream_t hs)
{
    tlin_status st;
    if ((st = check_device())) return st;
    const Workspace w = carve(ws, p, pd.nsplit);
    a.nsplit = pd.nsplit;
    a.tiles_per_split = pd.tiles_per_split;
    set_partial(a, w, pd.nsplit, 0);
    if ((st = launch_decode(p, a, hs))) return st;
    return launch_merge(p, merge_args(p, w, pd.nsplit, pd.nsplit, false, true, O, lse), hs);
}

// Address of this device's copy of `scratch`, looked up once per device ordinal with that device
// current (every GPU holds its own copy of the array at its own address).
tlin_status static_scratch(void **out)
{
    static std::mutex mu;
    static void *addr[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return TLIN_ERR_HIP;
    std::lock_guard<std::mutex> lk(mu);
    if (!addr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return TLIN_ERR_HIP;
        addr[dev] = ptr;
    }
    *out = addr[dev];
    return TLIN_OK;
}

}  // namespace

extern "C" {

size_t tlin_workspace_bytes(const tlin_params *p)
{
    if (check_common(p, true, true) != TLIN_OK) return 0;
    const Plan pl = plan_history(p);
    size_t need = ws_bytes_for(p, pl.nsplit + 1);
    if (use_decode(p)) {
        const size_t dec = ws_bytes_for(p, plan_decode(p).nsplit);
        if (dec > need) need = dec;
    }
    return need;
}

int32_t tlin_num_splits(const tlin_params *p)
{
    if (check_common(p, true, false) != TLIN_OK) return 0;
    return use_decode(p) ? plan_decode(p).nsplit : plan_history(p).nsplit;
}

tlin_status tlin_history_attn(const tlin_params *p, const void *Q_win, const void *K_hist, const void *V_hist,
                              void *O, float *lse, void *ws, size_t ws_bytes, void *stream)
{
    tlin_status st = check_common(p, true, false);
    if (st) return st;
    if ((st = check_dense_rows(p, T_Q | T_KH | T_VH | T_O))) return st;
    if (!Q_win || !K_hist || !V_hist || !O) return TLIN_ERR_INVALID_ARG;
    if (!aligned(Q_win, 16) || !aligned(K_hist, 16) || !aligned(V_hist, 16) || !aligned(O, 16)) return TLIN_ERR_INVALID_ARG;
    if (lse && !aligned(lse, 4)) return TLIN_ERR_INVALID_ARG;
    hipStream_t hs = (hipStream_t)stream;
    AttnArgs a = base_args(p, Q_win, K_hist, V_hist, p->kh_stride, p->vh_stride, p->N);
    if (use_decode(p)) {
        const Plan pd = plan_decode(p);
        // (its partitions may be more than the matrix-core path's, or that path's single one needs no workspace: a
        // call that brings only what that path needs is served by it)
        st = check_ws(ws, ws_bytes, ws_bytes_for(p, pd.nsplit));
        if (st && !decode_optional(p)) return st;
        if (!st) return history_attn_streamed(p, a, pd, O, lse, ws, hs);
    }
    const Plan pl = plan_history(p);
    a.nsplit = pl.nsplit;
    a.tiles_per_split = pl.tiles_per_split;
    if (pl.nsplit == 1) {
        if ((st = check_device())) return st;
        set_direct(a, p, O, lse);
        return launch_attn(p, false, a, hs);
    }
    if ((st = check_ws(ws, ws_bytes, ws_bytes_for(p, pl.nsplit)))) return st;
    if ((st = check_device())) return st;
    const Workspace w = carve(ws, p, pl.nsplit);
    set_partial(a, w, pl.nsplit, 0);
    if ((st = launch_attn(p, false, a, hs))) return st;
    return launch_merge(p, merge_args(p, w, pl.nsplit, pl.nsplit, false, true, O, lse), hs);
}

tlin_status tlin_window_causal_attn(const tlin_params *p, const void *Q_win, const void *K_win, const void *V_win,
                                    void *O, float *lse, void *ws, size_t ws_bytes, void *stream)
{
    (void)ws;
    (void)ws_bytes;
    tlin_status st = check_common(p, false, false);
    if (st) return st;
    if ((st = check_dense_rows(p, T_Q | T_KW | T_VW | T_O))) return st;
    if (!Q_win || !K_win || !V_win || !O) return TLIN_ERR_INVALID_ARG;
    if (!aligned(Q_win, 16) || !aligned(K_win, 16) || !aligned(V_win, 16) || !aligned(O, 16)) return TLIN_ERR_INVALID_ARG;
    if (lse && !aligned(lse, 4)) return TLIN_ERR_INVALID_ARG;
    if ((st = check_device())) return st;
    AttnArgs a = base_args(p, Q_win, K_win, V_win, p->kw_stride, p->vw_stride, p->W);
    set_direct(a, p, O, lse);
    return launch_attn(p, true, a, (hipStream_t)stream);
}

tlin_status tlin_layer_attn(const tlin_params *p, const void *Q_win, const void *K_hist, const void *V_hist,
                            const void *K_win, const void *V_win, void *O, void *ws, size_t ws_bytes, void *stream)
{
    tlin_status st = check_layer_args(p, Q_win, K_hist, V_hist, K_win, V_win, O);
    if (st) return st;
    if (p->N > 0 && (st = check_ws(ws, ws_bytes, ws_bytes_for(p, plan_history(p).nsplit + 1)))) return st;
    if ((st = check_device())) return st;
    return layer_attn(p, Q_win, K_hist, V_hist, K_win, V_win, O, ws, (hipStream_t)stream);
}

tlin_status tlin_layer_attn_static_ws(const tlin_params *p, const void *Q_win, const void *K_hist, const void *V_hist,
                                      const void *K_win, const void *V_win, void *O, void *stream)
{
    tlin_status st = check_layer_args(p, Q_win, K_hist, V_hist, K_win, V_win, O);
    if (st) return st;
    const size_t need = p->N > 0 ? ws_bytes_for(p, plan_history(p).nsplit + 1) : 0;
    if (need > TLIN_STATIC_WS_BYTES) return TLIN_ERR_WORKSPACE;
    if ((st = check_device())) return st;
    void *ws = nullptr;
    if (need > 0 && (st = static_scratch(&ws))) return st;
    return layer_attn(p, Q_win, K_hist, V_hist, K_win, V_win, O, ws, (hipStream_t)stream);
}

size_t tlin_slide_workspace_bytes(const tlin_params *p)
{
    if (check_common(p, true, false) != TLIN_OK) return 0;
    const SlidePlan pl = plan_slide(p);
    return slide_ws_bytes(p, pl);
}

tlin_status tlin_slide_layer_attn(const tlin_params *p, const void *Q, const void *K_hist, const void *V_hist,
                                  const void *K_win, const void *V_win, void *O, void *ws, size_t ws_bytes,
                                  void *stream)
{
    tlin_status st = check_common(p, true, false);
    if (st) return st;
    if ((st = check_dense_rows(p, T_Q | T_KH | T_VH | T_KW | T_VW | T_O))) return st;
    if (p->combine != TLIN_COMBINE_SUM && p->combine != TLIN_COMBINE_JOINT) return TLIN_ERR_INVALID_ARG;
    if (!Q || !K_hist || !V_hist || !K_win || !V_win || !O) return TLIN_ERR_INVALID_ARG;
    if (!aligned(Q, 16) || !aligned(K_hist, 16) || !aligned(V_hist, 16) || !aligned(K_win, 16) || !aligned(V_win, 16) ||
        !aligned(O, 16))
        return TLIN_ERR_INVALID_ARG;
    hipStream_t hs = (hipStream_t)stream;
    const SlidePlan pl = plan_slide(p);
    if ((int64_t)p->B * p->H * pl.nchunks * pl.nparts > 0x7fffffff) return TLIN_ERR_INVALID_ARG;
    if ((st = check_ws(ws, ws_bytes, slide_ws_bytes(p, pl)))) return st;
    if ((st = check_device())) return st;
    // partial slots: (b*H + h, chunk, part), W rows each
    const size_t rows = (size_t)p->B * p->H * pl.nchunks * pl.nparts * p->W;
    float *base = (float *)ws;
    const Workspace w = {base, base + rows * dpad(p->D), base + rows * dpad(p->D) + rows};

    // every tensor has p->N rows per head
    const Strides q = resolve(p->q_stride, p->H, p->N, p->D);
    const Strides o = resolve(p->o_stride, p->H, p->N, p->D);
    auto args = [&](const void *K, const void *V, const int64_t ks[3], const int64_t vs[3]) {
        AttnArgs a = base_args(p, Q, K, V, ks, vs, p->N);
        a.q_sb = q.b; a.q_sh = q.h; a.q_sr = q.r;
        a.nchunks = pl.nchunks;
        a.seq_rows = p->N;
        return a;
    };
    AttnArgs ah = args(K_hist, V_hist, p->kh_stride, p->vh_stride);
    ah.nsplit = pl.nsplit;
    set_partial(ah, w, pl.nparts, 0);
    AttnArgs aw = args(K_win, V_win, p->kw_stride, p->vw_stride);
    set_partial(aw, w, pl.nparts, pl.nsplit);
    if (pl.nchunks > 1) {
        if ((st = launch_partials(p, ah, aw, hs))) return st;
    } else if ((st = launch_attn(p, true, aw, hs))) {
        return st;
    }

    MergeArgs m = merge_args(p, w, pl.nparts, pl.nsplit, true, p->combine == TLIN_COMBINE_JOINT, O, nullptr);
    m.o_sb = o.b; m.o_sh = o.h; m.o_sr = o.r;
    m.nchunks = pl.nchunks;
    m.seq_rows = p->N;
    return launch_merge(p, m, hs);
}

tlin_status tlin_profile_stream_read(const void *buf, size_t bytes, int32_t nontemporal, void *stream)
{
    if (!buf || !aligned(buf, 16) || bytes < ((size_t)1 << 20)) return TLIN_ERR_INVALID_ARG;
    tlin_status st = check_device();
    if (st) return st;
    const int blocks = 8 * kNumCU;
    const StreamReadArgs a = {buf, bytes / 16 / blocks};
    const void *kernel = nontemporal ? (const void *)stream_read_kernel<true> : (const void *)stream_read_kernel<false>;
    return launch_kernel(kernel, dim3(blocks), dim3(256), 0, (hipStream_t)stream, a);
}

tlin_status tlin_profile_enable(int32_t enable)
{
    std::lock_guard<std::mutex> lk(g_prof.mu);
    g_prof.on = enable != 0;
    return TLIN_OK;
}

tlin_status tlin_profile_read(double ms[3], int64_t launches[3])
{
    if (!ms || !launches) return TLIN_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lk(g_prof.mu);
    for (int i = 0; i < KC_COUNT; ++i) { ms[i] = 0.0; launches[i] = 0; }
    tlin_status rc = TLIN_OK;
    for (const Timed &t : g_prof.used) {
        float e = 0.f;
        if (hipEventSynchronize(t.stop) != hipSuccess || hipEventElapsedTime(&e, t.start, t.stop) != hipSuccess) {
            rc = TLIN_ERR_HIP;
        } else {
            ms[t.cls] += e;
            launches[t.cls] += 1;
        }
        g_prof.pool.push_back({t.start, t.stop});
    }
    g_prof.used.clear();
    return rc;
}

const char *tlin_status_string(int status)
{
    switch (status) {
    case TLIN_OK: return "ok";
    case TLIN_ERR_INVALID_ARG: return "invalid argument";
    case TLIN_ERR_UNSUPPORTED: return "unsupported head dimension or dtype";
    case TLIN_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case TLIN_ERR_HIP: return "HIP runtime error";
    }
    return "unknown status";
}

int32_t tlin_version(void) { return kVersion; }

}  // extern "C"

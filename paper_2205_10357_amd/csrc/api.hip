// C-ABI of the fused block: argument validation (host only, before any HIP call), launch
// planning (tile shape, split count, workspace layout) and the calls into the kernels.
#include <limits.h>
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <atomic>
#include <map>
#include <mutex>

#include "../../include/sol_block.h"
#include "classes.h"
#include "launch.h"
#include "pack_tile.h"
#include "reduce_rows.h"

namespace sol {
namespace {

constexpr size_t kAlign = 256;
int builtin_scratch_address(void** out);      // device address of this GPU's built-in scratch array
inline size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }
inline bool misaligned(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }

struct Geometry {
    int Ho, Wo;
    long long M, K;
    long long x_elems, y_elems, w_elems;
};

int check_desc(const sol_block_desc* d, Geometry* g) {
    if (!d) return SOL_ERR_NULL;
    if (d->dtype != SOL_F32 && d->dtype != SOL_BF16) return SOL_ERR_UNSUPPORTED;
    if (d->flags & ~(uint32_t)(SOL_RELU | SOL_DW_ACCUMULATE)) return SOL_ERR_UNSUPPORTED;
    if (d->N < 1 || d->H < 1 || d->W < 1 || d->C_in < 1 || d->C_out < 1 || d->KH < 1 || d->KW < 1 ||
        d->stride < 1 || d->pad < 0)
        return SOL_ERR_SHAPE;
    if (d->H + 2 * (long long)d->pad < d->KH || d->W + 2 * (long long)d->pad < d->KW) return SOL_ERR_SHAPE;
    g->Ho = (d->H + 2 * d->pad - d->KH) / d->stride + 1;
    g->Wo = (d->W + 2 * d->pad - d->KW) / d->stride + 1;
    g->M = (long long)d->N * g->Ho * g->Wo;
    g->K = (long long)d->KH * d->KW * d->C_in;
    g->x_elems = (long long)d->N * d->H * d->W * d->C_in;
    g->y_elems = g->M * d->C_out;
    g->w_elems = g->K * d->C_out;
    const long long lim = 0x7fffffffLL;
    if (g->x_elems > lim || g->y_elems > lim || g->w_elems > lim) return SOL_ERR_UNSUPPORTED;
    return SOL_OK;
}

// hipGetLastError() reports the last error of ANY earlier HIP call on this thread (the caller's
// framework included); drop it so that the check after our launches sees only our own.
inline void clear_stale_error() { (void)hipGetLastError(); }

// Tuning-experiment overrides from the environment.  They are read once (at the first call that needs one,
// or when sol_reload_overrides() asks for it), never per call: every getenv walks the whole environment, and a
// backward call used to make some fifteen of them.
enum Knob {
    K_IGEMM_TILE, K_IGEMM_FAST, K_FAST_TILE, K_FAST_SHORTK, K_FAST_MANY, K_FAST_STAGES, K_WGRAD_SPLITS, K_WGRAD_TARGET,
    K_SMALLC, K_FILL_UNTOUCHED, K_WGRAD_FAST, K_PACK_FUSED, K_WGRAD_STAGES, K_PREMASK, K_PANEL, K_PANEL_TILES,
    K_REDUCE_RIDES, K_WIDE, K_KSPLIT, K_HALO, K_WGRAD_WIDE, K_COUNT
};
const char* const kKnobNames[K_COUNT] = {
    "SOL_IGEMM_TILE", "SOL_IGEMM_FAST", "SOL_FAST_TILE", "SOL_FAST_SHORTK", "SOL_FAST_MANY", "SOL_FAST_STAGES",
    "SOL_WGRAD_SPLITS", "SOL_WGRAD_TARGET", "SOL_SMALLC", "SOL_FILL_UNTOUCHED", "SOL_WGRAD_FAST", "SOL_PACK_FUSED",
    "SOL_WGRAD_STAGES", "SOL_PREMASK", "SOL_PANEL", "SOL_PANEL_TILES", "SOL_REDUCE_RIDES", "SOL_WIDE", "SOL_KSPLIT", "SOL_HALO", "SOL_WGRAD_WIDE"};
constexpr int kKnobUnset = INT32_MIN;
std::atomic<int> g_knobs[K_COUNT];
std::atomic<bool> g_knobs_loaded{false};
std::mutex g_knob_mutex;
void load_knobs() {
    std::lock_guard<std::mutex> lock(g_knob_mutex);
    for (int k = 0; k < K_COUNT; ++k) {
        const char* v = getenv(kKnobNames[k]);
        g_knobs[k].store(v && *v ? atoi(v) : kKnobUnset, std::memory_order_relaxed);
    }
    g_knobs_loaded.store(true, std::memory_order_release);
}
int knob(Knob k, int fallback) {
    if (!g_knobs_loaded.load(std::memory_order_acquire)) load_knobs();
    const int v = g_knobs[k].load(std::memory_order_relaxed);
    return v == kKnobUnset ? fallback : v;
}

// ---- installed launch plans (sol_block_set_plan): shape -> tile / ring depth / split count ----
struct PlanKey {
    int32_t v[11];
    bool operator<(const PlanKey& o) const { return memcmp(v, o.v, sizeof v) < 0; }
};
PlanKey plan_key(const sol_block_desc* d, int which) {
    return PlanKey{{d->N, d->H, d->W, d->C_in, d->C_out, d->KH, d->KW, d->stride, d->pad, d->dtype, which}};
}
std::mutex g_plan_mutex;
std::map<PlanKey, sol_plan> g_plans;
std::atomic<int> g_plan_count{0};              // lets the common case (no plans) skip the lock
sol_plan installed_plan(const sol_block_desc* d, int which) {
    sol_plan out{-1, 0, 0};
    if (g_plan_count.load(std::memory_order_acquire) == 0) return out;
    std::lock_guard<std::mutex> lock(g_plan_mutex);
    auto it = g_plans.find(plan_key(d, which));
    if (it != g_plans.end()) out = it->second;
    return out;
}

// Largest tile that still yields about one workgroup per compute unit; small problems fall
// back to the smallest tile.  SOL_IGEMM_TILE overrides (tuning experiments).
int pick_igemm_tile(const long long* class_rows, int ncls, int Nc) {
    const int forced = knob(K_IGEMM_TILE, -1);
    if (forced >= 0 && forced <= 3) return forced;
    const int order_wide[4] = {1, 0, 2, 3};
    const int order_narrow[2] = {2, 3};
    const int* order = Nc > 64 ? order_wide : order_narrow;
    const int n = Nc > 64 ? 4 : 2;
    for (int i = 0; i < n; ++i) {
        int bp, bc;
        igemm_tile_shape(order[i], &bp, &bc);
        long long tiles = 0;
        for (int c = 0; c < ncls; ++c) tiles += (class_rows[c] + bp - 1) / bp;
        tiles *= (Nc + bc - 1) / bc;
        if (tiles >= 192) return order[i];
    }
    return order[n - 1];
}

// A pipelined or panel launch of `gemm_wgs` workgroups (one per compute unit at a time) can carry the split
// reduction of the same block's weight gradient along, as workgroups behind its own: as many as its last wave
// leaves compute units idle, so that the reduction runs beside the tiles instead of after them.  Returns 0 when
// fewer than 32 are idle (the reduction then stays a launch of its own).  The two smaller tiles run several workgroups
// per compute unit in many waves: there the riders fill the launch's tail, one per compute unit at most and no more
// than there are passes over the rows.  So do those of the tiles that split the reduction, whose launches are short: with as
// many riders as units are idle, i.e. few, the launch waits for them (1x1 1024 -> 512, 196 pixels 20.2 us, 7.3 with 256).
// SOL_REDUCE_RIDES: 0 never, n > 1 that many.
int reduce_rider_blocks(int gemm_wgs, bool small_tile, const ReduceParams* rider) {
    const int forced = knob(K_REDUCE_RIDES, 1);
    if (!rider || forced == 0 || gemm_wgs <= 0 || !reduce_can_ride(*rider)) return 0;
    if (forced > 1) return forced < 1024 ? forced : 1024;
    if (small_tile) {
        const int rows_per_pass = rider->K <= 256 ? 4 : (rider->K <= 512 ? 2 : 1);
        const int passes = (rider->C_out + rows_per_pass - 1) / rows_per_pass;
        return passes < 256 ? passes : 256;
    }
    const int idle = (256 - gemm_wgs % 256) % 256;
    return idle >= 32 ? idle : 0;
}

// Which kernel family and tile a pipelined launch takes.
enum GemmFamily { GEMM_FAST, GEMM_WIDE, GEMM_KSPLIT, GEMM_HALO };
struct GemmChoice {
    GemmFamily family;
    int tile;
};

// Tiles of bp x bc (powers of two: every launch asks about a dozen shapes, which must not cost it a dozen divisions).
int tiles_of(const IgemmParams& p, const long long* rows, int bp, int bc) {
    const int lp = __builtin_ctz((unsigned)bp), lc = __builtin_ctz((unsigned)bc);
    long long t = 0;
    for (int c = 0; c < p.ncls; ++c) t += (rows[c] + bp - 1) >> lp;
    t *= (p.Nc + bc - 1) >> lc;
    return t < INT_MAX ? (int)t : INT_MAX;
}

// The choice between the four-wave tiles (`tile`: what the thresholds of run_igemm picked), the eight-wave tiles, the
// tiles that keep a 3x3 neighbourhood in LDS and the tiles whose waves split the reduction, by expected time.  All of them
// are bound by what a compute unit copies into LDS and multiplies, plus fixed costs per round of workgroups, so a launch
// of T workgroups with nk 64-deep slices takes, in ns (fits to launches over the benchmark network's layers at 1 .. 128
// images, inputs not in L2; 256 compute units):
//   64 x 64, two per compute unit              3600 + nk * max(200, 153 * ceil(T / 256))
//   128 x 64, three per compute unit           5000 + nk * max(300, 450 T / 256)
//     forward, 160 .. 256 tiles                5000 + 250 nk: each has a compute unit for itself, where 64 x 64 tiles come two by
//                                              two (us, 64 x 64 -> 128 x 64, operands in the caches / from HBM: 5x5 / stride 2
//                                              448 -> 448, 3600 pixels 55.8 / 64.2 -> 46.5 / 53.6; 3x3 448 -> 224, 6084 pixels 18.9 / 21.2
//                                              -> 15.8 / 19.9; 1x1 2048 -> 512, 3136 pixels 12.4 / 18.5 -> 11.4 / 16.5); a data gradient's
//                                              riders find no room beside such a tile (3x3 512 -> 512, 2352 pixels 25.5 -> 30.4)
//     many tiles, 129 .. 192 channels, >= 9 taps  320 for 450: three tiles of channels share a gather and 128-wide tiles pad a
//                                              quarter (3x3 128 -> 192, 82369 pixels 62.4 with a neighbourhood in LDS, 50.0; 512 -> 176
//                                              189 and 173)
//   128 x 128, eight waves                     ceil(T / 256) * (5100 + 390 nk)
//   256 x 128 and 128 x 256, eight waves       ceil(T / 256) * (6500 + 900 nk)
//   neighbourhood in LDS: 256 x 128            ceil(T / 256) * (8000 + 600 nk)
//                         128 x 128            ceil(T / 256) * (4200 + 370 nk)
//                         128 x 64             5000 + nk * max(300, 400 T / 256), where two workgroups fit a compute unit (64
//                                              source channels or narrow images; alone they lose to the gathering 128 x 64
//                                              tiles: 3x3 512 -> 64, 76176 pixels 70.5 and 74.5 us, 128 -> 64, 117077 pixels 27.9 and 29.9)
//   reduction split over the waves             2500 + ceil(T / 256) * (1200 + 1.28 nk (bp + bc))
// Short reductions (nk < 8) in many tiles are bound by HBM, which the fits do not know: they keep the four-wave tiles
// (1x1, 401408 pixels, 256 -> 128: 72 us with 128 x 64, 76 us with 256 x 128).  The splitting tiles are for launches that
// are at most 96 tiles of 64 x 64.
// Four- and eight-wave tiles add a reduction in the same order, the other two families in orders of their own: which
// family a launch takes depends on its sizes only, not on what rides along.  any_order = false (a plan is installed, even
// one that does not apply to this launch): four- and eight-wave tiles only.
GemmChoice choose_gemm(IgemmParams& p, const long long* rows, int tile, bool data_gradient, const ReduceParams* rider, bool any_order) {
    long long all_rows = 0, work = 0;
    for (int c = 0; c < p.ncls; ++c) {
        all_rows += rows[c];
        work += rows[c] * p.cls[c].Th * p.cls[c].Tw * p.Cs;
    }
    const bool ragged = (p.Cs & 63) != 0;                     // slices of the flattened (tap, channel) index
    const long long nk = p.ncls == 1 ? ((long long)p.cls[0].Th * p.cls[0].Tw * p.Cs + 63) >> 6          // slices of an average row
                       : all_rows > 0 ? (work / 64 + all_rows - 1) / all_rows : 0;
    auto rounds = [](long long t) { return (t + 255) >> 8; };
    // A split reduction that rides along: on the compute units that large tiles leave idle it moves about 25 bytes per ns
    // and unit (a launch of its own, 4000 ns, where fewer than 32 are idle); among many small workgroups it fills gaps.
    const long long rider_bytes = rider ? (long long)rider->splits * rider->C_out * rider->K * 4 : 0;
    auto with_rider = [&](long long e, long long t, bool small) {
        if (!rider) return e;
        if (small) return e + (rider_bytes >> 13);
        const int idle = (int)(-t & 255);
        if (idle < 32) return e + 4000 + (rider_bytes >> 12);
        const long long r = 2500 + (long long)((float)rider_bytes / (float)(idle * 25));
        return r > e ? r : e;
    };
    struct Best {
        GemmChoice choice{GEMM_FAST, 0};
        long long alone = INT64_MAX, loaded = INT64_MAX;      // least time without / with the rider, choice by the latter
        void offer(GemmChoice c, long long a, long long l) {
            if (a < alone) alone = a;
            if (l < loaded) {
                loaded = l;
                choice = c;
            }
        }
    } plain, halo, ksplit;
    int bp, bc;
    auto offer_fast = [&](int t) {
        igemm_fast_tile_shape(t, &bp, &bc);
        const long long n = tiles_of(p, rows, bp, bc), r = rounds(n);
        const int ns = n >= 1024 && p.Nc > 128 && p.Nc <= 192 && p.Cs > 64 && p.ncls == 1 && p.cls[0].Th * p.cls[0].Tw >= 9 ? 320 : 450;
        const bool one_each = !data_gradient && n >= 160 && n <= 256;
        const long long e = t == 2 ? 3600 + nk * (153 * r > 200 ? 153 * r : 200)
                          : t == 1 ? 5000 + nk * (one_each ? 250 : ns * n < 300 * 256 ? 300 : (ns * n) >> 8)
                                   : r * (5100 + 390 * nk);
        plain.offer(GemmChoice{GEMM_FAST, t}, e, with_rider(e, n, t == 1 || t == 2));
    };
    offer_fast(tile);
    // 64 x 64 beside 128 x 64 where its workgroups are resident at once; launches of up to eight slices come here with 64 x 64
    // already, see run_igemm (1x1 512 -> 2048, 539 pixels 8.0 -> 6.5 us, 1176 pixels
    // 10.4 -> 7.9; 512 -> 128, 12544 pixels 8.2 -> 6.0)
    if (ragged || (tile == 1 && tiles_of(p, rows, 64, 64) <= 640)) offer_fast(3 - tile);
    if (!ragged && knob(K_WIDE, 0) >= 0 && nk >= 8 && p.Nc > 64) {
        if (tile != 1) offer_fast(1);
        for (int w = 0; w < WIDE_TILES; ++w) {
            igemm_wide_tile_shape(w, &bp, &bc);
            const long long n = tiles_of(p, rows, bp, bc);
            const long long e = rounds(n) * (w == WIDE_128x128 ? 5100 + 390 * nk : 6500 + 900 * nk);
            plain.offer(GemmChoice{GEMM_WIDE, w}, e, with_rider(e, n, false));
        }
    }
    if (!ragged && any_order && knob(K_HALO, 0) == 0)
        for (int h = 0; h < HALO_TILES; ++h) {
            size_t lds = 0;
            if (!plan_igemm_halo(p, h, &bp, &bc, &lds) || (h == HALO_128x64 && lds > 80 * 1024)) continue;
            const long long n = tiles_of(p, rows, bp, bc);
            const long long e = h == HALO_256x128 ? rounds(n) * (8000 + 600 * nk)
                              : h == HALO_128x128 ? rounds(n) * (4200 + 370 * nk)
                                                  : 5000 + nk * (n < 192 ? 300 : (400 * n) >> 8);
            halo.offer(GemmChoice{GEMM_HALO, h}, e, with_rider(e, n, h == HALO_128x64));
        }
    if (any_order && knob(K_KSPLIT, 0) >= 0 && tiles_of(p, rows, 64, 64) <= 96)
        for (int k = 0; k < KSPLIT_TILES; ++k) {
            igemm_ksplit_tile_shape(k, &bp, &bc);
            const long long e = 2500 + rounds(tiles_of(p, rows, bp, bc)) * (1200 + ((nk * (bp + bc) * 328) >> 8));
            ksplit.offer(GemmChoice{GEMM_KSPLIT, k}, e, e);
        }
    // A tile whose waves split the reduction fills a compute unit's LDS, so a riding reduction runs after the tiles there and
    // beside them elsewhere: a data gradient (which carries one as a rule, and takes the same kernel when it does not) takes
    // such tiles where they save the 5 us of that.  Launch with its reduction, us, splitting tiles -> 64 x 64: 3x3 512 -> 512,
    // 392 pixels 17.4 and 19.0, 49 pixels 14.2 and 17.3; 3x3 256 -> 256, 196 pixels 10.0 and 11.1, 1372 pixels 10.9 and 11.0; 1x1
    // 1024 -> 512, 196 pixels 7.3 -> 6.4; 2048 -> 512, 49 pixels 8.0 -> 7.0; 3x3 / stride 2 256 -> 256, 784 pixels 10.5 -> 7.3.  (No
    // lead is asked of them in the forward pass: half a microsecond, which warm operands suggest (1x1 / stride 2 256 -> 512,
    // 304 pixels 4.4 -> 4.0), made the inference of one image, whose weights come from memory, 235 -> 243 us.)
    const long long lead = data_gradient ? 5000 : 0;
    if (ksplit.alone < INT64_MAX && ksplit.alone + lead < plain.alone && ksplit.alone + lead < halo.alone) return ksplit.choice;
    return halo.alone < plain.alone ? halo.choice : plain.choice;
}

// Fills tile-dependent fields of the launch (tile counts, class offsets) and launches either a pipelined kernel (channel
// counts multiples of 8, no mask on the gathered operand) or the general one.  SOL_IGEMM_FAST=0
// forces the general kernel; SOL_FAST_TILE / SOL_FAST_STAGES override the pipelined kernel's tile and ring depth,
// SOL_WIDE, SOL_HALO, SOL_KSPLIT = n > 0 force tile n - 1 of those families, -1 switches them off (tuning experiments); a
// launch that the forced neighbourhood tile cannot serve takes another family.
// `rider`: a split reduction the launch may carry along (see above); *rode tells whether it did.
int run_igemm(IgemmParams& p, const long long* rows, bool mask, bool data_gradient, const sol_plan& tuned, hipStream_t stream,
              const ReduceParams* rider = nullptr, bool* rode = nullptr) {
    if (rode) *rode = false;
    auto attach = [&](bool small_tile) {            // p.total_tiles is final
        p.red_blocks = reduce_rider_blocks(p.total_tiles, small_tile, rider);
        if (p.red_blocks > 0) p.red = *rider;
        if (rode) *rode = p.red_blocks > 0;
        return p.red_blocks > 0;
    };
    bool few_taps = true;                       // the pipelined kernel keeps one validity bit per tap
    for (int c = 0; c < p.ncls; ++c) few_taps = few_taps && p.cls[c].Th * p.cls[c].Tw <= 32;
    // the pipelined kernel starts its buffer descriptor a few image rows before the gathered tensor (the reach of the
    // taps around a pixel); tensor plus that reach must stay below 2^32 bytes
    long long reach = 0;
    for (int c = 0; c < p.ncls; ++c) {
        const RowClass& rc = p.cls[c];
        const long long first = ((long long)rc.h_off * p.Ws + rc.w_off) * p.Cs * 2;
        const long long last = (((long long)(rc.Th - 1) * p.Ws + (rc.Tw - 1)) * rc.tap_step) * p.Cs * 2;
        const long long m = (first < 0 ? -first : 0) + (last < 0 ? -last : 0);
        if (m > reach) reach = m;
    }
    const bool addressable = (long long)p.src_bytes + reach <= 0xffffffffLL && reach <= 0x7fffffffLL;
    // source channels that are no multiple of 64 take the pipelined tiles with a table of chunk addresses in LDS
    const bool ragged = (p.Cs % 64) != 0;
    const bool fast_ok = !mask && few_taps && addressable && (p.Cs % 8) == 0 && (p.Nc % 8) == 0 &&
                         (!ragged || igemm_chunk_table_bytes(p) <= 16384) && knob(K_IGEMM_FAST, 1) != 0;
    int bp, bc, tile = 0, stages = 0;
    GemmChoice choice{GEMM_FAST, 0};
    bool many_tiles = false;
    // 1x1 / stride 1 with a short reduction and a wide output: a workgroup keeps its pixel panel in LDS and walks over
    // several channel tiles (tile code 4)
    const bool panel_ok = fast_ok && !ragged && knob(K_PANEL, 1) != 0 && igemm_panel_eligible(p);
    if (fast_ok) {
        long long slices = 0;
        for (int c = 0; c < p.ncls; ++c) {
            const long long s = ((long long)p.cls[c].Th * p.cls[c].Tw * p.Cs + 63) >> 6;
            if (s > slices) slices = s;
        }
        tile = knob(K_FAST_TILE, -1);
        if (tile < 0 || tile > 4) tile = tuned.tile;              // an installed plan; the environment wins (experiments)
        if (tile == 4 && !panel_ok) tile = -1;                    // a plan for the panel kernel on a launch it cannot run
        const bool free_choice = tile < 0 || tile > 4;
        if (free_choice) {
            // 128 x 128 unless that leaves most compute units idle or the GEMM is narrow
            const long long t128 = tiles_of(p, rows, 128, 128);
            tile = p.Nc <= 64 ? 1 : (t128 >= 160 ? 0 : 1);
            // short reductions are dominated by per-workgroup latency (prologue, epilogue): many small
            // workgroups per compute unit hide it better than few large ones
            if (slices <= knob(K_FAST_SHORTK, 4) && t128 >= 512) tile = 2;
            // many tiles per compute unit: 128 x 64 tiles with two stages leave room for three workgroups per
            // compute unit, whose prologues and epilogues overlap (measured over the ResNet-50 layer shapes:
            // best or within a few percent of best from ~3 tiles of 128 x 128 per compute unit upwards)
            many_tiles = t128 >= knob(K_FAST_MANY, 700) * (slices <= 4 ? 2 : 1);   // short reductions: 64 x 64 holds up longer
            if (many_tiles) tile = 1;
            igemm_fast_tile_shape(tile, &bp, &bc);
            if (tiles_of(p, rows, bp, bc) < 160) tile = 2;
            // Short reductions whose small tiles are all resident at once pay one latency chain instead of a round after the
            // other.  1x1 with residual, panel kernel or 128 x 64 -> 64 x 64, us: 64 -> 256, 18207 pixels (1140 tiles) 10.4 -> 6.0,
            // 28611 9.2 -> 7.6, 62424 (3904) 14.3 and 13.9; 128 -> 512, 5488 pixels 6.0 -> 4.7, 8624 (1080) 8.7 -> 7.1; 256 -> 1024,
            // 1372 6.0 -> 4.9, 2156 (544) 6.5 -> 5.9, 3136 (784) 6.7 and 7.1; 512 -> 2048, 1176 (608) 10.4 -> 7.9.  With four slices
            // and more tiles than that 128 x 64 (256 -> 1024, 3136 pixels 6.1, 4704 10.2 -> 8.3), until the panel kernel leads.
            const long long t64 = tiles_of(p, rows, 64, 64);
            if (t64 <= (slices <= 2 ? 2560 : slices <= 4 ? 704 : slices <= 8 ? 640 : 0)) {
                tile = 2;
                many_tiles = false;
            } else if (slices <= 4 && t64 <= 1280 && p.Nc > 64) {
                tile = 1;
                many_tiles = true;
            } else if (panel_ok) {                  // where its launch is one wave of workgroups that fills most of the chip
                const long long panels = (rows[0] + 127) / 128;
                long long groups = 256 / (panels > 0 ? panels : 1);
                if (groups > p.Nc / 128) groups = p.Nc / 128;
                if (panels <= 256 && panels * groups >= 160) tile = 4;
            }
        }
        if (tile == 4) {
            plan_igemm_panel(p, knob(K_PANEL_TILES, 0));
            trace_point(stream, attach(false) ? SOL_TRACE_IGEMM_PANEL_REDUCE : SOL_TRACE_IGEMM_PANEL);
            return launch_igemm_panel(p, stream) == hipSuccess ? SOL_OK : SOL_ERR_LAUNCH;
        }
        if (ragged && tile != 2) tile = 1;
        choice = free_choice ? choose_gemm(p, rows, tile, data_gradient, knob(K_REDUCE_RIDES, 1) != 0 ? rider : nullptr, tuned.tile < 0) : GemmChoice{GEMM_FAST, tile};
        if (choice.family == GEMM_FAST && choice.tile != tile) {
            tile = choice.tile;
            igemm_fast_tile_shape(tile, &bp, &bc);      // deep rings: one 128 x 64 tile or two of 64 x 64 per compute unit
            many_tiles = tiles_of(p, rows, bp, bc) > (tile == 2 ? 512 : 256);
        }
        stages = knob(K_FAST_STAGES, 0);
        if (stages < 2 || stages > 4) stages = tuned.stages;
        if (stages < 2 || stages > 4) stages = (slices <= 4 || many_tiles) ? 2 : (slices <= 8 ? 3 : 4);
        if (tile == 3 && stages > 3) stages = 3;
        if (choice.family == GEMM_FAST && tile == 0 && stages == 4) choice = GemmChoice{GEMM_WIDE, WIDE_128x128};
        if (const int w = knob(K_WIDE, 0); w > 0 && w <= WIDE_TILES && !ragged) choice = GemmChoice{GEMM_WIDE, w - 1};
        if (const int k = knob(K_KSPLIT, 0); k > 0 && k <= KSPLIT_TILES) choice = GemmChoice{GEMM_KSPLIT, k - 1};
        if (const int h = knob(K_HALO, 0); h > 0 && h <= HALO_TILES && !ragged && plan_igemm_halo(p, h - 1, &bp, &bc)) choice = GemmChoice{GEMM_HALO, h - 1};
        if (choice.family == GEMM_HALO) plan_igemm_halo(p, choice.tile, &bp, &bc);
        else if (choice.family == GEMM_WIDE) igemm_wide_tile_shape(choice.tile, &bp, &bc);
        else if (choice.family == GEMM_KSPLIT) igemm_ksplit_tile_shape(choice.tile, &bp, &bc);
        else igemm_fast_tile_shape(tile, &bp, &bc);
    } else {
        tile = pick_igemm_tile(rows, p.ncls, p.Nc);
        igemm_tile_shape(tile, &bp, &bc);
    }
    p.tiles_c = (p.Nc + bc - 1) / bc;
    int tiles_p = 0;
    for (int c = 0; c < p.ncls; ++c) {
        RowClass& rc = p.cls[c];
        const bool lin_src = rc.Th == 1 && rc.Tw == 1 && rc.h_mul == 1 && rc.w_mul == 1 && rc.h_off == 0 &&
                             rc.w_off == 0 && rc.Rh == p.Hs && rc.Rw == p.Ws;
        const bool lin_out = rc.oh_mul == 1 && rc.ow_mul == 1 && rc.oh_off == 0 && rc.ow_off == 0 &&
                             rc.Rh == p.Hout && rc.Rw == p.Wout;
        rc.linear = (lin_src ? 1 : 0) | (lin_out ? 2 : 0);
        rc.div_img = make_fast_div((uint32_t)(rc.Rh * rc.Rw));
        rc.div_rw = make_fast_div((uint32_t)rc.Rw);
        p.cls[c].tile_begin = tiles_p;
        tiles_p += (int)((rows[c] + bp - 1) / bp);
    }
    p.total_tiles = tiles_p * p.tiles_c;
    hipError_t e;
    const bool rides = fast_ok && attach((choice.family == GEMM_FAST && (tile == 1 || tile == 2)) || choice.family == GEMM_KSPLIT ||
                                         (choice.family == GEMM_HALO && choice.tile == HALO_128x64));
    static const int kinds[][2] = {{SOL_TRACE_IGEMM, SOL_TRACE_IGEMM_REDUCE}, {SOL_TRACE_IGEMM_WIDE, SOL_TRACE_IGEMM_WIDE_REDUCE},
                                   {SOL_TRACE_IGEMM_KSPLIT, SOL_TRACE_IGEMM_KSPLIT_REDUCE}, {SOL_TRACE_IGEMM_HALO, SOL_TRACE_IGEMM_HALO_REDUCE}};
    trace_point(stream, fast_ok ? kinds[choice.family][rides] : SOL_TRACE_IGEMM_GENERAL);
    if (!fast_ok) e = launch_igemm(p, tile, (p.Cs % 8) == 0, mask, stream);
    else if (choice.family == GEMM_WIDE) e = launch_igemm_wide(p, choice.tile, stream);
    else if (choice.family == GEMM_HALO) e = launch_igemm_halo(p, choice.tile, stream);
    else if (choice.family == GEMM_KSPLIT) e = launch_igemm_ksplit(p, choice.tile, stream);
    else if (ragged) e = launch_igemm_fast_ragged(p, tile, stages, stream);
    else e = launch_igemm_fast(p, tile, stages, stream);
    return e == hipSuccess ? SOL_OK : SOL_ERR_LAUNCH;
}

struct BwdPlan {
    int splits, m_per_split, tiles_k, tiles_c;
    bool wide;                    // the weight gradient takes the eight-wave kernel (where it takes a pipelined one at all)
    size_t wpack_off, part_off, dshift_off, total;
    // few-input-channel layers: per-workgroup partials of their own weight-gradient kernel
    bool smallc;
    int sc_parts;
    size_t sc_part_off;
    // a block that masks dy itself (SOL_RELU): the masked gradient, written once by an element-wise launch so that
    // both gradient GEMMs take the pipelined kernels (which gather their operands without looking at y)
    bool premask;
    size_t gmask_off;
};

// channel counts the 16-byte operand pieces of the bf16 kernels need
inline bool bf16_vector_shape(const sol_block_desc* d) {
    return d->dtype == SOL_BF16 && (d->C_in % 8) == 0 && (d->C_out % 8) == 0;
}

// A backward pass of this block masks its gradient in a launch of its own, so that the GEMMs need not.
inline bool premasks(const sol_block_desc* d, bool smallc) {
    return (d->flags & SOL_RELU) != 0 && d->dtype == SOL_BF16 && (bf16_vector_shape(d) || smallc) && knob(K_PREMASK, 1) != 0;
}
// The weight gradient takes one of the pipelined kernels.
inline bool pipelined_wgrad(const sol_block_desc* d) {
    return bf16_vector_shape(d) && ((d->flags & SOL_RELU) == 0 || premasks(d, false)) && knob(K_WGRAD_FAST, 1) != 0;
}

// Kernel and split of a pipelined weight gradient of `slices` 64-row slices of the reduction and `tiles` 128 x 128 tiles.
//
// A split of S costs each workgroup slices / S and the launch, the reduction and the memory between them tiles * S fp32 tiles,
// so the best S goes with sqrt(slices / tiles).  Measured optima of weight gradient + reduction (7 .. 128 images, 4 .. 144 tiles)
// lie at S^2 tiles / slices = 18 .. 22 for 1x1 / stride 1 and 20 .. 35 for the gathering form.  1x1 / stride 1 runs three stages
// deep, one workgroup per compute unit, and leaves an eighth of them to the re-pack that rides along (1x1 2048 -> 512, 2352
// pixels: 256 workgroups 13.0 us, 192 10.7 us); the gathering form runs two per compute unit.  Before (256 / 512 workgroups
// whatever the slices are -> now, us of weight gradient + reduction + data gradient): 1x1 512 -> 128, 7436 pixels 23.2 -> 18.5;
// 3x3 128 -> 128 23.4 -> 19.7; 3x3 256 -> 256, 1372 pixels 30.4 -> 25.8.
struct WgradChoice {
    long long splits;
    bool wide;
};
WgradChoice choose_wgrad(long long slices, long long tiles, bool linear, int force_wide) {
    WgradChoice c{};
    // 4 T small workgroups re-pack (T = tiles)
    const long long pack = tiles < 16 ? 2 * tiles : 32;
    const float ratio = (float)slices / (float)tiles;
    // Gathering form with a long reduction: one eight-wave workgroup per compute unit instead of two of four waves, i.e. half
    // the partial tiles, beside the 2 T workgroups that re-pack (32 of them at most wait for their turn).  Weight gradient +
    // reduction + data gradient, us, four -> eight waves: 3x3 256 -> 256, 12544 pixels (T = 36, L = 196 slices) 44.2 -> 41.6;
    // 3x3 128 -> 128 (T = 9) L = 392 33.0 -> 30.3, L = 1568 72.5 -> 71.0; 1x1 / stride 2 256 -> 512 (T = 8), L = 1568 149 -> 141.
    // With few slices the two are equal or four waves ahead (T = 9, L = 117: 19.4 and 19.8; T = 6, L = 130 20.7 and 21.0;
    // T = 36, L = 22 26.5 and 27.2): the line is between.  Where one workgroup per compute unit leaves more than 96 idle
    // (T = 144), two splits finer balance better.
    const long long wide_splits = (256 - pack) / tiles;
    c.wide = force_wide > 0 ? wide_splits > 0
                            : !linear && force_wide == 0 && knob(K_WGRAD_TARGET, 0) <= 0 && wide_splits * tiles >= 160 && slices * tiles >= 2048;
    long long best = (long long)(sqrtf((linear ? 18.f : 34.f) * ratio) + 0.5f);
    // (the gathering form fills the chip once or twice, not one and a half times)
    const long long target = knob(K_WGRAD_TARGET, linear ? 256 - pack : (best * tiles <= 384 ? 256 : 512));
    const long long most = c.wide ? wide_splits : (target + (target > 256 ? tiles / 2 : 0)) / tiles;
    if (c.wide || best > most) best = most;
    c.splits = best < 1 ? 1 : best;
    if (best > 64) {
        // More than 64 splits cannot ride with the data gradient: a reduction of its own, which takes 4 us and 30 ns per split
        // more than one that rides along and so wants fewer of them.  It pays where it takes enough slices off each
        // workgroup, i.e. with few tiles and a long reduction.  Whole call, us, 64 riding -> finer splits: T = 1 (1x1 64 -> 64)
        // L = 6272 73 -> 47 (254 splits), L = 1568 26.6 -> 25.3 (131), L = 392 14.4 and 16.3 (96); T = 2 (1x1 64 -> 256) L = 6272
        // 99 -> 92 (126), L = 1568 30.0 and 30.5 (128); 1x1 256 -> 128 L = 6272 167 -> 164, L = 1568 39.0 and 42.8.
        long long alone = (long long)(sqrtf(11.f * ratio) + 0.5f);
        if (alone > most) alone = most;
        const bool pays = alone > 64 && slices / 64 - slices / alone >= 6 + 6 * tiles;
        c.splits = pays ? alone : 64;
    }
    return c;
}

BwdPlan plan_bwd(const sol_block_desc* d, const Geometry& g) {
    BwdPlan b{};
    int room = 1;                 // splits that the workspace has room for
    if (d->dtype == SOL_F32) {
        b.splits = 1;
        b.m_per_split = (int)g.M;
        b.wpack_off = 0;
        b.part_off = 0;
    } else {
        b.tiles_k = (int)((g.K + 127) / 128);
        b.tiles_c = (d->C_out + 127) / 128;
        const long long tiles = (long long)b.tiles_k * b.tiles_c;
        const sol_plan tuned = installed_plan(d, SOL_PLAN_WGRAD);
        const bool linear = d->KH == 1 && d->KW == 1 && d->stride == 1 && d->pad == 0;
        // At most 256 workgroups for 1x1 / stride 1 (one per compute unit) and 512 for the gathering form (two), in ranges of
        // whole 128 rows, with the fp32 partials below about 64 MiB: what the workspace has room for, whatever the split.  An
        // installed plan or an override takes the place of the workgroup count.
        const long long cap = (64LL << 20) / (g.w_elems * 4 > 0 ? g.w_elems * 4 : 1);
        long long asked = knob(K_WGRAD_SPLITS, 0);
        if (asked <= 0) asked = tuned.splits;
        const bool own = asked <= 0;             // the library's choice
        if (own) {
            asked = (knob(K_WGRAD_TARGET, linear ? 256 : 512) + tiles - 1) / tiles;
            if (asked > cap) asked = cap;
        }
        if (asked > (g.M + 127) / 128) asked = (g.M + 127) / 128;
        if (asked < 1) asked = 1;
        long long rows = ((g.M + asked - 1) / asked + 127) / 128 * 128;
        room = (int)((g.M + rows - 1) / rows);
        // (a ring depth that a plan or an override asks for is the four-wave kernel's)
        const bool staged = tuned.stages >= 2 || knob(K_WGRAD_STAGES, 0) >= 2;
        const int force_wide = staged ? -1 : knob(K_WGRAD_WIDE, 0);
        b.wide = force_wide > 0;
        if (own && pipelined_wgrad(d)) {
            const WgradChoice c = choose_wgrad((g.M + 63) / 64, tiles, linear, force_wide);
            const long long want = c.splits < room ? c.splits : room;
            b.wide = c.wide;
            rows = ((g.M + want - 1) / want + 63) / 64 * 64;
        }
        b.m_per_split = (int)rows;
        b.splits = (int)((g.M + rows - 1) / rows);
        b.wpack_off = 0;
        b.part_off = align_up((size_t)g.w_elems * 2);
    }
    b.dshift_off = b.part_off + align_up((size_t)room * g.w_elems * 4);
    b.total = b.dshift_off + align_up((size_t)room * d->C_out * 4);
    b.smallc = d->dtype == SOL_BF16 && smallc_wgrad_supported(d->C_in, d->C_out, d->KH, d->KW, d->stride) &&
               knob(K_SMALLC, 1) != 0;
    if (b.smallc) {
        b.sc_parts = smallc_wgrad_parts(d->N, g.Ho, g.Wo);
        b.sc_part_off = b.total;
        b.total += smallc_wgrad_workspace_bytes(d->N, d->H, d->W, g.Ho, g.Wo);
    }
    b.premask = premasks(d, b.smallc);
    if (b.premask) {
        b.gmask_off = b.total;
        b.total += align_up((size_t)g.y_elems * 2);
    }
    return b;
}

// Forward workspace: only layers with few input channels ask for one.
struct FwdPlan {
    bool smallc;
    size_t total;
};
FwdPlan plan_fwd(const sol_block_desc* d) {
    FwdPlan f{};
    f.smallc = d->dtype == SOL_BF16 && smallc_fwd_supported(d->C_in, d->C_out, d->KH, d->KW, d->stride) &&
               knob(K_SMALLC, 1) != 0;
    if (f.smallc) f.total = smallc_fwd_workspace_bytes(d->N, d->H, d->W, d->KH);
    return f;
}

int fwd_bf16(const sol_block_desc* d, const Geometry& g, const void* x, const void* W, const float* scale,
             const float* shift, const void* residual, void* y, hipStream_t stream) {
    if (plan_fwd(d).smallc && !residual) {
        SmallCParams sp{(const bf16_t*)x, (const bf16_t*)W, scale, shift, (bf16_t*)y, d->N, d->H, d->W, d->C_in, d->KH, d->KW,
                        d->pad, g.Ho, g.Wo, (d->flags & SOL_RELU) ? 1 : 0};
        trace_point(stream, SOL_TRACE_SMALLC_FWD);
        return launch_smallc_fwd(sp, stream) == hipSuccess ? SOL_OK : SOL_ERR_LAUNCH;
    }
    IgemmParams p{};
    p.src = (const bf16_t*)x;
    p.src_mask = nullptr;
    p.wmat = (const bf16_t*)W;
    p.out = (bf16_t*)y;
    p.scale = scale;
    p.shift = shift;
    p.addend = (const bf16_t*)residual;
    p.addend_mask = nullptr;
    p.src_bytes = (unsigned)(g.x_elems * 2);
    p.Hs = d->H;
    p.Ws = d->W;
    p.Cs = d->C_in;
    p.Nc = d->C_out;
    p.Hout = g.Ho;
    p.Wout = g.Wo;
    p.relu = (d->flags & SOL_RELU) ? 1 : 0;
    p.ncls = 1;
    RowClass& c = p.cls[0];
    c.rows = (int)g.M;
    c.Rh = g.Ho;
    c.Rw = g.Wo;
    c.h_mul = d->stride;
    c.h_off = -d->pad;
    c.w_mul = d->stride;
    c.w_off = -d->pad;
    c.Th = d->KH;
    c.Tw = d->KW;
    c.tap_step = 1;
    c.oh_mul = 1;
    c.oh_off = 0;
    c.ow_mul = 1;
    c.ow_off = 0;
    c.tile_begin = 0;
    c.b_off = 0;
    const long long rows[1] = {g.M};
    return run_igemm(p, rows, false, false, installed_plan(d, SOL_PLAN_FWD), stream);
}

int dgrad_bf16(const sol_block_desc* d, const Geometry& g, const void* dy, const void* ymask, const bf16_t* wpack,
               void* dx, const void* addend, const void* addend_mask, const void* dx_mask, hipStream_t stream,
               const ReduceParams* rider = nullptr, bool* rode = nullptr) {
    const int s = d->stride;
    IgemmParams p{};
    const bool relu = ymask != nullptr;          // mask dy by y > 0 while gathering it
    p.src = (const bf16_t*)dy;
    p.src_mask = (const bf16_t*)ymask;
    p.wmat = wpack;
    p.out = (bf16_t*)dx;
    p.scale = nullptr;
    p.shift = nullptr;
    p.addend = (const bf16_t*)addend;
    p.addend_mask = (const bf16_t*)addend_mask;
    p.out_mask = (const bf16_t*)dx_mask;
    p.src_bytes = (unsigned)(g.y_elems * 2);
    p.Hs = g.Ho;
    p.Ws = g.Wo;
    p.Cs = d->C_out;
    p.Nc = d->C_in;
    p.Hout = d->H;
    p.Wout = d->W;
    p.relu = 0;
    long long rows[kMaxClasses];
    int nc = 0;
    // pixels without a tap (1x1 / stride 2: three quarters of dx) are filled at memory speed by a launch of their
    // own; as GEMM tiles without a reduction they cost several times that.  Where dx is added to in place and not masked
    // they stay as they are (56x56, 128 images, 256 channels: a launch of 43 us).
    const bool fill_untouched = (d->C_in % 8) == 0 && knob(K_FILL_UNTOUCHED, 1) != 0;
    const bool in_place = addend == dx && !addend_mask && !dx_mask;
    bool any_untouched = false;
    for (int ph = 0; ph < s; ++ph)
        for (int pw = 0; pw < s; ++pw) {
            const int Rh = d->H > ph ? (d->H - ph + s - 1) / s : 0;
            const int Rw = d->W > pw ? (d->W - pw + s - 1) / s : 0;
            if (Rh == 0 || Rw == 0) continue;
            int fh, fw;
            RowClass& c = p.cls[nc];
            c.Th = class_taps(d->KH, s, d->pad, ph, &fh);
            c.Tw = class_taps(d->KW, s, d->pad, pw, &fw);
            if (c.Th == 0 || c.Tw == 0) {   // no tap reaches these pixels: K = 0, output = addend
                if (fill_untouched) {       // ... written by an element-wise launch instead of GEMM tiles
                    any_untouched = !in_place;
                    continue;
                }
                c.Th = 0;
                c.Tw = 1;
            }
            c.rows = d->N * Rh * Rw;
            c.Rh = Rh;
            c.Rw = Rw;
            c.h_mul = 1;
            c.h_off = (ph + d->pad - fh) / s;
            c.w_mul = 1;
            c.w_off = (pw + d->pad - fw) / s;
            c.tap_step = -1;
            c.oh_mul = s;
            c.oh_off = ph;
            c.ow_mul = s;
            c.ow_off = pw;
            c.b_off = class_weight_offset(d->C_in, d->C_out, d->KH, d->KW, s, d->pad, ph, pw);
            rows[nc] = c.rows;
            ++nc;
        }
    p.ncls = nc;
    if (any_untouched) trace_point(stream, SOL_TRACE_UNTOUCHED);
    if (any_untouched &&
        launch_untouched_pixels(dx, addend, addend_mask, dx_mask, d->N, d->H, d->W, d->C_in, d->KH, d->KW, s, d->pad,
                                stream) != hipSuccess)
        return SOL_ERR_LAUNCH;
    return run_igemm(p, rows, relu, true, installed_plan(d, SOL_PLAN_DGRAD), stream, rider, rode);
}

}  // namespace
}  // namespace sol

// ---- built-in scratch of the no-allocation backward entry point ---------------------------------------------
// One array per GPU, part of the loaded code object (it exists on every device the library runs on until the
// process ends).  In host code the array's NAME is only a stand-in: the device address is asked for once per
// device, with that device current, and only that address is ever handed to kernels.
static __device__ __align__(256) unsigned char scratch[SOL_NOALLOC_SCRATCH_BYTES];

namespace sol {
namespace {
constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch_ptr[kMaxDevices];
std::mutex g_scratch_mutex;

int builtin_scratch_address(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SOL_ERR_LAUNCH;
    void* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        p = g_scratch_ptr[dev].load(std::memory_order_relaxed);
        if (!p) {
            if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
                (void)hipGetLastError();
                return SOL_ERR_LAUNCH;
            }
            g_scratch_ptr[dev].store(p, std::memory_order_release);
        }
    }
    *out = p;
    return SOL_OK;
}
}  // namespace
}  // namespace sol

using namespace sol;

extern "C" {

SOL_API const char* sol_status_string(int status) {
    switch (status) {
        case SOL_OK: return "ok";
        case SOL_ERR_NULL: return "a required pointer is NULL";
        case SOL_ERR_SHAPE: return "invalid shape, stride or padding";
        case SOL_ERR_ALIGN: return "pointer not 16-byte aligned";
        case SOL_ERR_UNSUPPORTED: return "unsupported dtype, flag or size";
        case SOL_ERR_WORKSPACE: return "workspace missing or too small";
        case SOL_ERR_LAUNCH: return "HIP launch error";
        case SOL_ERR_SCRATCH_LIMIT: return "the call needs more scratch than the no-allocation entry point's built-in buffer holds";
        default: return "unknown status";
    }
}

SOL_API size_t sol_block_workspace_bytes(const sol_block_desc* desc, int pass) {
    Geometry g;
    if (check_desc(desc, &g) != SOL_OK) return 0;
    if (pass == SOL_PASS_FWD) return plan_fwd(desc).total;
    if (pass != SOL_PASS_BWD) return 0;
    return plan_bwd(desc, g).total;
}

SOL_API size_t sol_block_wgrad_partial_bytes(const sol_block_desc* desc) {
    Geometry g;
    if (check_desc(desc, &g) != SOL_OK) return 0;
    const BwdPlan plan = plan_bwd(desc, g);
    if (plan.smallc && (plan.premask || (desc->flags & SOL_RELU) == 0)) return smallc_wgrad_partial_bytes(plan.sc_parts, (int)g.K);
    return (size_t)plan.splits * (size_t)(g.w_elems + desc->C_out) * 4;
}

SOL_API int sol_block_fwd(const sol_block_desc* desc, const void* x, const void* W, const float* scale, const float* shift,
                  const void* residual, void* y, void* ws, size_t ws_bytes, void* hip_stream) {
    Geometry g;
    if (int e = check_desc(desc, &g); e != SOL_OK) return e;
    if (!x || !W || !scale || !shift || !y) return SOL_ERR_NULL;
    if (misaligned(x) || misaligned(W) || misaligned(scale) || misaligned(shift) || misaligned(y) ||
        misaligned(residual) || misaligned(ws))
        return SOL_ERR_ALIGN;
    const size_t need = plan_fwd(desc).total;
    if (need > 0 && (!ws || ws_bytes < need)) return SOL_ERR_WORKSPACE;
    hipStream_t stream = (hipStream_t)hip_stream;
    clear_stale_error();
    if (desc->dtype == SOL_BF16) {
        const int st = fwd_bf16(desc, g, x, W, scale, shift, residual, y, stream);
            return st;
    }
    DirectParams p{};
    p.x = (const float*)x;
    p.W = (const float*)W;
    p.scale = scale;
    p.shift = shift;
    p.res = (const float*)residual;
    p.y = (float*)y;
    p.N = desc->N; p.H = desc->H; p.W_ = desc->W; p.C_in = desc->C_in; p.C_out = desc->C_out;
    p.KH = desc->KH; p.KW = desc->KW; p.stride = desc->stride; p.pad = desc->pad;
    p.Ho = g.Ho; p.Wo = g.Wo; p.relu = (desc->flags & SOL_RELU) ? 1 : 0;
    trace_point(stream, SOL_TRACE_DIRECT);
    const int st = launch_direct_fwd_f32(p, stream) == hipSuccess ? SOL_OK : SOL_ERR_LAUNCH;
    return st;
}

// Both backward entry points: everything after the workspace has been chosen.  scratch_limit > 0 marks the
// built-in buffer of the no-allocation entry point, whose size is a property of the library, not of the call.
static int bwd_common(const sol_block_desc* desc, const void* dy, const void* x, const void* W, const void* y, void* dx,
                      float* dW, float* dscale, float* dshift, const float* scale, void* dres, const void* dx_addend,
                      const void* dx_addend_mask, const void* dx_mask, void* ws, size_t ws_bytes, bool builtin_scratch,
                      void* hip_stream) {
    Geometry g;
    if (int e = check_desc(desc, &g); e != SOL_OK) return e;
    bool relu = (desc->flags & SOL_RELU) != 0;
    if (!dy || !x || !W || !scale) return SOL_ERR_NULL;
    if (dW ? (!dscale || !dshift) : (dscale || dshift)) return SOL_ERR_NULL;   // the three come together
    if (!dW && !dx && !dres) return SOL_ERR_NULL;                              // nothing to compute
    if (relu && !y) return SOL_ERR_NULL;
    if (dx_addend_mask && !dx_addend) return SOL_ERR_NULL;
    if (misaligned(dy) || misaligned(x) || misaligned(W) || misaligned(y) || misaligned(dx) || misaligned(dW) ||
        misaligned(dscale) || misaligned(dshift) || misaligned(scale) || misaligned(dres) ||
        misaligned(dx_addend) || misaligned(dx_addend_mask) || misaligned(dx_mask) || misaligned(ws))
        return SOL_ERR_ALIGN;
    if (desc->dtype == SOL_BF16 && dx && desc->stride * desc->stride > kMaxClasses) return SOL_ERR_UNSUPPORTED;
    const BwdPlan plan = plan_bwd(desc, g);
    if (builtin_scratch) {
        if (plan.total > ws_bytes) return SOL_ERR_SCRATCH_LIMIT;
        if (int e = builtin_scratch_address(&ws); e != SOL_OK) return e;
    }
    if (!ws || ws_bytes < plan.total) return SOL_ERR_WORKSPACE;
    hipStream_t stream = (hipStream_t)hip_stream;
    clear_stale_error();
    unsigned char* wsb = (unsigned char*)ws;
    float* partial = (float*)(wsb + plan.part_off);
    float* dshift_partial = (float*)(wsb + plan.dshift_off);
    // A block that masks dy itself: write g = (y > 0 ? dy : 0) once (into dres when the caller wants it anyway) and
    // run everything below on g as a block without ReLU.
    bool dres_done = false;
    if (plan.premask) {
        void* gbuf = dres ? dres : (void*)(wsb + plan.gmask_off);
        trace_point(stream, SOL_TRACE_MASKED_COPY);
        if (launch_masked_copy(desc->dtype, dy, y, gbuf, g.y_elems, stream) != hipSuccess) return SOL_ERR_LAUNCH;
        dy = gbuf;
        relu = false;
        dres_done = dres != nullptr;
    }
    const void* ymask = relu ? y : nullptr;

    auto direct_params = [&]() {
        DirectParams p{};
        p.x = (const float*)x;
        p.W = (const float*)W;
        p.scale = scale;
        p.dy = (const float*)dy;
        p.ymask = (const float*)ymask;
        p.dx = (float*)dx;
        p.addend = (const float*)dx_addend;
        p.addend_mask = (const float*)dx_addend_mask;
        p.dx_mask = (const float*)dx_mask;
        p.G = partial;
        p.dshift_partial = dshift_partial;
        p.N = desc->N; p.H = desc->H; p.W_ = desc->W; p.C_in = desc->C_in; p.C_out = desc->C_out;
        p.KH = desc->KH; p.KW = desc->KW; p.stride = desc->stride; p.pad = desc->pad;
        p.Ho = g.Ho; p.Wo = g.Wo; p.relu = relu ? 1 : 0;
        return p;
    };

    // The re-pack of the weights for the data gradient rides along with the weight-gradient launch (as extra
    // workgroups) when one call computes both branches with the pipelined kernels; else it is a launch of its own.
    const bool bf16_vec = bf16_vector_shape(desc);
    const bool wgrad_pipelined = bf16_vec && !relu && knob(K_WGRAD_FAST, 1) != 0;
    PackParams pk{(const bf16_t*)W, scale, (bf16_t*)(wsb + plan.wpack_off), desc->C_in, desc->C_out, desc->KH,
                  desc->KW, desc->stride, desc->pad};
    const bool pack_rides = dx && dW && wgrad_pipelined && pack_tiled_ok(pk) && knob(K_PACK_FUSED, 1) != 0;

    // The reduction of the split weight gradient in turn may ride along with the data-gradient launch (run_igemm
    // decides); it needs the partial sums of the weight-gradient launch, which therefore goes first.
    ReduceParams rp{};
    rp.partial = partial;
    rp.dshift_partial = dshift_partial;
    rp.W = W;
    rp.scale = scale;
    rp.dW = dW;
    rp.dscale = dscale;
    rp.dshift = dshift;
    rp.C_out = desc->C_out;
    rp.K = (int)g.K;
    rp.splits = plan.splits;
    rp.accumulate = (desc->flags & SOL_DW_ACCUMULATE) ? 1 : 0;
    rp.w_is_bf16 = desc->dtype == SOL_BF16 ? 1 : 0;
    const bool reduce_may_ride = pack_rides;
    bool reduce_rode = false;

    // ---- data branch: shortcut gradient, weight re-pack, data-gradient GEMM ----
    auto data_branch = [&](hipStream_t st) -> int {
        if (dres && !dres_done) {
            trace_point(st, SOL_TRACE_MASKED_COPY);
            if (launch_masked_copy(desc->dtype, dy, ymask, dres, g.y_elems, st) != hipSuccess) return SOL_ERR_LAUNCH;
        }
        if (!dx) return SOL_OK;
        if (desc->dtype == SOL_BF16) {
            if (!pack_rides) trace_point(st, SOL_TRACE_PACK);
            if (!pack_rides && launch_pack_dgrad_weights(pk, st) != hipSuccess) return SOL_ERR_LAUNCH;
            return dgrad_bf16(desc, g, dy, ymask, pk.out, dx, dx_addend, dx_addend_mask, dx_mask, st,
                              reduce_may_ride ? &rp : nullptr, &reduce_rode);
        }
        DirectParams p = direct_params();        // with the weight gradient, which is one launch with it
        if (!dW) p.G = nullptr;
        trace_point(st, SOL_TRACE_DIRECT);
        return launch_direct_bwd_f32(p, st) == hipSuccess ? SOL_OK : SOL_ERR_LAUNCH;
    };

    // ---- weight branch: split weight-gradient GEMM, then the reduction that also finishes dscale, dshift ----
    auto weight_branch = [&](hipStream_t st) -> int {
        if (plan.smallc && !relu) {      // few input channels, gradient already masked: kernels of their own
            trace_point(st, SOL_TRACE_SMALLC_WGRAD);
            SmallCWgradParams wp{(const bf16_t*)dy, (const bf16_t*)x, (const bf16_t*)W, scale, (float*)(wsb + plan.sc_part_off), dW,
                                 dscale, dshift, desc->N, desc->H, desc->W, desc->C_in, desc->KH, desc->KW, desc->pad,
                                 g.Ho, g.Wo, plan.sc_parts, (desc->flags & SOL_DW_ACCUMULATE) ? 1 : 0};
            return launch_smallc_wgrad(wp, st) == hipSuccess ? SOL_OK : SOL_ERR_LAUNCH;
        }
        if (desc->dtype == SOL_BF16) {
            WgradParams wp{};
            wp.dy = (const bf16_t*)dy;
            wp.y = (const bf16_t*)ymask;
            wp.x = (const bf16_t*)x;
            wp.partial = partial;
            wp.dshift_partial = dshift_partial;
            wp.N = desc->N; wp.H = desc->H; wp.W = desc->W; wp.C_in = desc->C_in; wp.C_out = desc->C_out;
            wp.KH = desc->KH; wp.KW = desc->KW; wp.stride = desc->stride; wp.pad = desc->pad;
            wp.Ho = g.Ho; wp.Wo = g.Wo; wp.M = (int)g.M; wp.K = (int)g.K;
            wp.splits = plan.splits; wp.m_per_split = plan.m_per_split;
            wp.tiles_k = plan.tiles_k; wp.tiles_c = plan.tiles_c;
            wp.div_howo = make_fast_div((uint32_t)(g.Ho * g.Wo));
            wp.div_wo = make_fast_div((uint32_t)g.Wo);
            wp.pack = pk;
            wp.pack_tiles = pack_rides ? pack_tile_count(pk) : 0;
            wp.pack_blocks = wp.pack_tiles;
            const bool vec = bf16_vec;
            // pipelined kernel when dy needs no mask; SOL_WGRAD_FAST=0 forces the general kernel
            if (wgrad_pipelined) {
                int stages = knob(K_WGRAD_STAGES, 0);
                if (stages < 2 || stages > 4) stages = installed_plan(desc, SOL_PLAN_WGRAD).stages;
                if (stages < 2 || stages > 4)           // (a third stage has nothing to hold in ranges of two slices, and its LDS
                                                        // would keep the workgroups that re-pack from running two at a time:
                                                        // 3x3 512 -> 512, 49 pixels 14.2 -> 11.4 us)
                    stages = wp.m_per_split > 128 && (wp.splits * wp.tiles_k * wp.tiles_c <= 256 ||   // one workgroup per compute unit
                                                      (desc->KH == 1 && desc->KW == 1 && desc->stride == 1 && desc->pad == 0)) ? 3 : 2;
                trace_point(st, SOL_TRACE_WGRAD);
                if (plan.wide) {
                    // two tiles of the re-pack at a time per workgroup, on the compute units that the products leave idle
                    const int idle = (256 - (wp.splits * wp.tiles_k * wp.tiles_c) % 256) % 256, pairs = (wp.pack_tiles + 1) / 2;
                    const int blocks = idle > 32 ? idle : 32;
                    wp.pack_blocks = pairs < blocks ? pairs : blocks;
                    if (launch_wgrad_wide(wp, st) != hipSuccess) return SOL_ERR_LAUNCH;
                } else if (launch_wgrad_fast(wp, stages, st) != hipSuccess) return SOL_ERR_LAUNCH;
            } else {
                trace_point(st, SOL_TRACE_WGRAD_GENERAL);
                if (launch_wgrad(wp, vec, relu, st) != hipSuccess) return SOL_ERR_LAUNCH;
            }
        } else if (!dx) {
            DirectParams p = direct_params();
            trace_point(st, SOL_TRACE_DIRECT);
            if (launch_direct_bwd_f32(p, st) != hipSuccess) return SOL_ERR_LAUNCH;
        }
        if (reduce_may_ride) return SOL_OK;
        trace_point(st, SOL_TRACE_WGRAD_REDUCE);
        return launch_wgrad_reduce(rp, st) == hipSuccess ? SOL_OK : SOL_ERR_LAUNCH;
    };

    // the two branches share only inputs (dy, x, W, scale) and use disjoint parts of the workspace
    int status;
    if (pack_rides) {
        status = weight_branch(stream);
        if (status == SOL_OK) status = data_branch(stream);
        if (status == SOL_OK && !reduce_rode) {
            trace_point(stream, SOL_TRACE_WGRAD_REDUCE);
            if (launch_wgrad_reduce(rp, stream) != hipSuccess) status = SOL_ERR_LAUNCH;
        }
    } else {
        status = data_branch(stream);
        if (status == SOL_OK && dW) status = weight_branch(stream);
    }
    return status;
}

SOL_API int sol_block_bwd(const sol_block_desc* desc, const void* dy, const void* x, const void* W, const void* y, void* dx,
                  float* dW, float* dscale, float* dshift, const float* scale, void* dres, const void* dx_addend,
                  const void* dx_addend_mask, const void* dx_mask, void* ws, size_t ws_bytes, void* hip_stream) {
    return bwd_common(desc, dy, x, W, y, dx, dW, dscale, dshift, scale, dres, dx_addend, dx_addend_mask, dx_mask, ws,
                      ws_bytes, false, hip_stream);
}

SOL_API int sol_block_bwd_noalloc(const sol_block_desc* desc, const void* dy, const void* x, const void* W, const void* y,
                          void* dx, float* dW, float* dscale, float* dshift, const float* scale, void* dres,
                          const void* dx_addend, const void* dx_addend_mask, const void* dx_mask, void* hip_stream) {
    return bwd_common(desc, dy, x, W, y, dx, dW, dscale, dshift, scale, dres, dx_addend, dx_addend_mask, dx_mask, nullptr,
                      (size_t)SOL_NOALLOC_SCRATCH_BYTES, true, hip_stream);
}

SOL_API size_t sol_block_bwd_noalloc_limit(void) { return (size_t)SOL_NOALLOC_SCRATCH_BYTES; }

SOL_API int sol_block_set_plan(const sol_block_desc* desc, int which, const sol_plan* plan) {
    if (!desc) return SOL_ERR_NULL;
    if (which != SOL_PLAN_FWD && which != SOL_PLAN_DGRAD && which != SOL_PLAN_WGRAD) return SOL_ERR_UNSUPPORTED;
    Geometry g;
    if (int e = check_desc(desc, &g)) return e;
    if (plan) {
        const bool stages_ok = plan->stages == 0 || (plan->stages >= 2 && plan->stages <= 4);
        if (!stages_ok || plan->tile < -1 || plan->tile > 4 || (plan->tile == 3 && plan->stages == 4) ||
            plan->splits < 0 || plan->splits > 65535)
            return SOL_ERR_UNSUPPORTED;
    }
    std::lock_guard<std::mutex> lock(g_plan_mutex);
    if (plan) g_plans[plan_key(desc, which)] = *plan;
    else g_plans.erase(plan_key(desc, which));
    g_plan_count.store((int)g_plans.size(), std::memory_order_release);
    return SOL_OK;
}

SOL_API int sol_block_get_plan(const sol_block_desc* desc, int which, sol_plan* out) {
    if (!desc || !out) return SOL_ERR_NULL;
    if (which != SOL_PLAN_FWD && which != SOL_PLAN_DGRAD && which != SOL_PLAN_WGRAD) return SOL_ERR_UNSUPPORTED;
    *out = installed_plan(desc, which);
    return SOL_OK;
}

SOL_API void sol_reload_overrides(void) { load_knobs(); }

SOL_API void sol_clear_plans(void) {
    std::lock_guard<std::mutex> lock(g_plan_mutex);
    g_plans.clear();
    g_plan_count.store(0, std::memory_order_release);
}

SOL_API int sol_l1_loss_grad(int32_t dtype, const void* y, const void* t, void* dy, int64_t numel, int32_t mask_by_y,
                             void* hip_stream) {
    if (dtype != SOL_F32 && dtype != SOL_BF16) return SOL_ERR_UNSUPPORTED;
    if (numel < 1) return SOL_ERR_SHAPE;
    if (!y || !t || !dy) return SOL_ERR_NULL;
    if (misaligned(y) || misaligned(t) || misaligned(dy)) return SOL_ERR_ALIGN;
    clear_stale_error();
    trace_point((hipStream_t)hip_stream, SOL_TRACE_L1_GRAD);
    const int st = launch_l1_grad(dtype, y, t, dy, numel, mask_by_y, (hipStream_t)hip_stream) == hipSuccess ? SOL_OK : SOL_ERR_LAUNCH;
    return st;
}

SOL_API int sol_maxpool_fwd(int32_t dtype, const void* x, void* y, int32_t N, int32_t H, int32_t W, int32_t C, int32_t k,
                    int32_t stride, int32_t pad, void* hip_stream) {
    if (dtype != SOL_F32 && dtype != SOL_BF16) return SOL_ERR_UNSUPPORTED;
    if (N < 1 || H < 1 || W < 1 || C < 1 || k < 1 || stride < 1 || pad < 0 || pad >= k || H + 2 * pad < k ||
        W + 2 * pad < k)
        return SOL_ERR_SHAPE;
    if (!x || !y) return SOL_ERR_NULL;
    if (misaligned(x) || misaligned(y)) return SOL_ERR_ALIGN;
    clear_stale_error();
    trace_point((hipStream_t)hip_stream, SOL_TRACE_MAXPOOL);
    const int st = launch_maxpool(dtype, x, y, N, H, W, C, k, stride, pad, (hipStream_t)hip_stream) == hipSuccess
                       ? SOL_OK : SOL_ERR_LAUNCH;
    return st;
}

}  // extern "C"

// Pipelined implicit GEMM for stride-1 "same" convolutions (3x3, 5x5; forward and data gradient): the pixels a tile's taps
// need are copied into LDS once per 64-channel slice instead of once per tap.
//
// Tap (th, tw) of output pixel r reads source pixel r + dh * W + dw, counted through the whole tensor.  So the pixels of a
// tile of BP consecutive rows lie in one contiguous run of BP + 2 W + 2 source pixels (3x3), the region.  A tap is an
// offset into the region; lanes whose tap lies outside the image read a row of zeros instead.  Per slice and tap a
// workgroup copies the weights and a ninth of a region: 256 x 128 tile, 28 x 28 image 20 KiB instead of 48 KiB.  By the
// counters a 128 x 128 launch (12544 pixels, 256 -> 256) reads 1.06 M lines of 128 bytes from the L2, gathering tiles 1.72 M; its
// matrix units are busy 44 % of the time that its compute units are, with the four-wave gathering tile 40 %.  That alone makes
// it no faster than the eight-wave gathering tile; the larger tiles and those of 64 channels are.
//  * The reduction runs channel slice by channel slice, taps inside (the gathering tiles run taps outside: same products,
//    other order of the sums).  Weights stream through a ring of NSW slices, regions of two channel slices alternate: the
//    copies of the next region go out one or two per slice during the taps of this one.
//  * Region rows are swizzled by (row / 2) & 7, conflict-free for 16 rows from any start, so a tap costs a few vector
//    instructions per 32-pixel block (address, choice of the zero row) for 4 * TC MFMAs.
//  * Loop structure, barriers and epilogue are those of igemm_wide.hip.
// us on one box, operands rotating through HBM, 128 x 128 gathering tile of four waves / of eight waves (256 x 128 where that
// is marked) / here: 3x3 256 -> 256, 25088 pixels 44.3 / 33.6 (256 x 128) / 30.6 (970 TFLOP/s); 128 -> 128, 100352 pixels 51.6 / 40.5
// (256 x 128) / 39.7; 256 -> 256, 12544 pixels 23.4 / 19.0 / 19.2; 512 -> 512, 6272 pixels 46.0 / 34.1 / 34.4; 128 -> 128, 25088 pixels
// 14.6 / 11.9 / 11.6; 64 -> 64, 401408 pixels (128 x 64 in four waves) 77.5 / - / 47.1.
#include <type_traits>

#include "igemm_gather.h"
#include "launch.h"
#include "reduce_rows.h"

namespace sol {

// Rows are 128 bytes; any 16 consecutive rows at one logical chunk touch all 64 banks once, wherever they start.
__device__ __forceinline__ int halo_swizzle(int row) { return (row >> 1) & 7; }

template <int NC, int NM, int U = 0>
__device__ __forceinline__ void halo_pin() {
    if constexpr (U < NM) {
        constexpr int N = ((U + 1) * NC) / NM - (U * NC) / NM;
        if constexpr (N > 0) __builtin_amdgcn_sched_group_barrier(0x010, N, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        halo_pin<NC, NM, U + 1>();
    }
}

template <int BP, int BC, int WP, int WC, int NSW>
__global__ __launch_bounds__(64 * WP * WC) void igemm_halo_kernel(const IgemmParams p) {
    constexpr int NT = 64 * WP * WC, RPI = NT / 8;
    constexpr int LC = BC / RPI;           // weight copies per thread and slice
    constexpr int TP = BP / WP / 32, TC = BC / WC / 32;
    static_assert(TC == 2 && TP >= 1 && LC >= 1 && NSW >= 3, "a wave owns 64 channels");
    constexpr int WSTAGE = BC * 128;
    constexpr int ZERO = NSW * WSTAGE;     // byte offset of the row of zeros
    constexpr int REGION = ZERO + 128;     // ... of the first pixel region
    constexpr int EPITCH = 68;

    HIP_DYNAMIC_SHARED(uintx4, lds)
    unsigned char* const ldsb = reinterpret_cast<unsigned char*>(lds);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const RowClass rc = p.cls[0];
    SOL_FETCH_NOW_8(p.src, p.wmat, p.out, p.scale, p.shift, p.addend, p.addend_mask, p.out_mask);
    SOL_FETCH_NOW_8(p.src_bytes, p.Hs, p.Ws, p.Cs, p.Nc, p.tiles_c, p.total_tiles, p.relu);
    SOL_FETCH_NOW_8(rc.rows, rc.h_off, rc.w_off, rc.Th, rc.Tw, rc.tap_step, p.halo_first, p.halo_copies);
    SOL_FETCH_NOW_8(p.halo_pace, p.Nc, p.tiles_c, p.total_tiles, p.Ws, p.Cs, p.relu, rc.rows);
    SOL_FETCH_NOW_8(rc.Rh, rc.Rw, rc.div_img.magic, rc.div_img.shift, rc.div_rw.magic, rc.div_rw.shift, rc.h_mul, rc.w_mul);
    if ((int)blockIdx.x >= p.total_tiles) {    // workgroups behind the tiles: split reduction of the weight gradient
        reduce_rows_riding<(NT < 512), NT>(p.red, (int)blockIdx.x - p.total_tiles, p.red_blocks, reinterpret_cast<float*>(lds));
        return;
    }
    const int bid = xcd_remap(blockIdx.x, p.total_tiles);
    const int tc = bid % p.tiles_c, tp = bid / p.tiles_c;
    const int row0 = tp * BP, ch0 = tc * BC;
    const int cpt = p.Cs >> 6, ntaps = rc.Th * rc.Tw, nk = ntaps * cpt;
    const int K = ntaps * p.Cs;
    const int region_bytes = p.halo_copies * RPI * 128;
    const buffer_rsrc_t src_rs = make_buffer_rsrc(p.src, p.src_bytes);
    const buffer_rsrc_t w_rs = make_buffer_rsrc(p.wmat, (unsigned)((long long)K * p.Nc * 2));
    const int wp = wave % WP, wc = wave / WP;
    const int j8 = lane >> 3, pc = lane & 7;

    // ---- weights: slice (cs, tap) starts at tap * Cs + cs * 64 of every row
    unsigned wrowb[LC];
#pragma unroll
    for (int i = 0; i < LC; ++i) {
        const int lrow = RPI * i + 8 * wave + j8, c = ch0 + lrow;
        wrowb[i] = c < p.Nc ? (unsigned)(c * K + (pc ^ halo_swizzle(lrow)) * 8) * 2u : kOutOfRange;
    }
    int w_tap = 0;
    unsigned s_w = 0u;
    auto request_weights = [&](int stage) {
#pragma unroll
        for (int i = 0; i < LC; ++i) dma16_buf_to_lds(w_rs, wrowb[i], s_w, ldsb + stage * WSTAGE + (RPI * i + 8 * wave) * 128);
        if (++w_tap == ntaps) {
            w_tap = 0;
            s_w += 128u - (unsigned)((ntaps - 1) * p.Cs * 2);
        } else {
            s_w += (unsigned)(p.Cs * 2);
        }
    };
#pragma unroll
    for (int s = 0; s < NSW - 1; ++s)
        if (s < nk) request_weights(s);

    // ---- pixel region of a channel slice: source pixels row0 + halo_first + q, q = 0 .. BP + span - 1.  Rows before the
    // tensor wrap around to offsets beyond the descriptor's end, rows behind it lie there: both read zeros.
    const unsigned pix0 = (unsigned)((row0 + p.halo_first + 8 * wave + j8) * p.Cs + (pc ^ halo_swizzle(8 * wave + j8)) * 8) * 2u;
    auto request_pixels = [&](int buf, int i, int cs) {
        dma16_buf_to_lds(src_rs, pix0 + (unsigned)(i * RPI * p.Cs * 2), (unsigned)(cs * 128),
                         ldsb + REGION + buf * region_bytes + (i * RPI + 8 * wave) * 128);
    };
    for (int i = 0; i < p.halo_copies; ++i) request_pixels(0, i, 0);
    if (tid < 8) reinterpret_cast<uintx4*>(ldsb + ZERO)[tid] = uintx4{0u, 0u, 0u, 0u};

    // epilogue role, see igemm_wide.hip
    const int ecc = lane & 7, er0 = lane >> 3;
    const int ch = ch0 + wc * 64 + ecc * 8;
    const bool ch_ok = ch < p.Nc;
    floatx4 sc0 = {1.f, 1.f, 1.f, 1.f}, sc1 = sc0, sh0 = {0.f, 0.f, 0.f, 0.f}, sh1 = sh0;
    if (p.scale && ch_ok) {
        sc0 = *reinterpret_cast<const floatx4*>(p.scale + ch);
        sc1 = *reinterpret_cast<const floatx4*>(p.scale + ch + 4);
        sh0 = *reinterpret_cast<const floatx4*>(p.shift + ch);
        sh1 = *reinterpret_cast<const floatx4*>(p.shift + ch + 4);
    }

    // ---- taps that lie outside the image for this lane's pixels (one per 32-pixel block of the wave)
    const unsigned tap_rows = tap_row_bits(rc);
    unsigned badtap[TP];
#pragma unroll
    for (int j = 0; j < TP; ++j) {
        unsigned unused;
        gather_row(rc, row0 + wp * (BP / WP) + 32 * j + (lane & 31), 0, p.Hs, p.Ws, p.Cs, tap_rows, unused, badtap[j]);
    }

    floatx16 acc[TC][TP];
#pragma unroll
    for (int i = 0; i < TC; ++i)
#pragma unroll
        for (int j = 0; j < TP; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    // fragment addresses: weights per step; pixels per tap (step ks is the address with ks << 5 flipped)
    unsigned wad[4];
    {
        const int r = wc * 64 + (lane & 31);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) wad[ks] = (unsigned)(r * 128 + (((2 * ks + (lane >> 5)) ^ halo_swizzle(r)) << 4));
    }
    const int lrow = wp * (BP / WP) + (lane & 31);
    int t_tap = 0, t_tw = 0, t_th = 0, t_cs = 0;     // slice whose fragment addresses are set
    unsigned pad[TP];
    auto set_tap = [&]() {
        const int q = lrow + (rc.h_off + t_th * rc.tap_step) * p.Ws + rc.w_off + t_tw * rc.tap_step - p.halo_first;
        const unsigned a = (unsigned)(REGION + (t_cs & 1) * region_bytes + q * 128 + (((lane >> 5) ^ halo_swizzle(q)) << 4));
#pragma unroll
        for (int j = 0; j < TP; ++j)
            pad[j] = ((badtap[j] >> (t_tap & 31)) & 1u) ? (unsigned)(ZERO - j * 4096) : a;
    };
    auto next_tap = [&]() {
        ++t_tap;
        if (++t_tw == rc.Tw) {
            t_tw = 0;
            ++t_th;
        }
        if (t_tap == ntaps) {
            t_tap = 0;
            t_th = 0;
            ++t_cs;
        }
        set_tap();
    };
    set_tap();
    bf16x8 wf[2][TC], pf[2][TP];
    auto read_frags = [&](int buf, int stage, int ks) {
#pragma unroll
        for (int i = 0; i < TC; ++i)
            wf[buf][i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uintx4*>(ldsb + wad[ks] + (stage * WSTAGE + i * 4096)));
#pragma unroll
        for (int j = 0; j < TP; ++j)
            pf[buf][j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uintx4*>(ldsb + (pad[j] ^ (unsigned)(ks << 5)) + j * 4096));
    };
    auto multiply = [&](int buf) {
#pragma unroll
        for (int i = 0; i < TC; ++i)
#pragma unroll
            for (int j = 0; j < TP; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[buf][i], pf[buf][j], acc[i][j], 0, 0, 0);
    };
    auto slice = [&](auto stage, auto next_tag, auto more_tag) {
        constexpr int S = decltype(stage)::value;
        constexpr bool NEXT = decltype(next_tag)::value;
        constexpr bool MORE = decltype(more_tag)::value;
        constexpr int SN = (S + 1) % NSW, SR = (S + NSW - 1) % NSW;
        read_frags(1, S, 1);
        multiply(0);
        __builtin_amdgcn_sched_group_barrier(0x100, TC + TP, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, TC * TP, 0);
        read_frags(0, S, 2);
        __builtin_amdgcn_sched_group_barrier(0x100, TC + TP, 0);
        if constexpr (NEXT) {
            __builtin_amdgcn_s_waitcnt(MORE ? (0x0f70 | ((NSW - 3) * LC)) : 0x0f70);
            wg_barrier();
            // one copy of the next channel slice's region per slice; they come before the weight copies of this slice, so
            // the waits for weights cover them
            if (t_cs + 1 < cpt) {
                const int i = t_tap * p.halo_pace;
                if (i < p.halo_copies) request_pixels((t_cs + 1) & 1, i, t_cs + 1);
                if (p.halo_pace > 1 && i + 1 < p.halo_copies) request_pixels((t_cs + 1) & 1, i + 1, t_cs + 1);
            }
        }
        if constexpr (MORE) request_weights(SR);
        multiply(1);
        halo_pin<MORE ? LC : 0, TC * TP>();
        read_frags(1, S, 3);
        multiply(0);
        __builtin_amdgcn_sched_group_barrier(0x100, TC + TP, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, TC * TP, 0);
        if constexpr (NEXT) {
            next_tap();
            read_frags(0, SN, 0);
        }
        multiply(1);
        if constexpr (NEXT) __builtin_amdgcn_sched_group_barrier(0x100, TC + TP, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, TC * TP, 0);
    };
    wait_vm_and_lds<0>();
    wg_barrier();
    read_frags(0, 0, 0);
    auto run = [&](auto r_tag, auto all_tag) {
        constexpr int R = decltype(r_tag)::value;
        constexpr bool ALL = decltype(all_tag)::value;
        auto one = [&](auto i_tag) {
            constexpr int I = decltype(i_tag)::value;
            if constexpr (I < R)
                slice(std::integral_constant<int, I % NSW>{}, std::integral_constant<bool, ALL || (I < R - 1)>{},
                      std::integral_constant<bool, ALL || (I + NSW - 1 < R)>{});
        };
        one(std::integral_constant<int, 0>{});
        one(std::integral_constant<int, 1>{});
        one(std::integral_constant<int, 2>{});
        one(std::integral_constant<int, 3>{});
        one(std::integral_constant<int, 4>{});
        one(std::integral_constant<int, 5>{});
    };
    static_assert(2 * NSW - 2 <= 6, "the tail is written out for at most six slices");
    int kt = 0;
    for (; kt + 2 * NSW - 2 < nk; kt += NSW) run(std::integral_constant<int, NSW>{}, std::true_type{});
    switch (nk - kt) {
        case 1: run(std::integral_constant<int, 1>{}, std::false_type{}); break;
        case 2: run(std::integral_constant<int, 2>{}, std::false_type{}); break;
        case 3: run(std::integral_constant<int, 3>{}, std::false_type{}); break;
        case 4: run(std::integral_constant<int, 4>{}, std::false_type{}); break;
        case 5: if constexpr (NSW >= 4) run(std::integral_constant<int, 5>{}, std::false_type{}); break;
        default: if constexpr (NSW >= 4) run(std::integral_constant<int, 6>{}, std::false_type{}); break;
    }

    // ---- epilogue: every wave transposes its own pixels x 64 channels through LDS (fp32), no barrier after the first;
    // a lane then owns 8 consecutive channels of a pixel, a store instruction 8 whole 128-byte lines ----
    constexpr int PASSES = TP * 4;
    const uintx4 kOnes = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
    long long oofs[PASSES];
    bool ok[PASSES];
    uintx4 addv[PASSES], addm[PASSES], outm[PASSES];
    const int prow0 = row0 + wp * (BP / WP) + er0;
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
        const int r = prow0 + 8 * ps;
        ok[ps] = ch_ok && r < rc.rows;
        oofs[ps] = (long long)r * p.Nc + ch;
        addv[ps] = uintx4{0u, 0u, 0u, 0u};
        addm[ps] = kOnes;
        outm[ps] = kOnes;
    }
    if (p.addend) {
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps)
            if (ok[ps]) addv[ps] = *reinterpret_cast<const uintx4*>(p.addend + oofs[ps]);
        if (p.addend_mask) {
#pragma unroll
            for (int ps = 0; ps < PASSES; ++ps)
                if (ok[ps]) addm[ps] = *reinterpret_cast<const uintx4*>(p.addend_mask + oofs[ps]);
        }
    }
    if (p.out_mask) {
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps)
            if (ok[ps]) outm[ps] = *reinterpret_cast<const uintx4*>(p.out_mask + oofs[ps]);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    wg_barrier();                                   // every wave has read its last operands: the ring can be reused
    float* const stg = reinterpret_cast<float*>(ldsb) + wave * (32 * TP) * EPITCH;
#pragma unroll
    for (int j = 0; j < TP; ++j)
#pragma unroll
        for (int i = 0; i < TC; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<floatx4*>(stg + (32 * j + (lane & 31)) * EPITCH + i * 32 + 8 * q + 4 * (lane >> 5)) =
                    floatx4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
    floatx4 va[PASSES], vb[PASSES];
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
        va[ps] = *reinterpret_cast<const floatx4*>(stg + (er0 + 8 * ps) * EPITCH + ecc * 8);
        vb[ps] = *reinterpret_cast<const floatx4*>(stg + (er0 + 8 * ps) * EPITCH + ecc * 8 + 4);
    }
    const bool has_addend = p.addend != nullptr, has_outmask = p.out_mask != nullptr, relu = p.relu != 0;
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
        float v[8] = {va[ps][0], va[ps][1], va[ps][2], va[ps][3], vb[ps][0], vb[ps][1], vb[ps][2], vb[ps][3]};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[e] = fmaf(sc0[e], v[e], sh0[e]);
            v[e + 4] = fmaf(sc1[e], v[e + 4], sh1[e]);
        }
        if (has_addend) {
            const uintx4 a = mask_where_positive(addv[ps], addm[ps]);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[2 * e] += __uint_as_float(a[e] << 16);
                v[2 * e + 1] += __uint_as_float(a[e] & 0xffff0000u);
            }
        }
        if (relu) {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;   // never -0, NaN -> 0
        }
        uintx4 out = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])};
        if (has_outmask) out = mask_where_positive(out, outm[ps]);
        if (ok[ps]) store16_through(p.out + oofs[ps], out);
    }
}

template <int BP, int BC, int WP, int WC, int NSW>
static size_t halo_lds_bytes(const IgemmParams& p) {
    const size_t regions = p.Cs > 64 ? 2 : 1;
    const size_t loop = (size_t)NSW * BC * 128 + 128 + regions * p.halo_copies * (8 * WP * WC) * 128;
    const size_t epi = (size_t)BP * WC * 68 * 4;
    return loop > epi ? loop : epi;
}

template <int BP, int BC, int WP, int WC, int NSW>
static hipError_t launch_halo_tile(const IgemmParams& p, hipStream_t stream) {
    const size_t smem = halo_lds_bytes<BP, BC, WP, WC, NSW>(p);
    auto kern = igemm_halo_kernel<BP, BC, WP, WC, NSW>;
    static std::atomic<size_t> granted{0};
    if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), smem, granted); e != hipSuccess) return e;
    SOL_LAUNCH(kern, dim3(p.total_tiles + p.red_blocks), dim3(64 * WP * WC), smem, stream, p);
    return hipGetLastError();
}

// plans the tile (halo fields of p) and returns whether the launch can take it; *lds_bytes: of a workgroup
bool plan_igemm_halo(IgemmParams& p, int tile, int* bp, int* bc, size_t* lds_bytes) {
    static const int shapes[HALO_TILES][3] = {{256, 128, 64}, {128, 128, 64}, {128, 64, 32}};
    const RowClass& rc = p.cls[0];
    *bp = shapes[tile][0];
    *bc = shapes[tile][1];
    if (p.ncls != 1 || rc.h_mul != 1 || rc.w_mul != 1 || rc.Rh != p.Hs || rc.Rw != p.Ws || p.Hout != p.Hs || p.Wout != p.Ws ||
        rc.oh_mul != 1 || rc.ow_mul != 1 || rc.oh_off != 0 || rc.ow_off != 0 || rc.Th * rc.Tw < 9)
        return false;
    const int a = rc.h_off * p.Ws + rc.w_off;
    const int b = (rc.h_off + (rc.Th - 1) * rc.tap_step) * p.Ws + rc.w_off + (rc.Tw - 1) * rc.tap_step;
    p.halo_first = a < b ? a : b;
    const int rows = *bp + (a < b ? b - a : a - b), rpi = shapes[tile][2];
    p.halo_copies = (rows + rpi - 1) >> __builtin_ctz((unsigned)rpi);
    // the copies of the next region go out one or two per slice and must be done two slices before it is read
    p.halo_pace = p.halo_copies > rc.Th * rc.Tw - 2 ? 2 : 1;
    if (p.Cs > 64 && p.halo_copies > p.halo_pace * (rc.Th * rc.Tw - 2)) return false;
    size_t lds = 0;
    switch (tile) {
        case HALO_256x128: lds = halo_lds_bytes<256, 128, 4, 2, 4>(p); break;
        case HALO_128x128: lds = halo_lds_bytes<128, 128, 4, 2, 4>(p); break;
        default: lds = halo_lds_bytes<128, 64, 4, 1, 4>(p); break;
    }
    if (lds_bytes) *lds_bytes = lds;
    return lds <= 160 * 1024;
}

hipError_t launch_igemm_halo(const IgemmParams& p, int tile, hipStream_t stream) {
    if (p.total_tiles <= 0) return hipSuccess;
    switch (tile) {
        case HALO_256x128: return launch_halo_tile<256, 128, 4, 2, 4>(p, stream);
        case HALO_128x128: return launch_halo_tile<128, 128, 4, 2, 4>(p, stream);
        case HALO_128x64: return launch_halo_tile<128, 64, 4, 1, 4>(p, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace sol

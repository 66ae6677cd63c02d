// Pipelined implicit GEMM with eight waves per workgroup: 128 x 128, 256 x 128 and 128 x 256 tiles (pixels x channels).
//
// Same operand path as igemm_fast.hip (asynchronous 16-byte copies through buffer descriptors into a ring of 64-deep
// slices, one barrier in the middle of a slice, fragments of the next step requested before the MFMAs of this one), same
// order of the reduction, hence the same bits.  What differs:
//  * eight waves of (BP / WP) x 64 each, two per SIMD: while one waits for LDS or holds the issue port with a copy, the
//    other multiplies.
//  * The two larger tiles copy 48 KiB per 256 x 128 x 64 slice where two 128 x 128 tiles copy 64 KiB and need one
//    prologue and epilogue instead of two.
//    us on one box, operands that stay in the caches / that rotate through HBM, four waves of 64 x 64 (128 x 128, three stages)
//    -> here: 128 x 128: 3x3 256 -> 256, 12544 pixels 18.0 / 23.4 -> 17.6 / 19.0; 1x1 1024 -> 256 10.2 / 16.7 -> 9.8 / 13.5.
//    256 x 128: 3x3 256 -> 256, 25088 pixels 37.0 / 44.3 -> 30.1 / 33.6; 3x3 128 -> 128, 100352 pixels 45.6 / 51.6 -> 36.4 / 40.5;
//    1x1 1024 -> 512, 25088 pixels 47.9 / 59.1 -> 35.6 / 47.2 (128 x 256 35.2 / 42.1).  The 3x3 layers among them take the tiles
//    that keep a neighbourhood in LDS, which are up to a tenth faster still (igemm_halo.hip).
//  * Row r keeps logical chunk c at physical chunk c ^ ((r + r/8) & 7): 32 rows further that is chunk c ^ 4, so four
//    address registers per operand serve every fragment of every stage, the rest are immediates.
//  * The epilogue has one barrier (the ring is reused): every wave transposes its own pixels x 64 channels through LDS, a
//    lane then owns 8 channels of a pixel and a store instruction covers 8 whole 128-byte lines.
#include <type_traits>

#include "igemm_gather.h"
#include "launch.h"
#include "reduce_rows.h"

namespace sol {

__device__ __forceinline__ int wide_swizzle(int row) { return (row + (row >> 3)) & 7; }

template <int NC, int NM>
__device__ __forceinline__ void wide_pin_copies_between_mfmas() {
    constexpr int PAIRS = NC < NM ? NC : NM;
#pragma unroll
    for (int c = 0; c < PAIRS; ++c) {
        __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    }
    if constexpr (NC > PAIRS) __builtin_amdgcn_sched_group_barrier(0x010, NC - PAIRS, 0);
    if constexpr (NM > PAIRS) __builtin_amdgcn_sched_group_barrier(0x008, NM - PAIRS, 0);
}

template <int BP, int BC, int WP, int WC, int NS>
__global__ __launch_bounds__(64 * WP * WC) void igemm_wide_kernel(const IgemmParams p) {
    constexpr int NW = WP * WC, NT = 64 * NW;
    constexpr int RPI = NT / 8;            // rows covered by one copy instruction of every wave
    constexpr int LP = BP / RPI;           // async copies per thread and slice, pixel tile
    constexpr int LC = BC / RPI;           // ... weight tile
    constexpr int LPS = LP + LC;
    constexpr int TP = BP / WP / 32;
    constexpr int TC = BC / WC / 32;
    static_assert(NS >= 3 && TC == 2 && TP >= 1 && LP >= 1 && LC >= 1, "a wave owns 64 channels");
    constexpr int STAGEB = (BP + BC) * 128;   // bytes per stage
    constexpr int WCH = 64;
    constexpr int EPITCH = WCH + 4;           // fp32 pitch of a wave's epilogue staging block (32 pixels)

    HIP_DYNAMIC_SHARED(uintx4, lds)
    unsigned char* const ldsb = reinterpret_cast<unsigned char*>(lds);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    RowClass rc = p.cls[0];
    SOL_FETCH_NOW_8(p.src, p.wmat, p.out, p.scale, p.shift, p.addend, p.addend_mask, p.out_mask);
    SOL_FETCH_NOW_8(p.src_bytes, p.Hs, p.Ws, p.Cs, p.Nc, p.Hout, p.Wout, p.relu);
    SOL_FETCH_NOW_8(p.ncls, p.tiles_c, rc.rows, rc.Rh, rc.Rw, rc.h_mul, rc.h_off, rc.w_mul);
    SOL_FETCH_NOW_8(rc.w_off, rc.Th, rc.Tw, rc.tap_step, rc.oh_mul, rc.oh_off, rc.ow_mul, rc.ow_off);
    SOL_FETCH_NOW_8(rc.tile_begin, rc.linear, rc.b_off, rc.div_img.magic, rc.div_img.shift, rc.div_rw.magic,
                    rc.div_rw.shift, p.total_tiles);
    if ((int)blockIdx.x >= p.total_tiles) {    // workgroups behind the tiles: split reduction of the weight gradient
        reduce_rows_riding<false, NT>(p.red, (int)blockIdx.x - p.total_tiles, p.red_blocks, reinterpret_cast<float*>(lds));
        return;
    }
    const int bid = xcd_remap(blockIdx.x, p.total_tiles);
    const int tc = bid % p.tiles_c;
    int tp = bid / p.tiles_c;
    if (p.ncls > 1) {
        int cidx = 0;
#pragma unroll
        for (int i = 1; i < kMaxClasses; ++i)
            if (i < p.ncls && tp >= p.cls[i].tile_begin) cidx = i;
        rc = p.cls[cidx];
    }
    tp -= rc.tile_begin;
    const int row0 = tp * BP, ch0 = tc * BC;
    const int cpt = p.Cs >> 6;
    const int ntaps = rc.Th * rc.Tw;
    const int nk = ntaps * cpt;
    const long long K = (long long)ntaps * p.Cs;
    const bf16_t* wmat = p.wmat + rc.b_off;

    const int wp = wave % WP, wc = wave / WP;
    // epilogue role: 8 consecutive channels, rows er0 + 8 * pass of each 32-pixel block of this wave
    const int ecc = lane & 7, er0 = lane >> 3;
    const int ch = ch0 + wc * WCH + ecc * 8;
    const bool ch_ok = ch < p.Nc;
    floatx4 sc0 = {1.f, 1.f, 1.f, 1.f}, sc1 = sc0, sh0 = {0.f, 0.f, 0.f, 0.f}, sh1 = sh0;
    if (p.scale && ch_ok) {
        sc0 = *reinterpret_cast<const floatx4*>(p.scale + ch);
        sc1 = *reinterpret_cast<const floatx4*>(p.scale + ch + 4);
        sh0 = *reinterpret_cast<const floatx4*>(p.shift + ch);
        sh1 = *reinterpret_cast<const floatx4*>(p.shift + ch + 4);
    }

    const GatherBase gb = gather_base(rc, p.Ws, p.Cs);
    const unsigned margin = gb.margin;
    const int delta_min = gb.delta_min;
    const buffer_rsrc_t src_rs = make_buffer_rsrc(reinterpret_cast<const char*>(p.src) - margin, p.src_bytes + margin);
    const buffer_rsrc_t w_rs = make_buffer_rsrc(wmat, (unsigned)(K * p.Nc * 2));
    const int j8 = lane >> 3, pc = lane & 7;
    const bool weights_first = !(rc.linear & 1);
    unsigned wrowb[LC];
#pragma unroll
    for (int i = 0; i < LC; ++i) {
        const int lrow = RPI * i + 8 * wave + j8;
        const int c = ch0 + lrow;
        const int cl = pc ^ wide_swizzle(lrow);
        wrowb[i] = c < p.Nc ? (unsigned)(c * (int)K + cl * 8) * 2u : kOutOfRange;
    }
    auto weight_copies = [&](int stage, unsigned soff, int first, int last) {
#pragma unroll
        for (int iw = 0; iw < LC; ++iw)
            if (iw >= first && iw < last)
                dma16_buf_to_lds(w_rs, wrowb[iw], soff, ldsb + stage * STAGEB + (BP + RPI * iw + 8 * wave) * 128);
    };
    if (weights_first) {
#pragma unroll
        for (int s = 0; s < NS - 1; ++s)
            if (s < nk) weight_copies(s, (unsigned)(s * 128), 0, LC);
    }
    const unsigned tap_rows = tap_row_bits(rc);
    unsigned rowb[LP], badtap[LP];
#pragma unroll
    for (int i = 0; i < LP; ++i) {
        const int lrow = RPI * i + 8 * wave + j8;
        gather_row(rc, row0 + lrow, pc ^ wide_swizzle(lrow), p.Hs, p.Ws, p.Cs, tap_rows, rowb[i], badtap[i]);
    }
    // Requests are issued slice by slice in ring order, in parts between the MFMAs; the offsets of the next slice are
    // computed after the last copy of a request.
    int q_cs = 0, q_th = 0, q_tw = 0, q_tap = 0;
    unsigned s_pix = (unsigned)(-delta_min);
    unsigned s_w = 0u;
    unsigned voff[LP];
#pragma unroll
    for (int i = 0; i < LP; ++i) voff[i] = (rowb[i] + margin + (unsigned)delta_min) | (unsigned)__builtin_amdgcn_sbfe((int)badtap[i], 0, 1);
    auto next_pixel_slice = [&]() {
        if (__builtin_expect(++q_cs == cpt, 0)) {
            q_cs = 0;
            ++q_tap;
            if (++q_tw == rc.Tw) {
                q_tw = 0;
                ++q_th;
            }
            s_pix = (unsigned)((((q_th * p.Ws + q_tw) * rc.tap_step) * p.Cs) * 2 - delta_min);
#pragma unroll
            for (int i = 0; i < LP; ++i)
                voff[i] = (rowb[i] + margin + (unsigned)delta_min) | (unsigned)__builtin_amdgcn_sbfe((int)badtap[i], q_tap & 31, 1);
        } else {
            s_pix += 128u;
        }
    };
    auto request_part = [&](int stage, int part, int nparts) {
        unsigned char* st = ldsb + stage * STAGEB;
#pragma unroll
        for (int i = 0; i < LPS; ++i) {
            if (i < (part * LPS) / nparts || i >= ((part + 1) * LPS) / nparts) continue;
            if (i < LP) dma16_buf_to_lds(src_rs, voff[i], s_pix, st + (RPI * i + 8 * wave) * 128);
            else weight_copies(stage, s_w, i - LP, i - LP + 1);
        }
        if (part == nparts - 1) {
            s_w += 128u;
            next_pixel_slice();
        }
    };

    floatx16 acc[TC][TP];
#pragma unroll
    for (int i = 0; i < TC; ++i)
#pragma unroll
        for (int j = 0; j < TP; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
        if (s < nk) {
#pragma unroll
            for (int i = 0; i < LP; ++i) dma16_buf_to_lds(src_rs, voff[i], s_pix, ldsb + s * STAGEB + (RPI * i + 8 * wave) * 128);
            if (!weights_first) weight_copies(s, s_w, 0, LC);
            next_pixel_slice();
            s_w += 128u;
        }

    // Fragment addresses.  Row r keeps logical chunk c at physical chunk c ^ ((r + r/8) & 7).  32 rows further the
    // swizzle differs by 4 (mod 8), i.e. the chunk of step ks there is the chunk of step ks ^ 2 here: four address
    // registers per operand serve every fragment, the rest is an immediate.
    unsigned wad[4], pad[4];
    {
        const int h = lane >> 5;
        const int rw = wc * WCH + (lane & 31), rp = wp * (BP / WP) + (lane & 31);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            wad[ks] = (unsigned)(BP * 128 + rw * 128 + (((2 * ks + h) ^ wide_swizzle(rw)) << 4));
            pad[ks] = (unsigned)(rp * 128 + (((2 * ks + h) ^ wide_swizzle(rp)) << 4));
        }
    }
    bf16x8 wf[2][TC], pf[2][TP];
    auto read_frags = [&](int buf, int stage, int ks) {
#pragma unroll
        for (int i = 0; i < TC; ++i)
            wf[buf][i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uintx4*>(ldsb + wad[ks ^ (2 * (i & 1))] + (stage * STAGEB + i * 4096)));
#pragma unroll
        for (int j = 0; j < TP; ++j)
            pf[buf][j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uintx4*>(ldsb + pad[ks ^ (2 * (j & 1))] + (stage * STAGEB + j * 4096)));
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
        constexpr int SN = (S + 1) % NS, SR = (S + NS - 1) % NS;
        read_frags(1, S, 1);
        multiply(0);
        __builtin_amdgcn_sched_group_barrier(0x100, TC + TP, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, TC * TP, 0);
        read_frags(0, S, 2);
        __builtin_amdgcn_sched_group_barrier(0x100, TC + TP, 0);
        if constexpr (NEXT) {
            __builtin_amdgcn_s_waitcnt(MORE ? (0x0f70 | (((NS - 3) * LPS) & 15) | ((((NS - 3) * LPS) >> 4) << 14))
                                            : 0x0f70);
            wg_barrier();
        }
        if constexpr (MORE) request_part(SR, 0, 3);
        multiply(1);
        wide_pin_copies_between_mfmas<MORE ? LPS / 3 : 0, TC * TP>();
        read_frags(1, S, 3);
        if constexpr (MORE) request_part(SR, 1, 3);
        multiply(0);
        __builtin_amdgcn_sched_group_barrier(0x100, TC + TP, 0);
        wide_pin_copies_between_mfmas<MORE ? (2 * LPS) / 3 - LPS / 3 : 0, TC * TP>();
        if constexpr (NEXT) read_frags(0, SN, 0);
        if constexpr (MORE) request_part(SR, 2, 3);
        multiply(1);
        if constexpr (NEXT) __builtin_amdgcn_sched_group_barrier(0x100, TC + TP, 0);
        wide_pin_copies_between_mfmas<MORE ? LPS - (2 * LPS) / 3 : 0, TC * TP>();
    };
    if (nk < NS - 1) wait_vm_and_lds<0>();
    else if (weights_first) wait_vm_and_lds<LP>();
    else wait_vm_and_lds<(NS - 2) * LPS>();
    wg_barrier();
    if (nk > 0) {
        read_frags(0, 0, 0);
        auto run = [&](auto r_tag, auto all_tag) {
            constexpr int R = decltype(r_tag)::value;
            constexpr bool ALL = decltype(all_tag)::value;
            auto one = [&](auto i_tag) {
                constexpr int I = decltype(i_tag)::value;
                if constexpr (I < R)
                    slice(std::integral_constant<int, I % NS>{}, std::integral_constant<bool, ALL || (I < R - 1)>{},
                          std::integral_constant<bool, ALL || (I + NS - 1 < R)>{});
            };
            one(std::integral_constant<int, 0>{});
            one(std::integral_constant<int, 1>{});
            one(std::integral_constant<int, 2>{});
            one(std::integral_constant<int, 3>{});
            one(std::integral_constant<int, 4>{});
            one(std::integral_constant<int, 5>{});
        };
        static_assert(2 * NS - 2 <= 6, "the tail is written out for at most six slices");
        int kt = 0;
        for (; kt + 2 * NS - 2 < nk; kt += NS) run(std::integral_constant<int, NS>{}, std::true_type{});
        switch (nk - kt) {
            case 1: run(std::integral_constant<int, 1>{}, std::false_type{}); break;
            case 2: run(std::integral_constant<int, 2>{}, std::false_type{}); break;
            case 3: run(std::integral_constant<int, 3>{}, std::false_type{}); break;
            case 4: run(std::integral_constant<int, 4>{}, std::false_type{}); break;
            case 5: if constexpr (NS >= 4) run(std::integral_constant<int, 5>{}, std::false_type{}); break;
            default: if constexpr (NS >= 4) run(std::integral_constant<int, 6>{}, std::false_type{}); break;
        }
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
        oofs[ps] = ok[ps] ? output_offset(rc, r, p.Hout, p.Wout, p.Nc, ch) : 0;
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

template <int BP, int BC, int WP, int WC, int NS>
static hipError_t launch_wide_tile(const IgemmParams& p, hipStream_t stream) {
    const size_t stages = (size_t)NS * (BP + BC) * 128;
    const size_t epi = (size_t)BP * WC * 68 * 4;
    const size_t smem = stages > epi ? stages : epi;
    auto kern = igemm_wide_kernel<BP, BC, WP, WC, NS>;
    static std::atomic<size_t> granted{0};
    if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), smem, granted); e != hipSuccess) return e;
    SOL_LAUNCH(kern, dim3(p.total_tiles + p.red_blocks), dim3(64 * WP * WC), smem, stream, p);
    return hipGetLastError();
}

hipError_t launch_igemm_wide(const IgemmParams& p, int tile, hipStream_t stream) {
    if (p.total_tiles <= 0) return hipSuccess;
    switch (tile) {
        case WIDE_128x128: return launch_wide_tile<128, 128, 4, 2, 4>(p, stream);
        case WIDE_256x128: return launch_wide_tile<256, 128, 4, 2, 3>(p, stream);
        case WIDE_128x256: return launch_wide_tile<128, 256, 2, 4, 3>(p, stream);
        default: return hipErrorInvalidValue;
    }
}

void igemm_wide_tile_shape(int tile, int* bp, int* bc) {
    *bp = tile == WIDE_256x128 ? 256 : 128;
    *bc = tile == WIDE_128x256 ? 256 : 128;
}

}  // namespace sol

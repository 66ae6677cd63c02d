// Implicit GEMM for launches with few output tiles (small batches, the last stages of a network): the waves of a
// workgroup split the reduction instead of the tile.
//
// With 64 x 64 tiles such a launch leaves most compute units idle and every workgroup walks over the whole reduction, one
// memory latency per slice (0.2 us; 72 slices for a 3x3 over 512 channels).  Here a tile is as small as 16 x 16 (enough
// workgroups for the chip), and each of the 8 (6) waves takes every eighth (sixth) 64-deep slice of the reduction with a
// copy ring of its own: no barrier in the loop, every wave waits for its own copies only, and all their copies are in
// flight together.  By the fit of its times a compute unit copies about 100 bytes per ns into LDS, which bounds it.  The
// partial tiles meet in LDS and are added in the order of the waves (fixed, so runs repeat bit for bit; the sum of a
// reduction differs from the other kernels' in its last bits).
// One image, weights not in L2 (before: 64 x 64 tiles): 3x3 512 -> 512, 49 pixels 18.1 -> 6.2 us; 3x3 256 -> 256, 196
// pixels 10.9 -> 4.8; 1x1 2048 -> 512, 49 pixels 9.8 -> 4.2; 3x3 128 -> 128, 784 pixels 7.3 -> 4.5.  Six images: 18.6 ->
// 9.7, 11.0 -> 6.6, 10.1 -> 6.1, 7.3 -> 6.5.
#include <type_traits>

#include "igemm_gather.h"
#include "launch.h"
#include "reduce_rows.h"

namespace sol {

// Rows are 128 bytes (8 chunks of 16); 16 consecutive rows at one logical chunk touch all 64 banks once.
__device__ __forceinline__ int ksplit_swizzle(int row) { return (row >> 1) & 7; }

// Pins NC async copies and NM MFMAs in alternation.
template <int NC, int NM, int U = 0>
__device__ __forceinline__ void ksplit_pin() {
    if constexpr (U < NM) {
        constexpr int N = ((U + 1) * NC) / NM - (U * NC) / NM;
        if constexpr (N > 0) __builtin_amdgcn_sched_group_barrier(0x010, N, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        ksplit_pin<NC, NM, U + 1>();
    }
}

// RAGGED: source channels a multiple of 8 only; slices of the flattened (tap, channel) index and a chunk table, see
// igemm_fast.hip.
template <int MF, int TP, int TC, int KW, int NS, bool RAGGED>
__global__ __launch_bounds__(64 * KW) void igemm_ksplit_kernel(const IgemmParams p) {
    constexpr int BP = MF * TP, BC = MF * TC, NT = 64 * KW;
    constexpr int STEPS = MF == 32 ? 4 : 2;                     // MFMA steps per 64-deep slice: 32x32x16 or 16x16x32
    constexpr int LPC = 64 / MF;                                // lanes (k parts) per fragment row = 16-byte chunks per step
    constexpr int LP = BP / 8, LC = BC / 8, LPS = LP + LC;      // async copies of a wave per slice
    constexpr int STAGEB = (BP + BC) * 128;
    constexpr int RINGB = NS * STAGEB;                          // one wave's ring
    constexpr int PITCH = BC + 4;                               // fp32 pitch of a wave's partial tile
    static_assert(BP * PITCH * 4 <= RINGB, "the partial tile of a wave replaces its ring");
    static_assert((NS - 1) * LPS < 64, "vmcnt is a 6-bit field");

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
    const int K = ntaps * p.Cs;
    const int nk = RAGGED ? (K + 63) >> 6 : ntaps * cpt;
    const GatherBase gb = gather_base(rc, p.Ws, p.Cs);
    const buffer_rsrc_t src_rs = make_buffer_rsrc(reinterpret_cast<const char*>(p.src) - gb.margin, p.src_bytes + gb.margin);
    const buffer_rsrc_t w_rs = make_buffer_rsrc(p.wmat + rc.b_off, (unsigned)((long long)K * p.Nc * 2));
    unsigned char* const ring = ldsb + wave * RINGB;

    // copy i of a slice: rows 8 * i + (lane >> 3), physical chunk lane & 7
    const int j8 = lane >> 3, pc = lane & 7;
    unsigned wrowb[LC], rowb[LP], badtap[LP];
#pragma unroll
    for (int i = 0; i < LC; ++i) {
        const int lrow = 8 * i + j8, c = ch0 + lrow;
        wrowb[i] = c < p.Nc ? (unsigned)(c * K + (pc ^ ksplit_swizzle(lrow)) * 8) * 2u : kOutOfRange;
    }
    // slice of this wave that is requested next: tap and channel slice
    int q_sl = wave, q_cs = wave, q_th = 0, q_tw = 0, q_tap = 0;
    auto settle = [&]() {
        if constexpr (!RAGGED)
            while (q_cs >= cpt) {
                q_cs -= cpt;
                ++q_tap;
                if (++q_tw == rc.Tw) {
                    q_tw = 0;
                    ++q_th;
                }
            }
    };
    settle();
    uintx2* const table = reinterpret_cast<uintx2*>(ldsb + KW * RINGB);
    uintx2 chunk[2];                         // entries of this lane's two logical chunks of the slice that is requested
    if constexpr (RAGGED) {
        const int per_tap = p.Cs >> 3;
        for (int e = tid; e < nk * 8; e += NT) {
            const int tap = e / per_tap, c = e - tap * per_tap;
            const int th = tap / rc.Tw, tw = tap - th * rc.Tw;
            table[e] = e < (K >> 3) ? uintx2{(unsigned)((((th * p.Ws + tw) * rc.tap_step) * p.Cs + c * 8) * 2 - gb.delta_min), (unsigned)tap}
                                    : uintx2{0u, 0x80000000u};
        }
        __syncthreads();
    }
    auto request_weights = [&](int stage) {
        if constexpr (RAGGED) {
            const int mine = pc ^ ksplit_swizzle(j8);
            chunk[0] = table[q_sl * 8 + mine];
            chunk[1] = table[q_sl * 8 + (mine ^ 4)];
        }
#pragma unroll
        for (int i = 0; i < LC; ++i)
            dma16_buf_to_lds(w_rs, RAGGED ? wrowb[i] | (unsigned)((int)chunk[i & 1][1] >> 31) : wrowb[i], (unsigned)(q_sl * 128),
                             ring + stage * STAGEB + (BP + 8 * i) * 128);
    };
    auto request_pixels = [&](int stage) {
        if constexpr (RAGGED) {
#pragma unroll
            for (int i = 0; i < LP; ++i) {
                const uintx2 e = chunk[i & 1];
                const unsigned bad = (unsigned)__builtin_amdgcn_sbfe((int)badtap[i], e[1] & 31u, 1) | (unsigned)((int)e[1] >> 31);
                dma16_buf_to_lds(src_rs, (rowb[i] + gb.margin + (unsigned)gb.delta_min + e[0]) | bad, 0u, ring + stage * STAGEB + 8 * i * 128);
            }
        } else {
            const unsigned s_pix = (unsigned)((((q_th * p.Ws + q_tw) * rc.tap_step) * p.Cs + q_cs * 64) * 2 - gb.delta_min);
#pragma unroll
            for (int i = 0; i < LP; ++i)
                dma16_buf_to_lds(src_rs, (rowb[i] + gb.margin + (unsigned)gb.delta_min) | (unsigned)__builtin_amdgcn_sbfe((int)badtap[i], q_tap & 31, 1),
                                 s_pix, ring + stage * STAGEB + 8 * i * 128);
        }
        q_sl += KW;
        q_cs += KW;
        settle();
    };
    const int mine = nk > wave ? (nk - wave + KW - 1) / KW : 0;      // slices of this wave
    if (mine > 0) request_weights(0);                                // under the decoding of the rows
    const unsigned tap_rows = tap_row_bits(rc);
#pragma unroll
    for (int i = 0; i < LP; ++i)
        gather_row(rc, row0 + 8 * i + j8, RAGGED ? 0 : pc ^ ksplit_swizzle(8 * i + j8), p.Hs, p.Ws, p.Cs, tap_rows, rowb[i], badtap[i]);
    if (mine > 0) request_pixels(0);
#pragma unroll
    for (int s = 1; s < NS; ++s)
        if (s < mine) {
            request_weights(s);
            request_pixels(s);
        }

    typedef float acc_t __attribute__((ext_vector_type(MF * MF / 64)));
    acc_t acc[TC][TP];
#pragma unroll
    for (int i = 0; i < TC; ++i)
#pragma unroll
        for (int j = 0; j < TP; ++j)
#pragma unroll
            for (int v = 0; v < MF * MF / 64; ++v) acc[i][j][v] = 0.f;

    // epilogue role: 4 consecutive channels of row erow + pass * (rows per pass)
    constexpr int CPR = BC / 4, RPP = NT / CPR, PASSES = (BP + RPP - 1) / RPP;
    const int ecc = tid % CPR, erow = tid / CPR;
    const int ch = ch0 + ecc * 4;
    floatx4 sc = {1.f, 1.f, 1.f, 1.f}, sh = {0.f, 0.f, 0.f, 0.f};
    if (p.scale && ch < p.Nc) {
        sc = *reinterpret_cast<const floatx4*>(p.scale + ch);
        sh = *reinterpret_cast<const floatx4*>(p.shift + ch);
    }

    unsigned frow[STEPS];                    // byte offset of this lane's fragment row at the chunk of step ks
#pragma unroll
    for (int ks = 0; ks < STEPS; ++ks) {
        const int r = lane & (MF - 1);       // MF rows further the swizzle is the same
        frow[ks] = (unsigned)(r * 128 + (((LPC * ks + lane / MF) ^ ksplit_swizzle(r)) << 4));
    }
    // One slice.  Fragments are read one step ahead of their use; once the last step's are in registers the stage is free
    // and its next copies go out, under the MFMAs of the last two steps (the order is pinned: left alone, the scheduler
    // sinks every LDS read to its use and each step waits for it).
    auto multiply_slice = [&](int stage, auto more_tag) {
        constexpr bool MORE = decltype(more_tag)::value;
        const unsigned char* st = ring + stage * STAGEB;
        bf16x8 wf[STEPS][TC], pf[STEPS][TP];
        auto read_frags = [&](int ks) {
#pragma unroll
            for (int i = 0; i < TC; ++i) wf[ks][i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uintx4*>(st + frow[ks] + (BP + MF * i) * 128));
#pragma unroll
            for (int j = 0; j < TP; ++j) pf[ks][j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uintx4*>(st + frow[ks] + MF * j * 128));
            __builtin_amdgcn_sched_group_barrier(0x100, TC + TP, 0);
        };
        auto multiply = [&](int ks) {
#pragma unroll
            for (int i = 0; i < TC; ++i)
#pragma unroll
                for (int j = 0; j < TP; ++j) {
                    if constexpr (MF == 32) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[ks][i], pf[ks][j], acc[i][j], 0, 0, 0);
                    else acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[ks][i], pf[ks][j], acc[i][j], 0, 0, 0);
                }
        };
        auto pin_mfmas = [&]() { __builtin_amdgcn_sched_group_barrier(0x008, TC * TP, 0); };
        read_frags(0);
        read_frags(1);
        if constexpr (STEPS == 4) {
            multiply(0);
            pin_mfmas();
            read_frags(2);
            multiply(1);
            pin_mfmas();
            read_frags(3);
        }
        if constexpr (MORE) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            request_weights(stage);
            request_pixels(stage);
        }
        multiply(STEPS - 2);
        multiply(STEPS - 1);
        if constexpr (MORE) {                // copies and MFMAs alternate: a copy holds the wave's issue port for ~20 cycles
            ksplit_pin<LPS, 2 * TC * TP>();
        }
    };
    int stage = 0, t = 0;
    for (; t + NS < mine; ++t) {
        wait_vm_and_lds<(NS - 1) * LPS>();   // this wave's slice t has landed; nobody else touches the ring
        asm volatile("" ::: "memory");
        multiply_slice(stage, std::true_type{});
        stage = stage + 1 == NS ? 0 : stage + 1;
    }
    for (; t < mine; ++t) {
        if (NS >= 2 && t + 2 == mine) wait_vm_and_lds<LPS>();
        else if (NS >= 3 && t + 3 == mine) wait_vm_and_lds<NS >= 3 ? 2 * LPS : 0>();
        else if (NS >= 4 && t + 4 == mine) wait_vm_and_lds<NS >= 4 ? 3 * LPS : 0>();
        else wait_vm_and_lds<0>();
        asm volatile("" ::: "memory");
        multiply_slice(stage, std::false_type{});
        stage = stage + 1 == NS ? 0 : stage + 1;
    }

    // epilogue operands, requested before the waves meet
    long long oofs[PASSES];
    bool ok[PASSES];
    uintx2 addv[PASSES], addm[PASSES], outm[PASSES];
    const uintx2 kOnes = {0x3f803f80u, 0x3f803f80u};
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
        const int lr = erow + ps * RPP, r = row0 + lr;
        ok[ps] = lr < BP && r < rc.rows && ch < p.Nc;
        oofs[ps] = ok[ps] ? output_offset(rc, r, p.Hout, p.Wout, p.Nc, ch) : 0;
        addv[ps] = uintx2{0u, 0u};
        addm[ps] = kOnes;
        outm[ps] = kOnes;
        if (p.addend && ok[ps]) {
            addv[ps] = *reinterpret_cast<const uintx2*>(p.addend + oofs[ps]);
            if (p.addend_mask) addm[ps] = *reinterpret_cast<const uintx2*>(p.addend_mask + oofs[ps]);
        }
        if (p.out_mask && ok[ps]) outm[ps] = *reinterpret_cast<const uintx2*>(p.out_mask + oofs[ps]);
    }
    // partial tiles of the waves -> LDS [pixel][channel] (each over its own ring), added in the order of the waves
    float* const part = reinterpret_cast<float*>(ring);
#pragma unroll
    for (int j = 0; j < TP; ++j)
#pragma unroll
        for (int i = 0; i < TC; ++i)
#pragma unroll
            for (int q = 0; q < MF * MF / 256; ++q)       // a lane holds 4 consecutive channels of one pixel per group
                *reinterpret_cast<floatx4*>(part + (MF * j + (lane & (MF - 1))) * PITCH + i * MF + 8 * q + 4 * (lane / MF)) =
                    floatx4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    wg_barrier();
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
        const int lr = erow + ps * RPP;
        if (!ok[ps]) continue;
        floatx4 v = *reinterpret_cast<const floatx4*>(ldsb + (lr * PITCH + ecc * 4) * 4);
#pragma unroll
        for (int w = 1; w < KW; ++w) v += *reinterpret_cast<const floatx4*>(ldsb + w * RINGB + (lr * PITCH + ecc * 4) * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = fmaf(sc[e], v[e], sh[e]);
        if (p.addend) {
            const uintx2 a = mask_where_positive(addv[ps], addm[ps]);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                v[2 * e] += __uint_as_float(a[e] << 16);
                v[2 * e + 1] += __uint_as_float(a[e] & 0xffff0000u);
            }
        }
        if (p.relu) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;   // never -0, NaN -> 0
        }
        uintx2 out = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
        if (p.out_mask) out = mask_where_positive(out, outm[ps]);
        *reinterpret_cast<uintx2*>(p.out + oofs[ps]) = out;
    }
}

template <int MF, int TP, int TC, int KW, int NS, bool RAGGED>
static hipError_t launch_ksplit_tile(const IgemmParams& p, hipStream_t stream) {
    const size_t smem = (size_t)KW * NS * (TP + TC) * MF * 128 + (RAGGED ? igemm_chunk_table_bytes(p) : 0);
    auto kern = igemm_ksplit_kernel<MF, TP, TC, KW, NS, RAGGED>;
    static std::atomic<size_t> granted{0};
    if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), smem, granted); e != hipSuccess) return e;
    SOL_LAUNCH(kern, dim3(p.total_tiles + p.red_blocks), dim3(64 * KW), smem, stream, p);
    return hipGetLastError();
}

template <bool RAGGED>
static hipError_t launch_ksplit(const IgemmParams& p, int tile, hipStream_t stream) {
    switch (tile) {
        case KSPLIT_16x16: return launch_ksplit_tile<16, 1, 1, 8, 4, RAGGED>(p, stream);
        case KSPLIT_16x32: return launch_ksplit_tile<16, 1, 2, 8, 3, RAGGED>(p, stream);
        case KSPLIT_32x32: return launch_ksplit_tile<32, 1, 1, 8, 2, RAGGED>(p, stream);
        case KSPLIT_32x64: return launch_ksplit_tile<32, 1, 2, 6, 2, RAGGED>(p, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_igemm_ksplit(const IgemmParams& p, int tile, hipStream_t stream) {
    if (p.total_tiles <= 0) return hipSuccess;
    return (p.Cs & 63) == 0 ? launch_ksplit<false>(p, tile, stream) : launch_ksplit<true>(p, tile, stream);
}

void igemm_ksplit_tile_shape(int tile, int* bp, int* bc) {
    static const int shapes[4][2] = {{16, 16}, {16, 32}, {32, 32}, {32, 64}};
    const int t = tile < 0 || tile > 3 ? 3 : tile;
    *bp = shapes[t][0];
    *bc = shapes[t][1];
}

}  // namespace sol

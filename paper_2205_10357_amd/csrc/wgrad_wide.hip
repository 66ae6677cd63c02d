// Weight-gradient kernel with eight waves per workgroup (channel counts that are multiples of 8, dy already masked).
//
//   G[co][k] = sum_m g[m][co] * A[m][k]        A = im2col(x), k = (kh, kw, ci), ci fastest
//
// Tile, operand layout in LDS and transposing fragment reads are those of wgrad_fast_kernel (128 x 128 outputs, slices of
// 64 reduction rows of both operands); there four waves own a quarter of the tile each, one per SIMD, and every LDS wait and
// every barrier of that wave leaves its matrix unit idle.  Here two groups of four waves share the tile: group 0 multiplies
// the first 32 rows of every slice, group 1 the others, and the groups are added through LDS at the end.  Per flop the
// operands are copied as often as there, twice the waves hide the latencies, and a layer that ran two workgroups per
// compute unit needs half as many, i.e. half the fp32 partial tiles.
//
//  * The one barrier per slice sits between the slice's two steps: before it a wave has waited for its own copies of the
//    next slice, after it the first fragments of that slice are read, so the matrix unit has work queued across the barrier.
//  * The gather walks its rows: (row, column) of a thread's row advance by 64 rows per slice with two carries and a byte
//    offset that follows them, instead of two divisions and four 32-bit products per copy, and is ready before the barrier.
//
// 3x3 256 -> 256 channels, 12544 pixels, 6 splits: 21.8 us (680 TFLOP/s), and 17.5 for the data gradient that carries the
// reduction of 14 MB, where four waves and 13 splits took 23.0 and 20.1 for 31 MB.  A slice takes 0.42 us per compute unit, of
// which the matrix instructions are 0.21; launch, first copies and the partial tiles take the other 8 us.  1x1 / stride 1
// waits for memory either way (12.3 and 12.8 us for 1024 -> 256) and stays with four waves.
#include <type_traits>

#include "launch.h"
#include "pack_tile.h"
#include <sol_lds_tr.h>

namespace sol {

constexpr int WGW_TILE = 128;                 // tile edge along k and along co
constexpr int WGW_BM = 64;                    // reduction rows per slice
constexpr int WGW_OPER = WGW_BM * 16;         // 16-byte chunks of one operand tile
constexpr int WGW_STAGE = 2 * WGW_OPER;       // chunks per stage (x tile, then g tile)
constexpr int WGW_LDW = WGW_TILE + 4;         // fp32 pitch of the output staging tile

template <int NS>
__global__ __launch_bounds__(512) void wgrad_wide_kernel(const WgradParams p) {
    static_assert(NS >= 3, "the copies of slice s + NS - 1 replace slice s - 1");
    HIP_DYNAMIC_SHARED(uintx4, lds)
    constexpr int LPS = 4;                    // async copies per thread and slice (2 x rows + 2 g rows)

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);    // wave-uniform: keeps LDS bases scalar
    const int tiles = p.tiles_k * p.tiles_c;
    const int nwg = tiles * p.splits;         // workgroups that multiply; the launch may carry re-pack workgroups after them
    if ((int)blockIdx.x >= nwg) {
        for (int b = ((int)blockIdx.x - nwg) * 2; b < p.pack_tiles; b += p.pack_blocks * 2) {
            pack_dgrad_weights_tile(p.pack, b + (tid >> 8), p.pack_tiles, reinterpret_cast<bf16_t*>(lds) + (tid >> 8) * 64 * kPackTilePitch);
            __syncthreads();
        }
        return;
    }
    const int bid = xcd_remap(blockIdx.x, nwg);
    const int split = bid / tiles;
    const int t = bid - split * tiles;
    const int tk = t % p.tiles_k, tcn = t / p.tiles_k;
    const int k0 = tk * WGW_TILE, co0 = tcn * WGW_TILE;
    const int m_begin = split * p.m_per_split;
    const int m_end = min(p.M, m_begin + p.m_per_split);
    const int nsl = (m_end - m_begin + WGW_BM - 1) / WGW_BM;

    // ---- copy role: rows 32*i + 4*wave + (lane >> 4) of each operand tile, physical chunk lane & 15.
    // Copies go through buffer descriptors (see dma16_buf_to_lds): rows past the end of the range and taps outside the
    // image get an out-of-range offset, i.e. zeros.
    const buffer_rsrc_t x_rs = make_buffer_rsrc(p.x, (unsigned)((long long)p.N * p.H * p.W * p.C_in * 2));
    const buffer_rsrc_t g_rs = make_buffer_rsrc(p.dy, (unsigned)((long long)p.M * p.C_out * 2));
    const int mq = lane >> 4, pc = lane & 15;
    const int cl = pc ^ (4 * mq) ^ (2 * ((wave >> 1) & 1));       // logical chunk kept at physical chunk pc
    const int kx = k0 + cl * 8;               // first k of this thread's x chunk
    const bool kx_ok = kx < p.K;
    int kh = 0, kw = 0, ci = 0;
    if (kx_ok) {
        const int tap = kx / p.C_in;
        ci = kx - tap * p.C_in;
        kh = tap / p.KW;
        kw = tap - kh * p.KW;
    }
    const int cg = co0 + cl * 8;              // first channel of this thread's g chunk
    const bool cg_ok = cg < p.C_out;
    const int mrow0 = m_begin + 4 * wave + mq;            // this thread's row in slice 0, copy i adds 32*i
    unsigned xrow[2], grow[2];                             // byte offsets (x: of the next slice to make ready, g: at slice 0)
    int nvalid[2];                                         // slices in which copy i's row is inside [m_begin, m_end)
    // a row's position, the first valid one for this thread's tap and the last valid minus the first, and the advance by 64
    // rows = sa images, sb image rows, sc pixels
    int hpos[2], wpos[2], hlo = 0, wlo = 0;
    unsigned hspan = 0, wspan = 0;
    unsigned step0 = 0, step_w = 0, step_h = 0;
    int sb = 0, sc = 0;
    {
        const int sa = (int)fast_div(WGW_BM, p.div_howo), rest = WGW_BM - sa * p.Ho * p.Wo;
        sb = (int)fast_div((uint32_t)rest, p.div_wo);
        sc = rest - sb * p.Wo;
        const unsigned px = (unsigned)p.C_in * 2u;
        step0 = (unsigned)((sa * p.H + sb * p.stride) * p.W + sc * p.stride) * px;
        step_w = (unsigned)(p.stride * p.W - p.Wo * p.stride) * px;
        step_h = (unsigned)((p.H - p.Ho * p.stride) * p.W) * px;
        // image row h * stride + (kh - pad) lies in [0, H) for h in [hlo, hhi]
        const int dh = kh - p.pad, dw = kw - p.pad;
        hlo = dh < 0 ? (-dh + p.stride - 1) / p.stride : 0;
        wlo = dw < 0 ? (-dw + p.stride - 1) / p.stride : 0;
        // a tap that reaches no row or column of the image starts past any position
        const int hroom = p.H - 1 - dh, wroom = p.W - 1 - dw;         // h * stride <= hroom
        const int hhi = hroom >= 0 ? hroom / p.stride : -1, whi = wroom >= 0 ? wroom / p.stride : -1;
        const bool none = !kx_ok || hhi < hlo || whi < wlo;
        hspan = none ? 0u : (unsigned)(hhi - hlo);
        wspan = none ? 0u : (unsigned)(whi - wlo);
        if (none) hlo = 0x40000000;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int m = mrow0 + 32 * i;
        nvalid[i] = m < m_end ? (m_end - m + WGW_BM - 1) / WGW_BM : 0;
        grow[i] = cg_ok ? (unsigned)(m * p.C_out + cg) * 2u : kOutOfRange;
        const int n = (int)fast_div((uint32_t)m, p.div_howo), rem = m - n * p.Ho * p.Wo;
        hpos[i] = (int)fast_div((uint32_t)rem, p.div_wo);
        wpos[i] = rem - hpos[i] * p.Wo;
        xrow[i] = (unsigned)(((n * p.H + hpos[i] * p.stride - p.pad + kh) * p.W + wpos[i] * p.stride - p.pad + kw) * p.C_in + ci) * 2u;
    }

    // Requests go out right behind the barrier; the vector offsets of the next one are made ready long before, under the
    // matrix instructions.
    int q_sl = 0, q_stage = 0;                // next slice to request, and its stage
    unsigned gsoff = 0u, vx[2], vg[2];
    auto make_offsets = [&]() {               // of slice q_sl
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const unsigned inval = q_sl < nvalid[i] ? 0u : kOutOfRange;
            vg[i] = grow[i] | inval;
            const bool ok = (unsigned)(hpos[i] - hlo) <= hspan && (unsigned)(wpos[i] - wlo) <= wspan;
            vx[i] = (ok ? xrow[i] : kOutOfRange) | inval;
            wpos[i] += sc;
            const bool cw = wpos[i] >= p.Wo;
            wpos[i] -= cw ? p.Wo : 0;
            hpos[i] += sb + (cw ? 1 : 0);
            const bool ch = hpos[i] >= p.Ho;
            hpos[i] -= ch ? p.Ho : 0;
            xrow[i] += step0 + (cw ? step_w : 0u) + (ch ? step_h : 0u);
        }
    };
    auto request_x = [&]() {
        uintx4* st = lds + q_stage * WGW_STAGE + 4 * wave * 16;
#pragma unroll
        for (int i = 0; i < 2; ++i) dma16_buf_to_lds(x_rs, vx[i], 0u, st + 32 * i * 16);
    };
    auto request_g = [&]() {
        uintx4* st = lds + q_stage * WGW_STAGE + WGW_OPER + 4 * wave * 16;
#pragma unroll
        for (int i = 0; i < 2; ++i) dma16_buf_to_lds(g_rs, vg[i], gsoff, st + 32 * i * 16);
        gsoff += (unsigned)(WGW_BM * p.C_out * 2);
        ++q_sl;
        q_stage = q_stage + 1 == NS ? 0 : q_stage + 1;
    };
    make_offsets();

    // ---- MFMA role: group (steps 2 * group, 2 * group + 1 of a slice), wave grid 2 (k) x 2 (co), 64 x 64 each
    const int group = wave >> 2, wk = wave & 1, wcn = (wave >> 1) & 1;
    const int grp = lane >> 4, j = lane & 15;
    // byte offset (inside an operand tile) of this lane's first transposing read of fragment f:
    // row m = 8*(grp>>1) + (j>>2), channels r .. r+3 with r = base + 32*f + 16*(grp&1) + 4*(j&3)
    int xoff[2], goff[2];
#pragma unroll
    for (int f = 0; f < 2; ++f) {
        const int mrow = 8 * (grp >> 1) + (j >> 2);
        const int rx = wk * 64 + 32 * f + 16 * (grp & 1) + 4 * (j & 3);
        const int rg = wcn * 64 + 32 * f + 16 * (grp & 1) + 4 * (j & 3);
        const int sw = (4 * (mrow & 3)) ^ (2 * ((mrow >> 3) & 1));
        xoff[f] = mrow * 256 + (((rx >> 3) ^ sw) << 4) + ((rx >> 2) & 1) * 8 + group * 8192;
        goff[f] = mrow * 256 + (((rg >> 3) ^ sw) << 4) + ((rg >> 2) & 1) * 8 + group * 8192;
    }
    const bool do_shift = (tk == 0) && (wk == 0);
    // A group's two steps of a slice add up in accumulators of their own, which halves the chains of fp32 additions (relative
    // error of 3x3 256 -> 256, 12544 pixels against 64-bit sums 1.76e-7 -> 1.28e-7; 1.70e-7 with four waves and 14 splits).
    // The first product of each starts from the constant zero instead of cleared registers.
    floatx16 acc[2][2][2], accs[2];
    const floatx16 zero = {0.f};
    bf16x8 ones;
#pragma unroll
    for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.0f;

#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
        if (s < nsl) {
            request_x();
            request_g();
            make_offsets();
        }

    // Fragments of one 16-deep step: x^T rows (2 tiles) and g^T rows (2 tiles), two 8-byte transposing reads each.
    struct Frags {
        uintx2 r[8];
    };
    auto issue_frags = [&](Frags& fr, lds_addr_t base, auto step_tag) {
        constexpr int O = decltype(step_tag)::value * 4096;
        fr.r[0] = lds_tr_read_issue<O>(base + xoff[0]);
        fr.r[1] = lds_tr_read_issue<O + 1024>(base + xoff[0]);
        fr.r[2] = lds_tr_read_issue<O>(base + xoff[1]);
        fr.r[3] = lds_tr_read_issue<O + 1024>(base + xoff[1]);
        fr.r[4] = lds_tr_read_issue<O + WGW_OPER * 16>(base + goff[0]);
        fr.r[5] = lds_tr_read_issue<O + WGW_OPER * 16 + 1024>(base + goff[0]);
        fr.r[6] = lds_tr_read_issue<O + WGW_OPER * 16>(base + goff[1]);
        fr.r[7] = lds_tr_read_issue<O + WGW_OPER * 16 + 1024>(base + goff[1]);
    };
    auto frag = [](const Frags& fr, int i) {
        return __builtin_bit_cast(bf16x8, uintx4{fr.r[2 * i][0], fr.r[2 * i][1], fr.r[2 * i + 1][0], fr.r[2 * i + 1][1]});
    };
    auto multiply = [&](Frags& fr, auto set_tag, auto first_tag, auto newer_tag, auto shift_tag) {   // newer_tag: reads issued after fr's that may stay in flight
        lds_tr_wait<decltype(newer_tag)::value>(fr.r[0], fr.r[1], fr.r[2], fr.r[3], fr.r[4], fr.r[5], fr.r[6], fr.r[7]);
        constexpr int S = decltype(set_tag)::value;
        constexpr bool FIRST = decltype(first_tag)::value;      // the accumulators hold nothing yet
        const bf16x8 x0 = frag(fr, 0), x1 = frag(fr, 1), g0 = frag(fr, 2), g1 = frag(fr, 3);
        acc[S][0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x0, g0, FIRST ? zero : acc[S][0][0], 0, 0, 0);
        acc[S][0][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x0, g1, FIRST ? zero : acc[S][0][1], 0, 0, 0);
        acc[S][1][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x1, g0, FIRST ? zero : acc[S][1][0], 0, 0, 0);
        acc[S][1][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x1, g1, FIRST ? zero : acc[S][1][1], 0, 0, 0);
        if constexpr (decltype(shift_tag)::value) {
            accs[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, g0, FIRST && S == 0 ? zero : accs[0], 0, 0, 0);
            accs[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, g1, FIRST && S == 0 ? zero : accs[1], 0, 0, 0);
        }
    };
    const lds_addr_t lds0 = lds_byte_address(lds);
    auto stage_address = [&](int st) { return lds0 + (lds_addr_t)(st * WGW_STAGE * 16); };

    auto run = [&](auto shift_tag) {
        if (nsl < NS - 1) wait_vm_and_lds<0>();
        else wait_vm_and_lds<(NS - 2) * LPS>();
        wg_barrier();
        Frags fa, fb;
        int st = 0;
        issue_frags(fa, stage_address(0), std::integral_constant<int, 0>{});
        // (fragments in flight must not cross the loop's back edge, where the compiler may copy registers)
        auto settle = [&](Frags& fr) { lds_tr_wait<0>(fr.r[0], fr.r[1], fr.r[2], fr.r[3], fr.r[4], fr.r[5], fr.r[6], fr.r[7]); };
        settle(fa);
        // slice sl lies in stage st, its first step's fragments are in registers; MORE: slice sl + NS - 1 is requested
        auto slice = [&](auto first_tag, auto next_tag, auto more_tag) {
            constexpr bool NEXT = decltype(next_tag)::value, MORE = decltype(more_tag)::value;
            issue_frags(fb, stage_address(st), std::integral_constant<int, 1>{});
            multiply(fa, std::integral_constant<int, 0>{}, first_tag, std::integral_constant<int, 8>{}, shift_tag);
            if constexpr (NEXT) {
                constexpr int left = MORE ? (NS - 3) * LPS : 0;       // copies of slices sl + 2 .. may stay in flight
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_waitcnt(0x0f70 | (left & 15) | ((left >> 4) << 14));
                wg_barrier();                                         // slice sl + 1 has landed, slice sl - 1 is no longer read
                st = st + 1 == NS ? 0 : st + 1;
                issue_frags(fa, stage_address(st), std::integral_constant<int, 0>{});
                multiply(fb, std::integral_constant<int, 1>{}, first_tag, std::integral_constant<int, 8>{}, shift_tag);
                if constexpr (MORE) {
                    request_x();
                    request_g();
                    make_offsets();
#pragma unroll
                    for (int c = 0; c < 4; ++c) {                     // a copy holds the issue port while a product runs
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
                    }
                }
                settle(fa);                                           // under the MFMAs just issued
            } else {
                multiply(fb, std::integral_constant<int, 1>{}, first_tag, std::integral_constant<int, 0>{}, shift_tag);
            }
        };
        if (nsl > NS - 1) slice(std::true_type{}, std::true_type{}, std::true_type{});
        else if (nsl > 1) slice(std::true_type{}, std::true_type{}, std::false_type{});
        else slice(std::true_type{}, std::false_type{}, std::false_type{});
        int sl = 1;
        for (; sl + NS - 1 < nsl; ++sl) slice(std::false_type{}, std::true_type{}, std::true_type{});
        for (; sl + 1 < nsl; ++sl) slice(std::false_type{}, std::true_type{}, std::false_type{});
        if (sl < nsl) slice(std::false_type{}, std::false_type{}, std::false_type{});
    };
    if (do_shift) run(std::true_type{});
    else run(std::false_type{});
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[0][a][b] += acc[1][a][b];

    // ---- group 1 + group 0 through LDS; the partial tile leaves from there
    // (a lane holds channel co (lane & 31) and 4 consecutive k per quad; row 0 of the ones-product = accumulator element 0 of
    // lanes 0..31)
    float* stg = reinterpret_cast<float*>(lds);
    float* shift_sum = stg + WGW_TILE * WGW_LDW;              // [128], group 1's column sums
    auto staged = [&](auto f) {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    floatx4* at = reinterpret_cast<floatx4*>(stg + (wcn * 64 + 32 * b + (lane & 31)) * WGW_LDW + wk * 64 + 32 * a + 8 * q + 4 * (lane >> 5));
                    f(at, floatx4{acc[0][a][b][4 * q], acc[0][a][b][4 * q + 1], acc[0][a][b][4 * q + 2], acc[0][a][b][4 * q + 3]});
                }
    };
    wait_vm_and_lds<0>();
    wg_barrier();
    if (group == 1) {
        staged([](floatx4* at, floatx4 v) { *at = v; });
        if (do_shift && lane < 32) {
            shift_sum[wcn * 64 + lane] = accs[0][0];
            shift_sum[wcn * 64 + 32 + lane] = accs[1][0];
        }
    }
    __syncthreads();
    if (group == 0) {
        staged([](floatx4* at, floatx4 v) {
            const floatx4 w = *at;
            *at = floatx4{v[0] + w[0], v[1] + w[1], v[2] + w[2], v[3] + w[3]};
        });
        if (do_shift && lane < 32) {
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const int c = wcn * 64 + 32 * b + lane;
                if (co0 + c < p.C_out) p.dshift_partial[(long long)split * p.C_out + co0 + c] = accs[b][0] + shift_sum[c];
            }
        }
    }
    __syncthreads();
    float* part = p.partial + (long long)split * p.C_out * p.K;
    const int kq = (tid & 31) * 4, r0 = tid >> 5;
#pragma unroll
    for (int ps = 0; ps < WGW_TILE / 16; ++ps) {
        const int row = r0 + 16 * ps;
        const int co = co0 + row, k = k0 + kq;
        if (co < p.C_out && k < p.K)
            store16_through(part + (long long)co * p.K + k,
                            __builtin_bit_cast(uintx4, *reinterpret_cast<const floatx4*>(stg + row * WGW_LDW + kq)));
    }
}

hipError_t launch_wgrad_wide(const WgradParams& p, hipStream_t stream) {
    constexpr int NS = 4;
    const size_t smem = (size_t)NS * WGW_STAGE * 16;         // (the output staging tile and its column sums fit in the ring)
    static_assert(WGW_TILE * WGW_LDW * 4 + WGW_TILE * 4 <= NS * WGW_STAGE * 16, "output staging");
    auto kern = wgrad_wide_kernel<NS>;
    static std::atomic<size_t> granted{0};
    if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), smem, granted); e != hipSuccess) return e;
    SOL_LAUNCH(kern, dim3(p.tiles_k * p.tiles_c * p.splits + p.pack_blocks), dim3(512), smem, stream, p);
    return hipGetLastError();
}

}  // namespace sol

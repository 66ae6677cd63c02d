// Convolutions with very few input channels (the network stem: 7x7, stride 2, 3 -> 64 channels).
//
// With C_in = 3 a filter tap is 6 bytes of an NHWC row, so the implicit-GEMM kernels' 16-byte operand copies
// do not apply and their element-wise fallback is two orders of magnitude off the memory roofline of this
// layer (its output, not its arithmetic, is what must move).  Here:
//
//  * K is ordered (kh, kw', ci) with kw' = 0..7 and ci = 0..3: one filter row is a "run" of 8 consecutive
//    4-channel pixels = 32 K elements = two 16-deep MFMA steps, K = 32 * KH (taps kw' >= KW and channels >= C_in
//    carry zero weights);
//  * a workgroup computes 128 consecutive output pixels of one output row for all 64 output channels, then the row
//    below it, and so on.  The image rows under the window stay in a ring in LDS: an output row needs KH of them, but
//    only `stride` = 2 new ones, which are fetched as they lie in memory and widened to 4 channels on the way into
//    LDS.  The MFMA pixel operand of lane (pixel p, half h) at step (kh, half-run r) is the 16 bytes at pixel
//    p*2 + 4r + 2h of row kh -- an aligned ds_read_b128, consecutive lanes 16 bytes apart: no im2col copy exists
//    anywhere, and no widened copy of the image in memory;
//  * the accumulators hold 4 consecutive output channels per register group, so the epilogue (affine, ReLU, one
//    rounding) produces 8-byte pieces of NHWC rows.
//
// 32 images of 224 x 224, 7x7 / stride 2, 3 -> 64: forward 21.0 us, where a launch that wrote a widened copy of the image and
// a kernel that staged all KH rows of every tile from it took 6.5 + 22.0.  61 MB, so memory would allow 11 us; a launch
// costs 5 us before its first tile and a tile 0.8 us per compute unit, of which the matrix instructions are 0.4 and the LDS
// reads 0.5.
#include <stdlib.h>

#include <type_traits>

#include "launch.h"

namespace sol {

constexpr int SC_CO = 64;          // output channels (two 32-row MFMA tiles)
constexpr int SC_TILE = 128;       // output pixels of one row per workgroup tile
constexpr int SC_PW = SC_TILE * 2 + 8;      // staged pixels per image row (stride 2)
constexpr int SC_MAXKH = 8;

// ---- image rows: memory -> registers -> LDS ------------------------------------------------------------
// Three channels are 6 bytes at a 2-byte aligned address: a 2-byte and a 4-byte load, in the order that aligns the latter
// (by the parity of the pixel's first element), so that nothing outside the image is ever read.  Other channel counts
// (CIN = 0) take one 2-byte load per channel.  Pixels outside the image and missing channels lie outside the descriptor
// and read as zero.
template <int CIN>
struct RawPixel {
    uint32_t d, s;                 // three channels: the 4-byte and the 2-byte load; else channels 0, 1 and 2, 3
};

// The staged part of the image rows of one (image, row segment): pixel q of row i is image pixel (i - pad, wi0 + q),
// zero outside the image.
template <int CIN>
struct RowWindow {
    buffer_rsrc_t x;
    unsigned image;                // index of the image's first pixel in the tensor
    int H, W, C_in, pad, wi0;
    __device__ __forceinline__ unsigned index(int i, int q) const { return image + (unsigned)((i - pad) * W + wi0 + q); }
    __device__ __forceinline__ RawPixel<CIN> load(int i, int q, bool wanted = true) const {
        const bool in = wanted && (unsigned)(i - pad) < (unsigned)H && (unsigned)(wi0 + q) < (unsigned)W;
        const unsigned pixel = index(i, q);
        if (CIN == 3) {
            const unsigned odd = pixel & 1, a = pixel * 6;
            return {__builtin_amdgcn_raw_buffer_load_b32(x, in ? a + 2 * odd : kOutOfRange, 0, 0),
                    (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(x, in ? a + 4 - 4 * odd : kOutOfRange, 0, 0)};
        }
        uint32_t e[4];
#pragma unroll
        for (int c = 0; c < 4; ++c)
            e[c] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(x, in && c < C_in ? (pixel * C_in + c) * 2 : kOutOfRange, 0, 0);
        return {e[0] | (e[1] << 16), e[2] | (e[3] << 16)};
    }
    __device__ __forceinline__ uintx2 widen(RawPixel<CIN> r, int i, int q) const {
        const bool odd = CIN == 3 && (index(i, q) & 1);
        return odd ? uintx2{r.s | (r.d << 16), r.d >> 16} : uintx2{r.d, r.s};
    }
};

// Barrier after this wave's LDS operations only: global loads and stores stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("" ::: "memory");
    wait_vm_and_lds<63>();
    wg_barrier();
}

// ---- forward ---------------------------------------------------------------------------------------------
// Four waves of 32 pixels x 64 channels: a wave keeps the weights of all channels in registers (2 * 2 * KH x 16 bytes
// per lane) and reads each pixel fragment once for two MFMAs.  Tiles are numbered (image, segment, output row), row
// fastest, and a workgroup takes a contiguous range of them.  While tile i multiplies, the two rows of tile i + 1
// go from registers to the two ring slots that tile i does not read, so one barrier per tile suffices; those of tiles
// i + 2 and i + 3 are in flight, the latter issued before tile i's stores, whose completion they then need not wait for
// (vector memory operations complete in order).  Beyond the run the loads are issued all the same, out of range: the
// number in flight, which the waits count, is then the same on every path.  The epilogue's LDS staging is private to a wave.
constexpr int smallc_fwd_lds_bytes(int KH) {
    const int tile = (KH + 2) * SC_PW * 8 + 4 * 32 * 17 * 8, weights = 2 * KH * 4096;
    return tile > weights ? tile : weights;
}
template <int KH, int CIN>
__global__ __launch_bounds__(256, 2) void smallc_fwd_kernel(const SmallCParams p) {
    constexpr int KS = 2 * KH;                       // 16-deep MFMA steps
    constexpr int RING = KH + 2;
    constexpr int OP = 17;                           // 8-byte pieces per staged output pixel (16 + 1 of padding)
    constexpr int ROWS_BYTES = RING * SC_PW * 8;
    // the weights, as they lie and as operand image, share the LDS of ring and output staging
    extern __shared__ __align__(16) unsigned char smem[];            // smallc_fwd_lds_bytes(KH)
    __shared__ __align__(16) float affine[2][SC_CO];
    uintx2* ring = reinterpret_cast<uintx2*>(smem);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int segs = (p.Wo + SC_TILE - 1) / SC_TILE;
    const int tiles = p.N * p.Ho * segs;
    int t = (int)((long long)blockIdx.x * tiles / gridDim.x);
    const int end = (int)((long long)(blockIdx.x + 1) * tiles / gridDim.x);

    const buffer_rsrc_t image_rs = make_buffer_rsrc(p.x, (unsigned)(p.N * p.H * p.W * p.C_in) * 2u);
    // the run of consecutive output rows of one segment that starts at tile t: its first KH image rows, and those of its
    // next two tiles
    int seg, ho0, n, run;
    RowWindow<CIN> win;
    RawPixel<CIN> first[KH], firstx, next[2][3];
    const int xq = 256 + (tid & 7), xr = tid >> 3;   // the last eight pixels of a row: thread -> (row, pixel)
    auto request = [&](int i, RawPixel<CIN> (&v)[3]) {       // the two rows that tile i of the run needs beyond tile i - 1's
        const int r = ho0 * 2 + 2 * i + KH - 2;
        v[0] = win.load(r, tid, i < run);
        v[1] = win.load(r + 1, tid, i < run);
        v[2] = win.load(r + xr, xq, i < run && tid < 16);
    };
    auto begin_run = [&]() {
        seg = (t / p.Ho) % segs;
        ho0 = t % p.Ho;
        n = t / (p.Ho * segs);
        run = end - t < p.Ho - ho0 ? end - t : p.Ho - ho0;
        win = RowWindow<CIN>{image_rs, (unsigned)(n * p.H * p.W), p.H, p.W, p.C_in, p.pad, seg * SC_TILE * 2 - p.pad};
#pragma unroll
        for (int r = 0; r < KH; ++r) first[r] = win.load(ho0 * 2 + r, tid);
        firstx = win.load(ho0 * 2 + xr, xq, xr < KH);
        __builtin_amdgcn_sched_barrier(0);           // the order of the requests decides what a wait can leave in flight
        request(1, next[1]);
        __builtin_amdgcn_sched_barrier(0);
        request(2, next[0]);
        __builtin_amdgcn_sched_barrier(0);
    };

    // weights -> LDS as they lie -> operand image in LDS (element e of the piece of (step ks, channel co, half h):
    // W[co][ks/2][4*(ks&1) + 2*h + e/4][e%4] or 0) -> registers.  (Gathered from memory two bytes at a time the pieces kept the
    // address units of two workgroups busy for 3 us.)
    const int wpieces = SC_CO / 8 * KH * p.KW * p.C_in;
    uintx4 raw[KH];
#pragma unroll
    for (int k = 0; k < KH; ++k)
        if (tid + 256 * k < wpieces) raw[k] = reinterpret_cast<const uintx4*>(p.Wt)[tid + 256 * k];
    float affine_in = 0.f;
    if (tid < 2 * SC_CO) affine_in = tid < SC_CO ? p.scale[tid] : p.shift[tid - SC_CO];
    __builtin_amdgcn_sched_barrier(0);
    begin_run();                                     // arrives while the weights are sorted
    const uint16_t* wraw = reinterpret_cast<const uint16_t*>(smem + KH * 4096);
#pragma unroll
    for (int k = 0; k < KH; ++k)
        if (tid + 256 * k < wpieces) reinterpret_cast<uintx4*>(smem + KH * 4096)[tid + 256 * k] = raw[k];
    lds_barrier();
#pragma unroll
    for (int k = 0; k < KH; ++k) {
        const int i = tid + 256 * k, row = i >> 2, co = row / KH, kh = row % KH;        // row = co * KH + kh
        uint32_t e[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int kw = 2 * (i & 3) + (j >> 2), c = j & 3;
            const bool in = kw < p.KW && (CIN == 3 ? c < 3 : c < p.C_in);
            e[j] = CIN == 3 && c == 3 ? 0u : (uint32_t)wraw[in ? (row * p.KW + kw) * p.C_in + c : 0];
            e[j] = in ? e[j] : 0u;
        }
        reinterpret_cast<uintx4*>(smem)[((2 * kh + ((i >> 1) & 1)) * SC_CO + co) * 2 + (i & 1)] =
            uintx4{e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
    }
    if (tid < 2 * SC_CO) affine[tid >> 6][tid & 63] = affine_in;
    lds_barrier();
    uintx4 wf[KS][2];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int c = 0; c < 2; ++c)
            wf[ks][c] = reinterpret_cast<const uintx4*>(smem)[(ks * SC_CO + 32 * c + (lane & 31)) * 2 + (lane >> 5)];

    uintx2* outs = reinterpret_cast<uintx2*>(smem + ROWS_BYTES) + wave * 32 * OP;
    const int pl = wave * 32 + (lane & 31);          // output pixel of this lane inside the tile
    const uintx2* pixel0 = ring + pl * 2 + 2 * (lane >> 5);

    for (;;) {
        const int wo0 = seg * SC_TILE, row0 = ho0 * 2;       // row0: first image row under the window, pad added
        lds_barrier();                               // the previous run's rows (the weight image) have been read
#pragma unroll
        for (int r = 0; r < KH; ++r) ring[r * SC_PW + tid] = win.widen(first[r], row0 + r, tid);
        if (xr < KH) ring[xr * SC_PW + xq] = win.widen(firstx, row0 + xr, xq);
        lds_barrier();

        int base = 0;                                // ring slot of the window's first row
        auto tile = [&](int i, RawPixel<CIN> (&rows)[3]) {   // `rows`: what tile i + 1 needs beyond tile i
            floatx16 acc[2];
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[0][v] = acc[1][v] = 0.f;
#pragma unroll
            for (int kh = 0; kh < KH; ++kh) {
                const int slot = base + kh < RING ? base + kh : base + kh - RING;
                const uintx2* rowp = pixel0 + slot * SC_PW;
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const bf16x8 pf = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uintx4*>(rowp + 4 * r));
#pragma unroll
                    for (int c = 0; c < 2; ++c)
                        acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wf[2 * kh + r][c]), pf, acc[c], 0, 0, 0);
                }
            }
            {                                        // into the two slots that this tile does not read
                const int r = row0 + 2 * (i + 1) + KH - 2;
                int s0 = base + KH, s1 = base + KH + 1;
                s0 = s0 < RING ? s0 : s0 - RING;
                s1 = s1 < RING ? s1 : s1 - RING;
                ring[s0 * SC_PW + tid] = win.widen(rows[0], r, tid);
                ring[s1 * SC_PW + tid] = win.widen(rows[1], r + 1, tid);
                if (tid < 16) ring[(xr ? s1 : s0) * SC_PW + xq] = win.widen(rows[2], r + xr, xq);
                request(i + 3, rows);
            }
            // epilogue: affine, ReLU and the one rounding in the accumulator layout (channel 32c + 8g + 4*(lane/32) + e),
            // then through the wave's own LDS so that every store instruction writes whole 128-byte pixel rows
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int co = 32 * c + 8 * g + 4 * (lane >> 5);
                    const floatx4 sc = *reinterpret_cast<const floatx4*>(&affine[0][co]);
                    const floatx4 sh = *reinterpret_cast<const floatx4*>(&affine[1][co]);
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        v[e] = fmaf(sc[e], acc[c][4 * g + e], sh[e]);
                        if (p.relu) v[e] = v[e] > 0.f ? v[e] : 0.f;
                    }
                    outs[(lane & 31) * OP + 8 * c + 2 * g + (lane >> 5)] = uintx2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
                }
            asm volatile("" ::: "memory");           // a wave's LDS operations execute in order
            __builtin_amdgcn_wave_barrier();
            const int valid = p.Wo - wo0 < SC_TILE ? p.Wo - wo0 : SC_TILE;
            // pixels past the end of the row lie outside the descriptor, which drops their stores; write-through as in
            // store16_through, but known to the compiler, which counts it when it waits for the loads above
            const buffer_rsrc_t rs = make_buffer_rsrc(p.y + (((long long)n * p.Ho + ho0 + i) * p.Wo + wo0) * SC_CO, (unsigned)valid * SC_CO * 2);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int px = (lane >> 3) + 8 * j, c = lane & 7;
                const uintx2 a = outs[px * OP + 2 * c], b = outs[px * OP + 2 * c + 1];
                __builtin_amdgcn_raw_buffer_store_b128(uintx4{a[0], a[1], b[0], b[1]}, rs, (unsigned)((wave * 32 + px) * SC_CO * 2 + c * 16), 0, 17);
            }
            base = base + 2 < RING ? base + 2 : base + 2 - RING;
            lds_barrier();
        };
        int i = 0;
        for (; i + 1 < run; i += 2) {
            tile(i, next[1]);
            tile(i + 1, next[0]);
        }
        if (i < run) tile(i, next[1]);
        t += run;
        if (t >= end) break;
        begin_run();
    }
}

bool smallc_fwd_supported(int C_in, int C_out, int KH, int KW, int stride) {
    return C_in >= 1 && C_in <= 4 && C_out == SC_CO && KH >= 1 && KH <= SC_MAXKH && KW >= 1 && KW <= 8 && stride == 2;
}

// What a forward call asks of its workspace.  The kernels no longer use it; the sizes that the interface hands out (and
// with them which calls it takes) stay.
size_t smallc_fwd_workspace_bytes(int N, int H, int W, int KH) {
    return ((size_t)N * H * W * 4 * 2 + 255) / 256 * 256 + (size_t)2 * KH * SC_CO * 2 * 16;
}

template <int KH, int CIN>
static hipError_t launch_smallc_fwd_kh(const SmallCParams& p, hipStream_t stream) {
    const int segs = (p.Wo + SC_TILE - 1) / SC_TILE;
    const long long tiles = (long long)p.N * p.Ho * segs;
    const long long cap = 512;                                 // two workgroups per compute unit
    const int grid = (int)(tiles < cap ? tiles : cap);
    const size_t smem = smallc_fwd_lds_bytes(KH);
    auto kern = smallc_fwd_kernel<KH, CIN>;
    static std::atomic<size_t> granted{0};
    if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), smem, granted); e != hipSuccess) return e;
    SOL_LAUNCH(kern, dim3(grid), dim3(256), smem, stream, p);
    return hipGetLastError();
}

hipError_t launch_smallc_fwd(const SmallCParams& p, hipStream_t stream) {
    switch (p.KH) {
        case 1: return p.C_in == 3 ? launch_smallc_fwd_kh<1, 3>(p, stream) : launch_smallc_fwd_kh<1, 0>(p, stream);
        case 2: return p.C_in == 3 ? launch_smallc_fwd_kh<2, 3>(p, stream) : launch_smallc_fwd_kh<2, 0>(p, stream);
        case 3: return p.C_in == 3 ? launch_smallc_fwd_kh<3, 3>(p, stream) : launch_smallc_fwd_kh<3, 0>(p, stream);
        case 4: return p.C_in == 3 ? launch_smallc_fwd_kh<4, 3>(p, stream) : launch_smallc_fwd_kh<4, 0>(p, stream);
        case 5: return p.C_in == 3 ? launch_smallc_fwd_kh<5, 3>(p, stream) : launch_smallc_fwd_kh<5, 0>(p, stream);
        case 6: return p.C_in == 3 ? launch_smallc_fwd_kh<6, 3>(p, stream) : launch_smallc_fwd_kh<6, 0>(p, stream);
        case 7: return p.C_in == 3 ? launch_smallc_fwd_kh<7, 3>(p, stream) : launch_smallc_fwd_kh<7, 0>(p, stream);
        case 8: return p.C_in == 3 ? launch_smallc_fwd_kh<8, 3>(p, stream) : launch_smallc_fwd_kh<8, 0>(p, stream);
        default: return hipErrorInvalidValue;
    }
}

// ---- weight gradient ------------------------------------------------------------------------------------
// G[k'][co] = sum over pixels of P[px][k'] * g[px][co], with P the same (kh, kw', ci) view of the staged image
// rows as in the forward kernel: for filter row kh, P[px][0..31] are the 64 bytes at pixel 2*px of staged row kh
// (rows of this "matrix" are 16 bytes apart and overlap).  The reduction index is the pixel, which is the row
// index of both operands in memory, so both MFMA operands come from transposing LDS reads (ds_read_b64_tr_b16:
// per 16 lanes a 4 x 16 block, 4 reduction rows x 16 columns).
//
// A workgroup of eight waves takes two output rows at a time, and a contiguous range of such pairs: wave (slab, half)
// has 64 of the 256 pixels and filter-row slots 4*half .. 4*half + 3 for both channel tiles (4 x 2 register blocking: 12
// transposing reads per 8 MFMAs).  The image rows stay in a ring as in the forward kernel (a pair needs KH + 2, four of
// them new), the gradient rows have two buffers: one barrier per pair, the next pairs' operands on their way to registers.
// A slot without a filter row multiplies all-ones instead, and slot 7 (never a filter row) yields dshift.  At the end
// the slabs are added through LDS and the workgroup writes one fp32 partial, per channel KH*KW*C_in gradient columns, the
// column sum of g and its share of <W, G> (so that the sum over the workgroups can be split by columns);
// smallc_wgrad_reduce_kernel adds the workgroups in a fixed order.
// 32 images of 224 x 224, 7x7 / stride 2: 23.5 us + 5.4 us for the reduction.  With four waves, all KH rows per tile read from
// a widened copy of the image and one tile in flight: 6.3 (copy) + 39.0 + 9.7 us (the reduction on 64 compute units, each of
// which moves 25 bytes per ns at most).  64 MB, so memory would allow 12 us; a launch costs 8 us besides its pairs of rows,
// and a pair 1.9 us, of which the matrix instructions are 0.9.
constexpr int SC_GP = 160;         // bytes per staged gradient row (128 + 32: the 4 rows of a transposing read fall into
                                   // different banks)
constexpr int SC_SLAB = 8 * 2 * 16 * 64;             // accumulators of one slab (both halves), floats
constexpr int kExtraCols = 9;      // columns of a partial row behind the gradient: column sum, eight parts of <W, G>
constexpr int smallc_wgrad_lds_bytes(int KH) {
    const int operands = (KH + 6) * SC_PW * 8 + 4 * SC_TILE * SC_GP, slabs = 2 * SC_SLAB * 4;
    return operands > slabs ? operands : slabs;
}
template <int KH, int CIN>
__global__ __launch_bounds__(512, 2) void smallc_wgrad_kernel(const SmallCWgradParams p) {
    constexpr int RING = KH + 6;
    constexpr int ROWS_BYTES = RING * SC_PW * 8, G_BYTES = SC_TILE * SC_GP;       // G_BYTES: one row of gradients
    static_assert(KH <= 7, "filter-row slot 7 must be free for the column sums");
    extern __shared__ __align__(16) unsigned char smem[];            // smallc_wgrad_lds_bytes(KH), then W
    uintx2* ring = reinterpret_cast<uintx2*>(smem);
    unsigned char* gt = smem + ROWS_BYTES;                           // [buffer][row of the pair][pixel]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int slab = wave & 3, half = wave >> 2;
    const int grp = lane >> 4, j = lane & 15;
    const int segs = (p.Wo + SC_TILE - 1) / SC_TILE, pairs = (p.Ho + 1) >> 1;
    const int units = p.N * segs * pairs;
    int t = (int)((long long)blockIdx.x * units / gridDim.x);
    const int end = (int)((long long)(blockIdx.x + 1) * units / gridDim.x);

    const buffer_rsrc_t image_rs = make_buffer_rsrc(p.x, (unsigned)(p.N * p.H * p.W * p.C_in) * 2u);
    const buffer_rsrc_t grad_rs = make_buffer_rsrc(p.dy, (unsigned)(p.N * p.Ho * p.Wo * SC_CO) * 2u);
    uintx4* wstage = reinterpret_cast<uintx4*>(smem + smallc_wgrad_lds_bytes(KH));
    const int wpieces = SC_CO / 8 * KH * p.KW * p.C_in;
    uintx4 raw[(KH + 1) / 2];
#pragma unroll
    for (int k = 0; k < (KH + 1) / 2; ++k)
        if (tid + 512 * k < wpieces) raw[k] = reinterpret_cast<const uintx4*>(p.Wt)[tid + 512 * k];
#pragma unroll
    for (int k = 0; k < (KH + 1) / 2; ++k)
        if (tid + 512 * k < wpieces) wstage[tid + 512 * k] = raw[k];
    floatx16 acc[4][2];                              // [slot][channel tile]
#pragma unroll
    for (int v = 0; v < 16; ++v)
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[u][0][v] = acc[u][1][v] = 0.f;

    // lane part of the transposing-read addresses (reduction row 8*(grp>>1) + (j>>2), column piece 16*(grp&1) + 4*(j&3));
    // the slab is 64 pixels of row slab / 2 of the pair
    const int mrow = (slab & 1) * 64 + 8 * (grp >> 1) + (j >> 2);
    const unsigned char* gbase = gt + (slab >> 1) * G_BYTES + mrow * SC_GP + (16 * (grp & 1) + 4 * (j & 3)) * 2;
    const unsigned char* pbase = smem + mrow * 16 + 32 * (grp & 1) + 8 * (j & 3);
    const int gr = tid >> 8, gq = tid & 255;         // operand fetches: row parity, pixel (image) or 16-byte piece (gradient)
    const int xq = 256 + (tid & 7), xr = tid >> 3;   // the last eight pixels of a row: thread -> (row, pixel)

    while (t < end) {
        const int pair0 = t % pairs, seg = (t / pairs) % segs, n = t / (pairs * segs);
        const int run = end - t < pairs - pair0 ? end - t : pairs - pair0;
        const int wo0 = seg * SC_TILE;
        const int valid = p.Wo - wo0 < SC_TILE ? p.Wo - wo0 : SC_TILE;
        const RowWindow<CIN> win{image_rs, (unsigned)(n * p.H * p.W), p.H, p.W, p.C_in, p.pad, wo0 * 2 - p.pad};
        const int row0 = pair0 * 4;                  // first image row under the first pair's window, pad added

        struct Operands {
            uintx4 g[4];
            RawPixel<CIN> x[3];
        } next[2];
        RawPixel<CIN> first[(KH + 3) / 2], firstx;
        auto request_g = [&](int i, Operands& v) {   // gradient row gr of pair i; rows and pixels past the end are zero
            const int ho = 2 * (pair0 + i) + gr;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int px = (gq >> 3) + 32 * u;
                const unsigned at = (((unsigned)(n * p.Ho + ho) * p.Wo + wo0 + px) * SC_CO + (gq & 7) * 8) * 2u;
                v.g[u] = __builtin_amdgcn_raw_buffer_load_b128(grad_rs, i < run && ho < p.Ho && px < valid ? at : kOutOfRange, 0, 0);
            }
        };
        auto request = [&](int i, Operands& v) {     // pair i's gradients, and the four image rows it needs beyond pair i - 1's
            const int r = row0 + 4 * i + KH - 2;
            v.x[0] = win.load(r + gr, gq, i < run);
            v.x[1] = win.load(r + 2 + gr, gq, i < run);
            v.x[2] = win.load(r + xr, xq, i < run && tid < 32);
            request_g(i, v);
        };
        auto put_g = [&](int buf, const Operands& v) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                *reinterpret_cast<uintx4*>(gt + (2 * buf + gr) * G_BYTES + ((gq >> 3) + 32 * u) * SC_GP + (gq & 7) * 16) = v.g[u];
        };
        firstx = win.load(row0 + xr, xq, xr < KH + 2);
#pragma unroll
        for (int r = 0; r < (KH + 3) / 2; ++r) first[r] = win.load(row0 + 2 * r + gr, gq, 2 * r + gr < KH + 2);
        request_g(0, next[0]);
        __builtin_amdgcn_sched_barrier(0);           // the order of the requests decides what a wait can leave in flight
        request(1, next[1]);
        __builtin_amdgcn_sched_barrier(0);
        lds_barrier();                               // the previous run has been read
        put_g(0, next[0]);
#pragma unroll
        for (int r = 0; r < (KH + 3) / 2; ++r)
            if (2 * r + gr < KH + 2) ring[(2 * r + gr) * SC_PW + gq] = win.widen(first[r], row0 + 2 * r + gr, gq);
        if (xr < KH + 2) ring[xr * SC_PW + xq] = win.widen(firstx, row0 + xr, xq);
        __builtin_amdgcn_sched_barrier(0);
        request(2, next[0]);
        __builtin_amdgcn_sched_barrier(0);
        lds_barrier();

        int base = 0;                                // ring slot of the pair's first image row
        auto pair = [&](int i, Operands& v) {        // `v`: what pair i + 1 needs, for the buffers and slots that pair i does not read
            {
                const int r = row0 + 4 * (i + 1) + KH - 2;
                put_g((i + 1) & 1, v);
                int s0 = base + KH + 2 + gr, s1 = s0 + 2, sx = base + KH + 2 + xr;
                s0 = s0 < RING ? s0 : s0 - RING;
                s1 = s1 < RING ? s1 : s1 - RING;
                sx = sx < RING ? sx : sx - RING;
                ring[s0 * SC_PW + gq] = win.widen(v.x[0], r + gr, gq);
                ring[s1 * SC_PW + gq] = win.widen(v.x[1], r + 2 + gr, gq);
                if (tid < 32) ring[sx * SC_PW + xq] = win.widen(v.x[2], r + xr, xq);
                request(i + 3, v);                   // two pairs' operands in flight during this pair's arithmetic
            }
            const unsigned char* prow[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {            // slots without a filter row read the last one and discard it
                const int kh = 4 * half + u < KH ? 4 * half + u : KH - 1;
                int slot = base + 2 * (slab >> 1) + kh;
                slot = slot < RING ? slot : slot - RING;
                prow[u] = pbase + slot * SC_PW * 8;
            }
            const unsigned char* grow = gbase + 2 * (i & 1) * G_BYTES;
            // (the second row of the last pair of an odd height does not exist: its image rows must not be multiplied,
            // not even by zero)
            if (2 * (pair0 + i) + (slab >> 1) < p.Ho)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                bf16x8 gf[2];
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const unsigned char* a = grow + 16 * s * SC_GP + 64 * c;
                    const uintx2 g0 = lds_read_tr_b64(a), g1 = lds_read_tr_b64(a + 4 * SC_GP);
                    gf[c] = __builtin_bit_cast(bf16x8, uintx4{g0[0], g0[1], g1[0], g1[1]});
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const unsigned char* a = prow[u] + 16 * s * 16;
                    const uintx2 p0 = lds_read_tr_b64(a), p1 = lds_read_tr_b64(a + 64);
                    uintx4 pv = {p0[0], p0[1], p1[0], p1[1]};
                    if (u + 4 >= KH || u >= KH) {    // only then may the slot lack a filter row (no branch: a select)
                        const bool ones = 4 * half + u >= KH;
#pragma unroll
                        for (int e = 0; e < 4; ++e) pv[e] = ones ? 0x3f803f80u : pv[e];
                    }
#pragma unroll
                    for (int c = 0; c < 2; ++c)
                        acc[u][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, pv), gf[c], acc[u][c], 0, 0, 0);
                }
            }
            base = base + 4 < RING ? base + 4 : base + 4 - RING;
            lds_barrier();
        };
        int i = 0;
        for (; i + 1 < run; i += 2) {
            pair(i, next[1]);
            pair(i + 1, next[0]);
        }
        if (i < run) pair(i, next[1]);
        t += run;
    }

    // The four slabs are added through LDS: first a wave and its partner (slab ^ 1) exchange halves, the even slab keeps channel
    // tile 0, then with slab ^ 2 half of what is left, slabs 0 and 1 keep slots 0 and 1.  A wave's mail lies at its own place.
    floatx4* mail = reinterpret_cast<floatx4*>(smem);                 // [wave][piece][lane] of 16 bytes, 16 KiB per wave
    auto post = [&](int to, auto c_tag, auto u_tag) {                 // slots u .. u + 3 (or 1) of channel tile c
        constexpr int C = decltype(c_tag)::value, U = decltype(u_tag)::value;
#pragma unroll
        for (int u = 0; u < (U < 0 ? 4 : 2); ++u)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const floatx16& a = acc[(U < 0 ? 0 : U) + u][C];
                mail[to * 1024 + (u * 4 + g) * 64 + lane] = floatx4{a[4 * g], a[4 * g + 1], a[4 * g + 2], a[4 * g + 3]};
            }
    };
    auto open = [&](auto c_tag, auto u_tag) {
        constexpr int C = decltype(c_tag)::value, U = decltype(u_tag)::value;
#pragma unroll
        for (int u = 0; u < (U < 0 ? 4 : 2); ++u)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const floatx4 v = mail[wave * 1024 + (u * 4 + g) * 64 + lane];
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[(U < 0 ? 0 : U) + u][C][4 * g + e] += v[e];
            }
    };
    using std::integral_constant;
    __syncthreads();
    if (slab & 1) post(wave ^ 1, integral_constant<int, 0>{}, integral_constant<int, -1>{});
    else post(wave ^ 1, integral_constant<int, 1>{}, integral_constant<int, -1>{});
    __syncthreads();
    if (slab & 1) {
        open(integral_constant<int, 1>{}, integral_constant<int, -1>{});
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[u][0] = acc[u][1];
    } else {
        open(integral_constant<int, 0>{}, integral_constant<int, -1>{});
    }
    __syncthreads();
    if (slab & 2) post(wave ^ 2, integral_constant<int, 0>{}, integral_constant<int, 0>{});
    else post(wave ^ 2, integral_constant<int, 0>{}, integral_constant<int, 2>{});
    __syncthreads();
    if (slab & 2) {
        open(integral_constant<int, 0>{}, integral_constant<int, 2>{});
        acc[0][0] = acc[2][0];
        acc[1][0] = acc[3][0];
    } else {
        open(integral_constant<int, 0>{}, integral_constant<int, 0>{});
    }
    __syncthreads();

    // rows of the partial (gradient columns, column sum, eight parts of <W, G>) in LDS, then out as they lie
    // lane = channel (lane & 31); register group g holds filter column kw' = 2g + lane/32, element e channel e of the image
    const int K = KH * p.KW * p.C_in, cols = K + kExtraCols;
    float* rows = reinterpret_cast<float*>(smem);                     // [64][cols], at most 64 * 233 floats
    const bf16_t* wts = reinterpret_cast<const bf16_t*>(smem + smallc_wgrad_lds_bytes(KH));
    {
        const int co = 32 * (slab & 1) + (lane & 31);
        float dot = 0.f;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int kh = 4 * half + (slab & 2) + u;
            if (kh >= KH) {
                // slot 7 never has a filter row: every row of its ones-product is the column sum of g
                if (kh == 7 && lane < 32) rows[co * cols + K] = acc[u][0][0];
                continue;
            }
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int kw = 2 * g + (lane >> 5), o = (kh * p.KW + kw) * p.C_in;
                if (kw < p.KW) {
#pragma unroll
                    for (int e = 0; e < (CIN == 3 ? 3 : 4); ++e)
                        if (CIN == 3 || e < p.C_in) {
                            rows[co * cols + o + e] = acc[u][0][4 * g + e];
                            dot = fmaf(bf16_to_f32(wts[co * K + o + e]), acc[u][0][4 * g + e], dot);
                        }
                }
            }
        }
        rows[co * cols + K + 1 + 4 * half + (slab & 2) + (lane >> 5)] = dot;
    }
    __syncthreads();
    float* part = p.partial + (long long)blockIdx.x * SC_CO * cols;
    for (int i = tid; i < SC_CO * cols / 4; i += 512)
        store16_through(part + 4 * i, __builtin_bit_cast(uintx4, reinterpret_cast<const floatx4*>(rows)[i]));
}

// A workgroup of 512 threads sums 32 columns of one output channel over the partials (the last workgroup of a channel: the
// columns behind the gradient): 16 teams, team q takes partials q, q + 16, ... with 16 loads in flight, the team sums are
// added in a fixed order.  dW = scale * G, dshift = the column sum, dscale = <W[co,:], G[co,:]>.
__global__ __launch_bounds__(512) void smallc_wgrad_reduce_kernel(const SmallCWgradParams p) {
    __shared__ float team_sum[16][32];
    const int K = p.KH * p.KW * p.C_in, cols = K + kExtraCols, ranges = (K + 31) / 32 + 1;
    const int co = blockIdx.x / ranges, range = blockIdx.x - co * ranges;
    const int q = threadIdx.x >> 5, c = threadIdx.x & 31;
    const bool extra = range == ranges - 1;
    const int col = extra ? K + c : 32 * range + c;
    const bool live = col < (extra ? cols : K);
    const float* src = p.partial + (long long)co * cols + (live ? col : 0);
    const float sc = p.scale[co];
    float g = 0.f;
    for (int b = q; b < p.nparts; b += 16 * 16) {
        float a[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) a[u] = b + 16 * u < p.nparts ? src[(long long)(b + 16 * u) * SC_CO * cols] : 0.f;
#pragma unroll
        for (int u = 0; u < 16; ++u) g += a[u];
    }
    team_sum[q][c] = g;
    __syncthreads();
    if (q != 0 || !live) return;
    for (int u = 1; u < 16; ++u) g += team_sum[u][c];
    if (!extra) {
        const long long o = (long long)co * K + col;
        const float d = sc * g;
        p.dW[o] = p.accumulate ? p.dW[o] + d : d;
    } else {
        float d = g + __shfl_down(g, 1);                       // in lane 1: the eight parts of <W, G>
        d += __shfl_down(d, 2);
        d += __shfl_down(d, 4);
        if (c == 0) p.dshift[co] = p.accumulate ? p.dshift[co] + g : g;
        if (c == 1) p.dscale[co] = p.accumulate ? p.dscale[co] + d : d;
    }
}

bool smallc_wgrad_supported(int C_in, int C_out, int KH, int KW, int stride) {
    return smallc_fwd_supported(C_in, C_out, KH, KW, stride) && KH <= 7;
}

// What the weight gradient asks of the workspace: the partials (and, as in the forward pass, what the interface always
// asked for beyond them).
static int row_tiles(int N, int Ho, int Wo) {
    const long long tiles = (long long)N * Ho * ((Wo + SC_TILE - 1) / SC_TILE);
    return (int)(tiles < 256 ? tiles : 256);
}
size_t smallc_wgrad_workspace_bytes(int N, int H, int W, int Ho, int Wo) {
    return ((size_t)N * H * W * 4 * 2 + 255) / 256 * 256 + ((size_t)row_tiles(N, Ho, Wo) * SC_CO * 264 * 4 + 255) / 256 * 256;
}
// Workgroups: one per compute unit, at most one per pair of output rows.  Their partials, at most
// 64 * (7 * 8 * 4 + 9) floats each, fit the size above: there are no more of them than row tiles.
int smallc_wgrad_parts(int N, int Ho, int Wo) {
    const long long units = (long long)N * ((Ho + 1) / 2) * ((Wo + SC_TILE - 1) / SC_TILE);
    return (int)(units < 256 ? units : 256);
}

size_t smallc_wgrad_partial_bytes(int nparts, int K) { return (size_t)nparts * SC_CO * (K + kExtraCols) * 4; }

template <int KH, int CIN>
static hipError_t launch_smallc_wgrad_kh(const SmallCWgradParams& p, hipStream_t stream) {
    const size_t smem = smallc_wgrad_lds_bytes(KH) + SC_CO * KH * p.KW * p.C_in * 2;
    auto kern = smallc_wgrad_kernel<KH, CIN>;
    static std::atomic<size_t> granted{0};
    if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), smem, granted); e != hipSuccess) return e;
    SOL_LAUNCH(kern, dim3(p.nparts), dim3(512), smem, stream, p);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    const int ranges = (p.KH * p.KW * p.C_in + 31) / 32 + 1;
    SOL_LAUNCH(smallc_wgrad_reduce_kernel, dim3(SC_CO * ranges), dim3(512), 0, stream, p);
    return hipGetLastError();
}

hipError_t launch_smallc_wgrad(const SmallCWgradParams& p, hipStream_t stream) {
    switch (p.KH) {
        case 1: return p.C_in == 3 ? launch_smallc_wgrad_kh<1, 3>(p, stream) : launch_smallc_wgrad_kh<1, 0>(p, stream);
        case 2: return p.C_in == 3 ? launch_smallc_wgrad_kh<2, 3>(p, stream) : launch_smallc_wgrad_kh<2, 0>(p, stream);
        case 3: return p.C_in == 3 ? launch_smallc_wgrad_kh<3, 3>(p, stream) : launch_smallc_wgrad_kh<3, 0>(p, stream);
        case 4: return p.C_in == 3 ? launch_smallc_wgrad_kh<4, 3>(p, stream) : launch_smallc_wgrad_kh<4, 0>(p, stream);
        case 5: return p.C_in == 3 ? launch_smallc_wgrad_kh<5, 3>(p, stream) : launch_smallc_wgrad_kh<5, 0>(p, stream);
        case 6: return p.C_in == 3 ? launch_smallc_wgrad_kh<6, 3>(p, stream) : launch_smallc_wgrad_kh<6, 0>(p, stream);
        case 7: return p.C_in == 3 ? launch_smallc_wgrad_kh<7, 3>(p, stream) : launch_smallc_wgrad_kh<7, 0>(p, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace sol

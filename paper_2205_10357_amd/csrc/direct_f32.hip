// fp32 version of the block (SOL_F32): the small fp32 correctness configuration (tolerance 1e-5, which bf16 operands
// cannot meet); the throughput path is the bf16 MFMA code.
//
// The three passes are GEMMs on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32: fp32 products and sums).  At the sizes
// of this configuration a launch is latency, not arithmetic: a chain of dependent loads per output element took 18 us
// (forward), 26 us (data gradient) and 71 us (weight gradient) for 256 pixels of 16 channels.  So a workgroup owns one
// 16 x 16 tile of the result and its eight waves split the reduction, each with eight steps of operands in flight,
// gathered element by element straight into the registers the instruction reads; the partial tiles meet in LDS and are
// added in the order of the waves.  Data and weight gradient are one launch (workgroups of either kind), and the column
// sums of the gradient (dshift) come out of the operands of the first tile column.
// Measured for that block, forward + loss gradient + backward: 123 -> 27 us (of which the GPU works 19), 7 -> 4 launches.
// An operand that a tile shares between its rows or columns (weights, gradients) meets zeros where a filter tap lies outside
// the image or between the strides.  Such a product has to be skipped, not added: it is NaN for an infinite operand.  So a
// wave notes whether a shared operand is not finite, and such a tile is summed again product by product, taps skipped.
#include "launch.h"

namespace sol {

constexpr int kDirectWaves = 8;
constexpr int kDirectThreads = 64 * kDirectWaves;
constexpr int kDirectPitch = 17;
constexpr int kDirectUnroll = 8;
// A dimension of a launch may have at most 2^32 - 1 threads, and a tensor of few channels has more tiles than that allows
// (2^27 pixels of one channel: 2^23 tiles of 512 threads): tiles lie in rows of this many workgroups.  (A loop over tiles in
// a smaller grid took 77 registers instead of 50 and a tenth of the backward launch's speed.)
constexpr int kDirectRow = 1 << 20;
__device__ __forceinline__ int direct_tile_index() { return (int)(blockIdx.y * (unsigned)kDirectRow + blockIdx.x); }

struct DirectLds {
    float part[kDirectWaves * 16 * kDirectPitch];
    float colsum[kDirectWaves][16];
    int odd[kDirectWaves];                   // a shared operand of this wave was infinite or NaN
};

// The partial 16 x 16 tile of this wave over reduction indices [begin, end): a(k) is the element of row lane & 15 and
// b(k) that of column lane & 15 (0 where there is none); a lane feeds every fourth k.  odd: some shared(a, b) is not finite.
template <class A, class B, class S>
__device__ __forceinline__ floatx4 direct_tile(unsigned begin, unsigned end, int lane, bool& odd, A a, B b, S shared) {
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    float zero = 0.f;                        // becomes NaN: 0 x infinity, 0 x NaN
    for (unsigned k0 = begin + (lane >> 4); k0 < end + (lane >> 4); k0 += 4 * kDirectUnroll) {
        float av[kDirectUnroll], bv[kDirectUnroll];
#pragma unroll
        for (int u = 0; u < kDirectUnroll; ++u) {
            const unsigned k = k0 + 4 * u;
            av[u] = k < end ? a(k) : 0.f;
            bv[u] = k < end ? b(k) : 0.f;
        }
#pragma unroll
        for (int u = 0; u < kDirectUnroll; ++u) {
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u], bv[u], acc, 0, 0, 0);
            zero = fmaf(shared(av[u], bv[u]), 0.f, zero);
        }
    }
    odd = zero != 0.f;
    return acc;
}

// Sum of the waves' tiles at (row, column) = (tid % 16, tid / 16), for the first 256 threads; odd: some wave's was.
__device__ __forceinline__ float direct_sum(floatx4 acc, DirectLds& lds, int tid, bool& odd) {
    const int lane = tid & 63, wave = tid >> 6;
    float* mine = lds.part + wave * 16 * kDirectPitch;
#pragma unroll
    for (int v = 0; v < 4; ++v) mine[(lane & 15) * kDirectPitch + 4 * (lane >> 4) + v] = acc[v];
    const int any = __any(odd);
    if (lane == 0) lds.odd[wave] = any;
    __syncthreads();
    if (tid >= 256) return 0.f;
    float s = 0.f;
    int o = 0;
#pragma unroll
    for (int w = 0; w < kDirectWaves; ++w) {
        s += lds.part[w * 16 * kDirectPitch + (tid >> 4) * kDirectPitch + (tid & 15)];
        o |= lds.odd[w];
    }
    odd = o != 0;
    return s;
}

// the share of `total` reduction indices that wave `wave` takes: multiples of 4
__device__ __forceinline__ void direct_share(unsigned total, int wave, unsigned& begin, unsigned& end) {
    const unsigned q = ((total + 4 * kDirectWaves - 1) / (4 * kDirectWaves)) * 4;
    begin = min(total, wave * q);
    end = min(total, begin + q);
}

struct Pixel {
    int n, h, w;
    bool ok;
};
__device__ __forceinline__ Pixel pixel_of(unsigned i, unsigned count, FastDiv per_image, int image, FastDiv per_row, int row) {
    Pixel q;
    q.ok = i < count;
    const int j = q.ok ? (int)i : 0;
    q.n = (int)fast_div((uint32_t)j, per_image);
    const int rem = j - q.n * image;
    q.h = (int)fast_div((uint32_t)rem, per_row);
    q.w = rem - q.h * row;
    return q;
}

__device__ __forceinline__ float direct_gradient(const DirectParams& p, long long o) {
    const float g = p.dy[o];
    return p.ymask && !(p.ymask[o] > 0.f) ? 0.f : g;
}

// ---- one element of a result, product by product, taps outside the image skipped --------------------------------------
__device__ __forceinline__ float direct_fwd_element(const DirectParams& p, Pixel px, int co) {
    float acc = 0.f;
    for (int kh = 0; kh < p.KH; ++kh) {
        const int hi = px.h * p.stride - p.pad + kh;
        if ((unsigned)hi >= (unsigned)p.H) continue;
        for (int kw = 0; kw < p.KW; ++kw) {
            const int wi = px.w * p.stride - p.pad + kw;
            if ((unsigned)wi >= (unsigned)p.W_) continue;
            const float* xp = p.x + (((long long)px.n * p.H + hi) * p.W_ + wi) * p.C_in;
            const float* wp = p.W + (((long long)co * p.KH + kh) * p.KW + kw) * p.C_in;
            for (int ci = 0; ci < p.C_in; ++ci) acc = fmaf(xp[ci], wp[ci], acc);
        }
    }
    return acc;
}
__device__ __forceinline__ float direct_dgrad_element(const DirectParams& p, Pixel px, int ci) {
    float acc = 0.f;
    for (int kh = 0; kh < p.KH; ++kh) {
        const int th = px.h + p.pad - kh, ho = th / p.stride;
        if (th < 0 || ho * p.stride != th || ho >= p.Ho) continue;
        for (int kw = 0; kw < p.KW; ++kw) {
            const int tw = px.w + p.pad - kw, wo = tw / p.stride;
            if (tw < 0 || wo * p.stride != tw || wo >= p.Wo) continue;
            const long long o = (((long long)px.n * p.Ho + ho) * p.Wo + wo) * p.C_out;
            for (int co = 0; co < p.C_out; ++co)
                acc = fmaf(direct_gradient(p, o + co) * p.scale[co], p.W[(((long long)co * p.KH + kh) * p.KW + kw) * p.C_in + ci], acc);
        }
    }
    return acc;
}
__device__ __forceinline__ float direct_wgrad_element(const DirectParams& p, int kh, int kw, int ci, int co) {
    float acc = 0.f;
    for (int n = 0; n < p.N; ++n)
        for (int ho = 0; ho < p.Ho; ++ho) {
            const int hi = ho * p.stride - p.pad + kh;
            if ((unsigned)hi >= (unsigned)p.H) continue;
            for (int wo = 0; wo < p.Wo; ++wo) {
                const int wi = wo * p.stride - p.pad + kw;
                if ((unsigned)wi >= (unsigned)p.W_) continue;
                acc = fmaf(direct_gradient(p, (((long long)n * p.Ho + ho) * p.Wo + wo) * p.C_out + co),
                           p.x[(((long long)n * p.H + hi) * p.W_ + wi) * p.C_in + ci], acc);
            }
        }
    return acc;
}

// ---- tiles -------------------------------------------------------------------------------------------------------------
__device__ __forceinline__ void direct_fwd_tile(const DirectParams& p, int tile, DirectLds& lds) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const unsigned M = (unsigned)(p.N * p.Ho * p.Wo), K = (unsigned)(p.KH * p.KW * p.C_in);
    const int tiles_c = (p.C_out + 15) >> 4;
    const int tp = tile / tiles_c, tc = tile - tp * tiles_c;
    const Pixel px = pixel_of(tp * 16u + (lane & 15), M, p.div_howo, p.Ho * p.Wo, p.div_wo, p.Wo);
    const int co = tc * 16 + (lane & 15);
    const bool co_ok = co < p.C_out;
    unsigned begin, end;
    bool odd;
    direct_share(K, wave, begin, end);
    const floatx4 acc = direct_tile(begin, end, lane, odd,
        [&](unsigned k) { return co_ok ? p.W[(long long)co * K + k] : 0.f; },
        [&](unsigned k) {
            const int tap = (int)fast_div(k, p.div_cin), ci = (int)k - tap * p.C_in;
            const int kh = (int)fast_div((uint32_t)tap, p.div_kw), kw = tap - kh * p.KW;
            const int hi = px.h * p.stride - p.pad + kh, wi = px.w * p.stride - p.pad + kw;
            return px.ok && (unsigned)hi < (unsigned)p.H && (unsigned)wi < (unsigned)p.W_
                       ? p.x[(((long long)px.n * p.H + hi) * p.W_ + wi) * p.C_in + ci] : 0.f;
        },
        [](float w, float) { return w; });
    float z = direct_sum(acc, lds, tid, odd);
    const unsigned m = tp * 16u + (tid >> 4);
    const int c = tc * 16 + (tid & 15);
    if (tid >= 256 || m >= M || c >= p.C_out) return;
    if (odd) z = direct_fwd_element(p, pixel_of(m, M, p.div_howo, p.Ho * p.Wo, p.div_wo, p.Wo), c);
    const long long o = (long long)m * p.C_out + c;
    float v = fmaf(p.scale[c], z, p.shift[c]);
    if (p.res) v += p.res[o];
    if (p.relu) v = v > 0.f ? v : 0.f;
    p.y[o] = v;
}

__device__ __forceinline__ void direct_dgrad_tile(const DirectParams& p, int tile, DirectLds& lds) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const unsigned P = (unsigned)(p.N * p.H * p.W_), K = (unsigned)(p.KH * p.KW * p.C_out);      // k = (tap, output channel)
    const int tiles_c = (p.C_in + 15) >> 4;
    const int tp = tile / tiles_c, tc = tile - tp * tiles_c;
    const Pixel px = pixel_of(tp * 16u + (lane & 15), P, p.div_hw, p.H * p.W_, p.div_w, p.W_);
    const int ci = tc * 16 + (lane & 15);
    const bool ci_ok = ci < p.C_in;
    unsigned begin, end;
    bool odd;
    direct_share(K, wave, begin, end);
    const floatx4 acc = direct_tile(begin, end, lane, odd,
        [&](unsigned k) {
            const int tap = (int)fast_div(k, p.div_cout), co = (int)k - tap * p.C_out;
            return ci_ok ? p.W[((long long)co * p.KH * p.KW + tap) * p.C_in + ci] : 0.f;
        },
        [&](unsigned k) {
            const int tap = (int)fast_div(k, p.div_cout), co = (int)k - tap * p.C_out;
            const int kh = (int)fast_div((uint32_t)tap, p.div_kw), kw = tap - kh * p.KW;
            const int th = px.h + p.pad - kh, tw = px.w + p.pad - kw;
            if (!px.ok || th < 0 || tw < 0) return 0.f;
            const int ho = (int)fast_div((uint32_t)th, p.div_stride), wo = (int)fast_div((uint32_t)tw, p.div_stride);
            if (ho * p.stride != th || wo * p.stride != tw || ho >= p.Ho || wo >= p.Wo) return 0.f;
            return direct_gradient(p, (((long long)px.n * p.Ho + ho) * p.Wo + wo) * p.C_out + co) * p.scale[co];
        },
        [](float w, float) { return w; });
    float v = direct_sum(acc, lds, tid, odd);
    const unsigned m = tp * 16u + (tid >> 4);
    const int c = tc * 16 + (tid & 15);
    if (tid >= 256 || m >= P || c >= p.C_in) return;
    if (odd) v = direct_dgrad_element(p, pixel_of(m, P, p.div_hw, p.H * p.W_, p.div_w, p.W_), c);
    const long long o = (long long)m * p.C_in + c;
    if (p.addend && (!p.addend_mask || p.addend_mask[o] > 0.f)) v += p.addend[o];
    if (p.dx_mask && !(p.dx_mask[o] > 0.f)) v = 0.f;
    p.dx[o] = v;
}

__device__ __forceinline__ void direct_wgrad_tile(const DirectParams& p, int tile, DirectLds& lds) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const unsigned M = (unsigned)(p.N * p.Ho * p.Wo), K = (unsigned)(p.KH * p.KW * p.C_in);
    const int tiles_k = (int)((K + 15) >> 4);
    const int tc = tile / tiles_k, tk = tile - tc * tiles_k;
    auto tap_of = [&](unsigned k, int& kh, int& kw, int& ci) {
        const int tap = (int)fast_div(k, p.div_cin);
        ci = (int)k - tap * p.C_in;
        kh = (int)fast_div((uint32_t)tap, p.div_kw);
        kw = tap - kh * p.KW;
    };
    const unsigned k = tk * 16u + (lane & 15);
    const int co = tc * 16 + (lane & 15);
    const bool k_ok = k < K, co_ok = co < p.C_out;
    int kh, kw, ci;
    tap_of(k_ok ? k : 0u, kh, kw, ci);
    unsigned begin, end;
    bool odd;
    direct_share(M, wave, begin, end);
    float sum = 0.f;                         // of the gradients this lane feeds: its channel, every fourth pixel
    // (rows are the k of the weights, columns the output channels: a thread of the sum then stores along k)
    const floatx4 acc = direct_tile(begin, end, lane, odd,
        [&](unsigned m) {
            const Pixel px = pixel_of(m, M, p.div_howo, p.Ho * p.Wo, p.div_wo, p.Wo);
            const int hi = px.h * p.stride - p.pad + kh, wi = px.w * p.stride - p.pad + kw;
            return k_ok && (unsigned)hi < (unsigned)p.H && (unsigned)wi < (unsigned)p.W_
                       ? p.x[(((long long)px.n * p.H + hi) * p.W_ + wi) * p.C_in + ci] : 0.f;
        },
        [&](unsigned m) {
            const float g = co_ok ? direct_gradient(p, (long long)m * p.C_out + co) : 0.f;
            sum += g;
            return g;
        },
        [](float, float g) { return g; });
    if (tk == 0) {
        sum += __shfl_xor(sum, 16);
        sum += __shfl_xor(sum, 32);
        if (lane < 16) lds.colsum[wave][lane] = sum;
    }
    float g = direct_sum(acc, lds, tid, odd);
    const unsigned ke = tk * 16u + (tid & 15);
    const int ce = tc * 16 + (tid >> 4);
    if (tid < 256 && ke < K && ce < p.C_out) {
        if (odd) {
            tap_of(ke, kh, kw, ci);
            g = direct_wgrad_element(p, kh, kw, ci, ce);
        }
        p.G[(long long)ce * K + ke] = g;
    }
    if (tk == 0 && tid < 16 && tc * 16 + tid < p.C_out) {
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < kDirectWaves; ++w) s += lds.colsum[w][tid];
        p.dshift_partial[tc * 16 + tid] = s;
    }
}

__global__ __launch_bounds__(kDirectThreads) void direct_fwd_f32(const DirectParams p, int tiles) {
    __shared__ DirectLds lds;
    const int t = direct_tile_index();
    if (t < tiles) direct_fwd_tile(p, t, lds);
}

// Tiles [0, dgrad_tiles): data gradient; the rest: tiles of the unscaled weight gradient G.
__global__ __launch_bounds__(kDirectThreads) void direct_bwd_f32(const DirectParams p, int dgrad_tiles, int tiles) {
    __shared__ DirectLds lds;
    const int t = direct_tile_index();
    if (t < dgrad_tiles) direct_dgrad_tile(p, t, lds);
    else if (t < tiles) direct_wgrad_tile(p, t - dgrad_tiles, lds);
}

static void set_divisors(DirectParams& p) {
    p.div_cin = make_fast_div((uint32_t)p.C_in);
    p.div_cout = make_fast_div((uint32_t)p.C_out);
    p.div_kw = make_fast_div((uint32_t)p.KW);
    p.div_howo = make_fast_div((uint32_t)(p.Ho * p.Wo));
    p.div_wo = make_fast_div((uint32_t)p.Wo);
    p.div_hw = make_fast_div((uint32_t)(p.H * p.W_));
    p.div_w = make_fast_div((uint32_t)p.W_);
    p.div_stride = make_fast_div((uint32_t)p.stride);
}
// (a tensor has at most 2^31 - 1 elements: at most 2^27 tiles, as a column of 1 x n elements)
static inline long long tiles16(long long rows, long long cols) { return ((rows + 15) / 16) * ((cols + 15) / 16); }
static inline dim3 direct_grid(long long tiles) {
    if (tiles <= kDirectRow) return dim3((unsigned)tiles);
    return dim3(kDirectRow, (unsigned)((tiles + kDirectRow - 1) / kDirectRow));
}
static_assert((long long)kDirectRow * kDirectThreads < (1LL << 32), "threads of a launch");

hipError_t launch_direct_fwd_f32(const DirectParams& params, hipStream_t s) {
    DirectParams p = params;
    set_divisors(p);
    const long long tiles = tiles16((long long)p.N * p.Ho * p.Wo, p.C_out);
    SOL_LAUNCH(direct_fwd_f32, direct_grid(tiles), dim3(kDirectThreads), 0, s, p, (int)tiles);
    return hipGetLastError();
}

// data gradient (dx != null), weight gradient with its column sums (G != null), or both in one launch
hipError_t launch_direct_bwd_f32(const DirectParams& params, hipStream_t s) {
    DirectParams p = params;
    set_divisors(p);
    const long long dgrad = p.dx ? tiles16((long long)p.N * p.H * p.W_, p.C_in) : 0;
    const long long wgrad = p.G ? tiles16((long long)p.KH * p.KW * p.C_in, p.C_out) : 0;
    SOL_LAUNCH(direct_bwd_f32, direct_grid(dgrad + wgrad), dim3(kDirectThreads), 0, s, p, (int)dgrad, (int)(dgrad + wgrad));
    return hipGetLastError();
}

}  // namespace sol

// Gather addressing shared by the implicit-GEMM kernels that copy through buffer descriptors: where a GEMM row (pixel)
// starts in the source tensor and which of its filter taps lie inside the image.
#pragma once
#include "common.h"

namespace sol {

// The per-slice part of a gathered address is one wave-uniform scalar offset, which must not be negative, while the taps
// of a row may lie before it (padding) or run backwards (data gradient).  So the buffer descriptor starts `margin` bytes
// before the tensor and every vector offset carries the bias `margin + delta_min`; the scalar offset of a tap is its
// distance from tap 0 minus delta_min.  Only addresses inside the tensor are dereferenced.
struct GatherBase {
    int delta_min;
    unsigned margin;
};
__device__ __forceinline__ GatherBase gather_base(const RowClass& rc, int Ws, int Cs) {
    const int tap0_first = ((rc.h_off * Ws + rc.w_off) * Cs) * 2;
    const int tap_last = ((((rc.Th - 1) * Ws + (rc.Tw - 1)) * rc.tap_step) * Cs) * 2;
    const int delta_min = tap_last < 0 ? tap_last : 0;
    return GatherBase{delta_min, (unsigned)((tap0_first < 0 ? -tap0_first : 0) - delta_min)};
}

__device__ __forceinline__ unsigned low_bits(int n) { return n >= 32 ? 0xffffffffu : (1u << n) - 1u; }   // n in 0 .. 32

// bit th * Tw set for every row of taps (at most 32 taps in all)
__device__ __forceinline__ unsigned tap_row_bits(const RowClass& rc) {
    unsigned bits = 0u;
    for (int th = 0; th < rc.Th; ++th) bits |= 1u << (th * rc.Tw);
    return bits;
}

// GEMM row r: byte offset of (row, tap 0, channel chunk cl) modulo 2^32, and one bit per tap that lies outside the image
// (all ones for rows past the end).  Valid taps form an interval in either direction: the width interval is repeated in
// every row of taps by one multiplication and cut down to the valid rows of taps.
__device__ __forceinline__ void gather_row(const RowClass& rc, int r, int cl, int Hs, int Ws, int Cs, unsigned tap_rows, unsigned& rowb,
                                           unsigned& badtap) {
    rowb = 0u;
    badtap = 0xffffffffu;
    if (r >= rc.rows) return;
    if (rc.linear & 1) {
        rowb = (unsigned)(r * Cs + cl * 8) * 2u;
        badtap = 0xfffffffeu;
        return;
    }
    const int n = (int)fast_div((uint32_t)r, rc.div_img), rem = r - n * rc.Rh * rc.Rw;
    const int rh = (int)fast_div((uint32_t)rem, rc.div_rw), rw = rem - rh * rc.Rw;
    const int h0 = rh * rc.h_mul + rc.h_off, w0 = rw * rc.w_mul + rc.w_off;
    rowb = (unsigned)(((n * Hs + h0) * Ws + w0) * Cs + cl * 8) * 2u;
    auto interval = [&](int v0, int extent, int taps, int& l, int& h) {
        const int lo = rc.tap_step > 0 ? -v0 : v0 - extent + 1;
        const int hi = rc.tap_step > 0 ? extent - 1 - v0 : v0;
        l = lo > 0 ? lo : 0;
        h = hi < taps - 1 ? hi : taps - 1;
    };
    int hl, hh, wl, wh;
    interval(h0, Hs, rc.Th, hl, hh);
    interval(w0, Ws, rc.Tw, wl, wh);
    if (hh >= hl && wh >= wl) {
        const unsigned wgood = low_bits(wh + 1) & ~low_bits(wl);
        badtap = ~((wgood * tap_rows) & low_bits((hh + 1) * rc.Tw) & ~low_bits(hl * rc.Tw));
    }
}

// Element offset of output channel ch of GEMM row r (r must exist).
__device__ __forceinline__ long long output_offset(const RowClass& rc, int r, int Hout, int Wout, int Nc, int ch) {
    if (rc.linear & 2) return (long long)r * Nc + ch;
    const int n = (int)fast_div((uint32_t)r, rc.div_img), rem = r - n * rc.Rh * rc.Rw;
    const int rh = (int)fast_div((uint32_t)rem, rc.div_rw), rw = rem - rh * rc.Rw;
    return (((long long)n * Hout + (rh * rc.oh_mul + rc.oh_off)) * Wout + (rw * rc.ow_mul + rc.ow_off)) * Nc + ch;
}

}  // namespace sol

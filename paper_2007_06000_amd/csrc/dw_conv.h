// Depthwise 3x3 (stride 1) -> 1x1 convolution (stride 1) without LDS (included by kernels.hip; paper Table 1, a.2).
//
// The block moves its input and output once and does little else (16 channels of 80 x 80, batch 32: 26 MB, 164 MFLOP), so
// it is bound by memory as long as enough requests are in flight.  The general kernel (KIND_DW in block_kernel) runs in
// phases that a barrier separates -- input to LDS, depthwise layer to LDS, matrix operations, stores -- with a chip-wide
// single round of workgroups, so loads, arithmetic and stores do not overlap: 16.3 us.  Here a wave works alone: a
// lane owns a pixel column of R output rows and 4 of the 8 or 16 channels of a K step, which is what a matrix operation
// takes as its pixel operand, so the depthwise results go from the multiply-adds straight into the matrix operations.  A
// lane reads its (R + 2) x 3 window per channel from memory (neighbouring lanes share cache lines; R rows share window
// rows), every load of a K step in flight together, no barrier, no LDS.  12.7 us for that block (2.1 TB/s; a copy of as many
// bytes takes 5); 8 -> 24 channels of 100 x 90, batch 24: 14.7 -> 12.3 us.  R = 2 or 4 rows: the window's extra rows against
// waves in flight (13.4 and 13.8 us at R = 2 and 4 with 1600 and 800 workgroups, 15.2 us with 32-wide operations, which
// leave half of their rows idle at 16 channels).  From 3 K steps on, or with few waves, the general kernel is as fast
// (32 -> 64 channels of 50 x 61, batch 8: 8.3 and 8.4 us) or faster, so both stay and the planner's estimate decides.
//
// BlockParams used: x, y, N, Cin, H, W, Ho, Wo, Cy, c1 (depthwise tables: wp = [channel group][tap] float4, aff =
// [channel group][scale, shift] float4, pad, relu), c2[0] (pointwise), coff2[0], tw x th (pixels and rows of a wave's tile),
// tiles_x, tiles_y, csplit, nblocks.  A wave's tile is PW columns x (MF / PW) * R rows.
#pragma once

namespace xl {

template <int MF, int NRT, int R, int PW>
__global__ void __launch_bounds__(256) dw_pointwise_kernel(const BlockParams P)
{
    typedef MM<MF> M;
    touch_arguments();
    const int L = logical_block() * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tiles = P.tiles_x * P.tiles_y;
    if (L >= P.N * P.csplit * tiles) return;        // (wave-uniform; nothing below waits for another wave)
    const int lane = threadIdx.x & 63, sub = lane / MF, col = lane % MF;
    const int n = L / (tiles * P.csplit), in_image = L - n * (tiles * P.csplit);
    const int cs = in_image / tiles, tile = in_image - cs * tiles;
    const int ty = tile / P.tiles_x, tx = tile - ty * P.tiles_x;
    const int x = tx * PW + col % PW, y0 = ty * P.th + (col / PW) * R;
    const int HW = P.H * P.W, C = P.Cin;
    const ConvW &c1 = P.c1, &c2 = P.c2[0];

    // the lane's window: byte offsets from the first channel of its K step; outside the image past the end of the buffer
    // (an image has less than 2^30 elements)
    const __amdgpu_buffer_rsrc_t xr = make_rsrc(P.x + (size_t)n * C * HW, (unsigned long long)C * HW * 4ull);
    unsigned off[R + 2][3];
#pragma unroll
    for (int u = 0; u < R + 2; ++u)
#pragma unroll
        for (int v = 0; v < 3; ++v) {
            const int gy = y0 - c1.pad + u, gx = x - c1.pad + v;
            const bool in = gy >= 0 && gy < P.H && gx >= 0 && gx < P.W;
            off[u][v] = in ? (unsigned)((sub * 4 * HW + gy * P.W + gx) * 4) : 0xfffffffcu;
        }
    const int rt0 = cs * NRT, lo1 = relu_bound(c1.relu);
    typename M::Acc acc[NRT][R];
    init_acc<MF, NRT, R>(acc, c2, rt0);
    const f32x4 *wp = c2.wp + min(rt0, c2.nrt - 1) * 64 + lane;
    for (int kg = 0; kg < c2.nkg; ++kg) {
        const int g = min(kg * M::GPS + sub, ((C + 3) >> 2) - 1);        // channel group of 4; the last one stands in for those past C
        float xv[4][R + 2][3];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int u = 0; u < R + 2; ++u)
#pragma unroll
                for (int v = 0; v < 3; ++v)
                    xv[j][u][v] = kg * M::KC + j < C ? __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xr, off[u][v], (kg * M::KC + j) * HW * 4, 0)) : 0.f;
        f32x4 w[9];
#pragma unroll
        for (int t = 0; t < 9; ++t) w[t] = c1.wp[g * 9 + t];
        const f32x4 scale = c1.aff[g * 2], shift = c1.aff[g * 2 + 1];
        f32x4 a[NRT];
#pragma unroll
        for (int r = 0; r < NRT; ++r) a[r] = wp[(size_t)(kg * c2.nrt + min(r, c2.nrt - 1 - min(rt0, c2.nrt - 1))) * 64];
        const int live = C - (kg * M::KC + sub * 4);        // channels of this lane that exist
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float d[R];
#pragma unroll
            for (int p = 0; p < R; ++p) {
                float s = 0.f;
#pragma unroll
                for (int u = 0; u < 3; ++u)
#pragma unroll
                    for (int v = 0; v < 3; ++v) s = fmaf(xv[j][p + u][v], w[u * 3 + v][j], s);
                s = relu_from(s * scale[j] + shift[j], lo1);
                d[p] = j < live ? s : 0.f;
            }
#pragma unroll
            for (int r = 0; r < NRT; ++r)
#pragma unroll
                for (int p = 0; p < R; ++p) acc[r][p] = M::mma(a[r][j], d[p], acc[r][p]);
        }
    }
    const int plane = P.Ho * P.Wo, lo2 = max(relu_bound(c2.relu), relu_bound(P.relu_out));
    const __amdgpu_buffer_rsrc_t yr = make_rsrc(P.y + ((size_t)n * P.Cy + P.coff2[0]) * plane,
                                                ((unsigned long long)(P.N - n) * P.Cy - P.coff2[0]) * plane * 4ull);
#pragma unroll
    for (int p = 0; p < R; ++p) {
        if (x >= P.Wo || y0 + p >= P.Ho) continue;
        const unsigned voff = (unsigned)(((y0 + p) * P.Wo + x + sub * 4 * plane) * 4);
#pragma unroll
        for (int r = 0; r < NRT; ++r) {
#pragma unroll
            for (int e = 0; e < M::NQ * 4; ++e) {
                const int cu = (rt0 + r) * MF + M::quad_row(e >> 2, 0) + (e & 3);      // channel of lane half 0
                if (cu + sub * 4 < c2.cout)
                    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, relu_from(acc[r][p][e], lo2)), yr, voff, cu * plane * 4, 0);
            }
        }
    }
}

}  // namespace xl

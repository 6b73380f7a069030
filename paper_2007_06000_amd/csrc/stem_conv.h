// The stem of an image network on the bf16 matrix cores (included by kernels.hip): 3x3 convolution of 3 channels with stride 2, no
// padding -> 3x3 max pooling with stride 2, no padding (paper Fig. 3b).
//
// The layer is a reduction of 27 terms: bound by moving its input and output (88 MB at 224 x 224, batch 64, to 64 channels: 16 us)
// as long as the arithmetic is cheap, and on the vector ALU it is not (thin_conv.h: 73 us at the issue rate of multiply-adds with
// a scalar operand).  On operands in three bf16 parts (split_conv.h) the 27 terms and the shift fill two K steps of 16, so 32
// channels of 32 outputs are 12 operations of 33 cycles.  A wave works alone, without LDS:
//   - a lane stands for a pooled pixel; the 2x2 block of convolution outputs under it are four pixel tiles of the matrix
//     operations, so a lane has its block in registers, and what the pooling window needs of the block to the right it
//     takes from the next lane (31 of 32 pixels of a wave are its own) and of the block below from the next row: the
//     wave walks down the image and keeps one maximum per channel from row to row;
//   - the lane halves share a pixel and divide the reduction: half 0 takes filter rows (channel, u) 0 to 3, half 1 4 to 7, and row
//     8 goes into the spare slots (K slots below), so a lane loads five 16-byte pieces of the image per two convolution rows
//     and takes apart what it loads, nothing is shuffled between lanes but the fifth column of a piece;
//   - the filter, taken apart once, stays in registers, the shift in a K slot with the pixel value 1.
// K slots of step k and lane half h, filter row R = 4 h + 2 k:  R.0 R.1 (R+1).0 (R+1).1 R.2 (R+1).2 s s', where s s' are, for
// k = 0, row 8's taps 0 and 1 (h = 0) and 2 and nothing (h = 1), for k = 1 the shift and nothing (h = 0).  Where a slot has no filter
// value it is 0 and meets whatever lies there.
// Every value of a piece is taken apart once: the third column of a block is the first of its right tile too, and the fifth comes from the next lane
// in parts.
// What bounds it: some 600 vector instructions and 48 matrix operations per pooled row and wave, and the waits between them (5600 cycles a row and
// SIMD with two waves as with three).  Time per pass, on the vector ALU -> here with every K slot taken apart by itself -> here: to 64 channels at
// 224 x 224, batch 64: 67 -> 35.2 -> 33.6 us, batch 8: 16 -> 10.9 -> 10.1.  Before, to 96 at 150 x 200, batch 16: 29.5 -> 15.5; to 32 at 224 x 224,
// batch 50: 32 -> 21.
// 64 channels per wave were slower (46 us at batch 64, of 40 then: 248 registers, two waves per SIMD), a third of the filter in LDS equal.
// Where the chip is not filled the stream kernel stays ahead (to 64 channels at 224 x 224, xl_profile with its 2 to 3 us of events, batch 1:
// 8.6 us there, 9.5 here; batch 2: 9.5 and 9.6; batch 4: 12.3 and 10.0).
// A wave in which a value has no bf16 parts, or one is so large that a sum might overflow, takes fp32 matrix operations instead.
//
// BlockParams used: x, y, N, H, W, Ho, Wo, Cy, coff1, c1 (wp, aff: the tables of thin_conv_kernel; cout, relu), th (pooled rows of a
// wave), tiles_x, tiles_y, csplit (slices of 32 channels), nblocks.
#pragma once

namespace xl {

// the value of the next lane
__device__ __forceinline__ float next_lane(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x130, 0xf, 0xf, true));     // wave_shl:1
}

__device__ __forceinline__ unsigned next_lane(unsigned v)
{
    return __builtin_amdgcn_update_dpp(0, v, 0x130, 0xf, 0xf, true);
}

__global__ void __launch_bounds__(256, 3) stem_pool_kernel(const BlockParams P)
{
    touch_arguments();
    const int waves = P.N * P.csplit * P.tiles_y * P.tiles_x;
    const int L = logical_block() * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (L >= waves) return;         // (wave-uniform; nothing below waits for another wave)
    const int lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
    const int strips = P.tiles_y * P.tiles_x;
    // (the results of divisions are read through the first lane: the loads below take them as scalars)
    const int n = __builtin_amdgcn_readfirstlane(L / (strips * P.csplit)), in_image = L - n * (strips * P.csplit);
    const int cs = __builtin_amdgcn_readfirstlane(in_image / strips), strip = in_image - cs * strips;
    const int ty = __builtin_amdgcn_readfirstlane(strip / P.tiles_x), tx = strip - ty * P.tiles_x;
    const int px = tx * 31 + col, py0 = ty * P.th, py1 = min(py0 + P.th, P.Ho);
    const int H = P.H, W = P.W;

    // ---- the input: five pieces of 4 pixels per pair of convolution rows.  Pieces may run over the end of a row or of the
    // image: what they find there only reaches blocks without a pooled pixel (past the tensor the buffer ends: zeros).
    const __amdgpu_buffer_rsrc_t xr = make_rsrc(P.x + (size_t)n * 3 * H * W, (unsigned long long)(P.N - n) * 3 * H * W * 4ull);
    auto load = [&](f32x4 (&x)[5], int row) {           // row: first image row under the convolution row
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            auto piece = [&](int r) { return ((r * 11 >> 5) * H + (r - (r * 11 >> 5) * 3)) * W * 4; };      // row r of the filter
            int ln = lane;              // (an offset is worked out here: no registers for five of them)
            asm volatile("" : "+v"(ln));
            const int at = i < 4 ? (ln >= 32 ? piece(4 + i) : piece(i)) : piece(8) + (ln >= 32 ? 8 : 0);
            x[i] = __builtin_bit_cast(f32x4, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(xr, (unsigned)(at + (tx * 31 + (ln & 31)) * 16), row * W * 4, 0));
        }
    };
    f32x4 x[5];
    load(x, 4 * py0);

    // ---- the filter in parts
    const int rows16 = (P.c1.cout + 15) / 16 * 16;
    const __amdgpu_buffer_rsrc_t wr = make_rsrc(P.c1.wp, (unsigned long long)rows16 * thin_row_floats(27) * 4ull);
    const __amdgpu_buffer_rsrc_t sr = make_rsrc(P.c1.aff, (unsigned long long)rows16 * 4ull);
    // filter value of slot (k, e) for lane ln (rows past the table read as zeros)
    auto filter = [&](int ln, int k, int e) {
        const int oc = cs * 32 + (ln & 31), h = ln >> 5, R = h * 4 + k * 2;
        const int t = e < 2 ? R * 3 + e : e < 4 ? R * 3 + 3 + e - 2 : e < 6 ? R * 3 + 2 + (e - 4) * 3 : 24 + h * 2 + e - 6;
        if (k == 1 && e >= 6) return e == 6 && h == 0 ? __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(sr, oc * 4, 0, 0)) : 0.f;
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wr, (oc * thin_row_floats(27) + t) * 4, 0, 0));
    };
    constexpr float LARGE = 0x1p60f;        // 28 products of two such are below 2^125
    unsigned odd_filter = 0;
    float largest_filter = 0.f;
    u32x4 a[2][3];
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float f0 = filter(lane, k, 2 * j), f1 = filter(lane, k, 2 * j + 1);
            unsigned w[3];
            split_pair<2>(f0, f1, w, odd_filter);
            largest_filter = fmaxf(fmaxf(largest_filter, fabsf(f0)), fabsf(f1));
#pragma unroll
            for (int i = 0; i < 3; ++i) a[k][i][j] = w[i];
        }
    const bool whole_filter = __builtin_amdgcn_ballot_w64(odd_filter != 0u || largest_filter >= LARGE) != 0;

    const int oplane = P.Ho * P.Wo;
    const __amdgpu_buffer_rsrc_t yr = make_rsrc(P.y + ((size_t)n * P.Cy + P.coff1) * oplane,
                                                ((unsigned long long)P.Cy - P.coff1) * oplane * 4ull);       // (an image has less than 2^30 elements)
    const bool own = col < 31 && px < P.Wo;
    const int cout = P.c1.cout, Wo = P.Wo;
    int lo = relu_bound(P.c1.relu);
    asm volatile("" : "+s"(lo));

    // One convolution row of the blocks, `row` its first image row: the two tiles dx = 0, 1 from the pieces x, for which those of the image row
    // `next` are asked as soon as they are taken apart; use(dx, sums) takes the 16 sums of one.
    auto conv_row = [&](int row, bool more, int next, auto use) {
        float sum = 0.f;                // (NaN stays, and is not below LARGE)
#pragma unroll
        for (int i = 0; i < 5; ++i) sum += (fabsf(x[i][0]) + fabsf(x[i][1])) + (fabsf(x[i][2]) + fabsf(x[i][3]));
        // every value is taken apart once: the third column of a block is also the first of its right tile, and what a lane needs of the next
        // one's pieces comes in parts
        unsigned left = 0;
        unsigned front[5][3], back[5][3];       // columns 0, 1 and 2, 3 of the pieces
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            split_exact(x[i][0], x[i][1], front[i], left);
            split_exact(x[i][2], x[i][3], back[i], left);
        }
        const bool whole = whole_filter || __builtin_amdgcn_ballot_w64((left & 0xffffu) != 0u || !(sum < LARGE)) != 0;
        if (more) load(x, next);
#pragma unroll
        for (int dx = 0; dx < 2; ++dx) {
            u32x4 b[2][3];
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const int p = 2 * k, q = p + 1;
                    b[k][i][0] = dx ? back[p][i] : front[p][i];
                    b[k][i][1] = dx ? back[q][i] : front[q][i];
                    const unsigned third = dx ? __builtin_amdgcn_perm(front[q][i], front[p][i], 0x05040100u) : __builtin_amdgcn_perm(back[q][i], back[p][i], 0x05040100u);
                    b[k][i][2] = dx ? next_lane(third) : third;
                    b[k][i][3] = k == 0 ? (dx ? back[4][i] : front[4][i]) : i == 0 ? 0x3f80u : 0u;          // (1 for the shift)
                }
            __builtin_amdgcn_sched_barrier(0);
            f32x16 acc;
            zero_acc(acc);
            if (__builtin_expect(whole, 0)) {
                int ln = lane;          // (addresses are worked out here: no registers for them elsewhere)
                asm volatile("" : "+v"(ln));
                f32x4 z[5];
                load(z, row);
                // slot e of K step k
                auto slot = [&](int k, int e) {
                    const f32x4 &p = z[2 * k], &q = z[2 * k + 1];
                    if (e < 2) return p[2 * dx + e];
                    if (e < 4) return q[2 * dx + e - 2];
                    if (e == 4) return dx ? next_lane(p[0]) : p[2];
                    if (e == 5) return dx ? next_lane(q[0]) : q[2];
                    return z[4][2 * dx + e - 6];
                };
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        float v = 1.f;
                        if (!(k == 1 && e >= 6)) v = k == 0 && e == 7 && half == 1 ? 0.f : slot(k, e);
                        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(filter(ln, k, e), v, acc, 0, 0, 0);
                    }
                asm volatile("s_nop 15\n\ts_nop 3" : "+v"(acc));
            } else {
                // the small products of both K steps first, so that one accumulator loses none of their bits
#pragma unroll
                for (int large = 0; large < 2; ++large)
#pragma unroll
                    for (int k = 0; k < 2; ++k)
#pragma unroll
                        for (int i = 2; i >= 0; --i)
#pragma unroll
                            for (int j = 2 - i; j >= 0; --j)
                                if ((i + j == 0) == (large == 1))
                                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[k][j]), __builtin_bit_cast(bf16x8, b[k][i]), acc, 0, 0, 0);
                asm volatile("s_nop 15" : "+v"(acc));
            }
            use(dx, acc);
        }
    };

    // block: the left column of the block (first its top left sum); most: what is known of the window (of the row before,
    // until this row's top sums have joined it, then of this row)
    f32x16 block, most;
#pragma unroll 1
    for (int py = py0; py <= py1; ++py) {
        conv_row(4 * py, py < py1, 4 * py + 2, [&](int dx, const f32x16 &v) {
            if (dx == 0) {
                block = v;
                return;
            }
            if (py > py0) {
                // the row before is complete (lanes without a pixel of their own aim past the end of the image)
                const unsigned at = own ? (unsigned)(((py - 1) * Wo + px + half * 4 * oplane) * 4) : 0xfffffffcu;
                const int live = cout - cs * 32 - half * 4;          // channels from this lane's first one on
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int oc = (e >> 2) * 8 + (e & 3);
                    const float m = fmaxf(fmaxf(most[e], block[e]), fmaxf(v[e], next_lane(block[e])));
                    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, relu_from(m, lo)), yr, oc < live ? at : 0xfffffffcu, (cs * 32 + oc) * oplane * 4, 0);
                }
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) most[e] = fmaxf(block[e], v[e]);
        });
        if (py == py1) break;
        conv_row(4 * py + 2, true, 4 * py + 4, [&](int dx, const f32x16 &v) {
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                if (dx == 0) block[e] = fmaxf(block[e], v[e]);
                most[e] = fmaxf(most[e], v[e]);
                if (dx == 1) most[e] = fmaxf(most[e], next_lane(block[e]));
            }
        });
    }
}

}  // namespace xl

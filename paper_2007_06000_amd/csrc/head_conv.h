// Pointwise convolution -> global average pooling on bf16 parts (included by kernels.hip).
//
// The last layer of a classifier: every value of the input meets as many filter values as there are classes, and one number per image and class is kept.
// Layer by layer it wrote the product and read it again, and the workgroups of eight slices of output channels each took the whole input apart.  Here a
// workgroup has the image's pixels in front of it as fragments of the 16x16x32 bf16 operation (split_conv.h: three products of two parts or six of
// three), and the mean is taken from the accumulators.
//
// head_kernel: the waves of a workgroup take 16 * NRT channels each and all pixels (up to 16 * NPT; of larger images pw waves share the pixels).  The
// pixels of a K step of 32 channels are taken apart once per workgroup, tile by tile, by whichever wave's turn it is, and lie in LDS for all, in two
// buffers; one barrier per K step.  Half of the waves do this before their matrix operations and half in the middle of them, so that a SIMD always has a
// wave with matrix operations.  Filter rows of a wave are its own: they come to its place in LDS a K step ahead without passing registers, which the
// accumulators fill (2 x 11 tiles of two accumulators: 176 of 256).
// head_divided_kernel: where few workgroups are to be had (below).
//
// What bounds it: one K step of the 2 x 11 kernel takes 7000 cycles where its matrix operations take 4200, with four workgroups on the chip as with 256;
// by the counters a SIMD's matrix pipe works for 59 % of a launch and LDS reads (264 KB a step) meet no bank conflicts.  Two waits that stand in the
// source, neither of them timed by itself: the waves that stage first wait in stage() for the filter rows they have just asked for, though their pixels
// are there from the top of the step on; and the third part of a pixel is asked for 96 cycles of its own matrix work before it is due.
// 512 -> 1000 channels at 13 x 13, layer by layer -> here, three parts / two: batch 64 86.8 -> 50.4 / 54.5 -> 32.3 us, batch 8 20.6 -> 12.9 /
// 18.0 -> 9.8, batch 1 10.8 -> 9.7; at 7 x 7, batch 64: 25.2 -> 23.0; 300 -> 500 at 10 x 9, batch 16: 11.0 -> 8.0; 128 -> 100 at 14 x 14, batch 32:
// 8.0 -> 6.0.
#pragma once

namespace xl {

// The parts of 8 values as the pixel operand; what the third part does not hold is marked (split_conv.h).
template <int PR>
__device__ __forceinline__ void head_parts(const float (&x)[8], u32x4 (&b)[PR + 1])
{
    unsigned left = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        unsigned w[PR + 1];
        if constexpr (PR == 2) split_exact(x[2 * j], x[2 * j + 1], w, left);
        else split_pair<PR>(x[2 * j], x[2 * j + 1], w, left);
#pragma unroll
        for (int i = 0; i <= PR; ++i) b[i][j] = w[i];
    }
    if constexpr (PR == 2) {
        if (__builtin_expect((left & 0xffffu) != 0u, 0)) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                unsigned w[3];
                whole_parts(x[2 * j], x[2 * j + 1], w);
#pragma unroll
                for (int i = 0; i < 3; ++i) b[i][j] = w[i];
            }
        }
    }
}

template <int NRT, int NPT, int PR>
__device__ __forceinline__ void head_block()
{
    constexpr int NP = PR + 1, MAX_UNITS = HEAD_UNITS;
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const BlockParams &P = block_params();
    const int L = logical_block();
    if (L >= P.nblocks) return;
    const ConvW &c = P.c1;
    const int n = udiv(L, P.csplit, P.rcp_csplit), cs = L - n * P.csplit;
    const int lane = threadIdx.x & 63, sub = lane >> 4, col = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
    const int lr = __builtin_ctz(P.waves_r1), wr = wave & (P.waves_r1 - 1), wp = wave >> lr, pw = nw >> lr;
    const int npx = P.mh * P.mw, npt = (npx + 15) >> 4, nrt = c.nrt, nkg = c.nkg;
    const int per = (npt + pw - 1) >> __builtin_ctz(pw);            // pixel tiles of a wave: as many to each (11 and 2 of 13 lost more bits in the last sum than 7 and 6)
    const int rt0 = (cs * P.waves_r1 + wr) * NRT, pt0 = wp * per;
    const int live = rt0 < nrt ? min(per, npt - pt0) : 0;
    const int step = npx * 4;                                       // bytes from channel to channel

    float *a_lds = lds + wave * (NRT * NP * 256);                   // filter rows of a K step: every wave its own
    float *shift_lds = lds + nw * (NRT * NP * 256) + wave * (NRT * 256);
    float *b_lds = lds + nw * (NRT * (NP + 1) * 256);               // [buffer][pixel tile][part][lane]
    const int b_size = npt * (NP * 256);

    const __amdgpu_buffer_rsrc_t xr = make_rsrc(P.x + (size_t)n * P.Cin * npx, (unsigned long long)P.Cin * step);
    const __amdgpu_buffer_rsrc_t wsrc = make_rsrc(c.wp, (unsigned long long)nkg * nrt * (NP * 1024));
    const __amdgpu_buffer_rsrc_t ssrc = make_rsrc(c.aff, (unsigned long long)nrt * 1024);

    int w_at[NRT];              // byte offset of the row tiles in the K step requested next
#pragma unroll
    for (int r = 0; r < NRT; ++r) w_at[r] = min(rt0 + r, nrt - 1) * (NP * 1024);
    auto request_a = [&]() {
#pragma unroll
        for (int r = 0; r < NRT; ++r) {
#pragma unroll
            for (int i = 0; i < NP; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(wsrc, (__attribute__((address_space(3))) void *)(a_lds + (r * NP + i) * 256), 16, lane * 16, w_at[r] + i * 1024, 0, 0);
            w_at[r] += nrt * (NP * 1024);
        }
    };
    // units of a K step: 32 channels of one pixel tile, 8 per lane, wave after wave (the channel in the lane's offset: direct_conv.h)
    unsigned off[MAX_UNITS];
    float x[MAX_UNITS][8];
#pragma unroll
    for (int i = 0; i < MAX_UNITS; ++i) {
        const int px = (wave + i * nw) * 16 + col;
        off[i] = px < npx ? (unsigned)(px * 4 + sub * 8 * step) : 0x80000000u;
    }
    auto request_x = [&]() {
#pragma unroll
        for (int i = 0; i < MAX_UNITS; ++i) {
            if (wave + i * nw < npt) {
#pragma unroll
                for (int j = 0; j < 8; ++j) x[i][j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xr, off[i] + j * step, 0, 0));
            }
            off[i] += 32 * step;
        }
    };
    auto put_x = [&](float *dst) {
#pragma unroll
        for (int i = 0; i < MAX_UNITS; ++i) {
            if (wave + i * nw < npt) {
                u32x4 b[NP];
                head_parts<PR>(x[i], b);
#pragma unroll
                for (int q = 0; q < NP; ++q) *(u32x4 *)(dst + ((wave + i * nw) * NP + q) * 256 + lane * 4) = b[q];
            }
        }
    };

    f32x4 acc[NRT][NPT], low[PR == 2 ? NRT : 1][PR == 2 ? NPT : 1];
    request_a();
#pragma unroll
    for (int r = 0; r < NRT; ++r)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(ssrc, (__attribute__((address_space(3))) void *)(shift_lds + r * 256), 16, lane * 16, min(rt0 + r, nrt - 1) * 1024, 0, 0);
    request_x();
    __builtin_amdgcn_s_waitcnt(0);
    put_x(b_lds);
    request_x();
    // (sums begin with the shift: added behind them it is one rounding more)
#pragma unroll
    for (int r = 0; r < NRT; ++r) {
        const f32x4 shift = *(const f32x4 *)(shift_lds + r * 256 + lane * 4);
#pragma unroll
        for (int p = 0; p < NPT; ++p) {
            acc[r][p] = shift;
            if constexpr (PR == 2) zero_acc(low[r][p]);
        }
    }
    lds_barrier();

    const bool early = wave < nw / 2;
#pragma unroll 1
    for (int kg = 0; kg < nkg; ++kg) {
        const bool more = kg + 1 < nkg;
        __builtin_amdgcn_s_waitcnt(0x0f70);          // vmcnt(0): the filter rows (and pixels) asked for a K step ago
        __builtin_amdgcn_sched_barrier(0);
        f32x4 a[NRT][NP], b[NP];
#pragma unroll
        for (int r = 0; r < NRT; ++r)
#pragma unroll
            for (int i = 0; i < NP; ++i) a[r][i] = *(const f32x4 *)(a_lds + (r * NP + i) * 256 + lane * 4);
        const float *bs = b_lds + (kg & 1) * b_size + pt0 * (NP * 256) + lane * 4;
        auto fetch_b = [&](int p, int i) { b[i] = *(const f32x4 *)(bs + (p * NP + i) * 256); };
        // what the next step reads: pixels of it into the other buffer, its filter rows, the pixels of the step after it
        auto stage = [&]() {
            __builtin_amdgcn_s_waitcnt(0x0f70);
            put_x(b_lds + ((kg + 1) & 1) * b_size);
            request_x();
        };
        if (live > 0) {
#pragma unroll
            for (int i = NP - 1; i >= 0; --i) fetch_b(0, i);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        if (more) {
            request_a();
            if (early) stage();
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int p = 0; p < NPT; ++p) {
            if (p < live) {
#pragma unroll
                for (int i = NP - 1; i >= 0; --i) {
#pragma unroll
                    for (int j = NP - 1 - i; j >= 0; --j)
#pragma unroll
                        for (int r = 0; r < NRT; ++r) {
                            f32x4 &d = PR == 2 && i + j > 0 ? low[PR == 2 ? r : 0][PR == 2 ? p : 0] : acc[r][p];
                            d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[r][j]), __builtin_bit_cast(bf16x8, b[i]), d, 0, 0, 0);
                        }
                    if (p + 1 < NPT) {
                        fetch_b(p + 1 < live ? p + 1 : p, i);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
            if (p == NPT / 2 && more && !early) stage();
        }
        lds_barrier();
    }
    asm volatile("s_nop 15");
    float *red = b_lds;         // [pixel wave][channel]: no wave reads pixels any more
    const int rows_wg = P.waves_r1 * NRT * 16;
    if (live > 0) {
        bool again = false;
        const int lo = max(relu_bound(c.relu), relu_bound(P.relu_out));
        f32x4 s[NRT];
#pragma unroll
        for (int r = 0; r < NRT; ++r) {
#pragma unroll
            for (int p = 0; p < NPT; ++p) {
                asm volatile("" : "+v"(acc[r][p]));
                if constexpr (PR == 2) {
                    asm volatile("" : "+v"(low[r][p]));
                    acc[r][p] += low[r][p];
                }
                const bool valid = (p < live) & ((pt0 + p) * 16 + col < npx);
                float t = 0.f;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (PR == 2) t = fmaf(acc[r][p][e], 0.f, t);
                    acc[r][p][e] = valid ? relu_from(acc[r][p][e], lo) : 0.f;
                }
                again |= t != 0.f;
            }
            // (the tiles' sums meet in pairs: one after the other they lose more bits than a kernel that has four values to a lane)
#pragma unroll
            for (int m = 1; m < NPT; m <<= 1)
#pragma unroll
                for (int p = 0; p + m < NPT; p += 2 * m) acc[r][p] += acc[r][p + m];
            s[r] = acc[r][0];
        }
        if constexpr (PR == 2) {
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(again) != 0, 0)) {
#pragma unroll
                for (int r = 0; r < NRT; ++r) {
                    zero_acc(s[r]);
#pragma unroll 1
                    for (int p = 0; p < live; ++p) {
                        const int px = (pt0 + p) * 16 + col;
                        const unsigned at = px < npx ? (unsigned)(px * 4 + sub * 8 * step) : 0x80000000u;
                        const f32x4 v = direct_whole(c, min(rt0 + r, nrt - 1), [&](int kg, float (&xv)[8]) {
#pragma unroll
                            for (int j = 0; j < 8; ++j) xv[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xr, at + kg * 32 * step + j * step, 0, 0));
                        });
#pragma unroll
                        for (int e = 0; e < 4; ++e) s[r][e] += px < npx ? relu_from(v[e], lo) : 0.f;
                    }
                }
            }
        }
#pragma unroll
        for (int r = 0; r < NRT; ++r) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int m = 1; m < 16; m <<= 1) s[r][e] += __shfl_xor(s[r][e], m, 64);
            if (col == 0) *(f32x4 *)(red + wp * rows_wg + (wr * NRT + r) * 16 + sub * 4) = s[r];
        }
    }
    __syncthreads();
    const int npw = (npt + per - 1) / per;          // pixel waves with pixels
    for (int row = threadIdx.x; row < rows_wg; row += blockDim.x) {
        const int co = cs * rows_wg + row;
        if (co < c.cout) {
            float t = red[row];
            for (int w = 1; w < npw; ++w) t += red[w * rows_wg + row];
            P.y[(size_t)n * P.Cy + P.coff1 + co] = t / (float)npx;
        }
    }
}

// The same for launches with few workgroups: the waves of a workgroup divide the pixels, 64 to a wave, and the reduction, and all take the same NRT row
// tiles, so that the pixels are taken apart where they are multiplied (10000 of the 25000 cycles of a workgroup with 512 channels, 169 pixels and
// NRT = 2, which add up with the matrix operations').  A lane loads 8 channels of four neighbouring pixels, which are its columns of four pixel tiles
// (the mean asks for no order).  Partial sums meet in LDS: [row tile][pixel tile][K part][lane] float4.
template <int NRT, int PR>
__device__ __forceinline__ void head_divided_block()
{
    constexpr int NP = PR + 1;
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const BlockParams &P = block_params();
    const int L = logical_block();
    if (L >= P.nblocks) return;
    const ConvW &c = P.c1;
    const int n = udiv(L, P.csplit, P.rcp_csplit), cs = L - n * P.csplit;
    const int lane = threadIdx.x & 63, sub = lane >> 4, col = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
    const int lk = __builtin_ctz(P.waves_r1), wk = wave & (P.waves_r1 - 1), group = wave >> lk;
    const int npx = P.mh * P.mw, tiles = (nw >> lk) * 4, nrt = c.nrt, nkg = c.nkg;
    const int rt0 = cs * NRT, step = npx * 4;                       // bytes from channel to channel
    const int mine = (nkg - wk + P.waves_r1 - 1) >> lk;             // K steps wk, wk + K parts, ...
    const __amdgpu_buffer_rsrc_t xr = make_rsrc(P.x + (size_t)n * P.Cin * npx, (unsigned long long)P.Cin * step);
    const __amdgpu_buffer_rsrc_t wsrc = make_rsrc(c.wp, (unsigned long long)nkg * nrt * (NP * 1024));
    constexpr unsigned NOWHERE = 0x80000000u;

    const int px0 = group * 64 + col * 4;
    unsigned off = px0 < npx ? (unsigned)(px0 * 4 + (wk * 32 + sub * 8) * step) : NOWHERE;
    f32x4 x[8], a[NRT][NP];
    auto request_x = [&]() {
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = __builtin_bit_cast(f32x4, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(xr, off + j * step, 0, 0));
        off += (32 * step) << lk;
    };
    int w_at = min(wk, nkg - 1) * nrt * (NP * 1024);
    auto request_a = [&](int next) {            // (past the wave's last K step its rows once more: a scalar offset stays inside its buffer)
#pragma unroll
        for (int r = 0; r < NRT; ++r)
#pragma unroll
            for (int i = 0; i < NP; ++i)
                a[r][i] = __builtin_bit_cast(f32x4, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(wsrc, lane * 16, w_at + min(rt0 + r, nrt - 1) * (NP * 1024) + i * 1024, 0));
        w_at += next < mine ? (nrt * (NP * 1024)) << lk : 0;
    };
    request_x();
    request_a(1);
    const int r_sum = wave & (NRT - 1);         // the row tile whose sums the wave adds up
    f32x4 acc[NRT][4], low[NRT][4];
#pragma unroll
    for (int r = 0; r < NRT; ++r) {
        f32x4 shift;            // (the sums of the first part begin with it)
        zero_acc(shift);
        if (wk == 0) shift = c.aff[min(rt0 + r, nrt - 1) * 64 + lane];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            acc[r][t] = shift;
            zero_acc(low[r][t]);
        }
    }
#pragma unroll 1
    for (int k = 0; k < mine; ++k) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            u32x4 b[NP];
            const float px[8] = {x[0][t], x[1][t], x[2][t], x[3][t], x[4][t], x[5][t], x[6][t], x[7][t]};
            head_parts<PR>(px, b);
            if (t == 3) request_x();            // (past the last K step: zeros that nothing reads)
#pragma unroll
            for (int i = NP - 1; i >= 0; --i)
#pragma unroll
                for (int j = NP - 1 - i; j >= 0; --j)
#pragma unroll
                    for (int r = 0; r < NRT; ++r) {
                        f32x4 &d = PR == 2 && i + j > 0 ? low[r][t] : acc[r][t];
                        d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[r][j]), __builtin_bit_cast(bf16x8, b[i]), d, 0, 0, 0);
                    }
        }
        request_a(k + 2);
    }
    asm volatile("s_nop 15");
    float *part = lds, *red = lds + ((NRT * tiles) << lk) * 256;
#pragma unroll
    for (int r = 0; r < NRT; ++r)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            asm volatile("" : "+v"(acc[r][t]), "+v"(low[r][t]));
            if constexpr (PR == 2) acc[r][t] += low[r][t];
            *(f32x4 *)(part + ((((r * tiles + group * 4 + t) << lk) + wk) * 64 + lane) * 4) = acc[r][t];
        }
    lds_barrier();
    const int lo = max(relu_bound(c.relu), relu_bound(P.relu_out));
    f32x4 s;
    zero_acc(s);
    for (int p = wave / NRT; p < tiles; p += nw / NRT) {
        const int px = (p >> 2) * 64 + col * 4 + (p & 3);
        const float *from = part + (((r_sum * tiles + p) << lk) * 64 + lane) * 4;
        auto pair = [&](int k) { return *(const f32x4 *)(from + k * 256) + *(const f32x4 *)(from + k * 256 + 256); };
        f32x4 v = pair(0);
        if (lk > 1) v += pair(2);
        if (lk > 2) v += pair(4) + pair(6);
        if constexpr (PR == 2) {
            const float t = fmaf(v[0], 0.f, fmaf(v[1], 0.f, fmaf(v[2], 0.f, v[3] * 0.f)));
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(t != 0.f) != 0, 0)) {
                const unsigned at = px < npx ? (unsigned)(px * 4 + sub * 8 * step) : NOWHERE;
                v = direct_whole(c, min(rt0 + r_sum, nrt - 1), [&](int kg, float (&xv)[8]) {
#pragma unroll
                    for (int j = 0; j < 8; ++j) xv[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xr, at + kg * 32 * step + j * step, 0, 0));
                });
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] += px < npx ? relu_from(v[e], lo) : 0.f;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int m = 1; m < 16; m <<= 1) s[e] += __shfl_xor(s[e], m, 64);
    if (col == 0) *(f32x4 *)(red + wave * 16 + sub * 4) = s;
    lds_barrier();
    const int row = threadIdx.x, co = rt0 * 16 + row;
    if (row < NRT * 16 && co < c.cout) {
        // (in four sums: one after the other the waves' sums lost more bits than all that went before)
        float t[4] = {0.f, 0.f, 0.f, 0.f};
        for (int w = row >> 4; w < nw; w += 4 * NRT)
#pragma unroll
            for (int k = 0; k < 4; ++k) t[k] += w + k * NRT < nw ? red[(w + k * NRT) * 16 + (row & 15)] : 0.f;
        P.y[(size_t)n * P.Cy + P.coff1 + co] = ((t[0] + t[1]) + (t[2] + t[3])) / (float)npx;
    }
}

template <int NRT, int NPT, int PR>
__global__ void __launch_bounds__(MAX_THREADS, 2) head_kernel(const BlockParams args)
{
    touch_arguments();
    head_block<NRT, NPT, PR>();
}

template <int NRT, int PR>
__global__ void __launch_bounds__(head_threads(NRT, PR), head_threads(NRT, PR) / 256) head_divided_kernel(const BlockParams args)
{
    touch_arguments();
    head_divided_block<NRT, PR>();
}

}  // namespace xl

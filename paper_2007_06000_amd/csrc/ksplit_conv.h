// Fused convolutions on split-bf16 operands for launches with few workgroups (included by kernels.hip).
//
// A small batch leaves the chip idle: one image of 13 x 13 is 98 workgroups of the general kernel on 256 compute units, each a
// chain of input chunks, K steps, epilogue, K steps, epilogue, in which half of the waves have no tile of their own, and waves
// that share a row tile read the same filter rows at the 64 bytes per cycle of a compute unit's cache (fire module of 512 -> 64 ->
// {256, 256} channels: 7.8 us in layer 1, 6.0 in the 3x3 layer and 1.8 in the 1x1 layer of 16.3).  Here the waves of a workgroup
// divide the reduction: every wave takes all pixels and a part of the K steps, so it reads only its own part of the input and the
// filter, all of it requested within one or two trips to memory, and the partial sums meet in LDS:
//   layer 1, 1x1:  operands go from memory straight into registers, without LDS and barriers
//   layer 1, 3x3:  the whole input tile goes through LDS in one chunk
//   epilogue:      partial sums [wave][tile][quad][lane] float4; a wave adds up one (tile, quad) at a time, and activates,
//                  takes apart and writes it to the LDS tile of the intermediate, or adds the shortcut and stores it
//   layer 2:       as layer 1 from the LDS tile; its first filter rows are requested before layer 1's sums are added up
// The steps (K step, tap) of a wave are one counted loop for every filter size, a few hundred instructions.
//
// What bounds it: instructions and LDS around the matrix operations.  A wave that is almost alone on its SIMD issues one
// instruction per 5 to 7 cycles, so a quad of a tile costs it 0.7 us in an epilogue (eight partial sums of 1 KB each among that) and
// the loops run at 55 to 60 % of the operations' rate.  Time per pass, best of the other kernels -> here: fire module of 512 -> 64 ->
// {256, 256} channels at 13 x 13, batch 1: 16.9 -> 14.8 us, 256 -> 32 -> {128, 128} at 27 x 27 with its pooling: 15.2 -> 12.3;
// residual blocks of 50 channels at 20 x 20, batch 1: 14.8 -> 11.3, of 25 at 61 x 61, batch 2: 11.4 -> 9.9; 100 -> 20 -> 40 channels,
// 1x1 -> 5x5 at 20 x 20: 11.5 -> 9.3; the network at batch 1: 125.5 -> 113.5.  Where a launch fills the chip the general kernel is
// faster (96 -> 16 -> {64, 64} at 55 x 55, batch 16: 17.4 and 32 us), and with few K steps it is too (64 -> 16 -> {64, 64} at 55 x 55,
// batch 1: 7.3 and 10.5): the planner's estimate decides, and xl_tune times both.
//
// BlockParams used as in block_kernel, and: waves_r1 / pw1 (waves along row tiles and pixel tiles of layer 1; the others
// along K), waves_r2 / pw2, lds_buf_off (partial sums), w_off1 (input tile), tile2_off (tile to be pooled).
#pragma once

namespace xl {

// The sums of one tile again with fp32 matrix operations on whole operands (conv_whole of split_conv.h with the filter size
// as a number).
template <typename Pixels>
__device__ __forceinline__ void whole_tile(f32x16 &acc, const ConvW &c, int rt, Pixels pixels)
{
    const int lane = threadIdx.x & 63, taps = c.k * c.k;
#pragma unroll 1
    for (int kg = 0; kg < c.nkg; ++kg)
#pragma unroll 1
        for (int t = 0; t < taps; ++t) {
            uint4 w[3];
            float x[8];
#pragma unroll
            for (int i = 0; i < 3; ++i) w[i] = reinterpret_cast<const uint4 *>(c.wp)[(size_t)((kg * taps + t) * c.nrt + rt) * 192 + i * 64 + lane];
            pixels(kg, t / c.k, t % c.k, x);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(whole_value(w, e), x[e], acc, 0, 0, 0);
            asm volatile("s_nop 15\n\ts_nop 3" : "+v"(acc));        // a result may be read 18 wait states later, on the way out of the loops too
        }
}

// The part of a reduction that belongs to one wave: steps s0 .. s1 - 1 of nkg * taps, for NRT row tiles and NPT pixel tiles.
// Filter rows are requested PD steps ahead, and the first PD by open().
template <int NRT, int NPT, int PR>
struct KPart {
    static constexpr int NP = PR + 1, PD = NRT * NPT >= 4 ? 1 : 3, R = PD + 1;
    f32x4 a[R][NRT][NP];
    f32x16 acc[NRT][NPT], low[NRT][NPT];
    __amdgpu_buffer_rsrc_t wr;
    int w_next, w_step, s0, s1;

    __device__ __forceinline__ void fetch_a(int slot)
    {
        int w_lane = (threadIdx.x & 63) * 16;
        asm volatile("" : "+v"(w_lane));
        w_next = __builtin_amdgcn_readfirstlane(w_next);
#pragma unroll
        for (int r = 0; r < NRT; ++r)
#pragma unroll
            for (int i = 0; i < NP; ++i)
                a[slot][r][i] = __builtin_bit_cast(f32x4, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(wr, w_lane + (r * NP + i) * 1024, w_next, 0));
        w_next += w_step;
    }
    // share wk of 2^lkw of the steps of convolution c for row tiles from rt0 on (rows past the last one read what follows, or zeros)
    __device__ __forceinline__ void open(const ConvW &c, int rt0, int wk, int lkw)
    {
        const int steps = c.nkg * c.k * c.k;
        s0 = __builtin_amdgcn_readfirstlane(steps * wk >> lkw);
        s1 = __builtin_amdgcn_readfirstlane(steps * (wk + 1) >> lkw);
        wr = make_rsrc(c.wp, (unsigned long long)steps * c.nrt * (NP * 1024));
        w_step = c.nrt * (NP * 1024);
        w_next = __builtin_amdgcn_readfirstlane((s0 * c.nrt + rt0) * (NP * 1024));
#pragma unroll
        for (int i = 0; i < PD; ++i)
            if (s0 + i < s1) fetch_a(i);
    }
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int r = 0; r < NRT; ++r)
#pragma unroll
            for (int p = 0; p < NPT; ++p) {
                zero_acc(acc[r][p]);
                zero_acc(low[r][p]);
            }
    }
    __device__ __forceinline__ void mma(int slot, int j, const f32x4 (&b)[NPT][NP], int i)
    {
#pragma unroll
        for (int r = 0; r < NRT; ++r)
#pragma unroll
            for (int p = 0; p < NPT; ++p) {
                f32x16 &d = PR == 2 && i + j > 0 ? low[r][p] : acc[r][p];
                d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[slot][r][j]), __builtin_bit_cast(bf16x8, b[p][i]), d, 0, 0, 0);
            }
    }
    // Pixels in LDS, 16-byte planes [8-channel group][part][row][col] `gstride` floats apart; off: the lane's pixels, with the
    // planes of its lane half.
    __device__ __forceinline__ void run_lds(const float *src, const int (&off)[NPT], int ks, int src_w, int gstride)
    {
        clear();
        // s0 / taps and the rest / ks by multipliers (steps: planner)
        const int taps = ks * ks, kg = ks == 1 ? s0 : ks == 3 ? s0 * 7282 >> 16 : s0 * 2622 >> 16, t = s0 - kg * taps;
        int u = ks == 1 ? 0 : ks == 3 ? t * 11 >> 5 : t * 13 >> 6, v = t - u * ks;
        const int row_step = (src_w - ks) * 4, k_step = 2 * NP * gstride - ks * src_w * 4;
        int at = kg * (2 * NP) * gstride + (u * src_w + v) * 4;        // of the step whose pixels are read next
        f32x4 b[NPT][NP];
        auto fetch_b = [&](int i) {
#pragma unroll
            for (int p = 0; p < NPT; ++p) b[p][i] = *(const f32x4 *)(src + off[p] + (at + i * gstride));
        };
        auto next = [&](bool more) {        // (the last step is read once more, in place of one past the end)
            if (!more) return;
            const bool row = ++v == ks, step = row && u + 1 == ks;
            at += 4 + (row ? row_step : 0) + (step ? k_step : 0);
            v = row ? 0 : v;
            u = step ? 0 : u + (row ? 1 : 0);
        };
        if (s0 < s1) {
#pragma unroll
            for (int i = NP - 1; i >= 0; --i) fetch_b(i);
        }
#pragma unroll 1
        for (int s = s0; s < s1; s += R) {
#pragma unroll
            for (int q = 0; q < R; ++q) {
                if (s + q >= s1) continue;
                if (s + q + PD < s1) fetch_a((q + PD) % R);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = NP - 1; i >= 0; --i) {
#pragma unroll
                    for (int j = NP - 1 - i; j >= 0; --j) mma(q, j, b, i);
                    if (i == NP - 1) next(s + q + 1 < s1);
                    fetch_b(i);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    }
    // Pixels of a 1x1 layer from memory: load(kg, x) requests the 8 channels of every pixel tile.
    template <typename Load>
    __device__ __forceinline__ void run_memory(Load load)
    {
        clear();
        float x[R][NPT][8];
#pragma unroll
        for (int i = 0; i < PD; ++i)
            if (s0 + i < s1) load(s0 + i, x[i]);
#pragma unroll 1
        for (int s = s0; s < s1; s += R) {
#pragma unroll
            for (int q = 0; q < R; ++q) {
                if (s + q >= s1) continue;
                if (s + q + PD < s1) {
                    fetch_a((q + PD) % R);
                    load(s + q + PD, x[(q + PD) % R]);
                }
                f32x4 b[NPT][NP];
#pragma unroll
                for (int p = 0; p < NPT; ++p) {
                    unsigned w[4][NP];
                    bool odd = false;
#pragma unroll
                    for (int j = 0; j < 4; ++j) split_pair<PR>(x[q][p][2 * j], x[q][p][2 * j + 1], w[j], odd);
                    if constexpr (PR == 2) {
                        if (__builtin_expect(odd, 0)) {
#pragma unroll
                            for (int j = 0; j < 4; ++j) whole_parts(x[q][p][2 * j], x[q][p][2 * j + 1], w[j]);
                        }
                    }
#pragma unroll
                    for (int i = 0; i < NP; ++i) b[p][i] = __builtin_bit_cast(f32x4, u32x4{w[0][i], w[1][i], w[2][i], w[3][i]});
                }
#pragma unroll
                for (int i = NP - 1; i >= 0; --i)
#pragma unroll
                    for (int j = NP - 1 - i; j >= 0; --j) mma(q, j, b, i);
            }
        }
    }
    // this wave's partial sums -> LDS, [row tile][pixel tile][quad][K part][lane] float4; part: of the wave's first tile and K
    // part, `down` floats from one row tile to the next
    __device__ __forceinline__ void put(float *part, int down, int lkw)
    {
        asm volatile("s_nop 15" : "+v"(acc[0][0]));         // 12 wait states behind the last operation, however the loop ended
#pragma unroll
        for (int r = 0; r < NRT; ++r)
#pragma unroll
            for (int p = 0; p < NPT; ++p) {
                asm volatile("" : "+v"(acc[r][p]));
                if constexpr (PR == 2) asm volatile("" : "+v"(low[r][p]));
            }
#pragma unroll
        for (int r = 0; r < NRT; ++r)
#pragma unroll
            for (int p = 0; p < NPT; ++p)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    f32x4 s;
#pragma unroll
                    for (int i = 0; i < 4; ++i) s[i] = PR == 2 ? acc[r][p][q * 4 + i] + low[r][p][q * 4 + i] : acc[r][p][q * 4 + i];
                    *(f32x4 *)(part + r * down + ((p * 4 + q) << lkw) * 256 + (threadIdx.x & 63) * 4) = s;
                }
    }
};

// Numbers of the argument that a phase uses, loaded together: where each is loaded at its use, behind branches, a wave waits for
// every one of them (a tile of the epilogue took 1.5 us like that).
template <typename T>
__device__ __forceinline__ void keep(T &v) { asm volatile("" : "+s"(v)); }
template <typename... T>
__device__ __forceinline__ void loaded(T &...v) { (keep(v), ...); }

// K1 = 1: layer 1 is pointwise and reads memory; 3: of any filter size, from an LDS tile.  POOLED: KIND_FUSED2P.
// PR1, PR: of layer 1 (a pointwise one takes three parts in either precision, as the general kernels run it on fp32 operations)
// and of layer 2.
template <int K1, int NRT1, int NPT1, int NRT2, int NPT2, bool POOLED, int PR, int PR1>
__global__ void __launch_bounds__(MAX_THREADS, 2) ksplit_kernel(const BlockParams)
{
    constexpr int NP = PR + 1, NP1 = PR1 + 1;
    touch_arguments();
    const BlockParams &P = block_params();
    extern __shared__ __attribute__((aligned(16))) float lds[];
    int nblocks = P.nblocks, tiles_x = P.tiles_x, tiles_y = P.tiles_y, csplit = P.csplit, H = P.H, W = P.W, Cin = P.Cin, mh = P.mh, mw = P.mw;
    int stride1 = P.c1.stride, pad1 = P.c1.pad, s2 = P.s2, P2 = P.P2, th = P.th, tw = P.tw, rw1 = P.waves_r1, pw1 = P.pw1, mid_gstride = P.mid_gstride;
    int part_off = P.lds_buf_off, npp = P.pp, sy = POOLED ? P.pth * P.ps2 : th, sx = POOLED ? P.ptw * P.ps2 : tw;
    unsigned rcp_tcs = P.rcp_tcs, rcp_tiles = P.rcp_tiles, rcp_tiles_x = P.rcp_tiles_x, rcp_mw = P.rcp_mw;
    const float *x0 = P.x;
    loaded(nblocks, tiles_x, tiles_y, csplit, H, W, Cin, mh, mw, stride1, pad1, s2, P2, th, tw, rw1, pw1, mid_gstride, part_off, npp, sy, sx, rcp_tcs,
           rcp_tiles, rcp_tiles_x, rcp_mw, x0);
    const int L = logical_block();
    if (L >= nblocks) return;
    const int tiles = tiles_x * tiles_y;
    const int n = __builtin_amdgcn_readfirstlane(udiv(L, tiles * csplit, rcp_tcs));
    const int in_image = L - n * tiles * csplit;
    const int cs = __builtin_amdgcn_readfirstlane(udiv(in_image, tiles, rcp_tiles));
    const int tile = in_image - cs * tiles;
    const int ty = __builtin_amdgcn_readfirstlane(udiv(tile, tiles_x, rcp_tiles_x)), tx = tile - ty * tiles_x;
    const int oy0 = ty * sy - (POOLED ? npp : 0), ox0 = tx * sx - (POOLED ? npp : 0);
    const int my0 = oy0 * s2 - P2, mx0 = ox0 * s2 - P2;
    const int iy0 = my0 * stride1 - pad1, ix0 = mx0 * stride1 - pad1;
    const int lane = threadIdx.x & 63, sub = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
    const int HW = H * W;
    const float *ximg = x0 + (size_t)n * Cin * HW;
    const __amdgpu_buffer_rsrc_t xr = make_rsrc(ximg, (unsigned long long)Cin * HW * 4ull);       // (an image has less than 2^30 elements)
    float *mid = lds, *part = lds + part_off;
    const int npx1 = mh * mw;

    // row, pixel and K part of a wave (powers of two: their logarithms)
    struct Place { int r, p, k, lr, lp, lk; };
    auto place = [&](int rw, int pw) {
        const int lr = __builtin_ctz(rw), lp = __builtin_ctz(pw);
        return Place{wave & (rw - 1), (wave >> lr) & (pw - 1), wave >> (lr + lp), lr, lp, __builtin_ctz(nw) - lr - lp};
    };
    constexpr int LP1 = NPT1 == 2 ? 1 : 0, LP2 = NPT2 == 2 ? 1 : 0;
    // partial sums of row tile r, pixel tile p, quad q of a pass with 2^lp pixel tiles and 2^lk K parts
    auto part_of = [&](int r, int p, int q, int lp, int lk) { return part + ((((((r << lp) + p) << 2) + q) << lk) << 8); };
    // The shift and the partial sums of one quad.  The shift joins the first part and the parts meet in pairs, so that one of the eight
    // roundings is of the whole sum's size.  (One after the other with the shift last, half of them nearly were: over 60 blocks of up to
    // four images the error against 64 bits was 9 % larger, up to 1.13 instead of 1.01 times that of the general kernels on parts, in the mean
    // 0.68 instead of 0.63.)
    auto add_up = [&](const float *from, int lk, const f32x4 &shift) {
        from += lane * 4;
        auto sum = [&](auto count) {
            constexpr int N = decltype(count)::value;
            f32x4 t[N];
#pragma unroll
            for (int k = 0; k < N; ++k) t[k] = *(const f32x4 *)(from + k * 256);
            t[0] += shift;
#pragma unroll
            for (int d = 1; d < N; d *= 2)
#pragma unroll
                for (int k = 0; k < N; k += 2 * d) t[k] += t[k + d];
            return t[0];
        };
        return lk == 3 ? sum(std::integral_constant<int, 8>{}) : lk == 2 ? sum(std::integral_constant<int, 4>{})
             : lk == 1 ? sum(std::integral_constant<int, 2>{}) : sum(std::integral_constant<int, 1>{});
    };
    auto not_finite = [](const f32x4 &v) {
        const float t = fmaf(v[0], 0.f, fmaf(v[1], 0.f, fmaf(v[2], 0.f, v[3] * 0.f)));
        return __builtin_amdgcn_ballot_w64(t != 0.f) != 0;
    };
    auto quad_of = [](const f32x16 &a, int q) {
        f32x4 v;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = q == 0 ? a[i] : q == 1 ? a[4 + i] : q == 2 ? a[8 + i] : a[12 + i];
        return v;
    };
    // a wave adds up one quad of every (workgroup's waves / 4)-th tile
    const int q = wave & 3, t0 = wave >> 2, dt = nw >> 2;

    // ---- layer 1
    const Place w1 = place(rw1, pw1);
    // (what the epilogues add is requested before the filter rows: memory answers in order)
    int nrt1 = P.c1.nrt;
    const f32x4 *aff1 = P.c1.aff;
    loaded(nrt1, aff1);
    auto shift_of = [&](int t) { return aff1[(min(t >> (w1.lp + LP1), nrt1 - 1) * 4 + q) * 64 + lane]; };
    f32x4 shift1 = shift_of(t0);
    KPart<NRT1, NPT1, PR1> k1;
    k1.open(P.c1, w1.r * NRT1, w1.k, w1.lk);
    if constexpr (K1 == 1) {
        unsigned off[NPT1];
#pragma unroll
        for (int p = 0; p < NPT1; ++p) {
            // the pixel of the intermediate in the input, past the end outside the image
            const int pidx = (w1.p * NPT1 + p) * 32 + col;
            const int my = fdiv(pidx, rcp_mw), mx = pidx - my * mw;
            const int gy = iy0 + my * stride1, gx = ix0 + mx * stride1;
            off[p] = ((pidx < npx1) & ((unsigned)gy < (unsigned)H) & ((unsigned)gx < (unsigned)W)) ? (unsigned)((gy * W + gx + sub * 8 * HW) * 4) : 0xfffffffcu;
        }
        const int step = HW * 4, whole = Cin >> 4;
        k1.run_memory([&](int kg, float (&x)[NPT1][8]) {
            int at = kg * 16 * step;
            if (kg < whole) {
#pragma unroll
                for (int j = 0; j < 8; ++j, at += step)
#pragma unroll
                    for (int p = 0; p < NPT1; ++p) x[p][j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xr, off[p], at, 0));
            } else {
                const int live = Cin - kg * 16 - sub * 8;         // channels of this lane that exist
#pragma unroll
                for (int j = 0; j < 8; ++j, at += step)
#pragma unroll
                    for (int p = 0; p < NPT1; ++p) x[p][j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xr, j < live ? off[p] : 0xfffffffcu, at, 0));
            }
        });
    } else {
        // ---- the input tile in parts: a wave takes 64 pixels times 8 channels at a time, four of those in flight.  A unit's
        // buffer begins at its first channel and ends with the image: channels past the last one read as zeros.
        int in_off = P.w_off1, ih = P.ih, iw = P.iw, nkg1 = P.c1.nkg, k = P.c1.k;
        unsigned rcp_iw = P.rcp_qrow;
        loaded(in_off, ih, iw, nkg1, k, rcp_iw);
        float *in = lds + in_off;
        const int plane = ih * iw, groups = nkg1 * 2, units = groups * ((plane + 63) >> 6);
        constexpr int NU = 4;
        int u = wave, grp = wave, blk = 0;      // the unit requested next: 8-channel group, block of 64 pixels
        while (u < units) {
            float x[NU][8];
            int dst[NU];
#pragma unroll
            for (int i = 0; i < NU; ++i) {
                dst[i] = -1;
                if (u >= units) continue;
                while (grp >= groups) grp -= groups, ++blk;
                const int px = blk * 64 + lane, r = fdiv(px, rcp_iw), gy = iy0 + r, gx = ix0 + px - r * iw;
                if (px < plane) dst[i] = (grp * NP1 * plane + px) * 4;
                const bool inside = (px < plane) & ((unsigned)gy < (unsigned)H) & ((unsigned)gx < (unsigned)W);
                const unsigned off = inside ? (unsigned)((gy * W + gx) * 4) : 0xfffffffcu;
                const int ch = grp * 8;
                const __amdgpu_buffer_rsrc_t ur = make_rsrc(ximg + (size_t)min(ch, Cin) * HW, (unsigned long long)max(Cin - ch, 0) * HW * 4ull);
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    x[i][j] = ch + j < Cin ? __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(ur, off, j * HW * 4, 0)) : 0.f;
                u += nw;
                grp += nw;
            }
#pragma unroll
            for (int i = 0; i < NU; ++i) {
                if (dst[i] < 0) continue;
                unsigned w[4][NP1];
                bool odd = false;
#pragma unroll
                for (int j = 0; j < 4; ++j) split_pair<PR1>(x[i][2 * j], x[i][2 * j + 1], w[j], odd);
                if constexpr (PR1 == 2) {
                    if (__builtin_expect(odd, 0)) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) whole_parts(x[i][2 * j], x[i][2 * j + 1], w[j]);
                    }
                }
#pragma unroll
                for (int e = 0; e < NP1; ++e) *(uint4 *)(in + dst[i] + e * plane * 4) = uint4{w[0][e], w[1][e], w[2][e], w[3][e]};
            }
        }
        int off[NPT1];
#pragma unroll
        for (int p = 0; p < NPT1; ++p) {
            const int pidx = min((w1.p * NPT1 + p) * 32 + col, npx1 - 1);
            const int my = fdiv(pidx, rcp_mw), mx = pidx - my * mw;
            off[p] = (my * stride1 * iw + mx * stride1) * 4 + sub * NP1 * plane * 4;
        }
        lds_barrier();
        k1.run_lds(in, off, k, iw, plane * 4);
    }
    k1.put(part_of(w1.r * NRT1, w1.p * NPT1, 0, w1.lp + LP1, w1.lk) + (w1.k << 8), 4 << (w1.lp + LP1 + w1.lk + 8), w1.lk);

    // ---- layer 2: passes over (convolution, row tiles, pixel tiles)
    int rw2 = P.waves_r2, pw2 = P.pw2, convs = P.n2;
    unsigned rcp_csplit = P.rcp_csplit;
    loaded(rw2, pw2, convs, rcp_csplit);
    const Place w2 = place(rw2, pw2);
    const int npt2 = (th * tw + 31) >> 5, wg_rt2 = NRT2 << w2.lr, lp2 = w2.lp + LP2, wg_pt2 = 1 << lp2;
    KPart<NRT2, NPT2, PR> k2;
    // row tiles [first, end) of convolution c that belong to this workgroup
    struct Rows { int first, end; };
    auto rows_of = [&](int nrt) {
        const int per = __builtin_amdgcn_readfirstlane(udiv(nrt + csplit - 1, csplit, rcp_csplit));
        return Rows{cs * per, min(nrt, cs * per + per)};
    };
    auto open2 = [&](const ConvW &c, int rp) { k2.open(c, rp + w2.r * NRT2, w2.k, w2.lk); };
    {
        // (siblings of 5 and 8 row tiles in four slices: the last slice has none of the first sibling's)
        const BlockParams &P = block_params();
        const Rows rows0 = rows_of(P.c2[0].nrt);
        const ConvW &c = P.c2[rows0.first >= rows0.end && convs > 1 ? 1 : 0];
        open2(c, rows_of(c.nrt).first);
    }

    // ---- epilogue of layer 1: the LDS tile of the intermediate
    {
        const BlockParams &P = block_params();
        int nrt = nrt1, cout = P.c1.cout, lo = relu_bound(P.c1.relu), H1 = P.H1, W1 = P.W1;
        loaded(cout, lo, H1, W1);
        const int lp = w1.lp + LP1, tiles1 = (rw1 * NRT1) << lp;
        lds_barrier();
        for (int t = t0; t < tiles1; t += dt) {
            const f32x4 shift = shift1;
            shift1 = shift_of(t + dt);
            const int rt = t >> lp, pt = t & ((1 << lp) - 1);
            if (rt >= nrt || pt * 32 >= npx1) continue;
            f32x4 v = add_up(part_of(rt, pt, q, lp, w1.lk), w1.lk, shift);
            const int pidx = pt * 32 + col;
            const int my = fdiv(pidx, rcp_mw), mx = pidx - my * mw;
            if constexpr (PR1 == 2) {
                if (__builtin_expect(not_finite(v), 0)) {
                    f32x16 acc[1][1];
                    init_acc<32, 1, 1>(acc, P.c1, rt);
                    whole_tile(acc[0][0], P.c1, rt, [&](int kg, int uu, int vv, float (&x)[8]) {
                        const int gy = iy0 + my * stride1 + uu, gx = ix0 + mx * stride1 + vv, ch = kg * 16 + sub * 8;
                        const bool in = pidx < npx1 && gy >= 0 && gy < H && gx >= 0 && gx < W;
#pragma unroll
                        for (int e = 0; e < 8; ++e) x[e] = in && ch + e < Cin ? ximg[((ch + e) * H + gy) * W + gx] : 0.f;
                    });
                    v = quad_of(acc[0][0], q);
                }
            }
            const int cb = rt * 32 + q * 8 + sub * 4, gr = cb >> 2;
            const int live = (((unsigned)(my0 + my) < (unsigned)H1) & ((unsigned)(mx0 + mx) < (unsigned)W1)) ? cout - cb : 0;     // channels of the quad that hold a value
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float z = relu_from(v[i], lo);
                v[i] = i < live ? z : 0.f;
            }
            if (pidx < npx1) {
                float *dst = mid + (gr >> 1) * NP * mid_gstride + pidx * 4 + (gr & 1) * 2;
                bool odd = false;
                store_parts<PR>(v, dst, mid_gstride, odd);
                if constexpr (PR == 2) {
                    if (__builtin_expect(odd, 0)) store_whole_parts(v, dst, mid_gstride);
                }
            }
        }
    }
    lds_barrier();

#pragma unroll 1
    for (int ci = 0; ci < convs; ++ci) {
        const BlockParams &P = block_params();
        const ConvW &c = P.c2[ci];
        int nrt = c.nrt, k = c.k, cout = c.cout, lo1 = relu_bound(c.relu), lo2 = relu_bound(P.relu_out), d = P2 - c.pad, coff = P.coff2[ci];
        int Ho = P.Ho, Wo = P.Wo, Cy = P.Cy, H2 = P.H2, W2 = P.W2, tile2_off = P.tile2_off, Csc = P.Csc;
        unsigned rcp_tw = P.rcp_vw2;
        const f32x4 *aff = c.aff;
        float *y = P.y;
        const float *scp = P.sc;
        loaded(nrt, k, cout, lo1, lo2, d, coff, Ho, Wo, Cy, H2, W2, tile2_off, Csc, rcp_tw, aff, y, scp);
        const Rows rows = rows_of(nrt);
        const int plane = Ho * Wo;
        const bool shortcut = !POOLED && scp != nullptr;
        auto pixel_offset = [&](int pidx) {
            const int oyu = fdiv(pidx, rcp_tw);
            const int oy = min(oyu, th - 1), ox = min(pidx - oyu * tw, tw - 1);
            return ((oy * s2 + d) * mw + ox * s2 + d) * 4 + sub * NP * mid_gstride;
        };
        for (int rp = rows.first; rp < rows.end; rp += wg_rt2)
            for (int pp = 0; pp < npt2; pp += wg_pt2) {
                const __amdgpu_buffer_rsrc_t sr = make_rsrc(shortcut ? scp + (size_t)n * Csc * plane : x0, (unsigned long long)Csc * plane * 4ull);
                const __amdgpu_buffer_rsrc_t yr = make_rsrc(y + ((size_t)n * Cy + coff) * plane, ((unsigned long long)Cy - coff) * plane * 4ull);
                const int tiles2 = min(rows.end - rp, wg_rt2) << lp2;
                struct Out { int oy, ox, gy, gx, cb; bool pv; unsigned voff; };
                auto out_of = [&](int t) {
                    Out o;
                    const int pidx = (pp + (t & (wg_pt2 - 1))) * 32 + col;
                    o.oy = fdiv(pidx, rcp_tw);
                    o.ox = pidx - o.oy * tw;
                    o.gy = oy0 + o.oy;
                    o.gx = ox0 + o.ox;
                    o.cb = (rp + (t >> lp2)) * 32 + q * 8;          // channel of lane half 0
                    o.pv = (o.oy < th) & (o.ox < tw) & (POOLED | ((o.gy < Ho) & (o.gx < Wo)));
                    o.voff = (unsigned)((o.gy * Wo + o.gx + sub * 4 * plane) * 4);
                    return o;
                };
                // the shift and the shortcut of a tile are requested before the sums of the one before it are added up
                f32x4 shift = {0.f, 0.f, 0.f, 0.f}, sc = shift;
                auto request = [&](int t, const Out &o) {
                    if (t >= tiles2) return;
                    shift = aff[((rp + (t >> lp2)) * 4 + q) * 64 + lane];
                    if (!shortcut) return;
#pragma unroll
                    for (int i = 0; i < 4; ++i) sc[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(sr, (o.pv & (o.cb + i + sub * 4 < cout)) ? o.voff : 0xfffffffcu, (o.cb + i) * plane * 4, 0));
                };
                Out ahead = out_of(t0);
                request(t0, ahead);
                int off[NPT2];
#pragma unroll
                for (int p = 0; p < NPT2; ++p) off[p] = pixel_offset((pp + w2.p * NPT2 + p) * 32 + col);
                k2.run_lds(mid, off, k, mw, mid_gstride);
                k2.put(part_of(w2.r * NRT2, w2.p * NPT2, 0, lp2, w2.lk) + (w2.k << 8), 4 << (lp2 + w2.lk + 8), w2.lk);
                // the next pass's first filter rows
                const bool more = (pp + wg_pt2 < npt2) | (rp + wg_rt2 < rows.end);
                if (more || ci + 1 < convs) {
                    const ConvW &next = P.c2[more ? ci : ci + 1];
                    open2(next, more ? rp + (pp + wg_pt2 < npt2 ? 0 : wg_rt2) : rows_of(next.nrt).first);
                }
                float *tile2 = lds + tile2_off;
                const int npx2 = th * tw;
                lds_barrier();
                for (int t = t0; t < tiles2; t += dt) {
                    const Out o = ahead;
                    const f32x4 shift_now = shift, sc_now = sc;
                    ahead = out_of(t + dt);
                    request(t + dt, ahead);
                    const int rl = t >> lp2, pl = t & (wg_pt2 - 1), rt = rp + rl;
                    if (pp + pl >= npt2) continue;
                    f32x4 v = add_up(part_of(rl, pl, q, lp2, w2.lk), w2.lk, shift_now);
                    if constexpr (PR == 2) {
                        if (__builtin_expect(not_finite(v), 0)) {
                            f32x16 acc[1][1];
                            init_acc<32, 1, 1>(acc, c, rt);
                            const int at = pixel_offset((pp + pl) * 32 + col);
                            whole_tile(acc[0][0], c, rt, [&](int kg, int uu, int vv, float (&x)[8]) {
                                const float *from = mid + kg * 6 * mid_gstride + at + (uu * P.mw + vv) * 4;
                                const uint4 w[3] = {*(const uint4 *)from, *(const uint4 *)(from + mid_gstride), *(const uint4 *)(from + 2 * mid_gstride)};
#pragma unroll
                                for (int e = 0; e < 8; ++e) x[e] = whole_value(w, e);
                            });
                            v = quad_of(acc[0][0], q);
                        }
                    }
                    if constexpr (POOLED) {
                        // positions outside the layer's extent must not win a maximum
                        const bool inside = ((unsigned)o.gy < (unsigned)H2) & ((unsigned)o.gx < (unsigned)W2);
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] = inside ? relu_from(v[i], lo1) : -FLT_MAX;
                        if (o.pv) *(f32x4 *)(tile2 + ((rl * 8 + q * 2 + sub) * npx2 + o.oy * tw + o.ox) * 4) = v;
                    } else {
                        const bool whole = o.cb + 8 <= cout;          // (wave-uniform)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const float z = shortcut ? relu_from(relu_from(v[i], lo1) + sc_now[i], lo2) : relu_from(v[i], max(lo1, lo2));
                            if (o.pv & (whole | (o.cb + i + sub * 4 < cout)))
                                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, z), yr, o.voff, (o.cb + i) * plane * 4, 0);
                        }
                    }
                }
                lds_barrier();
                if constexpr (POOLED) {
                    // (one pixel pass covers the tile: planner; the next pass writes it behind a barrier of its own)
                    const BlockParams &P = block_params();
                    const int npo = P.pth * P.ptw, ngr = min(rows.end - rp, wg_rt2) * 8;
                    for (int it = threadIdx.x; it < ngr * npo; it += blockDim.x) {
                        const int gq = udiv(it, npo, P.rcp_npo), pidx = it - gq * npo;
                        const int py = fdiv(pidx, P.rcp_pw), px = pidx - py * P.ptw;
                        const int gy = ty * P.pth + py, gx = tx * P.ptw + px;
                        if (gy >= Ho || gx >= Wo) continue;
                        const float *sp = tile2 + (gq * npx2 + (py * P.ps2) * tw + px * P.ps2) * 4;
                        f32x4 m = {-FLT_MAX, -FLT_MAX, -FLT_MAX, -FLT_MAX};
                        if (P.pool_k == 3) {        // the usual window, unrolled: nine reads in flight together
                            f32x4 t[9];
#pragma unroll
                            for (int e = 0; e < 9; ++e) t[e] = *(const f32x4 *)(sp + (e / 3 * tw + e % 3) * 4);
#pragma unroll
                            for (int e = 0; e < 9; ++e)
#pragma unroll
                                for (int j = 0; j < 4; ++j) m[j] = fmaxf(m[j], t[e][j]);
                        } else {
                            for (int u = 0; u < P.pool_k; ++u)
                                for (int v = 0; v < P.pool_k; ++v) {
                                    const f32x4 t = *(const f32x4 *)(sp + (u * tw + v) * 4);
#pragma unroll
                                    for (int j = 0; j < 4; ++j) m[j] = fmaxf(m[j], t[j]);
                                }
                        }
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const int co = rp * 32 + gq * 4 + j;
                            if (co < cout) y[((size_t)n * Cy + coff + co) * plane + (size_t)gy * Wo + gx] = m[j];
                        }
                    }
                }
            }
    }
}

}  // namespace xl

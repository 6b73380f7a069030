// Pointwise first layers on three bf16 parts, operands from memory (included by kernels.hip).
//
// The first layer of a fire module is a pointwise reduction over many channels to a few: every input value meets 16 to 64 filter
// values.  Through LDS it is a chain of chunks (load, write, barrier, read), and on fp32 matrix operations in tiles of 16 pixels
// and one or two row tiles per wave it leaves waves idle; it took 30 to 45 % of the life of a workgroup of the fused fire kernels.  Here a
// wave takes 16 * NPT pixels and all row tiles: a lane loads 8 channels of its pixel, takes them apart in registers, where they are the
// pixel operand of the 16x16x32 bf16 operations as they are (split_conv.h: six products, the small ones in an accumulator of their own), and
// no value is loaded or taken apart twice.  Loads run DIRECT_AHEAD K steps of 32 channels ahead, across the pixel groups of a wave.  The filter
// lies in LDS, all of it or a chunk of K steps: every group of pixels reads all of it, and the vector cache returns 64 bytes per cycle where
// LDS returns 256.
//   waves_r1 = 1: waves take groups of 16 * NPT pixels in turn, each over all channels;
//   waves_r1 > 1: neighbouring waves divide the K steps of one group, for tiles with fewer groups than waves; partial sums meet in LDS,
//                 [row tile][pixel tile][K part][lane] float4, in the filter's place.
//
// What bounds it: where many workgroups start at once the input comes at 6 TB/s (a trip to memory of 2 us, then 3 to 8 us for 22 to 47 MB), and
// loads of 4 bytes a lane return 30 bytes per cycle and compute unit.  A second K step ahead is slower (fire module of 64 -> 16 -> {64, 64} at 55 x 55, batch
// 64: 49.8 us with three ahead, 45.9 with one: 32 registers and up to three empty steps behind every group), filter rows from
// memory instead of LDS too (51.9).  Layer 1 of 512 -> 64 at 13 x 13, batch 64, in the life of a workgroup: 17.5 -> 13.5 us.  Time per pass at batch 64,
// best of the other kernels -> here: 64 -> 16 -> {64, 64} at 55 x 55: 53.7 -> 46.0 us; 128 -> 32 -> {128, 128} at 27 x 27: 42.5 -> 36.7; 256 -> 32 ->
// {128, 128} at 27 x 27 with its pooling: 60.6 -> 52.7; at 13 x 13 256 -> 48 -> {192, 192}: 32.0 -> 28.5, 512 -> 64 -> {256, 256}: 49.7 -> 46.1; the network at batch
// 64: 494 -> 457.  Where a workgroup has few K steps and the launch one round, staging through LDS stays ahead (96 -> 16 -> {64, 64} at 55 x 55, batch 16:
// 20.3 us there, 21.3 here; 192 -> 16 -> 32, 1x1 -> 5x5 at 28 x 28, batch 32: 15.3 and 15.9, but 24.3 and 20.2 at batch 64), and with few workgroups the kernels that divide both
// layers (512 -> 64 -> {256, 256} at 13 x 13, batch 1: 16.4 and 18.5): the planner's estimate decides, and xl_tune times them all.
// (Over 138 blocks of 1 to 64 images the planner's first choice takes 0.945 times the time of its first one without these kernels, 0.967 on two parts in
// layer 2, and is behind it by 1 % at most, on two parts in three blocks by 1.5 to 4 %.)
#pragma once

namespace xl {

// The same sums of one 16x16 tile by fp32 matrix operations on whole values, as conv_whole does: pixels(kg, x) fetches the 8 values of
// the lane.
template <typename Pixels>
__device__ __forceinline__ f32x4 direct_whole(const ConvW &c, int rt, Pixels pixels)
{
    const int lane = threadIdx.x & 63;
    f32x4 acc = c.aff[rt * 64 + lane];
#pragma unroll 1
    for (int kg = 0; kg < c.nkg; ++kg) {
        uint4 w[3];
        float x[8];
#pragma unroll
        for (int i = 0; i < 3; ++i) w[i] = reinterpret_cast<const uint4 *>(c.wp)[(size_t)(kg * c.nrt + rt) * 192 + i * 64 + lane];
        pixels(kg, x);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(whole_value(w, e), x[e], acc, 0, 0, 0);
        asm volatile("s_nop 15" : "+v"(acc));        // a result may be read 10 wait states later, on the way out of the loop too
    }
    return acc;
}

template <int NRT, int NPT, int PR>
__device__ __forceinline__ void direct_stage1(const BlockParams &P, const ConvW &c, float *mid, float *buf, const float *ximg, int my0, int mx0,
                                              int iy0, int ix0)
{
    constexpr int XR = DIRECT_AHEAD + 1;        // K steps of pixels in registers or on their way
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
    const int lk = __builtin_ctz(P.waves_r1), wk = wave & (P.waves_r1 - 1), wp = wave >> lk, pw = nw >> lk;
    const int npx1 = P.mh * P.mw, npt = (npx1 + 15) >> 4, nrt = c.nrt, nkg = c.nkg, chunk = P.chunk_kg;
    const int step = P.H * P.W * 4;             // bytes from channel to channel

    // Pixel loads are never left out or made conditional: where they may or may not have been issued, the compiler's count of those in flight is
    // the smaller one, and a wait for old ones becomes a wait for new ones.  The buffer ends with the image, and what lies
    // behind it reads as zeros: channels past the last one too.  (An image and the K steps past its end have less than 2^31 bytes: planner.)
    // The channel is part of the lane's offset, which is what the bounds check is specified for: as a scalar offset it would pass the end of a buffer of
    // fewer than seven channels.  (Equally fast: the network's fires at batch 1, 8 and 64 within 1 %.)
    constexpr unsigned NOWHERE = 0x80000000u;
    const __amdgpu_buffer_rsrc_t xr = make_rsrc(ximg, (unsigned long long)P.Cin * step);
    const __amdgpu_buffer_rsrc_t wr = make_rsrc(c.wp, (unsigned long long)nkg * nrt * 3072);

    // byte offset of the lane's pixel of tile pt, with its 8 channels of a K step
    auto pixel_offset = [&](int pt, int ln) {
        const int pidx = pt * 16 + (ln & 15);
        const int my = fdiv(pidx, P.rcp_mw), mx = pidx - my * P.mw;
        const int gy = iy0 + my * c.stride, gx = ix0 + mx * c.stride;
        const bool in = (pidx < npx1) & ((unsigned)gy < (unsigned)P.H) & ((unsigned)gx < (unsigned)P.W);
        return in ? (unsigned)((gy * P.W + gx) * 4 + (ln >> 4) * 8 * step) : NOWHERE;
    };
    auto load8 = [&](unsigned off, float (&x)[8]) {
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xr, off + j * step, 0, 0));
    };
    // a tile by fp32 matrix operations, into the LDS tile
    auto put_whole = [&](int rt, int pt) {
        int ln = lane;          // (offsets are worked out here: no registers for them in the K loop)
        asm volatile("" : "+v"(ln));
        const unsigned off = pixel_offset(pt, ln);
        f32x4 v[1][1];
        v[0][0] = direct_whole(c, rt, [&](int kg, float (&x)[8]) { load8(off + kg * 32 * step, x); });
        store_mid<16, 1, 1, PR>(v, P, c, mid, my0, mx0, rt, nrt, pt, npx1, 0.f);
    };
    auto not_finite = [](const f32x4 &v) {
        const float t = fmaf(v[0], 0.f, fmaf(v[1], 0.f, fmaf(v[2], 0.f, v[3] * 0.f)));
        return __builtin_amdgcn_ballot_w64(t != 0.f) != 0;
    };

    // K steps wk, wk + K parts, ... of the reduction, XR of them per turn of the loop; the filter rows of `chunk` steps of all waves lie in LDS
    const int turns = __builtin_amdgcn_readfirstlane(((chunk + (1 << lk) - 1) >> lk) + XR - 1) / XR, chunks = (nkg + chunk - 1) / chunk;
    float x[XR][NPT][8];
    unsigned off[NPT];              // of the K step requested next
    auto fetch_x = [&](int slot) {
#pragma unroll
        for (int p = 0; p < NPT; ++p) {
            load8(off[p], x[slot][p]);
            off[p] += (32 * step) << lk;
        }
    };
    f32x4 acc[NRT][NPT], low[NRT][NPT];
    // the shifts lie in LDS behind the filter: behind the K loop a wave would wait for memory, and before it there are no registers for them
    const float *shift_lds = buf + P.chunk_kg * nrt * 768;
    auto shift = [&](int r) { return *(const f32x4 *)(shift_lds + (r * 64 + lane) * 4); };
    unsigned left = 0;              // bits that the parts do not hold
    const int first = wp * NPT;
    for (int ch = 0; ch < chunks; ++ch) {
        // the chunk's filter rows, from memory into LDS as they lie
        if (ch > 0) lds_barrier();
        const int rows = min(chunk, nkg - ch * chunk) * nrt * 3;
        for (int r = wave; r < rows; r += nw)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, (__attribute__((address_space(3))) void *)(buf + r * 256), 16, lane * 16, (ch * chunk * nrt * 3 + r) * 1024, 0, 0);
        if (ch == 0 && wave < nrt)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(make_rsrc(c.aff, (unsigned long long)nrt * 1024), (__attribute__((address_space(3))) void *)(buf + (chunk * nrt * 3 + wave) * 256), 16,
                                                     lane * 16, wave * 1024, 0, 0);
        if (ch == 0 && first < npt) {
#pragma unroll
            for (int p = 0; p < NPT; ++p) off[p] = pixel_offset(first + p, lane) + wk * 32 * step;
#pragma unroll
            for (int i = 0; i < XR - 1; ++i) fetch_x(i);
        }
        __builtin_amdgcn_s_waitcnt(0);
        lds_barrier();
        const float *a_lds = buf + (wk * nrt * 192 + lane) * 4;
        const int a_step = (nrt << lk) * 768, mine = (min(chunk, nkg - ch * chunk) - wk + (1 << lk) - 1) >> lk;       // K steps of the wave in the chunk
        // (the reduction of a group that shares a wave with others is one chunk: planner)
#pragma unroll 1
        for (int pt = first; pt < npt; pt += pw * NPT) {
            const bool more = lk == 0 && pt + pw * NPT < npt;       // (divided reductions: one group)
            if (ch == 0) {
#pragma unroll
                for (int r = 0; r < NRT; ++r)
#pragma unroll
                    for (int p = 0; p < NPT; ++p) {
                        zero_acc(acc[r][p]);
                        zero_acc(low[r][p]);
                    }
            }
            f32x4 a[2][3];
            int a_at = 0;
            auto fetch_a = [&](int slot, int r) {
                asm volatile("" : "+v"(a_at));
#pragma unroll
                for (int i = 0; i < 3; ++i) a[slot][i] = *(const f32x4 *)(a_lds + a_at + (r * 3 + i) * 256);
            };
            fetch_a(0, 0);
#pragma unroll 1
            for (int t = 0; t < turns; ++t) {
                const bool last = ch + 1 == chunks && t + 1 == turns;
#pragma unroll
                for (int u = 0; u < XR; ++u) {
                    // pixels XR - 1 steps on: of this group or of the next
                    if (u == 1 && last) {
#pragma unroll
                        for (int p = 0; p < NPT; ++p) off[p] = more ? pixel_offset(pt + pw * NPT + p, lane) : NOWHERE;
                    }
                    fetch_x((u + XR - 1) % XR);
                    const bool live = t * XR + u < mine;
                    u32x4 b[NPT][3];
                    if (live) {
#pragma unroll
                        for (int p = 0; p < NPT; ++p)
#pragma unroll
                            for (int j = 0; j < 4; ++j) {
                                unsigned w[3];
                                split_exact(x[u][p][2 * j], x[u][p][2 * j + 1], w, left);
#pragma unroll
                                for (int i = 0; i < 3; ++i) b[p][i][j] = w[i];
                            }
                    }
#pragma unroll
                    for (int r = 0; r < NRT; ++r) {
                        const int slot = (u * NRT + r) & 1;
                        if (r + 1 == NRT) a_at += t * XR + u + 1 < mine ? a_step : 0;       // (the last row is read once more, in place of one past the end)
                        fetch_a(slot ^ 1, (r + 1) % NRT);
                        if (live && (r == 0 || r < nrt)) {
#pragma unroll
                            for (int i = 2; i >= 0; --i)
#pragma unroll
                                for (int j = 2 - i; j >= 0; --j)
#pragma unroll
                                    for (int p = 0; p < NPT; ++p) {
                                        f32x4 &d = i + j > 0 ? low[r][p] : acc[r][p];
                                        d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[slot][j]), __builtin_bit_cast(bf16x8, b[p][i]), d, 0, 0, 0);
                                    }
                        }
                    }
                }
            }
            if (ch + 1 < chunks) break;
            // (results are asked for here; 8 wait states behind the last operation, however the loop ended)
            asm volatile("s_nop 15");
#pragma unroll
            for (int r = 0; r < NRT; ++r)
#pragma unroll
                for (int p = 0; p < NPT; ++p) {
                    asm volatile("" : "+v"(acc[r][p]), "+v"(low[r][p]));
                    acc[r][p] += low[r][p];
                }
            if (lk == 0) {
                bool again = __builtin_amdgcn_ballot_w64((left & 0xffffu) != 0u) != 0;
#pragma unroll
                for (int r = 0; r < NRT; ++r) {
                    if (r >= nrt) continue;
#pragma unroll
                    for (int p = 0; p < NPT; ++p) {
                        acc[r][p] += shift(r);
                        again |= not_finite(acc[r][p]);
                    }
                }
                if (__builtin_expect(again, 0)) {
#pragma unroll 1
                    for (int t = 0; t < nrt * NPT; ++t) put_whole(t / NPT, pt + t % NPT);
                } else {
                    store_mid<16, NRT, NPT, PR>(acc, P, c, mid, my0, mx0, 0, nrt, pt, npx1, 0.f);
                }
                left = 0;
            }
        }
    }
    if (lk == 0) return;
    // divided reductions: the partial sums take the filter's place
    const bool odd = __builtin_amdgcn_ballot_w64((left & 0xffffu) != 0u) != 0;
    float *part = buf;
    if (wk == 0) {
#pragma unroll
        for (int r = 0; r < NRT; ++r)
#pragma unroll
            for (int p = 0; p < NPT; ++p)
                if (r < nrt) acc[r][p] += shift(r);
    }
    lds_barrier();
#pragma unroll
    for (int r = 0; r < NRT; ++r)
#pragma unroll
        for (int p = 0; p < NPT; ++p)
            if (r < nrt && first + p < npt) *(f32x4 *)(part + ((((r * npt + first + p) << lk) + wk) * 64 + lane) * 4) = odd ? f32x4{NAN, NAN, NAN, NAN} : acc[r][p];
    lds_barrier();
    // (the shift is in the first part; the parts meet in pairs: ksplit_conv.h)
    auto sum_of = [&](int t) {
        const float *from = part + ((t << lk) * 64 + lane) * 4;
        auto pair = [&](int k) { return *(const f32x4 *)(from + k * 256) + *(const f32x4 *)(from + k * 256 + 256); };
        f32x4 v = pair(0);
        if (lk > 1) v += pair(2);
        if (lk > 2) v += pair(4) + pair(6);
        return v;
    };
    const int tiles = nrt * npt;
    f32x4 v[1][1], ahead = {0.f, 0.f, 0.f, 0.f};
    if (wave < tiles) ahead = sum_of(wave);
    for (int t = wave; t < tiles; t += nw) {
        const int rt = t / npt, pt = t - rt * npt;
        v[0][0] = ahead;
        if (t + nw < tiles) ahead = sum_of(t + nw);
        if (__builtin_expect(not_finite(v[0][0]), 0)) put_whole(rt, pt);
        else store_mid<16, 1, 1, PR>(v, P, c, mid, my0, mx0, rt, nrt, pt, npx1, 0.f);
    }
}

}  // namespace xl

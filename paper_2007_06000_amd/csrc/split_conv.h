// Convolutions on split-bf16 operands (included by kernels.hip).
//
// A float is held as PR + 1 bf16 parts, each the rounding of what the parts before it leave:
//   PR = 1: x ~ hi + lo (16 bits), a product is hi*hi + hi*lo + lo*hi: at most 3 * 2^-16 of |a||b| is left out;
//   PR = 2: x = hi + mid + lo, all 24 bits of a float, exactly.  A product is six of the nine part products; mid*lo, lo*mid
//           and lo*lo, at most 2^-23 and typically 2^-27 of |a||b| together, are left out.
// bf16 products are exact in the fp32 accumulators, so what remains is the rounding of the sums, and there PR = 2
// keeps TWO accumulators per tile: hi*hi in one, the five small products, which would lose their last bits against
// the large sum, in the other; they are added once at the end.  Error against 64 bits (relative 2-norm, reductions of
// 64 / 576 / 4608 non-negative x signed normal terms): fp32 matrix operations 1.0e-7 / 3.0e-7 / 8.8e-7, six products in
// one accumulator 1.1e-7 / 3.5e-7 / 1.0e-6, in two 4.0e-8 / 1.0e-7 / 3.5e-7 -- so the second accumulator is what makes
// PR = 2 a replacement for the fp32 operations.  Six 32x32x16 bf16 operations take 192 cycles for what takes the fp32
// 32x32x2 operation 8 x 64.
//
// What cannot be taken apart: infinities and NaN (inf - inf), values the first rounding takes to infinity (above
// 3.39e38), and values with bits below 2^-133, the smallest bf16 number (many of those below 2^-110 = 7.7e-34; the matrix
// operations themselves keep parts, products and sums below 2^-126).  In place of the parts of such a value stand a NaN and
// its upper and lower half (whole_parts), so that every sum it goes into is NaN.  A wave whose sums are not all finite
// after the K loop computes them again with fp32 matrix operations on the reassembled operands (conv_whole), as the fp32
// kernels do.  That also covers sums that overflow: hi*hi may round a product just below FLT_MAX up to infinity.  What a
// wave does depends on its own sums alone.
//
// The filter goes from memory to registers, one (K step, tap) or two ahead of the matrix operations, not
// through LDS: six operations on one 3 KB row of parts last 192 cycles per pixel tile, so a wave with two or more pixel
// tiles per row asks its vector cache for at most half of what it delivers; and a K loop that reads only pixels from LDS
// has no barriers, no filter buffers and no chunks.  The LDS tile of the intermediate then takes the place of the
// staging buffers of layer 1.
//
// What bounds it: power.  A K loop of this header alone keeps the matrix cores 86 to 90 % busy (36 to 37 cycles per
// operation and SIMD where 32 are nominal), but with real operands the clock falls to 1.65 - 1.75 GHz: 1.55 PFLOP/s in
// bf16, 258 TFLOP/s of fp32-exact products against 155 of the fp32 operations.  Time per pass, fp32 kernels -> PR = 2: the
// residual block of 64 channels at 56 x 56, batch 32: 158.6 -> 94 to 99 us from card to card; two 1x1 producers 64 -> 256 and
// their consumer, batch 32: 179 -> 124 us; 1x1 into 5x5, 28 x 28, batch 32: 17.6 -> 13.5 us; the batch-64 network: 688 -> 552 us.
#pragma once

namespace xl {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((vector_size(16)));     // what the 128-bit buffer load returns

__device__ __forceinline__ float bf16_low(unsigned w) { return __builtin_bit_cast(float, w << 16); }
__device__ __forceinline__ float bf16_high(unsigned w) { return __builtin_bit_cast(float, w & 0xffff0000u); }

// The parts of two floats, packed (first float in the low half of each word).  `odd` is raised (is not 0) when one of the two
// does not come apart (PR = 2).
template <int PR>
__device__ __forceinline__ void split_pair(float a, float b, unsigned (&w)[PR + 1], unsigned &odd)
{
#pragma unroll
    for (int i = 0; i <= PR; ++i) {
        w[i] = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{a, b}, bf16x2));
        if (i < PR || PR == 2) {
            a -= bf16_low(w[i]);
            b -= bf16_high(w[i]);
        }
    }
    // what is left is 0, except where a part was infinite or NaN (NaN) or bits lie below the smallest bf16 number
    if constexpr (PR == 2) odd |= __builtin_bit_cast(unsigned, a) | __builtin_bit_cast(unsigned, b);
}
template <int PR>
__device__ __forceinline__ void split_pair(float a, float b, unsigned (&w)[PR + 1], bool &odd)
{
    unsigned left = 0;
    split_pair<PR>(a, b, w, left);
    if constexpr (PR == 2) odd |= left != 0u;
}

// The three parts of two values for sums that are looked at afterwards and computed again from the values themselves: nothing is marked.
// `left` collects, in its lower 16 bits, what the parts do not hold (bits below the smallest bf16 number); parts of values that are infinite, NaN or too large are
// infinite or NaN, and so are their sums.  What is left for the third part has 8 bits: it is cut off, not rounded.
__device__ __forceinline__ void split_exact(float a, float b, unsigned (&w)[3], unsigned &left)
{
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(w[i]) : "v"(a), "v"(b));      // (a vector of the two costs a move)
        a -= bf16_low(w[i]);
        b -= bf16_high(w[i]);
    }
    const unsigned x = __builtin_bit_cast(unsigned, a), y = __builtin_bit_cast(unsigned, b);
    w[2] = __builtin_amdgcn_perm(y, x, 0x07060302u);
    left |= x | y;
}

// What is held in place of the parts of two values of which one does not come apart (PR = 2).
constexpr unsigned WHOLE_MARK = 0x7fc0u;        // no part of a value that comes apart is NaN
__device__ __forceinline__ void whole_parts(float a, float b, unsigned (&w)[3])
{
    const unsigned x = __builtin_bit_cast(unsigned, a), y = __builtin_bit_cast(unsigned, b);
    w[0] = WHOLE_MARK | WHOLE_MARK << 16;
    w[1] = x >> 16 | (y & 0xffff0000u);
    w[2] = (x & 0xffffu) | y << 16;
}

// The value of three parts, whichever way it is held; the parts of 8 values in 3 x 16 bytes (e: which value).
__device__ __forceinline__ float whole_value(unsigned hi, unsigned mid, unsigned lo)
{
    return hi == WHOLE_MARK ? __builtin_bit_cast(float, mid << 16 | lo) : bf16_low(hi) + (bf16_low(mid) + bf16_low(lo));
}
__device__ __forceinline__ float whole_value(const uint4 (&w)[3], int e)
{
    unsigned part[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const unsigned word = e < 2 ? w[i].x : e < 4 ? w[i].y : e < 6 ? w[i].z : w[i].w;
        part[i] = e & 1 ? word >> 16 : word & 0xffffu;
    }
    return whole_value(part[0], part[1], part[2]);
}

// The same for a value of PR + 1 parts (two parts hold every value as their sum).
template <int PR>
__device__ __forceinline__ float held_value(const uint4 (&w)[PR + 1], int e)
{
    if constexpr (PR == 2) return whole_value(w, e);
    const unsigned hi = e < 2 ? w[0].x : e < 4 ? w[0].y : e < 6 ? w[0].z : w[0].w, lo = e < 2 ? w[1].x : e < 4 ? w[1].y : e < 6 ? w[1].z : w[1].w;
    return e & 1 ? bf16_high(hi) + bf16_high(lo) : bf16_low(hi) + bf16_low(lo);
}

// Four consecutive channels of one pixel into the part planes: part p goes 8 bytes wide to dst + p * plane.
template <int PR>
__device__ __forceinline__ void store_parts(const f32x4 &v, float *dst, int plane, bool &odd)
{
    unsigned a[PR + 1], b[PR + 1];
    split_pair<PR>(v[0], v[1], a, odd);
    split_pair<PR>(v[2], v[3], b, odd);
#pragma unroll
    for (int i = 0; i <= PR; ++i) *(uint2 *)(dst + i * plane) = uint2{a[i], b[i]};
}
__device__ __forceinline__ void store_whole_parts(const f32x4 &v, float *dst, int plane)
{
    unsigned a[3], b[3];
    whole_parts(v[0], v[1], a);
    whole_parts(v[2], v[3], b);
#pragma unroll
    for (int i = 0; i < 3; ++i) *(uint2 *)(dst + i * plane) = uint2{a[i], b[i]};
}

// Workgroup barrier for data in LDS: waits for this wave's LDS operations only, so that loads of the next chunk and
// of the next filter rows stay in flight (__syncthreads would wait for nothing less than the compiler's fence asks).
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// ----------------------------------------------------------------------------
// K loop: acc (+ accl) [r][p] += filter (row tile rt0 + r) x pixels (pixel tile p), K steps kg0 .. kg0 + nkg - 1, for the
// first LIVE of the wave's pixel tiles.
// Pixels in LDS: 16-byte planes [8-channel group][part][row][col][8 bf16], `gstride` floats apart; `off` is the lane's
// pixel plus the planes of its lane half; `bsrc` starts at K step kg0.  Filter in memory:
// [K step][tap][row tile][part][lane] 16 bytes.  The operands of the next (K step, tap) steps are requested before the
// matrix operations of the current one: filter rows PD steps ahead, pixels one.  `hook` runs once the first filter
// rows have been requested: what it requests (the next input chunk) comes after them in the queue.  From K step `lower_at` on the wave has priority 0.
// ----------------------------------------------------------------------------
template <int KS, int NRT, int NPT, int PR, int LIVE, typename Hook>
__device__ __forceinline__ void conv_tiles(f32x16 (&acc)[NRT][NPT], f32x16 (&accl)[NRT][NPT], const float *bsrc,
                                           const int (&off)[NPT], int src_w, int gstride, const ConvW &c, int rt0,
                                           int kg0, int nkg, Hook hook, int lower_at)
{
    constexpr int T = KS * KS, NP = PR + 1, GROUPS = 2 * NP;     // planes per K step
    constexpr int PD = NRT >= 2 ? 1 : 2;                        // steps the filter rows are requested ahead
    constexpr int R = PD + 1;
    const __amdgpu_buffer_rsrc_t wr = make_rsrc(c.wp, (unsigned long long)c.nkg * T * c.nrt * (NP * 1024));
    // Addresses are kept as few running values that the compiler cannot see through: left to itself it keeps one
    // induction variable per tap and part in vector registers, 60 to 100 of them.
    int w_lane = (threadIdx.x & 63) * 16;
    const int w_step = c.nrt * (NP * 1024);
    int w_next = __builtin_amdgcn_readfirstlane((kg0 * T * c.nrt + rt0) * (NP * 1024));     // the step requested next
    int px[LIVE];                                                                          // the K step read next
#pragma unroll
    for (int p = 0; p < LIVE; ++p) px[p] = off[p];
    f32x4 a[R][NRT][NP], b[LIVE][NP];
    auto fetch_a = [&](int slot) {                  // one (K step, tap) after the other
        asm volatile("" : "+v"(w_lane), "+s"(w_next));
#pragma unroll
        for (int r = 0; r < NRT; ++r)
#pragma unroll
            for (int i = 0; i < NP; ++i)
                a[slot][r][i] = __builtin_bit_cast(f32x4, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(wr, w_lane + (r * NP + i) * 1024, w_next, 0));
        w_next += w_step;
    };
    auto fetch_b = [&](int i, int t) {              // part i of tap t of the K step that px stands at
        const float *s = bsrc + ((t / KS) * src_w + t % KS) * 4 + i * gstride;
#pragma unroll
        for (int p = 0; p < LIVE; ++p) {
            asm volatile("" : "+v"(px[p]));
            b[p][i] = *(const f32x4 *)(s + px[p]);
        }
    };
    auto next_px = [&](bool more) {                 // (the last K step is read once more, in place of one past the end)
#pragma unroll
        for (int p = 0; p < LIVE; ++p) px[p] += more ? GROUPS * gstride : 0;
    };
    // (results are asked for where they are due: matrix operations have no side effect that would keep them in place)
    auto pin = [&](f32x16 (&d)[NRT][NPT]) {
#pragma unroll
        for (int r = 0; r < NRT; ++r)
#pragma unroll
            for (int p = 0; p < LIVE; ++p) asm volatile("" : "+v"(d[r][p]));
    };
    auto mma = [&](int as, int ai, int bi, f32x16 (&d)[NRT][NPT]) {
#pragma unroll
        for (int r = 0; r < NRT; ++r)
#pragma unroll
            for (int p = 0; p < LIVE; ++p)
                d[r][p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[as][r][ai]), __builtin_bit_cast(bf16x8, b[p][bi]), d[r][p], 0, 0, 0);
    };
    // One (K step, tap): the filter rows PD steps on are requested, then part by part, the smallest first, the products
    // that need it and the request of the same part for the next tap `tn`, so that pixels need one register set.
    auto step = [&](int as, bool more_a, int slot, int tn) {
        if (more_a) fetch_a(slot);
        __builtin_amdgcn_sched_barrier(0);
        f32x16 (&low)[NRT][NPT] = PR == 2 ? accl : acc;
#pragma unroll
        for (int i = NP - 1; i >= 0; --i) {
#pragma unroll
            for (int j = NP - 1 - i; j >= 0; --j) mma(as, j, i, i + j == 0 ? acc : low);
            pin(low);
            if (i == 0) pin(acc);
            fetch_b(i, tn);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // A result of the matrix operations may be read 12 wait states after the last one.  An earlier form of this loop read an
    // accumulator too early where paths of different length met behind it, so they stand here; the matrix pipe is busy for
    // longer anyway.  As the kernels are now the compiler's own count holds on every path, with these states and without
    // them, behind conv_whole too (tests/test_matrix_operation_waits.py follows them in the built library).
    auto settle = [] { asm volatile("s_nop 15"); };
    const int nsteps = nkg * T;
#pragma unroll
    for (int i = 0; i < PD; ++i)
        if (i < nsteps) fetch_a(i);
    hook();
#pragma unroll
    for (int i = NP - 1; i >= 0; --i) fetch_b(i, 0);
    if constexpr (T == 1) {
#pragma unroll 1
        for (int kg = 0; kg < nkg; kg += R) {
#pragma unroll
            for (int u = 0; u < R; ++u)
                if (kg + u < nkg) {
                    next_px(kg + u + 1 < nkg);
                    step(u, kg + u + PD < nkg, (u + PD) % R, 0);
                    settle();
                }
        }
    } else {
#pragma unroll 1
        for (int kg = 0; kg < nkg; ++kg) {
            const bool last = kg + 1 >= nkg;
            if (kg == lower_at) __builtin_amdgcn_s_setprio(0);
#pragma unroll
            for (int t = 0; t < T; ++t) {
                if (t == T - 1) next_px(!last);
                step(t % R, t + PD < T || !last, (t + PD) % R, (t + 1) % T);
            }
            settle();
            // the next K step starts again from slot 0 of the ring
            if constexpr (T % R != 0) {
                f32x4 keep[PD][NRT][NP];
#pragma unroll
                for (int i = 0; i < PD; ++i)
#pragma unroll
                    for (int r = 0; r < NRT; ++r)
#pragma unroll
                        for (int q = 0; q < NP; ++q) keep[i][r][q] = a[(T + i) % R][r][q];
#pragma unroll
                for (int i = 0; i < PD; ++i)
#pragma unroll
                    for (int r = 0; r < NRT; ++r)
#pragma unroll
                        for (int q = 0; q < NP; ++q) a[i][r][q] = keep[i][r][q];
            }
        }
    }
}

// conv_tiles for a wave of which all or only the first pixel tile holds pixels (`live`, wave-uniform): work on a tile of
// padding costs as much power as any, and these kernels run at the power limit.
template <int KS, int NRT, int NPT, int PR, typename Hook>
__device__ __forceinline__ void conv_direct(f32x16 (&acc)[NRT][NPT], f32x16 (&accl)[NRT][NPT], const float *bsrc,
                                            const int (&off)[NPT], int src_w, int gstride, const ConvW &c, int rt0,
                                            int kg0, int nkg, int live, Hook hook, int lower_at = -1)
{
    if (NPT == 1 || live > 1) conv_tiles<KS, NRT, NPT, PR, NPT>(acc, accl, bsrc, off, src_w, gstride, c, rt0, kg0, nkg, hook, lower_at);
    else conv_tiles<KS, NRT, NPT, PR, 1>(acc, accl, bsrc, off, src_w, gstride, c, rt0, kg0, nkg, hook, lower_at);
}

// The same sums by fp32 matrix operations on whole operands, for a wave whose sums are not all finite: rare, so it is
// short, and it starts from the shift again.  Element e of a lane's 8 channels is K index `lane half` of the operation, for
// both operands alike; pixels(p, kg, t, x) fetches those of pixel tile p.  (Residual block of 64 channels at 56 x 56, batch
// 32, every value NaN: 371 us, 811 with the operands fetched element by element; 164 with the fp32 kernels.)
template <int KS, int NRT, int NPT, typename Pixels>
__device__ __forceinline__ void conv_whole(f32x16 (&acc)[NRT][NPT], const ConvW &c, int rt0, Pixels pixels)
{
    const int lane = threadIdx.x & 63;
#pragma unroll 1
    for (int kg = 0; kg < c.nkg; ++kg)
#pragma unroll 1
        for (int t = 0; t < KS * KS; ++t) {
            uint4 w[NRT][3];
            float x[NPT][8];
#pragma unroll
            for (int r = 0; r < NRT; ++r)
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    w[r][i] = reinterpret_cast<const uint4 *>(c.wp)[(size_t)((kg * KS * KS + t) * c.nrt + min(rt0 + r, c.nrt - 1)) * 192 + i * 64 + lane];
#pragma unroll
            for (int p = 0; p < NPT; ++p) pixels(p, kg, t, x[p]);
#pragma unroll
            for (int e = 0; e < 8; ++e)
#pragma unroll
                for (int r = 0; r < NRT; ++r) {
                    const float a = whole_value(w[r], e);
#pragma unroll
                    for (int p = 0; p < NPT; ++p) acc[r][p] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, x[p][e], acc[r][p], 0, 0, 0);
                }
        }
}

// Whether a sum of the wave is infinite or NaN.
template <int NRT, int NPT>
__device__ __forceinline__ bool any_not_finite(const f32x16 (&acc)[NRT][NPT])
{
    float t = 0.f;
#pragma unroll
    for (int r = 0; r < NRT; ++r)
#pragma unroll
        for (int p = 0; p < NPT; ++p)
#pragma unroll
            for (int i = 0; i < 16; ++i) t = fmaf(acc[r][p][i], 0.f, t);
    return __builtin_amdgcn_ballot_w64(t != 0.f) != 0;
}

// The two accumulators of a tile become one.
template <int NRT, int NPT>
__device__ __forceinline__ void add_small(f32x16 (&acc)[NRT][NPT], const f32x16 (&accl)[NRT][NPT])
{
#pragma unroll
    for (int r = 0; r < NRT; ++r)
#pragma unroll
        for (int p = 0; p < NPT; ++p)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[r][p][i] += accl[r][p][i];
}

// ----------------------------------------------------------------------------
// Layer 1 on split operands: the halo-extended input tile goes through LDS in chunks of `chunk_kg` K steps, taken
// apart on the way.  Two LDS buffers; the values of chunk i + 1 are in registers when chunk i begins and are written at
// its start, the loads of chunk i + 2 follow the first filter rows of chunk i; one barrier per chunk.
// A wave stages 64 consecutive pixels of the tile (row-major, no padding) times 8 channels: a lane loads its pixel's 8
// values, consecutive lanes consecutive pixels, and writes 16 bytes per part, consecutive lanes consecutive addresses.
// (Units of 4 channels x 4 pixels per lane load wider but write with a stride of 64 bytes: four bank groups of LDS for
// 64 lanes; 55 % of the LDS cycles of the residual block were conflicts.)  The buffer ends with the image, and lanes
// outside the image aim past it: zeros without a mask.
// ----------------------------------------------------------------------------
template <int KS, int NRT, int NPT, int PR, typename Init>
__device__ __forceinline__ void conv_pass_split(f32x16 (&acc)[NRT][NPT], const BlockParams &P, const ConvW &c, int rt0,
                                                int pt0, int live, const int (&off)[NPT], float *buf,
                                                const float *__restrict__ ximg, int iy0, int ix0, Init init)
{
    constexpr int NP = PR + 1, KC = 16;
    const int tid = threadIdx.x;
    const int HW = P.H * P.W;
    const int plane = P.ih * P.iws;                                // pixels of the tile, and of an LDS plane
    const int chunk = P.chunk_kg;
    constexpr int NU = SPLIT_STAGE_UNITS;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nwaves = blockDim.x >> 6;
    const int groups = chunk * 2, units = groups * ((plane + 63) >> 6);
    int xgrp[NU];                   // 8-channel group of the chunk (wave-uniform)
    unsigned xoff[NU];              // byte offset of the lane's pixel in its plane
    int xdst[NU];                   // float offset in the LDS chunk; -1: no pixel
#pragma unroll
    for (int i = 0; i < NU; ++i) {
        const int u = i * nwaves + wave;
        const int blk = u / groups;
        xgrp[i] = u < units ? u - blk * groups : -1;
        const int px = blk * 64 + (tid & 63);
        const int r = fdiv(px, P.rcp_qrow), gy = iy0 + r, gx = ix0 + px - r * P.iws;
        xdst[i] = px < plane ? (xgrp[i] * NP * plane + px) * 4 : -1;
        const bool in = px < plane && gy >= 0 && gy < P.H && gx >= 0 && gx < P.W;
        xoff[i] = in ? (unsigned)((gy * P.W + gx) * 4) : 0xfffffffcu;
    }
    float xst[NU][8];
    auto load_x = [&](int c0) {                     // chunk whose first channel is c0
#pragma unroll
        for (int i = 0; i < NU; ++i) {
            if (xgrp[i] < 0) continue;
            const int ch = c0 + xgrp[i] * 8, live = P.Cin - ch;     // channels that exist (wave-uniform)
            const __amdgpu_buffer_rsrc_t xr = make_rsrc(ximg + (size_t)ch * HW, live > 0 ? (unsigned long long)live * HW * 4ull : 0ull);
            if (live >= 8) {
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    xst[i][j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xr, xoff[i], j * HW * 4, 0));
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    xst[i][j] = j < live ? __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xr, xoff[i], j * HW * 4, 0)) : 0.f;
            }
        }
    };
    auto store_x = [&](float *dst) {
#pragma unroll
        for (int i = 0; i < NU; ++i) {
            if (xgrp[i] < 0 || xdst[i] < 0) continue;
            unsigned w[4][NP];
            bool odd = false;
#pragma unroll
            for (int j = 0; j < 4; ++j) split_pair<PR>(xst[i][2 * j], xst[i][2 * j + 1], w[j], odd);
            if constexpr (PR == 2) {
                if (__builtin_expect(odd, 0)) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) whole_parts(xst[i][2 * j], xst[i][2 * j + 1], w[j]);
                }
            }
#pragma unroll
            for (int q = 0; q < NP; ++q) *(uint4 *)(dst + xdst[i] + q * plane * 4) = uint4{w[0][q], w[1][q], w[2][q], w[3][q]};
        }
    };
    f32x16 accl[NRT][NPT];
#pragma unroll
    for (int r = 0; r < NRT; ++r)
#pragma unroll
        for (int p = 0; p < NPT; ++p) zero_acc(accl[r][p]);
    const int nchunks = (c.nkg + chunk - 1) / chunk;
    load_x(0);
    store_x(buf);
    if (nchunks > 1) load_x(chunk * KC);
    lds_barrier();
    for (int ch = 0; ch < nchunks; ++ch) {
        const int kg0 = ch * chunk;
        if (ch + 1 < nchunks) store_x(buf + ((ch + 1) & 1) * P.buf_stride);
        auto next = [&]() {
            if (ch + 2 < nchunks) load_x((kg0 + 2 * chunk) * KC);
        };
        if (live > 0)
            conv_direct<KS, NRT, NPT, PR>(acc, accl, buf + (ch & 1) * P.buf_stride, off, P.iws, P.in_gstride, c, rt0, kg0,
                                          min(chunk, c.nkg - kg0), live, next);
        else
            next();
        lds_barrier();
    }
    if constexpr (PR == 2) {
        add_small<NRT, NPT>(acc, accl);
        if (live > 0 && any_not_finite<NRT, NPT>(acc)) {
            init(acc);
            const int lane = tid & 63, sub = lane >> 5;
            conv_whole<KS, NRT, NPT>(acc, c, rt0, [&](int p, int kg, int t, float (&x)[8]) {
                const int pidx = min((pt0 + p) * 32 + (lane & 31), P.mh * P.mw - 1);
                const int my = fdiv(pidx, P.rcp_mw), mx = pidx - my * P.mw;
                const int gy = iy0 + my * c.stride + t / KS, gx = ix0 + mx * c.stride + t % KS, ch = kg * 16 + sub * 8;
                const bool in = gy >= 0 && gy < P.H && gx >= 0 && gx < P.W;
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] = in && ch + e < P.Cin ? ximg[((ch + e) * P.H + gy) * P.W + gx] : 0.f;
            });
        }
    }
}

}  // namespace xl

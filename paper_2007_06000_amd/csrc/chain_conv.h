// Pointwise -> pointwise convolutions on split-bf16 operands, without LDS for the intermediate (included by kernels.hip;
// paper Fig. 4c, Table 1 c.1: {1x1, 1x1} -> add -> 1x1, and the straight 1x1 -> 1x1).
//
// Both layers are matrix products over the same pixels, so a wave can take 32 pixels through both alone.  The accumulator of
// a 32x32 operation leaves a lane with 16 channels of its pixel, 8 per half of the row tile, and a lane of the next operation
// wants 8 channels of its pixel per K step: the same lanes, and the same channels once the filter rows of layer 1 are
// dealt to the accumulator rows in that order (row_channel).  So the intermediate goes from the accumulators through
// activation and splitting straight into the operands of layer 2, 32 channels at a time, and never leaves the
// registers; the input of the wave stays in registers in parts, read and taken apart once for both producers.
//
// The filters go through LDS, the rows of 32 intermediate channels at a time (two buffers, one barrier): four waves share
// them, so a compute unit asks its L2 for 1/4 of what waves on their own would (36 KB per 72 operations of 32 cycles and wave:
// 64 bytes per cycle, all that the path delivers).  Two workgroups per compute unit, so that vector instructions of one wave of
// a SIMD (taking apart, activation) run under the matrix operations of the other.
//
// What bounds it: the matrix cores, 60 % busy with two workgroups per compute unit (38 us of operations at the power limit for
// the block below), and the last round: 3136 waves of 32 pixels on 1024 SIMDs take four rounds instead of 3.06.  A wave alone on
// its SIMD takes 1.7 us per row tile, 1.0 of it operations; staging and barriers cost 5 % (measured without them).  Time per
// pass, before (three passes of the general kernel with the intermediate in LDS) -> here: {64 -> 256, 64 -> 256} -> 64 channels of
// 56 x 56, batch 32: 123 -> 59 us (layer 2 on two parts: 68 -> 55), batch 8: 40 -> 22; {20 -> 45, 20 -> 45} -> 19 of 44 x 49, batch 45: 28 ->
// 11; 20 -> 16 -> 16 of 50 x 50, batch 64: 17.5 -> 10.6; 64 -> 64 -> 64 of 56 x 56, batch 32: 27.8 -> 21.  Below about 100 waves the
// general kernel's smaller tiles are faster ({64 -> 256, 64 -> 256} -> 64 of one image: 17.1 and 18.9 us), so both stay.
#pragma once

namespace xl {

// Channel (inside a tile of 32) that accumulator row m holds, and source lane of the filter row of the layout
// [part][lane]: after this a lane's accumulator values 8 s .. 8 s + 7 are channels 16 s + 8 * (lane half) + 0 .. 7.
__device__ __forceinline__ int row_channel(int m) { return (m >> 4) * 16 + ((m >> 2) & 1) * 8 + ((m >> 3) & 1) * 4 + (m & 3); }

// What a wave of the kernel below needs for its pixels' input: channel c of the lane's pixel, 0 where there is none.
struct ChainInput {
    __amdgpu_buffer_rsrc_t rsrc;
    unsigned off;           // the lane's pixel, channel 8 * (lane half)
    int channels, plane;    // of the input; pixels per image
    __device__ __forceinline__ void load(float (&v)[8], int kg, int lane) const
    {
        const int live = channels - kg * 16 - (lane >> 5) * 8;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            v[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, j < live ? off : 0xfffffffcu, (kg * 16 + j) * plane * 4, 0));
    }
};

// The whole chain again with fp32 matrix operations on whole operands, for a wave that met a sum that is not finite
// (conv_whole of split_conv.h: values without bf16 parts, sums that overflow).  The intermediate stays in fp32.
template <int NRT2, int PR>
__device__ __forceinline__ void chain_whole(f32x16 (&acc2)[NRT2][1], const BlockParams &P, const ChainInput &in, int lane)
{
    const int from = (lane & 32) + row_channel(lane & 31);
    init_acc<32, NRT2, 1>(acc2, P.c2[0], 0);
#pragma unroll 1
    for (int rt = 0; rt < P.c1.nrt; ++rt) {
        f32x16 v;
        zero_acc(v);
#pragma unroll 1
        for (int p = 0; p < P.n1; ++p) {
            const ConvW &c = p ? P.c1b : P.c1;
            f32x16 acc;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 sh = c.aff[(rt * 4 + (q >> 1) * 2 + (lane >> 5)) * 64 + (q & 1) * 32];
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[q * 4 + i] = sh[i];
            }
#pragma unroll 1
            for (int kg = 0; kg < c.nkg; ++kg) {
                uint4 w[3];
#pragma unroll
                for (int i = 0; i < 3; ++i) w[i] = reinterpret_cast<const uint4 *>(c.wp)[(size_t)(kg * c.nrt + rt) * 192 + i * 64 + from];
                float x[8];
                in.load(x, kg, lane);
#pragma unroll
                for (int e = 0; e < 8; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(whole_value(w, e), x[e], acc, 0, 0, 0);
                asm volatile("s_nop 15\n\ts_nop 3" : "+v"(acc));      // a result may be read 18 wait states later, on the way out of the loop too
            }
            const int lo = relu_bound(c.relu), lo_sum = relu_bound(P.relu_mid);
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = p ? relu_from(v[i] + relu_from(acc[i], lo), lo_sum) : relu_from(acc[i], lo);
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int kg = rt * 2 + s;
            if (kg >= P.c2[0].nkg) continue;
#pragma unroll
            for (int r = 0; r < NRT2; ++r) {
                uint4 w[PR + 1];
#pragma unroll
                for (int i = 0; i <= PR; ++i)
                    w[i] = reinterpret_cast<const uint4 *>(P.c2[0].wp)[(size_t)(kg * NRT2 + r) * (64 * (PR + 1)) + i * 64 + lane];
#pragma unroll
                for (int e = 0; e < 8; ++e) acc2[r][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(held_value<PR>(w, e), v[s * 8 + e], acc2[r][0], 0, 0, 0);
            }
        }
    }
}

// N1: producers, NKG1: K steps of layer 1, NRT2: row tiles of layer 2.  Layer 1 takes three parts in either precision (the general
// kernel it stands for may run it on fp32 operations); PR: of layer 2.
// BlockParams used: x, y, N, Cin, H, W, Cy, c1, c1b (N1 == 2), n1, relu_mid, c2[0], coff2[0], relu_out, nblocks, and buf_stride
// (floats per filter buffer), lds_buf_off (floats of the shift tables before them).
template <int PR, int N1, int NKG1, int NRT2>
__global__ void __launch_bounds__(256, 2) chain_kernel(const BlockParams P)
{
    constexpr int PR1 = 2, NP1 = PR1 + 1, NP = PR + 1, ROWS1 = NKG1 * NP1;      // filter rows of 1 KB per producer and row tile
    constexpr int GROUPS = N1 * NKG1 + 2 * NRT2;       // K steps per row tile of layer 1: of the producers, then of layer 2
    extern __shared__ __attribute__((aligned(16))) float lds[];
    touch_arguments();
    const int L = logical_block();
    if (L >= P.nblocks) return;
    const int lane = threadIdx.x & 63, sub = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int HW = P.H * P.W;
    const ConvW &c2 = P.c2[0];

    // ---- this lane's pixel; images are as far apart as 32 pixels reach (offsets fit 32 bits: planner)
    const unsigned first = (unsigned)(L * 4 + wave) * 32u, pixels = (unsigned)P.N * (unsigned)HW;
    const unsigned n0 = min(first, pixels - 1u) / (unsigned)HW;
    const unsigned g = first + (lane & 31);
    const unsigned n = g / (unsigned)HW, p = g - n * (unsigned)HW;
    const bool own = g < pixels;
    ChainInput in;
    const unsigned reach = min((unsigned)P.N - n0, 31u / (unsigned)HW + 2u);        // images that 32 pixels touch
    in.rsrc = make_rsrc(P.x + (size_t)n0 * P.Cin * HW, (unsigned long long)reach * P.Cin * HW * 4ull);
    in.channels = P.Cin;
    in.plane = HW;
    in.off = own ? ((n - n0) * (unsigned)(P.Cin * HW) + p + (unsigned)(sub * 8 * HW)) * 4u : 0xfffffffcu;
    float xv[NKG1][8];
#pragma unroll
    for (int kg = 0; kg < NKG1; ++kg) in.load(xv[kg], kg, lane);

    // ---- shift tables of layer 1 -> LDS, [producer][channel]
    for (int i = threadIdx.x; i < N1 * P.c1.nrt * 8; i += 256) {
        const int pr = i >= P.c1.nrt * 8, q = i - (pr ? P.c1.nrt * 8 : 0);
        *(f32x4 *)(lds + i * 4) = (pr ? P.c1b : P.c1).aff[(q >> 1) * 64 + (q & 1) * 32];
    }
    // ---- filter rows of row tile rt of layer 1 (in the order of row_channel) and of the two K steps of layer 2 that it feeds:
    // rows of 1 KB, [producer][K step][part], then [K step][row tile][part]
    const __amdgpu_buffer_rsrc_t wa = make_rsrc(P.c1.wp, (unsigned long long)P.c1.nrt * (ROWS1 * 1024));
    const __amdgpu_buffer_rsrc_t wb = make_rsrc(N1 == 2 ? P.c1b.wp : P.c1.wp, (unsigned long long)P.c1.nrt * (ROWS1 * 1024));
    const __amdgpu_buffer_rsrc_t wc = make_rsrc(c2.wp, (unsigned long long)c2.nkg * (NRT2 * NP * 1024));
    const int permuted = ((lane & 32) + row_channel(lane & 31)) * 16, straight = lane * 16;
    float *buf = lds + P.lds_buf_off;
    // (few scalar instructions and branches: they stand in the way of a wave's matrix operations like any other)
    constexpr int R1 = (ROWS1 + 3) / 4, R2 = (2 * NRT2 * NP + 3) / 4;       // rows of a wave
    int at1[R1];
#pragma unroll
    for (int i = 0; i < R1; ++i) {
        const int r = i * 4 + wave, kg = r / NP1;
        at1[i] = (kg * P.c1.nrt * NP1 + r - kg * NP1) * 1024;
    }
    auto stage = [&](int rt, float *to) {
        auto row = [&](__amdgpu_buffer_rsrc_t from, int lane_at, int at, int r) {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(from, (__attribute__((address_space(3))) void *)(to + r * 256), 16, lane_at, at, 0, 0);
        };
#pragma unroll
        for (int i = 0; i < R1; ++i) {
            if (ROWS1 % 4 && i * 4 + wave >= ROWS1) continue;
            row(wa, permuted, at1[i] + rt * (NP1 * 1024), i * 4 + wave);
            if (N1 == 2) row(wb, permuted, at1[i] + rt * (NP1 * 1024), ROWS1 + i * 4 + wave);
        }
        const int live = min(2, c2.nkg - rt * 2) * (NRT2 * NP);        // rows of K steps that exist
#pragma unroll
        for (int i = 0; i < R2; ++i)
            if (i * 4 + wave < live) row(wc, straight, (rt * (2 * NRT2 * NP) + i * 4 + wave) * 1024, N1 * ROWS1 + i * 4 + wave);
    };
    // The rows of a K step past the last one are read (an intermediate of zeros meets them): they hold zeros, or what the row
    // tile before the last but one left there.
    if ((c2.nkg & 1) && P.c1.nrt <= 2)
        for (int r = NRT2 * NP + wave; r < 2 * NRT2 * NP; r += 4)
            *(f32x4 *)(buf + (P.c1.nrt - 1 & 1) * P.buf_stride + (N1 * ROWS1 + r) * 256 + lane * 4) = f32x4{0.f, 0.f, 0.f, 0.f};
    stage(0, buf);

    f32x16 acc2[NRT2][1], small2[NRT2][1];
    init_acc<32, NRT2, 1>(acc2, c2, 0);
#pragma unroll
    for (int r = 0; r < NRT2; ++r) zero_acc(small2[r][0]);

    // ---- the input in parts.  Bits that are left raise `odd` (split_pair), as those of the intermediate do below: the wave then
    // starts again with whole operands, so nothing needs to stand for such a value here.
    unsigned odd = 0;
    u32x4 xp[NKG1][NP1];
#pragma unroll
    for (int kg = 0; kg < NKG1; ++kg)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            unsigned w[NP1];
            split_pair<PR1>(xv[kg][2 * j], xv[kg][2 * j + 1], w, odd);
#pragma unroll
            for (int q = 0; q < NP1; ++q) xp[kg][q][j] = w[q];
        }
    // The largest sum of layer 1 as an unsigned number: 0xff800000 and above are -inf and NaN with the sign set, which an activation
    // turns to 0 (+inf and NaN do not come apart).
    unsigned least = 0;
    int lo1 = relu_bound(P.c1.relu), lo1b = relu_bound(P.c1b.relu), lo_sum = relu_bound(P.relu_mid);
    asm volatile("" : "+s"(lo1), "+s"(lo1b), "+s"(lo_sum));     // (seen through, a maximum against one becomes a maximum and a select)
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
#pragma unroll 1
    for (int rt = 0; rt < P.c1.nrt; ++rt) {
        const float *w = buf + (rt & 1) * P.buf_stride + lane * 4;
        // the filter rows of K step g + 2 of the tile are read before the matrix operations of K step g
        f32x4 a[3][NP1];
        auto fetch = [&](int g) {
            if (g >= GROUPS) return;
            constexpr int G1 = N1 * NKG1;
#pragma unroll
            for (int i = 0; i < (g < G1 ? NP1 : NP); ++i) a[g % 3][i] = *(const f32x4 *)(w + (g < G1 ? g * NP1 + i : G1 * NP1 + (g - G1) * NP + i) * 256);
        };
        // acc gets the large products, low the small ones; `beside(i)` are vector instructions for the time of the i-th operation
        auto mma = [&](f32x16 &acc, f32x16 &low, int g, const auto &b, auto beside) {
            constexpr int parts = sizeof(b) / 16;
            fetch(g + 2);
            int at = 0;
#pragma unroll
            for (int i = parts - 1; i >= 0; --i)
#pragma unroll
                for (int j = parts - 1 - i; j >= 0; --j) {
                    f32x16 &d = parts == 3 && i + j > 0 ? low : acc;
                    d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[g % 3][j]), __builtin_bit_cast(bf16x8, b[i]), d, 0, 0, 0);
                    beside(at++);
                    __builtin_amdgcn_sched_barrier(0);
                }
        };
        f32x16 acc[N1], low[N1];
        fetch(0);
        fetch(1);
#pragma unroll
        for (int pr = 0; pr < N1; ++pr) {
            zero_acc(low[pr]);
            const float *sh = lds + (pr * P.c1.nrt + rt) * 32 + sub * 8;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 s4 = *(const f32x4 *)(sh + (q >> 1) * 16 + (q & 1) * 4);
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[pr][q * 4 + i] = s4[i];
            }
        }
        if (rt + 1 < P.c1.nrt) stage(rt + 1, buf + ((rt + 1) & 1) * P.buf_stride);
        constexpr int OPS1 = products_of(PR1), OPS = products_of(PR);
        f32x16 v;
        u32x4 mp[2][NP];
        auto sum = [&](int pr, int i) {
            const float t = acc[pr][i] + low[pr][i];
            least = max(least, __builtin_bit_cast(unsigned, t));
            v[i] = pr == 0 ? relu_from(t, lo1) : relu_from(v[i] + relu_from(t, lo1b), lo_sum);
        };
        auto split = [&](u32x4 (&to)[NP], int from, int j) {
            unsigned w[NP];
            split_pair<PR>(v[from + 2 * j], v[from + 2 * j + 1], w, odd);
#pragma unroll
            for (int q = 0; q < NP; ++q) to[q][j] = w[q];
        };
        // part k of `all` in the time of operation k of `ops`
        auto share = [](int k, int ops, int all, auto f) {
#pragma unroll
            for (int i = 0; i < all; ++i)
                if (i * ops / all == k) f(i);
        };
#pragma unroll
        for (int kg = 0; kg < NKG1; ++kg) mma(acc[0], low[0], kg, xp[kg], [](int) {});
        if constexpr (N1 == 2) {
#pragma unroll
            for (int kg = 0; kg < NKG1; ++kg)
                mma(acc[1], low[1], NKG1 + kg, xp[kg], [&](int k) { share(kg * OPS1 + k, NKG1 * OPS1, 16, [&](int i) { sum(0, i); }); });
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) sum(N1 - 1, i);
#pragma unroll
        for (int j = 0; j < 4; ++j) split(mp[0], 0, j);
#pragma unroll
        for (int r = 0; r < NRT2; ++r)
            mma(acc2[r][0], small2[r][0], N1 * NKG1 + r, mp[0], [&](int k) { share(r * OPS + k, NRT2 * OPS, 4, [&](int j) { split(mp[1], 8, j); }); });
#pragma unroll
        for (int r = 0; r < NRT2; ++r) mma(acc2[r][0], small2[r][0], N1 * NKG1 + NRT2 + r, mp[1], [](int) {});
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
    }
    if constexpr (PR == 2) add_small<NRT2, 1>(acc2, small2);
    const bool again = __builtin_amdgcn_ballot_w64(odd != 0u || least >= 0xff800000u) != 0;
    if (again || any_not_finite<NRT2, 1>(acc2)) chain_whole<NRT2, PR>(acc2, P, in, lane);
    if (!own) return;
    const __amdgpu_buffer_rsrc_t yr = make_rsrc(P.y + ((size_t)n0 * P.Cy + P.coff2[0]) * HW,
                                                ((unsigned long long)reach * P.Cy - P.coff2[0]) * HW * 4ull);
    const unsigned off = ((n - n0) * (unsigned)(P.Cy * HW) + p + (unsigned)(sub * 4 * HW)) * 4u;
    const int lo2 = max(relu_bound(c2.relu), relu_bound(P.relu_out));
#pragma unroll
    for (int r = 0; r < NRT2; ++r)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int cu = r * 32 + (e >> 2) * 8 + (e & 3);        // channel of lane half 0
            if (cu + sub * 4 < c2.cout)
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, relu_from(acc2[r][0][e], lo2)), yr, off, cu * HW * 4, 0);
        }
}

}  // namespace xl

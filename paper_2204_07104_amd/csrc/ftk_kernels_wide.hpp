// Gradient pass for ranks above 32 (padded to 64) at orders 2 and 3: a workgroup works on one tile of 32 samples together.
//
// A wave that takes a tile of its own (grad_tiled_kernel) needs all P x P blocks of every contraction: 192 accumulators for the
// core gradient alone, so a SIMD holds one wave, and nothing covers that wave's trips through LDS.  Here the 64 columns are cut
// into four blocks of 16 and a wave works on one of them, for all 32 samples: its share of the core factors stays in registers
// as operands (72 registers for one product), its share of the core gradient takes 48.  Two teams of four waves, one of each per SIMD,
// work on tiles one behind the other:
//
//   team 0, tile i:      rows -> bf16 parts in LDS | projections C = A B, partial predictions | errors, -e W -> parts in LDS,
//                        core gradient GB += A^T (-e W)
//   team 1, tile i - 1:  -e GS = (-e W) B^T, one-hot sums and float atomics, a mode between two barriers; draws the samples
//
// Products are those of ftk_split.hpp (three bf16 parts, six partial products).  The samples' rows and -e W sit in LDS as 16 x 16
// blocks of their parts, for two tiles: 147 KB at order 3, which is what limits it to one workgroup per CU and to order 3.
// A contraction over a tile's samples fills the instruction's 32 slots, so no part is taken twice.
//
// What bounds it, J = R = 64, 1e6 samples (649 us a launch with 40 + 47 table rows, modes by power laws; with 16 + 16, as for the
// variants that follow, 706, where the general kernel took 765): products (3 900 clocks of a
// SIMD per tile), vector instructions (3 600) and LDS (4 600 of the CU) that come one after the other more than side by side,
// because a SIMD has one wave of each team and the teams meet three times a tile.  Without atomics 666 us, without rows
// from memory either 568.  Core gradients dealt to both teams: 708 us.  Rows asked for two tiles ahead, and all core gradients with
// team 1: 758 us; spilled registers are dear, as their reloads wait behind the atomics (799 us with 36).
// Small sample sets gain most: there are no core factors to write to LDS first and no accumulators of several waves to sum last.
// A tile of order 2 takes 3.3 us, which is more than the general kernel needs for the same samples: the general kernel serves
// large sets there, and some at order 3 (where the line lies: wide_pass in ftk_api.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "ftk_kernels_tiled.hpp"

namespace ftk {

constexpr int kWideMaxOrder = 3, kWideThreads = 512, kWideTile = 32;
constexpr int kWideDraw = 8, kWideParks = 2 * kWideDraw;   // tiles whose samples are drawn at a time; tiles parked
constexpr int kWidePartStride = 2 * 4 * kSplitBlockBytes;          // bytes between the parts of a block: [part][half of the tile][column block]
__host__ __device__ constexpr int wide_park_words(int order) { return (2 * order + 1) * kWideTile; }   // row offsets | route words | values
__host__ __device__ constexpr size_t wide_lds_bytes(int order) {
    return (size_t)4 * order * 3 * kWidePartStride + 4 * ((size_t)kWideParks * wide_park_words(order) + 4 * kWideTile);
}

template <int N, bool X4>
__global__ void __launch_bounds__(kWideThreads) grad_wide_kernel(TiledArgs g) {
    static_assert(N >= 2 && N <= kWideMaxOrder, "two tiles' operands fit LDS up to order 3");
    extern __shared__ float lds[];
    constexpr int D = 64;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), cb = wave & 3;   // cb: the wave's block of columns
    const int c = lane & 15, g4 = lane >> 4;
    lds_char* blocks = (lds_char*)lds;
    unsigned int* parks = reinterpret_cast<unsigned int*>(lds) + 4 * N * 3 * kWidePartStride / 4;   // tile t at slot t % kWideParks
    float* partial = reinterpret_cast<float*>(parks + kWideParks * wide_park_words(N));                      // [column block][sample]: predictions
    const int straight = split_slot(c, g4), transposed = split_slot(4 * g4 + (c >> 2), c & 3);
    const SplitConst sc = split_const();
    // block (half, col) of part 0 of the rows (what 0) or of -e W (what 1) of mode n, in the buffer of tile t
    auto block = [&](int t, int what, int n, int half, int col) {
        return blocks + ((((t & 1) * 2 + what) * N + n) * 3) * kWidePartStride + (half * 4 + col) * kSplitBlockBytes;
    };
    // What the waves exchange goes through LDS: its own requests are waited for, not those to memory (a tile's rows and its
    // atomics stay under way).
    auto meet = [&]() {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // what the bf16 instructions cut off towards -inf goes the other way in every other workgroup (see ftk_split.hpp)
    const unsigned int sign = (blockIdx.x & 1u) << 31;
    auto turned = [&](float v) { return __uint_as_float(__float_as_uint(v) ^ sign); };

    // the workgroup's samples: whole tiles of 16, as the host deals them
    const int wg = (int)blockIdx.x;
    const int wg_tiles = g.tiles_each + (wg < g.tiles_more ? 1 : 0);
    const long long first = ((long long)wg * g.tiles_each + (wg < g.tiles_more ? wg : g.tiles_more)) * 16;
    const int mine = first < g.M ? (int)min((long long)wg_tiles * 16, g.M - first) : 0;
    const int T = (mine + kWideTile - 1) / kWideTile;

    // an operand of a product over a block row or column of 64: parts h, m, l of column blocks (0, 1) and (2, 3)
    auto straight_parts = [&](const lds_char* b, bf16x8 (&x)[2][3]) {
#pragma unroll
        for (int kc = 0; kc < 2; ++kc)
#pragma unroll
            for (int q = 0; q < 3; ++q)
                x[kc][q] = pair_up(lds_straight(b + q * kWidePartStride + (2 * kc) * kSplitBlockBytes + straight),
                                   lds_straight(b + q * kWidePartStride + (2 * kc + 1) * kSplitBlockBytes + straight));
    };
    // ... over the tile's samples: parts of one column block, both halves of the tile
    auto transposed_parts = [&](const lds_char* b, bf16x8 (&x)[3]) {
#pragma unroll
        for (int q = 0; q < 3; ++q)
            x[q] = pair_up(lds_transposed(b + q * kWidePartStride + transposed), lds_transposed(b + q * kWidePartStride + 4 * kSplitBlockBytes + transposed));
    };
    const floatx4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    // the six partial products of a contraction over 64, smallest first, in two sums
    auto contract = [&](const bf16x8 (&x)[2][3], const bf16x8 (&y)[2][3]) {
        floatx4 sum[2] = {zero, zero};
#pragma unroll
        for (int part = 2; part >= 0; --part)
#pragma unroll
            for (int q = 2 - part; q >= 0; --q)
#pragma unroll
                for (int kc = 0; kc < 2; ++kc) sum[kc] = mfma_bf16(x[kc][part], y[kc][q], sum[kc]);
        return sum[0] + sum[1];
    };
    // Core gradient of a mode over a tile's samples: this wave's columns 16 cb .. 16 cb + 15 of all rows.  Each tile's sum starts
    // from zero and is then added (see ftk_split.hpp).
    auto core_gradient = [&](int t, int n, floatx4 (&GB)[4]) {
        bf16x8 ew[3], a[2][2][3];
        transposed_parts(block(t, 1, n, 0, cb), ew);
#pragma unroll
        for (int u = 0; u < 2; ++u) transposed_parts(block(t, 0, n, 0, u), a[0][u]);
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            if (p == 0) {
#pragma unroll
                for (int u = 0; u < 2; ++u) transposed_parts(block(t, 0, n, 0, 2 + u), a[1][u]);
                __builtin_amdgcn_sched_barrier(0x6);
            }
            floatx4 sum[2] = {zero, zero};
#pragma unroll
            for (int part = 2; part >= 0; --part)
#pragma unroll
                for (int q = 2 - part; q >= 0; --q)
#pragma unroll
                    for (int u = 0; u < 2; ++u) sum[u] = mfma_bf16(a[p][u][part], ew[q], sum[u]);
            GB[2 * p] += sum[0];
            GB[2 * p + 1] += sum[1];
        }
    };
    auto store_core = [&](int n, const floatx4 (&GB)[4]) {
        float* out = g.gb_partial + (size_t)blockIdx.x * g.B_total + g.B_off[n];
        const int r = 16 * cb + c;
#pragma unroll
        for (int jb = 0; jb < 4; ++jb)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int j = 16 * jb + 4 * g4 + v;
                if (j < g.J[n] && r < g.R) out[j * g.R + r] = turned(GB[jb][v]);
            }
    };
    // LDS reads stay in front of the products of the step before theirs: all waves come from a barrier, and would else read
    // together and multiply together (with 16 + 16 table rows 706 us against 718)
    auto hold_reads = [&]() { __builtin_amdgcn_sched_barrier(0x6); };

    if (wave < 4) {
        __amdgpu_buffer_rsrc_t rsrc_A[N];
        bf16x8 Bp[N][2][3];    // B^(n)[j][16 cb + c]: slots of block kc are j = 32 kc + 4 g .. +3 and 32 kc + 16 + 4 g .. +3
#pragma unroll
        for (int n = 0; n < N; ++n) {
            rsrc_A[n] = make_rsrc(g.A + g.A_off[n], g.mode_bytes[n] + kRowSlack);
            const int r = 16 * cb + c;
#pragma unroll
            for (int kc = 0; kc < 2; ++kc) {
                floatx4 lo, hi;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int j = 32 * kc + 4 * g4 + i;
                    lo[i] = j < g.J[n] && r < g.R ? g.B[g.B_off[n] + j * g.R + r] : 0.0f;
                    hi[i] = j + 16 < g.J[n] && r < g.R ? g.B[g.B_off[n] + (j + 16) * g.R + r] : 0.0f;
                }
                split2<true>(lo, hi, sc, Bp[n][kc]);
            }
        }
        // this wave's block of columns of the rows of a tile: 16 bytes per lane, straight into the layout of a block
        floatx4 rows[N][2];
        floatx4 GB[N][4];      // core gradient: rows 16 jb + 4 g + v, column 16 cb + c
#pragma unroll
        for (int n = 0; n < N; ++n)
#pragma unroll
            for (int jb = 0; jb < 4; ++jb) GB[n][jb] = zero;
        auto request = [&](int t) {
            const unsigned int* park = parks + (t % kWideParks) * wide_park_words(N);
            const int col = 16 * cb + 4 * g4;
#pragma unroll
            for (int n = 0; n < N; ++n)
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const unsigned int row = park[n * kWideTile + half * 16 + c];
                    const unsigned int off = col < g.J[n] ? row + (unsigned int)col * 4u : g.mode_bytes[n] + kRowSlack;
                    rows[n][half] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(rsrc_A[n], (int)off, 0, 0));
                }
        };
        meet();   // the first tiles are parked
        if (T > 0) request(0);
#pragma unroll 1
        for (int t = 0; t <= T; ++t) {
            if (t < T) {
#pragma unroll
                for (int n = 0; n < N; ++n)
#pragma unroll
                    for (int half = 0; half < 2; ++half) {
                        if constexpr (!X4) {   // columns past J_n: the row behind, no part of this one
#pragma unroll
                            for (int v = 1; v < 4; ++v) rows[n][half][v] = 16 * cb + 4 * g4 + v < g.J[n] ? rows[n][half][v] : 0.0f;
                        }
                        store_block(block(t, 0, n, half, cb) + straight, kWidePartStride, split<true>(rows[n][half], sc));
                    }
            }
            if (t + 1 < T) request(t + 1);
            meet();
            floatx4 w[2][N];
            float x[2] = {0.0f, 0.0f};
            if (t < T) {
                const float* val = reinterpret_cast<const float*>(parks + (t % kWideParks) * wide_park_words(N)) + 2 * N * kWideTile;
                // projections: w[half][n][v] = c^(n)_{r = 16 cb + 4 g + v} of sample 16 half + c
                bf16x8 a[2][2][3];
                straight_parts(block(t, 0, 0, 0, 0), a[0]);
#pragma unroll
                for (int st = 0; st < 2 * N; ++st) {
                    if (st + 1 < 2 * N) straight_parts(block(t, 0, (st + 1) >> 1, (st + 1) & 1, 0), a[(st + 1) & 1]);
                    hold_reads();
                    w[st & 1][st >> 1] = contract(Bp[st >> 1], a[st & 1]);
                }
                // leave-one-out products (in the place of the projections) and this block's share of the predictions
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    x[half] = val[half * 16 + c];
                    floatx4 before[N], run = {1.0f, 1.0f, 1.0f, 1.0f};
#pragma unroll
                    for (int n = 0; n < N; ++n) {
                        before[n] = run;
                        run *= w[half][n];
                    }
                    const float sum = sum_over_groups((run[0] + run[1]) + (run[2] + run[3]));
                    if (g4 == 0) partial[cb * kWideTile + half * 16 + c] = sum;
                    run = floatx4{1.0f, 1.0f, 1.0f, 1.0f};
#pragma unroll
                    for (int n = N - 1; n >= 0; --n) {
                        const floatx4 s = w[half][n];
                        w[half][n] = before[n] * run;
                        run *= s;
                    }
                }
            }
            meet();
            if (t < T) {
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const float* p = partial + half * 16 + c;
                    const float neg_e = turned(((p[0] + p[kWideTile]) + (p[2 * kWideTile] + p[3 * kWideTile])) - x[half]);
#pragma unroll
                    for (int n = 0; n < N; ++n)
                        store_block(block(t, 1, n, half, cb) + straight, kWidePartStride, split(w[half][n] * neg_e, sc));
                }
                lds_wave_sync();   // (the wave's own blocks of -e W, read back)
#pragma unroll
                for (int n = 0; n < N; ++n) core_gradient(t, n, GB[n]);
            }
            meet();
        }
#pragma unroll
        for (int n = 0; n < N; ++n) store_core(n, GB[n]);
    } else {
        __amdgpu_buffer_rsrc_t rsrc_dA[N];
        bf16x8 Bg[N][2][3];   // B^(n)[16 cb + c][r]: slots as above, with r for j
        floatx4 Top[N];       // gradient sums of rows 0..15: [row 4 g + v][column 16 cb + c]
#pragma unroll
        for (int n = 0; n < N; ++n) {
            rsrc_dA[n] = make_rsrc(g.dA + g.A_off[n], g.dA_bytes[n]);
            const int j = 16 * cb + c;
#pragma unroll
            for (int kc = 0; kc < 2; ++kc) {
                floatx4 lo, hi;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int r = 32 * kc + 4 * g4 + i;
                    lo[i] = j < g.J[n] && r < g.R ? g.B[g.B_off[n] + j * g.R + r] : 0.0f;
                    hi[i] = j < g.J[n] && r + 16 < g.R ? g.B[g.B_off[n] + j * g.R + r + 16] : 0.0f;
                }
                split2<true>(lo, hi, sc, Bg[n][kc]);
            }
            Top[n] = zero;
        }
        shortx4 diagonal;   // the all-one diagonal as a bf16 operand: column c of rows 4g .. 4g+3
#pragma unroll
        for (int i = 0; i < 4; ++i) diagonal[i] = 4 * g4 + i == c ? (short)0x3f80 : (short)0;
        const bf16x8 diagonal2 = pair_up(diagonal, diagonal), diagonal_high = pair_up(shortx4{0, 0, 0, 0}, diagonal);
        const unsigned int top_key = kRouteOneHot | ((unsigned int)c << 2);
        const unsigned int kDropped = 0x40000000u;

        bf16x8 x[2][2][3];
        // the gradients of mode n of tile t, and where they go
        auto gradient = [&](auto mode, int t) {
            constexpr int n = decltype(mode)::value;
            const unsigned int* routes = parks + (t % kWideParks) * wide_park_words(N) + (N + n) * kWideTile;
            const unsigned int col4 = 16 * cb + c < g.J[n] ? (unsigned int)((16 * cb + c) * 4) : kDropped;
            floatx4 gs[2], grad[2];
            shortx4 onehot[2];
            Split rows_y[2];
            // x[0] holds the first operand; the next step's is read before a step's products
            straight_parts(block(t, 1, n, 1, 0), x[1]);
            hold_reads();
            gs[0] = contract(x[0], Bg[n]);
#pragma unroll
            for (int half = 0; half < 2; ++half) rows_y[half] = transposed_block(block(t, 0, n, half, cb) + transposed, kWidePartStride);
            if constexpr (n + 1 < N) straight_parts(block(t, 1, n + 1, 0, 0), x[0]);   // the next mode's first operand
            hold_reads();
            gs[1] = contract(x[1], Bg[n]);
            bool any = false;
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                // the rows whole, for the regulariser term: the all-one diagonal times their parts (exact)
                floatx4 ay = mfma_bf16(diagonal_high, pair_up(high_half(rows_y[half].mh), rows_y[half].l), zero);
                ay = mfma_bf16(diagonal2, rows_y[half].mh, ay);
                const uint4 route4 = *reinterpret_cast<const uint4*>(routes + half * 16 + 4 * g4);
                const unsigned int route[4] = {route4.x, route4.y, route4.z, route4.w};   // samples 16 half + 4g ..
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    grad[half][v] = turned(g.scale) * fmaf(turned(g.lambda_A), ay[v], gs[half][v]);
                    __builtin_amdgcn_raw_ptr_buffer_atomic_fadd_f32(grad[half][v], rsrc_dA[n], (int)(route[v] + col4), 0, 0);
                    const bool is_top = route[v] == top_key;
                    onehot[half][v] = is_top ? (short)0x3f80 : (short)0;
                    any = any || is_top;
                }
            }
            if (g.top[n] > 0 && __builtin_amdgcn_ballot_w64(any) != 0) {
                floatx4 back[2], sum = zero;
#pragma unroll
                for (int half = 0; half < 2; ++half)
#pragma unroll
                    for (int v = 0; v < 4; ++v) back[half][v] = turned(grad[half][v]);
                bf16x8 parts[3];
                split2(back[0], back[1], sc, parts);
                const bf16x8 rows_hit = pair_up(onehot[0], onehot[1]);
#pragma unroll
                for (int q = 2; q >= 0; --q) sum = mfma_bf16(rows_hit, parts[q], sum);
                Top[n] += sum;
            }
        };
        // Records: the team draws those of kWideDraw tiles at a time, a lane a sample, and parks them that many tiles later: row
        // offsets and route words as grad_tiled_kernel does (see tiled_grad_park_words).
        const uint4* rec4 = reinterpret_cast<const uint4*>(g.coo.rec);
        uint4 rec = {0u, 0u, 0u, 0u};
        const int my_tile = 2 * cb + (lane >> 5), my_place = lane & 31;
        auto load_records = [&](int t0) {
            const int local = (t0 + my_tile) * kWideTile + my_place;
            rec = rec4[local < mine ? sample_place(g.seed, (uint64_t)(first + local), g.rule) : 0u];
        };
        auto park_records = [&](int t0) {
            unsigned int* park = parks + ((t0 + my_tile) % kWideParks) * wide_park_words(N) + my_place;
            const bool act = (t0 + my_tile) * kWideTile + my_place < mine;
            const uint32_t flat[4] = {rec.x, rec.y, rec.z, rec.w};
#pragma unroll
            for (int n = 0; n < N; ++n) {
                const int row = (int)flat[n];
                const unsigned int in_mode = act ? (unsigned int)(row * g.J[n] * 4) : g.mode_bytes[n] + kRowSlack;
                park[n * kWideTile] = in_mode;
                park[(N + n) * kWideTile] =
                    !act ? kRouteNone : row < g.top[n] ? kRouteOneHot | ((unsigned int)row << 2)
                    : row < g.K[n] ? g.table_off[n] + blockIdx.x * g.table_stride + (unsigned int)((g.hot_off[n] + row) * D * 4) : in_mode;
            }
            park[2 * N * kWideTile] = act ? flat[N] : 0u;
        };
        static_assert(kWideDraw == 8, "four waves draw two tiles each");
        load_records(0);
        park_records(0);
        load_records(kWideDraw);
        meet();
#pragma unroll 1
        for (int t = 0; t <= T; ++t) {
            if (t > 0) {
                straight_parts(block(t - 1, 1, 0, 0, 0), x[0]);
                gradient(std::integral_constant<int, 0>{}, t - 1);
            }
            meet();
            if (t > 0) gradient(std::integral_constant<int, 1>{}, t - 1);
            meet();
            if constexpr (N > 2)
                if (t > 0) gradient(std::integral_constant<int, 2>{}, t - 1);
            if (t % kWideDraw == kWideDraw - 2) {   // team 0 asks for the first of them in the next turn
                park_records(t + 2);
                load_records(t + 2 + kWideDraw);
            }
            meet();
        }
        float* hot = g.hot_partial + (size_t)blockIdx.x * g.H * D;
#pragma unroll
        for (int n = 0; n < N; ++n)
            if (g.top[n] > 0)
#pragma unroll
                for (int v = 0; v < 4; ++v) hot[(g.hot_off[n] + 4 * g4 + v) * D + 16 * cb + c] = turned(Top[n][v]);
    }
}

}  // namespace ftk

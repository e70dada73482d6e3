// Synchronous step in the space of the projections with atomics: for ranks R <= 8 on tensors that the row owners
// (ftk_kernels_owners.hpp) do not suit, such as those with frequent rows.
//
//   S^(n) = A^(n) B^(n)                  projected rows, one streaming pass (project_rows_kernel)
//   v_k^(n) = -e_k w_k^(n)               per sample from N gathered rows of S: products only
//   D^(n)_i = sum of v_k^(n), h_i = number of the samples that hit row i      (scatter_projected_kernel)
//   A^(n)_i <- A^(n)_i - lr_A ( D^(n)_i (B^(n))^T + lambda_A h_i A^(n)_i ),
//   GB^(n)  = sum_i A^(n)_i (x) D^(n)_i                                        (apply_projected_kernel)
//
// The step of the other kernels with the sums over samples drawn in front of the products with B^(n) and A^(n).  Those are
// done once per touched row, so nothing per sample needs the matrix cores (padded to 16 x 16, they spent a half to three
// quarters of their work on zeros at these ranks), and a sample is one lane's work: no exchange between register layouts.  The
// count h_i, which the regulariser needs, rides as one more column of D: a row of R + 1 floats is still one 64-byte request
// to the atomic unit.
//
// Rows take the three routes of the J = R = 16 kernel: rows 0..15 of a mode, where they are frequent, are summed 16 samples at
// a time by the matrix core against a one-hot operand; rows [16, K_n) in a table per workgroup in LDS; the others by float
// atomics into the accumulator, whose rows (16 floats apart, as the padded A^(n)) have room for the count.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ftk_kernels_mfma16.hpp"

namespace ftk {

constexpr int kProjectedMaxOrder = 5, kProjectedMaxRank = 8;
constexpr int kScatterWaves = 16, kScatterThreads = kScatterWaves * 64;
// Q: float4 pieces of a row of S.  A row of sums has 4 Q columns and the count.
__host__ __device__ constexpr int projected_width(int Q) { return 4 * Q + 1; }
// floats of LDS next to the table: per wave 64 rows of sums and where they go
__host__ __device__ constexpr int scatter_wave_floats(int Q) { return kScatterWaves * 64 * (projected_width(Q) + 1); }
// floats of one workgroup's table as it is stored
__host__ __device__ constexpr int scatter_table_floats(int H, int Q) { return (H * projected_width(Q) + 3) & ~3; }

struct ScatterArgs {
    Coo coo;
    SampleRule rule;
    uint64_t seed;
    long long M;
    int groups_each, groups_more;              // groups of 64 samples over the workgroups: each gets groups_each, the first groups_more one more
    const float* S[kProjectedMaxOrder];
    int K[kProjectedMaxOrder], top[kProjectedMaxOrder], hot_off[kProjectedMaxOrder];
    unsigned int acc_off[kProjectedMaxOrder];  // bytes from dA to the accumulator of the mode's row 0
    int H;
    float* dA;
    unsigned int all_bytes;                    // of dA, below 2^31 - 64
    float* tables;                             // [gridDim.x][scatter_table_floats(H, Q)]
};

// One workgroup per CU, 16 waves, a sample per lane.  A wave's turn: the rows of S of 64 samples (requested while the turn
// before it was scattered), the products, then mode by mode the 64 rows of sums are written to the wave's LDS buffer in the
// order of their routes, so that each route reads its own share of them without gaps, whole rows at a time.
// What bounds it: see launch_projected's figures.
template <int N, int Q>
__global__ void __launch_bounds__(kScatterThreads) scatter_projected_kernel(ScatterArgs g) {
    extern __shared__ float lds[];
    constexpr int W4 = (N + 1 + 3) / 4, WD = projected_width(Q), ROWS = 64 / WD;   // ROWS: rows one instruction takes
    constexpr unsigned int kNowhere = 0x7fffffc0u;   // past the end of dA: dropped by the buffer check
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g4 = lane >> 4;         // operand layout of the matrix instruction
    const int mine = lane / WD, col = lane - mine * WD;   // row and column of this lane where whole rows are moved
    const bool mover = mine < ROWS;
    float* table = lds;
    float* stage = lds + scatter_table_floats(g.H, Q) + wave * (64 * (WD + 1));
    unsigned int* word = reinterpret_cast<unsigned int*>(stage + 64 * WD);
    const uint4* rec4 = reinterpret_cast<const uint4*>(g.coo.rec);
    const __amdgpu_buffer_rsrc_t rsrc_dA = make_rsrc(g.dA, g.all_bytes);

    // the wave's share: whole groups of 64 samples, first to first + n_turns
    const int blk = (int)blockIdx.x;
    const int in_block = g.groups_each + (blk < g.groups_more ? 1 : 0);
    const long long block0 = (long long)blk * g.groups_each + (blk < g.groups_more ? blk : g.groups_more);
    const int n_turns = in_block / kScatterWaves + (wave < in_block % kScatterWaves ? 1 : 0);
    const long long first = block0 + (long long)wave * (in_block / kScatterWaves) + (wave < in_block % kScatterWaves ? wave : in_block % kScatterWaves);
    // Entry rule: two turns share their Philox blocks (a block yields the positions of samples 2 k and 2 k + 1: the even turn
    // takes the 2 l-th of the 128 samples, the odd one the next).
    uint32_t odd_place = 0u;
    auto paired = [&](int t) { return g.rule.n_runs == 0 && (t | 1) < n_turns; };
    auto sample_of = [&](int t) -> long long {
        const long long base = (first + t) * 64;
        return paired(t) ? ((t & 1) ? base - 64 : base) + 2 * lane + (t & 1) : base + lane;
    };
    uint4 rec[W4];
    auto load_record = [&](int t) {
        const long long k = sample_of(t);
        uint32_t p;
        if (!paired(t)) {
            p = sample_place(g.seed, (uint64_t)k, g.rule);
        } else if ((t & 1) == 0) {
            const uint64_t ctr = (uint64_t)k >> 1;
            const U4 o = philox4x32_10((uint32_t)ctr, (uint32_t)(ctr >> 32), 0u, 0u, (uint32_t)g.seed, (uint32_t)(g.seed >> 32));
            p = (uint32_t)__umul64hi(((uint64_t)o.y << 32) | (uint64_t)o.x, g.rule.nnz);
            odd_place = (uint32_t)__umul64hi(((uint64_t)o.w << 32) | (uint64_t)o.z, g.rule.nnz);
        } else {
            p = odd_place;
        }
        if (k >= g.M) p = 0u;
#pragma unroll
        for (int q = 0; q < W4; ++q) rec[q] = rec4[(size_t)p * W4 + q];
    };
    uint32_t flat[4 * W4];
    floatx4 s[N][Q];
    auto gather = [&]() {   // the rows that the records in `rec` name
#pragma unroll
        for (int q = 0; q < W4; ++q) {
            flat[4 * q + 0] = rec[q].x;
            flat[4 * q + 1] = rec[q].y;
            flat[4 * q + 2] = rec[q].z;
            flat[4 * q + 3] = rec[q].w;
        }
#pragma unroll
        for (int n = 0; n < N; ++n)
#pragma unroll
            for (int q = 0; q < Q; ++q) s[n][q] = *reinterpret_cast<const floatx4*>(g.S[n] + (uint64_t)flat[n] * (4u * Q) + 4 * q);
    };
    if (n_turns > 0) load_record(0);
    for (int q = tid; q < g.H * WD; q += kScatterThreads) table[q] = 0.0f;
    __syncthreads();

    floatx4 Top[N];   // rows 0..15 of each mode: [row 4 g4 + v][column c]
#pragma unroll
    for (int n = 0; n < N; ++n) Top[n] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    if (n_turns > 0) {
        gather();
        if (n_turns > 1) load_record(1);
    }
    for (int t = 0; t < n_turns; ++t) {
        const bool act = sample_of(t) < g.M;
        uint32_t row[N];
        floatx4 v[N][Q];
        {
            // leave-one-out products by a prefix and a suffix sweep, times -e
            const float x = __uint_as_float(flat[N]);
            floatx4 run[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) run[q] = floatx4{1.0f, 1.0f, 1.0f, 1.0f};
#pragma unroll
            for (int n = 0; n < N; ++n) {
                row[n] = flat[n];
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    v[n][q] = run[q];
                    run[q] *= s[n][q];
                }
            }
            float sum = 0.0f;
#pragma unroll
            for (int q = 0; q < Q; ++q) sum += (run[q][0] + run[q][1]) + (run[q][2] + run[q][3]);
            const float minus_e = act ? sum - x : 0.0f;
#pragma unroll
            for (int q = 0; q < Q; ++q) run[q] = floatx4{minus_e, minus_e, minus_e, minus_e};
#pragma unroll
            for (int n = N - 1; n >= 0; --n)
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    v[n][q] *= run[q];
                    run[q] *= s[n][q];
                }
        }
        if (t + 1 < n_turns) {   // the next turn's rows, and the records of the one after it
            gather();
            if (t + 2 < n_turns) load_record(t + 2);
        }
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const bool one = act && (int)row[n] < g.top[n];
            const bool tab = act && !one && (int)row[n] < g.K[n];
            const bool atm = act && (int)row[n] >= g.K[n];
            const unsigned long long b_atm = __builtin_amdgcn_ballot_w64(atm), b_tab = __builtin_amdgcn_ballot_w64(tab),
                                     b_one = __builtin_amdgcn_ballot_w64(one);
            const int n_atm = __popcll(b_atm), n_tab = __popcll(b_tab), n_one = __popcll(b_one);
            // place in the buffer: atomics | table | one-hot | slots with no sample
            const unsigned long long same = atm ? b_atm : tab ? b_tab : one ? b_one : ~(b_atm | b_tab | b_one);
            const int at = (atm ? 0 : tab ? n_atm : one ? n_atm + n_tab : n_atm + n_tab + n_one) +
                           __popcll(same & ((1ull << lane) - 1ull));
            float* mine_out = stage + at * WD;
#pragma unroll
            for (int q = 0; q < Q; ++q)
#pragma unroll
                for (int i = 0; i < 4; ++i) mine_out[4 * q + i] = v[n][q][i];
            mine_out[4 * Q] = 1.0f;
            word[at] = atm ? g.acc_off[n] + row[n] * 64u : tab ? (unsigned int)(g.hot_off[n] + (int)row[n]) * (unsigned int)WD : row[n];
            lds_wave_sync();
            // rows 0..15: [row x sample] . [sample x column], four samples an instruction
            if (n_one > 0) {
                const int begin = n_atm + n_tab, end = begin + n_one;
                for (int e0 = begin; e0 < end; e0 += 16)
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int e = e0 + 4 * k + g4, in = e < 63 ? e : 63;
                        const float is = (e < end && word[in] == (unsigned int)c) ? 1.0f : 0.0f;
                        const float val = c < WD ? stage[in * WD + c] : 0.0f;
                        Top[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(is, val, Top[n], 0, 0, 0);
                    }
            }
            // the workgroup's table, by compare-and-swap (the native LDS float add takes 3 clocks per lane)
            for (int e0 = n_atm; e0 < n_atm + n_tab; e0 += 2 * ROWS) {
                float val[2];
                unsigned int cell[2], want[2], got[2];
                bool todo[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int e = e0 + i * ROWS + mine;
                    todo[i] = mover && e < n_atm + n_tab;
                    const int in = todo[i] ? e : n_atm;
                    val[i] = stage[in * WD + col];
                    cell[i] = lds_address(table) + (word[in] + (unsigned int)col) * 4u;
                    want[i] = *(lds_u32*)(uintptr_t)cell[i];
                }
                do {
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        if (todo[i]) got[i] = lds_cas(cell[i], want[i], __float_as_uint(__uint_as_float(want[i]) + val[i]));
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        if (todo[i]) {
                            todo[i] = got[i] != want[i];
                            want[i] = got[i];
                        }
                } while (todo[0] || todo[1]);
            }
            // everything else: float atomics into the accumulator
            for (int e0 = 0; e0 < n_atm; e0 += 2 * ROWS)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int e = e0 + i * ROWS + mine;
                    const bool there = mover && e < n_atm;
                    const int in = there ? e : 0;
                    const float val = stage[in * WD + col];
                    const unsigned int off = there ? word[in] + (unsigned int)col * 4u : kNowhere;
                    __builtin_amdgcn_raw_ptr_buffer_atomic_fadd_f32(val, rsrc_dA, (int)off, 0, 0);
                }
            lds_wave_sync();   // the next mode overwrites the buffer
        }
    }
#pragma unroll
    for (int n = 0; n < N; ++n)
        if (g.top[n] > 0 && c < WD)
#pragma unroll
            for (int i = 0; i < 4; ++i) lds_float_add(table + (g.hot_off[n] + 4 * g4 + i) * WD + c, Top[n][i]);
    __syncthreads();
    float* out = g.tables + (size_t)blockIdx.x * scatter_table_floats(g.H, Q);
    for (int q = tid; q < g.H * WD; q += kScatterThreads) out[q] = table[q];
}

constexpr int kApplyProjectedThreads = 1024;

struct ApplyProjectedArgs {
    int order, H, parts;                     // parts: workgroups (tables) of the scatter pass
    int block0[kProjectedMaxOrder + 1];      // blocks [block0[n], block0[n + 1]) work on mode n,
    int dense[kProjectedMaxOrder];           // the first dense[n] of them on rows [K[n], rows[n]), the others on the table rows
    int K[kProjectedMaxOrder], hot_off[kProjectedMaxOrder], J[kProjectedMaxOrder], R;   // J, R: the caller's
    long long rows[kProjectedMaxOrder], A_off[kProjectedMaxOrder];
    int B_off[kProjectedMaxOrder];
    float* A;
    float* dA;
    const float* B;
    const float* tables;
    float* core;                             // [gridDim.x][core_floats]
    int core_floats;
    float lr_A, lambda_A;
};

#ifndef FTK_TEMPLATE_KERNELS_ONLY
// value of lane `L` of the 16 lanes this one belongs to
template <int L>
__device__ __forceinline__ float row_lane(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x150 + L, 0xf, 0xf, true));
}

// The rows' update: 16 lanes a row, lane j its column j.  Every row of the accumulator is looked at (64 bytes), those that
// were hit are applied and cleared.  A block's share of the core gradient leaves as one table of plain stores.
template <int Q>
__global__ void __launch_bounds__(kApplyProjectedThreads) apply_projected_kernel(ApplyProjectedArgs g) {
    constexpr int WD = projected_width(Q), HOT_ROWS = 256 / WD, WAVES = kApplyProjectedThreads / 64;
    __shared__ float red[4][256];
    __shared__ float part[WAVES][16 * 4 * Q];
    const int tid = threadIdx.x, j = tid & 15, lane = tid & 63, wave = tid >> 6;
    int n = 0;
    while (n + 1 < g.order && (int)blockIdx.x >= g.block0[n + 1]) ++n;
    const int blk = (int)blockIdx.x - g.block0[n], K = g.K[n];
    const bool column = j < g.J[n];
    float Bj[4 * Q], core[4 * Q];
#pragma unroll
    for (int r = 0; r < 4 * Q; ++r) {
        Bj[r] = g.B[g.B_off[n] + j * 16 + r];   // (zeros outside J x R)
        core[r] = 0.0f;
    }
    float* A = g.A + g.A_off[n];
    float* acc = g.dA + g.A_off[n];
    // x: this lane's column of the row's sums; a: its column of the row
    auto moved = [&](float x, float a) {
        float d[4 * Q];
        d[0] = row_lane<0>(x); d[1] = row_lane<1>(x); d[2] = row_lane<2>(x); d[3] = row_lane<3>(x);
        if constexpr (Q == 2) { d[4] = row_lane<4>(x); d[5] = row_lane<5>(x); d[6] = row_lane<6>(x); d[7] = row_lane<7>(x); }
        float grad = g.lambda_A * row_lane<4 * Q>(x) * a;
#pragma unroll
        for (int r = 0; r < 4 * Q; ++r) {
            grad = fmaf(d[r], Bj[r], grad);
            core[r] = fmaf(a, d[r], core[r]);
        }
        return fmaf(-g.lr_A, grad, a);
    };
    if (blk < g.dense[n]) {
        constexpr int U = 4;   // rows in flight per lane
        const long long rows = g.rows[n], step = (long long)g.dense[n] * (64 * U);
        for (long long i0 = K + (long long)blk * (64 * U) + (tid >> 4); i0 - (tid >> 4) < rows; i0 += step) {
            float x[U], a[U];
            bool hit[U];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = i0 + 64 * u < rows ? acc[(i0 + 64 * u) * 16 + j] : 0.0f;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                hit[u] = row_lane<4 * Q>(x[u]) != 0.0f;
                a[u] = hit[u] ? A[(i0 + 64 * u) * 16 + j] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float now = moved(x[u], a[u]);
                if (hit[u]) {
                    if (column) A[(i0 + 64 * u) * 16 + j] = now;
                    acc[(i0 + 64 * u) * 16 + j] = 0.0f;
                }
            }
        }
    } else {
        // table rows: summed over the workgroups' tables first, four threads per element
        const int r0 = (blk - g.dense[n]) * HOT_ROWS, count = min(HOT_ROWS, K - r0);
        const int q = tid & 255, sub = tid >> 8;
        const size_t stride = (size_t)scatter_table_floats(g.H, Q);
        float sum0 = 0.0f, sum1 = 0.0f;
        if (q < count * WD) {
            const float* src = g.tables + (size_t)(g.hot_off[n] + r0) * WD + q;
            int b = sub;
            for (; b + 28 < g.parts; b += 32) {
                float t[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) t[u] = src[(size_t)(b + 4 * u) * stride];
                sum0 += (t[0] + t[2]) + (t[4] + t[6]);
                sum1 += (t[1] + t[3]) + (t[5] + t[7]);
            }
            for (; b < g.parts; b += 4) sum0 += src[(size_t)b * stride];
        }
        red[sub][q] = sum0 + sum1;
        __syncthreads();
        const int i = tid >> 4;
        float x = 0.0f;
        if (i < count && j < WD) {
            const int e = i * WD + j;
            x = (red[0][e] + red[1][e]) + (red[2][e] + red[3][e]);
        }
        const bool hit = row_lane<4 * Q>(x) != 0.0f;
        const long long at = (long long)(r0 + i) * 16 + j;
        const float a = hit ? A[at] : 0.0f;
        const float now = moved(x, a);
        if (hit && column) A[at] = now;
    }
    // the block's share of the core gradient
#pragma unroll
    for (int r = 0; r < 4 * Q; ++r) {
        float sum = core[r] + __shfl_xor(core[r], 16);
        sum += __shfl_xor(sum, 32);
        if (lane < 16) part[wave][j * (4 * Q) + r] = sum;
    }
    __syncthreads();
    for (int q = tid; q < g.J[n] * g.R; q += kApplyProjectedThreads) {
        const int jj = q / g.R, r = q - jj * g.R;
        float sum = 0.0f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) sum += part[w][jj * (4 * Q) + r];
        g.core[(size_t)blockIdx.x * g.core_floats + q] = sum;
    }
}
#endif

}  // namespace ftk

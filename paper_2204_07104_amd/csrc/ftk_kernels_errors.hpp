// Evaluation pass over a set of entries (RMSE / MAE, Section 5.1) by way of the projected rows.
//
// A prediction needs c^(n) = a^(n) B^(n) of its N rows, and a row is needed by many entries: the rows are projected
// once, S^(n) = A^(n) B^(n) (project_rows_kernel, one streaming pass over A), and an entry then only gathers N rows of S
// and multiplies them, x^ = sum_r prod_n S^(n)[i_n, r].  No matrix instruction and no exchange between layouts is left
// per entry; what bounds the pass is the gathering of N rows of 4 R bytes per entry out of the L2 and last-level caches.
// At order 3 with J = R = 16 (1e8 entries) that is 1.2 ns per row and CU, where rows that sit in L2 take 1.0, so rows that
// are short and often asked for are kept in LDS (HOT: 1 430 -> 934 us); what the passes with a projection per entry take
// stands at the dispatch (launch_errors_rows).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ftk_kernels_generic.hpp"

namespace ftk {

constexpr int kProjectRows = 4;      // rows per thread
constexpr int kProjectMaxRank = 64;  // J_n, R

struct ProjectArgs {
    const float* A[kMaxOrder];
    const float* B[kMaxOrder];
    float* S[kMaxOrder];
    long long rows[kMaxOrder];
    int J[kMaxOrder], stride_A[kMaxOrder];
    int block0[kMaxOrder + 1];   // blocks [block0[n], block0[n + 1]) work on mode n
    int order, R, stride_B, Rs;
};

struct ErrorRows {
    const float* S[kMaxOrder];
    int Rs;          // floats per row of S, a multiple of four
    // HOT: rows [0, K[n]) of S, the most frequent ones, are kept in LDS (table row hot0[n] on); bytes[n] is the size of S^(n)
    int K[kMaxOrder], hot0[kMaxOrder], hot_rows;
    unsigned int bytes[kMaxOrder];
};
constexpr int kErrorHotThreads = 1024;
// floats of LDS next to the table: a row of zeros and what the waves park
__host__ __device__ constexpr int error_hot_floats(int order) { return 64 + kErrorHotThreads / 64 * (order + 1) * 64; }

#ifndef FTK_TEMPLATE_KERNELS_ONLY
// S[i][0..Rs) = A[i][:] B for every mode (columns R .. Rs - 1 zero), Rs = R rounded up to four.  A thread makes four columns of
// kProjectRows rows; B sits in LDS.
__global__ void __launch_bounds__(256) project_rows_kernel(ProjectArgs p) {
    __shared__ float4 Bl[kProjectMaxRank * kProjectMaxRank / 4];
    int n = 0;
    while (n + 1 < p.order && (int)blockIdx.x >= p.block0[n + 1]) ++n;
    const float* __restrict__ A = p.A[n];
    const float* __restrict__ B = p.B[n];
    float* __restrict__ S = p.S[n];
    const long long rows = p.rows[n];
    const int J = p.J[n], stride_A = p.stride_A[n], Rs = p.Rs, quads = Rs / 4;
    for (int q = threadIdx.x; q < J * quads; q += 256) {
        const int j = q / quads, r = 4 * (q - j * quads);
        float b[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) b[i] = r + i < p.R ? B[j * p.stride_B + r + i] : 0.0f;
        Bl[q] = make_float4(b[0], b[1], b[2], b[3]);
    }
    __syncthreads();
    const int per_block = 256 / quads, mine = (int)threadIdx.x / quads, quad = (int)threadIdx.x - mine * quads;
    if (mine >= per_block) return;
    const long long step = (long long)(p.block0[n + 1] - p.block0[n]) * per_block * kProjectRows;
    for (long long i0 = ((long long)((int)blockIdx.x - p.block0[n]) * per_block + mine) * kProjectRows; i0 < rows; i0 += step) {
        float4 acc[kProjectRows];
        const float* row[kProjectRows];
#pragma unroll
        for (int u = 0; u < kProjectRows; ++u) {
            acc[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            row[u] = A + (i0 + u < rows ? i0 + u : i0) * stride_A;
        }
        int j = 0;
        for (; j + 4 <= J; j += 4) {
            typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));   // rows start where they may
            floatx4u a[kProjectRows];
#pragma unroll
            for (int u = 0; u < kProjectRows; ++u) a[u] = *reinterpret_cast<const floatx4u*>(row[u] + j);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float4 b = Bl[(j + k) * quads + quad];
#pragma unroll
                for (int u = 0; u < kProjectRows; ++u) {
                    acc[u].x = fmaf(a[u][k], b.x, acc[u].x);
                    acc[u].y = fmaf(a[u][k], b.y, acc[u].y);
                    acc[u].z = fmaf(a[u][k], b.z, acc[u].z);
                    acc[u].w = fmaf(a[u][k], b.w, acc[u].w);
                }
            }
        }
        for (; j < J; ++j) {
            const float4 b = Bl[j * quads + quad];
#pragma unroll
            for (int u = 0; u < kProjectRows; ++u) {
                const float a = row[u][j];
                acc[u].x = fmaf(a, b.x, acc[u].x);
                acc[u].y = fmaf(a, b.y, acc[u].y);
                acc[u].z = fmaf(a, b.z, acc[u].z);
                acc[u].w = fmaf(a, b.w, acc[u].w);
            }
        }
#pragma unroll
        for (int u = 0; u < kProjectRows; ++u)
            if (i0 + u < rows) *reinterpret_cast<float4*>(S + (i0 + u) * Rs + 4 * quad) = acc[u];
    }
}
#endif

// sum over groups of G neighbouring lanes (G a power of two up to 16), in every lane of the group: moves inside a lane row
template <int G>
__device__ __forceinline__ float group_sum(float x) {
    auto add = [](float v, int moved) { return v + __int_as_float(moved); };
    if constexpr (G >= 2) x = add(x, __builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xf, 0xf, true));    // lane ^ 1
    if constexpr (G >= 4) x = add(x, __builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x4E, 0xf, 0xf, true));    // lane ^ 2
    if constexpr (G >= 8) x = add(x, __builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x141, 0xf, 0xf, true));   // the other quad of eight
    if constexpr (G >= 16) x = add(x, __builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x140, 0xf, 0xf, true));  // the other half of sixteen
    return x;
}

// G lanes work on one entry (four columns each, 4 G >= Rs), a wave on 64 / G entries at a time and on 64 in turn; all
// rows of kDepth such turns are asked for before the first is used.
// HOT: one workgroup per CU with the most frequent rows in LDS.  Every row is asked for twice, from LDS and from memory; the
// one that is not meant aims at the row of zeros or past the end of the buffer, where the request is dropped, and the two
// are added.
template <int N, int G, bool HOT>
__global__ void __launch_bounds__(HOT ? kErrorHotThreads : 256) errors_rows_kernel(Coo coo, uint64_t nnz, ErrorRows s, double* __restrict__ sums /* [gridDim.x][2]: sse, sae */) {
    constexpr int W4 = (N + 1 + 3) / 4, E = 64 / G;
    constexpr int kDepth = N * G <= 12 ? G : N <= 3 ? (G < 4 ? G : 4) : N <= 6 ? (G < 2 ? G : 2) : 1;
    constexpr int THREADS = HOT ? kErrorHotThreads : 256, WAVES = THREADS / 64;
    __shared__ int parked_all[HOT ? 1 : WAVES][(N + 1) * 64];   // per wave: [N][64] row numbers | [64] values
    __shared__ double red[2][WAVES];
    extern __shared__ float error_lds[];   // HOT: table [hot_rows][Rs] | 64 zeros | parked_all
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int sub = lane % G, who = lane / G;
    int* parked = HOT ? reinterpret_cast<int*>(error_lds + (size_t)s.hot_rows * s.Rs + 64) + wave * ((N + 1) * 64) : parked_all[HOT ? 0 : wave];
    const float* zeros = error_lds + (size_t)s.hot_rows * s.Rs;
    __amdgpu_buffer_rsrc_t rsrc[N];
    if constexpr (HOT) {
#pragma unroll
        for (int n = 0; n < N; ++n) {
            rsrc[n] = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(s.S[n]), 0, s.bytes[n], 0x00020000);
            const float4* from = reinterpret_cast<const float4*>(s.S[n]);
            float4* to = reinterpret_cast<float4*>(error_lds + (size_t)s.hot0[n] * s.Rs);
            for (int q = tid; q < s.K[n] * (s.Rs / 4); q += THREADS) to[q] = from[q];
        }
        if (tid < 64) error_lds[(size_t)s.hot_rows * s.Rs + tid] = 0.0f;
        __syncthreads();
    }
    const bool column = 4 * sub < s.Rs;
    const int col = column ? 4 * sub : 0;
    const uint4* rec4 = reinterpret_cast<const uint4*>(coo.rec);
    const uint64_t n_groups = (nnz + 63) / 64, stride = (uint64_t)gridDim.x * WAVES;
    double sse = 0.0, sae = 0.0;
    uint4 rec[W4];
    uint64_t group = (uint64_t)blockIdx.x * WAVES + wave;
    auto load = [&](uint64_t g) {
        const uint64_t p = g * 64 + lane;
#pragma unroll
        for (int q = 0; q < W4; ++q) rec[q] = rec4[(p < nnz ? p : 0) * W4 + q];
    };
    if (group < n_groups) load(group);
    for (; group < n_groups; group += stride) {
        uint32_t flat[4 * W4];
#pragma unroll
        for (int q = 0; q < W4; ++q) {
            flat[4 * q + 0] = rec[q].x;
            flat[4 * q + 1] = rec[q].y;
            flat[4 * q + 2] = rec[q].z;
            flat[4 * q + 3] = rec[q].w;
        }
        asm volatile("" ::: "memory");   // lanes of a wave exchange through LDS in program order, no wait needed
#pragma unroll
        for (int n = 0; n <= N; ++n) parked[n * 64 + lane] = (int)flat[n];
        asm volatile("" ::: "memory");
        if (group + stride < n_groups) load(group + stride);
        float kept = 0.0f;   // the prediction of entry number sub * E + who of the group: one per lane
#pragma unroll
        for (int t0 = 0; t0 < G; t0 += kDepth) {
            float4 v[kDepth][N];
#pragma unroll
            for (int u = 0; u < kDepth; ++u)
#pragma unroll
                for (int n = 0; n < N; ++n) {
                    const uint32_t row = (uint32_t)parked[n * 64 + (t0 + u) * E + who];
                    if constexpr (HOT) {
                        typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));
                        const bool hot = row < (uint32_t)s.K[n];
                        const uint32_t at = row * (uint32_t)s.Rs + (uint32_t)col;
                        const uintx4 q = __builtin_amdgcn_raw_buffer_load_b128(rsrc[n], hot ? (int)0xfffffff0u : (int)(at * 4u), 0, 0);
                        const float4 h = *reinterpret_cast<const float4*>(hot ? error_lds + (uint32_t)(s.hot0[n] * s.Rs) + at : zeros);
                        v[u][n] = make_float4(__uint_as_float(q[0]) + h.x, __uint_as_float(q[1]) + h.y, __uint_as_float(q[2]) + h.z,
                                              __uint_as_float(q[3]) + h.w);
                    } else {
                        v[u][n] = *reinterpret_cast<const float4*>(s.S[n] + (uint64_t)row * (uint32_t)s.Rs + col);
                    }
                }
#pragma unroll
            for (int u = 0; u < kDepth; ++u) {
                float4 p = v[u][0];
#pragma unroll
                for (int n = 1; n < N; ++n) {
                    p.x *= v[u][n].x;
                    p.y *= v[u][n].y;
                    p.z *= v[u][n].z;
                    p.w *= v[u][n].w;
                }
                const float xhat = group_sum<G>(column ? (p.x + p.y) + (p.z + p.w) : 0.0f);
                if (sub == t0 + u) kept = xhat;
            }
        }
        const int mine = sub * E + who;
        if (group * 64 + mine < nnz) {
            const double e = (double)__int_as_float(parked[N * 64 + mine]) - (double)kept;
            sse += e * e;
            sae += fabs(e);
        }
    }
    sse = wave_sum(sse);
    sae = wave_sum(sae);
    if (lane == 0) {
        red[0][wave] = sse;
        red[1][wave] = sae;
    }
    __syncthreads();
    if (tid == 0) {
        double a = 0.0, b = 0.0;
        for (int w = 0; w < WAVES; ++w) {
            a += red[0][w];
            b += red[1][w];
        }
        sums[2 * blockIdx.x + 0] = a;
        sums[2 * blockIdx.x + 1] = b;
    }
}

}  // namespace ftk

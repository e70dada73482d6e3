// Synchronous step without atomics on factor rows, in the space of the projections: for tensors whose modes are hit
// evenly, so that nearly every row update would leave the chip as an atomic of its own (20e9 of them per second is what
// the whole chip retires, whatever their size up to 64 bytes, while plain stores go at 90e9).
//
//   S^(n) = A^(n) B^(n)                  projected rows, one streaming pass (project_rows_kernel)
//   v_k^(n) = -e_k w_k^(n)               per sample from N gathered rows of S: products only (append_lists_kernel)
//   D^(n)_i = sum_{i_n(k) = i} v_k^(n),  h_i = number of samples that hit row i
//   A^(n)_i <- A^(n)_i - lr_A ( D^(n)_i (B^(n))^T + lambda_A h_i A^(n)_i )
//   GB^(n)  = sum_i A^(n)_i (x) D^(n)_i  (both contractions per touched row, not per sample: own_rows_kernel)
//
// which is the step of the other kernels with the sums over samples drawn in front of the products with B^(n) and A^(n).
// The rows of every mode are cut into buckets; a workgroup of the first pass keeps one list per bucket and appends v_k and
// the row's number, with plain stores; a workgroup of the second owns a bucket, sums its lists in LDS and updates its rows.
// A list that is full sends its row to the accumulator of the atomic kernels instead, which the owner folds in.
//
// Order 10, J = R = 4, 1e6 samples: 537 us per step with atomics, 244 us this way: 157 us for the appending pass, where 10e6
// entries of 16 bytes at the rate of scattered stores take 110 us, and 92 us for the owners, which read 200 MB (40 us).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ftk_kernels_errors.hpp"
#include "ftk_kernels_mfma16.hpp"

namespace ftk {

constexpr int kOwnersMaxRank = 8;        // R
constexpr int kAppendThreads = 1024, kOwnThreads = 512;
constexpr int kOwnersMaxBuckets = 1024;

struct AppendArgs {
    Coo coo;
    SampleRule rule;
    uint64_t seed;
    long long M;
    const float* S[kMaxOrder];
    int Rs;                                // floats per row of S and per list entry
    unsigned int rows_per_bucket[kMaxOrder], bucket0[kMaxOrder];
    float inv_rows_per_bucket[kMaxOrder];
    unsigned int cap[kMaxOrder];           // places in one workgroup's list of a bucket of mode n
    unsigned int place0[kMaxOrder];        // first place of mode n's lists among the workgroup's places
    unsigned int places;                   // of one workgroup
    int n_buckets;
    float* values;                         // [gridDim.x][places][Rs]
    unsigned short* ids;                   // [gridDim.x][places]: row number inside the bucket
    unsigned int* fill;                    // [n_buckets][gridDim.x]
    // rows whose list is full
    const float* A;
    const float* B;
    float* dA;
    float* GB;
    long long A_off[kMaxOrder];
    int B_off[kMaxOrder], J[kMaxOrder], R, stride_B;
    float lambda_A;
    unsigned int* overflow;
};

// G lanes per sample (four columns each), 64 / G samples per wave at a time.  LDS: cursors [n_buckets] | row numbers [places].
// A workgroup takes one share of Psi; what bounds it is the scattered stores of the entries (one request of 16 G bytes each)
// and the gathering of the rows.
template <int N, int G>
__global__ void __launch_bounds__(kAppendThreads) append_lists_kernel(AppendArgs g) {
    extern __shared__ unsigned int append_lds[];
    constexpr int W4 = (N + 1 + 3) / 4, E = 64 / G, WAVES = kAppendThreads / 64;
    unsigned int* cursor = append_lds;
    unsigned short* id_lds = reinterpret_cast<unsigned short*>(append_lds + g.n_buckets);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, sub = lane % G, who = lane / G;
    for (int q = tid; q < g.n_buckets; q += kAppendThreads) cursor[q] = 0u;
    __syncthreads();
    const bool column = 4 * sub < g.Rs;
    const int col = column ? 4 * sub : 0;
    const uint4* rec4 = reinterpret_cast<const uint4*>(g.coo.rec);
    // A wave takes 64 samples in G turns of E.  Lane l draws the position of the l-th of them, once for all turns.
    const long long groups = (g.M + 63) / 64;
    const long long stride = (long long)gridDim.x * WAVES;
    float* values = g.values + (size_t)blockIdx.x * g.places * g.Rs;
    long long group = (long long)wave * gridDim.x + blockIdx.x;
    uint4 rec[W4];
    uint32_t position = 0u;
    auto draw = [&](long long grp) {
        const long long k = grp * 64 + lane;
        position = k < g.M ? sample_place(g.seed, (uint64_t)k, g.rule) : 0u;
    };
    auto load = [&](int turn) {
        const uint32_t p = G == 1 ? position : (uint32_t)__shfl((int)position, turn * E + who);
#pragma unroll
        for (int q = 0; q < W4; ++q) rec[q] = rec4[(size_t)p * W4 + q];
    };
    if (group < groups) {
        draw(group);
        load(0);
    }
    int turn = 0;
    while (group < groups) {
        const bool act = group * 64 + turn * E + who < g.M;
        uint32_t flat[4 * W4];
#pragma unroll
        for (int q = 0; q < W4; ++q) {
            flat[4 * q + 0] = rec[q].x;
            flat[4 * q + 1] = rec[q].y;
            flat[4 * q + 2] = rec[q].z;
            flat[4 * q + 3] = rec[q].w;
        }
        float4 c[N];
#pragma unroll
        for (int n = 0; n < N; ++n) c[n] = *reinterpret_cast<const float4*>(g.S[n] + (uint64_t)flat[n] * (uint32_t)g.Rs + col);
        // the places in the lists while the rows are on their way
        unsigned int place[N], in_bucket[N];
#pragma unroll
        for (int n = 0; n < N; ++n) {
            // row / rows_per_bucket: rows stay below 2^24, where the float quotient is off by one at most
            const unsigned int row = flat[n];
            unsigned int b = (unsigned int)((float)row * g.inv_rows_per_bucket[n]);
            unsigned int rest = row - b * g.rows_per_bucket[n];
            if ((int)rest < 0) { b -= 1u; rest += g.rows_per_bucket[n]; }
            if (rest >= g.rows_per_bucket[n]) { b += 1u; rest -= g.rows_per_bucket[n]; }
            in_bucket[n] = rest;
            unsigned int p = 0u;
            if (act && sub == 0) p = atomicAdd(cursor + g.bucket0[n] + b, 1u);
            if constexpr (G == 2) p = (unsigned int)__builtin_amdgcn_update_dpp(0, (int)p, 0xA0, 0xf, 0xf, true);   // lanes 0, 0, 2, 2 of a quad
            place[n] = p < g.cap[n] ? g.place0[n] + b * g.cap[n] + p : 0xffffffffu;
        }
        // the next turn's records
        turn += 1;
        if (turn == G) {
            turn = 0;
            group += stride;
            if (group < groups) draw(group);
        }
        if (group < groups) load(turn);
        const float x = __uint_as_float(flat[N]);
        // leave-one-out products by a prefix and a suffix sweep
        float4 w[N], run = make_float4(1.0f, 1.0f, 1.0f, 1.0f);
        auto times = [](float4 a, const float4& b) { return make_float4(a.x * b.x, a.y * b.y, a.z * b.z, a.w * b.w); };
#pragma unroll
        for (int n = 0; n < N; ++n) {
            w[n] = run;
            run = times(run, c[n]);
        }
        const float minus_e = group_sum<G>(column ? (run.x + run.y) + (run.z + run.w) : 0.0f) - x;
        run = make_float4(minus_e, minus_e, minus_e, minus_e);
#pragma unroll
        for (int n = N - 1; n >= 0; --n) {
            w[n] = times(w[n], run);
            run = times(run, c[n]);
        }
        bool full = false;
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const bool fits = act && place[n] != 0xffffffffu;
            full = full || (act && !fits);
            if (fits && column) *reinterpret_cast<float4*>(values + (size_t)place[n] * g.Rs + col) = w[n];
            if (fits && sub == 0) id_lds[place[n]] = (unsigned short)in_bucket[n];
        }
        if (full) {   // rare: this row's share of the step goes through atomics
#pragma unroll 1
            for (int n = 0; n < N; ++n) {
                if (place[n] != 0xffffffffu) continue;
                if (sub == 0) atomicAdd(g.overflow, 1u);
                float4 v = w[0];
                uint32_t row = flat[0];
#pragma unroll
                for (int m = 1; m < N; ++m)
                    if (m == n) {
                        v = w[m];
                        row = flat[m];
                    }
                const float vr[4] = {v.x, v.y, v.z, v.w};
                const float* a = g.A + g.A_off[n] + (long long)row * g.J[n];
                float* d = g.dA + g.A_off[n] + (long long)row * g.J[n];
                for (int j = 0; j < g.J[n]; ++j) {
                    float sum = sub == 0 ? g.lambda_A * a[j] : 0.0f;
                    for (int i = 0; i < 4; ++i)
                        if (column && col + i < g.R) {
                            sum = fmaf(vr[i], g.B[g.B_off[n] + j * g.stride_B + col + i], sum);
                            atomicAdd(g.GB + g.B_off[n] + j * g.stride_B + col + i, a[j] * vr[i]);
                        }
                    atomicAdd(d + j, sum);
                }
            }
        }
    }
    __syncthreads();
    unsigned short* ids = g.ids + (size_t)blockIdx.x * g.places;
    for (unsigned int q = tid; q < g.places / 2; q += kAppendThreads)   // (places is even)
        reinterpret_cast<unsigned int*>(ids)[q] = reinterpret_cast<const unsigned int*>(id_lds)[q];
#pragma unroll
    for (int n = 0; n < N; ++n) {
        const unsigned int end = n + 1 < N ? g.bucket0[n + 1 < N ? n + 1 : n] : (unsigned int)g.n_buckets;
        for (unsigned int b = g.bucket0[n] + tid; b < end; b += kAppendThreads)
            g.fill[(size_t)b * gridDim.x + blockIdx.x] = min(cursor[b], g.cap[n]);
    }
}

struct OwnArgs {
    const float* values;
    const unsigned short* ids;
    const unsigned int* fill;
    int order, Rs, R, stride_B, lists;          // lists: workgroups of the appending launch
    unsigned int rows_per_bucket[kMaxOrder], bucket0[kMaxOrder + 1], cap[kMaxOrder], place0[kMaxOrder], places;
    long long rows[kMaxOrder], A_off[kMaxOrder];
    int B_off[kMaxOrder], J[kMaxOrder], J_user[kMaxOrder];
    float* A;
    float* dA;
    const float* B;
    float* core;                                // [n_buckets][core_floats]: sums of a (x) D of the bucket's rows
    int core_floats;
    const unsigned int* overflow;
    float lr_A, lambda_A;
};

// One workgroup per bucket.  LDS: D [rows][Rs] | h [rows] (as counters) | fill [lists]; core gradient sums [threads][Rs] in the
// place of D at the end.  Entries are added by compare-and-swap on pairs of floats (the native LDS float add takes 3 clocks
// per lane).
template <int G>
__global__ void __launch_bounds__(kOwnThreads) own_rows_kernel(OwnArgs g);

#ifndef FTK_TEMPLATE_KERNELS_ONLY
// Four floats added in LDS by compare-and-swap on pairs, both pairs' swaps under way at a time.
__device__ __forceinline__ void add_four(float* cell, const float4& x) {
    unsigned long long* p = reinterpret_cast<unsigned long long*>(cell);
    auto plus = [](unsigned long long old, float a, float b) {
        return (unsigned long long)__float_as_uint(__uint_as_float((unsigned int)(old >> 32)) + b) << 32 |
               __float_as_uint(__uint_as_float((unsigned int)old) + a);
    };
    unsigned long long want0 = p[0], want1 = p[1];
    bool again0 = true, again1 = true;
    do {
        unsigned long long got0 = want0, got1 = want1;
        if (again0) got0 = atomicCAS(p, want0, plus(want0, x.x, x.y));
        if (again1) got1 = atomicCAS(p + 1, want1, plus(want1, x.z, x.w));
        again0 = again0 && got0 != want0;
        again1 = again1 && got1 != want1;
        want0 = got0;
        want1 = got1;
    } while (again0 || again1);
}

template <int G>
__global__ void __launch_bounds__(kOwnThreads) own_rows_kernel(OwnArgs g) {
    extern __shared__ float own_lds[];
    constexpr int E = 64 / G, WAVES = kOwnThreads / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, sub = lane % G, who = lane / G;
    const int b = (int)blockIdx.x;
    int n = 0;
    while (n + 1 < g.order && b >= (int)g.bucket0[n + 1]) ++n;
    const unsigned int in_mode = (unsigned int)b - g.bucket0[n];
    const long long row0 = (long long)in_mode * g.rows_per_bucket[n];
    const int rows = (int)min((long long)g.rows_per_bucket[n], g.rows[n] - row0), Rs = g.Rs;
    float* D = own_lds;
    unsigned int* hits = reinterpret_cast<unsigned int*>(own_lds + (size_t)g.rows_per_bucket[n] * Rs);
    unsigned int* fill = hits + g.rows_per_bucket[n];
    for (int q = tid; q < rows * Rs; q += kOwnThreads) D[q] = 0.0f;
    for (int q = tid; q < rows; q += kOwnThreads) hits[q] = 0u;
    for (int q = tid; q < g.lists; q += kOwnThreads) fill[q] = g.fill[(size_t)b * g.lists + q];
    __syncthreads();
    const bool column = 4 * sub < Rs;
    const int col = column ? 4 * sub : 0;
    const size_t first = g.place0[n] + (size_t)in_mode * g.cap[n];
    // Work items: the pieces of E places of every list, dealt to the waves list by list; the next kAhead of them are on
    // their way while the last ones are added.
    constexpr int kAhead = 4;
    const int pieces = ((int)g.cap[n] + E - 1) / E, items = g.lists * pieces;
    const float per_list = 1.0f / (float)pieces;
    float4 x[kAhead];
    unsigned int row[kAhead];
    auto ask = [&](int item0) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int item = item0 + u * WAVES;
            const int list = (int)(((float)item + 0.5f) * per_list);   // item / pieces: both stay far below 2^20
            const int e = (item - list * pieces) * E + who;
            const bool there = item < items && e < (int)fill[list < g.lists ? list : 0];
            const size_t at = (size_t)list * g.places + first + e;
            row[u] = there ? g.ids[at] : 0xffffffffu;
            x[u] = there ? *reinterpret_cast<const float4*>(g.values + at * Rs + col) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
    };
    ask(wave);
    for (int item0 = wave; item0 < items; item0 += kAhead * WAVES) {
        float4 y[kAhead];
        unsigned int to[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            y[u] = x[u];
            to[u] = row[u];
        }
        ask(item0 + kAhead * WAVES);
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            if (to[u] != 0xffffffffu) {
                if (column) add_four(D + (size_t)to[u] * Rs + col, y[u]);
                if (sub == 0) atomicAdd(hits + to[u], 1u);
            }
    }
    __syncthreads();
    // rows: thread (group of rows, j) holds row j of B and its sums of the core gradient
    const int J = g.J_user[n];
    int Jp = 1;
    while (Jp < J) Jp *= 2;   // at most 64
    const int j = tid % Jp;
    float Bj[kOwnersMaxRank], core[kOwnersMaxRank];
#pragma unroll
    for (int r = 0; r < kOwnersMaxRank; ++r) {
        Bj[r] = (j < J && r < g.R) ? g.B[g.B_off[n] + j * g.stride_B + r] : 0.0f;
        core[r] = 0.0f;
    }
    const bool spilled = *g.overflow != 0u;
    if (j < J)
        for (int i = tid / Jp; i < rows; i += kOwnThreads / Jp) {
            const unsigned int h = hits[i];
            const long long off = g.A_off[n] + (row0 + i) * g.J[n] + j;
            float grad = 0.0f;
            if (h != 0u || spilled) {
                const float a = g.A[off];
#pragma unroll
                for (int q = 0; q < kOwnersMaxRank / 4; ++q)
                    if (4 * q < Rs) {
                        const float4 d = *reinterpret_cast<const float4*>(D + (size_t)i * Rs + 4 * q);
                        const float dr[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            grad = fmaf(dr[u], Bj[4 * q + u], grad);
                            core[4 * q + u] = fmaf(a, dr[u], core[4 * q + u]);
                        }
                    }
                grad = fmaf(g.lambda_A * (float)h, a, grad);
                if (spilled) {
                    grad += g.dA[off];
                    g.dA[off] = 0.0f;
                }
                g.A[off] = fmaf(-g.lr_A, grad, a);
            }
        }
    __syncthreads();
    float* part = own_lds;   // [threads][Rs]
#pragma unroll
    for (int r = 0; r < kOwnersMaxRank; ++r)
        if (r < Rs) part[tid * Rs + r] = core[r];
    __syncthreads();
    float* out = g.core + (size_t)b * g.core_floats;
    for (int q = tid; q < J * g.R; q += kOwnThreads) {
        const int jj = q / g.R, r = q - jj * g.R;
        float sum = 0.0f;
        for (int t = jj; t < kOwnThreads; t += Jp) sum += part[t * Rs + r];
        out[q] = sum;
    }
}

struct FinishArgs {
    const float* core;          // [n_buckets][core_floats]
    int core_floats, order, R, stride_B;
    unsigned int bucket0[kMaxOrder + 1];
    int B_off[kMaxOrder], J[kMaxOrder];
    float* B;
    float* GB;                  // what went through atomics
    unsigned int* overflow;     // [2]: of this step, of all before it
    float lr_B, lambda_B, inv_M;
};
// B <- B - lr_B (GB / M + lambda_B B): one workgroup per mode and 64 elements, four threads per element over the buckets
__global__ void __launch_bounds__(256) finish_core_kernel(FinishArgs g, int blocks_per_mode) {
    __shared__ float red[4][64];
    const int n = (int)blockIdx.x / blocks_per_mode, q = ((int)blockIdx.x - n * blocks_per_mode) * 64 + ((int)threadIdx.x & 63), part = (int)threadIdx.x >> 6;
    const int count = g.J[n] * g.R;
    float sum = 0.0f;
    if (q < count) {
        // eight loads in flight: a mode has up to some hundred buckets
        const float* src = g.core + q;
        unsigned int b = g.bucket0[n] + part;
        const unsigned int end = g.bucket0[n + 1];
        for (; b + 28 < end; b += 32) {
            float t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = src[(size_t)(b + 4 * u) * g.core_floats];
            sum += ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
        }
        for (; b < end; b += 4) sum += src[(size_t)b * g.core_floats];
    }
    red[part][threadIdx.x & 63] = sum;
    __syncthreads();
    if (part == 0 && q < count) {
        const int jj = q / g.R, r = q - jj * g.R, l = (int)threadIdx.x;
        float* gb = g.GB + g.B_off[n] + jj * g.stride_B + r;
        const float total = ((red[0][l] + red[1][l]) + (red[2][l] + red[3][l])) + *gb;
        *gb = 0.0f;
        float* b = g.B + g.B_off[n] + jj * g.stride_B + r;
        *b = *b - g.lr_B * fmaf(total, g.inv_M, g.lambda_B * *b);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        g.overflow[1] += g.overflow[0];
        g.overflow[0] = 0u;
    }
}
#endif

}  // namespace ftk

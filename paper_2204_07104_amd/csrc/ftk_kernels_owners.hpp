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
// Order 10, J = R = 4, 1e6 samples: 537 us per step with atomics, 186 us this way: 118 us for the appending pass and 58 us for
// the owners, which read 200 MB (40 us).
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

// A meeting of the workgroup's waves over what they have in LDS.  Unlike __syncthreads it waits for LDS only, so that records and
// rows asked for and entries on their way out stay under way.
__device__ __forceinline__ void lds_meet() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Words of LDS: [4][n_buckets] counts of the round, filled places, place of a bucket in the round, the same against its list |
// for every thread and mode the staged entry (four floats) and, per sample and mode, the entry's bucket and row.
__host__ __device__ inline int append_bucket_words(int n_buckets) { return 4 * ((n_buckets + 3) / 4 * 4); }
// Samples a thread takes in a round: at low orders a round of one each holds too few entries of a bucket to leave side by side.
// Whole steps with one -> four, order 2, R = 8, 2e6 samples 224 -> 180 us; with one -> two, 1e6 samples: order 3, 60 000 rows a mode R = 4
// 109 -> 98, R = 8 153 -> 134 (180 000 rows 134 -> 123, 183 -> 167); order 4, 40 000 rows 133 -> 123, 174 -> 172, 10 000 rows 115 -> 107, but R = 8
// 155 -> 160; 3e5 samples the same either way.  (Order 3 with three: R = 8 157.)
__host__ __device__ constexpr int append_samples(int order) { return order <= 2 ? 4 : order <= 4 ? 2 : 1; }
__host__ __device__ constexpr int append_wave_words(int order, int G) { return append_samples(order) * order * (64 * 4 + 64 / G); }
// from order 8 on a wave needs more than the 128 registers that 16 waves leave it: 161 at order 8, R <= 8, 157 and 168 (16 more spilled) at
// order 10, where 12 waves leave 168.  (Order 8, R <= 4 gets by with 127.)
__host__ __device__ constexpr int append_max_waves(int order) { return order < 8 ? kAppendThreads / 64 : 12; }

// A workgroup takes one share of Psi in rounds of append_samples(N) samples per G threads (four columns each).  The entries of a round are put in
// the order of their buckets in LDS first: an entry's place is counted by an atomic that returns it, one wave per mode adds the
// counts up, and entries of one list then leave side by side (order 10, J = R = 4: some 15 of 16 bytes), in far fewer requests
// than when each is stored where it belongs, which bound the launch before.  What bounds it now is the gathering of the rows (10e6 of
// 16 bytes, 40 us at 1 ns a row and CU), the records, and what a round does in turn between its three meetings.
// Launch for 1e6 samples of order 10, J = R = 4: 152 -> 118 us.  Whole steps of 1e6 samples: order 10 R = 4 247 -> 211, R = 8 371 -> 346; order 7 R = 8
// 277 -> 258; order 6 R = 4 193 -> 150; order 4 R = 4 168 -> 127; order 3 R = 8 165 -> 153; order 2 R = 8 135 -> 113.
template <int N, int G>
__global__ void __launch_bounds__(append_max_waves(N) * 64) append_lists_kernel(AppendArgs g) {
    extern __shared__ __align__(16) unsigned int append_lds[];
    constexpr int W4 = (N + 1 + 3) / 4, U = append_samples(N);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), sub = tid % G, who = tid / G;
    const int threads = (int)blockDim.x, waves = threads >> 6, turn = threads / G, S = turn * U;   // S: samples of a round
    const int nb4 = append_bucket_words(g.n_buckets) / 4;
    unsigned int* count = append_lds;
    unsigned int* filled = count + nb4;
    unsigned int* base = filled + nb4;     // first staged entry of the bucket in this round
    unsigned int* start = base + nb4;      // place in the bucket's list = start + staged place
    float4* staged = reinterpret_cast<float4*>(append_lds + 4 * nb4);                          // [N][S][G]
    unsigned int* tag = reinterpret_cast<unsigned int*>(staged + (size_t)N * U * threads);         // [N][S]: bucket << 16 | row in it
    for (int q = tid; q < 2 * nb4; q += threads) append_lds[q] = 0u;   // counts and filled places
    const bool column = 4 * sub < g.Rs;
    const int col = column ? 4 * sub : 0;
    const uint4* rec4 = reinterpret_cast<const uint4*>(g.coo.rec);
    float* values = g.values + (size_t)blockIdx.x * g.places * g.Rs;
    unsigned short* ids = g.ids + (size_t)blockIdx.x * g.places;
    // the workgroup's share: groups of 64 samples, dealt evenly
    const long long groups = (g.M + 63) / 64, each = groups / gridDim.x, more = groups % gridDim.x, b0 = blockIdx.x;
    const long long first = 64 * (b0 * each + (b0 < more ? b0 : more));
    const long long end = min(g.M, first + 64 * (each + (b0 < more ? 1 : 0)));
    uint4 rec[U][W4];
    auto load = [&](long long from) {   // records of this thread's samples of the round that starts at `from`
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const long long k = from + u * turn + who;
            const uint32_t p = k < end ? sample_place(g.seed, (uint64_t)k, g.rule) : 0u;
#pragma unroll
            for (int q = 0; q < W4; ++q) rec[u][q] = rec4[(size_t)p * W4 + q];
        }
    };
    uint32_t flat[U][4 * W4];
    float4 c[U][N];
    auto gather = [&]() {
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int q = 0; q < W4; ++q) {
                flat[u][4 * q + 0] = rec[u][q].x;
                flat[u][4 * q + 1] = rec[u][q].y;
                flat[u][4 * q + 2] = rec[u][q].z;
                flat[u][4 * q + 3] = rec[u][q].w;
            }
#pragma unroll
            for (int n = 0; n < N; ++n) c[u][n] = *reinterpret_cast<const float4*>(g.S[n] + (uint64_t)flat[u][n] * (uint32_t)g.Rs + col);
        }
    };
    if (first < end) {
        load(first);
        gather();
    }
    __syncthreads();
    for (long long s0 = first; s0 < end; s0 += S) {
        const int here = (int)min((long long)S, end - s0);   // samples of this round
        auto act = [&](int u) { return u * turn + who < here; };
        // the entries' places in their buckets while the rows are on their way
        unsigned int place[U][N], where[U][N];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
        for (int n = 0; n < N; ++n) {
            // row / rows_per_bucket: rows stay below 2^24, where the float quotient is off by one at most
            const unsigned int row = flat[u][n];
            unsigned int b = (unsigned int)((float)row * g.inv_rows_per_bucket[n]);
            unsigned int rest = row - b * g.rows_per_bucket[n];
            if ((int)rest < 0) { b -= 1u; rest += g.rows_per_bucket[n]; }
            if (rest >= g.rows_per_bucket[n]) { b += 1u; rest -= g.rows_per_bucket[n]; }
            b += g.bucket0[n];
            where[u][n] = b << 16 | rest;
            unsigned int p = 0u;
            if (act(u) && sub == 0) p = atomicAdd(count + b, 1u);
            if constexpr (G == 2) p = (unsigned int)__builtin_amdgcn_update_dpp(0, (int)p, 0xA0, 0xf, 0xf, true);   // lanes 0, 0, 2, 2 of a quad
            place[u][n] = p;
        }
        float x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = __uint_as_float(flat[u][N]);
        load(s0 + S);   // the next round's records
        // leave-one-out products by a prefix and a suffix sweep
        float4 w[U][N];
        auto times = [](float4 a, const float4& b) { return make_float4(a.x * b.x, a.y * b.y, a.z * b.z, a.w * b.w); };
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float4 run = make_float4(1.0f, 1.0f, 1.0f, 1.0f);
#pragma unroll
            for (int n = 0; n < N; ++n) {
                w[u][n] = run;
                run = times(run, c[u][n]);
            }
            const float minus_e = group_sum<G>(column ? (run.x + run.y) + (run.z + run.w) : 0.0f) - x[u];
            run = make_float4(minus_e, minus_e, minus_e, minus_e);
#pragma unroll
            for (int n = N - 1; n >= 0; --n) {
                w[u][n] = times(w[u][n], run);
                run = times(run, c[u][n]);
            }
        }
        lds_meet();   // all counted; the round before has left
        // a wave per mode: where its buckets' entries start in the round (a mode has `here` of them)
        for (int n = wave; n < N; n += waves) {
            const unsigned int last = n + 1 < N ? g.bucket0[n + 1 < N ? n + 1 : n] : (unsigned int)g.n_buckets;
            unsigned int before = (unsigned int)(n * S);
            for (unsigned int b = g.bucket0[n]; b < last; b += 64) {
                const bool mine = b + lane < last;
                const unsigned int cnt = mine ? count[b + lane] : 0u;
                unsigned int sum = cnt;
#pragma unroll
                for (int d = 1; d < 64; d *= 2) {
                    const unsigned int up = (unsigned int)__shfl_up((int)sum, d);
                    sum += lane >= d ? up : 0u;
                }
                if (mine) {
                    const unsigned int f = filled[b + lane], at = before + sum - cnt;
                    base[b + lane] = at;
                    start[b + lane] = f - at;
                    filled[b + lane] = f + cnt;
                    count[b + lane] = 0u;
                }
                before += (unsigned int)__builtin_amdgcn_readlane((int)sum, 63);
            }
        }
        lds_meet();
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (act(u)) {
#pragma unroll
                for (int n = 0; n < N; ++n) {
                    const unsigned int at = base[where[u][n] >> 16] + place[u][n];
                    staged[at * G + sub] = w[u][n];
                    if (sub == 0) tag[at] = where[u][n];
                }
            }
        gather();   // the next round's rows
        lds_meet();
        // out: a thread takes the staged entries `who`, `who` + turn ... of every mode
        unsigned int full = 0u;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (!act(u)) continue;
#pragma unroll
            for (int n = 0; n < N; ++n) {
                const unsigned int at = (unsigned int)(n * S + u * turn + who), t = tag[at], p = start[t >> 16] + at;
                if (p < g.cap[n]) {
                    const size_t to = g.place0[n] + ((t >> 16) - g.bucket0[n]) * g.cap[n] + p;
                    if (column) *reinterpret_cast<float4*>(values + to * g.Rs + col) = staged[at * G + sub];
                    if (sub == 0) ids[to] = (unsigned short)t;
                } else {
                    full |= 1u << (u * N + n);
                }
            }
        }
        if (full != 0u) {   // rare: no room in the list, this row's share of the step goes through atomics
#pragma unroll 1
            for (int un = 0; un < U * N; ++un) {
                if (!(full >> un & 1u)) continue;
                const int n = un % N;
                const unsigned int at = (unsigned int)(n * S + un / N * turn + who), t = tag[at];
                const long long row = (long long)((t >> 16) - g.bucket0[n]) * g.rows_per_bucket[n] + (t & 0xffffu);
                if (sub == 0) atomicAdd(g.overflow, 1u);
                const float4 v = staged[at * G + sub];
                const float vr[4] = {v.x, v.y, v.z, v.w};
                const float* a = g.A + g.A_off[n] + row * g.J[n];
                float* d = g.dA + g.A_off[n] + row * g.J[n];
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
#pragma unroll
    for (int n = 0; n < N; ++n) {
        const unsigned int last = n + 1 < N ? g.bucket0[n + 1 < N ? n + 1 : n] : (unsigned int)g.n_buckets;
        for (unsigned int b = g.bucket0[n] + tid; b < last; b += threads)
            g.fill[(size_t)b * gridDim.x + blockIdx.x] = min(filled[b], g.cap[n]);
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

// One workgroup per bucket.  LDS: D [rows][Rs] | (a chunk's entries) | h [rows] (as counters) | (counts and places of the chunk
// [2][rows]) | fill [lists]; core gradient sums [threads][Rs] in the place of D at the end.
// How entries are added: where a bucket has many rows, by compare-and-swap on pairs of floats (the native LDS float add takes 3 clocks
// per lane).  Where it has few (SORT), the lanes of a wave meet on them and repeat their swaps: there a chunk of entries is put in the order of
// its rows in LDS, by an atomic that counts an entry's place in its row, and threads that own a row add its entries up in
// registers.  Order 10, J = R = 4, 1e6 samples, 196 rows a bucket: 85 -> 58 us.  Whole steps with 100 / 150 / 200 / 235 / 300 / 400 rows in a bucket:
//   order 5, R = 4, 5e5      swaps 85 / 83 / 83 / 83 / 83 / 84        order 72 / 75 / 79 / 79 / 82 / 88
//   order 4, R = 4, 1e6            126 / 123 / 122 / 122 / 122 / 125        107 / 112 / 116 / 118 / 123 / 133
//   order 10, R = 4, 5e5           132 / 128 / 128 / 127 / 129 / 129        110 / 115 / 120 / 119 / 126 / 136
//   order 7, R = 8, 5e5            137 / 136 / 135 / 136 / 137 / 143        123 / 131 / 133 / 134 / 142 / 154
//   order 3, R = 8, 1e6            126 / 127 / 127 / 128 / 131 / 136        115 / 122 / 127 / 128 / 137 / 150
//   order 4, R = 8, 1e6            162 / 164 / 168 / 170 / 172 / 179        156 / 167 / 175 / 177 / 187 / 203
// The two meet at 300 rows for R <= 4 and between 120 and 250 for R <= 8; the line lies at 200 for both.
constexpr int kOwnSortRows = 200, kOwnSortPieces = 6;   // most rows of a bucket; pieces of 64 / G entries a wave brings to a chunk
__host__ __device__ constexpr int own_sort_floats() { return kOwnSortPieces * kOwnThreads * 4; }
template <int G, bool SORT>
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

template <int G, bool SORT>
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
    float4* staged = reinterpret_cast<float4*>(own_lds + (size_t)g.rows_per_bucket[n] * Rs);
    unsigned int* hits = reinterpret_cast<unsigned int*>(own_lds + (size_t)g.rows_per_bucket[n] * Rs + (SORT ? own_sort_floats() : 0));
    unsigned int* count = hits + g.rows_per_bucket[n];    // SORT: entries of the chunk per row
    unsigned int* base = count + g.rows_per_bucket[n];    // SORT: the first of them
    unsigned int* fill = SORT ? base + g.rows_per_bucket[n] : count;
    if constexpr (SORT) {   // (D and h are stored once all entries are in)
        for (int q = tid; q < rows; q += kOwnThreads) count[q] = 0u;
    } else {
        for (int q = tid; q < rows * Rs; q += kOwnThreads) D[q] = 0.0f;
        for (int q = tid; q < rows; q += kOwnThreads) hits[q] = 0u;
    }
    for (int q = tid; q < g.lists; q += kOwnThreads) fill[q] = g.fill[(size_t)b * g.lists + q];
    __syncthreads();
    const bool column = 4 * sub < Rs;
    const int col = column ? 4 * sub : 0;
    const size_t first = g.place0[n] + (size_t)in_mode * g.cap[n];
    // Work items: the pieces of E places of every list, dealt to the waves list by list; the next kAhead of them are on
    // their way while the last ones are added.
    constexpr int kAhead = SORT ? kOwnSortPieces : 4;
    const int pieces = ((int)g.cap[n] + E - 1) / E, items = g.lists * pieces;
    const float per_list = 1.0f / (float)pieces;
    float4 x[kAhead];
    unsigned int row[kAhead];
    auto ask = [&](int item0) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int item = item0 + u * WAVES;
            const int list = (int)(((float)item + 0.5f) * per_list);   // item / pieces: exact below 2^21 items, of which the plan leaves 2^18
            const int e = (item - list * pieces) * E + who;
            const bool there = item < items && e < (int)fill[list < g.lists ? list : 0];
            const size_t at = (size_t)list * g.places + first + e;
            row[u] = there ? g.ids[at] : 0xffffffffu;
            x[u] = there ? *reinterpret_cast<const float4*>(g.values + at * Rs + col) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
    };
    ask(wave);
    if constexpr (SORT) {
        // `team` threads per row and column piece, next to each other: row tid / (team G)
        int team = 1;
        while (2 * team * G * rows <= kOwnThreads && 2 * team * G <= 64) team *= 2;
        const int width = team * G, at_once = kOwnThreads / width, my_part = tid % width / G;
        constexpr int kRowsOfThread = (kOwnSortRows * G + kOwnThreads - 1) / kOwnThreads;
        float4 acc[kRowsOfThread];
        unsigned int my_hits[kRowsOfThread];
#pragma unroll
        for (int v = 0; v < kRowsOfThread; ++v) {
            acc[v] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            my_hits[v] = 0u;
        }
        for (int chunk = 0; chunk < items; chunk += kAhead * WAVES) {   // the same number of chunks for every wave
            float4 y[kAhead];
            unsigned int to[kAhead], rank[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                y[u] = x[u];
                to[u] = row[u];
                unsigned int r = 0u;
                if (to[u] != 0xffffffffu && sub == 0) r = atomicAdd(count + to[u], 1u);
                if constexpr (G == 2) r = (unsigned int)__builtin_amdgcn_update_dpp(0, (int)r, 0xA0, 0xf, 0xf, true);   // lanes 0, 0, 2, 2 of a quad
                rank[u] = r;
            }
            ask(chunk + kAhead * WAVES + wave);
            lds_meet();   // all counted
            if (wave == 0) {
                unsigned int before = 0u;
                for (int r0 = 0; r0 < rows; r0 += 64) {
                    const bool mine = r0 + lane < rows;
                    const unsigned int cnt = mine ? count[r0 + lane] : 0u;
                    unsigned int sum = cnt;
#pragma unroll
                    for (int d = 1; d < 64; d *= 2) {
                        const unsigned int up = (unsigned int)__shfl_up((int)sum, d);
                        sum += lane >= d ? up : 0u;
                    }
                    if (mine) base[r0 + lane] = before + sum - cnt;
                    before += (unsigned int)__builtin_amdgcn_readlane((int)sum, 63);
                }
            }
            lds_meet();
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
                if (to[u] != 0xffffffffu) staged[(base[to[u]] + rank[u]) * G + sub] = y[u];
            lds_meet();
#pragma unroll
            for (int v = 0; v < kRowsOfThread; ++v) {
                const int i = v * at_once + tid / width;
                if (i < rows) {
                    const unsigned int cnt = count[i], b0 = base[i];
                    for (unsigned int k = my_part; k < cnt; k += team) {
                        const float4 t = staged[(b0 + k) * G + sub];
                        acc[v] = make_float4(acc[v].x + t.x, acc[v].y + t.y, acc[v].z + t.z, acc[v].w + t.w);
                    }
                    my_hits[v] += cnt;
                    if (tid % width == 0) count[i] = 0u;   // (the threads of a row are one wave's: they have read it)
                }
            }
            lds_meet();   // the next chunk may be counted and staged
        }
#pragma unroll
        for (int v = 0; v < kRowsOfThread; ++v) {
            for (int d = G; d < width; d *= 2) {
                acc[v].x += __shfl_xor(acc[v].x, d);
                acc[v].y += __shfl_xor(acc[v].y, d);
                acc[v].z += __shfl_xor(acc[v].z, d);
                acc[v].w += __shfl_xor(acc[v].w, d);
            }
            const int i = v * at_once + tid / width;
            if (i < rows && my_part == 0) {
                if (column) *reinterpret_cast<float4*>(D + (size_t)i * Rs + col) = acc[v];
                if (sub == 0) hits[i] = my_hits[v];
            }
        }
    } else {
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

// Low-rank update of projections (adapters): the work of one block, shared by the launch of its own and by the
// few-row GEMM launches that carry it as extra blocks.
#pragma once
#include "sd_internal.h"

// Block (row, projection, part of lora_part(WAVES) outputs).  Bound: latency - a row reads 2 * rank * (K + N) floats of factors
// per projection (49 KB at rank 8, width 768) and multiplies each once - so the block is laid out to have everything in
// flight at once: the rows of B that its threads will need go out first, then wave w takes the dot products
// w, w + WAVES, ... with A, row of X and row of A straight into registers, and one barrier later every thread
// finishes its outputs from registers.  A grid dimension per projection puts three times the blocks on the chip.
// RQ = rank / 4 reads the rows of B (rank contiguous floats) as 16-byte vectors; 0 takes any rank, element by element; -1
// finds out (one instance for every rank: what a GEMM launch carries).
#define LORA_MAX_RANK 16
#define LORA_MAX_K 8192
#define LORA_WAVES 8 // of a launch of its own
constexpr int lora_out(int waves) { return waves == 8 ? 2 : 3; } // outputs per thread
constexpr int lora_part(int waves) { return lora_out(waves) * waves * 64; }

__device__ __forceinline__ float4 load_act4(const float *b, size_t i, size_t) { return *(const float4 *)(b + i); }
__device__ __forceinline__ float4 load_act4(const bf16_t *b, size_t i, size_t plane)
{
    const uint2 h = *(const uint2 *)(b + i), l = *(const uint2 *)(b + i + plane);
    return make_float4(__uint_as_float(h.x << 16) + __uint_as_float(l.x << 16),
                       __uint_as_float(h.x & 0xffff0000u) + __uint_as_float(l.x & 0xffff0000u),
                       __uint_as_float(h.y << 16) + __uint_as_float(l.y << 16),
                       __uint_as_float(h.y & 0xffff0000u) + __uint_as_float(l.y & 0xffff0000u));
}

template <typename T, int RQ, int WAVES>
__device__ __forceinline__ void lora_block(const T *X, ActView x_av, int K, const LoraArgs la, int r, int p, int part)
{
    constexpr int THREADS = WAVES * 64, NB = RQ > 0 ? RQ * 4 : LORA_MAX_RANK, OUT = lora_out(WAVES);
    __shared__ float st[LORA_MAX_RANK];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, N = la.N, rank = la.rank;
    const float *Ap = p == 0 ? la.a0 : p == 1 ? la.a1 : la.a2, *Bp = p == 0 ? la.b0 : p == 1 ? la.b1 : la.b2;
    const int valid = la.row_valid[r];
    int a = la.adapter[la.row_b[r]]; // (row_b of an unused row is in range too)
    if (!valid || a >= la.n_adapters) a = -1;
    float *orow = la.out + (size_t)r * la.n_proj * N + (size_t)p * N;
    const int n0 = part * lora_part(WAVES) + threadIdx.x;
    if (a < 0 || !Ap || !Bp) { // (uniform) no update for this row and projection
        if (!la.accumulate) {
#pragma unroll
            for (int o = 0; o < OUT; o++)
                if (n0 + o * THREADS < N) orow[n0 + o * THREADS] = 0.f;
        }
        return;
    }
    const bool vec = RQ > 0 || (RQ < 0 && (rank & 3) == 0 && ((uintptr_t)Bp & 15) == 0);
    float bv[OUT][NB], old[OUT];
#pragma unroll
    for (int o = 0; o < OUT; o++) {
        const int n = min(n0 + o * THREADS, N - 1); // (outputs past the end re-read the last one; never stored)
        old[o] = la.accumulate ? orow[n] : 0.f;
        const float *brow = Bp + ((size_t)a * N + n) * rank;
        if (vec) { // (uniform)
#pragma unroll
            for (int i = 0; i < NB / 4; i++) {
                const float4 v = RQ > 0 || 4 * i < rank ? *(const float4 *)(brow + 4 * i) : make_float4(0.f, 0.f, 0.f, 0.f);
                bv[o][4 * i] = v.x, bv[o][4 * i + 1] = v.y, bv[o][4 * i + 2] = v.z, bv[o][4 * i + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int i = 0; i < NB; i++) bv[o][i] = i < rank ? brow[i] : 0.f;
        }
    }
    // Dot products a wave takes at a time: with four waves a rank of 8 is two, with one read of X.  Three draft tokens of the
    // 768-wide model at rank 8: 32 sequences 321 -> 311 us so, 304 with four pieces of each row requested together (a loop
    // over K of 768 is three trips, one after the other); 16 sequences 297 -> 279, one 245 -> 233.
    constexpr int JS = WAVES == 8 ? 1 : 2;
    for (int j = wave; j < rank; j += JS * WAVES) {
        const float *arow[JS];
        float acc[JS];
#pragma unroll
        for (int i = 0; i < JS; i++) arow[i] = Ap + ((size_t)a * rank + min(j + i * WAVES, rank - 1)) * K, acc[i] = 0.f; // (past the last: read again, not stored)
        for (int k0 = 4 * lane; k0 < K; k0 += 1024) { // 16 bytes per lane and load (K is a multiple of 4), four of each row in flight
            float4 xv[4], av[JS][4];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int k = k0 + 256 * u < K ? k0 + 256 * u : k0;
                xv[u] = load_act4(X, act_index(x_av, r, k, K), x_av.plane);
#pragma unroll
                for (int i = 0; i < JS; i++) av[i][u] = *(const float4 *)(arow[i] + k);
            }
#pragma unroll
            for (int u = 0; u < 4; u++)
#pragma unroll
                for (int i = 0; i < JS; i++) {
                    const float t = acc[i] + (av[i][u].x * xv[u].x + av[i][u].y * xv[u].y + av[i][u].z * xv[u].z + av[i][u].w * xv[u].w);
                    acc[i] = k0 + 256 * u < K ? t : acc[i];
                }
        }
#pragma unroll
        for (int i = 0; i < JS; i++) {
            acc[i] = wave_sum_dpp(acc[i]);
            if (lane == 0 && j + i * WAVES < rank) st[j + i * WAVES] = acc[i];
        }
    }
    __syncthreads();
#pragma unroll
    for (int o = 0; o < OUT; o++) {
        float acc = 0.f;
#pragma unroll
        for (int i = 0; i < NB; i++)
            if (RQ > 0 || i < rank) acc += bv[o][i] * st[i];
        if (n0 + o * THREADS < N) orow[n0 + o * THREADS] = old[o] + la.scale * acc;
    }
}

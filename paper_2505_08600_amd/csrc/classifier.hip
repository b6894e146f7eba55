// Prompt classifier (Sections 2.4, 3.3.3): embedding -> one selective state-space layer ->
// average pooling over the prompt -> linear layer -> arg max, as the second backend of routing.
//
// One workgroup per prompt or (classifier_run_kernel) per run of tokens.  The recurrence over tokens is sequential, so everything a channel
// needs between tokens (its state row, its weights) stays in registers; only the small per-token
// projection (dt_rank + 2 d_state outputs) crosses threads, through LDS.  Everything without a
// dependence between tokens is done for a chunk of tokens at a time.  Pooling and the output
// projection commute (both linear), so the channel outputs are averaged first and projected once
// per prompt.  Up to 192 channels four threads share a channel's states (classifier_quad_kernel, classifier_run_kernel),
// above that a thread has a channel to itself (classifier_kernel).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdint>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/sd.h"
#include "sd_internal.h"

#define CLS_TC 8          // tokens per chunk: everything but the state update is done a chunk at a time
#define CLS_MAX_STATE 16
#define CLS_MAX_RANK 16
#define CLS_MAX_CONV 4
#define CLS_MAX_INNER 512
#define CLS_MAX_MODEL 512
#define CLS_MAX_CLASSES 64
#define CLS_LDS_LIMIT (65536 - 64) // dynamic part; the kernel also holds one static word

struct ClsView {
    // table[v] = emb[v] W_in, [vocab][2 d_inner]: the embedding and the input projection are both
    // functions of the token id alone, so the library multiplies them out once at creation.
    const float *table, *conv_w, *conv_b, *w_x, *w_dt, *b_dt, *a_log, *d, *w_out, *w_fc, *b_fc;
    // w_head[k][c] = sum_m W_out[c][m] W_fc[k][m] (added in 64 bits at creation): pooling, output projection and linear layer are
    // all linear, so the averaged channels meet one matrix (classifier_run_kernel)
    const float *w_head;
    int vocab, d_model, d_inner, d_state, dt_rank, d_conv, n_classes;
};

struct sd_classifier {
    ClsView v;
    void *mem;
    int device;
    size_t lds_bytes;
};

__host__ __device__ static inline size_t cls_align4(size_t n) { return (n + 3) & ~(size_t)3; }

// LDS layout in floats:
//   W_x [d_inner][J] | x [d_inner][CLS_TC] | part [waves][CLS_TC][64] | dbc [CLS_TC][64] | o [d_model + 64]
__host__ __device__ static inline size_t cls_lds_floats(int d_inner, int J, int d_model)
{
    return cls_align4((size_t)d_inner * J) + (size_t)d_inner * CLS_TC + (size_t)(d_inner / 64) * CLS_TC * 64 +
           CLS_TC * 64 + cls_align4((size_t)d_model + CLS_MAX_CLASSES);
}

// table[v][c] = sum_k emb[v][k] W_in[k][c]; one block per vocabulary entry.
__global__ void __launch_bounds__(256)
classifier_table_kernel(const float *__restrict__ emb, const float *__restrict__ w_in, int d_model, int cols,
                        float *__restrict__ table)
{
    __shared__ float e[CLS_MAX_MODEL];
    const size_t v = blockIdx.x;
    for (int k = threadIdx.x; k < d_model; k += blockDim.x) e[k] = emb[v * d_model + k];
    __syncthreads();
    for (int c = threadIdx.x; c < cols; c += blockDim.x) {
        float acc = 0.f;
        for (int k = 0; k < d_model; ++k) acc = fmaf(e[k], w_in[(size_t)k * cols + c], acc);
        table[v * cols + c] = acc;
    }
}

// head[k][c] = sum_m w_out[c][m] w_fc[k][m]; one block per class.
__global__ void __launch_bounds__(256)
classifier_head_kernel(const float *__restrict__ w_out, const float *__restrict__ w_fc, int d_inner, int d_model, float *__restrict__ head)
{
    const int k = blockIdx.x;
    for (int c = threadIdx.x; c < d_inner; c += blockDim.x) {
        double acc = 0.0;
        for (int m = 0; m < d_model; ++m) acc = fma((double)w_out[(size_t)c * d_model + m], (double)w_fc[(size_t)k * d_model + m], acc);
        head[(size_t)k * d_inner + c] = (float)acc;
    }
}

__global__ void __launch_bounds__(CLS_MAX_INNER)
classifier_kernel(ClsView v, const int32_t *__restrict__ tokens, const int32_t *__restrict__ lens, int max_len,
                  float *__restrict__ logits, int32_t *__restrict__ draft_id)
{
    extern __shared__ __align__(16) float lds[];
    const int J = v.dt_rank + 2 * v.d_state;
    const int di = v.d_inner, dm = v.d_model, waves = di >> 6;
    float *s_wx = lds;
    float *s_x = s_wx + cls_align4((size_t)di * J);
    float *s_part = s_x + (size_t)di * CLS_TC;
    float *s_dbc = s_part + (size_t)waves * CLS_TC * 64;
    float *s_o = s_dbc + CLS_TC * 64;
    __shared__ int s_bad;

    const int c = threadIdx.x, lane = c & 63, wave = c >> 6;
    const int i = blockIdx.x;
    int L = lens[i];
    L = L < 0 ? 0 : (L > max_len ? max_len : L);
    const int32_t *tok = tokens + (size_t)i * max_len;

    if (c == 0) s_bad = 0;
    for (int k = c; k < di * J; k += di) s_wx[k] = v.w_x[k];
    // per token, r sits in slots [0, 16), B in [16, 32), C in [32, 48): slots beyond dt_rank / d_state stay
    // zero, so the loops over them below run to the fixed maxima without a branch
    for (int k = c; k < CLS_TC * 64; k += di) s_dbc[k] = 0.f;

    // this channel's constants
    float cw[CLS_MAX_CONV], A[CLS_MAX_STATE], wdt[CLS_MAX_RANK], h[CLS_MAX_STATE], xh[CLS_MAX_CONV];
#pragma unroll
    for (int j = 0; j < CLS_MAX_CONV; ++j) {
        const int src = j - (CLS_MAX_CONV - v.d_conv); // taps right-aligned: the last one meets the current token
        cw[j] = src >= 0 ? v.conv_w[c * v.d_conv + src] : 0.f;
        xh[j] = 0.f;
    }
#pragma unroll
    for (int n = 0; n < CLS_MAX_STATE; ++n) {
        A[n] = n < v.d_state ? -expf(v.a_log[c * v.d_state + n]) * 1.44269504088896f : 0.f; // times log2(e): decay = 2^(Delta A)
        h[n] = 0.f;
    }
#pragma unroll
    for (int r = 0; r < CLS_MAX_RANK; ++r) wdt[r] = r < v.dt_rank ? v.w_dt[r * di + c] : 0.f;
    const float cb = v.conv_b[c], bdt = v.b_dt[c], D = v.d[c];
    float pooled = 0.f;

    // The input projection's two values of this channel for one chunk of tokens, gathered from the
    // table.  Two loads depend on each other (token id, then table row), so both run ahead: lane t of
    // every wave holds the id of token t of the chunk after next while the next chunk's rows fly.
    float nx[CLS_TC], nz[CLS_TC];
    bool bad = false;
    int idv = 0;
    auto load_ids = [&](int t0) {
        const int t = t0 + (lane & (CLS_TC - 1));
        idv = t < L ? tok[t] : 0;
    };
    auto gather = [&](int t0) {
#pragma unroll
        for (int t = 0; t < CLS_TC; ++t) {
            nx[t] = nz[t] = 0.f;
            const int id = __builtin_amdgcn_readlane(idv, t);
            if (t0 + t < L) {
                if ((unsigned)id < (unsigned)v.vocab) {
                    const float *row = v.table + (size_t)id * 2 * di + c;
                    nx[t] = row[0];
                    nz[t] = row[di];
                } else
                    bad = true;
            }
        }
    };
    load_ids(0);
    gather(0);
    load_ids(CLS_TC);

    for (int t0 = 0; t0 < L; t0 += CLS_TC) {
        const int nt = min(CLS_TC, L - t0);
        float x[CLS_TC], z[CLS_TC];
        // causal depthwise convolution and SiLU: no dependence on the state, so the whole chunk at once
#pragma unroll
        for (int t = 0; t < CLS_TC; ++t) {
            xh[0] = xh[1]; xh[1] = xh[2]; xh[2] = xh[3]; xh[3] = nx[t];
            float pre = cb;
#pragma unroll
            for (int j = 0; j < CLS_MAX_CONV; ++j) pre = fmaf(cw[j], xh[j], pre);
            x[t] = pre * __builtin_amdgcn_rcpf(1.f + __expf(-pre));
            z[t] = nz[t];
        }
        *(float4 *)(s_x + c * CLS_TC) = make_float4(x[0], x[1], x[2], x[3]);
        *(float4 *)(s_x + c * CLS_TC + 4) = make_float4(x[4], x[5], x[6], x[7]);
        gather(t0 + CLS_TC); // the next chunk's rows fly while this one is worked on
        load_ids(t0 + 2 * CLS_TC);
        __syncthreads();

        // (r, B, C) = x W_x for the chunk: each wave sums its 64 channels for output `lane`
        if (lane < J) {
            float p[CLS_TC];
#pragma unroll
            for (int t = 0; t < CLS_TC; ++t) p[t] = 0.f;
            const float *wx = s_wx + (size_t)wave * 64 * J + lane;
            const float *xs = s_x + (size_t)wave * 64 * CLS_TC;
#pragma unroll 4
            for (int k = 0; k < 64; ++k) {
                const float w = wx[k * J];
                const float4 a = *(const float4 *)(xs + k * CLS_TC), b = *(const float4 *)(xs + k * CLS_TC + 4);
                p[0] = fmaf(a.x, w, p[0]); p[1] = fmaf(a.y, w, p[1]); p[2] = fmaf(a.z, w, p[2]); p[3] = fmaf(a.w, w, p[3]);
                p[4] = fmaf(b.x, w, p[4]); p[5] = fmaf(b.y, w, p[5]); p[6] = fmaf(b.z, w, p[6]); p[7] = fmaf(b.w, w, p[7]);
            }
#pragma unroll
            for (int t = 0; t < CLS_TC; ++t) s_part[(wave * CLS_TC + t) * 64 + lane] = p[t];
        }
        __syncthreads();
        for (int q = c; q < CLS_TC * 64; q += di) {
            const int j = q & 63;
            if (j < J) {
                float p = 0.f;
                for (int w = 0; w < waves; ++w) p += s_part[w * CLS_TC * 64 + q];
                const int slot = j < v.dt_rank ? j : (j < v.dt_rank + v.d_state ? 16 + j - v.dt_rank : 32 + j - v.dt_rank - v.d_state);
                s_dbc[(q & ~63) + slot] = p;
            }
        }
        __syncthreads();

        // the state update, token by token, all in this thread's registers
#pragma unroll
        for (int t = 0; t < CLS_TC; ++t) {
            if (t >= nt) break; // uniform over the block
            const float *dbc = s_dbc + t * 64;
            float dt = bdt;
#pragma unroll
            for (int r = 0; r < CLS_MAX_RANK; ++r) dt = fmaf(dbc[r], wdt[r], dt);
            // softplus = log1p(e^dt): log(u) e / (u - 1) with u = 1 + e undoes the rounding of u (steps are ~1e-3..0.1)
            const float e = __expf(dt), u = 1.f + e;
            const float delta = dt > 20.f ? dt : (u == 1.f ? e : logf(u) * e * __builtin_amdgcn_rcpf(u - 1.f));
            const float dx = delta * x[t];
            float acc = 0.f;
#pragma unroll
            for (int n = 0; n < CLS_MAX_STATE; ++n) {
                h[n] = fmaf(__builtin_amdgcn_exp2f(delta * A[n]), h[n], dx * dbc[16 + n]);
                acc = fmaf(dbc[32 + n], h[n], acc);
            }
            pooled += (acc + D * x[t]) * z[t] * __builtin_amdgcn_rcpf(1.f + __expf(-z[t]));
        }
    }
    if (bad) s_bad = 1;

    // mean over tokens, output projection, linear layer, arg max
    __syncthreads();
    s_x[c] = L > 0 ? pooled / (float)L : 0.f;
    __syncthreads();
    for (int m = c; m < dm; m += di) {
        float o = 0.f;
        for (int k = 0; k < di; ++k) o = fmaf(s_x[k], v.w_out[(size_t)k * dm + m], o);
        s_o[m] = o;
    }
    __syncthreads();
    float *s_logit = s_o + dm;
    for (int k = c; k < v.n_classes; k += di) {
        float o = v.b_fc[k];
        for (int m = 0; m < dm; ++m) o = fmaf(s_o[m], v.w_fc[(size_t)k * dm + m], o);
        s_logit[k] = o;
        if (logits) logits[(size_t)i * v.n_classes + k] = o;
    }
    __syncthreads();
    if (c == 0) {
        int best = 0;
        for (int k = 1; k < v.n_classes; ++k)
            if (s_logit[k] > s_logit[best]) best = k;
        draft_id[i] = s_bad ? -1 : best;
    }
}

// Up to 192 channels: 4 d_inner threads per prompt, chunks of 16 tokens.
// Bound: the chain of the longest prompt - its tokens' state updates (four exponentials and some twenty other
// instructions per token and thread, 12 waves of 192 channels on 4 SIMDs) and four barriers per chunk.  So the work of a
// chunk is split three ways: (1) input convolution, SiLU, softplus: wave w has channels 16 w .. 16 w + 15, lane (channel
// l % 16, token group l / 16) four tokens of one of them; (2) the two small projections run on the matrix cores in fp32:
// [16 x d_inner] . [d_inner x 48] for r, B and C, a wave per 16 outputs and share of the channels, and [16 x 16] .
// [16 x d_inner] for the step sizes, whose result lands in exactly the lanes of (1); the weights stay in registers;
// (3) state update: thread (channel, quarter) has four of the states in registers and adds its share of silu(z) (C . h)
// to its pooled sum, so nothing is reduced per token.
// Measured, 400 prompts of 1 to 128 tokens, 192 channels: 47.7 us (120 with a thread per channel; 59 where 80 registers per thread let a second prompt
// onto the unit: the operands then spill).
#define CQ_TC 16
#define CQ_OUT 48 // r | B | C, 16 slots each
#define CQ_ROW 52 // ... in rows of 52: 16 rows fall into distinct banks
__host__ __device__ static inline size_t cq_lds_floats(int di, int dm)
{
    // x [TC][di + 4] | delta [TC][di + 4] (the projection's partial sums before that) | (delta x, silu(z)) [TC][di + 4] | r, B, C [TC][52]
    const size_t chunk = 4 * (size_t)CQ_TC * (di + 4) + CQ_TC * CQ_ROW;
    const size_t tail = (size_t)di * 5 + 4 * (size_t)di + cls_align4(dm) + CLS_MAX_CLASSES; // pooled shares, mean | partial outputs | output | logits
    return chunk > tail ? chunk : tail;
}

// a barrier that waits for LDS traffic only: the table rows of the next chunk stay in flight across it
__device__ __forceinline__ void lds_sync() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int DI> // d_inner: 64, 128 or 192
__global__ void __launch_bounds__(4 * DI, DI / 64)
classifier_quad_kernel(ClsView v, const int32_t *__restrict__ tokens, const int32_t *__restrict__ lens, int max_len,
                       float *__restrict__ logits, int32_t *__restrict__ draft_id)
{
    typedef __attribute__((ext_vector_type(4))) float f32x4;
    extern __shared__ __align__(16) float lds[];
    __shared__ int s_bad;
    constexpr int di = DI, sx = DI + 4; // (rows 4 banks apart)
    constexpr int waves = DI / 16, nkq = waves / 3, per = DI / 4 / nkq; // (2): a wave's share is `per` instructions
    static_assert(nkq * per * 4 == DI, "shares of whole instructions");
    const int dm = v.d_model;
    float *s_x = lds, *s_delta = s_x + CQ_TC * sx, *s_part = s_delta;
    float2 *s_dz = (float2 *)(s_delta + CQ_TC * sx);
    float *s_dbc = s_delta + 3 * CQ_TC * sx;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, tq = lane >> 4, c = wave * 16 + l16; // (1): channel, group of four tokens
    const int cs = tid >> 2, sub = tid & 3;                         // (3): channel, quarter of the states
    const int i = blockIdx.x;
    int L = lens[i];
    L = L < 0 ? 0 : (L > max_len ? max_len : L);
    const int32_t *tok = tokens + (size_t)i * max_len;
    if (tid == 0) s_bad = 0;

    // (2): this wave's 16 outputs and channels (four per instruction); its 16 channels of the step sizes
    const int tile = wave % 3, kq = wave / 3;
    const bool proj = kq < nkq;
    const int k_lo = proj ? kq * per : 0;
    const int J = v.dt_rank + 2 * v.d_state;
    const int col = tile == 0 ? l16 : v.dt_rank + (tile - 1) * v.d_state + l16;
    const bool has_col = l16 < (tile == 0 ? v.dt_rank : v.d_state);
    float bd[4];
    float bw[per];
#pragma unroll
    for (int k = 0; k < per; ++k) {
        const float w = v.w_x[((k_lo + k) * 4 + tq) * J + (has_col ? col : 0)];
        bw[k] = has_col ? w : 0.f;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float w = v.w_dt[min(4 * k + tq, v.dt_rank - 1) * di + c];
        bd[k] = 4 * k + tq < v.dt_rank ? w : 0.f;
    }
    // (1): this channel's constants
    float cw[CLS_MAX_CONV];
#pragma unroll
    for (int j = 0; j < CLS_MAX_CONV; ++j) {
        const int src = j - (CLS_MAX_CONV - v.d_conv); // taps right-aligned: the last one meets the current token
        cw[j] = src >= 0 ? v.conv_w[c * v.d_conv + src] : 0.f;
    }
    const float cb = v.conv_b[c], bdt = v.b_dt[c], D = v.d[c];
    // (3): decay rates (times log2 e: decay = 2^(Delta A)) and states
    float A[4], h[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        const int st = sub * 4 + n;
        A[n] = st < v.d_state ? -expf(v.a_log[cs * v.d_state + st]) * 1.44269504088896f : 0.f;
        h[n] = 0.f;
    }
    float pooled = 0.f, pooled_d = 0.f;

    // The table rows of this lane's four tokens.  Ids run one chunk ahead of the rows (lane t of every wave holds the id of
    // token t), the rows one chunk ahead of their use; the convolution's history is the neighbouring token group's.
    float nx[4], nz[4], px[4]; // next rows; this lane's inputs of the chunk before (the last three count)
    bool bad = false;
    int idv = 0;
    auto load_ids = [&](int t0) { idv = t0 + l16 < L ? tok[t0 + l16] : 0; };
    auto gather = [&](int t0) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int id = __shfl(idv, 4 * tq + j, 64);
            const bool live = t0 + 4 * tq + j < L, in = (unsigned)id < (unsigned)v.vocab;
            bad |= live && !in;
            const float *row = v.table + (size_t)(in ? id : 0) * 2 * di + c;
            const float a = row[0], b = row[di];
            nx[j] = live && in ? a : 0.f;
            nz[j] = live && in ? b : 0.f;
        }
    };
#pragma unroll
    for (int j = 0; j < 4; ++j) px[j] = 0.f;
    load_ids(0);
    gather(0);
    load_ids(CQ_TC);

    for (int t0 = 0; t0 < L; t0 += CQ_TC) {
        const int nt = min(CQ_TC, L - t0);
        // (1) causal depthwise convolution and SiLU
        float z[4], raw[CLS_MAX_CONV + 3];
#pragma unroll
        for (int j = 0; j < 3; ++j) raw[j] = __shfl(tq == 3 ? px[j + 1] : nx[j + 1], (lane + 48) & 63, 64);
#pragma unroll
        for (int j = 0; j < 4; ++j) raw[3 + j] = px[j] = nx[j];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            float pre = cb;
#pragma unroll
            for (int j = 0; j < CLS_MAX_CONV; ++j) pre = fmaf(cw[j], raw[t + j], pre);
            z[t] = nz[t] * __builtin_amdgcn_rcpf(1.f + __expf(-nz[t]));
            s_x[(4 * tq + t) * sx + c] = pre * __builtin_amdgcn_rcpf(1.f + __expf(-pre));
        }
        gather(t0 + CQ_TC); // the next chunk's rows fly while this one is worked on
        load_ids(t0 + 2 * CQ_TC);
        lds_sync();
        // (2) lane (token l % 16, channel l / 16 of four) against (channel, output l % 16); the result leaves tokens
        // 4 (l / 16) .. + 3 of output l % 16
        if (proj) {
            f32x4 acc = {0.f, 0.f, 0.f, 0.f}, acc2 = {0.f, 0.f, 0.f, 0.f};
            const float *xs = s_x + l16 * sx + tq + 4 * k_lo;
#pragma unroll
            for (int k = 0; k < per; k += 2) { // (two chains)
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(xs[4 * k], bw[k], acc, 0, 0, 0);
                acc2 = __builtin_amdgcn_mfma_f32_16x16x4f32(xs[4 * k + 4], bw[k + 1], acc2, 0, 0, 0);
            }
            float *dst = s_part + kq * CQ_TC * CQ_OUT + tq * 4 * CQ_OUT + tile * 16 + l16;
#pragma unroll
            for (int r = 0; r < 4; ++r) dst[r * CQ_OUT] = acc[r] + acc2[r];
        }
        lds_sync();
        for (int q = tid; q < CQ_TC * CQ_OUT; q += 4 * di) {
            float p = 0.f;
#pragma unroll
            for (int w = 0; w < nkq; ++w) p += s_part[w * CQ_TC * CQ_OUT + q];
            s_dbc[q / CQ_OUT * CQ_ROW + q % CQ_OUT] = p;
        }
        lds_sync();
        // (2), (1) step sizes
        f32x4 dt4 = {bdt, bdt, bdt, bdt};
#pragma unroll
        for (int k = 0; k < 4; ++k) dt4 = __builtin_amdgcn_mfma_f32_16x16x4f32(s_dbc[l16 * CQ_ROW + 4 * k + tq], bd[k], dt4, 0, 0, 0);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int row = 4 * tq + t;
            const float dt = dt4[t];
            // softplus = log1p(e^dt): log(u) e / (u - 1) with u = 1 + e undoes the rounding of u (steps are ~1e-3..0.1)
            const float e = __expf(dt), u = 1.f + e;
            const float delta = dt > 20.f ? dt : (u == 1.f ? e : logf(u) * e * __builtin_amdgcn_rcpf(u - 1.f));
            s_delta[row * sx + c] = delta;
            const float x = s_x[row * sx + c];
            s_dz[row * sx + c] = make_float2(delta * x, z[t]);
            if (row < nt) pooled_d = fmaf(x * D, z[t], pooled_d);
        }
        lds_sync();
        // (3) the state update, token by token, in this thread's registers
        const float *sd = s_delta + cs;
        const float2 *sz = s_dz + cs;
        const float *sb = s_dbc + 16 + sub * 4;
        auto token = [&](int t) {
            const float delta = sd[t * sx];
            const float2 dz = sz[t * sx];
            const float4 B = *(const float4 *)(sb + t * CQ_ROW), C = *(const float4 *)(sb + t * CQ_ROW + 16);
            h[0] = fmaf(__builtin_amdgcn_exp2f(delta * A[0]), h[0], dz.x * B.x);
            h[1] = fmaf(__builtin_amdgcn_exp2f(delta * A[1]), h[1], dz.x * B.y);
            h[2] = fmaf(__builtin_amdgcn_exp2f(delta * A[2]), h[2], dz.x * B.z);
            h[3] = fmaf(__builtin_amdgcn_exp2f(delta * A[3]), h[3], dz.x * B.w);
            const float acc = fmaf(C.w, h[3], fmaf(C.z, h[2], fmaf(C.y, h[1], C.x * h[0])));
            pooled = fmaf(acc, dz.y, pooled);
        };
        int t = 0;
        for (; t + 4 <= nt; t += 4) { // (four tokens' operands in flight)
            token(t);
            token(t + 1);
            token(t + 2);
            token(t + 3);
        }
        for (; t < nt; ++t) token(t);
    }
    if (bad) s_bad = 1;

    // mean over tokens, output projection, linear layer, arg max
    __syncthreads();
    float *s_pool = lds, *s_mean = s_pool + 4 * di, *s_po = s_mean + di, *s_o = s_po + 4 * di, *s_logit = s_o + cls_align4(dm);
    s_pool[tq * di + c] = pooled_d;
    pooled += dpp_f<0xB1>(pooled);
    pooled += dpp_f<0x4E>(pooled);
    __syncthreads();
    if (sub == 0) {
        const float t = pooled + ((s_pool[cs] + s_pool[di + cs]) + (s_pool[2 * di + cs] + s_pool[3 * di + cs]));
        s_mean[cs] = L > 0 ? t / (float)L : 0.f;
    }
    __syncthreads();
    // the block's threads share the channels of every output: np shares of kc channels (at most 4 di partial sums)
    const int np = max(1, 4 * di / dm), kc = (di + np - 1) / np;
    for (int q = tid; q < np * dm; q += 4 * di) {
        const int m = q % dm, k0 = q / dm * kc, k1 = min(di, k0 + kc);
        float o = 0.f;
#pragma unroll 8
        for (int k = k0; k < k1; ++k) o = fmaf(s_mean[k], v.w_out[(size_t)k * dm + m], o);
        if (np > 1) s_po[q] = o;
        else s_o[m] = o;
    }
    __syncthreads();
    if (np > 1) {
        for (int m = tid; m < dm; m += 4 * di) {
            float o = 0.f;
            for (int w = 0; w < np; ++w) o += s_po[w * dm + m];
            s_o[m] = o;
        }
        __syncthreads();
    }
    for (int k = wave; k < v.n_classes; k += waves) {
        float o = 0.f;
        for (int m = lane; m < dm; m += 64) o = fmaf(s_o[m], v.w_fc[(size_t)k * dm + m], o);
        o = wave_sum_dpp(o);
        if (lane == 0) {
            o += v.b_fc[k];
            s_logit[k] = o;
            if (logits) logits[(size_t)i * v.n_classes + k] = o;
        }
    }
    __syncthreads();
    if (tid == 0) {
        int best = 0;
        for (int k = 1; k < v.n_classes; ++k)
            if (s_logit[k] > s_logit[best]) best = k;
        draft_id[i] = s_bad ? -1 : best;
    }
}

// The same work in equal runs of chunks, a block per compute unit, for callers that bring a workspace.
// A block per prompt spends 6 us on launch, weights and the first dependent loads of every prompt, and the longest prompt
// sets the time of a small batch (128 tokens: 34 us of chunks).  Here the chunks of all prompts are dealt out in equal runs, weights
// are loaded once per run, and the head is one matrix.  A run that starts inside a prompt works from a zero state; with P
// the product of its decays and G the sum of C P silu(z) over its tokens, the state before it enters the pooled sum as G . h and the
// state behind it as P h.  So the block leaves the record (G, P, state, sums) of that prompt's part in the workspace, the block a
// prompt starts in leaves what it has, and whichever of the prompt's blocks ends last joins them in order: no block waits for
// another, and the sums are the same whoever joins.  Where cutting would save a chunk at most, each block has a prompt.
// Bound: vector issue and barriers, 4.3 - 4.6 us a chunk, 4.4 us from the start of a block to its first chunk, about 7 us for a cut
// batch's hand-over (the stores' arrival, one write-back of the die's L2 and an atomic per block, the join's loads; fences of all
// twelve waves instead of one cost 70).  A second launch for the joins cost 5 - 8 us, and 2 where nothing was cut.
// Measured, 192 channels, a block per prompt / runs (us): 8 prompts of up to 64 tokens 24.9 / 17.3, 40 of up to 128 28.7 / 18.0, 100 of
// up to 40 19.7 / 17.2, 200 of up to 200 32.6 / 24.7, 400 of up to 128 55.6 / 34.0, 1000 87 / 58, 4000 284 / 185, 100000 of up to 40
// 5920 / 3784; 3000 of up to 16 124 / 73; all of one length: 200 x 128 44.1 / 43.8, 100 x 200 64 / 44, 400 x 128 86.5 / 80.7, 2000 x 200
// 515 / 494, 250 x 512 153 / 156, 20 of 900 - 1000 285 / 48.
#define CQ_BLOCKS 256 // blocks at most: one per compute unit
__host__ __device__ static constexpr size_t cq_run_lds_floats(int di)
{
    // x [TC][di + 4] | delta [TC][di + 4] (the projection's partial sums before that) | (delta x, silu(z)) [TC][di + 4] | r, B, C [TC][52]
    return 4 * (size_t)CQ_TC * (di + 4) + CQ_TC * CQ_ROW;
}
// Workspace of nb blocks of t threads, in floats: arrivals [nb] (64 bits each) | records [nb][14][t] | open prompts [nb][6][t] |
// invalid ids seen in a block's record, in its open prompt [nb][2]
__host__ __device__ static inline size_t cq_rec_at(size_t nb, size_t b, int t) { return 2 * nb + b * 14 * (size_t)t; }
__host__ __device__ static inline size_t cq_open_at(size_t nb, size_t b, int t) { return 2 * nb + (nb * 14 + b * 6) * (size_t)t; }
__host__ __device__ static inline size_t cq_bad_at(size_t nb, size_t b, int t) { return 2 * nb + nb * 20 * (size_t)t + b * 2; }

// What blocks hand to each other goes past the caches that only one die sees.
__device__ __forceinline__ void put(float *p, float x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ float get(const float *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// One of `parts` arrivals at *word; true for the last.  The word counts for this call only where its upper 48 bits are the call's
// tag, so the workspace may hold anything; the last arrival leaves 0 (a replay of a captured call has the same tag).
__device__ __forceinline__ bool cq_arrive(unsigned long long *word, unsigned long long tag, int parts)
{
    unsigned long long old = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (;;) { // (repeated only when another part has arrived in between)
        const unsigned long long seen = (old & ~0xffffull) == tag ? old & 0xffff : 0;
        const bool last = (int)seen + 1 == parts;
        if (__hip_atomic_compare_exchange_strong(word, &old, last ? 0 : tag | (seen + 1), __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            return last;
    }
}

__device__ __forceinline__ int cls_len(const int32_t *lens, int i, int max_len) { return min(max(lens[i], 0), max_len); }
struct CqChunk {
    int p, at, len; // prompt, first token, the prompt's length
};
__device__ __forceinline__ int cls_chunks(int L) { return max(1, (L + CQ_TC - 1) / CQ_TC); } // (an empty prompt has one, of no tokens)

// Mean over tokens, head, arg max of a prompt whose sums are complete: pooled per (channel, quarter) thread, pooled_d per
// (channel, token group) thread.  bad: uniform.
template <int DI>
__device__ __forceinline__ void classifier_finish(const ClsView &v, int i, int L, float pooled, float pooled_d, bool bad, float *s_pool, float *s_mean,
                                                  float *s_logit, float *logits, int32_t *draft_id)
{
    constexpr int waves = DI / 16;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    s_pool[(lane >> 4) * DI + wave * 16 + (lane & 15)] = pooled_d;
    pooled += dpp_f<0xB1>(pooled);
    pooled += dpp_f<0x4E>(pooled);
    lds_sync();
    if ((tid & 3) == 0) {
        const int c = tid >> 2;
        const float t = pooled + ((s_pool[c] + s_pool[DI + c]) + (s_pool[2 * DI + c] + s_pool[3 * DI + c]));
        s_mean[c] = L > 0 ? t / (float)L : 0.f;
    }
    lds_sync();
    for (int k = wave; k < v.n_classes; k += waves) {
        float o = 0.f;
#pragma unroll
        for (int m = 0; m < DI; m += 64) o = fmaf(s_mean[m + lane], v.w_head[(size_t)k * DI + m + lane], o);
        o = wave_sum_dpp(o);
        if (lane == 0) {
            o += v.b_fc[k];
            s_logit[k] = o;
            if (logits) logits[(size_t)i * v.n_classes + k] = o;
        }
    }
    lds_sync();
    if (tid == 0) {
        int best = 0;
        for (int k = 1; k < v.n_classes; ++k)
            if (s_logit[k] > s_logit[best]) best = k;
        draft_id[i] = bad ? -1 : best;
    }
}

__device__ __forceinline__ void cq_record(float *rec, int T, const float *G, const float *P, const float *h, float pooled, float pooled_d)
{
#pragma unroll
    for (int k = 0; k < 4; ++k) put(rec + k * T, G[k]), put(rec + (4 + k) * T, P[k]), put(rec + (8 + k) * T, h[k]);
    put(rec + 12 * T, pooled);
    put(rec + 13 * T, pooled_d);
}

// Joins prompt i, which block b0 left open, with the records of blocks b0 + 1 .. b1.
template <int DI>
__device__ __forceinline__ void cq_join(const ClsView &v, int i, int L, int b0, int b1, int nb, const float *ws, float *s_pool, float *s_mean,
                                        float *s_logit, float *logits, int32_t *draft_id)
{
    constexpr int T = 4 * DI;
    const int tid = threadIdx.x;
    const float *o = ws + cq_open_at(nb, b0, T) + tid;
    bool bad = get(ws + cq_bad_at(nb, b0, T) + 1) != 0.f;
    float h[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) h[k] = get(o + k * T);
    float pooled = get(o + 4 * T), pooled_d = get(o + 5 * T);
    for (int b = b0 + 1; b <= b1; ++b) {
        const float *rec = ws + cq_rec_at(nb, b, T) + tid;
        float r[14];
#pragma unroll
        for (int k = 0; k < 14; ++k) r[k] = get(rec + k * T);
        bad |= get(ws + cq_bad_at(nb, b, T)) != 0.f;
        pooled += fmaf(r[3], h[3], fmaf(r[2], h[2], fmaf(r[1], h[1], fmaf(r[0], h[0], r[12]))));
        pooled_d += r[13];
#pragma unroll
        for (int k = 0; k < 4; ++k) h[k] = fmaf(r[4 + k], h[k], r[8 + k]);
    }
    classifier_finish<DI>(v, i, L, pooled, pooled_d, bad, s_pool, s_mean, s_logit, logits, draft_id);
}

template <int DI> // d_inner: 64, 128 or 192
__global__ void __launch_bounds__(4 * DI, DI / 64)
classifier_run_kernel(ClsView v, const int32_t *__restrict__ tokens, const int32_t *__restrict__ lens, int n, int max_len,
                      float *__restrict__ logits, int32_t *__restrict__ draft_id, float *ws, unsigned long long tag)
{
    typedef __attribute__((ext_vector_type(4))) float f32x4;
    __shared__ __align__(16) float lds[cq_run_lds_floats(DI)];
    __shared__ float s_pool[4 * DI], s_mean[DI], s_logit[CLS_MAX_CLASSES];
    __shared__ int s_sum[16], s_max[16], s_start[3], s_last[2];
    constexpr int di = DI, sx = DI + 4, T = 4 * DI; // (rows 4 banks apart)
    constexpr int waves = DI / 16, nkq = waves / 3, per = DI / 4 / nkq; // (2): a wave's share is `per` instructions
    static_assert(nkq * per * 4 == DI, "shares of whole instructions");
    float *s_x = lds, *s_delta = s_x + CQ_TC * sx, *s_part = s_delta;
    float2 *s_dz = (float2 *)(s_delta + CQ_TC * sx);
    float *s_dbc = s_delta + 3 * CQ_TC * sx;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, tq = lane >> 4, c = wave * 16 + l16; // (1): channel, group of four tokens
    const int cs = tid >> 2, sub = tid & 3;                         // (3): channel, quarter of the states

    // (for a batch in which nothing is cut: this block's prompt)
    const int own = min((int)blockIdx.x, n - 1), own_len = cls_len(lens, own, max_len);
    const int own_id = l16 < max_len ? tokens[(size_t)own * max_len + l16] : 0;
    // chunks of the prompts this thread looks after (pp in a row), and of those before them
    const int pp = (n + T - 1) / T, p_lo = min(n, tid * pp), p_hi = min(n, p_lo + pp);
    int mine = 0, longest = 0;
    for (int p = p_lo; p < p_hi; ++p) {
        const int nc = cls_chunks(cls_len(lens, p, max_len));
        mine += nc;
        longest = max(longest, nc);
    }

    // (2): this wave's 16 outputs and channels (four per instruction); its 16 channels of the step sizes
    const int tile = wave % 3, kq = wave / 3;
    const bool proj = kq < nkq;
    const int k_lo = proj ? kq * per : 0;
    const int J = v.dt_rank + 2 * v.d_state;
    const int col = tile == 0 ? l16 : v.dt_rank + (tile - 1) * v.d_state + l16;
    const bool has_col = l16 < (tile == 0 ? v.dt_rank : v.d_state);
    float bd[4];
    float bw[per];
#pragma unroll
    for (int k = 0; k < per; ++k) {
        const float w = v.w_x[((k_lo + k) * 4 + tq) * J + (has_col ? col : 0)];
        bw[k] = has_col ? w : 0.f;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float w = v.w_dt[min(4 * k + tq, v.dt_rank - 1) * di + c];
        bd[k] = 4 * k + tq < v.dt_rank ? w : 0.f;
    }
    // (1): this channel's constants
    float cw[CLS_MAX_CONV];
#pragma unroll
    for (int j = 0; j < CLS_MAX_CONV; ++j) {
        const int src = j - (CLS_MAX_CONV - v.d_conv); // taps right-aligned: the last one meets the current token
        cw[j] = src >= 0 ? v.conv_w[c * v.d_conv + src] : 0.f;
    }
    const float cb = v.conv_b[c], bdt = v.b_dt[c], D = v.d[c];
    // (3): decay rates (times log2 e: decay = 2^(Delta A))
    float A[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int st = sub * 4 + k;
        A[k] = st < v.d_state ? -expf(v.a_log[cs * v.d_state + st]) * 1.44269504088896f : 0.f;
    }

    // this block's run of chunks
    int incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int x = __shfl_up(incl, o, 64);
        if (lane >= o) incl += x;
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) longest = max(longest, __shfl_xor(longest, o, 64));
    if (lane == 63) {
        s_sum[wave] = incl;
        s_max[wave] = longest;
    }
    lds_sync();
    int first = incl - mine, total = 0; // (first: chunks before this thread's prompts)
    for (int w = 0; w < waves; ++w) {
        const int x = s_sum[w];
        if (w < wave) first += x;
        total += x;
        longest = max(longest, s_max[w]);
    }
    total = __builtin_amdgcn_readfirstlane(total); // (the loops below are uniform: keep their bounds in scalar registers)
    longest = __builtin_amdgcn_readfirstlane(longest);
    const int nb = gridDim.x, run = (total + nb - 1) / nb;
    // cutting would save a chunk at most: a block per prompt
    const bool whole = n <= nb && longest <= run + 1;
    int run0, run1;
    CqChunk cur = {own, 0, own_len};
    if (whole) {
        run0 = 0;
        run1 = (int)blockIdx.x < n ? cls_chunks(own_len) : 0;
    } else {
        run0 = (int)min((int64_t)total, (int64_t)blockIdx.x * run), run1 = min(total, run0 + run);
        if (run0 < run1 && first <= run0 && run0 < first + mine) { // (one thread's prompts hold chunk run0)
            int p = p_lo, q = first, L = cls_len(lens, p, max_len);
            while (q + cls_chunks(L) <= run0) {
                q += cls_chunks(L);
                L = cls_len(lens, ++p, max_len);
            }
            s_start[0] = p;
            s_start[1] = (run0 - q) * CQ_TC;
            s_start[2] = L;
        }
        lds_sync();
        cur.p = __builtin_amdgcn_readfirstlane(s_start[0]);
        cur.at = __builtin_amdgcn_readfirstlane(s_start[1]);
        cur.len = __builtin_amdgcn_readfirstlane(s_start[2]);
    }
    if (run0 >= run1) return; // (uniform)
    // The chunks behind this one: the same prompt's, or the first of the next prompt, whose length was requested two prompts
    // before.
    CqChunk ahead = cur;
    int len1 = 0, len2 = 0; // of prompts ahead.p + 1, ahead.p + 2
    if (!whole) {
        len1 = cls_len(lens, min(cur.p + 1, n - 1), max_len);
        len2 = cls_len(lens, min(cur.p + 2, n - 1), max_len);
    }
    auto advance = [&]() {
        if (ahead.at + CQ_TC < ahead.len) ahead.at += CQ_TC;
        else {
            ahead = {ahead.p + 1, 0, len1};
            len1 = len2;
            if (!whole) len2 = cls_len(lens, min(ahead.p + 2, n - 1), max_len);
        }
        return ahead;
    };

    // The table rows of this lane's four tokens.  Ids run one chunk ahead of the rows (lane t of every wave holds the id of
    // token t), the rows one chunk ahead of their use; the convolution's history is the neighbouring token group's.
    // (Every chunk gathers, past the run's end row 0: in a branch the rows would be waited for where it ends, 0.4 us a chunk.)
    float nx[4], nz[4], px[4]; // next rows; this lane's inputs of the chunk before (the last three count)
    bool take[4], bad = false, bad_next = false; // rows of valid tokens
    int idv = 0;
    auto load_ids = [&](const CqChunk &e) { idv = e.at + l16 < e.len ? tokens[(size_t)e.p * max_len + e.at + l16] : 0; };
    auto gather = [&](const CqChunk &e) {
        bad_next = false;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int id = __shfl(idv, 4 * tq + j, 64);
            const bool live = e.at + 4 * tq + j < e.len, in = (unsigned)id < (unsigned)v.vocab;
            bad_next |= live && !in;
            take[j] = live && in;
            const float *row = v.table + (size_t)(in ? id : 0) * 2 * di + c;
            nx[j] = row[0];
            nz[j] = row[di];
        }
    };
    // state and sums of the prompt, or of the part of the prompt the run starts inside, with its decay product and G
    float h[4], pooled = 0.f, pooled_d = 0.f;
    const CqChunk start = cur;
    const bool head_part = start.at > 0;
    bool part_bad = false; // an invalid id in the part of the prompt the run starts inside
#pragma unroll
    for (int k = 0; k < 4; ++k) h[k] = px[k] = 0.f;
    if (whole) idv = l16 < cur.len ? own_id : 0;
    else load_ids(cur);
    if (head_part) { // the convolution's history of the four tokens before
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int id = tokens[(size_t)cur.p * max_len + cur.at - 4 + j];
            const bool in = (unsigned)id < (unsigned)v.vocab;
            const float a = v.table[(size_t)(in ? id : 0) * 2 * di + c];
            px[j] = in ? a : 0.f;
        }
    }
    gather(cur);
    const CqChunk none = {0, 0, 0};
    CqChunk next = run0 + 1 < run1 ? advance() : none, next2 = run0 + 2 < run1 ? advance() : none;
    load_ids(next);
    int kc = run0;
    // One chunk; `each` looks at the decays, delta x silu(z) and C of a token's states after their update.
    auto chunk = [&](auto each) {
        const int nt = min(CQ_TC, cur.len - cur.at);
        bad |= bad_next;
        // (1) causal depthwise convolution and SiLU
        float z[4], raw[CLS_MAX_CONV + 3];
#pragma unroll
        for (int j = 0; j < 4; ++j) nx[j] = take[j] ? nx[j] : 0.f, nz[j] = take[j] ? nz[j] : 0.f;
#pragma unroll
        for (int j = 0; j < 3; ++j) raw[j] = __shfl(tq == 3 ? px[j + 1] : nx[j + 1], (lane + 48) & 63, 64);
#pragma unroll
        for (int j = 0; j < 4; ++j) raw[3 + j] = px[j] = nx[j];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            float pre = cb;
#pragma unroll
            for (int j = 0; j < CLS_MAX_CONV; ++j) pre = fmaf(cw[j], raw[t + j], pre);
            z[t] = nz[t] * __builtin_amdgcn_rcpf(1.f + __expf(-nz[t]));
            s_x[(4 * tq + t) * sx + c] = pre * __builtin_amdgcn_rcpf(1.f + __expf(-pre));
        }
        gather(next); // the next chunk's rows fly while this one is worked on
        load_ids(next2);
        lds_sync();
        // (2) lane (token l % 16, channel l / 16 of four) against (channel, output l % 16); the result leaves tokens
        // 4 (l / 16) .. + 3 of output l % 16
        if (proj) {
            f32x4 acc = {0.f, 0.f, 0.f, 0.f}, acc2 = {0.f, 0.f, 0.f, 0.f};
            const float *xs = s_x + l16 * sx + tq + 4 * k_lo;
#pragma unroll
            for (int k = 0; k < per; k += 2) { // (two chains)
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(xs[4 * k], bw[k], acc, 0, 0, 0);
                acc2 = __builtin_amdgcn_mfma_f32_16x16x4f32(xs[4 * k + 4], bw[k + 1], acc2, 0, 0, 0);
            }
            float *dst = s_part + kq * CQ_TC * CQ_OUT + tq * 4 * CQ_OUT + tile * 16 + l16;
#pragma unroll
            for (int r = 0; r < 4; ++r) dst[r * CQ_OUT] = acc[r] + acc2[r];
        }
        lds_sync();
        for (int q = tid; q < CQ_TC * CQ_OUT; q += T) {
            float p = 0.f;
#pragma unroll
            for (int w = 0; w < nkq; ++w) p += s_part[w * CQ_TC * CQ_OUT + q];
            s_dbc[q / CQ_OUT * CQ_ROW + q % CQ_OUT] = p;
        }
        lds_sync();
        // (2), (1) step sizes
        f32x4 dt4 = {bdt, bdt, bdt, bdt};
#pragma unroll
        for (int k = 0; k < 4; ++k) dt4 = __builtin_amdgcn_mfma_f32_16x16x4f32(s_dbc[l16 * CQ_ROW + 4 * k + tq], bd[k], dt4, 0, 0, 0);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int row = 4 * tq + t;
            const float dt = dt4[t];
            // softplus = log1p(e^dt): log(u) e / (u - 1) with u = 1 + e undoes the rounding of u (steps are ~1e-3..0.1)
            const float ex = __expf(dt), u = 1.f + ex;
            const float delta = dt > 20.f ? dt : (u == 1.f ? ex : logf(u) * ex * __builtin_amdgcn_rcpf(u - 1.f));
            s_delta[row * sx + c] = delta;
            const float x = s_x[row * sx + c];
            s_dz[row * sx + c] = make_float2(delta * x, z[t]);
            if (row < nt) pooled_d = fmaf(x * D, z[t], pooled_d);
        }
        lds_sync();
        // (3) the state update, token by token, in this thread's registers
        const float *sd = s_delta + cs;
        const float2 *sz = s_dz + cs;
        const float *sb = s_dbc + 16 + sub * 4;
        auto token = [&](int t) {
            const float delta = sd[t * sx];
            const float2 dz = sz[t * sx];
            const float4 B = *(const float4 *)(sb + t * CQ_ROW), C = *(const float4 *)(sb + t * CQ_ROW + 16);
            float a[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) a[k] = __builtin_amdgcn_exp2f(delta * A[k]);
            h[0] = fmaf(a[0], h[0], dz.x * B.x);
            h[1] = fmaf(a[1], h[1], dz.x * B.y);
            h[2] = fmaf(a[2], h[2], dz.x * B.z);
            h[3] = fmaf(a[3], h[3], dz.x * B.w);
            const float acc = fmaf(C.w, h[3], fmaf(C.z, h[2], fmaf(C.y, h[1], C.x * h[0])));
            pooled = fmaf(acc, dz.y, pooled);
            each(a, C, dz.y);
        };
        int t = 0;
        for (; t + 4 <= nt; t += 4) { // (four tokens' operands in flight)
            token(t);
            token(t + 1);
            token(t + 2);
            token(t + 3);
        }
        for (; t < nt; ++t) token(t);
    };
    auto step = [&]() {
        ++kc;
        cur = next;
        next = next2;
        next2 = kc + 2 < run1 ? advance() : none;
    };
    // The part of a prompt that started in an earlier run (a loop of its own: in one with the other chunks, choosing the update
    // by a uniform test costs 60 register copies a chunk).
    if (head_part) {
        float P[4], G[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) P[k] = 1.f, G[k] = 0.f;
        bool more = true;
        while (more) {
            chunk([&](const float *a, const float4 &C, float z) {
#pragma unroll
                for (int k = 0; k < 4; ++k) P[k] *= a[k];
                G[0] = fmaf(C.x * z, P[0], G[0]);
                G[1] = fmaf(C.y * z, P[1], G[1]);
                G[2] = fmaf(C.z * z, P[2], G[2]);
                G[3] = fmaf(C.w * z, P[3], G[3]);
            });
            more = cur.at + CQ_TC < cur.len && kc + 1 < run1;
            step();
        }
        part_bad = __any(bad); // (every wave sees all token ids)
        cq_record(ws + cq_rec_at(nb, blockIdx.x, T) + tid, T, G, P, h, pooled, pooled_d);
    }
    // prompts from their start
    CqChunk last = start;
    bool open = false;
    while (kc < run1) {
        if (cur.at == 0) {
            bad = false;
            pooled = pooled_d = 0.f;
#pragma unroll
            for (int k = 0; k < 4; ++k) h[k] = px[k] = 0.f;
        }
        chunk([](const float *, const float4 &, float) {});
        last = cur;
        open = cur.at + CQ_TC < cur.len;
        if (!open) classifier_finish<DI>(v, cur.p, cur.len, pooled, pooled_d, __any(bad), s_pool, s_mean, s_logit, logits, draft_id);
        step();
    }
    // parts of cut prompts: the one the run starts inside, and the one it ends in
    if (!head_part && !open) return; // (uniform)
    if (open) {
        float *o = ws + cq_open_at(nb, blockIdx.x, T) + tid;
#pragma unroll
        for (int k = 0; k < 4; ++k) put(o + k * T, h[k]);
        put(o + 4 * T, pooled);
        put(o + 5 * T, pooled_d);
    }
    const bool open_bad = __any(bad);
    if (tid == 0) {
        put(ws + cq_bad_at(nb, blockIdx.x, T), part_bad ? 1.f : 0.f);
        put(ws + cq_bad_at(nb, blockIdx.x, T) + 1, open_bad ? 1.f : 0.f);
    }
    // (first and last blocks of the prompts: chunk numbers over the run's length)
    const int head_chunk = run0 - start.at / CQ_TC, tail_chunk = run1 - 1 - last.at / CQ_TC;
    const int head_b0 = head_chunk / run, head_b1 = (head_chunk + cls_chunks(start.len) - 1) / run;
    const int tail_b1 = (tail_chunk + cls_chunks(last.len) - 1) / run;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // every wave's stores have arrived
    __syncthreads();
    if (tid == 0) {
        unsigned long long *arrivals = (unsigned long long *)ws;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        s_last[0] = head_part && cq_arrive(arrivals + head_b0, tag, head_b1 - head_b0 + 1);
        s_last[1] = open && cq_arrive(arrivals + blockIdx.x, tag, tail_b1 - (int)blockIdx.x + 1);
        if (s_last[0] || s_last[1]) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
    if (s_last[0]) cq_join<DI>(v, start.p, start.len, head_b0, head_b1, nb, ws, s_pool, s_mean, s_logit, logits, draft_id);
    if (s_last[1]) cq_join<DI>(v, last.p, last.len, blockIdx.x, tail_b1, nb, ws, s_pool, s_mean, s_logit, logits, draft_id);
}

// ---------------------------------------------------------------- C ABI

extern "C" int sd_classifier_create(const sd_classifier_shape *s, const sd_classifier_weights *w, sd_classifier **out)
{
    if (!s || !w || !out) return sd_fail(SD_EINVAL, "sd_classifier_create: null argument");
    *out = nullptr;
    if (s->vocab < 1 || s->n_classes < 1 || s->n_classes > CLS_MAX_CLASSES)
        return sd_fail(SD_EINVAL, "sd_classifier_create: vocab >= 1 and 1 <= n_classes <= 64 required");
    if (s->d_model < 1 || s->d_model > CLS_MAX_MODEL || s->d_inner < 64 || s->d_inner > CLS_MAX_INNER || s->d_inner % 64)
        return sd_fail(SD_EINVAL, "sd_classifier_create: d_model in [1, 512] and d_inner a multiple of 64 in [64, 512] required");
    if (s->d_state < 1 || s->d_state > CLS_MAX_STATE || s->dt_rank < 1 || s->dt_rank > CLS_MAX_RANK || s->d_conv < 1 ||
        s->d_conv > CLS_MAX_CONV)
        return sd_fail(SD_EINVAL, "sd_classifier_create: d_state, dt_rank in [1, 16] and d_conv in [1, 4] required");
    const float *src[12] = {w->emb, w->w_in, w->conv_w, w->conv_b, w->w_x, w->w_dt, w->b_dt, w->a_log, w->d, w->w_out,
                            w->w_fc, w->b_fc};
    for (const float *p : src)
        if (!p) return sd_fail(SD_EINVAL, "sd_classifier_create: null weight pointer");
    const size_t J = (size_t)s->dt_rank + 2 * (size_t)s->d_state;
    const size_t lds_bytes = cls_lds_floats(s->d_inner, (int)J, s->d_model) * sizeof(float);
    if (lds_bytes > CLS_LDS_LIMIT)
        return sd_fail(SD_EINVAL, "sd_classifier_create: d_inner * (dt_rank + 2 d_state) does not fit the 64 KB of LDS "
                                  "the per-token projection is staged in");
    // slot 0 holds the table emb W_in, slot 1 the head W_out W_fc (emb and W_in go to a temporary allocation), the rest are
    // copies of the caller's arrays.
    const size_t cols = 2 * (size_t)s->d_inner;
    const size_t count[12] = {(size_t)s->vocab * cols, (size_t)s->n_classes * s->d_inner,
                              (size_t)s->d_inner * s->d_conv, (size_t)s->d_inner, (size_t)s->d_inner * J,
                              (size_t)s->dt_rank * s->d_inner, (size_t)s->d_inner, (size_t)s->d_inner * s->d_state,
                              (size_t)s->d_inner, (size_t)s->d_inner * s->d_model, (size_t)s->n_classes * s->d_model,
                              (size_t)s->n_classes};
    size_t total = 0, off[12];
    for (int k = 0; k < 12; ++k) { off[k] = total; total += (count[k] * sizeof(float) + 255) & ~(size_t)255; }
    const size_t emb_bytes = (size_t)s->vocab * s->d_model * sizeof(float), emb_slot = (emb_bytes + 255) & ~(size_t)255;
    const size_t win_bytes = (size_t)s->d_model * cols * sizeof(float);

    sd_classifier *c = new sd_classifier();
    c->v.vocab = s->vocab; c->v.d_model = s->d_model; c->v.d_inner = s->d_inner; c->v.d_state = s->d_state;
    c->v.dt_rank = s->dt_rank; c->v.d_conv = s->d_conv; c->v.n_classes = s->n_classes;
    c->lds_bytes = lds_bytes;
    c->mem = nullptr;
    void *tmp = nullptr;
    hipError_t e = hipGetDevice(&c->device);
    if (e == hipSuccess) e = hipMalloc(&c->mem, total);
    if (e == hipSuccess) e = hipMalloc(&tmp, emb_slot + win_bytes);
    const float **dst[12] = {&c->v.table, &c->v.w_head, &c->v.conv_w, &c->v.conv_b, &c->v.w_x, &c->v.w_dt, &c->v.b_dt,
                             &c->v.a_log, &c->v.d, &c->v.w_out, &c->v.w_fc, &c->v.b_fc};
    for (int k = 0; k < 12 && e == hipSuccess; ++k) {
        *dst[k] = (const float *)((char *)c->mem + off[k]);
        if (k >= 2) e = hipMemcpy((char *)c->mem + off[k], src[k], count[k] * sizeof(float), hipMemcpyHostToDevice);
    }
    if (e == hipSuccess) e = hipMemcpy(tmp, w->emb, emb_bytes, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy((char *)tmp + emb_slot, w->w_in, win_bytes, hipMemcpyHostToDevice);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(classifier_table_kernel, dim3(s->vocab), dim3(256), 0, (hipStream_t)0, (const float *)tmp,
                           (const float *)((char *)tmp + emb_slot), s->d_model, (int)cols, (float *)c->mem);
        hipLaunchKernelGGL(classifier_head_kernel, dim3(s->n_classes), dim3(256), 0, (hipStream_t)0, c->v.w_out, c->v.w_fc, s->d_inner,
                           s->d_model, (float *)c->v.w_head);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (tmp) (void)hipFree(tmp);
    if (e != hipSuccess) {
        if (c->mem) (void)hipFree(c->mem);
        delete c;
        return sd_fail(SD_EHIP, std::string("sd_classifier_create: ") + hipGetErrorString(e));
    }
    *out = c;
    return SD_OK;
}

extern "C" void sd_classifier_destroy(sd_classifier *c)
{
    if (!c) return;
    (void)hipFree(c->mem);
    delete c;
}

// Blocks of classifier_run_kernel for a call with a workspace (0: the call has no use for it).
static int cq_blocks(const sd_classifier *c, int32_t n, int32_t max_len)
{
    if (c->v.d_inner > 192 || (max_len <= CQ_TC && n <= CQ_BLOCKS)) return 0; // (no form for it; nothing to deal out)
    const int64_t chunks = (int64_t)n * ((max_len + (int64_t)CQ_TC - 1) / CQ_TC);
    if (chunks > 1 << 30) return 0; // (chunk numbers are 32 bits)
    return (int)std::min<int64_t>(CQ_BLOCKS, chunks);
}

extern "C" int64_t sd_classifier_workspace(const sd_classifier *c, int32_t n, int32_t max_len)
{
    if (!c || n < 1 || max_len < 1) return sd_fail(SD_EINVAL, "sd_classifier_workspace: null classifier or non-positive size");
    const int nb = cq_blocks(c, n, max_len);
    return nb ? (int64_t)cq_bad_at(nb, nb, 4 * c->v.d_inner) * (int64_t)sizeof(float) + 4 : 0; // (4: to align the arrivals)
}

// A number of 48 bits (in the upper ones) that no other call's has but by chance: the workspace of a call may hold what any
// other has left there.
static unsigned long long cq_call_tag()
{
    static std::atomic<unsigned long long> calls{(unsigned long long)std::chrono::steady_clock::now().time_since_epoch().count()};
    unsigned long long x = calls.fetch_add(1, std::memory_order_relaxed) * 0x9E3779B97F4A7C15ull; // (Weyl sequence, mixed as in splitmix64)
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    x = (x ^ (x >> 31)) & ~0xffffull;
    return x ? x : 1ull << 63;
}

static int route_classifier(const char *who, const sd_classifier *c, const int32_t *tokens, const int32_t *lens, int32_t n,
                            int32_t max_len, float *logits, int32_t *draft_id, float *ws, void *stream)
{
    if (!c || !tokens || !lens || !draft_id) return sd_fail(SD_EINVAL, std::string(who) + ": null argument");
    if (n < 1 || max_len < 1) return sd_fail(SD_EINVAL, std::string(who) + ": non-positive size");
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev != c->device)
        return sd_fail(SD_EINVAL, std::string(who) + ": the classifier was created on another device");
    const int nb = ws ? cq_blocks(c, n, max_len) : 0;
    // Up to 192 channels the four-threads-per-channel kernel is ahead at every batch and prompt length measured (thread per
    // channel -> this, us): 192 channels, one prompt of 128 tokens 124 -> 44, 4096 ragged ones 378 -> 298, 4096 of 16 tokens
    // 191 -> 168, 2000 of 512 tokens 1772 -> 1213; 64 channels 127 -> 30, 198 -> 92, 71 -> 45, 586 -> 381.  At 256 channels
    // its 16 waves no longer share the projection out evenly, above that its block would exceed 1024 threads.
#define SD_QUAD(DI)                                                                                                           \
    do {                                                                                                                      \
        if (!nb)                                                                                                              \
            hipLaunchKernelGGL(classifier_quad_kernel<DI>, dim3(n), dim3(4 * DI), cq_lds_floats(DI, c->v.d_model) * sizeof(float), \
                               (hipStream_t)stream, c->v, tokens, lens, max_len, logits, draft_id);                           \
        else {                                                                                                                \
            hipLaunchKernelGGL(classifier_run_kernel<DI>, dim3(nb), dim3(4 * DI), 0, (hipStream_t)stream, c->v, tokens, lens, \
                               n, max_len, logits, draft_id, ws, tag);                                                        \
        }                                                                                                                     \
    } while (0)
    ws = (float *)(((uintptr_t)ws + 7) & ~(uintptr_t)7);
    const unsigned long long tag = nb ? cq_call_tag() : 0;
    if (c->v.d_inner == 64) SD_QUAD(64);
    else if (c->v.d_inner == 128) SD_QUAD(128);
    else if (c->v.d_inner == 192) SD_QUAD(192);
    else
        hipLaunchKernelGGL(classifier_kernel, dim3(n), dim3(c->v.d_inner), c->lds_bytes, (hipStream_t)stream, c->v, tokens,
                           lens, max_len, logits, draft_id);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return sd_fail(SD_EHIP, std::string(who) + ": " + hipGetErrorString(e));
    return SD_OK;
}

extern "C" int sd_route_classifier(const sd_classifier *c, const int32_t *tokens, const int32_t *lens, int32_t n,
                                   int32_t max_len, float *logits, int32_t *draft_id, void *stream)
{
    return route_classifier("sd_route_classifier", c, tokens, lens, n, max_len, logits, draft_id, nullptr, stream);
}

extern "C" int sd_route_classifier_ws(const sd_classifier *c, const int32_t *tokens, const int32_t *lens, int32_t n,
                                      int32_t max_len, float *logits, int32_t *draft_id, float *workspace, void *stream)
{
    return route_classifier("sd_route_classifier_ws", c, tokens, lens, n, max_len, logits, draft_id, workspace, stream);
}

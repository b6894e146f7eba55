// bf16 weight-streaming GEMMs: C[M][N] = A[M][K] . W[N][K]^T for the decoder's linear layers.
//
// At batch 1 (M = gamma+1 verify rows, or one draft row) the work is reading each
// weight once from HBM, so the kernels are organised around the weight stream and
// the matrix cores only keep the ALUs out of the way; at batch 32-64 (M = 192-576)
// the same weight stream feeds enough rows for the matrix cores to matter.
//
//  * weights are stored in 16-row x 128-element tiles in MFMA operand order, so each
//    of the four load instructions of a K step reads one contiguous kilobyte straight
//    into operand registers (v_mfma_f32_16x16x32_bf16: lane l supplies row l%16,
//    k-group l/16).  Row-major weights would spread every such load over 16 rows 2K
//    bytes apart, which lands on one L2 channel and limits a compute unit to about a
//    third of the rate it reaches on the tiles;
//  * activations are two bf16 planes (hi + lo, ~16 mantissa bits).  For M <= 8 both
//    planes ride in ONE operand: MFMA columns 0..7 carry the hi rows, columns 8..15
//    the lo rows, and the epilogue adds the two halves; for larger M every weight
//    fragment is multiplied twice;
//  * few rows (gemm_ksplit_kernel up to 8 rows or where the norm is split, gemm_wide_kernel
//    from 9 to 16, and to 64 in layers narrower than 4096): the waves of a block split K, fetch their
//    activation fragments straight from L2 and meet in LDS - no barrier in the K loop;
//    17 to 96 rows of wide layers (gemm_lds_kernel): weights and rows staged through LDS;
//    more rows (gemm_tile_kernel): row blocks share a staged activation chunk in LDS;
//  * results leave either directly (store; SwiGLU: silu(gate)*up split to bf16
//    hi/lo) or as fp32 partial sums per K split, which the consuming kernel adds in
//    a fixed order (the fused attention prologue for QKV, add_rmsnorm for the residual
//    GEMMs), so results are bit-reproducible run to run.
//
// Paper (arXiv 2505.08600): Section 1, Figure 1 (draft steps and the parallel
// verify pass whose linear layers these are); Section 3.1 (LLaMA blocks).
#include "lora.h"
#include "sd_internal.h"

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

// Pins the program order of the memory operations around it, for the optimiser and the scheduler alike.
#define SD_ORDER()                          \
    do {                                    \
        asm volatile("" ::: "memory");       \
        __builtin_amdgcn_sched_barrier(0);  \
    } while (0)
#define GS_PAD 8 // row padding in LDS (16 bytes): operand rows fall into distinct banks

// Row-blocked GEMM for M > 32 (batched verify, prefill chunks of many sequences).
// MODE: GEMM_STORE (C = acc, or partial sums when grid.y > 1) / GEMM_SWIGLU (the block's WAVES * NT tiles are,
// alternately, the gate and the up tile of WAVES * NT / 2 groups of 16 output columns; tile q belongs to wave
// q / NT, so with an odd NT every second pair straddles two waves and the gate accumulators change wave
// through LDS before the epilogue; a last block may hold fewer pairs than the others).  A block owns BM rows (hi plane in operand rows 0..BM-1, lo
// plane in BM..2BM-1 of the staged chunk) and WAVES * NT 16-column weight tiles; every wave keeps its NT
// weight fragments of a 128-element K step in registers (loaded straight from the tiled weights, two steps
// in flight) and all waves share the activation chunk, staged once per block in LDS (double buffered).
// The row blocks of one column tile re-read the same weights, so they are mapped to the SAME XCD and to
// adjacent dispatch slots: block id = xcd + 8 * (row block + n_mblocks * (tile / 8)); the re-reads then
// hit that XCD's L2 and HBM still sees every weight once.  The grid is padded to a multiple of 8 tiles.
template <int MODE, int BM, int KC, int NT, int WAVES, int NB>
__global__ __launch_bounds__(WAVES * 64) void gemm_tile_kernel(const uint16_t *A, ActView a_av,
                                                               WeightSeg w, int M, int N, int K, int k_per_split,
                                                               int n_mblocks, int n_ntiles, float *__restrict__ C,
                                                               size_t c_split_stride, uint16_t *__restrict__ Cact,
                                                               ActView c_av)
{
    constexpr int MT = BM / 16;      // 16-row tiles of A
    constexpr int OPROWS = 2 * BM;   // staged operand rows (hi | lo)
    constexpr int NI = KC / 32;      // MFMA k-groups per chunk (KC = 128: a whole K step, 64: half of one)
    static_assert(KC == 64 || KC == 128, "chunk is a K step or half of one");
    constexpr int LDROW = KC + GS_PAD;
    constexpr int THREADS = WAVES * 64;
    constexpr int VEC_PER_ROW = KC / 8; // 16-byte vectors per operand row
    constexpr int NVEC = OPROWS * VEC_PER_ROW;
    constexpr int LPT = NVEC / THREADS;
    static_assert(NVEC % THREADS == 0, "staging must divide evenly");
    constexpr bool SW = MODE == GEMM_SWIGLU;
    constexpr bool XCH = SW && (NT & 1); // gate/up pairs straddle waves
    static_assert(!SW || (NT * WAVES) % 2 == 0, "gate and up tiles come in pairs");
    constexpr int COLS = SW ? NT * WAVES * 8 : NT * 16 * WAVES; // output columns of a block
    __shared__ __attribute__((aligned(16))) uint16_t sA[2][OPROWS][LDROW];
    __shared__ f32x4 xch[XCH ? WAVES * MT * 64 : 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row = lane & 15, grp = lane >> 4;
    const int r8 = blockIdx.x >> 3;
    const int mblk = r8 % n_mblocks;
    const int ntile = (r8 / n_mblocks) * 8 + (blockIdx.x & 7);
    if (ntile >= n_ntiles) return; // padded grid
    const int n0 = ntile * COLS;
    const int m0 = mblk * BM;
    const int kb = blockIdx.y * k_per_split;
    const int ke = min(K, kb + k_per_split);
    const int nchunks = (ke - kb) / KC; // k_per_split and K are multiples of 128
    // this lane's 16 bytes inside the first K step of each of the wave's weight tiles
    const size_t tile_elems = (size_t)(K >> 7) * 2048;
    const uint16_t *Wp[NT];
    if (SW) {
        const int last_pair = N / 16 - 1; // pairs past the end (last block) re-read the last one; never stored
#pragma unroll
        for (int c = 0; c < NT; c++) {
            const int q = wave * NT + c;
            Wp[c] = (const uint16_t *)w.p[q & 1] + (size_t)min(n0 / 16 + (q >> 1), last_pair) * tile_elems +
                    (size_t)(kb >> 7) * 2048 + lane * 8;
        }
    } else {
        const int seg_tiles = w.n_per_seg / 16; // a block's tiles may lie in different segments (q | k | v)
#pragma unroll
        for (int c = 0; c < NT; c++) {
            const int tile = n0 / 16 + wave * NT + c;
            const int seg = tile / seg_tiles;
            const uint16_t *base = (const uint16_t *)(seg == 0 ? w.p[0] : seg == 1 ? w.p[1] : w.p[2]);
            Wp[c] = base + (size_t)(tile - seg * seg_tiles) * tile_elems + (size_t)(kb >> 7) * 2048 + lane * 8;
        }
    }
    // cooperative staging of the activation chunk: vector v -> operand row v / VEC_PER_ROW.  Rows past M
    // are loaded like any other (the buffers are over-allocated by SD_ACT_PAD_ROWS rows, so the addresses
    // are valid); whatever they hold only reaches accumulator rows that are never stored.
    uint32_t a_off[LPT];
    int a_dst[LPT];
#pragma unroll
    for (int j = 0; j < LPT; j++) {
        const int v = threadIdx.x + j * THREADS;
        const int orow = v / VEC_PER_ROW, ov = v % VEC_PER_ROW;
        a_off[j] = (uint32_t)((orow < BM ? 0 : a_av.plane) + (size_t)(m0 + orow % BM) * 128 + ov * 8);
        a_dst[j] = orow * LDROW + ov * 8;
    }
    const size_t step_stride = (size_t)a_av.rows * 128; // step-major activations
    // Loads for chunks past the end of the K range (issued by the last iterations so that every
    // iteration issues the same loads, which keeps the compiler's outstanding-load counts exact)
    // re-read the last chunk; their data is never used.
    bf16x8 a_reg[LPT];
    auto a_fetch = [&](int chunk) {
        const int k0 = min(chunk, nchunks - 1) * KC; // offset inside this block's K range
        const uint16_t *base = A + ((size_t)(kb >> 7) + (k0 >> 7)) * step_stride + (k0 & 127);
#pragma unroll
        for (int j = 0; j < LPT; j++) a_reg[j] = *(const bf16x8 *)(base + a_off[j]);
    };
    auto a_commit = [&](int buf) {
#pragma unroll
        for (int j = 0; j < LPT; j++) *(bf16x8 *)(&sA[buf][0][0] + a_dst[j]) = a_reg[j];
    };
    f32x4 acc[NT][MT];
#pragma unroll
    for (int c = 0; c < NT; c++)
#pragma unroll
        for (int t = 0; t < MT; t++) acc[c][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    bf16x8 wv[NB][NT][NI];
    auto w_issue = [&](int chunk, int b) {
        const int cc = min(chunk, nchunks - 1);
#pragma unroll
        for (int c = 0; c < NT; c++)
#pragma unroll
            for (int i = 0; i < NI; i++) wv[b][c][i] = *(const bf16x8 *)(Wp[c] + ((size_t)cc * NI + i) * 512);
    };
    // Activation fragments: two register sets used alternately by the MFMA groups of a chunk (group i
    // contracts elements 32*i .. 32*i+31 and reads set i & 1); the fragments of group i+1 are read from LDS
    // while group i runs.
    static_assert(NI % 2 == 0, "the last MFMA group of a chunk uses fragment set 1");
    bf16x8 fh[2][MT], fl[2][MT];
    auto frags = [&](int lb, int i, int fb) {
        const uint16_t *sa = &sA[lb][0][0] + row * LDROW + grp * 8;
#pragma unroll
        for (int t = 0; t < MT; t++) {
            fh[fb][t] = *(const bf16x8 *)(sa + t * 16 * LDROW + i * 32);
            fl[fb][t] = *(const bf16x8 *)(sa + (BM + t * 16) * LDROW + i * 32);
        }
    };
    auto mfma_group = [&](int b, int i) {
#pragma unroll
        for (int t = 0; t < MT; t++) {
#pragma unroll
            for (int c = 0; c < NT; c++)
                acc[c][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv[b][c][i], fh[i & 1][t], acc[c][t], 0, 0, 0);
#pragma unroll
            for (int c = 0; c < NT; c++)
                acc[c][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv[b][c][i], fl[i & 1][t], acc[c][t], 0, 0, 0);
        }
    };
    // Pipeline, iteration ch (weight buffer b = ch % NB):
    //   1. the activation rows of chunk ch+1 (fetched into registers during iteration ch-1) go to the
    //      other LDS buffer;
    //   2. chunk ch is multiplied, and in between its MFMAs the loads of later chunks are issued: the
    //      activation rows of chunk ch+2 first, then the weights of chunk ch+NB-1 into the buffer that
    //      iteration ch-1 released (so NB-1 weight chunks are in flight or in use at any time);
    //   3. barrier.  With EARLY the barrier stands before the last MFMA group instead, and the first
    //      fragments of chunk ch+1 are read from LDS behind it, under that group's MFMAs: no MFMA then
    //      waits for the LDS round trip that follows a barrier (it costs 8 more registers of live range,
    //      which only the 3-tile shape has to spare).
    // Every iteration issues the same loads in the same order, activation rows before weights: waiting
    // for the rows never waits for the (much slower) weight stream, and the wait counts stay exact.
    constexpr bool EARLY = BM == 96 && NT == 3;
    a_fetch(0);
    SD_ORDER();
    w_issue(0, 0);
    SD_ORDER();
    a_commit(0);
    a_fetch(1);
    SD_ORDER();
#pragma unroll
    for (int b = 1; b < NB - 1; b++) w_issue(b, b);
    SD_ORDER();
    __syncthreads();
    if (EARLY) {
        frags(0, 0, 0);
        SD_ORDER();
    }
    auto chunk = [&](int ch, int b) {
        a_commit((ch + 1) & 1);
        SD_ORDER();
        a_fetch(ch + 2);
        w_issue(ch + NB - 1, (b + NB - 1) % NB);
        if (!EARLY) frags(ch & 1, 0, 0);
#pragma unroll
        for (int i = 0; i < (EARLY ? NI - 1 : NI); i++) {
            if (i < NI - 1) frags(ch & 1, i + 1, (i + 1) & 1);
            mfma_group(b, i);
        }
        // instruction order of this stretch: (the LDS reads of the first fragment group, then) one
        // global load (activation rows first) and one LDS read after every third MFMA
        if (!EARLY) __builtin_amdgcn_sched_group_barrier(0x100, 2 * MT, 0);
#pragma unroll
        for (int k = 0; k < (NT * MT * 2 * (EARLY ? NI - 1 : NI)) / 3; k++) {
            __builtin_amdgcn_sched_group_barrier(0x008, 3, 0); // MFMA
            if (k < LPT + NT * NI) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);     // VMEM read
            if (k < 2 * MT * (NI - 1)) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0); // DS read
        }
        SD_ORDER();
        __syncthreads();
        if (EARLY) {
            frags((ch + 1) & 1, 0, 0); // (after the last chunk: a stale buffer, never used)
            mfma_group(b, NI - 1);
#pragma unroll
            for (int k = 0; k < (NT * MT * 2) / 3; k++) {
                __builtin_amdgcn_sched_group_barrier(0x008, 3, 0); // MFMA
                if (k < 2 * MT) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0); // DS read
            }
            SD_ORDER();
        }
    };
    // whole rounds of NB chunks in one loop with a single exit (exits inside the unrolled round make the register
    // allocator copy accumulators from round to round), then the at most NB - 1 chunks that remain
    const int n_main = nchunks / NB * NB;
    for (int ch0 = 0; ch0 < n_main; ch0 += NB) {
#pragma unroll
        for (int b = 0; b < NB; b++) chunk(ch0 + b, b);
    }
#pragma unroll
    for (int b = 0; b < NB - 1; b++)
        if (n_main + b < nchunks) chunk(n_main + b, b);
    // epilogue: lane (m' = row, grp) holds D[n = 4*grp + r][m'] of each of its tiles
    f32x4 gin[MT]; // gate accumulators of the pair whose up tile is this wave's first tile
#pragma unroll
    for (int t = 0; t < MT; t++) gin[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    if (XCH) { // xch is used nowhere else; every wave is past the loop's last barrier
        if (((wave * NT + NT - 1) & 1) == 0) {
#pragma unroll
            for (int t = 0; t < MT; t++) xch[(wave * MT + t) * 64 + lane] = acc[NT - 1][t];
        }
        __syncthreads();
        if ((wave * NT) & 1) {
#pragma unroll
            for (int t = 0; t < MT; t++) gin[t] = xch[((wave - 1) * MT + t) * 64 + lane];
        }
    }
#pragma unroll
    for (int t = 0; t < MT; t++) {
        const int m = m0 + t * 16 + row;
        if (m >= M) continue;
        if (SW) {
#pragma unroll
            for (int c = 0; c < NT; c++) { // the wave that holds a pair's up tile writes the pair
                const int q = wave * NT + c;
                const int n = n0 + (q >> 1) * 16;
                if (!(q & 1) || n >= N) continue;
                const f32x4 g = c > 0 ? acc[c > 0 ? c - 1 : 0][t] : gin[t];
                const size_t o = act_index(c_av, m, n + 4 * grp, N); // 4 columns inside one K step: contiguous
                float y[4];
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    const float g0 = g[r];
                    y[r] = g0 / (1.0f + expf(-g0)) * acc[c][t][r];
                }
                uint32_t h0, l0, h1, l1;
                bf16x2_split(y[0], y[1], h0, l0);
                bf16x2_split(y[2], y[3], h1, l1);
                *(uint2 *)(Cact + o) = make_uint2(h0, h1);
                *(uint2 *)(Cact + c_av.plane + o) = make_uint2(l0, l1);
            }
        } else {
            float *Cs = C + (size_t)blockIdx.y * c_split_stride;
#pragma unroll
            for (int c = 0; c < NT; c++) {
                const size_t o = (size_t)m * N + n0 + (wave * NT + c) * 16 + 4 * grp;
                *(f32x4 *)(Cs + o) = acc[c][t];
            }
        }
    }
}

// K range per split (a multiple of 128) and the number of splits that actually results
static void split_geometry(int K, int ks, int *kps, int *ny)
{
    if (ks < 1) ks = 1;
    if (K < 128) K = 128;
    *kps = ((K / 128 + ks - 1) / ks) * 128;
    *ny = (K + *kps - 1) / *kps;
}

// Few-row GEMM with the K range split over the 4 waves of a block (and optionally over grid.y).
// A block owns NTW 16-column tiles of NMAT matrices: NMAT = 1 stores fp32 sums (one slab per grid.y
// split), NMAT = 2 is the gate/up pair of the same columns with the SwiGLU epilogue (silu(gate)*up needs
// complete sums, so there grid.y is 1).  The waves interleave the 128-element K steps, fetch their
// activation fragments straight from global memory (L2) - no barrier inside the K loop - and keep the
// loads of U steps in flight in registers; the four partial accumulators meet in LDS.
template <int NMAT, bool PACKED, int MT, int U, int NTW, bool NT_HINT, int WAVES = 4>
__global__ __launch_bounds__(WAVES * 64) void gemm_ksplit_kernel(const uint16_t *__restrict__ A, ActView a_av, WeightSeg w,
                                                          int M, int N, int K, int steps_per_split,
                                                          float *__restrict__ C, size_t c_split_stride,
                                                          uint16_t *__restrict__ Cact, ActView c_av, LmStats ls,
                                                          NormFold nf)
{
    constexpr int THREADS = WAVES * 64;
    constexpr int NW = NMAT * NTW; // weight tiles per wave and step
    __shared__ float red[WAVES][NW][MT][64][4];
    __shared__ float s_inv[32]; // consumer side of a split norm: 1 / rms of every output row
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row = lane & 15, grp = lane >> 4;
    const int n0 = blockIdx.x * 16 * NTW;
    // tiled weights: step st of a tile starts 2048*st elements after the tile, instruction i of a step
    // 512*i after that; tile j of matrix c is Wp[c] + j * tile_elems
    const size_t tile_elems = (size_t)(K >> 7) * 2048;
    const uint16_t *Wp[NMAT];
    if (NMAT == 2) {
#pragma unroll
        for (int c = 0; c < NMAT; c++) Wp[c] = (const uint16_t *)w.p[c] + (size_t)(n0 / 16) * tile_elems + lane * 8;
    } else {
        const int seg = n0 / w.n_per_seg;
        Wp[0] = (const uint16_t *)w.p[seg] + (size_t)((n0 - seg * w.n_per_seg) / 16) * tile_elems + lane * 8;
    }
    const uint16_t *Ap[MT], *Al[MT];
    bool a_live[MT];
#pragma unroll
    for (int t = 0; t < MT; t++) {
        const int m = PACKED ? (row & 7) : t * 16 + row;
        a_live[t] = m < M;
        const int src = !a_live[t] ? 0 : nf.row_map ? nf.row_map[m] : m;
        // step-major activations: row m of K step st starts at (st * rows + m) * 128
        Ap[t] = A + ((PACKED && row >= 8) ? a_av.plane : 0) + (size_t)src * 128 + grp * 8;
        Al[t] = Ap[t] + a_av.plane;
    }
    constexpr int ROWS_MAX = PACKED ? 8 : 16 * MT;
    constexpr int SSR = (ROWS_MAX + WAVES - 1) / WAVES, SSB = SD_NORMFOLD_MAX_BLOCKS / 256; // (a lane loads 4 entries at once)
    constexpr int EPI = (16 * NTW * ROWS_MAX + THREADS - 1) / THREADS; // epilogue elements per thread
    float4 ssl[SSR][SSB]; // consumer side of a split norm: wave w sums the producer's per-block shares of rows w, w + 4, ...
    int ss_src[SSR];
    float xres[EPI], gval[EPI]; // producer side: residual and gain of this thread's epilogue elements
    if (nf.ss_in) {
#pragma unroll
        for (int r = 0; r < SSR; r++) {
            const int m = wave + r * WAVES;
            ss_src[r] = m < M ? (nf.row_map ? nf.row_map[m] : m) : 0;
        }
    }
    const size_t step_stride = (size_t)a_av.rows * 128;
    f32x4 acc[NW][MT];
#pragma unroll
    for (int c = 0; c < NW; c++)
#pragma unroll
        for (int t = 0; t < MT; t++) acc[c][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const int s_begin = blockIdx.y * steps_per_split;
    const int s_end = min(K / 128, s_begin + steps_per_split);
    const bf16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
    // U register buffers: the loads of the wave's next U-1 steps are in flight while one step is consumed
    bf16x8 wv[U][NW][4], av[U][MT][4], al[U][PACKED ? 1 : MT][4];
    auto issue = [&](int st, int b) {
#pragma unroll
        for (int t = 0; t < MT; t++)
#pragma unroll
            for (int i = 0; i < 4; i++) {
                av[b][t][i] = a_live[t] ? *(const bf16x8 *)(Ap[t] + step_stride * st + i * 32) : zero;
                if (!PACKED) al[b][t][i] = a_live[t] ? *(const bf16x8 *)(Al[t] + step_stride * st + i * 32) : zero;
            }
#pragma unroll
        for (int c = 0; c < NW; c++)
#pragma unroll
            for (int i = 0; i < 4; i++)
                wv[b][c][i] = ld_stream<NT_HINT>((const bf16x8 *)(Wp[c % NMAT] + (size_t)(c / NMAT) * tile_elems + (size_t)st * 2048 + i * 512));
    };
    // the small loads of a split norm go out ahead of the weight stream (loads return in order: behind the
    // first weight loads they would hold up everything issued after them for as long as they take) and are used
    // after the K loop; every address is clamped into range, so the loads are unconditional
    if (nf.ss_in) { // (uniform)
#pragma unroll
        for (int r = 0; r < SSR; r++)
#pragma unroll
            for (int i = 0; i < SSB; i++) // (entries past ss_nb are stale or never written: masked when summed)
                ssl[r][i] = *(const float4 *)(nf.ss_in + ss_src[r] * SD_NORMFOLD_MAX_BLOCKS + 4 * (lane + 64 * i));
    }
    if (NMAT == 1 && nf.x) { // (uniform)
#pragma unroll
        for (int k = 0; k < EPI; k++) {
            const int e = threadIdx.x + THREADS * k;
            const int m = min(e / (16 * NTW), M - 1), n = n0 + (e & (16 * NTW - 1));
            xres[k] = nf.x[(size_t)m * N + n];
            gval[k] = nf.g[n];
        }
    }
#pragma unroll
    for (int u = 0; u < U; u++)
        if (s_begin + wave + u * WAVES < s_end) issue(s_begin + wave + u * WAVES, u);
    // The wave's rows of 1 / rms: summed once its first K step has been consumed - the small loads went out
    // before that step's and have therefore arrived - so that nothing of it is left for the block's tail.
    bool ss_pending = nf.ss_in != nullptr;
    auto ss_reduce = [&]() {
#pragma unroll
        for (int r = 0; r < SSR; r++) {
            float a = 0.f;
#pragma unroll
            for (int i = 0; i < SSB; i++) {
                const int b = 4 * (lane + 64 * i);
                a += b < nf.ss_nb ? ssl[r][i].x : 0.f;
                a += b + 1 < nf.ss_nb ? ssl[r][i].y : 0.f;
                a += b + 2 < nf.ss_nb ? ssl[r][i].z : 0.f;
                a += b + 3 < nf.ss_nb ? ssl[r][i].w : 0.f;
            }
            a = wave_sum_dpp(a);
            const int m = wave + r * WAVES;
            if (lane == 0 && m < ROWS_MAX) s_inv[m] = 1.0f / sqrtf(a / (float)K + nf.eps);
        }
        ss_pending = false;
    };
    for (int s = s_begin + wave; s < s_end; s += U * WAVES) {
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int cur = s + u * WAVES;
            if (cur < s_end) {
#pragma unroll
                for (int i = 0; i < 4; i++)
#pragma unroll
                    for (int t = 0; t < MT; t++)
#pragma unroll
                        for (int c = 0; c < NW; c++) {
                            acc[c][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv[u][c][i], av[u][t][i], acc[c][t], 0, 0, 0);
                            if (!PACKED)
                                acc[c][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv[u][c][i], al[u][t][i], acc[c][t], 0, 0, 0);
                        }
                if (cur + U * WAVES < s_end) issue(cur + U * WAVES, u);
                if (u == 0 && ss_pending) ss_reduce(); // (uniform; true in the first round only)
            }
        }
    }
#pragma unroll
    for (int c = 0; c < NW; c++)
#pragma unroll
        for (int t = 0; t < MT; t++)
#pragma unroll
            for (int r = 0; r < 4; r++) red[wave][c][t][lane][r] = acc[c][t][r];
    if (ss_pending) ss_reduce(); // (a wave without a K step of its own)
    __syncthreads();
    // tile element D[n = 4*(slot/16) + r][m' = slot%16] sits at red[.][c][t][slot][r]
    constexpr int ROWS = PACKED ? 8 : 16 * MT;
    for (int e = threadIdx.x, ek = 0; e < 16 * NTW * ROWS; e += THREADS, ek++) {
        const int nn = e & 15, j = (e >> 4) % NTW, m = e / (16 * NTW);
        if (m >= M) continue;
        const int t = PACKED ? 0 : m >> 4;
        const int slot = (nn >> 2) * 16 + (m & 15), r = nn & 3;
        float v[NMAT];
#pragma unroll
        for (int c = 0; c < NMAT; c++) {
            v[c] = 0.f;
#pragma unroll
            for (int wv2 = 0; wv2 < WAVES; wv2++) {
                v[c] += red[wv2][j * NMAT + c][t][slot][r];
                if (PACKED) v[c] += red[wv2][j * NMAT + c][t][slot + 8][r];
            }
            if (nf.ss_in) v[c] *= s_inv[m];
        }
        if (NMAT == 1 && nf.x) { // (uniform) producer side of a split norm; the launcher rules out K splits
            const int n = n0 + j * 16 + nn;
            float xr = xres[0], gg = gval[0];
#pragma unroll
            for (int k = 1; k < EPI; k++)
                if (k == ek) xr = xres[k], gg = gval[k];
            const float xn = xr + v[0];
            nf.x[(size_t)m * N + n] = xn;
            const float y = xn * gg;
            const uint16_t hi = bf16_bits_rne(y);
            const size_t o = act_index(c_av, m, n, N);
            Cact[o] = hi;
            Cact[c_av.plane + o] = bf16_bits_rne(y - __uint_as_float((uint32_t)hi << 16));
            float sq = row16_sum(xn * xn); // the block's 16 * NTW columns of row m sit in adjacent lanes
            if (NTW == 2) sq += __shfl_xor(sq, 16, 64);
            if ((e & (16 * NTW - 1)) == 0) nf.ss_out[m * SD_NORMFOLD_MAX_BLOCKS + blockIdx.x] = sq;
            continue;
        }
        if (NMAT == 2) {
            const float y = v[0] / (1.0f + expf(-v[0])) * v[NMAT - 1];
            const uint16_t hi = bf16_bits_rne(y);
            const size_t o = act_index(c_av, m, n0 + j * 16 + nn, N);
            Cact[o] = hi;
            Cact[c_av.plane + o] = bf16_bits_rne(y - __uint_as_float((uint32_t)hi << 16));
        } else {
            C[(size_t)blockIdx.y * c_split_stride + (size_t)m * N + n0 + j * 16 + nn] = v[0];
            if (NTW == 2 && ls.p) { // (uniform) the block's 32 columns of row m sit in the 32 lanes of a half wave
                float mx = v[0];
                int ai = n0 + j * 16 + nn;
#pragma unroll
                for (int o = 16; o > 0; o >>= 1) {
                    const float ov = __shfl_xor(mx, o, 64);
                    const int oi = __shfl_xor(ai, o, 64);
                    if (ov > mx || (ov == mx && oi < ai)) {
                        mx = ov;
                        ai = oi;
                    }
                }
                float ex = ls.invT > 0.f ? expf((v[0] - mx) * ls.invT) : 0.f;
#pragma unroll
                for (int o = 16; o > 0; o >>= 1) ex += __shfl_xor(ex, o, 64);
                if ((e & 31) == 0) {
                    float *sp = ls.p + ((size_t)m * gridDim.x + blockIdx.x) * 3;
                    sp[0] = mx;
                    sp[1] = ex;
                    sp[2] = __int_as_float(ai);
                }
            }
        }
    }
}

// Wide few-row GEMM (9 to 16 rows, to 64 where gemm_lds_kernel does not take the shape): like gemm_ksplit_kernel the waves
// of a block share out the K steps and meet in LDS, but a block owns NW weight tiles instead of one or two.
// Bound: bytes through L2 into the compute units (about 8.5 TB/s on this part for 16-byte loads), of which HBM only
// supplies the weights: a block re-reads the activation rows of its K range, 4 M bytes per K element against 32 NW of
// weights, so at M = 24 one gate/up pair per block pulled 270 MB of rows beside 180 MB of weights; six tiles pull 90 MB.
// The loads of a wave's next step go out group by group while the current one is multiplied, into the registers just
// used.  Measured at M = 24, 7B shape, weights from HBM (before: gemm_ksplit_kernel; us): QKV 27.3 -> 20.3, O 11.1 -> 9,
// gate/up 50.0 -> 36.3, down 24.3 -> 19.0, LM head 66.3 -> 46.7; at M = 64 (before: gemm_tile_kernel in 48-row blocks)
// 36.4 -> 29.4, 15.1 -> 12.7, 61.2 -> 53.1, 28.5 -> 25.5, 67.4 -> 63.7, and a 768-wide QKV 10.5 -> 5.0.
// LORA: the blocks behind the first n_cols columns of the grid take the low-rank update of the same rows (a block per row,
// projection and part), which would otherwise be a launch of 4.7 us between this one and its consumer.
#define WIDE_WAVES 4
template <int NMAT, int MT, int NW, bool NT_HINT, bool LORA>
__global__ __launch_bounds__(WIDE_WAVES * 64) void gemm_wide_kernel(const uint16_t *__restrict__ A, ActView a_av, WeightSeg w, int M,
                                                               int N, int K, int steps_per_split, float *__restrict__ C,
                                                               size_t c_split_stride, uint16_t *__restrict__ Cact, ActView c_av,
                                                               LmStats ls, int n_cols, LoraArgs la)
{
    constexpr int WAVES = WIDE_WAVES;
    static_assert(NW % 2 == 0, "tiles are finished in pairs");
    if (LORA && (int)blockIdx.x >= n_cols) { // (uniform)
        const int id = ((int)blockIdx.x - n_cols) * gridDim.y + blockIdx.y, r = id % M, p = id / M % la.n_proj, part = id / M / la.n_proj;
        if (part * lora_part(WAVES) < la.N) lora_block<bf16_t, -1, WAVES>((const bf16_t *)A, a_av, K, la, r, p, part);
        return;
    }
    __shared__ f32x4 red[WAVES][NW][MT][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row = lane & 15, grp = lane >> 4;
    const size_t tile_elems = (size_t)(K >> 7) * 2048;
    constexpr int CT = NW / NMAT; // 16-column tiles of the result per block
    const int t0 = blockIdx.x * CT, n_t = N / 16;
    // tile c of the block (NMAT = 2: gate and up alternate); tiles past the end (last block) re-read the last one
    const uint16_t *Wp[NW];
    const int seg_tiles = w.n_per_seg / 16;
#pragma unroll
    for (int c = 0; c < NW; c++) {
        const int t = min(t0 + c / NMAT, n_t - 1), seg = NMAT == 2 ? c & 1 : t / seg_tiles;
        const uint16_t *base = (const uint16_t *)(seg == 0 ? w.p[0] : seg == 1 ? w.p[1] : w.p[2]);
        Wp[c] = base + (size_t)(NMAT == 2 ? t : t - seg * seg_tiles) * tile_elems;
    }
    const uint16_t *Ap[MT]; // rows past M re-read the last one; they only reach result columns that are never stored
#pragma unroll
    for (int t = 0; t < MT; t++) Ap[t] = A + (size_t)min(t * 16 + row, M - 1) * 128 + grp * 8;
    const size_t step_stride = (size_t)a_av.rows * 128;
    f32x4 acc[NW][MT];
#pragma unroll
    for (int c = 0; c < NW; c++)
#pragma unroll
        for (int t = 0; t < MT; t++) acc[c][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    bf16x8 wv[NW][4], ah[MT][4], al[MT][4];
    auto issue = [&](int st, int i) { // group i (32 of the step's 128 elements)
#pragma unroll
        for (int t = 0; t < MT; t++) {
            ah[t][i] = *(const bf16x8 *)(Ap[t] + step_stride * st + i * 32);
            al[t][i] = *(const bf16x8 *)(Ap[t] + a_av.plane + step_stride * st + i * 32);
        }
#pragma unroll
        for (int c = 0; c < NW; c++)
            wv[c][i] = ld_stream<NT_HINT>((const bf16x8 *)(Wp[c] + (size_t)st * 2048 + i * 512 + lane * 8));
    };
    auto consume = [&](int i) {
#pragma unroll
        for (int t = 0; t < MT; t++)
#pragma unroll
            for (int c = 0; c < NW; c++) acc[c][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv[c][i], ah[t][i], acc[c][t], 0, 0, 0);
#pragma unroll
        for (int t = 0; t < MT; t++)
#pragma unroll
            for (int c = 0; c < NW; c++) acc[c][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv[c][i], al[t][i], acc[c][t], 0, 0, 0);
    };
    const int s_begin = blockIdx.y * steps_per_split, s_end = min(K / 128, s_begin + steps_per_split);
    int st = s_begin + wave;
    if (st < s_end) { // (uniform over the wave)
#pragma unroll
        for (int i = 0; i < 4; i++) issue(st, i);
        for (; st + WAVES < s_end; st += WAVES) {
#pragma unroll
            for (int i = 0; i < 4; i++) {
                consume(i);
                issue(st + WAVES, i);
            }
        }
#pragma unroll
        for (int i = 0; i < 4; i++) consume(i);
    }
#pragma unroll
    for (int c = 0; c < NW; c++)
#pragma unroll
        for (int t = 0; t < MT; t++) red[wave][c][t][lane] = acc[c][t];
    __syncthreads();
    // unit = (pair of tiles, row tile): lane (m' = lane % 16, g = lane / 16) finishes columns 4 g .. 4 g + 3 of row m'
    for (int u = wave; u < NW / 2 * MT; u += WAVES) {
        const int c = u / MT * 2, t = u % MT, m = t * 16 + row;
        f32x4 v0 = red[0][c][t][lane], v1 = red[0][c + 1][t][lane];
#pragma unroll
        for (int x = 1; x < WAVES; x++) {
            v0 += red[x][c][t][lane];
            v1 += red[x][c + 1][t][lane];
        }
        if (NMAT == 2) {
            const int n = (t0 + c / 2) * 16 + 4 * grp;
            if (m < M && n < N) {
                float y[4];
#pragma unroll
                for (int r = 0; r < 4; r++) y[r] = v0[r] / (1.0f + expf(-v0[r])) * v1[r];
                uint32_t h0, l0, h1, l1;
                bf16x2_split(y[0], y[1], h0, l0);
                bf16x2_split(y[2], y[3], h1, l1);
                const size_t o = act_index(c_av, m, n, N); // 4 columns inside one K step
                *(uint2 *)(Cact + o) = make_uint2(h0, h1);
                *(uint2 *)(Cact + c_av.plane + o) = make_uint2(l0, l1);
            }
        } else {
            const int n = (t0 + c) * 16 + 4 * grp;
            float *dst = C + (size_t)blockIdx.y * c_split_stride + (size_t)m * N + n;
            if (m < M && n < N) *(f32x4 *)dst = v0;
            if (m < M && n + 16 < N) *(f32x4 *)(dst + 16) = v1;
            if (ls.p && n < N) { // (uniform; N is a multiple of 32) partials of the 32 columns this unit covers
                float mx = v0[0];
                int ai = n;
#pragma unroll
                for (int r = 1; r < 4; r++)
                    if (v0[r] > mx) mx = v0[r], ai = n + r;
#pragma unroll
                for (int r = 0; r < 4; r++)
                    if (v1[r] > mx) mx = v1[r], ai = n + 16 + r;
#pragma unroll
                for (int o = 16; o <= 32; o <<= 1) {
                    const float ov = __shfl_xor(mx, o, 64);
                    const int oi = __shfl_xor(ai, o, 64);
                    if (ov > mx || (ov == mx && oi < ai)) mx = ov, ai = oi;
                }
                float ex = 0.f;
                if (ls.invT > 0.f) {
#pragma unroll
                    for (int r = 0; r < 4; r++) ex += expf((v0[r] - mx) * ls.invT) + expf((v1[r] - mx) * ls.invT);
                }
                ex += __shfl_xor(ex, 16, 64);
                ex += __shfl_xor(ex, 32, 64);
                if (grp == 0 && m < M) {
                    float *sp = ls.p + ((size_t)m * (N / 32) + (t0 + c) / 2) * 3;
                    sp[0] = mx;
                    sp[1] = ex;
                    sp[2] = __int_as_float(ai);
                }
            }
        }
    }
}

// Few-row GEMM of wide layers (17 to 96 rows, 4096 elements of K and more): a block of WR x WC waves, each with one 32 x 32
// tile of the result (v_mfma_f32_32x32x16_bf16, weights as the first operand), and one block per compute unit.
// Bound: what a compute unit pulls through L2 (50 - 60 GB/s), of which HBM only supplies the weights.  gemm_wide_kernel reads
// the activation rows once per wave and K step into registers, as many bytes of rows as of weights at M = 32; here both operands go to LDS
// (global_load_lds, 16 bytes a lane, no registers in between), so a block pulls its rows once for all of its weight
// tiles, and NB - 1 chunks of 64 elements are in flight while one is multiplied, whatever the registers hold.
// One barrier per chunk, in front of its last MFMA group: behind it the next chunk's fragments are read and the buffer
// just emptied is refilled.  Weight tiles lie in LDS as in memory (operand order, conflict free); rows of 128 bytes have their eight 16-byte
// pieces exchanged by (row / 2) % 8, so that the 32 rows of an operand fall into all banks.
// Measured alone, the slabs' reader included (gemm_wide_kernel before -> now, us): 4096 wide, M = 24: gate/up 34.6 -> 31.5, QKV
// 19.4 -> 19.6 (in a whole pass 0.8 ahead), down 18.5 -> 17.8; M = 64: gate/up 53.0 -> 42.9, QKV 30.7 -> 24.7, O 14.4 -> 13.1, down
// 27.5 -> 24.2, LM head 63.7 -> 49.0; 5120 wide, M = 24: gate/up 52.2 -> 45.8, QKV 28.5 -> 27.3, down 27.3 -> 24.4; M = 64:
// gate/up 73.8 -> 57.1, QKV 42.5 -> 34.2, down 40.0 -> 32.7; M = 80 (gemm_tile_kernel before, weights cold): gate/up 59.0 -> 53.5,
// QKV 35.6 -> 30.6, O 15.7 -> 16.0, down 27.0 -> 26.9, LM head 60.1 -> 53.1, at 5120 wide 79.9 -> 68.8, 44.8 -> 40.6, 20.3 -> 19.9,
// 38.4 -> 39.2.  Deeper rings (5 stages of 64 x 96, 7 of 32 x 96) change nothing.  Verify pass, four 4096-wide layers: 468 -> 448 at
// 18 rows, 495 -> 461 at 24, 520 -> 476 at 30, 624 -> 560 at 48, 685 -> 596 at 64, 766 -> 697 at 72, 811 -> 758 at 96; two 8192 wide
// 730 -> 690 at 18, 840 -> 734 at 30, 1079 -> 889 at 64.  Which launches it gets: lds_plan, lds_choice.
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) const void global_cvoid;
template <int MODE, int WR, int WC, int NB, bool NT_HINT>
__global__ __launch_bounds__(WR *WC * 64) void gemm_lds_kernel(const uint16_t *__restrict__ A, ActView a_av, WeightSeg w, int M, int N, int K,
                                                            int k_per_split, float *__restrict__ C, size_t c_split_stride,
                                                            uint16_t *__restrict__ Cact, ActView c_av, LmStats ls)
{
    constexpr bool SW = MODE == GEMM_SWIGLU; // weight tiles of the block: gate and up alternate
    constexpr int WAVES = WR * WC, BM = 32 * WR, BN = 32 * WC, COLS = SW ? BN / 2 : BN;
    constexpr int KC = 64;                             // elements per chunk
    constexpr int NA = 2 * BM / 8, NW = BN / 16 * 2;   // loads of 1 KiB per chunk: 8 rows of a plane, 32 elements of a weight tile
    constexpr int PA = (NA + WAVES - 1) / WAVES, PB = (NW + WAVES - 1) / WAVES, PD = PA + PB; // per wave (some load a piece twice where the waves don't divide)
    constexpr int STAGE = (NA + NW) * 1024;
    static_assert(NB * STAGE <= 160 * 1024 && (NB - 2) * PD < 64, "LDS, vmcnt");
    __shared__ __attribute__((aligned(1024))) char lds[NB * STAGE];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wr = wave / WC, wc = wave % WC;
    const int n0 = blockIdx.x * COLS;
    const int kb = blockIdx.y * k_per_split, ke = min(K, kb + k_per_split);
    const int nchunks = (ke - kb) / KC;
    const size_t tile_elems = (size_t)(K >> 7) * 2048;
    const uint16_t *Wp[PB]; // (uniform) tiles past the end (last block) re-read the last one
    {
        const int seg_tiles = w.n_per_seg / 16, last = N / 16 - 1;
#pragma unroll
        for (int j = 0; j < PB; j++) {
            const int id = min(j * WAVES + wave, NW - 1), q = id / 2;
            const int t = min(n0 / 16 + (SW ? q >> 1 : q), last), seg = SW ? q & 1 : t / seg_tiles;
            const uint16_t *base = (const uint16_t *)(seg == 0 ? w.p[0] : seg == 1 ? w.p[1] : w.p[2]);
            Wp[j] = base + (size_t)(SW ? t : t - seg * seg_tiles) * tile_elems + (size_t)(kb >> 7) * 2048 + id % 2 * 512;
        }
    }
    uint32_t a_off[PA]; // rows past M re-read the last one; they only reach result rows that are never stored
#pragma unroll
    for (int j = 0; j < PA; j++) {
        const int id = min(j * WAVES + wave, NA - 1), plane = id / (BM / 8), r = id % (BM / 8) * 8 + lane / 8;
        a_off[j] = (uint32_t)((plane ? a_av.plane : 0) + (size_t)min(r, M - 1) * 128 + ((lane & 7) ^ (r >> 1 & 7)) * 8);
    }
    const size_t step_stride = (size_t)a_av.rows * 128;
    const uint16_t *Ab = A + (size_t)(kb >> 7) * step_stride;
    auto dma = [&](int ch, int buf) { // chunks past the end re-read the last one (the count of loads in flight stays the same)
        const int cc = min(ch, nchunks - 1);
        const uint16_t *ab = Ab + (size_t)(cc >> 1) * step_stride + (cc & 1) * KC;
        char *st = lds + buf * STAGE;
#pragma unroll
        for (int j = 0; j < PA; j++)
            __builtin_amdgcn_global_load_lds((global_cvoid *)(ab + a_off[j]), (lds_void *)(st + min(j * WAVES + wave, NA - 1) * 1024), 16, 0, 0);
#pragma unroll
        for (int j = 0; j < PB; j++)
            __builtin_amdgcn_global_load_lds((global_cvoid *)(Wp[j] + (size_t)cc * (KC * 16) + lane * 8),
                                             (lds_void *)(st + (NA + min(j * WAVES + wave, NW - 1)) * 1024), 16, 0, NT_HINT ? 2 : 0);
    };
    const int lr = lane & 31, lg = lane >> 5;
    uint32_t fa[4];
#pragma unroll
    for (int kk = 0; kk < 4; kk++) fa[kk] = (wr * 32 + lr) * 128 + (((2 * kk + lg) ^ (lr >> 1 & 7)) << 4);
    const uint32_t fb = NA * 1024 + (wc * 2 + (lr >> 4)) * 2048 + lg * 256 + (lr & 15) * 16;
    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; e++) acc[e] = 0.f;
    bf16x8 ah[2], al[2], bw[2];
    auto frags = [&](int buf, int kk, int s) { // 16 of the chunk's elements
        const char *b = lds + buf * STAGE;
        bw[s] = *(const bf16x8 *)(b + fb + (kk >> 1) * 1024 + (kk & 1) * 512);
        ah[s] = *(const bf16x8 *)(b + fa[kk]);
        al[s] = *(const bf16x8 *)(b + fa[kk] + BM * 128);
    };
    auto mfmas = [&](int s) {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bw[s], ah[s], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bw[s], al[s], acc, 0, 0, 0);
    };
    constexpr int VM = (NB - 2) * PD, VMCNT = (VM & 15) | (VM >> 4 << 14); // this wave's part of the next chunk has landed
#pragma unroll
    for (int b = 0; b < NB - 1; b++) dma(b, b);
    __builtin_amdgcn_s_waitcnt(0x0f70 | VMCNT);
    __builtin_amdgcn_s_barrier();
    SD_ORDER();
    dma(NB - 1, NB - 1);
    frags(0, 0, 0);
    // chunk ch in buffer b; at entry the fragments of its group 0 are requested and the loads of chunks up to ch + NB - 1 issued
    auto chunk = [&](int ch, int b) {
#pragma unroll
        for (int kk = 0; kk < 3; kk++) {
            frags(b, kk + 1, (kk + 1) & 1);
            mfmas(kk & 1);
            SD_ORDER();
        }
        // everything of this chunk is in registers; the next one has landed once all waves are past the barrier
        __builtin_amdgcn_s_waitcnt(0x0070 | VMCNT);
        __builtin_amdgcn_s_barrier();
        SD_ORDER();
        frags((b + 1) % NB, 0, 0);
        SD_ORDER();
        dma(ch + NB, b);
        mfmas(1);
        SD_ORDER();
    };
    const int n_main = nchunks / NB * NB;
    for (int c0 = 0; c0 < n_main; c0 += NB) {
#pragma unroll
        for (int b = 0; b < NB; b++) chunk(c0 + b, b);
    }
#pragma unroll
    for (int b = 0; b < NB - 1; b++)
        if (n_main + b < nchunks) chunk(n_main + b, b);
    __builtin_amdgcn_s_waitcnt(0x0f70); // nothing may land in LDS after the block has ended
    // lane (m' = lane % 32, g = lane / 32) holds columns 8 i + 4 g + 0 .. 3, i = 0 .. 3, of row m'
    const int m = wr * 32 + lr;
    if (SW) {
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int n = n0 + wc * 16 + 8 * h + 4 * lg;
            if (m >= M || n >= N) continue;
            float y[4];
#pragma unroll
            for (int r = 0; r < 4; r++) y[r] = acc[4 * h + r] / (1.0f + expf(-acc[4 * h + r])) * acc[8 + 4 * h + r];
            uint32_t h0, l0, h1, l1;
            bf16x2_split(y[0], y[1], h0, l0);
            bf16x2_split(y[2], y[3], h1, l1);
            const size_t o = act_index(c_av, m, n, N); // 4 columns inside one K step
            *(uint2 *)(Cact + o) = make_uint2(h0, h1);
            *(uint2 *)(Cact + c_av.plane + o) = make_uint2(l0, l1);
        }
    } else {
        const int nb = n0 + wc * 32 + 4 * lg;
        float *dst = C + (size_t)blockIdx.y * c_split_stride + (size_t)m * N + nb;
#pragma unroll
        for (int i = 0; i < 4; i++)
            if (m < M && nb + 8 * i < N) *(f32x4 *)(dst + 8 * i) = (f32x4){acc[4 * i], acc[4 * i + 1], acc[4 * i + 2], acc[4 * i + 3]};
        if (ls.p && n0 + wc * 32 < N) { // (uniform; N is a multiple of 32) partials of the wave's 32 columns
            float mx = acc[0];
            int ai = nb;
#pragma unroll
            for (int e = 1; e < 16; e++)
                if (acc[e] > mx) mx = acc[e], ai = nb + e / 4 * 8 + e % 4;
            const float ov = __shfl_xor(mx, 32, 64);
            const int oi = __shfl_xor(ai, 32, 64);
            if (ov > mx || (ov == mx && oi < ai)) mx = ov, ai = oi;
            float ex = 0.f;
            if (ls.invT > 0.f) {
#pragma unroll
                for (int e = 0; e < 16; e++) ex += expf((acc[e] - mx) * ls.invT);
            }
            ex += __shfl_xor(ex, 32, 64);
            if (lg == 0 && m < M) {
                float *sp = ls.p + ((size_t)m * (N / 32) + n0 / 32 + wc) * 3;
                sp[0] = mx;
                sp[1] = ex;
                sp[2] = __int_as_float(ai);
            }
        }
    }
}

// fp32 slabs of a K split: written by the launch and read by its consumer, 32 bytes per element spread over the 256 units (KiB each).
static float slab_kib(int ny, int M, int N) { return ny > 1 ? (float)ny * M * N * (32.f / (256 * 1024)) : 0.f; }
// Block shape of the wide kernel: NW weight tiles per block and the K splits (nw = 0: not a shape of it).  The estimate
// is what the busiest compute unit pulls in, in KiB: rounds of blocks over 256 units x K steps per split x (4 NW for the
// weights + M / 2 for the rows), plus the splits' fp32 slabs, written here and read by the consumer (32 bytes per element
// spread over the units).  Against a sweep of NW, 4 and 8 waves and 1 to 8 splits over QKV / O / gate-up / down / LM head of the
// 7B, 13B and draft shapes at 9 to 64 rows its choice is the fastest or within 8 % of it (8 waves were never more than 2 % ahead).
struct WidePlan {
    int nw, ncol, ks;
};
static WidePlan wide_plan(int mode, int M, int N, int K, int n_per_seg, int force_ks, int max_ks = 8)
{
    WidePlan best = {0, 0, 1};
    if (M > 64 || N % 16 != 0 || n_per_seg % 16 != 0 || K % 128 != 0 || K < 128) return best;
    // 41 to 48 rows fit one 48-row block of the row-blocked kernel, which stages them once for 128 weight rows: where
    // its unsplit grid fills the chip it is ahead of this one (gate/up at M = 48: 44.7 against 45.9 us at 4096 / 11008, 55.5 against 65.2
    // at 5120 / 13824; the 32000-column head 52.8 against 55.0; from a K of 4096 on gemm_lds_kernel has these shapes)
    const int nmat = mode == GEMM_SWIGLU ? 2 : 1, rows_w = N * nmat, steps = K / 128;
    if (M > 40 && M <= 48 && steps >= 16 && rows_w % 128 == 0 && n_per_seg % 128 == 0 && N == n_per_seg && rows_w / 128 >= 160) return best;
    float best_cost = 0.f;
    for (int nw = 2; nw <= 8; nw += 2) {
        const int ct = nw / nmat, ncol = (N / 16 + ct - 1) / ct;
        for (int ks = force_ks > 0 ? force_ks : 1; ks <= (force_ks > 0 ? force_ks : mode == GEMM_SWIGLU ? 1 : max_ks); ks++) {
            int kps, ny;
            split_geometry(K, ks, &kps, &ny);
            if (force_ks <= 0 && ks > 1 && (ny != ks || kps < 256)) continue;
            const float rounds = (float)((ncol * ny + 255) / 256);
            const float cost = rounds * (float)(kps / 128) * (4.f * nw + 0.5f * M) + slab_kib(ny, M, N);
            if (best.nw == 0 || cost < best_cost) {
                best = {nw, ncol, ny};
                best_cost = cost;
            }
        }
    }
    return best;
}

// Does the norm split between producer and consumer GEMM (NormFold) pay at M rows of width d?  Up to 8 rows (hi and lo rows
// share one operand) the weights dominate and two launches per layer less are ahead.  From 9 rows on the unfolded launches run on
// the wide kernel and split K over the chip, while a folded projection runs unsplit in blocks that re-read the rows; only
// where those blocks cover the compute units in one full round does the fold last two rows longer.  Verify pass of two
// layers, folded / not (us): 4096 wide 229.9 / 233.6 at 8 rows, 248.0 / 253.9 at 9, 254.4 / 255.1 at 10, 263.2 / 257.4 at 11,
// 297 / 262 at 16, 442 / 311 at 32; 8192 wide 361 / 370 at 9, 380 / 375 at 11; 5120 wide 391 / 331 at 9; 3072 wide 177 / 171 at
// 9; 768 wide 81.6 / 78.8 at 9, 89.0 / 82.5 at 16, 120 / 96 at 32.
bool gemm_normfold_pays(int M, int d) { return M <= 8 || (M <= 10 && gemm_normfold_blocks(d) == 256); }

// Block shapes of the row-blocked kernel (unsplit: the launch has one K split).  More than 64 rows: 96 rows x 256 columns (4
// waves x 4 tiles; chunks of half a K step) - the bytes a block pulls through L2 per MFMA halve against 48 x 128, which is what
// bounds these GEMMs - or x 192 columns (3 tiles per wave) where that fills the 256 compute units better
// (QKV at M = 192: 128 blocks x 2 K splits instead of 96 x 2); 64-row blocks of the same widths where they
// pad M less (M = 128).  Up to 64 rows: 48-row blocks of 2 waves x
// 128 columns, two resident per unit.  A block of the 96-row shapes has a compute unit to itself
// (~500 registers per wave), so the K splits are chosen to cover the chip in one round of blocks.
struct TileShape {
    int cols;  // weight rows per block (0: shape not supported)
    int bm;    // rows per block
    int ncol;  // column tiles
    int nmb;   // row blocks
    int slots; // blocks resident at once on the whole chip
};
// Column tile t runs on die t % 8 with all its row blocks and K splits (they share the die's L2), so the busiest
// die carries ceil(ncol / 8) tiles: 20 tiles put 3 on four dies and 2 on the others.  A launch is one round of
// blocks only if that die's share fits its eighth of the slots - counting blocks over the whole chip instead let
// the 5120-wide projections run a second round on half the dies (44 against 31 us for the O projection at M = 192).
static int die_blocks(int ncol, int nmb, int ks) { return (ncol + 7) / 8 * nmb * ks; }
static int one_round_splits(int ncol, int nmb, int slots, int steps)
{
    int ks = 1;
    while (ks < 8 && die_blocks(ncol, nmb, ks + 1) * 8 <= slots && (steps + ks) / (ks + 1) >= 4) ks++;
    return ks;
}
static int die_rounds(int ncol, int nmb, int ks, int slots) { return (die_blocks(ncol, nmb, ks) * 8 + slots - 1) / slots; }
// K splits of a launch: as many as keep the busiest die at one round of blocks; where not even the unsplit launch fits one
// round, the count that makes rounds x (K steps per split + 5 steps of fixed cost) smallest (by more than 5 %): the 96-row
// QKV blocks of a 4096-wide model at M = 576 come to one and a half rounds, two splits to three full ones of half the
// length (measured 120 -> 107 us; three and four splits 124 us, as the model has it).
static int tile_splits(int ncol, int nmb, int slots, int steps)
{
    if (die_rounds(ncol, nmb, 1, slots) == 1) return one_round_splits(ncol, nmb, slots, steps);
    int best = 1;
    float best_cost = (float)die_rounds(ncol, nmb, 1, slots) * ((float)steps + 5.f);
    for (int ks = 2; ks <= 8 && (steps + ks - 1) / ks >= 4; ks++) {
        const float cost = (float)die_rounds(ncol, nmb, ks, slots) * ((float)steps / (float)ks + 5.f);
        if (cost < 0.95f * best_cost) {
            best = ks;
            best_cost = cost;
        }
    }
    return best;
}
// Block shape and K splits of gemm_lds_kernel (cols = 0: not a shape of it).  Blocks of 32, 64 or 96 rows, all of the
// launch's; 96 or 128 weight rows; the estimate is rounds of blocks over 256 units x (K steps per split + 2), a step of 128
// weight rows 1.05 of one of 96, plus the splits' fp32 slabs; no split of fewer than four steps, and none in more than one round
// of blocks (two from 33 rows on): every round fills its ring anew.  QKV, whole passes, us per launch against the present choice:
// 8192 wide in four splits, three rounds, 13 to 18 behind up to 32 rows, 9 to 15 at 36 to 64; 6144 and 7168 wide in three splits, two rounds,
// 2 to 6 behind up to 32 rows, at 36 to 64 the unsplit launch is 2 to 4 behind and 3 ahead to 5 behind.  Over QKV / O / gate-up / down / LM head of the 4096- and
// 5120-wide models at 20 to 64 rows its choice is the fastest of the sweep (both widths, 1 to 8 splits) or within 3 % but for
// one (O at M = 48: 13.0 against 11.7).
// Up to 16 rows gemm_wide_kernel is ahead (QKV 17.3 against 19.0, O 7.1 against 7.9 at M = 16), so it is on narrower models (2048
// wide, M = 32: gate/up 15.6 against 16.4, down 7.6 against 9.3), whose few K steps don't repay filling the ring, and up to 48
// rows where a unit's share of the launch is fewer than five steps of 128 weight rows (O at 4096 wide, in a whole pass: 2.0 us ahead at 18 and
// 24 rows, 1.4 at 32, 0.5 at 48, 1.1 behind at 64; at 5120 wide, a share of six, the two are equal).
// Above 96 rows one block takes too much LDS for a ring, and two row blocks per column tile are slower than gemm_tile_kernel (gate/up
// at M = 128: 84 against 59).
struct LdsPlan {
    int cols, ncol, ks;
    float pull; // what the busiest unit pulls in, KiB
};
static LdsPlan lds_plan(int mode, int M, int N, int K, int n_per_seg, int force_ks, int max_ks = 8)
{
    LdsPlan best = {0, 0, 1, 0.f};
    const int rows_w = N * (mode == GEMM_SWIGLU ? 2 : 1), steps = K / 128;
    if (M < 17 || M > 96 || N % 16 != 0 || n_per_seg % 16 != 0 || K % 128 != 0 || steps < 32 || rows_w < 4096) return best;
    if (M <= 48 && (long)rows_w * steps < 5L * 256 * 128) return best;
    float best_cost = 0.f;
    for (int cols = 96; cols <= 128; cols += 32) {
        const int ncol = (rows_w + cols - 1) / cols;
        for (int ks = force_ks > 0 ? force_ks : 1; ks <= (force_ks > 0 ? force_ks : mode == GEMM_SWIGLU ? 1 : max_ks); ks++) {
            int kps, ny;
            split_geometry(K, ks, &kps, &ny);
            if (force_ks <= 0 && ks > 1 && (ny != ks || steps / ks < 4 || ncol * ny > (M <= 32 ? 256 : 512))) continue;
            const float turns = (float)((ncol * ny + 255) / 256) * (float)(kps / 128 + 2);
            const float cost = turns * (cols == 128 ? 1.05f : 1.f) + (ny > 1 ? 0.2f * 4e-6f * (float)ny * M * N : 0.f);
            if (best.cols == 0 || cost < best_cost) {
                best = {cols, ncol, ny, turns * (cols / 4 + (M + 31) / 32 * 16) + slab_kib(ny, M, N)};
                best_cost = cost;
            }
        }
    }
    return best;
}

int g_force_tile_cols = 0; // weight rows per 96-row block forced by option "gemm_tile_cols" (0 = automatic)
static TileShape tile_shape(int mode, int M, int N, int n_per_seg, int K, bool unsplit)
{
    const int out_per_col = mode == GEMM_SWIGLU ? 2 : 1; // weight rows per output column
    const int rows_w = N * out_per_col;                  // weight rows streamed
    TileShape t = {0, 0, 0, 0, 0};
    if (M > 64) {
        const int nmb = (M + 95) / 96, steps = K / 128;
        const bool ok256 = rows_w % 256 == 0 && (mode == GEMM_SWIGLU || n_per_seg % 256 == 0);
        // (SwiGLU blocks of 192 weight rows = 96 output columns may end in a partial block)
        const bool ok192 = mode == GEMM_SWIGLU || (rows_w % 192 == 0 && n_per_seg % 16 == 0);
        auto fill = [&](int cols) { // fraction of the 256 units busy, averaged over the rounds of blocks
            const int ncol = (rows_w + cols - 1) / cols;
            const int ks = mode == GEMM_SWIGLU ? 1 : one_round_splits(ncol, nmb, 256, steps);
            return (float)(ncol * nmb * ks) / (256.f * (float)die_rounds(ncol, nmb, ks, 256));
        };
        int cols = 0;
        if (ok256) cols = 256;
        if (ok192 && (!ok256 || fill(192) > fill(256) + 0.1f)) cols = 192;
        // Plain projections with few column tiles may do better with 128-column blocks.  A block's time is modelled as
        // rounds on the busiest die x (K steps per split + 5 steps of fixed cost) x the cost of one of its steps (a
        // 128-column step costs 0.68 of a 256-column one: half the weights and MFMAs, the same activation chunk).
        // Against measurements at widths 4096 and 5120, M = 66 ... 576, it picks 128 columns for O and down at M <= 96
        // (twice the blocks in flight), for O at M = 192 (4 K splits of 8 steps instead of 8 of 4: also half the slabs
        // for the add + norm launch behind it) and for the 5120-wide O and down where 20 wide tiles would leave four
        // dies with half as much again as the others; 256 columns for the 4096-wide down projection at M > 96 and for
        // QKV.
        const bool ok128 = mode != GEMM_SWIGLU && rows_w % 128 == 0 && n_per_seg % 128 == 0;
        if (cols == 256 && ok128) {
            auto est = [&](int c, float step_cost) {
                const int ncol = rows_w / c, sp = one_round_splits(ncol, nmb, 256, steps);
                return (float)die_rounds(ncol, nmb, sp, 256) * ((float)steps / (float)sp + 5.f) * step_cost;
            };
            if (est(128, 0.68f) < est(256, 1.f)) cols = 128;
        }
        if (g_force_tile_cols == 256 && ok256) cols = 256;
        if (g_force_tile_cols == 192 && ok192) cols = 192;
        if (g_force_tile_cols == 128 && ok128) cols = 128;
        if (cols) {
            // 64-row blocks when they pad M less (M = 128: 2 x 64 instead of 96 + 32) and do not cost more rounds; from 65 to 96
            // rows also where K is not split: one row block of the gate/up pair or the LM head leaves units idle (43 and 125
            // blocks at 2048 wide), and two of 64 rows pull little more than one of 96 (weights outweigh rows in every block):
            // gate/up at 2048 / 5504 40 -> 25 us, a verify pass of four 2048-wide layers 480 -> 439 at 66 rows, 497 -> 457 at 96, 3072 wide
            // 645 -> 589, 664 -> 613 (from a K of 4096 on gemm_lds_kernel has most of these launches)
            const int ncol = (rows_w + cols - 1) / cols, nmb64 = (M + 63) / 64;
            auto rounds = [&](int rb) {
                return die_rounds(ncol, rb, mode == GEMM_SWIGLU ? 1 : one_round_splits(ncol, rb, 256, steps), 256);
            };
            const bool use64 = (nmb64 * 64 < nmb * 96 || (unsplit && M <= 96)) && rounds(nmb64) * 64 <= rounds(nmb) * 96;
            return use64 ? TileShape{cols, 64, ncol, nmb64, 256} : TileShape{cols, 96, ncol, nmb, 256};
        }
    }
    if (rows_w % 128 == 0 && (mode == GEMM_SWIGLU || n_per_seg % 128 == 0))
        t = TileShape{128, 48, rows_w / 128, (M + 47) / 48, 512};
    return t;
}

template <int MODE>
static hipError_t tile_launch(hipStream_t s, const uint16_t *a, ActView a_av, WeightSeg w, int M, int N, int K, int ks,
                              float *C, size_t c_split_stride, uint16_t *ca, ActView c_av)
{
    int kps, ny;
    split_geometry(K, ks, &kps, &ny);
    const TileShape t = tile_shape(MODE, M, N, w.n_per_seg, K, ks == 1);
    if (!t.cols) return hipErrorNotSupported;
    constexpr int OUT_PER_COL = MODE == GEMM_SWIGLU ? 2 : 1;
    const int ntiles = (N * OUT_PER_COL + t.cols - 1) / t.cols, nmb = (M + t.bm - 1) / t.bm;
    const int gx = ((ntiles + 7) / 8) * 8 * nmb;
#define SD_TILE(BM, KC, NT, WAVES, NB)                                                                              \
    hipLaunchKernelGGL((gemm_tile_kernel<MODE, BM, KC, NT, WAVES, NB>), dim3(gx, ny), dim3(WAVES * 64), 0, s, a, a_av, w, \
                       M, N, K, kps, nmb, ntiles, C, c_split_stride, ca, c_av)
    if (t.cols == 256 && t.bm == 96) SD_TILE(96, 64, 4, 4, 3);
    else if (t.cols == 192 && t.bm == 96) SD_TILE(96, 64, 3, 4, 3);
    else if (t.cols == 256) SD_TILE(64, 64, 4, 4, 3);
    else if (t.cols == 192) SD_TILE(64, 64, 3, 4, 3);
    else if (t.cols == 128 && t.bm == 96) SD_TILE(96, 64, 2, 4, 3);
    else if (t.cols == 128 && t.bm == 64) SD_TILE(64, 64, 2, 4, 3);
    else SD_TILE(48, 128, 4, 2, 3);
    return hipGetLastError();
}

template <int NMAT, int MT, bool NT>
static void wide_launch_nw(hipStream_t s, WidePlan p, const uint16_t *a, ActView a_av, WeightSeg w, int M, int N, int K, int sps,
                           float *C, size_t c_split_stride, uint16_t *ca, ActView c_av, LmStats ls, const LoraArgs *la)
{
    dim3 grid(p.ncol, p.ks);
    const dim3 block(WIDE_WAVES * 64);
    if constexpr (NMAT == 1 && !NT) {
        if (la) {
            const int parts = (la->N + lora_part(WIDE_WAVES) - 1) / lora_part(WIDE_WAVES);
            grid.x += (M * la->n_proj * parts + p.ks - 1) / p.ks;
#define SD_WIDE_LORA(NW_)                                                                                                     \
    hipLaunchKernelGGL((gemm_wide_kernel<NMAT, MT, NW_, NT, true>), grid, block, 0, s, a, a_av, w, M, N, K, sps, C, c_split_stride, ca, c_av, ls, p.ncol, *la)
            if (p.nw == 2) SD_WIDE_LORA(2);
            else SD_WIDE_LORA(4);
#undef SD_WIDE_LORA
            return;
        }
    }
#define SD_WIDE(NW_)                                                                                                          \
    hipLaunchKernelGGL((gemm_wide_kernel<NMAT, MT, NW_, NT, false>), grid, block, 0, s, a, a_av, w, M, N, K, sps, C, c_split_stride, ca, c_av, ls, p.ncol, LoraArgs{})
    if (p.nw == 2) SD_WIDE(2);
    else if (p.nw == 4) SD_WIDE(4);
    else if (p.nw == 6) SD_WIDE(6);
    else SD_WIDE(8);
#undef SD_WIDE
}
template <int NMAT>
static hipError_t wide_launch(hipStream_t s, WidePlan p, const uint16_t *a, ActView a_av, WeightSeg w, int M, int N, int K, float *C,
                              size_t c_split_stride, uint16_t *ca, ActView c_av, LmStats ls, const LoraArgs *la = nullptr)
{
    int kps, ny;
    split_geometry(K, p.ks, &kps, &ny);
    const int mt = (M + 15) / 16, sps = kps / 128;
#define SD_WIDE_MT(MT_)                                                                                                   \
    do {                                                                                                                  \
        if (w.nt) wide_launch_nw<NMAT, MT_, true>(s, p, a, a_av, w, M, N, K, sps, C, c_split_stride, ca, c_av, ls, la);        \
        else wide_launch_nw<NMAT, MT_, false>(s, p, a, a_av, w, M, N, K, sps, C, c_split_stride, ca, c_av, ls, la);            \
    } while (0)
    if (mt == 1) SD_WIDE_MT(1);
    else if (mt == 2) SD_WIDE_MT(2);
    else if (mt == 3) SD_WIDE_MT(3);
    else SD_WIDE_MT(4);
#undef SD_WIDE_MT
    return hipGetLastError();
}

template <int MODE, bool NT>
static hipError_t lds_launch(hipStream_t s, LdsPlan p, const uint16_t *a, ActView a_av, WeightSeg w, int M, int N, int K, float *C,
                             size_t c_split_stride, uint16_t *ca, ActView c_av, LmStats ls)
{
    int kps, ny;
    split_geometry(K, p.ks, &kps, &ny);
#define SD_LDS(WR, WC, NB)                                                                                                    \
    hipLaunchKernelGGL((gemm_lds_kernel<MODE, WR, WC, NB, NT>), dim3(p.ncol, ny), dim3(WR * WC * 64), 0, s, a, a_av, w, M, N, K, \
                       kps, C, c_split_stride, ca, c_av, ls)
    if constexpr (!NT) {
        if (M > 64) {
            if (p.cols == 96) SD_LDS(3, 3, 4);
            else SD_LDS(3, 4, 3);
            return hipGetLastError();
        }
    }
    if (M <= 32 && p.cols == 96) SD_LDS(1, 3, 5);
    else if (M <= 32) SD_LDS(1, 4, 4);
    else if (p.cols == 96) SD_LDS(2, 3, 3);
    else SD_LDS(2, 4, 4);
#undef SD_LDS
    return hipGetLastError();
}

int g_force_splits[3] = {0, 0, 0}; // [mode] -> K splits (0 = automatic); a tuning knob for sweeps

// K splits of the row-blocked kernel.  Measured at M = 192: a block costs about five K steps of fixed time, so one round
// of blocks with the K range cut as finely as that allows beats several rounds of shorter blocks.
static int tile_ks(int mode, int M, int N, int K, int n_per_seg)
{
    if (mode == GEMM_SWIGLU) return 1;
    const TileShape t = tile_shape(mode, M, N, n_per_seg, K, false);
    int kps, ny;
    split_geometry(K, g_force_splits[mode] > 0 ? g_force_splits[mode] : t.cols ? tile_splits(t.ncol, t.nmb, t.slots, K / 128) : 1, &kps, &ny);
    return ny;
}

// Does the launch run on gemm_lds_kernel?  From 65 to 96 rows its 96-row blocks pull two thirds of their bytes for rows, and
// gemm_tile_kernel, whose blocks have up to 256 columns, pulls less where the matrix fills the chip with those: the kernel
// whose busiest unit has less to pull, as measured (whole passes at 4096 to 12288 wide and 32000 or 128256 columns, 66 to 96
// rows, us per launch): gate/up at 4096 / 5120 / 6144 / 7168 / 8192 wide 3.7 to 6.7, 5.7 to 9.7 and 6.3 to 11.7 ahead, 23 to 35 and 27 to 47
// behind; QKV 3.5 ahead at 4096, equal at 5120, 5 to 8 behind at 6144, 6 to 14 at 7168, 19 to 26 at 8192; down equal up to 5120, 2 to 6
// behind at 6144, up to 13 at 8192 / 28672; the head 5 to 20 ahead at 32000 columns, 3 to 15 behind at 128256.  The
// estimates' ratio is 0.92 and less where this kernel is ahead or equal, 1.0 and more where it is behind.
// splits: those of the launch, or 0 while they are being chosen.
static LdsPlan lds_choice(int mode, int M, int N, int K, int n_per_seg, int splits, int max_ks = 8)
{
    const LdsPlan lp = lds_plan(mode, M, N, K, n_per_seg, splits, max_ks);
    if (!lp.cols || M <= 64) return lp;
    const int ks = splits == 1 ? 1 : tile_ks(mode, M, N, K, n_per_seg);
    const TileShape t = tile_shape(mode, M, N, n_per_seg, K, ks == 1);
    if (!t.cols) return lp;
    int kps, ny;
    split_geometry(K, ks, &kps, &ny);
    const float pull = (float)(die_rounds(t.ncol, t.nmb, ny, t.slots) * (t.slots / 256)) * (float)(kps / 128 + 5) *
                           (float)(t.cols / 4 + t.bm / 2) + slab_kib(ny, M, N);
    return lp.pull <= 0.95f * pull ? lp : LdsPlan{0, 0, 1, 0.f};
}

// Number of K splits the launcher will use for this shape (the caller sizes and reduces the partials).  folded: the launch is
// part of a split norm, which stays on the K-split kernel; max_ks: slabs the caller has room for.
int gemm_skinny_splits(int mode, int M, int N, int K, int n_per_seg, bool folded, int max_ks)
{
    if (mode == GEMM_SWIGLU || K < 128 || K % 128 != 0) return 1; // (the launcher rejects such K)
    int kps, ny;
    if (g_force_splits[mode] > 0) {
        split_geometry(K, g_force_splits[mode], &kps, &ny);
        return ny;
    }
    const int steps = K / 128;
    int ks;
    if (M > 8 && !folded) {
        const LdsPlan lp = lds_choice(mode, M, N, K, n_per_seg, 0, max_ks);
        if (lp.cols) return lp.ks;
        const WidePlan wp = wide_plan(mode, M, N, K, n_per_seg, 0, max_ks);
        if (wp.nw) return wp.ks;
    }
    if (M <= 32) { // K-split kernel: 32 columns per block, a step for each of its four waves
        const int blocks = N / 32;
        ks = steps >= 16 ? 2 : 1; // measured: two half-length blocks per tile stream faster than one
        while (blocks * ks < 256 && ks < 8 && steps / (ks * 2) >= 4) ks *= 2;
    } else {
        ks = tile_ks(mode, M, N, K, n_per_seg);
    }
    split_geometry(K, ks, &kps, &ny);
    return ny;
}

// What tile_launch would do for this shape (host only; for tests of the choice itself).
int gemm_tile_plan(int mode, int M, int N, int K, int n_per_seg, int plan[6])
{
    if (M <= 32 || K < 128 || K % 128 != 0 || (mode != GEMM_STORE && mode != GEMM_SWIGLU)) return -1;
    const int ks = tile_ks(mode, M, N, K, n_per_seg);
    const TileShape t = tile_shape(mode, M, N, n_per_seg, K, ks == 1);
    if (!t.cols) return -1;
    plan[0] = t.cols;
    plan[1] = t.bm;
    plan[2] = t.ncol;
    plan[3] = t.nmb;
    plan[4] = ks;
    plan[5] = die_blocks(t.ncol, t.nmb, ks);
    return 0;
}

// Blocks (= entries of NormFold::ss_out per row) of a producer launch with N output columns.
int gemm_normfold_blocks(int N) { return N % 32 == 0 && N / 32 >= 256 ? N / 32 : N / 16; }

// mode GEMM_STORE: C receives `splits` partial slabs [split][M][N] (split stride c_split_stride floats);
// mode GEMM_SWIGLU: Cact receives the bf16 hi/lo planes.  GEMM_RESID is expressed by the caller as a
// store into partial slabs followed by the fused add + norm kernel.
hipError_t launch_gemm_skinny_bf16(hipStream_t s, int mode, const void *A, ActView a_av, WeightSeg w, int M, int N,
                                   int K, float *C, size_t c_split_stride, int splits, void *Cact, ActView c_av,
                                   LmStats ls, int *ls_done, NormFold nf, const LoraArgs *lora, int *lora_done)
{
    if (ls_done) *ls_done = 0;
    if (lora_done) *lora_done = 0;
    const LmStats no_ls = {nullptr, 0.f};
    const bool folded = nf.ss_in || nf.x || nf.row_map;
    if (folded && (M > 32 || nf.ss_nb > SD_NORMFOLD_MAX_BLOCKS)) return hipErrorNotSupported;
    if (nf.x && (mode != GEMM_STORE || splits != 1 || !c_av.sm || N % 128 != 0 || N / 16 > SD_NORMFOLD_MAX_BLOCKS))
        return hipErrorNotSupported;
    if (M < 1 || K % 128 != 0 || K < 128 || (mode != GEMM_STORE && mode != GEMM_SWIGLU)) return hipErrorNotSupported;
    if (!w.tiled) return hipErrorNotSupported; // these kernels read the 16 x 128 tile order only
    for (int i = 0; i < 3; i++)
        if (w.p[i] && ((uintptr_t)w.p[i] & 15)) return hipErrorNotSupported;
    if (((uintptr_t)A & 15) || (a_av.plane & 7) || (N & 3) || !a_av.sm || a_av.rows < M) return hipErrorNotSupported;
    if (2 * a_av.plane + (size_t)SD_ACT_PAD_ROWS * 128 >= ((size_t)1 << 32)) return hipErrorNotSupported; // 32-bit offsets
    if (mode == GEMM_SWIGLU && (!c_av.sm || (c_av.plane & 7) || N % 128 != 0 || ((uintptr_t)Cact & 15))) return hipErrorNotSupported;
    const uint16_t *a = (const uint16_t *)A;
    uint16_t *ca = (uint16_t *)Cact;
    // (weights that stay cached - the instances of the wide kernel that carry an update are for those - in blocks of two or four
    // tiles, as the projections of small models run; with an update to carry, 8 rows and fewer run on it too)
    const bool can_carry = mode == GEMM_STORE && lora && lora_done && !w.nt && lora_valid(M, K, *lora);
    if ((M > 8 || can_carry) && !folded) {
        const LdsPlan lp = lds_choice(mode, M, N, K, w.n_per_seg, mode == GEMM_SWIGLU ? 1 : splits);
        if (lp.cols) {
            const LmStats lsk = mode == GEMM_STORE && lp.ks == 1 && N % 32 == 0 ? ls : no_ls; // (partial sums of a K split have no softmax)
            if (ls_done && lsk.p) *ls_done = 1;
            const bool nt = w.nt && M <= 64; // (80 rows, 4096 wide: the LM head 61.3 us with the hint, 53.1 without; at 64 and fewer even or ahead with it)
            if (mode == GEMM_SWIGLU)
                return nt ? lds_launch<GEMM_SWIGLU, true>(s, lp, a, a_av, w, M, N, K, C, c_split_stride, ca, c_av, lsk)
                            : lds_launch<GEMM_SWIGLU, false>(s, lp, a, a_av, w, M, N, K, C, c_split_stride, ca, c_av, lsk);
            return nt ? lds_launch<GEMM_STORE, true>(s, lp, a, a_av, w, M, N, K, C, c_split_stride, ca, c_av, lsk)
                        : lds_launch<GEMM_STORE, false>(s, lp, a, a_av, w, M, N, K, C, c_split_stride, ca, c_av, lsk);
        }
        const WidePlan wp = wide_plan(mode, M, N, K, w.n_per_seg, mode == GEMM_SWIGLU ? 1 : splits);
        if (wp.nw && (M > 8 || wp.nw <= 4)) {
            const LmStats lsk = mode == GEMM_STORE && wp.ks == 1 && N % 32 == 0 ? ls : no_ls; // (partial sums of a K split have no softmax)
            if (ls_done && lsk.p) *ls_done = 1;
            if (mode == GEMM_SWIGLU) return wide_launch<2>(s, wp, a, a_av, w, M, N, K, C, c_split_stride, ca, c_av, lsk);
            const bool carry = can_carry && wp.nw <= 4;
            if (carry) *lora_done = 1;
            return wide_launch<1>(s, wp, a, a_av, w, M, N, K, C, c_split_stride, ca, c_av, lsk, carry ? lora : nullptr);
        }
    }
    if (M > 32) { // row-blocked
        if (mode == GEMM_SWIGLU) return tile_launch<GEMM_SWIGLU>(s, a, a_av, w, M, N, K, 1, C, 0, ca, c_av);
        return tile_launch<GEMM_STORE>(s, a, a_av, w, M, N, K, splits, C, c_split_stride, ca, c_av);
    }
#define SD_KSPLIT(NMAT, PACKED, MT, U, NTW, GRID, SPS, LS)                                                               \
    do {                                                                                                                  \
        if (w.nt)                                                                                                         \
            hipLaunchKernelGGL((gemm_ksplit_kernel<NMAT, PACKED, MT, U, NTW, true>), GRID, dim3(256), 0, s, a, a_av, w, M, \
                               N, K, SPS, C, c_split_stride, ca, c_av, LS, nf);                                           \
        else                                                                                                              \
            hipLaunchKernelGGL((gemm_ksplit_kernel<NMAT, PACKED, MT, U, NTW, false>), GRID, dim3(256), 0, s, a, a_av, w,  \
                               M, N, K, SPS, C, c_split_stride, ca, c_av, LS, nf);                                        \
    } while (0)
    if (mode == GEMM_SWIGLU) { // K split inside the block only
        if (N % 16 != 0) return hipErrorNotSupported;
        dim3 grid(N / 16);
        if (M <= 8) SD_KSPLIT(2, true, 1, 2, 1, grid, K / 128, no_ls);
        else if (M <= 16) SD_KSPLIT(2, false, 1, 2, 1, grid, K / 128, no_ls);
        else SD_KSPLIT(2, false, 2, 1, 1, grid, K / 128, no_ls);
        return hipGetLastError();
    }
    int kps, ny;
    split_geometry(K, splits, &kps, &ny);
    if (nf.x && ny != 1) return hipErrorNotSupported;
    // (a producer of a split norm has no K split to fill the chip with: 16-column blocks where 32-column ones would
    // leave compute units idle, and four K steps in flight per wave instead of two)
    if (N % 32 == 0 && w.n_per_seg % 32 == 0 && !(nf.x && N / 32 < 256)) {
        dim3 grid(N / 32, ny);
        const LmStats lsk = ny == 1 ? ls : no_ls; // (partial sums of a K split have no softmax)
        if (ls_done && lsk.p) *ls_done = 1;
        if (M <= 8) SD_KSPLIT(1, true, 1, 2, 2, grid, kps / 128, lsk);
        else if (M <= 16) SD_KSPLIT(1, false, 1, 2, 2, grid, kps / 128, lsk);
        else SD_KSPLIT(1, false, 2, 1, 2, grid, kps / 128, lsk);
    } else if (N % 16 == 0 && w.n_per_seg % 16 == 0) {
        dim3 grid(N / 16, ny);
        if (M <= 8 && nf.x) SD_KSPLIT(1, true, 1, 4, 1, grid, kps / 128, no_ls);
        else if (M <= 8) SD_KSPLIT(1, true, 1, 2, 1, grid, kps / 128, no_ls);
        else if (M <= 16) SD_KSPLIT(1, false, 1, 2, 1, grid, kps / 128, no_ls);
        else SD_KSPLIT(1, false, 2, 1, 1, grid, kps / 128, no_ls);
    } else {
        return hipErrorNotSupported;
    }
    return hipGetLastError();
}

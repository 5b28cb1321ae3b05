// mlp.hip -- learned refinement flags: per-block features, a 512-128-128-1 MLP
// on bf16 MFMA (fp32 accumulate), its backward pass and Adam.
//
// The network predicts, from a block's primitive variables, whether the plain
// refinement criterion (Loehner density/velocity estimator with div V < 0 in
// the Earth/CME windows, paper Sect. 3.2) will ask for refinement of that
// block; the plain criterion stays the judge and the fallback.
//
// Rounding points (the CPU reference follows the same ones): inputs X, the
// weights W1, W2, w3 and the hidden activations H1 = relu(Z1), H2 = relu(Z2)
// are bf16 (round to nearest even from fp32); products accumulate in fp32; in
// the backward pass dZ2 and dZ1 enter the GEMMs as bf16 while the bias
// gradients sum the fp32 values.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <stdexcept>
#include <string>
#include <type_traits>
#include <utility>
#include <vector>

#include "devmem.h"
#include "kernels.h"
#include "mlp.h"

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

__device__ inline uint16_t f2bf(float x)
{
    uint32_t u = __float_as_uint(x);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ inline float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
#define DEV_EPI __device__ __forceinline__

// ---------------------------------------------------------------------------
// features: 8 primitives x 4^3 patch means, [prim][k][j][i]
// ---------------------------------------------------------------------------
// A work-group takes one of the four layers of patches along phi: all threads
// turn its cells into primitives (consecutive cells, into LDS), then a thread
// a patch and variable adds the patch's cells in order.  With a thread a patch
// that read its own cells (strided, 192 of 256 threads idle) the launches of
// three days of a level-5 run (1,400 leaves on average) took 46 us, now 29; about
// 300 blocks 13.6 us, now 12.
// On 4^3 blocks a patch is a cell: a lane takes one through, four blocks a
// work-group (4,096 blocks 7.7 us, with a thread a patch over one block 8.9; by
// layers through LDS 16,384 blocks took 58 us, a thread a patch 20).
constexpr int FEATURE_BLOCKS = 4;

template <int BI, int BJ, int BK>
__global__ void __launch_bounds__(256) k_features(KArgs a, const int *items, const int *nitems_ptr, float *raw,
                                                  const float *mean, const float *istd, uint16_t *xb)
{
    using S = Shape<BI, BJ, BK>;
    constexpr int PI = BI / 4, PJ = BJ / 4, PK = BK / 4, LC = BI * BJ * PK;      // cells of a layer
    __shared__ double sw[8][LC];
    const int n = *nitems_ptr, pk = blockIdx.y, t = threadIdx.x;
    auto put = [&](int it, int idx, double m) {
        if (idx < 64 || idx >> 6 == 4) m = log10(m);          // density and pressure
        const float f = (float)m;
        if (raw) raw[(size_t)it * IC_MLP_IN + idx] = f;
        if (xb) xb[(size_t)it * IC_MLP_IN + idx] = f2bf((f - mean[idx]) * istd[idx]);
    };
    if constexpr (S::NC == 64) {
        for (int it = blockIdx.x * FEATURE_BLOCKS + t / 64; it < n; it += gridDim.x * FEATURE_BLOCKS) {
            const int slot = items[it], c = t % 64;
            double u[8], w[8];
#pragma unroll
            for (int v = 0; v < 8; ++v) u[v] = a.U[((size_t)slot * a.nv + v) * S::NC + c];
            cons_to_prim<true>(u, w, a.gas);
#pragma unroll
            for (int v = 0; v < 8; ++v) put(it, v * 64 + c, 0.0 + w[v]);
        }
        return;
    }
    for (int it = blockIdx.x; it < n; it += gridDim.x) {
        const int slot = items[it];
        for (int c = t; c < LC; c += 256) {
            double u[8], w[8];
#pragma unroll
            for (int v = 0; v < 8; ++v) u[v] = a.U[((size_t)slot * a.nv + v) * S::NC + pk * LC + c];
            cons_to_prim<true>(u, w, a.gas);
#pragma unroll
            for (int v = 0; v < 8; ++v) sw[v][c] = w[v];
        }
        __syncthreads();
        if (t < 128) {
            const int v = t >> 4, pi = t & 3, pj = (t >> 2) & 3;
            double sum = 0;
#pragma unroll
            for (int k = 0; k < PK; ++k)
#pragma unroll
                for (int j = 0; j < PJ; ++j)
#pragma unroll
                    for (int i = 0; i < PI; ++i) sum += sw[v][pi * PI + i + BI * (pj * PJ + j + BJ * k)];
            put(it, v * 64 + pk * 16 + (t & 15), sum * (1.0 / (PI * PJ * PK)));
        }
        __syncthreads();               // the cells are read before the next block's are written
    }
}

// ---------------------------------------------------------------------------
// inference in one launch: z-score, bf16 rounding of inputs and weights, both
// layers, head.  Bound by latency and by the 320 KB of fp32 weights each
// work-group reads from the L2 (2.2 us at 64 B/clock), so the two layers share
// one launch and the weights are asked for all at once, up to 160 loads a lane
// in flight, and stay in registers as MFMA operands for every 16-row tile the
// group takes.  Eight waves: wave w owns columns 16 w .. 16 w + 15 of both
// layers, so a row tile is 16 + 4 MFMA steps a wave, the k-steps of 32 in
// ascending order and the head's 128 products in column order (the rounding
// points and orders of the training pass).  Raw inputs, calls queued one after
// another: 1 row 22.8 -> 8.0 us, 677 rows 30.3 -> 7.9, 4,096 rows 34.1 -> 8.4
// against six launches (1/std, weights to bf16, z-score, two GEMMs, head).
// ---------------------------------------------------------------------------
constexpr int NET_TH = 512;                // threads: eight waves of 16 columns
constexpr int NET_XP = IC_MLP_IN + 8;      // padded LDS rows, bf16
constexpr int NET_HP = IC_MLP_HID + 8;

// two fp32 values as bf16 (nearest even, as f2bf), packed
DEV_EPI uint32_t f2bf2(float lo, float hi)
{
    uint32_t a = __float_as_uint(lo), b = __float_as_uint(hi);
    a += 0x7FFFu + ((a >> 16) & 1u);
    b += 0x7FFFu + ((b >> 16) & 1u);
    return __builtin_amdgcn_perm(b, a, 0x07060302u);
}

DEV_EPI bf16x8_t pack8(const float *v)
{
    const uint4 q = make_uint4(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]), f2bf2(v[4], v[5]), f2bf2(v[6], v[7]));
    return __builtin_bit_cast(bf16x8_t, q);
}

// B operands of NK MFMA steps from the fp32 weights W[k][128]: lane l holds
// column n = 16 wave + l % 16 and k = 32 step + 8 (l / 16) + 0..7
template <int NK>
DEV_EPI void weights_ask(const float *W, int wave, int lane, float (*v)[8])
{
    const float *q = W + (lane >> 4) * 8 * IC_MLP_HID + wave * 16 + (lane & 15);
#pragma unroll
    for (int kk = 0; kk < NK; ++kk)
#pragma unroll
        for (int e = 0; e < 8; ++e) v[kk][e] = q[(kk * 32 + e) * IC_MLP_HID];
}

// C rows 16 i + 4 (l / 16) + 0..3, column l % 16, of the NB 16-row blocks of L
// (rows of `pitch` bf16) times the NK operands b
template <int NK, int NB>
DEV_EPI void tile_mfma(const uint16_t *L, int pitch, int lane, const bf16x8_t *b, float4_t *acc)
{
#pragma unroll
    for (int i = 0; i < NB; ++i) acc[i] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < NK; ++kk)
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const bf16x8_t a = *(const bf16x8_t *)&L[(16 * i + (lane & 15)) * pitch + kk * 32 + (lane >> 4) * 8];
            acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[kk], acc[i], 0, 0, 0);
            // no further than 16 operands read ahead: more would spill
            if (NB > 1 && kk % 4 == 3 && i == NB - 1) __builtin_amdgcn_sched_barrier(0);
        }
}

DEV_EPI float relu(float v) { return v > 0.f ? v : 0.f; }

// logit of a row: sum_j H2[j] w3[j] + b3 (fp32, j ascending), w3 rounded to
// bf16; both 16-byte aligned in LDS
DEV_EPI float head_row(const uint16_t *H2, const float *w3, float b3)
{
    float s = 0.f;
#pragma unroll 4
    for (int j = 0; j < IC_MLP_HID; j += 8) {
        const uint4 h = *(const uint4 *)&H2[j];
        const float4_t wa = *(const float4_t *)&w3[j], wb = *(const float4_t *)&w3[j + 4];
        const uint32_t u[4] = {h.x, h.y, h.z, h.w};
#pragma unroll
        for (int e = 0; e < 8; ++e)
            s += bf2f((uint16_t)(u[e >> 1] >> (16 * (e & 1)))) * (e < 4 ? wa[e & 3] : wb[e & 3]);
    }
    return s + b3;
}

// RAW: x is fp32 raw inputs, z-scored here with mean and std; else bf16, normalised.
// HOLD: one work-group takes all rows (at most IC_MLP_NOALLOC_ROWS) and writes
// the probabilities when it has read every input, so prob may lie on them.
template <bool RAW, bool HOLD = false>
__global__ void __launch_bounds__(NET_TH) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_infer(const void *x, const float *mean, const float *std, const float *P, int n, float *prob)
{
    __shared__ __attribute__((aligned(16))) uint16_t Xs[16 * NET_XP];
    __shared__ __attribute__((aligned(16))) uint16_t Hs[16 * NET_HP];
    __shared__ __attribute__((aligned(16))) uint16_t Gs[16 * NET_HP];
    __shared__ __attribute__((aligned(16))) float w3s[IC_MLP_HID];
    __shared__ float held[HOLD ? IC_MLP_NOALLOC_ROWS : 1];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int col = wave * 16 + (lane & 15), row4 = (lane >> 4) * 4;
    const int ntile = (n + 15) / 16;
    // a thread's share of a tile's inputs: RAW one column of 16 rows (any
    // alignment of the caller's array), else two 16-byte pieces
    constexpr int NX = RAW ? 16 : 2;
    using XT = typename std::conditional<RAW, float, uint4>::type;
    XT xr[NX];
    auto ask = [&](int tile) {
#pragma unroll
        for (int e = 0; e < NX; ++e) {
            if constexpr (RAW) {
                const int b = tile * 16 + e;
                xr[e] = b < n ? ((const float *)x)[(long)b * IC_MLP_IN + tid] : 0.f;
            } else {
                const int b = tile * 16 + e * 8 + (tid >> 6);
                xr[e] = b < n ? ((const uint4 *)x)[(long)b * (IC_MLP_IN / 8) + lane] : make_uint4(0u, 0u, 0u, 0u);
            }
        }
    };
    int tile = blockIdx.x;
    ask(tile);
    float mu = 0.f, is = 1.f;
    if constexpr (RAW) {
        mu = mean[tid];
        is = 1.0f / std[tid];
    }
    float v1[16][8], v2[4][8];
    weights_ask<16>(P + IC_MLP_OFF_W1, wave, lane, v1);
    weights_ask<4>(P + IC_MLP_OFF_W2, wave, lane, v2);
    const float b1 = P[IC_MLP_OFF_B1 + col], b2 = P[IC_MLP_OFF_B2 + col], b3 = P[IC_MLP_OFF_B3];
    if (tid < IC_MLP_HID) w3s[tid] = bf2f(f2bf(P[IC_MLP_OFF_W3 + tid]));
    bf16x8_t w1[16], w2[4];
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) w1[kk] = pack8(v1[kk]);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) w2[kk] = pack8(v2[kk]);
    for (; tile < ntile; tile += gridDim.x) {
#pragma unroll
        for (int e = 0; e < NX; ++e) {
            if constexpr (RAW)
                Xs[e * NET_XP + tid] = f2bf((xr[e] - mu) * is);
            else
                *(uint4 *)&Xs[(e * 8 + (tid >> 6)) * NET_XP + lane * 8] = xr[e];
        }
        __syncthreads();
        if (tile + (int)gridDim.x < ntile) ask(tile + gridDim.x);
        float4_t z1, z2;
        tile_mfma<16, 1>(Xs, NET_XP, lane, w1, &z1);
#pragma unroll
        for (int t = 0; t < 4; ++t) Hs[(row4 + t) * NET_HP + col] = f2bf(relu(z1[t] + b1));
        __syncthreads();
        tile_mfma<4, 1>(Hs, NET_HP, lane, w2, &z2);
#pragma unroll
        for (int t = 0; t < 4; ++t) Gs[(row4 + t) * NET_HP + col] = f2bf(relu(z2[t] + b2));
        __syncthreads();
        // Gs is written again two barriers on, Xs was last read one barrier ago
        if (tid < 16 && tile * 16 + tid < n) {
            const float s = head_row(&Gs[tid * NET_HP], w3s, b3);
            (HOLD ? held : prob)[tile * 16 + tid] = 1.f / (1.f + expf(-s));
        }
    }
    if constexpr (HOLD) {
        __syncthreads();
        for (int b = tid; b < n; b += NET_TH) prob[b] = held[b];
    }
}

// ---------------------------------------------------------------------------
// weight gradients: dW = A^T D over the n rows of a minibatch, bf16 operands,
// fp32 accumulate on v_mfma_f32_16x16x32_bf16; dW1 (A = X, 512 columns) and
// dW2 (A = H1, 128 columns) in one launch.  A work-group of 4 waves computes a
// 64x64 tile of one slice of the rows, each wave a 32x32 quarter as 2x2 MFMA
// blocks.  Rows advance in MFMA steps of 32, staged through LDS four steps at
// a time and transposed there (row index contiguous), so that a lane's operand
// -- one column and eight consecutive rows -- is one 16-byte LDS read (pitch
// padded by 8 bf16 to spread them over the banks).  Each thread moves 16-byte
// pieces (eight columns of a row); the next stage's loads are in flight while
// the MFMAs of the current one run, from the other of two LDS buffers.  The
// slices' fp32 sums go to P[slice][m][n]; k_update adds them in slice order.
// 4,096 rows, both matrices: 17 us in two launches -> 7.4 us, of which pairs
// of rows stored as one word and the order of tile_at gave 4.
// ---------------------------------------------------------------------------
struct GradArgs {
    const uint16_t *A, *D;    // [n][M], [n][128]
    int M, nz;                // columns of A, slices
    float *P;                 // [nz][M][128]
};

constexpr int GEMM_KS = 128;               // rows per LDS stage (four MFMA steps)
constexpr int GEMM_KP = GEMM_KS + 8;       // padded LDS row, bf16

// The pieces of one stage of a 64-column tile of X[n][ld], rows 2p and 2p + 1
// of a piece in turn; rows from n on are zero.
DEV_EPI void tile_load(const uint16_t *X, int ld, int c0, int kb, int n, int tid, uint4 *out)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int k = kb + 2 * ((e >> 1) * 32 + (tid >> 3)) + (e & 1);
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (k < n) v = *(const uint4 *)(X + (long)k * ld + c0 + (tid & 7) * 8);
        out[e] = v;
    }
}

// Column r's eight-row pieces lie in the order p ^ (r / 8 % 8): the eight
// lanes that write one pair of rows then meet different banks (a row of 8
// columns further is 32 banks on, whatever the padding).
DEV_EPI int tile_at(int r, int k) { return r * GEMM_KP + (((k >> 3) ^ ((r >> 3) & 7)) << 3) + (k & 7); }

DEV_EPI void tile_store(uint16_t *L, int tid, const uint4 *in)
{
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int r = (tid & 7) * 8, k = 2 * (h * 32 + (tid >> 3));
        const uint32_t a[4] = {in[2 * h].x, in[2 * h].y, in[2 * h].z, in[2 * h].w};
        const uint32_t b[4] = {in[2 * h + 1].x, in[2 * h + 1].y, in[2 * h + 1].z, in[2 * h + 1].w};
#pragma unroll
        for (int i = 0; i < 8; ++i)
            *(uint32_t *)&L[tile_at(r + i, k)] =
                __builtin_amdgcn_perm(b[i >> 1], a[i >> 1], i & 1 ? 0x07060302u : 0x05040100u);
    }
}

__global__ void __launch_bounds__(256) k_wgrad(GradArgs g1, GradArgs g2, int n)
{
    __shared__ __attribute__((aligned(16))) uint16_t As[2][64 * GEMM_KP];
    __shared__ __attribute__((aligned(16))) uint16_t Bt[2][64 * GEMM_KP];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    int q = blockIdx.x;
    const int first = 2 * (g1.M / 64) * g1.nz;
    const bool two = q >= first;
    const GradArgs g = two ? g2 : g1;
    if (two) q -= first;
    const int n0 = (q & 1) * 64, m0 = ((q >> 1) % (g.M / 64)) * 64, z = (q >> 1) / (g.M / 64);
    const int wm = (wave & 1) * 32, wn = (wave >> 1) * 32;
    const int r = lane & 15, kq = (lane >> 4) * 8;
    const int nstep = (n + 31) / 32;
    const int s0 = (int)((long)nstep * z / g.nz), s1 = (int)((long)nstep * (z + 1) / g.nz);
    float4_t acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = float4_t{0.f, 0.f, 0.f, 0.f};
    const int kend = s1 * 32;
    uint4 ra[4], rb[4];
    int kb = s0 * 32;
    if (kb < kend) {
        tile_load(g.A, g.M, m0, kb, n, tid, ra);
        tile_load(g.D, IC_MLP_HID, n0, kb, n, tid, rb);
    }
    for (int buf = 0; kb < kend; kb += GEMM_KS, buf ^= 1) {
        // the buffer written here was last read two stages ago, before the
        // barrier of the previous stage
        tile_store(As[buf], tid, ra);
        tile_store(Bt[buf], tid, rb);
        __syncthreads();
        if (kb + GEMM_KS < kend) {
            tile_load(g.A, g.M, m0, kb + GEMM_KS, n, tid, ra);
            tile_load(g.D, IC_MLP_HID, n0, kb + GEMM_KS, n, tid, rb);
        }
        const int nk = (kend - kb < GEMM_KS ? kend - kb : GEMM_KS) / 32;
        for (int kk = 0; kk < nk; ++kk) {
            bf16x8_t a[2], b[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) a[i] = *(const bf16x8_t *)&As[buf][tile_at(wm + 16 * i + r, kk * 32 + kq)];
#pragma unroll
            for (int j = 0; j < 2; ++j) b[j] = *(const bf16x8_t *)&Bt[buf][tile_at(wn + 16 * j + r, kk * 32 + kq)];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
        }
    }
    float *P = g.P + (long)z * g.M * IC_MLP_HID;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                P[(m0 + wm + 16 * i + (lane >> 4) * 4 + t) * IC_MLP_HID + n0 + wn + 16 * j + r] = acc[i][j][t];
}

// ---------------------------------------------------------------------------
// training: forward and backward of a minibatch's rows in one launch
//
// One work-group takes one chunk of the rows (the chunks in which the bias and
// w3 gradients are summed), in tiles of 64: both layers, the head, the loss,
// dZ2 = dz w3 [H2 > 0], dZ1 = (dZ2 W2^T) [H1 > 0] and the chunk's column sums
// (rows ascending), with every operand between them in LDS.  What the weight
// gradients need goes to memory as bf16: the gathered rows, H1, dZ2, dZ1.  The
// weights come as packed operands (below), W2 a second time transposed.  Bound
// by the latency of the phases of a tile (at 4,096 rows, where a chunk is one
// tile: layers, dZ2 and dZ1 5 us, head 1.2, sums 0.7, the rest the rows and the
// weights on their way; two tiles of 32 rows took 26 us).  A minibatch of 4,096 rows: 205 us in 17
// launches -> 35 us in three, this one 21 us.
// ---------------------------------------------------------------------------
// The bf16 weights of k_rows, as each lane's 16-byte MFMA B operands: operand
// (step kk, wave, lane) of W1, then W2, then W2^T.  k_update writes them with
// the parameters, so that a work-group asks for 24 pieces a lane and rounds
// nothing (192 fp32 values a lane and their rounding: 31 us a launch against 26).
constexpr int PACK_W2 = IC_MLP_IN * IC_MLP_HID, PACK_W2T = PACK_W2 + IC_MLP_HID * IC_MLP_HID;
constexpr int PACK_N = PACK_W2T + IC_MLP_HID * IC_MLP_HID;

DEV_EPI int pack_at(int k, int n)
{
    return ((((k >> 5) * 8 + (n >> 4)) * 64) + ((k >> 3) & 3) * 16 + (n & 15)) * 8 + (k & 7);
}

// parameter q as bf16 to its places (biases and w3 have none)
DEV_EPI void pack_param(uint16_t *wp, int q, float w)
{
    if (q < IC_MLP_OFF_B1) {
        wp[pack_at(q / IC_MLP_HID, q % IC_MLP_HID)] = f2bf(w);
    } else if (q >= IC_MLP_OFF_W2 && q < IC_MLP_OFF_B2) {
        const int k = (q - IC_MLP_OFF_W2) / IC_MLP_HID, n = (q - IC_MLP_OFF_W2) % IC_MLP_HID;
        const uint16_t b = f2bf(w);
        wp[PACK_W2 + pack_at(k, n)] = b;
        wp[PACK_W2T + pack_at(n, k)] = b;
    }
}

__global__ void k_pack(const float *w, uint16_t *wp)
{
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q < IC_MLP_NPARAM) pack_param(wp, q, w[q]);
}

constexpr int ROWS_T = 64, ROWS_NB = ROWS_T / 16;   // rows of a tile, MFMA blocks
constexpr int ROWS_FP = IC_MLP_HID + 4;             // padded fp32 row of dZ1
constexpr int SUMS = 3 * IC_MLP_HID + 1;            // column sums of a chunk: db1, db2, dw3, db3

struct RowArgs {
    const uint16_t *X;        // normalised inputs, bf16
    const long *order;        // GATHER: row b of the minibatch is order[b] of X and y; else row b
    const uint8_t *y;
    const float *P;           // parameters
    const uint16_t *wp;       // their packed bf16 weights
    int n;                    // rows
    float pw;
    uint16_t *xb;             // GATHER: the gathered rows
    uint16_t *H1, *dZ2, *dZ1;
    float *loss;              // per row
    float *S;                 // [chunks][SUMS]
};

template <bool GATHER>
__global__ void __launch_bounds__(NET_TH) __attribute__((amdgpu_waves_per_eu(2, 2))) k_rows(RowArgs g)
{
    __shared__ __attribute__((aligned(16))) uint16_t Xs[ROWS_T * NET_XP];
    __shared__ __attribute__((aligned(16))) uint16_t Hs[ROWS_T * NET_HP], Gs[ROWS_T * NET_HP], Ds[ROWS_T * NET_HP];
    __shared__ __attribute__((aligned(16))) float Fs[ROWS_T * ROWS_FP];
    __shared__ __attribute__((aligned(16))) float w3s[IC_MLP_HID], dzs[ROWS_T];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int col = wave * 16 + (lane & 15), row4 = (lane >> 4) * 4;
    const int b0 = (int)((long)g.n * blockIdx.x / gridDim.x), b1 = (int)((long)g.n * (blockIdx.x + 1) / gridDim.x);
    // A tile's rows, one a lane (from b1 on the last one again: read, not
    // used), asked for a tile ahead of the inputs: wave w moves rows w, w + 8,
    // ..., a 16-byte piece a lane.
    constexpr int NX = ROWS_T / 8;
    long idx;
    u32x4_t xr[NX];
    uint8_t yr = 0;
    auto ask_rows = [&](int t0) {
        const int b = min(t0 + lane, b1 - 1);
        idx = GATHER ? g.order[b] : (long)b;
    };
    auto ask = [&]() {
        const int lo = (int)idx, hi = (int)(idx >> 32), w = __builtin_amdgcn_readfirstlane(wave);
#pragma unroll
        for (int e = 0; e < NX; ++e) {
            const long row = (long)(uint32_t)__builtin_amdgcn_readlane(lo, e * 8 + w) |
                             (long)__builtin_amdgcn_readlane(hi, e * 8 + w) << 32;
            xr[e] = ((const u32x4_t *)g.X)[row * (IC_MLP_IN / 8) + lane];
        }
        if (wave == 0) yr = g.y[idx];
    };
    ask_rows(b0);
    bf16x8_t w1[16], w2[4], w2t[4];
    const bf16x8_t *wp = (const bf16x8_t *)g.wp + wave * 64 + lane;
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) w1[kk] = wp[kk * 512];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        w2[kk] = wp[PACK_W2 / 8 + kk * 512];
        w2t[kk] = wp[PACK_W2T / 8 + kk * 512];
    }
    const float bias1 = g.P[IC_MLP_OFF_B1 + col], bias2 = g.P[IC_MLP_OFF_B2 + col], bias3 = g.P[IC_MLP_OFF_B3];
    if (tid < IC_MLP_HID) w3s[tid] = bf2f(f2bf(g.P[IC_MLP_OFF_W3 + tid]));
    ask();
    ask_rows(b0 + ROWS_T);
    float sum = 0.f;                        // this thread's column sum over the chunk
    for (int t0 = b0; t0 < b1; t0 += ROWS_T) {
        const int nr = min(ROWS_T, b1 - t0);
#pragma unroll
        for (int e = 0; e < NX; ++e) *(u32x4_t *)&Xs[(e * 8 + wave) * NET_XP + lane * 8] = xr[e];
        if (GATHER) {                        // rows past the chunk write its last row once more
#pragma unroll
            for (int e = 0; e < NX; ++e)
                ((u32x4_t *)g.xb)[(long)min(t0 + e * 8 + wave, b1 - 1) * (IC_MLP_IN / 8) + lane] = xr[e];
        }
        const float yy = (float)yr;
        __syncthreads();
        if (t0 + ROWS_T < b1) {
            ask();
            ask_rows(t0 + 2 * ROWS_T);
        }
        float4_t z[ROWS_NB];
        tile_mfma<16, ROWS_NB>(Xs, NET_XP, lane, w1, z);
#pragma unroll
        for (int q = 0; q < 4 * ROWS_NB; ++q)
            Hs[(16 * (q >> 2) + row4 + (q & 3)) * NET_HP + col] = f2bf(relu(z[q >> 2][q & 3] + bias1));
        __syncthreads();
        tile_mfma<4, ROWS_NB>(Hs, NET_HP, lane, w2, z);
#pragma unroll
        for (int q = 0; q < 4 * ROWS_NB; ++q)
            Gs[(16 * (q >> 2) + row4 + (q & 3)) * NET_HP + col] = f2bf(relu(z[q >> 2][q & 3] + bias2));
        __syncthreads();
        if (tid < ROWS_T) {
            float dz = 0.f;
            if (tid < nr) {
                const float s = head_row(&Gs[tid * NET_HP], w3s, bias3);
                const float p = 1.f / (1.f + expf(-s)), pw = g.pw;
                const int b = t0 + tid;
                // gradient of the mean weighted BCE
                dz = (p * (pw * yy + 1.f - yy) - pw * yy) / (float)g.n;
                // stable log-sigmoid terms: log p and log (1 - p)
                const float l = log1pf(expf(s >= 0.f ? -s : s));
                const float lsp = s >= 0.f ? -l : s - l;
                const float lsn = s >= 0.f ? -s - l : -l;
                g.loss[b] = -(pw * yy * lsp + (1.f - yy) * lsn);
            }
            dzs[tid] = dz;
        }
        __syncthreads();
        // this thread's eights of the 64 x 128 arrays: columns ec.., rows er and er + 32
        const int er = tid >> 4, ec = (tid & 15) * 8;
#pragma unroll
        for (int r = er; r < ROWS_T; r += NET_TH / 16) {
            float v[8];
            const float dz = dzs[r];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = bf2f(Gs[r * NET_HP + ec + e]) > 0.f ? dz * w3s[ec + e] : 0.f;
            const bf16x8_t d = pack8(v);
            *(bf16x8_t *)&Ds[r * NET_HP + ec] = d;
            if (r < nr) {
                *(bf16x8_t *)&g.dZ2[(long)(t0 + r) * IC_MLP_HID + ec] = d;
                *(uint4 *)&g.H1[(long)(t0 + r) * IC_MLP_HID + ec] = *(const uint4 *)&Hs[r * NET_HP + ec];
            }
        }
        __syncthreads();
        tile_mfma<4, ROWS_NB>(Ds, NET_HP, lane, w2t, z);
#pragma unroll
        for (int q = 0; q < 4 * ROWS_NB; ++q) {
            const int r = 16 * (q >> 2) + row4 + (q & 3);
            Fs[r * ROWS_FP + col] = bf2f(Hs[r * NET_HP + col]) > 0.f ? z[q >> 2][q & 3] : 0.f;
        }
        __syncthreads();
        // column sums, rows ascending, sixteen LDS reads in flight; waves 0-1
        // db1, 2-3 db2, 4-5 dw3, then db3
        const int j = tid & (IC_MLP_HID - 1);
        auto add_rows = [&](auto term) {
            int r = 0;
#pragma unroll 1
            for (; r + 16 <= nr; r += 16) {
                float v[16];
#pragma unroll
                for (int e = 0; e < 16; ++e) v[e] = term(r + e);
#pragma unroll
                for (int e = 0; e < 16; ++e) sum += v[e];
            }
#pragma unroll 1
            for (; r < nr; ++r) sum += term(r);
        };
        if (wave < 2) add_rows([&](int r) { return Fs[r * ROWS_FP + j]; });
        else if (wave < 4) add_rows([&](int r) { return bf2f(Gs[r * NET_HP + j]) > 0.f ? dzs[r] * w3s[j] : 0.f; });
        else if (wave < 6) add_rows([&](int r) { return dzs[r] * bf2f(Gs[r * NET_HP + j]); });
        else if (wave < 7) add_rows([&](int r) { return dzs[r]; });
#pragma unroll
        for (int r = er; r < ROWS_T; r += NET_TH / 16)
            if (r < nr) *(bf16x8_t *)&g.dZ1[(long)(t0 + r) * IC_MLP_HID + ec] = pack8(&Fs[r * ROWS_FP + ec]);
        // the next tile's first barriers order these reads before its writes
    }
    if (tid < SUMS) g.S[(long)blockIdx.x * SUMS + tid] = sum;
}

// The minibatch's gradient from its partial sums -- slices of the weights'
// (k_wgrad) and chunks of the others' (k_rows), each in order -- and Adam's
// step with it, or (grad) the gradient itself.  The group after the
// parameters' sums the rows' losses in fp64 (fixed order: thread-strided, then
// a pairwise tree).
struct StepArgs {
    const float *P1, *P2, *S;
    int nz1, nz2, nc;
    float *grad;                           // the gradient; NULL: Adam
    float *w, *m1, *m2;
    uint16_t *wp;                          // packed weights
    float lr, b1, b2, eps, c1, c2;
    const float *loss;
    int n;
    double *loss_out;
};

DEV_EPI float ordered_sum(const float *p, int count, int stride)
{
    float s = 0.f;
    int z = 0;
    for (; z + 16 <= count; z += 16) {
        float v[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = p[(z + e) * stride];
#pragma unroll
        for (int e = 0; e < 16; ++e) s += v[e];
    }
    for (; z < count; ++z) s += p[z * stride];
    return s;
}

__global__ void __launch_bounds__(256) k_update(StepArgs g)
{
    const int q = blockIdx.x * 256 + threadIdx.x;
    if (blockIdx.x == gridDim.x - 1) {
        __shared__ double sh[256];
        double s = 0.0;
        for (int b = threadIdx.x; b < g.n; b += 256) s += (double)g.loss[b];
        sh[threadIdx.x] = s;
        __syncthreads();
        for (int w = 128; w > 0; w >>= 1) {
            if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
            __syncthreads();
        }
        if (threadIdx.x == 0) *g.loss_out = sh[0];
        return;
    }
    if (q >= IC_MLP_NPARAM) return;
    float gg;
    if (q < IC_MLP_OFF_B1) gg = ordered_sum(g.P1 + q, g.nz1, IC_MLP_IN * IC_MLP_HID);
    else if (q < IC_MLP_OFF_W2) gg = ordered_sum(g.S + (q - IC_MLP_OFF_B1), g.nc, SUMS);
    else if (q < IC_MLP_OFF_B2) gg = ordered_sum(g.P2 + (q - IC_MLP_OFF_W2), g.nz2, IC_MLP_HID * IC_MLP_HID);
    else gg = ordered_sum(g.S + IC_MLP_HID + (q - IC_MLP_OFF_B2), g.nc, SUMS);      // db2, dw3, db3
    if (g.grad) {
        g.grad[q] = gg;
        return;
    }
    const float m1 = g.b1 * g.m1[q] + (1.f - g.b1) * gg;
    const float m2 = g.b2 * g.m2[q] + (1.f - g.b2) * gg * gg;
    g.m1[q] = m1;
    g.m2[q] = m2;
    const float mh = m1 / g.c1, vh = m2 / g.c2;
    float w = g.w[q];
    w -= g.lr * mh / (sqrtf(vh) + g.eps);
    g.w[q] = w;
    pack_param(g.wp, q, w);
}

// z-score statistics of n rows x 512 columns in fp64, rows ascending within a
// column: mu (MEAN) or the sum of (x - mu)^2.  A column's sum is one chain of
// n dependent additions, so a work-group takes 16 columns: all 16 waves bring
// tiles of 512 rows (64 bytes a row) into LDS as the terms of the sum, and 16
// lanes of the first wave add the previous tile meanwhile: 0.27 ms a pass over
// 40,000 rows, 16 cycles an addition (on the host, and after the upload, both
// passes took about 9 ms).
constexpr int STAT_C = 16, STAT_R = 512, STAT_P = STAT_C + 1;

template <bool MEAN>
__global__ void __launch_bounds__(1024) k_stats(const float *raw, long n, double *mu, double *var)
{
    __shared__ double T[2][STAT_R * STAT_P];
    const int tid = threadIdx.x, f0 = blockIdx.x * STAT_C;
    const int c4 = (tid & 3) * 4, r = tid >> 2;                  // four columns of rows r and r + 256
    double m[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) m[e] = MEAN ? 0.0 : mu[f0 + c4 + e];
    float4 v[2];
    auto ask = [&](long b) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
            v[h] = b + r + 256 * h < n ? *(const float4 *)(raw + (b + r + 256 * h) * IC_MLP_IN + f0 + c4)
                                       : make_float4(0.f, 0.f, 0.f, 0.f);
    };
    double sum = 0.0;
    ask(0);
    int buf = 0;
    for (long b = 0; b < n; b += STAT_R, buf ^= 1) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float x[4] = {v[h].x, v[h].y, v[h].z, v[h].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                double d = (double)x[e];
                if (!MEAN) {
                    d = d - m[e];
                    d = d * d;
                }
                T[buf][(r + 256 * h) * STAT_P + c4 + e] = d;
            }
        }
        __syncthreads();               // the other buffer was read before this barrier
        if (b + STAT_R < n) ask(b + STAT_R);
        if (tid < STAT_C) {
            const int nr = (int)min((long)STAT_R, n - b);
            const double *q = &T[buf][tid];
            int i = 0;
            double d[2][16];           // the next sixteen terms are read while these are added
            auto get = [&](int i0, double *t) {
#pragma unroll
                for (int e = 0; e < 16; ++e) t[e] = q[(i0 + e) * STAT_P];
            };
            get(0, d[0]);
            for (; i + 32 <= nr; i += 32) {
                get(i + 16, d[1]);
#pragma unroll
                for (int e = 0; e < 16; ++e) sum += d[0][e];
                get(min(i + 32, STAT_R - 16), d[0]);
#pragma unroll
                for (int e = 0; e < 16; ++e) sum += d[1][e];
            }
            for (; i < nr; ++i) sum += q[i * STAT_P];
        }
    }
    if (tid < STAT_C) (MEAN ? mu : var)[f0 + tid] = MEAN ? sum / (double)n : sum;
}

__global__ void k_to_bf16(const float *x, uint16_t *y, long n)
{
    const long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q < n) y[q] = f2bf(x[q]);
}

// normalised bf16 inputs from raw fp32 features
__global__ void k_normalise(const float *raw, const float *mean, const float *istd, long n, uint16_t *xb)
{
    const long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n * IC_MLP_IN) return;
    const int f = (int)(q % IC_MLP_IN);
    xb[q] = f2bf((raw[q] - mean[f]) * istd[f]);
}

// learned flags: p >= threshold -> refine, else coarsen-eligible
__global__ void k_prob_flags(const float *prob, const int *items, int n, float threshold, int8_t *flags)
{
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q < n) flags[items[q]] = prob[q] >= threshold ? 1 : -1;
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
namespace {

template <class T>
struct Buf {
    T *p = nullptr;
    size_t n = 0;
    explicit Buf(size_t count = 0) { alloc(count); }
    void alloc(size_t count)
    {
        dev_free(p);
        p = nullptr;
        n = count;
        if (count && !(p = (T *)dev_malloc(count * sizeof(T)))) throw std::runtime_error("device allocation failed");
    }
    ~Buf() { dev_free(p); }
    Buf(const Buf &) = delete;
    Buf &operator=(const Buf &) = delete;
};

}  // namespace

MlpDevice::MlpDevice() = default;

MlpDevice::~MlpDevice()
{
    for (void *q : {(void *)w, (void *)mean, (void *)istd, (void *)xb, (void *)prob}) dev_free(q);
}

void MlpDevice::set(const float *params, const float *mean_h, const float *std_h)
{
    if (!w) {
        w = (float *)dev_malloc(IC_MLP_NPARAM * sizeof(float));
        mean = (float *)dev_malloc(IC_MLP_IN * sizeof(float));
        istd = (float *)dev_malloc(IC_MLP_IN * sizeof(float));
        if (!w || !mean || !istd) throw std::runtime_error("device allocation failed");
    }
    std::vector<float> is(IC_MLP_IN);
    for (int f = 0; f < IC_MLP_IN; ++f) is[f] = 1.0f / std_h[f];
    if (hipMemcpy(w, params, IC_MLP_NPARAM * sizeof(float), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(mean, mean_h, IC_MLP_IN * sizeof(float), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(istd, is.data(), IC_MLP_IN * sizeof(float), hipMemcpyHostToDevice) != hipSuccess)
        throw std::runtime_error("hipMemcpy failed");
    if (hipDeviceSynchronize() != hipSuccess) throw std::runtime_error("device error");
    ready = true;
}

void MlpDevice::reserve(int n)
{
    if (n <= cap) return;
    for (void *q : {(void *)xb, (void *)prob}) dev_free(q);
    xb = nullptr;
    prob = nullptr;
    cap = n + n / 2 + 64;
    xb = (uint16_t *)dev_malloc((size_t)cap * IC_MLP_IN * sizeof(uint16_t));
    prob = (float *)dev_malloc((size_t)cap * sizeof(float));
    if (!xb || !prob) throw std::runtime_error("device allocation failed");
}

// One work-group per 16-row tile up to one per compute unit: beyond that a
// group takes several tiles with the weights it holds, which saves their
// 320 KB a tile.
static dim3 infer_grid(long n) { return dim3((unsigned)std::min((n + 15) / 16, 256L)); }

// forward pass over n rows of xb (already filled) -> prob
void MlpDevice::forward(hipStream_t s, int n)
{
    hipLaunchKernelGGL((k_infer<false>), infer_grid(n), dim3(NET_TH), 0, s, (const void *)xb, (const float *)nullptr,
                       (const float *)nullptr, (const float *)w, n, prob);
}

void mlp_features(hipStream_t s, const KArgs &a, int bi, int bj, int bk, const int *items,
                  const int *nitems, int n, float *raw, const float *mean, const float *istd, uint16_t *xb)
{
#define IC_INSTANTIATE(BI, BJ, BK)                                                                      \
    if (bi == BI && bj == BJ && bk == BK) {                                                            \
        const dim3 g = BI * BJ * BK == 64 ? dim3(std::max(1, (n + FEATURE_BLOCKS - 1) / FEATURE_BLOCKS))  \
                                          : dim3(std::max(1, std::min(n, 16384)), 4);                   \
        hipLaunchKernelGGL((k_features<BI, BJ, BK>), g, dim3(256), 0, s, a, items, nitems, raw, mean,   \
                           istd, xb);                                                                   \
        return;                                                                                        \
    }
#include "shapes.inc"
#undef IC_INSTANTIATE
}

void mlp_prob_flags(hipStream_t s, const float *prob, const int *items, int n, float threshold, int8_t *flags)
{
    hipLaunchKernelGGL(k_prob_flags, dim3((n + 255) / 256), dim3(256), 0, s, prob, items, n, threshold, flags);
}

// The buffers and launches of one forward and backward pass of n rows.
struct Pass {
    int n = 0, nc = 0, nz1 = 0, nz2 = 0;
    Buf<uint16_t> wp, H1, dZ2, dZ1;
    Buf<float> loss, P1, P2, S;
    // Slices of the rows in the weight gradients: enough for about 256
    // work-groups a matrix, at most 32, each at least 4 MFMA steps.
    static int slices(int n, int tiles) { return std::max(1, std::min({32, (n + 31) / 32 / 4, (256 + tiles - 1) / tiles})); }
    void alloc(int rows)
    {
        n = rows;
        nc = std::max(1, std::min(64, n / 32));
        nz1 = slices(n, 2 * IC_MLP_IN / 64);
        nz2 = slices(n, 2 * IC_MLP_HID / 64);
        wp.alloc(PACK_N);
        for (Buf<uint16_t> *b : {&H1, &dZ2, &dZ1}) b->alloc((size_t)n * IC_MLP_HID);
        loss.alloc(n);
        P1.alloc((size_t)nz1 * IC_MLP_IN * IC_MLP_HID);
        P2.alloc((size_t)nz2 * IC_MLP_HID * IC_MLP_HID);
        S.alloc((size_t)nc * SUMS);
    }
    // the packed weights of the first pass; each Adam step then leaves the next one's
    void pack(hipStream_t s, const float *w)
    {
        hipLaunchKernelGGL(k_pack, dim3((IC_MLP_NPARAM + 255) / 256), dim3(256), 0, s, w, wp.p);
    }
    // X, y: all rows; order: the minibatch's (NULL: rows 0 .. n-1); xb: room for its gathered inputs
    void run(hipStream_t s, const uint16_t *X, const long *order, const uint8_t *y, float pw, const float *w,
             uint16_t *xb, StepArgs st)
    {
        RowArgs r{X, order, y, w, wp.p, n, pw, xb, H1.p, dZ2.p, dZ1.p, loss.p, S.p};
        if (order) hipLaunchKernelGGL((k_rows<true>), dim3(nc), dim3(NET_TH), 0, s, r);
        else hipLaunchKernelGGL((k_rows<false>), dim3(nc), dim3(NET_TH), 0, s, r);
        GradArgs g1{order ? xb : X, dZ1.p, IC_MLP_IN, nz1, P1.p}, g2{H1.p, dZ2.p, IC_MLP_HID, nz2, P2.p};
        hipLaunchKernelGGL(k_wgrad, dim3(2 * (IC_MLP_IN / 64) * nz1 + 2 * (IC_MLP_HID / 64) * nz2), dim3(256), 0, s,
                           g1, g2, n);
        st.wp = wp.p;
        st.P1 = P1.p;
        st.P2 = P2.p;
        st.S = S.p;
        st.nz1 = nz1;
        st.nz2 = nz2;
        st.nc = nc;
        st.loss = loss.p;
        st.n = n;
        hipLaunchKernelGGL(k_update, dim3((IC_MLP_NPARAM + 255) / 256 + 1), dim3(256), 0, s, st);
    }
};

// Gradients (fp32, params layout) and mean loss of n rows of normalised fp32
// inputs (converted to bf16 here); params: fp32 weights.
void mlp_grad(const float *xnorm, const uint8_t *y, int n, float pw, const float *params, float *grad_out,
              float *loss_out)
{
    hipStream_t s = nullptr;
    Buf<float> x((size_t)n * IC_MLP_IN), w(IC_MLP_NPARAM), grad(IC_MLP_NPARAM);
    Buf<uint16_t> xb((size_t)n * IC_MLP_IN);
    Buf<uint8_t> yd(n);
    Buf<double> lsum(1);
    Pass pass;
    pass.alloc(n);
    if (hipMemcpy(x.p, xnorm, (size_t)n * IC_MLP_IN * sizeof(float), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(w.p, params, IC_MLP_NPARAM * sizeof(float), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(yd.p, y, n, hipMemcpyHostToDevice) != hipSuccess)
        throw std::runtime_error("hipMemcpy failed");
    hipLaunchKernelGGL(k_to_bf16, dim3(((long)n * IC_MLP_IN + 255) / 256), dim3(256), 0, s, x.p, xb.p,
                       (long)n * IC_MLP_IN);
    pass.pack(s, w.p);
    StepArgs st{};
    st.grad = grad.p;
    st.loss_out = lsum.p;
    pass.run(s, xb.p, nullptr, yd.p, pw, w.p, nullptr, st);
    std::vector<float> lrow(n);
    if (hipMemcpy(grad_out, grad.p, IC_MLP_NPARAM * sizeof(float), hipMemcpyDeviceToHost) != hipSuccess ||
        hipMemcpy(lrow.data(), pass.loss.p, n * sizeof(float), hipMemcpyDeviceToHost) != hipSuccess)
        throw std::runtime_error("hipMemcpy failed");
    double l = 0.0;
    for (int b = 0; b < n; ++b) l += lrow[b];
    *loss_out = (float)(l / n);
}

void mlp_train(const float *raw, const uint8_t *y, long n, const MlpHparams &hp, float *params, float *mean_out,
               float *std_out, float *loss_epochs)
{
    hipStream_t s = nullptr;
    auto H2D = [](void *d, const void *h, size_t bytes) {
        if (hipMemcpy(d, h, bytes, hipMemcpyHostToDevice) != hipSuccess) throw std::runtime_error("hipMemcpy failed");
    };
    auto D2H = [](void *h, const void *d, size_t bytes) {
        if (hipMemcpy(h, d, bytes, hipMemcpyDeviceToHost) != hipSuccess) throw std::runtime_error("hipMemcpy failed");
    };
    const int B = hp.batch;
    const long nbatch = n / B;
    Buf<float> rawd((size_t)n * IC_MLP_IN), mean(IC_MLP_IN), istd(IC_MLP_IN), w(IC_MLP_NPARAM), m1(IC_MLP_NPARAM),
        m2(IC_MLP_NPARAM);
    Buf<double> stat(2 * IC_MLP_IN), lossacc;            // lossacc: per-minibatch loss sums, read once per epoch
    Buf<uint16_t> xall, xb;
    Buf<uint8_t> yall;
    Buf<long> orderd;
    Pass pass;
    // the device is done with the buffers before any of them is given back, also
    // where an allocation fails while the statistics run
    struct Idle {
        ~Idle() { (void)hipStreamSynchronize(nullptr); }
    } idle;
    H2D(rawd.p, raw, (size_t)n * IC_MLP_IN * sizeof(float));
    // per-feature z-score statistics of the training set (fp64)
    hipLaunchKernelGGL((k_stats<true>), dim3(IC_MLP_IN / STAT_C), dim3(1024), 0, s, (const float *)rawd.p, n, stat.p,
                       stat.p + IC_MLP_IN);
    hipLaunchKernelGGL((k_stats<false>), dim3(IC_MLP_IN / STAT_C), dim3(1024), 0, s, (const float *)rawd.p, n, stat.p,
                       stat.p + IC_MLP_IN);
    xall.alloc((size_t)n * IC_MLP_IN);
    xb.alloc((size_t)B * IC_MLP_IN);
    yall.alloc(n);
    orderd.alloc(n);
    lossacc.alloc(std::max(nbatch, 1L));
    pass.alloc(B);
    long npos = 0;
    for (long b = 0; b < n; ++b) npos += y[b] ? 1 : 0;
    const float pw = hp.pos_weight > 0.f ? hp.pos_weight : (npos > 0 ? (float)(n - npos) / (float)npos : 1.f);
    // deterministic shuffle per epoch (xorshift on the host)
    std::vector<long> order(n);
    for (long b = 0; b < n; ++b) order[b] = b;
    uint64_t st = hp.seed * 2654435761ull + 88172645463325252ull;
    auto rnd = [&]() {
        st ^= st << 13;
        st ^= st >> 7;
        st ^= st << 17;
        return st;
    };
    auto shuffle = [&]() {
        for (long b = n - 1; b > 0; --b) std::swap(order[b], order[rnd() % (uint64_t)(b + 1)]);
    };
    if (hp.epochs > 0) shuffle();                        // while the statistics run
    std::vector<double> stat_h(2 * IC_MLP_IN);
    D2H(stat_h.data(), stat.p, 2 * IC_MLP_IN * sizeof(double));
    std::vector<float> mean_h(IC_MLP_IN), std_h(IC_MLP_IN), istd_h(IC_MLP_IN);
    for (int f = 0; f < IC_MLP_IN; ++f) {
        mean_h[f] = (float)stat_h[f];
        double sd = std::sqrt(stat_h[IC_MLP_IN + f] / (double)n);
        if (!(sd > 1e-6)) sd = 1.0;
        std_h[f] = (float)sd;
        istd_h[f] = 1.0f / std_h[f];
    }
    H2D(mean.p, mean_h.data(), IC_MLP_IN * sizeof(float));
    H2D(istd.p, istd_h.data(), IC_MLP_IN * sizeof(float));
    H2D(w.p, params, IC_MLP_NPARAM * sizeof(float));
    H2D(yall.p, y, n);
    (void)hipMemset(m1.p, 0, IC_MLP_NPARAM * sizeof(float));
    (void)hipMemset(m2.p, 0, IC_MLP_NPARAM * sizeof(float));
    hipLaunchKernelGGL(k_normalise, dim3(((long)n * IC_MLP_IN + 255) / 256), dim3(256), 0, s, rawd.p, mean.p, istd.p,
                       n, xall.p);
    pass.pack(s, w.p);
    std::vector<double> lsums(std::max(nbatch, 1L));
    auto read_losses = [&](int ep) {                     // an epoch's minibatch losses, summed in batch order
        D2H(lsums.data(), lossacc.p, nbatch * sizeof(double));
        double lsum = 0.0;
        for (long i = 0; i < nbatch; ++i) lsum += lsums[i];
        if (loss_epochs) loss_epochs[ep] = (float)(lsum / (double)(nbatch * B));
    };
    long t = 0;
    for (int ep = 0; ep < hp.epochs; ++ep) {
        if (ep > 0) {
            shuffle();                                   // while the last epoch's steps run
            read_losses(ep - 1);
        }
        H2D(orderd.p, order.data(), n * sizeof(long));
        long q = 0;
        for (long b0 = 0; b0 + B <= n; b0 += B, ++q) {
            ++t;
            const float c1 = 1.f - std::pow(hp.beta1, (float)t), c2 = 1.f - std::pow(hp.beta2, (float)t);
            StepArgs st{};
            st.w = w.p;
            st.m1 = m1.p;
            st.m2 = m2.p;
            st.lr = hp.lr;
            st.b1 = hp.beta1;
            st.b2 = hp.beta2;
            st.eps = hp.eps;
            st.c1 = c1;
            st.c2 = c2;
            st.loss_out = lossacc.p + q;
            pass.run(s, xall.p, orderd.p + b0, yall.p, pw, w.p, xb.p, st);
        }
    }
    if (hp.epochs > 0) read_losses(hp.epochs - 1);
    D2H(params, w.p, IC_MLP_NPARAM * sizeof(float));
    std::memcpy(mean_out, mean_h.data(), IC_MLP_IN * sizeof(float));
    std::memcpy(std_out, std_h.data(), IC_MLP_IN * sizeof(float));
}

void mlp_infer(const float *raw, long n, const float *params, const float *mean, const float *std, float *prob)
{
    MlpDevice d;
    d.set(params, mean, std);
    const long chunk = 65536;
    d.reserve((int)std::min(n, chunk));
    Buf<float> rawd((size_t)std::min(n, chunk) * IC_MLP_IN);
    for (long b0 = 0; b0 < n; b0 += chunk) {
        const long m = std::min(chunk, n - b0);
        if (hipMemcpy(rawd.p, raw + b0 * IC_MLP_IN, (size_t)m * IC_MLP_IN * sizeof(float), hipMemcpyHostToDevice) !=
            hipSuccess)
            throw std::runtime_error("hipMemcpy failed");
        hipLaunchKernelGGL(k_normalise, dim3((m * IC_MLP_IN + 255) / 256), dim3(256), 0, 0, rawd.p, d.mean, d.istd, m,
                           d.xb);
        d.forward(0, (int)m);
        if (hipMemcpy(prob + b0, d.prob, m * sizeof(float), hipMemcpyDeviceToHost) != hipSuccess)
            throw std::runtime_error("hipMemcpy failed");
    }
}

// ---------------------------------------------------------------------------
// inference without allocation: the launch reads the caller's arrays and writes
// the probabilities, with no intermediate value in device memory.  Where the
// probabilities overlie inputs (a caller that is done with them), no
// work-group may write before the inputs under its rows are read: the rows of
// raw under prob go first, in one work-group that holds their results back
// (prob's n values lie on at most 9 rows when n is 4,096); the other rows'
// probabilities then fall on those rows or outside raw.  On the network's own
// arrays all rows go that way.
// ---------------------------------------------------------------------------
void mlp_infer_noalloc(const float *raw, long n, const float *params, const float *mean, const float *std,
                       float *prob, hipStream_t s)
{
    if (n < 0 || n > IC_MLP_NOALLOC_ROWS) throw std::invalid_argument("row count outside 0 .. IC_MLP_NOALLOC_ROWS");
    if (n == 0) return;
    const uintptr_t p0 = (uintptr_t)prob, p1 = (uintptr_t)(prob + n);
    auto on_prob = [&](const float *q, long count) { return (uintptr_t)q < p1 && (uintptr_t)(q + count) > p0; };
    long r0 = n, r1 = n;                     // rows r0 .. r1 - 1 first
    if (on_prob(params, IC_MLP_NPARAM) || on_prob(mean, IC_MLP_IN) || on_prob(std, IC_MLP_IN)) {
        r0 = 0;
    } else if (on_prob(raw, n * IC_MLP_IN)) {
        const uintptr_t base = (uintptr_t)raw, row = IC_MLP_IN * sizeof(float);
        r0 = p0 > base ? (long)((p0 - base) / row) : 0;
        r1 = std::min(n, (long)((p1 - base + row - 1) / row));
    }
    if (r0 < r1)
        hipLaunchKernelGGL((k_infer<true, true>), dim3(1), dim3(NET_TH), 0, s, (const void *)(raw + r0 * IC_MLP_IN), mean,
                           std, params, (int)(r1 - r0), prob + r0);
    for (const auto &part : {std::pair<long, long>{0, r0}, {r1, n}})
        if (part.first < part.second)
            hipLaunchKernelGGL((k_infer<true>), infer_grid(part.second - part.first), dim3(NET_TH), 0, s,
                               (const void *)(raw + part.first * IC_MLP_IN), mean, std, params,
                               (int)(part.second - part.first), prob + part.first);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) throw std::runtime_error(std::string("launch failed: ") + hipGetErrorString(e));
}

// Per-step kernels of the certified sub-vocabulary LM-head path and the entry points that enqueue them.
//
//   bound_rows_kernel, bound_kernel / bound_tile_kernel / bound_mfma_kernel + bound_finish_kernel
//                      U[b,c] = <mu_c,h_b> + R_c ||h_b|| + bmax_c  for up to four sequences / up to 16 with short rows or many
//                      clusters / more                                                          (Eq. "cluster_bound")
//   round0_kernel      per sequence: shortest prefix of the bound order holding >= max(k,1) rows, next bound, log tail
//                      mass (Algorithm 1: queue, PopMax); logits of the prefix rows of W' (Algorithm 1: sparse GEMV);
//                      top-k, log-sum-exp and both certificates, or the plan of the next round
//                                                                                      (Definitions 1-2, Theorems 1-2)
//   tail_kernel        only when some sequence needs it: further rounds (tile GEMV + certification), then all V logits,
//                      top-k and log-sum-exp for the sequences that fall back                          (Eq. "logit")
//   full_gemv_kernel / full_mfma_kernel   all V logits as an entry point of their own
//
// Everything is enqueued on the caller's stream; decisions (round 1, fallback) are taken on the device.
// The open set of a sequence is {c : key_c >= kappa} for a 64-bit key that encodes (bound, cluster id), so the
// common path needs reductions only; the bound order is sorted only when the softmax test asks for a longer prefix.
#include "csv_common.h"

#include <math.h>
#include <type_traits>
#include <stdarg.h>
#include <stdlib.h>
#include <string.h>
#include <pthread.h>

// ------------------------------------------------------------------------------------------------ errors
static thread_local char g_err[512] = "";
void csv_set_error(const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
}
extern "C" const char* csv_last_error(void) { return g_err; }

typedef unsigned long long u64;

// ------------------------------------------------------------------------------------------------ arguments
struct StepArgs {
    int V, d, C;
    const uint16_t* Wp;
    const float* bp;
    const int32_t* perm;
    const float* mu;
    const uint16_t* mu16;   // bf16 copy of the centroids, or NULL
    const float* R;
    const float* bmax;
    const int32_t* n;
    const int32_t* off;
    const float* lnn;
    const int4* cmeta;      // per cluster {first row, rows, bits of ln n, 0}
    const float2* bt;       // top-m bias table, [C * bt_m] pairs (radius, bias), or NULL
    const float4* ang;      // angular index: {cos, sin of the angular radius, largest, smallest row norm} per cluster, or NULL
    int bt_m;
    float ln_nmax;
    int B, B_max, K_cap, Npad, n_chunks, tile_stride;
    int sp_chunks;     // most STAGE_CAP-sized chunks a sequence's scored rows can span
    int cand_chunks;   // chunk stride of the candidate buffers
    int tail_lds;      // dynamic LDS bytes of the tail kernel
    int spin_limit;    // polls a grid barrier of the tail kernel waits before it gives the step up
    int* host_history; // pinned host word for the history of steps that needed the tail (device-visible address)
    int r0_h_off;      // offset of h in the round-0 kernel's LDS arena, in 128-bit units (behind the cluster data)
    float* U;
    float* hnorm;
    float* bound_partial;   // [BOUND_KS_MAX * B * C] K-slice partial sums of the batched bound product
    SeqState* st;
    int32_t* sel;
    float* slog;
    int32_t* sid;
    u64* slots;        // [B*CSV_SLOT_ROWS] round-0 hand-over words
    Tile* tiles[2];
    int32_t* counters;
    int32_t* fb_list;
    float* fb_logits;
    float* cand_val;
    int32_t* cand_id;
    float* cand_max;
    float* cand_sum;
    const uint16_t* h;
    int k, K_max, combine, use_k, use_s;
    int max_rounds, delta_clusters, relax;   // fallback levels
    float lam;   // ln(eps/(1-eps)); +inf when eps >= 1
    float lam2;  // the same for the relaxed tolerance 2 eps
    float top_p; // nucleus mass asked for (0 = none)
    csv_step_out out;
};

#define TILE_ROWS 8        // rows per work item of the gathered GEMV (4 waves x 2 rows)
#define SEQ_THREADS 512    // block size of the per-sequence kernels (seed, cert, fallback top-k)
#define STAGE_CAP 4096     // scored logits kept in LDS by cert_kernel when a sequence has at most this many
static_assert(STAGE_CAP == CSV_SLOT_ROWS, "the round-0 slots hold exactly what one block certifies from LDS");
#define FB_CHUNK 8192      // rows per block of the fallback top-k first stage
#define FULL_G 4           // sequences per pass of the vector full-vocabulary product
#define BIGQ 32            // clusters whose tiles are written cooperatively per emit call

#define CSV_STATIC_MAX_DEVICES 64   // devices the per-device host tables of this file cover

// Key of a value for ordering: -0 and +0 compare equal.
__device__ __forceinline__ uint32_t lkey(float v) { return fkey(v + 0.0f); }
__device__ __forceinline__ u64 ckey(float U, int c) { return ((u64)lkey(U) << 32) | (u64)(0xFFFFFFFFu - (uint32_t)c); }
__device__ __forceinline__ float ckey_bound(u64 k) { return fkey_inv((uint32_t)(k >> 32)); }

// Zero the step's counters: the fixed slots and, of every per-sequence row, the entries of the B sequences in use.
// Before that, whether the previous step needed anything after round 0 is shifted into the history word (device
// copy behind the reset range, and a pinned host copy that the next calls read without synchronising).
__device__ __forceinline__ void reset_step_counters(int* counters, int B, int nthreads, int* host_history, u64* slots, int B_max) {
    constexpr int rows = (CNT_TOTAL - CNT_TILES) / CSV_MAX_BATCH;
    if (counters[CNT_SLOTS_DIRTY] != 0) {     // an earlier step gave up with logits still on their way: empty every slot
        for (size_t i = threadIdx.x; i < (size_t)B_max * CSV_SLOT_ROWS; i += nthreads) slots[i] = CSV_SLOT_EMPTY;
        __syncthreads();
        if (threadIdx.x == 0) counters[CNT_SLOTS_DIRTY] = 0;
    }
    if (threadIdx.x == 0) {      // low half: steps that needed the tail; high half: steps with a fallback
        const unsigned old = (unsigned)counters[CNT_HISTORY];
        const unsigned lo = ((old << 1) | (unsigned)(counters[CNT_TAIL_NEEDED] != 0)) & 0xffffu;
        const unsigned hi = (((old >> 16) << 1) | (unsigned)(counters[CNT_FALLBACK] != 0)) & 0x7fffu;
        const int h = (int)(lo | (hi << 16));
        counters[CNT_HISTORY] = h;
        if (host_history) *host_history = h;
    }
    __syncthreads();             // called by every thread of one block: the zeroing below must not overtake the reads
    for (int i = threadIdx.x; i < CNT_TILES + rows * B; i += nthreads) {
        const int j = i - CNT_TILES;
        counters[i < CNT_TILES ? i : CNT_TILES + (j / B) * CSV_MAX_BATCH + (j % B)] = 0;
    }
}

// ================================================================================================ bounds
// What a cluster adds to <mu_c,h>: R_c ||h|| + max bias (Eq. "cluster_bound"), or, with a top-m bias table, the
// largest of its m terms rho_j ||h|| + beta_j (the m-1 tokens with the largest biases one by one, the rest together).
// With an angular index (spherical clustering) mu_c is a unit direction and the bound is
//   rho ||h|| cos(phi - theta_c) = rho (t cos(theta_c) + sqrt(||h||^2 - t^2) sin(theta_c)),  t = <mu_c,h> = ||h|| cos(phi),
// outside the cluster's cone and rho_max ||h|| inside it; rho is the largest row norm for a positive value, the smallest
// for a negative one.
__device__ __forceinline__ float bound_value(const StepArgs& a, int c, float dot, float Rc, float bm, float hn) {
    if (a.ang) {
        const float4 g = a.ang[c];
        const float perp = sqrtf(fmaxf(hn * hn - dot * dot, 0.f));
        const float v = dot * g.x + perp * g.y;
        const float val = dot >= hn * g.x ? g.z * hn : (v >= 0.f ? g.z * v : g.w * v);
        return val + bm;
    }
    if (!a.bt) return dot + Rc * hn + bm;
    const float2* t = a.bt + (size_t)c * a.bt_m;
    float best = -INFINITY;
    for (int j = 0; j < a.bt_m; ++j) {
        const float2 e = t[j];
        best = fmaxf(best, fmaf(e.x, hn, e.y));
    }
    return dot + best;
}

#define BOUND_PF 8
// A "unit" is one 128-bit load of a centroid row: four float32 values, or eight bfloat16 values when the index
// stores its centroids rounded (MU16).  The matching piece of h is 8 resp. 16 bytes of bf16.
template <bool MU16>
__device__ __forceinline__ const uint4* mu_row(const StepArgs& a, int c) {
    return MU16 ? reinterpret_cast<const uint4*>(a.mu16 + (size_t)c * a.d) : reinterpret_cast<const uint4*>(a.mu + (size_t)c * a.d);
}
template <bool MU16>
__device__ __forceinline__ int mu_units(int d) { return MU16 ? d >> 3 : d >> 2; }
// acc += <unit of mu, matching piece of h>;  hrow: the sequence's h as 32-bit words (two bf16 each)
template <bool MU16, class HP>
__device__ __forceinline__ float mu_fma(const uint4& m, HP hrow, int unit, float acc) {
    if constexpr (MU16) {
        const uint4 hv = reinterpret_cast<const uint4*>(hrow)[unit];
        return dot8_bf16(m, hv, acc);
    } else {
        const uint2 hv = reinterpret_cast<const uint2*>(hrow)[unit];
        acc = fmaf(__uint_as_float(m.x), bf16_lo(hv.x), acc);
        acc = fmaf(__uint_as_float(m.y), bf16_hi(hv.x), acc);
        acc = fmaf(__uint_as_float(m.z), bf16_lo(hv.y), acc);
        acc = fmaf(__uint_as_float(m.w), bf16_hi(hv.y), acc);
        return acc;
    }
}
#define BOUND_THREADS 512
#define BOUND_LDS_MAX (128 * 1024)   // most LDS for the h of four sequences
#define BOUND_HREG 8       // 128-bit pieces of h per thread: 8 x 512 x 16 B covers the 64 KB that BT sequences may take in LDS
// Three or four sequences, bf16 centroids: h of the sequences is staged in LDS once, then every wave walks over whole clusters
// (cluster = wave index among all waves of the grid, then + their number, ...): a centroid row goes through the wave
// in chunks of BOUND_PFB 128-bit loads per lane, the next chunk (of this or of the wave's next cluster) always
// requested before the current one is used, and nothing in the loop waits for another wave.  With more clusters
// than resident waves the staging of h is paid once per block, not once per cluster.
#ifndef BOUND_PFB
#define BOUND_PFB 16      // 128-bit loads per lane and chunk of a centroid row (two chunks in flight)
#endif
__global__ __launch_bounds__(BOUND_THREADS) void bound_kernel(StepArgs a, float* __restrict__ U_out, float* __restrict__ hn_out, int reset_counters) {
    constexpr int BT = 4;
    constexpr bool MU16 = true;
    extern __shared__ uint4 hs4[];
    __shared__ float hn[BT];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nb = min(BT, a.B);
    const int nch = a.d >> 3, nq = mu_units<MU16>(a.d), C = a.C;
    const int GW = gridDim.x * (BOUND_THREADS / 64);
    const int nchk = (nq + 64 * BOUND_PFB - 1) / (64 * BOUND_PFB);
    int c = blockIdx.x * (BOUND_THREADS / 64) + wave, chunk = 0;
    uint4 pfA[BOUND_PFB], pfB[BOUND_PFB];
    auto issue = [&](uint4 (&buf)[BOUND_PFB], int cc, int ch) {      // unconditional loads from clamped addresses, then a select
        const uint4* mrow = mu_row<MU16>(a, min(cc, C - 1));
#pragma unroll
        for (int j = 0; j < BOUND_PFB; ++j) {
            const int i = ch * 64 * BOUND_PFB + lane + 64 * j;
            const uint4 v = mrow[min(i, nq - 1)];
            buf[j] = (cc < C && i < nq) ? v : make_uint4(0, 0, 0, 0);
        }
    };
    issue(pfA, c, 0);                 // in flight while h is staged
    const uint4* hsrc = reinterpret_cast<const uint4*>(a.h);
    for (int base = 0; base < BT * nch; base += BOUND_HREG * BOUND_THREADS) {
        uint4 hreg[BOUND_HREG];
#pragma unroll
        for (int q = 0; q < BOUND_HREG; ++q) {
            const int i = base + tid + q * BOUND_THREADS;
            const uint4 v = hsrc[min(i, nb * nch - 1)];
            hreg[q] = i < nb * nch ? v : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int q = 0; q < BOUND_HREG; ++q) {
            const int i = base + tid + q * BOUND_THREADS;
            if (i < BT * nch) hs4[i] = hreg[q];
        }
    }
    if (reset_counters && blockIdx.x == 0)
        reset_step_counters(a.counters, a.B, BOUND_THREADS, a.host_history, a.slots, a.B_max);
    __syncthreads();
    for (int s = wave; s < BT; s += BOUND_THREADS / 64) {
        float acc = 0.f;
        for (int i = lane; i < nch; i += 64) {
            uint4 v = hs4[s * nch + i];
            acc = dot8_bf16(v, v, acc);
        }
        acc = wave_sum(acc);
        if (lane == 0) hn[s] = sqrtf(acc);
    }
    __syncthreads();
    if (blockIdx.x == 0 && tid < nb && hn_out) hn_out[tid] = hn[tid];

    float acc[BT];
#pragma unroll
    for (int s = 0; s < BT; ++s) acc[s] = 0.f;
    // one trip: request the chunk after (c, chunk) into `nxt`, use `cur`, finish the cluster when that was its last chunk
    auto trip = [&](uint4 (&cur)[BOUND_PFB], uint4 (&nxt)[BOUND_PFB]) {
        const bool last = chunk + 1 == nchk;
        const int c2 = last ? c + GW : c, ch2 = last ? 0 : chunk + 1;
        float Rc = 0.f, bm = 0.f;
        int ncl = 0;
        if (last) {                    // every lane the same address; needed only after the reduction below
            Rc = a.R[c];
            bm = a.bmax[c];
            ncl = a.n[c];
        }
        if (c2 < C) issue(nxt, c2, ch2);
#pragma unroll
        for (int j = 0; j < BOUND_PFB; ++j) {
            const int i = min(chunk * 64 * BOUND_PFB + lane + 64 * j, nq - 1);     // units past the row are zero
#pragma unroll
            for (int s = 0; s < BT; ++s) acc[s] = mu_fma<MU16>(cur[j], hs4 + s * nch, i, acc[s]);
        }
        if (last) {
#pragma unroll
            for (int s = 0; s < BT; ++s) {
                const float t = wave_sum(acc[s]);
                if (lane == 0 && s < nb) U_out[(size_t)s * C + c] = ncl == 0 ? -INFINITY : bound_value(a, c, t, Rc, bm, hn[s]);
                acc[s] = 0.f;
            }
        }
        c = c2;
        chunk = ch2;
    };
    while (c < C) {
        trip(pfA, pfB);
        if (c >= C) break;
        trip(pfB, pfA);
    }
}

// BT sequences (1..4).  Block = 8 waves = 8/WPC clusters x WPC column slices (WPC = 1, 2 or 4, chosen so that a wave's slice of the centroid row is one batch of
// loads per lane, where four slices are enough).  Blocks are dealt round-robin to the 8 XCDs, so group g = (block % 8) * groups_per_xcd + block / 8 keeps
// every XCD on the same centroid slice step after step.  No LDS staging at all:  h is 2d bytes a sequence that every wave of the device reads, so it comes from
// L2 / L1 with the same addresses in every block; each wave takes its slice of h straight from global memory next to
// its centroid slice, and ||h||^2 is the sum of the slices' partial sums of squares (slice order: the same value
// in every block).
// Units of a centroid row a lane has requested at once: with more than two sequences four, which leaves registers for four sequences' pieces of h for them and for
// five waves per SIMD (us with four / eight: B = 3, C = 4096, d = 4608 15.5 / 20.9; B = 4, C = 2048, d = 5120 11.6 / 14.0, C = 1024, d = 4096 6.0 / 6.3).
// Walking over whole clusters with h in LDS took B = 2..4 at C = 1024, d = 4096 6.1 / 7.0 / 7.1 us, this 5.1 / 5.4 / 6.0, at C = 601, d = 2056 (3) 6.9, now 5.1.
#define BOUND_ROWS_PF(BT) ((BT) > 2 ? 4 : BOUND_PF)
template <int BT, bool MU16>
__global__ __launch_bounds__(BOUND_THREADS) void bound_rows_kernel(StepArgs a, float* __restrict__ U_out, float* __restrict__ hn_out,
                                                                   int reset_counters, int groups, int groups_per_xcd, int wpc) {
    constexpr int PF = BOUND_ROWS_PF(BT);
    __shared__ float part[BT][BOUND_THREADS / 64], parth[BT][BOUND_THREADS / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nq = mu_units<MU16>(a.d);
    const int cpb = (BOUND_THREADS / 64) / wpc, cl = wave / wpc, slice = wave - cl * wpc;
    const int g = (blockIdx.x & 7) * groups_per_xcd + (blockIdx.x >> 3);
    const int c = g * cpb + cl;
    const bool valid = g < groups && c < a.C;
    const int seg = (nq + wpc - 1) / wpc, lo = slice * seg, hi = min(nq, lo + seg);
    const uint4* mrow = mu_row<MU16>(a, valid ? c : 0);
    typedef typename std::conditional<MU16, uint4, uint2>::type hpiece;   // the piece of h that goes with one unit
    const hpiece* hp = reinterpret_cast<const hpiece*>(a.h);
    uint4 pf[PF];
    hpiece ph[BT][PF];
#pragma unroll
    for (int j = 0; j < PF; ++j) {
        const int i = lo + lane + 64 * j;
        pf[j] = (valid && i < hi) ? mrow[i] : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int s = 0; s < BT; ++s)
#pragma unroll
        for (int j = 0; j < PF; ++j) {
            const int i = lo + lane + 64 * j;
            ph[s][j] = i < hi ? hp[(size_t)s * nq + i] : hpiece{};
        }
    float Rc = 0.f, bm = 0.f;
    int ncl = 0;
    if (valid && slice == 0 && lane < BT) {
        Rc = a.R[c];
        bm = a.bmax[c];
        ncl = a.n[c];
    }
    if (reset_counters && blockIdx.x == 0)
        reset_step_counters(a.counters, a.B, BOUND_THREADS, a.host_history, a.slots, a.B_max);
    float acc[BT], hh[BT];
#pragma unroll
    for (int s = 0; s < BT; ++s) acc[s] = hh[s] = 0.f;
    auto step = [&](int s, const uint4& m, const hpiece& hv) {
        acc[s] = mu_fma<MU16>(m, &hv, 0, acc[s]);
        const uint32_t* w = reinterpret_cast<const uint32_t*>(&hv);
#pragma unroll
        for (int e = 0; e < (int)(sizeof(hpiece) / 4); ++e) {
            hh[s] = fmaf(bf16_lo(w[e]), bf16_lo(w[e]), hh[s]);
            hh[s] = fmaf(bf16_hi(w[e]), bf16_hi(w[e]), hh[s]);
        }
    };
#pragma unroll
    for (int j = 0; j < PF; ++j)
#pragma unroll
        for (int s = 0; s < BT; ++s) step(s, pf[j], ph[s][j]);
#pragma unroll 4
    for (int i = lo + lane + 64 * PF; i < hi; i += 64) {
        const uint4 m = valid ? mrow[i] : make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int s = 0; s < BT; ++s) step(s, m, hp[(size_t)s * nq + i]);
    }
#pragma unroll
    for (int s = 0; s < BT; ++s) {
        acc[s] = wave_sum(acc[s]);
        hh[s] = wave_sum(hh[s]);
        if (lane == 0) {
            part[s][wave] = acc[s];
            parth[s][wave] = hh[s];
        }
    }
    __syncthreads();
    if (slice == 0 && lane < BT) {                           // lane s finishes sequence s
        float t = part[lane][wave], th = parth[lane][wave];
        for (int q = 1; q < wpc; ++q) {
            t += part[lane][wave + q];
            th += parth[lane][wave + q];
        }
        const float hn = sqrtf(th);
        if (blockIdx.x == 0 && wave == 0 && hn_out) hn_out[lane] = hn;
        if (valid) U_out[(size_t)lane * a.C + c] = ncl == 0 ? -INFINITY : bound_value(a, c, t, Rc, bm, hn);
    }
}

// Bounds for larger batches (B >= BOUND_MFMA_MIN_B): [C x d] fp32 centroids times [d x B] bf16 hidden states is a dense contraction,
// done with v_mfma_f32_16x16x32_bf16.  A float32 centroid value is split exactly into three bf16 pieces
// (x = hi + mid + lo, 8 mantissa bits each), so three MFMAs per k-block give the float32-exact products with float32
// accumulation; the split costs a handful of vector instructions per value, independent of B.
// A wave owns 16 clusters and one slice of K; lane (li, g) feeds cluster/sequence li with the eight k values
// 32 kb + 8 g.  Partial sums of the K slices go to P[slice][sequence][cluster]; bound_finish_kernel adds them in a
// fixed order together with R_c ||h|| + bmax_c, so the result does not depend on scheduling.
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4_t;

__device__ __forceinline__ void split3_bf16(const float4& x0, const float4& x1, uint4& hi, uint4& mid, uint4& lo) {
    const float v[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
    uint32_t h[8], m[8], l[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        h[i] = __float_as_uint(v[i]) & 0xffff0000u;
        const float r1 = v[i] - __uint_as_float(h[i]);
        m[i] = __float_as_uint(r1) & 0xffff0000u;
        const float r2 = r1 - __uint_as_float(m[i]);
        l[i] = __float_as_uint(r2) & 0xffff0000u;
    }
    hi = make_uint4((h[0] >> 16) | h[1], (h[2] >> 16) | h[3], (h[4] >> 16) | h[5], (h[6] >> 16) | h[7]);
    mid = make_uint4((m[0] >> 16) | m[1], (m[2] >> 16) | m[3], (m[4] >> 16) | m[5], (m[6] >> 16) | m[7]);
    lo = make_uint4((l[0] >> 16) | l[1], (l[2] >> 16) | l[3], (l[4] >> 16) | l[5], (l[6] >> 16) | l[7]);
}

#define BOUND_TILES_PER_BLOCK 8   // waves of a block: each owns 16 clusters, all share the block's K slice (and its h in LDS)
#define BOUND_MFMA_MIN_B 5       // from this many sequences on the matrix cores: a lane of the vector kernels reads h of every sequence for each piece of a
                                 // centroid (eight sequences: 128 bytes for 16, 23 us against 15 at C = 2048, d = 5120)
#ifndef BOUND_BLOCK_TARGET
#define BOUND_BLOCK_TARGET 256   // (groups of cluster tiles x K slices) aimed at: one block per compute unit (64..2048 swept)
#endif
#define BOUND_KS_MAX 32
#ifndef BOUND_PIPE
#define BOUND_PIPE 4             // k-blocks (of 32) a wave has requested ahead: 8 KB of float32 centroids
#endif
#define BOUND_LDS_KB 48          // most LDS for the h of one K slice (1 KB per k-block and 16 sequences)
#define BOUND_LDS_KB_MANY 64     // with more than 64 sequences
__device__ __forceinline__ uint4 keep_if(bool c, const uint4& v) {     // v or zero, component by component (no select between objects in memory)
    return make_uint4(c ? v.x : 0u, c ? v.y : 0u, c ? v.z : 0u, c ? v.w : 0u);
}
__device__ __forceinline__ void lds_barrier() {      // all LDS accesses of the block's waves are done; global loads stay in flight
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Grid (groups of 8 cluster tiles, K slices, 64 sequences each: 256 sequences at C = 1024, d = 4096 take 4 x 8 us as launches of
// their own).  The block's slice of h goes to LDS once, in fragment order (1 KB per
// k-block and sequence tile, read without bank conflicts), zero where the sequence, the k-block or k itself lies
// outside: centroid values can then be read from clamped addresses without a select, which would be waited for right
// behind the load.  Every wave has BOUND_PIPE k-blocks of its 16 centroid rows requested ahead; a register buffer is
// requested again as soon as its values are split.  The last chunk is a copy of the loop body without requests, so
// that the waits the compiler places are counted at compile time.
template <int NT, bool MU16, bool MANY = false>
__global__ __launch_bounds__(512) void bound_mfma_kernel(StepArgs a, float* __restrict__ P, int kb_per_slice,
                                                         int reset_counters) {
    extern __shared__ uint4 bound_lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int li = lane & 15, g = lane >> 4;
    if (reset_counters && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0)
        reset_step_counters(a.counters, a.B, 512, a.host_history, a.slots, a.B_max);
    const int ks = blockIdx.y, seq0 = blockIdx.z * 64;
    const int nkb = (a.d + 31) >> 5;
    const int kb0 = ks * kb_per_slice, kb1 = min(nkb, kb0 + kb_per_slice);      // the host gives every slice at least one k-block
    const int nchunk = (kb1 - kb0 + BOUND_PIPE - 1) / BOUND_PIPE;
    const int c0 = (blockIdx.x * BOUND_TILES_PER_BLOCK + wave) * 16;            // past C: the wave computes a copy of the last rows and stores nothing
    const size_t crow = (size_t)min(c0 + li, a.C - 1) * a.d;
    const uint4* ap = MU16 ? reinterpret_cast<const uint4*>(a.mu16 + crow) : reinterpret_cast<const uint4*>(a.mu + crow);
    uint4 X[BOUND_PIPE][MU16 ? 1 : 2];
    auto load_x = [&](int u, int kb) {          // the lane's eight values of k-block kb, or (k past d) eight finite values that meet zeros
        const int k = min(kb * 32 + g * 8, a.d - 8);
        if constexpr (MU16) {
            X[u][0] = ap[k >> 3];
        } else {
            X[u][0] = ap[k >> 2];
            X[u][1] = ap[(k >> 2) + 1];
        }
    };
    // h first (older loads are waited for first), then the centroid requests, which stay in flight across the staging
    constexpr int HS = ((MANY ? BOUND_LDS_KB_MANY : BOUND_LDS_KB) * 64 + 511) / 512;           // staged 128-bit pieces per thread at most
    const int items = nchunk * BOUND_PIPE * NT * 64;
    const uint4* hsrc = reinterpret_cast<const uint4*>(a.h);
    uint4 hreg[HS];
    bool hok[HS];
#pragma unroll
    for (int q = 0; q < HS; ++q) {
        const int it = tid + q * 512;
        const int ln = it & 63, t = (it >> 6) % NT, kbl = (it >> 6) / NT;
        const int sq = seq0 + t * 16 + (ln & 15), kb = kb0 + kbl, k = kb * 32 + (ln >> 4) * 8;
        hok[q] = it < items && sq < a.B && kb < kb1 && k < a.d;
        hreg[q] = make_uint4(0, 0, 0, 0);
        if (it < items) hreg[q] = hsrc[(size_t)(hok[q] ? sq : 0) * (a.d >> 3) + (hok[q] ? k >> 3 : 0)];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < BOUND_PIPE; ++u) load_x(u, kb0 + u);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < HS; ++q) {
        const int it = tid + q * 512;
        if (it < items) bound_lds[it] = keep_if(hok[q], hreg[q]);
    }
    lds_barrier();
    floatx4_t acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    auto chunk = [&](auto more_t, int c) {
        constexpr bool more = decltype(more_t)::value;
#pragma unroll
        for (int u = 0; u < BOUND_PIPE; ++u) {
            const uint4* hb = bound_lds + ((c * BOUND_PIPE + u) * NT << 6) + lane;
            if constexpr (MU16) {       // bf16 centroids feed the MFMA as they are
                const bf16x8_t xv = __builtin_bit_cast(bf16x8_t, X[u][0]);
                __builtin_amdgcn_sched_barrier(0);
                if (more) load_x(u, kb0 + (c + 1) * BOUND_PIPE + u);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, hb[t << 6]), xv, acc[t], 0, 0, 0);
            } else {
                uint4 hi, mid, lo;
                split3_bf16(__builtin_bit_cast(float4, X[u][0]), __builtin_bit_cast(float4, X[u][1]), hi, mid, lo);
                __builtin_amdgcn_sched_barrier(0);
                if (more) load_x(u, kb0 + (c + 1) * BOUND_PIPE + u);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const bf16x8_t bv = __builtin_bit_cast(bf16x8_t, hb[t << 6]);
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bv, __builtin_bit_cast(bf16x8_t, hi), acc[t], 0, 0, 0);
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bv, __builtin_bit_cast(bf16x8_t, mid), acc[t], 0, 0, 0);
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bv, __builtin_bit_cast(bf16x8_t, lo), acc[t], 0, 0, 0);
                }
            }
        }
    };
    for (int c = 0; c + 1 < nchunk; ++c) chunk(std::true_type{}, c);
    chunk(std::false_type{}, nchunk - 1);
    // h is the first operand: accumulator register r of lane (li, g) is  [sequence 4g + r][cluster li], so the 16
    // lanes of a group store 64 contiguous bytes of one sequence's partial bounds
    const int c = c0 + li;
    if (c < a.C) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int sq = seq0 + t * 16 + 4 * g + r;
                if (sq < a.B) P[((size_t)ks * a.B + sq) * a.C + c] = acc[t][r];
            }
    }
}

// Up to 16 sequences in one launch: block = 16 clusters and the whole of K, so that nothing has to meet outside the block.  K goes by in chunks of 32 k-blocks,
// two to each of the 16 waves; h of a chunk lies in LDS in fragment order (places turned by the k group, so that rows can be read from memory in runs of
// 1 KB and written without bank conflicts), the next chunk's is requested a chunk ahead and stored to the other half; every wave has the centroid values of its next two
// k-blocks requested.  The waves' sums are added in wave order.
// Bound by latency, for long rows and many clusters by reading the centroids: C = 4096, d = 5120 in bf16 10.7 us = 3.9 TB/s.  (With chunks of 64 k-blocks, twice the
// time until the first products, 12.7; with h read from L2 by every wave 13.7-15.5.)
#define BOUND_TILE_KB 32
#define BOUND_TILE_LDS (2 * BOUND_TILE_KB * 1024)
template <bool MU16>
__global__ __launch_bounds__(1024) void bound_tile_kernel(StepArgs a, float* __restrict__ U_out, float* __restrict__ hn_out, int reset_counters) {
    extern __shared__ uint4 bound_lds[];
    constexpr int PER = BOUND_TILE_KB / 16;                  // k-blocks of a chunk per wave = pieces of h a lane stages
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, g = lane >> 4, nch = a.d >> 3, nchunk = (a.d + 32 * BOUND_TILE_KB - 1) / (32 * BOUND_TILE_KB), c0 = blockIdx.x * 16;
    const size_t crow = (size_t)min(c0 + li, a.C - 1) * a.d;
    const uint4* ap = MU16 ? reinterpret_cast<const uint4*>(a.mu16 + crow) : reinterpret_cast<const uint4*>(a.mu + crow);
    const uint4* hp = reinterpret_cast<const uint4*>(a.h) + (size_t)min(wave, a.B - 1) * nch;      // the wave stages one sequence (past B: one whose sums nobody takes)
    uint4 X[PER][MU16 ? 1 : 2], H[PER];
    auto request_h = [&](int ch) {
#pragma unroll
        for (int q = 0; q < PER; ++q) H[q] = hp[min(ch * 4 * BOUND_TILE_KB + lane + 64 * q, nch - 1)];
    };
    auto store_h = [&](int ch) {                             // zeros past d: they meet the centroid row's last values
        uint4* o = bound_lds + (ch & 1) * BOUND_TILE_KB * 64;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int p = lane + 64 * q;
            o[p * 16 + ((wave + p) & 15)] = keep_if(ch * 4 * BOUND_TILE_KB + p < nch, H[q]);
        }
    };
    auto request_x = [&](int u, int ch) {                    // the wave's k-blocks lie side by side
        const int q = min((ch * BOUND_TILE_KB + wave * PER + u) * 4 + g, nch - 1);
        if constexpr (MU16) {
            X[u][0] = ap[q];
        } else {
            X[u][0] = ap[2 * q];
            X[u][1] = ap[2 * q + 1];
        }
    };
    request_h(0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < PER; ++u) request_x(u, 0);
    __builtin_amdgcn_sched_barrier(0);
    if (reset_counters && blockIdx.x == 0) reset_step_counters(a.counters, a.B, 1024, a.host_history, a.slots, a.B_max);
    store_h(0);
    __builtin_amdgcn_sched_barrier(0);
    request_h(1);
    lds_barrier();
    floatx4_t acc = {0.f, 0.f, 0.f, 0.f};
    float ss = 0.f;
    for (int ch = 0; ch < nchunk; ++ch) {
        const uint4* hb = bound_lds + (ch & 1) * BOUND_TILE_KB * 64;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int p = (wave * PER + u) * 4 + g;
            const uint4 hv = hb[p * 16 + ((li + p) & 15)];
            ss = dot8_bf16(hv, hv, ss);
            const bf16x8_t bv = __builtin_bit_cast(bf16x8_t, hv);
            if constexpr (MU16) {
                const bf16x8_t xv = __builtin_bit_cast(bf16x8_t, X[u][0]);
                __builtin_amdgcn_sched_barrier(0);
                request_x(u, ch + 1);
                __builtin_amdgcn_sched_barrier(0);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bv, xv, acc, 0, 0, 0);
            } else {
                uint4 hi, mid, lo;
                split3_bf16(__builtin_bit_cast(float4, X[u][0]), __builtin_bit_cast(float4, X[u][1]), hi, mid, lo);
                __builtin_amdgcn_sched_barrier(0);
                request_x(u, ch + 1);
                __builtin_amdgcn_sched_barrier(0);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bv, __builtin_bit_cast(bf16x8_t, hi), acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bv, __builtin_bit_cast(bf16x8_t, mid), acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bv, __builtin_bit_cast(bf16x8_t, lo), acc, 0, 0, 0);
            }
        }
        if (ch + 1 < nchunk) {
            store_h(ch + 1);                                 // to the half that was read a chunk ago: every wave has passed its barrier
            __builtin_amdgcn_sched_barrier(0);
            request_h(ch + 2);
        }
        lds_barrier();
    }
    // accumulator register r of lane (li, g) is [sequence 4g + r][cluster li]; the squares of sequence li are in its four lanes
    float* red = reinterpret_cast<float*>(bound_lds);        // [wave][sequence][cluster], then [wave][sequence]
    float* redh = red + 16 * 256;
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave * 256 + (4 * g + r) * 16 + li] = acc[r];
    ss += __shfl_xor(ss, 16, CSV_WAVE);
    ss += __shfl_xor(ss, 32, CSV_WAVE);
    if (g == 0) redh[wave * 16 + li] = ss;
    __syncthreads();
    const int sq = tid >> 4, c = c0 + (tid & 15);
    if (sq >= a.B || sq >= 16) return;
    float u = 0.f, th = 0.f;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
        u += red[w * 256 + tid];
        th += redh[w * 16 + sq];
    }
    const float hn = sqrtf(th);
    if (c0 == 0 && (tid & 15) == 0 && hn_out) hn_out[sq] = hn;
    if (c < a.C) U_out[(size_t)sq * a.C + c] = a.n[c] == 0 ? -INFINITY : bound_value(a, c, u, a.R[c], a.bmax[c], hn);
}

// Block (x, b): ||h_b|| (every block of the sequence recomputes it: d values), then for 256 clusters
// U[b,c] = sum of the K-slice partials (ascending slice) + R_c ||h_b|| + bmax_c.
__global__ __launch_bounds__(256) void bound_finish_kernel(StepArgs a, const float* __restrict__ P, int KS,
                                                           float* __restrict__ U_out, float* __restrict__ hn_out) {
    __shared__ float red[16];
    const int b = blockIdx.y, tid = threadIdx.x;
    const int c = blockIdx.x * 256 + tid;
    const bool in = c < a.C;
    float part[BOUND_KS_MAX];
#pragma unroll
    for (int ks = 0; ks < BOUND_KS_MAX; ++ks) part[ks] = (in && ks < KS) ? P[((size_t)ks * a.B + b) * a.C + c] : 0.f;
    const float Rc = in ? a.R[c] : 0.f, bm = in ? a.bmax[c] : 0.f;
    const int nc = in ? a.n[c] : 0;
    const uint4* hsrc = reinterpret_cast<const uint4*>(a.h) + (size_t)b * (a.d >> 3);
    float ss = 0.f;
    for (int i = tid; i < (a.d >> 3); i += 256) {
        const uint4 v = hsrc[i];
        ss = dot8_bf16(v, v, ss);
    }
    const float hn = sqrtf(block_sum(ss, red));
    if (blockIdx.x == 0 && tid == 0 && hn_out) hn_out[b] = hn;
    if (!in) return;
    float u = 0.f;
#pragma unroll
    for (int ks = 0; ks < BOUND_KS_MAX; ++ks) u += part[ks];
    U_out[(size_t)b * a.C + c] = nc == 0 ? -INFINITY : bound_value(a, c, u, Rc, bm, hn);
}

// ================================================================================================ block scans
// Combination of everything owned by the threads AFTER this one (exclusive suffix), for log-sum-exp partials.
__device__ __forceinline__ LseAcc block_excl_suffix_lse(LseAcc v, LseAcc* wtot) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    LseAcc x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        LseAcc y;
        y.m = __shfl_down(x.m, o, CSV_WAVE);
        y.s = __shfl_down(x.s, o, CSV_WAVE);
        if (lane + o < 64) x = lse_combine(x, y);
    }
    LseAcc after;
    after.m = __shfl_down(x.m, 1, CSV_WAVE);
    after.s = __shfl_down(x.s, 1, CSV_WAVE);
    if (lane == 63) {
        after.m = -INFINITY;
        after.s = 0.f;
    }
    __syncthreads();
    if (lane == 0) wtot[w] = x;
    __syncthreads();
    LseAcc tail;
    tail.m = -INFINITY;
    tail.s = 0.f;
    for (int i = nw - 1; i > w; --i) tail = lse_combine(wtot[i], tail);
    return lse_combine(after, tail);
}

// ================================================================================================ shared LDS of the per-sequence kernels
struct BigItem {
    int row0, n, pos, tbase;
};
#define CAND_CAP SEQ_THREADS
#define RANK_DIRECT 256      // up to this many values are ranked against each other directly (a multiple of four, at most SEQ_THREADS)
struct SeqShared {
    unsigned hist[256];
    float redf[16];
    int redi[16];
    int scan3[48];
    int rank[SEQ_THREADS];
    u64 redu[32];
    LseAcc redl[16];
    unsigned sel, rem, eq, cnt;
    int tbase, nbig;
    BigItem big[BIGQ];
    float wval[CSV_MAX_K];
    int wid[CSV_MAX_K];
};
// Later rounds collect the values at or above the previous round's k-th logit, and their ids, behind the staged
// logits in the dynamic LDS (a region the cluster data of a large index covers anyway).
#define CAND_OFF (STAGE_CAP * 8)
#define CAND_BYTES ((CAND_CAP + 4) * 4 + CAND_CAP * 4)

// ================================================================================================ helpers shared by seed/cert
__device__ __forceinline__ void write_invalid(const StepArgs& a, int b) {
    for (int t = threadIdx.x; t < a.k; t += blockDim.x) {
        a.out.d_ids[(size_t)b * a.k + t] = -1;
        a.out.d_logits[(size_t)b * a.k + t] = NAN;
        if (a.out.d_probs) a.out.d_probs[(size_t)b * a.k + t] = NAN;
        if (a.out.d_cum) a.out.d_cum[(size_t)b * a.k + t] = NAN;
    }
    if (threadIdx.x == 0 && a.out.d_nucleus) a.out.d_nucleus[b] = 0;
    if (threadIdx.x == 0) {
        a.out.d_lse[b] = NAN;
        a.out.d_flags[b] = CSV_FLAG_INVALID_INPUT;
        a.out.d_n_rows[b] = 0;
        a.out.d_n_clusters[b] = 0;
        if (a.out.d_rounds) a.out.d_rounds[b] = 0;
        a.st[b].status = ST_INVALID;
    }
}

// Called by one thread: hand sequence b to the full-vocabulary path.
__device__ __forceinline__ void push_fallback(const StepArgs& a, int b, int rounds) {
    const int slot = atomicAdd(&a.counters[CNT_FALLBACK], 1);
    __hip_atomic_store(&a.counters[CNT_TAIL_NEEDED], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    a.fb_list[slot] = b;
    a.st[b].status = ST_FALLBACK;
    a.st[b].fb_slot = slot;
    if (a.out.d_rounds) a.out.d_rounds[b] = rounds;
}

// Per-sequence cluster data in LDS: keys[Npad], first permuted row of each cluster offl[C+1], and
// vl[c] = ln n_c + U_c (the cluster's term of the log tail mass; -inf for an empty cluster).
struct ClusterLds {
    u64* keys;
    int* offl;
    float* vl;
};
__device__ __forceinline__ ClusterLds carve_clusters(u64* arena, int Npad, int C) {
    ClusterLds L;
    L.keys = arena;
    L.offl = reinterpret_cast<int*>(arena + Npad);
    L.vl = reinterpret_cast<float*>(L.offl + C + 1);
    return L;
}
__device__ __forceinline__ void load_clusters(const StepArgs& a, int b, const ClusterLds& L) {
    const int tid = threadIdx.x, nt = blockDim.x;
    // four clusters per thread and trip, all sixteen loads issued before the first use (n_c = off[c+1] - off[c])
    for (int c0 = 0; c0 < a.C; c0 += 4 * nt) {
        float u[4], ln[4];
        int o0[4], o1[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int c = c0 + q * nt + tid;
            const bool in = c < a.C;
            u[q] = in ? a.U[(size_t)b * a.C + c] : 0.f;
            ln[q] = in ? a.lnn[c] : 0.f;
            o0[q] = in ? a.off[c] : 0;
            o1[q] = in ? a.off[c + 1] : 0;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int c = c0 + q * nt + tid;
            if (c < a.C) {
                const bool some = o1[q] > o0[q];
                L.offl[c] = o0[q];
                if (c == a.C - 1) L.offl[a.C] = o1[q];
                L.keys[c] = some ? ckey(u[q], c) : 0ull;
                L.vl[c] = some ? ln[q] + u[q] : -INFINITY;
            }
        }
    }
}

// fn(c, key, rows, term) for the thread's clusters, four at a time: all LDS reads of a trip are issued, from clamped indexes, before the
// first is looked at (a read behind a test of another would add its latency to every cluster).  Past the end: key 0.
template <bool ROWS, bool TERMS, class Fn>
__device__ __forceinline__ void for_clusters(int C, const ClusterLds& L, Fn fn) {
    const int nt = blockDim.x;
    for (int c0 = threadIdx.x; c0 < C; c0 += 4 * nt) {
        u64 k[4];
        int o0[4], o1[4];
        float v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int cc = min(c0 + q * nt, C - 1);
            k[q] = L.keys[cc];
            if (ROWS) {
                o0[q] = L.offl[cc];
                o1[q] = L.offl[cc + 1];
            }
            if (TERMS) v[q] = L.vl[cc];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) fn(c0 + q * nt, c0 + q * nt < C ? k[q] : 0ull, ROWS ? o1[q] - o0[q] : 0, TERMS ? v[q] : 0.f);
    }
}

// Exclusive prefix sums of three ints per thread in one pass.  wtot: 48 ints of LDS.
__device__ __forceinline__ void block_excl_scan3(int& v0, int& v1, int& v2, int* wtot, int& t0, int& t1, int& t2) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    int x0 = v0, x1 = v1, x2 = v2;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y0 = __shfl_up(x0, o, CSV_WAVE), y1 = __shfl_up(x1, o, CSV_WAVE), y2 = __shfl_up(x2, o, CSV_WAVE);
        if (lane >= o) {
            x0 += y0;
            x1 += y1;
            x2 += y2;
        }
    }
    __syncthreads();
    if (lane == 63) {
        wtot[w] = x0;
        wtot[16 + w] = x1;
        wtot[32 + w] = x2;
    }
    __syncthreads();
    int b0 = 0, b1 = 0, b2 = 0;
    t0 = t1 = t2 = 0;
    for (int i = 0; i < nw; ++i) {
        const int a0 = wtot[i], a1 = wtot[16 + i], a2 = wtot[32 + i];
        if (i < w) {
            b0 += a0;
            b1 += a1;
            b2 += a2;
        }
        t0 += a0;
        t1 += a1;
        t2 += a2;
    }
    v0 = b0 + x0 - v0;
    v1 = b1 + x1 - v1;
    v2 = b2 + x2 - v2;
}

// Opens every cluster c with flag(c): its rows get consecutive positions from pos_base on (cluster id order), its
// row tiles go to the sequence's region of the round's work list (two lists, used by even and odd rounds), its id is appended to the sequence's list of
// opened clusters.  All threads of the block call; flag must be the same function of c in both passes.
template <class FlagFn>
__device__ __forceinline__ void emit_clusters(const StepArgs& a, int b, int round, int pos_base, int sel_base, FlagFn flag,
                                              const ClusterLds& L, SeqShared& s) {
    const int tid = threadIdx.x, nt = blockDim.x, C = a.C;
    const int E = (C + nt - 1) / nt;
    const int c0 = min(C, tid * E), c1 = min(C, c0 + E);
    int cnt = 0, rows = 0, tiles = 0;
    for (int c = c0; c < c1; ++c)
        if (flag(c)) {
            const int n = L.offl[c + 1] - L.offl[c];
            cnt += 1;
            rows += n;
            tiles += (n + TILE_ROWS - 1) / TILE_ROWS;
        }
    int tot_cnt, tot_rows, tot_tiles;
    block_excl_scan3(cnt, rows, tiles, s.scan3, tot_cnt, tot_rows, tot_tiles);
    if (tid == 0) {
        a.counters[CNT_TILES + round * CSV_MAX_BATCH + b] = tot_tiles;
        __hip_atomic_store(&a.counters[CNT_TAIL_NEEDED], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s.nbig = 0;
    }
    __syncthreads();
    Tile* tl = a.tiles[round & 1] + (size_t)b * a.tile_stride;
    int tb = tiles, pos = pos_base + rows, si = sel_base + cnt;
    for (int c = c0; c < c1; ++c)
        if (flag(c)) {
            const int r0 = L.offl[c], n = L.offl[c + 1] - r0, ntc = (n + TILE_ROWS - 1) / TILE_ROWS;
            a.sel[(size_t)b * C + si++] = c;
            int slot = BIGQ;
            if (ntc > 16) slot = atomicAdd(&s.nbig, 1);
            if (slot < BIGQ) {
                BigItem it;
                it.row0 = r0; it.n = n; it.pos = pos; it.tbase = tb;
                s.big[slot] = it;
            } else {
                for (int t = 0; t < ntc; ++t) {
                    Tile x;
                    x.b = b; x.row0 = r0 + t * TILE_ROWS; x.nrows = min(TILE_ROWS, n - t * TILE_ROWS); x.pos = pos + t * TILE_ROWS;
                    tl[tb + t] = x;
                }
            }
            tb += ntc;
            pos += n;
        }
    __syncthreads();
    const int nbig = min(s.nbig, BIGQ);
    for (int q = 0; q < nbig; ++q) {
        const BigItem it = s.big[q];
        const int ntc = (it.n + TILE_ROWS - 1) / TILE_ROWS;
        for (int t = tid; t < ntc; t += nt) {
            Tile x;
            x.b = b; x.row0 = it.row0 + t * TILE_ROWS; x.nrows = min(TILE_ROWS, it.n - t * TILE_ROWS); x.pos = it.pos + t * TILE_ROWS;
            tl[it.tbase + t] = x;
        }
    }
    __syncthreads();
}

// The same for at most SEQ_THREADS opened clusters, cnt of them (the block has SEQ_THREADS
// threads): the opened ids go into a list in id order, a thread takes one of them for the prefix sums, and the
// tiles are then written one per thread, neighbouring threads side by side.  emit_clusters gives each thread a run of neighbouring
// clusters, whose LDS reads fall on few banks, and mostly one thread writes all the tiles of a cluster: 4.2-5.0 us
// against 3.2 at C = 2048 with clusters of very unequal sizes; at C = 4096 with 8 to 52 clusters of 62 rows 3.7-5.6 against 4.0.
// opens: a test of a cluster's key (false for 0).  Uses s.hist, s.rank, s.wval and s.wid (the
// caller's top-k list is dead by then); the caller passes a barrier before it uses them again.
// s.hist counts 256 groups of 64 clusters; a thread keeps its up to 32 answers in one word
static_assert(CSV_MAX_CLUSTERS <= 256 * 64 && CSV_MAX_CLUSTERS <= 32 * SEQ_THREADS, "emit_list: groups and answers");
template <class OpensFn>
__device__ __forceinline__ void emit_list(const StepArgs& a, int b, int round, int pos_base, int sel_base, int cnt, OpensFn opens,
                                          const ClusterLds& L, SeqShared& s) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, C = a.C;
    constexpr int NW = SEQ_THREADS / 64;
    __syncthreads();
    if (tid < 256) s.hist[tid] = 0u;
    __syncthreads();
    // trip i of a thread is cluster tid + SEQ_THREADS i, and the 64 clusters of a wave's trip are group wave + NW i
    unsigned mine = 0;
    int trip = 0;
    for_clusters<false, false>(C, L, [&](int, u64 kx, int, float) {
        mine |= (opens(kx) ? 1u : 0u) << trip;
        ++trip;
    });
    const int trips = (C + SEQ_THREADS - 1) / SEQ_THREADS;
    for (int i = 0; i < trips; ++i) {
        const unsigned long long bal = __ballot((mine >> i) & 1u);
        if (lane == 0) s.hist[wave + NW * i] = (unsigned)__popcll(bal);
    }
    __syncthreads();
    if (tid < 64) {                                                  // groups before each one, lane l: groups 4l..4l+3
        unsigned h[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) h[q] = s.hist[4 * lane + q];
        const unsigned sum = h[0] + h[1] + h[2] + h[3];
        unsigned x = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned y = __shfl_up(x, o, CSV_WAVE);
            if (lane >= o) x += y;
        }
        x -= sum;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            s.hist[4 * lane + q] = x;
            x += h[q];
        }
    }
    __syncthreads();
    for (int i = 0; i < trips; ++i) {
        const bool on = (mine >> i) & 1u;
        const unsigned long long bal = __ballot(on);
        if (on) s.rank[s.hist[wave + NW * i] + __popcll(bal & ((1ull << lane) - 1ull))] = tid + SEQ_THREADS * i;
    }
    __syncthreads();
    int one = 0, rows = 0, tiles = 0, c = 0, n = 0;
    if (tid < cnt) {
        c = s.rank[tid];
        n = L.offl[c + 1] - L.offl[c];
        rows = n;
        tiles = (n + TILE_ROWS - 1) / TILE_ROWS;
    }
    int tot_one, tot_rows, tot_tiles;
    block_excl_scan3(one, rows, tiles, s.scan3, tot_one, tot_rows, tot_tiles);
    int* pos = reinterpret_cast<int*>(s.wval);
    if (tid < cnt) {
        s.wid[tid] = tiles;
        pos[tid] = pos_base + rows;
    }
    __syncthreads();                       // no store to global memory before this: a barrier waits for those too
    if (tid < cnt) a.sel[(size_t)b * C + sel_base + tid] = c;
    if (tid == 0) {
        a.counters[CNT_TILES + round * CSV_MAX_BATCH + b] = tot_tiles;
        __hip_atomic_store(&a.counters[CNT_TAIL_NEEDED], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    Tile* tl = a.tiles[round & 1] + (size_t)b * a.tile_stride;
    for (int g = tid; g < tot_tiles; g += SEQ_THREADS) {
        int lo = 0, hi = cnt;               // the last cluster whose tiles start at or before g (every one has at least one)
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (s.wid[mid] <= g) lo = mid; else hi = mid;
        }
        const int t = g - s.wid[lo], cc = s.rank[lo], r0 = L.offl[cc], m = L.offl[cc + 1] - r0;
        Tile x;
        x.b = b; x.row0 = r0 + t * TILE_ROWS; x.nrows = min(TILE_ROWS, m - t * TILE_ROWS); x.pos = pos[lo] + t * TILE_ROWS;
        tl[g] = x;
    }
}

// Largest bound and log tail mass over the unopened clusters {c : 0 < key_c < kappa}: a max pass, then a sum pass.
// (best, vmax: the largest key and term among them)
__device__ __forceinline__ void tail_mass(const StepArgs& a, const ClusterLds& L, u64 kappa, u64 best, float vmax, SeqShared& s, float& nxtU, float& T) {
    float sum = 0.f;
    if (vmax > -INFINITY)
        for_clusters<false, true>(a.C, L, [&](int, u64 kx, int, float v) { sum += kx != 0 && kx < kappa ? expf(v - vmax) : 0.f; });
    sum = block_sum(sum, s.redf);
    nxtU = best ? ckey_bound(best) : -INFINITY;
    T = vmax > -INFINITY ? vmax + logf(sum) : -INFINITY;
}
__device__ __forceinline__ void tail_stats(const StepArgs& a, const ClusterLds& L, u64 kappa, SeqShared& s, float& nxtU, float& T) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    u64 best = 0;
    float vmax = -INFINITY;
    for (int c = threadIdx.x; c < a.C; c += blockDim.x) {
        const u64 kx = L.keys[c];
        if (kx != 0 && kx < kappa) {
            best = kx > best ? kx : best;
            vmax = fmaxf(vmax, L.vl[c]);
        }
    }
    best = wave_max_u64(best);
    vmax = wave_max(vmax);
    __syncthreads();
    if (lane == 0) {
        s.redu[w] = best;
        s.redf[w] = vmax;
    }
    __syncthreads();
    best = s.redu[0];
    vmax = s.redf[0];
    for (int i = 1; i < nw; ++i) {
        best = s.redu[i] > best ? s.redu[i] : best;
        vmax = fmaxf(vmax, s.redf[i]);
    }
    tail_mass(a, L, kappa, best, vmax, s, nxtU, T);
}

// What a plan needs to know of the clusters, in one pass and one reduction instead of two passes and three (C = 4096: with the
// log tail mass 7.0 us, 7.7 before): the clusters with kappa1 <= key < kappa0 (those
// it opens) and their rows, and of those below kappa1 the largest key and the largest term of the log tail mass (kappa1 <= kappa0).
struct PlanSums {
    int cnt, rows;
    u64 best;
    float vmax;
};
__device__ __forceinline__ PlanSums plan_sweep(const StepArgs& a, const ClusterLds& L, u64 kappa0, u64 kappa1, SeqShared& s) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    PlanSums p;
    p.cnt = p.rows = 0; p.best = 0; p.vmax = -INFINITY;
    for_clusters<true, true>(a.C, L, [&](int, u64 kx, int n, float v) {
        const bool on = kx != 0 && kx >= kappa1 && kx < kappa0, rest = kx != 0 && kx < kappa1;
        p.cnt += on ? 1 : 0;
        p.rows += on ? n : 0;
        p.best = rest && kx > p.best ? kx : p.best;
        p.vmax = fmaxf(p.vmax, rest ? v : -INFINITY);
    });
    p.cnt = wave_sum_i(p.cnt);
    p.rows = wave_sum_i(p.rows);
    p.best = wave_max_u64(p.best);
    p.vmax = wave_max(p.vmax);
    __syncthreads();
    if (lane == 0) {
        s.scan3[w] = p.cnt;
        s.scan3[16 + w] = p.rows;
        s.redu[w] = p.best;
        s.redf[w] = p.vmax;
    }
    __syncthreads();
    p.cnt = s.scan3[0]; p.rows = s.scan3[16]; p.best = s.redu[0]; p.vmax = s.redf[0];
    for (int i = 1; i < nw; ++i) {
        p.cnt += s.scan3[i];
        p.rows += s.scan3[16 + i];
        p.best = s.redu[i] > p.best ? s.redu[i] : p.best;
        p.vmax = fmaxf(p.vmax, s.redf[i]);
    }
    return p;
}

// ================================================================================================ gathered GEMV
// Work item = up to TILE_ROWS consecutive rows of W' for one sequence; one row per wave (8 waves).  Tiles of
// sequence b sit in its own region of the round's list; a prefix over the per-sequence counts maps a global tile
// number to (sequence, tile).  A block takes a contiguous run of tiles and has two of them in flight: both tiles' rows are requested in full (up to
// 16 KB per row) before anything is reduced, and the descriptors of the next pair are requested behind them, so an
// iteration costs one memory round trip for 16 rows.  h of the two tiles' sequences sits in two LDS slots (bf16)
// that are refilled only when the sequence changes.  128-bit loads, float32 accumulation, DPP wave reduction.
#define TILE_PF 16         // 128-bit pieces of a row requested at once per lane: a whole row up to d = 8192
struct GemvShared {
    int pre[CSV_MAX_BATCH + 1];
    int wsum[16];
};
// block / nblocks: this block's position in the set of blocks that share the work.  hs4: 2 * d * 2 bytes of LDS.
__device__ __forceinline__ void gemv_tiles_device(const StepArgs& a, int round, uint4* hs4, GemvShared& gs, int block, int nblocks) {
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wave = tid >> 6;
    {
        const int mine = tid < a.B ? a.counters[CNT_TILES + round * CSV_MAX_BATCH + tid] : 0;
        int x = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(x, o, CSV_WAVE);
            if (lane >= o) x += y;
        }
        __syncthreads();
        if (lane == 63) gs.wsum[wave] = x;
        __syncthreads();
        int base = 0;
        for (int i = 0; i < wave; ++i) base += gs.wsum[i];
        if (tid == 0) gs.pre[0] = 0;
        if (tid < CSV_MAX_BATCH) gs.pre[tid + 1] = base + x;
        __syncthreads();
    }
    const int total = gs.pre[a.B];
    const int nch = a.d >> 3;
    const Tile* tl = a.tiles[round & 1];
    auto fetch = [&](int g) {        // descriptor of global tile g; an empty tile past the end
        Tile t;
        t.b = 0; t.row0 = 0; t.nrows = 0; t.pos = 0;
        if (g < total) {
            int lo = 0, hi = a.B;   // largest b with pre[b] <= g
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (gs.pre[mid] <= g) lo = mid; else hi = mid;
            }
            t = tl[(size_t)lo * a.tile_stride + (g - gs.pre[lo])];
        }
        return t;
    };
    // a block takes a contiguous run of the list: mostly one sequence (h is staged once or twice per block, not
    // once per tile) and neighbouring rows
    const int per = (total + nblocks - 1) / nblocks;
    const int g0 = block * per, g1 = min(total, g0 + per);
    int cached[2] = {-1, -1};
    Tile tA = fetch(g0 < g1 ? g0 : total), tB = fetch(g0 + 1 < g1 ? g0 + 1 : total);
    for (int g = g0; g < g1; g += 2) {
        const Tile t[2] = {tA, tB};
        uint4 pf[2][TILE_PF];
        const uint4* w[2];
        float bias[2];
        int ids[2];
        bool act[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            act[q] = wave < t[q].nrows;
            const int r = t[q].row0 + (act[q] ? wave : 0);
            w[q] = reinterpret_cast<const uint4*>(a.Wp + (size_t)r * a.d);
#pragma unroll
            for (int j = 0; j < TILE_PF; ++j) {
                const int i = lane + 64 * j;
                pf[q][j] = (act[q] && i < nch) ? w[q][i] : make_uint4(0, 0, 0, 0);
            }
            bias[q] = 0.f;
            ids[q] = 0;
            if (act[q] && lane == 0) {
                bias[q] = a.bp[r];
                ids[q] = a.perm[r];
            }
        }
        // next pair's descriptors ride behind the row requests
        tA = fetch(g + 2 < g1 ? g + 2 : total);
        tB = fetch(g + 3 < g1 ? g + 3 : total);
        // h of the two sequences: slot q holds the sequence of tile q
        bool staged = false;
#pragma unroll
        for (int q = 0; q < 2; ++q)
            if (t[q].nrows > 0 && cached[q] != t[q].b) {
                if (!staged) __syncthreads();          // everyone is done with the slots' previous contents
                staged = true;
                const uint4* hsrc = reinterpret_cast<const uint4*>(a.h) + (size_t)t[q].b * nch;
                for (int i = tid; i < nch; i += nt) hs4[q * nch + i] = hsrc[i];
                cached[q] = t[q].b;
            }
        if (staged) __syncthreads();
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (!act[q]) continue;
            const uint4* hq = hs4 + q * nch;
            float acc = 0.f;
#pragma unroll
            for (int j = 0; j < TILE_PF; ++j) {
                const int i = lane + 64 * j;
                if (i < nch) acc = dot8_bf16(pf[q][j], hq[i], acc);
            }
            for (int i = lane + 64 * TILE_PF; i < nch; i += 64) acc = dot8_bf16(w[q][i], hq[i], acc);
            acc = wave_sum(acc);
            if (lane == 0) {
                const size_t o = (size_t)t[q].b * a.K_cap + t[q].pos + wave;
                a.slog[o] = acc + bias[q];
                a.sid[o] = ids[q];
            }
        }
    }
}

// Copy n 32-bit words from global memory to LDS.  Every trip issues eight loads per thread before the first
// store, also in the ragged last trip (out-of-range lanes load nothing), so a copy of up to 8 x blockDim words is
// one memory round trip.
template <class T>
__device__ __forceinline__ void stage_to_lds(T* dst, const T* __restrict__ src, int n) {
    const int tid = threadIdx.x, nt = blockDim.x;
    for (int i = tid; i < n; i += 8 * nt) {
        T r[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) r[q] = i + q * nt < n ? src[i + q * nt] : T(0);
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (i + q * nt < n) dst[i + q * nt] = r[q];
    }
}
// Two arrays of the same length at once (logits and token ids): both arrays' loads are in flight together.
__device__ __forceinline__ void stage2_to_lds(float* dv, const float* __restrict__ sv, int* di, const int* __restrict__ si, int n) {
    const int tid = threadIdx.x, nt = blockDim.x;
    for (int i = tid; i < n; i += 8 * nt) {
        float rv[8];
        int ri[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const bool in = i + q * nt < n;
            rv[q] = in ? sv[i + q * nt] : 0.f;
            ri[q] = in ? si[i + q * nt] : 0;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (i + q * nt < n) {
                dv[i + q * nt] = rv[q];
                di[i + q * nt] = ri[q];
            }
    }
}

// ================================================================================================ block top-k
// kk-th largest key among the elements for which key(i, kx) returns true (1 <= kk <= their number).
// On return: kth = that key, need_eq = how many elements equal to it belong to the largest kk, n_eq = how many equal it.
// Needs blockDim.x >= 256.
template <class KeyFn>
__device__ __forceinline__ void radix_select(int n, unsigned kk, KeyFn key, SeqShared& s, unsigned& kth,
                                             unsigned& need_eq, unsigned& n_eq) {
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, w = tid >> 6, nw = (nt + 63) >> 6;
    // Bytes that all keys share from the top need no pass (logits of one cluster differ only in their low bits,
    // and a histogram pass over a shared byte would send every element to the same bin).
    unsigned kmin = 0xffffffffu, kmax = 0u;
    for (int i = tid; i < n; i += nt) {
        unsigned kx;
        if (key(i, kx)) {
            kmin = kx < kmin ? kx : kmin;
            kmax = kx > kmax ? kx : kmax;
        }
    }
    kmax = wave_max_u(kmax);
    kmin = ~wave_max_u(~kmin);
    __syncthreads();
    if (lane == 0) {
        s.hist[w] = kmax;
        s.hist[16 + w] = kmin;
    }
    __syncthreads();
    for (int i = 0; i < nw; ++i) {
        kmax = s.hist[i] > kmax ? s.hist[i] : kmax;
        kmin = s.hist[16 + i] < kmin ? s.hist[16 + i] : kmin;
    }
    __syncthreads();
    const unsigned diff = kmin ^ kmax;
    int first_shift = 24;
    unsigned prefix = 0, mask = 0, rem = kk, eq = 0;
    while (first_shift > 0 && ((diff >> first_shift) & 0xffu) == 0) {
        prefix |= kmax & (0xffu << first_shift);
        mask |= 0xffu << first_shift;
        first_shift -= 8;
    }
    for (int shift = first_shift; shift >= 0; shift -= 8) {
        for (int t = tid; t < 256; t += nt) s.hist[t] = 0;
        __syncthreads();
        for (int i0 = 0; i0 < n; i0 += nt) {
            const int i = i0 + tid;
            unsigned kx = 0;
            const bool in = i < n && key(i, kx) && (kx & mask) == prefix;
            const unsigned dg = (kx >> shift) & 255u;
            // one atomic per wave when every participating lane has the same digit
            const unsigned long long act = __ballot(in);
            if (act) {
                const unsigned d0 = __shfl(dg, __ffsll((long long)act) - 1, CSV_WAVE);
                const unsigned long long same = __ballot(in && dg == d0);
                if (same == act) {
                    if (lane == __ffsll((long long)act) - 1) atomicAdd(&s.hist[d0], (unsigned)__popcll(act));
                } else if (in) {
                    atomicAdd(&s.hist[dg], 1u);
                }
            }
        }
        __syncthreads();
        if (tid < 64) {
            // lane l owns bins 4l..4l+3; suffix sums by a descending scan inside the first wave
            const unsigned h0 = s.hist[4 * lane], h1 = s.hist[4 * lane + 1], h2 = s.hist[4 * lane + 2], h3 = s.hist[4 * lane + 3];
            const unsigned mine = h0 + h1 + h2 + h3;
            unsigned x = mine;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const unsigned y = __shfl_down(x, o, CSV_WAVE);
                if (lane + o < 64) x += y;
            }
            const unsigned gt3 = x - mine;          // elements in bins above 4l+3
            const unsigned gt2 = gt3 + h3, gt1 = gt2 + h2, gt0 = gt1 + h1, ge0 = gt0 + h0;
            if (ge0 >= rem && gt3 < rem) {           // the kk-th falls into one of my bins
                unsigned selb, gt, cntb;
                if (gt2 >= rem) { selb = 3; gt = gt3; cntb = h3; }
                else if (gt1 >= rem) { selb = 2; gt = gt2; cntb = h2; }
                else if (gt0 >= rem) { selb = 1; gt = gt1; cntb = h1; }
                else { selb = 0; gt = gt0; cntb = h0; }
                s.sel = 4u * lane + selb;
                s.rem = rem - gt;
                s.eq = cntb;
            }
        }
        __syncthreads();
        prefix |= s.sel << shift;
        mask |= 0xffu << shift;
        rem = s.rem;
        eq = s.eq;
        if (shift > 0 && eq <= 256u) {
            // few candidates left in the selected bin: list them and rank them directly instead of more passes
            __syncthreads();
            if (tid == 0) s.cnt = 0;
            __syncthreads();
            for (int i = tid; i < n; i += nt) {
                unsigned kx = 0;
                if (key(i, kx) && (kx & mask) == prefix) s.hist[atomicAdd(&s.cnt, 1u)] = kx;
            }
            __syncthreads();
            if (tid < (int)eq) {
                const unsigned v = s.hist[tid];
                unsigned gt = 0, ge = 0;
                for (unsigned j = 0; j < eq; ++j) {
                    const unsigned x = s.hist[j];
                    gt += x > v;
                    ge += x >= v;
                }
                if (gt < rem && rem <= ge) {     // every thread holding this value writes the same three numbers
                    s.sel = v;
                    s.rem = rem - gt;
                    s.eq = ge - gt;
                }
            }
            __syncthreads();
            kth = s.sel;
            need_eq = s.rem;
            n_eq = s.eq;
            __syncthreads();
            return;
        }
    }
    kth = prefix;
    need_eq = rem;
    n_eq = eq;
}

// Largest min(k,n) of n values in order (value descending, id ascending).  Result in s.wval / s.wid.
// val(i) and id_of(i) may read LDS or global memory.  Returns min(k,n).
template <class ValFn, class IdFn>
__device__ __forceinline__ int block_topk(int n, int k, ValFn val, IdFn id_of, SeqShared& s) {
    const int tid = threadIdx.x, nt = blockDim.x;
    const int kk = min(k, n);
    if (kk <= 0) return 0;
    if (n <= nt) {
        // rank of every element = number of larger values.  The n x n comparisons are spread over all threads:
        // thread (e, slice) compares element e with one slice of the others and adds its count (larger values in
        // the low half, equal values in the high half) to rank[e].  Ids are looked at only by elements that have
        // an equal somewhere else.  blockDim.x must be a power of two.
        int lg = 0;
        while ((1 << lg) < n) ++lg;
        const int npad = 1 << lg, slices = nt >> lg;
        const int e = tid & (npad - 1), sl = tid >> lg;
        __syncthreads();
        if (tid < npad) s.rank[tid] = 0;
        __syncthreads();
        const int len = ((n + slices - 1) / slices + 3) & ~3;
        const int j0 = sl * len, j1 = min(n, j0 + len);
        if (e < n && j0 < j1) {
            const float v = val(e);
            int gt = 0, eq = 0;
            int j = j0;
#pragma unroll 2
            for (; j + 4 <= j1; j += 4) {
                const float q0 = val(j), q1 = val(j + 1), q2 = val(j + 2), q3 = val(j + 3);
                gt += (q0 > v) + (q1 > v) + (q2 > v) + (q3 > v);
                eq += (q0 == v) + (q1 == v) + (q2 == v) + (q3 == v);
            }
            for (; j < j1; ++j) {
                const float vj = val(j);
                gt += vj > v;
                eq += vj == v;
            }
            atomicAdd(&s.rank[e], gt | (eq << 16));
        }
        __syncthreads();
        if (tid < n) {
            const float v = val(tid);
            const int id = id_of(tid);
            const int packed = s.rank[tid];
            int rank = packed & 0xffff;
            if ((packed >> 16) > 1)
                for (int i = 0; i < n; ++i)
                    if (val(i) == v && id_of(i) < id) rank += 1;
            if (rank < kk) {
                s.wval[rank] = v;
                s.wid[rank] = id;
            }
        }
        __syncthreads();
        return kk;
    }
    if (kk < n) {
        unsigned kth, need, neq;
        radix_select(n, (unsigned)kk, [&](int i, unsigned& kx) { kx = lkey(val(i)); return true; }, s, kth, need, neq);
        unsigned idkey = 0;   // boundary elements win when ~id >= idkey
        if (need < neq) {
            unsigned u1, u2;
            radix_select(n, need,
                         [&](int i, unsigned& kx) {
                             if (lkey(val(i)) != kth) return false;
                             kx = ~(unsigned)id_of(i);
                             return true;
                         },
                         s, idkey, u1, u2);
        }
        if (tid == 0) s.cnt = 0;
        __syncthreads();
        for (int i = tid; i < n; i += nt) {
            const float v = val(i);
            const unsigned kx = lkey(v);
            if (kx >= kth) {
                const int id = id_of(i);
                if (kx > kth || (~(unsigned)id) >= idkey) {
                    const unsigned slot = atomicAdd(&s.cnt, 1u);
                    if (slot < CSV_MAX_K) {
                        s.wval[slot] = v;
                        s.wid[slot] = id;
                    }
                }
            }
        }
        __syncthreads();
    } else {
        for (int i = tid; i < n; i += nt) {
            s.wval[i] = val(i);
            s.wid[i] = id_of(i);
        }
        __syncthreads();
    }
    // order the winners in place: ranks first, then a permuted write (CSV_MAX_K <= 4 * 256 threads)
    float mv[4];
    int mi[4], mr[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int t = tid + e * nt;
        mr[e] = -1;
        if (t < kk) {
            const float v = s.wval[t];
            const int id = s.wid[t];
            int rank = 0;
            for (int j = 0; j < kk; ++j) {
                const float vj = s.wval[j];
                rank += (vj > v) || (vj == v && s.wid[j] < id);
            }
            mv[e] = v; mi[e] = id; mr[e] = rank;
        }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (mr[e] >= 0) {
            s.wval[mr[e]] = mv[e];
            s.wid[mr[e]] = mi[e];
        }
    __syncthreads();
    return kk;
}

// max and sum exp(x - max) of n values, fixed reduction order
template <class ValFn>
__device__ __forceinline__ LseAcc block_lse(int n, ValFn val, SeqShared& s) {
    float mx = -INFINITY;
    for (int i = threadIdx.x; i < n; i += blockDim.x) mx = fmaxf(mx, val(i));
    mx = block_max(mx, s.redf);
    float sm = 0.f;
    if (mx > -INFINITY)
        for (int i = threadIdx.x; i < n; i += blockDim.x) sm += expf(val(i) - mx);
    sm = block_sum(sm, s.redf);
    LseAcc r;
    r.m = mx;
    r.s = sm;
    return r;
}

// ================================================================================================ prefix search
// The first wave: of 256 classes of ascending keys (H: weights, cnt: members) the largest that is not empty and has at most the
// limit (2^40) below it, base included.  Leaves it in s.sel and the weight below it in s.redu[0].
__device__ __forceinline__ void prefix_pick(const u64* H, const unsigned* cnt, u64 base, SeqShared& s) {
    const int lane = threadIdx.x & 63;
    // lane l owns digits 4l..4l+3; weights below a digit by an ascending scan inside the first wave
    u64 h[4];
    unsigned n4[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        h[q] = H[4 * lane + q];
        n4[q] = cnt[4 * lane + q];
    }
    const u64 mine = h[0] + h[1] + h[2] + h[3];
    u64 x = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const u64 y = __shfl_up(x, o, CSV_WAVE);
        if (lane >= o) x += y;
    }
    u64 below[4];
    below[0] = base + (x - mine);
    below[1] = below[0] + h[0];
    below[2] = below[1] + h[1];
    below[3] = below[2] + h[2];
    int pick = -1;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (n4[q] != 0 && below[q] <= (1ull << 40)) pick = 4 * lane + q;
    const int best = (int)wave_max_u((unsigned)(pick + 1)) - 1;
    if (best >= 0 && (best >> 2) == lane) {
        s.sel = (unsigned)best;
        s.redu[0] = below[best & 3];
    }
    if (best < 0 && lane == 0) {                  // cannot happen (the smallest key has nothing below it); stay defined
        s.sel = 0u;
        s.redu[0] = base;
    }
}
// The shortest prefix of the bound order, no shorter than the open one, whose log tail mass is within lam of Z0
// (Theorem 2): returns the key of its last cluster.  In terms of keys: the largest key kappa <= kappa0 such that the
// clusters below it weigh  sum_{key_c < kappa} n_c exp(U_c)  <=  exp(Z0 + lam).  No sort: the key is found digit by
// digit from the top (eight bits a pass).  Among the keys that share the digits fixed so far, the clusters of a
// smaller digit all lie below those of a larger one, so a digit can hold the answer when it is not empty and the
// weight below its smallest key (everything below the fixed digits, plus the smaller digits) is within the limit;
// the largest such digit is taken.  Weights are summed as 64-bit fixed point relative to the limit (2^-40 steps, each
// term capped at 2^9, which already exceeds the limit of 1): integer sums do not depend on the order of the atomic
// additions, so the result is the same in every run.  Leaves the cluster data in LDS as it is.  Uses s.rank and s.hist.
// among: the clusters to search, base: the weight of everything below them (all clusters and 0 unless softmax_prefix_fast has
// narrowed them down).
template <class AmongFn>
__device__ __forceinline__ u64 softmax_prefix_key(const StepArgs& a, const ClusterLds& L, u64 kappa0, float Z0, SeqShared& s, AmongFn among, u64 base) {
    const int tid = threadIdx.x, nt = blockDim.x;
    u64* H = reinterpret_cast<u64*>(s.rank);               // 256 weights
    unsigned* cnt = s.hist;                                // 256 counts
    const float shift = Z0 + a.lam;
    u64 prefix = 0;
    for (int sb = 56; sb >= 0; sb -= 8) {
        if (sb == 24 || sb == 16) {                        // bits 16..31 of ~c: ones for every cluster id below 65536
            prefix |= 0xffull << sb;
            continue;
        }
        if (tid < 256) {
            H[tid] = 0ull;
            cnt[tid] = 0u;
        }
        __syncthreads();
        for (int c = tid; c < a.C; c += nt) {
            const u64 kx = L.keys[c];
            const bool match = sb == 56 || ((kx ^ prefix) >> (sb + 8)) == 0;
            if (kx != 0 && kx <= kappa0 && match && among(kx)) {
                const float e = expf(fminf(L.vl[c] - shift, 6.f));         // e^6 < 2^9
                const unsigned dg = (unsigned)(kx >> sb) & 255u;
                atomicAdd(reinterpret_cast<unsigned long long*>(&H[dg]), (unsigned long long)(e * 1099511627776.f));
                atomicAdd(&cnt[dg], 1u);
            }
        }
        __syncthreads();
        if (tid < 64) prefix_pick(H, cnt, base, s);
        __syncthreads();
        prefix |= (u64)s.sel << sb;
        base = s.redu[0];
    }
    __syncthreads();
    return prefix;
}

// The same key, found sooner: 256 classes of equal width between the smallest and the largest bound instead of leading digits.
// Nearly all bounds share their first digits, and 64-bit LDS additions to one address go one after the other (the
// digits took 7.4 us at C = 1024, mostly that; this way 4.2 us).  The class of a bound is a monotone function of it, so the class that holds the
// answer is picked as a digit is; up to 64 members of it then settle it in every wave alone: each lane adds up what lies
// below its own key.  The sums are the same integers, so the answer is the same key.  More members: the digits, among
// them only.  Bounds that are not finite, or too close together for a finite class width: the digits, from the start.
__device__ __forceinline__ u64 softmax_prefix_fast(const StepArgs& a, const ClusterLds& L, u64 kappa0, float Z0, SeqShared& s) {
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63;
    const float shift = Z0 + a.lam;
    float up = -INFINITY, down = -INFINITY;                // the largest bound, the largest negated bound
    for_clusters<false, false>(a.C, L, [&](int, u64 kx, int, float) {
        const bool on = kx != 0 && kx <= kappa0;
        const float u = ckey_bound(kx);
        up = fmaxf(up, on ? (isfinite(u) ? u : INFINITY) : -INFINITY);
        down = fmaxf(down, on ? -u : -INFINITY);
    });
    up = wave_max(up);
    down = wave_max(down);
    __syncthreads();
    if (lane == 0) {
        s.redf[tid >> 6] = up;
        s.redi[tid >> 6] = __float_as_int(down);
    }
    __syncthreads();
    for (int i = 0; i < (nt >> 6); ++i) {
        up = fmaxf(up, s.redf[i]);
        down = fmaxf(down, __int_as_float(s.redi[i]));
    }
    const float lo = -down, scale = 256.f / (up - lo);
    if (!(isfinite(up) && isfinite(lo) && isfinite(scale) && scale > 0.f))
        return softmax_prefix_key(a, L, kappa0, Z0, s, [](u64) { return true; }, 0ull);
    auto cls = [&](u64 kx) { return (unsigned)fminf((ckey_bound(kx) - lo) * scale, 255.f); };
    auto weight = [&](float v) { return (u64)(expf(fminf(v - shift, 6.f)) * 1099511627776.f); };       // as in the digit search
    u64* H = reinterpret_cast<u64*>(s.rank);
    unsigned* cnt = s.hist;
    if (tid < 256) {
        H[tid] = 0ull;
        cnt[tid] = 0u;
    }
    __syncthreads();
    for_clusters<false, true>(a.C, L, [&](int, u64 kx, int, float v) {
        if (kx == 0 || kx > kappa0) return;
        const unsigned q = cls(kx);
        atomicAdd(reinterpret_cast<unsigned long long*>(&H[q]), (unsigned long long)weight(v));
        atomicAdd(&cnt[q], 1u);
    });
    __syncthreads();
    if (tid < 64) prefix_pick(H, cnt, 0ull, s);
    if (tid == 0) s.cnt = 0;
    __syncthreads();
    const unsigned q0 = s.sel;
    const int m = (int)cnt[q0];
    const u64 base = s.redu[0];
    __syncthreads();                                       // everyone has read the class: its members take its place
    if (m > 64) return softmax_prefix_key(a, L, kappa0, Z0, s, [&](u64 kx) { return cls(kx) == q0; }, base);
    u64* mk = H;
    u64* mw = H + 64;
    for_clusters<false, true>(a.C, L, [&](int, u64 kx, int, float v) {
        if (kx == 0 || kx > kappa0 || cls(kx) != q0) return;
        const unsigned i = atomicAdd(&s.cnt, 1u);
        mk[i] = kx;
        mw[i] = weight(v);
    });
    __syncthreads();
    const u64 mine = lane < m ? mk[lane] : 0ull;
    u64 below = base;
    for (int i = 0; i < m; ++i) below += mk[i] < mine ? mw[i] : 0ull;
    const u64 best = wave_max_u64(mine != 0 && below <= (1ull << 40) ? mine : 0ull);
    __syncthreads();
    return best;
}

// Ordered top-kk (value descending, id ascending) of len <= blockDim.x values V in LDS with ids I; V is followed by
// -inf up to the next multiple of four.  One pass, one barrier: thread (e, slice) compares value e with one slice of
// the others (larger ones, equal ones) and notes the slice's maximum; after the barrier thread e adds the slices'
// counts to its rank (ids are looked at only among equal values) and writes itself to its place in s.wval / s.wid.
// Returns the largest value; v is the value of element threadIdx.x (threadIdx.x < len).  The caller's next barrier
// publishes the list.  blockDim.x is a power of two.
__device__ __forceinline__ float rank_small(const float* V, const int* I, int len, int kk, SeqShared& s, float& v) {
    const int tid = threadIdx.x, nt = blockDim.x;
    int lg = 5;
    while ((1 << lg) < len) ++lg;
    const int npad = 1 << lg, slices = nt >> lg;           // slices <= 16
    const int e = tid & (npad - 1), sl = tid >> lg;
    const int len4 = (len + 3) >> 2;                         // slices of whole float4's
    const int seg4 = (len4 + slices - 1) / slices;
    const int q0 = min(len4, sl * seg4), q1 = min(len4, q0 + seg4);
    const float ve = V[min(e, max(len, 1) - 1)];
    int gt = 0, eq = 0;
    float mx = -INFINITY;
    const float4* v4 = reinterpret_cast<const float4*>(V);
#pragma unroll 8
    for (int q = q0; q < q1; ++q) {
        const float4 x = v4[q];
        gt += (x.x > ve) + (x.y > ve) + (x.z > ve) + (x.w > ve);
        eq += (x.x == ve) + (x.y == ve) + (x.z == ve) + (x.w == ve);
        mx = fmaxf(fmaxf(mx, fmaxf(x.x, x.y)), fmaxf(x.z, x.w));
    }
    s.rank[tid] = gt | (eq << 16);                          // rank[sl * npad + e]
    if (e == 0) s.redf[sl] = mx;
    __syncthreads();
    float vmax = s.redf[0];
    for (int q = 1; q < slices; ++q) vmax = fmaxf(vmax, s.redf[q]);
    v = ve;                                                 // tid < len <= npad: e is tid
    if (tid < len) {
        int packed = 0;
        for (int q = 0; q < slices; ++q) packed += s.rank[q * npad + tid];
        int rank = packed & 0xffff;
        const int id = I[tid];
        if ((packed >> 16) > 1)
            for (int i = 0; i < len; ++i)
                if (V[i] == v && I[i] < id) rank += 1;
        if (rank < kk) {
            s.wval[rank] = v;
            s.wid[rank] = id;
        }
    }
    return vmax;
}

// Ordered top-kk of m <= blockDim.x candidates V / I in LDS (one per thread), none of them below lo: a counting
// sort into 256 equal-width buckets between lo and hi, largest values first, then every candidate whose bucket starts within the first
// kk places ranks itself against the members of its bucket (equal values by id); values above hi share the first bucket.  Exact for any distribution of the
// values (a crowded bucket only costs time); the comparisons of rank_small grow with m * m, these with m.  V / I are
// reordered (bucket by bucket; the order inside a bucket depends on timing, the ranks do not).  The caller's next
// barrier publishes s.wval / s.wid.  Uses s.hist, s.rank, s.redi.
__device__ __forceinline__ void rank_buckets(float* V, int* I, int m, int kk, float lo, float hi, SeqShared& s) {
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const float scale = (hi > lo && lo > -INFINITY && hi < INFINITY) ? 255.f / (hi - lo) : 0.f;
    float v = 0.f;
    int id = 0, d = 0;
    if (tid < m) {
        v = V[tid];
        id = I[tid];
        d = scale > 0.f ? 255 - min(255, max(0, (int)((v - lo) * scale))) : 0;
    }
    if (tid < 256) s.hist[tid] = 0;
    __syncthreads();
    unsigned slot = 0;
    if (tid < m) slot = atomicAdd(&s.hist[d], 1u);
    __syncthreads();
    if (tid < 256) {
        const int c = (int)s.hist[tid];
        int x = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(x, o, CSV_WAVE);
            if (lane >= o) x += y;
        }
        if (lane == 63) s.redi[w] = x;
        s.rank[tid] = x - c;                                // first place of the bucket, counted within its wave of buckets
    }
    __syncthreads();
    int start = 0, cnt = 0;
    if (tid < m) {
        start = s.rank[d];
        for (int i = 0; i < (d >> 6); ++i) start += s.redi[i];
        cnt = (int)s.hist[d];
        V[start + (int)slot] = v;
        I[start + (int)slot] = id;
    }
    __syncthreads();
    if (tid < m && start < kk) {
        int r = start;
#pragma unroll 4
        for (int j = start; j < start + cnt; ++j) {
            const float x = V[j];
            r += (x > v || (x == v && I[j] < id)) ? 1 : 0;
        }
        if (r < kk) {
            s.wval[r] = v;
            s.wid[r] = id;
        }
    }
}
#define RANK_BUCKETS_MIN 128     // more candidates than this (with a finite range) take rank_buckets instead of rank_small

// Ordered top-k of len > RANK_DIRECT values staged at the start of the dynamic LDS (ranking all of them against each
// other costs len^2 comparisons: 10 us at 512).  Everything below a threshold that k of the values are known to reach
// is out; the values at or above it (usually few more than k) are collected behind the staged data and ranked in one
// pass.  First threshold: theta, a value the caller knows k of the values to reach (-inf: none).  Failing that, or
// when more than CAND_CAP values reach it: the k-th largest of RANK_DIRECT group maxima.  short_ok: the values are one chunk of several
// and fewer than k of them may reach theta (the merged lists still hold the overall top-k).  The collected order
// depends on timing, the ranking does not.  On success s.wval / s.wid hold kkv entries once the caller has passed a
// barrier, vmax is the largest value; on failure (k > RANK_DIRECT, too many survivors) nothing is decided.
// MERGE: the values are lists of several chunks, unused places marked by the id 0x7fffffff (and the value -inf): those are
// left out, and the first attempt also runs without a threshold (len may then be RANK_DIRECT or less).
// LATE_IDS: idf reads global memory: the candidates are collected with their positions and all look their ids up
// together afterwards (a load in the collecting loop would be waited for in every trip that collects something).
template <bool MERGE = false, bool LATE_IDS = false, class IdFn>
__device__ __forceinline__ bool threshold_topk(int len, int k, float theta, bool short_ok, IdFn idf, SeqShared& s, int& kkv, float& vmax) {
    extern __shared__ __align__(16) u64 arena[];
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63;
    const float* V = reinterpret_cast<const float*>(arena);
    const int k0 = min(k, len);
    auto attempt = [&](float th) -> bool {
        float* wmax = reinterpret_cast<float*>(s.redu);        // not s.hist / s.redf: the ranking writes those while others still read here
        float* cval = reinterpret_cast<float*>(reinterpret_cast<char*>(arena) + CAND_OFF);
        int* cid = reinterpret_cast<int*>(cval + CAND_CAP + 4);
        if (tid < CAND_CAP) cval[tid] = -INFINITY;
        if (tid < 4) cval[CAND_CAP + tid] = -INFINITY;
        if (tid == 0) s.cnt = 0;
        __syncthreads();
        float mx = -INFINITY, over = 0.f;                  // over: sum of (v - th) over the collected values
        for (int i0 = 0; i0 < len; i0 += nt) {
            const int i = i0 + tid;
            const float v = i < len ? V[i] : -INFINITY;
            mx = fmaxf(mx, v);
            const bool in = i < len && v >= th && (!MERGE || idf(i) != 0x7fffffff);
            if (in) over += v - th;
            const unsigned long long bal = __ballot(in);
            if (bal) {
                const int lead = __ffsll((long long)bal) - 1;
                unsigned base = 0;
                if (lane == lead) base = atomicAdd(&s.cnt, (unsigned)__popcll(bal));
                base = __shfl(base, lead, CSV_WAVE);
                const unsigned slot = base + (unsigned)__popcll(bal & ((1ull << lane) - 1ull));
                if (in && slot < CAND_CAP) {
                    cval[slot] = v;
                    cid[slot] = LATE_IDS ? i : idf(i);
                }
            }
        }
        mx = wave_max(mx);
        over = wave_sum(over);
        if (lane == 0) {
            wmax[tid >> 6] = mx;
            wmax[16 + (tid >> 6)] = over;
        }
        __syncthreads();
        const int m = (int)s.cnt;
        if (m > CAND_CAP || (!short_ok && m < k0)) return false;
        vmax = wmax[0];
        for (int q = 1; q < (nt >> 6); ++q) vmax = fmaxf(vmax, wmax[q]);
        if (LATE_IDS) {
            if (tid < m) cid[tid] = idf(cid[tid]);
            __syncthreads();
        }
        kkv = min(k, m);
        if (m > RANK_BUCKETS_MIN && th > -INFINITY) {
            // the values thin out above the threshold: equal-width buckets up to eight times their mean excess hold a
            // few values each, whatever lies beyond (a handful of outstanding logits) shares the first bucket
            float tot = 0.f;
            for (int q = 0; q < (nt >> 6); ++q) tot += wmax[16 + q];
            rank_buckets(cval, cid, m, kkv, th, fminf(vmax, th + 8.f * tot / (float)m), s);
        } else {
            float v;
            rank_small(cval, cid, m, kkv, s, v);
        }
        return true;
    };
    bool ok = false;
    if (MERGE || theta > -INFINITY) ok = attempt(theta);
    if (!ok && k <= RANK_DIRECT && len > RANK_DIRECT) {
        // RANK_DIRECT group maxima (group g: the values i with i % RANK_DIRECT == g; len > RANK_DIRECT, so no group is
        // empty): k of them, hence k of the values, reach their k-th largest, and since the largest values mostly sit
        // in different groups few more do
        float* cval = reinterpret_cast<float*>(reinterpret_cast<char*>(arena) + CAND_OFF);
        float mx = -INFINITY;
        for (int i = tid; i < len; i += nt) mx = fmaxf(mx, V[i]);
        __syncthreads();
        if (tid < CAND_CAP) cval[tid] = mx;
        __syncthreads();
        float m2 = -INFINITY;
        if (tid < RANK_DIRECT) {
            m2 = cval[tid];
            for (int j = tid + RANK_DIRECT; j < min(nt, CAND_CAP); j += RANK_DIRECT) m2 = fmaxf(m2, cval[j]);
        }
        __syncthreads();
        if (tid < RANK_DIRECT) cval[tid] = m2;
        __syncthreads();
        float v;
        rank_small(cval, reinterpret_cast<const int*>(cval), RANK_DIRECT, k, s, v);      // only the k-th value is wanted: any ids do
        __syncthreads();
        const float th = fmaxf(s.wval[k - 1], theta);
        __syncthreads();
        ok = attempt(th);
    }
    return ok;
}

// ================================================================================================ certified distribution
// Optional outputs (Section III, top-p certification): over the returned list, in its order, the sub-vocabulary
// probabilities p~_t = exp(l_t - Z_S), their running sums, and the length of the shortest prefix whose running sum
// reaches top_p (0: not reached within the list).  kk entries of s.wval are valid; Z is the log-sum-exp that goes
// to d_lse.  Every thread of the block calls.  Each running sum is taken in list order by one thread.
__device__ __forceinline__ void write_distribution(const StepArgs& a, int b, int kk, float Z, SeqShared& s) {
    if (!a.out.d_probs && !a.out.d_cum && !a.out.d_nucleus) return;
    const int tid = threadIdx.x, nt = blockDim.x;
    int below = 0;
    for (int t = tid; t < a.k; t += nt) {
        float p = 0.f, cum = 0.f;
        const int last = min(t, kk - 1);
        for (int j = 0; j <= last; ++j) {
            const float pj = expf(s.wval[j] - Z);
            cum += pj;
            if (j == t) p = pj;
        }
        if (a.out.d_probs) a.out.d_probs[(size_t)b * a.k + t] = p;
        if (a.out.d_cum) a.out.d_cum[(size_t)b * a.k + t] = cum;
        below += (t < kk && cum < a.top_p) ? 1 : 0;
    }
    if (a.out.d_nucleus) {
        below = block_sum_i(below, s.redi);
        if (tid == 0) a.out.d_nucleus[b] = (a.top_p > 0.f && below < kk) ? below + 1 : 0;
    }
}

// ================================================================================================ certification
// One block per sequence.  round 0: certify, or plan round 1 (or fall back on budget); round 1: certify or fall back.
// Sequences with more than STAGE_CAP scored rows are handled by several blocks: each takes one chunk of STAGE_CAP
// logits, publishes the chunk's top-k candidates and log-sum-exp partial, and the block that arrives last (a
// device-scope counter; nobody waits) merges them and goes on to the tests.
// staged: the caller has already put the sequence's logits and ids where the staging below would put them
// Returns true when the sequence is finished (its outputs are written), false when work was queued for later phases
// (another round, the full vocabulary) or nothing was done.
// THRESH: compile the threshold selection for more than RANK_DIRECT values.  The fused step kernel leaves it out (its
// rare larger selections take the general path): with that code in the kernel a single-sequence step took 0.3 us
// longer, although the step never runs it.
// PLANS: compile the quicker forms of a plan (softmax_prefix_fast, plan_sweep, emit_list).  They pay where plans are made
// (us a step without / with them: 8 sequences, C = 1500 121 / 113; 34, C = 2445 545 / 525; 25, C = 1108 64 / 61) and cost, as code
// that is never run, where none is (11 sequences certified at once, C = 1550: 36.3 / 37.7; 3, C = 825: 20.2 / 21.0).
template <bool THRESH, bool PLANS>
__device__ __forceinline__ bool cert_body(const StepArgs& a, int b, int chunk, int round, const SeqState& st, SeqShared& s,
                                          bool staged = false, int* settled_count = nullptr) {
    extern __shared__ __align__(16) u64 arena[];
    const int tid = threadIdx.x, nt = blockDim.x, C = a.C;
    if (st.status != ST_ACTIVE || st.rounds != round) return false;
    const int n = st.n_rows;
    const int nchunks = (n + STAGE_CAP - 1) / STAGE_CAP;
    if (chunk >= nchunks) return false;
    const int c0 = chunk * STAGE_CAP, len = min(STAGE_CAP, n - c0);
    if (!staged) {
        const float* gv = a.slog + (size_t)b * a.K_cap + c0;
        const int32_t* gi = a.sid + (size_t)b * a.K_cap + c0;
        stage2_to_lds(reinterpret_cast<float*>(arena), gv, reinterpret_cast<int*>(arena) + STAGE_CAP, gi, len);
        if (tid < 4 && len + tid < STAGE_CAP) reinterpret_cast<float*>(arena)[len + tid] = -INFINITY;   // see the small path below
        __syncthreads();
    }
    // the accessors name the LDS array itself so that the reads compile to LDS instructions
    auto val = [](int i) { return reinterpret_cast<const float*>(arena)[i]; };
    auto idf = [](int i) { return reinterpret_cast<const int*>(arena)[STAGE_CAP + i]; };
    // with a top-k the largest logit is already known when the sum is taken: one block reduction instead of two
    LseAcc l;
    int kkv = min(a.k, len);                 // entries of the ordered list this chunk contributes
    bool have_topk = false;
    if (a.use_k && len <= RANK_DIRECT) {
        // few values: ordered top-k and log-sum-exp in one pass with two barriers
        float v;
        const float vmax = rank_small(reinterpret_cast<const float*>(arena), reinterpret_cast<const int*>(arena) + STAGE_CAP, len, kkv, s, v);
        float pe = (tid < len && vmax > -INFINITY) ? expf(v - vmax) : 0.f;
        pe = wave_sum(pe);
        float* wsum = reinterpret_cast<float*>(s.hist);
        if ((tid & 63) == 0) wsum[tid >> 6] = pe;
        __syncthreads();
        float tot = 0.f;
        for (int q = 0; q < (nt >> 6); ++q) tot += wsum[q];
        l.m = vmax;
        l.s = tot;
        have_topk = true;
    } else if (THRESH && a.use_k) {
        // more values: through a threshold (see threshold_topk); the log-sum-exp runs over all values
        float vmax;
        if (threshold_topk(len, a.k, st.theta, nchunks > 1, idf, s, kkv, vmax)) {
            float sm = 0.f;
            if (vmax > -INFINITY)
                for (int i = tid; i < len; i += nt) sm += expf(val(i) - vmax);
            l.m = vmax;
            l.s = block_sum(sm, s.redf);
            have_topk = true;
        }
    }
    if (have_topk) {
        // list and log-sum-exp are set
    } else if (a.use_k) {
        block_topk(len, a.k, val, idf, s);
        l.m = s.wval[0];
        float sm = 0.f;
        if (l.m > -INFINITY)
            for (int i = tid; i < len; i += nt) sm += expf(val(i) - l.m);
        l.s = block_sum(sm, s.redf);
    } else {
        l = block_lse(len, val, s);
    }
    if (nchunks > 1) {
        const size_t pb = (size_t)b * a.cand_chunks, pc = pb + chunk;
        const int kk = kkv;
        for (int t = tid; t < a.k; t += nt) {
            a.cand_val[pc * a.k + t] = t < kk ? s.wval[t] : -INFINITY;
            a.cand_id[pc * a.k + t] = t < kk ? s.wid[t] : 0x7fffffff;
        }
        if (tid == 0) {
            a.cand_max[pc] = l.m;
            a.cand_sum[pc] = l.s;
        }
        __threadfence();
        __syncthreads();
        if (tid == 0) s.sel = atomicAdd(&a.counters[CNT_CHUNKS + round * CSV_MAX_BATCH + b], 1) == nchunks - 1;
        __syncthreads();
        if (!s.sel) return false;
        __threadfence();
        float mx = -INFINITY;
        for (int i = tid; i < nchunks; i += nt) mx = fmaxf(mx, a.cand_max[pb + i]);
        mx = block_max(mx, s.redf);
        float sm = 0.f;
        for (int i = tid; i < nchunks; i += nt) sm += a.cand_sum[pb + i] * expf(a.cand_max[pb + i] - mx);
        l.m = mx;
        l.s = block_sum(sm, s.redf);
        if (a.use_k) {
            const float* cv = a.cand_val + pb * a.k;
            const int32_t* ci = a.cand_id + pb * a.k;
            const int nc = nchunks * a.k;
            if (nc <= STAGE_CAP) {
                __syncthreads();
                stage2_to_lds(reinterpret_cast<float*>(arena), cv, reinterpret_cast<int*>(arena) + STAGE_CAP, ci, nc);
                __syncthreads();
                bool merged = false;
                if (THRESH) {
                    int kq;
                    float vm;
                    merged = threshold_topk<true>(nc, a.k, st.theta, false, idf, s, kq, vm);
                    __syncthreads();
                }
                if (!merged) block_topk(nc, a.k, val, idf, s);
            } else {
                block_topk(nc, a.k, [&](int i) { return cv[i]; }, [&](int i) { return ci[i]; }, s);
            }
        }
    }
    const float Z = lse_value(l);
    float theta = -INFINITY;
    if (a.use_k) theta = s.wval[a.k - 1];
    const bool tk = (st.nxtU == -INFINITY) || (st.nxtU < theta);
    const bool sm = (st.T - Z <= a.lam) || (st.T == -INFINITY);
    bool ok;
    if (a.combine == CSV_COMBINE_ALL)
        ok = (tk || !a.use_k) && (sm || !a.use_s);
    else
        ok = (tk && a.use_k) || (sm && a.use_s);

    auto finish = [&](unsigned flags) {
        // the fused step kernel's parked blocks wait for this count: a finished sequence leaves nothing for them to
        // read, so they are told before the outputs are written rather than after
        if (settled_count && tid == 0) atomicAdd(settled_count, 1);
        for (int t = tid; t < a.k; t += nt) {
            a.out.d_ids[(size_t)b * a.k + t] = s.wid[t];
            a.out.d_logits[(size_t)b * a.k + t] = s.wval[t];
        }
        if (a.use_k) write_distribution(a, b, min(a.k, n), Z, s);
        if (a.out.d_sel_clusters)
            for (int j = tid; j < st.n_open; j += nt) a.out.d_sel_clusters[(size_t)b * C + j] = a.sel[(size_t)b * C + j];
        if (tid == 0) {
            a.out.d_lse[b] = Z;
            a.out.d_flags[b] = flags;
            a.out.d_n_rows[b] = n;
            a.out.d_n_clusters[b] = st.n_open;
            if (a.out.d_rounds) a.out.d_rounds[b] = round + 1;
            a.st[b].status = ST_DONE;
        }
    };
    if (ok) {
        finish(((tk && a.use_k) ? CSV_FLAG_TOPK_CERT : 0u) | ((sm && a.use_s) ? CSV_FLAG_SOFTMAX_CERT : 0u));
        return true;
    }
    if (round + 1 < a.max_rounds) {
        // ---- plan the next round: the open set grows from {key >= kappa0} to {key >= kappa1}
        __syncthreads();                                   // the staged logits are dead; the arena is reused
        const ClusterLds L = carve_clusters(arena, a.Npad, C);
        const u64 kappa0 = st.kappa;
        u64 kappa_a = kappa0, kappa_s = kappa0;
        if (a.use_k && !tk) kappa_a = (u64)lkey(theta) << 32;                 // every cluster with U_c >= theta
        bool intact = false;                               // the by-cluster data is in LDS
        if (a.use_s && !sm) {
            load_clusters(a, b, L);
            __syncthreads();
            bool hopeless = false;
            if (a.use_k && !tk && a.combine == CSV_COMBINE_ALL && a.delta_clusters == 0) {
                // when the top-k threshold alone opens more rows than allowed, the joint plan (a superset) does too:
                // the sorted prefix search for the softmax threshold would change nothing
                int r2 = 0;
                for_clusters<true, false>(C, L, [&](int, u64 kx, int m, float) { r2 += kx >= kappa_a && kx < kappa0 && kx != 0 ? m : 0; });
                hopeless = n + block_sum_i(r2, s.redi) > a.K_max;
            }
            if (!hopeless) {
                if constexpr (PLANS) kappa_s = softmax_prefix_fast(a, L, kappa0, Z, s);
                else kappa_s = softmax_prefix_key(a, L, kappa0, Z, s, [](u64) { return true; }, 0ull);
            }
            intact = true;
        }
        u64 kappa1;
        if (a.use_k && a.use_s)
            kappa1 = a.combine == CSV_COMBINE_ALL ? (kappa_a < kappa_s ? kappa_a : kappa_s) : (kappa_a > kappa_s ? kappa_a : kappa_s);
        else
            kappa1 = a.use_k ? kappa_a : kappa_s;
        if (!intact) {
            load_clusters(a, b, L);
            __syncthreads();
        }
        int cnt = 0, rows = 0;
        PlanSums ps;
        if constexpr (PLANS) {
            ps = plan_sweep(a, L, kappa0, kappa1, s);
            cnt = ps.cnt;
            rows = ps.rows;
        } else {
            for (int c = tid; c < C; c += nt) {
                const u64 kx = L.keys[c];
                if (kx >= kappa1 && kx < kappa0 && kx != 0) {
                    cnt += 1;
                    rows += L.offl[c + 1] - L.offl[c];
                }
            }
            cnt = block_sum_i(cnt, s.redi);
            rows = block_sum_i(rows, s.redi);
        }
        bool whole = true;                                 // the plan as swept, not a part of it
        bool expand = n + rows <= a.K_max;
        if (!expand) {
            if (tid == 0) {          // sizes of the plan that did not fit (reported if the sequence falls back)
                a.st[b].n_open = st.n_open + cnt;
                a.st[b].n_rows = n + rows;
            }
            // partial expansion: the next clusters of the bound order, at most delta_clusters of them, not past
            // the planned set, while the rows stay within the budget
            u64 kp = kappa0;
            int add = 0, radd = 0;
            for (int i = 0; i < a.delta_clusters; ++i) {
                u64 best = 0;
                for (int c = tid; c < C; c += nt) {
                    const u64 kx = L.keys[c];
                    if (kx < kp && kx > best) best = kx;
                }
                best = block_max_u64(best, s.redu);
                if (best == 0 || best < kappa1) break;
                const int cw = (int)(0xFFFFFFFFu - (uint32_t)best);
                const int nr = L.offl[cw + 1] - L.offl[cw];
                if (n + radd + nr > a.K_max) break;
                kp = best;
                add += 1;
                radd += nr;
            }
            if (add > 0) {
                kappa1 = kp;
                whole = false;
                cnt = add;
                rows = radd;
                expand = true;
            }
        }
        if (expand) {
            auto opens = [&](u64 kx) { return kx >= kappa1 && kx < kappa0 && kx != 0; };
            auto isnew = [&](int c) { return opens(L.keys[c]); };
            float nxtU, T1;
            if (PLANS && whole) tail_mass(a, L, kappa1, ps.best, ps.vmax, s, nxtU, T1);
            else tail_stats(a, L, kappa1, s, nxtU, T1);
            if (PLANS && cnt <= SEQ_THREADS) emit_list(a, b, round + 1, n, st.n_open, cnt, opens, L, s);
            else emit_clusters(a, b, round + 1, n, st.n_open, isnew, L, s);
            if (tid == 0) {
                SeqState o = st;
                o.n_open = st.n_open + cnt; o.n_rows = n + rows; o.rounds = round + 1; o.kappa = kappa1; o.nxtU = nxtU; o.T = T1;
                o.theta = (a.use_k && n >= a.k) ? theta : -INFINITY;
                a.st[b] = o;
            }
            return false;
        }
    }
    // ---- no further expansion: the relaxed tolerance, then the full vocabulary
    if (a.relax && a.use_s) {
        const bool sm2 = (st.T - Z <= a.lam2) || (st.T == -INFINITY);
        const bool ok2 = a.combine == CSV_COMBINE_ALL ? ((tk || !a.use_k) && sm2) : ((tk && a.use_k) || sm2);
        if (ok2) {
            finish(((tk && a.use_k) ? CSV_FLAG_TOPK_CERT : 0u) | (sm ? CSV_FLAG_SOFTMAX_CERT : (sm2 ? CSV_FLAG_SOFTMAX_RELAXED : 0u)));
            return true;
        }
    }
    if (tid == 0) push_fallback(a, b, round + 1);
    return false;
}

template <bool THRESH>
__device__ __forceinline__ void cert_device(const StepArgs& a, int b, int chunk, int round, SeqShared& s) {
    const SeqState st = a.st[b];
    cert_body<THRESH, THRESH>(a, b, chunk, round, st, s);
}

// ================================================================================================ round 0
// Grid (NB, B): the NB blocks of a sequence each derive the same seed prefix from the sequence's bounds (the
// prefix is a handful of clusters found by repeated block-wide arg-max over the keys, no sort), so no block
// waits for another to plan the work; they share the prefix rows wave by wave, and the block that arrives last at
// the sequence's counter (nobody waits) certifies, or plans round 1, or hands the sequence to the full product.
// A prefix with more rows than the NB blocks should score themselves (one giant cluster) goes to the round-0
// work list instead and is scored and certified by the tail kernel with the whole device.
#define ROUND0_ROWS_PER_BLOCK 4     // rows of the largest possible seed prefix per block (2..8 swept: 3-4 fastest; 8 costs 1 us)
#define ROUND0_NB_MAX 64           // most blocks of a sequence in the round-0 kernel (8..128 swept: 32-64 fastest)
#define ROUND0_ROWS_PER_WAVE 8     // with at most 32 blocks of 8 waves a sequence: no more than 2048 <= STAGE_CAP rows;
                                   // with a single block: 64 rows, larger prefixes go to the tail kernel
#define ROUND0_HREG 4     // 128-bit pieces of h a thread carries in registers across the seed (d <= 4 * 8 * SEQ_THREADS)
// log tail mass of the clusters below the threshold key kappa, shifted by an upper bound of its largest term
// (nxt: the largest unopened key, 0 if none; nxtU: its bound)
__device__ __forceinline__ float seed_tail_mass(const StepArgs& a, const ClusterLds& L, u64 kappa, u64 nxt, float nxtU, SeqShared& s) {
    if (!nxt) return -INFINITY;
    const float shift = a.ln_nmax + nxtU;
    float sum = 0.f;
    for (int c = threadIdx.x; c < a.C; c += blockDim.x) {
        const u64 kx = L.keys[c];
        if (kx != 0 && kx < kappa) sum += expf(L.vl[c] - shift);
    }
    sum = block_sum(sum, s.redf);
    return shift + logf(sum);
}
__device__ __forceinline__ SeqState seed_state(int m0, int rows, u64 kappa, float nxtU, float T0) {
    SeqState st;
    st.status = ST_ACTIVE; st.n_open = m0; st.n_rows = rows; st.rounds = 0; st.kappa = kappa; st.nxtU = nxtU; st.T = T0;
    st.fb_slot = -1; st.theta = -INFINITY; st.pad[0] = st.pad[1] = 0;
    return st;
}

// Seed selection for indexes of at most 64 * SEED_E clusters.  The block stages the sequence's bounds and ln n_c
// in LDS once (one barrier, shared with the staging of h); after that every wave works alone: lane l looks at
// clusters l, l + 64, ..., the wave takes the arg-max of the 64-bit keys and fetches the winner's packed metadata.
// Every wave of every block of the sequence gets the same answer.  When the best cluster alone holds max(k,1) rows
// (the common case: clusters larger than k) it is the whole seed prefix; the wave requests its row and only then
// takes, from the same registers, the next bound and the log tail mass of everything else, while the row is in
// flight.  Otherwise the caller falls through to the general selection.
#define SEED_E 16
struct WaveSeed {
    int c, row0, rows;
    u64 kappa;
    float u[SEED_E], l[SEED_E];     // bounds and ln n of the lane's clusters (-inf: empty or out of range)
};
// sU, sL, sR: LDS copies of U[b,:], of ln n_c and of {first row, rows} per cluster.  All LDS reads are issued from
// clamped indexes before anything is compared (a conditional read would put every read in a basic block of its own,
// one LDS round trip after the other).
__device__ __forceinline__ void wave_seed_pick(const StepArgs& a, const float* sU, const float* sL, const int2* sR, WaveSeed& r) {
    const int lane = threadIdx.x & 63, C = a.C;
#pragma unroll
    for (int i = 0; i < SEED_E; ++i) {
        const int cc = min(lane + 64 * i, C - 1);
        r.u[i] = sU[cc];
        r.l[i] = sL[cc];
    }
    // 32-bit keys: the largest bound first, then the smallest cluster id among its holders (the order of the 64-bit keys)
    unsigned bk = 0;
    int bc = 0x7fffffff;
#pragma unroll
    for (int i = 0; i < SEED_E; ++i) {
        const int c = lane + 64 * i;
        const bool some = c < C && r.l[i] > -INFINITY;
        r.u[i] = some ? r.u[i] : -INFINITY;
        r.l[i] = some ? r.l[i] : -INFINITY;
        const unsigned kx = some ? lkey(r.u[i]) : 0u;      // lkey is never 0 for a bound that is not NaN
        const bool better = kx > bk;                       // c grows with i: a tie keeps the smaller id
        bk = better ? kx : bk;
        bc = better ? c : bc;
    }
    const unsigned top = wave_max_u(bk);
    const int cw = wave_min_i((bk == top && top != 0u) ? bc : 0x7fffffff);
    r.kappa = 0;
    r.c = 0;
    r.row0 = 0;
    r.rows = 0;
    if (top != 0u) {
        const int2 rr = sR[cw];
        r.c = cw;
        r.row0 = rr.x;
        r.rows = rr.y;
        r.kappa = ((u64)top << 32) | (u64)(0xFFFFFFFFu - (uint32_t)cw);
    }
}
// next bound and log tail mass with cluster r.c open and everything else unopened
__device__ __forceinline__ void wave_seed_tail(const StepArgs& a, const WaveSeed& r, float& nxtU, float& T0) {
    const int lane = threadIdx.x & 63;
    float mx = -INFINITY;
    float v[SEED_E];
#pragma unroll
    for (int i = 0; i < SEED_E; ++i) {
        const bool rest = (lane + 64 * i) != r.c;          // empty and out-of-range clusters already carry -inf
        v[i] = rest ? r.l[i] + r.u[i] : -INFINITY;
        mx = fmaxf(mx, rest ? r.u[i] : -INFINITY);
    }
    mx = wave_max(mx + 0.0f);
    nxtU = mx;
    T0 = -INFINITY;
    if (mx == -INFINITY) return;                              // the prefix is the whole vocabulary
    const float shift = a.ln_nmax + nxtU;
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < SEED_E; ++i) sum += expf(v[i] - shift);     // exp(-inf) = 0
    sum = wave_sum(sum);
    T0 = shift + logf(sum);
}

// One sequence's round 0 as seen by block j of its NB blocks.  Returns nonzero in the one block that settled the
// sequence: 1 when the sequence is finished (certified, or flagged invalid), 2 when it left work for later phases
// (a planned round, a hand-over, a fallback) or gave up.
// settled_count: where a sequence that finishes here is counted as soon as that is decided (the return value is then 3).
template <bool THRESH, bool PLANS>
__device__ __forceinline__ int round0_device(const StepArgs& a, int b, int j, int NB, SeqShared& s, int* settled_count = nullptr) {
    extern __shared__ __align__(16) u64 arena[];
    const int tid = threadIdx.x, nt = SEQ_THREADS, lane = tid & 63, wave = tid >> 6, C = a.C;
    const int nch = a.d >> 3;
    const ClusterLds L = carve_clusters(arena, a.Npad, C);
    // h is requested now and parked in registers: it moves to LDS once the cluster data there is dead
    uint4 hreg[ROUND0_HREG];
    {
        const uint4* hsrc = reinterpret_cast<const uint4*>(a.h) + (size_t)b * nch;
#pragma unroll
        for (int q = 0; q < ROUND0_HREG; ++q) {
            const int i = tid + q * nt;
            hreg[q] = i < nch ? hsrc[i] : make_uint4(0, 0, 0, 0);
        }
    }
    const float hn = a.hnorm[b];
    if (j == 0 && tid == 0) a.out.d_flags[b] = CSV_FLAG_ABORTED;   // pending: overwritten by whichever path finishes the sequence
    const int need = max(a.k, 1);
    const int GW = NB * (nt >> 6);
    const int cap_rows = min(GW * ROUND0_ROWS_PER_WAVE, STAGE_CAP);
    int* scl = s.wid;
    int* spos = reinterpret_cast<int*>(s.wval);
    int rows = 0, m0 = 0;
    u64 kappa = ~0ull, nxt = 0;
    float nxtU, T0;
    uint4* hs4 = reinterpret_cast<uint4*>(arena) + a.r0_h_off;
    u64* slots = a.slots + (size_t)b * CSV_SLOT_ROWS;
    uint4 pf[TILE_PF];
    const uint4* w = nullptr;
    float bias = 0.f;
    int id = 0;
    auto request_row = [&](int r) {       // unconditional loads from clamped addresses, then a select: no branches
        w = reinterpret_cast<const uint4*>(a.Wp + (size_t)r * a.d);
#pragma unroll
        for (int q = 0; q < TILE_PF; ++q) {
            const int i = lane + 64 * q;
            const uint4 v = w[min(i, nch - 1)];
            pf[q] = i < nch ? v : make_uint4(0, 0, 0, 0);
        }
        bias = a.bp[r];                   // every lane the same address: one transaction
        id = a.perm[r];
    };
    int p = wave * NB + j;   // neighbouring rows go to different compute units
    bool fast = false;
    WaveSeed ws;
    ws.row0 = 0;
    if (C <= 64 * SEED_E && nch <= ROUND0_HREG * nt) {
        // bounds, ln n and h to LDS with one barrier; then every wave picks the seed cluster by itself
        float* sU = reinterpret_cast<float*>(arena);
        float* sL = sU + C;
        int2* sR = reinterpret_cast<int2*>(sL + C + (C & 1));
        {
            const float* Ub = a.U + (size_t)b * C;
            float ru[2];
            int4 rm[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int cc = min(tid + q * nt, C - 1);
                ru[q] = Ub[cc];
                rm[q] = a.cmeta[cc];
            }
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int c = tid + q * nt;
                if (c < C) {
                    sU[c] = ru[q];
                    sL[c] = __int_as_float(rm[q].z);
                    sR[c] = make_int2(rm[q].x, rm[q].y);
                }
            }
#pragma unroll
            for (int q = 0; q < ROUND0_HREG; ++q) {
                const int i = tid + q * nt;
                if (i < nch) hs4[i] = hreg[q];
            }
        }
        __syncthreads();
        if (!isfinite(hn)) {
            if (j == 0) write_invalid(a, b);
            return j == 0 ? 1 : 0;
        }
        wave_seed_pick(a, sU, sL, sR, ws);
        fast = ws.kappa != 0 && ws.rows >= need && ws.rows <= cap_rows && ws.rows <= a.K_max;
        if (!fast) __syncthreads();          // every wave has read the staged bounds: the general path reuses the LDS
    }
    if (fast) {
        // the prefix is one cluster: the row first, then the next bound and the tail mass while it is in flight
        m0 = 1; rows = ws.rows; kappa = ws.kappa;
        if (p < rows) request_row(ws.row0 + p);
        if (j == 0 && tid == 0) a.sel[(size_t)b * C] = ws.c;
        nxtU = -INFINITY;        // the next bound and the tail mass are needed by the certifying block only: taken after its rows
        T0 = -INFINITY;
    } else {
        load_clusters(a, b, L);
        if (!isfinite(hn)) {
            if (j == 0) write_invalid(a, b);
            return j == 0 ? 1 : 0;
        }
        __syncthreads();
        // Open clusters one at a time by block-wide arg-max until max(k,1) rows are open.  Every opened cluster has
        // at least one row, so at most max(k,1) <= CSV_MAX_K clusters open: their ids and positions fit the k-sized
        // arrays.  Nothing is written to global memory inside the loop (a store would be waited for at the next barrier).
        while (true) {
            // the best unopened cluster and the one after it, in one reduction: when the best completes the prefix,
            // the runner-up is already the next unopened bound
            Top2 t2{0ull, 0ull};
            for (int c = tid; c < C; c += nt) {
                const u64 kx = L.keys[c];
                if (kx < kappa) t2 = top2_push(t2, kx);
            }
            t2 = block_top2(t2, s.redu);
            if (t2.a == 0) {                   // nothing left to open
                nxt = 0;
                break;
            }
            const int cw = (int)(0xFFFFFFFFu - (uint32_t)t2.a);
            if (tid == 0) {
                scl[m0] = cw;
                spos[m0] = rows;
            }
            rows += L.offl[cw + 1] - L.offl[cw];
            m0 += 1;
            kappa = t2.a;
            if (rows >= need) {
                nxt = t2.b;
                break;
            }
        }
        if (rows > a.K_max) {
            if (j == 0 && tid == 0) {
                a.st[b].n_open = m0;
                a.st[b].n_rows = rows;
                push_fallback(a, b, 0);
            }
            return j == 0 ? 2 : 0;
        }
        __syncthreads();   // scl / spos complete
        if (j == 0)
            for (int i = tid; i < m0; i += nt) a.sel[(size_t)b * C + i] = scl[i];
        nxtU = nxt ? ckey_bound(nxt) : -INFINITY;
        if (rows > cap_rows || nch > ROUND0_HREG * nt) {
            // too much for these blocks: the first block queues the prefix for the tail
            if (j != 0) return 0;
            T0 = seed_tail_mass(a, L, kappa, nxt, nxtU, s);
            Tile* tl = a.tiles[0] + (size_t)b * a.tile_stride;
            int ntile = 0;
            for (int i = 0; i < m0; ++i) {
                const int r0 = L.offl[scl[i]], p0 = spos[i], n = (i + 1 < m0 ? spos[i + 1] : rows) - p0;
                const int ntc = (n + TILE_ROWS - 1) / TILE_ROWS;
                for (int t = tid; t < ntc; t += nt) {
                    Tile x;
                    x.b = b; x.row0 = r0 + t * TILE_ROWS; x.nrows = min(TILE_ROWS, n - t * TILE_ROWS); x.pos = p0 + t * TILE_ROWS;
                    tl[ntile + t] = x;
                }
                ntile += ntc;
            }
            if (tid == 0) {
                a.counters[CNT_TILES + b] = ntile;
                __hip_atomic_store(&a.counters[CNT_TAIL_NEEDED], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                a.st[b] = seed_state(m0, rows, kappa, nxtU, T0);
            }
            return 2;
        }
        // h goes to its own LDS region behind the cluster data; the wave's first row is requested before the tail
        // mass is summed, so that sum runs while the loads are in flight
#pragma unroll
        for (int q = 0; q < ROUND0_HREG; ++q) {
            const int i = tid + q * nt;
            if (i < nch) hs4[i] = hreg[q];
        }
    }
    auto row_of = [&](int pp) {
        if (fast) return ws.row0 + pp;
        int lo = 0, hi = m0;   // largest i with spos[i] <= pp
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (spos[mid] <= pp) lo = mid; else hi = mid;
        }
        return L.offl[scl[lo]] + (pp - spos[lo]);
    };
    if (!fast) {
        if (p < rows) request_row(row_of(p));
        __syncthreads();                   // h staged (the fast path staged it before its barrier)
    }
    while (p < rows) {
        float acc = 0.f, acc2 = 0.f;          // two chains: a dependent FMA costs two issue slots of a lone wave
#pragma unroll
        for (int q = 0; q < TILE_PF; q += 2) {     // pieces past the row are zero and h is finite: no branch needed
            const int i = lane + 64 * q;
            acc = dot8_bf16(pf[q], hs4[min(i, nch - 1)], acc);
            acc2 = dot8_bf16(pf[q + 1], hs4[min(i + 64, nch - 1)], acc2);
        }
        acc += acc2;
        int i = lane + 64 * TILE_PF;
        for (; i + 192 < nch; i += 256) {
            const uint4 x0 = w[i], x1 = w[i + 64], x2 = w[i + 128], x3 = w[i + 192];
            acc = dot8_bf16(x0, hs4[i], acc);
            acc = dot8_bf16(x1, hs4[i + 64], acc);
            acc = dot8_bf16(x2, hs4[i + 128], acc);
            acc = dot8_bf16(x3, hs4[i + 192], acc);
        }
        for (; i < nch; i += 64) acc = dot8_bf16(w[i], hs4[i], acc);
        acc = wave_sum(acc);
        if (lane == 0)      // one word carries the row's token id and logit: whoever reads it gets both or neither
            __hip_atomic_store(&slots[p], ((u64)(uint32_t)id << 32) | (u64)__float_as_uint(acc + bias), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        p += GW;
        if (p < rows) request_row(row_of(p));
    }
    // Block 0 of the sequence collects: each of its threads waits for its rows' words (no counter, no fence: a word
    // is either still empty or complete), puts the logit and the id where the certification expects its staged
    // input, copies them to the row arrays that later rounds read, and empties the word for the next step.  All NB
    // blocks of a sequence are resident together (the host sizes the grid so), and the wait is bounded.
    if (j != 0) return 0;
    // the tail mass, which only this block needs, while the other blocks' words are on their way (the cluster data
    // in LDS is still whole: h sits behind it)
    if (fast) wave_seed_tail(a, ws, nxtU, T0);
    else T0 = seed_tail_mass(a, L, kappa, nxt, nxtU, s);
    const SeqState st = seed_state(m0, rows, kappa, nxtU, T0);
    __syncthreads();                       // every wave is done with h in LDS: the staging area overlaps it
    float* sv = reinterpret_cast<float*>(arena);
    int* si = reinterpret_cast<int*>(arena) + STAGE_CAP;
    int gave_up = 0;
    for (int t = tid; t < rows; t += nt) {
        u64 v;
        int spins = 0;
        while ((v = __hip_atomic_load(&slots[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == CSV_SLOT_EMPTY) {
            if (++spins > a.spin_limit) {
                gave_up = 1;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        if (gave_up) break;
        __hip_atomic_store(&slots[t], CSV_SLOT_EMPTY, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const float lv = __uint_as_float((uint32_t)v);
        const int iv = (int)(uint32_t)(v >> 32);
        sv[t] = lv;
        si[t] = iv;
        a.slog[(size_t)b * a.K_cap + t] = lv;
        a.sid[(size_t)b * a.K_cap + t] = iv;
    }
    if (tid < 4 && rows + tid < STAGE_CAP) sv[rows + tid] = -INFINITY;     // the certification reads the values four at a time
    if (__syncthreads_or(gave_up)) {
        // a row never arrived: the step is given up for this sequence (flag ABORTED stays); words may still arrive
        // later, so the next step has to empty the slots before it uses them
        if (tid == 0) {
            atomicExch(&a.counters[CNT_ABORT], 1);
            __hip_atomic_store(&a.counters[CNT_SLOTS_DIRTY], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        return 2;
    }
    return cert_body<THRESH, PLANS>(a, b, 0, 0, st, s, true, settled_count) ? (settled_count ? 3 : 1) : 2;     // every path of it that leaves work behind writes the state it needs
}

// ================================================================================================ Algorithm 1's own order
// One cluster per iteration, the tests after every opening: the shortest certifying prefix of the bound order
// (Algorithm 1, Section III-C).  A reference mode, not the fast path: one block per sequence does everything itself, so
// an iteration is a block-wide arg-max, the rows of one cluster (a row per wave at a time) and a top-k update, with
// no dependency between blocks.  Dynamic LDS: staged values and ids with the candidates behind them (as the
// certification lays them out), then the sequence's cluster data, then h.
#define ALG1_PIECE 2048            // rows of a cluster scored between two updates of the list (a piece plus the list fit the staging area)
#define ALG1_CL_OFF (CAND_OFF + CAND_BYTES + 16)      // bytes; a multiple of 16
static_assert(ALG1_PIECE + CSV_MAX_K <= STAGE_CAP && ALG1_CL_OFF % 16 == 0, "Algorithm-1 mode: staging layout");
__global__ __launch_bounds__(SEQ_THREADS) void alg1_kernel(StepArgs a, int h_off16) {
    extern __shared__ __align__(16) u64 arena[];
    __shared__ SeqShared s;
    const int b = blockIdx.x, tid = threadIdx.x, nt = SEQ_THREADS, lane = tid & 63, wave = tid >> 6, C = a.C;
    const int nch = a.d >> 3;
    float* sv = reinterpret_cast<float*>(arena);
    int* si = reinterpret_cast<int*>(arena) + STAGE_CAP;
    const ClusterLds L = carve_clusters(reinterpret_cast<u64*>(reinterpret_cast<char*>(arena) + ALG1_CL_OFF), a.Npad, C);
    uint4* hs4 = reinterpret_cast<uint4*>(arena) + h_off16;
    auto val = [](int i) { return reinterpret_cast<const float*>(arena)[i]; };
    auto idf = [](int i) { return reinterpret_cast<const int*>(arena)[STAGE_CAP + i]; };
    const float hn = a.hnorm[b];
    if (!isfinite(hn)) {
        write_invalid(a, b);
        return;
    }
    load_clusters(a, b, L);
    for (int i = tid; i < nch; i += nt) hs4[i] = (reinterpret_cast<const uint4*>(a.h) + (size_t)b * nch)[i];
    __syncthreads();
    u64 kappa = ~0ull;
    int rows = 0, m = 0, kcur = 0;         // rows scored, clusters open, entries of the list in s.wval / s.wid
    LseAcc run;
    run.m = -INFINITY;
    run.s = 0.f;
    while (true) {
        // ---- both tests on the open prefix (m = 0: nothing scored, only "no cluster at all" certifies)
        float nxtU, T;
        tail_stats(a, L, kappa, s, nxtU, T);
        __syncthreads();
        const float Z = lse_value(run);
        const float theta = (a.use_k && kcur >= a.k) ? s.wval[a.k - 1] : -INFINITY;
        const bool none_left = nxtU == -INFINITY;
        const bool tk = none_left || (kcur >= a.k && nxtU < theta);
        const bool sm = none_left || (rows > 0 && T - Z <= a.lam);
        const bool tk_ok = a.use_k ? tk : (a.combine == CSV_COMBINE_ALL);
        const bool sm_ok = a.use_s ? sm : (a.combine == CSV_COMBINE_ALL);
        const bool ok = a.combine == CSV_COMBINE_ALL ? (tk_ok && sm_ok) : (tk_ok || sm_ok);
        if (ok) {
            for (int t = tid; t < a.k; t += nt) {
                a.out.d_ids[(size_t)b * a.k + t] = t < kcur ? s.wid[t] : -1;
                a.out.d_logits[(size_t)b * a.k + t] = t < kcur ? s.wval[t] : -INFINITY;
            }
            if (a.use_k) write_distribution(a, b, kcur, Z, s);
            if (tid == 0) {
                a.out.d_lse[b] = Z;
                a.out.d_flags[b] = ((tk && a.use_k) ? CSV_FLAG_TOPK_CERT : 0u) | ((sm && a.use_s) ? CSV_FLAG_SOFTMAX_CERT : 0u);
                a.out.d_n_rows[b] = rows;
                a.out.d_n_clusters[b] = m;
                if (a.out.d_rounds) a.out.d_rounds[b] = m;
                a.st[b].status = ST_DONE;
            }
            if (a.out.d_sel_clusters)
                for (int j = tid; j < m; j += nt)       // written by thread 0 of this block: read past the first-level cache
                    a.out.d_sel_clusters[(size_t)b * C + j] = __hip_atomic_load(&a.sel[(size_t)b * C + j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
        // ---- open the next cluster of the bound order; the budget is tested before its rows are scored
        u64 best = 0;
        for (int c = tid; c < C; c += nt) {
            const u64 kx = L.keys[c];
            if (kx < kappa && kx > best) best = kx;
        }
        best = block_max_u64(best, s.redu);
        const int cw = (int)(0xFFFFFFFFu - (uint32_t)best);       // best != 0: some cluster is unopened, or the tests had held
        const int r0 = L.offl[cw], nc = L.offl[cw + 1] - r0;
        if (rows + nc > a.K_max) {
            if (tid == 0) {
                a.st[b].n_open = m + 1;
                a.st[b].n_rows = rows + nc;
                push_fallback(a, b, m + 1);
            }
            return;
        }
        if (tid == 0) a.sel[(size_t)b * C + m] = cw;
        kappa = best;
        m += 1;
        for (int p0 = 0; p0 < nc; p0 += ALG1_PIECE) {
            const int P = min(ALG1_PIECE, nc - p0);
            __syncthreads();                                  // the staging area is free
            // two rows per wave at a time, a whole row (up to TILE_PF pieces per lane) requested before anything is added up
            for (int p = 2 * wave; p < P; p += 2 * (nt >> 6)) {
                uint4 pf[2][TILE_PF];
                const uint4* w[2];
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    w[q] = reinterpret_cast<const uint4*>(a.Wp + (size_t)(r0 + p0 + min(p + q, P - 1)) * a.d);
#pragma unroll
                    for (int j = 0; j < TILE_PF; ++j) pf[q][j] = w[q][min(lane + 64 * j, nch - 1)];
                }
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    float acc = 0.f;
#pragma unroll
                    for (int j = 0; j < TILE_PF; ++j) {
                        const int i = lane + 64 * j;
                        if (i < nch) acc = dot8_bf16(pf[q][j], hs4[i], acc);
                    }
                    for (int i = lane + 64 * TILE_PF; i < nch; i += 64) acc = dot8_bf16(w[q][i], hs4[i], acc);
                    acc = wave_sum(acc);
                    if (lane == 0 && p + q < P) {
                        const int r = r0 + p0 + p + q;
                        sv[p + q] = acc + a.bp[r];
                        si[p + q] = a.perm[r];
                    }
                }
            }
            __syncthreads();
            // log-sum-exp of the piece joins the running one; the list joins the piece and the top k of both is the new list
            const LseAcc lp = block_lse(P, val, s);
            run = lse_combine(run, lp);
            __syncthreads();
            for (int t = tid; t < kcur; t += nt) {
                sv[P + t] = s.wval[t];
                si[P + t] = s.wid[t];
            }
            const int ntot = P + kcur;
            if (tid < 4 && ntot + tid < STAGE_CAP) sv[ntot + tid] = -INFINITY;
            __syncthreads();
            if (a.use_k) {
                const int knew = min(a.k, ntot);
                bool done = false;
                if (ntot <= RANK_DIRECT) {
                    float v;
                    rank_small(sv, si, ntot, knew, s, v);
                    done = true;
                } else {
                    int kk = 0;
                    float vmax;
                    done = threshold_topk(ntot, a.k, kcur >= a.k ? s.wval[a.k - 1] : -INFINITY, false, idf, s, kk, vmax);
                }
                __syncthreads();
                if (!done) block_topk(ntot, a.k, val, idf, s);
                kcur = knew;
            }
            rows += P;
        }
        __syncthreads();
    }
}

// ================================================================================================ full-vocabulary product
struct FullArgs {
    int V, d;
    const uint16_t* Wp;
    const float* bp;
    const int32_t* perm;
    const uint16_t* h;
    const int32_t* list;    // sequences to score
    int n_fixed;            // their number (the fallback products pass their own, counted on the device)
    float* out;             // [slot*out_stride + row*row_stride]
    long long out_stride;
    int row_stride;         // 1, or (MFMA product) the number of sequences with out_stride = 1: a row's logits side by side
    int scatter;            // 1: write at the original token id instead of the permuted row
};

// Vector path: NG <= FULL_G sequences (g0 ...) in one pass over W', their h in LDS, two rows per wave at a time and PF pieces of
// each requested together, of what is left two, then one.
template <int NG, int PF>
__device__ __forceinline__ void full_gemv_pass(const FullArgs& f, int g0, uint4* hs4, int block, int nblocks) {
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wave = tid >> 6;
    const int nch = f.d >> 3;
    const int rpt = (nt >> 6) * 2;                 // rows per tile: two per wave
    const int ntiles = (f.V + rpt - 1) / rpt;
    __syncthreads();
    for (int i = tid; i < NG * nch; i += nt) {
        const int s = NG == 1 ? 0 : i / nch, j = i - s * nch;
        hs4[i] = (reinterpret_cast<const uint4*>(f.h) + (size_t)f.list[g0 + s] * nch)[j];
    }
    __syncthreads();
    for (int tile = block; tile < ntiles; tile += nblocks) {
        const int r0 = tile * rpt + wave * 2;
        if (r0 >= f.V) continue;
        const bool two = r0 + 1 < f.V;
        const int r1 = two ? r0 + 1 : r0;
        const uint4* w0 = reinterpret_cast<const uint4*>(f.Wp + (size_t)r0 * f.d);
        const uint4* w1 = reinterpret_cast<const uint4*>(f.Wp + (size_t)r1 * f.d);
        float acc0[NG], acc1[NG];
#pragma unroll
        for (int s = 0; s < NG; ++s) acc0[s] = acc1[s] = 0.f;
        auto add = [&](const uint4& a, const uint4& c, int i) {
#pragma unroll
            for (int s = 0; s < NG; ++s) {
                const uint4 h = hs4[s * nch + i];
                acc0[s] = dot8_bf16(a, h, acc0[s]);
                acc1[s] = dot8_bf16(c, h, acc1[s]);
            }
        };
        int i = lane;
        auto trip = [&](auto pieces_t) {
            constexpr int N = decltype(pieces_t)::value;
            uint4 a[N], c[N];
#pragma unroll
            for (int q = 0; q < N; ++q) a[q] = w0[i + 64 * q];
#pragma unroll
            for (int q = 0; q < N; ++q) c[q] = w1[i + 64 * q];
#pragma unroll
            for (int q = 0; q < N; ++q) add(a[q], c[q], i + 64 * q);
            i += 64 * N;
        };
        while (i + 64 * (PF - 1) < nch) trip(std::integral_constant<int, PF>{});
        if (PF > 2 && i + 64 < nch) trip(std::integral_constant<int, 2>{});
        while (i < nch) trip(std::integral_constant<int, 1>{});
#pragma unroll
        for (int s = 0; s < NG; ++s) {
            const float v0 = wave_sum(acc0[s]), v1 = wave_sum(acc1[s]);
            if (lane == 0) {
                float* dst = f.out + (size_t)(g0 + s) * f.out_stride;
                dst[f.scatter ? f.perm[r0] : r0] = v0 + f.bp[r0];
                if (two) dst[f.scatter ? f.perm[r1] : r1] = v1 + f.bp[r1];
            }
        }
    }
}
template <int PF = 4>
__device__ __forceinline__ void full_gemv_device(const FullArgs& f, int n, uint4* hs4, int block, int nblocks) {
    for (int g0 = 0; g0 < n; g0 += FULL_G) {
        switch (min(FULL_G, n - g0)) {
            case 1: full_gemv_pass<1, PF>(f, g0, hs4, block, nblocks); break;
            case 2: full_gemv_pass<2, PF>(f, g0, hs4, block, nblocks); break;
            case 3: full_gemv_pass<3, PF>(f, g0, hs4, block, nblocks); break;
            default: full_gemv_pass<4, PF>(f, g0, hs4, block, nblocks); break;
        }
    }
}

// Dense logits of up to FULL_G sequences.  PF: 4 where a row has that many pieces per lane (d >= 2048), 2 for shorter rows, which never
// fill a trip of four: the registers then allow eight waves per SIMD, which hide what fewer requests per wave leave open
// (us with four pieces and four waves / two and five / two and eight: V = 24000, d = 768, one sequence 9.5 / 8.9 / 7.4, four 16.2 /
// 15.0 / 12.0; V = 128256, d = 1536, four 103 / 102 / 81.  V = 32000, d = 4096, one 39.4 / 43.7 with two pieces).
template <int PF>
__global__ __launch_bounds__(256, PF == 2 ? 8 : 4) void full_gemv_kernel(FullArgs f) {
    extern __shared__ uint4 hs4[];
    full_gemv_device<PF>(f, f.n_fixed, hs4, blockIdx.x, gridDim.x);
}

// MFMA path of the full-vocabulary product, used when more than FULL_G sequences share the pass over W' (then it
// is a real dense contraction: [V x d] . [d x n]).  v_mfma_f32_16x16x32_bf16.  A block of eight waves owns
// 128 TW consecutive rows of W' at a time, a wave 16 TW of them (TW row tiles) for 16 NT sequences, and keeps the
// logits of its tiles in accumulator registers over the whole of K: every logit is written once.
//   h  (shared by all waves) moves through LDS in chunks of one to four K blocks of 128, already in fragment order
//      (the 64 lanes of a fragment read 1 KB contiguously: no bank conflicts), double-buffered: while a chunk is
//      consumed the next one is fetched into registers and stored to the other buffer; one barrier per chunk, which
//      waits for LDS traffic only, so the W' loads in flight cross it.  A fragment read from LDS serves TW MFMAs.
//   W' goes straight from global memory to registers: lane (li = lane%16, g = lane/16) feeds row li of a tile and, for
//      the jj-th MFMA of a K block, the eight k values at  128 block + 32 jj + 8 g.  A wave always has a chunk's worth
//      of K blocks requested ahead (register buffer kb is refilled for the next chunk as soon as its MFMAs are
//      issued): 8 to 32 KB per wave in flight at any time, in 256-byte runs per row.
// h is fed as the first operand and W' as the second, so accumulator register r of lane (li, g) is
// out[sequence 4g + r][row li]: stores are 64-byte runs per sequence instead of 4-byte pieces 4V bytes apart.
#define MFMA_THREADS 512
// Order of K.  In step, all the blocks' rows ask for the same columns at the same time, and with rows of a multiple of
// 4 KB those sit behind few of the memory channels.  There K is cut into 2^levels parts, which a group of rows takes in the order
// p ^ rot, rot its own; the parts' sums are added as a binary tree, ((0 + 1) + (2 + 3)) + ..., each pair in either order, so a row's logit
// has the same bits whatever its group, the grid and the launch form: equal rows get equal logits, and none depends on
// how the step was launched.  (rot by both the group and its octet: groups are dealt round-robin to the eight XCDs,
// and each of those then has all parts in flight.)  V = 128256, us for one order / with parts: 8 sequences, d = 2048 120 / 99,
// 4096 243 / 188, 6144 325 / 283, 8192 371 / 365; 64 sequences at d = 8192 412 / 390.  Eight parts rather than four at
// d = 8192: the same there, but not up to 10 % more where W' comes to lie less well (8 sequences 365 in each of five places, with
// four parts 353-390); at d = 4096 four are 1-3 % faster.  Other lengths spread by themselves: d = 4608 (V = 256000) 410 without /
// 420 with, 5120 (V = 151552) 299 / 304, 3072 and 7168 no difference.
__host__ __device__ __forceinline__ int full_k_levels(int d) { return d % 8192 == 0 ? 3 : (d % 2048 == 0 ? 2 : 0); }
// Dynamic LDS: two buffers of K blocks x 4 fragments x 1 KB x groups of 16 sequences, at most 2 x 4; where K is cut also the
// sums of the last level, 128 bytes a thread
__host__ __device__ constexpr int mfma_lds(int levels) { return levels > 0 ? 128 * 1024 : 64 * 1024; }
// LEVELS: at least the full_k_levels of d
template <int NT, int TW, int MFMA_PIPE, int LEVELS>
__device__ __forceinline__ void full_mfma_device(const FullArgs& f, int n, int seq0, uint4* lds, int block, int nblocks) {
    constexpr int NW = MFMA_THREADS / 64;
    constexpr int CH = MFMA_PIPE * 4 * NT * 64;       // 16-byte pieces per LDS buffer
    constexpr int SPT = CH / MFMA_THREADS;            // pieces a thread stages per chunk
    static_assert(CH % MFMA_THREADS == 0 && NW % NT == 0 && 2 * CH * 16 + (LEVELS > 0 ? TW * NT * MFMA_THREADS * 16 : 0) <= mfma_lds(LEVELS), "staging layout");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int li = lane & 15, g = lane >> 4;
    const int ntiles = (f.V + 15) >> 4;
    const int nq = f.d >> 3;                          // 16-byte pieces per row
    const int nsb = (f.d + 127) >> 7;                 // K blocks of 128
    const int nchunk = (nsb + MFMA_PIPE - 1) / MFMA_PIPE;
    const int ngroups = (ntiles + NW * TW - 1) / (NW * TW);
    // Staging: piece p = tid + 512 s of a buffer is lane p % 64 = lane of fragment p / 64 = (4 kb + jj) NT + t.  NT divides
    // the eight waves, so t, and with it the sequence 16 t + li, is the same for every piece a thread stages.
    const int st_sq = seq0 + (wave % NT) * 16 + li;
    const bool st_on = st_sq < n;
    const uint4* st_h = reinterpret_cast<const uint4*>(f.h) + (size_t)f.list[st_on ? st_sq : seq0] * nq;
    for (int grp = block; grp < ngroups; grp += nblocks) {
        const int tile0 = (grp * NW + wave) * TW;
        const uint4* ap[TW];
#pragma unroll
        for (int tw = 0; tw < TW; ++tw) ap[tw] = reinterpret_cast<const uint4*>(f.Wp + (size_t)min((tile0 + tw) * 16 + li, f.V - 1) * f.d);
        floatx4_t acc[TW][NT];
#pragma unroll
        for (int tw = 0; tw < TW; ++tw)
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[tw][t] = floatx4_t{0.f, 0.f, 0.f, 0.f};
        uint4 A[MFMA_PIPE][TW][4];
        uint4 sreg[SPT];
        // Nothing is done to a loaded value before its MFMA or its LDS store: an instruction on it would be waited for
        // where it stands, right behind the load.  Past the end of a row W' is read from a clamped address (the row's
        // own last piece) and meets zeros staged for h there; the zeros are selected when the piece is stored.
        auto load_A = [&](int kb, int sb) {           // K block sb of the wave's rows
#pragma unroll
            for (int tw = 0; tw < TW; ++tw)
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) A[kb][tw][jj] = ap[tw][min(sb * 16 + jj * 4 + g, nq - 1)];
        };
        const int levels = LEVELS == 0 ? 0 : full_k_levels(f.d), rot = (grp + (grp >> 3)) & ((1 << levels) - 1);
        auto part_at = [&](int q) { return (q * nchunk) >> levels; };        // first chunk of part q (d >= 2048: no part is empty)
        int part = 0, cur_c = part_at(rot), next_c = 0;                      // parts done, the chunk in use, the one after it
        floatx4_t held[LEVELS > 1 ? LEVELS - 1 : 1][TW][NT];                 // the levels but the last, which lies in LDS
        floatx4_t* park = reinterpret_cast<floatx4_t*>(lds + 2 * CH) + tid;
        // behind part i: acc joins the sum held on every level that is full, and is held on the first that is not
        auto fold = [&](int i) {
            bool carry = true;
#pragma unroll
            for (int l = 0; l < LEVELS; ++l) {
                if (l >= levels || !carry) continue;
                carry = (i >> l) & 1;
#pragma unroll
                for (int tw = 0; tw < TW; ++tw)
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        floatx4_t& h = l < LEVELS - 1 ? held[l < LEVELS - 1 ? l : 0][tw][t] : park[(tw * NT + t) * MFMA_THREADS];
                        if (carry) {
                            acc[tw][t] = acc[tw][t] + h;
                        } else {
                            h = acc[tw][t];
                            acc[tw][t] = floatx4_t{0.f, 0.f, 0.f, 0.f};
                        }
                    }
            }
        };
        auto stage_q = [&](int c, int s) {
            const int kbjj = wave / NT + (NW / NT) * s;
            return (c * MFMA_PIPE + (kbjj >> 2)) * 16 + (kbjj & 3) * 4 + g;
        };
        auto stage_load = [&](int c) {
#pragma unroll
            for (int s = 0; s < SPT; ++s) sreg[s] = st_h[min(stage_q(c, s), nq - 1)];
        };
        auto stage_store = [&](uint4* buf, int c) {
#pragma unroll
            for (int s = 0; s < SPT; ++s) buf[tid + MFMA_THREADS * s] = keep_if(st_on && stage_q(c, s) < nq, sreg[s]);
        };
        stage_load(cur_c);
#pragma unroll
        for (int kb = 0; kb < MFMA_PIPE; ++kb) load_A(kb, cur_c * MFMA_PIPE + kb);
        stage_store(lds, cur_c);
        lds_barrier();
        // The last chunk is a copy of the loop body without the requests for a next one: with the requests under a
        // condition the compiler could not count, at compile time, how many younger loads a wait may leave open.
        auto chunk = [&](auto more_t, int c) {
            constexpr bool more = decltype(more_t)::value;
            const uint4* cur = lds + (c & 1) * CH;
            if (more) stage_load(next_c);
            __builtin_amdgcn_sched_barrier(0);      // requests are issued where they are written: the scheduler would sink them
#pragma unroll
            for (int kb = 0; kb < MFMA_PIPE; ++kb) {
#pragma unroll
                for (int jj = 0; jj < 4; ++jj)
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        const uint4 Bv = cur[(((kb * 4 + jj) * NT + t) << 6) + lane];
#pragma unroll
                        for (int tw = 0; tw < TW; ++tw)
                            acc[tw][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, Bv),
                                                                                 __builtin_bit_cast(bf16x8_t, A[kb][tw][jj]), acc[tw][t], 0, 0, 0);
                    }
                __builtin_amdgcn_sched_barrier(0);
                if (more) load_A(kb, next_c * MFMA_PIPE + kb);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (more) stage_store(lds + ((c + 1) & 1) * CH, next_c);
            lds_barrier();          // the chunk just consumed may be overwritten, the next one is complete
        };
        for (int c = 0; c + 1 < nchunk; ++c) {
            next_c = cur_c + 1;
            const bool ends = next_c == part_at((part ^ rot) + 1);
            if (ends) next_c = part_at((part + 1) ^ rot);
            chunk(std::true_type{}, c);
            if (ends) fold(part++);
            cur_c = next_c;
        }
        chunk(std::false_type{}, nchunk - 1);
        fold(part);
#pragma unroll
        for (int tw = 0; tw < TW; ++tw) {
            const int row = (tile0 + tw) * 16 + li;
            if (row < f.V) {
                const float bias = f.bp[row];
                const size_t col = f.scatter ? (size_t)f.perm[row] : (size_t)row;
                float* dst = f.out + col * f.row_stride;
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const int sq = seq0 + t * 16 + 4 * g;
                    if (f.row_stride > 1 && (n & 3) == 0) {       // four sequences of a row: one 16-byte store
                        if (sq < n) *reinterpret_cast<float4*>(dst + sq) = make_float4(acc[tw][t][0] + bias, acc[tw][t][1] + bias, acc[tw][t][2] + bias, acc[tw][t][3] + bias);
                        continue;
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (sq + r < n) dst[(size_t)(sq + r) * f.out_stride] = acc[tw][t][r] + bias;
                }
            }
        }
    }
}

// All n sequences through the MFMA path: up to 64 per pass over W'.  Two K blocks (of 128) are requested ahead: four
// measured 2-8 % slower at d = 8192 for up to 32 sequences (and spill with 64), one no faster, eight far slower.  The groups of 128 TW rows are dealt to the blocks in rounds:
// two row tiles per wave (a fragment of h read from LDS then serves two MFMAs) unless one tile per wave saves a
// round's worth of idle blocks.  Four tiles per wave with half the K blocks ahead measured 4-7 % slower at d = 8192.
template <int TW, int LEVELS>
__device__ __forceinline__ void full_mfma_pass(const FullArgs& f, int n, uint4* lds, int block, int nblocks) {
    for (int s0 = 0; s0 < n; s0 += 64) {
        const int m = n - s0;
        if (m <= 16) full_mfma_device<1, TW, 2, LEVELS>(f, n, s0, lds, block, nblocks);
        else if (m <= 32) full_mfma_device<2, TW, 2, LEVELS>(f, n, s0, lds, block, nblocks);
        else full_mfma_device<4, TW, 2, LEVELS>(f, n, s0, lds, block, nblocks);
    }
}
template <int LEVELS>
__device__ __forceinline__ void full_mfma_all(const FullArgs& f, int n, uint4* lds, int block, int nblocks) {
    const int ntiles = (f.V + 15) >> 4, NW = MFMA_THREADS / 64;
    auto cost = [&](int tw) {           // rounds of groups x time of a group
        const int groups = (ntiles + NW * tw - 1) / (NW * tw);
        return (groups + nblocks - 1) / nblocks * tw;
    };
    if (cost(2) <= cost(1)) full_mfma_pass<2, LEVELS>(f, n, lds, block, nblocks);
    else full_mfma_pass<1, LEVELS>(f, n, lds, block, nblocks);
}

// Of this kernel and the fallback product there is a form per full_k_levels: sums held for levels that a length does not
// use cost registers (d = 4096, 8 sequences in a step 217 us, with three levels compiled in 223).
template <int LEVELS>
__global__ __launch_bounds__(MFMA_THREADS) void full_mfma_kernel(FullArgs f) {
    extern __shared__ uint4 stage_lds[];
    full_mfma_all<LEVELS>(f, f.n_fixed, stage_lds, blockIdx.x, gridDim.x);
}

// The first stage for k <= RANK_DIRECT < n with the chunk's logits in registers (blockDim.x = SEQ_THREADS, sixteen values
// a thread): no staging, two passes over the registers.  Pass one: the thread's maximum, hence the maxima of 256 groups
// (the values i with i % 256 == g); their k-th largest is a threshold that k values reach (each thread counts the
// groups above its own, over half of them), their largest the chunk's maximum.  Pass two: the sum for the log-sum-exp,
// in block_lse's order (the same bits), and the values at or above the threshold, which are ranked like any other
// candidates.  Returns false (nothing decided) when more than CAND_CAP values reach the threshold.
template <class IdFn>
__device__ __forceinline__ bool fb_topk_regs(const float* __restrict__ vals, int n, int k, IdFn idf, SeqShared& s, LseAcc& l, int& kk) {
    extern __shared__ __align__(16) u64 arena[];
    constexpr int PER = FB_CHUNK / SEQ_THREADS;
    const int tid = threadIdx.x, lane = tid & 63;
    float v[PER];
    // all sixteen loads first, from clamped addresses; values past the end are replaced afterwards (a select behind each
    // load would be waited for where it stands: sixteen round trips one after the other)
#pragma unroll
    for (int j = 0; j < PER; ++j) v[j] = vals[min(tid + SEQ_THREADS * j, n - 1)];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (tid + SEQ_THREADS * j >= n) v[j] = -INFINITY;
    float* gm = reinterpret_cast<float*>(arena);
    float* cval = reinterpret_cast<float*>(reinterpret_cast<char*>(arena) + CAND_OFF);
    int* cid = reinterpret_cast<int*>(cval + CAND_CAP + 4);
    float mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < PER; ++j) mx = fmaxf(mx, v[j]);
    gm[tid] = mx;
    if (tid < CAND_CAP) cval[tid] = -INFINITY;
    if (tid < 4) cval[CAND_CAP + tid] = -INFINITY;
    if (tid == 0) {
        s.cnt = 0;
        s.eq = 0xFFFFFFFFu;
    }
    __syncthreads();
    const int e = tid & 255, half = tid >> 8;
    const float ve = fmaxf(gm[e], gm[e + 256]);                  // the maximum of group e
    int gt = 0;
    const float4* gm4 = reinterpret_cast<const float4*>(gm);
#pragma unroll 8
    for (int q = half * 32; q < half * 32 + 32; ++q) {
        const float4 x = gm4[q], y = gm4[64 + q];
        gt += (fmaxf(x.x, y.x) > ve) + (fmaxf(x.y, y.y) > ve) + (fmaxf(x.z, y.z) > ve) + (fmaxf(x.w, y.w) > ve);
    }
    s.rank[tid] = gt;
    __syncthreads();
    if (tid < 256) {
        const int g = s.rank[tid] + s.rank[tid + 256];           // groups with a larger maximum
        if (g < k) atomicMin(&s.eq, lkey(ve));                   // the k-th largest is the smallest of those with fewer than k above
        if (g == 0) s.rem = __float_as_uint(ve);                 // the chunk's maximum (equal writes if it comes twice)
    }
    __syncthreads();
    const float th = fkey_inv(s.eq), vmax = __uint_as_float(s.rem);
    float sm = 0.f, over = 0.f;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int i = tid + SEQ_THREADS * j;
        if (vmax > -INFINITY && i < n) sm += expf(v[j] - vmax);
        const bool in = i < n && v[j] >= th;
        if (in) over += v[j] - th;
        const unsigned long long bal = __ballot(in);
        if (bal) {
            const int lead = __ffsll((long long)bal) - 1;
            unsigned base = 0;
            if (lane == lead) base = atomicAdd(&s.cnt, (unsigned)__popcll(bal));
            base = __shfl(base, lead, CSV_WAVE);
            const unsigned slot = base + (unsigned)__popcll(bal & ((1ull << lane) - 1ull));
            if (in && slot < CAND_CAP) {
                cval[slot] = v[j];
                cid[slot] = i;           // the token id is looked up below, for all candidates at once: a load from global
            }                            // memory in this loop would be waited for in every trip that collects something
        }
    }
    over = wave_sum(over);
    float* wover = reinterpret_cast<float*>(s.redu);
    if (lane == 0) wover[tid >> 6] = over;
    l.m = vmax;
    l.s = block_sum(sm, reinterpret_cast<float*>(s.redl));        // its barriers also publish the candidates and wover; not s.redf, which the ranking writes
    const int m = (int)s.cnt;
    if (m > CAND_CAP) return false;
    if (tid < m) cid[tid] = idf(cid[tid]);
    __syncthreads();
    kk = min(k, m);
    if (m > RANK_BUCKETS_MIN && th > -INFINITY) {
        float tot = 0.f;
        for (int q = 0; q < (SEQ_THREADS >> 6); ++q) tot += wover[q];
        rank_buckets(cval, cid, m, kk, th, fminf(vmax, th + 8.f * tot / (float)m), s);
    } else {
        float dummy;
        rank_small(cval, cid, m, kk, s, dummy);
    }
    return true;
}

// First stage of top-k / log-sum-exp over V: one block per (chunk of rows, fallback slot).  The chunk's logits
// are staged in LDS; token ids come from the permutation only for elements at the selection boundary.
template <bool THRESH>
__device__ __forceinline__ void fb_topk_device(const StepArgs& a, int slot, int chunk, SeqShared& s) {
    extern __shared__ __align__(16) u64 arena[];
    const int tid = threadIdx.x, nt = blockDim.x;
    const int c0 = chunk * FB_CHUNK;
    const int n = min(FB_CHUNK, a.V - c0);
    const float* vals = a.fb_logits + (size_t)slot * a.V + c0;
    auto idf = [&](int i) { return a.perm[c0 + i]; };
    const size_t pc = (size_t)slot * a.n_chunks + chunk;
    if (THRESH && a.k > 0 && a.k <= RANK_DIRECT && n > RANK_DIRECT) {
        LseAcc lr;
        int kr = 0;
        const bool done = fb_topk_regs(vals, n, a.k, idf, s, lr, kr);
        __syncthreads();
        if (done) {
            if (tid == 0) {
                a.cand_max[pc] = lr.m;
                a.cand_sum[pc] = lr.s;
            }
            for (int t = tid; t < a.k; t += nt) {
                a.cand_val[pc * a.k + t] = t < kr ? s.wval[t] : -INFINITY;
                a.cand_id[pc * a.k + t] = t < kr ? s.wid[t] : 0x7fffffff;
            }
            return;
        }
    }
    stage_to_lds(reinterpret_cast<float*>(arena), vals, n);
    __syncthreads();
    auto val = [](int i) { return reinterpret_cast<const float*>(arena)[i]; };
    const LseAcc l = block_lse(n, val, s);
    if (tid == 0) {
        a.cand_max[pc] = l.m;
        a.cand_sum[pc] = l.s;
    }
    if (a.k > 0) {
        int kk = 0;
        float vmax;
        bool done = false;
        if (THRESH && n > RANK_DIRECT) {
            __syncthreads();
            done = threshold_topk<false, true>(n, a.k, -INFINITY, false, idf, s, kk, vmax);
            __syncthreads();
        }
        if (!done) kk = block_topk(n, a.k, val, idf, s);
        for (int t = tid; t < a.k; t += nt) {
            a.cand_val[pc * a.k + t] = t < kk ? s.wval[t] : -INFINITY;
            a.cand_id[pc * a.k + t] = t < kk ? s.wid[t] : 0x7fffffff;
        }
    }
}

// Second stage: merge the chunk candidates of one fallback sequence and write its outputs.
template <bool THRESH>
__device__ __forceinline__ void fb_final_device(const StepArgs& a, int slot, SeqShared& s) {
    extern __shared__ __align__(16) u64 arena[];
    const int tid = threadIdx.x, nt = blockDim.x;
    const int b = a.fb_list[slot];
    const float* cm = a.cand_max + (size_t)slot * a.n_chunks;
    const float* cs = a.cand_sum + (size_t)slot * a.n_chunks;
    float mx = -INFINITY;
    for (int i = tid; i < a.n_chunks; i += nt) mx = fmaxf(mx, cm[i]);
    mx = block_max(mx, s.redf);
    float sm = 0.f;
    for (int i = tid; i < a.n_chunks; i += nt) sm += cs[i] * expf(cm[i] - mx);
    sm = block_sum(sm, s.redf);
    if (a.k > 0) {
        const float* cv = a.cand_val + (size_t)slot * a.n_chunks * a.k;
        const int32_t* ci = a.cand_id + (size_t)slot * a.n_chunks * a.k;
        const int n = a.n_chunks * a.k;
        if (n <= STAGE_CAP) {
            stage2_to_lds(reinterpret_cast<float*>(arena), cv, reinterpret_cast<int*>(arena) + STAGE_CAP, ci, n);
            __syncthreads();
            auto sval = [](int i) { return reinterpret_cast<const float*>(arena)[i]; };
            auto sid = [](int i) { return reinterpret_cast<const int*>(arena)[STAGE_CAP + i]; };
            int kk = 0;
            float vmax;
            bool done = false;
            if (THRESH && n > RANK_DIRECT) {
                done = threshold_topk(n, a.k, -INFINITY, false, sid, s, kk, vmax);
                __syncthreads();
            }
            if (!done) block_topk(n, a.k, sval, sid, s);
        } else {
            block_topk(n, a.k, [&](int i) { return cv[i]; }, [&](int i) { return ci[i]; }, s);
        }
        for (int t = tid; t < a.k; t += nt) {
            a.out.d_ids[(size_t)b * a.k + t] = s.wid[t];
            a.out.d_logits[(size_t)b * a.k + t] = s.wval[t];
        }
        write_distribution(a, b, min(a.k, a.V), mx + logf(sm), s);
    }
    if (tid == 0) {
        a.out.d_lse[b] = mx + logf(sm);
        a.out.d_flags[b] = CSV_FLAG_FALLBACK | CSV_FLAG_TOPK_CERT | CSV_FLAG_SOFTMAX_CERT;
        a.out.d_n_rows[b] = a.V;
        a.out.d_n_clusters[b] = a.C;
        if (a.out.d_fallback_count) atomicAdd(a.out.d_fallback_count, 1ull);
    }
}

// ================================================================================================ tail of a step
// Everything that is rarely needed runs in ONE kernel, so that a step whose sequences were all certified in round 0
// pays for one (immediately returning) launch instead of five: round-1 gathered GEMV, round-1 certification, the
// full-vocabulary product for fallback sequences, and the two stages of their top-k / log-sum-exp.  The phases
// depend on each other grid-wide, so the blocks meet at barriers built on device-scope atomics.  The grid is sized
// by the host so that all blocks are resident together; every wait is bounded: a block that waits too long raises
// the abort flag and every block leaves (the step's unfinished sequences keep the INVALID flag seed_kernel gave them).
#define TAIL_THREADS 512
static_assert(TAIL_THREADS == SEQ_THREADS, "the per-sequence phases assume one block size");
#define TAIL_SPIN_LIMIT (1 << 22)

// Returns false when the step was aborted.  Each barrier of a step uses its own counter.
__device__ __forceinline__ bool grid_barrier(int* counters, int which, int nblocks, int* s_flag, int spin_limit) {
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        atomicAdd(&counters[CNT_BARRIER + which], 1);
        int ok = 1, spins = 0;
        // relaxed polls (an acquire per poll would invalidate the XCD's L2 every time); the fence below acquires once
        while (__hip_atomic_load(&counters[CNT_BARRIER + which], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < nblocks) {
            if (__hip_atomic_load(&counters[CNT_ABORT], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) { ok = 0; break; }
            if (++spins > spin_limit) {
                atomicExch(&counters[CNT_ABORT], 1);
                ok = 0;
                break;
            }
            __builtin_amdgcn_s_sleep(32);
        }
        __threadfence();
        *s_flag = ok;
    }
    __syncthreads();
    return *s_flag != 0;
}

// block / nblocks: this block's position among the blocks that run the tail together (all resident).
template <bool THRESH, bool MANY>
__device__ __forceinline__ void tail_device(const StepArgs& a, const FullArgs& f, int from, int block, int nblocks,
                                            SeqShared& s, GemvShared& gs, int* s_flag) {
    extern __shared__ __align__(16) u64 arena[];
    const int tid = threadIdx.x;
    if (a.counters[CNT_TAIL_NEEDED] == 0) return;      // the common case at small batches: one word, no reduction
    if (from == CSV_MAX_ROUNDS && a.counters[CNT_FALLBACK] == 0) return;
    // is any sequence waiting for round 0 (a seed prefix too large for the round-0 blocks), for round 1 or for the
    // full product?  Every block reads the same, settled values.
    int mine0 = 0, mine1 = 0;
    if (tid < a.B && from < CSV_MAX_ROUNDS) {
        mine0 = from ? 0 : a.counters[CNT_TILES + tid];
        mine1 = a.counters[CNT_TILES + (from ? from : 1) * CSV_MAX_BATCH + tid];
    }
    const int n_fb0 = a.counters[CNT_FALLBACK];
    const int tiles0 = block_sum_i(mine0, s.redi);
    int tiles = block_sum_i(mine1, s.redi);
    if (tiles0 == 0 && tiles == 0 && n_fb0 == 0) return;

    // Rounds: the GEMV over the round's work list, then the certification, which may plan the next round.
    // Round 0 is here only for seed prefixes that the round-0 blocks handed over.
    const int first = from ? from : tiles0 > 0 ? 0 : 1;
    for (int r = first; r < a.max_rounds; ++r) {
        if (r > 0) {
            if (r > first) {             // planned by a certification earlier in this kernel: read past the barrier
                const int mine = tid < a.B ? __hip_atomic_load(&a.counters[CNT_TILES + r * CSV_MAX_BATCH + tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
                tiles = block_sum_i(mine, s.redi);
            }
            if (tiles == 0) break;
            if (from && block == 0 && tid == 0) a.host_history[1] = 1;      // the host launches these rounds for the next steps
        }
        gemv_tiles_device(a, r, reinterpret_cast<uint4*>(arena), gs, block, nblocks);
        if (!grid_barrier(a.counters, 2 * r, nblocks, s_flag, a.spin_limit)) return;
        // chunk-major items: the first chunks of all sequences (often the only ones with work) go to distinct blocks
        for (int item = block; item < a.B * a.sp_chunks; item += nblocks) {
            cert_device<THRESH>(a, item % a.B, item / a.B, r, s);
            __syncthreads();
        }
        if (!grid_barrier(a.counters, 2 * r + 1, nblocks, s_flag, a.spin_limit)) return;
    }
    const int n_fb = __hip_atomic_load(&a.counters[CNT_FALLBACK], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
    if (n_fb == 0) return;
    // the same rule as the separate launches, so that a sequence's logits do not depend on how the step was launched
    if (MANY && n_fb > FULL_G)
        full_mfma_all<3>(f, n_fb, reinterpret_cast<uint4*>(arena), block, nblocks);
    else
        full_gemv_device(f, n_fb, reinterpret_cast<uint4*>(arena), block, nblocks);
    if (!grid_barrier(a.counters, 2 * CSV_MAX_ROUNDS, nblocks, s_flag, a.spin_limit)) return;
    for (int item = block; item < n_fb * a.n_chunks; item += nblocks) {
        fb_topk_device<THRESH>(a, item / a.n_chunks, item % a.n_chunks, s);
        __syncthreads();
    }
    if (!grid_barrier(a.counters, 2 * CSV_MAX_ROUNDS + 1, nblocks, s_flag, a.spin_limit)) return;
    for (int slot = block; slot < n_fb; slot += nblocks) {
        fb_final_device<THRESH>(a, slot, s);
        __syncthreads();
    }
}

// from: the first round it runs, those before were launches of their own (0: as queued; CSV_MAX_ROUNDS: the fallback only)
__global__ __launch_bounds__(TAIL_THREADS) void tail_kernel(StepArgs a, FullArgs f, int from) {
    __shared__ SeqShared s;
    __shared__ GemvShared gs;
    __shared__ int s_flag;
    tail_device<true, true>(a, f, from, blockIdx.x, gridDim.x, s, gs, &s_flag);
}

// ------------------------------------------------------------------------------------------------ round 0 as a launch
// Plain form, grid NB x B: round 0 only; what follows is launched separately.  THRESH, PLANS: see cert_body.
template <bool THRESH, bool PLANS>
__global__ __launch_bounds__(SEQ_THREADS) void round0_kernel(StepArgs a, int NB) {
    __shared__ SeqShared s;
    round0_device<THRESH, PLANS>(a, blockIdx.x / NB, blockIdx.x % NB, NB, s);
}

// Fused form, used while recent steps rarely needed anything after round 0: the first NB x B blocks run round 0,
// the remaining blocks are the tail's blocks, parked until every sequence's round 0 is settled.  When nothing is
// queued for them (the common case) they leave at once: the step has saved a kernel launch.  Otherwise they run the
// tail exactly as tail_kernel does (the round-0 blocks have left by then; the tail's blocks are all resident: the
// host sizes the grid for one block per compute unit).  Blocks start in index order, so the blocks waited for are
// already running when a parked block starts; the wait is bounded all the same (the poll limit of the grid barriers).
// MANY: the product for more than FULL_G fallback sequences is compiled in, for batches that can have them (in the kernel of smaller
// ones it costs a step that never runs it up to 0.7 us of 14).
template <bool MANY>
__global__ __launch_bounds__(SEQ_THREADS) void step_kernel(StepArgs a, FullArgs f, int NB) {
    __shared__ SeqShared s;
    __shared__ GemvShared gs;
    __shared__ int s_flag;
    const int n0 = NB * a.B;
    if ((int)blockIdx.x < n0) {
        const int settled = round0_device<false, false>(a, blockIdx.x / NB, blockIdx.x % NB, NB, s, &a.counters[CNT_R0_DONE]);
        if (!settled || settled == 3) return;          // 3: finished and already counted
        __syncthreads();                      // all of the block's writes are issued
        if (threadIdx.x == 0) {
            // One word tells the parked blocks both things: sequences settled (low half) and whether any of them
            // left work for the tail (high half).  Work is released before the count; a finished sequence left
            // nothing for the tail to read.
            if (settled == 2) __threadfence();
            atomicAdd(&a.counters[CNT_R0_DONE], settled == 2 ? 0x10001 : 1);
        }
        return;
    }
    if (threadIdx.x == 0) {
        int ok = 1, spins = 0, v;
        while (((v = __hip_atomic_load(&a.counters[CNT_R0_DONE], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) & 0xffff) < a.B) {
            if (++spins > a.spin_limit) {
                atomicExch(&a.counters[CNT_ABORT], 1);
                ok = 0;
                break;
            }
            __builtin_amdgcn_s_sleep(4);
        }
        if (ok && (v >> 16) == 0) ok = 0;     // every sequence finished in round 0: nothing to do, nothing to acquire
        if (ok) __threadfence();              // acquire
        s_flag = ok;
    }
    __syncthreads();
    if (!s_flag) return;
    tail_device<false, MANY>(a, f, 0, (int)blockIdx.x - n0, (int)gridDim.x - n0, s, gs, &s_flag);   // the lean form: see cert_body
}

// ------------------------------------------------------------------------------------------------ the tail, one launch per phase
// The same phases as tail_kernel as separate launches, used while recent steps needed them: a kernel boundary
// costs about 2.5 us on this machine, a grid barrier among 256 resident blocks 14-24 us (every block's device-scope
// release and acquire writes back and invalidates its XCD's L2).  Every kernel finds out on the device whether it
// has anything to do.
__global__ __launch_bounds__(TAIL_THREADS, 2) void round_gemv_kernel(StepArgs a, int r) {
    extern __shared__ __align__(16) u64 arena[];
    __shared__ GemvShared gs;
    if (a.counters[CNT_TAIL_NEEDED] == 0) return;
    gemv_tiles_device(a, r, reinterpret_cast<uint4*>(arena), gs, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(SEQ_THREADS) void round_cert_kernel(StepArgs a, int r) {   // grid (B, chunks per sequence)
    __shared__ SeqShared s;
    if (a.counters[CNT_TAIL_NEEDED] == 0) return;
    cert_device<true>(a, blockIdx.x, blockIdx.y, r, s);
}

// Up to FULL_G fallback sequences take the vector product, more the MFMA product, which needs a compute unit's whole
// register file.  A batch of at most FULL_G sequences launches the first kernel, a larger one the second, which holds
// both products and picks by the number of fallback sequences.
__global__ __launch_bounds__(TAIL_THREADS, 2) void fb_product_kernel(StepArgs a, FullArgs f) {
    extern __shared__ __align__(16) u64 arena[];
    const int n_fb = a.counters[CNT_FALLBACK];
    if (n_fb == 0 || n_fb > FULL_G) return;
    full_gemv_device(f, n_fb, reinterpret_cast<uint4*>(arena), blockIdx.x, gridDim.x);
}

template <int LEVELS>
__global__ __launch_bounds__(MFMA_THREADS) void fb_product_mfma_kernel(StepArgs a, FullArgs f) {
    extern __shared__ uint4 stage_lds[];
    const int n_fb = a.counters[CNT_FALLBACK];
    if (n_fb == 0) return;
    if (n_fb > FULL_G) full_mfma_all<LEVELS>(f, n_fb, stage_lds, blockIdx.x, gridDim.x);
    else full_gemv_device(f, n_fb, stage_lds, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(SEQ_THREADS) void fb_topk_kernel(StepArgs a) {             // grid (chunks of V, B)
    __shared__ SeqShared s;
    if ((int)blockIdx.y >= a.counters[CNT_FALLBACK]) return;
    fb_topk_device<true>(a, blockIdx.y, blockIdx.x, s);
}

__global__ __launch_bounds__(SEQ_THREADS) void fb_final_kernel(StepArgs a) {            // grid B
    __shared__ SeqShared s;
    if ((int)blockIdx.x >= a.counters[CNT_FALLBACK]) return;
    fb_final_device<true>(a, blockIdx.x, s);
}

// ================================================================================================ host side
static void profile_release(csv_workspace* ws);

static int next_pow2(int x) {
    int p = 1;
    while (p < x) p <<= 1;
    return p;
}

// dynamic LDS of the per-sequence kernels
static size_t seed_lds(const csv_workspace* ws) {
    const size_t general = (size_t)ws->Npad * 8 + (size_t)ws->C * 8 + 8;       // keys, offsets, tail terms
    const size_t staged = (size_t)ws->C * 16 + 32;                             // bounds, ln n, {first row, rows} (small indexes)
    return general > staged ? general : staged;
}
static size_t cert_lds(const csv_workspace* ws) {
    const size_t plan = seed_lds(ws), stage = (size_t)CAND_OFF + CAND_BYTES;      // staged logits and ids, then the candidates of a later round
    return plan > stage ? plan : stage;
}
static size_t round0_h_off(const csv_workspace* ws) { return (seed_lds(ws) + 15) / 16 * 16; }
static size_t round0_lds(const csv_workspace* ws) {
    const size_t c = cert_lds(ws), h = round0_h_off(ws) + (size_t)ws->d * 2;
    return c > h ? c : h;
}

static void fill_args(StepArgs& a, const csv_workspace* ws, const csv_index* idx) {
    memset(&a, 0, sizeof(a));
    a.V = idx->V; a.d = idx->d; a.C = idx->C;
    a.Wp = idx->Wp; a.bp = idx->bp; a.perm = idx->perm; a.mu = idx->mu; a.mu16 = idx->mu16; a.R = idx->R; a.bmax = idx->bmax;
    a.n = idx->n; a.off = idx->off; a.lnn = idx->lnn; a.cmeta = idx->cmeta; a.bt = idx->bt; a.bt_m = idx->bt_m; a.ang = idx->ang; a.ln_nmax = idx->ln_nmax;
    a.K_cap = ws->K_cap; a.Npad = ws->Npad; a.n_chunks = ws->n_chunks; a.tile_stride = ws->tile_stride; a.sp_chunks = ws->sp_chunks; a.cand_chunks = ws->cand_chunks;
    a.U = ws->U; a.hnorm = ws->hnorm; a.bound_partial = ws->bound_partial; a.st = ws->st; a.sel = ws->sel; a.slog = ws->slog; a.sid = ws->sid; a.slots = ws->slots; a.B_max = ws->B_max;
    a.tiles[0] = ws->tiles[0]; a.tiles[1] = ws->tiles[1]; a.counters = ws->counters;
    a.r0_h_off = (int)(round0_h_off(ws) / 16);
    a.tail_lds = (int)ws->tail_lds;
    a.spin_limit = ws->spin_limit;
    a.host_history = ws->d_history;
    a.fb_list = ws->fb_list; a.fb_logits = ws->fb_logits; a.cand_val = ws->cand_val; a.cand_id = ws->cand_id;
    a.cand_max = ws->cand_max; a.cand_sum = ws->cand_sum;
}

static int check_pair(const csv_workspace* ws, const csv_index* idx, const void* d_h, int B) {
    if (!ws || !idx || !d_h) { csv_set_error("null workspace, index or h"); return CSV_EINVAL; }
    if (ws->V != idx->V || ws->d != idx->d || ws->C != idx->C) { csv_set_error("workspace was created for another index shape"); return CSV_ESHAPE; }
    if (B < 1 || B > ws->B_max) { csv_set_error("B=%d outside 1..%d", B, ws->B_max); return CSV_ESHAPE; }
    return CSV_OK;
}

// The dynamic-LDS limit of a kernel is one attribute per process and device, shared by every workspace: it is only
// ever raised, so a workspace created later with smaller needs cannot take away what an earlier one's launches rely on.
enum { K_ROUND0, K_ROUND0_THRESH, K_ROUND0_PLANS, K_STEP, K_STEP_MANY, K_TAIL, K_RCERT, K_FBPROD, K_FBPRODM /* + levels */, K_FULLMFMA = K_FBPRODM + 4 /* + levels */, K_ALG1 = K_FULLMFMA + 4, K_BOUND, K_BOUNDT, K_BOUNDT16, K_NKERN };
static size_t g_lds_limit[CSV_STATIC_MAX_DEVICES][K_NKERN];
static pthread_mutex_t g_attr_lock = PTHREAD_MUTEX_INITIALIZER;
#define CSV_STATIC_LDS_MAX 16384     // at least the static shared memory of any kernel here
static hipError_t raise_lds(int dev, int which, const void* fn, size_t bytes) {
    if (dev < 0 || dev >= CSV_STATIC_MAX_DEVICES) return hipErrorInvalidDevice;
    hipError_t e = hipSuccess;
    pthread_mutex_lock(&g_attr_lock);
    if (bytes > g_lds_limit[dev][which]) {
        if (bytes + CSV_STATIC_LDS_MAX > 65536) e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (e == hipSuccess) g_lds_limit[dev][which] = bytes;
    }
    pthread_mutex_unlock(&g_attr_lock);
    return e;
}

// K slices of the batched bound product and k-blocks (of 32) per slice: enough slices that (groups of cluster tiles x
// slices) fills the device, a whole number of request chunks per slice, a slice's h within BOUND_LDS_KB of LDS, at most
// BOUND_KS_MAX slices (the partial buffer holds KS x B x C floats).  B decides how many sequence tiles a block carries.
static int bound_mfma_nt(int B) { return B > 32 ? 4 : (B > 16 ? 2 : 1); }
static void bound_mfma_plan(int C, int d, int B, int& KS, int& kbs, bool many, bool m16 = false) {
    const int tiles = (C + 15) / 16, groups = (tiles + BOUND_TILES_PER_BLOCK - 1) / BOUND_TILES_PER_BLOCK, nkb = (d + 31) / 32;
    KS = (BOUND_BLOCK_TARGET + groups - 1) / groups;
    if (KS > BOUND_KS_MAX) KS = BOUND_KS_MAX;
    if (KS > nkb) KS = nkb;
    kbs = (nkb + KS - 1) / KS;
    kbs = (kbs + BOUND_PIPE - 1) / BOUND_PIPE * BOUND_PIPE;     // whole chunks
    const int cap = BOUND_LDS_KB / bound_mfma_nt(B) / BOUND_PIPE * BOUND_PIPE;
    if (kbs > cap) kbs = cap;                                   // d <= 8192: 256 k-blocks in at most 32 slices of 8 always fit
    KS = (nkb + kbs - 1) / kbs;
    if (!many) return;
    // More than 64 sequences, whose groups of 64 are blocks of their own: of the slice lengths that need no more slices than that, the one that costs least.
    // A block takes 0.5 us per k-block of float32 centroids, 0.25 of bf16, in as many rounds over the compute units as the blocks make; partial sums, which
    // the launch writes and the next one reads, 2.2 us a million (fitted to 90 plans; over 110 shapes, B = 65..256, the choice is 0.4 % slower than the
    // best on average, 5 % at most).  us with the slices of 64 sequences / always the longest / now: C = 1024, d = 4096, 256 sequences 26.8 / 18.9 / 19.1,
    // 130 18.7 / 20.1 / 17.3; C = 3614, d = 2184, 65 22.3 / 23.7 / 20.8; bf16 C = 2000, d = 5000, 72 15.0 / 16.4 / 15.0, 150 20.4 / 18.3 / 18.3.
    const int most = KS;
    double best = 0.0;
    for (int len = BOUND_PIPE; len <= BOUND_LDS_KB_MANY / bound_mfma_nt(B); len += BOUND_PIPE) {
        const int n = (nkb + len - 1) / len, rounds = (groups * n * ((B + 63) / 64) + BOUND_BLOCK_TARGET - 1) / BOUND_BLOCK_TARGET;
        const double cost = rounds * len * (m16 ? 0.25 : 0.5) + 2.2e-6 * n * B * C;
        if (n <= most && (best == 0.0 || cost <= best)) {
            best = cost;
            KS = n;
            kbs = len;
        }
    }
}

// Where the one launch beats the product over K slices and the launch that adds them up: its blocks are as many as tiles (4096 clusters are one
// round of them on 256 compute units) and each reads its rows alone, so rows must be short or tiles many.  us, two launches / one, B = 16:
// bf16, d = 1024: C = 1024 9.2 / 6.6, C = 8192 9.6 / 7.2; d = 4096: C = 1024 9.4 / 7.9, C = 4096 11.5 / 8.6, but C = 8192 16.1 / 17.3;
//   d = 5120: C = 1024 8.9 / 8.8, C = 2048 9.6 / 8.8, C = 4096 13.0 / 10.8; d = 5376 (a sixth chunk): C = 1024 8.9 / 9.8, C = 2048 9.7 / 10.0; the line
//   is theirs: C = 2304 and more would gain up to d = 7168 (C = 2560, d = 6144 11.0 / 10.3, C = 4096, d = 7168 15.3 / 13.2, but d = 8192 16.4 / 18.9);
//   more than 4096 clusters: C = 5000, d = 2048 9.6 / 9.5, d = 2304 9.9 / 11.2.
// float32, d = 2048: C = 256 9.5 / 8.1, C = 1024 10.0 / 8.1, C = 4096 11.2 / 8.8; d = 2304: C = 1024 9.8 / 9.9; d = 4096: C = 1024 9.3 / 11.8;
//   d = 5120: C = 2048 13.9 / 14.6; many tiles: C = 3072, d = 3072 13.2 / 10.9, C = 3072, d = 6144 17.7 / 16.7, d = 6400 18.1 / 18.7,
//   C = 4096, d = 4608 17.4 / 16.3, but d = 4096 16.1 / 20.5 (rows 16 KB apart ask for the same memory channels).  The line keeps clear of all
//   rows a multiple of 4 KB apart, though those of 12, 20 and 24 KB would gain (C = 4096, d = 5120 18.7 / 16.8).
static bool bound_tile_pays(int C, int d, int B, bool m16) {
    if (B > 16) return false;
    if (m16) return d <= (C <= 4096 ? 5120 : 2048);
    return C <= 4096 && (d <= 2048 || (C >= 3072 && d <= 6144 && d % 1024 != 0));
}
static int launch_bounds_kernel(const StepArgs& a, float* U, float* hn, int reset, hipStream_t st) {
    if (a.B >= BOUND_MFMA_MIN_B) {
        const int tiles = (a.C + 15) / 16;
        if (bound_tile_pays(a.C, a.d, a.B, a.mu16 != nullptr)) {
            int dev = 0;
            CSV_HIP(hipGetDevice(&dev));
            CSV_HIP(raise_lds(dev, a.mu16 ? K_BOUNDT16 : K_BOUNDT, a.mu16 ? (const void*)bound_tile_kernel<true> : (const void*)bound_tile_kernel<false>, BOUND_TILE_LDS));
            if (a.mu16) bound_tile_kernel<true><<<tiles, 1024, BOUND_TILE_LDS, st>>>(a, U, hn, reset);
            else bound_tile_kernel<false><<<tiles, 1024, BOUND_TILE_LDS, st>>>(a, U, hn, reset);
            CSV_LAUNCH_CHECK("bound_tile_kernel");
            return CSV_OK;
        }
        int KS, kbs;
        bound_mfma_plan(a.C, a.d, a.B, KS, kbs, a.B > 64, a.mu16 != nullptr);
        dim3 grid((tiles + BOUND_TILES_PER_BLOCK - 1) / BOUND_TILES_PER_BLOCK, KS, (a.B + 63) / 64);
        const int nt = bound_mfma_nt(a.B);
        const size_t lds = (size_t)kbs * nt * 1024;
        if (a.mu16) {
            if (nt == 1) bound_mfma_kernel<1, true><<<grid, 512, lds, st>>>(a, a.bound_partial, kbs, reset);
            else if (nt == 2) bound_mfma_kernel<2, true><<<grid, 512, lds, st>>>(a, a.bound_partial, kbs, reset);
            else if (a.B <= 64) bound_mfma_kernel<4, true><<<grid, 512, lds, st>>>(a, a.bound_partial, kbs, reset);
            else bound_mfma_kernel<4, true, true><<<grid, 512, lds, st>>>(a, a.bound_partial, kbs, reset);
        } else {
            if (nt == 1) bound_mfma_kernel<1, false><<<grid, 512, lds, st>>>(a, a.bound_partial, kbs, reset);
            else if (nt == 2) bound_mfma_kernel<2, false><<<grid, 512, lds, st>>>(a, a.bound_partial, kbs, reset);
            else if (a.B <= 64) bound_mfma_kernel<4, false><<<grid, 512, lds, st>>>(a, a.bound_partial, kbs, reset);
            else bound_mfma_kernel<4, false, true><<<grid, 512, lds, st>>>(a, a.bound_partial, kbs, reset);
        }
        CSV_LAUNCH_CHECK("bound_mfma_kernel");
        bound_finish_kernel<<<dim3((a.C + 255) / 256, a.B), 256, 0, st>>>(a, a.bound_partial, KS, U, hn);
        CSV_LAUNCH_CHECK("bound_finish_kernel");
        return CSV_OK;
    }
    const bool m16 = a.mu16 != nullptr;
    const int nq = m16 ? a.d >> 3 : a.d >> 2;         // 128-bit units per centroid row
    int wpc = 1;
    while (wpc < 4 && (nq + wpc - 1) / wpc > 64 * BOUND_ROWS_PF(a.B)) wpc <<= 1;
    // Three and four sequences against many long bf16 rows: a wave reads twice and more as many bytes of h as of its centroid, and from the second round of
    // waves on (4096 at once) reading h from LDS wins (us, from L2 / from LDS: C = 4096, d = 5120 21.7 / 16.5, C = 2048, d = 7168 9.4 / 7.7, C = 1500,
    // d = 5120 8.6 / 7.1; but C = 1024, d = 8192 6.9 / 7.7, C = 2048, d = 4096 6.4 / 7.5, C = 8192, d = 1024 10.3 / 20.3).
    const size_t lds = (size_t)4 * a.d * 2;
    if (m16 && a.B > 2 && wpc > 1 && a.C * wpc > 4096 && lds <= BOUND_LDS_MAX) {
        int dev = 0, cus = 0;
        CSV_HIP(hipGetDevice(&dev));
        CSV_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
        // as many blocks as are resident together (LDS decides), at most one wave per cluster
        int per_cu = (int)((size_t)(150 * 1024) / (lds + 1024));
        per_cu = per_cu < 1 ? 1 : (per_cu > 4 ? 4 : per_cu);
        int gx = (a.C + (BOUND_THREADS / 64) - 1) / (BOUND_THREADS / 64);
        if (gx > cus * per_cu) gx = cus * per_cu;
        // more dynamic LDS than the default limit: raise the attribute (only ever upwards)
        if (lds + 4096 > 65536) CSV_HIP(raise_lds(dev, K_BOUND, (const void*)bound_kernel, BOUND_LDS_MAX));
        bound_kernel<<<gx, BOUND_THREADS, lds, st>>>(a, U, hn, reset);
        CSV_LAUNCH_CHECK("bound_kernel");
        return CSV_OK;
    }
    const int cpb = (BOUND_THREADS / 64) / wpc;
    const int groups = (a.C + cpb - 1) / cpb;
    const int gpx = (groups + 7) / 8;
#define CSV_BOUND_ROWS(BT)                                                                                            \
    do {                                                                                                              \
        if (m16) bound_rows_kernel<BT, true><<<gpx * 8, BOUND_THREADS, 0, st>>>(a, U, hn, reset, groups, gpx, wpc);   \
        else bound_rows_kernel<BT, false><<<gpx * 8, BOUND_THREADS, 0, st>>>(a, U, hn, reset, groups, gpx, wpc);      \
    } while (0)
    switch (a.B) {
        case 1: CSV_BOUND_ROWS(1); break;
        case 2: CSV_BOUND_ROWS(2); break;
        case 3: CSV_BOUND_ROWS(3); break;
        default: CSV_BOUND_ROWS(4); break;            // more sequences take the MFMA product
    }
#undef CSV_BOUND_ROWS
    CSV_LAUNCH_CHECK("bound_rows_kernel");
    return CSV_OK;
}

// out[s][t] = tmp[inv[t]][s]: the product leaves the n logits of a row side by side, so a token's are read as one run (of up
// to 256 bytes a block) and turned in LDS, and everything is written in 256-byte runs.  Grid (tiles of 64 tokens, slabs of
// 64 sequences).  A scatter of single logits to out[s][perm[r]], one 4-byte request each, was bound by the number of
// requests: 53 us for 32 sequences at V = 256000, also with every sequence kept behind one XCD's L2.
#define UNPERM_TILE 64
__global__ __launch_bounds__(256) void unpermute_kernel(const float* __restrict__ tmp, const int32_t* __restrict__ inv, int V, int n,
                                                        float* __restrict__ out) {
    __shared__ float tile[UNPERM_TILE][UNPERM_TILE + 1];       // [token][sequence]
    __shared__ int32_t row[UNPERM_TILE];
    const int tid = threadIdx.x, t0 = blockIdx.x * UNPERM_TILE, s0 = blockIdx.y * UNPERM_TILE;
    const int nt = min(UNPERM_TILE, V - t0), ns = min(UNPERM_TILE, n - s0);
    if (tid < nt) row[tid] = inv[t0 + tid];
    __syncthreads();
    // the lanes of a wave read 64 / w runs of w values, w = ns rounded up to a power of two
    int lw = 0;
    while ((1 << lw) < ns) ++lw;
    const int s = tid & ((1 << lw) - 1), per = 256 >> lw;
    if (s < ns) {
        const float* src = tmp + s0 + s;
#pragma unroll 4
        for (int t = tid >> lw; t < nt; t += per) tile[t][s] = src[(size_t)row[t] * n];
    }
    __syncthreads();
    const int t = tid & 63;
    if (t < nt)
#pragma unroll 4
        for (int q = tid >> 6; q < ns; q += 4) out[(size_t)(s0 + q) * V + t0 + t] = tile[t][q];
}

// (a full_k_levels of zero, two or three)
static void launch_fb_product_mfma(int grid, const StepArgs& a, const FullArgs& f, hipStream_t st) {
    switch (full_k_levels(f.d)) {
        case 3: fb_product_mfma_kernel<3><<<grid, MFMA_THREADS, mfma_lds(3), st>>>(a, f); break;
        case 2: fb_product_mfma_kernel<2><<<grid, MFMA_THREADS, mfma_lds(2), st>>>(a, f); break;
        default: fb_product_mfma_kernel<0><<<grid, MFMA_THREADS, mfma_lds(0), st>>>(a, f); break;
    }
}

// tmp: [n_fixed x V] scratch for the MFMA path when the result is wanted in token-id order (may be NULL otherwise)
static int launch_full(const csv_index* idx, const uint16_t* d_h, const int32_t* list, int n_fixed,
                       float* out, long long stride, int scatter, float* tmp, hipStream_t st) {
    FullArgs f;
    f.V = idx->V; f.d = idx->d; f.Wp = idx->Wp; f.bp = idx->bp; f.perm = idx->perm; f.h = d_h;
    f.list = list; f.n_fixed = n_fixed; f.out = out; f.out_stride = stride; f.row_stride = 1; f.scatter = scatter;
    if (n_fixed > FULL_G) {
        int dev = 0, cus = 0;
        CSV_HIP(hipGetDevice(&dev));
        CSV_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
        const bool two_step = scatter && tmp && stride == idx->V;
        if (two_step) {
            f.out = tmp;
            f.scatter = 0;
            f.out_stride = 1;
            f.row_stride = n_fixed;
        }
        switch (full_k_levels(idx->d)) {
            case 3: full_mfma_kernel<3><<<cus, MFMA_THREADS, mfma_lds(3), st>>>(f); break;
            case 2: full_mfma_kernel<2><<<cus, MFMA_THREADS, mfma_lds(2), st>>>(f); break;
            default: full_mfma_kernel<0><<<cus, MFMA_THREADS, mfma_lds(0), st>>>(f); break;
        }
        CSV_LAUNCH_CHECK("full_mfma_kernel");
        if (two_step) {
            unpermute_kernel<<<dim3((idx->V + UNPERM_TILE - 1) / UNPERM_TILE, (n_fixed + UNPERM_TILE - 1) / UNPERM_TILE), 256, 0, st>>>(tmp, idx->inv, idx->V, n_fixed, out);
            CSV_LAUNCH_CHECK("unpermute_kernel");
        }
        return CSV_OK;
    }
    // Blocks.  Many short ones rather than few that stay keep the rows in flight close together (the hardware hands them out in
    // order), but each stages h: a share of n / 8 of a tile's bytes per tile it computes.
    // Long rows: 8192 for one and two sequences (V = 128256, d = 4096: 177 and 182 us, with 2048 blocks 188 and 191), for three
    // where that leaves a block more than one tile (190 / 194); 2048 for four (V = 64000, d = 4096 103 us, with 8192 115).
    // Short rows: four tiles a block, 2048 to 8192 blocks (d = 1024, four sequences, us with 2048 / 4096 / 8192, at five waves per SIMD:
    // V = 32000 18.5 / 19.5 / 19.5, V = 128256 60 / 58 / 59, V = 256000 154 / 146 / 139).
    const int ntiles = (idx->V + 7) / 8, n = n_fixed;
    const bool rows_long = idx->d >= 2048;
    int grid = rows_long ? (n <= 2 || (n == 3 && ntiles >= 12288) ? 8192 : 2048) : (ntiles / 4 < 2048 ? 2048 : (ntiles / 4 < 8192 ? ntiles / 4 : 8192));
    grid = grid < ntiles ? grid : ntiles;
    const size_t lds = (size_t)n * idx->d * 2;
    if (rows_long) full_gemv_kernel<4><<<grid, 256, lds, st>>>(f);
    else full_gemv_kernel<2><<<grid, 256, lds, st>>>(f);
    CSV_LAUNCH_CHECK("full_gemv_kernel");
    return CSV_OK;
}

extern "C" int csv_workspace_create(const csv_index* idx, int B_max, int K_cap_rows, csv_workspace** out) {
    if (out) *out = nullptr;
    if (!idx || !out) { csv_set_error("null index or out"); return CSV_EINVAL; }
    if (B_max < 1 || B_max > CSV_MAX_BATCH) { csv_set_error("B_max=%d outside 1..%d", B_max, CSV_MAX_BATCH); return CSV_ESHAPE; }
    if (K_cap_rows < 0 || K_cap_rows > idx->V) { csv_set_error("K_cap_rows=%d outside 0..V", K_cap_rows); return CSV_EINVAL; }
    if ((size_t)FULL_G * idx->d * 2 > 65536) { csv_set_error("d=%d too large for the LDS staging of h", idx->d); return CSV_ESHAPE; }
    csv_workspace* ws = (csv_workspace*)calloc(1, sizeof(csv_workspace));
    if (!ws) { csv_set_error("host allocation failed"); return CSV_ENOMEM; }
    ws->B_max = B_max; ws->K_cap = K_cap_rows > 0 ? K_cap_rows : 1; ws->V = idx->V; ws->d = idx->d; ws->C = idx->C;
    ws->Npad = next_pow2(idx->C);
    ws->n_chunks = (idx->V + FB_CHUNK - 1) / FB_CHUNK;
    ws->device = idx->device;
    ws->sp_chunks = (ws->K_cap + STAGE_CAP - 1) / STAGE_CAP;
    ws->cand_chunks = ws->n_chunks > ws->sp_chunks ? ws->n_chunks : ws->sp_chunks;
    const size_t B = B_max, C = idx->C, V = idx->V, K = ws->K_cap, NC = ws->cand_chunks;
    ws->tile_stride = (int)(K / TILE_ROWS + C + 1);
    const size_t tcap = B * (size_t)ws->tile_stride;
    hipError_t e = hipSuccess;
    auto A = [&](void** p, size_t bytes) { if (e == hipSuccess) e = hipMalloc(p, bytes ? bytes : 16); };
    A((void**)&ws->U, B * C * 4); A((void**)&ws->bound_partial, B_max >= BOUND_MFMA_MIN_B ? B * C * 4 * BOUND_KS_MAX : 16); A((void**)&ws->hnorm, B * 4); A((void**)&ws->st, B * sizeof(SeqState));
    A((void**)&ws->sel, B * C * 4); A((void**)&ws->slog, B * K * 4); A((void**)&ws->sid, B * K * 4);
    A((void**)&ws->slots, B * CSV_SLOT_ROWS * 8);
    A((void**)&ws->tiles[0], tcap * sizeof(Tile)); A((void**)&ws->tiles[1], tcap * sizeof(Tile));
    A((void**)&ws->counters, CNT_ALLOC * 4); A((void**)&ws->fb_list, B * 4); A((void**)&ws->all_list, B * 4);
    A((void**)&ws->fb_logits, B * V * 4); A((void**)&ws->cand_val, B * NC * CSV_MAX_K * 4); A((void**)&ws->cand_id, B * NC * CSV_MAX_K * 4);
    A((void**)&ws->cand_max, B * NC * 4); A((void**)&ws->cand_sum, B * NC * 4);
    if (e == hipSuccess) e = hipMemset(ws->counters, 0, CNT_ALLOC * 4);
    if (e == hipSuccess) e = hipHostMalloc((void**)&ws->h_history, 64, hipHostMallocDefault);
    if (e == hipSuccess) {
        ws->h_history[0] = ws->h_history[1] = 0;
        e = hipHostGetDevicePointer((void**)&ws->d_history, ws->h_history, 0);
    }
    if (e == hipSuccess) e = hipMemset(ws->slots, 0xFF, B * CSV_SLOT_ROWS * 8);     // every slot empty
    if (e == hipSuccess) e = hipMemset(ws->st, 0, B * sizeof(SeqState));
    if (e == hipSuccess) e = hipMemset(ws->tiles[0], 0, tcap * sizeof(Tile));
    if (e == hipSuccess) e = hipMemset(ws->tiles[1], 0, tcap * sizeof(Tile));
    if (e == hipSuccess) {
        int32_t* tmp = (int32_t*)malloc(B * 4);
        for (size_t i = 0; i < B; ++i) tmp[i] = (int32_t)i;
        e = hipMemcpy(ws->all_list, tmp, B * 4, hipMemcpyHostToDevice);
        free(tmp);
    }
    // the per-sequence kernels may need more dynamic LDS than the default limit when C is large
    const int levels = full_k_levels(idx->d);
    if (e == hipSuccess) e = raise_lds(ws->device, K_FULLMFMA + levels, levels == 3 ? (const void*)full_mfma_kernel<3> : levels == 2 ? (const void*)full_mfma_kernel<2> : (const void*)full_mfma_kernel<0>, mfma_lds(levels));
    if (e == hipSuccess) e = raise_lds(ws->device, K_ROUND0, (const void*)round0_kernel<false, false>, round0_lds(ws));
    if (e == hipSuccess) e = raise_lds(ws->device, K_ROUND0_THRESH, (const void*)round0_kernel<true, false>, round0_lds(ws));
    if (e == hipSuccess) e = raise_lds(ws->device, K_ROUND0_PLANS, (const void*)round0_kernel<true, true>, round0_lds(ws));
    if (e == hipSuccess) {
        size_t l = cert_lds(ws);
        const size_t cand[] = {(size_t)FULL_G * idx->d * 2 /* also covers the two h slots of the tile loop */, (size_t)FB_CHUNK * 4, (size_t)STAGE_CAP * 8,
                               B_max > FULL_G ? (size_t)mfma_lds(levels) : 0 /* more than FULL_G fallback sequences: the MFMA product's h fragments */};
        for (size_t c : cand) l = c > l ? c : l;
        ws->tail_lds = l;
        e = raise_lds(ws->device, K_TAIL, (const void*)tail_kernel, l);
        int per_cu = 0, dev = 0, cus = 0;
        if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, tail_kernel, TAIL_THREADS, l);
        if (e == hipSuccess) e = hipGetDevice(&dev);
        if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e == hipSuccess && (per_cu < 1 || cus < 1)) {
            csv_set_error("tail kernel does not fit a compute unit (dynamic LDS %zu bytes)", l);
            csv_workspace_free(ws);
            return CSV_ESHAPE;
        }
        // All blocks of the tail kernel must be resident together, which the occupancy check above guarantees
        // for one block per compute unit.  A second block per unit measured slower at every batch size: the
        // grid barriers cost more with twice the arrivals, and the row loops already keep enough loads in flight.
        ws->tail_grid = cus;
        ws->spin_limit = TAIL_SPIN_LIMIT;
        ws->split_min_B = 0;      // decided per step from the history
        if (e == hipSuccess) e = raise_lds(ws->device, K_RCERT, (const void*)round_cert_kernel, cert_lds(ws));
        if (e == hipSuccess) e = raise_lds(ws->device, K_FBPROD, (const void*)fb_product_kernel, (size_t)FULL_G * idx->d * 2);
        if (e == hipSuccess) e = raise_lds(ws->device, K_FBPRODM + levels, levels == 3 ? (const void*)fb_product_mfma_kernel<3> : levels == 2 ? (const void*)fb_product_mfma_kernel<2> : (const void*)fb_product_mfma_kernel<0>, mfma_lds(levels));
        int r0_per_cu = 0x7fffffff;          // of every form of the kernel: the blocks of a sequence wait for each other
        auto fits = [&](auto kernel) {
            int n = 0;
            if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, SEQ_THREADS, round0_lds(ws));
            r0_per_cu = n < r0_per_cu ? n : r0_per_cu;
        };
        fits(round0_kernel<false, false>);
        fits(round0_kernel<true, false>);
        fits(round0_kernel<true, true>);
        if (e == hipSuccess && r0_per_cu < 1) {
            csv_set_error("round-0 kernel does not fit a compute unit (dynamic LDS %zu bytes)", round0_lds(ws));
            csv_workspace_free(ws);
            return CSV_ESHAPE;
        }
        ws->round0_capacity = r0_per_cu * cus;
        // round 0 and the tail in one launch: every block of that grid (one per compute unit) must be resident
        ws->fused_lds = round0_lds(ws) > l ? round0_lds(ws) : l;
        int few_per_cu = 0, many_per_cu = 0;
        if (e == hipSuccess) e = raise_lds(ws->device, K_STEP, (const void*)step_kernel<false>, ws->fused_lds);
        if (e == hipSuccess) e = raise_lds(ws->device, K_STEP_MANY, (const void*)step_kernel<true>, ws->fused_lds);
        if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&few_per_cu, step_kernel<false>, SEQ_THREADS, ws->fused_lds);
        if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&many_per_cu, step_kernel<true>, SEQ_THREADS, ws->fused_lds);
        ws->fused_ok = few_per_cu >= 1 && many_per_cu >= 1;
    }
    if (e != hipSuccess) {
        csv_set_error("workspace allocation failed: %s", hipGetErrorString(e));
        csv_workspace_free(ws);
        return e == hipErrorOutOfMemory ? CSV_ENOMEM : CSV_EHIP;
    }
    *out = ws;
    return CSV_OK;
}

extern "C" void csv_workspace_free(csv_workspace* ws) {
    if (!ws) return;
    void* ptrs[] = {ws->U, ws->bound_partial, ws->hnorm, ws->st, ws->sel, ws->slog, ws->sid, ws->slots, ws->tiles[0], ws->tiles[1],
                    ws->counters, ws->fb_list, ws->all_list, ws->fb_logits, ws->cand_val, ws->cand_id, ws->cand_max, ws->cand_sum};
    for (void* p : ptrs)
        if (p) (void)hipFree(p);
    if (ws->h_history) (void)hipHostFree(ws->h_history);
    profile_release(ws);
    free(ws);
}

extern "C" int csv_bounds(csv_workspace* ws, const csv_index* idx, const uint16_t* d_h, int B, float* d_U, float* d_hnorm,
                          void* stream) {
    int rc = check_pair(ws, idx, d_h, B);
    if (rc) return rc;
    if (!d_U) { csv_set_error("null d_U"); return CSV_EINVAL; }
    StepArgs a;
    fill_args(a, ws, idx);
    a.B = B; a.h = d_h;
    return launch_bounds_kernel(a, d_U, d_hnorm, 0, (hipStream_t)stream);
}

// ------------------------------------------------------------------------------------------------ bounds without a workspace
// For callers that cannot allocate: the K-slice partial sums of the batched bound product (the only scratch the
// bound kernels use) live in a file-scope device array instead of a workspace buffer.  Every GPU holds its own copy
// of the array at its own address; the address is looked up once per device and handed to the kernels as an argument.
#define CSV_STATIC_SCRATCH_BYTES (8u << 20)
static __device__ __align__(256) unsigned char scratch[CSV_STATIC_SCRATCH_BYTES];
static void* g_scratch_ptr[CSV_STATIC_MAX_DEVICES];          // per device: address of `scratch` there (NULL = not looked up yet)
static pthread_mutex_t g_scratch_lock = PTHREAD_MUTEX_INITIALIZER;

// Address of the array on the current device (looked up on the first call there).
static int static_scratch(int dev, void** out) {
    if (dev < 0 || dev >= CSV_STATIC_MAX_DEVICES) { csv_set_error("device %d outside 0..%d", dev, CSV_STATIC_MAX_DEVICES - 1); return CSV_EINVAL; }
    pthread_mutex_lock(&g_scratch_lock);
    void* p = g_scratch_ptr[dev];
    if (!p) {
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            pthread_mutex_unlock(&g_scratch_lock);
            csv_set_error("hipGetSymbolAddress(scratch) failed on device %d: %s", dev, hipGetErrorString(e));
            return CSV_EHIP;
        }
        g_scratch_ptr[dev] = p;
    }
    pthread_mutex_unlock(&g_scratch_lock);
    *out = p;
    return CSV_OK;
}

extern "C" int csv_bounds_static(const csv_index* idx, const uint16_t* d_h, int B, float* d_U, float* d_hnorm, void* stream) {
    if (!idx || !d_h || !d_U) { csv_set_error("null index, h or d_U"); return CSV_EINVAL; }
    if (B < 1 || B > CSV_MAX_BATCH) { csv_set_error("B=%d outside 1..%d", B, CSV_MAX_BATCH); return CSV_ESHAPE; }
    int dev = -1;
    CSV_HIP(hipGetDevice(&dev));
    if (dev != idx->device) { csv_set_error("the index lives on device %d, the current device is %d", idx->device, dev); return CSV_EINVAL; }
    StepArgs a;
    memset(&a, 0, sizeof(a));
    a.V = idx->V; a.d = idx->d; a.C = idx->C;
    a.mu = idx->mu; a.mu16 = idx->mu16; a.R = idx->R; a.bmax = idx->bmax; a.n = idx->n; a.bt = idx->bt; a.bt_m = idx->bt_m; a.ang = idx->ang;
    a.B = B; a.h = d_h;
    if (B >= BOUND_MFMA_MIN_B) {       // the batched product is the only bound kernel with scratch: KS x B x C partial sums; the limit is that of 64
                                       // sequences' slices for every batch, also where the launch takes fewer slices or none
        int KS, kbs;
        bound_mfma_plan(idx->C, idx->d, B, KS, kbs, false);
        const size_t need = (size_t)KS * B * idx->C * sizeof(float);
        if (need > CSV_STATIC_SCRATCH_BYTES) {
            csv_set_error("B=%d sequences x C=%d clusters need %zu bytes of partial sums, the static scratch holds %u: "
                          "use csv_bounds with a workspace", B, idx->C, need, CSV_STATIC_SCRATCH_BYTES);
            return CSV_ESHAPE;
        }
        void* p = nullptr;
        const int rc = static_scratch(dev, &p);
        if (rc) return rc;
        a.bound_partial = (float*)p;
    }
    return launch_bounds_kernel(a, d_U, d_hnorm, 0, (hipStream_t)stream);
}

extern "C" int csv_full_logits(csv_workspace* ws, const csv_index* idx, const uint16_t* d_h, int B, float* d_logits,
                               void* stream) {
    int rc = check_pair(ws, idx, d_h, B);
    if (rc) return rc;
    if (!d_logits) { csv_set_error("null d_logits"); return CSV_EINVAL; }
    return launch_full(idx, d_h, ws->all_list, B, d_logits, idx->V, 1, ws->fb_logits, (hipStream_t)stream);
}

#define DEEP_HOLD 256
extern "C" int csv_decode_step(csv_workspace* ws, const csv_index* idx, const uint16_t* d_h, int B,
                               const csv_step_params* p, const csv_step_out* o, void* stream) {
    int rc = check_pair(ws, idx, d_h, B);
    if (rc) return rc;
    if (!p || !o) { csv_set_error("null params or out"); return CSV_EINVAL; }
    const bool use_k = p->k >= 1, use_s = p->eps > 0.f;
    if (!use_k && !use_s) { csv_set_error("both certificates disabled (k=%d, eps=%g)", p->k, (double)p->eps); return CSV_EINVAL; }
    if (p->k < 0 || p->k > CSV_MAX_K || p->k > idx->V) { csv_set_error("k=%d outside 0..min(V,%d)", p->k, CSV_MAX_K); return CSV_EINVAL; }
    if (p->K_max_rows < 0 || p->K_max_rows > ws->K_cap) { csv_set_error("K_max_rows=%d exceeds workspace capacity %d", p->K_max_rows, ws->K_cap); return CSV_EINVAL; }
    if (p->combine != CSV_COMBINE_ALL && p->combine != CSV_COMBINE_ANY) { csv_set_error("bad combine=%d", p->combine); return CSV_EINVAL; }
    const int max_rounds = p->max_rounds == 0 ? 2 : p->max_rounds;
    if (max_rounds < 2 || max_rounds > CSV_MAX_ROUNDS) { csv_set_error("max_rounds=%d outside 2..%d", p->max_rounds, CSV_MAX_ROUNDS); return CSV_EINVAL; }
    if (p->delta_clusters < 0) { csv_set_error("delta_clusters=%d is negative", p->delta_clusters); return CSV_EINVAL; }
    if (!o->d_lse || !o->d_flags || !o->d_n_rows || !o->d_n_clusters || (use_k && (!o->d_ids || !o->d_logits))) {
        csv_set_error("null output buffer");
        return CSV_EINVAL;
    }
    hipStream_t st = (hipStream_t)stream;
    StepArgs a;
    fill_args(a, ws, idx);
    a.B = B; a.h = d_h; a.k = p->k; a.K_max = p->K_max_rows; a.combine = p->combine; a.use_k = use_k; a.use_s = use_s;
    if (!use_s) a.lam = -INFINITY;
    else if (p->eps >= 1.f) a.lam = INFINITY;
    else a.lam = (float)log((double)p->eps / (1.0 - (double)p->eps));
    a.max_rounds = max_rounds; a.delta_clusters = p->delta_clusters; a.relax = p->relax != 0;
    if (!(p->top_p >= 0.f && p->top_p <= 1.f)) { csv_set_error("top_p=%g outside 0..1", (double)p->top_p); return CSV_EINVAL; }
    a.top_p = p->top_p;
    if (!use_s) a.lam2 = -INFINITY;
    else if (2.0 * (double)p->eps >= 1.0) a.lam2 = INFINITY;
    else a.lam2 = (float)log(2.0 * (double)p->eps / (1.0 - 2.0 * (double)p->eps));
    a.out = *o;

    hipEvent_t* ev = nullptr;
    if (ws->prof_on && ws->prof_n < ws->prof_cap) ev = ws->prof_ev + (size_t)ws->prof_n++ * (CSV_PROFILE_STAGES + 1);
#define CSV_MARK(i) do { if (ev) CSV_HIP(hipEventRecord(ev[i], st)); } while (0)
    CSV_MARK(0);
    rc = launch_bounds_kernel(a, ws->U, ws->hnorm, 1, st);
    if (rc) return rc;
    CSV_MARK(1);
    FullArgs f;
    f.V = idx->V; f.d = idx->d; f.Wp = idx->Wp; f.bp = idx->bp; f.perm = idx->perm; f.h = d_h;
    f.list = ws->fb_list; f.n_fixed = 0; f.out = ws->fb_logits; f.out_stride = idx->V; f.row_stride = 1; f.scatter = 0;
    if (p->schedule == CSV_SCHEDULE_ALG1) {
        // Algorithm 1's own order: one block per sequence opens one cluster per iteration; then the fallback launches
        const size_t general = (size_t)ws->Npad * 8 + (size_t)ws->C * 8 + 8;
        const size_t h_off = (ALG1_CL_OFF + general + 15) / 16 * 16;
        const size_t lds = h_off + (size_t)idx->d * 2;
        if (lds + sizeof(SeqShared) + 256 > 160u * 1024u) {
            csv_set_error("schedule=ALG1: C=%d, d=%d need %zu bytes of LDS per block, more than a compute unit has", idx->C, idx->d, lds);
            return CSV_ESHAPE;
        }
        if (p->max_rounds > 2 || p->delta_clusters != 0 || p->relax) {
            csv_set_error("schedule=ALG1 has no fallback levels (max_rounds, delta_clusters, relax must be 0)");
            return CSV_EINVAL;
        }
        CSV_HIP(raise_lds(ws->device, K_ALG1, (const void*)alg1_kernel, lds));
        alg1_kernel<<<B, SEQ_THREADS, lds, st>>>(a, (int)(h_off / 16));
        CSV_LAUNCH_CHECK("alg1_kernel");
        CSV_MARK(2);
        if (B > FULL_G) {
            launch_fb_product_mfma(ws->tail_grid, a, f, st);
            CSV_LAUNCH_CHECK("fb_product_mfma_kernel");
        } else {
            fb_product_kernel<<<ws->tail_grid, TAIL_THREADS, (size_t)FULL_G * idx->d * 2, st>>>(a, f);
            CSV_LAUNCH_CHECK("fb_product_kernel");
        }
        fb_topk_kernel<<<dim3(ws->n_chunks, B), SEQ_THREADS, (size_t)CAND_OFF + CAND_BYTES, st>>>(a);
        CSV_LAUNCH_CHECK("fb_topk_kernel");
        fb_final_kernel<<<B, SEQ_THREADS, (size_t)CAND_OFF + CAND_BYTES, st>>>(a);
        CSV_LAUNCH_CHECK("fb_final_kernel");
        CSV_MARK(3);
        return CSV_OK;
    }
    if (p->schedule != CSV_SCHEDULE_ROUNDS) { csv_set_error("bad schedule=%d", p->schedule); return CSV_EINVAL; }
    // One launch per phase pays when the tail is needed (kernel boundaries instead of grid barriers: 30 % of a
    // step even at B = 1), the single kernel when it is not (one launch that returns at once instead of seven).
    // Unless the caller fixed the choice, follow the recent steps: the bound kernel keeps a bit per step in a
    // pinned host word, read here without synchronising (it may lag a few steps; either choice is correct).
    bool split, fb_launches = true, deep = true;
    const unsigned history = (unsigned)*(volatile int*)ws->h_history;
    if (ws->split_min_B > 0) {
        split = B >= ws->split_min_B;
    } else {
        split = __builtin_popcount(history & 0xffu) >= 2;
        // the three fallback phases as launches of their own only while fallbacks occur; otherwise one launch
        // of the single kernel restricted to them, which returns at once when nobody fell back
        fb_launches = (history >> 16) != 0;         // any of the last 15 steps
        // Rounds after round 1 likewise: that single kernel takes them, too, unless it met one lately, and says so in the second pinned word (a pair of launches
        // that return at once takes 4-6 us: steps with max_rounds = 4, 203 sequences at C = 294 78.7 -> 69.5 us, 232 at C = 1054 157 -> 139; a round
        // inside it costs two grid barriers, so it is tried again after DEEP_HOLD steps only).
        volatile int* met = ws->h_history + 1;
        if (*met) {
            *met = 0;
            ws->deep_hold = DEEP_HOLD;
        }
        deep = fb_launches || ws->deep_hold > 0;
        if (split && max_rounds > 2 && ws->deep_hold > 0) --ws->deep_hold;
    }
    // blocks per sequence in round 0: as many as stay resident together (a second wave of blocks would double the
    // kernel's time), at most ROUND0_NB_MAX, and no more than the largest possible seed prefix needs at
    // ROUND0_ROWS_PER_BLOCK rows a block (max(k,1) - 1 rows before its last cluster plus that cluster)
    const long long prefix_max = (long long)(p->k > 1 ? p->k : 1) - 1 + idx->n_max;
    int nb = ws->round0_capacity / B;
    nb = nb < 1 ? 1 : (nb > ROUND0_NB_MAX ? ROUND0_NB_MAX : nb);
    {
        const long long want = (prefix_max + ROUND0_ROWS_PER_BLOCK - 1) / ROUND0_ROWS_PER_BLOCK;
        if (want < nb) nb = (int)(want < 1 ? 1 : want);
    }
    // the tail's blocks ride in the round-0 launch when they all fit next to the round-0 blocks (one block per unit)
    const bool fused = !split && ws->fused_ok && nb * B * 2 <= ws->tail_grid;
    if (fused) {
        if (B > FULL_G) step_kernel<true><<<ws->tail_grid, SEQ_THREADS, ws->fused_lds, st>>>(a, f, nb);
        else step_kernel<false><<<ws->tail_grid, SEQ_THREADS, ws->fused_lds, st>>>(a, f, nb);
        CSV_LAUNCH_CHECK("step_kernel");
    } else {
        // Plans are made where recent steps needed later rounds; lists of more than RANK_DIRECT rows only where a seed prefix can
        // be that long (5 sequences certified on 478 rows each: 53 us without the threshold selection, 30 with it).
        if (split) round0_kernel<true, true><<<nb * B, SEQ_THREADS, round0_lds(ws), st>>>(a, nb);
        else if (prefix_max > RANK_DIRECT) round0_kernel<true, false><<<nb * B, SEQ_THREADS, round0_lds(ws), st>>>(a, nb);
        else round0_kernel<false, false><<<nb * B, SEQ_THREADS, round0_lds(ws), st>>>(a, nb);
        CSV_LAUNCH_CHECK("round0_kernel");
    }
    CSV_MARK(2);
    if (!fused) {
        if (!split) {
            // one launch that returns at once when no sequence needs it
            tail_kernel<<<ws->tail_grid, TAIL_THREADS, ws->tail_lds, st>>>(a, f, 0);
            CSV_LAUNCH_CHECK("tail_kernel");
        } else {
            const size_t hl = (size_t)2 * idx->d * 2;
            // Round 0 appears here only for seed prefixes that the round-0 kernel hands over.  A prefix holds fewer
            // than max(k,1) rows before its last cluster, so with small clusters that cannot happen: no launches.
            const long long cap = (long long)nb * (SEQ_THREADS / 64) * ROUND0_ROWS_PER_WAVE;
            const bool may_hand_over = prefix_max > (cap < STAGE_CAP ? cap : STAGE_CAP) || (idx->d >> 3) > ROUND0_HREG * SEQ_THREADS;
            const int launched = deep ? max_rounds : 2;          // rounds before this one are launches of their own
            for (int r = may_hand_over ? 0 : 1; r < launched; ++r) {
                round_gemv_kernel<<<ws->tail_grid, TAIL_THREADS, hl, st>>>(a, r);   // more blocks measured slower
                CSV_LAUNCH_CHECK("round_gemv_kernel");
                round_cert_kernel<<<dim3(B, ws->sp_chunks), SEQ_THREADS, cert_lds(ws), st>>>(a, r);
                CSV_LAUNCH_CHECK("round_cert_kernel");
            }
            if (fb_launches) {
                if (B > FULL_G) {
                    launch_fb_product_mfma(ws->tail_grid, a, f, st);
                    CSV_LAUNCH_CHECK("fb_product_mfma_kernel");
                } else {
                    fb_product_kernel<<<ws->tail_grid, TAIL_THREADS, (size_t)FULL_G * idx->d * 2, st>>>(a, f);
                    CSV_LAUNCH_CHECK("fb_product_kernel");
                }
                fb_topk_kernel<<<dim3(ws->n_chunks, B), SEQ_THREADS, (size_t)CAND_OFF + CAND_BYTES, st>>>(a);
                CSV_LAUNCH_CHECK("fb_topk_kernel");
                fb_final_kernel<<<B, SEQ_THREADS, (size_t)CAND_OFF + CAND_BYTES, st>>>(a);
                CSV_LAUNCH_CHECK("fb_final_kernel");
            } else {
                tail_kernel<<<ws->tail_grid, TAIL_THREADS, ws->tail_lds, st>>>(a, f, launched < max_rounds ? launched : CSV_MAX_ROUNDS);
                CSV_LAUNCH_CHECK("tail_kernel");
            }
        }
    }
    CSV_MARK(3);
#undef CSV_MARK
    return CSV_OK;
}

extern "C" int csv_workspace_set_tail_split(csv_workspace* ws, int min_batch) {
    if (!ws) { csv_set_error("null workspace"); return CSV_EINVAL; }
    if (min_batch < 0) { csv_set_error("min_batch=%d is negative", min_batch); return CSV_EINVAL; }
    ws->split_min_B = min_batch;
    return CSV_OK;
}

extern "C" int csv_workspace_set_spin_limit(csv_workspace* ws, int polls) {
    if (!ws) { csv_set_error("null workspace"); return CSV_EINVAL; }
    if (polls < 0) { csv_set_error("polls=%d is negative", polls); return CSV_EINVAL; }
    ws->spin_limit = polls == 0 ? TAIL_SPIN_LIMIT : polls;
    return CSV_OK;
}

// ------------------------------------------------------------------------------------------------ stage timing
static void profile_release(csv_workspace* ws) {
    if (ws->prof_ev) {
        for (size_t i = 0; i < (size_t)ws->prof_cap * (CSV_PROFILE_STAGES + 1); ++i)
            if (ws->prof_ev[i]) (void)hipEventDestroy(ws->prof_ev[i]);
        free(ws->prof_ev);
    }
    ws->prof_ev = nullptr;
    ws->prof_cap = ws->prof_n = ws->prof_on = 0;
}

extern "C" int csv_profile_begin(csv_workspace* ws, int max_steps) {
    if (!ws || max_steps < 1 || max_steps > (1 << 16)) { csv_set_error("bad workspace or max_steps"); return CSV_EINVAL; }
    profile_release(ws);
    const size_t n = (size_t)max_steps * (CSV_PROFILE_STAGES + 1);
    ws->prof_ev = (hipEvent_t*)calloc(n, sizeof(hipEvent_t));
    if (!ws->prof_ev) { csv_set_error("host allocation failed"); return CSV_ENOMEM; }
    ws->prof_cap = max_steps;
    for (size_t i = 0; i < n; ++i) {
        hipError_t e = hipEventCreate(&ws->prof_ev[i]);
        if (e != hipSuccess) {
            csv_set_error("hipEventCreate failed: %s", hipGetErrorString(e));
            profile_release(ws);
            return CSV_EHIP;
        }
    }
    ws->prof_on = 1;
    return CSV_OK;
}

extern "C" int csv_profile_end(csv_workspace* ws, float* h_stage_ms, int* h_steps) {
    if (!ws || !h_stage_ms || !h_steps) { csv_set_error("null argument"); return CSV_EINVAL; }
    for (int i = 0; i < CSV_PROFILE_STAGES; ++i) h_stage_ms[i] = 0.f;
    *h_steps = ws->prof_n;
    int rc = CSV_OK;
    for (int s = 0; s < ws->prof_n && rc == CSV_OK; ++s) {
        hipEvent_t* ev = ws->prof_ev + (size_t)s * (CSV_PROFILE_STAGES + 1);
        hipError_t e = hipEventSynchronize(ev[CSV_PROFILE_STAGES]);
        for (int i = 0; i < CSV_PROFILE_STAGES && e == hipSuccess; ++i) {
            float ms = 0.f;
            e = hipEventElapsedTime(&ms, ev[i], ev[i + 1]);
            h_stage_ms[i] += ms;
        }
        if (e != hipSuccess) {
            csv_set_error("event timing failed: %s", hipGetErrorString(e));
            rc = CSV_EHIP;
        }
    }
    profile_release(ws);
    return rc;
}

// ------------------------------------------------------------------------------------------------ adaptive budget
extern "C" int csv_kmax_init(csv_kmax_ctl* c, int K0, int K_min, int K_cap, double alpha, double rho_target, int literal) {
    if (!c) { csv_set_error("null controller"); return CSV_EINVAL; }
    if (K_min < 0 || K_cap < K_min || K0 < K_min || K0 > K_cap) { csv_set_error("need 0 <= K_min <= K0 <= K_cap (got %d, %d, %d)", K_min, K0, K_cap); return CSV_EINVAL; }
    if (!(alpha >= 0.0) || !(rho_target >= 0.0 && rho_target <= 1.0)) { csv_set_error("bad alpha=%g or rho_target=%g", alpha, rho_target); return CSV_EINVAL; }
    c->K_max = (double)K0; c->alpha = alpha; c->rho_target = rho_target; c->K_min = K_min; c->K_cap = K_cap; c->literal = literal != 0;
    return CSV_OK;
}

extern "C" int csv_kmax_update(csv_kmax_ctl* c, int n_fallback, int n_sequences) {
    if (!c) { csv_set_error("null controller"); return CSV_EINVAL; }
    if (n_sequences < 1 || n_fallback < 0 || n_fallback > n_sequences) { csv_set_error("bad counts %d of %d", n_fallback, n_sequences); return CSV_EINVAL; }
    const double rho = (double)n_fallback / (double)n_sequences;
    const double err = c->literal ? (c->rho_target - rho) : (rho - c->rho_target);
    double K = c->K_max * (1.0 + c->alpha * err);
    // the state itself stays inside the range, so a long run at one end does not have to be unwound
    if (K < (double)c->K_min) K = (double)c->K_min;
    if (K > (double)c->K_cap) K = (double)c->K_cap;
    c->K_max = K;
    return (int)floor(K);
}

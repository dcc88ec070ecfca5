// Offline preprocessing: Lloyd's k-means over the rows of W, cluster metadata (centroid, radius, bias maximum)
// and the row permutation that makes every cluster contiguous (Section III-A.1; Section IV "Offline Preprocessing").
// Off the per-step hot path.  Everything stays on the device until the metadata is done; float64 accumulation for the metadata.
#include "csv_common.h"

#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <type_traits>
#include <vector>

// ------------------------------------------------------------------------------------------------ kernels
// W'[r] = W[perm[r]], b'[r] = b[perm[r]] (0 without bias).  One block per permuted row.
__global__ __launch_bounds__(256) void gather_rows_kernel(const uint16_t* __restrict__ W, const float* __restrict__ b,
                                                          const int32_t* __restrict__ perm, int V, int d,
                                                          uint16_t* __restrict__ Wp, float* __restrict__ bp) {
    const int r = blockIdx.x;
    if (r >= V) return;
    const int src = perm[r];
    const uint4* s = reinterpret_cast<const uint4*>(W + (size_t)src * d);
    uint4* t = reinterpret_cast<uint4*>(Wp + (size_t)r * d);
    for (int i = threadIdx.x; i < (d >> 3); i += 256) t[i] = s[i];
    if (threadIdx.x == 0) bp[r] = b ? b[src] : 0.f;
}

// ------------------------------------------------------------------------------------------------ labels -> layout
// Sizes, offsets and the permutation from the labels (clusters in id order, tokens by ascending id inside a cluster), on
// the device: the build of an index then has no copy to the host and no wait between its iterations.  A stable counting
// sort: one wave per LAY_TOKENS tokens counts its labels, the counts are summed up per cluster over the waves, and the same
// wave places its tokens in order.  All of it is latency (V = 128256, C = 1024: four launches, 40 us in all; the copy of the labels, the host's
// sort and three copies back took 0.4 ms).
#define LAY_TOKENS 512
// hist[wave][c] = its tokens of cluster c.  cand != NULL: the labels are made here, as the smallest word over the
// assignment's column blocks (equal distances: the smaller cluster id is the smaller word).  A negative label ~i stands for
// the cluster in the low half of win[i] (rows whose nearest centroid took a second look).
__global__ __launch_bounds__(64) void label_hist_kernel(const unsigned long long* __restrict__ cand, int ncol, const unsigned long long* __restrict__ win,
                                                        int32_t* __restrict__ labels, int V,
                                                        int C, int32_t* __restrict__ hist) {
    extern __shared__ int32_t lay_cnt[];
    const int lane = threadIdx.x, base = blockIdx.x * LAY_TOKENS;
    for (int c = lane; c < C; c += 64) lay_cnt[c] = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < LAY_TOKENS / 64; ++i) {
        const int t = base + lane + 64 * i;
        if (t < V) {
            int l;
            if (cand) {
                unsigned long long x = cand[t];
                for (int q = 1; q < ncol; ++q) {
                    const unsigned long long y = cand[(size_t)q * V + t];
                    x = y < x ? y : x;
                }
                l = (int)(unsigned)x;
                labels[t] = l;
            } else {
                l = labels[t];
                if (l < 0) {
                    l = (int)(unsigned)win[~l];
                    labels[t] = l;
                }
            }
            atomicAdd(&lay_cnt[l], 1);
        }
    }
    __syncthreads();
    for (int c = lane; c < C; c += 64) hist[(size_t)blockIdx.x * C + c] = lay_cnt[c];
}

// hist[w][c] becomes the tokens of cluster c before wave w; n[c] their number.  64 clusters per block, a segment of the waves per wave.
__global__ __launch_bounds__(512) void layout_scan_kernel(int32_t* __restrict__ hist, int nw, int C, int32_t* __restrict__ n) {
    __shared__ int32_t seg_sum[8][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c = blockIdx.x * 64 + lane;
    const int seg = (nw + 7) / 8, w0 = min(nw, wave * seg), w1 = min(nw, w0 + seg);
    int sum = 0;
    if (c < C)
#pragma unroll 8
        for (int w = w0; w < w1; ++w) sum += hist[(size_t)w * C + c];
    seg_sum[wave][lane] = sum;
    __syncthreads();
    int run = 0, total = 0;
    for (int q = 0; q < 8; ++q) {
        if (q < wave) run += seg_sum[q][lane];
        total += seg_sum[q][lane];
    }
    if (c >= C) return;
#pragma unroll 8
    for (int w = w0; w < w1; ++w) {
        const int x = hist[(size_t)w * C + c];
        hist[(size_t)w * C + c] = run;
        run += x;
    }
    if (wave == 0) n[c] = total;
}

// off, and the list of row chunks of the centroid and distance passes: chunks[i] = {cluster, first permuted row}, coff[c] =
// first chunk of cluster c, coff[C] = their number; poff[c] = the partial sums of cluster c's chunks, which only clusters of several
// have (PART_SLOTS of them at most).  One block.
#define CHUNK_ROWS 128
// a cluster of n > CHUNK_ROWS rows has at most n / CHUNK_ROWS + 1 chunks, and there are at most V / (CHUNK_ROWS + 1) such clusters
#define PART_SLOTS(V) ((V) / CHUNK_ROWS + (V) / (CHUNK_ROWS + 1) + 1)
__global__ __launch_bounds__(1024) void layout_offsets_kernel(const int32_t* __restrict__ n, int C, int32_t* __restrict__ off,
                                                              int32_t* __restrict__ coff, int32_t* __restrict__ poff, int2* __restrict__ chunks) {
    __shared__ int32_t ws[3][16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int per = (C + 1023) / 1024, c0 = min(C, tid * per), c1 = min(C, c0 + per);
    int rows = 0, nch = 0, nparts = 0;
    for (int c = c0; c < c1; ++c) {
        const int m = (n[c] + CHUNK_ROWS - 1) / CHUNK_ROWS;
        rows += n[c];
        nch += m;
        nparts += m > 1 ? m : 0;
    }
    int x = rows, y = nch, z = nparts;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int xx = __shfl_up(x, o, CSV_WAVE), yy = __shfl_up(y, o, CSV_WAVE), zz = __shfl_up(z, o, CSV_WAVE);
        if (lane >= o) {
            x += xx;
            y += yy;
            z += zz;
        }
    }
    if (lane == 63) {
        ws[0][wave] = x;
        ws[1][wave] = y;
        ws[2][wave] = z;
    }
    __syncthreads();
    x -= rows;
    y -= nch;
    z -= nparts;
    for (int q = 0; q < wave; ++q) {
        x += ws[0][q];
        y += ws[1][q];
        z += ws[2][q];
    }
    for (int c = c0; c < c1; ++c) {
        off[c] = x;
        coff[c] = y;
        poff[c] = z;
        if (n[c] > CHUNK_ROWS) z += (n[c] + CHUNK_ROWS - 1) / CHUNK_ROWS;
        for (int r = 0; r < n[c]; r += CHUNK_ROWS) chunks[y++] = make_int2(c, x + r);
        x += n[c];
    }
    if (c1 == C && c0 < C) {
        off[C] = x;
        coff[C] = y;
    }
}

__global__ __launch_bounds__(64) void layout_scatter_kernel(const int32_t* __restrict__ labels, const int32_t* __restrict__ hist,
                                                            const int32_t* __restrict__ off, int V, int C, int label_bits,
                                                            int32_t* __restrict__ perm) {
    extern __shared__ int32_t lay_cnt[];                     // next permuted row of each cluster
    const int lane = threadIdx.x, base = blockIdx.x * LAY_TOKENS;
    for (int c = lane; c < C; c += 64) lay_cnt[c] = off[c] + hist[(size_t)blockIdx.x * C + c];
    __syncthreads();
    for (int i = 0; i < LAY_TOKENS / 64; ++i) {
        const int t = base + lane + 64 * i;
        const bool in = t < V;
        const int l = in ? labels[t] : 0;
        unsigned long long same = __ballot(in);              // the lanes with this lane's label
        for (int bit = 0; bit < label_bits; ++bit) {
            const bool one = (l >> bit) & 1;
            const unsigned long long m = __ballot(one);
            same &= one ? m : ~m;
        }
        const int before = __popcll(same & ((1ull << lane) - 1ull));
        const int pos = lay_cnt[l] + before;
        __syncthreads();                                     // every lane has read its counter
        if (in) {
            perm[pos] = t;
            if (before == 0) lay_cnt[l] = pos + __popcll(same);
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------------------------------------------ centroids
// Sums of the rows of W of one chunk (at most CHUNK_ROWS rows of one cluster, read through the permutation: the gathered
// copy is made once, after the last iteration), in float64.  Block = 4 waves x 512 columns; a wave takes every fourth
// row, eight rows requested at once; the waves' sums are added in wave order.  A cluster of one chunk is finished here, the
// chunks of a larger one leave partial sums for centroid_finish_kernel, so a cluster of any size is spread over the device.
// Bound by reading W: V = 128256, d = 4096 in 208 us = 5.05 TB/s, with the blocks of one chunk side by side.  (With those of one column slice side by side
// 215 us; one thread per column going down all rows of a cluster 1.7 ms with clusters of up to 2900 rows, and 0.38 ms for a gathered copy per iteration.)
// UNIT (spherical clustering): rows are divided by their norm nrm[token], the sums themselves go to out_sum.
template <bool UNIT>
__global__ __launch_bounds__(256) void centroid_chunk_kernel(const uint16_t* __restrict__ W, const int32_t* __restrict__ perm, const int32_t* __restrict__ off,
                                                             const int32_t* __restrict__ coff, const int32_t* __restrict__ poff, const int2* __restrict__ chunks, int d, int C, int nslices,
                                                             const double* __restrict__ nrm, float* __restrict__ mu, double* __restrict__ out_sum,
                                                             double* __restrict__ part) {
    __shared__ double red[4][8][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, chunk = blockIdx.x / nslices;
    if (chunk >= coff[C]) return;
    const int c = chunks[chunk].x, r0 = chunks[chunk].y;
    const int first = off[c], last = off[c + 1], rows = min(CHUNK_ROWS, last - r0);
    const int piece = (blockIdx.x - chunk * nslices) * 64 + lane, np = d >> 3;
    const int mine = (rows - wave + 3) / 4;                  // rows r0 + wave, r0 + wave + 4, ...
    const int token = lane < mine ? perm[r0 + wave + 4 * lane] : 0;
    double acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.0;
    const uint4* w = reinterpret_cast<const uint4*>(W) + min(piece, np - 1);
    auto add = [&](const uint4& x, int tok) {
        const double nr = UNIT ? nrm[tok] : 1.0;
        const uint32_t xs[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const double v = (double)__uint_as_float(e & 1 ? xs[e >> 1] & 0xffff0000u : xs[e >> 1] << 16);
            acc[e] += UNIT && nr > 0.0 ? v / nr : v;
        }
    };
    int i = 0;
    for (; i + 8 <= mine; i += 8) {
        uint4 x[8];
        int tk[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            tk[q] = __builtin_amdgcn_readlane(token, i + q);
            x[q] = w[(size_t)tk[q] * np];
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) add(x[q], tk[q]);
    }
    if (i < mine) {                                          // the last few together, too: one by one they took as long as all before
        uint4 x[8];
        int tk[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            tk[q] = __builtin_amdgcn_readlane(token, min(i + q, mine - 1));
            x[q] = w[(size_t)tk[q] * np];
        }
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (i + q < mine) add(x[q], tk[q]);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) red[wave][e][lane] = acc[e];
    __syncthreads();
    if (piece >= np) return;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int e = 2 * wave + q, col = piece * 8 + e;
        const double sum = ((red[0][e][lane] + red[1][e][lane]) + red[2][e][lane]) + red[3][e][lane];
        if (last - first > CHUNK_ROWS) part[(size_t)(poff[c] + chunk - coff[c]) * d + col] = sum;
        else if (UNIT) out_sum[(size_t)c * d + col] = sum;
        else mu[(size_t)c * d + col] = (float)(sum / (double)rows);
    }
}

// Clusters of several chunks: the partial sums, in chunk order.  An empty cluster keeps its centroid (Lloyd) or is zeroed
// (final metadata; direction_finish_kernel does that for directions).
template <bool UNIT>
__global__ __launch_bounds__(256) void centroid_finish_kernel(const int32_t* __restrict__ off, const int32_t* __restrict__ poff, int d, int zero_empty,
                                                              const double* __restrict__ part, float* __restrict__ mu, double* __restrict__ out_sum) {
    const int c = blockIdx.x, n = off[c + 1] - off[c];
    const int col = blockIdx.y * 256 + threadIdx.x;
    if (col >= d) return;
    if (n == 0 && zero_empty && !UNIT) mu[(size_t)c * d + col] = 0.f;
    if (n <= CHUNK_ROWS) return;
    double sum = 0.0;
#pragma unroll 4
    for (int q = 0; q < (n + CHUNK_ROWS - 1) / CHUNK_ROWS; ++q) sum += part[(size_t)(poff[c] + q) * d + col];
    if (UNIT) out_sum[(size_t)c * d + col] = sum;
    else mu[(size_t)c * d + col] = (float)(sum / (double)n);
}

__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, CSV_WAVE);
    return v;
}

// R_c = max_i ||W_i - mu_c||_2 to the stored float32 centroid, in float64; stored radius
// roundup_f32(R_c (1+rho) + rho ||mu_c||); bias maximum; ln n_c.
// Pass 1, together with the gathered copy W'[r] = W[perm[r]], b'[r] = b[perm[r]] (0 without bias), so that W is read once:
// one block per chunk, one wave per row: squared distance in float64, folded into d2max[c] with an integer atomic max
// (non-negative doubles order like their bit patterns).  A row passes through the wave in batches of four 128-bit loads.
// Bound by reading W and writing W': V = 128256, d = 4096 in 495 us (separate passes: 380 + 305 us).
__global__ __launch_bounds__(256) void gather_dist_kernel(const uint16_t* __restrict__ W, const float* __restrict__ b, const int32_t* __restrict__ perm,
                                                          const int32_t* __restrict__ off, const int32_t* __restrict__ coff, const int2* __restrict__ chunks,
                                                          const float* __restrict__ mu, int d, int C, uint16_t* __restrict__ Wp, float* __restrict__ bp,
                                                          unsigned long long* __restrict__ d2max, double* __restrict__ d2row) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, chunk = blockIdx.x >> 2;
    if (chunk >= coff[C]) return;
    const int c = chunks[chunk].x, r0 = chunks[chunk].y, r1 = min(r0 + CHUNK_ROWS, off[c + 1]), np = d >> 3;
    const float4* m = reinterpret_cast<const float4*>(mu + (size_t)c * d);
    unsigned long long most = 0ull;                          // bit pattern: a row with NaN or infinity keeps its cluster's radius from being finite
    // a quarter of the chunk's rows per block, every fourth of those per wave
    for (int r = r0 + (blockIdx.x & 3) * 4 + wave; r < r1; r += 16) {
        const int src = perm[r];
        const uint4* w = reinterpret_cast<const uint4*>(W + (size_t)src * d);
        uint4* o = reinterpret_cast<uint4*>(Wp + (size_t)r * d);
        double acc = 0.0;
        for (int q0 = lane; q0 < np; q0 += 256) {
            uint4 x[4];
            float4 m0[4], m1[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int q = min(q0 + 64 * i, np - 1);
                x[i] = w[q];
                m0[i] = m[2 * q];
                m1[i] = m[2 * q + 1];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (q0 + 64 * i >= np) break;
                o[q0 + 64 * i] = x[i];
                const uint32_t xs[4] = {x[i].x, x[i].y, x[i].z, x[i].w};
                const float ms[8] = {m0[i].x, m0[i].y, m0[i].z, m0[i].w, m1[i].x, m1[i].y, m1[i].z, m1[i].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double d0 = (double)__uint_as_float(xs[e] << 16) - (double)ms[2 * e];
                    const double d1 = (double)__uint_as_float(xs[e] & 0xffff0000u) - (double)ms[2 * e + 1];
                    acc = fma(d0, d0, acc);
                    acc = fma(d1, d1, acc);
                }
            }
        }
        acc = wave_sum_d(acc);
        const unsigned long long bits = (unsigned long long)__double_as_longlong(acc);
        most = bits > most ? bits : most;
        if (lane == 0) {
            bp[r] = b ? b[src] : 0.f;
            if (d2row) d2row[r] = acc;      // squared distance of every row, for the bias table
        }
    }
    if (lane == 0) atomicMax(&d2max[c], most);
}

// Top-m bias table of one cluster (one block per cluster): the m-1 rows with the largest bias (equal biases: the
// earlier permuted row, i.e. the smaller token id) get entries of their own (distance to the centroid, bias); the
// remaining rows share one entry (their largest distance, their largest bias).  Radii are stored like R_c:
// roundup_f32(r (1+rho) + rho ||mu_c||).  Unused entries are (0, -inf).
__global__ __launch_bounds__(256) void bias_table_kernel(const float* __restrict__ bp, const int32_t* __restrict__ off,
                                                         const float* __restrict__ mu, int d, double rho, int m,
                                                         const double* __restrict__ d2row, float2* __restrict__ bt) {
    __shared__ float sb[256];
    __shared__ int si[256];
    __shared__ double sd[256];
    __shared__ int picked[CSV_MAX_BIAS_TABLE];
    __shared__ double mun;
    const int c = blockIdx.x, tid = threadIdx.x;
    const int r0 = off[c], r1 = off[c + 1], n = r1 - r0;
    float2* out = bt + (size_t)c * m;
    for (int j = tid; j < m; j += 256) out[j] = make_float2(0.f, -INFINITY);
    if (n == 0) return;
    {
        double acc = 0.0;
        for (int j = tid; j < d; j += 256) acc += (double)mu[(size_t)c * d + j] * (double)mu[(size_t)c * d + j];
        sd[tid] = acc;
        __syncthreads();
        for (int o = 128; o > 0; o >>= 1) {
            if (tid < o) sd[tid] += sd[tid + o];
            __syncthreads();
        }
        if (tid == 0) mun = sqrt(sd[0]);
        __syncthreads();
    }
    auto store = [&](int slot, double d2, float bias) {
        const double x = sqrt(d2) * (1.0 + rho) + rho * mun;
        float y = (float)x;
        if ((double)y < x) y = nextafterf(y, INFINITY);
        out[slot] = make_float2(y, bias);
    };
    const int ne = min(m - 1, n);
    for (int e = 0; e < ne; ++e) {
        // arg-max of (bias, -row) over the rows not picked yet
        float bb = -INFINITY;
        int bi = 0x7fffffff;
        for (int r = r0 + tid; r < r1; r += 256) {
            bool taken = false;
            for (int q = 0; q < e; ++q) taken |= picked[q] == r;
            const float v = bp[r];
            if (!taken && (v > bb || (v == bb && r < bi))) {
                bb = v;
                bi = r;
            }
        }
        sb[tid] = bb;
        si[tid] = bi;
        __syncthreads();
        for (int o = 128; o > 0; o >>= 1) {
            if (tid < o) {
                const float v = sb[tid + o];
                const int i = si[tid + o];
                if (v > sb[tid] || (v == sb[tid] && i < si[tid])) {
                    sb[tid] = v;
                    si[tid] = i;
                }
            }
            __syncthreads();
        }
        if (tid == 0) {
            picked[e] = si[0];
            store(e, d2row[si[0]], sb[0]);
        }
        __syncthreads();
    }
    if (n > ne) {       // the rest: largest distance and largest bias among the rows not picked
        float bb = -INFINITY;
        double dd = 0.0;
        for (int r = r0 + tid; r < r1; r += 256) {
            bool taken = false;
            for (int q = 0; q < ne; ++q) taken |= picked[q] == r;
            if (!taken) {
                bb = fmaxf(bb, bp[r]);
                dd = fmax(dd, d2row[r]);
            }
        }
        sb[tid] = bb;
        sd[tid] = dd;
        __syncthreads();
        for (int o = 128; o > 0; o >>= 1) {
            if (tid < o) {
                sb[tid] = fmaxf(sb[tid], sb[tid + o]);
                sd[tid] = fmax(sd[tid], sd[tid + o]);
            }
            __syncthreads();
        }
        if (tid == 0) store(ne, sd[0], sb[0]);
    }
}

// Pass 2, one block per cluster: bias maximum, ||mu_c||, the stored radius and ln n_c.
__global__ __launch_bounds__(256) void radius_finish_kernel(const float* __restrict__ bp, const int32_t* __restrict__ off,
                                                            const float* __restrict__ mu, int d, double rho,
                                                            const unsigned long long* __restrict__ d2max,
                                                            float* __restrict__ R, float* __restrict__ bmax,
                                                            float* __restrict__ lnn) {
    __shared__ float wb[4];
    __shared__ double wm[4];
    const int c = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r0 = off[c], r1 = off[c + 1];
    const float* m = mu + (size_t)c * d;
    float bm = -INFINITY;
    for (int r = r0 + tid; r < r1; r += 256) bm = fmaxf(bm, bp[r]);
    bm = wave_max(bm);
    double acc = 0.0;
    for (int j = tid; j < d; j += 256) acc += (double)m[j] * (double)m[j];
    acc = wave_sum_d(acc);
    if (lane == 0) {
        wb[wave] = bm;
        wm[wave] = acc;
    }
    __syncthreads();
    if (tid == 0) {
        const int n = r1 - r0;
        if (n == 0) {
            R[c] = 0.f;
            bmax[c] = -INFINITY;
            lnn[c] = -INFINITY;
        } else {
            const double mun2 = (wm[0] + wm[1]) + (wm[2] + wm[3]);
            const double d2 = __longlong_as_double((long long)d2max[c]);
            const double x = sqrt(d2) * (1.0 + rho) + rho * sqrt(mun2);
            float y = (float)x;
            if ((double)y < x) y = nextafterf(y, INFINITY);
            R[c] = y;
            bmax[c] = fmaxf(fmaxf(wb[0], wb[1]), fmaxf(wb[2], wb[3]));
            lnn[c] = (float)log((double)n);
        }
    }
}

// Lloyd assignment: labels[i] = argmin_c ||W_i - mu_c||^2, ties to the smaller cluster id.
// ||W_i - mu_c||^2 = ||W_i||^2 - 2 <W_i,mu_c> + ||mu_c||^2 and the first term does not depend on c, so the work is the
// dense contraction [V x d] . [d x C].  W is bf16, the centroids are float32: split exactly into three bf16 pieces, three MFMAs
// per k-block give exact products (assign_exact_kernel), at three times the matrix work of bf16 centroids.
// One piece settles nearly every row: with mu_c rounded to bf16 a score is off by at most 2 ||W_i|| ||mu_c - bf16(mu_c)|| and what the float32 sums
// differ by (round_centroids_kernel), and only centroids within twice that of the best can be the nearest.  So, where there is enough work to pay for the passes
// (assign_near_pays): round_centroids_kernel rounds the centroids and measures what the rounding left out; assign_near_kernel scores
// all pairs with the rounded ones and keeps, per row and group of clusters, the three best; assign_pick_kernel labels the rows with one
// centroid in reach and lists the others' pairs, which assign_pairs_kernel scores exactly; rows with many in reach, or
// whose reach is not finite, go to assign_exact_kernel.  An exact score is one sum in one order (k-blocks ascending, a value's
// pieces one after the other) wherever it is taken, so the labels are the same whichever way they were found.
// Rows with more than one in reach: 20 % where clusters were planted and some share their seeds or have none, 0.2-6 % of heads
// without or with blurred clusters (V = 16384, d = 1024 and 4096, C = 256 and 512), 2.0-2.4 centroids each.
// V = 128256, d = 4096, C = 1024: 1.01 ms an assignment (0.80 the rounded scores, 0.03 the look through them, 0.16 the pairs, 0.02 the rest), the
// exact product over all rows 2.35.
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 as_bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float as_floatx4_t;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t as_uintx4_t;     // a 16-byte piece in registers (uint4 arrays held across the loop went to scratch)
#define CSV_ANGLE_SLACK (1.0 / 4096.0)     // added to every angular radius (radians), next to the relative slack
#define AS_THREADS 512

__device__ __forceinline__ uint32_t as_tops(float lo, float hi) {         // the upper halves of two floats in one word
    return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
}
// v = hi + mid + lo, three bf16 values that add up to v exactly; what is cut off is never rounded, so the halves need no masks
__device__ __forceinline__ void as_split3(const float4& x0, const float4& x1, uint4& hi, uint4& mid, uint4& lo) {
    const float v[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
    float r1[8], r2[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        r1[i] = v[i] - __uint_as_float(__float_as_uint(v[i]) & 0xffff0000u);
        r2[i] = r1[i] - __uint_as_float(__float_as_uint(r1[i]) & 0xffff0000u);
    }
    hi = make_uint4(as_tops(v[0], v[1]), as_tops(v[2], v[3]), as_tops(v[4], v[5]), as_tops(v[6], v[7]));
    mid = make_uint4(as_tops(r1[0], r1[1]), as_tops(r1[2], r1[3]), as_tops(r1[4], r1[5]), as_tops(r1[6], r1[7]));
    lo = make_uint4(as_tops(r2[0], r2[1]), as_tops(r2[2], r2[3]), as_tops(r2[4], r2[5]), as_tops(r2[6], r2[7]));
}
// minimum over the 16 lanes of a DPP row (lanes 16g .. 16g+15); every lane of the row gets it
__device__ __forceinline__ unsigned row16_min_u(unsigned v) {
    v = min(v, (unsigned)dpp_move<0xB1, 0xf>((int)v, (int)v));    // quad_perm [1,0,3,2]
    v = min(v, (unsigned)dpp_move<0x4E, 0xf>((int)v, (int)v));    // quad_perm [2,3,0,1]
    v = min(v, (unsigned)dpp_move<0x141, 0xf>((int)v, (int)v));   // row_half_mirror
    v = min(v, (unsigned)dpp_move<0x140, 0xf>((int)v, (int)v));   // row_mirror
    return v;
}

// ||mu_c||^2.  The sum is that of round_centroids_kernel: 512 partial sums, value k to the partial sum k % 512, which meet as a binary
// tree, neighbours first.
// unit != 0 (spherical clustering): every direction counts as of length one, so the arg-min is the largest cosine
__global__ __launch_bounds__(512) void centroid_norm_kernel(const float* __restrict__ mu, int d, int unit, float* __restrict__ cn) {
    __shared__ double red[8];
    const int c = blockIdx.x, tid = threadIdx.x;
    if (unit) {
        if (tid == 0) cn[c] = 1.f;
        return;
    }
    double acc = 0.0;
    for (int j = tid; j < d; j += 512) acc = fma((double)mu[(size_t)c * d + j], (double)mu[(size_t)c * d + j], acc);
#pragma unroll
    for (int o = 1; o < CSV_WAVE; o <<= 1) acc += __shfl_xor(acc, o, CSV_WAVE);
    if ((tid & 63) == 0) red[tid >> 6] = acc;
    __syncthreads();
    if (tid == 0) cn[c] = (float)(((red[0] + red[1]) + (red[2] + red[3])) + ((red[4] + red[5]) + (red[6] + red[7])));
}

// The three bf16 pieces of every centroid value in fragment order: out[((kb * CT + ct) * 3 + piece) * 64 + lane], lane =
// 16 g + li: cluster 16 ct + li, the eight k values 32 kb + 8 g ...; zero past C and past d.  One wave per (kb, ct).  needed: nothing is done where it counts nothing.
__global__ __launch_bounds__(256) void split_centroids_kernel(const float* __restrict__ mu, int d, int C, int CT, int nkb, const int* __restrict__ needed, uint4* __restrict__ out) {
    const int lane = threadIdx.x & 63;
    const int ct = blockIdx.x, kb = blockIdx.y * 4 + (threadIdx.x >> 6);
    if (kb >= nkb || (needed && *needed == 0)) return;
    const int c = ct * 16 + (lane & 15), k = kb * 32 + (lane >> 4) * 8;
    uint4 hi = make_uint4(0, 0, 0, 0), mid = hi, lo = hi;
    if (c < C && k < d) {                                    // d is a multiple of 8: the eight values are all in or all out
        const float4* src = reinterpret_cast<const float4*>(mu + (size_t)c * d + k);
        as_split3(src[0], src[1], hi, mid, lo);
    }
    uint4* o = out + ((size_t)kb * CT + ct) * 192 + lane;
    o[0] = hi;
    o[64] = mid;
    o[128] = lo;
}

// All LDS accesses of the block's waves are done; global loads stay in flight.
__device__ __forceinline__ void as_lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int N, int I = 0, class F>
__device__ __forceinline__ void as_for(F f) {              // f(0), f(1), ... with the index as a constant
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        as_for<N, I + 1>(f);
    }
}

// The exact scores of rows against all centroids.  The centroids' pieces are split once per assignment (split_centroids_kernel): they lie in
// fragment order, [k-block of 32][cluster tile of 16][piece][lane], so that a block's share of a k-block is one run.
// Block = 8 waves, 2 (rows) x 4 (clusters); a wave owns 16 MT rows x 16 NT clusters in accumulators over the whole of K.
// Both operands go through LDS in fragment order (1 KB reads, no bank conflicts), one k-block per stage, two stages:
// while a stage is consumed the next one, requested an iteration ahead into registers, is stored between the MFMAs, and
// one barrier (for LDS traffic only: the requests cross it) ends the iteration.  A fragment of W serves 3 NT MFMAs, one
// of the centroids MT: at MT = 8, NT = 4 a stage is 3072 matrix-core cycles per SIMD for 1792 cycles of LDS traffic.
// Accumulator register r of lane (li, g) is [row 4g + r][cluster li]: the arg-min over a tile's 16 clusters is a
// reduction inside a 16-lane DPP row, over a block's four column waves through LDS.  Each block writes, per row, the best
// (distance key, cluster) of its columns as one 64-bit word, to win[column block * V + row]; label_hist_kernel takes the smallest.
// LISTED: the rows are rows[list[i]], i < *count (blocks beyond leave at once: few heads list any, then mostly few), and their best words meet in
// win[list[i]].
// Bound by the matrix cores: V = 128256, d = 4096, C = 1024 takes 2.45 ms = 1.32 PFLOP/s (8 waves of 16 rows x 64 clusters, each
// block splitting its own centroids: 7.45 ms); V = 32000, d = 1024, C = 256 (128 x 256 tiles) 49 us, was 124 us.
// Bs: CT cluster tiles (a multiple of 4 NT) of pieces.
template <int MT, int NT, bool LISTED>
__global__ __launch_bounds__(AS_THREADS) void assign_exact_kernel(const uint16_t* __restrict__ W, const uint4* __restrict__ Bs,
                                                                  const float* __restrict__ cn, int V, int d, int C, int CT,
                                                                  int ncol, int ntot, const int* __restrict__ count, const int* __restrict__ list,
                                                                  const int* __restrict__ rows, unsigned long long* __restrict__ win) {
    extern __shared__ as_uintx4_t as_lds[];
    constexpr int AP = 2 * MT * 64 / AS_THREADS, BP = 4 * NT * 192 / AS_THREADS;      // 16-byte pieces a thread stages of W, of the centroids
    constexpr int ASZ = 2 * MT * 64, STAGE = ASZ + 4 * NT * 192;                      // pieces per stage
    static_assert(AP * AS_THREADS == ASZ && BP * AS_THREADS == 4 * NT * 192, "staging layout");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int li = lane & 15, g = lane >> 4, wm = wave >> 2, wn = wave & 3;
    // blocks are dealt round-robin to the eight XCDs: each gets a contiguous run of tiles, columns fastest, so that the
    // blocks that share rows of W and the centroids of a k-block sit behind one L2
    const int tile = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    if (tile >= ntot) return;
    const int bn = tile % ncol, row0 = tile / ncol * (2 * MT * 16);
    if (LISTED) {
        V = *count;
        if (row0 >= V) return;
    }
    const int nq = d >> 3, nkb = (d + 31) >> 5;
    const as_uintx4_t* ap[AP];
#pragma unroll
    for (int i = 0; i < AP; ++i) {
        const int r = min(row0 + (wave + 8 * i) * 16 + li, V - 1);
        ap[i] = reinterpret_cast<const as_uintx4_t*>(W + (size_t)(LISTED ? rows[list[r]] : r) * d);
    }
    const as_uintx4_t* bp = reinterpret_cast<const as_uintx4_t*>(Bs) + (size_t)bn * (4 * NT) * 192 + tid;
    as_uintx4_t ra[AP], rb[BP];
    bool in_row = true;                                      // the requested pieces of W lie inside their rows
    auto request = [&](int kb) {
        const int q = kb * 4 + g;
        in_row = q < nq;
#pragma unroll
        for (int i = 0; i < AP; ++i) ra[i] = ap[i][min(q, nq - 1)];
        const as_uintx4_t* b = bp + (size_t)kb * CT * 192;
#pragma unroll
        for (int i = 0; i < BP; ++i) rb[i] = b[i * AS_THREADS];
    };
    auto store_a = [&](as_uintx4_t* buf, int i) { buf[tid + i * AS_THREADS] = in_row ? ra[i] : as_uintx4_t{0, 0, 0, 0}; };
    auto store_b = [&](as_uintx4_t* buf, int i) { buf[ASZ + tid + i * AS_THREADS] = rb[i]; };
    as_floatx4_t acc[MT][NT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[m][t] = as_floatx4_t{0.f, 0.f, 0.f, 0.f};
    request(0);
#pragma unroll
    for (int i = 0; i < AP; ++i) store_a(as_lds, i);
#pragma unroll
    for (int i = 0; i < BP; ++i) store_b(as_lds, i);
    request(min(1, nkb - 1));
    as_lds_barrier();
    for (int kb = 0; kb < nkb; ++kb) {
        const as_uintx4_t* cur = as_lds + (kb & 1) * STAGE;
        as_uintx4_t* nxt = as_lds + ((kb + 1) & 1) * STAGE;        // last read in the iteration before: every wave has passed its barrier
        as_bf16x8_t A[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m) A[m] = __builtin_bit_cast(as_bf16x8_t, cur[(wm * MT + m) * 64 + lane]);
        // a slot: one centroid fragment, its MT MFMAs, then its share of the next stage's pieces (stored between the MFMAs;
        // in the last iteration to a stage nobody reads)
        as_for<3 * NT>([&](auto slot_t) {
            constexpr int slot = decltype(slot_t)::value, t = slot / 3;
            const as_bf16x8_t B = __builtin_bit_cast(as_bf16x8_t, cur[ASZ + (wn * NT * 3 + slot) * 64 + lane]);
#pragma unroll
            for (int m = 0; m < MT; ++m) acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[m], B, acc[m][t], 0, 0, 0);
            as_for<AP + BP>([&](auto i_t) {
                constexpr int i = decltype(i_t)::value;
                if constexpr (i * 3 * NT / (AP + BP) == slot) {
                    if constexpr (i < AP) store_a(nxt, i);
                    else store_b(nxt, i - AP);
                }
            });
        });
        request(min(kb + 2, nkb - 1));
        as_lds_barrier();
    }
    // ||mu_c||^2 - 2 <W_i,mu_c> for row 4g + r of a tile and cluster li of another; best over the wave's tiles, then over the
    // 16 lanes of the row, then over the four column waves
    unsigned long long* best = reinterpret_cast<unsigned long long*>(as_lds);        // [2 MT 16 rows][4]
    const int c0 = (bn * 4 + wn) * NT * 16 + li;
    float norm[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) norm[t] = c0 + 16 * t < C ? cn[c0 + 16 * t] : 0.f;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            unsigned bk = 0xffffffffu;
            int bc = 0x7fffffff;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int c = c0 + 16 * t;
                const float v = norm[t] - 2.f * acc[m][t][r];
                const unsigned kx = c < C ? fkey(v + 0.0f) : 0xffffffffu;
                if (kx < bk) {                               // tiles in ascending cluster order: a tie keeps the smaller id
                    bk = kx;
                    bc = c;
                }
            }
            const unsigned mk = row16_min_u(bk);
            const unsigned cm = row16_min_u(bk == mk ? (unsigned)bc : 0x7fffffffu);
            if (li == 0) best[((wm * MT + m) * 16 + 4 * g + r) * 4 + wn] = ((unsigned long long)mk << 32) | cm;
        }
    __syncthreads();
    for (int r = tid; r < 2 * MT * 16; r += AS_THREADS)
        if (row0 + r < V) {
            unsigned long long x = best[r * 4];
#pragma unroll
            for (int q = 1; q < 4; ++q) x = best[r * 4 + q] < x ? best[r * 4 + q] : x;
            if (LISTED) atomicMin(&win[list[row0 + r]], x);
            else win[(size_t)bn * V + row0 + r] = x;
        }
}

// Centroids rounded to bf16 (nearest even) in fragment order, out[(kb * CT + ct) * 64 + lane], lane = (cluster li of the tile, k
// group g); zeros past C and past d.  With them cn[c] = ||mu_c||^2 and left[c], what a score with the rounded centroid can differ by from the exact product's
// per unit of ||W_i||: 2 (||mu_c - bf16(mu_c)|| + (0.501 d + 64) 2^-24 ||mu_c||).  The second term is for the float32 sums of both:  an MFMA adds its 32 products
// to the accumulator in four groups of eight, each rounded to nearest (measured: off by 4 2^-24 of the accumulator at most, which is reached); no partial sum
// is larger than ||W_i|| ||mu_c||, and there are d/8 such roundings with one piece (of a centroid up to 1 + 2^-8 times as long), 3 d/8 with three.  Inside a group,
// products are cut off where the bits of the largest end: at most 16 2^-24 of the sum of |products| in all, for either way (4 seen).  The other 32: the
// norm of W_i in float32 and the scores' own last operations (in proportion to cn[c] only where that is less than about 2 ||W_i|| ||mu_c||: a centroid farther
// out is in nobody's reach, unless it is the best: assign_pick_kernel adds 2^-20 of it).  Sums in float64.  (A centroid that rounding takes out of range has no finite
// score: left = 0.  One with a value that is not finite, which counts as zero here: left is not a number.)
// unit != 0 (spherical clustering): every direction counts as of length one, so the arg-min is the largest cosine.
// One block per tile of 16 clusters, a k-block per wave at a time; cn is summed in the order of centroid_norm_kernel, so that a score has the same bits
// whichever of the two made its norm.  Also empties the lists.
__global__ __launch_bounds__(1024) void round_centroids_kernel(const float* __restrict__ mu, int d, int C, int CT, int nkb, int unit, as_uintx4_t* __restrict__ out,
                                                              float* __restrict__ cn, float* __restrict__ left, int* __restrict__ counts) {
    __shared__ double red[2][16][16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, ct = blockIdx.x, c = ct * 16 + (lane & 15), g = lane >> 4;
    if (ct == 0 && threadIdx.x < 3) counts[threadIdx.x] = 0;
    double n8[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0}, rr = 0.0;
    for (int kb = wave; kb < nkb; kb += 16) {
        const int k = kb * 32 + g * 8;
        as_uintx4_t x = {0, 0, 0, 0};
        if (c < C && k < d) {                                    // d is a multiple of 8: the eight values are all in or all out
            const float4* src = reinterpret_cast<const float4*>(mu + (size_t)c * d + k);
            const float4 x0 = src[0], x1 = src[1];
            const float v[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint32_t u = __float_as_uint(v[e]), r = (u & 0x7f800000u) == 0x7f800000u ? 0u : (u + 0x7fffu + ((u >> 16) & 1u)) & 0xffff0000u;
                const double whole = (double)v[e], rest = whole - (double)__uint_as_float(r);
                n8[e] = fma(whole, whole, n8[e]);
                rr = fma(rest, rest, rr);
                x[e >> 1] |= e & 1 ? r : r >> 16;
            }
        }
        out[((size_t)kb * CT + ct) * 64 + lane] = x;
    }
    double nn = ((n8[0] + n8[1]) + (n8[2] + n8[3])) + ((n8[4] + n8[5]) + (n8[6] + n8[7]));
#pragma unroll
    for (int o = 16; o < 64; o <<= 1) {
        nn += __shfl_xor(nn, o, CSV_WAVE);
        rr += __shfl_xor(rr, o, CSV_WAVE);
    }
    if (g == 0) {
        red[0][wave][lane] = nn;
        red[1][wave][lane] = rr;
    }
    __syncthreads();
    if (threadIdx.x >= 16 || ct * 16 + threadIdx.x >= C) return;
    double part[16];
#pragma unroll
    for (int w = 0; w < 16; ++w) part[w] = red[0][w][threadIdx.x];
#pragma unroll
    for (int o = 1; o < 16; o <<= 1)
#pragma unroll
        for (int w = 0; w < 16; w += 2 * o) part[w] += part[w + o];
    nn = part[0];
    rr = 0.0;
    for (int w = 0; w < 16; ++w) rr += red[1][w][threadIdx.x];
    cn[ct * 16 + threadIdx.x] = unit ? 1.f : (float)nn;
    const double off = 2.0 * (sqrt(rr) + (0.501 * d + 64.0) * 0x1p-24 * sqrt(nn)) * (1.0 + 1e-6);
    left[ct * 16 + threadIdx.x] = nn < (double)INFINITY ? (off < (double)INFINITY ? (float)off : 0.f) : NAN;
}

// The three smallest of a set of words, ascending.
struct Low3 {
    unsigned a, b, c;
};
__device__ __forceinline__ Low3 low3_merge(const Low3& x, const Low3& y) {             // of two disjoint sets
    return Low3{min(x.a, y.a), min(max(x.a, y.a), min(x.b, y.b)), min(min(x.c, y.c), min(max(x.b, y.a), max(x.a, y.b)))};
}
template <int CTRL>
__device__ __forceinline__ Low3 low3_move(const Low3& x) {
    return Low3{(unsigned)dpp_move<CTRL, 0xf>((int)x.a, (int)x.a), (unsigned)dpp_move<CTRL, 0xf>((int)x.b, (int)x.b), (unsigned)dpp_move<CTRL, 0xf>((int)x.c, (int)x.c)};
}
// The lane keeps its second set if odd, else its first, and merges it with the same set of the lane that CTRL pairs it with, which keeps the other.
template <int CTRL>
__device__ __forceinline__ Low3 low3_trade(bool odd, const Low3& first, const Low3& second) {
    const Low3 keep = {odd ? second.a : first.a, odd ? second.b : first.b, odd ? second.c : first.c};
    const Low3 give = {odd ? first.a : second.a, odd ? first.b : second.b, odd ? first.c : second.c};
    return low3_merge(keep, low3_move<CTRL>(give));
}

// The row tiles of a launch.  The first assignment with rounded centroids looks at a sample of them first: part 1, one tile of every `every`, at changing
// places among them; part 2, the others; part 0, all.
struct AssignRows {
    int part, every, tiles;              // tiles: of all rows
    __host__ __device__ int count() const {
        const int sample = (tiles + every - 1) / every;
        return part == 0 ? tiles : part == 1 ? sample : tiles - sample;
    }
    __device__ int tile(int i) const {
        if (part == 0) return i;
        const int e = part == 1 ? i : i / (every - 1), k = i - e * (every - 1), at = min(e * 11 % every, tiles - 1 - e * every);
        return e * every + (part == 1 ? at : k < at ? k : k + 1);
    }
};

// Score word of a (row, cluster) pair: the monotone key of the score with the cluster's place in its group in the low AS_ID_BITS bits.
#define AS_ID_BITS 6
#define AS_ID_MASK 63u

// Scores ||mu_c||^2 - 2 <W_i, bf16(mu_c)> of all pairs, less what they can be off by; per row and group of 16 NT clusters the three smallest words, to
// words[(group * 3 + place) * V + row].  Rows are taken in the given order (of the clusters so far: the rows of a block then mostly
// have the same centroids in reach), row being the place in it.  Block = 8 waves, 2 (rows) x 4 (clusters); a wave owns 16 MT rows x 16 NT clusters (one
// group) in accumulators over the whole of K.  Both operands go from memory to LDS without passing registers: W by whole 128-byte lines,
// 64 values of K of every row a stage (three stages, its 16-byte pieces swapped within a line by the row's low bits, so that the
// fragment reads are free of bank conflicts), the centroids 32 values of K a stage (four stages) in the fragment order in which
// they lie in memory.  A wave requests its share of the pieces three to four k-blocks ahead; a k-block issues as many requests in every wave, so "all but
// the last two k-blocks' requests" is a count of vmcnt.  The block's two halves (waves 0-3 and 4-7, one of each per SIMD) run half a k-block
// apart: while one reads its fragments the other has the matrix cores, a barrier after each half.
// A wave passes 2 nkb + 2 barriers, the second half one before the loop, the first half one after it.
// V = 128256, d = 4096, C = 1024 (256 x 256 tiles): 0.80 ms = 1.35 PFLOP/s with the three best, 0.86 with the best and the norms; the product alone 0.77,
// without the two halves 0.91, with W by 64-byte pieces 0.85, through registers 1.10 ms; without any requests in the loop it would take 0.61-0.64 ms.
// FINAL: the centroids are bf16 values (rows of W, the first assignment's), so the scores are exact; the best (distance key, cluster) of a row over the
// block's columns goes to win[column block * V + row] as assign_exact_kernel leaves it: there the zero pieces make "not a number" of every score of a row with
// a value that is not finite.  So where a score is not finite, the block looks whether the row itself is (a sum may overflow, too, and minus infinity is the
// nearest).  norms: ||W_i||, a little more than that, for the assignments to come.
template <int MT, int NT, bool FINAL>
__global__ __launch_bounds__(AS_THREADS) void assign_near_kernel(const uint16_t* __restrict__ W, const int32_t* __restrict__ order, const as_uintx4_t* __restrict__ Bs,
                                                                 const float* __restrict__ cn, int V, int d, int C, int CT,
                                                                 int ncol, AssignRows rows, const float* __restrict__ left, double* __restrict__ norms, unsigned* __restrict__ words, unsigned long long* __restrict__ win) {
    extern __shared__ as_uintx4_t as_lds[];
    constexpr int ASZ = 2 * MT * 128, BSZ = 4 * NT * 64;                                  // 16-byte pieces per stage of W, of the centroids
    constexpr int AP = ASZ / AS_THREADS, BP = BSZ / AS_THREADS, AH = AP / 2, OPEN = 2 * (AH + BP);
    static_assert(AP * AS_THREADS == ASZ && BP * AS_THREADS == BSZ && AP % 2 == 0 && (OPEN == 8 || OPEN == 6), "staging layout");
    as_uintx4_t* ldb = as_lds + 3 * ASZ;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, g = lane >> 4, wm = wave >> 2, wn = wave & 3;
    // blocks are dealt round-robin to the eight XCDs: each gets a contiguous run of tiles, columns fastest, so that the
    // blocks that share rows of W and the centroids of a k-block sit behind one L2
    const int tile = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    if (tile >= rows.count() * ncol) return;
    const int bn = tile % ncol, row0 = rows.tile(tile / ncol) * (2 * MT * 16);
    const int nq = d >> 3, nst = (d + 63) >> 6, nkb = 2 * nst;
    const int piece = (lane & 7) ^ (lane >> 3);              // of the eight of a line; rows go to LDS by eights, so lane >> 3 is the row's low bits
    const as_uintx4_t* ap[AP];
#pragma unroll
    for (int i = 0; i < AP; ++i) {
        const int p = min(row0 + (wave + 8 * i) * 8 + (lane >> 3), V - 1);
        ap[i] = reinterpret_cast<const as_uintx4_t*>(W + (size_t)(order ? order[p] : p) * d);
    }
    const as_uintx4_t* bp = Bs + (size_t)bn * (4 * NT) * 64 + tid;
    auto load = [&](const as_uintx4_t* src, as_uintx4_t* dst) {          // lane l's piece to dst + l
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src, (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
    };
    // past the last stage: requests from the last one to a stage nobody reads again; past d: some piece of the row, which meets zeros
    auto request_w = [&](int s, int slot, int half) {
        const int q = min(min(s, nst - 1) * 8 + piece, nq - 1);
#pragma unroll
        for (int i = 0; i < AH; ++i) load(ap[half * AH + i] + q, as_lds + slot * ASZ + wave * 64 + (half * AH + i) * AS_THREADS);
    };
    auto request_c = [&](int kb) {
#pragma unroll
        for (int i = 0; i < BP; ++i) load(bp + (size_t)min(kb, nkb - 1) * CT * 64 + i * AS_THREADS, ldb + (kb & 3) * BSZ + wave * 64 + i * AS_THREADS);
    };
    auto wait_open = [&]() {                                 // all requests but the last two k-blocks' have arrived
        if constexpr (OPEN == 8) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
    };
    auto barrier = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    as_floatx4_t acc[MT][NT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[m][t] = as_floatx4_t{0.f, 0.f, 0.f, 0.f};
    // in the order of their k-blocks: the first stage's pieces and centroids are older than the last OPEN requests
    request_w(0, 0, 0);
    request_w(0, 0, 1);
    request_c(0);
    request_c(1);
    request_w(1, 1, 0);
    request_w(1, 1, 1);
    request_c(2);
    wait_open();
    barrier();
    if (wm == 1) barrier();
    int slot = 0;
    constexpr int NM = MT / 4;                               // FINAL: of the tile rows that four waves read, each sums the squares of a quarter
    float ss[NM];
#pragma unroll
    for (int i = 0; i < NM; ++i) ss[i] = 0.f;
    const int abase = (wm * MT * 2 + (li >> 3)) * 64 + (li & 7) * 8;
    auto step = [&](auto odd_t, int kb) {
        constexpr int odd = decltype(odd_t)::value;
        const as_uintx4_t* cur = as_lds + slot * ASZ;
        const as_uintx4_t* cub = ldb + (kb & 3) * BSZ;
        as_bf16x8_t A[MT], B[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) B[t] = __builtin_bit_cast(as_bf16x8_t, cub[(wn * NT + t) * 64 + lane]);
        const int q = (odd * 4 + g) ^ (li & 7);
#pragma unroll
        for (int m = 0; m < MT; ++m) A[m] = __builtin_bit_cast(as_bf16x8_t, cur[abase + m * 128 + q]);
        uint4 sq[NM];
        if constexpr (FINAL)
#pragma unroll
            for (int i = 0; i < NM; ++i) sq[i] = __builtin_bit_cast(uint4, cur[abase + (wn * NM + i) * 128 + q]);
        // into the slots of the stage before this one, of the k-block before this one: both halves of the block have read them
        request_w((kb >> 1) + 2, slot == 0 ? 2 : slot - 1, odd);
        request_c(kb + 3);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (wm == 1) wait_open();
        barrier();
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[m], B[t], acc[m][t], 0, 0, 0);
        __builtin_amdgcn_s_setprio(0);
        if constexpr (FINAL)
#pragma unroll
            for (int i = 0; i < NM; ++i) ss[i] = dot8_bf16(sq[i], sq[i], ss[i]);
        if (wm == 0) wait_open();
        barrier();
    };
    for (int kb = 0; kb < nkb; kb += 2) {
        step(std::integral_constant<int, 0>{}, kb);
        step(std::integral_constant<int, 1>{}, kb + 1);
        slot = slot == 2 ? 0 : slot + 1;
    }
    if (wm == 0) barrier();
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // no request may land in what the results go through
    __syncthreads();
    // accumulator register r of lane (li, g) is [row 4g + r][cluster li]: the three best of the wave's tiles, then of the 16 lanes
    const int c0 = (bn * 4 + wn) * NT * 16 + li;
    float norm[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) norm[t] = c0 + 16 * t < C ? cn[c0 + 16 * t] : INFINITY;        // past C: in nobody's reach
    float off[NT];
    bool odd_c[NT];                                          // the centroid is not finite: FINAL, a seed row, nobody's nearest; else in everybody's reach
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const float x = c0 + 16 * t < C ? left[c0 + 16 * t] : 0.f;
        odd_c[t] = x != x;
        off[t] = odd_c[t] ? 0.f : x;
    }
    if constexpr (FINAL) {
        if (norms && bn == 0) {
#pragma unroll
            for (int i = 0; i < NM; ++i) {                   // lane (li, g) holds a quarter of row li's squares
                const float x = ss[i] + __shfl_xor(ss[i], 16, CSV_WAVE), y = x + __shfl_xor(x, 32, CSV_WAVE);
                const int row = row0 + (wm * MT + wn * NM + i) * 16 + li;
                // (up to d = 2^16 the sum, d / 8 steps in float32 to a lane, is short of less than that)
                if (g == 0 && row < V) norms[row] = sqrt((double)y) * (1.0 + 0x1p-10);
            }
        }
        unsigned long long* best = reinterpret_cast<unsigned long long*>(as_lds);        // [2 MT 16 rows][4]
        int* odd = reinterpret_cast<int*>(best + 2 * MT * 16 * 4);                        // per row: it has a value that is not finite; then: look for such
        if (tid <= 2 * MT * 16) odd[tid] = 0;
        __syncthreads();
        bool look = false;
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int t = 0; t < NT; ++t) look = look || (c0 + 16 * t < C && !(fabsf(norm[t] - 2.f * acc[m][t][r]) < INFINITY));
        if (look) odd[2 * MT * 16] = 1;
        __syncthreads();
        if (odd[2 * MT * 16]) {
            for (int r = wave; r < 2 * MT * 16 && row0 + r < V; r += AS_THREADS / 64) {
                const as_uintx4_t* w = reinterpret_cast<const as_uintx4_t*>(W + (size_t)(row0 + r) * d);         // order is NULL here
                bool any = false;
                for (int q = lane; q < nq; q += 64) {
                    const as_uintx4_t x = w[q];
#pragma unroll
                    for (int e = 0; e < 4; ++e) any = any || (x[e] & 0x7f80u) == 0x7f80u || (x[e] & 0x7f800000u) == 0x7f800000u;
                }
                if (__any(any) && lane == 0) odd[r] = 1;
            }
            __syncthreads();
        }
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                unsigned bk = 0xffffffffu;
                int bc = 0x7fffffff;
                const int none = odd[(wm * MT + m) * 16 + 4 * g + r];
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const float v = norm[t] - 2.f * acc[m][t][r];
                    const unsigned kx = c0 + 16 * t >= C ? 0xffffffffu : none || odd_c[t] ? 0xffc00000u : fkey(v + 0.0f);
                    if (kx < bk) {                           // tiles in ascending cluster order: a tie keeps the smaller id
                        bk = kx;
                        bc = c0 + 16 * t;
                    }
                }
                const unsigned mk = row16_min_u(bk);
                const unsigned cm = row16_min_u(bk == mk ? (unsigned)bc : 0x7fffffffu);
                if (li == 0) best[((wm * MT + m) * 16 + 4 * g + r) * 4 + wn] = ((unsigned long long)mk << 32) | cm;
            }
        __syncthreads();
        for (int r = tid; r < 2 * MT * 16; r += AS_THREADS)
            if (row0 + r < V) win[(size_t)bn * V + row0 + r] = min(min(best[r * 4], best[r * 4 + 1]), min(best[r * 4 + 2], best[r * 4 + 3]));
        return;
    } else {
        unsigned* best = reinterpret_cast<unsigned*>(as_lds);    // [column wave][3][2 MT 16 rows]
        float* wnorm = reinterpret_cast<float*>(as_lds) + 12 * 2 * MT * 16;
        if (tid < 2 * MT * 16) {
            const int p = min(row0 + tid, V - 1);
            wnorm[tid] = (float)norms[order ? order[p] : p];
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) norm[t] = odd_c[t] ? -INFINITY : norm[t];
        __syncthreads();
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            Low3 w[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                unsigned x[NT];
                const float wr = wnorm[(wm * MT + m) * 16 + 4 * g + r];
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    x[t] = (fkey(norm[t] - 2.f * acc[m][t][r] - wr * off[t]) & ~AS_ID_MASK) | (unsigned)(t * 16 + li);
                const unsigned p = min(x[0], x[1]), P = max(x[0], x[1]), q = min(x[2], x[3]), Q = max(x[2], x[3]);
                const unsigned m1 = max(p, q), m2 = min(P, Q);
                w[r] = Low3{min(p, q), min(m1, m2), max(m1, m2)};
            }
            // a lane hands half of its rows to its neighbour, then half of the rest to the next but one: lane li goes on with one row
            const Low3 x0 = low3_trade<0xB1>(li & 1, w[0], w[2]), x1 = low3_trade<0xB1>(li & 1, w[1], w[3]);
            Low3 y = low3_trade<0x4E>(li & 2, x0, x1);
            y = low3_merge(y, low3_move<0x128>(y));          // row_ror by 8, then by 4: the other lanes with this row
            y = low3_merge(y, low3_move<0x124>(y));
            const int row = (wm * MT + m) * 16 + 4 * g + (li & 1) * 2 + ((li >> 1) & 1);
            if (li < 12) best[(wn * 3 + (li >> 2)) * (2 * MT * 16) + row] = li < 4 ? y.a : li < 8 ? y.b : y.c;
        }
        __syncthreads();
        for (int i = tid; i < 12 * 2 * MT * 16; i += AS_THREADS) {
            const int row = row0 + i % (2 * MT * 16);
            if (row < V) words[(size_t)(bn * 12 + i / (2 * MT * 16)) * V + row] = best[i];
        }
    }
}

// Labels from the score words.  A word is a lower bound of a centroid's exact score, with twice what it can be off by an upper one; a row's reach is its
// smallest upper bound.  One centroid in reach: the label.  Else the label is ~(a place in rows) until the place's win word holds the nearest: the row's
// pairs with the centroids in reach are listed (all of a group whose third is in reach), or, where they are more than AS_PAIRS_ROW, or more than
// the list holds, or the reach is not finite, the place itself is.  Whole groups and more than AS_PAIRS_CHEAP
// pairs are listed only while less than an eighth of the list is in use: on heads with many such rows the exact product is the cheaper way.  (The blocks of a
// launch mostly run together and see an empty list; those of part 2 see the sample's pairs, which were found to be few enough: no such limit.)
// most: pairs that the list may hold so far, for a sample its share.
// counts: {rows, pairs, rows for all centroids}.  64 rows per block, four threads per row; a block takes its places and pairs in one piece, so
// that pairs of neighbours in the row order, which share centroids, are neighbours in the list.
// Bound by reading the words: V = 128256, C = 1024 in 30 us.
#define AS_PAIRS_ROW 160
#define AS_PAIRS_CHEAP 16
#define AS_PAIRS_SHARE 2      // the list holds that many pairs per row of W, or C / 512 of them: a pair takes as long as 100 columns of the exact product
__global__ __launch_bounds__(256) void assign_pick_kernel(const int32_t* __restrict__ order, const float* __restrict__ cn, const float* __restrict__ left,
                                                          const double* __restrict__ nrm, const unsigned* __restrict__ words, int ngroups, int group, int V, int C,
                                                          AssignRows tiles, int tile_rows, int most, int cap, int32_t* __restrict__ labels, int* __restrict__ counts, int* __restrict__ rows,
                                                          unsigned long long* __restrict__ win, int2* __restrict__ pairs, int* __restrict__ list) {
    __shared__ float s_lim[4][64];
    __shared__ int s_cnt[4][64], s_one[4][64], s_place[64], s_pair[64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, per_tile = tile_rows >> 6;
    const int at = tiles.tile(blockIdx.x / per_tile) * tile_rows + (blockIdx.x % per_tile) * 64 + lane, row = min(at, V - 1);
    const bool mine = at < V;
    const int token = order ? order[row] : row;
    const float wr = (float)nrm[token];
    float lim = INFINITY;
#pragma unroll 4
    for (int g = wave; g < ngroups; g += 4) {
        const unsigned a = words[(size_t)(g * 3) * V + row];
        const int c = min(g * group + (int)(a & AS_ID_MASK), C - 1);
        const float lo = fkey_inv(a | AS_ID_MASK);
        lim = fminf(lim, lo + (2.00001f * wr * left[c] + 0x1p-20f * (fabsf(lo) + cn[c])));
    }
    s_lim[wave][lane] = lim;
    __syncthreads();
    lim = fminf(fminf(s_lim[0][lane], s_lim[1][lane]), fminf(s_lim[2][lane], s_lim[3][lane]));
    const bool finite = fabsf(lim) < INFINITY;
    const unsigned reach = fkey(lim) | AS_ID_MASK;
    auto reached = [&](auto fn) {                            // this thread's share of the row's centroids in reach, in runs
#pragma unroll 4
        for (int g = wave; g < ngroups; g += 4) {
            const unsigned* w = words + (size_t)(g * 3) * V + row;
            const unsigned a = w[0];
            if (finite && a <= reach) {
                const unsigned b = w[V];
                if (b <= reach && w[2 * (size_t)V] <= reach) {
                    fn(g * group, min(group, C - g * group));
                } else {
                    fn(g * group + (int)(a & AS_ID_MASK), 1);
                    if (b <= reach) fn(g * group + (int)(b & AS_ID_MASK), 1);
                }
            }
        }
    };
    int cnt = 0, one = 0;
    reached([&](int c, int n) {
        cnt += n;
        one = n > 1 ? -1 : one < 0 ? one : c;                // -1: a whole group
    });
    s_cnt[wave][lane] = cnt;
    s_one[wave][lane] = one;
    __syncthreads();
    if (wave == 0) {
        int total = 0;
        one = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int n = s_cnt[q][lane];
            s_cnt[q][lane] = total;                          // becomes the row's pairs of the threads before
            if (n) one = one < 0 ? one : s_one[q][lane];
            total += n;
        }
        const bool settled = finite && total == 1 && one >= 0;
        const int used = __builtin_amdgcn_readfirstlane(counts[1]);
        bool few = mine && !settled && finite && total <= AS_PAIRS_ROW && ((one >= 0 && total <= AS_PAIRS_CHEAP) || used < (tiles.part == 2 ? most : most >> 3));
        int upto = few ? total : 0;                          // inclusive sum over the lanes
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(upto, o, CSV_WAVE);
            if (lane >= o) upto += y;
        }
        const unsigned long long open = __ballot(mine && !settled), below = (1ull << lane) - 1ull;
        const int npairs = __builtin_amdgcn_readlane(upto, 63);
        int place0 = 0, pair0 = 0;
        if (open && lane == 0) {
            place0 = atomicAdd(&counts[0], __popcll(open));
            if (npairs) pair0 = atomicAdd(&counts[1], npairs);
        }
        place0 = __builtin_amdgcn_readfirstlane(place0);
        pair0 = __builtin_amdgcn_readfirstlane(pair0);
        if (pair0 > most - npairs) {                         // the list is full (of the sample's share of it): these places of it hold no pairs
            for (int i = pair0 + lane; i < cap && i < pair0 + npairs; i += 64) pairs[i] = make_int2(0, -1);
            few = false;
        }
        const unsigned long long all = __ballot(mine && !settled && !few);
        int list0 = 0;
        if (all && lane == 0) list0 = atomicAdd(&counts[2], __popcll(all));
        list0 = __builtin_amdgcn_readfirstlane(list0);
        const int place = place0 + __popcll(open & below);
        s_place[lane] = few ? place : -1;
        s_pair[lane] = pair0 + upto - total;
        if (mine && settled) labels[token] = one;
        if (mine && !settled) {
            labels[token] = ~place;
            rows[place] = token;
            win[place] = ~0ull;
            if (!few) list[list0 + __popcll(all & below)] = place;
        }
    }
    __syncthreads();
    if (s_place[lane] < 0) return;
    int next = s_pair[lane] + s_cnt[wave][lane];
    reached([&](int c, int n) {
        for (int i = 0; i < n; ++i) pairs[next++] = make_int2(s_place[lane], c + i);
    });
}

// Exact scores of the listed pairs {place, centroid}.  Sixteen pairs at a time are the diagonal of a 16 x 16 product whose first operand is
// the pairs' rows and whose second is their centroids, split as they are read; a wave has AS_PIPE k-blocks requested ahead.
// Bound by the splitting and, with few pairs a wave, by latency: 62000 pairs at d = 4096 in 0.16 ms (the rows in token order, so that
// no two pairs of a wave share a centroid: 0.24; eight k-blocks ahead and half the waves: 1 % of a build slower).
#define AS_PIPE 4
__global__ __launch_bounds__(256) void assign_pairs_kernel(const uint16_t* __restrict__ W, const float* __restrict__ mu, const float* __restrict__ cn, int d,
                                                           int cap, const int* __restrict__ counts, const int2* __restrict__ pairs,
                                                           const int* __restrict__ rows, unsigned long long* __restrict__ win) {
    const int lane = threadIdx.x & 63, li = lane & 15, g = lane >> 4, nkb = (d + 31) >> 5, nq = d >> 3, npairs = min(counts[1], cap);
    for (int i0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * 16; i0 < npairs; i0 += gridDim.x * 64) {
        const int2 pair = pairs[min(i0 + li, npairs - 1)];
        const bool in = i0 + li < npairs && pair.y >= 0;
        const as_uintx4_t* w = reinterpret_cast<const as_uintx4_t*>(W + (size_t)(pair.y >= 0 ? rows[pair.x] : 0) * d);
        const float4* m = reinterpret_cast<const float4*>(mu + (size_t)max(pair.y, 0) * d);
        as_uintx4_t x[AS_PIPE];
        float4 m0[AS_PIPE], m1[AS_PIPE];
        auto request = [&](int u, int kb) {                  // past d: the row's last values, which meet zeros
            const int q = min(kb * 4 + g, nq - 1);
            x[u] = w[q];
            m0[u] = m[2 * q];
            m1[u] = m[2 * q + 1];
        };
        as_floatx4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < AS_PIPE; ++u) request(u, u);
        for (int kb = 0; kb < nkb; kb += AS_PIPE) {
#pragma unroll
            for (int u = 0; u < AS_PIPE; ++u) {
                uint4 hi, mid, lo;
                as_uintx4_t xv = x[u];
                as_split3(m0[u], m1[u], hi, mid, lo);
                if ((kb + u) * 4 + 4 > nq && (kb + u) * 4 + g >= nq) xv = as_uintx4_t{0, 0, 0, 0};
                __builtin_amdgcn_sched_barrier(0);
                request(u, kb + u + AS_PIPE);
                __builtin_amdgcn_sched_barrier(0);
                const as_bf16x8_t A = __builtin_bit_cast(as_bf16x8_t, xv);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, __builtin_bit_cast(as_bf16x8_t, hi), acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, __builtin_bit_cast(as_bf16x8_t, mid), acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, __builtin_bit_cast(as_bf16x8_t, lo), acc, 0, 0, 0);
            }
        }
        if ((li >> 2) == g && in) {                          // register li & 3 of this lane is [row li][centroid li]
            const float dot = li & 2 ? (li & 1 ? acc[3] : acc[2]) : (li & 1 ? acc[1] : acc[0]), v = cn[pair.y] - 2.f * dot;
            atomicMin(&win[pair.x], ((unsigned long long)fkey(v + 0.0f) << 32) | (unsigned)pair.y);
        }
    }
}

// mu[c] = row init_rows[c] of W widened to float32 (starting centroids).
__global__ __launch_bounds__(256) void init_centroid_kernel(const uint16_t* __restrict__ W, const int32_t* __restrict__ rows,
                                                            int d, float* __restrict__ mu) {
    const int c = blockIdx.x;
    const uint16_t* w = W + (size_t)rows[c] * d;
    for (int j = threadIdx.x; j < d; j += 256) mu[(size_t)c * d + j] = __uint_as_float((uint32_t)w[j] << 16);
}

// ------------------------------------------------------------------------------------------------ spherical clustering
// (Section III, "Advanced Theoretical Improvements", spherical clustering metrics)
// ||W_r|| of every row (original or permuted order, whichever W is), float64.  One wave per row.
__global__ __launch_bounds__(256) void row_norm_kernel(const uint16_t* __restrict__ W, int V, int d, double* __restrict__ nrm) {
    const int lane = threadIdx.x & 63;
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= V) return;
    const uint4* w = reinterpret_cast<const uint4*>(W + (size_t)r * d);
    double acc = 0.0;
    for (int q = lane; q < (d >> 3); q += 64) {
        const uint4 x = w[q];
        const uint32_t xs[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double a0 = (double)__uint_as_float(xs[e] << 16), a1 = (double)__uint_as_float(xs[e] & 0xffff0000u);
            acc = fma(a0, a0, acc);
            acc = fma(a1, a1, acc);
        }
    }
    acc = wave_sum_d(acc);
    if (lane == 0) nrm[r] = sqrt(acc);
}

// Starting directions: row init_rows[c] of W, normalised, as float32.
__global__ __launch_bounds__(256) void init_direction_kernel(const uint16_t* __restrict__ W, const int32_t* __restrict__ rows,
                                                             const double* __restrict__ nrm, int d, float* __restrict__ mu) {
    const int c = blockIdx.x;
    const uint16_t* w = W + (size_t)rows[c] * d;
    const double nr = nrm[rows[c]];
    for (int j = threadIdx.x; j < d; j += 256) {
        const double v = (double)__uint_as_float((uint32_t)w[j] << 16);
        mu[(size_t)c * d + j] = (float)(nr > 0.0 ? v / nr : v);
    }
}

// mu[c] = sums[c] / ||sums[c]|| as float32; an empty cluster keeps its direction (Lloyd) or is zeroed (final metadata).
__global__ __launch_bounds__(256) void direction_finish_kernel(const double* __restrict__ sums, const int32_t* __restrict__ off, int d,
                                                               int zero_empty, float* __restrict__ mu) {
    __shared__ double red[4];
    const int c = blockIdx.x, tid = threadIdx.x;
    if (off[c + 1] == off[c]) {
        if (zero_empty)
            for (int j = tid; j < d; j += 256) mu[(size_t)c * d + j] = 0.f;
        return;
    }
    double acc = 0.0;
    for (int j = tid; j < d; j += 256) acc += sums[(size_t)c * d + j] * sums[(size_t)c * d + j];
    acc = wave_sum_d(acc);
    if ((tid & 63) == 0) red[tid >> 6] = acc;
    __syncthreads();
    const double nr = sqrt((red[0] + red[1]) + (red[2] + red[3]));
    for (int j = tid; j < d; j += 256) {
        const double v = sums[(size_t)c * d + j];
        mu[(size_t)c * d + j] = (float)(nr > 0.0 ? v / nr : v);
    }
}

// Per row (one wave): cosine to its cluster's stored direction and its norm, folded into per-cluster extremes with
// integer atomics: cosines are shifted by +2 (positive doubles order like their bit patterns).
// ext[c] = {min (cos + 2), max ||w||^2 bits, min ||w||^2 bits}
__global__ __launch_bounds__(256) void row_angle_kernel(const uint16_t* __restrict__ Wp, const int32_t* __restrict__ off,
                                                        const float* __restrict__ mu, int V, int d, int C,
                                                        unsigned long long* __restrict__ ext) {
    const int lane = threadIdx.x & 63;
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= V) return;
    int lo = 0, hi = C;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (off[mid] <= r) lo = mid; else hi = mid;
    }
    const uint4* w = reinterpret_cast<const uint4*>(Wp + (size_t)r * d);
    const float4* m = reinterpret_cast<const float4*>(mu + (size_t)lo * d);
    double ww = 0.0, wm = 0.0, mm = 0.0;
    for (int q = lane; q < (d >> 3); q += 64) {
        const uint4 x = w[q];
        const float4 m0 = m[2 * q], m1 = m[2 * q + 1];
        const uint32_t xs[4] = {x.x, x.y, x.z, x.w};
        const float ms[8] = {m0.x, m0.y, m0.z, m0.w, m1.x, m1.y, m1.z, m1.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double a0 = (double)__uint_as_float(xs[e] << 16), a1 = (double)__uint_as_float(xs[e] & 0xffff0000u);
            const double b0 = (double)ms[2 * e], b1 = (double)ms[2 * e + 1];
            ww = fma(a0, a0, ww); ww = fma(a1, a1, ww);
            wm = fma(a0, b0, wm); wm = fma(a1, b1, wm);
            mm = fma(b0, b0, mm); mm = fma(b1, b1, mm);
        }
    }
    ww = wave_sum_d(ww);
    wm = wave_sum_d(wm);
    mm = wave_sum_d(mm);
    if (lane == 0) {
        const double nw = sqrt(ww), nm = sqrt(mm);
        double cs = nw > 0.0 ? wm / (nw * (nm > 0.0 ? nm : 1.0)) : 1.0;
        cs = fmin(1.0, fmax(-1.0, cs));
        atomicMin(&ext[3 * lo], (unsigned long long)__double_as_longlong(cs + 2.0));
        atomicMax(&ext[3 * lo + 1], (unsigned long long)__double_as_longlong(ww));
        atomicMin(&ext[3 * lo + 2], (unsigned long long)__double_as_longlong(ww));
    }
}

// ang[c] = {cos, sin of the angular radius with slack, largest norm (1+slack) rounded up, smallest (1-slack) rounded down}
__global__ __launch_bounds__(256) void angular_finish_kernel(const int32_t* __restrict__ off, int C, double slack, double angle_slack,
                                                             const unsigned long long* __restrict__ ext, float4* __restrict__ ang) {
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (c >= C) return;
    if (off[c + 1] == off[c]) {
        ang[c] = make_float4(1.f, 0.f, 0.f, 0.f);
        return;
    }
    const double mincos = __longlong_as_double((long long)ext[3 * c]) - 2.0;
    double theta = acos(fmin(1.0, fmax(-1.0, mincos)));
    const double pi = 3.14159265358979323846;
    theta = fmin(pi, theta * (1.0 + slack) + angle_slack);
    auto up = [](double x) { float y = (float)x; if ((double)y < x) y = nextafterf(y, INFINITY); return y; };
    auto down = [](double x) { float y = (float)x; if ((double)y > x) y = nextafterf(y, -INFINITY); return y; };
    const float ct = theta < pi ? down(cos(theta)) : -1.f;
    const float st = up(sin(theta));
    const double nmax = sqrt(__longlong_as_double((long long)ext[3 * c + 1])), nmin = sqrt(__longlong_as_double((long long)ext[3 * c + 2]));
    ang[c] = make_float4(ct, st, up(nmax * (1.0 + slack)), down(nmin * (1.0 - slack)));
}

// cmeta[c] = {off[c], off[c+1] - off[c], bits of ln n_c, 0};  inv[perm[r]] = r
__global__ __launch_bounds__(256) void pack_tables_kernel(const int32_t* __restrict__ off, const float* __restrict__ lnn, const int32_t* __restrict__ perm,
                                                          int C, int V, int4* __restrict__ cmeta, int32_t* __restrict__ inv) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < C) cmeta[i] = make_int4(off[i], off[i + 1] - off[i], __float_as_int(lnn[i]), 0);
    if (i < V) inv[perm[i]] = i;
}

// ------------------------------------------------------------------------------------------------ host side
int csv_index_pack_tables(csv_index* x, hipStream_t st) {          // C <= V
    pack_tables_kernel<<<(x->V + 255) / 256, 256, 0, st>>>(x->off, x->lnn, x->perm, x->C, x->V, x->cmeta, x->inv);
    CSV_LAUNCH_CHECK("pack_tables_kernel");
    return CSV_OK;
}

static int check_shape(int V, int d, int C) {
    if (V < 1 || d < 8 || (d & 7) != 0) { csv_set_error("need V >= 1 and d a positive multiple of 8 (V=%d, d=%d)", V, d); return CSV_ESHAPE; }
    if (C < 1 || C > V || C > CSV_MAX_CLUSTERS) { csv_set_error("C=%d outside 1..min(V,%d)", C, CSV_MAX_CLUSTERS); return CSV_ESHAPE; }
    return CSV_OK;
}

int csv_index_alloc(int V, int d, int C, csv_index** out) {
    csv_index* x = (csv_index*)calloc(1, sizeof(csv_index));
    if (!x) { csv_set_error("host allocation failed"); return CSV_ENOMEM; }
    x->V = V; x->d = d; x->C = C;
    hipError_t e = hipGetDevice(&x->device);
    auto A = [&](void** p, size_t bytes) { if (e == hipSuccess) e = hipMalloc(p, bytes); };
    A((void**)&x->Wp, (size_t)V * d * 2); A((void**)&x->bp, (size_t)V * 4); A((void**)&x->perm, (size_t)V * 4); A((void**)&x->inv, (size_t)V * 4);
    A((void**)&x->mu, (size_t)C * d * 4); A((void**)&x->R, (size_t)C * 4); A((void**)&x->bmax, (size_t)C * 4);
    A((void**)&x->n, (size_t)C * 4); A((void**)&x->off, (size_t)(C + 1) * 4); A((void**)&x->lnn, (size_t)C * 4);
    A((void**)&x->cmeta, (size_t)C * sizeof(int4));
    if (e != hipSuccess) {
        csv_set_error("index allocation failed: %s", hipGetErrorString(e));
        csv_index_free(x);
        return e == hipErrorOutOfMemory ? CSV_ENOMEM : CSV_EHIP;
    }
    *out = x;
    return CSV_OK;
}

extern "C" void csv_index_free(csv_index* x) {
    if (!x) return;
    void* ptrs[] = {x->Wp, x->bp, x->perm, x->inv, x->mu, x->mu16, x->R, x->bmax, x->n, x->off, x->lnn, x->cmeta, x->bt, x->ang};
    for (void* p : ptrs)
        if (p) (void)hipFree(p);
    free(x);
}

extern "C" int csv_index_dims(const csv_index* x, int* V, int* d, int* C) {
    if (!x) { csv_set_error("null index"); return CSV_EINVAL; }
    if (V) *V = x->V;
    if (d) *d = x->d;
    if (C) *C = x->C;
    return CSV_OK;
}

// Centroids stored as bfloat16: mu is rounded in place (nearest even) and the 16-bit patterns go to mu16.
// check != 0: nothing is rounded; *bad is set when a value is not already a bfloat16.
__global__ __launch_bounds__(256) void centroid_bf16_kernel(float* __restrict__ mu, uint16_t* __restrict__ mu16, size_t n, int check,
                                                            int* __restrict__ bad) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const uint32_t u = __float_as_uint(mu[i]);
    if (check) {
        if (u & 0xffffu) *bad = 1;
        mu16[i] = (uint16_t)(u >> 16);
        return;
    }
    const uint32_t r = (u + 0x7fffu + ((u >> 16) & 1u)) & 0xffff0000u;
    mu[i] = __uint_as_float(r);
    mu16[i] = (uint16_t)(r >> 16);
}

static int store_centroids_bf16(csv_index* x, int check, hipStream_t st) {
    const size_t n = (size_t)x->C * x->d;
    if (!x->mu16 && hipMalloc((void**)&x->mu16, n * 2) != hipSuccess) { csv_set_error("out of device memory (bf16 centroids)"); return CSV_ENOMEM; }
    int* d_bad = nullptr;
    if (hipMalloc((void**)&d_bad, 4) != hipSuccess) { csv_set_error("out of device memory"); return CSV_ENOMEM; }
    int h_bad = 0;
    hipError_t e = hipMemsetAsync(d_bad, 0, 4, st);
    if (e == hipSuccess) {
        centroid_bf16_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(x->mu, x->mu16, n, check, d_bad);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpyAsync(&h_bad, d_bad, 4, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    (void)hipFree(d_bad);
    if (e != hipSuccess) { csv_set_error("bf16 centroid conversion failed: %s", hipGetErrorString(e)); return CSV_EHIP; }
    if (h_bad) {
        (void)hipFree(x->mu16);
        x->mu16 = nullptr;
        csv_set_error("centroids are not bfloat16 values: the radii of this index were not measured to rounded centroids");
        return CSV_EINVAL;
    }
    return CSV_OK;
}

extern "C" int csv_index_use_bf16_centroids(csv_index* x, void* stream) {
    if (!x) { csv_set_error("null index"); return CSV_EINVAL; }
    if (x->mu16) return CSV_OK;
    return store_centroids_bf16(x, 1, (hipStream_t)stream);
}

static int upload_layout(csv_index* x, const std::vector<int32_t>& n, const std::vector<int32_t>& off,
                         const std::vector<int32_t>& perm, hipStream_t st) {
    CSV_HIP(hipMemcpyAsync(x->n, n.data(), (size_t)x->C * 4, hipMemcpyHostToDevice, st));
    CSV_HIP(hipMemcpyAsync(x->off, off.data(), (size_t)(x->C + 1) * 4, hipMemcpyHostToDevice, st));
    CSV_HIP(hipMemcpyAsync(x->perm, perm.data(), (size_t)x->V * 4, hipMemcpyHostToDevice, st));
    CSV_HIP(hipStreamSynchronize(st));   // the host vectors may go away after this
    return CSV_OK;
}

static int gather(csv_index* x, const uint16_t* d_W, const float* d_b, hipStream_t st) {
    gather_rows_kernel<<<x->V, 256, 0, st>>>(d_W, d_b, x->perm, x->V, x->d, x->Wp, x->bp);
    CSV_LAUNCH_CHECK("gather_rows_kernel");
    return CSV_OK;
}

// Which tile a block of the assignment computes: the one whose rounds over the compute units cost least.  Per k-block of the exact
// product a 256 x 256 tile takes 3072 cycles of a SIMD's matrix core, a 128 x 256 tile 1536 (with 1464 of LDS traffic), and two
// 128 x 128 tiles, which share a compute unit, 1792 of LDS traffic between them; of the product with bf16 centroids 1024 (matrix core
// and LDS) and 704 (LDS), while two 128 x 128 tiles would take 1024, never less than one of 256 x 256.
struct AssignPlan {
    int kind, nt, ncol, CT, ntot;
};
static AssignPlan assign_plan(int V, int C, bool near) {
    static const struct { int mt, nt, per_cu, exact, near; } kind[3] = {{8, 4, 1, 3072, 1024}, {4, 4, 1, 1536, 704}, {4, 2, 2, 1792, 0}};
    AssignPlan best = {0, 0, 0, 0, 0};
    long long cost = 0;
    for (int i = 0; i < (near ? 2 : 3); ++i) {
        const int bm = 2 * kind[i].mt * 16, bn = 4 * kind[i].nt * 16;
        const int ncol = (C + bn - 1) / bn, ntot = (V + bm - 1) / bm * ncol, at_once = 256 * kind[i].per_cu;
        const long long c = (long long)((ntot + at_once - 1) / at_once) * (near ? kind[i].near : kind[i].exact);
        if (i == 0 || c < cost) {
            cost = c;
            best = {i, kind[i].nt, ncol, ncol * 4 * kind[i].nt, ntot};
        }
    }
    return best;
}
// Whether the rounded centroids come first.  They save two thirds of the exact product, V d C, and cost four launches and the pairs, which do not shrink with
// C; where most rows stay open (hundreds of seeds in one centre) the look at them is lost.  Builds of four iterations, exact against rounded first: V = 32000,
// d = 1024, C = 256 661 / 813 us, C = 512 799 / 786; V = 32000, d = 4096, C = 256 1763 / 1914; V = 64000, d = 2048, C = 384 2137 / 1970; V = 128256, d = 4096,
// C = 384 6764 / 6471, C = 256 4849 / 3939 (but C = 336 with rows left open 5503 / 5598).
static bool assign_near_pays(int V, int d, int C) { return C >= 384 && (double)V * d * C >= 20e9; }
struct AssignRun {                       // what an assignment reads and writes, in the build's scratch
    const uint16_t* W;
    const float* mu;
    float* cn;
    int V, d, C;
    uint4* pieces;                       // exact: the centroids' pieces; near: the same, for listed rows
    unsigned long long* win;             // exact: [column block][V]; near: by place
    as_uintx4_t* rounded;                // near only, as all below
    float* left;
    double* nrm;
    unsigned* words;
    int *counts, *rows, *list, cap;
    int2* pairs;
    int32_t* labels;
    hipStream_t st;
};
template <int MT, int NT, bool LISTED>
static int launch_exact(const AssignPlan& p, const AssignRun& r) {
    constexpr int lds = 2 * (2 * MT + 12 * NT) * 1024;
    CSV_HIP(hipFuncSetAttribute((const void*)assign_exact_kernel<MT, NT, LISTED>, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    assign_exact_kernel<MT, NT, LISTED><<<(p.ntot + 7) / 8 * 8, AS_THREADS, lds, r.st>>>(r.W, r.pieces, r.cn, r.V, r.d, r.C, p.CT, p.ncol, p.ntot,
                                                                                        r.counts + 2, r.list, r.rows, r.win);
    CSV_LAUNCH_CHECK("assign_exact_kernel");
    return CSV_OK;
}
template <int MT, int NT, bool FINAL>
static int launch_near(const AssignPlan& p, const AssignRun& r, const int32_t* order, const AssignRows& rows) {
    constexpr int lds = (3 * 2 * MT * 128 + 4 * 4 * NT * 64) * 16;
    CSV_HIP(hipFuncSetAttribute((const void*)assign_near_kernel<MT, NT, FINAL>, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    assign_near_kernel<MT, NT, FINAL><<<(rows.count() * p.ncol + 7) / 8 * 8, AS_THREADS, lds, r.st>>>(r.W, order, r.rounded, r.cn, r.V, r.d, r.C, p.CT, p.ncol, rows, r.left, r.nrm, r.words, r.win);
    CSV_LAUNCH_CHECK("assign_near_kernel");
    return CSV_OK;
}
static int round_centroids(const AssignPlan& p, const AssignRun& r, int unit) {
    round_centroids_kernel<<<p.CT, 1024, 0, r.st>>>(r.mu, r.d, r.C, p.CT, (r.d + 63) / 64 * 2, unit, r.rounded, r.cn, r.left, r.counts);
    CSV_LAUNCH_CHECK("round_centroids_kernel");
    return CSV_OK;
}
static int assign_exact(const AssignPlan& p, const AssignRun& r, int unit) {
    centroid_norm_kernel<<<r.C, 512, 0, r.st>>>(r.mu, r.d, unit, r.cn);
    CSV_LAUNCH_CHECK("centroid_norm_kernel");
    const int nkb = (r.d + 31) / 32;
    split_centroids_kernel<<<dim3(p.CT, (nkb + 3) / 4), 256, 0, r.st>>>(r.mu, r.d, r.C, p.CT, nkb, nullptr, r.pieces);
    CSV_LAUNCH_CHECK("split_centroids_kernel");
    return p.kind == 0 ? launch_exact<8, 4, false>(p, r) : p.kind == 1 ? launch_exact<4, 4, false>(p, r) : launch_exact<4, 2, false>(p, r);
}
// the first assignment: the centroids are rows of W
static int assign_first(const AssignPlan& p, const AssignRun& r) {
    const int rc = round_centroids(p, r, 0);
    if (rc) return rc;
    const AssignRows all = {0, 2, p.ntot / p.ncol};
    return p.kind == 0 ? launch_near<8, 4, true>(p, r, nullptr, all) : launch_near<4, 4, true>(p, r, nullptr, all);
}
// order: the rows by the clusters so far.  give_up: looked at once the rounded scores of a sample of the rows are in (of all, where those are few tiles), at
// the cost of a wait; set, and no labels made, where they leave so many rows for the exact product that it is cheaper over all rows.  Builds of skewed heads,
// us without any look / looking at all rows / at the sample: V = 26000, d = 800, C = 1024, 2 iterations 660 / 690 / 660; V = 40000, d = 1024, C = 512, 4 iterations
// 1050 / 1080 / 1050.
static int assign_near(const AssignPlan& p, const AssignRun& r, int unit, const int32_t* order, bool* give_up) {
    int rc = round_centroids(p, r, unit);
    if (rc) return rc;
    const int tiles = p.ntot / p.ncol, tile_rows = p.kind == 0 ? 256 : 128;
    // the sample: as few tiles as take, with the others in a launch of their own, no more rounds over the compute units than all in one launch
    auto rounds = [&](int t) { return (t * p.ncol + 255) / 256; };
    int every = 16;
    while (every > 1 && rounds((tiles + every - 1) / every) + rounds(tiles - (tiles + every - 1) / every) > rounds(tiles)) --every;
    for (int part = give_up && tiles >= 32 && every > 1 ? 1 : 0; part < 3; ++part) {
        const AssignRows rows = {part, every, tiles};
        const double share = (double)rows.count() / tiles;
        const int most = part == 1 ? (int)(r.cap * share) : r.cap;       // pairs so far
        rc = p.kind == 0 ? launch_near<8, 4, false>(p, r, order, rows) : launch_near<4, 4, false>(p, r, order, rows);
        if (rc) return rc;
        assign_pick_kernel<<<rows.count() * (tile_rows / 64), 256, 0, r.st>>>(order, r.cn, r.left, r.nrm, r.words, p.ncol * 4, p.nt * 16, r.V, r.C, rows, tile_rows, most, r.cap, r.labels,
                                                                              r.counts, r.rows, r.win, r.pairs, r.list);
        CSV_LAUNCH_CHECK("assign_pick_kernel");
        if (give_up && part < 2) {
            int n[3] = {0, 0, 0};
            CSV_HIP(hipMemcpyAsync(n, r.counts, 12, hipMemcpyDeviceToHost, r.st));
            CSV_HIP(hipStreamSynchronize(r.st));
            // in passes of the exact product over all rows: the rounded scores and the look through them; 30 us of launches; a pair takes as long as 100
            // columns of a row; listed rows go through smaller tiles
            const double work = (double)r.V * r.d * r.C, V = r.V * share;
            *give_up = 0.4 + 6.5e9 / work + 100.0 * std::min(n[1], most) / (V * r.C) + 1.15 * n[2] / V > 0.85;
            if (*give_up) return CSV_OK;
        }
        if (part == 0) break;
    }
    assign_pairs_kernel<<<1024, 256, 0, r.st>>>(r.W, r.mu, r.cn, r.d, r.cap, r.counts, r.pairs, r.rows, r.win);
    CSV_LAUNCH_CHECK("assign_pairs_kernel");
    const int nkb = (r.d + 31) / 32, ncol = (r.C + 255) / 256;
    const AssignPlan all = {1, 4, ncol, ncol * 16, (r.V + 127) / 128 * ncol};
    split_centroids_kernel<<<dim3(all.CT, (nkb + 3) / 4), 256, 0, r.st>>>(r.mu, r.d, r.C, all.CT, nkb, r.counts + 2, r.pieces);
    CSV_LAUNCH_CHECK("split_centroids_kernel");
    return launch_exact<4, 4, true>(all, r);
}

extern "C" int csv_build_index(const uint16_t* d_W, const float* d_b, int V, int d, int C, const csv_build_opts* o,
                               void* stream, csv_index** out) {
    if (out) *out = nullptr;
    if (!d_W || !o || !out) { csv_set_error("null W, opts or out"); return CSV_EINVAL; }
    int rc = check_shape(V, d, C);
    if (rc) return rc;
    if (o->iters < 0 || !(o->radius_slack >= 0.f)) { csv_set_error("iters and radius_slack must be >= 0"); return CSV_EINVAL; }
    if (o->bias_table_m < 0 || o->bias_table_m > CSV_MAX_BIAS_TABLE) { csv_set_error("bias_table_m=%d outside 0..%d", o->bias_table_m, CSV_MAX_BIAS_TABLE); return CSV_EINVAL; }

    hipStream_t st = (hipStream_t)stream;
    csv_index* x = nullptr;
    rc = csv_index_alloc(V, d, C, &x);
    if (rc) return rc;
    // One scratch allocation for the whole build: labels, the layout's counts and chunk list, norms, squared distances; for spherical clustering
    // sums of unit rows.
    const int sph = o->spherical != 0, bt_m = o->bias_table_m >= 2 ? o->bias_table_m : 0;
    const bool assigns = !o->h_init_labels || o->iters > 0;
    const int nkb = (d + 31) / 32, nw = (V + LAY_TOKENS - 1) / LAY_TOKENS, max_chunks = V / CHUNK_ROWS + C;
    // first: the centroids are rows of W and one bf16 piece is exact; may_near: the centroids rounded come first
    const bool first = !o->h_init_labels && !o->spherical, may_near = o->iters > 0 && assign_near_pays(V, d, C);
    const AssignPlan fp = assign_plan(V, C, true), ap = assign_plan(V, C, false);
    bool near = may_near;                // until an assignment shows that most rows are out of its reach
    char* arena = nullptr;
    size_t used = 0;
    auto take = [&](size_t bytes) {
        const size_t at = used;
        used += (bytes + 255) / 256 * 256;
        return at;
    };
    // Partial centroid sums and what an assignment needs (pieces, words, lists) are never live together: they share their bytes, and those are the
    // index's own copy of W, which is written last, wherever they fit into it (an allocation of 64 MB or more takes 30 us to get and 225 us to give back).
    // Given labels that stay say how many partial sums there are.
    size_t part_slots = PART_SLOTS(V) < max_chunks ? PART_SLOTS(V) : max_chunks;
    if (o->h_init_labels) {
        std::vector<int32_t> rows(C, 0);
        for (int i = 0; i < V; ++i) {
            const int l = o->h_init_labels[i];
            if (l < 0 || l >= C) { csv_set_error("label %d of token %d outside 0..C-1", l, i); csv_index_free(x); return CSV_EINVAL; }
            ++rows[l];
        }
        if (o->iters == 0) {
            part_slots = 0;
            for (int c = 0; c < C; ++c)
                if (rows[c] > CHUNK_ROWS) part_slots += (rows[c] + CHUNK_ROWS - 1) / CHUNK_ROWS;
        }
    }
    const size_t part_bytes = part_slots * d * 8, piece_tiles = assigns ? std::max(ap.CT, (C + 255) / 256 * 16) : 0,
                 piece_bytes = (size_t)nkb * piece_tiles * 192 * sizeof(uint4), near_rows = near ? V : 0;
    const int pair_cap = near ? (int)std::min(std::min((long long)V * AS_PAIRS_SHARE, (long long)V * C / 512), (long long)INT32_MAX / 2) : 0;
    size_t assign_bytes = 0;
    auto share = [&](size_t bytes) {
        const size_t at = assign_bytes;
        assign_bytes += (bytes + 255) / 256 * 256;
        return at;
    };
    const size_t a_pieces = share(piece_bytes), a_rounded = share(first || near ? (size_t)(d + 63) / 64 * 2 * fp.CT * 64 * sizeof(as_uintx4_t) : 0),
                 a_win = share(assigns ? (size_t)V * std::max(fp.ncol, ap.ncol) * 8 : 0), a_words = share(near_rows * fp.ncol * 48), a_rows = share(near_rows * 4),
                 a_list = share(near_rows * 4), a_pairs = share((size_t)pair_cap * sizeof(int2)), shared_bytes = std::max(part_bytes, assign_bytes);
    const bool in_copy = shared_bytes <= (size_t)V * d * 2;
    const size_t o_labels = take((size_t)V * 4), o_hist = take((size_t)nw * C * 4), o_coff = take((size_t)(C + 1) * 4), o_poff = take((size_t)C * 4), o_chunks = take((size_t)max_chunks * sizeof(int2)),
                 o_shared = take(in_copy ? 0 : shared_bytes), o_cn = take((size_t)C * 4), o_left = take((size_t)C * 4), o_counts = take(256), o_d2max = take((size_t)C * 8),
                 o_d2row = take(bt_m ? (size_t)V * 8 : 0), o_nrm = take(sph ? (size_t)V * 8 : near_rows * 8), o_sums = take(sph ? (size_t)C * d * 8 : 0),
                 o_ext = take(sph ? (size_t)3 * C * 8 : 0);
    auto fail = [&](int code) {
        if (arena) {
            (void)hipStreamSynchronize(st);
            (void)hipFree(arena);
        }
        csv_index_free(x);
        return code;
    };
    if (sph && (o->centroid_bf16 || bt_m)) { csv_set_error("spherical clustering takes neither bf16 centroids nor a bias table"); return fail(CSV_EINVAL); }
    if (hipMalloc((void**)&arena, used) != hipSuccess) { csv_set_error("out of device memory (index build scratch, %zu bytes)", used); return fail(CSV_ENOMEM); }
    int32_t *d_labels = (int32_t*)(arena + o_labels), *d_hist = (int32_t*)(arena + o_hist), *d_coff = (int32_t*)(arena + o_coff), *d_poff = (int32_t*)(arena + o_poff);
    int2* d_chunks = (int2*)(arena + o_chunks);
    char* shared = in_copy ? (char*)x->Wp : arena + o_shared;
    double *d_part = (double*)shared, *d_nrm = (double*)(arena + o_nrm), *d_sums = (double*)(arena + o_sums), *d_d2row = bt_m ? (double*)(arena + o_d2row) : nullptr;
    unsigned long long *d_win = (unsigned long long*)(shared + a_win), *d_d2max = (unsigned long long*)(arena + o_d2max), *d_ext = (unsigned long long*)(arena + o_ext);
    if (sph || (near && !first)) {
        row_norm_kernel<<<(V + 3) / 4, 256, 0, st>>>(d_W, V, d, d_nrm);
        if (hipGetLastError() != hipSuccess) { csv_set_error("launch of row_norm_kernel failed"); return fail(CSV_EHIP); }
    }
    const AssignRun run = {d_W, x->mu, (float*)(arena + o_cn), V, d, C, (uint4*)(shared + a_pieces), d_win, (as_uintx4_t*)(shared + a_rounded), (float*)(arena + o_left),
                           near || sph ? d_nrm : nullptr, (unsigned*)(shared + a_words), (int*)(arena + o_counts), (int*)(shared + a_rows), (int*)(shared + a_list), pair_cap,
                           (int2*)(shared + a_pairs), d_labels, st};
    int made = 0;                        // column blocks whose best words the labels come from (0: they are there already)
    std::vector<int32_t> seed;
    if (o->h_init_labels) {
        if (hipMemcpyAsync(d_labels, o->h_init_labels, (size_t)V * 4, hipMemcpyHostToDevice, st) != hipSuccess) { csv_set_error("copy of the labels failed"); return fail(CSV_EHIP); }
    } else {
        // seeding rule when the caller names no rows: C tokens evenly spread over the vocabulary, token floor(c V / C)
        seed.resize(C);
        for (int c = 0; c < C; ++c) seed[c] = o->h_init_rows ? o->h_init_rows[c] : (int32_t)((long long)c * V / C);
        for (int c = 0; c < C; ++c)
            if (seed[c] < 0 || seed[c] >= V) { csv_set_error("init row %d outside 0..V-1", seed[c]); return fail(CSV_EINVAL); }
        // x->n doubles as the staging buffer for the starting rows
        if (hipMemcpyAsync(x->n, seed.data(), (size_t)C * 4, hipMemcpyHostToDevice, st) != hipSuccess) { csv_set_error("copy of init rows failed"); return fail(CSV_EHIP); }
        if (sph) init_direction_kernel<<<C, 256, 0, st>>>(d_W, x->n, d_nrm, d, x->mu);
        else init_centroid_kernel<<<C, 256, 0, st>>>(d_W, x->n, d, x->mu);
        if ((rc = first ? assign_first(fp, run) : assign_exact(ap, run, sph))) return fail(rc);
        made = first ? fp.ncol : ap.ncol;
    }
    int label_bits = 1;
    while ((1 << label_bits) < C) ++label_bits;
    for (int it = 0;; ++it) {
        const bool last = it == o->iters;
        label_hist_kernel<<<nw, 64, (size_t)C * 4, st>>>(made ? d_win : nullptr, made, d_win, d_labels, V, C, d_hist);
        layout_scan_kernel<<<(C + 63) / 64, 512, 0, st>>>(d_hist, nw, C, x->n);
        layout_offsets_kernel<<<1, 1024, 0, st>>>(x->n, C, x->off, d_coff, d_poff, d_chunks);
        layout_scatter_kernel<<<nw, 64, (size_t)C * 4, st>>>(d_labels, d_hist, x->off, V, C, label_bits, x->perm);
        const int nslices = (d + 511) / 512;
        const dim3 kgrid(max_chunks * nslices), fgrid(C, (d + 255) / 256);
        if (sph) {
            centroid_chunk_kernel<true><<<kgrid, 256, 0, st>>>(d_W, x->perm, x->off, d_coff, d_poff, d_chunks, d, C, nslices, d_nrm, x->mu, d_sums, d_part);
            centroid_finish_kernel<true><<<fgrid, 256, 0, st>>>(x->off, d_poff, d, 0, d_part, x->mu, d_sums);
            direction_finish_kernel<<<C, 256, 0, st>>>(d_sums, x->off, d, last ? 1 : 0, x->mu);
        } else {
            centroid_chunk_kernel<false><<<kgrid, 256, 0, st>>>(d_W, x->perm, x->off, d_coff, d_poff, d_chunks, d, C, nslices, nullptr, x->mu, nullptr, d_part);
            centroid_finish_kernel<false><<<fgrid, 256, 0, st>>>(x->off, d_poff, d, last ? 1 : 0, d_part, x->mu, nullptr);
        }
        if (hipGetLastError() != hipSuccess) { csv_set_error("launch of the centroid kernels failed"); return fail(CSV_EHIP); }
        if (last) break;
        bool give_up = false;
        if (near && (rc = assign_near(fp, run, sph, x->perm, it == 0 ? &give_up : nullptr))) return fail(rc);
        near = near && !give_up;
        if (!near && (rc = assign_exact(ap, run, sph))) return fail(rc);
        made = near ? 0 : ap.ncol;
    }
    if (o->centroid_bf16 && (rc = store_centroids_bf16(x, 0, st))) return fail(rc);
    if (bt_m && hipMalloc((void**)&x->bt, (size_t)C * bt_m * sizeof(float2)) != hipSuccess) { csv_set_error("out of device memory (bias table)"); return fail(CSV_ENOMEM); }
    x->bt_m = bt_m;
    bool launched = hipMemsetAsync(d_d2max, 0, (size_t)C * 8, st) == hipSuccess;
    if (launched) {
        gather_dist_kernel<<<max_chunks * 4, 256, 0, st>>>(d_W, d_b, x->perm, x->off, d_coff, d_chunks, x->mu, d, C, x->Wp, x->bp, d_d2max, d_d2row);
        launched = hipGetLastError() == hipSuccess;
    }
    if (launched && bt_m) {
        bias_table_kernel<<<C, 256, 0, st>>>(x->bp, x->off, x->mu, d, (double)o->radius_slack, bt_m, d_d2row, x->bt);
        launched = hipGetLastError() == hipSuccess;
    }
    if (launched) {
        radius_finish_kernel<<<C, 256, 0, st>>>(x->bp, x->off, x->mu, d, (double)o->radius_slack, d_d2max, x->R, x->bmax, x->lnn);
        launched = hipGetLastError() == hipSuccess;
    }
    if (launched) launched = csv_index_pack_tables(x, st) == CSV_OK;
    std::vector<unsigned long long> ext0;
    if (launched && sph) {          // angular metadata in place of the Euclidean radius (which stays unused)
        ext0.resize((size_t)3 * C);
        for (int c = 0; c < C; ++c) {
            ext0[3 * c] = ~0ull;
            ext0[3 * c + 1] = 0ull;
            ext0[3 * c + 2] = ~0ull;
        }
        launched = hipMalloc((void**)&x->ang, (size_t)C * sizeof(float4)) == hipSuccess &&
                   hipMemcpyAsync(d_ext, ext0.data(), (size_t)3 * C * 8, hipMemcpyHostToDevice, st) == hipSuccess;
        if (launched) {
            row_angle_kernel<<<(V + 3) / 4, 256, 0, st>>>(x->Wp, x->off, x->mu, V, d, C, d_ext);
            angular_finish_kernel<<<(C + 255) / 256, 256, 0, st>>>(x->off, C, (double)o->radius_slack, CSV_ANGLE_SLACK, d_ext, x->ang);
            launched = hipGetLastError() == hipSuccess;
        }
    }
    std::vector<int32_t> n(C);
    if (launched) launched = hipMemcpyAsync(n.data(), x->n, (size_t)C * 4, hipMemcpyDeviceToHost, st) == hipSuccess;
    const bool synced = hipStreamSynchronize(st) == hipSuccess;
    if (!launched) { csv_set_error("launch of the radius kernels failed"); return fail(CSV_EHIP); }
    if (!synced) { csv_set_error("index build failed on the device: %s", hipGetErrorString(hipGetLastError())); return fail(CSV_EHIP); }
    {
        int nmax = 1;
        for (int c = 0; c < C; ++c) nmax = n[c] > nmax ? n[c] : nmax;
        x->ln_nmax = (float)log((double)nmax);
        x->n_max = nmax;
    }
    (void)hipFree(arena);
    *out = x;
    return CSV_OK;
}

extern "C" int csv_index_from_arrays(const uint16_t* d_W, const float* d_b, int V, int d, int C, const float* h_mu,
                                     const float* h_R, const float* h_bmax, const int32_t* h_n, const int32_t* h_perm,
                                     void* stream, csv_index** out) {
    if (out) *out = nullptr;
    if (!d_W || !h_mu || !h_R || !h_bmax || !h_n || !h_perm || !out) { csv_set_error("null argument"); return CSV_EINVAL; }
    int rc = check_shape(V, d, C);
    if (rc) return rc;
    std::vector<int32_t> n(h_n, h_n + C), off(C + 1, 0), perm(h_perm, h_perm + V);
    std::vector<float> lnn(C);
    for (int c = 0; c < C; ++c) {
        if (n[c] < 0) { csv_set_error("negative cluster size"); return CSV_EINVAL; }
        off[c + 1] = off[c] + n[c];
        lnn[c] = n[c] > 0 ? (float)log((double)n[c]) : -INFINITY;
    }
    if (off[C] != V) { csv_set_error("cluster sizes sum to %d, not V=%d", off[C], V); return CSV_EINVAL; }
    std::vector<char> seen(V, 0);
    for (int i = 0; i < V; ++i) {
        if (perm[i] < 0 || perm[i] >= V || seen[perm[i]]) { csv_set_error("h_perm is not a permutation of 0..V-1"); return CSV_EINVAL; }
        seen[perm[i]] = 1;
    }
    hipStream_t st = (hipStream_t)stream;
    csv_index* x = nullptr;
    rc = csv_index_alloc(V, d, C, &x);
    if (rc) return rc;
    auto fail = [&](int code) { csv_index_free(x); return code; };
    {
        int nmax = 1;
        for (int c = 0; c < C; ++c) nmax = n[c] > nmax ? n[c] : nmax;
        x->ln_nmax = (float)log((double)nmax);
        x->n_max = nmax;
    }
    hipError_t e = hipMemcpyAsync(x->mu, h_mu, (size_t)C * d * 4, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync(x->R, h_R, (size_t)C * 4, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync(x->bmax, h_bmax, (size_t)C * 4, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync(x->lnn, lnn.data(), (size_t)C * 4, hipMemcpyHostToDevice, st);
    if (e != hipSuccess) { csv_set_error("metadata upload failed: %s", hipGetErrorString(e)); return fail(CSV_EHIP); }
    if ((rc = upload_layout(x, n, off, perm, st))) return fail(rc);
    if ((rc = gather(x, d_W, d_b, st))) return fail(rc);
    if ((rc = csv_index_pack_tables(x, st))) return fail(rc);
    if (hipStreamSynchronize(st) != hipSuccess) { csv_set_error("index import failed on the device"); return fail(CSV_EHIP); }
    *out = x;
    return CSV_OK;
}

extern "C" int csv_index_export(const csv_index* x, float* h_mu, float* h_R, float* h_bmax, int32_t* h_n, int32_t* h_perm) {
    if (!x) { csv_set_error("null index"); return CSV_EINVAL; }
    if (h_mu) CSV_HIP(hipMemcpy(h_mu, x->mu, (size_t)x->C * x->d * 4, hipMemcpyDeviceToHost));
    if (h_R) CSV_HIP(hipMemcpy(h_R, x->R, (size_t)x->C * 4, hipMemcpyDeviceToHost));
    if (h_bmax) CSV_HIP(hipMemcpy(h_bmax, x->bmax, (size_t)x->C * 4, hipMemcpyDeviceToHost));
    if (h_n) CSV_HIP(hipMemcpy(h_n, x->n, (size_t)x->C * 4, hipMemcpyDeviceToHost));
    if (h_perm) CSV_HIP(hipMemcpy(h_perm, x->perm, (size_t)x->V * 4, hipMemcpyDeviceToHost));
    return CSV_OK;
}

extern "C" int csv_index_set_bias_table(csv_index* x, int m, const float* h_table, void* stream) {
    if (!x) { csv_set_error("null index"); return CSV_EINVAL; }
    if (m < 0 || m > CSV_MAX_BIAS_TABLE || (m >= 1 && !h_table)) { csv_set_error("bias table: m=%d outside 0..%d, or null table", m, CSV_MAX_BIAS_TABLE); return CSV_EINVAL; }
    hipStream_t st = (hipStream_t)stream;
    if (x->bt) {
        CSV_HIP(hipStreamSynchronize(st));
        (void)hipFree(x->bt);
        x->bt = nullptr;
        x->bt_m = 0;
    }
    if (m == 0) return CSV_OK;
    const size_t bytes = (size_t)x->C * m * sizeof(float2);
    if (hipMalloc((void**)&x->bt, bytes) != hipSuccess) { csv_set_error("out of device memory (bias table)"); return CSV_ENOMEM; }
    CSV_HIP(hipMemcpyAsync(x->bt, h_table, bytes, hipMemcpyHostToDevice, st));
    CSV_HIP(hipStreamSynchronize(st));
    x->bt_m = m;
    return CSV_OK;
}

extern "C" int csv_index_get_bias_table(const csv_index* x, int* m, float* h_table) {
    if (!x || !m) { csv_set_error("null index or m"); return CSV_EINVAL; }
    *m = x->bt_m;
    if (h_table && x->bt_m) CSV_HIP(hipMemcpy(h_table, x->bt, (size_t)x->C * x->bt_m * sizeof(float2), hipMemcpyDeviceToHost));
    return CSV_OK;
}

extern "C" int csv_index_set_angular(csv_index* x, const float* h_ang, void* stream) {
    if (!x) { csv_set_error("null index"); return CSV_EINVAL; }
    hipStream_t st = (hipStream_t)stream;
    if (!h_ang) {
        if (x->ang) {
            CSV_HIP(hipStreamSynchronize(st));
            (void)hipFree(x->ang);
            x->ang = nullptr;
        }
        return CSV_OK;
    }
    if (x->bt || x->mu16) { csv_set_error("an angular index takes neither a bias table nor bf16 centroids"); return CSV_EINVAL; }
    if (!x->ang && hipMalloc((void**)&x->ang, (size_t)x->C * sizeof(float4)) != hipSuccess) { csv_set_error("out of device memory (angular metadata)"); return CSV_ENOMEM; }
    CSV_HIP(hipMemcpyAsync(x->ang, h_ang, (size_t)x->C * sizeof(float4), hipMemcpyHostToDevice, st));
    CSV_HIP(hipStreamSynchronize(st));
    return CSV_OK;
}

extern "C" int csv_index_get_angular(const csv_index* x, int* present, float* h_ang) {
    if (!x || !present) { csv_set_error("null index or present"); return CSV_EINVAL; }
    *present = x->ang != nullptr;
    if (h_ang && x->ang) CSV_HIP(hipMemcpy(h_ang, x->ang, (size_t)x->C * sizeof(float4), hipMemcpyDeviceToHost));
    return CSV_OK;
}

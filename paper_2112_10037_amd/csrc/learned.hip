// Learned output-size predictor and the one-pass product it enables.
//
// The network is a fully connected 8-64-64-1 ReLU MLP in FP32.  Its inputs
// are the per-row features of the row-statistics kernel; its output
// estimates log2(1 + row_nnz) / 16.  The capacity of row i is
//     cap_i = clamp(ceil(2^(16 y_i + delta)), lo_i, hi_i)
// with the exact bounds lo_i = max_k nnz(B(k,:)) (the union is at least its
// largest set) and hi_i = min(prod_i, ncols(B)); delta is a calibrated
// quantile of the training residuals.  Rows whose bounds are small take
// cap_i = hi_i without running the network.
//
// The one-pass product bins rows by capacity, runs the numeric kernels in
// capacity mode into a padded C (each row's true count, or -1 when it did
// not fit), recomputes the overflowed rows exactly with the plain two-phase
// path on the sub-matrix of those rows, and compacts everything into a
// tight CSR.  The structure is exact whatever the network predicts.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <functional>
#include <vector>

#include "internal.hpp"
#include "kernels.hpp"
#include "msp.h"

using namespace msp;

namespace msp {

constexpr int kNF = 8, kH1 = 64, kH2 = 64;
constexpr int kOffW1 = 0, kOffB1 = 512, kOffW2 = 576, kOffB2 = 4672, kOffW3 = 4736, kOffB3 = 4800;
constexpr int kNParam = 4801;
constexpr int kSmallCap = 32;      // rows with hi <= this skip the network

// ---------------------------------------------------------------------------
// network evaluation (weights in LDS, one row per thread)
// ---------------------------------------------------------------------------
__device__ __forceinline__ float mlp_eval(const float* __restrict__ w, const float* __restrict__ xin) {
    float x[kNF];
#pragma unroll
    for (int f = 0; f < kNF; ++f) x[f] = xin[f];
    float h1[kH1];
#pragma unroll
    for (int i = 0; i < kH1; ++i) {
        float z = w[kOffB1 + i];
#pragma unroll
        for (int f = 0; f < kNF; ++f) z += w[kOffW1 + i * kNF + f] * x[f];
        h1[i] = z > 0.f ? z : 0.f;
    }
    float y = w[kOffB3];
#pragma unroll 1
    for (int j = 0; j < kH2; ++j) {
        const float4* row = reinterpret_cast<const float4*>(w + kOffW2 + j * kH1);
        float z = w[kOffB2 + j];
#pragma unroll
        for (int i4 = 0; i4 < kH1 / 4; ++i4) {
            const float4 q = row[i4];
            z += q.x * h1[4 * i4] + q.y * h1[4 * i4 + 1] + q.z * h1[4 * i4 + 2] + q.w * h1[4 * i4 + 3];
        }
        y += w[kOffW3 + j] * (z > 0.f ? z : 0.f);
    }
    return y;
}

// (at least 4 waves per SIMD: the weight loads are not hoisted into registers)
__global__ void __launch_bounds__(256, 4)
k_mlp_predict(long long n, const float* __restrict__ feats, const float* __restrict__ params, float* __restrict__ y) {
    __shared__ __align__(16) float w[kNParam + 3];
    for (int i = threadIdx.x; i < kNParam; i += 256) w[i] = params[i];
    __syncthreads();
    // one row per thread (a row loop would let the compiler hoist every
    // weight load out of it into registers)
    const long long r = (long long)blockIdx.x * 256 + threadIdx.x;
    if (r < n) y[r] = mlp_eval(w, feats + r * kNF);
}

// capacity rule; rows with small bounds skip the network.  Rows without
// products (cap 0) are in no numeric bin: their count is set to 0 here.
__global__ void __launch_bounds__(256, 4)
k_capacity(int m, const float* __restrict__ feats, const int32_t* __restrict__ hi, const int32_t* __restrict__ lo,
           const float* __restrict__ params, float delta, int32_t* __restrict__ cap, int32_t* __restrict__ cnt,
           BinTable nt, int big, int* __restrict__ nbig, unsigned long long* __restrict__ big_hi) {
    __shared__ __align__(16) float w[kNParam + 3];
    for (int i = threadIdx.x; i < kNParam; i += 256) w[i] = params[i];
    __syncthreads();
    const long long r = (long long)blockIdx.x * 256 + threadIdx.x;
    bool to_exact = false;
    unsigned long long exact_hi = 0;
    if (r < m) {
        const int h = hi[r];
        const int l = lo[r] < h ? lo[r] : h;
        int c = h;
        if (h > kSmallCap && l < h) {
            const float y = mlp_eval(w, feats + r * kNF);
            const double est = exp2((double)(16.f * y + delta));
            c = est < (double)h ? (int)ceil(est) : h;    // NaN or overflow: the upper bound
            c = c < l ? l : c;
            if (nt.nb > 0) {
                // the margin alone lifts the row past the bound of its point
                // prediction's bin: keep it in that bin, at the bin's bound
                const double pt = exp2((double)(16.f * y));
                if (pt < (double)h) {
                    int cp = (int)ceil(pt);
                    cp = cp < l ? l : cp;
                    const int bp = bin_of(nt, cp);
                    if (bp < nt.nb && bin_of(nt, c) > bp) c = nt.umax[bp];
                }
            }
            // the exact bound costs nothing more when it keeps the row in
            // the same numeric bin (same kernel, same accumulator): only
            // unused padding, which the compaction never reads; and it
            // costs at most twice the predicted room when it is within a
            // factor 2, where a row just above the prediction would
            // otherwise overflow into the exact recomputation
            if ((long long)h <= 2LL * c || (nt.nb > 0 && bin_of(nt, c) == bin_of(nt, h))) c = h;
        }
        // a capacity in the global bin: the row goes to the exact two-phase
        // path (its per-window counts come from the symbolic pass there),
        // with no padded room here
        to_exact = big >= 0 && c > big;
        if (to_exact) {
            c = 0;
            exact_hi = (unsigned long long)h;
        }
        cap[r] = c;
        if (c == 0) cnt[r] = to_exact ? -2 : 0;
    }
    const uint64_t bm = __ballot(to_exact);
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) exact_hi += __shfl_xor(exact_hi, d);
    if (bm && (threadIdx.x & 63) == __builtin_ctzll(bm)) {
        atomicAdd(nbig, __builtin_popcountll(bm));
        atomicAdd(big_hi, exact_hi);
    }
}

// ---------------------------------------------------------------------------
// training: forward, backward and gradient of a batch tile on the matrix
// cores, then the tiles' sums and Adam
// ---------------------------------------------------------------------------
// A workgroup of four waves takes tiles of 16 samples.  Wave w owns the hidden
// units 16 w .. 16 w + 15 of both layers: its part of every product is a 16 x
// 16 FP64 matrix-core tile (v_mfma_f64_16x16x4: lane l holds A[l % 16][l / 16]
// and B[l / 16][l % 16]; register r of the result is row 4 r + l / 16, column
// l % 16).  A product's terms may come in any order, so lane group g takes the
// terms 16 g + k in step k: its weights are then consecutive in memory and
// stay in registers over the tiles.  Activations and deltas pass between the
// waves through LDS in FP64; the gradient's sums over the workgroup's samples
// stay in the result registers and leave as one partial sum per workgroup, so
// the gradient is deterministic.
//
// Bound by latency: a step of 4096 samples is 115 MFLOP, 1.6 us at the FP64
// matrix rate, and takes 11.9 us here (256 workgroups of one tile: 11.6, but
// 5.9 instead of 4.5 us for the sum of twice the partial sums).  Before (a
// thread per sample, 16 workgroups, activations and deltas through memory, one
// thread per parameter and tile): 51 + 25 + 37 us for forward and backward,
// tile sums and their sum.  FP64 keeps every sum at least as close as the FP32
// forward pass with FP64 gradient sums was.
constexpr int kTile = 16;                      // samples per tile
constexpr int kTileWG = 128;                   // most workgroups of a step
constexpr int kPartRow = 4864;                 // doubles per workgroup's partial sums (whole 512-byte lines)
constexpr int kTilePad = 66;                   // doubles per LDS row of 64 (rows start on different banks)
static_assert(kPartRow >= kNParam, "a partial row holds every parameter");

typedef double f64x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f64x4 mfma_f64(double a, double b, f64x4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

__global__ void __launch_bounds__(256)
k_mlp_tiles(int batch, long long n, const int32_t* __restrict__ idx, const float* __restrict__ feats,
            const float* __restrict__ targets, const float* __restrict__ params, double* __restrict__ partial,
            double* __restrict__ partial_loss, int* __restrict__ bad) {
    __shared__ __align__(16) double h1[kTile][kTilePad], dz2[kTile][kTilePad], dz1[kTile][kTilePad];
    __shared__ double ypart[4][kTile];
    __shared__ float sx[kTile][kNF], st[kTile];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
    const int u = 16 * w + c;                   // this lane's hidden unit
    // a tile's samples: lane group g takes the features 2 g and 2 g + 1 of sample c
    float x[2], target;
    auto samples = [&](int s0) {
        x[0] = x[1] = target = 0.f;
        if (s0 + c >= batch) return;
        long long r = idx[s0 + c];
        if (r < 0 || r >= n) {                  // flagged; the sample reads row 0 instead
            atomicOr(bad, 1);
            r = 0;
        }
        x[0] = feats[r * kNF + 2 * g];
        x[1] = feats[r * kNF + 2 * g + 1];
        target = targets[r];
    };
    samples(blockIdx.x * kTile);
    // the wave's weights: rows of W1 and W2 for the forward pass, columns of W2 for the backward one
    double w1[2], w2f[16], w2b[16];
    for (int k = 0; k < 2; ++k) w1[k] = params[kOffW1 + u * kNF + 2 * g + k];
#pragma unroll
    for (int k = 0; k < 16; ++k) w2f[k] = params[kOffW2 + u * kH1 + 16 * g + k];
#pragma unroll
    for (int k = 0; k < 16; ++k) w2b[k] = params[kOffW2 + (16 * g + k) * kH1 + u];
    const double b1 = params[kOffB1 + u], b2 = params[kOffB2 + u], w3 = params[kOffW3 + u], b3 = params[kOffB3];
    const double scale = 2.0 / (double)batch;
    f64x4 gw2[4] = {}, gw1 = {};
    double gb1 = 0.0, gb2 = 0.0, gw3 = 0.0, gb3 = 0.0, loss = 0.0;
    for (int s0 = blockIdx.x * kTile; s0 < batch; s0 += gridDim.x * kTile) {
        // layer 1, then the next tile's samples
        if (w == 0) {
            sx[c][2 * g] = x[0];
            sx[c][2 * g + 1] = x[1];
            if (g == 0) st[c] = target;
        }
        f64x4 z = {b1, b1, b1, b1};
        z = mfma_f64(x[0], w1[0], z);
        z = mfma_f64(x[1], w1[1], z);
        samples(s0 + gridDim.x * kTile);
        bool on1[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            on1[r] = z[r] > 0.0;
            h1[4 * r + g][u] = on1[r] ? z[r] : 0.0;
        }
        __syncthreads();
        // layer 2 and the output
        z = f64x4{b2, b2, b2, b2};
#pragma unroll
        for (int k = 0; k < 16; ++k) z = mfma_f64(h1[c][16 * g + k], w2f[k], z);
        double h2[4], y[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            h2[r] = z[r] > 0.0 ? z[r] : 0.0;
            y[r] = h2[r] * w3;
        }
        {
            // over the 16 units: lanes that differ in bits 3 and 2 share out the
            // four samples (lane c ends with sample register c / 4), then the rest
            const bool up = c & 8;
            double p = up ? y[2] : y[0], q = up ? y[3] : y[1];
            p += __shfl_xor(up ? y[0] : y[2], 8);
            q += __shfl_xor(up ? y[1] : y[3], 8);
            const bool odd = c & 4;
            const double o = __shfl_xor(odd ? p : q, 4);
            double v = (odd ? q : p) + o;
            v += __shfl_xor(v, 2);
            v += __shfl_xor(v, 1);
            if ((c & 3) == 0) ypart[w][4 * (c >> 2) + g] = v;
        }
        __syncthreads();
        // the samples' errors and the second layer's deltas
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int s = 4 * r + g;
            double d = 0.0;
            if (s0 + s < batch) d = b3 + ypart[0][s] + ypart[1][s] + ypart[2][s] + ypart[3][s] - (double)st[s];
            const double dy = scale * d;
            const double dz = z[r] > 0.0 ? dy * w3 : 0.0;
            dz2[s][u] = dz;
            gb2 += dz;
            gw3 += dy * h2[r];
            gb3 += dy;
            loss += d * d;
        }
        __syncthreads();
        // the first layer's deltas, and W2's gradient: rows of this wave, all columns
        z = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < 16; ++k) z = mfma_f64(dz2[c][16 * g + k], w2b[k], z);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const double dz = on1[r] ? z[r] : 0.0;
            dz1[4 * r + g][u] = dz;
            gb1 += dz;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double a = dz2[4 * g + k][u];
#pragma unroll
            for (int t = 0; t < 4; ++t) gw2[t] = mfma_f64(a, h1[4 * g + k][16 * t + c], gw2[t]);
        }
        __syncthreads();
        // W1's gradient (columns past the features are not kept)
#pragma unroll
        for (int k = 0; k < 4; ++k) gw1 = mfma_f64(dz1[4 * g + k][u], c < kNF ? (double)sx[4 * g + k][c] : 0.0, gw1);
        __syncthreads();
    }
    double* const out = partial + (long long)blockIdx.x * kPartRow;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = 16 * w + 4 * r + g;
        if (c < kNF) out[kOffW1 + row * kNF + c] = gw1[r];
#pragma unroll
        for (int t = 0; t < 4; ++t) out[kOffW2 + row * kH1 + 16 * t + c] = gw2[t][r];
    }
#pragma unroll
    for (int d = 16; d < 64; d <<= 1) {         // over the lane groups
        gb1 += __shfl_xor(gb1, d);
        gb2 += __shfl_xor(gb2, d);
        gw3 += __shfl_xor(gw3, d);
        gb3 += __shfl_xor(gb3, d);
        loss += __shfl_xor(loss, d);
    }
    if (g == 0) {
        out[kOffB1 + u] = gb1;
        out[kOffB2 + u] = gb2;
        out[kOffW3 + u] = gw3;
        if (u == 0) {
            out[kOffB3] = gb3;
            partial_loss[blockIdx.x] = loss;
        }
    }
}

// The workgroups' partial sums in a fixed order, and with ADAM the update
// (Kingma and Ba, 2015, bias-corrected moments; step is 1-based).  A
// workgroup takes 32 parameters, eight threads each; the last one the loss.
constexpr int kSumP = 32, kSumT = 8;
template <bool ADAM>
__global__ void __launch_bounds__(kSumP * kSumT)
k_mlp_sum(int parts, int batch, const double* __restrict__ partial, const double* __restrict__ partial_loss,
          float* __restrict__ grad, float* __restrict__ loss, float* __restrict__ params, float* __restrict__ m,
          float* __restrict__ v, int step, float lr, float beta1, float beta2, float eps) {
    __shared__ double acc[kSumT][kSumP];
    const int pl = threadIdx.x % kSumP, t = threadIdx.x / kSumP;
    const bool is_loss = blockIdx.x == gridDim.x - 1;
    const int p = blockIdx.x * kSumP + pl;
    double s = 0.0;
    if (is_loss) {
        for (int i = threadIdx.x; i < parts; i += kSumP * kSumT) s += partial_loss[i];
    } else if (p < kNParam) {
#pragma unroll 4
        for (int i = t; i < parts; i += kSumT) s += partial[(long long)i * kPartRow + p];
    }
    acc[t][pl] = s;
    __syncthreads();
    if (t != 0) return;
    s = 0.0;
#pragma unroll
    for (int i = 0; i < kSumT; ++i) s += acc[i][pl];
    if (is_loss) {
#pragma unroll
        for (int d = kSumP / 2; d > 0; d >>= 1) s += __shfl_xor(s, d, kSumP);
        if (pl == 0 && loss) *loss = (float)(s / batch);
        return;
    }
    if (p >= kNParam) return;
    const float g = (float)s;
    grad[p] = g;
    if constexpr (ADAM) {
        const float mm = beta1 * m[p] + (1.f - beta1) * g;
        const float vv = beta2 * v[p] + (1.f - beta2) * g * g;
        m[p] = mm;
        v[p] = vv;
        const float mhat = mm / (1.f - powf(beta1, (float)step));
        const float vhat = vv / (1.f - powf(beta2, (float)step));
        params[p] -= lr * mhat / (sqrtf(vhat) + eps);
    }
}
constexpr int kSumGrid = (kNParam + kSumP - 1) / kSumP + 1;

// training target of a row: log2(1 + row_nnz) / 16
__global__ void __launch_bounds__(256)
k_targets(int m, const int32_t* __restrict__ row_nnz, float* __restrict__ t) {
    const long long r = (long long)blockIdx.x * 256 + threadIdx.x;
    if (r < m) t[r] = log2f(1.f + (float)row_nnz[r]) * kFeatLogScale;
}

// ---------------------------------------------------------------------------
// one-pass product helpers
// ---------------------------------------------------------------------------
// Overflowed rows (cnt < 0): list them in row order per wave, with their A
// lengths, and count them.
__global__ void __launch_bounds__(256)
k_collect_overflow(int m, const int32_t* __restrict__ cnt, const int64_t* __restrict__ arp,
                   int32_t* __restrict__ list, int* __restrict__ count, unsigned long long* __restrict__ sum_len) {
    const long long r = (long long)blockIdx.x * 256 + threadIdx.x;
    const bool o = r < m && cnt[r] < 0;
    const int lane = threadIdx.x & 63;
    const uint64_t mask = __ballot(o);
    if (!mask) return;
    int base = 0;
    const int leader = __builtin_ctzll(mask);
    if (lane == leader) base = atomicAdd(count, __builtin_popcountll(mask));
    base = __shfl(base, leader);
    if (o) {
        list[base + __builtin_popcountll(mask & ((1ull << lane) - 1))] = (int32_t)r;
        atomicAdd(sum_len, (unsigned long long)(arp[r + 1] - arp[r]));
    }
}

// Row pointers of the gathered sub-matrix (rows of A listed in `list`),
// computed serially per block chunk: lens then a single-block scan.
__global__ void __launch_bounds__(1024)
k_sub_rowptr(int ns, const int32_t* __restrict__ list, const int64_t* __restrict__ arp, int64_t* __restrict__ srp) {
    __shared__ BlockScanSmem<1024> sm;
    long long carry = 0;
    for (int c0 = 0; c0 < ns; c0 += 1024) {
        const int j = c0 + threadIdx.x;
        const long long len = j < ns ? arp[list[j] + 1] - arp[list[j]] : 0;
        long long tot;
        const long long incl = block_incl_scan<1024>(len, sm, &tot);
        if (j < ns) srp[j] = carry + incl - len;
        carry += tot;
    }
    if (threadIdx.x == 0) srp[ns] = carry;
}

template <typename VT>
__global__ void __launch_bounds__(256)
k_sub_gather(int ns, const int32_t* __restrict__ list, const int64_t* __restrict__ arp,
             const int32_t* __restrict__ acol, const VT* __restrict__ aval, const int64_t* __restrict__ srp,
             int32_t* __restrict__ scol, VT* __restrict__ sval) {
    // one wave per listed row
    const long long wid = ((long long)blockIdx.x * 256 + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63;
    if (wid >= ns) return;
    const long long a0 = arp[list[wid]], a1 = arp[list[wid] + 1], d0 = srp[wid];
    for (long long p = a0 + lane; p < a1; p += 64) {
        scol[d0 + p - a0] = acol[p];
        sval[d0 + p - a0] = aval[p];
    }
}

// Overflowed rows take their counts and sources from the sub-product.
__global__ void __launch_bounds__(256)
k_patch_overflow(int ns, const int32_t* __restrict__ list, const int64_t* __restrict__ crp_sub,
                 int32_t* __restrict__ cnt, int64_t* __restrict__ src_off) {
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= ns) return;
    const int r = list[j];
    cnt[r] = (int32_t)(crp_sub[j + 1] - crp_sub[j]);
    src_off[r] = -(crp_sub[j] + 1);              // negative: from the sub-product
}

// Compaction into the tight CSR, balanced by output entries: workgroup b
// writes destination entries [b CH, (b+1) CH) whatever the row lengths, so
// a hub row is spread over many workgroups.  chunk_row[b] is the row that
// holds entry b CH.  A row's source is the padded product at rp_pad[row],
// or the sub-product at -src_off[row]-1 when src_off[row] < 0.
constexpr int kCompactChunk = 4096;
constexpr int kCompactRows = 1024;      // rows staged in LDS per chunk

static __global__ void __launch_bounds__(256)
k_chunk_rows(int m, const int64_t* __restrict__ rp, int32_t* __restrict__ chunk_row) {
    const long long r = (long long)blockIdx.x * 256 + threadIdx.x;
    if (r >= m) return;
    const long long d0 = rp[r], d1 = rp[r + 1];
    for (long long c = (d0 + kCompactChunk - 1) / kCompactChunk; c * kCompactChunk < d1; ++c)
        chunk_row[c] = (int32_t)r;
}

template <typename VT>
__global__ void __launch_bounds__(256)
k_compact(int m, long long nnz, const int32_t* __restrict__ chunk_row, const int64_t* __restrict__ rp,
          const int64_t* __restrict__ rp_pad, const int64_t* __restrict__ src_off, const int32_t* __restrict__ pcol,
          const VT* __restrict__ pval, const int32_t* __restrict__ scol, const VT* __restrict__ sval,
          int32_t* __restrict__ ccol, VT* __restrict__ cval) {
    __shared__ long long s_rp[kCompactRows + 1];
    __shared__ long long s_src[kCompactRows];
    const long long nch = (nnz + kCompactChunk - 1) / kCompactChunk;
    const long long b = blockIdx.x;
    const long long d0 = b * kCompactChunk;
    const long long d1 = d0 + kCompactChunk < nnz ? d0 + kCompactChunk : nnz;
    const int r0 = chunk_row[b];
    const int r1 = b + 1 < nch ? chunk_row[b + 1] : m - 1;   // rows r0..r1 cover [d0, d1)
    const int nr = r1 - r0 + 1;
    // a row's source position of its first entry (negative: from the sub-product)
    auto src_of = [&](int r) -> long long {
        const long long so = src_off ? src_off[r] : 0;
        return so < 0 ? so : rp_pad[r];
    };
    if (nr <= kCompactRows) {
        for (int j = threadIdx.x; j <= nr; j += 256) {
            s_rp[j] = rp[r0 + j];
            if (j < nr) s_src[j] = src_of(r0 + j);
        }
        __syncthreads();
        for (long long d = d0 + threadIdx.x; d < d1; d += 256) {
            int lo = 0, hi = nr;                       // s_rp[lo] <= d < s_rp[hi]
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (s_rp[mid] <= d) lo = mid; else hi = mid;
            }
            const long long so = s_src[lo];
            const long long k = d - s_rp[lo];
            if (so < 0) { ccol[d] = scol[-so - 1 + k]; cval[d] = sval[-so - 1 + k]; }
            else { ccol[d] = pcol[so + k]; cval[d] = pval[so + k]; }
        }
    } else {
        // many short rows: one thread per row, clipped to the chunk
        for (int j = threadIdx.x; j < nr; j += 256) {
            const int r = r0 + j;
            const long long e0 = rp[r], e1 = rp[r + 1];
            const long long a = e0 > d0 ? e0 : d0, z = e1 < d1 ? e1 : d1;
            if (a >= z) continue;
            const long long so = src_of(r);
            for (long long d = a; d < z; ++d) {
                const long long k = d - e0;
                if (so < 0) { ccol[d] = scol[-so - 1 + k]; cval[d] = sval[-so - 1 + k]; }
                else { ccol[d] = pcol[so + k]; cval[d] = pval[so + k]; }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// predictor object
// ---------------------------------------------------------------------------
struct ExtraState {
    DevBuf feat, lo, cap, rp_pad, cnt, src_off, pad, list, sub_rp, sub_a, sub_c, sub_crp, chunk;
};

static ExtraState* extra(msp_handle* h) {
    if (!h->extra) h->extra = new (std::nothrow) ExtraState();
    return h->extra;
}

void release_extra(msp_handle* h) {
    if (!h->extra) return;
    ExtraState* x = h->extra;
    for (DevBuf* b : {&x->feat, &x->lo, &x->cap, &x->rp_pad, &x->cnt, &x->src_off, &x->pad, &x->list, &x->sub_rp,
                      &x->sub_a, &x->sub_c, &x->sub_crp, &x->chunk})
        b->release();
    delete x;
    h->extra = nullptr;
}

static msp_status launch_check2(const char* what) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, what);
    return MSP_OK;
}

}  // namespace msp

struct msp_predictor {
    int device = 0;
    msp::DevBuf params, m, v, grad, loss, bad, part, part_loss;
    float delta = 0.f;
    long long step = 0;
};

extern "C" msp_status msp_predictor_create(msp_handle* h, const float* init_params, msp_predictor** out) {
    if (!h || !init_params || !out) return fail(MSP_ERR_INVALID_ARG, "null argument");
    *out = nullptr;
    hipError_t e = hipSetDevice(h->device);
    if (e != hipSuccess) return hip_fail(e, "hipSetDevice");
    msp_predictor* p = new (std::nothrow) msp_predictor();
    if (!p) return fail(MSP_ERR_OOM, "host allocation failed");
    p->device = h->device;
    msp_status s;
    for (DevBuf* b : {&p->params, &p->m, &p->v, &p->grad, &p->bad}) {
        if ((s = b->ensure(kNParam * sizeof(float))) != MSP_OK) { msp_predictor_destroy(p); return s; }
        if ((e = hipMemsetAsync(b->ptr, 0, kNParam * sizeof(float), h->stream)) != hipSuccess) {
            msp_predictor_destroy(p);
            return hip_fail(e, "hipMemsetAsync");
        }
    }
    if ((e = hipMemcpyAsync(p->params.ptr, init_params, kNParam * sizeof(float), hipMemcpyHostToDevice, h->stream)) !=
            hipSuccess ||
        (e = hipStreamSynchronize(h->stream)) != hipSuccess) {
        msp_predictor_destroy(p);
        return hip_fail(e, "hipMemcpyAsync(params)");
    }
    *out = p;
    return MSP_OK;
}

extern "C" msp_status msp_predictor_destroy(msp_predictor* p) {
    if (!p) return MSP_OK;
    (void)hipSetDevice(p->device);
    for (DevBuf* b :
         {&p->params, &p->m, &p->v, &p->grad, &p->loss, &p->bad, &p->part, &p->part_loss})
        b->release();
    delete p;
    return MSP_OK;
}

extern "C" msp_status msp_predictor_get(msp_handle* h, const msp_predictor* p, float* params, float* delta) {
    if (!h || !p) return fail(MSP_ERR_INVALID_ARG, "null argument");
    if (params) {
        hipError_t e = hipMemcpyAsync(params, p->params.ptr, kNParam * sizeof(float), hipMemcpyDeviceToHost, h->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
        if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync(params)");
    }
    if (delta) *delta = p->delta;
    return MSP_OK;
}

extern "C" msp_status msp_predictor_set(msp_handle* h, msp_predictor* p, const float* params, float delta) {
    if (!h || !p) return fail(MSP_ERR_INVALID_ARG, "null argument");
    if (params) {
        hipError_t e = hipMemcpyAsync(p->params.ptr, params, kNParam * sizeof(float), hipMemcpyHostToDevice, h->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
        if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync(params)");
    }
    p->delta = delta;
    return MSP_OK;
}

// ---------------------------------------------------------------------------
// serialized form (little-endian): magic "MSPP", u32 version, u32 parameter
// count, f32 delta, i64 Adam step count, then the parameters and Adam's two
// moment arrays (f32 each), then a u64 FNV-1a hash of every byte before it
// ---------------------------------------------------------------------------
namespace {
constexpr uint32_t kBlobVersion = 1;
constexpr size_t kBlobHeader = 24;
constexpr size_t kBlobBytes = kBlobHeader + 3 * (size_t)kNParam * 4 + 8;
static_assert(kBlobBytes == MSP_PREDICTOR_BLOB_BYTES, "blob layout and its declared size agree");

uint64_t fnv1a64(const unsigned char* p, size_t n) {
    uint64_t x = 0xcbf29ce484222325ull;
    for (size_t i = 0; i < n; ++i) {
        x ^= p[i];
        x *= 0x100000001b3ull;
    }
    return x;
}
}  // namespace

extern "C" msp_status msp_predictor_blob_pack(const float* params, const float* adam_m, const float* adam_v,
                                              float delta, int64_t step, void* blob, size_t cap, size_t* size) {
    if (size) *size = kBlobBytes;
    if (!blob) return size ? MSP_OK : fail(MSP_ERR_INVALID_ARG, "blob and size are both NULL");
    if (!params) return fail(MSP_ERR_INVALID_ARG, "params is NULL");
    if (cap < kBlobBytes) return fail(MSP_ERR_INVALID_ARG, "blob buffer of %zu bytes, %zu needed", cap, kBlobBytes);
    unsigned char* b = (unsigned char*)blob;
    const uint32_t np = kNParam;
    memcpy(b, "MSPP", 4);
    memcpy(b + 4, &kBlobVersion, 4);
    memcpy(b + 8, &np, 4);
    memcpy(b + 12, &delta, 4);
    memcpy(b + 16, &step, 8);
    unsigned char* q = b + kBlobHeader;
    for (const float* a : {params, adam_m, adam_v}) {
        if (a) memcpy(q, a, (size_t)kNParam * 4);
        else memset(q, 0, (size_t)kNParam * 4);
        q += (size_t)kNParam * 4;
    }
    const uint64_t hsh = fnv1a64(b, kBlobBytes - 8);
    memcpy(q, &hsh, 8);
    return MSP_OK;
}

extern "C" msp_status msp_predictor_blob_unpack(const void* blob, size_t size, float* params, float* adam_m,
                                                float* adam_v, float* delta, int64_t* step) {
    if (!blob) return fail(MSP_ERR_INVALID_ARG, "blob is NULL");
    const unsigned char* b = (const unsigned char*)blob;
    if (size < kBlobHeader || memcmp(b, "MSPP", 4) != 0)
        return fail(MSP_ERR_INVALID_ARG, "not a predictor blob (magic)");
    uint32_t ver = 0, np = 0;
    memcpy(&ver, b + 4, 4);
    memcpy(&np, b + 8, 4);
    if (ver != kBlobVersion)
        return fail(MSP_ERR_UNSUPPORTED, "predictor blob version %u; this library reads version %u", ver, kBlobVersion);
    if (np != (uint32_t)kNParam) return fail(MSP_ERR_INVALID_ARG, "predictor blob holds %u parameters, not %d", np, kNParam);
    if (size != kBlobBytes) return fail(MSP_ERR_INVALID_ARG, "predictor blob of %zu bytes, %zu expected", size, kBlobBytes);
    uint64_t hsh = 0;
    memcpy(&hsh, b + kBlobBytes - 8, 8);
    if (hsh != fnv1a64(b, kBlobBytes - 8)) return fail(MSP_ERR_INVALID_ARG, "predictor blob checksum mismatch");
    if (delta) memcpy(delta, b + 12, 4);
    if (step) memcpy(step, b + 16, 8);
    const unsigned char* q = b + kBlobHeader;
    for (float* a : {params, adam_m, adam_v}) {
        if (a) memcpy(a, q, (size_t)kNParam * 4);
        q += (size_t)kNParam * 4;
    }
    return MSP_OK;
}

extern "C" msp_status msp_predictor_save(msp_handle* h, const msp_predictor* p, void* blob, size_t cap, size_t* size) {
    if (!h || !p) return fail(MSP_ERR_INVALID_ARG, "null argument");
    if (size) *size = kBlobBytes;
    if (!blob) return size ? MSP_OK : fail(MSP_ERR_INVALID_ARG, "blob and size are both NULL");
    if (cap < kBlobBytes) return fail(MSP_ERR_INVALID_ARG, "blob buffer of %zu bytes, %zu needed", cap, kBlobBytes);
    hipError_t e = hipSetDevice(h->device);
    if (e != hipSuccess) return hip_fail(e, "hipSetDevice");
    std::vector<float> host(3 * (size_t)kNParam);
    const DevBuf* src[3] = {&p->params, &p->m, &p->v};
    for (int i = 0; i < 3 && e == hipSuccess; ++i)
        e = hipMemcpyAsync(host.data() + (size_t)i * kNParam, src[i]->ptr, (size_t)kNParam * 4, hipMemcpyDeviceToHost,
                           h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync(predictor state)");
    return msp_predictor_blob_pack(host.data(), host.data() + kNParam, host.data() + 2 * kNParam, p->delta, p->step,
                                   blob, cap, nullptr);
}

extern "C" msp_status msp_predictor_load(msp_handle* h, msp_predictor* p, const void* blob, size_t size) {
    if (!h || !p) return fail(MSP_ERR_INVALID_ARG, "null argument");
    std::vector<float> host(3 * (size_t)kNParam);
    float delta = 0.f;
    int64_t step = 0;
    msp_status s = msp_predictor_blob_unpack(blob, size, host.data(), host.data() + kNParam,
                                             host.data() + 2 * kNParam, &delta, &step);
    if (s != MSP_OK) return s;
    if (step < 0) return fail(MSP_ERR_INVALID_ARG, "predictor blob has a negative step count");
    hipError_t e = hipSetDevice(h->device);
    if (e != hipSuccess) return hip_fail(e, "hipSetDevice");
    DevBuf* dst[3] = {&p->params, &p->m, &p->v};
    for (int i = 0; i < 3 && e == hipSuccess; ++i)
        e = hipMemcpyAsync(dst[i]->ptr, host.data() + (size_t)i * kNParam, (size_t)kNParam * 4, hipMemcpyHostToDevice,
                           h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync(predictor state)");
    p->delta = delta;
    p->step = step;
    return MSP_OK;
}

// One forward and backward pass on batch rows idx[0..batch) and the gradient;
// with `adam`, also the parameters' update (p->step counts this step).
// (k_mlp_tiles steps over the batch in 32 bits, kTileWG tiles at a time)
constexpr int kMaxBatch = INT32_MAX - 2 * kTile * kTileWG;
static msp_status grad_step(msp_handle* h, msp_predictor* p, const float* feats, const float* targets, int64_t n,
                            const int32_t* idx, int batch, float* loss_dev, const msp_train_opts* adam) {
    if (batch > kMaxBatch) return fail(MSP_ERR_INDEX_OVERFLOW, "at most %d samples a batch", kMaxBatch);
    const int parts = std::min((batch + kTile - 1) / kTile, kTileWG);
    msp_status s;
    if ((s = p->part.ensure((size_t)parts * kPartRow * 8)) != MSP_OK ||
        (s = p->part_loss.ensure((size_t)parts * 8)) != MSP_OK)
        return s;
    k_mlp_tiles<<<parts, 256, 0, h->stream>>>(batch, n, idx, feats, targets, p->params.as<float>(),
                                              p->part.as<double>(), p->part_loss.as<double>(), p->bad.as<int>());
    if ((s = launch_check2("k_mlp_tiles")) != MSP_OK) return s;
    if (adam)
        k_mlp_sum<true><<<kSumGrid, kSumP * kSumT, 0, h->stream>>>(
            parts, batch, p->part.as<double>(), p->part_loss.as<double>(), p->grad.as<float>(), loss_dev,
            p->params.as<float>(), p->m.as<float>(), p->v.as<float>(), (int)p->step, adam->lr, adam->beta1,
            adam->beta2, adam->eps);
    else
        k_mlp_sum<false><<<kSumGrid, kSumP * kSumT, 0, h->stream>>>(
            parts, batch, p->part.as<double>(), p->part_loss.as<double>(), p->grad.as<float>(), loss_dev, nullptr,
            nullptr, nullptr, 0, 0.f, 0.f, 0.f, 0.f);
    return launch_check2("k_mlp_sum");
}

// Sample indices outside [0, n) were flagged by the forward/backward kernel:
// report them (and clear the flag) once the stream has drained.
static msp_status take_bad_index(msp_handle* h, msp_predictor* p) {
    int bad = 0;
    hipError_t e = hipMemcpyAsync(&bad, p->bad.ptr, sizeof(int), hipMemcpyDeviceToHost, h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync(index flag)");
    if (!bad) return MSP_OK;
    if ((e = hipMemsetAsync(p->bad.ptr, 0, sizeof(int), h->stream)) != hipSuccess) return hip_fail(e, "hipMemsetAsync");
    return fail(MSP_ERR_INVALID_ARG, "a batch index is outside [0, n)");
}

extern "C" msp_status msp_predictor_grad(msp_handle* h, msp_predictor* p, const float* feats, const float* targets,
                                         int64_t n, const int32_t* idx, int batch, float* grad_host,
                                         float* loss_host) {
    if (!h || !p || !feats || !targets || !idx || batch <= 0 || n <= 0) return fail(MSP_ERR_INVALID_ARG, "bad argument");
    hipError_t e = hipSetDevice(h->device);
    if (e != hipSuccess) return hip_fail(e, "hipSetDevice");
    msp_status s = p->loss.ensure(sizeof(float));
    if (s != MSP_OK) return s;
    if ((s = grad_step(h, p, feats, targets, n, idx, batch, p->loss.as<float>(), nullptr)) != MSP_OK) return s;
    if (grad_host &&
        (e = hipMemcpyAsync(grad_host, p->grad.ptr, kNParam * 4, hipMemcpyDeviceToHost, h->stream)) != hipSuccess)
        return hip_fail(e, "hipMemcpyAsync(grad)");
    if (loss_host && (e = hipMemcpyAsync(loss_host, p->loss.ptr, 4, hipMemcpyDeviceToHost, h->stream)) != hipSuccess)
        return hip_fail(e, "hipMemcpyAsync(loss)");
    if ((e = hipStreamSynchronize(h->stream)) != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
    return take_bad_index(h, p);
}

extern "C" msp_status msp_predictor_train(msp_handle* h, msp_predictor* p, const float* feats, const float* targets,
                                          int64_t n, const int32_t* batch_idx, int steps, int batch,
                                          const msp_train_opts* o, float* losses_host) {
    if (!h || !p || !feats || !targets || !batch_idx || n <= 0 || steps < 0 || batch <= 0)
        return fail(MSP_ERR_INVALID_ARG, "bad argument");
    hipError_t e = hipSetDevice(h->device);
    if (e != hipSuccess) return hip_fail(e, "hipSetDevice");
    msp_train_opts a;
    a.lr = o && o->lr > 0 ? o->lr : 1e-3f;
    a.beta1 = o && o->beta1 > 0 ? o->beta1 : 0.9f;
    a.beta2 = o && o->beta2 > 0 ? o->beta2 : 0.999f;
    a.eps = o && o->eps > 0 ? o->eps : 1e-8f;
    msp_status s = p->loss.ensure((size_t)std::max(steps, 1) * sizeof(float));
    if (s != MSP_OK) return s;
    for (int t = 0; t < steps; ++t) {
        ++p->step;
        if ((s = grad_step(h, p, feats, targets, n, batch_idx + (size_t)t * batch, batch, p->loss.as<float>() + t,
                           &a)) != MSP_OK) {
            --p->step;
            return s;
        }
    }
    if (losses_host && steps > 0 &&
        (e = hipMemcpyAsync(losses_host, p->loss.ptr, (size_t)steps * 4, hipMemcpyDeviceToHost, h->stream)) !=
            hipSuccess)
        return hip_fail(e, "hipMemcpyAsync(losses)");
    if ((e = hipStreamSynchronize(h->stream)) != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
    return take_bad_index(h, p);
}

extern "C" msp_status msp_predictor_infer(msp_handle* h, const msp_predictor* p, const float* feats, int64_t n,
                                          float* y) {
    if (!h || !p || (n > 0 && (!feats || !y)) || n < 0) return fail(MSP_ERR_INVALID_ARG, "bad argument");
    hipError_t e = hipSetDevice(h->device);
    if (e != hipSuccess) return hip_fail(e, "hipSetDevice");
    if (n == 0) return MSP_OK;
    const long long blocks = (n + 255) / 256;
    if (blocks > INT32_MAX) return fail(MSP_ERR_INDEX_OVERFLOW, "too many rows");
    k_mlp_predict<<<(int)blocks, 256, 0, h->stream>>>(n, feats, p->params.as<float>(), y);
    return launch_check2("k_mlp_predict");
}

// delta = the q-quantile of 16 (t - y) over the rows given (log2 units).
extern "C" msp_status msp_predictor_calibrate(msp_handle* h, msp_predictor* p, const float* feats,
                                              const float* targets, int64_t n, double q) {
    if (!h || !p || !feats || !targets || n <= 0 || !(q > 0 && q < 1)) return fail(MSP_ERR_INVALID_ARG, "bad argument");
    DevBuf y;
    msp_status s = y.ensure((size_t)n * 4);
    if (s != MSP_OK) return s;
    if ((s = msp_predictor_infer(h, p, feats, n, y.as<float>())) != MSP_OK) { y.release(); return s; }
    std::vector<float> yh((size_t)n), th((size_t)n);
    hipError_t e = hipMemcpyAsync(yh.data(), y.ptr, (size_t)n * 4, hipMemcpyDeviceToHost, h->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(th.data(), targets, (size_t)n * 4, hipMemcpyDeviceToHost, h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    y.release();
    if (e != hipSuccess) return hip_fail(e, "calibration copy");
    std::vector<float> res((size_t)n);
    for (size_t i = 0; i < (size_t)n; ++i) res[i] = 16.f * (th[i] - yh[i]);
    const size_t k = std::min((size_t)n - 1, (size_t)std::ceil(q * (double)n) - 1);
    std::nth_element(res.begin(), res.begin() + k, res.end());
    p->delta = res[k];
    return MSP_OK;
}

// ---------------------------------------------------------------------------
// the one-pass product
// ---------------------------------------------------------------------------
extern "C" msp_status msp_spgemm_learned(msp_handle* h, const msp_predictor* p, const msp_csr* A, const msp_csr* B,
                                         msp_csr_out* C, const msp_opts* opts, msp_learned_stats* st) {
    if (!h || !p) return fail(MSP_ERR_INVALID_ARG, "null handle or predictor");
    if (!C) return fail(MSP_ERR_INVALID_ARG, "C is NULL");
    msp_status s = check_pair(A, B);
    if (s != MSP_OK) return s;
    hipError_t e = hipSetDevice(h->device);
    if (e != hipSuccess) return hip_fail(e, "hipSetDevice");
    ExtraState* x = extra(h);
    if (!x) return fail(MSP_ERR_OOM, "host allocation failed");
    const msp_tuning t = effective_tuning(h, opts);
    const int m = (int)A->nrows;
    const size_t vsz = A->dtype == MSP_F64 ? 8 : 4;
    if (opts && opts->validate && (s = validate_inputs(h, A, B)) != MSP_OK) return s;
    msp_learned_stats stats;
    memset(&stats, 0, sizeof(stats));

    const size_t mm = (size_t)std::max(m, 1);
    if ((s = h->rnnz.ensure(mm * 4)) != MSP_OK || (s = x->feat.ensure(mm * kNF * 4)) != MSP_OK ||
        (s = x->lo.ensure(mm * 4)) != MSP_OK || (s = x->cap.ensure(mm * 4)) != MSP_OK ||
        (s = x->rp_pad.ensure((mm + 1) * 8)) != MSP_OK || (s = x->cnt.ensure(mm * 4)) != MSP_OK)
        return s;

    bool own_rp = false;
    if (!C->row_ptr) {
        C->row_ptr = (int64_t*)h->alloc(h->alloc_ctx, (size_t)(m + 1) * 8, h->stream);
        if (!C->row_ptr) return fail(MSP_ERR_OOM, "allocation of C.row_ptr failed");
        own_rp = true;
    }
    C->col = nullptr;
    C->val = nullptr;
    auto cleanup = [&](msp_status r) {
        if (C->col) h->free_fn(h->alloc_ctx, C->col, h->stream);
        C->col = nullptr;
        C->val = nullptr;
        if (own_rp) { h->free_fn(h->alloc_ctx, C->row_ptr, h->stream); C->row_ptr = nullptr; }
        return r;
    };

    // 1. features and bounds, 2. capacities
    BinPlan none;
    memset(&none, 0, sizeof(none));
    if ((s = zero_info(h)) != MSP_OK) return cleanup(s);
    h->prof.begin(MSP_PHASE_ROW_STATS, h->stream);
    if ((s = run_row_stats(h, A, B, none, nullptr, x->feat.as<float>(), x->lo.as<int32_t>())) != MSP_OK)
        return cleanup(s);
    h->prof.end(h->stream);
    const BinPlan np = numeric_plan(t, opts && opts->force_spill);
    h->prof.begin(MSP_PHASE_PREDICT, h->stream);
    if (m > 0) {
        const int blocks = (m + 255) / 256;
        // rows whose capacity falls in the global bin take the exact path
        const int big = (opts && opts->force_spill) || np.table.nb <= 1 ? -1 : np.table.umax[np.table.nb - 1];
        k_capacity<<<blocks, 256, 0, h->stream>>>(m, x->feat.as<float>(), h->u.as<int32_t>(), x->lo.as<int32_t>(),
                                                  p->params.as<float>(), p->delta, x->cap.as<int32_t>(),
                                                  x->cnt.as<int32_t>(),
                                                  numeric_plan(t, opts && opts->force_spill, true).table, big,
                                                  &h->info.as<DevInfo>()->learned_big,
                                                  &h->info.as<DevInfo>()->learned_big_hi);
        if ((s = launch_check2("k_capacity")) != MSP_OK) return cleanup(s);
    }
    h->prof.end(h->stream);
    // 3. padded row pointers and bins by capacity
    h->prof.begin(MSP_PHASE_SCAN, h->stream);
    if ((s = run_scan(h, m, x->cap.as<int32_t>(), x->rp_pad.as<int64_t>(), &np)) != MSP_OK) return cleanup(s);
    h->prof.end(h->stream);
    if ((s = read_info(h)) != MSP_OK) return cleanup(s);
    if ((s = device_error(h->hinfo->err)) != MSP_OK) return cleanup(s);
    const long long sum_cap = h->hinfo->nnz;
    stats.sum_cap = sum_cap;
    stats.exact_rows = h->hinfo->learned_big;
    if (stats.exact_rows > 0 && (long long)h->hinfo->learned_big_hi > sum_cap) {
        // more of the bounded work is in rows that take the exact path anyway
        // than in the predicted rows: the two-phase product of the whole
        // matrix does less than the two paths together
        msp_opts so;
        memset(&so, 0, sizeof(so));
        so.tuning = t;
        s = spgemm_core(
            h, A, B, C, &so, [h](size_t bytes) -> void* { return h->alloc(h->alloc_ctx, bytes, h->stream); },
            [h](void* ptr) { h->free_fn(h->alloc_ctx, ptr, h->stream); });
        if (s != MSP_OK) return cleanup(s);
        stats.exact_rows = m;
        stats.sum_cap = 0;
        stats.overflow_rows = 0;
        stats.nnz = C->nnz;
        if (st) *st = stats;
        return MSP_OK;
    }
    int counts[kNB];
    sum_parts(h->hinfo->num_part, counts);
    // 4. numeric pass in capacity mode into the padded area
    if ((s = x->pad.ensure((size_t)std::max(sum_cap, 1LL) * (4 + vsz) + 256)) != MSP_OK) return cleanup(s);
    int32_t* pcol = x->pad.as<int32_t>();
    char* pval = (char*)x->pad.ptr + (((size_t)std::max(sum_cap, 1LL) * 4 + 255) & ~(size_t)255);
    // (the device info is not cleared here: the scatter of rows into bins
    // reads the per-partition bin counts that the scan just wrote)
    h->prof.begin(MSP_PHASE_NUMERIC, h->stream);
    if ((s = run_numeric_bins(h, A, B, np, counts, x->cap.as<int32_t>(), x->rp_pad.as<int64_t>(), pcol, pval,
                              x->cnt.as<int32_t>())) != MSP_OK)
        return cleanup(s);
    h->prof.end(h->stream);
    // 5. final row pointers (overflowed rows count 0 for now) and overflow count
    h->prof.begin(MSP_PHASE_COMPACT, h->stream);
    if ((s = zero_info(h)) != MSP_OK) return cleanup(s);
    if ((s = run_scan(h, m, x->cnt.as<int32_t>(), C->row_ptr, nullptr)) != MSP_OK) return cleanup(s);
    h->prof.end(h->stream);
    if ((s = read_info(h)) != MSP_OK) return cleanup(s);
    if ((s = device_error(h->hinfo->err)) != MSP_OK) return cleanup(s);
    const int novf = h->hinfo->neg_count;
    stats.overflow_rows = novf - stats.exact_rows;
    int64_t* src_off = nullptr;
    int32_t* scol = nullptr;
    char* sval = nullptr;
    if (novf > 0) {
        // 6. exact recomputation of the overflowed rows on their sub-matrix
        h->prof.begin(MSP_PHASE_FALLBACK, h->stream);
        if ((s = x->list.ensure((size_t)novf * 4)) != MSP_OK || (s = x->src_off.ensure(mm * 8)) != MSP_OK ||
            (s = x->sub_rp.ensure(((size_t)novf + 1) * 8)) != MSP_OK)
            return cleanup(s);
        if ((e = hipMemsetAsync(x->src_off.ptr, 0, mm * 8, h->stream)) != hipSuccess)
            return cleanup(hip_fail(e, "hipMemsetAsync"));
        if ((s = zero_info(h)) != MSP_OK) return cleanup(s);
        DevInfo* info = h->info.as<DevInfo>();
        k_collect_overflow<<<(m + 255) / 256, 256, 0, h->stream>>>(m, x->cnt.as<int32_t>(), A->row_ptr,
                                                                   x->list.as<int32_t>(), &info->neg_count,
                                                                   (unsigned long long*)&info->nnz);
        if ((s = launch_check2("k_collect_overflow")) != MSP_OK) return cleanup(s);
        if ((s = read_info(h)) != MSP_OK) return cleanup(s);
        const long long sub_nnz = h->hinfo->nnz;
        if (h->hinfo->neg_count != novf) return cleanup(fail(MSP_ERR_HIP, "internal: overflow list size"));
        if ((s = x->sub_a.ensure((size_t)std::max(sub_nnz, 1LL) * (4 + vsz) + 256)) != MSP_OK) return cleanup(s);
        int32_t* sacol = x->sub_a.as<int32_t>();
        char* saval = (char*)x->sub_a.ptr + (((size_t)std::max(sub_nnz, 1LL) * 4 + 255) & ~(size_t)255);
        k_sub_rowptr<<<1, 1024, 0, h->stream>>>(novf, x->list.as<int32_t>(), A->row_ptr, x->sub_rp.as<int64_t>());
        if ((s = launch_check2("k_sub_rowptr")) != MSP_OK) return cleanup(s);
        const int gb = (int)(((long long)novf * 64 + 255) / 256);
        if (A->dtype == MSP_F64)
            k_sub_gather<double><<<gb, 256, 0, h->stream>>>(novf, x->list.as<int32_t>(), A->row_ptr, A->col,
                                                            (const double*)A->val, x->sub_rp.as<int64_t>(), sacol,
                                                            (double*)saval);
        else
            k_sub_gather<float><<<gb, 256, 0, h->stream>>>(novf, x->list.as<int32_t>(), A->row_ptr, A->col,
                                                           (const float*)A->val, x->sub_rp.as<int64_t>(), sacol,
                                                           (float*)saval);
        if ((s = launch_check2("k_sub_gather")) != MSP_OK) return cleanup(s);
        msp_csr Asub{novf, A->ncols, sub_nnz, x->sub_rp.as<int64_t>(), sacol, saval, A->dtype};
        if ((s = x->sub_crp.ensure(((size_t)novf + 1) * 8)) != MSP_OK) return cleanup(s);
        msp_csr_out Csub;
        memset(&Csub, 0, sizeof(Csub));
        Csub.row_ptr = x->sub_crp.as<int64_t>();
        DevBuf* subc = &x->sub_c;
        auto ws_alloc = [subc](size_t bytes) -> void* {
            if (subc->ensure(std::max(bytes, (size_t)256)) != MSP_OK) return nullptr;
            return subc->ptr;
        };
        msp_opts so;
        memset(&so, 0, sizeof(so));
        so.tuning = t;
        if ((s = spgemm_core(h, &Asub, B, &Csub, &so, ws_alloc, [](void*) {})) != MSP_OK) return cleanup(s);
        scol = Csub.col;
        sval = (char*)Csub.val;
        k_patch_overflow<<<(novf + 255) / 256, 256, 0, h->stream>>>(novf, x->list.as<int32_t>(), Csub.row_ptr,
                                                                    x->cnt.as<int32_t>(), x->src_off.as<int64_t>());
        if ((s = launch_check2("k_patch_overflow")) != MSP_OK) return cleanup(s);
        if ((s = zero_info(h)) != MSP_OK) return cleanup(s);
        if ((s = run_scan(h, m, x->cnt.as<int32_t>(), C->row_ptr, nullptr)) != MSP_OK) return cleanup(s);
        if ((s = read_info(h)) != MSP_OK) return cleanup(s);
        if ((s = device_error(h->hinfo->err)) != MSP_OK) return cleanup(s);
        if (h->hinfo->neg_count != 0) return cleanup(fail(MSP_ERR_HIP, "internal: rows left after the fallback"));
        src_off = x->src_off.as<int64_t>();
        h->prof.end(h->stream);
    }
    // 7. tight output
    const long long nnz = h->hinfo->nnz;
    stats.nnz = nnz;
    C->nrows = m;
    C->ncols = B->ncols;
    C->nnz = nnz;
    C->dtype = A->dtype;
    if (nnz > 0) {
        const size_t voff = ((size_t)nnz * 4 + 255) & ~(size_t)255;
        void* base = h->alloc(h->alloc_ctx, voff + (size_t)nnz * vsz, h->stream);
        if (!base) return cleanup(fail(MSP_ERR_OOM, "allocation of C (%lld nonzeros) failed", nnz));
        C->col = (int32_t*)base;
        C->val = (char*)base + voff;
        const long long nch = (nnz + kCompactChunk - 1) / kCompactChunk;
        if (nch > INT32_MAX) return cleanup(fail(MSP_ERR_INDEX_OVERFLOW, "too many output entries"));
        if ((s = x->chunk.ensure((size_t)nch * 4)) != MSP_OK) return cleanup(s);
        h->prof.begin(MSP_PHASE_COMPACT, h->stream);
        k_chunk_rows<<<(m + 255) / 256, 256, 0, h->stream>>>(m, C->row_ptr, x->chunk.as<int32_t>());
        if ((s = launch_check2("k_chunk_rows")) != MSP_OK) return cleanup(s);
        if (A->dtype == MSP_F64)
            k_compact<double><<<(int)nch, 256, 0, h->stream>>>(m, nnz, x->chunk.as<int32_t>(), C->row_ptr,
                                                              x->rp_pad.as<int64_t>(), src_off, pcol,
                                                              (const double*)pval, scol, (const double*)sval, C->col,
                                                              (double*)C->val);
        else
            k_compact<float><<<(int)nch, 256, 0, h->stream>>>(m, nnz, x->chunk.as<int32_t>(), C->row_ptr,
                                                             x->rp_pad.as<int64_t>(), src_off, pcol,
                                                             (const float*)pval, scol, (const float*)sval, C->col,
                                                             (float*)C->val);
        if ((s = launch_check2("k_compact")) != MSP_OK) return cleanup(s);
        h->prof.end(h->stream);
        hipError_t e2 = hipMemcpyAsync(h->hpending, &h->info.as<DevInfo>()->err, sizeof(int), hipMemcpyDeviceToHost,
                                       h->stream);
        if (e2 != hipSuccess) return cleanup(hip_fail(e2, "hipMemcpyAsync(error flags)"));
    }
    if (st) *st = stats;
    return MSP_OK;
}

extern "C" msp_status msp_training_rows(msp_handle* h, const msp_csr* A, const msp_csr* B, float* features,
                                        float* targets) {
    if (!h) return fail(MSP_ERR_INVALID_ARG, "null handle");
    msp_status s = check_pair(A, B);
    if (s != MSP_OK) return s;
    const int m = (int)A->nrows;
    if (m > 0 && (!features || !targets)) return fail(MSP_ERR_INVALID_ARG, "null output");
    if ((s = msp_row_features(h, A, B, nullptr, features)) != MSP_OK) return s;
    int64_t tot = 0;
    DevBuf rn;
    if ((s = rn.ensure((size_t)std::max(m, 1) * 4)) != MSP_OK) return s;
    if ((s = msp_spgemm_symbolic(h, A, B, rn.as<int32_t>(), &tot, nullptr)) != MSP_OK) { rn.release(); return s; }
    if (m > 0) k_targets<<<(m + 255) / 256, 256, 0, h->stream>>>(m, rn.as<int32_t>(), targets);
    s = launch_check2("k_targets");
    hipError_t e = hipStreamSynchronize(h->stream);
    rn.release();
    if (s == MSP_OK && e != hipSuccess) s = hip_fail(e, "hipStreamSynchronize");
    return s;
}

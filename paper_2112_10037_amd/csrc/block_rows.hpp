// Workgroup row kernels: one workgroup of BS threads per row, the row's
// products in registers (R a thread) while they are ordered in LDS.
#pragma once

#include "list_walk.hpp"

namespace msp {

// Numeric, one workgroup per row of at most BS R products and fewer than 3/4 as
// many A entries, by a counting sort: the columns' span is cut into 16 BS buckets of equal
// width (a power of two), an LDS atomic counts the buckets and gives each
// product its place, the counts are scanned, (column, value) pairs placed,
// and each pair counts its bucket's smaller columns.  The pairs are ranked in
// place order, so that the lanes of a wave work on neighbouring buckets and
// a skewed matrix's full buckets hold up few waves.  Sums over equal columns,
// now neighbours, go out in order.  A row of one nonempty B row is its copy,
// scaled.  Rows past those limits, or with more than kSortBucket products in
// a bucket, are left to a hash kernel with a table of the bin's size: rows whose
// products merge several to an output can be most of a bin.  left_of[row] says
// which (1 or 0), *left how many.
//
// The walk finds a product's A entry as the row kernels of one wave do: a mark
// per entry at its last product, counted below the lane.
//
// Bound by LDS and barriers (about ten a row, spread over the compute unit's
// two to nine workgroups).  Measured on a sparse power-law matrix of 2^20 rows
// (FP32): rows of 2049 to 4096 outputs 3272 us in the LDS hash with its radix
// sort before, 1257 us here and 373 in the hash behind; rows of 1025 to 2048
// 2741 us (with those of 513 to 1024), 800 and 146 here; rows of 513 to 1024
// outputs of a uniform FP64 matrix 1329 -> 284 us.  Without the check of each
// column's neighbour and the rows' marks, and with one draw a row, these took
// 1138, 767 and 488 us; then nine products a thread, which spill, 1708, 1022 and
// 543; half the buckets 1160, 888 and 489; 128 registers for the smaller
// workgroups too 1139, 765 and 524.
constexpr int kSortBucket = 256;
constexpr int kSortR = 8;

// The slots a workgroup of the sort draws from the row queue, thread 0's, in
// LDS.  The draws of one queue follow each other at some 12 ns, more than a
// row that the sort leaves takes (60,000 of them 711 us, drawn one by one): a
// draw takes half of the workgroup's share of what is left, up to eight slots,
// so that the last rows still go one by one (a fixed eighth of the whole share
// made the last rows of a sparse power-law matrix's 2049- to 4096-output bin
// wait, 1163 -> 1495 us).  The pointers are kept here too, out of the kernel's
// registers.
struct SortRows {
    unsigned* q;
    int32_t* left_of;
    int* left;
    long long at;
    int rows, held, nleft;

    __device__ __forceinline__ void open(unsigned* q_, int rows_, int32_t* left_of_, int* left_, long long slot,
                                         long long* s_slot) {
        q = q_;
        rows = rows_;
        at = 0;
        left_of = left_of_;
        left = left_;
        held = nleft = 0;
        draw(slot, s_slot);
    }
    __device__ __forceinline__ void draw(long long slot, long long* s_slot) {
        if (!q) {
            *s_slot = slot + gridDim.x;
            return;
        }
        int n = held;
        long long to = at;
        if (n == 0) {
            // (what is left at this workgroup's last draw)
            n = (int)min(8ll, (rows - to) / (2 * (long long)gridDim.x));
            n = max(n, 1);
            to = (long long)atomicAdd(q, (unsigned)n);
        }
        *s_slot = to;
        at = to + 1;
        held = n - 1;
    }
    __device__ __forceinline__ void close(int row, bool done) {
        left_of[row] = !done;
        nleft += !done;
    }
    __device__ __forceinline__ void finish() {
        if (nleft > 0) atomicAdd(left, nleft);
    }
};

template <int BS, int R>
struct SortCfg {
    static constexpr int kCap = BS * R;                  // products
    static constexpr int kBuckets = 16 * BS;
    static constexpr int kWords = kCap / 64;             // mark words
    static constexpr int kEntries = kCap / 4 * 3 - 1;    // A entries: their 16 bytes take the pairs' place
    static_assert(kWords <= 128, "two mark words a lane");
};

template <int BS, int R, typename VT, bool BATCH = false>
__global__ void __launch_bounds__(BS, BS <= 256 ? 3 : 4)
k_num_sort(Work wk,
           const int64_t* __restrict__ arp, const int32_t* __restrict__ acol, const VT* __restrict__ aval,
           const int64_t* __restrict__ brp, const int32_t* __restrict__ bcol, const VT* __restrict__ bval,
           const int64_t* __restrict__ crp, int32_t* __restrict__ ccol, VT* __restrict__ cval,
           int32_t* __restrict__ cnt_out, DevInfo* info, RowMap mp, unsigned* q,
           int32_t* left_of, int* left) {
    using Cfg = SortCfg<BS, R>;
    constexpr int CAP = Cfg::kCap, NB = Cfg::kBuckets, NW = BS / 64, WORDS = Cfg::kWords;
    int nrows_bin;
    const int32_t* perm;
    work_rows(wk, &nrows_bin, &perm);
    __shared__ __align__(16) uint32_t cw[NB / 2];        // two 16-bit counters, later first positions, a word
    __shared__ __align__(16) unsigned char area[CAP * 12];
    double* const sv = reinterpret_cast<double*>(area);                  // the pairs; before them the entries
    int32_t* const sc = reinterpret_cast<int32_t*>(area + CAP * 8);
    long long* const base = reinterpret_cast<long long*>(area);
    VT* const av = reinterpret_cast<VT*>(area + (Cfg::kEntries + 1) * 8);
    __shared__ unsigned long long mark[WORDS];
    __shared__ long long s_slot;
    __shared__ SortRows rows;
    __shared__ int s_sum[NW], s_some[NW], s_min[NW], s_max[NW], s_tot[NW], s_most[NW], s_heads[NW];
    const uint16_t* const cs = reinterpret_cast<const uint16_t*>(cw);
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    int err = 0;

    struct Head {
        int row, expect;
        long long a0, a1, rp, bo;
    };
    auto head_of = [&](long long slot) {
        Head h;
        h.row = __builtin_amdgcn_readfirstlane(perm ? perm[slot] : (int)slot);
        h.a0 = arp[h.row];
        h.a1 = arp[h.row + 1];
        h.rp = crp[h.row];
        h.expect = (int)(crp[h.row + 1] - h.rp);
        h.bo = row_boff<BATCH>(mp, h.row);
        return h;
    };
    // threads past a row's entries repeat its last one
    auto load_entry = [&](const Head& h, int* k, VT* a) {
        if (h.a1 <= h.a0) return;
        const long long p = h.a0 + tid < h.a1 ? h.a0 + tid : h.a1 - 1;
        *k = acol[p];
        *a = aval[p];
    };
    auto load_bounds = [&](const Head& h, int k, long long* b0, long long* b1) {
        if (h.a1 <= h.a0) return;
        *b0 = brp[k + h.bo];
        *b1 = brp[k + h.bo + 1];
    };

    if (tid == 0) rows.open(q, nrows_bin, left_of, left, (long long)blockIdx.x - gridDim.x, &s_slot);
    __syncthreads();
    long long slot = s_slot;
    __syncthreads();                                       // (a row may come to the next draw without another)
    if (slot < nrows_bin) {                                // uniform
        Head cur = head_of(slot);
        int k = 0, kn = 0;
        VT a = (VT)0, an = (VT)0;
        long long b0 = 0, b1 = 0, b0n = 0, b1n = 0;
        load_entry(cur, &k, &a);
        load_bounds(cur, k, &b0, &b1);
        while (true) {
            const int row = cur.row, expect = cur.expect;
            const long long rp = cur.rp, na = cur.a1 - cur.a0;
            // A entries, BS at a time (the first ones were loaded ahead): prefix
            // of the B-row lengths, marks, positions
            for (int i = tid; i < WORDS; i += BS) mark[i] = 0ull;
            for (int i = tid; i < NB / 8; i += BS) reinterpret_cast<uint4*>(cw)[i] = make_uint4(0, 0, 0, 0);
            int total = 0, entries = 0;
            for (long long e0 = 0; e0 < na && na <= Cfg::kEntries && total <= CAP; e0 += BS) {     // uniform
                if (e0 > 0) {
                    if (e0 + tid < na) {
                        const long long kk = acol[cur.a0 + e0 + tid] + cur.bo;
                        a = aval[cur.a0 + e0 + tid];
                        b0 = brp[kk];
                        b1 = brp[kk + 1];
                    }
                    __syncthreads();                       // the wave sums before are read
                }
                int n = 0;
                if (e0 + tid < na) n = (int)(b1 - b0 < CAP + 1 ? b1 - b0 : CAP + 1);
                const int incl = wave_scan(n);
                const uint64_t some = __ballot(n > 0);
                if (lane == 63) {
                    s_sum[wv] = incl;
                    s_some[wv] = __builtin_popcountll(some);
                }
                __syncthreads();
                int first = total + incl - n, idx = entries;
#pragma unroll
                for (int i = 0; i < NW; ++i) {
                    if (i < wv) {
                        first += s_sum[i];
                        idx += s_some[i];
                    }
                    total = min(total + s_sum[i], 1 << 24);
                    entries += s_some[i];
                }
                if (n > 0 && first + n <= CAP) {
                    idx = lanes_below(some, idx);
                    base[idx] = b0 - first;
                    av[idx] = a;
                    const int last = first + n - 1;
                    atomicOr(reinterpret_cast<uint32_t*>(mark) + (last >> 5), 1u << (last & 31));
                }
            }
            const bool takes = na <= Cfg::kEntries && total <= CAP;   // uniform
            if (tid == 0) rows.draw(slot, &s_slot);
            __syncthreads();
            const long long next = s_slot;
            const bool more = next < nrows_bin;            // uniform
            const Head nxt = head_of(more ? next : slot);
            bool done = false;
            int c[R];
            VT v[R], ae[R];
            // lane i of every wave: mark words i and 64 + i, and the marks before them
            int lo0 = 0, hi0 = 0, pre0 = 0, lo1 = 0, hi1 = 0, pre1 = 0;
            auto entry = [&](int s) {                      // entry of product ((s NW + wave) 64 + lane)
                const int i = (s * NW & 63) + wv;
                if (s * NW < 64)
                    return lanes_below((uint32_t)__builtin_amdgcn_readlane(lo0, i),
                                       (uint32_t)__builtin_amdgcn_readlane(hi0, i), __builtin_amdgcn_readlane(pre0, i));
                return lanes_below((uint32_t)__builtin_amdgcn_readlane(lo1, i),
                                   (uint32_t)__builtin_amdgcn_readlane(hi1, i), __builtin_amdgcn_readlane(pre1, i));
            };
            auto place_of = [&](int s) { return (s * NW + wv) * 64 + lane; };
            if (takes) {
                const unsigned long long w0 = lane < WORDS ? mark[lane] : 0ull;
                const unsigned long long w1 = 64 + lane < WORDS ? mark[64 + lane] : 0ull;
                lo0 = (int)(uint32_t)w0;
                hi0 = (int)(uint32_t)(w0 >> 32);
                lo1 = (int)(uint32_t)w1;
                hi1 = (int)(uint32_t)(w1 >> 32);
                const int n0 = __builtin_popcountll(w0), n1 = __builtin_popcountll(w1);
                pre0 = wave_scan(n0);
                pre1 = __builtin_amdgcn_readlane(pre0, 63) + wave_scan(n1) - n1;
                pre0 -= n0;
            }
            load_entry(nxt, &kn, &an);
            int mn = 0x7fffffff, mx = -1;
            if (takes) {
                // lanes past the last product repeat the row's first one
                const long long at0 = base[0];
#pragma unroll
                for (int s = 0; s < R; ++s) {
                    c[s] = 0;
                    v[s] = ae[s] = (VT)0;
                    if ((s * NW + wv) * 64 < total) {      // wave-uniform
                        const int p = place_of(s), e = min(entry(s), entries - 1);
                        const long long at = p < total ? base[e] + p : at0;
                        ae[s] = av[e];
                        c[s] = bcol[at];
                        v[s] = bval[at];
                    }
                }
#pragma unroll
                for (int s = 0; s < R; ++s)
                    if ((s * NW + wv) * 64 < total) {
                        mn = min(mn, c[s]);
                        mx = max(mx, c[s]);
                    }
                mn = wave_least(mn);
                mx = wave_most(mx);
                if (lane == 0) {
                    s_min[wv] = mn;
                    s_max[wv] = mx;
                }
            }
            load_bounds(nxt, kn, &b0n, &b1n);
            __syncthreads();
            if (takes && entries <= 1) {
                // one B row (or none): its scaled copy
                if (cnt_out ? total <= expect : total == expect) {
#pragma unroll
                    for (int s = 0; s < R; ++s)
                        if (place_of(s) < total) {
                            ccol[rp + place_of(s)] = c[s];
                            cval[rp + place_of(s)] = (VT)(0.0 + to_f64(ae[s]) * to_f64(v[s]));
                        }
                    if (cnt_out && tid == 0) cnt_out[row] = total;
                } else if (cnt_out) {
                    if (tid == 0) cnt_out[row] = -1;
                } else {
                    err |= kErrCount;
                }
                done = true;
            } else if (takes) {
#pragma unroll
                for (int i = 0; i < NW; ++i) {
                    mn = min(mn, s_min[i]);
                    mx = max(mx, s_max[i]);
                }
                const int sh = max(0, 32 - __builtin_clz((unsigned)(mx - mn) | 1u) - __builtin_ctz(NB));
                // place in the bucket (16 bits: at most CAP)
                int at[R];
#pragma unroll
                for (int s = 0; s < R; ++s) {
                    at[s] = 0;
                    if ((s * NW + wv) * 64 < total) {
                        const int b = (c[s] - mn) >> sh, half = (b & 1) * 16;
                        at[s] = (int)((atomicAdd(&cw[b >> 1], place_of(s) < total ? 1u << half : 0u) >> half) & 0xffffu);
                    }
                }
                __syncthreads();
                // counts to first positions, eight words (two buckets each) a thread
                uint32_t w[8];
                int sum = 0, most = 0;
#pragma unroll
                for (int i = 0; i < 8; i += 4) {
                    const uint4 x = reinterpret_cast<const uint4*>(cw)[tid * 2 + i / 4];
                    w[i] = x.x; w[i + 1] = x.y; w[i + 2] = x.z; w[i + 3] = x.w;
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int x = (int)(w[i] & 0xffffu), y = (int)(w[i] >> 16);
                    most = max(most, max(x, y));
                    w[i] = (uint32_t)sum | (uint32_t)(sum + x) << 16;
                    sum += x + y;
                }
                const int incl = wave_scan(sum);
                most = wave_most(most);
                if (lane == 63) {
                    s_tot[wv] = incl;
                    s_most[wv] = most;
                }
                __syncthreads();
                int before = incl - sum;
#pragma unroll
                for (int i = 0; i < NW; ++i) {
                    if (i < wv) before += s_tot[i];
                    most = max(most, s_most[i]);
                }
                if (most <= kSortBucket) {                 // uniform
                    const uint32_t add = (uint32_t)before | (uint32_t)before << 16;
#pragma unroll
                    for (int i = 0; i < 8; i += 4)
                        reinterpret_cast<uint4*>(cw)[tid * 2 + i / 4] =
                            make_uint4(w[i] + add, w[i + 1] + add, w[i + 2] + add, w[i + 3] + add);
                    __syncthreads();
#pragma unroll
                    for (int s = 0; s < R; ++s)
                        if (place_of(s) < total) {
                            const int p = cs[(c[s] - mn) >> sh] + at[s];
                            sc[p] = c[s];
                            sv[p] = 0.0 + to_f64(ae[s]) * to_f64(v[s]);    // (a sum from zero: -0 becomes +0)
                        }
                    __syncthreads();
                    // in place order: rank within the bucket, then move
                    double x[R];
#pragma unroll
                    for (int s = 0; s < R; ++s) {
                        const int p = s * BS + tid;
                        at[s] = 0;
                        if (p < total) {
                            c[s] = sc[p];
                            x[s] = sv[p];
                            const int b = (c[s] - mn) >> sh;
                            const int p0 = cs[b], p1 = b + 1 < NB ? (int)cs[b + 1] : total;
                            int r = p0;
                            for (int o = p0; o < p1; ++o) {
                                const int y = sc[o];
                                r += y < c[s] || (y == c[s] && o < p);
                            }
                            at[s] = r;
                        }
                    }
                    __syncthreads();
#pragma unroll
                    for (int s = 0; s < R; ++s)
                        if (s * BS + tid < total) {
                            sc[at[s]] = c[s];
                            sv[at[s]] = x[s];
                        }
                    __syncthreads();
                    if (!cnt_out && total == expect) {     // no two products in one column
                        bool twice = false;
                        for (int j = tid; j < total; j += BS) {
                            const int x = sc[j];
                            twice = twice || (j > 0 && sc[j - 1] == x);
                            ccol[rp + j] = x;
                            cval[rp + j] = (VT)sv[j];
                        }
                        if (twice) err |= kErrCount;       // (the symbolic count was too high)
                    } else {
                        // each column's sum at its rank; a wave takes R 64-entry steps in a row
                        int heads = 0;
#pragma unroll
                        for (int s = 0; s < R; ++s) {
                            const int j = (wv * R + s) * 64 + lane;
                            heads += __builtin_popcountll(__ballot(j < total && (j == 0 || sc[j - 1] != sc[j])));
                        }
                        if (lane == 0) s_heads[wv] = heads;
                        __syncthreads();
                        int rank0 = 0, all = 0;
#pragma unroll
                        for (int i = 0; i < NW; ++i) {
                            if (i < wv) rank0 += s_heads[i];
                            all += s_heads[i];
                        }
                        const bool fits = cnt_out ? all <= expect : all == expect;
                        if (cnt_out && tid == 0) cnt_out[row] = fits ? all : -1;
                        if (!cnt_out && !fits) err |= kErrCount;
                        if (fits)
#pragma unroll
                            for (int s = 0; s < R; ++s) {
                                const int j = (wv * R + s) * 64 + lane;
                                const bool head = j < total && (j == 0 || sc[j - 1] != sc[j]);
                                const uint64_t m = __ballot(head);
                                const int rank = lanes_below(m, rank0);
                                rank0 += __builtin_popcountll(m);
                                if (head) {
                                    const int col = sc[j];
                                    double y = sv[j];
                                    for (int i = j + 1; i < total && sc[i] == col; ++i) y += sv[i];
                                    ccol[rp + rank] = col;
                                    cval[rp + rank] = (VT)y;
                                }
                            }
                    }
                    done = true;
                }
            }
            if (tid == 0) rows.close(row, done);
            if (!more) break;
            slot = next;
            cur = nxt;
            k = kn;
            a = an;
            b0 = b0n;
            b1 = b1n;
            __syncthreads();                               // the next row writes what this one still reads
        }
    }
    if (tid == 0) rows.finish();
    block_slots_done(rows.q);
    if (err) atomicOr(&info->err, err);
}

// Symbolic, one workgroup per row of at most BS R products: the products'
// columns in registers, each joins the list of its column's hash slot with one
// LDS exchange and counts unless an earlier member has its column.  An A
// entry's position in B (less its first product's number) waits in its
// members' place: 32 bits of it where the members' columns will lie and, with
// WIDE (B of 2^32 entries or more), 16 above them in their predecessors'.
// Rows of more products (their bound was B's width) are appended to fb_list for
// the bitmap kernel.  Rows above the records'
// threshold leave their outputs per window, as every symbolic workgroup
// kernel does.
//
// Bound by LDS, as k_num_sort.  On a sparse power-law matrix of 2^20 rows the
// LDS hash before took 2077 us for the rows of 2049 to 8192 products (1041
// here), 1487 for those up to 16,384 (1250) and 548 for those up to 2048
// (564); a single row of 1030 short B rows took it 49 us, walking from product
// to product (the rows above 2048 products of a power-law matrix of 171,000
// rows: 123 and 68 us before, 50 and 30 here).
template <int BS, int R, bool WIDE, bool BATCH = false>
__global__ void __launch_bounds__(BS, BS <= 256 ? 5 : 4)
k_sym_list(Work wk,
           const int64_t* __restrict__ arp, const int32_t* __restrict__ acol,
           const int64_t* __restrict__ brp, const int32_t* __restrict__ bcol,
           int32_t* __restrict__ row_nnz, DevInfo* info, RowMap mp, WinRec rec, unsigned* q,
           int32_t* __restrict__ fb_list, int* fb_count) {
    constexpr int CAP = BS * R, NW = BS / 64, WORDS = CAP / 64, H = CAP <= 2048 ? CAP : CAP / 2;
    constexpr int WL = (WORDS + 63) / 64;                // mark words a lane
    static_assert(CAP < 65536 && 64 % NW == 0, "16-bit members; a step's words lie in one lane register");
    int nrows_bin;
    const int32_t* perm;
    work_rows(wk, &nrows_bin, &perm);
    __shared__ __align__(16) int32_t head[H];
    __shared__ int32_t lc[CAP];                          // members' columns; before them the entries' positions
    __shared__ uint16_t lp[CAP];                         // the member before (kListEnd: none); before, positions' bits 32-47
    __shared__ unsigned long long mark[WORDS];
    __shared__ int s_wc[BATCH ? 1 : kWinMaxNw];
    __shared__ int s_rslot;
    __shared__ long long s_slot;
    __shared__ int s_sum[NW], s_some[NW], s_cnt[NW];
    uint32_t* const base = reinterpret_cast<uint32_t*>(lc);
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);

    struct Head {
        int row;
        long long a0, a1, bo;
    };
    auto head_of = [&](long long slot) {
        Head h;
        h.row = __builtin_amdgcn_readfirstlane(perm ? perm[slot] : (int)slot);
        h.a0 = arp[h.row];
        h.a1 = arp[h.row + 1];
        h.bo = row_boff<BATCH>(mp, h.row);
        return h;
    };
    auto load_entry = [&](const Head& h, int* k) {
        if (h.a1 > h.a0) *k = acol[h.a0 + tid < h.a1 ? h.a0 + tid : h.a1 - 1];
    };
    auto load_bounds = [&](const Head& h, int k, long long* b0, long long* b1) {
        if (h.a1 <= h.a0) return;
        *b0 = brp[k + h.bo];
        *b1 = brp[k + h.bo + 1];
    };

    long long slot = block_open(q, &s_slot);
    if (slot < nrows_bin) {                              // uniform
        Head cur = head_of(slot);
        int k = 0, kn = 0;
        long long b0 = 0, b1 = 0, b0n = 0, b1n = 0;
        load_entry(cur, &k);
        load_bounds(cur, k, &b0, &b1);
        while (true) {
            const long long na = cur.a1 - cur.a0;
            // A entries, BS at a time (the first ones were loaded ahead)
            for (int i = tid; i < WORDS; i += BS) mark[i] = 0ull;
            for (int i = tid; i < H / 4; i += BS) reinterpret_cast<int4*>(head)[i] = make_int4(-1, -1, -1, -1);
            int total = 0, entries = 0;
            for (long long e0 = 0; e0 < na && total <= CAP; e0 += BS) {     // uniform
                if (e0 > 0) {
                    if (e0 + tid < na) {
                        const long long kk = acol[cur.a0 + e0 + tid] + cur.bo;
                        b0 = brp[kk];
                        b1 = brp[kk + 1];
                    }
                    __syncthreads();                     // the wave sums before are read
                }
                int n = 0;
                if (e0 + tid < na) n = (int)(b1 - b0 < CAP + 1 ? b1 - b0 : CAP + 1);
                const int incl = wave_scan(n);
                const uint64_t some = __ballot(n > 0);
                if (lane == 63) {
                    s_sum[wv] = incl;
                    s_some[wv] = __builtin_popcountll(some);
                }
                __syncthreads();
                int first = total + incl - n, idx = entries;
#pragma unroll
                for (int i = 0; i < NW; ++i) {
                    if (i < wv) {
                        first += s_sum[i];
                        idx += s_some[i];
                    }
                    total = min(total + s_sum[i], 1 << 26);
                    entries += s_some[i];
                }
                if (n > 0 && first + n <= CAP) {         // (then fewer than CAP entries lie before)
                    idx = lanes_below(some, idx);
                    const long long at = b0 - first;
                    base[idx] = (uint32_t)at;
                    if constexpr (WIDE) lp[idx] = (uint16_t)(at >> 32);
                    const int last = first + n - 1;
                    atomicOr(reinterpret_cast<uint32_t*>(mark) + (last >> 5), 1u << (last & 31));
                }
            }
            const bool takes = total <= CAP;             // uniform
            block_draw(q, slot, &s_slot);
            __syncthreads();
            const long long next = s_slot;
            const bool more = next < nrows_bin;          // uniform
            const Head nxt = head_of(more ? next : slot);
            load_entry(nxt, &kn);
            int c[R];
            if (takes) {
                // lane i of every wave: mark words i, 64 + i, ..., and the marks before them
                int lo[WL], hi[WL], pre[WL], sum = 0;
#pragma unroll
                for (int j = 0; j < WL; ++j) {
                    const unsigned long long w = 64 * j + lane < WORDS ? mark[64 * j + lane] : 0ull;
                    lo[j] = (int)(uint32_t)w;
                    hi[j] = (int)(uint32_t)(w >> 32);
                    const int m = __builtin_popcountll(w), incl = wave_scan(m);
                    pre[j] = sum + incl - m;
                    sum += __builtin_amdgcn_readlane(incl, 63);
                }
#pragma unroll
                for (int s = 0; s < R; ++s) {
                    c[s] = 0;
                    if ((s * NW + wv) * 64 < total) {    // wave-uniform
                        const int p = (s * NW + wv) * 64 + lane, i = (s * NW & 63) + wv, j = s * NW / 64;
                        const int e = lanes_below((uint32_t)__builtin_amdgcn_readlane(lo[j], i),
                                                  (uint32_t)__builtin_amdgcn_readlane(hi[j], i),
                                                  __builtin_amdgcn_readlane(pre[j], i));
                        // lanes past the last product read it again
                        const int i0 = min(e, entries - 1);
                        if constexpr (WIDE)
                            c[s] = bcol[list_position(base[i0], lp[i0], min(p, total - 1))];
                        else
                            c[s] = bcol[base[i0] + (uint32_t)min(p, total - 1)];
                    }
                }
            }
            load_bounds(nxt, kn, &b0n, &b1n);
            __syncthreads();                             // the entries' positions are read
            if (takes) {
                int prev[R];
#pragma unroll
                for (int s = 0; s < R; ++s) {
                    const int p = (s * NW + wv) * 64 + lane;
                    prev[s] = -1;
                    if (p < total) {
                        prev[s] = atomicExch(&head[hash_slot<H>(c[s])], p);
                        lc[p] = c[s];
                        lp[p] = (uint16_t)prev[s];
                    }
                }
                __syncthreads();
                uint32_t own = 0;                        // steps whose product counts
#pragma unroll
                for (int g = 0; g < R; g += 4) {
                    // four products a lane at once, back through the lists
                    int live = 0;
                    uint32_t four = 0;
#pragma unroll
                    for (int s = g; s < g + 4; ++s) {
                        four |= (uint32_t)((s * NW + wv) * 64 + lane < total) << (s - g);
                        live |= (prev[s] >= 0) << (s - g);
                    }
                    while (__ballot(live != 0))
                        list_step<4>(c + g, prev + g, live, four, [&](int m) { return lc[m]; },
                                     [&](int m) { return (int)lp[m]; });
                    own |= four << g;
                }
                const int cnt = __builtin_amdgcn_readlane(wave_scan(__builtin_popcount(own)), 63);
                if (lane == 0) s_cnt[wv] = cnt;
                __syncthreads();
                int tot = 0;
#pragma unroll
                for (int i = 0; i < NW; ++i) tot += s_cnt[i];
                if (tid == 0) row_nnz[cur.row] = tot;
                if constexpr (!BATCH) {
                    if (win_record_open((int*)rec.cnt, rec.nw, rec.thresh, rec.nrec, tot, s_wc, &s_rslot)) {
#pragma unroll
                        for (int s = 0; s < R; ++s)
                            if ((own >> s) & 1u) atomicAdd(&s_wc[c[s] >> kWinLog], 1);
                        win_record_close(rec, cur.row, s_wc, &s_rslot);
                    }
                }
            } else if (tid == 0) {
                fb_list[atomicAdd(fb_count, 1)] = cur.row;
            }
            if (!more) break;
            slot = next;
            cur = nxt;
            k = kn;
            b0 = b0n;
            b1 = b1n;
            __syncthreads();                             // the next row writes what this one still reads
        }
    }
    block_slots_done(q);
    (void)info;
}

}  // namespace msp

// Whole-wave row kernels: one wave per row, the row's products in registers.
//
// A wave takes a row of at most 64 A entries and at most 64 R products.  Lane
// e holds A entry e; the nonempty entries' B positions and values go to LDS
// in order, and a bit mask marks the last product of each entry.  Step s of
// the walk gives product q = 64 s + lane to a lane, and the product's entry
// is the number of marks before q: the count in the words before word s plus
// the marks below the lane in word s (two mbcnt instructions on a word that
// every lane of the wave shares).  So every lane has a product whatever the
// B rows' lengths, with no search, and all loads of a row are independent:
// they are in flight together.
#pragma once

namespace msp {

// The walk over a row's products (see the head of this file).  `mark` is an
// LDS array of R 64-bit words; base[i] and, with values, av[i] are LDS arrays
// of 65 entries for the i-th nonempty A entry: the B position of product q of
// that entry is base[i] + q.
template <int R>
struct RowWalk {
    int total;                  // products of the row; above 64 R: not walked
    int lo, hi, pre;            // lane s: word s of the marks and the marks before it

    // lane e's entry: B rows' position bst and length len (0 past the row's entries)
    __device__ __forceinline__ void open(int lane, long long bst, long long len, unsigned long long* mark,
                                         long long* base, double* av, double a) {
        const int n = (int)(len < 64 * R + 1 ? len : 64 * R + 1);      // (the sum stays in 32 bits)
        const int incl = wave_scan(n);
        total = __builtin_amdgcn_readlane(incl, 63);
        if (total > 64 * R) return;
        if (lane < R) mark[lane] = 0ull;
        const uint64_t some = __ballot(n > 0);
        lds_fence();
        if (n > 0) {
            const int i = lanes_below(some, 0);
            base[i] = bst - (incl - n);
            if (av) av[i] = a;
            atomicOr(reinterpret_cast<uint32_t*>(mark) + ((incl - 1) >> 5), 1u << ((incl - 1) & 31));
        }
        lds_fence();
        const unsigned long long w = lane < R ? mark[lane] : 0ull;
        lo = (int)(uint32_t)w;
        hi = (int)(uint32_t)(w >> 32);
        const int c = __builtin_popcountll(w);
        pre = wave_scan(c) - c;
    }
    // Forget what was computed from the words: entry() is cheaper than the
    // registers that would keep every step's answer.
    __device__ __forceinline__ void again() { asm volatile("" : "+v"(lo), "+v"(hi), "+v"(pre)); }
    // the entry of product 64 s + lane (s a constant; meaningless past the total)
    __device__ __forceinline__ int entry(int s) const {
        return lanes_below((uint32_t)__builtin_amdgcn_readlane(lo, s), (uint32_t)__builtin_amdgcn_readlane(hi, s),
                           __builtin_amdgcn_readlane(pre, s));
    }
};

// A row by a whole wave through an LDS hash of T (column, FP64) slots, for
// rows that the register paths of k_num_row do not take.  The occupied slots
// are compacted and each output's position is its rank among the row's
// columns: from a bitmap of the span when it is under 32 T, else through 64
// buckets of equal column width while none holds more than kBucketMax keys
// (rows of at least 64 outputs), by a sort across the wave past 160 outputs,
// or counted with 16-byte LDS reads.  Returns error bits.
constexpr int kBucketMax = 24;
template <int T, typename VT>
__device__ __forceinline__ int row_hash(
    long long a0, long long a1, long long bo, int expect, long long rp, int row, const int32_t* __restrict__ acol,
    const VT* __restrict__ aval, const int64_t* __restrict__ brp, const int32_t* __restrict__ bcol,
    const VT* __restrict__ bval, int32_t* __restrict__ ccol, VT* __restrict__ cval, int32_t* __restrict__ cnt_out,
    int32_t* kt, double* vt, long long* s_off, long long* s_bst, double* s_a) {
    const int lane = threadIdx.x & 63;
    int re = 0;                                  // the table or the room overflowed
    int ncol = 0;                                // columns that this lane saw added
#pragma unroll
    for (int i = 0; i < T / 64; ++i) { kt[lane + i * 64] = kEmpty; vt[lane + i * 64] = 0.0; }
    lds_fence();
    for (long long c0 = a0; c0 < a1; c0 += 64) {
        const long long p = c0 + lane;
        long long len = 0, bst = 0;
        double a = 0.0;
        if (p < a1) {
            const long long k = acol[p] + bo;
            a = to_f64(aval[p]);
            bst = brp[k];
            len = brp[k + 1] - bst;
        }
        const long long incl = group_incl_scan<64>(len, lane);
        const long long total = __shfl(incl, 63);
        s_off[lane] = incl;
        s_bst[lane] = bst - (incl - len);
        s_a[lane] = a;
        lds_fence();
        const int nact = (int)((a1 - c0) < 64 ? (a1 - c0) : 64);
        int t = -1;                              // owner of q: one search, then it only moves forward
        for (long long q = lane; q < total; q += 64) {
            if (t < 0) t = owner_search(s_off, nact, q);
            else while (s_off[t] <= q) ++t;
            const long long bi = s_bst[t] + q;
            const int32_t j = bcol[bi];
            const double prod = s_a[t] * to_f64(bval[bi]);
            // A full table ends the row (every further column would be looked for
            // in all of it), and so do more columns than the room, which is only
            // looked at where registers allow it.
            if constexpr (T > 512) {
                bool fresh = false;
                const int h = hash_slot_of<T>(kt, j, &re, &fresh);
                if (h >= 0) atomicAdd(&vt[h], prod);
                ncol += __builtin_popcountll(__ballot(fresh));
                if ((cnt_out && ncol > expect) || __ballot(h < 0)) { re = 1; break; }
            } else {
                const int h = hash_slot_of<T>(kt, j, &re);
                if (h >= 0) atomicAdd(&vt[h], prod);
                if (__ballot(h < 0)) break;
            }
        }
        lds_fence();
        if (__ballot(re != 0)) break;
    }
    // compact the occupied slots to the front, in place: a slot moves to a
    // position no later than its own, and the wave reads its 64 slots before
    // any of them is written
    int n = 0;
#pragma unroll
    for (int s0 = 0; s0 < T; s0 += 64) {
        const int s = s0 + lane;
        const int32_t k = kt[s];
        const double v = vt[s];
        const bool occ = k != kEmpty;
        const uint64_t mask = __ballot(occ);
        if (occ) {
            const int pos = lanes_below(mask, n);
            kt[pos] = k;
            vt[pos] = v;
        }
        n += __builtin_popcountll(mask);
    }
    const bool failed = __ballot(re != 0) != 0;
    if (cnt_out) {                               // capacity mode
        const bool fits = !failed && n <= expect && n <= T / 2;
        if (lane == 0) cnt_out[row] = fits ? n : -1;
        if (!fits) { lds_fence(); return 0; }
    } else if (failed || n != expect || n > T / 2) {
        lds_fence();
        return failed ? kErrProbe : kErrCount;
    }
    {
        // rows whose columns span less than 32 T: column order from a
        // bitmap of the span (the free upper half of the value table, T / 2
        // words) and a rank per word (the free upper half of the key
        // table), O(n / 64 + T / 128) steps a lane instead of a sort
        int kmn = 0x7fffffff, kmx = -1;
        for (int e = lane; e < n; e += 64) {
            kmn = min(kmn, kt[e]);
            kmx = max(kmx, kt[e]);
        }
        kmn = wave_least(kmn);
        kmx = wave_most(kmx);
        if (n > 0 && (long long)kmx - kmn < 32LL * T) {       // wave-uniform
            unsigned long long* bm = reinterpret_cast<unsigned long long*>(vt + T / 2);
            int* wr = kt + T / 2;
            const int nwd = ((kmx - kmn) >> 6) + 1;            // <= T / 2
            for (int i = lane; i < nwd; i += 64) bm[i] = 0ull;
            lds_fence();
            for (int e = lane; e < n; e += 64) {
                const int d = kt[e] - kmn;
                atomicOr(&bm[d >> 6], 1ull << (d & 63));
            }
            lds_fence();
            // lane l ranks the E consecutive words from l E
            const int E = (nwd + 63) >> 6;
            const int i0 = lane * E, i1 = min(i0 + E, nwd);
            int loc = 0;
            for (int i = i0; i < i1; ++i) loc += __builtin_popcountll(bm[i]);
            int run = wave_scan(loc) - loc;
            for (int i = i0; i < i1; ++i) {
                wr[i] = run;
                run += __builtin_popcountll(bm[i]);
            }
            lds_fence();
            for (int e = lane; e < n; e += 64) {
                const int32_t k = kt[e];
                const int d = k - kmn;
                const int rank = wr[d >> 6] + __builtin_popcountll(bm[d >> 6] & ((1ull << (d & 63)) - 1ull));
                ccol[rp + rank] = k;
                cval[rp + rank] = (VT)vt[e];
            }
            lds_fence();
            return 0;
        }
        // (the counters and slots below need T >= 256)
        if (T >= 256 && n >= 64) {                            // wave-uniform
            // wider rows: the keys counted into 64 buckets of equal column
            // width, placed bucket by bucket, and each ranked by comparison
            // within its bucket; taken while no bucket holds more than
            // kBucketMax keys (else the sort or the rank count below)
            int* cnt = reinterpret_cast<int*>(vt + T / 2);    // the free upper half
            int* cur = cnt + 64;
            int* sidx = cur + 64;                             // n <= T / 2 entries
            int32_t* skey = kt + T / 2;                       // n <= T / 2 entries
            const float scale = 64.0f / (float)((long long)kmx - kmn + 1);
            auto bucket = [&](int32_t k) { return min(63, (int)((float)(k - kmn) * scale)); };
            cnt[lane] = 0;
            lds_fence();
            for (int e = lane; e < n; e += 64) atomicAdd(&cnt[bucket(kt[e])], 1);
            lds_fence();
            const int c = cnt[lane];
            const int cmax = wave_most(c);
            if (cmax <= kBucketMax) {                         // wave-uniform
                cur[lane] = wave_scan(c) - c;
                lds_fence();
                for (int e = lane; e < n; e += 64) {
                    const int32_t k = kt[e];
                    const int slot = atomicAdd(&cur[bucket(k)], 1);
                    skey[slot] = k;
                    sidx[slot] = e;
                }
                lds_fence();
                // cur[b] is now the end of bucket b
                for (int sl = lane; sl < n; sl += 64) {
                    const int32_t k = skey[sl];
                    const int b = bucket(k);
                    const int b1 = cur[b], b0 = b1 - cnt[b];
                    int rank = b0;
                    for (int j = b0; j < b1; ++j) rank += skey[j] < k;
                    ccol[rp + rank] = k;
                    cval[rp + rank] = (VT)vt[sidx[sl]];
                }
                lds_fence();
                return 0;
            }
        }
    }
    if constexpr (T / 2 > 128) {
        // long rows: a bitonic sort across the wave (the rank count below
        // costs n / 4 LDS reads and n compares per output, n / 64 outputs a
        // lane; the sort of T / 2 elements costs less from about 160 on)
        if (n > 160) {                                  // wave-uniform (a row per wave)
            lds_fence();
            wave_sort_out<T / 128>(kt, vt, n, ccol + rp, cval + rp, lane);
            lds_fence();
            return 0;
        }
    }
    const int n4 = (n + 3) & ~3;
    if (lane < n4 - n) kt[n + lane] = 0x7fffffff;         // pads sort after every key
    lds_fence();
    for (int e = lane; e < n; e += 64) {
        const int32_t k = kt[e];
        int rank = 0;
        for (int f = 0; f < n4; f += 4) {
            const int4 q = *reinterpret_cast<const int4*>(&kt[f]);
            rank += (q.x < k) + (q.y < k) + (q.z < k) + (q.w < k);
        }
        ccol[rp + rank] = k;
        cval[rp + rank] = (VT)vt[e];
    }
    return 0;
}

// Products a lane of the row kernels holds, and the most columns a row's
// products may span for the bitmap paths (32 columns a word, 4 + 2 LDS bytes
// a word with the words' ranks).  43008 columns cover the 27-point rows of a
// 101^3 grid (41,212).
constexpr int kRowR = 12;
constexpr int kRowWords = 1344;
constexpr int kRowStep = 4;

// Numeric, one wave per row of at most T / 2 outputs.
//
// Rows of at most 64 A entries and 64 kRowR products:
//   narrow (products' columns within 32 kRowWords): a bitmap of the span, the
//     words' ranks, then every product adds into the FP64 sum at its column's
//     rank.  Column offset and rank share a register, so the sums take the
//     bitmap's place.
//   wide (at most P products): counting sort.  The span is cut into NB
//     buckets of equal width (a power of two); an LDS atomic counts the
//     buckets and gives each product its place in its bucket, the counts are
//     scanned, the columns placed, and each product counts its bucket's
//     smaller columns (equal ones by place).  Sums over equal columns, now
//     neighbours, go out in order.  While no bucket holds more than
//     kRowBucket products.
// Other rows: an LDS hash of T (column, FP64) slots, compacted, then ordered
// by a bitmap of the span, by buckets, by a sort across the wave or by
// counting.
//
// What bounds it: instruction issue and LDS (a hash probe loop runs as long as
// its unluckiest lane, and finding a product's entry by search cost more than
// the product), so both went; HBM is at 15-20%.  One wave a workgroup, so that
// LDS is handed out a row at a time: 16 waves a compute unit up to T = 512.
// Measured against the hash kernels it replaced: 300,763 27-point rows (FP64,
// 729 products, 125 outputs) 1311 -> 588 us; 260,000 banded rows (FP32, 256
// products) 735 -> 303 us; the 257- to 512-output rows of a uniform FP64
// matrix of 262,144 rows 2820 -> 523 us (a workgroup a row before; 475 without
// the count of distinct columns where there are as many outputs as products).  At three
// waves a SIMD without spills the FP64 kernel up to T = 512 is no faster (657
// us on the 27-point rows at two, 670 at three, 617 at four); T = 1024, where
// LDS leaves 11 waves a compute unit, takes 475 us at two and 620 at three
// with spills.  Two steps between checks instead of four: 1-5% slower.
//
// Rows of 257 outputs and more that have past kRowMost products go to a workgroup:
// a wave hashes 60,000 rows of 6400 products onto 390 outputs in 2147 us, of
// 25,600 onto 440 in 7480, a workgroup of 256 threads in 2199 and 4616.
constexpr int kRowBucket = 24;
constexpr int kRowMost = 8192;
template <int T>
struct RowCfg {
    static constexpr int P = T <= 512 ? 512 : 768;            // most products of a wide row
    static constexpr int NB = T <= 512 ? 1024 : 2048;         // buckets (16-bit counters)
    static constexpr int kWide = (P + 2) * 12 + NB * 2;      // (a spare entry for lanes past the last product)
    static constexpr int kNarrow = kRowWords * 6 > T / 2 * 12 ? kRowWords * 6 : T / 2 * 12;
    static constexpr int kHash = (T + 4) * 4 + (T + 1) * 8;
    static constexpr int a0 = kWide > kNarrow ? kWide : kNarrow;
    static constexpr int kArea = ((a0 > kHash ? a0 : kHash) + 15) & ~15;
};

template <int T, typename VT, bool BATCH = false>
__global__ void __launch_bounds__(64, T <= 512 ? 4 : 2)
k_num_row(Work wk,
          const int64_t* __restrict__ arp, const int32_t* __restrict__ acol, const VT* __restrict__ aval,
          const int64_t* __restrict__ brp, const int32_t* __restrict__ bcol, const VT* __restrict__ bval,
          const int64_t* __restrict__ crp, int32_t* __restrict__ ccol, VT* __restrict__ cval,
          int32_t* __restrict__ cnt_out, DevInfo* info, RowMap mp, int32_t* left_of, int* left) {
    using Cfg = RowCfg<T>;
    constexpr int R = kRowR, OUT = T / 2;
    constexpr bool LEAVES = T > 512;                // rows past kRowMost products: left (see k_num_block)
    int nleft = 0;
    constexpr int GS = kRowStep;                    // steps between checks of the row's length
    static_assert(Cfg::P <= 64 * R, "a wide row's products are in registers");
    int nrows_bin;
    const int32_t* perm;
    work_rows(wk, &nrows_bin, &perm);
    __shared__ long long s_off[65];                 // hash path: offsets; else the walk's marks
    __shared__ long long s_bst[65];
    __shared__ double s_a[65];
    __shared__ __align__(16) unsigned char area[Cfg::kArea];
    static_assert(R <= 65, "the marks take the offsets' place");
    const int lane = threadIdx.x;
    int err = 0;
    const long long per = (nrows_bin + gridDim.x - 1) / gridDim.x;
    const long long first = (long long)xcd_block() * per;
    const long long last = first + per < nrows_bin ? first + per : nrows_bin;
    if (first >= last) return;

    // The next row's head is loaded at the start of a row, its A entries
    // before the row's products and its B bounds behind them; the values are
    // not touched before the next row starts, so nothing waits for them.
    // Lanes past a row's entries repeat its last one.
    struct Head {
        int row, expect;
        long long a0, a1, rp, bo;
    };
    int listed = 0;                                 // 64 slots of the list, one a lane
    auto head_of = [&](long long slot) {
        Head h;
        h.row = (int)slot;
        if (perm) {
            const int i = (int)(slot - first) & 63;
            if (i == 0) listed = perm[slot + lane < last ? slot + lane : last - 1];
            h.row = __builtin_amdgcn_readlane(listed, i);
        }
        h.a0 = arp[h.row];
        h.a1 = arp[h.row + 1];
        h.rp = crp[h.row];
        h.expect = (int)(crp[h.row + 1] - h.rp);
        h.bo = row_boff<BATCH>(mp, h.row);
        return h;
    };
    auto load_entry = [&](const Head& h, int* k, VT* a) {
        if (h.a1 <= h.a0) return;                   // wave-uniform
        const long long p = h.a0 + lane < h.a1 ? h.a0 + lane : h.a1 - 1;
        *k = acol[p];
        *a = aval[p];
    };
    auto load_bounds = [&](const Head& h, int k, long long* b0, long long* b1) {
        if (h.a1 <= h.a0) return;
        *b0 = brp[k + h.bo];
        *b1 = brp[k + h.bo + 1];
    };
    Head cur = head_of(first);
    int k = 0, kn = 0;
    VT a = (VT)0, an = (VT)0;
    long long b0 = 0, b1 = 0, b0n = 0, b1n = 0;
    load_entry(cur, &k, &a);
    load_bounds(cur, k, &b0, &b1);
    for (long long slot = first; slot < last; ++slot) {
        const Head nxt = head_of(slot + 1 < last ? slot + 1 : slot);
        const int row = cur.row, expect = cur.expect;
        const long long rp = cur.rp;
        bool done = false;
        RowWalk<R> walk;
        walk.total = 64 * R + 1;
        if (cur.a1 - cur.a0 <= 64)
            walk.open(lane, b0, cur.a0 + lane < cur.a1 ? b1 - b0 : 0, reinterpret_cast<unsigned long long*>(s_off),
                      s_bst, s_a, to_f64(a));
        const int total = walk.total;
        load_entry(nxt, &kn, &an);
        if (total <= 64 * R) {                      // wave-uniform
            // Every product's column and value.  Lanes past the last product
            // repeat the row's first one, which the minimum, the bitmap and
            // the output columns may take twice.
            int c[R];
            VT v[R];
            const long long at0 = s_bst[0];
#pragma unroll
            for (int g = 0; g < R; g += GS)
                if (64 * g < total) {
                    long long at[GS];
#pragma unroll
                    for (int s = g; s < g + GS; ++s) at[s - g] = s_bst[walk.entry(s)] + (64 * s + lane);
#pragma unroll
                    for (int s = g; s < g + GS; ++s) {
                        const long long p = 64 * s + lane < total ? at[s - g] : at0;
                        c[s] = bcol[p];
                        v[s] = bval[p];
                    }
                }
            walk.again();
            int mn = 0x7fffffff, mx = -1;
#pragma unroll
            for (int g = 0; g < R; g += GS)
                if (64 * g < total) {
#pragma unroll
                    for (int s = g; s < g + GS; ++s) {
                        mn = min(mn, c[s]);
                        mx = max(mx, c[s]);
                    }
                }
            load_bounds(nxt, kn, &b0n, &b1n);
            mn = wave_least(mn);
            mx = wave_most(mx);
            const int span = total > 0 ? mx - mn : 0;
            if (span < 32 * kRowWords) {
                // narrow: bitmap of the span and the words' ranks
                uint32_t* const bm = reinterpret_cast<uint32_t*>(area);
                uint16_t* const wr = reinterpret_cast<uint16_t*>(area + kRowWords * 4);
                const int nwd = total > 0 ? (span >> 5) + 1 : 0;
                for (int i = lane * 4; i < nwd; i += 256) *reinterpret_cast<uint4*>(bm + i) = make_uint4(0, 0, 0, 0);
                lds_fence();
#pragma unroll
                for (int g = 0; g < R; g += GS)
                    if (64 * g < total) {
#pragma unroll
                        for (int s = g; s < g + GS; ++s) {
                            c[s] -= mn;
                            atomicOr(&bm[c[s] >> 5], 1u << (c[s] & 31));
                        }
                    }
                lds_fence();
                // lane l ranks the E words from l E (E odd: the lanes' words spread over the banks)
                const int E = ((nwd + 63) >> 6) | 1;
                const int i0 = min(lane * E, nwd), i1 = min(i0 + E, nwd);
                int loc = 0;
                for (int i = i0; i < i1; ++i) loc += __builtin_popcount(bm[i]);
                const int incl = wave_scan(loc);
                int run = incl - loc;
                const int n = __builtin_amdgcn_readlane(incl, 63);
                for (int i = i0; i < i1; ++i) {
                    wr[i] = (uint16_t)run;
                    run += __builtin_popcount(bm[i]);
                }
                const bool fits = n <= expect && n <= OUT;
                if (cnt_out) {
                    if (lane == 0) cnt_out[row] = fits ? n : -1;
                } else if (n != expect || !fits) {
                    err |= kErrCount;
                }
                if (fits) {
                    lds_fence();
#pragma unroll
                    for (int g = 0; g < R; g += GS)
                        if (64 * g < total) {
                            int x[GS];
                            uint32_t y[GS];
#pragma unroll
                            for (int s = g; s < g + GS; ++s) {
                                x[s - g] = wr[c[s] >> 5];
                                y[s - g] = bm[c[s] >> 5];
                            }
#pragma unroll
                            for (int s = g; s < g + GS; ++s) {        // column offset (below 2^16) and rank
                                const int rk = x[s - g] + __builtin_popcount(y[s - g] & ((1u << (c[s] & 31)) - 1u));
                                c[s] |= rk << 16;
                            }
                        }
                    lds_fence();
                    walk.again();
                    double* const acc = reinterpret_cast<double*>(area);
                    int32_t* const oc = reinterpret_cast<int32_t*>(area + OUT * 8);
                    const bool apart = total == n;                    // no two products in one column
                    if (!apart) {
                        for (int i = lane; i < n; i += 64) acc[i] = 0.0;
                        lds_fence();
                    }
#pragma unroll
                    for (int g = 0; g < R; g += GS)
                        if (64 * g < total) {
                            double x[GS];
#pragma unroll
                            for (int s = g; s < g + GS; ++s) x[s - g] = s_a[walk.entry(s)];
#pragma unroll
                            for (int s = g; s < g + GS; ++s) {
                                const int rk = c[s] >> 16;
                                oc[rk] = c[s] & 0xffff;
                                const double y = x[s - g] * to_f64(v[s]);
                                if (64 * s + lane < total) {
                                    if (apart) acc[rk] = 0.0 + y;     // (a sum from zero: -0 becomes +0)
                                    else atomicAdd(&acc[rk], y);
                                }
                            }
                        }
                    lds_fence();
                    for (int i = lane; i < n; i += 64) {
                        ccol[rp + i] = oc[i] + mn;
                        cval[rp + i] = (VT)acc[i];
                    }
                }
                lds_fence();
                done = true;
            } else if (total <= Cfg::P) {
                // wide: counting sort by buckets of 2^sh columns
                constexpr int RP = Cfg::P / 64, NB = Cfg::NB, PER = NB / 128;      // counter words a lane scans
                static_assert(RP % GS == 0 && NB % 512 == 0, "whole steps, 16-byte clears");
                uint32_t* const cw = reinterpret_cast<uint32_t*>(area);
                uint16_t* const cs = reinterpret_cast<uint16_t*>(area);
                int32_t* const sc = reinterpret_cast<int32_t*>(area + NB * 2);     // entry P: lanes past the last product
                double* const sv = reinterpret_cast<double*>(area + NB * 2 + (Cfg::P + 2) * 4);
                const int sh = max(0, 32 - __builtin_clz((unsigned)span) - __builtin_ctz(NB));
#pragma unroll
                for (int i = 0; i < NB / 512; ++i) reinterpret_cast<uint4*>(area)[64 * i + lane] = make_uint4(0, 0, 0, 0);
                lds_fence();
                // the bucket and, from bit 24, the place within it; later the
                // bucket's first position, its size (from bit 16) and the place
                int bk[RP];
#pragma unroll
                for (int g = 0; g < RP; g += GS)
                    if (64 * g < total) {
                        uint32_t x[GS];
#pragma unroll
                        for (int s = g; s < g + GS; ++s) {
                            bk[s] = (c[s] - mn) >> sh;
                            x[s - g] = atomicAdd(&cw[bk[s] >> 1],
                                                 64 * s + lane < total ? 1u << ((bk[s] & 1) * 16) : 0u);
                        }
#pragma unroll
                        for (int s = g; s < g + GS; ++s)              // (a place past 255: the bucket is too full)
                            bk[s] |= (int)((x[s - g] >> ((bk[s] & 1) * 16)) << 24);
                    }
                lds_fence();
                // counts to first positions, PER words (two buckets each) a lane
                uint32_t w[PER];
                int sum = 0, most = 0;
#pragma unroll
                for (int i = 0; i < PER; i += 4) {
                    const uint4 x = reinterpret_cast<const uint4*>(cw)[(lane * PER + i) / 4];
                    w[i] = x.x; w[i + 1] = x.y; w[i + 2] = x.z; w[i + 3] = x.w;
                }
#pragma unroll
                for (int i = 0; i < PER; ++i) {
                    const int x = (int)(w[i] & 0xffffu), y = (int)(w[i] >> 16);
                    most = max(most, max(x, y));
                    w[i] = (uint32_t)sum | (uint32_t)(sum + x) << 16;
                    sum += x + y;
                }
                most = wave_most(most);
                if (most <= kRowBucket) {
                    const uint32_t before = (uint32_t)(wave_scan(sum) - sum);
                    const uint32_t add = before | before << 16;
#pragma unroll
                    for (int i = 0; i < PER; i += 4)
                        reinterpret_cast<uint4*>(cw)[(lane * PER + i) / 4] =
                            make_uint4(w[i] + add, w[i + 1] + add, w[i + 2] + add, w[i + 3] + add);
                    lds_fence();
#pragma unroll
                    for (int g = 0; g < RP; g += GS)
                        if (64 * g < total) {
                            int x[GS], y[GS];
#pragma unroll
                            for (int s = g; s < g + GS; ++s) {
                                const int b = bk[s] & 0xffff;
                                x[s - g] = cs[b];
                                y[s - g] = cs[b + 1 < NB ? b + 1 : b];
                            }
#pragma unroll
                            for (int s = g; s < g + GS; ++s) {
                                const int place = (int)((unsigned)bk[s] >> 24), p0 = x[s - g];
                                const int p1 = (bk[s] & 0xffff) + 1 < NB ? y[s - g] : total;
                                const bool in = 64 * s + lane < total;
                                sc[in ? p0 + place : Cfg::P] = c[s];
                                bk[s] = p0 | (p1 - p0) << 16 | place << 24;
                            }
                        }
                    lds_fence();
                    // the smaller columns of the bucket (equal ones by place)
                    int pos[RP];
#pragma unroll
                    for (int s = 0; s < RP; ++s) pos[s] = 0;
                    for (int o = 0; o < most; ++o) {                  // wave-uniform
#pragma unroll
                        for (int g = 0; g < RP; g += GS)
                            if (64 * g < total) {
                                int x[GS];
#pragma unroll
                                for (int s = g; s < g + GS; ++s)
                                    x[s - g] = sc[(bk[s] & 0xffff) + min(o, ((bk[s] >> 16) & 0xff) - 1)];
#pragma unroll
                                for (int s = g; s < g + GS; ++s)
                                    pos[s] += o < ((bk[s] >> 16) & 0xff) &&
                                              (x[s - g] < c[s] || (x[s - g] == c[s] && o < (bk[s] >> 24)));
                            }
                    }
                    lds_fence();
                    walk.again();
#pragma unroll
                    for (int g = 0; g < RP; g += GS)
                        if (64 * g < total) {
                            double x[GS];
#pragma unroll
                            for (int s = g; s < g + GS; ++s) x[s - g] = s_a[walk.entry(s)];
#pragma unroll
                            for (int s = g; s < g + GS; ++s) {
                                const int q = 64 * s + lane < total ? (bk[s] & 0xffff) + pos[s] : Cfg::P;
                                sc[q] = c[s];
                                sv[q] = 0.0 + x[s - g] * to_f64(v[s]);        // (a sum from zero: -0 becomes +0)
                            }
                        }
                    lds_fence();
                    int n = 0;
                    if (T <= 512 && !cnt_out && total == expect) {    // no two products in one column
                        n = total;
                        for (int j = lane; j < total; j += 64) {
                            ccol[rp + j] = sc[j];
                            cval[rp + j] = (VT)sv[j];
                        }
                    } else {
                        // each column's sum at its rank
                        for (int j0 = 0; j0 < total; j0 += 64) {
                            const int j = j0 + lane;
                            int x = -1;
                            bool head = false;
                            if (j < total) {
                                x = sc[j];
                                head = j == 0 || sc[j - 1] != x;
                            }
                            const uint64_t heads = __ballot(head);
                            const int rank = lanes_below(heads, n);
                            n += __builtin_popcountll(heads);
                            if (head && rank < expect) {
                                double y = sv[j];
                                for (int i = j + 1; i < total && sc[i] == x; ++i) y += sv[i];
                                ccol[rp + rank] = x;
                                cval[rp + rank] = (VT)y;
                            }
                        }
                    }
                    if (cnt_out) {
                        if (lane == 0) cnt_out[row] = n <= expect ? n : -1;
                    } else if (n != expect) {
                        err |= kErrCount;
                    }
                    done = true;
                }
                lds_fence();
            }
        } else {
            load_bounds(nxt, kn, &b0n, &b1n);
        }
        if constexpr (LEAVES) {
            bool heavy = false;                     // wave-uniform
            if (!done) {
                int n = cur.a0 + lane < cur.a1 ? (int)min(b1 - b0, kRowMost + 1ll) : 0;
                n = __builtin_amdgcn_readlane(wave_scan(n), 63);
                for (long long p = cur.a0 + 64; p < cur.a1 && n <= kRowMost; p += 64) {
                    int x = 0;
                    if (p + lane < cur.a1) {
                        const long long kk = acol[p + lane] + cur.bo;
                        x = (int)min((long long)(brp[kk + 1] - brp[kk]), kRowMost + 1ll);
                    }
                    n += __builtin_amdgcn_readlane(wave_scan(x), 63);
                }
                heavy = n > kRowMost;
            }
            if (lane == 0) left_of[row] = heavy;
            nleft += heavy;
            done = done || heavy;
        }
        if (!done)
            err |= row_hash<T, VT>(cur.a0, cur.a1, cur.bo, expect, rp, row, acol, aval, brp, bcol, bval, ccol, cval,
                                   cnt_out, reinterpret_cast<int32_t*>(area),
                                   reinterpret_cast<double*>(area + (T + 4) * 4), s_off, s_bst, s_a);
        cur = nxt;
        k = kn;
        a = an;
        b0 = b0n;
        b1 = b1n;
    }
    if (LEAVES && lane == 0 && nleft > 0) atomicAdd(left, nleft);
    if (err) atomicOr(&info->err, err);
}

// Symbolic, one wave per row of at most T / 2 products (or columns of B).
//
// Rows of at most 64 A entries and T / 2 products: the products' columns in
// registers; within 32 kRowWords columns their bits are counted in a bitmap
// of the span, else every product joins the list of its column's hash slot
// (one LDS exchange) and counts unless an earlier member has its column.
// Other rows: a bitmap of the span, products taken as they come, when they have at most 64 A entries and the span is narrow; else an LDS hash of T
// keys.  (With the hash for both, 60,000 rows of 2500 products over 950 columns
// took 558 us, 405 in the kernel before, which had the bitmap.)
//
// Bound by LDS and instruction issue, as k_num_row.  The lists need one
// returning LDS operation a product and then only reads, where a hash of
// compare-and-swaps repeats the slow operation on every collision of the
// wave's unluckiest lane: the 257- to 512-product rows of a uniform matrix of
// 262,144 rows take 134 us (compare-and-swap four keys a lane at once 573, the
// kernel before, read first, 326), the 513- to 1024-product ones 78 (148
// before), the 129- to 256-product ones 62 (103 before).  Bitmap rows: 260,000
// banded rows 208 -> 142 us, 300,763 27-point rows 626 -> 331 us.
template <int T, bool BATCH = false>
__global__ void __launch_bounds__(64, 4)
k_sym_row(Work wk,
          const int64_t* __restrict__ arp, const int32_t* __restrict__ acol,
          const int64_t* __restrict__ brp, const int32_t* __restrict__ bcol,
          int32_t* __restrict__ row_nnz, DevInfo* info, RowMap mp) {
    constexpr int R = T / 128, GS = R < kRowStep ? R : kRowStep;
    int nrows_bin;
    const int32_t* perm;
    work_rows(wk, &nrows_bin, &perm);
    __shared__ long long s_off[65];                 // general path: offsets; else the walk's marks
    __shared__ long long s_bst[65];
    // the bitmap; or the lists' heads and members (column, earlier member); or the hash
    constexpr int H = T <= 1024 ? T / 2 : T / 4;
    __shared__ __align__(16) int32_t keys[H + T > kRowWords ? H + T : kRowWords];
    static_assert(R <= 65, "the marks take the offsets' place");
    const int lane = threadIdx.x;
    int err = 0;
    const long long per = (nrows_bin + gridDim.x - 1) / gridDim.x;
    const long long first = (long long)xcd_block() * per;
    const long long last = first + per < nrows_bin ? first + per : nrows_bin;
    if (first >= last) return;

    // the next row is loaded ahead, as in k_num_row
    struct Head {
        int row;
        long long a0, a1, bo;
    };
    int listed = 0;
    auto head_of = [&](long long slot) {
        Head h;
        h.row = (int)slot;
        if (perm) {
            const int i = (int)(slot - first) & 63;
            if (i == 0) listed = perm[slot + lane < last ? slot + lane : last - 1];
            h.row = __builtin_amdgcn_readlane(listed, i);
        }
        h.a0 = arp[h.row];
        h.a1 = arp[h.row + 1];
        h.bo = row_boff<BATCH>(mp, h.row);
        return h;
    };
    auto load_entry = [&](const Head& h, int* k) {
        if (h.a1 <= h.a0) return;                   // wave-uniform
        *k = acol[h.a0 + lane < h.a1 ? h.a0 + lane : h.a1 - 1];
    };
    auto load_bounds = [&](const Head& h, int k, long long* b0, long long* b1) {
        if (h.a1 <= h.a0) return;
        *b0 = brp[k + h.bo];
        *b1 = brp[k + h.bo + 1];
    };
    Head cur = head_of(first);
    int k = 0, kn = 0;
    long long b0 = 0, b1 = 0, b0n = 0, b1n = 0;
    load_entry(cur, &k);
    load_bounds(cur, k, &b0, &b1);
    for (long long slot = first; slot < last; ++slot) {
        const Head nxt = head_of(slot + 1 < last ? slot + 1 : slot);
        RowWalk<R> walk;
        walk.total = 64 * R + 1;
        if (cur.a1 - cur.a0 <= 64)
            walk.open(lane, b0, cur.a0 + lane < cur.a1 ? b1 - b0 : 0, reinterpret_cast<unsigned long long*>(s_off),
                      s_bst, nullptr, 0.0);
        const int total = walk.total;
        load_entry(nxt, &kn);
        int cnt = 0;
        if (total <= 64 * R) {                      // wave-uniform
            // lanes past the last product repeat the row's first one
            int c[R];
            const long long at0 = s_bst[0];
#pragma unroll
            for (int g = 0; g < R; g += GS)
                if (64 * g < total) {
                    long long at[GS];
#pragma unroll
                    for (int s = g; s < g + GS; ++s) at[s - g] = s_bst[walk.entry(s)] + (64 * s + lane);
#pragma unroll
                    for (int s = g; s < g + GS; ++s) c[s] = bcol[64 * s + lane < total ? at[s - g] : at0];
                }
            int mn = 0x7fffffff, mx = -1;
#pragma unroll
            for (int g = 0; g < R; g += GS)
                if (64 * g < total) {
#pragma unroll
                    for (int s = g; s < g + GS; ++s) {
                        mn = min(mn, c[s]);
                        mx = max(mx, c[s]);
                    }
                }
            load_bounds(nxt, kn, &b0n, &b1n);
            mn = wave_least(mn);
            mx = wave_most(mx);
            const int span = total > 0 ? mx - mn : 0;
            if (span < 32 * kRowWords) {
                uint32_t* const bm = reinterpret_cast<uint32_t*>(keys);
                const int nwd = total > 0 ? (span >> 5) + 1 : 0;
                for (int i = lane * 4; i < nwd; i += 256) *reinterpret_cast<uint4*>(bm + i) = make_uint4(0, 0, 0, 0);
                lds_fence();
#pragma unroll
                for (int g = 0; g < R; g += GS)
                    if (64 * g < total) {
#pragma unroll
                        for (int s = g; s < g + GS; ++s) {
                            const int d = c[s] - mn;
                            atomicOr(&bm[d >> 5], 1u << (d & 31));
                        }
                    }
                lds_fence();
                for (int i = lane * 4; i < nwd; i += 256) {
                    const uint4 x = *reinterpret_cast<const uint4*>(bm + i);
                    cnt += __builtin_popcount(x.x) + __builtin_popcount(x.y) + __builtin_popcount(x.z) +
                           __builtin_popcount(x.w);
                }
            } else {
                int32_t* const head = keys;
                int2* const list = reinterpret_cast<int2*>(keys + H);
                for (int i = lane; i < H / 4; i += 64)
                    reinterpret_cast<int4*>(head)[i] = make_int4(-1, -1, -1, -1);
                lds_fence();
                int prev[R];
#pragma unroll
                for (int g = 0; g < R; g += GS)
                    if (64 * g < total) {
#pragma unroll
                        for (int s = g; s < g + GS; ++s) {
                            const int q = 64 * s + lane;
                            prev[s] = -1;
                            if (q < total) prev[s] = atomicExch(&head[hash_slot<H>(c[s])], q);
                        }
#pragma unroll
                        for (int s = g; s < g + GS; ++s) {
                            list[64 * s + lane] = make_int2(c[s], prev[s]);
                            cnt += 64 * s + lane < total;
                        }
                    }
                lds_fence();
#pragma unroll
                for (int g = 0; g < R; g += GS)
                    if (64 * g < total) {
                        // the members before this one, GS products a lane at once
                        while (true) {
                            bool more = false;
#pragma unroll
                            for (int s = g; s < g + GS; ++s) more |= prev[s] >= 0;
                            if (!__ballot(more)) break;
                            int2 x[GS];
#pragma unroll
                            for (int s = g; s < g + GS; ++s) x[s - g] = list[max(prev[s], 0)];
#pragma unroll
                            for (int s = g; s < g + GS; ++s) {
                                const bool same = prev[s] >= 0 && x[s - g].x == c[s];
                                cnt -= same;
                                prev[s] = prev[s] < 0 || same ? -1 : x[s - g].y;
                            }
                        }
                    }
                lds_fence();
            }
        } else {
            // The first and last columns of the B rows bound the span of a row
            // of at most 64 A entries: a bitmap of it when it is narrow (B's
            // width bounds these rows, so it is), else a hash.
            int mn = 0x7fffffff, mx = -1;
            if (cur.a1 - cur.a0 <= 64) {
                if (cur.a0 + lane < cur.a1 && b1 > b0) {
                    mn = bcol[b0];
                    mx = bcol[b1 - 1];
                }
                mn = wave_least(mn);
                mx = wave_most(mx);
            }
            load_bounds(nxt, kn, &b0n, &b1n);
            const bool narrow = mx >= mn && (long long)mx - mn < 32 * kRowWords;     // wave-uniform
            uint32_t* const bm = reinterpret_cast<uint32_t*>(keys);
            const int nwd = narrow ? ((mx - mn) >> 5) + 1 : 0;
            const int clear = narrow ? (nwd + 3) >> 2 : T / 4, empty = narrow ? 0 : kEmpty;
            for (int i = lane; i < clear; i += 64)
                reinterpret_cast<int4*>(keys)[i] = make_int4(empty, empty, empty, empty);
            lds_fence();
            int full = 0;
            for (long long c0 = cur.a0; c0 < cur.a1; c0 += 64) {
                const long long p = c0 + lane;
                long long len = 0, bst = 0;
                if (p < cur.a1) {
                    const long long kk = acol[p] + cur.bo;
                    bst = brp[kk];
                    len = brp[kk + 1] - bst;
                }
                const long long incl = group_incl_scan<64>(len, lane);
                const long long all = __shfl(incl, 63);
                s_off[lane] = incl;
                s_bst[lane] = bst - (incl - len);
                lds_fence();
                const int nact = (int)((cur.a1 - c0) < 64 ? (cur.a1 - c0) : 64);
                // (GS products a lane in flight)
                int t = -1;                          // owner of q: one search, then it only moves forward
                for (long long q0 = lane; q0 < all; q0 += 64 * GS) {
                    int32_t j[GS];
#pragma unroll
                    for (int u = 0; u < GS; ++u) {
                        const long long q = q0 + 64 * u;
                        j[u] = -1;
                        if (q < all) {
                            if (t < 0) t = owner_search(s_off, nact, q);
                            else while (s_off[t] <= q) ++t;
                            j[u] = bcol[s_bst[t] + q];
                        }
                    }
#pragma unroll
                    for (int u = 0; u < GS; ++u) {
                        if (j[u] < 0) continue;
                        if (narrow) {
                            // (in the span for canonical B; unsorted rows, which
                            // the input contract excludes, stay in bounds)
                            const int d = j[u] - mn;
                            if ((unsigned)d < (unsigned)(nwd << 5)) atomicOr(&bm[d >> 5], 1u << (d & 31));
                        } else {
                            cnt += hash_insert_key<T>(keys, j[u], &full);
                        }
                    }
                }
                lds_fence();
            }
            for (int i = lane; i < nwd; i += 64) cnt += __builtin_popcount(bm[i]);
            if (full) err |= kErrProbe;
        }
        cnt = __builtin_amdgcn_readlane(wave_scan(cnt), 63);
        if (lane == 0) row_nnz[cur.row] = cnt;
        lds_fence();
        cur = nxt;
        k = kn;
        b0 = b0n;
        b1 = b1n;
    }
    if (err) atomicOr(&info->err, err);
}

}  // namespace msp

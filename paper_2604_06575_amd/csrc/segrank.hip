// simplify of a batch whose total degree D is known, one workgroup per
// polynomial (Section 3.3, simplify).
//
// In n variables there are C(n + D, n) monomials of degree at most D, and a
// term's place among them in lexicographic order (muldense.hip) is a key of a
// few bits beside the tens of bits of its exponents: 18 in 20 variables at
// degree 6, against 60.  A polynomial of up to 20,480 terms then fits in LDS
// as (rank, term index) pairs of six bytes, and its terms are read once:
//   * ranks from the exponent rows, two variables to a table read;
//   * a stable radix sort in LDS by the rank's bits (the operation order of
//     equal digits is that of lds_radix_sort);
//   * coefficients gathered in sorted order, each run summed left to right in
//     storage order, as the definition has it;
//   * runs above the tolerance staged as (rank, sum); once the polynomials'
//     counts are scanned, k_sr_unpack writes rows and coefficients.  (Copying a
//     term's row from the input instead: 300 us against 172.)
// Four sizes of workgroup take the polynomials by their number of terms, so
// that short ones share a CU.  The largest size, one workgroup to a CU, is bound
// by its end: CUs are busy for 52% of its time, and then vector instructions
// take 52% of the cycles and LDS 20%.  10.6 million terms in 4,096 polynomials of 10 to
// 20,000, 20 variables, degree 6: k_sr_merge 166 + 85 + 18 + 18 us, k_sr_unpack
// 146, k_max_degree 76, the call 614 us; 1,810 with a device-wide radix sort of
// two key words.  1,024 polynomials of 64 terms: 104 against 264 us.
#include "kernels.h"
#include "ranks.h"

// products and sums are rounded separately, as in the definition (no FMA)
#pragma clang fp contract(off)

namespace polyhip {

namespace {

// Place of a row among the monomials of degree at most D:
//   C(n + D, n) - 1 - sum_j pairs[j][c_(2 j) (D + 1) + c_(2 j + 1)]
// with c_i the degree in the variables up to i.  A row past the declared
// exponent or degree bound sets POLY_ERR_EXPONENT and gets place 0.
__device__ inline uint32_t row_rank(const SegRankArgs &A, const uint8_t *row, const uint32_t *s_pairs)
{
    const uint32_t D1 = (uint32_t)A.D + 1, n = (uint32_t)A.n, last = D1 * D1 - 1;
    uint32_t c = 0, sum = 0, worst = 0;
    const uint32_t *tab = s_pairs;
    const bool check = A.max_exp < A.D;   // else a degree within its bound says it
    auto pair = [&](uint32_t e0, uint32_t e1) {
        if (check) {
            worst = e0 > worst ? e0 : worst;
            worst = e1 > worst ? e1 : worst;
        }
        const uint32_t c0 = c + e0;
        c = c0 + e1;
        const uint32_t x = c0 * D1 + c;
        sum += tab[x < last ? x : last];   // in bounds whatever the row holds
        tab += D1 * D1;
    };
    if (((n | (uint32_t)reinterpret_cast<uintptr_t>(A.exps)) & 3) == 0) {
        const uint32_t *r4 = reinterpret_cast<const uint32_t *>(row);
        for (uint32_t i0 = 0; i0 < n / 4; i0 += 8) {
            uint32_t x[8];
#pragma unroll
            for (uint32_t i = 0; i < 8; ++i) x[i] = i0 + i < n / 4 ? r4[i0 + i] : 0;
#pragma unroll
            for (uint32_t i = 0; i < 8; ++i)
                if (i0 + i < n / 4) {
                    pair(x[i] & 0xffu, (x[i] >> 8) & 0xffu);
                    pair((x[i] >> 16) & 0xffu, x[i] >> 24);
                }
        }
    } else {
        uint32_t i = 0;
        for (; i + 2 <= n; i += 2) pair(row[i], row[i + 1]);
        if (i < n) pair(row[i], 0);
    }
    if (worst > (uint32_t)A.max_exp || c > (uint32_t)A.D) {
        set_status(A.status, POLY_ERR_EXPONENT);
        return 0;
    }
    return A.cells - 1 - sum;
}

// value of v in lane k (k uniform)
__device__ inline double lane_value(double v, int k)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, k);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), k);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

}  // namespace

// Dynamic LDS: CAP ranks, CAP indices, 1 KB per wave (counters of up to nine
// bits of digit; then the coefficients of a round), the rank table.
template <int THREADS, int ITEMS, int DB>
__global__ void __launch_bounds__(THREADS) k_sr_merge(SegRankArgs A, int64_t first)
{
    constexpr int W = THREADS / kWave, CAP = THREADS * ITEMS;
    extern __shared__ double s_dyn[];
    __shared__ uint32_t s_scan[W];
    uint16_t *s_cnt = (uint16_t *)s_dyn;
    uint32_t *key = (uint32_t *)(s_cnt + W * 512);
    uint16_t *idx = (uint16_t *)(key + CAP);
    uint32_t *s_pairs = (uint32_t *)(idx + CAP);
    const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
    const int64_t p = A.order[first + blockIdx.x];
    const int64_t base = A.rp[p], len = A.rp[p + 1] - base;
    const int m = len < CAP ? (int)len : CAP;
    if (m <= 0) {
        if (tid == 0) A.seg_count[p] = 0;
        return;
    }
    const int np = (A.n + 1) / 2 * (A.D + 1) * (A.D + 1);
    for (int x = tid; x < np; x += THREADS) s_pairs[x] = A.pairs[x];
    __syncthreads();
    const int its = (m + THREADS - 1) / THREADS;   // items of each thread, the same for all
    const unsigned long long lt = lane ? (~0ull >> (kWave - lane)) : 0ull;
#pragma unroll 2
    for (int it = 0; it < its; ++it) {
        const int e = (w * its + it) * kWave + lane;
        key[e] = e < m ? row_rank(A, A.exps + (base + e) * A.n, s_pairs) : ~0u;
        idx[e] = (uint16_t)e;
    }
    __syncthreads();
    // passes over the rank's bits; the padding past m has every bit set and is
    // last in the order, where it stays
    constexpr int nbins = 1 << DB;
    for (int sh = 0; sh < A.rank_bits; sh += DB) {
        uint32_t k[ITEMS], v[ITEMS], pos[ITEMS];
#pragma unroll
        for (int it = 0; it < ITEMS; ++it)
            if (it < its) {
                const int e = (w * its + it) * kWave + lane;
                k[it] = key[e];
                v[it] = idx[e];
            }
        for (int i = tid; i < W * nbins; i += THREADS) s_cnt[i] = 0;
        __syncthreads();
        uint16_t *cnt = s_cnt + w * nbins;
#pragma unroll
        for (int it = 0; it < ITEMS; ++it)
            if (it < its) {
                const uint32_t d = (k[it] >> sh) & (uint32_t)(nbins - 1);
                uint32_t lo = ~0u, hi = ~0u;   // lanes with the same digit
#pragma unroll
                for (int b = 0; b < DB; ++b) {
                    const int32_t bit = __builtin_amdgcn_sbfe((int32_t)d, b, 1);   // 0 or -1
                    const unsigned long long bb = __ballot(bit != 0);
                    lo &= ~((uint32_t)bb ^ (uint32_t)bit);
                    hi &= ~((uint32_t)(bb >> 32) ^ (uint32_t)bit);
                }
                const uint32_t before = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
                const uint32_t prior = cnt[d];
                pos[it] = prior + before;
                if (before == 0) cnt[d] = (uint16_t)(prior + __popc(lo) + __popc(hi));
            }
        __syncthreads();
        // exclusive scan over (digit, wave), digit-major
        uint32_t pre[W], tot = 0, bins;
        for (int d0 = 0, run = 0; d0 < nbins; d0 += THREADS) {
            const int d = d0 + tid;
            tot = 0;
#pragma unroll
            for (int ww = 0; ww < W; ++ww) {
                pre[ww] = tot;
                if (d < nbins) tot += s_cnt[ww * nbins + d];
            }
            const uint32_t at = (uint32_t)run + block_exclusive_scan<THREADS>(tot, s_scan, bins);
            run += (int)bins;
            if (d < nbins) {
#pragma unroll
                for (int ww = 0; ww < W; ++ww) s_cnt[ww * nbins + d] = (uint16_t)(at + pre[ww]);
            }
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < ITEMS; ++it)
            if (it < its) {
                const uint32_t q = cnt[(k[it] >> sh) & (uint32_t)(nbins - 1)] + pos[it];
                key[q] = k[it];
                idx[q] = (uint16_t)v[it];
            }
        __syncthreads();
    }
    // runs: a wave takes the runs that begin in its its * 64 elements, 64
    // elements a round, a run's sum carried from round to round and past the
    // wave's last element
    double sum[ITEMS];
    uint32_t kept[ITEMS];   // place among the wave's kept runs, or ~0
    double *s_c = s_dyn + w * kWave;
    const int e0 = w * its * kWave, e1 = e0 + its * kWave < m ? e0 + its * kWave : m;
    uint32_t found = 0;
    double carry = 0.0;
    bool open = false;      // a run of this wave goes on from the round before
    uint32_t last = e0 > 0 && e0 < m ? key[e0 - 1] : 0;
    double next = e0 + lane < m ? A.coefs[base + idx[e0 + lane]] : 0.0;
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        sum[it] = 0.0;
        kept[it] = ~0u;
        const int i = e0 + it * kWave + lane, c0 = e0 + it * kWave;
        if (it >= its || c0 >= m) continue;   // the same on every lane
        __builtin_amdgcn_wave_barrier();
        s_c[lane] = next;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (i + kWave < m) next = A.coefs[base + idx[i + kWave]];
        const uint32_t k = i < m ? key[i] : ~0u;
        uint32_t prev = (uint32_t)__shfl_up((int)k, 1, kWave);
        if (lane == 0) prev = last;
        last = (uint32_t)__builtin_amdgcn_readlane((int)k, kWave - 1);
        const bool head = i < m && (i == 0 || prev != k);
        const bool on = head || (lane == 0 && open);
        const unsigned long long after = __ballot(head) & ~(lt | (1ull << lane));   // heads past this lane
        double s = 0.0;
        bool done = false;
        if (on) {
            s = head ? s_c[lane] : carry + s_c[0];
            const int size = m - c0 < kWave ? m - c0 : kWave;
            const int end = after ? __ffsll((long long)after) - 1 : size;
            int q = lane + 1;
            for (; q + 4 <= end; q += 4) {   // the reads of four together, the additions in order
                const double a = s_c[q], b = s_c[q + 1], c = s_c[q + 2], d = s_c[q + 3];
                s = s + a;
                s = s + b;
                s = s + c;
                s = s + d;
            }
            for (; q < end; ++q) s = s + s_c[q];
            done = end < kWave || c0 + kWave >= m || key[c0 + kWave] != k;
        }
        const unsigned long long undone = __ballot(on && !done);   // one lane at most
        open = undone != 0;
        if (open) carry = lane_value(s, __ffsll((long long)undone) - 1);
        const bool keep = done && !(fabs(s) <= A.tol);
        const unsigned long long kb = __ballot(keep);
        if (keep) {
            sum[it] = s;
            kept[it] = found + (uint32_t)__popcll(kb & lt);
        }
        found += (uint32_t)__popcll(kb);
    }
    // the run that goes on past the wave's elements
    uint32_t tail_key = last;
    double tail = 0.0;
    bool tail_keep = false;
    for (int c0 = e1; open; c0 += kWave) {
        __builtin_amdgcn_wave_barrier();
        s_c[lane] = c0 + lane < m ? A.coefs[base + idx[c0 + lane]] : 0.0;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const unsigned long long same = __ballot(c0 + lane < m && key[c0 + lane] == tail_key);
        const int cnt = ~same ? __ffsll((long long)~same) - 1 : kWave;   // sorted: a prefix
#pragma unroll 8
        for (int q = 0; q < cnt; ++q) carry = carry + s_c[q];
        if (cnt < kWave) {
            open = false;
            tail = carry;
            tail_keep = !(fabs(tail) <= A.tol);
        }
    }
    const uint32_t mine = found + (tail_keep ? 1u : 0u);
    __syncthreads();
    if (lane == 0) s_scan[w] = mine;
    __syncthreads();
    uint32_t off = 0, all = 0;
#pragma unroll
    for (int ww = 0; ww < W; ++ww) {
        off += ww < w ? s_scan[ww] : 0u;
        all += s_scan[ww];
    }
#pragma unroll
    for (int it = 0; it < ITEMS; ++it)
        if (kept[it] != ~0u) {
            A.st_rank[base + off + kept[it]] = key[e0 + it * kWave + lane];
            A.st_coef[base + off + kept[it]] = sum[it];
        }
    if (tail_keep && lane == 0) {
        A.st_rank[base + off + found] = tail_key;
        A.st_coef[base + off + found] = tail;
    }
    if (tid == 0) A.seg_count[p] = all;
}

// Rows and coefficients of the result: 64 consecutive output terms per wave,
// each lane finds its polynomial from the wave's first.  Exponent rows go
// through the wave's LDS buffer and leave as one contiguous run.
// Dynamic LDS: rank table, then 64 * n bytes per wave.
__global__ void __launch_bounds__(256) k_sr_unpack(SegRankArgs A, int64_t P, const int64_t *__restrict__ row_ptr,
                                                   uint8_t *out_exps, double *out_coefs, int64_t capacity)
{
    extern __shared__ double s_dyn[];
    const int n = A.n, D = A.D, lane = lane_id(), wv = wave_id();
    uint32_t *s_tab = (uint32_t *)s_dyn;
    uint8_t *buf = (uint8_t *)(s_tab + n * (D + 2)) + (size_t)wv * kWave * n;
    for (int x = threadIdx.x; x < n * (D + 2); x += 256) s_tab[x] = A.table[x];
    __syncthreads();
    int64_t total = row_ptr[P];
    if (total > capacity) {
        if (blockIdx.x == 0 && threadIdx.x == 0) set_status(A.status, POLY_ERR_CAPACITY);
        total = capacity;
    }
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t q0 = (int64_t)blockIdx.x * 256 + wv * kWave; q0 < total; q0 += stride) {
        const int rows = total - q0 < kWave ? (int)(total - q0) : kWave;
        int64_t lo = 0, hi = P - 1;   // the last polynomial that starts at or before q0
        while (lo < hi) {
            const int64_t mid = (lo + hi + 1) >> 1;
            if (row_ptr[mid] <= q0) lo = mid;
            else hi = mid - 1;
        }
        if (lane < rows) {
            const int64_t q = q0 + lane;
            while (row_ptr[lo + 1] <= q) ++lo;
            const int64_t st = A.rp[lo] + (q - row_ptr[lo]);
            const uint32_t rank = A.st_rank[st];
            const double c = A.st_coef[st];
            unrank_row(rank, n, D, s_tab, buf + lane * n);
            out_coefs[q] = c;
        }
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const uint32_t bytes = (uint32_t)rows * (uint32_t)n;
        uint8_t *o = out_exps + q0 * n;
        if ((reinterpret_cast<uintptr_t>(o) & 3) == 0) {   // whole words, then the bytes left over
            const uint32_t *b4 = reinterpret_cast<const uint32_t *>(buf);
            uint32_t *o4 = reinterpret_cast<uint32_t *>(o);
            for (uint32_t d = lane; d < bytes / 4; d += kWave) o4[d] = b4[d];
            for (uint32_t d = (bytes & ~3u) + lane; d < bytes; d += kWave) o[d] = buf[d];
        } else {
            for (uint32_t d = lane; d < bytes; d += kWave) o[d] = buf[d];
        }
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

#define SR_INSTANCES(DB)                                                  \
    template __global__ void k_sr_merge<1024, 20, DB>(SegRankArgs, int64_t); \
    template __global__ void k_sr_merge<512, 16, DB>(SegRankArgs, int64_t);  \
    template __global__ void k_sr_merge<256, 4, DB>(SegRankArgs, int64_t);   \
    template __global__ void k_sr_merge<64, 4, DB>(SegRankArgs, int64_t);
SR_INSTANCES(7)
SR_INSTANCES(9)
#undef SR_INSTANCES

}  // namespace polyhip

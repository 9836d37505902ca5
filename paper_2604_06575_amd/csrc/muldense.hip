// times and mtimes on a dense range of monomials (Section 3.3, products
// followed by simplify).
//
// When the operands' total degrees are known (dA, dB; D = dA + dB), every
// product monomial has degree at most D, and there are only C(n + D, n) of
// those: the cells of an output entry, numbered by their rank in
// lexicographic order.  Where the raw product is not much sparser than the
// cells, an output entry is cut into ranges of consecutive cells, one
// workgroup each, and the raw product is never stored or sorted in memory:
//   * a row (a term of the left operand, in storage order) meets one
//     contiguous interval of the partner's sorted terms in each range (keys
//     are mixed-radix numbers, so a product key is a sum and sums with a fixed
//     row keep the partner's order); k_md_cut finds all intervals, neighbouring
//     lanes searching for neighbouring range bounds of one row, which costs the
//     ranges' workgroups a read instead of two binary searches per row;
//   * the range's raw products are generated in chunks, in (row, partner)
//     order, which is the order of the definition; each gets its cell from
//     table reads: with c_i the partial degree e_1 + ... + e_i of the product,
//       rank = C(n + D, n) - 1 - sum_i C(n - i + D - c_i, n - i + 1),
//     two variables to a read: a term carries c_i (D + 1) + c_(i+1) in 16 bits
//     per pair, and the operands' values add;
//   * a chunk's products are added to their cells' sums in rounds: in each, the
//     earliest pending product of every cell claims it (an LDS minimum) and is
//     added, so every sum is that of the definition, left to right, whatever
//     the number of chunks.  Chunks are as long as ranges are wide, so a cell
//     meets few products of one chunk and a handful of rounds do;
//   * cells with a sum above the tolerance are staged in order; exponents are
//     recovered from the rank when the result is unpacked.
// The raw product stays on chip.  k_md_range is bound by the latency of its LDS
// rounds: of the cycles that its CUs are busy, vector instructions take 43% and
// LDS 44% (20 of them bank conflicts), and a wave waits for 56% of its time.
// 5,000 x 5,000 terms in 10 variables (25 million raw products, 5.3 million
// cells): k_md_range 317 us (79 G raw products/s), k_md_cut 71, the whole call
// 0.56 ms with read-backs; the radix sort of the raw product's 41-bit keys took
// 1.36 ms.  600 pairs of
// 6 to 300 terms in 8 variables: 77 + 31 us, the call 0.26 against 0.98 ms.
// Ordering each chunk by an LDS counting sort instead of claims: 592 us.
#include "kernels.h"
#include "ranks.h"

// products and sums are rounded separately, as in the definition (no FMA)
#pragma clang fp contract(off)

namespace polyhip {

namespace {

// C(m + d, m) by exact partial products; d may be -1 (zero)
__device__ inline uint32_t monomials_below(int m, int d)
{
    if (d < 0) return 0;
    uint64_t r = 1;
    for (int k = 1; k <= m; ++k) r = r * (uint64_t)(d + k) / (uint64_t)k;
    return (uint32_t)r;
}

}  // namespace

// Largest total degree of the rows of two batches, into host[0] and host[1]
// (host memory that the device can write).  One block writes them itself;
// several meet in deg[0..2] (zero before the launch: two maxima and a count of
// finished blocks), and the last one writes them.
__global__ void __launch_bounds__(1024) k_max_degree(const uint8_t *ea, int64_t Ta, const uint8_t *eb, int64_t Tb,
                                                     int n, uint32_t *deg, int64_t *host)
{
    __shared__ uint32_t s_m[2][16];
    uint32_t m[2] = {0, 0};
    auto rows = [&](auto sum) {   // sum(row): its exponents'
#pragma unroll 2
        for (int64_t t = (int64_t)blockIdx.x * 1024 + threadIdx.x; t < Ta + Tb; t += (int64_t)gridDim.x * 1024) {
            const bool second = t >= Ta;
            const uint32_t d = sum(second ? eb + (t - Ta) * n : ea + t * n);
            if (second) m[1] = d > m[1] ? d : m[1];
            else m[0] = d > m[0] ? d : m[0];
        }
    };
    if (((reinterpret_cast<uintptr_t>(ea) | reinterpret_cast<uintptr_t>(eb) | (uintptr_t)n) & 3) == 0) {
        rows([&](const uint8_t *row) {
            const uint32_t *r4 = reinterpret_cast<const uint32_t *>(row);
            uint32_t d = 0;
            int i = 0;
            for (; i + 4 <= n / 4; i += 4) {
                uint32_t x[4];
                __builtin_memcpy(x, r4 + i, 16);
#pragma unroll
                for (int k = 0; k < 4; ++k) d = __builtin_amdgcn_sad_u8(x[k], 0u, d);
            }
            for (; i < n / 4; ++i) d = __builtin_amdgcn_sad_u8(r4[i], 0u, d);
            return d;
        });
    } else {   // the bytes before the row's first whole word, its words, the bytes after the last
        rows([&](const uint8_t *row) {
            uint32_t d = 0;
            int i = 0;
            for (; i < n && ((reinterpret_cast<uintptr_t>(row) + i) & 3) != 0; ++i) d += row[i];
#pragma unroll 4
            for (; i + 4 <= n; i += 4) d = __builtin_amdgcn_sad_u8(*reinterpret_cast<const uint32_t *>(row + i), 0u, d);
            for (; i < n; ++i) d += row[i];
            return d;
        });
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        uint32_t v = m[k];
#pragma unroll
        for (int o = kWave / 2; o > 0; o >>= 1) {
            const uint32_t y = (uint32_t)__shfl_xor((int)v, o, kWave);
            v = y > v ? y : v;
        }
        if (lane_id() == 0) s_m[k][threadIdx.x >> 6] = v;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    uint32_t v[2] = {0, 0};
    for (int k = 0; k < 2; ++k)
        for (int w = 0; w < 16; ++w) v[k] = s_m[k][w] > v[k] ? s_m[k][w] : v[k];
    if (gridDim.x > 1) {
        atomicMax(deg, v[0]);
        atomicMax(deg + 1, v[1]);
        __threadfence();
        if (atomicAdd(deg + 2, 1u) + 1 != gridDim.x) return;
        __threadfence();
        v[0] = __hip_atomic_load(deg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        v[1] = __hip_atomic_load(deg + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    host[0] = v[0];
    host[1] = v[1];
}

// The status word and a row pointer for the host: one launch that writes to
// host memory instead of two copies, each with its own wait.
__global__ void __launch_bounds__(256) k_read_back(const int32_t *status, const int64_t *row_ptr, int64_t count,
                                                   int64_t *host)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i == 0) host[0] = *status;
    if (i < count) host[1 + i] = row_ptr[i];
}

// Keys and pair words of both operands' terms, and the rank tables:
//   table[i * (D + 2) + x] = B(D - x), the number of monomials of degree at
//     most D - x in the variables from i (from 0) on, C(n - i + D - x, n - i);
//     zero at x = D + 1;
//   pairs[j * (D + 1)^2 + c (D + 1) + c'] = B(D - c - 1) of variable 2 j plus
//     B(D - c' - 1) of variable 2 j + 1 (absent past an odd n).
// Every value is at most the number of cells, below 2^31.  A row past the
// declared exponent or degree bound sets POLY_ERR_EXPONENT and gets zero words.
__global__ void __launch_bounds__(256) k_md_prep(MulDenseArgs A, const uint8_t *ea, int64_t Ta, int amax, int adeg,
                                                 const uint8_t *eb, int64_t Tb, int bmax, int bdeg, uint64_t *ka,
                                                 uint64_t *wa, uint64_t *kb, uint64_t *wb, uint32_t *table,
                                                 uint32_t *pairs)
{
    const int n = A.n, D = A.D, D1 = D + 1;
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x, nt = (int64_t)gridDim.x * 256;
    for (int64_t x = t; x < n * (D + 2); x += nt) table[x] = monomials_below(n - (int)x / (D + 2), D - (int)x % (D + 2));
    for (int64_t x = t; x < (int64_t)((n + 1) / 2) * D1 * D1; x += nt) {
        const int i = 2 * ((int)x / (D1 * D1)), y = (int)x % (D1 * D1);
        uint32_t v = monomials_below(n - i, D - y / D1 - 1);
        if (i + 1 < n) v += monomials_below(n - i - 1, D - y % D1 - 1);
        pairs[x] = v;
    }
    if (t >= Ta + Tb) return;
    const bool second = t >= Ta;
    const int64_t u = second ? t - Ta : t;
    const uint8_t *row = (second ? eb : ea) + u * n;
    uint64_t k = 0, w0 = 0, w1 = 0;
    uint32_t deg = 0;
    int bad = 0;
    for (int i = 0; i < n; ++i) {
        const uint32_t e = row[i];
        bad |= (int)(e > (uint32_t)(second ? bmax : amax));
        k = k * A.radix + e;
        deg += e;
        const uint64_t v = (uint64_t)((i & 1) ? deg : deg * (uint32_t)D1) << (16 * ((i >> 1) & 3));
        if (i < 8) w0 += v;
        else w1 += v;
    }
    bad |= (int)(deg > (uint32_t)(second ? bdeg : adeg));
    if (bad) {
        set_status(A.status, POLY_ERR_EXPONENT);
        w0 = w1 = 0;
        k = 0;
    }
    uint64_t *kk = second ? kb : ka, *ww = second ? wb : wa;
    kk[u] = k;
    ww[2 * u] = w0;
    ww[2 * u + 1] = w1;
}

// Stable sort of each polynomial's terms by key, by counting: a term's place
// is the number of its polynomial's terms with a smaller key, or an equal one
// earlier in storage.  Sixteen threads count for each term.  Blocks from
// sort_blocks on write the first key of every cell range (the last: past every key).
__global__ void __launch_bounds__(256) k_md_sort(MulDenseArgs A, const int64_t *rp, int64_t P, int64_t T,
                                                 const uint64_t *k, const uint64_t *w, const double *c, uint64_t *ks,
                                                 uint64_t *ws, double *cs, int64_t sort_blocks, uint64_t *bounds)
{
    constexpr int G = 16;
    if ((int64_t)blockIdx.x >= sort_blocks) {
        const int64_t b = ((int64_t)blockIdx.x - sort_blocks) * 256 + threadIdx.x;
        if (b > A.nr) return;
        uint64_t key = ~0ull;
        if (b < A.nr) {
            // A product's exponents are below the radix, the range's first
            // monomial's need not be: from one that is not, the key is the
            // smallest above every product with the same leading exponents
            // (that digit the radix, the later ones zero; at most radix^n).
            key = 0;
            bool past = false;
            unrank((uint32_t)(b * A.cpr), A.n, A.D, A.table, [&](int, int e) {
                const uint64_t v = (uint64_t)e < A.radix ? (uint64_t)e : A.radix;
                key = key * A.radix + (past ? 0 : v);
                past = past || v == A.radix;
            });
        }
        bounds[b] = key;
        return;
    }
    const int64_t t = (int64_t)blockIdx.x * (256 / G) + threadIdx.x / G;
    const int g = threadIdx.x % G;
    if (t >= T) return;
    int64_t lo = 0, hi = P - 1;   // polynomial of term t
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (rp[mid] <= t) lo = mid;
        else hi = mid - 1;
    }
    const int64_t b0 = rp[lo], b1 = rp[lo + 1];
    if (t >= b1) return;   // T is the host's, rp may hold fewer terms
    const uint64_t key = k[t];
    uint32_t before = 0;
#pragma unroll 4
    for (int64_t u = b0 + g; u < b1; u += G) {
        const uint64_t x = k[u];
        before += (uint32_t)(x < key || (x == key && u < t));
    }
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) before += (uint32_t)__shfl_xor((int)before, o, kWave);
    if (g == 0) {
        const int64_t d = b0 + before;
        ks[d] = key;
        ws[2 * d] = w[2 * t];
        ws[2 * d + 1] = w[2 * t + 1];
        cs[d] = c[t];
    }
}

// cut[...][b][r]: how many partners of row r (of the entry's rows) have a
// product key below bound b.  Entries lie one after another, each (nr + 1)
// bounds by its rows: entry column j, left polynomials from term a0 on, at
// (j * Ta + a0) * (nr + 1).  A block takes CUT_ROWS left terms and a stretch of
// bounds; tiles of 64 bounds go through LDS so that they leave along the rows.
// grid: x = left terms / CUT_ROWS, y = columns, z = stretches of bounds.
constexpr int CUT_ROWS = 32, CUT_THREADS = 256;

__global__ void __launch_bounds__(CUT_THREADS) k_md_cut(MulDenseArgs A, int64_t P, int64_t Ta, int64_t stretch,
                                                       uint16_t *cut)
{
    extern __shared__ uint64_t s_key[];      // the partners' keys, where every row has the same
    __shared__ uint16_t s_tile[64][CUT_ROWS + 2];
    __shared__ int64_t s_dst[CUT_ROWS], s_rows[CUT_ROWS];
    constexpr int W = CUT_THREADS / kWave, RPW = CUT_ROWS / W;
    const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
    const int64_t t0 = (int64_t)blockIdx.x * CUT_ROWS, j = blockIdx.y;
    const int64_t nb = A.nr + 1;
    const int64_t z0 = (int64_t)blockIdx.z * stretch, z1 = z0 + stretch < nb ? z0 + stretch : nb;
    if (A.kb_lds)
        for (int64_t x = tid; x < A.max_partners; x += CUT_THREADS) s_key[x] = A.kb_s[x];
    // this wave's rows: key, partner list
    uint64_t kr[RPW];
    int64_t base[RPW];
    uint32_t len[RPW], longest = 0;
#pragma unroll
    for (int u = 0; u < RPW; ++u) {
        const int64_t t = t0 + w * RPW + u < Ta ? t0 + w * RPW + u : Ta - 1;
        int64_t lo = 0, hi = P;   // the term's polynomial: the last p with a_rp[p] <= t
        while (hi - lo > 1) {
            const int64_t mid = (lo + hi) >> 1;
            if (A.a_rp[mid] <= t) lo = mid;
            else hi = mid;
        }
        const int64_t pb = A.J ? (lo % A.K) * A.J + j : lo;
        const int64_t i0 = A.J ? lo - lo % A.K : lo;
        kr[u] = A.ka[t];
        base[u] = A.b_rp[pb];
        len[u] = (uint32_t)(A.b_rp[pb + 1] - base[u]);
        if (A.kb_lds && len[u] > A.max_partners) len[u] = (uint32_t)A.max_partners;
        longest = len[u] > longest ? len[u] : longest;
        if (lane == 0) {
            const int64_t a0 = A.a_rp[i0];
            s_dst[w * RPW + u] = (j * Ta + a0) * nb + (t - a0);
            // none past the batch's last term (Ta is the host's, a_rp may hold fewer)
            s_rows[w * RPW + u] = t0 + w * RPW + u < Ta && t < A.a_rp[lo + 1] ? A.a_rp[i0 + A.K] - a0 : 0;
        }
    }
    __syncthreads();
    for (int64_t b0 = z0; b0 < z1; b0 += 64) {
        const uint64_t bound = b0 + lane < z1 ? A.bounds[b0 + lane] : 0;
        // the wave's rows side by side: their probes are in flight together
        uint64_t x[RPW];
        uint32_t c[RPW];
#pragma unroll
        for (int u = 0; u < RPW; ++u) {
            x[u] = bound == ~0ull ? ~0ull : (bound > kr[u] ? bound - kr[u] : 0);
            c[u] = 0;
        }
        for (uint32_t st = longest ? 1u << (31 - __clz((int)longest)) : 0u; st > 0; st >>= 1) {
            uint64_t k[RPW];
#pragma unroll
            for (int u = 0; u < RPW; ++u) {
                const uint32_t p = c[u] + st;
                const uint32_t pi = p <= len[u] ? p - 1 : 0;
                k[u] = A.kb_lds ? s_key[pi] : A.kb_s[base[u] + pi];
            }
#pragma unroll
            for (int u = 0; u < RPW; ++u)
                if (c[u] + st <= len[u] && k[u] < x[u]) c[u] += st;
        }
#pragma unroll
        for (int u = 0; u < RPW; ++u) s_tile[lane][w * RPW + u] = (uint16_t)c[u];
        __syncthreads();
        for (int i = tid; i < 64 * CUT_ROWS; i += CUT_THREADS) {
            const int b = i / CUT_ROWS, r = i % CUT_ROWS;
            if (b0 + b < z1 && s_rows[r] > 0) cut[s_dst[r] + (b0 + b) * s_rows[r]] = s_tile[b][r];
        }
        __syncthreads();
    }
}

namespace {

// Block-wide "any of v", with the barrier that follows a round (one wave: none).
template <int NT>
__device__ inline bool block_any(bool v)
{
    if (NT == kWave) {
        const bool a = __any(v);
        __syncthreads();
        return a;
    }
    return __syncthreads_or(v) != 0;
}

}  // namespace

// One workgroup per cell range: entry q = blockIdx.x / nr, cells [c0, c1).
// Rows are taken NT * RB at a time, their products chunk by chunk.  Dynamic
// LDS: cell sums [cpr], pair tables, claims [cpr], and per row of a step that
// meets the range its first raw position [NT * RB + 1], first partner and
// index [NT * RB].
template <int NT, int IT, int NWORD>
__global__ void __launch_bounds__(NT) k_md_range(MulDenseArgs A)
{
    constexpr int CH = NT * IT, W = NT / kWave, RB = MD_STEP_ROWS, SR = NT * RB;
    extern __shared__ double s_dyn[];
    __shared__ uint64_t s_scan[W];
    const int n = A.n, D1 = A.D + 1, tid = threadIdx.x;
    const int npair = (n + 1) / 2, psize = D1 * D1;
    double *s_acc = s_dyn;                                     // [cpr]
    uint32_t *s_tab = (uint32_t *)(s_acc + A.cpr);             // [npair][D1 * D1]
    uint32_t *s_claim = s_tab + npair * psize;                 // [cpr]
    uint32_t *s_pos = s_claim + A.cpr;                         // [SR + 1]
    uint32_t *s_lo = s_pos + SR + 1;                           // [SR]
    uint16_t *s_row = (uint16_t *)(s_lo + SR);                 // [SR]
    const int64_t q = blockIdx.x / A.nr, rg = blockIdx.x % A.nr;
    const uint32_t c0 = (uint32_t)rg * A.cpr;
    const uint32_t c1 = c0 + A.cpr < A.cells ? c0 + A.cpr : A.cells;
    // entry q: rows = terms of the left polynomials i * K .. i * K + K - 1
    // (contiguous), partners of polynomial k: right polynomial k * J + j;
    // entrywise products (J = 0): left and right polynomial q
    const int64_t i0 = A.J ? (q / A.J) * A.K : q, jb = A.J ? q % A.J : q;
    const int64_t a0 = A.a_rp[i0], rows = A.a_rp[i0 + A.K] - a0;
    const int64_t b0 = A.b_rp[jb];
    const uint16_t *cut0 = A.cut + ((A.J ? jb * A.Ta : 0) + a0) * (A.nr + 1) + rg * rows, *cut1 = cut0 + rows;
    for (int x = tid; x < npair * psize; x += NT) s_tab[x] = A.pairs[x];
    for (uint32_t c = tid; c < A.cpr; c += NT) {
        s_acc[c] = 0.0;
        s_claim[c] = ~0u;
    }
    bool any = false;
    uint32_t last = 0;   // largest cell met: within the range, if the cuts are those of the products' keys
    for (int64_t r0 = 0; r0 < rows; r0 += SR) {
        // ---- rows of this step that meet the range, in row order
        const int64_t rb = r0 + tid * RB;
        uint32_t lo[RB], hi[RB];
#pragma unroll
        for (int u = 0; u < RB; ++u) {
            const int64_t rr = rb + u < rows ? rb + u : rows - 1;
            lo[u] = cut0[rr];
            hi[u] = cut1[rr];
        }
        uint64_t mine = 0;   // rows with partners above, raw products below
#pragma unroll
        for (int u = 0; u < RB; ++u) {
            if (rb + u >= rows) hi[u] = lo[u];
            if (hi[u] > lo[u]) mine += (1ull << 32) + (hi[u] - lo[u]);
        }
        uint64_t tot;
        const uint64_t ex = block_exclusive_scan<NT>(mine, s_scan, tot);
        const uint32_t m = (uint32_t)tot, nz = (uint32_t)(tot >> 32);
        if (m == 0) continue;
        any = true;
        uint32_t k = (uint32_t)(ex >> 32), pos = (uint32_t)ex;
#pragma unroll
        for (int u = 0; u < RB; ++u)
            if (hi[u] > lo[u]) {
                int64_t base = b0;
                if (A.K > 1) {   // the row's polynomial: the last x with a_rp[i0 + x] <= its term
                    int64_t x = 0, y = A.K;
                    while (y - x > 1) {
                        const int64_t mid = (x + y) >> 1;
                        if (A.a_rp[i0 + mid] <= a0 + rb + u) x = mid;
                        else y = mid;
                    }
                    base = A.b_rp[x * A.J + jb];
                }
                s_pos[k] = pos;
                s_lo[k] = (uint32_t)base + lo[u];
                s_row[k] = (uint16_t)(tid * RB + u);
                ++k;
                pos += hi[u] - lo[u];
            }
        if (tid == 0) s_pos[nz] = m;
        __syncthreads();
        const int64_t ar = a0 + r0;
        for (uint32_t q0 = 0; q0 < m; q0 += CH) {
            // ---- products and cells of IT consecutive raw positions per thread
            const uint32_t e0 = (uint32_t)tid * IT;
            const uint32_t left = m - q0;
            uint32_t cell[IT];
            double p[IT];
            uint32_t pend = 0;
#pragma unroll
            for (int u = 0; u < IT; ++u) {
                cell[u] = 0;
                p[u] = 0.0;
            }
            if (e0 < left) {
                uint32_t x = 0, y = nz;   // the row: last k with s_pos[k] <= q0 + e0
                while (y - x > 1) {
                    const uint32_t mid = (x + y) >> 1;
                    if (s_pos[mid] <= q0 + e0) x = mid;
                    else y = mid;
                }
                uint32_t start = s_pos[x], next = s_pos[x + 1], fp = s_lo[x], row = s_row[x];
                uint64_t x0[IT], x1[IT];
#pragma unroll
                for (int u = 0; u < IT; ++u) {
                    const uint32_t e = q0 + e0 + u;
                    const bool live = e0 + u < left;
                    if (live && next <= e) {   // every row holds a product: one step
                        ++x;
                        start = next;
                        next = s_pos[x + 1];
                        fp = s_lo[x];
                        row = s_row[x];
                    }
                    pend |= (uint32_t)live << u;
                    const int64_t ia = ar + row, ib = fp + ((live ? e : next - 1) - start);
                    x0[u] = A.wa[2 * ia] + A.wb_s[2 * ib];
                    x1[u] = NWORD > 1 ? A.wa[2 * ia + 1] + A.wb_s[2 * ib + 1] : 0ull;
                    p[u] = A.ca[ia] * A.cb_s[ib];
                }
                const uint32_t *tab = s_tab;
                const int n0 = npair < 4 ? npair : 4;
                for (int i = 0; i < n0; ++i, tab += psize)
#pragma unroll
                    for (int u = 0; u < IT; ++u) {
                        cell[u] += tab[x0[u] & 0xffffull];
                        x0[u] >>= 16;
                    }
                if (NWORD > 1)
                    for (int i = 4; i < npair; ++i, tab += psize)
#pragma unroll
                        for (int u = 0; u < IT; ++u) {
                            cell[u] += tab[x1[u] & 0xffffull];
                            x1[u] >>= 16;
                        }
#pragma unroll
                for (int u = 0; u < IT; ++u) {
                    const uint32_t c = A.cells - 1u - cell[u] - c0;
                    last = c > last ? c : last;
                    cell[u] = c < A.cpr ? c : A.cpr - 1;
                }
            }
            // ---- rounds: the earliest pending product of each cell is added.
            // A round's claims, then its sums, are read together.
            do {
#pragma unroll
                for (int u = 0; u < IT; ++u)
                    if ((pend >> u) & 1u) atomicMin(&s_claim[cell[u]], e0 + u);
                __syncthreads();
                uint32_t cl[IT], win = 0;
                double sum[IT];
#pragma unroll
                for (int u = 0; u < IT; ++u) cl[u] = s_claim[cell[u]];
#pragma unroll
                for (int u = 0; u < IT; ++u) {
                    win |= (uint32_t)(cl[u] == e0 + u) << u;
                    sum[u] = s_acc[cell[u]];
                }
                win &= pend;
#pragma unroll
                for (int u = 0; u < IT; ++u)
                    if ((win >> u) & 1u) {   // winners hold distinct cells
                        s_acc[cell[u]] = sum[u] + p[u];
                        s_claim[cell[u]] = ~0u;
                    }
                pend &= ~win;
            } while (block_any<NT>(pend != 0));
        }
    }
    if (last >= A.cpr) set_status(A.status, POLY_ERR_EXPONENT);
    __syncthreads();
    // ---- kept cells in order
    const uint32_t span = c1 - c0;
    const uint32_t cpt = (span + NT - 1) / NT;
    const uint32_t cb = (uint32_t)tid * cpt < span ? (uint32_t)tid * cpt : span;
    const uint32_t ce = cb + cpt < span ? cb + cpt : span;
    uint32_t keep = 0;
    if (any)
        for (uint32_t c = cb; c < ce; ++c) keep += (uint32_t)!(fabs(s_acc[c]) <= A.tol);
    uint64_t kept;
    uint32_t d = (uint32_t)block_exclusive_scan<NT>((uint64_t)keep, s_scan, kept);
    const int64_t st = (int64_t)blockIdx.x * A.cpr;
    if (any)
        for (uint32_t c = cb; c < ce; ++c) {
            const double s = s_acc[c];
            if (!(fabs(s) <= A.tol)) {
                A.st_cell[st + d] = c0 + c;
                A.st_coef[st + d] = s;
                ++d;
            }
        }
    if (tid == 0) A.count[blockIdx.x] = (int64_t)kept;
}

// Unpack of cell ranges: each wave takes up to 256 kept cells of a range, 64
// at a time; exponent rows are unranked into the wave's LDS buffer and leave as
// one contiguous run.  Thread q of block 0 .. writes row_ptr as well.
// Dynamic LDS: rank table, then 64 * n bytes per wave.
__global__ void __launch_bounds__(256) k_md_unpack(MulDenseArgs A, const int64_t *out_off, int64_t ranges,
                                                   int64_t entries, uint8_t *out_exps, double *out_coefs,
                                                   int64_t capacity, int64_t *row_ptr)
{
    extern __shared__ double s_dyn[];
    const int n = A.n, D = A.D, lane = lane_id(), wv = wave_id();
    uint32_t *s_tab = (uint32_t *)s_dyn;
    uint8_t *buf = (uint8_t *)(s_tab + n * (D + 2)) + (size_t)wv * kWave * n;
    for (int x = threadIdx.x; x < n * (D + 2); x += 256) s_tab[x] = A.table[x];
    for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q <= entries; q += (int64_t)gridDim.x * 256)
        row_ptr[q] = out_off[q * A.nr];
    __syncthreads();
    if (blockIdx.x == 0 && threadIdx.x == 0 && out_off[ranges] > capacity) set_status(A.status, POLY_ERR_CAPACITY);
    constexpr int64_t UNIT = 4 * kWave;
    const int64_t parts = (A.cpr + UNIT - 1) / UNIT;
    for (int64_t u = (int64_t)blockIdx.x * 4 + wv; u < ranges * parts; u += (int64_t)gridDim.x * 4) {
      const int64_t b = u / parts;
      const int64_t cnt = A.count[b], off = out_off[b];
      const int64_t kend = (u % parts + 1) * UNIT < cnt ? (u % parts + 1) * UNIT : cnt;
      for (int64_t k0 = (u % parts) * UNIT; k0 < kend; k0 += kWave) {
        const int64_t dst = off + k0;
        int64_t rows = kend - k0 < kWave ? kend - k0 : kWave;
        if (dst + rows > capacity) rows = capacity > dst ? capacity - dst : 0;
        if (rows <= 0) break;
        if (lane < rows) {
            const int64_t s = b * A.cpr + k0 + lane;
            out_coefs[dst + lane] = A.st_coef[s];
            uint8_t *row = buf + lane * n;
            unrank_row(A.st_cell[s], n, D, s_tab, row);
        }
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const uint32_t total = (uint32_t)rows * (uint32_t)n;
        uint8_t *o = out_exps + dst * n;
        const uint32_t head = (uint32_t)((4 - (reinterpret_cast<uintptr_t>(o) & 3)) & 3);
        if (head == 0) {   // whole words, then the bytes left over
            const uint32_t *b4 = reinterpret_cast<const uint32_t *>(buf);
            uint32_t *o4 = reinterpret_cast<uint32_t *>(o);
            for (uint32_t d = lane; d < total / 4; d += kWave) o4[d] = b4[d];
            for (uint32_t d = (total & ~3u) + lane; d < total; d += kWave) o[d] = buf[d];
        } else {
            for (uint32_t d = lane; d < total; d += kWave) o[d] = buf[d];
        }
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
    }
}

template __global__ void k_md_range<512, 4, 1>(MulDenseArgs);
template __global__ void k_md_range<512, 4, 2>(MulDenseArgs);
template __global__ void k_md_range<256, 4, 1>(MulDenseArgs);
template __global__ void k_md_range<256, 4, 2>(MulDenseArgs);
template __global__ void k_md_range<64, 4, 1>(MulDenseArgs);
template __global__ void k_md_range<64, 4, 2>(MulDenseArgs);

}  // namespace polyhip

// Affine-normal direction of one polynomial at a batch of points (Section 5,
// the exact log-determinant route).
//
// At a point x with g = grad f(x), e = g / |g| and an orthonormal frame
// Q = [Q_T, e], the direction is nu = Q [tau; -1] with
//   A   = Q_T' H Q_T + reg I          (regularized tangent block, H = Hess f(x))
//   a_i = tr(A^-1 Q_T' D^3f[Q_T e_i] Q_T)
//   tau = A^-1 (Q_T' H e - |g| / (n + 1) a).
// With M = Q_T A^-1 Q_T' (n x n) the correction needs no third-order tensor:
// a = Q_T' w with w_l = sum_jk M_jk d^3 f / dx_j dx_k dx_l (x), and since
// Q_T' e = 0,
//   nu = M (H e - |g| / (n + 1) w) - e.
// Q_T is taken from the Householder reflector P = I - beta v v' that maps e
// to -s e_n (s the sign of e_n): its first n - 1 columns are orthonormal and
// orthogonal to e, so A is the leading block of P H P (a rank-two update of
// H) and M = P [A^-1 0; 0 0] P (applied as such, never formed).  The
// direction does not depend on the choice of Q_T.
//
// One workgroup per point does all of it.  The gradient and the Hessian are
// added up term by term in LDS from each monomial's factor list (variables in
// ascending order, degree <= EV_MAX_DEG): every pair of factor slots adds the
// product of the other factors, so repeated variables get their multiplicity
// by themselves (lists longer than four factors also by runs of a variable).
// The gradient adds up in a fixed order, the Hessian, H e and w as they come.
// (Streaming the formed derivative polynomials over all points, and passing the
// Hessians through memory, took 0.42 of 1.48 ms at n = 64, 4,096 points, most of
// it in 29 small launches.)  A is inverted in place by a blocked Gauss-Jordan
// elimination with partial pivoting:
//   * a panel of NB columns is eliminated with one row per lane in registers,
//     the pivot row broadcast by readlane (one panel wave) or through LDS (several);
//     rows are not swapped, the pivots' permutation is applied when the
//     inverse is read;
//   * the panel then holds D = (pivot block)^-1 in the pivot rows and -A D in
//     the others (G), and every other column is updated at once,
//     A <- mask A + G U, with U the pivot rows' old entries and the mask
//     dropping them: a product of depth NB on v_mfma_f64_16x16x4f64.
// The matrix lives in LDS up to n = AN_MAX_N_LDS and in the workgroup's slot
// of the workspace beyond.  n <= AN_WAVE_N takes four waves per point, one of
// which holds the whole panel (no barrier within it), and four points per CU,
// so that one point's panel runs beside another's MFMAs; larger n eight waves,
// four of them for the panel.  At n = 64 the panels, a serial chain of a pivot
// search, a reciprocal and a row update per column, take 40% of a point's clocks,
// the updates 24 and the gradient and Hessian 13; at n = 160 the updates take
// 53%, each going through the matrix in the workspace (0.96 GB of traffic for
// 256 points), and the panels 28.
// n = 64, 320 terms, 4,096 points: 1,050 us as the kernels before it, 281 us.
// n = 160, 800 terms, 256 points: 7,060 us, 473 us.
#include <limits.h>

#include "kernels.h"

namespace polyhip {

typedef double d4v __attribute__((ext_vector_type(4)));

namespace {

__device__ inline double readlane_d(double v, int lane)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, lane);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), lane);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// v of the lane that the DPP control names; lanes without a source keep v
template <int CTRL>
__device__ inline double dpp_d(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const int lo = (int)(unsigned)b, hi = (int)(unsigned)(b >> 32);
    const unsigned l = (unsigned)__builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false);
    const unsigned h = (unsigned)__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false);
    return __longlong_as_double((long long)(((unsigned long long)h << 32) | l));
}

// largest v of the wave (no NaN): row shifts, then row broadcasts, end in lane 63
__device__ inline double wave_max_d(double v)
{
    v = fmax(v, dpp_d<0x111>(v));
    v = fmax(v, dpp_d<0x112>(v));
    v = fmax(v, dpp_d<0x114>(v));
    v = fmax(v, dpp_d<0x118>(v));
    v = fmax(v, dpp_d<0x142>(v));
    v = fmax(v, dpp_d<0x143>(v));
    return readlane_d(v, 63);
}

template <int NW>
__device__ inline double sum_block(double v, double *red)
{
    v = wave_sum(v);
    if (lane_id() == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < NW; ++i) t += red[i];
    __syncthreads();
    return t;
}

__device__ inline void lds_add(double *p, double v)
{
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// factor r of a list, and the product of a list's d factors but for three
__device__ inline int factor(const uint4 &f, int r)
{
    const uint32_t w = r < 4 ? f.x : (r < 8 ? f.y : f.z);
    return (int)((w >> (8 * (r & 3))) & 0xffu);
}

__device__ inline double product_but(const uint4 &f, int d, const double *x, int a, int b, int l)
{
    double val = 1.0;
    for (int r = 0; r < d; ++r) val *= r == a || r == b || r == l ? 1.0 : x[factor(f, r)];
    return val;
}

// A list's runs of one variable: bit r where one begins at slot r; its length.
// Derivatives of a list longer than a word are formed by runs, a variable's
// multiplicity as a number, where every lane's are few, else slot by slot, the
// same slots on every lane.  1,000 terms of degree up to 12 in 8 variables,
// 1,000 points: 1,570 us by runs, 4,200 by slots; 5,000 terms of degree up to 6
// in 20 variables, 500 points: 1,275 by runs, 815 by slots.
__device__ inline uint32_t run_starts(const uint4 &f, int d)
{
    uint32_t m = 1;
    for (int r = 1; r < d; ++r) m |= (uint32_t)(factor(f, r) != factor(f, r - 1)) << r;
    return m;
}

__device__ inline int run_length(uint32_t runs, int d, int a)
{
    const uint32_t after = runs >> a >> 1;
    return after ? __ffs((int)after) : d - a;
}

// Whether the active lanes' lists (d > 4) are taken by runs: an eighth of the
// steps is the price of slots that differ from lane to lane.
__device__ inline bool by_runs(uint32_t runs, int d)
{
    const int s = __popc(runs);
    int most = 0, longest = 0;
#pragma unroll
    for (int k = 1; k <= EV_MAX_DEG; ++k) {
        most = __any(s >= k) ? k : most;
        longest = __any(d >= k) ? k : longest;
    }
    return 2 * most * most * (most + 1) <= longest * (longest - 1) * (longest - 2);
}

}  // namespace

template <int NW, int PW, int NB, bool LDSM>
__global__ void __launch_bounds__(NW * kWave, NW == 4 ? 4 : 2) k_affine_normal(int n, const uint4 *__restrict__ enc,
                                                              const double *__restrict__ coefs, int64_t T,
                                                              const double *__restrict__ X, int64_t N, double *slots,
                                                              double reg, double *D, double *gnorm, int32_t *status)
{
    constexpr int NT = NW * kWave;
    constexpr int KK = NB / 4;                       // MFMAs per tile and panel
    constexpr int MAXU = PW == 1 ? 2 : 4;            // half column blocks per wave (at most PW * 4 blocks)
    extern __shared__ double s_dyn[];
    const AffineShape sh = affine_shape(n);
    const int ld = sh.ld, mp = sh.mp;
    double *S = LDSM ? s_dyn : slots + (size_t)blockIdx.x * sh.L * ld;   // [L][ld]
    double *e = LDSM ? s_dyn + (size_t)sh.L * ld : s_dyn + AN_BLOCK_DOUBLES;   // [n] unit gradient
    double *v = e + n;                               // [n] Householder vector
    double *t = v + n;                               // [n] H v, then K v
    double *u = t + n;                               // [n] v' K
    double *he = u + n;                              // [n] H e
    double *w = he + n;                              // [n] third-derivative contraction
    double *z = w + n;                               // [n] vectors multiplied by K
    double *x = z + n;                               // [n + 1] coordinates, 1
    int *piv = (int *)(x + n + 1);                   // [mp] pivot row of step k
    int *kinv = piv + mp;                            // [mp] step of pivot row i
    __shared__ double s_red[NW];
    __shared__ double s_row[2][PW][NB];
    __shared__ double s_cval[2][PW];
    __shared__ int s_crow[2][PW];
    const int tid = threadIdx.x;
    const int lane = lane_id(), wv = wave_id();
    // the panel wave where there is one: workgroups that share a CU (numbers
    // 256 apart at first) put theirs on different SIMDs
    const int pw = (int)(blockIdx.x >> 8) % NW;
    const int m = n - 1;
    // The gradient adds up by waves, in vectors that are free until it is
    // complete: in the waves' order it is the same from call to call.
    auto grad_sum = [&](int q) { return q < 7 ? e + q * n : reinterpret_cast<double *>(piv); };
    for (int64_t pt = blockIdx.x; pt < N; pt += gridDim.x) {
        __syncthreads();
        for (int i = tid; i < n; i += NT) {
            x[i] = X[pt * n + i];
#pragma unroll
            for (int q = 0; q < NW; ++q) grad_sum(q)[i] = 0.0;
        }
        if (tid == 0) x[n] = 1.0;
        // ---- gradient (by waves) and Hessian, term by term: the upper
        // triangle adds up in LDS (in row blocks where the matrix does not
        // fit), then both triangles are stored
        double *const gw = grad_sum(wv);
        const int rows = LDSM ? n : AN_BLOCK_DOUBLES / (n | 1);
        const int pitch = LDSM ? ld : (n | 1);
        for (int r0 = 0; r0 < n; r0 += rows) {
            const int r1 = r0 + rows < n ? r0 + rows : n;
            double *A = s_dyn;
            for (int i = r0 + wv; i < r1; i += NW)
                for (int j = lane; j < n; j += kWave) A[(i - r0) * pitch + j] = 0.0;
            __syncthreads();
            for (int64_t q = tid; q < T; q += NT) {
                const uint4 f = enc[q];
                const int d = (int)f.w;
                const double c = coefs[q];
                if (d > EV_MAX_DEG) {
                    set_status(status, POLY_ERR_UNSUPPORTED);
                } else if (d <= 4) {
                    const int fi[4] = {(int)(f.x & 0xffu), (int)((f.x >> 8) & 0xffu), (int)((f.x >> 16) & 0xffu),
                                       (int)(f.x >> 24)};
                    const double y0 = x[fi[0]], y1 = x[fi[1]], y2 = x[fi[2]], y3 = x[fi[3]];
                    if (r0 == 0) {
                        const double c01 = c * y0 * y1, c23 = c * y2 * y3;
                        if (d > 0) lds_add(&gw[fi[0]], y1 * c23);
                        if (d > 1) lds_add(&gw[fi[1]], y0 * c23);
                        if (d > 2) lds_add(&gw[fi[2]], y3 * c01);
                        if (d > 3) lds_add(&gw[fi[3]], y2 * c01);
                    }
                    auto pair = [&](int a, int b, double val) {
                        if (b < d && (LDSM || (fi[a] >= r0 && fi[a] < r1)))
                            lds_add(&A[(fi[a] - r0) * pitch + fi[b]], fi[a] == fi[b] ? 2.0 * val : val);
                    };
                    pair(0, 1, c * (y2 * y3));
                    pair(0, 2, c * (y1 * y3));
                    pair(1, 2, c * (y0 * y3));
                    pair(0, 3, c * (y1 * y2));
                    pair(1, 3, c * (y0 * y2));
                    pair(2, 3, c * (y0 * y1));
                } else {
                    const uint32_t runs = run_starts(f, d);
                    const bool whole = by_runs(runs, d);
                    for (int a = 0; a < d && !whole; ++a) {
                        const int fa = factor(f, a);
                        if (r0 == 0) lds_add(&gw[fa], c * product_but(f, d, x, a, a, a));
                        if (fa < r0 || fa >= r1) continue;
                        for (int b = a + 1; b < d; ++b) {
                            const int fb = factor(f, b);
                            const double val = c * product_but(f, d, x, a, b, b);
                            lds_add(&A[(fa - r0) * pitch + fb], fa == fb ? 2.0 * val : val);
                        }
                    }
                    for (uint32_t ma = whole ? runs : 0u; ma; ma &= ma - 1) {
                        const int a = __ffs((int)ma) - 1, fa = factor(f, a), ka = run_length(runs, d, a);
                        if (r0 == 0) lds_add(&gw[fa], (double)ka * c * product_but(f, d, x, a, a, a));
                        if (fa < r0 || fa >= r1) continue;
                        for (uint32_t mb = ma; mb; mb &= mb - 1) {
                            const int b = __ffs((int)mb) - 1, kb = b == a ? ka - 1 : run_length(runs, d, b);
                            if (kb > 0)
                                lds_add(&A[(fa - r0) * pitch + factor(f, b)],
                                        (double)(ka * kb) * c * product_but(f, d, x, a, b == a ? a + 1 : b, a));
                        }
                    }
                }
            }
            __syncthreads();
            if (LDSM) {
                for (int i = wv; i < n; i += NW)
                    for (int j = lane; j < i; j += kWave) S[i * ld + j] = A[j * pitch + i];
            } else {
                for (int i = r0 + wv; i < r1; i += NW)
                    for (int j = i + lane; j < n; j += kWave) S[i * ld + j] = A[(i - r0) * pitch + j];
                for (int j = r0 + 1 + wv; j < n; j += NW)
                    for (int i = r0 + lane; i < (j < r1 ? j : r1); i += kWave) S[j * ld + i] = A[(i - r0) * pitch + j];
            }
            __syncthreads();
        }
        double part = 0.0;
        for (int i = tid; i < n; i += NT) {
            double ei = e[i];
#pragma unroll
            for (int q = 1; q < NW; ++q) ei += grad_sum(q)[i];
            e[i] = ei;
            part += ei * ei;
            w[i] = he[i] = t[i] = 0.0;
        }
        const double gn = sqrt(sum_block<NW>(part, s_red));
        const double sgn = e[m] / gn >= 0.0 ? 1.0 : -1.0;
        __syncthreads();
        for (int i = tid; i < n; i += NT) {
            const double ei = e[i] / gn;
            e[i] = ei;
            v[i] = i == m ? ei + sgn : ei;
        }
        __syncthreads();
        // H e and H v (H is symmetric: columns read along rows)
        for (int i = lane; i < n; i += kWave) {
            double a = 0.0, b = 0.0;
#pragma unroll 4
            for (int j = wv; j < n; j += NW) {
                const double hij = S[j * ld + i];
                a += hij * e[j];
                b += hij * v[j];
            }
            lds_add(&he[i], a);
            lds_add(&t[i], b);
        }
        __syncthreads();
        part = 0.0;
        double part2 = 0.0;
        for (int i = tid; i < n; i += NT) {
            part += v[i] * v[i];
            part2 += v[i] * t[i];
        }
        const double beta = 2.0 / sum_block<NW>(part, s_red);
        const double bv = beta * beta * sum_block<NW>(part2, s_red);   // beta^2 v'Hv
        // P H P = H - beta (v t' + t v') + beta^2 (v'Hv) v v', in place: the
        // regularized tangent block A in the leading m x m corner, padded to a
        // multiple of 16 by the identity
        for (int j = lane; j < mp; j += kWave) {
            const double vj = j < m ? v[j] : 0.0, tj = j < m ? t[j] : 0.0;
            constexpr int UN = 4;                   // rows in flight
            for (int i0 = wv * UN; i0 < mp; i0 += NW * UN) {   // mp is a multiple of UN
                double h[UN], vi[UN], ti[UN];
#pragma unroll
                for (int r = 0; r < UN; ++r) {
                    const int i = i0 + r < n ? i0 + r : n - 1;
                    h[r] = S[(i0 + r) * ld + j];
                    vi[r] = v[i];
                    ti[r] = t[i];
                }
#pragma unroll
                for (int r = 0; r < UN; ++r) {
                    const int i = i0 + r;
                    double b = h[r] - beta * (vi[r] * tj + ti[r] * vj) + bv * vi[r] * vj;
                    if (i == j) b += reg;
                    S[i * ld + j] = i < m && j < m ? b : (i == j ? 1.0 : 0.0);
                }
            }
        }
        __syncthreads();
        // ---- A^-1 in place
        const int row = PW == 1 ? lane : tid;       // this lane's panel row
        bool used = row >= mp;
        for (int kb = 0; kb < mp; kb += NB) {
            if (PW == 1 ? wv == pw : wv < PW) {
                double a[NB];
#pragma unroll
                for (int j = 0; j < NB; ++j) a[j] = row < mp ? S[row * ld + kb + j] : 0.0;
#pragma unroll
                for (int k = 0; k < NB; ++k) {
                    // the unused row with the largest entry in column k (the
                    // smallest row on ties; NaN last)
                    const double mag = fabs(a[k]);
                    const double key = used ? -1.0 : (mag >= 0.0 ? mag : -0.5);
                    const double best = wave_max_d(key);
                    const int il = __ffsll((long long)__ballot(key == best)) - 1;
                    double prow[NB];
                    int ip = il;
                    if (PW == 1) {
#pragma unroll
                        for (int j = 0; j < NB; ++j) prow[j] = readlane_d(a[j], il);
                    } else {
                        const int par = k & 1;
                        if (lane == il) {
#pragma unroll
                            for (int j = 0; j < NB; ++j) s_row[par][wv][j] = a[j];
                            s_cval[par][wv] = best;
                            s_crow[par][wv] = row;
                        }
                        __syncthreads();
                        double bb = s_cval[par][0];
                        int ws = 0;
#pragma unroll
                        for (int q = 1; q < PW; ++q) {
                            const double c = s_cval[par][q];
                            if (c > bb) {
                                bb = c;
                                ws = q;
                            }
                        }
                        ip = s_crow[par][ws];
#pragma unroll
                        for (int j = 0; j < NB; ++j) prow[j] = s_row[par][ws][j];
                    }
                    const double pinv = 1.0 / prow[k];
                    if (row == ip) {   // the pivot row, scaled; its column holds the reciprocal
#pragma unroll
                        for (int j = 0; j < NB; ++j) a[j] = j == k ? pinv : a[j] * pinv;
                        used = true;
                        piv[kb + k] = row;
                        kinv[row] = kb + k;
                    } else {
                        const double g = a[k] * pinv;
#pragma unroll
                        for (int j = 0; j < NB; ++j) a[j] = j == k ? -g : a[j] - g * prow[j];
                    }
                }
                if (row < mp)
#pragma unroll
                    for (int j = 0; j < NB; ++j) S[row * ld + kb + j] = a[j];
            } else if (PW > 1) {
                for (int k = 0; k < NB; ++k) __syncthreads();
            }
            __syncthreads();
            // pivot rows of the panel: this lane's rows of U, and bit masks
            int ur[KK];
#pragma unroll
            for (int q = 0; q < KK; ++q) ur[q] = piv[kb + 4 * q + (lane >> 4)];
            unsigned long long pm[PW] = {};
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const int p = __builtin_amdgcn_readfirstlane(piv[kb + j]);
#pragma unroll
                for (int q = 0; q < PW; ++q) pm[q] |= (p >> 6) == q ? 1ull << (p & 63) : 0ull;
            }
            const int ncb = mp >> 4;
            const int col = lane & 15, lr = lane >> 4;
            // this wave's units: halves of column blocks, their U entries read
            // before any tile is overwritten
            const int units = 2 * ncb;
            double bu[MAXU][KK];
#pragma unroll
            for (int q = 0; q < MAXU; ++q) {
                const int un = wv + q * NW;
                const int cb = un >> 1;
#pragma unroll
                for (int k = 0; k < KK; ++k) bu[q][k] = un < units ? S[ur[k] * ld + cb * 16 + col] : 0.0;
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < MAXU; ++q) {
                const int un = wv + q * NW;
                if (un >= units) break;
                const int cb = un >> 1;
                if (NB == 16 && cb * 16 == kb) continue;
                const int half = (ncb + 1) >> 1;
                const int ra = (un & 1) * half;
                const int rb = (un & 1) ? ncb : half;
                // panel columns keep G
                const bool live = NB == 16 || (unsigned)(cb * 16 + col - kb) >= (unsigned)NB;
                constexpr int RU = LDSM ? 2 : 4;    // tiles in flight
                for (int rt = ra; rt < rb; rt += RU) {
                    d4v c[RU];
                    double ga[RU][KK];
#pragma unroll
                    for (int r = 0; r < RU; ++r) {
                        const int tr = rt + r < rb ? rt + r : rb - 1;
#pragma unroll
                        for (int k = 0; k < KK; ++k) ga[r][k] = S[(tr * 16 + col) * ld + kb + 4 * k + lr];
                        unsigned long long mk = pm[0];
#pragma unroll
                        for (int p = 1; p < PW; ++p) mk = (tr >> 2) == p ? pm[p] : mk;
                        mk >>= (tr & 3) * 16 + lr;
#pragma unroll
                        for (int y = 0; y < 4; ++y) {
                            const double s = S[(tr * 16 + lr + 4 * y) * ld + cb * 16 + col];
                            c[r][y] = (mk >> (4 * y)) & 1ull ? 0.0 : s;
                        }
                    }
#pragma unroll
                    for (int k = 0; k < KK; ++k)
#pragma unroll
                        for (int r = 0; r < RU; ++r)
                            c[r] = __builtin_amdgcn_mfma_f64_16x16x4f64(ga[r][k], bu[q][k], c[r], 0, 0, 0);
#pragma unroll
                    for (int r = 0; r < RU; ++r)
                        if (rt + r < rb && live)
#pragma unroll
                            for (int y = 0; y < 4; ++y) S[((rt + r) * 16 + lr + 4 * y) * ld + cb * 16 + col] = c[r][y];
                }
            }
            __syncthreads();
        }
        // ---- K = A^-1: K_ab = S[piv[a]][kinv[b]] for a, b < m, else 0.
        // t = K v, u = v' K
        for (int i = tid; i < n; i += NT) t[i] = u[i] = 0.0;
        __syncthreads();
        auto kv = [&](const double *y, int q) { return q < m ? y[q] : 0.0; };
        for (int i = lane; i < n; i += kWave) {
            double a = 0.0, b = 0.0;
            if (i < m) {
                const double *Sr = S + piv[i] * ld;
                const int ci = kinv[i];
#pragma unroll 4
                for (int c = wv; c < mp; c += NW) {
                    a += Sr[c] * kv(v, piv[c]);
                    b += kv(v, kinv[c]) * S[c * ld + ci];
                }
            }
            lds_add(&t[i], a);
            lds_add(&u[i], b);
        }
        __syncthreads();
        part = 0.0;
        for (int i = tid; i < n; i += NT) part += v[i] * t[i];
        const double bk = beta * beta * sum_block<NW>(part, s_red);   // beta^2 v'Kv
        // ---- w_l = sum_jk M_jk f_jkl(x), term by term, M = P K P
        auto entry = [&](int a, int b) {
            const double k = a < m && b < m ? S[piv[a] * ld + kinv[b]] : 0.0;
            return k - beta * (t[a] * v[b] + v[a] * u[b]) + bk * v[a] * v[b];
        };
        for (int64_t q = tid; q < T; q += NT) {
            const uint4 f = enc[q];
            const int d = (int)f.w;
            if (d < 3 || d > EV_MAX_DEG) continue;
            const double c = coefs[q];
            if (d <= 4) {
                const int f0 = (int)(f.x & 0xffu), f1 = (int)((f.x >> 8) & 0xffu), f2 = (int)((f.x >> 16) & 0xffu);
                const double m01 = c * (entry(f0, f1) + entry(f1, f0)), m02 = c * (entry(f0, f2) + entry(f2, f0)),
                             m12 = c * (entry(f1, f2) + entry(f2, f1));
                if (d == 3) {
                    lds_add(&w[f0], m12);
                    lds_add(&w[f1], m02);
                    lds_add(&w[f2], m01);
                } else {
                    const int f3 = (int)(f.x >> 24);
                    const double m03 = c * (entry(f0, f3) + entry(f3, f0)), m13 = c * (entry(f1, f3) + entry(f3, f1)),
                                 m23 = c * (entry(f2, f3) + entry(f3, f2));
                    const double y0 = x[f0], y1 = x[f1], y2 = x[f2], y3 = x[f3];
                    lds_add(&w[f0], m12 * y3 + m13 * y2 + m23 * y1);
                    lds_add(&w[f1], m02 * y3 + m03 * y2 + m23 * y0);
                    lds_add(&w[f2], m01 * y3 + m03 * y1 + m13 * y0);
                    lds_add(&w[f3], m01 * y2 + m02 * y1 + m12 * y0);
                }
            } else {
                const uint32_t runs = run_starts(f, d);
                const bool whole = by_runs(runs, d);
                for (int a = 0; a < d && !whole; ++a)
                    for (int b = a + 1; b < d; ++b) {
                        const int fa = factor(f, a), fb = factor(f, b);
                        const double mab = c * (entry(fa, fb) + entry(fb, fa));
                        for (int l = 0; l < d; ++l)
                            if (l != a && l != b) lds_add(&w[factor(f, l)], mab * product_but(f, d, x, a, b, l));
                    }
                for (uint32_t ma = whole ? runs : 0u; ma; ma &= ma - 1) {
                    const int a = __ffs((int)ma) - 1, fa = factor(f, a), ka = run_length(runs, d, a);
                    for (uint32_t mb = ma; mb; mb &= mb - 1) {
                        // slots a and b, and how many pairs of slots are of these variables
                        const int b0 = __ffs((int)mb) - 1, b = b0 == a ? a + 1 : b0;
                        const int pairs = b0 == a ? ka * (ka - 1) / 2 : ka * run_length(runs, d, b);
                        if (pairs == 0) continue;
                        const int fb = factor(f, b);
                        const double mab = (double)pairs * c * (entry(fa, fb) + entry(fb, fa));
                        for (uint32_t ml = runs; ml; ml &= ml - 1) {
                            const int l0 = __ffs((int)ml) - 1, used = (l0 == a) + (l0 == b0);
                            const int kl = run_length(runs, d, l0) - used;
                            if (kl > 0)
                                lds_add(&w[factor(f, l0)], (double)kl * mab * product_but(f, d, x, a, b, l0 + used));
                        }
                    }
                }
            }
        }
        __syncthreads();
        // ---- nu = P K P (H e - |g| / (n + 1) w) - e
        const double cg = gn / (double)(n + 1);
        part = 0.0;
        for (int i = tid; i < n; i += NT) {
            const double r = he[i] - cg * w[i];
            z[i] = r;
            part += v[i] * r;
        }
        const double bz = beta * sum_block<NW>(part, s_red);
        for (int i = tid; i < n; i += NT) {
            z[i] -= bz * v[i];
            t[i] = 0.0;
        }
        __syncthreads();
        for (int i = lane; i < m; i += kWave) {
            const double *Sr = S + piv[i] * ld;
            double a = 0.0;
#pragma unroll 4
            for (int c = wv; c < mp; c += NW) a += Sr[c] * kv(z, piv[c]);
            lds_add(&t[i], a);
        }
        __syncthreads();
        part = 0.0;
        for (int i = tid; i < n; i += NT) part += v[i] * t[i];
        const double by = beta * sum_block<NW>(part, s_red);
        for (int i = tid; i < n; i += NT) D[pt * n + i] = (t[i] - by * v[i]) - e[i];
        if (gnorm && tid == 0) gnorm[pt] = gn;
    }
}

template __global__ void k_affine_normal<4, 1, 8, true>(int, const uint4 *, const double *, int64_t, const double *,
                                                     int64_t, double *, double, double *, double *, int32_t *);
template __global__ void k_affine_normal<8, 4, 16, true>(int, const uint4 *, const double *, int64_t, const double *,
                                                      int64_t, double *, double, double *, double *, int32_t *);
template __global__ void k_affine_normal<8, 4, 16, false>(int, const uint4 *, const double *, int64_t, const double *,
                                                       int64_t, double *, double, double *, double *, int32_t *);

}  // namespace polyhip

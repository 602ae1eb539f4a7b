// Edge correction on the device (Section 3.2, eqs. edge-correction-matrix and
// edge-corrected-NPCF), FP64 throughout: one n x n system per radial-bin tuple B,
//
//   A[L''][L] = M_{L L''}(B) = sum_{L'} f_{L'}(B) E(L'') G^{L L' L''},  f = R_{L'} / R_0,
//   sum_L A[L''][L] zeta_L = N_{L''} / R_0   (eq. edge-correction-matrix as written:
//   M transposed).
//
// k_edge_ell lays the Gaunt terms out for k_edge_matrix, which forms A of several bin
// tuples per pass over the terms, each entry a fixed-order sum; M is symmetric in the
// real numbers used here, so only the 64 x 64 blocks on and above the diagonal are
// summed and k_edge_mirror copies them below it.  The systems are then
// solved together by a blocked right-looking LU with partial pivoting (row exchanges
// chosen by the first largest |pivot|, so the result does not depend on timing): the
// right-hand side is column n of A and takes part in every step.  Per 128 columns:
//   k_lu_panel  factors 64 columns (one workgroup per system),
//   k_lu_rows   exchanges rows right of them and forms U12 (one column per lane),
//   k_lu_gemm   updates the next 64 columns (FP64 matrix cores); then the second 64
//               columns the same way, their rows updated by the first 64's before U12,
//   k_lu_gemm   updates the trailing matrix with all 128,
// and k_lu_back substitutes back; k_edge_small solves systems of up to 32 multiplets
// whole.  B with R_0 = 0 or a zero pivot get NaN and are counted.
//
// Measured, 10 radial bins: 6PCF lmax 3 (2,212 multiplets, 252 systems) 392 -> 87 ms a
// call, matrix build 85 -> 18 ms, solve 307 -> 68 ms of which the trailing updates 43
// ms (41 TFLOP/s; the FP64 16 x 16 x 4 instructions alone reach 48); 5PCF lmax 4 (585 x
// 210) 14.5 -> 4.2 ms, of which the panels 1.5 ms.  Before, one workgroup per system
// did every step, with panels of 32 columns eliminated in global memory.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <utility>

#include "device.h"

namespace encore {

namespace {

constexpr int kEdgeThreads = 1024;
constexpr int kPanel = 64;          // columns of one panel
constexpr int kOuter = 2 * kPanel;  // columns per update of the trailing matrix
constexpr int kSub = 8;             // columns a panel eliminates in registers
constexpr int kSmall = 32;          // multiplets of a system that one wave solves

typedef double d2 __attribute__((ext_vector_type(2)));
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));   // a pair at any column
typedef double d4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------ matrix build
// Terms of the entries (L'', 64 consecutive L) as a block [t][lane] padded to the
// longest of the 64 lists (value 0, L' = n: f is 0 there): a wave reads them with two coalesced
// loads per term.  Read as one list per entry, each lane's loads were 4 bytes and 8
// bytes of cache lines of its own.
__global__ void __launch_bounds__(256) k_edge_ell(int n, const int64_t* __restrict__ row_start,
                                                  const int32_t* __restrict__ term_lp,
                                                  const double* __restrict__ term_val,
                                                  const int64_t* __restrict__ ell_off, uint16_t* __restrict__ lp,
                                                  double* __restrict__ val)
{
    const int nblk = (n + kWave - 1) / kWave;
    const int64_t unit = (int64_t)blockIdx.x * 4 + threadIdx.x / kWave;   // (L'', block of L)
    if (unit >= (int64_t)n * nblk) return;
    const int lane = threadIdx.x & (kWave - 1);
    const int Lpp = (int)(unit / nblk), L = (int)(unit % nblk) * kWave + lane;
    const int64_t o = ell_off[unit], w = (ell_off[unit + 1] - o) / kWave;
    int64_t t0 = 0, cnt = 0;
    if (L < n) {
        t0 = row_start[(int64_t)L * n + Lpp];
        cnt = row_start[(int64_t)L * n + Lpp + 1] - t0;
    }
    for (int64_t t = 0; t < w; ++t) {
        lp[o + t * kWave + lane] = t < cnt ? (uint16_t)term_lp[t0 + t] : (uint16_t)n;
        val[o + t * kWave + lane] = t < cnt ? term_val[t0 + t] : 0.0;
    }
}

// One workgroup per (group of G bin tuples, range of L''): f of the G bin tuples sits
// in LDS ([L'][G], zeros in row n); a wave takes 64 entries (L'', 64 L), a lane per L, and adds each
// term to all G sums (6PCF lmax 3, 112M terms above the diagonal times 252 bin tuples:
// 15.4 ms).  Bound by the LDS reads of f (G values per lane and term, at
// random L'): the lanes start their G / 2 reads of 16 bytes at different pairs, since
// the same pair of every row lies on a quarter (G = 8) of the banks.
template <int G>
__global__ void __launch_bounds__(kEdgeThreads) k_edge_matrix(EdgeArgs a, int B_lo, int nB_here, int rows_per_block)
{
    extern __shared__ __align__(16) double f[];   // [nlam + 1][G]
    constexpr int NC = G / 2;
    const int n = a.nlam;
    const int B0 = B_lo + blockIdx.x * G;
    const int nb = min(G, B_lo + nB_here - B0);
    for (int i = threadIdx.x; i < (n + 1) * G; i += kEdgeThreads) {
        const int lp = i / G, g = i - lp * G;
        f[i] = lp < n && g < nb ? a.rmult[(size_t)lp * a.nB + B0 + g] / a.rmult[B0 + g] : 0.0;
    }
    __syncthreads();
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int nblk = (n + kWave - 1) / kWave;
    const int q0 = blockIdx.y * rows_per_block, q1 = min(n, q0 + rows_per_block);
    const int rot = lane & (NC - 1);
    for (int u = q0 * nblk + wave; u < q1 * nblk; u += kEdgeThreads / kWave) {
        const int Lpp = u / nblk, blk = u - Lpp * nblk, L = blk * kWave + lane;
        if (blk < Lpp / kWave) continue;            // below the diagonal
        const int64_t o = a.ell_off[u], o1 = a.ell_off[u + 1];
        double2 s[NC];
#pragma unroll
        for (int r = 0; r < NC; ++r) s[r] = make_double2(0.0, 0.0);
        for (int64_t t = o; t < o1; t += kWave) {
            const double v = a.ell_val[t + lane];
            const double2* fp = reinterpret_cast<const double2*>(f) + (size_t)a.ell_lp[t + lane] * NC;
#pragma unroll
            for (int r = 0; r < NC; ++r) {
                const double2 w = fp[(r + rot) & (NC - 1)];
                s[r].x += v * w.x;
                s[r].y += v * w.y;
            }
        }
        if (L >= n) continue;
#pragma unroll
        for (int c = 0; c < NC; ++c) {   // pair c of the lane's sums is s[(c - rot) mod NC]
            double2 v = s[c];
#pragma unroll
            for (int k = 1; k < NC; ++k)
                if (rot == k) v = s[(c - k + NC) & (NC - 1)];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int g = 2 * c + h;
                if (g >= nb) continue;
                a.A[((size_t)(B0 - B_lo + g) * n + Lpp) * a.ld + L] = h ? v.y : v.x;
            }
        }
    }
}

// The 64 x 64 block (I, J >= I) of A to (J, I), through LDS (of a block on the diagonal
// the part above it)
__global__ void __launch_bounds__(256) k_edge_mirror(double* __restrict__ A0, int n, int ld)
{
    __shared__ double t[kWave][kWave + 1];
    const int I = blockIdx.y, J = blockIdx.x;
    if (J < I) return;
    double* A = A0 + (size_t)blockIdx.z * n * ld;
    const int c = threadIdx.x & (kWave - 1);
    for (int i = threadIdx.x / kWave; i < kWave; i += 4) {
        const int row = I * kWave + i, col = J * kWave + c;
        t[i][c] = (row < n && col < n) ? A[(size_t)row * ld + col] : 0.0;
    }
    __syncthreads();
    for (int i = threadIdx.x / kWave; i < kWave; i += 4) {
        const int row = J * kWave + i;
        if (row < n && (J > I || c < i)) A[(size_t)row * ld + I * kWave + c] = t[c][i];
    }
}

// M[L][L''] of the bin tuples for the caller
__global__ void __launch_bounds__(256) k_edge_copy_out(const double* __restrict__ A, int n, int ld,
                                                       double* __restrict__ M)
{
    const size_t row = blockIdx.x;                  // of all the systems' rows
    for (int c = threadIdx.x; c < n; c += 256) M[row * n + c] = A[row * ld + c];
}

template <int G>
int launch_edge_matrix(const EdgeArgs& a, int B_lo, int nB_here, hipStream_t stream)
{
    const int gx = (nB_here + G - 1) / G;
    // ~2048 blocks: the first row ranges hold twice the average work
    const int gy = std::max(1, std::min(a.nlam, (2048 + gx - 1) / gx));
    const int rows = (a.nlam + gy - 1) / gy;
    const size_t lds = sizeof(double) * (size_t)(a.nlam + 1) * G;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_edge_matrix<G>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return (int)e;
    k_edge_matrix<G><<<dim3((unsigned)gx, (unsigned)((a.nlam + rows - 1) / rows)), dim3(kEdgeThreads), lds, stream>>>(
        a, B_lo, nB_here, rows);
    e = hipGetLastError();
    if (e != hipSuccess) return (int)e;
    if (a.nlam <= kSmall && !a.M_out) return (int)hipSuccess;   // k_edge_small reads above the diagonal alone
    const unsigned nblk = (unsigned)((a.nlam + kWave - 1) / kWave);
    k_edge_mirror<<<dim3(nblk, nblk, (unsigned)nB_here), dim3(256), 0, stream>>>(a.A, a.nlam, a.ld);
    if (a.M_out)
        k_edge_copy_out<<<dim3((unsigned)(nB_here * a.nlam)), dim3(256), 0, stream>>>(
            a.A, a.nlam, a.ld, a.M_out + (size_t)B_lo * a.nlam * a.nlam);
    return (int)hipGetLastError();
}

// ------------------------------------------------------------------ LU
// Systems of one chunk of bin tuples: matrix b at A + b n ld (row-major, column n the
// right-hand side); panel workspace P + b kOuter mp (column-major: P[c mp + i] holds
// row o + i of the outer block's column c, L below and on the diagonal block U).
struct LuArgs {
    int n, ld, mp, nb;
    double* A;
    double* P;
    int32_t* perm;    // [nb][3 kPanel]: the row now in panel row t; exchanged row or -1; its new content's row
    unsigned* bad;    // [nb]
};

// right-hand sides and the check of R_0
__global__ void __launch_bounds__(256) k_lu_rhs(LuArgs u, const double* __restrict__ nmult,
                                                const double* __restrict__ rmult, int B_lo, int nB)
{
    const int b = blockIdx.x;
    const double r0 = rmult[B_lo + b];
    if (threadIdx.x == 0) u.bad[b] = (!(r0 != 0.0) || !std::isfinite(r0)) ? 1u : 0u;
    double* A = u.A + (size_t)b * u.n * u.ld;
    for (int i = threadIdx.x; i < u.n; i += 256) A[(size_t)i * u.ld + u.n] = nmult[(size_t)i * nB + B_lo + b] / r0;
}

template <int CTRL>
__device__ __forceinline__ double dpp(double v)
{
    const long long u = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)u, CTRL, 0xf, 0xf, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(u >> 32), CTRL, 0xf, 0xf, false);
    return __longlong_as_double(((long long)hi << 32) | lo);
}
// maximum over each row of 16 lanes (NaN ignored), in every lane: rotations by 8, 4, 2, 1
__device__ __forceinline__ double row_max(double v)
{
    v = fmax(v, dpp<0x128>(v));
    v = fmax(v, dpp<0x124>(v));
    v = fmax(v, dpp<0x122>(v));
    return fmax(v, dpp<0x121>(v));
}
__device__ __forceinline__ int row_min(int v)
{
    v = min(v, __builtin_amdgcn_update_dpp(0, v, 0x128, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(0, v, 0x124, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(0, v, 0x122, 0xf, 0xf, false));
    return min(v, __builtin_amdgcn_update_dpp(0, v, 0x121, 0xf, 0xf, false));
}
// maximum over the wave's 64 lanes, in every lane: the rows', then across odd and even
// rows and across halves (each swap of a register with itself gives both operands)
__device__ __forceinline__ double wave_max(double v)
{
    v = row_max(v);
    auto both = [](unsigned lo0, unsigned lo1, unsigned hi0, unsigned hi1) {
        return fmax(__longlong_as_double(((long long)hi0 << 32) | lo0),
                    __longlong_as_double(((long long)hi1 << 32) | lo1));
    };
    {
        const long long u = __double_as_longlong(v);
        const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)u, (unsigned)u, false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(u >> 32), (unsigned)(u >> 32), false, false);
        v = both(lo[0], lo[1], hi[0], hi[1]);
    }
    const long long u = __double_as_longlong(v);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)u, (unsigned)u, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(u >> 32), (unsigned)(u >> 32), false, false);
    return both(lo[0], lo[1], hi[0], hi[1]);
}

// Factors the panel of kb columns from column o + jo on (rows from o + jo on); the
// panel's columns are jo .. jo + kb - 1 of P.  Eight columns at a time are eliminated
// in registers (R rows per thread), then applied to the rest of the panel: the
// pivot search and the exchanges of a column cost two barriers and no memory access.
// The one-column-at-a-time elimination in global memory before this took most of the
// solve: each search read a strided column.
template <int R>
__global__ void __launch_bounds__(kEdgeThreads) k_lu_panel(LuArgs u, int o, int jo, int kb)
{
    constexpr int kT = kPanel + 1;
    __shared__ double tile[kPanel * kT];            // transposes
    __shared__ double slots[kOuter][2 * kSub + 1];  // a column's rows that an exchange touches
    __shared__ double U8[kPanel][kSub];
    __shared__ double L8[kSub][kSub];
    __shared__ double wmax[2][16];
    __shared__ int wrow[2][16];
    __shared__ double rows[2][2][kSub];             // pivot row, row k
    __shared__ int piv8[kSub], sid8[kSub];
    __shared__ int piv[kPanel], sid[kPanel], src[kOuter];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    if (u.bad[b]) return;
    const int n = u.n, m = n - o;                   // rows of P
    double* A = u.A + (size_t)b * n * u.ld;
    double* P = u.P + (size_t)b * kOuter * u.mp;

    // the panel's columns into P
    for (int r0 = jo; r0 < m; r0 += kPanel) {
        const int i = r0 + tid / 16;
        if (i < m)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int c = (tid & 15) + 16 * k;
                tile[(tid / 16) * kT + c] = c < kb ? A[(size_t)(o + i) * u.ld + o + jo + c] : 0.0;
            }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int c = wave + 16 * k;
            if (c < kb && r0 + lane < m) P[(size_t)(jo + c) * u.mp + r0 + lane] = tile[lane * kT + c];
        }
        __syncthreads();
    }

    for (int s = 0; s < kb; s += kSub) {
        const int w = min(kSub, kb - s);
        const int base = jo + s;                    // first active row, and column, of P
        double a[R][kSub];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = base + tid + kEdgeThreads * r;
#pragma unroll
            for (int k = 0; k < kSub; ++k) a[r][k] = (i < m && k < w) ? P[(size_t)(base + k) * u.mp + i] : 0.0;
        }
        bool stop = false;
#pragma unroll
        for (int k = 0; k < kSub; ++k) {
            if (k >= w) break;
            const int par = k & 1;
            // first row with the largest |a| in column k, from row k on
            double v = -1.0;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int q = tid + kEdgeThreads * r;
                if (q >= k && base + q < m) v = fmax(v, fabs(a[r][k]));
            }
            const double wm = wave_max(v);
            int q1 = INT_MAX;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int q = tid + kEdgeThreads * r;
                const unsigned long long hit =
                    __builtin_amdgcn_ballot_w64(q >= k && base + q < m && fabs(a[r][k]) == wm);
                if (hit && q1 == INT_MAX) q1 = kEdgeThreads * r + wave * kWave + (int)__builtin_ctzll(hit);
            }
            if (lane == 0) { wmax[par][wave] = wm; wrow[par][wave] = q1; }
            __syncthreads();
            const double bm = wmax[par][lane & 15];
            const double gm = row_max(bm);
            const int p = __builtin_amdgcn_readfirstlane(row_min(bm == gm ? wrow[par][lane & 15] : INT_MAX));
            if (p != INT_MAX)
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (tid + kEdgeThreads * r == p)
#pragma unroll
                        for (int c = 0; c < kSub; ++c) rows[par][0][c] = a[r][c];
            if (tid == k)
#pragma unroll
                for (int c = 0; c < kSub; ++c) rows[par][1][c] = a[0][c];
            if (tid == 0) piv8[k] = p;
            __syncthreads();
            const double pv = p == INT_MAX ? 0.0 : rows[par][0][k];
            if (!(pv != 0.0) || !std::isfinite(pv)) { stop = true; break; }
            double pr[kSub];
#pragma unroll
            for (int c = 0; c < kSub; ++c) pr[c] = rows[par][0][c];
            if (p != k) {
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (tid + kEdgeThreads * r == p)
#pragma unroll
                        for (int c = 0; c < kSub; ++c) a[r][c] = rows[par][1][c];
                if (tid == k)
#pragma unroll
                    for (int c = 0; c < kSub; ++c) a[0][c] = pr[c];
            }
            // multipliers, and the rank-1 update of the columns right of k
            const bool big = fabs(pv) >= 1e-290;    // its reciprocal is finite and normal
            const double ip = 1.0 / pv;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (tid + kEdgeThreads * r <= k) continue;
                const double l = big ? a[r][k] * ip : a[r][k] / pv;
                a[r][k] = l;
#pragma unroll
                for (int c = k + 1; c < kSub; ++c) a[r][c] -= l * pr[c];
            }
        }
        if (stop) {
            if (tid == 0) u.bad[b] = 1u;
            return;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = base + tid + kEdgeThreads * r;
#pragma unroll
            for (int k = 0; k < kSub; ++k)
                if (i < m && k < w) P[(size_t)(base + k) * u.mp + i] = a[r][k];
        }
        if (tid < kSub)
#pragma unroll
            for (int k = 0; k < kSub; ++k) L8[tid][k] = a[0][k];
        if (tid < w) {
            // slot of the row that step tid exchanged with: one of the first w rows, or
            // the first step that met the same row
            int sl = piv8[tid];
            if (sl >= w) {
                int first = tid;
                for (int t = tid - 1; t >= 0; --t)
                    if (piv8[t] == piv8[tid]) first = t;
                sl = kSub + first;
            }
            sid8[tid] = sl;
            piv[s + tid] = base + piv8[tid];
        }
        __syncthreads();
        // the exchanges in P's other columns, and U of the panel's columns right of
        // the eight: a thread per column
        if (tid < jo + kb && (tid < base || tid >= base + w)) {
            double* Pc = P + (size_t)tid * u.mp;
            double* x = slots[tid];
#pragma unroll
            for (int t = 0; t < kSub; ++t)
                if (t < w) {
                    x[t] = Pc[base + t];
                    if (sid8[t] == kSub + t) x[kSub + t] = Pc[base + piv8[t]];
                }
            for (int t = 0; t < w; ++t) {
                const int q = sid8[t];
                const double y = x[t];
                x[t] = x[q];
                x[q] = y;
            }
#pragma unroll
            for (int t = 0; t < kSub; ++t)
                if (t < w && sid8[t] == kSub + t) Pc[base + piv8[t]] = x[kSub + t];
            double y[kSub];
#pragma unroll
            for (int t = 0; t < kSub; ++t) y[t] = t < w ? x[t] : 0.0;
            if (tid >= base + w) {
#pragma unroll
                for (int t = 1; t < kSub; ++t)
#pragma unroll
                    for (int k = 0; k < t; ++k)
                        if (t < w) y[t] -= L8[t][k] * y[k];
#pragma unroll
                for (int t = 0; t < kSub; ++t) U8[tid - jo][t] = y[t];
            }
#pragma unroll
            for (int t = 0; t < kSub; ++t)
                if (t < w) Pc[base + t] = y[t];
        }
        __syncthreads();
        // the panel's columns right of the eight lose L U (w = 8 and a multiple of eight
        // columns whenever there are any, but for a ragged panel's last ones): eight
        // columns at a time, their loads in flight together
        for (int c0 = s + kSub; c0 < kb; c0 += kSub) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int q = tid + kEdgeThreads * r;
                if (q < kSub || base + q >= m) continue;
                double* e = P + (size_t)(jo + c0) * u.mp + base + q;
                double v[kSub];
#pragma unroll
                for (int c = 0; c < kSub; ++c) v[c] = c0 + c < kb ? e[(size_t)c * u.mp] : 0.0;
#pragma unroll
                for (int c = 0; c < kSub; ++c)
                    if (c0 + c < kb) {
                        double p = a[r][0] * U8[c0 + c][0];
#pragma unroll
                        for (int k = 1; k < kSub; ++k) p = fma(a[r][k], U8[c0 + c][k], p);
                        e[(size_t)c * u.mp] = v[c] - p;
                    }
            }
        }
        __syncthreads();
    }

    // U of the panel into A
    for (int e = tid; e < kb * kPanel; e += kEdgeThreads) {
        const int t = e / kPanel, c = e % kPanel;
        if (c >= t && c < kb) A[(size_t)(o + jo + t) * u.ld + o + jo + c] = P[(size_t)(jo + c) * u.mp + jo + t];
    }
    // all kb exchanges as one permutation of the rows they touch: slot t < 64 is panel
    // row t, slot 64 + t the row outside the panel that step t was the first to meet
    if (tid < kb) {
        int sl = piv[tid] - jo;
        if (sl >= kb) {
            int first = tid;
            for (int t = tid - 1; t >= 0; --t)
                if (piv[t] == piv[tid]) first = t;
            sl = kPanel + first;
        }
        sid[tid] = sl;
    }
    if (tid < kOuter) src[tid] = tid;
    __syncthreads();
    if (tid == 0)
        for (int t = 0; t < kb; ++t) {
            const int q = sid[t], y = src[t];
            src[t] = src[q];
            src[q] = y;
        }
    __syncthreads();
    if (tid < kb) {
        auto row_of = [&](int sl) { return o + (sl < kPanel ? jo + sl : piv[sl - kPanel]); };
        int32_t* pm = u.perm + (size_t)b * 3 * kPanel;
        pm[tid] = row_of(src[tid]);
        const bool ext = sid[tid] == kPanel + tid;
        pm[kPanel + tid] = ext ? row_of(kPanel + tid) : -1;
        pm[2 * kPanel + tid] = ext ? row_of(src[kPanel + tid]) : 0;
    }
}

// Columns c0 .. n right of the panel at column o + jo (kb columns): EXCH the panel's row
// exchanges, SOLVE U12 = L11^-1 A12.  One column per lane, its 64 panel rows in
// registers; L11 in LDS, read as broadcasts.  (L read through the scalar cache took
// 5 times as long: two CUs share 16 KB of it, and 64 values exceed the registers.)
template <bool EXCH, bool SOLVE>
__global__ void __launch_bounds__(256) k_lu_rows(LuArgs u, int o, int jo, int kb, int c0)
{
    __shared__ __align__(16) double Ls[SOLVE ? kPanel * kPanel : 1];   // [t][i]: column t of L11
    const int b = blockIdx.y;
    if (u.bad[b]) return;
    const int n = u.n;
    if (SOLVE) {
        const double* P = u.P + (size_t)b * kOuter * u.mp + (size_t)jo * u.mp + jo;
        for (int e = threadIdx.x; e < kPanel * kPanel; e += 256) {
            const int t = e / kPanel, i = e % kPanel;
            Ls[e] = (t < kb && i < kb) ? P[(size_t)t * u.mp + i] : 0.0;
        }
        __syncthreads();
    }
    const int c = c0 + blockIdx.x * 256 + threadIdx.x;
    if (c > n) return;
    const size_t ld = u.ld;
    double* A = u.A + (size_t)b * n * ld + c;
    const int32_t* pm = u.perm + (size_t)b * 3 * kPanel;
    double a[kPanel];
    if (EXCH) {
        double e[kPanel];
#pragma unroll
        for (int t = 0; t < kPanel; ++t) a[t] = t < kb ? A[(size_t)pm[t] * ld] : 0.0;
#pragma unroll
        for (int t = 0; t < kPanel; ++t) e[t] = (t < kb && pm[kPanel + t] >= 0) ? A[(size_t)pm[2 * kPanel + t] * ld] : 0.0;
#pragma unroll
        for (int t = 0; t < kPanel; ++t)
            if (t < kb && pm[kPanel + t] >= 0) A[(size_t)pm[kPanel + t] * ld] = e[t];
    } else {
#pragma unroll
        for (int t = 0; t < kPanel; ++t) a[t] = t < kb ? A[(size_t)(o + jo + t) * ld] : 0.0;
    }
    // eight rows at a time: among themselves one by one, the rows below by their sum
    [&]<int... G>(std::integer_sequence<int, G...>) {
        ([&] {
            constexpr int T0 = G * kSub;
            if (SOLVE && T0 < kb) {
#pragma unroll
                for (int t = T0; t < T0 + kSub; ++t)
#pragma unroll
                    for (int i = t + 1; i < T0 + kSub; ++i) a[i] -= Ls[t * kPanel + i] * a[t];
#pragma unroll
                for (int i = T0 + kSub; i < kPanel; ++i) {
                    double p = Ls[T0 * kPanel + i] * a[T0];
#pragma unroll
                    for (int t = T0 + 1; t < T0 + kSub; ++t) p = fma(Ls[t * kPanel + i], a[t], p);
                    a[i] -= p;
                }
            }
#pragma unroll
            for (int t = T0; t < T0 + kSub; ++t)
                if (t < kb) A[(size_t)(o + jo + t) * ld] = a[t];
        }(), ...);
    }(std::make_integer_sequence<int, kPanel / kSub>{});
}

// A[r][c] -= sum_{k < K} P[k][r] A[o + k][c] for rows r0 <= r < r1 and columns
// c0 <= c < c1: tiles of TM x TN by four waves, the operands of 16 k staged in LDS while
// the next 16 are on their way to registers, 16 x 16 x 4 FP64 matrix instructions.  The
// products are summed by themselves and then subtracted, here and in the panels and U12:
// with A as the accumulator each was rounded at the size of A, and systems of 65 to 585
// multiplets were solved 1.5 to 10 times less exactly (6PCF lmax 3, 252 systems: 86.0 ms,
// 84.3 with A as the accumulator, 100 with a wave's part of A read at once at the end).
// The LDS rows are 16 doubles longer than a multiple of 32, so that the two k rows a
// half-wave reads lie on different halves of the banks.  Tiles at the edge read L and U
// past the panel's rows and columns: those products land in rows and columns that are
// not stored.
constexpr int kGemmM = 128, kGemmK = 16;
template <int TM, int TN>
__global__ void __launch_bounds__(256, 2) k_lu_gemm(LuArgs u, int o, int K, int r0, int r1, int c0, int c1, int tx,
                                                    int tiles)
{
    constexpr int SA = TM + 16, SB = TN + 16;
    constexpr int WN = TN / 64, WM = 4 / WN;        // waves along columns and rows
    constexpr int MT = TM / WM / 16, NT = 4;        // 16 x 16 tiles of a wave
    constexpr int NA = kGemmK * TM / 512, NB = kGemmK * TN / 512;   // pairs a thread stages
    __shared__ __align__(16) double As[kGemmK * SA];
    __shared__ __align__(16) double Bs[kGemmK * SB];
    // every tile of one system on one XCD (workgroup i runs on XCD i % 8): they share
    // its L and U rows through that XCD's L2
    const int slot = blockIdx.x / 8;
    const int b = slot / tiles * 8 + (int)(blockIdx.x % 8);
    if (b >= u.nb || u.bad[b]) return;
    const int tile = slot % tiles;
    const int rt = r0 + tile / tx * TM, ct = c0 + tile % tx * TN;
    double* A = u.A + (size_t)b * u.n * u.ld;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int ka = tid / (TM / 2), ra = tid % (TM / 2) * 2, kc = tid / (TN / 2), cc = tid % (TN / 2) * 2;
    const double* P = u.P + (size_t)b * kOuter * u.mp + (rt - o) + (size_t)ka * u.mp + ra;
    const double* Ur = A + (size_t)(o + kc) * u.ld + ct + cc;
    const int wm = wave / WN, wn = wave % WN;
    const int li = lane & 15, lk = lane >> 4;
    const int rw = rt + wm * MT * 16 + lk, cw = ct + wn * 64 + li;   // the lane's first row and column
    auto row = [&](int i, int q) { return rw + 16 * i + 4 * q; };
    auto col = [&](int j) { return cw + 16 * j; };
    // a system is below 2^32 bytes: 32-bit offsets from its base
    auto at = [&](int r, int c) {
        return reinterpret_cast<double*>(reinterpret_cast<char*>(A) + (unsigned)(r * u.ld + c) * 8u);
    };
    d2 pa[NA], pb[NB];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int e = 0; e < NA; ++e)
            pa[e] = *reinterpret_cast<const d2*>(P + (size_t)(k0 + e * (512 / TM)) * u.mp);
#pragma unroll
        for (int e = 0; e < NB; ++e)
            pb[e] = *reinterpret_cast<const d2u*>(Ur + (size_t)(k0 + e * (512 / TN)) * u.ld);
    };
    fetch(0);
    d4 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[i][j][q] = 0.0;
    for (int k0 = 0; k0 < K; k0 += kGemmK) {
        __syncthreads();
#pragma unroll
        for (int e = 0; e < NA; ++e)
            *reinterpret_cast<d2*>(&As[(ka + e * (512 / TM)) * SA + ra]) = pa[e];
#pragma unroll
        for (int e = 0; e < NB; ++e) *reinterpret_cast<d2*>(&Bs[(kc + e * (512 / TN)) * SB + cc]) = pb[e];
        __syncthreads();
        if (k0 + kGemmK < K) fetch(k0 + kGemmK);
#pragma unroll
        for (int k = 0; k < kGemmK; k += 4) {
            double x[MT], y[NT];
#pragma unroll
            for (int i = 0; i < MT; ++i) x[i] = As[(k + lk) * SA + wm * MT * 16 + i * 16 + li];
#pragma unroll
            for (int j = 0; j < NT; ++j) y[j] = Bs[(k + lk) * SB + wn * 64 + j * 16 + li];
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[i], y[j], acc[i][j], 0, 0, 0);
        }
    }
    // A of one row of tiles, on its way while the row before is stored
    d4 old[2][NT];
    auto load = [&](int i) {
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                old[i & 1][j][q] = (row(i, q) < r1 && col(j) < c1) ? *at(row(i, q), col(j)) : 0.0;
    };
    load(0);
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        if (i + 1 < MT) load(i + 1);
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (row(i, q) < r1 && col(j) < c1) *at(row(i, q), col(j)) = old[i & 1][j][q] - acc[i][j][q];
    }
}

// Back substitution on U, 64 unknowns at a time: wave 0 solves their triangle, then
// every row above loses its 64 products (8 lanes per row).  Writes the kept multiplets.
__global__ void __launch_bounds__(kEdgeThreads) k_lu_back(LuArgs u, const int32_t* __restrict__ keep, int nout,
                                                          double* __restrict__ zeta, int B_lo, int nB,
                                                          unsigned* __restrict__ nbad)
{
    extern __shared__ double x[];                   // [n]
    __shared__ double Ub[kPanel][kPanel + 1];
    __shared__ double xb[kPanel];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & (kWave - 1);
    const int n = u.n;
    const double* A = u.A + (size_t)b * n * u.ld;
    const bool bad = u.bad[b] != 0;
    if (!bad) {
        for (int i = tid; i < n; i += kEdgeThreads) x[i] = A[(size_t)i * u.ld + n];
        for (int k0 = (n - 1) / kPanel * kPanel; k0 >= 0; k0 -= kPanel) {
            const int kb = min(kPanel, n - k0);
            for (int e = tid; e < kPanel * kPanel; e += kEdgeThreads) {
                const int i = e / kPanel, c = e % kPanel;
                Ub[i][c] = (i < kb && c < kb && c >= i) ? A[(size_t)(k0 + i) * u.ld + k0 + c] : 0.0;
            }
            __syncthreads();
            if (tid < kWave) {
                double v = lane < kb ? x[k0 + lane] : 0.0;
                for (int k = kb - 1; k >= 0; --k) {
                    const double xk = __shfl(v, k) / Ub[k][k];
                    if (lane == k) v = xk;
                    else if (lane < k) v -= Ub[lane][k] * xk;
                }
                xb[lane] = v;
                if (lane < kb) x[k0 + lane] = v;
            }
            __syncthreads();
            const int sub = tid & 7;
            for (int r = tid / 8; r < k0; r += kEdgeThreads / 8) {
                double s = 0.0;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const int c = sub + 8 * k;
                    if (c < kb) s += A[(size_t)r * u.ld + k0 + c] * xb[c];
                }
                s += __shfl_xor(s, 1);
                s += __shfl_xor(s, 2);
                s += __shfl_xor(s, 4);
                if (sub == 0) x[r] -= s;
            }
            __syncthreads();
        }
    }
    for (int i = tid; i < nout; i += kEdgeThreads) zeta[(size_t)i * nB + B_lo + b] = bad ? NAN : x[keep[i]];
    if (tid == 0 && bad) atomicAdd(nbad, 1u);
}

// Systems of up to kSmall multiplets whole, a wave each, matrix and right-hand side in
// LDS, instead of the steps above, whose 6 launches of a few us were most of a small
// call (device time, steps above / here / one workgroup per system in global memory:
// 3PCF lmax 10, 10 bins, 11 multiplets 0.062 / 0.018 / 0.044 ms; 6PCF lmax 1, 16 bins, 26
// multiplets x 4,368 systems 1.47 / 0.08 / 1.98).  A lane per row up to 32 rows.
__global__ void __launch_bounds__(kWave) k_edge_small(const double* __restrict__ A0, int n, int ld,
                                                      const double* __restrict__ nmult,
                                                      const double* __restrict__ rmult, int B_lo, int nB,
                                                      const int32_t* __restrict__ keep, int nout,
                                                      double* __restrict__ zeta, unsigned* __restrict__ nbad)
{
    __shared__ double a[kSmall][kSmall + 1];        // column n: the right-hand side
    __shared__ double xs[kSmall];
    const int b = blockIdx.x, lane = threadIdx.x, B = B_lo + b;
    const double* A = A0 + (size_t)b * n * ld;
    const double r0 = rmult[B];
    bool bad = !(r0 != 0.0) || !std::isfinite(r0);
    for (int e = lane; e < n * n; e += kWave) {     // the part above the diagonal, as k_edge_mirror
        const int i = e / n, c = e - i * n;
        a[i][c] = A[(size_t)min(i, c) * ld + max(i, c)];
    }
    if (lane < n) a[lane][n] = nmult[(size_t)lane * nB + B] / r0;
    __syncthreads();
    for (int k = 0; k < n && !bad; ++k) {
        const bool in = lane >= k && lane < n;
        const double v = in ? fabs(a[lane][k]) : -1.0;
        const double wm = wave_max(v);
        const unsigned long long hit = __builtin_amdgcn_ballot_w64(in && v == wm);
        const int p = hit ? (int)__builtin_ctzll(hit) : k;
        const double pv = a[p][k];
        bad = !hit || !(pv != 0.0) || !std::isfinite(pv);
        if (bad) break;
        if (p != k && lane >= k && lane <= n) {
            const double y = a[k][lane];
            a[k][lane] = a[p][lane];
            a[p][lane] = y;
        }
        __syncthreads();
        if (lane > k && lane < n) {
            const double l = a[lane][k] / pv;
            for (int c = k + 1; c <= n; ++c) a[lane][c] -= l * a[k][c];
        }
        __syncthreads();
    }
    double x = lane < n ? a[lane][n] : 0.0;
    for (int k = n - 1; k >= 0 && !bad; --k) {
        const double xk = __shfl(x, k) / a[k][k];
        if (lane == k) x = xk;
        else if (lane < k) x -= a[lane][k] * xk;
    }
    if (lane < n) xs[lane] = x;
    __syncthreads();
    for (int i = lane; i < nout; i += kWave) zeta[(size_t)i * nB + B] = bad ? NAN : xs[keep[i]];
    if (lane == 0 && bad) atomicAdd(nbad, 1u);
}

template <int TM, int TN>
int launch_lu_gemm(const LuArgs& u, int o, int K, int r0, int r1, int c0, int c1, hipStream_t s)
{
    if (r0 >= r1 || c0 >= c1) return (int)hipSuccess;
    const int tx = (c1 - c0 + TN - 1) / TN, ty = (r1 - r0 + TM - 1) / TM;
    const int64_t blocks = (int64_t)(u.nb + 7) / 8 * 8 * tx * ty;
    k_lu_gemm<TM, TN><<<dim3((unsigned)blocks), dim3(256), 0, s>>>(u, o, K, r0, r1, c0, c1, tx, tx * ty);
    return (int)hipGetLastError();
}

int launch_lu_panel(const LuArgs& u, int o, int jo, int kb, hipStream_t s)
{
    const dim3 g((unsigned)u.nb), t(kEdgeThreads);
    const int rows = u.n - o - jo;
    if (rows <= kEdgeThreads) k_lu_panel<1><<<g, t, 0, s>>>(u, o, jo, kb);
    else if (rows <= 2 * kEdgeThreads) k_lu_panel<2><<<g, t, 0, s>>>(u, o, jo, kb);
    else if (rows <= 3 * kEdgeThreads) k_lu_panel<3><<<g, t, 0, s>>>(u, o, jo, kb);
    else return (int)hipErrorInvalidValue;
    return (int)hipGetLastError();
}

template <bool EXCH, bool SOLVE>
int launch_lu_rows(const LuArgs& u, int o, int jo, int kb, hipStream_t s)
{
    const int c0 = o + jo + kb;   // up to the right-hand side, column n
    const dim3 g((unsigned)((u.n - c0) / 256 + 1), (unsigned)u.nb), t(256);
    k_lu_rows<EXCH, SOLVE><<<g, t, 0, s>>>(u, o, jo, kb, c0);
    return (int)hipGetLastError();
}

#define LUTRY(x)                             \
    do {                                     \
        const int e__ = (x);                 \
        if (e__ != (int)hipSuccess) return e__; \
    } while (0)

int launch_lu(const LuArgs& u, hipStream_t s)
{
    const int n = u.n;
    for (int o = 0; o < n; o += kOuter) {
        const int ka = std::min(kPanel, n - o);
        LUTRY(launch_lu_panel(u, o, 0, ka, s));
        LUTRY((launch_lu_rows<true, true>(u, o, 0, ka, s)));
        const int j = o + kPanel;
        if (j >= n) break;
        const int kb = std::min(kPanel, n - j);
        LUTRY((launch_lu_gemm<128, 64>(u, o, kPanel, j, n, j, j + kb, s)));
        LUTRY(launch_lu_panel(u, o, kPanel, kb, s));
        LUTRY((launch_lu_rows<true, false>(u, o, kPanel, kb, s)));
        LUTRY((launch_lu_gemm<64, 128>(u, o, kPanel, j, j + kb, j + kb, n + 1, s)));
        LUTRY((launch_lu_rows<false, true>(u, o, kPanel, kb, s)));
        if (o + kOuter >= n) break;
        LUTRY((launch_lu_gemm<128, 128>(u, o, kOuter, o + kOuter, n, o + kOuter, n + 1, s)));
    }
    return (int)hipSuccess;
}

}  // namespace

int edge_ld(int n) { return (n + 1 + 15) / 16 * 16; }

size_t edge_matrix_bytes(int n, int nb)
{
    // one tile past the last row and column may be read
    return sizeof(double) * ((size_t)nb * n * edge_ld(n) + kGemmM + 16);
}

size_t edge_panel_bytes(int n, int nb) { return sizeof(double) * (size_t)nb * kOuter * ((n + 15) / 16 * 16 + kGemmM); }

size_t edge_perm_bytes(int nb) { return (sizeof(int32_t) * 3 * kPanel + sizeof(unsigned)) * (size_t)nb; }

int launch_edge_ell(int n, const int64_t* row_start, const int32_t* term_lp, const double* term_val,
                    const int64_t* ell_off, uint16_t* lp, double* val, hipStream_t stream)
{
    const int64_t units = (int64_t)n * ((n + kWave - 1) / kWave);
    k_edge_ell<<<dim3((unsigned)((units + 3) / 4)), dim3(256), 0, stream>>>(n, row_start, term_lp, term_val, ell_off, lp,
                                                                         val);
    return (int)hipGetLastError();
}

int launch_edge(const EdgeArgs& a, int B_lo, int nb, hipStream_t stream)
{
    if (nb == 0 || a.nlam == 0) return (int)hipSuccess;
    if (a.nlam > kEdgeMaxMultiplets) return (int)hipErrorInvalidValue;
    // eight bin tuples per block while their f tables fit the LDS, else four
    LUTRY((a.nlam + 1) * 8 * sizeof(double) <= 150 * 1024 ? launch_edge_matrix<8>(a, B_lo, nb, stream)
                                                    : launch_edge_matrix<4>(a, B_lo, nb, stream));
    if (a.nlam <= kSmall) {
        k_edge_small<<<dim3((unsigned)nb), dim3(kWave), 0, stream>>>(a.A, a.nlam, a.ld, a.nmult, a.rmult, B_lo, a.nB,
                                                                    a.keep, a.nout, a.zeta, a.nbad);
        return (int)hipGetLastError();
    }
    LuArgs u;
    u.n = a.nlam;
    u.ld = a.ld;
    u.mp = (a.nlam + 15) / 16 * 16 + kGemmM;
    u.nb = nb;
    u.A = a.A;
    u.P = a.P;
    u.perm = a.perm;
    u.bad = reinterpret_cast<unsigned*>(a.perm + (size_t)nb * 3 * kPanel);
    k_lu_rhs<<<dim3((unsigned)nb), dim3(256), 0, stream>>>(u, a.nmult, a.rmult, B_lo, a.nB);
    LUTRY((int)hipGetLastError());
    LUTRY(launch_lu(u, stream));
    LUTRY((int)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_lu_back), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)(sizeof(double) * kEdgeMaxMultiplets)));
    k_lu_back<<<dim3((unsigned)nb), dim3(kEdgeThreads), sizeof(double) * (size_t)a.nlam, stream>>>(
        u, a.keep, a.nout, a.zeta, B_lo, a.nB, a.nbad);
    return (int)hipGetLastError();
}

}  // namespace encore

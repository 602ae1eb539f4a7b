// Coupling step (eq. NPCF-mult-discrete-binned-estimator with the Appendix B half
// sum), reassociated so that the sum over primaries comes first:
//
//   T[t][B]  = sum_i w_i Q_t[ prod_k a~^{b_k}_{l_k m_k}(i) ]          (k_couple)
//   Z[L][B]  = sum_{terms (L, t)} 2 S(m_{N-1}) E(L) C^L_M  T[t][B]      (k_contract)
//
// t runs over the distinct (l_k, m_k)_k tuples with m_{N-1} >= 0 that carry a
// nonzero coupling; Q_t is Re for parity-even and Im for parity-odd tuples.  The
// identity is exact in real arithmetic (the coupling does not depend on i).
// a~ for m < 0 comes from a~_{l,-m} = (-1)^m conj(a~_{l,m}) (Appendix B).
//
// k_couple: one thread per (t, B) output, FP64 accumulator; the block stages a tile
// of primaries' coefficients in LDS and every thread walks the tile.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <utility>

#include "device.h"

namespace encore {

namespace {

constexpr int kBlock = 256;
constexpr int kMaxK = 5;

template <typename T> struct C2;
template <> struct C2<float> { using type = float2; };
template <> struct C2<double> { using type = double2; };

template <typename T, int NK>
__global__ void __launch_bounds__(kBlock) k_couple(CoupleArgs a, int ptile)
{
    using V = typename C2<T>::type;
    extern __shared__ __align__(16) unsigned char smem[];
    V* tile = reinterpret_cast<V*>(smem);
    const int per = a.nbins * a.nlm;                       // complex values per primary
    double* wtile = reinterpret_cast<double*>(smem + sizeof(V) * (size_t)ptile * per);

    const int64_t gid = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const bool valid = gid < (int64_t)a.ntuple * a.nB;
    const int t = valid ? (int)(gid / a.nB) : 0;
    const int b = valid ? (int)(gid - (int64_t)t * a.nB) : 0;
    const int split = blockIdx.y;
    const int p_lo = a.split_lo[split];
    const int p_hi = a.split_hi[split];

    int off[NK];
    T cs[NK];
    int flags = 0;
#pragma unroll
    for (int k = 0; k < NK; ++k) { off[k] = 0; cs[k] = (T)1; }
    if (valid) {
        flags = a.tuple_flags[t];
#pragma unroll
        for (int k = 0; k < NK; ++k) {
            off[k] = a.btab[b * a.nk + k] * a.nlm + a.tuple_off[t * a.nk + k];
            cs[k] = ((flags >> k) & 1) ? (T)-1 : (T)1;
        }
    }
    const bool take_im = (flags >> 16) & 1;
    double acc = 0.0;

    for (int p0 = p_lo; p0 < p_hi; p0 += ptile) {
        const int np = min(ptile, p_hi - p0);
        __syncthreads();
        const V* src = reinterpret_cast<const V*>(a.alm) + (size_t)p0 * per;
        for (int q = threadIdx.x; q < np * per; q += kBlock) tile[q] = src[q];
        for (int q = threadIdx.x; q < np; q += kBlock) wtile[q] = a.wprim[p0 + q];
        __syncthreads();
        if (valid) {
            for (int pp = 0; pp < np; ++pp) {
                const V* ap = tile + pp * per;
                V v = ap[off[0]];
                T pr = v.x, pi = cs[0] * v.y;
#pragma unroll
                for (int k = 1; k < NK; ++k) {
                    const V u = ap[off[k]];
                    const T ur = u.x, ui = cs[k] * u.y;
                    const T nr = pr * ur - pi * ui;
                    const T ni = pr * ui + pi * ur;
                    pr = nr; pi = ni;
                }
                const T q = take_im ? pi : pr;
                acc += wtile[pp] * (double)q;
            }
        }
    }
    if (valid) {
        if ((flags >> 8) & 1) acc = -acc;
        a.T[((size_t)split * a.ntuple + t) * a.nB + b] = acc;
    }
}

// 4PCF: one block per (256 tuples, first bin b1, primary split).  For each primary each
// thread loads a~^{b1} of its first factor, the second factor's a~^{b2} and the third
// factor's a~^{b3} once each, forms P = w a1 a2 once per b2 and adds Q[P a3] for every
// b3 > b2: about one product per output and primary instead of k_couple's three.
// TI: the coefficients' type, TC: that of the products.  TILED (10 bins): the sums over a
// tile of primaries are added to the FP64 sums, so that a split's thousands of terms are
// not rounded one by one at the size of their sum; otherwise the terms are added to the
// FP64 sums directly, over splits as couple_split_rows cuts them.  Bound by FP64 issue and
// the LDS reads alike at b1 = 0 (17 reads of 16 bytes for 104 multiply-adds).  With the
// products as multiply-adds into the sums, and several b1 per launch, 10 bins at lmax 5
// over 60k primaries take 2.96 ms in FP64 (3.53 with products, then sums; 2.53 without
// tiles, whose sums are rounded 2 to 3 times as far).
constexpr int kNB4 = 10;
constexpr int kNB4Max = 12;   // its 55 FP64 sums and 2 x 12 coefficients per thread fit the registers
__host__ __device__ constexpr int pair_count(int nr) { return (nr - 1) * (nr - 2) / 2; }   // b1 < b2 < b3 of nr bins

template <typename TI, typename TC, bool TILED, int NR>
__device__ __forceinline__ void couple4_bins(const CoupleArgs& a, int ptile, int t, unsigned char* smem)
{
    using V = typename C2<TI>::type;
    constexpr int NA = pair_count(NR);
    const int B1 = a.nbins - NR;
    V* tile = reinterpret_cast<V*>(smem);
    const int per = NR * a.nlm;                           // staged complex values per primary
    double* wtile = reinterpret_cast<double*>(smem + sizeof(V) * (size_t)ptile * per);

    const bool valid = t < a.ntuple;
    const int split = blockIdx.y;
    const int p_lo = a.split_lo[split];
    const int p_hi = a.split_hi[split];

    int lm0 = 0, lm1 = 0, lm2 = 0, flags = 0;
    if (valid) {
        lm0 = a.tuple_off[t * 3 + 0];
        lm1 = a.tuple_off[t * 3 + 1];
        lm2 = a.tuple_off[t * 3 + 2];
        flags = a.tuple_flags[t];
    }
    const TC c0 = (flags & 1) ? (TC)-1 : (TC)1;
    const TC c1 = (flags & 2) ? (TC)-1 : (TC)1;
    const TC c2 = (flags & 4) ? (TC)-1 : (TC)1;
    const bool take_im = (flags >> 16) & 1;

    double acc[NA];
    TC part[TILED ? NA : 1];
#pragma unroll
    for (int q = 0; q < NA; ++q) acc[q] = 0.0;

    for (int p0 = p_lo; p0 < p_hi; p0 += ptile) {
        const int np = min(ptile, p_hi - p0);
        __syncthreads();
        // stage bins B1 .. nbins - 1 of each primary of the tile
        const V* src = reinterpret_cast<const V*>(a.alm);
        const int full = a.nbins * a.nlm;
        for (int q = threadIdx.x; q < np * per; q += kBlock) {
            const int pp = q / per, r = q - pp * per;
            tile[q] = src[(size_t)(p0 + pp) * full + B1 * a.nlm + r];
        }
        for (int q = threadIdx.x; q < np; q += kBlock) wtile[q] = a.wprim[p0 + q];
        __syncthreads();
        if constexpr (TILED)
#pragma unroll
            for (int q = 0; q < NA; ++q) part[q] = (TC)0;
        if (valid) {
            for (int pp = 0; pp < np; ++pp) {
                const V* ap = tile + pp * per;
                const TC w = (TC)wtile[pp];
                const V v0 = ap[lm0];
                const TC a1r = w * (TC)v0.x, a1i = w * (c0 * (TC)v0.y);
                TC u3r[NR], u3i[NR];
#pragma unroll
                for (int b = 2; b < NR; ++b) {
                    const V u = ap[b * a.nlm + lm2];
                    u3r[b] = (TC)u.x; u3i[b] = c2 * (TC)u.y;
                }
                int q = 0;
#pragma unroll
                for (int b2 = 1; b2 < NR - 1; ++b2) {
                    const V u = ap[b2 * a.nlm + lm1];
                    const TC ur = (TC)u.x, ui = c1 * (TC)u.y;
                    TC pr = a1r * ur - a1i * ui;
                    TC pi = a1r * ui + a1i * ur;
                    if (take_im) { const TC tmp = pr; pr = pi; pi = -tmp; }   // Im(z) = Re(-i z)
#pragma unroll
                    for (int b3 = b2 + 1; b3 < NR; ++b3) {
                        if constexpr (sizeof(TC) == 4) part[q] += pr * u3r[b3] - pi * u3i[b3];
                        else if constexpr (TILED) part[q] = fma(-pi, u3i[b3], fma(pr, u3r[b3], part[q]));
                        else acc[q] = fma(-pi, u3i[b3], fma(pr, u3r[b3], acc[q]));
                        ++q;
                    }
                }
            }
        }
        if constexpr (TILED)
#pragma unroll
            for (int q = 0; q < NA; ++q) acc[q] += (double)part[q];
    }
    if (valid) {
        const double sgn = ((flags >> 8) & 1) ? -1.0 : 1.0;
        // B index of (B1, b2, b3): tuples with first bin < B1 come first
        int bidx = 0;
        for (int b = 0; b < B1; ++b) bidx += pair_count(a.nbins - b);
        double* dst = a.T + ((size_t)split * a.ntuple + t) * a.nB + bidx;
#pragma unroll
        for (int q = 0; q < NA; ++q) dst[q] = sgn * acc[q];
    }
}

// the first bins b1 = nbins - nr of nr = NRLO .. NRHI, the one with the most tuples of
// bins first
template <typename TI, typename TC, bool TILED, int NRLO, int NRHI>
__global__ void __launch_bounds__(kBlock) k_couple4(CoupleArgs a, int ptile, int tblocks, int nr_first)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int j = blockIdx.x / tblocks;
    const int t = (blockIdx.x - j * tblocks) * kBlock + threadIdx.x;
    const int nr = nr_first - j;                          // uniform over the block
    [&]<int... R>(std::integer_sequence<int, R...>) {
        ((nr == R + NRLO ? couple4_bins<TI, TC, TILED, R + NRLO>(a, ptile, t, smem) : (void)0), ...);
    }(std::make_integer_sequence<int, NRHI - NRLO + 1>{});
}

__global__ void __launch_bounds__(kBlock) k_contract(ContractArgs a)
{
    const int64_t gid = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (gid >= (int64_t)a.nlam * a.nB) return;
    const int l = (int)(gid / a.nB);
    const int b = (int)(gid - (int64_t)l * a.nB);
    double z = 0.0;
    for (int q = a.term_start[l]; q < a.term_start[l + 1]; ++q) {
        const int t = a.term_tuple[q];
        double s = 0.0;
        if (a.tmap) {
            const int32_t mv = a.tmap[(size_t)t * a.nB + b];
            s = a.T[mv & 0x7fffffff];
            if (mv < 0) s = -s;
        } else {
            for (int sp = 0; sp < a.nsplit; ++sp) s += a.T[((size_t)sp * a.ntuple + t) * a.nB + b];
        }
        z += a.term_coef[q] * s;
    }
    if (a.bscale) z *= a.bscale[b];
    a.zeta[gid] = z;
}

}  // namespace

// k_couple4 couples this job: up to 12 bins, and with enough tuples that its blocks,
// whose lanes are tuples, are not mostly idle (4PCF, 60k primaries, k_couple / k_couple4
// in ms: FP64 lmax 3 8 bins 0.64 / 0.39, lmax 5 8 bins 5.0 / 1.45, 12 bins 25.1 / 5.5;
// FP32 path lmax 4 6 bins 0.56 / 0.49).  10 bins always, where k_couple took longer at
// every lmax.
static bool use_couple4(int nk, int nbins, int64_t ntuple, int64_t nB)
{
    return nk == 3 && nbins >= 3 &&
           (nbins == kNB4 || (nbins <= kNB4Max && ntuple >= 128 && ntuple * nB >= 8192));
}

int couple_split_rows(int nk, int nbins, int64_t ntuple, int64_t nB, int64_t nrows)
{
    auto rows_of = [&](int64_t ns, int64_t least) {
        ns = std::max<int64_t>(1, std::min<int64_t>(ns, 1024));
        return std::max<int64_t>(least, (nrows + ns - 1) / ns);
    };
    const int64_t ns = (int64_t)(1 << 20) / std::max<int64_t>(ntuple * nB, 1);
    if (!use_couple4(nk, nbins, ntuple, nB)) return (int)rows_of(ns, 64);
    // one block per (b1, 256 tuples, split): aim at ~1024 blocks per b1
    const int64_t tblocks = (ntuple + kBlock - 1) / kBlock;
    const int64_t want = (1024 + tblocks - 1) / std::max<int64_t>(tblocks, 1);
    if (nbins == kNB4) return (int)rows_of(want, 64);
    // Bin counts without tiles of primaries: a split's sum and the sum over the splits
    // round least when both are sqrt(nrows) long, and no more than k_couple's would
    // up to as many splits as those have rows: the former, or within the latter as many
    // as make 1024 blocks (FP32 path, 9 bins, lmax 3, 8k primaries: 0.106 ms, k_couple
    // 0.130), and no more than 64 MiB of partial sums.
    const int64_t few = std::min(rows_of(ns, 64), 1024 / (tblocks * (nbins - 2)) + 1);
    const int64_t most = std::min(want, ((int64_t)64 << 20) / (8 * ntuple * nB));
    return (int)rows_of(std::max(ns, std::min(most, std::max((int64_t)std::sqrt((double)nrows), few))), 32);
}

__global__ void k_reduce(ReduceArgs a)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int r = blockIdx.y;
    if (i >= a.per) return;
    // left fold from the running total, split by split in row order: the same
    // association however the job's splits were distributed over slices
    double* dst = a.dst[r] + i;
    double s = *dst;
    for (int y = a.red_lo[r]; y < a.red_hi[r]; ++y) s += a.T[(size_t)y * a.per + i];
    *dst = s;
}

int launch_reduce(const ReduceArgs& a, hipStream_t stream)
{
    if (a.nred == 0 || a.per == 0) return (int)hipSuccess;
    k_reduce<<<dim3((unsigned)((a.per + kBlock - 1) / kBlock), (unsigned)a.nred), kBlock, 0, stream>>>(a);
    return (int)hipGetLastError();
}

int couple_ptile(int nbins, int nlm, int precision)
{
    const int per = nbins * nlm * (precision == 0 ? 16 : 8) + 8;
    int pt = 32768 / per;
    return pt < 1 ? 1 : (pt > 64 ? 64 : pt);
}

template <typename TI, typename TC, bool TILED, int NRLO, int NRHI>
int launch4(const CoupleArgs& a, hipStream_t stream)
{
    const int hi = std::min(NRHI, a.nbins);
    if (hi < NRLO) return (int)hipSuccess;
    const int ptile = std::max(1, std::min(64, 32768 / (a.nbins * a.nlm * (int)sizeof(typename C2<TI>::type) + 8)));
    const int tblocks = (a.ntuple + kBlock - 1) / kBlock;
    const size_t lds = (size_t)ptile * hi * a.nlm * sizeof(typename C2<TI>::type) + 8 * (size_t)ptile;
    k_couple4<TI, TC, TILED, NRLO, NRHI><<<dim3((unsigned)(tblocks * (hi - NRLO + 1)), (unsigned)a.nsplit), kBlock, lds,
                                    stream>>>(a, ptile, tblocks, hi);
    return (int)hipGetLastError();
}

// Several first bins share a launch so that no launch's end leaves the chip idle for
// long; the register use of a launch is that of its largest, which keeps the largest
// apart at 10 bins (4PCF lmax 5, 60k primaries, ms: FP64 {8..10} in one launch 3.08, {10}
// alone 2.96; FP32 2.30, 2.07).  Other counts, with one set of sums, take one launch (8
// bins 1.45, in two launches 1.59; FP32 path, 4k primaries, lmax 3, 9 bins 0.081, 0.104).
template <typename T>
int launch4_tiled(const CoupleArgs& a, hipStream_t stream)   // 10 bins
{
    int rc = launch4<T, T, true, kNB4, kNB4>(a, stream);
    if (rc == (int)hipSuccess) rc = launch4<T, T, true, 8, 9>(a, stream);
    return rc != (int)hipSuccess ? rc : launch4<T, T, true, 3, 7>(a, stream);
}
template <typename TI>
int launch4_fp64(const CoupleArgs& a, hipStream_t stream)    // other bin counts
{
    return a.nbins > kNB4 ? launch4<TI, double, false, 3, kNB4Max>(a, stream)
                          : launch4<TI, double, false, 3, kNB4 - 1>(a, stream);
}

int launch_couple(const CoupleArgs& a, int precision, hipStream_t stream)
{
    if (a.nk > kMaxK) return (int)hipErrorInvalidValue;
    if (a.nsplit == 0 || a.ntuple == 0) return (int)hipSuccess;
    if (use_couple4(a.nk, a.nbins, a.ntuple, a.nB)) {
        // The FP32 products of 10 bins are summed in FP32 over a tile of primaries (2.07 ms
        // at lmax 5 over 60k primaries, 2.96 for FP64 products and sums).  At other bin
        // counts, where k_couple added each FP32 product to an FP64 sum, the products are
        // formed in FP64 too: a conversion and an addition in FP64 for each FP32 product
        // would issue as long as the two FP64 multiply-adds.
        if (a.nbins == kNB4)
            return precision == 0 ? launch4_tiled<double>(a, stream) : launch4_tiled<float>(a, stream);
        return precision == 0 ? launch4_fp64<double>(a, stream) : launch4_fp64<float>(a, stream);
    }
    const int64_t nthreads = (int64_t)a.ntuple * a.nB;
    const int64_t nblk = (nthreads + kBlock - 1) / kBlock;
    if (nblk == 0) return (int)hipSuccess;
    const int ptile = couple_ptile(a.nbins, a.nlm, precision);
    const size_t lds = (size_t)ptile * a.nbins * a.nlm * (precision == 0 ? 16 : 8) + 8 * (size_t)ptile;
    dim3 grid((unsigned)nblk, (unsigned)a.nsplit);
#define ENCORE_COUPLE_CASE(NKV)                                                      \
    case NKV:                                                                        \
        if (precision == 0)                                                          \
            k_couple<double, NKV><<<grid, kBlock, lds, stream>>>(a, ptile);          \
        else                                                                         \
            k_couple<float, NKV><<<grid, kBlock, lds, stream>>>(a, ptile);           \
        break;
    switch (a.nk) {
        ENCORE_COUPLE_CASE(2)
        ENCORE_COUPLE_CASE(3)
        ENCORE_COUPLE_CASE(4)
        ENCORE_COUPLE_CASE(5)
    default: return (int)hipErrorInvalidValue;
    }
#undef ENCORE_COUPLE_CASE
    return (int)hipGetLastError();
}

int launch_contract(const ContractArgs& a, hipStream_t stream)
{
    const int64_t n = (int64_t)a.nlam * a.nB;
    if (n == 0) return (int)hipSuccess;
    k_contract<<<(unsigned)((n + kBlock - 1) / kBlock), kBlock, 0, stream>>>(a);
    return (int)hipGetLastError();
}

}  // namespace encore

// mtpt_device.h -- device code of the MTPT step for gfx950 (wave64): the
// helpers, the phase bodies and the tiled mass-transfer kernels, shared by
// the translation units that instantiate them (mtpt_kernels.hip: binning,
// exports and the host launchers; mtpt_tiles_*.hip: the two tiled passes per
// dimension and metric, compiled in parallel).
//
// One step of the method (Schauer et al., arXiv 2204.03756, Sec. 3) runs as:
//   bin        random walk + reflection (Sec. 3 random-walk update, zero-flux
//              walls), cell id of the walked position, cell histogram
//   scan       exclusive scan of the histogram -> cell offsets
//   scatter    slot of every particle inside its cell
//   place      rank inside the cell by (x, pid), gather positions, masses and
//              pids into that slot: the layout, and with it every
//              floating-point sum, does not depend on the order of atomics
//   rowsum     s_i = sum_j K_ij, K_ii = 1 included (Eq. (2)-(3) without the
//              prefactor, which cancels in W)
//   transfer   W_ij = 2 K_ij / (s_i + s_j), M_i' = M_i + beta sum_j W_ij (M_j - M_i)
//              (Eq. (4)-(5)), optional A+B->C epilogue, per-workgroup mass sums
//   finalize   FP64 totals and pair counters, summed in a fixed order
// The K-D tree search of the paper is replaced by the cell list (cell side
// >= the cutoff's reach along each axis).  The two mass-transfer passes run
// per tile of cells: the workgroup stages the positions (and row sums) of
// every cell row of the tile and its one-cell halo in LDS -- each such row is
// one contiguous, x-sorted run of the sorted arrays -- and every particle
// scans its 3^(d-1) neighbouring rows (trimmed to its x-window where rows are
// long).  With a dispersion tensor the distance is the Mahalanobis form
// q = |M dx|^2 (M = L^-1, T = L L^T), the cutoff an ellipsoid.
#pragma once
#include "mtpt_kernels.h"
#include "mtpt_rng.h"

#include <math.h>

#include <type_traits>

namespace mtpt {

// ------------------------------------------------------------------ basics
template <int PREC> struct Types;
template <> struct Types<0> { using T = double; using M = double; using A = double; };
template <> struct Types<1> { using T = float;  using M = double; using A = double; };
template <> struct Types<2> { using T = float;  using M = float;  using A = float;  };

// Particles a tile (cells plus halo) can stage in LDS: positions, and for the
// transfer pass also row sums and masses.  The row-sum pass (one
// instantiation for every species count) takes the capacity of the
// one-species transfer pass, so that it needs no more LDS than its tiles use
// (it stages positions only); each pass has its own tile plan.
template <int D, int PREC, int NS, bool TRANSFER> struct TileCap {
    using T = typename Types<PREC>::T;
    using M = typename Types<PREC>::M;
    static constexpr int bytes = D * static_cast<int>(sizeof(T)) + static_cast<int>(sizeof(T) + NS * sizeof(M));
    static constexpr int value = LdsBudget<D, PREC, NS>::value / bytes;
};

__device__ __forceinline__ int cell_coord(double x, double glo, double inv, int nc)
{
#pragma clang fp contract(off)
    int c = static_cast<int>((x - glo) * inv);
    c = c < 0 ? 0 : c;
    return c > nc - 1 ? nc - 1 : c;
}

template <int D>
__device__ __forceinline__ double r2_canonical(const double* xi, const double* xj)
{
#pragma clang fp contract(off)
    const double d0 = xj[0] - xi[0];
    const double d1 = xj[1] - xi[1];
    double r2 = d0 * d0 + d1 * d1;
    if (D == 3) {
        const double d2 = xj[2] - xi[2];
        r2 = r2 + d2 * d2;
    }
    return r2;
}

// Inside test and kernel value in the arithmetic of the path.  FP64: the
// canonical r^2 against psi^2.  FP32: the FP32 r^2 decides outside a 1e-5
// relative band around psi^2 (its error is below 1e-6 relative); inside the
// band the canonical FP64 r^2 of the same FP32 positions decides.
template <int D, typename T> struct Pair;

template <int D> struct Pair<D, double> {
    __device__ __forceinline__ static double r2(const double* xi, const double* xj)
    {
        return r2_canonical<D>(xi, xj);
    }
    __device__ __forceinline__ static bool inside(const SimArgs& a, const double* xi,
                                                  const double* xj, double* r2o)
    {
        const double r2 = r2_canonical<D>(xi, xj);
        *r2o = r2;
        return r2 <= a.psi2;
    }
    __device__ __forceinline__ static double kernel(const SimArgs& a, double r2) { return exp(-a.kc * r2); }
    __device__ __forceinline__ static double weight(double k, double si, double sj)
    {
        return (k + k) / (si + sj);
    }
};

template <int D> struct Pair<D, float> {
    // FP32 r^2 with a fixed contraction: fma(d0, d0, d1 d1) (+ fma(d2, d2, .))
    __device__ __forceinline__ static float r2(const float* xi, const float* xj)
    {
        const float d0 = xj[0] - xi[0];
        const float d1 = xj[1] - xi[1];
        float r = __builtin_fmaf(d0, d0, d1 * d1);
        if (D == 3) {
            const float d2 = xj[2] - xi[2];
            r = __builtin_fmaf(d2, d2, r);
        }
        return r;
    }
    __device__ __forceinline__ static bool inside(const SimArgs& a, const float* xi,
                                                  const float* xj, float* r2o)
    {
        const float r2 = Pair::r2(xi, xj);
        *r2o = r2;
        // below psi2_in inside for sure, above psi2_out outside; between the
        // two the FP64 test decides
        bool in = r2 <= a.psi2_out;
        if (__builtin_expect(in && r2 >= a.psi2_in, 0)) {
            double pi[3], pj[3];
#pragma unroll
            for (int k = 0; k < D; ++k) {
                pi[k] = static_cast<double>(xi[k]);
                pj[k] = static_cast<double>(xj[k]);
            }
            in = r2_canonical<D>(pi, pj) <= a.psi2;
        }
        return in;
    }
    __device__ __forceinline__ static float kernel(const SimArgs& a, float r2)
    {
        return __builtin_amdgcn_exp2f(a.kcf2 * r2);
    }
    __device__ __forceinline__ static float weight(float k, float si, float sj)
    {
        return (k + k) * __builtin_amdgcn_rcpf(si + sj);
    }
};

// Distance in the cutoff's metric.  Isotropic (TN = false): the squared
// distance of Pair.  Tensor (TN = true): the Mahalanobis form q = |M dx|^2,
// M = L^-1 lower triangular, in FP64 in the canonical order
//   y0 = M00 d0, y1 = M10 d0 + M11 d1, y2 = (M20 d0 + M21 d1) + M22 d2,
//   q = (y0 y0 + y1 y1) + y2 y2   (no contraction),
// or in FP32 with fused multiply-adds; the FP32 q decides outside a relative
// band around psi^2 sized on the host from the tensor's conditioning, the
// canonical FP64 q of the same FP32 positions inside it.
template <int D>
__device__ __forceinline__ double q_canonical(const double* m, const double* xi, const double* xj)
{
#pragma clang fp contract(off)
    const double d0 = xj[0] - xi[0];
    const double d1 = xj[1] - xi[1];
    const double y0 = m[0] * d0;
    const double y1 = m[1] * d0 + m[2] * d1;
    double q = y0 * y0 + y1 * y1;
    if (D == 3) {
        const double d2 = xj[2] - xi[2];
        const double y2 = (m[3] * d0 + m[4] * d1) + m[5] * d2;
        q = q + y2 * y2;
    }
    return q;
}

template <int D, typename T, bool TN> struct Metric;

template <int D, typename T> struct Metric<D, T, false> {
    __device__ __forceinline__ static T r2(const SimArgs&, const T* xi, const T* xj)
    {
        return Pair<D, T>::r2(xi, xj);
    }
    __device__ __forceinline__ static bool inside(const SimArgs& a, const T* xi, const T* xj, T* r2o)
    {
        return Pair<D, T>::inside(a, xi, xj, r2o);
    }
};

template <int D> struct Metric<D, double, true> {
    __device__ __forceinline__ static double r2(const SimArgs& a, const double* xi, const double* xj)
    {
        return q_canonical<D>(a.minv, xi, xj);
    }
    __device__ __forceinline__ static bool inside(const SimArgs& a, const double* xi, const double* xj,
                                                  double* r2o)
    {
        const double q = q_canonical<D>(a.minv, xi, xj);
        *r2o = q;
        return q <= a.psi2;
    }
};

template <int D> struct Metric<D, float, true> {
    __device__ __forceinline__ static float r2(const SimArgs& a, const float* xi, const float* xj)
    {
        const float* m = a.minvf;
        const float d0 = xj[0] - xi[0];
        const float d1 = xj[1] - xi[1];
        const float y0 = m[0] * d0;
        const float y1 = __builtin_fmaf(m[2], d1, m[1] * d0);
        float q = __builtin_fmaf(y1, y1, y0 * y0);
        if (D == 3) {
            const float d2 = xj[2] - xi[2];
            const float y2 = __builtin_fmaf(m[5], d2, __builtin_fmaf(m[4], d1, m[3] * d0));
            q = __builtin_fmaf(y2, y2, q);
        }
        return q;
    }
    __device__ __forceinline__ static bool inside(const SimArgs& a, const float* xi, const float* xj, float* r2o)
    {
        const float q = r2(a, xi, xj);
        *r2o = q;
        bool in = q <= a.psi2_out;
        if (__builtin_expect(in && q >= a.psi2_in, 0)) {
            double pi[3], pj[3];
#pragma unroll
            for (int k = 0; k < D; ++k) {
                pi[k] = static_cast<double>(xi[k]);
                pj[k] = static_cast<double>(xj[k]);
            }
            in = q_canonical<D>(a.minv, pi, pj) <= a.psi2;
        }
        return in;
    }
};

// The displacement of one coordinate in the type of the positions: the FP64
// z sdev + v dt (each operation rounded), rounded once more for FP32
// positions; then the position after the jump, reflected at the walls.
template <typename T>
__device__ __forceinline__ T jump_of(double z, double sdev, double drift)
{
#pragma clang fp contract(off)
    const double j = z * sdev + drift;
    return static_cast<T>(j);
}
template <typename T>
__device__ __forceinline__ T reflect_jump(T x, T jump, double lo, double hi, float lof, float hif);
template <>
__device__ __forceinline__ double reflect_jump<double>(double x, double jump, double lo, double hi, float, float)
{
#pragma clang fp contract(off)
    double v = x + jump;
    while (v < lo || v > hi)
        v = (v < lo) ? 2.0 * lo - v : 2.0 * hi - v;
    return v;
}
template <>
__device__ __forceinline__ float reflect_jump<float>(float x, float jump, double, double, float lof, float hif)
{
#pragma clang fp contract(off)
    float v = x + jump;
    while (v < lof || v > hif)
        v = (v < lof) ? 2.0f * lof - v : 2.0f * hif - v;
    return v;
}

// The D displacements of one particle from its standard normals z: with a
// dispersion tensor z is first replaced by u = L z (FP64, ascending column
// order, no contraction: u0 = L00 z0, u1 = L10 z0 + L11 z1,
// u2 = (L20 z0 + L21 z1) + L22 z2).
template <int D, typename T>
__device__ __forceinline__ void make_jumps(const SimArgs& a, const double* z, T* jv)
{
#pragma clang fp contract(off)
    double u[3] = {z[0], z[1], D == 3 ? z[2] : 0.0};
    if (a.tensor) {
        const double* l = a.lch;
        u[0] = l[0] * z[0];
        u[1] = l[1] * z[0] + l[2] * z[1];
        if (D == 3)
            u[2] = (l[3] * z[0] + l[4] * z[1]) + l[5] * z[2];
    }
#pragma unroll
    for (int k = 0; k < D; ++k)
        jv[k] = jump_of<T>(u[k], a.sdev, a.drift[k]);
}

// x-window [x_i - win, x_i + win] in the type of the positions, rounded
// outward so that no x within the exact window falls outside it
template <typename T> struct Window;
template <> struct Window<double> {
    __device__ __forceinline__ static void make(double xi, double win, double* lo, double* hi)
    {
        *lo = xi - win;
        *hi = xi + win;
    }
};
// next float below / above a finite v
__device__ __forceinline__ float float_down(float v)
{
    const uint32_t b = __float_as_uint(v);
    if (v == 0.0f)
        return __uint_as_float(0x80000001u);
    return __uint_as_float(v > 0.0f ? b - 1u : b + 1u);
}
__device__ __forceinline__ float float_up(float v)
{
    const uint32_t b = __float_as_uint(v);
    if (v == 0.0f)
        return __uint_as_float(0x00000001u);
    return __uint_as_float(v > 0.0f ? b + 1u : b - 1u);
}

template <> struct Window<float> {
    __device__ __forceinline__ static void make(float xi, double win, float* lo, float* hi)
    {
        const double l = static_cast<double>(xi) - win;
        const double h = static_cast<double>(xi) + win;
        float lf = static_cast<float>(l);
        float hf = static_cast<float>(h);
        if (static_cast<double>(lf) > l)
            lf = float_down(lf);
        if (static_cast<double>(hf) < h)
            hf = float_up(hf);
        *lo = lf;
        *hi = hf;
    }
};

// v / d for 0 <= v < 4096 and 1 <= d <= 256, with inv = 1.0f / d: the exact
// quotient plus (v mod d + 0.5) / d lies at least 0.5 / d >= 2^-9 from an
// integer, and the FP32 product is off by less than 4096 * 2^-22 = 2^-10, so
// the truncation is exact (no integer divide sequence)
__device__ __forceinline__ int small_div(int v, float inv)
{
    return static_cast<int>((static_cast<float>(v) + 0.5f) * inv);
}

// predicates of the compare builtins (ordered <= and >=, unsigned <)
constexpr int kFcmpLe = 5, kFcmpGe = 3, kIcmpUlt = 36;

// Wave64 primitives on DPP lane moves (no LDS round trip).  Every lane of
// the wave must be active.
// one DPP move: lane value from the lane that dpp_ctrl selects, 0 where that
// lane is outside the row or the row is masked off
template <int Ctrl, int RowMask = 0xF>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v)
{
    return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), Ctrl, RowMask, 0xF, true));
}

// inclusive scan over the 64 lanes: shifts by 1, 2, 4 and 8 inside each row
// of 16 lanes, then the last lane of row 0 (2) added to row 1 (3) and the
// last lane of row 1 added to rows 2 and 3
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v)
{
    v += dpp_u32<0x111>(v);          // row_shr:1
    v += dpp_u32<0x112>(v);          // row_shr:2
    v += dpp_u32<0x114>(v);          // row_shr:4
    v += dpp_u32<0x118>(v);          // row_shr:8
    v += dpp_u32<0x142, 0xA>(v);     // row_bcast:15 into rows 1 and 3
    v += dpp_u32<0x143, 0xC>(v);     // row_bcast:31 into rows 2 and 3
    return v;
}

// maximum over the 64 lanes, wave-uniform: the maximum of every quad, then of
// every row (rotations by 4 and 8), then of the four rows' lanes 0
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
    v = max(v, dpp_u32<0xB1>(v));    // quad_perm [1,0,3,2]
    v = max(v, dpp_u32<0x4E>(v));    // quad_perm [2,3,0,1]
    v = max(v, dpp_u32<0x124>(v));   // row_ror:4
    v = max(v, dpp_u32<0x128>(v));   // row_ror:8
    const uint32_t r0 = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), 0));
    const uint32_t r1 = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), 16));
    const uint32_t r2 = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), 32));
    const uint32_t r3 = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), 48));
    return max(max(r0, r1), max(r2, r3));
}

__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* total)
{
    __shared__ uint32_t wsum[kBlock / 64];
    const int lane = threadIdx.x & 63;
    const int wid = threadIdx.x >> 6;
    const uint32_t inc = wave_incl_scan(v);
    if (lane == 63)
        wsum[wid] = inc;
    __syncthreads();
    uint32_t base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kBlock / 64; ++w) {
        base += (w < wid) ? wsum[w] : 0u;
        tot += wsum[w];
    }
    __syncthreads();
    *total = tot;
    return base + inc - v;
}

// workgroup sum in a fixed order; result valid in thread 0
template <int NT, typename V>
__device__ __forceinline__ V block_sum(V v)
{
    __shared__ V red[NT / 64];
    const int lane = threadIdx.x & 63;
    const int wid = threadIdx.x >> 6;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        v += __shfl_down(v, off, 64);
    if (lane == 0)
        red[wid] = v;
    __syncthreads();
    V t = V(0);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 0; w < NT / 64; ++w)
            t += red[w];
    }
    __syncthreads();
    return t;
}

// N workgroup sums at once, each in the order of block_sum (wave shuffle
// tree, then the waves in order); results valid in thread 0.  One barrier
// for all N (the caller's last use of the workgroup, so none after it).
template <int NT, int N, typename V>
__device__ __forceinline__ void block_sum_n_final(V* v)
{
    __shared__ V red[N][NT / 64];
    const int lane = threadIdx.x & 63;
    const int wid = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < N; ++q) {
        V x = v[q];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1)
            x += __shfl_down(x, off, 64);
        if (lane == 0)
            red[q][wid] = x;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int q = 0; q < N; ++q) {
            V t = V(0);
#pragma unroll
            for (int w = 0; w < NT / 64; ++w)
                t += red[q][w];
            v[q] = t;
        }
    }
}

// Workgroups are dispatched to the 8 XCDs round-robin (workgroup b on XCD
// b mod 8), each XCD with its own L2.  Remapping b so that every XCD runs one
// contiguous chunk of logical blocks keeps neighbouring tiles and slot ranges,
// which share halo rows and gather sources, in the same L2.  The map is a
// bijection of [0, n) whatever the dispatch order.
__device__ __forceinline__ uint32_t xcd_block(uint32_t b, uint32_t n)
{
    constexpr uint32_t kXcd = 8;
    const uint32_t per = n / kXcd, rem = n % kXcd;
    const uint32_t x = b % kXcd, k = b / kXcd;
    return x * per + (x < rem ? x : rem) + k;
}

// -------------------------------------------------------------- binning
template <int D, typename T>
__device__ __forceinline__ void bin_body(const SimArgs& a, uint32_t blk)
{
    const int64_t i = static_cast<int64_t>(blk) * kBlock + threadIdx.x;
    if (i >= a.n)
        return;
    T v[3];
#pragma unroll
    for (int k = 0; k < D; ++k)
        v[k] = static_cast<const T*>(a.x[k])[i];
    if (a.walk) {
        const uint32_t pid = a.pid_src[i];
        double z[3] = {0.0, 0.0, 0.0}, spare;
        normal_pair(a.seed, a.step, pid, 0u, &z[0], &z[1]);
        if (D == 3)
            normal_pair(a.seed, a.step, pid, 1u, &z[2], &spare);
        T jv[3];
        make_jumps<D, T>(a, z, jv);
#pragma unroll
        for (int k = 0; k < D; ++k)
            v[k] = reflect_jump<T>(v[k], jv[k], a.lo[k], a.hi[k], a.lof[k], a.hif[k]);
    }
    uint32_t c = 0;
#pragma unroll
    for (int k = D - 1; k >= 0; --k) {
        static_cast<T*>(a.xt[k])[i] = v[k];
        c = c * static_cast<uint32_t>(a.nc[k]) +
            static_cast<uint32_t>(cell_coord(static_cast<double>(v[k]), a.glo[k], a.inv_side[k], a.nc[k]));
    }
    a.cell[i] = c;
    a.rank[i] = atomicAdd(&a.counts[c], 1u);
}

// Counts to scan are in[c] (+ in2[c] when in2 is given).
__device__ __forceinline__ void scan_reduce_body(const uint32_t* in, const uint32_t* in2, uint32_t* bsum,
                                                 uint32_t blk)
{
    const size_t base = static_cast<size_t>(blk) * kScanTile + threadIdx.x * kScanItems;
    const uint4* p = reinterpret_cast<const uint4*>(in + base);
    uint32_t s = 0;
#pragma unroll
    for (int q = 0; q < kScanItems / 4; ++q) {
        const uint4 w = p[q];
        s += w.x + w.y + w.z + w.w;
    }
    if (in2) {
        const uint4* p2 = reinterpret_cast<const uint4*>(in2 + base);
#pragma unroll
        for (int q = 0; q < kScanItems / 4; ++q) {
            const uint4 w = p2[q];
            s += w.x + w.y + w.z + w.w;
        }
    }
    const uint32_t t = block_sum<kBlock, uint32_t>(s);
    if (threadIdx.x == 0)
        bsum[blk] = t;
}

// Exclusive scan of the nb tile totals in place, by one workgroup: each
// thread takes 16 consecutive totals per round (its loads in flight
// together), so a round covers 4096 totals.
__device__ __forceinline__ void scan_top_body(uint32_t* bsum, uint32_t nb)
{
    constexpr uint32_t kTop = 16;
    uint32_t carry = 0;
    for (uint32_t base = 0; base < nb; base += kBlock * kTop) {
        const uint32_t i0 = base + threadIdx.x * kTop;
        uint32_t v[kTop];
#pragma unroll
        for (uint32_t q = 0; q < kTop; ++q)
            v[q] = i0 + q < nb ? bsum[i0 + q] : 0u;
        uint32_t sum = 0;
#pragma unroll
        for (uint32_t q = 0; q < kTop; ++q)
            sum += v[q];
        uint32_t tot;
        uint32_t run = carry + block_excl_scan(sum, &tot);
#pragma unroll
        for (uint32_t q = 0; q < kTop; ++q) {
            if (i0 + q < nb)
                bsum[i0 + q] = run;
            run += v[q];
        }
        carry += tot;
    }
}

// bsum holds the exclusive prefix of the tile totals (after the top pass),
// or with fold the raw totals, summed here over the tiles before blk.
__device__ __forceinline__ void scan_down_body(uint32_t* in, const uint32_t* in2, uint32_t* out,
                                               const uint32_t* bsum, uint32_t blk, bool zero_in,
                                               bool fold = false)
{
    __shared__ uint32_t pre_s;
    if (fold) {
        uint32_t t = 0;
        for (uint32_t b = threadIdx.x; b < blk; b += kBlock)
            t += bsum[b];
        t = block_sum<kBlock, uint32_t>(t);
        if (threadIdx.x == 0)
            pre_s = t;
        __syncthreads();
    }
    const uint32_t pre = fold ? pre_s : bsum[blk];
    const size_t base = static_cast<size_t>(blk) * kScanTile + threadIdx.x * kScanItems;
    uint4* p = reinterpret_cast<uint4*>(in + base);
    uint32_t v[kScanItems];
#pragma unroll
    for (int q = 0; q < kScanItems / 4; ++q) {
        const uint4 w = p[q];
        v[4 * q + 0] = w.x; v[4 * q + 1] = w.y; v[4 * q + 2] = w.z; v[4 * q + 3] = w.w;
    }
    if (in2) {
        const uint4* p2 = reinterpret_cast<const uint4*>(in2 + base);
#pragma unroll
        for (int q = 0; q < kScanItems / 4; ++q) {
            const uint4 w = p2[q];
            v[4 * q + 0] += w.x; v[4 * q + 1] += w.y; v[4 * q + 2] += w.z; v[4 * q + 3] += w.w;
        }
    }
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const uint32_t t = v[k];
        v[k] = s;
        s += t;
    }
    uint32_t tot;
    const uint32_t ex = block_excl_scan(s, &tot) + pre;
    uint4* o = reinterpret_cast<uint4*>(out + base);
#pragma unroll
    for (int q = 0; q < kScanItems / 4; ++q)
        o[q] = make_uint4(ex + v[4 * q], ex + v[4 * q + 1], ex + v[4 * q + 2], ex + v[4 * q + 3]);
    if (zero_in) {
#pragma unroll
        for (int q = 0; q < kScanItems / 4; ++q)
            p[q] = make_uint4(0u, 0u, 0u, 0u);
    }
}

__device__ __forceinline__ void scatter_body(const SimArgs& a, uint32_t blk)
{
    const int64_t i = static_cast<int64_t>(blk) * kBlock + threadIdx.x;
    if (i >= a.n)
        return;
    const uint32_t c = a.cell[i];
    const uint32_t r = a.rank[i];
    uint32_t slot = a.starts[c];
    if (a.tcounts_valid) {
        // slots of a cell: its tile's own particles first, then the arrivals
        // from other tiles (rank flagged in bit 31)
        slot += (r >> 31) ? a.tcounts[c] : 0u;
        slot += r & 0x7fffffffu;
    } else {
        slot += r;
    }
    a.perm[slot] = static_cast<uint32_t>(i);
}

// Linear cell index of a position (x fastest), as the binning computes it.
template <int D, typename T>
__device__ __forceinline__ uint32_t cell_index(const SimArgs& a, const T* v)
{
    uint32_t c = 0;
#pragma unroll
    for (int k = D - 1; k >= 0; --k)
        c = c * static_cast<uint32_t>(a.nc[k]) +
            static_cast<uint32_t>(cell_coord(static_cast<double>(v[k]), a.glo[k], a.inv_side[k], a.nc[k]));
    return c;
}

// Slot k holds particle src after the scatter, in arbitrary order inside its
// cell.  Its final slot is the cell start plus the number of cell members
// with a smaller (x, pid) key.  The workgroup gathers the keys of its 256
// slots once into LDS; only members of a cell that straddles the range of
// the workgroup are read from global memory.
template <int D, typename T, typename M>
__device__ __forceinline__ void place_body(const SimArgs& a, uint32_t blk)
{
    __shared__ T lkx[kBlock];
    __shared__ uint32_t lkp[kBlock];
    const int64_t k0 = static_cast<int64_t>(blk) * kBlock;
    const int64_t k = k0 + threadIdx.x;
    const bool live = k < a.n;
    const T* xt0 = static_cast<const T*>(a.xt[0]);
    uint32_t src = 0, kp = 0, b = 0, e = 0;
    T xv[3];
    M mv[3];
    T jv[3];
    if (live) {
        src = a.perm[k];
#pragma unroll
        for (int d = 0; d < D; ++d)
            xv[d] = static_cast<const T*>(a.xt[d])[src];
        kp = a.pid_src[src];
        // the masses are gathered with the keys, not after the ranking
        // (unless the row-sum pass moves them)
        if (!a.src_slot) {
#pragma unroll
            for (int s = 0; s < 3; ++s)
                if (s < a.ns)
                    mv[s] = static_cast<const M*>(a.m_src[s])[src];
        }
        const uint32_t c = cell_index<D, T>(a, xv);
        b = a.starts[c];
        e = a.starts[c + 1];
        lkx[threadIdx.x] = xv[0];
        lkp[threadIdx.x] = kp;
        if (a.fuse_bin) {
            // the jumps of the step after a.step, for the transfer pass's
            // walk, drawn while the cell's offsets are in flight
            double z[3] = {0.0, 0.0, 0.0}, spare;
            normal_pair(a.seed, a.step + 1, kp, 0u, &z[0], &z[1]);
            if (D == 3)
                normal_pair(a.seed, a.step + 1, kp, 1u, &z[2], &spare);
            make_jumps<D, T>(a, z, jv);
        }
    }
    __syncthreads();
    if (!live)
        return;
    const uint32_t lo = static_cast<uint32_t>(k0);
    const uint32_t hi = static_cast<uint32_t>(min(k0 + kBlock, a.n));
    const T kx = xv[0];
    uint32_t rank = 0;
    for (uint32_t q = b; q < e; ++q) {
        T ox;
        uint32_t op;
        if (q >= lo && q < hi) {
            ox = lkx[q - lo];
            op = lkp[q - lo];
        } else {
            const uint32_t o = a.perm[q];
            ox = xt0[o];
            op = a.pid_src[o];
        }
        rank += (ox < kx || (ox == kx && op < kp)) ? 1u : 0u;
    }
    const uint32_t dst = b + rank;
#pragma unroll
    for (int d = 0; d < D; ++d)
        static_cast<T*>(a.x[d])[dst] = xv[d];
    if (a.src_slot) {
        a.src_slot[dst] = src;
    } else {
#pragma unroll
        for (int s = 0; s < 3; ++s)
            if (s < a.ns)
                static_cast<M*>(a.m_mid[s])[dst] = mv[s];
    }
    a.pid_dst[dst] = kp;
    if (a.fuse_bin) {
#pragma unroll
        for (int d = 0; d < D; ++d)
            static_cast<T*>(a.jmp[d])[dst] = jv[d];
    }
}

// ------------------------------------------------------------ tiled passes
// A+B->C inside one particle over dt, exact solution of da/dt = db/dt = -k a b
// on concentrations (c = N M / V): with D = a - b >= 0,
// a' = a D / (D - b expm1(-k D dt)), or a/(1 + k a dt) when D = 0; b' = a' - D.
__device__ __forceinline__ void react3(double* m, const SimArgs& a)
{
    double ca = m[0] * a.to_c, cb = m[1] * a.to_c;
    const bool sw = cb > ca;
    if (sw) {
        const double t = ca;
        ca = cb;
        cb = t;
    }
    const double d = ca - cb;
    // one division for both cases (operands chosen first)
    const bool dpos = d > 0.0;
    const double num = dpos ? ca * d : ca;
    const double den = dpos ? d - cb * expm1(-a.k_react * d * a.dt) : 1.0 + a.k_react * ca * a.dt;
    const double an = num / den;
    const double bn = an - d;
    const double reacted = ca - an;
    m[0] = (sw ? bn : an) * a.to_m;
    m[1] = (sw ? an : bn) * a.to_m;
    m[2] = m[2] + reacted * a.to_m;
}

// Rows are trimmed to the particle's x-window (per row, from its y/z
// distance) before the candidate loop when rows are long (a.trim_rows, set
// by the host from the mean cell occupancy); short rows are scanned whole.

template <typename T> __device__ __forceinline__ T win2_of(const SimArgs& a);
template <> __device__ __forceinline__ double win2_of<double>(const SimArgs& a) { return a.win2d; }
template <> __device__ __forceinline__ float win2_of<float>(const SimArgs& a) { return a.win2f; }
template <typename T> __device__ __forceinline__ T wmargin_of(const SimArgs& a);
template <> __device__ __forceinline__ double wmargin_of<double>(const SimArgs& a) { return a.wmargind; }
template <> __device__ __forceinline__ float wmargin_of<float>(const SimArgs& a) { return a.wmarginf; }

// Half width of a row's x-window, sqrt(w2) plus the rounding margin, 0 < w2
// <= win^2.  The square root may be off by a relative 1e-6 upwards only (a
// wider window costs candidates, a narrower one would lose pairs): FP32 takes
// the hardware's (1 ulp, within the margin's 8 ulps of the window), FP64 the
// hardware FP32 root of w2 / win^2 scaled up by 1e-6 (a ratio too small for
// FP32 stands for a window far below the margin).
__device__ __forceinline__ float row_window(const SimArgs& a, float w2)
{
    return __builtin_amdgcn_sqrtf(w2) + a.wmarginf;
}
__device__ __forceinline__ double row_window(const SimArgs& a, double w2)
{
    const float r = __builtin_amdgcn_sqrtf(static_cast<float>(w2 * a.iwin2d)) * 1.000001f;
    return static_cast<double>(r) * a.win + a.wmargind;
}

// element of an LDS array at a byte offset
template <typename V>
__device__ __forceinline__ V lds_at(const V* base, int off)
{
    return *reinterpret_cast<const V*>(reinterpret_cast<const char*>(base) + off);
}

// Cutoff test of one candidate per lane, as a lane mask in scalar registers.
// FP64: exact.  FP32: r2 <= psi2_out; in_band, the lanes whose r2 lies in the
// band in which only the FP64 test decides (the caller then repeats its chunk
// with Metric::inside).
__device__ __forceinline__ uint64_t within(const SimArgs& a, double r2)
{
    return __builtin_amdgcn_fcmp(r2, a.psi2, kFcmpLe);
}
__device__ __forceinline__ uint64_t within(const SimArgs& a, float r2)
{
    return __builtin_amdgcn_fcmpf(r2, a.psi2_out, kFcmpLe);
}
__device__ __forceinline__ uint64_t in_band(const SimArgs&, double) { return 0ull; }
__device__ __forceinline__ uint64_t in_band(const SimArgs& a, float r2)
{
    return __builtin_amdgcn_fcmpf(r2, a.psi2_in, kFcmpGe);
}
// in[u] = near[u] & valid[u], and w with this lane's bits of them shifted in, in
// order: one add each with the mask as its carry-in (the compiler takes a select,
// a shift and an or).  The scalar ands stand in the same block: a vector
// instruction may not read a mask that a compare has just written, and the
// compiler does not look into the block to keep them apart, but the hardware
// orders it behind a scalar one.  Ands first, so that an add does not wait for
// its own (one by one the 1e5-particle 3-d walk's step lost 1.3 %).
template <int U>
__device__ __forceinline__ uint32_t shift_in(uint32_t w, const uint64_t (&near)[U], const uint64_t (&valid)[U],
                                             uint64_t (&in)[U])
{
    static_assert(U == 1 || U == 2 || U == 4, "groups of one, two and four");
    uint32_t r;
    uint64_t carry_out;
    if constexpr (U == 4)
        asm("s_and_b64 %0, %6, %10\n\ts_and_b64 %1, %7, %11\n\ts_and_b64 %2, %8, %12\n\ts_and_b64 %3, %9, %13\n\t"
            "v_addc_co_u32_e64 %4, %5, %14, %14, %0\n\tv_addc_co_u32_e64 %4, %5, %4, %4, %1\n\t"
            "v_addc_co_u32_e64 %4, %5, %4, %4, %2\n\tv_addc_co_u32_e64 %4, %5, %4, %4, %3"
            : "=&s"(in[0]), "=&s"(in[1]), "=&s"(in[2]), "=&s"(in[3]), "=v"(r), "=s"(carry_out)
            : "s"(near[0]), "s"(near[1]), "s"(near[2]), "s"(near[3]), "s"(valid[0]), "s"(valid[1]), "s"(valid[2]),
              "s"(valid[3]), "v"(w)
            : "scc");
    else if constexpr (U == 2)
        asm("s_and_b64 %0, %4, %6\n\ts_and_b64 %1, %5, %7\n\t"
            "v_addc_co_u32_e64 %2, %3, %8, %8, %0\n\tv_addc_co_u32_e64 %2, %3, %2, %2, %1"
            : "=&s"(in[0]), "=&s"(in[1]), "=v"(r), "=s"(carry_out)
            : "s"(near[0]), "s"(near[1]), "s"(valid[0]), "s"(valid[1]), "v"(w)
            : "scc");
    else
        asm("s_and_b64 %0, %3, %4\n\tv_addc_co_u32_e64 %1, %2, %5, %5, %0"
            : "=s"(in[0]), "=v"(r), "=s"(carry_out)
            : "s"(near[0]), "s"(valid[0]), "v"(w)
            : "scc");
    return r;
}

// Per-particle accumulator of the two passes.
template <int PREC, int NS, bool TRANSFER> struct Acc;

template <int PREC, int NS> struct Acc<PREC, NS, false> {
    using T = typename Types<PREC>::T;
    T s = T(0);
    uint32_t cnt = 0;
};

template <int PREC, int NS> struct Acc<PREC, NS, true> {
    using T = typename Types<PREC>::T;
    using M = typename Types<PREC>::M;
    using A = typename Types<PREC>::A;
    T si;
    M mi[NS];
    A dl[NS];
    A comp[NS];
};

// Candidates of one halo row: positions p[k] (k in [b, e), x-sorted), and for
// the transfer pass row sums sr[k] and masses ms[c][k]; slot j = k + jofs.
// Only the x-window [xlo, xhi] is visited.  rec(k) sees every candidate
// within the cutoff other than the particle itself.
template <int D, int PREC, int NS, bool TRANSFER, bool TN, typename PX, typename PS, typename PM, typename PR>
__device__ __forceinline__ void scan_row(const SimArgs& a, PX p, PS sr, PM ms, uint32_t b, uint32_t e,
                                         uint32_t jofs, const typename Types<PREC>::T* xi,
                                         typename Types<PREC>::T xlo, typename Types<PREC>::T xhi,
                                         uint32_t i, Acc<PREC, NS, TRANSFER>& acc, PR rec)
{
    using T = typename Types<PREC>::T;
    using M = typename Types<PREC>::M;
    using A = typename Types<PREC>::A;
    for (uint32_t k = b; k < e; ++k) {
        T xj[3];
        xj[0] = p(0, k);
        if (xj[0] < xlo)
            continue;
        if (xj[0] > xhi)
            break;
#pragma unroll
        for (int d = 1; d < D; ++d)
            xj[d] = p(d, k);
        if (TRANSFER && k + jofs == i)
            continue;
        T r2;
        if (!Metric<D, T, TN>::inside(a, xi, xj, &r2))
            continue;
        if (k + jofs != i)
            rec(k);
        const T kv = Pair<D, T>::kernel(a, r2);
        if constexpr (!TRANSFER) {
            acc.s += kv;
            acc.cnt += 1;
        } else {
            const T w = Pair<D, T>::weight(kv, acc.si, sr(k));
#pragma unroll
            for (int c = 0; c < NS; ++c) {
                const M mj = ms(c, k);
                if (PREC == 2) {
                    // Kahan-compensated FP32 accumulation
                    const A y = static_cast<A>(w) * static_cast<A>(mj - acc.mi[c]) - acc.comp[c];
                    const A t = acc.dl[c] + y;
                    acc.comp[c] = (t - acc.dl[c]) - y;
                    acc.dl[c] = t;
                } else {
                    acc.dl[c] = __builtin_fma(static_cast<A>(w), static_cast<A>(mj - acc.mi[c]), acc.dl[c]);
                }
            }
        }
    }
}

// Walk (with the jumps the place pass drew), cell id and histogram slot of
// sorted particle i for the step after a.step (the next step's binning,
// done while its position is in registers).
// A particle that stays inside the tile (cells [tlo, thi) per axis) takes
// its slot from the tile's LDS histogram hist (two 16-bit counts per word,
// used when the tile holds fewer than 65536 particles: tile_hist); one that
// leaves takes it from the global histogram, flagged in bit 31 of its rank.
// The slot is returned, not stored: the caller stores it after other work,
// so that the atomic's round trip overlaps that work.
template <int D, typename T>
__device__ __forceinline__ uint32_t bin_next(const SimArgs& a, uint32_t i, const T* x, const T* jump,
                                             const int* tlo, const int* thi, uint32_t* hist, bool tile_hist)
{
    uint32_t c = 0, lc = 0;
    bool inside = true;
#pragma unroll
    for (int k = D - 1; k >= 0; --k) {
        const T v = reflect_jump<T>(x[k], jump[k], a.lo[k], a.hi[k], a.lof[k], a.hif[k]);
        static_cast<T*>(a.xt[k])[i] = v;
        const int ck = cell_coord(static_cast<double>(v), a.glo[k], a.inv_side[k], a.nc[k]);
        c = c * static_cast<uint32_t>(a.nc[k]) + static_cast<uint32_t>(ck);
        inside = inside && ck >= tlo[k] && ck < thi[k];
        // tile-local index < 2^16 (a 24-bit multiply)
        lc = __umul24(lc, static_cast<uint32_t>(thi[k] - tlo[k])) + static_cast<uint32_t>(ck - tlo[k]);
    }
    a.cell[i] = c;
    uint32_t rank;
    if (inside && tile_hist) {
        const uint32_t sh = (lc & 1u) << 4;
        rank = (atomicAdd(&hist[lc >> 1], 1u << sh) >> sh) & 0xFFFFu;
    } else {
        rank = 0x80000000u | atomicAdd(&a.counts[c], 1u);
    }
    return rank;
}

}  // namespace mtpt
#include "mtpt_lists.h"
namespace mtpt {

// One tile: tx * ty * tz cells (tz = 1 in 2-d).  Halo rows (cells xa..xb-1
// of rows y0-1..y1 of planes z0-1..z1) are staged in LDS with the offsets of
// their cell boundaries; a particle in cell cx visits cells cx-1..cx+1 of
// each of its 3^(d-1) neighbouring rows, restricted to the x-window.  Halo
// and own rows are numbered y fastest with a fixed pitch per plane (see
// TileLimits); rows past the tile's extent are empty.
// With EXPORT the pass changes nothing: it records, for every own particle,
// the pairs it would use -- a.nb_col == nullptr: their count plus one (self)
// into a.nb_cnt[pid]; else the pids, self first, into a.nb_col from
// a.nb_row[pid] -- and skips every store of the step.
// With LIST the tile is that of mtpt_lists.h, for kListBlock threads.
template <int D, int PREC, int NS, bool TRANSFER, bool TN, bool EXPORT = false, bool LIST = false>
__device__ __forceinline__ void tile_body(const SimArgs& a, uint32_t blk)
{
    using T = typename Types<PREC>::T;
    using M = typename Types<PREC>::M;
    static_assert(!LIST || (D == 3 && PREC == 0 && !TN), "neighbour lists: 3-d, FP64, isotropic");
    constexpr int NT = LIST ? kListBlock : kBlock;
    constexpr int CAP = LIST ? kListCap
                             : TileCap<D, PREC, NS, TRANSFER>::value + (D == 3 && PREC == 0 && NS == 3 && !TN ? kSpareCap : 0);
    constexpr int planes = D == 3 ? 3 : 1;
    constexpr int SCAP = TRANSFER ? CAP : 1;
    // rows are trimmed to the spherical cutoff's x-window; an ellipsoidal
    // cutoff scans its rows whole (the host never sets trim_rows for it)
    constexpr bool kTrim = !TN && !LIST;
    // the FP64 row-sum pass evaluates its (software) exp only for the
    // candidates within the cutoff, after each chunk of 32, where rows are
    // not trimmed (about one candidate in six is in; in trimmed rows most
    // are, and the second loop costs more than it saves: measured)
    constexpr bool kExpAfter = !TRANSFER && PREC == 0;
    const bool exp_after = kExpAfter && !(kTrim && a.trim_rows);
    __shared__ T lpos[D][CAP];
    __shared__ T lsr[SCAP];
    __shared__ M lms[NS][SCAP];
    constexpr int kSegs = TileLimits<D>::segs;
    constexpr int kRows = TileLimits<D>::own_rows;   // own rows (pitch kSY per plane)
    constexpr int kSY = TileLimits<D>::seg_y;
    static_assert(kSegs <= 64, "a lane of a wave stands for each halo row");
    constexpr bool kHalves = LIST && TRANSFER && !EXPORT;   // sums of two transfer tiles (mtpt_lists.h)
    __shared__ uint32_t rbound[kHalves ? 5 : 4][kSegs];
    __shared__ uint32_t cst[kSegs][TileLimits<D>::cols];
    __shared__ uint32_t seg_gb[EXPORT ? kSegs : 1], seg_off[EXPORT ? kSegs : 1];
    // 2-d FP64 row-sum pass: own cells in order of their candidate count, so
    // that a wave's trip count is near its lanes' mean (the pass's only sum
    // over particles, the pair count, is an integer: the order changes no
    // result).  The FP32 pass's candidates are too cheap to repay the ordering.
    constexpr bool kCellOrder = D == 2 && !TRANSFER && (PREC == 0 ? MTPT_CELL_ORDER_2D : MTPT_CELL_ORDER_2D_F32) != 0;
    constexpr int kCells = kCellOrder ? TileLimits<D>::max_x * TileLimits<D>::max_y : 1;
    __shared__ uint16_t ord[kCellOrder ? CAP : 1];
    __shared__ uint32_t own_pre[kCellOrder ? kRows : 1];
    __shared__ uint8_t row_of[kCellOrder ? CAP : 1];   // own row of each own particle
    __shared__ uint8_t ckey[kCells];
    __shared__ uint32_t obase[64];
    // per-cell counts of the particles that stay in the tile, two 16-bit
    // counts per word
    constexpr int kHist =
        TRANSFER ? (TileLimits<D>::max_x * TileLimits<D>::max_y * TileLimits<D>::max_z + 1) / 2 : 1;
    __shared__ uint32_t hist[kHist];
    // list variant's row-sum pass: LDS offsets of every lane's neighbours
    __shared__ uint16_t found[LIST && !TRANSFER ? kListDepth : 1][LIST && !TRANSFER ? NT : 1];

    const int tid = threadIdx.x;
    const int nc0 = a.nc[0], nc1 = a.nc[1], nc2 = a.nc[2];
    // this pass's tile plan
    constexpr bool kOwnPlan = TRANSFER && !LIST;
    const int* const tl = kOwnPlan ? a.ttile : a.tile;
    const uint32_t tiles_x = kOwnPlan ? a.ttiles_x : a.tiles_x;
    const uint32_t per_slab = tiles_x * (kOwnPlan ? a.ttiles_y : a.tiles_y);
    const int tzi = static_cast<int>(blk / per_slab);
    const uint32_t rem = blk - static_cast<uint32_t>(tzi) * per_slab;
    const int tyi = static_cast<int>(rem / tiles_x);
    const int txi = static_cast<int>(rem - static_cast<uint32_t>(tyi) * tiles_x);
    const int x0 = txi * tl[0];
    const int x1 = min(x0 + tl[0], nc0);
    const int y0 = tyi * tl[1];
    const int y1 = min(y0 + tl[1], nc1);
    const int z0 = D == 3 ? tzi * tl[2] : 0;
    const int z1 = D == 3 ? min(z0 + tl[2], nc2) : 1;
    const int nrow = y1 - y0;                      // own rows per own plane
    const int nz = z1 - z0;                        // own planes (1 in 2-d)
    const int nown = nrow * nz;                    // own rows
    const int rows = nrow + 2;                     // halo rows per halo plane
    // Halo row sg = pz * kSY + py holds cells xa..xb-1 of grid row y0 - 1 + py
    // of plane z0 - 1 + pz (py < rows, pz < nz + 2; the others are empty).
    // Own row r = rz * kSY + ry holds cells x0..x1-1 of row y0 + ry of plane
    // z0 + rz (ry < nrow, rz < nz); its halo row is srow(r), and the halo rows
    // of its lowest candidate plane start at r.
    auto srow = [](int r) { return D == 3 ? r + kSY + 1 : r + 1; };
    const int xa = x0 > 0 ? x0 - 1 : 0;
    const int xb = x1 < nc0 ? x1 + 1 : nc0;
    const int ncol = xb - xa;
    const int tw = x1 - x0;
    if (TRANSFER && a.fuse_bin)
        for (int k = tid; k < (tw * nown + 1) / 2; k += NT)
            hist[k] = 0u;

    // Tile setup, bound by latency: two dependent rounds of global loads (the
    // cell boundaries of the halo rows, then their particles) and two
    // barriers.  Every wave works out the halo rows' and own rows' extents
    // for itself, lane r for row r, and finds the row of a slot by a search
    // through those lanes (ds_bpermute), so that no scan and no table crosses
    // waves.  Against block-wide scans (seven barriers) and searches in LDS
    // tables: 2-d transfer pass 93 -> 89 us (4e6 particles, FP32W) and 46.6 ->
    // 45.5 us (1e6, FP64), 1000 particles 8.1 -> 7.6 us and their row-sum pass
    // 7.8 -> 7.2 us, reacting 3-d FP64 (1e6) 108.5 -> 106.5 us, the other 3-d
    // passes within 1 %.
    const int lane = tid & 63;
    auto lane_u32 = [](uint32_t v, int l) {
        return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), l));
    };
    auto from_lane = [](uint32_t v, uint32_t l) {
        return static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(static_cast<int>(l * 4u), static_cast<int>(v)));
    };
    // last row r < n whose start (lane r of start) is <= at[k], for every k at
    // once: an empty row shares its start with the next one, which then wins
    auto find_rows = [&](uint32_t start, auto n, const auto& at, auto& row) {
        constexpr int N = std::extent_v<std::remove_reference_t<decltype(at)>>;
#pragma unroll
        for (int k = 0; k < N; ++k)
            row[k] = 0u;
#pragma unroll
        for (int len = n; len > 1;) {
            const uint32_t half = static_cast<uint32_t>(len >> 1);
#pragma unroll
            for (int k = 0; k < N; ++k)
                row[k] = from_lane(start, row[k] + half) <= at[k] ? row[k] + half : row[k];
            len -= static_cast<int>(half);
        }
    };
    // Every cell boundary of the halo rows in one round of loads, as global
    // slots (a row outside the grid is empty).  Thread k of a round takes
    // boundary c = k % kCP of halo row k / kCP (a power-of-two pitch: no
    // integer division); the values stay in registers until the rows' LDS
    // offsets are known.
    const int ncb = ncol + 1;
    constexpr int kCP = TileLimits<D>::col_p;
    constexpr int kCstIt = (kSegs * kCP + NT - 1) / NT;
    const int cc = tid % kCP;
    uint32_t cv[kCstIt];
#pragma unroll
    for (int it = 0; it < kCstIt; ++it) {
        const int sg = (tid + it * NT) / kCP;
        const int pzr = D == 3 ? sg / kSY : 0;
        const int pyr = D == 3 ? sg % kSY : sg;
        const int pz = z0 - 1 + pzr;
        const int py = y0 - 1 + pyr;
        const bool in = sg < kSegs && cc < ncb && pyr < rows && (D == 2 || pzr < nz + 2) && py >= 0 &&
                        py < nc1 && (D == 2 || (pz >= 0 && pz < nc2));
        cv[it] = in ? a.starts[(static_cast<uint32_t>(D == 3 ? pz : 0) * nc1 + py) * nc0 + xa + cc] : 0u;
    }
    // the ends of every halo row and of its own part, for the other waves
    if (cc == 0 || cc == ncol) {
#pragma unroll
        for (int it = 0; it < kCstIt; ++it)
            if ((tid + it * NT) / kCP < kSegs)
                rbound[cc == 0 ? 0 : 1][(tid + it * NT) / kCP] = cv[it];
    }
    if (cc == x0 - xa || cc == x1 - xa) {
#pragma unroll
        for (int it = 0; it < kCstIt; ++it)
            if ((tid + it * NT) / kCP < kSegs)
                rbound[cc == x0 - xa ? 2 : 3][(tid + it * NT) / kCP] = cv[it];
    }
    if constexpr (kHalves) {
        if (cc == min(x0 + a.ttile[0], x1) - xa) {
#pragma unroll
            for (int it = 0; it < kCstIt; ++it)
                if ((tid + it * NT) / kCP < kSegs)
                    rbound[4][(tid + it * NT) / kCP] = cv[it];
        }
    }
    __syncthreads();
    // lane r: halo row r, staged at LDS slots s_off .. from sorted slots s_off + s_dd ..;
    // own row r, own particles o_pre .., their sorted slots o_pre + o_dd ..,
    // their LDS slots o_pre + o_ld ..
    uint32_t s_len = 0, s_gb = 0;
    if (lane < kSegs) {
        s_gb = rbound[0][lane];
        s_len = rbound[1][lane] - s_gb;
    }
    const uint32_t s_inc = wave_incl_scan(s_len);
    const uint32_t s_off = s_inc - s_len;
    const uint32_t s_dd = s_gb - s_off;
    const uint32_t total = lane_u32(s_inc, 63);
    uint32_t o_len = 0, o_gb = 0;
    const int o_seg = srow(lane < kRows ? lane : 0);
    if (lane < kRows) {
        const int ry = D == 3 ? lane % kSY : lane;
        const int rz = D == 3 ? lane / kSY : 0;
        if (ry < nrow && rz < nz) {
            o_gb = rbound[2][o_seg];
            o_len = rbound[3][o_seg] - o_gb;
        }
    }
    // list variant: the part of own row r in the first of the two transfer tiles
    uint32_t a_len = 0;
    if constexpr (kHalves) {
        const int rr = lane < kRows ? lane : 0;
        const bool first = (a.lsplit != 1 || rr % kSY < a.ttile[1]) && (a.lsplit != 2 || rr / kSY < a.ttile[2]);
        a_len = a.lsplit == 0 ? min(o_len, rbound[4][o_seg] - o_gb) : (first ? o_len : 0u);
    }
    const uint32_t o_inc = wave_incl_scan(o_len);
    const uint32_t o_pre = o_inc - o_len;
    const uint32_t o_dd = o_gb - o_pre;
    const uint32_t o_ld = o_dd - from_lane(s_dd, static_cast<uint32_t>(o_seg));
    const uint32_t own_total = lane_u32(o_inc, 63);
    if constexpr (EXPORT) {
        if (tid < kSegs) {
            seg_gb[tid] = s_gb;
            seg_off[tid] = s_off;
        }
    }

    const bool use_lds = total <= static_cast<uint32_t>(CAP);
    // cell boundaries of every halo row as LDS offsets, or as sorted slots
    // when the tile does not fit the LDS (read by the particle loop after the
    // staging barrier)
#pragma unroll
    for (int it = 0; it < kCstIt; ++it) {
        const int sg = (tid + it * NT) / kCP;
        const uint32_t dd = from_lane(s_dd, static_cast<uint32_t>(sg & 63));
        if (sg < kSegs && cc < ncb)
            cst[sg][cc] = use_lds ? cv[it] - dd : cv[it];
    }
    // own row of every own particle, when they fit the table
    const bool rows_tab = kCellOrder && own_total <= static_cast<uint32_t>(CAP);
    if constexpr (kCellOrder) {
        if (tid < kRows)
            own_pre[tid] = o_pre;
        if (rows_tab)
            for (int r = __builtin_amdgcn_readfirstlane(tid >> 6); r < kRows; r += NT / 64)
                for (uint32_t j = static_cast<uint32_t>(lane); j < lane_u32(o_len, r); j += 64)
                    row_of[lane_u32(o_pre, r) + j] = static_cast<uint8_t>(r);
    }
    if (use_lds) {
        // Each halo row is one contiguous run in HBM and in LDS.  A thread
        // stages slots tid, tid + NT, ...: it finds every slot's row
        // first (the searches advance together), then issues all its loads,
        // then all its LDS stores, so that its loads are in flight at once.
        constexpr int kIt = (CAP + NT - 1) / NT;
        T vx[kIt][D];
        T vs[kIt];
        M vm[kIt][NS];
        uint32_t slots[kIt], sdd[kIt];
#pragma unroll
        for (int it = 0; it < kIt; ++it)
            slots[it] = static_cast<uint32_t>(tid + it * NT);
        find_rows(s_off, std::integral_constant<int, kSegs>{}, slots, sdd);
#pragma unroll
        for (int it = 0; it < kIt; ++it)
            sdd[it] = from_lane(s_dd, sdd[it]);
#pragma unroll
        for (int it = 0; it < kIt; ++it) {
            const uint32_t slot = static_cast<uint32_t>(tid + it * NT);
            if (slot < total) {
                const uint32_t g = slot + sdd[it];
#pragma unroll
                for (int d = 0; d < D; ++d)
                    vx[it][d] = static_cast<const T*>(a.x[d])[g];
                if (TRANSFER) {
                    vs[it] = static_cast<const T*>(a.srow)[g];
#pragma unroll
                    for (int c = 0; c < NS; ++c)
                        vm[it][c] = static_cast<const M*>(a.m_mid[c])[g];
                }
            }
        }
#pragma unroll
        for (int it = 0; it < kIt; ++it) {
            const uint32_t idx = static_cast<uint32_t>(tid + it * NT);
            if (idx < total) {
#pragma unroll
                for (int d = 0; d < D; ++d)
                    lpos[d][idx] = vx[it][d];
                if (TRANSFER) {
                    lsr[idx] = vs[it];
#pragma unroll
                    for (int c = 0; c < NS; ++c)
                        lms[c][idx] = vm[it][c];
                }
            }
        }
    }
    __syncthreads();

    const bool cell_order = kCellOrder && use_lds && rows_tab;
    if constexpr (kCellOrder) {
        if (cell_order) {
            if (tid < 64)
                obase[tid] = 0;
            __syncthreads();
            // own row r is halo row r + 1; own column cx is staged column x0 - xa + cx
            for (int j = tid; j < tw * nrow; j += NT) {
                const int r = j / tw;
                const int cxr = x0 - xa + (j - r * tw);
                const int cl = cxr > 0 ? cxr - 1 : 0;
                const int ch = cxr + 2 < ncol ? cxr + 2 : ncol;
                uint32_t tot = 0;
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    tot += cst[r + q][ch] - cst[r + q][cl];
                const uint32_t key = min(tot, 63u);
                ckey[j] = static_cast<uint8_t>(key);
                atomicAdd(&obase[key], cst[r + 1][cxr + 1] - cst[r + 1][cxr]);
            }
            __syncthreads();
            if (tid < 64) {
                const uint32_t v = obase[tid];
                obase[tid] = wave_incl_scan(v) - v;
            }
            __syncthreads();
            for (int j = tid; j < tw * nrow; j += NT) {
                const int r = j / tw;
                const int cxr = x0 - xa + (j - r * tw);
                const uint32_t c0 = cst[r + 1][cxr];
                const uint32_t nin = cst[r + 1][cxr + 1] - c0;
                if (nin == 0)
                    continue;
                const uint32_t pos = atomicAdd(&obase[ckey[j]], nin);
                const uint32_t t0 = own_pre[r] + (c0 - cst[r + 1][x0 - xa]);
                for (uint32_t q = 0; q < nin; ++q)
                    ord[pos + q] = static_cast<uint16_t>(t0 + q);
            }
            __syncthreads();
        }
    }

    uint32_t pairs = 0;
    double msum[NS];
#pragma unroll
    for (int c = 0; c < NS; ++c)
        msum[c] = 0.0;
    // Every lane of a wave runs every pass the wave takes (own_total is
    // uniform, and the loop holds no workgroup barrier), so the wave-wide
    // maxima below see only live lanes.  A wave leaves once all its lanes are
    // past the last own particle.
    for (uint32_t base = 0; base < own_total; base += NT) {
        if (base + static_cast<uint32_t>(tid & ~63) >= own_total)
            break;
        const uint32_t t = base + tid;
        const bool act = t < own_total;
        uint32_t tt = act ? t : own_total - 1u;
        int r;
        if (cell_order) {
            tt = ord[kCellOrder ? tt : 0u];
            r = row_of[kCellOrder ? tt : 0u];
        } else {
            const uint32_t at[1] = {tt};
            uint32_t row[1];
            find_rows(o_pre, std::integral_constant<int, kRows>{}, at, row);
            r = static_cast<int>(row[0]);
        }
        // the particle's sorted slot and its LDS slot; its own position (and,
        // in the transfer pass, row sum and masses) from there when the tile
        // is staged, else coalesced global loads (LDS reads and global loads
        // stay separate instructions: a select of the two addresses would
        // make them flat loads)
        const uint32_t i = tt + from_lane(o_dd, static_cast<uint32_t>(r));
        const uint32_t lself = tt + from_lane(o_ld, static_cast<uint32_t>(r));
        const uint32_t lq = use_lds ? lself : 0u;
        // first halo row of the particle's lowest candidate plane
        const int rbase = r;
        T xi[3];
#pragma unroll
        for (int d = 0; d < D; ++d)
            xi[d] = lpos[d][lq];
        if (!use_lds) {
#pragma unroll
            for (int d = 0; d < D; ++d)
                xi[d] = static_cast<const T*>(a.x[d])[i];
        }
        const int cxr = cell_coord(static_cast<double>(xi[0]), a.glo[0], a.inv_side[0], nc0) - xa;
        const int cl = cxr > 0 ? cxr - 1 : 0;
        const int ch = cxr + 2 < ncol ? cxr + 2 : ncol;
        Acc<PREC, NS, TRANSFER> acc;
        // export: the particle's pid and its next column in a.nb_col
        uint32_t ecnt = 0;
        int64_t ebase = 0;
        uint32_t epid = 0;
        if constexpr (EXPORT) {
            if (act) {
                epid = a.pid_dst[i];
                if (a.nb_col)
                    ebase = a.nb_row[epid] + 1;
            }
        }
        // one pair of particle i with sorted slot g
        auto record = [&](uint32_t g) {
            if constexpr (EXPORT) {
                if (a.nb_col)
                    a.nb_col[ebase + ecnt] = static_cast<int64_t>(a.pid_dst[g]);
                ++ecnt;
            }
        };
        // the particle's jumps and neighbour masks are loaded before its
        // candidate loops, all at once (issued later, each would stall the
        // wave in front of its use: measured 10 % of the 3-d three-species
        // transfer pass)
        constexpr bool kEarly = TRANSFER;
        T jv[3] = {T(0), T(0), T(0)};
        uint64_t mkp[planes], wkp[planes];
        uint32_t lw[kListWords] = {};
#pragma unroll
        for (int pzr = 0; pzr < planes; ++pzr)
            mkp[pzr] = wkp[pzr] = 0ull;
        if constexpr (TRANSFER) {
            const uint32_t ls = lq < SCAP ? lq : 0u;
            acc.si = lsr[ls];
#pragma unroll
            for (int c = 0; c < NS; ++c) {
                acc.mi[c] = lms[c][ls];
                acc.dl[c] = 0;
                acc.comp[c] = 0;
            }
            if (!use_lds) {
                acc.si = static_cast<const T*>(a.srow)[i];
#pragma unroll
                for (int c = 0; c < NS; ++c)
                    acc.mi[c] = static_cast<const M*>(a.m_mid[c])[i];
            }
            if constexpr (LIST) {
                // (the last word only where a lane of the wave needs it)
#pragma unroll
                for (int w = 0; w < kListWords - 1; ++w)
                    lw[w] = act ? list_word(a, w)[i] : 0u;
            }
            if (kEarly && a.fuse_bin) {
#pragma unroll
                for (int d = 0; d < D; ++d)
                    jv[d] = static_cast<const T*>(a.jmp[d])[i];
            }
            if (!LIST && kEarly && act) {
#pragma unroll
                for (int pzr = 0; pzr < planes; ++pzr)
                    mkp[pzr] = a.cmask[static_cast<size_t>(pzr) * static_cast<size_t>(a.n) + i];
            }
            if (kEarly && NS == 1 && use_lds && kTrim && a.trim_rows && act) {
#pragma unroll
                for (int pzr = 0; pzr < planes; ++pzr)
                    wkp[pzr] = a.cwin[static_cast<size_t>(pzr) * static_cast<size_t>(a.n) + i];
            }
        }
        if constexpr (LIST) {
            if (use_lds) {
                auto export_slot = [&](uint32_t slot) {
                    if constexpr (EXPORT) {
                        int sgi = 0;
                        for (int q = 1; q < kSegs; ++q)
                            sgi = seg_off[q] <= slot ? q : sgi;
                        record(seg_gb[sgi] + (slot - seg_off[sgi]));
                    }
                };
                if constexpr (TRANSFER)
                    list_transfer<NS, EXPORT, CAP>(a, lpos, lsr, lms, cst, rbase, cl, ch, lself, i, act, lw, xi, acc,
                                                   export_slot);
                else
                    list_rowsum<EXPORT, CAP>(a, lpos, cst, found, rbase, cl, ch, lself, i, act, xi, acc,
                                             export_slot);
            }
        }
        if (!LIST && use_lds) {
            // LDS slot of particle i itself (the self pair is skipped by slot)
            const uint32_t li = lself;
            if constexpr (!TRANSFER)
                acc.cnt = 1;   // self; the neighbours are counted from the masks
            // distances from the particle to the y (and z) slabs of the rows
            // below and above its own, less a rounding margin (for trimming)
            T dyv[3] = {T(0), T(0), T(0)};
            T dzv[3] = {T(0), T(0), T(0)};
            if (kTrim && a.trim_rows) {
                const int cyc = cell_coord(static_cast<double>(xi[1]), a.glo[1], a.inv_side[1], nc1);
                const T ylo = static_cast<T>(a.glo[1] + cyc * a.side[1]);
                dyv[0] = xi[1] - ylo - wmargin_of<T>(a);
                dyv[2] = ylo + static_cast<T>(a.side[1]) - xi[1] - wmargin_of<T>(a);
                if (D == 3) {
                    const int czc = cell_coord(static_cast<double>(xi[2]), a.glo[2], a.inv_side[2], nc2);
                    const T zlo = static_cast<T>(a.glo[2] + czc * a.side[2]);
                    dzv[0] = xi[2] - zlo - wmargin_of<T>(a);
                    dzv[2] = zlo + static_cast<T>(a.side[2]) - xi[2] - wmargin_of<T>(a);
                }
            }
#pragma unroll
            for (int pzr = 0; pzr < planes; ++pzr) {
                const int s0 = rbase + pzr * kSY;
                uint32_t b0 = cst[s0][cl], l0 = cst[s0][ch] - b0;
                uint32_t b1 = cst[s0 + 1][cl], l1 = cst[s0 + 1][ch] - b1;
                uint32_t b2 = cst[s0 + 2][cl], l2 = cst[s0 + 2][ch] - b2;
                if (kTrim && a.trim_rows) {
                    uint32_t bb[3] = {b0, b1, b2}, ll[3] = {l0, l1, l2};
                    uint64_t* const pwin = a.cwin + static_cast<size_t>(pzr) * static_cast<size_t>(a.n);
                    // the one-species transfer pass takes the windows the
                    // row-sum pass recorded when every lane's fit the packing
                    // (offset into the row and length, 10 bits each per row,
                    // bit 63 set); otherwise the wave searches again, to the
                    // same result (the three-species kernels always search:
                    // their registers are the tighter limit)
                    bool have = false;
                    if constexpr (TRANSFER && NS == 1) {
                        const uint64_t wv = act ? (kEarly ? wkp[pzr] : pwin[i]) : (1ull << 63);
                        have = __builtin_amdgcn_ballot_w64((wv >> 63) == 0ull) == 0ull;
                        if (have) {
#pragma unroll
                            for (int q = 0; q < 3; ++q) {
                                bb[q] += static_cast<uint32_t>(wv >> (20 * q)) & 0x3ffu;
                                ll[q] = static_cast<uint32_t>(wv >> (20 * q + 10)) & 0x3ffu;
                            }
                        }
                    }
                    if (!have) {
                        // x-window of each row from its y/z distance: |dx|^2 <= psi^2 - dy^2 - dz^2
                        const T dz = dzv[D == 3 ? pzr : 1] > T(0) ? dzv[D == 3 ? pzr : 1] : T(0);
                        T wlo[3], whi[3];
                        uint32_t lmax = 0;
#pragma unroll
                        for (int q = 0; q < 3; ++q) {
                            const T dy = dyv[q] > T(0) ? dyv[q] : T(0);
                            const T w2 = win2_of<T>(a) - dy * dy - dz * dz;
                            const T w = w2 > T(0) ? row_window(a, w2) : T(0);
                            wlo[q] = xi[0] - w;
                            whi[q] = xi[0] + w;
                            ll[q] = w2 > T(0) ? ll[q] : 0u;
                            lmax = max(lmax, ll[q]);
                        }
                        lmax = wave_max_u32(lmax);
                        const int nsteps = 32 - __builtin_clz(lmax | 1u);
                        // per row, the first slot with x >= wlo and the first with
                        // x > whi, both searched over the whole (x-sorted) row:
                        // wlo <= whi, so the second is never before the first.
                        // Powers of two downwards: pl[q] (ph[q]) is the LDS byte
                        // offset of the last slot known to lie before the result
                        // (one slot before the row at first); a step tries the
                        // slot st further on, if the row has it (pe: the row's
                        // last slot; a slot past it reads the row's end, or for an
                        // empty row the slot after it, and is not taken).  The six
                        // searches of a step are free of branches, so their LDS
                        // reads are in flight together; behind branches each
                        // waited for its own.
                        constexpr int kS = static_cast<int>(sizeof(T));
                        int pl[3], ph[3], pe[3], pc[3];
#pragma unroll
                        for (int q = 0; q < 3; ++q) {
                            pl[q] = ph[q] = (static_cast<int>(bb[q]) - 1) * kS;
                            pe[q] = pl[q] + static_cast<int>(ll[q]) * kS;
                            pc[q] = max(pe[q], pl[q] + kS);
                        }
                        for (int st = kS << (nsteps - 1); st >= kS; st >>= 1) {
                            T vl[3], vh[3];
#pragma unroll
                            for (int q = 0; q < 3; ++q) {
                                vl[q] = lds_at(lpos[0], min(pl[q] + st, pc[q]));
                                vh[q] = lds_at(lpos[0], min(ph[q] + st, pc[q]));
                            }
#pragma unroll
                            for (int q = 0; q < 3; ++q) {
                                const bool gl = (pl[q] + st <= pe[q]) & (vl[q] < wlo[q]);
                                const bool gh = (ph[q] + st <= pe[q]) & !(vh[q] > whi[q]);
                                pl[q] = gl ? pl[q] + st : pl[q];
                                ph[q] = gh ? ph[q] + st : ph[q];
                            }
                        }
                        uint64_t pack = 1ull << 63;
#pragma unroll
                        for (int q = 0; q < 3; ++q) {
                            const uint32_t slo = static_cast<uint32_t>(pl[q] / kS + 1);
                            const uint32_t off = slo - bb[q];
                            bb[q] = slo;
                            ll[q] = static_cast<uint32_t>(ph[q] - pl[q]) / kS;
                            pack = (off < 1024u && ll[q] < 1024u)
                                       ? pack | (static_cast<uint64_t>(off) << (20 * q)) |
                                             (static_cast<uint64_t>(ll[q]) << (20 * q + 10))
                                       : 0ull;
                        }
                        if constexpr (!TRANSFER && !EXPORT) {
                            if (act)
                                pwin[i] = pack;
                        }
                    }
                    b0 = bb[0]; l0 = ll[0];
                    b1 = bb[1]; l1 = ll[1];
                    b2 = bb[2]; l2 = ll[2];
                }
                const uint32_t tot = act ? l0 + l1 + l2 : 0u;
                // LDS byte offset of candidate k of the concatenated rows: k
                // sizeof(T) plus its row's offset (kept opaque so that the
                // scaling is not folded back into the candidate loops); a
                // candidate past the lane's rows reads the particle's own slot
                constexpr uint32_t kT = static_cast<uint32_t>(sizeof(T));
                uint32_t ob0 = b0 * kT, ob1 = (b1 - l0) * kT, ob2 = (b2 - l0 - l1) * kT, obs = li * kT;
                asm volatile("" : "+v"(ob0), "+v"(ob1), "+v"(ob2), "+v"(obs));
                const uint32_t e0 = l0, e1 = l0 + l1;
                auto slot_of = [ob0, ob1, ob2, obs, e0, e1](uint32_t k, bool valid) {
                    const uint32_t off = k * kT + (k < e0 ? ob0 : (k < e1 ? ob1 : ob2));
                    return valid ? off : obs;
                };
                auto ld = [](const auto* base, uint32_t off) { return lds_at(base, static_cast<int>(off)); };
                // the recorded neighbours serve the wave when every lane has
                // them (its row-sum tile was staged) and no lane has more
                // than 63 candidates (ballots: the wave-wide maximum is needed
                // only by the candidate loop)
                uint64_t mk = 0ull;
                bool use_mask = false, fits32 = false;
                if constexpr (TRANSFER) {
                    mk = kEarly ? mkp[pzr] : (act ? a.cmask[static_cast<size_t>(pzr) * static_cast<size_t>(a.n) + i] : 0ull);
                    use_mask = __builtin_amdgcn_ballot_w64(tot > 63u || (mk & kMaskInvalid) != 0ull) == 0ull;
                    fits32 = __builtin_amdgcn_ballot_w64(tot > 32u) == 0ull;
                }
                const uint32_t kmax = use_mask ? 0u : wave_max_u32(tot);
                constexpr int kUnroll = D == 3 ? (TRANSFER && NS == 3 ? MTPT_CAND_UNROLL_3D_S3 : MTPT_CAND_UNROLL_3D)
                                               : (PREC == 0 ? MTPT_CAND_UNROLL_2D_F64 : MTPT_CAND_UNROLL_2D);
                // one candidate at LDS byte offset off (of the T arrays), pair
                // counted when in
                auto visit = [&](uint32_t off, bool in, T r2) {
                    if constexpr (EXPORT) {
                        // LDS slot -> sorted slot: the halo row holding it
                        if (in && off != obs && act) {
                            const uint32_t lidx = off / kT;
                            int sgi = 0;
                            for (int q = 1; q < kSegs; ++q)
                                sgi = seg_off[q] <= lidx ? q : sgi;
                            record(seg_gb[sgi] + (lidx - seg_off[sgi]));
                        }
                    }
                    if constexpr (!TRANSFER) {
                        // the FP64 pass sums its kernel values after each
                        // chunk, over the chunk's neighbours only
                        if (!exp_after) {
                            const T kv = Pair<D, T>::kernel(a, r2);
                            acc.s += in ? kv : T(0);
                        }
                    } else {
                        const T kv = Pair<D, T>::kernel(a, r2);
                        using A = typename Types<PREC>::A;
                        const T w = Pair<D, T>::weight(kv, acc.si, ld(lsr, off));
#pragma unroll
                        for (int c = 0; c < NS; ++c) {
                            const M mj = ld(lms[c], off * static_cast<uint32_t>(sizeof(M) / sizeof(T)));
                            if (PREC == 2) {
                                const A y = static_cast<A>(w) * static_cast<A>(mj - acc.mi[c]) - acc.comp[c];
                                const A tk = acc.dl[c] + y;
                                const A cn = (tk - acc.dl[c]) - y;
                                acc.comp[c] = in ? cn : acc.comp[c];
                                acc.dl[c] = in ? tk : acc.dl[c];
                            } else {
                                // one rounding per increment, in the mask loop
                                // and the full loop alike
                                const A dm = static_cast<A>(mj - acc.mi[c]);
                                acc.dl[c] = __builtin_fma(static_cast<A>(w), in ? dm : A(0), acc.dl[c]);
                            }
                        }
                    }
                };
                uint64_t* const pmask = a.cmask + static_cast<size_t>(pzr) * static_cast<size_t>(a.n);
                if (TRANSFER && use_mask) {
                    // neighbours recorded by the row-sum pass: bit k of the
                    // mask is candidate k (same rows, same order) within psi
                    uint32_t cmax = static_cast<uint32_t>(__builtin_popcountll(mk));
                    cmax = wave_max_u32(cmax);
                    // a lane without a neighbour left visits its own slot:
                    // r^2 = 0 and m_j - m_i = 0 give an increment of exactly
                    // zero, which only the compensated sum has to skip
                    auto visit_bit = [&](uint32_t k, bool valid) {
                        const uint32_t off = slot_of(k, valid);
                        T xj[3];
#pragma unroll
                        for (int d = 0; d < D; ++d)
                            xj[d] = ld(lpos[d], off);
                        visit(off, PREC == 2 ? valid : true, Metric<D, T, TN>::r2(a, xi, xj));
                    };
                    if (fits32) {
                        // every lane's candidates fit the low word
                        uint32_t m32 = static_cast<uint32_t>(mk);
#pragma unroll kUnroll
                        for (uint32_t q = 0; q < cmax; ++q) {
                            const bool valid = m32 != 0u;
                            const uint32_t k = valid ? static_cast<uint32_t>(__builtin_ctz(m32)) : 0u;
                            m32 &= m32 - 1u;
                            visit_bit(k, valid);
                        }
                    } else {
#pragma unroll kUnroll
                        for (uint32_t q = 0; q < cmax; ++q) {
                            const bool valid = mk != 0ull;
                            const uint32_t k = valid ? static_cast<uint32_t>(__builtin_ctzll(mk)) : 0u;
                            mk &= mk - 1ull;
                            visit_bit(k, valid);
                        }
                    }
                    continue;
                }
                uint32_t mlo = 0, mhi = 0;
                // Candidates in chunks of 32, one mask word per chunk (shifted in,
                // first candidate highest, then bit-reversed).  The row-sum
                // pass's chunk is free of branches: FP32 pairs in the band
                // around the cutoff (about one in 10^5) are only noted, and a
                // chunk of a wave that met one is run again with the FP64
                // test.  The pass is bound by VALU issue on large sims and by
                // the latency of one wave's chain on small ones; a branch per
                // candidate kept the LDS reads of successive candidates apart,
                // each waiting for its own.  With the branch-free window search
                // and the one-instruction mask bit, against a branch per
                // candidate and per search step: 2e6-particle 3-d walk 288 ->
                // 244 us a launch, 3.2e7 reacting 1.48 -> 1.40 ms, 4e6 2-d 92
                // -> 82 us, 1e5 3-d (one wave per SIMD) 62 -> 45 us.
                for (uint32_t k0 = 0; k0 < kmax; k0 += 32u) {
                    const uint32_t kend = min(kmax, k0 + 32u);
                    uint32_t mw = 0;
                    // candidates k .. k + U - 1, their LDS reads first
                    auto group = [&](auto width, uint32_t k, uint64_t& band) {
                        constexpr int U = width;
                        uint32_t off[U];
                        T xj[U][3];
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            off[u] = slot_of(k + u, k + u < tot);
#pragma unroll
                            for (int d = 0; d < D; ++d)
                                xj[u][d] = ld(lpos[d], off[u]);
                        }
                        T r2[U];
                        uint64_t near[U], valid[U], in[U];
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            r2[u] = Metric<D, T, TN>::r2(a, xi, xj[u]);
                            near[u] = within(a, r2[u]);
                            valid[u] = __builtin_amdgcn_uicmp(k + u, tot, kIcmpUlt);
                        }
                        mw = shift_in(mw, near, valid, in);
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            band |= in_band(a, r2[u]) & in[u];
                            visit(off[u], __builtin_amdgcn_inverse_ballot_w64(in[u]), r2[u]);
                        }
                    };
                    // one candidate, with the exact test
                    auto single = [&](uint32_t k) {
                        const bool valid = k < tot;
                        const uint32_t off = slot_of(k, valid);
                        T xj[3];
#pragma unroll
                        for (int d = 0; d < D; ++d)
                            xj[d] = ld(lpos[d], off);
                        T r2;
                        bool in = Metric<D, T, TN>::inside(a, xi, xj, &r2) && valid;
                        if (TRANSFER)
                            in = in && off != obs;
                        visit(off, in, r2);
                        mw = (mw << 1) | (in ? 1u : 0u);
                    };
                    if constexpr (TRANSFER || EXPORT) {
#pragma unroll kUnroll
                        for (uint32_t k = k0; k < kend; ++k)
                            single(k);
                    } else {
                        constexpr int kGroup = D == 3 ? MTPT_ROW_GROUP_3D
                                                      : (PREC == 0 ? MTPT_ROW_GROUP_2D_F64 : MTPT_ROW_GROUP_2D);
                        const auto before = acc;
                        uint64_t band = 0ull;
                        uint32_t k = k0;
                        for (; k + kGroup <= kend; k += kGroup)
                            group(std::integral_constant<int, kGroup>{}, k, band);
                        if constexpr (kGroup > 2)
                            if (k + 2 <= kend) {
                                group(std::integral_constant<int, 2>{}, k, band);
                                k += 2;
                            }
                        if constexpr (kGroup > 1)
                            if (k < kend)
                                group(std::integral_constant<int, 1>{}, k, band);
                        if (__builtin_expect(band != 0ull, 0)) {
                            acc = before;
                            mw = 0;
                            for (k = k0; k < kend; ++k)
                                single(k);
                        }
                    }
                    if constexpr (!TRANSFER) {
                        // candidate k0 + j at bit j
                        mw = __builtin_bitreverse32(mw) >> (32u - (kend - k0));
                        if (exp_after) {
                            // kernel values of the chunk's candidates within
                            // the cutoff (the particle itself included), in
                            // candidate order: the same sum as adding every
                            // candidate's value or zero, with the software
                            // FP64 exp evaluated for about one candidate in
                            // six instead of all
                            uint32_t mr = mw;
                            uint32_t rmax = static_cast<uint32_t>(__builtin_popcount(mr));
                            rmax = wave_max_u32(rmax);
                            for (uint32_t q = 0; q < rmax; ++q) {
                                const bool valid = mr != 0u;
                                const uint32_t kb = valid ? static_cast<uint32_t>(__builtin_ctz(mr)) : 0u;
                                mr &= mr - 1u;
                                const uint32_t off = slot_of(k0 + kb, valid);
                                T xj[3];
#pragma unroll
                                for (int d = 0; d < D; ++d)
                                    xj[d] = ld(lpos[d], off);
                                const T kv = Pair<D, T>::kernel(a, Metric<D, T, TN>::r2(a, xi, xj));
                                acc.s += valid ? kv : T(0);
                            }
                        }
                        // the particle itself is candidate l0 + (li - b1) of
                        // its own plane's middle row
                        if (pzr == planes / 2) {
                            const uint32_t ks = l0 + (li - b1) - k0;
                            mw &= (act && ks < 32u) ? ~(1u << ks) : ~0u;
                        }
                        acc.cnt += static_cast<uint32_t>(__builtin_popcount(mw));
                        mlo = k0 == 0u ? mw : mlo;
                        mhi = k0 == 32u ? mw : mhi;
                    }
                }
                if (!TRANSFER && !EXPORT && act)
                    pmask[i] = tot <= 63u ? ((static_cast<uint64_t>(mhi) << 32) | mlo) : kMaskInvalid;
            }
        }
        if (!use_lds) {
#pragma unroll
            for (int pzr = 0; pzr < planes; ++pzr) {
#pragma unroll
                for (int dy = 0; dy < 3; ++dy) {
                    const int sg = rbase + pzr * kSY + dy;
                    const uint32_t b = cst[sg][cl];
                    const uint32_t e = act ? cst[sg][ch] : b;
                    T xlo, xhi;
                    Window<T>::make(xi[0], a.win, &xlo, &xhi);
                    scan_row<D, PREC, NS, TRANSFER, TN>(
                        a, [&](int d, uint32_t k) { return static_cast<const T*>(a.x[d])[k]; },
                        [&](uint32_t k) { return static_cast<const T*>(a.srow)[k]; },
                        [&](int c, uint32_t k) { return static_cast<const M*>(a.m_mid[c])[k]; }, b, e, 0u, xi,
                        xlo, xhi, i, acc, [&](uint32_t k) { if (act) record(k); });
                }
            }
            // no recorded neighbours or windows for the transfer pass (whose
            // tile may be staged)
            if constexpr (LIST && !TRANSFER && !EXPORT) {
                if (act) {
                    list_word(a, 0)[i] = kListNone;
                    count_unlisted(a, acc.cnt);
                }
            }
            if (!LIST && !TRANSFER && !EXPORT && act) {
#pragma unroll
                for (int pzr = 0; pzr < planes; ++pzr) {
                    a.cmask[static_cast<size_t>(pzr) * static_cast<size_t>(a.n) + i] = kMaskInvalid;
                    if (kTrim && a.trim_rows)
                        a.cwin[static_cast<size_t>(pzr) * static_cast<size_t>(a.n) + i] = 0ull;
                }
            }
        }
        if (!act)
            continue;
        if constexpr (EXPORT) {
            if (a.nb_col)
                a.nb_col[ebase - 1] = static_cast<int64_t>(epid);
            else
                a.nb_cnt[epid] = ecnt + 1u;
            continue;
        }
        if constexpr (!TRANSFER) {
            static_cast<T*>(a.srow)[i] = acc.s;
            pairs += acc.cnt - 1u;
            if (a.src_slot) {
                // the masses of the sorted slot, from the order before
                // re-binning (the place pass recorded the source slot): a
                // gather whose latency the arithmetic of the other waves hides
                const uint32_t src = a.src_slot[i];
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    if (c < a.ns)
                        static_cast<M*>(a.m_mid[c])[i] = static_cast<const M*>(a.m_src[c])[src];
            }
        } else {
            // the next step's walk and binning first: the slot's atomic (for
            // a particle that leaves the tile) is in flight during the mass
            // update and the reaction
            uint32_t nrank = 0;
            if (a.fuse_bin) {
                const int tlo[3] = {x0, y0, z0};
                const int thi[3] = {x1, y1, z1};
                if (!kEarly) {
#pragma unroll
                    for (int d = 0; d < D; ++d)
                        jv[d] = static_cast<const T*>(a.jmp[d])[i];
                }
                nrank = bin_next<D, T>(a, i, xi, jv, tlo, thi, hist, own_total < 65536u);
            }
            double mo[3];
#pragma unroll
            for (int c = 0; c < NS; ++c) {
                if (PREC == 2) {
                    const float nv = acc.mi[c] + a.betaf * acc.dl[c];
                    mo[c] = static_cast<double>(nv);
                } else {
                    mo[c] = static_cast<double>(acc.mi[c]) + a.beta * static_cast<double>(acc.dl[c]);
                }
            }
            if (NS == 3 && a.k_react > 0.0)
                react3(mo, a);
#pragma unroll
            for (int c = 0; c < NS; ++c) {
                const M st = static_cast<M>(mo[c]);
                static_cast<M*>(a.m_dst[c])[i] = st;
                msum[c] += static_cast<double>(st);
            }
            if (a.fuse_bin)
                a.rank[i] = nrank;
        }
    }
    if constexpr (EXPORT)
        return;
    if (TRANSFER && a.fuse_bin) {
        // counts of the tile's cells from the particles that stayed in it
        __syncthreads();
        const float inv_tw = 1.0f / static_cast<float>(tw);
        const float inv_nrow = 1.0f / static_cast<float>(nrow);
        for (int k = tid; k < tw * nown; k += NT) {
            const int rr = small_div(k, inv_tw);   // own row, y fastest (dense)
            const int rz = small_div(rr, inv_nrow);
            const uint32_t c = (static_cast<uint32_t>(z0 + rz) * nc1 + (y0 + rr - rz * nrow)) * nc0 + x0 + (k - rr * tw);
            a.tcounts[c] = (hist[k >> 1] >> ((k & 1) << 4)) & 0xFFFFu;
        }
    }
    if constexpr (!TRANSFER) {
        const uint32_t p = block_sum<NT, uint32_t>(pairs);
        if (tid == 0)
            a.pair_part[blk] = p;
    } else if constexpr (LIST) {
        const uint32_t a_inc = wave_incl_scan(a_len);
        const uint32_t a_pre = a_inc - a_len, a_total = lane_u32(a_inc, 63);
        // the transfer tile that this thread sums for
        const bool upper = __builtin_amdgcn_readfirstlane(tid / kBlock) != 0;
        const uint32_t v = static_cast<uint32_t>(tid % kBlock);
        const uint32_t count = upper ? own_total - a_total : a_total;
        auto row_at = [&](uint32_t start, uint32_t k) {
            const uint32_t at[1] = {k};
            uint32_t row[1];
            find_rows(start, std::integral_constant<int, kRows>{}, at, row);
            return row[0];
        };
        double sum[NS] = {};
        __syncthreads();                     // (the staged masses are read no more)
        if (own_total <= static_cast<uint32_t>(NT)) {
            // each thread's mass to its place in its transfer tile's order
            const uint32_t t = min(static_cast<uint32_t>(tid), own_total > 0u ? own_total - 1u : 0u);
            const uint32_t r = row_at(o_pre, t);
            const uint32_t op = from_lane(o_pre, r), ap = from_lane(a_pre, r), al = from_lane(a_len, r);
            const uint32_t to = t - op < al ? ap + (t - op) : a_total + (op - ap) + (t - op - al);
            if (static_cast<uint32_t>(tid) < own_total)
#pragma unroll
                for (int c = 0; c < NS; ++c)
                    lms[c][to] = msum[c];
            __syncthreads();
            for (uint32_t k = v; k < count; k += kBlock)
#pragma unroll
                for (int c = 0; c < NS; ++c)
                    sum[c] += lms[c][(upper ? a_total : 0u) + k];
        } else {
            for (uint32_t k0 = 0; k0 < count; k0 += kBlock) {
                const uint32_t k = min(k0 + v, count - 1u);
                const uint32_t r = row_at(upper ? o_pre - a_pre : a_pre, k);
                const uint32_t op = from_lane(o_pre, r), ap = from_lane(a_pre, r), al = from_lane(a_len, r);
                const uint32_t i = from_lane(o_dd, r) + op + (upper ? al + (k - (op - ap)) : k - ap);
                if (k0 + v < count)
#pragma unroll
                    for (int c = 0; c < NS; ++c)
                        sum[c] += static_cast<const double*>(a.m_dst[c])[i];
            }
        }
        const int sub[3] = {txi * (a.lsplit == 0 ? 2 : 1) + (upper && a.lsplit == 0 ? 1 : 0),
                            tyi * (a.lsplit == 1 ? 2 : 1) + (upper && a.lsplit == 1 ? 1 : 0),
                            tzi * (a.lsplit == 2 ? 2 : 1) + (upper && a.lsplit == 2 ? 1 : 0)};
        list_totals<NS>(a, upper, sub, sum);
    } else {
        block_sum_n_final<NT, NS, double>(msum);
        if (tid == 0) {
#pragma unroll
            for (int c = 0; c < NS; ++c)
                a.partials[static_cast<size_t>(blk) * NS + c] = msum[c];
        }
    }
}

// Totals and pair counters of one step (mode 0) or totals only (mode 1),
// summed over the per-workgroup partials in a fixed order; counted: the step
// ran the row-sum pass, which left its pair counts.
template <int NT>
__device__ __forceinline__ void finalize_body(const SimArgs& a, const double* partials, bool counted,
                                              uint32_t nparts, int mode)
{
    const int ns = a.ns;
    DevStats* st = a.st;
    unsigned long long pairs = 0;
    if (mode == 0 && counted) {
        unsigned long long p = 0;
#pragma unroll 8
        for (uint32_t b = threadIdx.x; b < a.ntiles; b += NT)
            p += a.pair_part[b];
        pairs = block_sum<NT, unsigned long long>(p);
    }
    for (int c = 0; c < ns; ++c) {
        double s = 0.0;
#pragma unroll 8
        for (uint32_t b = threadIdx.x; b < nparts; b += NT)
            s += partials[static_cast<size_t>(b) * ns + c];
        const double t = block_sum<NT, double>(s);
        if (threadIdx.x == 0) {
            st->totals[c] = t;
            if (!isfinite(t))
                st->nonfinite = 1;
        }
    }
    if (threadIdx.x == 0 && mode == 0) {
        if (counted)
            st->pairs_last = pairs;
        st->pairs_total += st->pairs_last;
        st->steps += 1;
    }
}

// ---------------------------------------------------------- tiled kernels
__device__ __forceinline__ int find_sim(const Batch& b, uint32_t blk, uint32_t* local)
{
    int lo = 0, hi = b.nsims - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (b.blk_off[mid] <= blk)
            lo = mid;
        else
            hi = mid - 1;
    }
    *local = blk - b.blk_off[lo];
    return lo;
}

// The arguments of a tiled pass, read where they are used.  A tile's chain of
// barriers, searches and candidate loops uses some sixty of them: taken by
// value they are all loaded at the start and kept, in 106 scalar registers
// and 40 to 140 spilled ones, each spill and its return an instruction of the
// vector unit; taken from a batch's array, every load behind a store is a
// vector load that waits for the memory.  Through the constant address space
// (nothing writes them while the kernel runs) they are scalar loads wherever
// they stand, and the hidden pointer keeps the compiler from gathering them at
// the start again.  One word of each 64 bytes is read first, all at once: the
// first use of a line would otherwise wait for the memory, in turn (1000
// particles: row sum 7.1 us by value, 7.6 without, 7.2 with).  By value / so,
// us a launch: 3-d transfer of 3.2e7 reacting particles 2065 / 1980, of a
// 2e6-particle walk 184 / 177, 2-d FP64 transfer (1e4 particles) 11.2 / 8.4, 2-d
// row sum (4e6) 75 / 72, 3-d (5e4) 37.9 / 34.9; batches of a pool, 2-d
// transfer 45 / 31, 3-d 160 / 120.
using ConstArgs = const __attribute__((address_space(4))) SimArgs;
__device__ __forceinline__ const SimArgs& args_at(ConstArgs* p)
{
    using Word = const __attribute__((address_space(4))) uint32_t;
    static_assert(sizeof(SimArgs) > 13 * 64 && sizeof(SimArgs) <= 14 * 64, "one word of each 64 bytes");
    Word* w = (Word*)p;
    asm volatile("" ::"s"(w[0]), "s"(w[16]), "s"(w[32]), "s"(w[48]), "s"(w[64]), "s"(w[80]), "s"(w[96]), "s"(w[112]),
                 "s"(w[128]), "s"(w[144]), "s"(w[160]), "s"(w[176]), "s"(w[192]), "s"(w[208]));
    asm volatile("" : "+s"(p));
    return *(const SimArgs*)p;
}
// a single sim's kernel has them as its first argument
__device__ __forceinline__ const SimArgs& kernel_args()
{
    return args_at((ConstArgs*)__builtin_amdgcn_kernarg_segment_ptr());
}

#define MTPT_BATCH_PROLOGUE                                                                     \
    uint32_t l;                                                                                 \
    const SimArgs& a = b.args[find_sim(b, xcd_block(blockIdx.x, gridDim.x), &l)]

// The 3-d FP32W isotropic row-sum pass is held to the seven waves per SIMD
// that its LDS allows (72 registers).
template <int D, int PREC, bool TN>
__global__ __launch_bounds__(kBlock, D == 3 && PREC == 1 && !TN ? 7 : 1) void rowsum_k(SimArgs a)
{
    // (ellipsoidal cutoff: by value.  By value / through the constant address
    // space, us a launch: 2-d FP32W 1e4 10.4 / 10.7, 5e4 12.2 / 12.3, 5e5 24.6 / 24.7,
    // 2e6 53.2 / 52.2, FP64 2e6 95.7 / 94.9; 3-d 5e4 to 1e6 within 1 % both ways.  A
    // whole step of 1e4 takes 30.3 / 32.0, of 5e4 33.7 / 35.4.)
    tile_body<D, PREC, 1, false, TN>(TN ? a : kernel_args(), xcd_block(blockIdx.x, gridDim.x));
}
template <int D, int PREC, bool TN>
__global__ __launch_bounds__(kBlock, D == 3 && PREC == 1 && !TN ? 7 : 1) void rowsum_kb(Batch b)
{
    MTPT_BATCH_PROLOGUE;
    tile_body<D, PREC, 1, false, TN>(args_at((ConstArgs*)&a), l);
}

// the 2-d FP64 one-species transfer kernel is held to the registers of 5
// workgroups per CU, which its LDS allows
#ifndef MTPT_S3_MIN_BLOCKS
#define MTPT_S3_MIN_BLOCKS 1
#endif
template <int D, int PREC, int NS>
constexpr int transfer_min_blocks()
{
    return PREC == 0 && D == 2 && NS == 1 ? 5 : (D == 3 && PREC == 1 && NS == 3 ? MTPT_S3_MIN_BLOCKS : 1);
}
template <int D, int PREC, int NS, bool TN>
__global__ __launch_bounds__(kBlock, (transfer_min_blocks<D, PREC, NS>())) void transfer_k(SimArgs a)
{
    // A static sim's launch has one more workgroup, the first, that finalizes
    // the previous step: the step is bound by launch latency, and the finalize
    // launch and the gap before it are gone (50 steps and a read: 1e4
    // particles FP64 805 -> 680 us, 3e5 FP32W 1248 -> 1119 us; with the steps
    // made since, 516 and 1110 us).
    uint32_t blk = blockIdx.x, n = gridDim.x;
    if (a.fin_partials) {
        if (blk == 0) {
            finalize_body<kBlock>(a, a.fin_partials, a.fin_counted != 0, a.nttiles, 0);
            return;
        }
        --blk;
        --n;
    }
    tile_body<D, PREC, NS, true, TN>(kernel_args(), xcd_block(blk, n));
}
template <int D, int PREC, int NS, bool TN>
__global__ __launch_bounds__(kBlock, (transfer_min_blocks<D, PREC, NS>())) void transfer_kb(Batch b)
{
    MTPT_BATCH_PROLOGUE;
    tile_body<D, PREC, NS, true, TN>(args_at((ConstArgs*)&a), l);
}

// Launch of the row-sum (ph = PH_ROWSUM) or transfer (PH_TRANSFER) pass of
// dimension D and metric TN: one sim (a) or a batch (b).  Instantiated by
// the mtpt_tiles_*.hip units, one per (D, TN).
template <int D, bool TN>
hipError_t launch_tiles(int ph, int prec, int ns, const SimArgs* a, const Batch* b, hipStream_t s)
{
    const uint32_t grid =
        a ? (ph == PH_ROWSUM ? a->ntiles : a->nttiles + (a->fin_partials ? 1u : 0u)) : b->total_blocks;
    if (grid == 0 || (b && b->nsims == 0) || (a && a->n <= 0))
        return hipSuccess;
#define MTPT_TILE_LAUNCH(KSIM, KBAT)                                                             \
    do {                                                                                         \
        if (a) KSIM<<<grid, kBlock, 0, s>>>(*a);                                                 \
        else KBAT<<<grid, kBlock, 0, s>>>(*b);                                                   \
    } while (0)
    if (ph == PH_ROWSUM) {
        if (prec == 0) MTPT_TILE_LAUNCH((rowsum_k<D, 0, TN>), (rowsum_kb<D, 0, TN>));
        else if (prec == 1) MTPT_TILE_LAUNCH((rowsum_k<D, 1, TN>), (rowsum_kb<D, 1, TN>));
        else MTPT_TILE_LAUNCH((rowsum_k<D, 2, TN>), (rowsum_kb<D, 2, TN>));
    } else if (ph == PH_TRANSFER) {
        if (ns == 1) {
            if (prec == 0) MTPT_TILE_LAUNCH((transfer_k<D, 0, 1, TN>), (transfer_kb<D, 0, 1, TN>));
            else if (prec == 1) MTPT_TILE_LAUNCH((transfer_k<D, 1, 1, TN>), (transfer_kb<D, 1, 1, TN>));
            else MTPT_TILE_LAUNCH((transfer_k<D, 2, 1, TN>), (transfer_kb<D, 2, 1, TN>));
        } else {
            if (prec == 0) MTPT_TILE_LAUNCH((transfer_k<D, 0, 3, TN>), (transfer_kb<D, 0, 3, TN>));
            else if (prec == 1) MTPT_TILE_LAUNCH((transfer_k<D, 1, 3, TN>), (transfer_kb<D, 1, 3, TN>));
            else MTPT_TILE_LAUNCH((transfer_k<D, 2, 3, TN>), (transfer_kb<D, 2, 3, TN>));
        }
    } else {
        return hipErrorInvalidValue;
    }
#undef MTPT_TILE_LAUNCH
    return hipGetLastError();
}

// Export launches (mtpt_step_neighbors): the row-sum or transfer pass of
// the last step, recording instead of storing.
template <int D, int PREC, bool TN>
__global__ __launch_bounds__(kBlock) void rowsum_export_k(SimArgs a)
{
    tile_body<D, PREC, 1, false, TN, true>(a, xcd_block(blockIdx.x, gridDim.x));
}
template <int D, int PREC, int NS, bool TN>
__global__ __launch_bounds__(kBlock) void transfer_export_k(SimArgs a)
{
    tile_body<D, PREC, NS, true, TN, true>(a, xcd_block(blockIdx.x, gridDim.x));
}

template <int D, bool TN>
hipError_t launch_tiles_export(int ph, int prec, int ns, const SimArgs& a, hipStream_t s)
{
    const uint32_t grid = ph == PH_ROWSUM ? a.ntiles : a.nttiles;
    if (grid == 0 || a.n <= 0)
        return hipSuccess;
    if (ph == PH_ROWSUM) {
        if (prec == 0) rowsum_export_k<D, 0, TN><<<grid, kBlock, 0, s>>>(a);
        else if (prec == 1) rowsum_export_k<D, 1, TN><<<grid, kBlock, 0, s>>>(a);
        else rowsum_export_k<D, 2, TN><<<grid, kBlock, 0, s>>>(a);
    } else if (ph == PH_TRANSFER) {
        if (ns == 1) {
            if (prec == 0) transfer_export_k<D, 0, 1, TN><<<grid, kBlock, 0, s>>>(a);
            else if (prec == 1) transfer_export_k<D, 1, 1, TN><<<grid, kBlock, 0, s>>>(a);
            else transfer_export_k<D, 2, 1, TN><<<grid, kBlock, 0, s>>>(a);
        } else {
            if (prec == 0) transfer_export_k<D, 0, 3, TN><<<grid, kBlock, 0, s>>>(a);
            else if (prec == 1) transfer_export_k<D, 1, 3, TN><<<grid, kBlock, 0, s>>>(a);
            else transfer_export_k<D, 2, 3, TN><<<grid, kBlock, 0, s>>>(a);
        }
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace mtpt

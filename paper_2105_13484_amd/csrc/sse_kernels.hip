// HIP kernels of the split-explicit step for gfx950.
//
// Column kernels (3D): one 64-lane wavefront owns one vertical column of a
// cell, an edge or a vertex; lane k holds layer k (layers >= 64 live in a
// second register chunk).  Mesh indices are therefore wave-uniform (scalar
// loads) and every neighbour access is one contiguous column read; vertical
// sums and scans are cross-lane operations inside the wavefront.  Lanes past
// the last layer load a copy of the last layer; what they hold is zeroed
// before it reaches a sum or a scan over the layers.
//
// 2D kernels (barotropic loop, reconciliation): one thread per edge or cell,
// reading slot-major neighbour tables.
//
// R is double (FP64 mode) or float (mixed mode); the split between the two
// types is described in sse_kernels.h.
#include <hip/hip_runtime.h>

#include <cmath>

#include "sse_kernels.h"

namespace sse {

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

// Workgroups are dispatched to the 8 XCDs round-robin (block b runs on XCD
// b mod 8) and every XCD has its own L2.  Launches use 8 * ceil(nb / 8)
// blocks and renumber them so that XCD x processes the contiguous logical
// range [x * per, (x + 1) * per): neighbouring columns then share one L2.
// Returns -1 for the padding blocks.
__device__ __forceinline__ int xcd_block(int nb) {
    const int per = (nb + kXcd - 1) / kXcd;
    const int b = blockIdx.x;
    const int logical = (b % kXcd) * per + b / kXcd;
    return logical < nb ? logical : -1;
}

// Index of the column owned by this wavefront among n columns (n: none); a
// workgroup of w wavefronts owns w consecutive columns.
// readfirstlane tells the compiler the value is wave-uniform, so mesh-table
// reads that depend on it become scalar loads instead of 64 identical vector
// loads.
__device__ __forceinline__ int column_id(int n) {
    const int cpb = blockDim.x >> 6;
    const int lb = xcd_block((n + cpb - 1) / cpb);
    const int col = lb * cpb + (threadIdx.x >> 6);
    return __builtin_amdgcn_readfirstlane(lb < 0 ? n : col);
}

// ---------------------------------------------------------------------------
// Cross-lane operations of a column; every caller runs them with all 64
// lanes active.  Two forms, chosen by the kernel (kDpp):
//  * DPP: values move inside rows of 16 lanes, and by one lane across the
//    wavefront, as DPP operands, with no LDS round trip and no wait.  An FP32
//    step is one instruction (the move folds into the addition); an FP64
//    step takes two moves besides the addition.
//  * shuffles: lane permutes through the LDS crossbar, fewer VALU
//    instructions for FP64 values.
// The kernels of both precisions use DPP for every value type (the FP64
// edge pass, once its column loads took 32-bit scalar offsets, had the
// registers for it and became 3.7% faster than with shuffles; the assembly
// pass, 11%).  The butterfly steps that cross rows (i ^ 32, i ^ 16) are
// shuffles in both forms, and the butterfly keeps its pairwise order, so a
// column sum has the same bits in both.
// ---------------------------------------------------------------------------
template <typename R>
constexpr bool kDppFor = true;

constexpr int kDppQuadXor1 = 0xB1;      // quad_perm [1,0,3,2]
constexpr int kDppQuadXor2 = 0x4E;      // quad_perm [2,3,0,1]
constexpr int kDppRowShl = 0x100;       // + n: lane j of a row reads lane j + n of the row
constexpr int kDppRowShr = 0x110;       // + n: lane j of a row reads lane j - n of the row
constexpr int kDppRowRor = 0x120;       // + n: rotation within a row
constexpr int kDppWaveShl1 = 0x130;     // lane i reads lane i + 1
constexpr int kDppWaveShr1 = 0x138;     // lane i reads lane i - 1
constexpr int kDppRowBcast15 = 0x142;   // lane 15 of a row to the lanes of the next row
constexpr int kDppRowBcast31 = 0x143;   // lane 31 to the lanes of rows 2 and 3

// Lane i receives x from the lane the control names; lanes without a source
// lane, and rows outside kRowMask, receive `old`.
template <int kCtrl, int kRowMask = 0xF, typename T>
__device__ __forceinline__ T dpp(T old, T x) {
    return __builtin_amdgcn_update_dpp(old, x, kCtrl, kRowMask, 0xF, false);
}

// The same with zero for lanes without a source lane (bound control), every
// row written: no register has to be cleared first, which matters for FP64
// values, whose moves cannot fold into the addition that consumes them.
template <int kCtrl, typename T>
__device__ __forceinline__ T dpp_z(T x) {
    return __builtin_amdgcn_update_dpp(T(0), x, kCtrl, 0xF, 0xF, true);
}

// x of lane l, as a wave-uniform value
template <typename T>
__device__ __forceinline__ T lane_value(T x, int l) {
    if constexpr (sizeof(T) == 8) {
        const unsigned long long v = __builtin_bit_cast(unsigned long long, x);
        const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)v, l);
        const unsigned hi = __builtin_amdgcn_readlane((int)(unsigned)(v >> 32), l);
        return __builtin_bit_cast(T, ((unsigned long long)hi << 32) | lo);
    } else {
        return __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), l));
    }
}

// One butterfly step of two values at once, by the swap instructions: lanes
// 0 - 31 hold a_i + a_{i+32}, lanes 32 - 63 b's; and across rows of 16, rows 0
// and 2 a's sum over their two rows, rows 1 and 3 b's.
template <typename T>
__device__ __forceinline__ T merge32(T a, T b) {
    constexpr int W = sizeof(T) / 4;
    unsigned x[W], y[W];
    __builtin_memcpy(x, &a, sizeof(T));
    __builtin_memcpy(y, &b, sizeof(T));
#pragma unroll
    for (int i = 0; i < W; ++i) {
        const auto v = __builtin_amdgcn_permlane32_swap(x[i], y[i], false, false);
        x[i] = v[0];
        y[i] = v[1];
    }
    __builtin_memcpy(&a, x, sizeof(T));
    __builtin_memcpy(&b, y, sizeof(T));
    return a + b;
}
template <typename T>
__device__ __forceinline__ T merge16(T a, T b) {
    constexpr int W = sizeof(T) / 4;
    unsigned x[W], y[W];
    __builtin_memcpy(x, &a, sizeof(T));
    __builtin_memcpy(y, &b, sizeof(T));
#pragma unroll
    for (int i = 0; i < W; ++i) {
        const auto v = __builtin_amdgcn_permlane16_swap(x[i], y[i], false, false);
        x[i] = v[0];
        y[i] = v[1];
    }
    __builtin_memcpy(&a, x, sizeof(T));
    __builtin_memcpy(&b, y, sizeof(T));
    return a + b;
}
// Sum over the 16 lanes of every row.
template <typename T>
__device__ __forceinline__ T row_sum(T x) {
    x += dpp_z<kDppRowRor + 8>(x);
    x += dpp_z<kDppRowRor + 4>(x);
    x += dpp_z<kDppQuadXor2>(x);
    x += dpp_z<kDppQuadXor1>(x);
    return x;
}

// Sum over the 64 lanes as a butterfly: every lane adds the value of lane
// i ^ 32, then i ^ 16, i ^ 8, i ^ 4, i ^ 2, i ^ 1; the result is the pairwise
// halving sum, the same bits in both forms.  (DPP: after the i ^ 8 step the
// values repeat with period 8 inside a row, so the rotation by 4 hands every
// lane the value of lane i ^ 4.)
template <bool kDpp, typename T>
__device__ __forceinline__ T wave_sum(T x) {
    if constexpr (!kDpp) {
#pragma unroll
        for (int o = kWave / 2; o > 0; o >>= 1) x += __shfl_xor(x, o, kWave);
        return __shfl(x, 0, kWave);  // one value for the whole column
    } else {
        x += __shfl_xor(x, 32, kWave);
        x += __shfl_xor(x, 16, kWave);
        return lane_value(row_sum(x), 0);
    }
}

// The sums of two columns in one butterfly, the same bits as one each.
template <int NK, typename T>
__device__ __forceinline__ void col_sum2(const T (&a)[NK], const T (&b)[NK], T &sa, T &sb) {
    T x = a[0], y = b[0];
#pragma unroll
    for (int c = 1; c < NK; ++c) {
        x += a[c];
        y += b[c];
    }
    x = merge32(x, y);
    x = row_sum(merge16(x, x));
    sa = lane_value(x, 0);
    sb = lane_value(x, 32);
}

// Inclusive scan over the lanes.  DPP: steps of 1, 2, 4, 8 inside each row,
// then the row totals carried into the rows after them.
template <bool kDpp, typename T>
__device__ __forceinline__ T wave_incl_prefix(T x) {
    if constexpr (!kDpp) {
        const int l = lane_id();
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const T y = __shfl_up(x, d, kWave);
            if (l >= d) x += y;
        }
    } else {
        x += dpp_z<kDppRowShr + 1>(x);
        x += dpp_z<kDppRowShr + 2>(x);
        x += dpp_z<kDppRowShr + 4>(x);
        x += dpp_z<kDppRowShr + 8>(x);
        x += dpp<kDppRowBcast15, 0xA>(T(0), x);
        x += dpp<kDppRowBcast31, 0xC>(T(0), x);
    }
    return x;
}

// Inclusive suffix scan.  DPP: steps of 1, 2, 4, 8 inside each row, after
// which lane 16 r holds the total t_r of row r; row 0 then adds
// t1 + (t2 + t3), row 1 t2 + t3, row 2 t3.
template <bool kDpp, typename T>
__device__ __forceinline__ T wave_incl_suffix(T x) {
    if constexpr (!kDpp) {
        const int l = lane_id();
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const T y = __shfl_down(x, d, kWave);
            if (l + d < kWave) x += y;
        }
        return x;
    } else {
        x += dpp_z<kDppRowShl + 1>(x);
        x += dpp_z<kDppRowShl + 2>(x);
        x += dpp_z<kDppRowShl + 4>(x);
        x += dpp_z<kDppRowShl + 8>(x);
        const T t3 = lane_value(x, 48);
        const T t23 = lane_value(x, 32) + t3;
        const T t123 = lane_value(x, 16) + t23;
        const int row = lane_id() >> 4;
        const T add = row == 0 ? t123 : row == 1 ? t23 : row == 2 ? t3 : T(0);
        return x + add;
    }
}

// v of lane i - 1 (lane 0: fill) and of lane i + 1 (lane 63: fill)
template <bool kDpp, typename T>
__device__ __forceinline__ T lane_prev(T fill, T v) {
    if constexpr (!kDpp) {
        const T y = __shfl_up(v, 1, kWave);
        return lane_id() == 0 ? fill : y;
    } else {
        return dpp<kDppWaveShr1>(fill, v);
    }
}
template <bool kDpp, typename T>
__device__ __forceinline__ T lane_next(T fill, T v) {
    if constexpr (!kDpp) {
        const T y = __shfl_down(v, 1, kWave);
        return lane_id() == kWave - 1 ? fill : y;
    } else {
        return dpp<kDppWaveShl1>(fill, v);
    }
}

// Sum over the layers: per-lane chunks first, then the butterfly; the result
// is the pairwise (halving) sum over the layers padded to 128.
template <int NK, bool kDpp = false, typename T>
__device__ __forceinline__ T col_sum(const T (&v)[NK]) {
    T s = v[0];
#pragma unroll
    for (int c = 1; c < NK; ++c) s += v[c];
    return wave_sum<kDpp>(s);
}

// o_k = sum_{l<k} v_l
template <int NK, bool kDpp = false, typename T>
__device__ __forceinline__ void col_excl_prefix(const T (&v)[NK], T (&o)[NK]) {
    T carry = T(0);
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        const T inc = wave_incl_prefix<kDpp>(v[c]);
        o[c] = (kDpp ? dpp_z<kDppWaveShr1>(inc) : lane_prev<false>(T(0), inc)) + carry;
        if (c + 1 < NK) carry += __shfl(inc, kWave - 1, kWave);
    }
}

// o_k = sum_{l>k} v_l
template <int NK, bool kDpp = false, typename T>
__device__ __forceinline__ void col_excl_suffix(const T (&v)[NK], T (&o)[NK]) {
    T carry = T(0);
#pragma unroll
    for (int c = NK - 1; c >= 0; --c) {
        const T inc = wave_incl_suffix<kDpp>(v[c]);
        o[c] = (kDpp ? dpp_z<kDppWaveShl1>(inc) : lane_next<false>(T(0), inc)) + carry;
        if (c > 0) carry += __shfl(inc, 0, kWave);
    }
}

// o_k = sum_{l>=k} v_l
template <int NK, bool kDpp = false, typename T>
__device__ __forceinline__ void col_incl_suffix(const T (&v)[NK], T (&o)[NK]) {
    T carry = T(0);
#pragma unroll
    for (int c = NK - 1; c >= 0; --c) {
        const T inc = wave_incl_suffix<kDpp>(v[c]);
        o[c] = inc + carry;
        if (c > 0) carry += __shfl(inc, 0, kWave);
    }
}

// o_k = v_{k-1}, o_0 = 0
template <int NK, bool kDpp = false, typename T>
__device__ __forceinline__ void col_up1(const T (&v)[NK], T (&o)[NK]) {
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        const T prev_last = (c > 0) ? __shfl(v[c > 0 ? c - 1 : 0], kWave - 1, kWave) : T(0);
        o[c] = (kDpp && c == 0) ? dpp_z<kDppWaveShr1>(v[c]) : lane_prev<kDpp>(prev_last, v[c]);
    }
}

// o_k = v_{k+1}; zero past the last layer (lanes past L hold zeros)
template <int NK, bool kDpp = false, typename T>
__device__ __forceinline__ void col_down1(const T (&v)[NK], T (&o)[NK]) {
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        const T next_first = (c < NK - 1) ? __shfl(v[c < NK - 1 ? c + 1 : c], 0, kWave) : T(0);
        o[c] = (kDpp && c == NK - 1) ? dpp_z<kDppWaveShl1>(v[c]) : lane_next<kDpp>(next_first, v[c]);
    }
}

// o_k = v_{k-s} (fill where k < s), 1 <= s <= 64, k = lane + 64 c
template <int NK, typename T>
__device__ __forceinline__ void col_shift_up(const T (&v)[NK], int s, T fill, T (&o)[NK]) {
    const int l = lane_id();
    if (s >= kWave) {
#pragma unroll
        for (int c = 0; c < NK; ++c) o[c] = c > 0 ? v[c > 0 ? c - 1 : 0] : fill;
        return;
    }
    const int src = (l - s) & (kWave - 1);
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        const T a = __shfl(v[c], src, kWave);
        const T b = c > 0 ? __shfl(v[c > 0 ? c - 1 : 0], src, kWave) : fill;
        o[c] = l >= s ? a : b;
    }
}

// o_k = v_{k+s} (fill past the last register chunk), 1 <= s <= 64
template <int NK, typename T>
__device__ __forceinline__ void col_shift_down(const T (&v)[NK], int s, T fill, T (&o)[NK]) {
    const int l = lane_id();
    if (s >= kWave) {
#pragma unroll
        for (int c = 0; c < NK; ++c) o[c] = c < NK - 1 ? v[c < NK - 1 ? c + 1 : c] : fill;
        return;
    }
    const int src = (l + s) & (kWave - 1);
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        const T a = __shfl(v[c], src, kWave);
        const T b = c < NK - 1 ? __shfl(v[c < NK - 1 ? c + 1 : c], src, kWave) : fill;
        o[c] = l + s < kWave ? a : b;
    }
}

// a b + c rounded once
__device__ __forceinline__ double fmadd(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fmadd(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// 1 / x (layer thicknesses, pivots): the hardware reciprocal refined to the
// last place in three (FP64: five) instructions, where the division takes
// eleven (with divisions and the FP64 root in their places, in turn on one
// device: level-7 globe of 60 layers, mixed, 84.3 against 80.5 ms; 256 x 256 x
// 60 with the column solve 69.2 against 66.6; 512 x 512 x 60 1.002x).  Not
// rounded correctly, but the results' errors against 64 bits come out the same
// with either.  0 and infinity give NaN where a division gives infinity and 0:
// a column with such a thickness has no finite value either way, since its sums
// (of thickness, and of thickness x velocity) are then not finite or 0 x
// infinity.
template <typename R>
__device__ __forceinline__ R recip(R x) {
    R r;
    if constexpr (sizeof(R) == 4) {
        r = __builtin_amdgcn_rcpf(x);
    } else {
        r = __builtin_amdgcn_rcp(x);
        r = fmadd(fmadd(-x, r, R(1)), r, r);
    }
    return fmadd(fmadd(-x, r, R(1)), r, r);
}

// o_k = v_{k-s} and v_{k+s}, for rows whose values from outside the column are
// multiplied by zero: with one register chunk they may be any row's.
template <int NK, typename T>
__device__ __forceinline__ void col_shift_any(const T (&v)[NK], int s, T (&a)[NK], T (&b)[NK]) {
    if constexpr (NK == 1) {
        const int l = lane_id();
        a[0] = __shfl(v[0], (l - s) & (kWave - 1), kWave);
        b[0] = __shfl(v[0], (l + s) & (kWave - 1), kWave);
    } else {
        col_shift_up<NK>(v, s, T(0), a);
        col_shift_down<NK>(v, s, T(0), b);
    }
}

// Solves lo_k x_{k-1} + di_k x_k + up_k x_{k+1} = d_k over the layers of a
// column, x returned in d.  Rows past the last layer must be the identity
// (lo = up = 0, di = 1, d = 0) and the first and last rows must not couple
// outwards (lo_0 = up_{L-1} = 0).  Parallel cyclic reduction (Hockney): in
// round r every row eliminates its couplings to the rows s = 2^r above and
// below with those rows' equations, so after ceil(log2 L) rounds each row
// holds one unknown.  Every lane works in every round, the cross-lane reads
// are register shuffles, and for the diagonally dominant systems of implicit
// diffusion no pivoting is needed.
//
// The shuffles' LDS port bounds it (six rounds of eight FP64 shuffles were a
// third of the edge pass with mixing).  Rows are kept divided by their
// diagonal, which leaves three columns to shift each way; the first round
// shifts by DPP, the round of 32 reads the same lane for above and below, and
// the last round moves on the right-hand side only.  A row's coupling past
// the column's end is zero in every round, so with one chunk the shifts wrap
// around without a select.  One edge pass with mixing on 256 x 256 x 60: FP64
// 282 -> 192 us, FP32 219 -> 154; level-6 globe, 100 layers, biharmonic: FP64
// 320 -> 253 us, FP32 191 -> 158.
template <int NK, typename T>
__device__ __forceinline__ void col_tridiag_solve(int L, T (&lo)[NK], T (&di)[NK], T (&up)[NK], T (&d)[NK]) {
    T loA[NK], upA[NK], dA[NK], loB[NK], upB[NK], dB[NK];
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        const T q = recip<T>(di[c]);
        lo[c] *= q;
        up[c] *= q;
        d[c] *= q;
    }
    auto round = [&](bool last) {
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            const T q = recip<T>(fmadd(-lo[c], upA[c], fmadd(-up[c], loB[c], T(1))));
            d[c] = fmadd(-lo[c], dA[c], fmadd(-up[c], dB[c], d[c])) * q;
            if (!last) {
                lo[c] = -lo[c] * loA[c] * q;
                up[c] = -up[c] * upB[c] * q;
            }
        }
    };
    if (L > 1) {
        col_up1<NK, true>(lo, loA);
        col_up1<NK, true>(up, upA);
        col_up1<NK, true>(d, dA);
        col_down1<NK, true>(lo, loB);
        col_down1<NK, true>(up, upB);
        col_down1<NK, true>(d, dB);
        round(false);
    }
    int s = 2;
    for (; 2 * s < L && s < 32; s <<= 1) {
        col_shift_any<NK>(lo, s, loA, loB);
        col_shift_any<NK>(up, s, upA, upB);
        col_shift_any<NK>(d, s, dA, dB);
        round(false);
    }
    if constexpr (NK == 1) {
        if (s >= L) return;
        if (s == 32) {
            const int other = lane_id() ^ 32;
            loB[0] = __shfl(lo[0], other, kWave);
            upA[0] = __shfl(up[0], other, kWave);
            dA[0] = dB[0] = __shfl(d[0], other, kWave);
        } else {
            col_shift_any<NK>(lo, s, loA, loB);
            col_shift_any<NK>(up, s, upA, upB);
            col_shift_any<NK>(d, s, dA, dB);
        }
        round(true);
    } else {
        for (; s < L; s <<= 1) {
            col_shift_any<NK>(lo, s, loA, loB);
            col_shift_any<NK>(up, s, upA, upB);
            col_shift_any<NK>(d, s, dA, dB);
            round(2 * s >= L);
        }
    }
}

// Quotients by 3 and 6 in the bits of x / d but without the division
// sequence (about ten instructions).  With r = RN(1/d), q = RN(x r) and the
// residual x - q d (exact in one fused multiply-add), Markstein's theorem
// makes RN(q + (x - q d) r) the correctly rounded quotient whenever q lies
// within one ulp of x / d, which holds when |1 - d r| <= 2^-(p+1) for
// precision p: 1 - 3 RN(1/3) is 2^-54 in FP64 and 2^-25 in FP32 (and RN(1/6)
// is RN(1/3) / 2).  Valid while the quotient and the residual stay normal
// (|x / d| above about 2^-960 in FP64, 2^-100 in FP32); x = -0 gives +0.
template <typename T>
__device__ __forceinline__ T div_by_near(T x, T d, T r) {
    const T q = x * r;
    return fmadd(fmadd(-q, d, x), r, q);
}

// The 3/4 combination is one fused multiply-add with an explicit operand
// order (1/4 x is exact), so every kernel that forms it rounds alike.
template <typename T>
__device__ __forceinline__ T combine(int mode, T b, T x) {
    switch (mode) {
        case COMB_34: return fmadd(T(0.75), b, T(0.25) * x);
        case COMB_THIRD: return div_by_near(b, T(3), T(1) / T(3)) + div_by_near(T(2) * x, T(3), T(1) / T(3));
        case COMB_HALF: return T(0.5) * (b + x);
        default: return x;
    }
}

// Lane k holds layer k (chunk c: layer k + 64 c).  Lanes past the last layer
// load layer L - 1 (always in bounds), so loads are never predicated: no
// branches split the load stream and all loads of a stencil can be in flight
// together.  What those lanes loaded is zeroed where it can reach a sum or a
// scan over the layers; elsewhere it only feeds results that are not stored.
template <int NK>
__device__ __forceinline__ void lane_layers(int L, int (&kk)[NK], bool (&ok)[NK]) {
    const int lane = lane_id();
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        const int k = lane + c * kWave;
        ok[c] = k < L;
        kk[c] = ok[c] ? k : L - 1;
    }
}

// Column access.  `col` is the first layer of a column and must be
// wave-uniform; the lane reads or writes layer k.  The address is a scalar
// base plus a 32-bit lane offset, a form the load and store instructions take
// directly, so the columns of a stencil share one offset register and need no
// 64-bit address arithmetic per lane (where scalar registers run short, the
// compiler still forms some of the addresses in vector registers).  Measured
// on the C1 edge pass: 6% faster than per-lane 64-bit addresses.
typedef __attribute__((address_space(1))) char global_char;

template <typename T>
__device__ __forceinline__ global_char *uniform_global(const T *col) {
    const unsigned long long p = reinterpret_cast<unsigned long long>(col);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)p);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(p >> 32));
    return (global_char *)(((unsigned long long)hi << 32) | lo);
}

template <typename T>
__device__ __forceinline__ T col_ld(const T *col, int k) {
    return *(const __attribute__((address_space(1))) T *)(uniform_global(col) + (unsigned)k * (unsigned)sizeof(T));
}

template <typename T>
__device__ __forceinline__ void col_st(T *col, int k, T v) {
    *(__attribute__((address_space(1))) T *)(uniform_global(col) + (unsigned)k * (unsigned)sizeof(T)) = v;
}

// Layer k of the column that starts off elements into arr.  kWide: a 64-bit
// scalar base per column (col_ld).  Otherwise (arrays below 4 GiB) through
// one buffer descriptor of the whole array, with the column's byte offset in
// a single 32-bit scalar register and the layer's in the lane's: half the
// scalar registers per column and no 64-bit address arithmetic, which keeps
// the edge pass, with its ~30 columns, from spilling scalar registers.
template <bool kWide, typename T>
__device__ __forceinline__ T col_ldv(const T *arr, size_t off, int k) {
    if constexpr (kWide) {
        return col_ld(arr + off, k);
    } else {
        const __amdgpu_buffer_rsrc_t r =
            __builtin_amdgcn_make_buffer_rsrc((void *)uniform_global(arr), (short)0, -1, 0x00020000);
        const unsigned so = __builtin_amdgcn_readfirstlane((unsigned)(off * sizeof(T)));
        if constexpr (sizeof(T) == 8)
            return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, (unsigned)k * 8u, so, 0));
        else
            return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, (unsigned)k * 4u, so, 0));
    }
}

// ---------------------------------------------------------------------------
// Baroclinic forward Euler (Algorithm 1): cell pass.
// kAdd: the velocity is X + ubar_add (ubar_add non-null), else X itself.
// ---------------------------------------------------------------------------
template <int NK, typename R, bool kAdd>
__device__ __forceinline__ void fe_cell_body(const FECellArgs<R> &a, int col) {
    const DevMesh &m = a.m;
    const int i = col;
    if (i >= m.C) return;
    const int L = a.L;
    const size_t base = (size_t)i * L;
    int kk[NK];
    bool ok[NK];
    lane_layers<NK>(L, kk, ok);
    if (!m.cmask[i]) {
#pragma unroll
        for (int c = 0; c < NK; ++c)
            if (ok[c]) {
                a.B[base + kk[c]] = R(0);
                a.Wtop[base + kk[c]] = R(0);
                if (a.D1) a.D1[base + kk[c]] = R(0);
            }
        if (lane_id() == 0) a.Kbot[i] = 0.0;
        return;
    }
    double hi[NK];
    R divhu[NK], divu[NK], K[NK];
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        hi[c] = col_ld(a.h + base, kk[c]);
        divhu[c] = divu[c] = K[c] = R(0);
    }
    // Padded slots hold a valid index with zero coefficients, so the stencil
    // is unrolled to its full width.
#pragma unroll
    for (int j = 0; j < kMaxEdges; ++j) {
        const int e = m.cell_edges[i * kMaxEdges + j];
        const int nb = m.cell_nbrs[i * kMaxEdges + j];
        const R cd = (R)m.cell_div[i * kMaxEdges + j];
        const R ck = (R)m.cell_ke[i * kMaxEdges + j];
        const R add = kAdd ? (R)a.ubar_add[e] : R(0);
        const size_t eb = (size_t)e * L, nbb = (size_t)nb * L;
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            const R x = col_ld(a.X + eb, kk[c]);
            const double hn = col_ld(a.h + nbb, kk[c]);
            const R u = ok[c] ? x + add : R(0);
            const R he = (R)(0.5 * (hi[c] + hn));
            divhu[c] += cd * (he * u);
            divu[c] += cd * u;
            K[c] += ck * (u * u);
        }
    }
    R w[NK];
    if (a.frac) {
        // z-star: T^h_k = -frac_k sum_l div(h u)_l, and w_k - w_{k+1} = -div_k - T^h_k
        const R tot = col_sum<NK, kDppFor<R>>(divhu);
        R src[NK];
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            const R th = -(R)col_ld(a.frac + base, kk[c]) * tot;
            src[c] = ok[c] ? (-divhu[c] - th) : R(0);
        }
        col_incl_suffix<NK, kDppFor<R>>(src, w);
    } else {
#pragma unroll
        for (int c = 0; c < NK; ++c) w[c] = R(0);
    }
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        if (ok[c]) {
            col_st(a.B + base, kk[c], K[c] - (R)a.nu_h * divu[c]);
            if (a.D1) col_st(a.D1 + base, kk[c], divu[c]);
            col_st(a.Wtop + base, kk[c], w[c]);
            if (kk[c] == L - 1) a.Kbot[i] = (double)K[c];
        }
    }
}

// ---------------------------------------------------------------------------
// Baroclinic forward Euler split by cells (meshes with factored weights).
//
// The direct edge pass gathers 30 layer columns per edge, 11 GB per launch of
// a 512 x 512 x 60 mesh, and those gathers bound it (0.87 of its 1.07 ms).
// With factored weights the 20 columns of the reconstruction belong to the two
// cells: one wavefront per cell loads its 6 edges, the 6 edges that leave its
// vertices, h of itself and its neighbours (20 columns for 6 half edges, and
// no vorticity array in between), and writes the cell's share of each edge's
// horizontal terms.  The edge pass then reads the two shares.  On that mesh in
// FP64 the cell, vertex and edge passes took 0.22 + 0.12 + 1.07 ms; the split
// takes 0.55 (cells) + 0.53 (edges), in FP32 0.14 + 0.09 + 0.76 against 0.29 +
// 0.48.  Both parts are now near the rate of HBM: 2.45 and 2.41 GB per launch
// by the counters, 4.4 and 4.5 TB/s where a copy reaches 5.1.
//
// With x = s l u / 2, t the same of ut, f / 2, q = zeta_e / 2 (zeta_e the mean
// of the edge's two vertex vorticities) and y = f t + q x, edge a's share of
// d_a (Coriolis on ut + vorticity flux of u) is, as in half_sums,
//   S_a (f_a T + q_a X + Y') + f_a (T - Yt) + q_a (X - Yx) + (Y' - Yy) - 2 y_a
//     - S_n (f_a Pt_a + q_a Px_a + Py_a),
// capitals the sums over the cell (Y weighted by S), P the sums before a.
// ---------------------------------------------------------------------------
// Layer k of the column that starts off elements into arr, through the array's
// base and a 32-bit lane offset (arrays below 4 GiB), or (kWide) the column's
// 64-bit base.
template <bool kWide, typename T>
__device__ __forceinline__ T col_ldo(const T *arr, size_t off, int k) {
    if constexpr (kWide) return col_ld(arr + off, k);
    const unsigned vo = (unsigned)(off * sizeof(T)) + (unsigned)k * (unsigned)sizeof(T);
    return *(const __attribute__((address_space(1))) T *)((const global_char *)(unsigned long long)arr + vo);
}
template <bool kWide, typename T>
__device__ __forceinline__ void col_sto(T *arr, size_t off, int k, T v) {
    if constexpr (kWide) {
        col_st(arr + off, k, v);
    } else {
        const unsigned vo = (unsigned)(off * sizeof(T)) + (unsigned)k * (unsigned)sizeof(T);
        *(__attribute__((address_space(1))) T *)((global_char *)(unsigned long long)arr + vo) = v;
    }
}

template <typename T>
using const_ptr = const __attribute__((address_space(4))) T *;

template <int NK, typename R, bool kAdd, bool kWide>
__device__ __forceinline__ void fe_split_body(const FESplitArgs<R> &a, int i) {
    if (i >= a.C) return;
    const int L = a.L;
    const size_t base = (size_t)i * L;
    int kk[NK];
    bool ok[NK];
    lane_layers<NK>(L, kk, ok);
    if (!a.cmask[i]) {
#pragma unroll
        for (int c = 0; c < NK; ++c)
            if (ok[c]) {
                a.Wtop[base + kk[c]] = R(0);
                if (a.D1) a.D1[base + kk[c]] = R(0);
            }
        if (lane_id() == 0) a.Kbot[i] = 0.0;
        return;
    }
    // The record through the constant address space, so that its loads stay
    // scalar also past the stores.  They are issued in three groups, each well
    // before its use and held there by scheduling barriers: left alone the
    // compiler loads every coefficient where it is used, and a wavefront spends
    // its time in a dozen scalar waits one after another.
    const_ptr<CellRec<R>> q = (const_ptr<CellRec<R>>)(unsigned long long)(a.rec + i);
    const double *ubar = kAdd ? a.ubar_add : a.ubar_sub;
    int own[6];
    const int n = q->n;
    const unsigned side = q->side;
    R u[6][NK], o[6][NK], hs[6][NK], fr[NK];
    R lhs[6], ke[6], ub[6], uo[6], curl[18];
    {
        double hi[NK], hn[6][NK];
#pragma unroll
        for (int b = 0; b < 6; ++b) {
            own[b] = q->own[b];
            const size_t eb = (size_t)own[b] * L, ob = (size_t)q->out[b] * L, nb = (size_t)q->nbr[b] * L;
#pragma unroll
            for (int c = 0; c < NK; ++c) {
                u[b][c] = col_ldo<kWide>(a.X, eb, kk[c]);
                o[b][c] = col_ldo<kWide>(a.X, ob, kk[c]);
                hn[b][c] = col_ldo<kWide>(a.h, nb, kk[c]);
            }
        }
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            hi[c] = col_ldo<kWide>(a.h, base, kk[c]);
            fr[c] = a.frac ? (R)col_ldo<kWide>(a.frac, base, kk[c]) : R(0);
        }
#pragma unroll
        for (int b = 0; b < 6; ++b) {
            ub[b] = (R)ubar[own[b]];
            if constexpr (kAdd) uo[b] = (R)ubar[q->out[b]];
        }
#pragma unroll
        for (int m = 0; m < 18; ++m) curl[m] = q->curl[m];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int b = 0; b < 6; ++b)
#pragma unroll
            for (int c = 0; c < NK; ++c) hs[b][c] = (R)(hi[c] + hn[b][c]);
    }
    R tot[NK], K[NK], x[6][NK], t[6][NK], z[6][NK], bern[NK], X[NK];
#pragma unroll
    for (int b = 0; b < 6; ++b)
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            t[b][c] = kAdd ? u[b][c] : u[b][c] - ub[b];
            if constexpr (kAdd) {
                u[b][c] += ub[b];
                o[b][c] += uo[b];
            }
        }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int b = 0; b < 6; ++b) {
        lhs[b] = q->lhs[b];
        ke[b] = q->ke[b];
    }
    const R ia = q->ia;
#pragma unroll
    for (int c = 0; c < NK; ++c) {
#pragma unroll
        for (int m = 0; m < 6; ++m)
            z[m][c] = curl[3 * m] * u[m][c] + curl[3 * m + 1] * u[(m + 1) % 6][c] + curl[3 * m + 2] * o[m][c];
        if (n < 6) z[5][c] = z[4][c];   // the vertex before edge 0 of a pentagon
    }
    __builtin_amdgcn_sched_barrier(0);
    R fh[6], S[6], nr[6];
#pragma unroll
    for (int b = 0; b < 6; ++b) {
        fh[b] = q->fh[b];
        S[b] = q->S[b];
        nr[b] = q->rk[b];
    }
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        tot[c] = K[c] = X[c] = R(0);
#pragma unroll
        for (int b = 0; b < 6; ++b) {
            x[b][c] = lhs[b] * u[b][c];
            t[b][c] = lhs[b] * t[b][c];
            K[c] += ke[b] * (u[b][c] * u[b][c]);
            X[c] += x[b][c];
            tot[c] += x[b][c] * hs[b][c];
        }
        const R divu = R(2) * ia * X[c];
        bern[c] = K[c] - (R)a.nu_h * divu;
        if (a.D1 && ok[c]) col_sto<kWide>(a.D1, base, kk[c], divu);
    }
    __builtin_amdgcn_sched_barrier(0);
    // z-star: T^h_k = -frac_k sum_l div(h u)_l, and w_k - w_{k+1} = -div_k - T^h_k
    R w[NK];
    if (a.frac) {
        R src[NK];
#pragma unroll
        for (int c = 0; c < NK; ++c) tot[c] = ok[c] ? ia * tot[c] : R(0);
        const R sum = col_sum<NK, kDppFor<R>>(tot);
#pragma unroll
        for (int c = 0; c < NK; ++c) src[c] = ok[c] ? fr[c] * sum - tot[c] : R(0);
        col_incl_suffix<NK, kDppFor<R>>(src, w);
    } else {
#pragma unroll
        for (int c = 0; c < NK; ++c) w[c] = R(0);
    }
#pragma unroll
    for (int c = 0; c < NK; ++c)
        if (ok[c]) {
            col_sto<kWide>(a.Wtop, base, kk[c], w[c]);
            if (kk[c] == L - 1) a.Kbot[i] = (double)K[c];
        }
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        R T = R(0), Y = R(0), Yx = R(0), Yt = R(0), Yy = R(0), y[6];
#pragma unroll
        for (int b = 0; b < 6; ++b) {
            const R qb = z[(b + 5) % 6][c] + z[b][c];
            y[b] = fh[b] * t[b][c] + qb * x[b][c];
            T += t[b][c];
            Y += y[b];
            if (b > 0) {
                Yx += S[b - 1] * x[b][c];
                Yt += S[b - 1] * t[b][c];
                Yy += S[b - 1] * y[b];
            }
        }
        const R Dx = X[c] - Yx, Dt = T - Yt, Dy = Y - Yy;
        R Px = R(0), Pt = R(0), Py = R(0);
#pragma unroll
        for (int b = 0; b < 6; ++b) {
            const R zp = z[(b + 5) % 6][c], f = fh[b], qb = zp + z[b][c];
            R g = bern[c] + (f * Dt + (qb * Dx + Dy)) - R(2) * y[b] - ((R)a.nu_h * nr[b]) * (z[b][c] - zp);
            if (b > 0) g += S[b - 1] * (f * T + (qb * X[c] + Y)) - S[5] * (f * Pt + (qb * Px + Py));
            Px += x[b][c];
            Pt += t[b][c];
            Py += y[b];
            if (b < n && ok[c]) {
                R *const G = ((side >> b) & 1u) ? a.GB : a.GA;
                col_sto<kWide>(G, (size_t)own[b] * L, kk[c], g);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Baroclinic forward Euler: vertex pass (relative vorticity of X + ubar_add)
// ---------------------------------------------------------------------------
template <int NK, typename R, bool kAdd, int Q>
__device__ __forceinline__ void fe_vertex_body(const FEVertexArgs<R> &a, int first) {
    const DevMesh &m = a.m;
    if (first >= m.V) return;
    const int L = a.L;
    int kk[NK];
    bool ok[NK];
    lane_layers<NK>(L, kk, ok);
    int vi[Q];
    bool has[Q];
    R x[Q][3][NK], cr[Q][3], add[Q][3];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        has[q] = first + q < m.V;
        vi[q] = has[q] ? first + q : first;
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const int e = m.vert_edges[vi[q] * 3 + j];
            cr[q][j] = (R)m.vert_curl[vi[q] * 3 + j];
            add[q][j] = kAdd ? (R)a.ubar_add[e] : R(0);
            const size_t eb = (size_t)e * L;
#pragma unroll
            for (int c = 0; c < NK; ++c) x[q][j][c] = col_ld(a.X + eb, kk[c]);
        }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        if (!has[q]) continue;
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            R z = R(0);
#pragma unroll
            for (int j = 0; j < 3; ++j) z += cr[q][j] * (x[q][j][c] + add[q][j]);
            if (ok[c]) col_st(a.Z + (size_t)vi[q] * L, kk[c], z);
        }
    }
}

// ---------------------------------------------------------------------------
// Biharmonic viscosity: the vector Laplacian of u at edges, then the
// divergence of that field at cells (its curl at vertices is the vertex pass
// applied to it).
// ---------------------------------------------------------------------------
template <int NK, typename R, int Q>
__device__ __forceinline__ void lap_body(const LapArgs<R> &a, int first) {
    const DevMesh &m = a.m;
    if (first >= m.E) return;
    const int L = a.L;
    int kk[NK];
    bool ok[NK];
    lane_layers<NK>(L, kk, ok);
    int ei[Q];
    bool has[Q];
    R d1[Q][NK], d2[Q][NK], z1[Q][NK], z2[Q][NK];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        has[q] = first + q < m.E;
        const int e = ei[q] = has[q] ? first + q : first;
        const size_t b1 = (size_t)m.edge_cells[2 * e] * L, b2 = (size_t)m.edge_cells[2 * e + 1] * L;
        const size_t w1 = (size_t)m.edge_verts[2 * e] * L, w2 = (size_t)m.edge_verts[2 * e + 1] * L;
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            d1[q][c] = col_ld(a.D + b1, kk[c]);
            d2[q][c] = col_ld(a.D + b2, kk[c]);
            z1[q][c] = col_ld(a.Z + w1, kk[c]);
            z2[q][c] = col_ld(a.Z + w2, kk[c]);
        }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        if (!has[q]) continue;
        const int e = ei[q];
        const bool wet = m.emask[e] != 0;
        const R idc = (R)m.inv_dc[e], idv = (R)m.inv_dv[e];
#pragma unroll
        for (int c = 0; c < NK; ++c)
            if (ok[c])
                col_st(a.out + (size_t)e * L, kk[c],
                       wet ? (d2[q][c] - d1[q][c]) * idc - (z2[q][c] - z1[q][c]) * idv : R(0));
    }
}

template <int NK, typename R, int Q>
__device__ __forceinline__ void div_body(const DivArgs<R> &a, int first) {
    const DevMesh &m = a.m;
    if (first >= m.C) return;
    const int L = a.L;
    int kk[NK];
    bool ok[NK];
    lane_layers<NK>(L, kk, ok);
    int ci[Q];
    bool has[Q];
    R x[Q][kMaxEdges][NK], cd[Q][kMaxEdges];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        has[q] = first + q < m.C;
        const int i = ci[q] = has[q] ? first + q : first;
#pragma unroll
        for (int j = 0; j < kMaxEdges; ++j) {
            const size_t eb = (size_t)m.cell_edges[i * kMaxEdges + j] * L;
            cd[q][j] = (R)m.cell_div[i * kMaxEdges + j];
#pragma unroll
            for (int c = 0; c < NK; ++c) x[q][j][c] = col_ld(a.X + eb, kk[c]);
        }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        if (!has[q]) continue;
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            R d = R(0);
#pragma unroll
            for (int j = 0; j < kMaxEdges; ++j) d += cd[q][j] * x[q][j][c];
            if (ok[c]) col_st(a.out + (size_t)ci[q] * L, kk[c], d);
        }
    }
}

// ---------------------------------------------------------------------------
// Baroclinic forward Euler: edge pass (Algorithm 1 and the stage combination)
//
// The direct-gather and the LDS-staged kernels share everything after the
// operand loads: fe_edge_finish receives the column values of the edge, its
// cells and vertices and the accumulated reconstruction sums.
// ---------------------------------------------------------------------------
// TRiSK weight pairs (W / 4, W (f_e + f_j) / 2) of the edge pass in its real type.
template <typename R>
__device__ __forceinline__ const R *wpair_of(const DevMesh &m);
template <>
__device__ __forceinline__ const double *wpair_of<double>(const DevMesh &m) { return m.wpair; }
template <>
__device__ __forceinline__ const float *wpair_of<float>(const DevMesh &m) { return m.wpair_f; }

// The barotropic velocity at edge e as the pass computes with it: FP64 as
// stored, or (FP32 pass) the copy rounded to FP32 once per pass.
template <typename R>
__device__ __forceinline__ R ubar_at(const FEEdgeArgs<R> &a, const double *ubar, int e) {
    if constexpr (sizeof(R) == 4) return a.ubar_r[e];
    else return ubar[e];
}

template <int NK, typename R>
struct EdgeOperands {
    R u[NK], ut[NK], za[NK], zb[NK], B1[NK], B2[NK], W1[NK], W2[NK];
    double h1[NK], h2[NK], r1[NK], r2[NK];
    R cor[NK], vor[NK];
    R lap2[NK];   // lap(lap u) (biharmonic runs; zero otherwise)
    // split pass: u^n of the stage combination, and the two cells' scalars
    R un[NK];
    double K1, K2, z1, z2, H1, H2, ubn;
};

// sqrt(x) rounded to R (of the bottom layer's kinetic energy; NaN of an infinite
// one).  FP32: one Newton step from the hardware's reciprocal root is good to
// about 1e-15 before the rounding.
template <typename R>
__device__ __forceinline__ R sqrt_to(double x) {
    if constexpr (sizeof(R) == 4) {
        const double y = __builtin_amdgcn_rsq(x), v = x * y;
        const double w = fmadd(fmadd(-v, v, x), 0.5 * y, v);
        return x > 1e-300 ? (R)w : (x >= 0.0 ? R(0) : R(NAN));
    } else {
        return sqrt(x);
    }
}

// kMix: D^u is left out of the tendency and applied by the implicit column
// solve of Algorithm 2 (the vertical-mixing form of the stage).
template <int NK, typename R, bool kMix, bool kWide, bool kSplit = false>
__device__ __forceinline__ void fe_edge_finish(const FEEdgeArgs<R> &a, int e, int c1, int c2, double idc, double idv,
                                               const EdgeOperands<NK, R> &o) {
    const int lane = lane_id();
    const DevMesh &m = a.m;
    const int L = a.L;
    const size_t base = (size_t)e * L;
    int kk[NK];
    bool ok[NK];
    lane_layers<NK>(L, kk, ok);
    // Operands of lanes past the last layer are copies of layer L - 1; the
    // edge thickness and the PGF differences, which reach the column sums and
    // scans, are zeroed there.
    R he[NK];
    double hed[NK];
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        hed[c] = ok[c] ? 0.5 * (o.h1[c] + o.h2[c]) : 0.0;
        he[c] = (R)hed[c];
    }
    // Pressure gradient in z-star layers from the column differences, in FP64
    // in both modes: its two terms cancel down to the density anomaly.
    double pgf[NK];
    {
        double drh[NK], dh[NK], sp[NK], ss[NK];
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            drh[c] = ok[c] ? o.r2[c] * o.h2[c] - o.r1[c] * o.h1[c] : 0.0;
            dh[c] = ok[c] ? o.h2[c] - o.h1[c] : 0.0;
        }
        col_excl_prefix<NK, kDppFor<R>>(drh, sp);
        col_excl_suffix<NK, kDppFor<R>>(dh, ss);
        const double dH = kSplit ? o.H2 - o.H1 : m.H[c2] - m.H[c1];
        const double pgf_scale = idc * a.irho0;
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            const double dp = a.g * (sp[c] + 0.5 * drh[c]);
            const double dz = -dH + ss[c] + 0.5 * dh[c];
            pgf[c] = -(dp + a.g * (0.5 * (o.r1[c] + o.r2[c])) * dz) * pgf_scale;
        }
    }

    // Vertical advection and vertical viscosity at interior interfaces.
    R uu[NK], hu[NK], at[NK], tau[NK], atn[NK], taun[NK];
    col_up1<NK, kDppFor<R>>(o.u, uu);
    col_up1<NK, kDppFor<R>>(he, hu);
    const R nu_v = (R)a.nu_v;
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        const int k = lane + c * kWave;
        if (k >= 1 && k < L) {
            const R dzt = (uu[c] - o.u[c]) * recip<R>(R(0.5) * (hu[c] + he[c]));
            const R we = R(0.5) * (o.W1[c] + o.W2[c]);
            at[c] = we * dzt;
            tau[c] = nu_v * dzt;
        } else {
            at[c] = R(0);
            tau[c] = R(0);
        }
    }
    col_down1<NK, kDppFor<R>>(at, atn);
    col_down1<NK, kDppFor<R>>(tau, taun);
    const R speed = sqrt_to<R>(kSplit ? o.K1 + o.K2 : a.Kbot[c1] + a.Kbot[c2]);
    const R gz = (R)(a.g * (kSplit ? o.z2 - o.z1 : a.zeta[c2] - a.zeta[c1]) * idc);
    const R dt = (R)a.dt, nu_h = (R)a.nu_h, c_drag = (R)a.c_drag;
    const R ridc = (R)idc, ridv = (R)idv;

    // (lanes past the last layer run along and are cleared, rather than
    // branched around: a branch keeps their loads from starting early)
    R ut1[NK];
    double hut1[NK], hu_in[NK];
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        const int k = lane + c * kWave;
        if (k == L - 1) taun[c] = c_drag * speed * o.u[c];
        const R vadv = R(0.5) * (at[c] + atn[c]);
        const R du = kMix ? R(0) : (tau[c] - taun[c]) * recip<R>(he[c]);
        R next;
        if constexpr (kSplit) {
            // B1, B2: the two cells' shares of the horizontal terms
            const R hor = (o.B1[c] - o.B2[c]) * ridc;
            const R tu = hor - vadv + (R)pgf[c] - (R)a.nu4 * o.lap2[c];
            next = o.ut[c] + dt * (tu + du + gz);
        } else {
            const R gradB = (o.B2[c] - o.B1[c]) * ridc;
            const R curlp = (o.zb[c] - o.za[c]) * ridv;
            const R tu = -gradB + o.vor[c] - vadv + (R)pgf[c] - nu_h * curlp - (R)a.nu4 * o.lap2[c];
            next = o.ut[c] + dt * (o.cor[c] + tu + du + gz);
        }
        ut1[c] = k < L ? next : R(0);
        hut1[c] = hed[c] * (double)ut1[c];
        hu_in[c] = hed[c] * (double)o.u[c];
    }
    // Column sums that feed the barotropic forcing and the reconciliation are
    // formed in FP64 in both modes.
    double Sh, Shut;
    col_sum2<NK>(hed, hut1, Sh, Shut);
    const double G = Shut / (Sh * a.dt);
    const R dtG = (R)(a.dt * G);
    R x[NK];
#pragma unroll
    for (int c = 0; c < NK; ++c) x[c] = (lane + c * kWave < L) ? ut1[c] - dtG : R(0);
    if constexpr (kMix) {
        // Algorithm 2: u1 - dt D^u(u1) = ut1 + ubar with the drag speed of the
        // input, then ut1 = u1 - ubar (ubar: the input's barotropic velocity).
        // Solved for the change y of ut1: (1 - dt D^u) y = dt D^u(ut1 + ubar),
        // whose right-hand side takes the differences between layers, in which
        // ubar drops out but for the drag.  The rounding of the solve is then
        // relative to y, not to the whole velocity.  Relative error of u against
        // 64 bits after 20 mixed steps on 64 x 64 cells, solved for u1 with rows
        // as they are, with rows divided by their diagonal, and for y (6.1e-7
        // without mixing): 30 layers 7.1e-7, 7.9e-7, 6.2e-7; 60 layers 2.0e-6,
        // 1.1e-6, 6.3e-7.  Times within 1% (256 x 256 x 60 FP64, level-6 globe x 100 mixed).
        const R ubin = (R)((a.ubar_add ? a.ubar_add[e] : 0.0) + (a.ubar_sub ? a.ubar_sub[e] : 0.0));
        R Aup[NK], Adn[NK], lo[NK], di[NK], up[NK], xu[NK], xd[NK], y[NK];
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            const int k = lane + c * kWave;
            Aup[c] = (k >= 1 && k < L) ? nu_v / (R(0.5) * (hu[c] + he[c])) : R(0);
        }
        col_down1<NK, kDppFor<R>>(Aup, Adn);
        col_up1<NK, kDppFor<R>>(x, xu);
        col_down1<NK, kDppFor<R>>(x, xd);
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            const int k = lane + c * kWave;
            if (k == L - 1) Adn[c] = c_drag * speed;
            const bool in = k < L;
            lo[c] = in ? -dt * Aup[c] / he[c] : R(0);
            const R below = dt * Adn[c] / he[c];   // the drag's, at the bottom
            up[c] = (in && k < L - 1) ? -below : R(0);
            di[c] = in ? R(1) + dt * (Aup[c] + Adn[c]) / he[c] : R(1);
            y[c] = lo[c] * (x[c] - xu[c]) + up[c] * (x[c] - xd[c]);
            if (k == L - 1) y[c] -= below * (x[c] + ubin);
        }
        col_tridiag_solve<NK, R>(L, lo, di, up, y);
#pragma unroll
        for (int c = 0; c < NK; ++c) x[c] = (lane + c * kWave < L) ? x[c] + y[c] : R(0);
    }
    const double ubn = a.Un ? (kSplit ? o.ubn : a.ubar_n[e]) : 0.0;
    R outv[NK];
    double hp[NK];
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        const int k = lane + c * kWave;
        R utn = R(0);
        if (a.Un) {
            const double un = kSplit ? (double)o.un[c] : (double)col_ldv<kWide>(a.Un, base, kk[c]);
            utn = k < L ? (R)(un - ubn) : R(0);
        }
        outv[c] = (k < L) ? combine<R>(a.comb, utn, x[c]) : R(0);
        if (k < L) col_st(a.out + base, k, outv[c]);
        hp[c] = hed[c] * (a.psum_a * (double)utn + a.psum_b * (double)outv[c]);
    }
    double shu = 0.0, shp = 0.0;
    if (a.sum_hu || a.sum_hp) col_sum2<NK>(hu_in, hp, shu, shp);
    if (lane == 0) {
        a.G[e] = G;
        a.sum_h[e] = Sh;
        if (a.sum_hu) a.sum_hu[e] = shu;
        if (a.sum_hp) a.sum_hp[e] = shp;
        if (a.Gi) {
            if (a.interp == 3)
                a.Gi[e] = div_by_near(a.Ga[e], 6.0, 1.0 / 6.0) + div_by_near(a.Gb[e], 6.0, 1.0 / 6.0) +
                          div_by_near(2.0 * G, 3.0, 1.0 / 3.0);
            else
                a.Gi[e] = 0.5 * a.Ga[e] + 0.5 * G;
        }
    }
}

template <int NK, typename R>
__device__ __forceinline__ void fe_edge_dry(const FEEdgeArgs<R> &a, int e) {
    const int lane = lane_id();
    const size_t base = (size_t)e * a.L;
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        const int k = lane + c * kWave;
        if (k < a.L) a.out[base + k] = R(0);
    }
    if (lane == 0) {
        a.G[e] = 0.0;
        a.sum_h[e] = 0.0;
        if (a.sum_hu) a.sum_hu[e] = 0.0;
        if (a.sum_hp) a.sum_hp[e] = 0.0;
        if (a.Gi) a.Gi[e] = 0.0;
    }
}

// kChain: the stencil is in canonical two-cell order (sse_mesh.cpp) and the
// edge record holds the two cells' vertex chains, so the vorticity of the 10
// distinct vertices is read once instead of at both ends of every stencil
// edge; otherwise every stencil edge carries its own two vertices.
// kVar bit 0: kChain; bit 1: kMix (see fe_edge_finish); bit 2: kDel4, the
// biharmonic operand lap(lap u) is gathered (div and curl of lap u at the
// edge's cells and vertices).
template <int NK, typename R, bool kAdd, int kVar>
__device__ __forceinline__ void fe_edge_body(const FEEdgeArgs<R> &a, int col) {
    constexpr bool kChain = (kVar & 1) != 0;
    constexpr bool kMix = (kVar & 2) != 0;
    constexpr bool kDel4 = (kVar & 4) != 0;
    constexpr bool kWide = (kVar & 8) != 0;
    const DevMesh &m = a.m;
    const int E = m.E;
    const int e = col;
    if (e >= E) return;
    const int L = a.L;
    const size_t base = (size_t)e * L;
    if (!m.emask[e]) {
        fe_edge_dry<NK, R>(a, e);
        return;
    }
    int kk[NK];
    bool ok[NK];
    lane_layers<NK>(L, kk, ok);
    // u = X + ubar (kAdd) or ut = X - ubar (otherwise); the other one equals X.
    const double *ubar = kAdd ? a.ubar_add : a.ubar_sub;
    const int32_t *rec = m.erec + (size_t)e * kEdgeRec;
    const int c1 = rec[30], c2 = rec[31];
    const double idc = m.inv_dc[e], idv = m.inv_dv[e];
    const R ub_e = ubar_at<R>(a, ubar, e);
    const size_t b1 = (size_t)c1 * L, b2 = (size_t)c2 * L;

    EdgeOperands<NK, R> o;
    R q[NK];
    // vertex vorticity: chain A0..A5 around c1 (A0, A5 the end points of e),
    // B0..B3 the inner vertices of the chain around c2
    R zA[6][NK], zB[4][NK];
    if constexpr (kChain) {
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            const size_t zo = (size_t)rec[10 + i] * L;
#pragma unroll
            for (int c = 0; c < NK; ++c) zA[i][c] = col_ldv<kWide>(a.Z, zo, kk[c]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const size_t zo = (size_t)rec[16 + i] * L;
#pragma unroll
            for (int c = 0; c < NK; ++c) zB[i][c] = col_ldv<kWide>(a.Z, zo, kk[c]);
        }
    }
    const bool a0_is_v1 = kChain ? rec[20] != 0 : false;
    const size_t bv1 = kChain ? 0 : (size_t)m.edge_verts[2 * e] * L;
    const size_t bv2 = kChain ? 0 : (size_t)m.edge_verts[2 * e + 1] * L;
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        const int k = kk[c];
        const R x = col_ldv<kWide>(a.X, base, k);
        R za, zb;
        if constexpr (kChain) {
            za = a0_is_v1 ? zA[0][c] : zA[5][c];
            zb = a0_is_v1 ? zA[5][c] : zA[0][c];
        } else {
            za = col_ldv<kWide>(a.Z, bv1, k);
            zb = col_ldv<kWide>(a.Z, bv2, k);
        }
        o.u[c] = kAdd ? x + ub_e : x;
        o.ut[c] = kAdd ? x : x - ub_e;
        o.h1[c] = col_ldv<kWide>(a.h, b1, k);
        o.h2[c] = col_ldv<kWide>(a.h, b2, k);
        o.r1[c] = col_ldv<kWide>(a.rho, b1, k);
        o.r2[c] = col_ldv<kWide>(a.rho, b2, k);
        o.za[c] = za;
        o.zb[c] = zb;
        o.B1[c] = col_ldv<kWide>(a.B, b1, k);
        o.B2[c] = col_ldv<kWide>(a.B, b2, k);
        o.W1[c] = col_ldv<kWide>(a.Wtop, b1, k);
        o.W2[c] = col_ldv<kWide>(a.Wtop, b2, k);
        q[c] = o.za[c] + o.zb[c];  // twice the edge vorticity
        o.cor[c] = o.vor[c] = R(0);
        o.lap2[c] = R(0);
    }
    if constexpr (kDel4) {
        // lap(lap u) at the edge from div(lap u) at its cells and curl(lap u)
        // at its vertices
        const int v1 = kChain ? (a0_is_v1 ? rec[10] : rec[15]) : m.edge_verts[2 * e];
        const int v2 = kChain ? (a0_is_v1 ? rec[15] : rec[10]) : m.edge_verts[2 * e + 1];
        const size_t w1 = (size_t)v1 * L, w2 = (size_t)v2 * L;
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            const int k = kk[c];
            const R d1 = col_ldv<kWide>(a.D2, b1, k), d2 = col_ldv<kWide>(a.D2, b2, k);
            const R z1 = col_ldv<kWide>(a.Z2, w1, k), z2 = col_ldv<kWide>(a.Z2, w2, k);
            o.lap2[c] = (d2 - d1) * (R)idc - (z2 - z1) * (R)idv;
        }
    }

    // Coriolis on the baroclinic velocity (-f ut^perp) and the vorticity flux
    // -(k.curl u) u^perp through the TRiSK tangential reconstruction.  The
    // table holds W / 4 beside W (f_e + f_j) / 2, and the vertex sums are
    // twice the edge vorticities, so W ((q_e + q_j) / 2) is (W / 4)(2 q_e +
    // 2 q_j): the same bits with two multiplications fewer per stencil term
    // (scaling by powers of two is exact).  Padded
    // stencil slots point at the edge itself with zero weights, so the loop
    // runs its full width; its column loads carry no branch between them.
    // the weight pairs in R (mixed precision: the FP32 table, the same values
    // as converting the FP64 ones, without a conversion per term)
    const R *wp = wpair_of<R>(m) + (size_t)e * 2 * kMaxEdges2;
#pragma unroll
    for (int j = 0; j < kMaxEdges2; ++j) {
        const int ep = rec[j];
        const R wj = wp[2 * j], wfj = wp[2 * j + 1];
        const R ubp = ubar_at<R>(a, ubar, ep);
        const size_t pb = (size_t)ep * L;
        const size_t pb1 = kChain ? 0 : (size_t)rec[10 + 2 * j] * L;
        const size_t pb2 = kChain ? 0 : (size_t)rec[11 + 2 * j] * L;
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            const R xp = col_ldv<kWide>(a.X, pb, kk[c]);
            const R up = kAdd ? xp + ubp : xp, utp = kAdd ? xp : xp - ubp;
            R qp;
            if constexpr (kChain) {
                // chain of c1: A_j, A_{j+1}; chain of c2: A5, B0, B1, B2, B3, A0
                const int s = j - 5;
                const R za_ = j < 5 ? zA[j < 5 ? j : 0][c] : (s == 0 ? zA[5][c] : zB[s > 0 ? s - 1 : 0][c]);
                const R zb_ = j < 5 ? zA[j < 5 ? j + 1 : 0][c] : (s == 4 ? zA[0][c] : zB[s < 4 && s >= 0 ? s : 0][c]);
                qp = za_ + zb_;
            } else {
                qp = col_ldv<kWide>(a.Z, pb1, kk[c]) + col_ldv<kWide>(a.Z, pb2, kk[c]);
            }
            o.cor[c] += wfj * utp;
            o.vor[c] += (wj * (q[c] + qp)) * up;
        }
    }
    fe_edge_finish<NK, R, kMix, kWide>(a, e, c1, c2, idc, idv, o);
}

// The edge part of the split pass: per edge the two shares g, h, rho and w at
// both cells, the edge itself and u^n, ten columns in the place of thirty.
// Between its bytes (FP64 512 x 512 x 60: 2.5 GB a call) and about 250 vector
// instructions per edge, a wavefront has little else to wait with, so all of
// its loads, vector and scalar, start before the first wait: left to the
// compiler, u^n, the shares and the cells' scalars came one after the other
// behind the scans.  With the column sums two to a butterfly and the
// reciprocals refined rather than divided, one call on 512 x 512 x 60 went
// from 595 to 526 us (FP64, 4.5 TB/s) and 523 to 458 (FP32), on a level-7
// globe from 343 to 285 and 305 to 241.
template <int NK, typename R, bool kAdd, int kVar>
__device__ __forceinline__ void fe_edge_split_body(const FEEdgeArgs<R> &a, int e) {
    constexpr bool kMix = (kVar & 2) != 0;
    constexpr bool kDel4 = (kVar & 4) != 0;
    constexpr bool kWide = (kVar & 8) != 0;
    const DevMesh &m = a.m;
    if (e >= m.E) return;
    const int L = a.L;
    const size_t base = (size_t)e * L;
    // the mask's word by a scalar load, beside the edge's cells (the table is
    // padded to whole words)
    const uint32_t wet = reinterpret_cast<const uint32_t *>(m.emask)[e >> 2] >> (8 * (e & 3)) & 0xffu;
    const int c1 = m.edge_cells[2 * e], c2 = m.edge_cells[2 * e + 1];
    if (!wet || c1 < 0) {  // (c1 is a cell; read here so that its load starts with the mask's)
        fe_edge_dry<NK, R>(a, e);
        return;
    }
    int kk[NK];
    bool ok[NK];
    lane_layers<NK>(L, kk, ok);
    const double idc = m.inv_dc[e], idv = kDel4 ? m.inv_dv[e] : 0.0;
    const R ub = (R)(kAdd ? a.ubar_add : a.ubar_sub)[e];
    const size_t b1 = (size_t)c1 * L, b2 = (size_t)c2 * L;
    EdgeOperands<NK, R> o;
    o.K1 = a.Kbot[c1];
    o.K2 = a.Kbot[c2];
    o.z1 = a.zeta[c1];
    o.z2 = a.zeta[c2];
    o.H1 = m.H[c1];
    o.H2 = m.H[c2];
    o.ubn = (a.Un ? a.ubar_n : m.inv_dc)[e];  // (used with u^n only)
    const R *const un = a.Un ? a.Un : a.X;
    R x[NK];
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        const int k = kk[c];
        x[c] = col_ldv<kWide>(a.X, base, k);
        o.B1[c] = col_ldv<kWide>(a.out, base, k);
        o.B2[c] = col_ldv<kWide>(a.B, base, k);
        o.h1[c] = col_ldv<kWide>(a.h, b1, k);
        o.h2[c] = col_ldv<kWide>(a.h, b2, k);
        o.r1[c] = col_ldv<kWide>(a.rho, b1, k);
        o.r2[c] = col_ldv<kWide>(a.rho, b2, k);
        o.W1[c] = col_ldv<kWide>(a.Wtop, b1, k);
        o.W2[c] = col_ldv<kWide>(a.Wtop, b2, k);
        o.un[c] = col_ldv<kWide>(un, base, k);
        o.lap2[c] = R(0);
    }
    // every load has started before the first value is waited for
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        o.u[c] = kAdd ? x[c] + ub : x[c];
        o.ut[c] = kAdd ? x[c] : x[c] - ub;
    }
    if constexpr (kDel4) {
        const size_t w1 = (size_t)m.edge_verts[2 * e] * L, w2 = (size_t)m.edge_verts[2 * e + 1] * L;
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            const int k = kk[c];
            const R d1 = col_ldv<kWide>(a.D2, b1, k), d2 = col_ldv<kWide>(a.D2, b2, k);
            const R z1 = col_ldv<kWide>(a.Z2, w1, k), z2 = col_ldv<kWide>(a.Z2, w2, k);
            o.lap2[c] = (d2 - d1) * (R)idc - (z2 - z1) * (R)idv;
        }
    }
    fe_edge_finish<NK, R, kMix, kWide, true>(a, e, c1, c2, idc, idv, o);
}

// ---------------------------------------------------------------------------
// Measurement aid: the edge pass's column loads without its arithmetic.
// Each wavefront gathers the columns the direct edge pass reads for its edge
// (canonical stencils, one register chunk): u and u^n at the edge, h, rho,
// K - nu div u and w at both cells, the 10 stencil edges and the 10 chain
// vertices, and writes their sum; a launch takes the pass's gather time at
// its access pattern.  kSplit: the ten columns of the split pass's edge part.
// ---------------------------------------------------------------------------
template <typename R, bool kSplit>
__global__ void __launch_bounds__(1024, 8) edge_gather_kernel(FEEdgeArgs<R> a) {
    const DevMesh &m = a.m;
    const int e = column_id(m.E);
    if (e >= m.E) return;
    const int L = a.L;
    int kk[1];
    bool ok[1];
    lane_layers<1>(L, kk, ok);
    const int k = kk[0];
    if (!m.emask[e]) {
        if (ok[0]) col_st(a.out + (size_t)e * L, k, R(0));
        return;
    }
    const int32_t *rec = m.erec + (size_t)e * kEdgeRec;
    const size_t b1 = (size_t)rec[30] * L, b2 = (size_t)rec[31] * L;
    R v[30];
    v[0] = col_ldv<false>(a.X, (size_t)e * L, k);
    v[1] = col_ldv<false>(a.Un, (size_t)e * L, k);
    v[2] = (R)col_ldv<false>(a.h, b1, k);
    v[3] = (R)col_ldv<false>(a.h, b2, k);
    v[4] = (R)col_ldv<false>(a.rho, b1, k);
    v[5] = (R)col_ldv<false>(a.rho, b2, k);
    v[6] = kSplit ? col_ldv<false>(a.B, (size_t)e * L, k) : col_ldv<false>(a.B, b1, k);
    v[7] = kSplit ? col_ldv<false>(a.out, (size_t)e * L, k) : col_ldv<false>(a.B, b2, k);
    v[8] = col_ldv<false>(a.Wtop, b1, k);
    v[9] = col_ldv<false>(a.Wtop, b2, k);
#pragma unroll
    for (int j = 0; j < (kSplit ? 0 : 10); ++j) {
        v[10 + j] = col_ldv<false>(a.X, (size_t)rec[j] * L, k);
        v[20 + j] = col_ldv<false>(a.Z, (size_t)rec[10 + j] * L, k);
    }
    R sum = R(0);
#pragma unroll
    for (int j = 0; j < (kSplit ? 10 : 30); ++j) sum += v[j];
    if (ok[0]) col_st(a.out + (size_t)e * L, k, sum);
}

// ---------------------------------------------------------------------------
// Baroclinic forward Euler: edge pass staged through LDS.
//
// One workgroup of T wavefronts owns a tile of T consecutive edges.  It first
// copies every column the tile reads (stencil edges, their vertices, the
// edges' cells for h, rho, K - nu div u and w) from global memory into LDS,
// each column exactly once, then each wavefront evaluates its edge from LDS.
// The copy uses 16-byte loads, so one load instruction moves two FP64 (four
// FP32) layers per lane and several columns per wavefront; the vector-memory
// address path, which bounds the direct-gather kernel, then handles about a
// quarter of the instructions.
// ---------------------------------------------------------------------------

constexpr int kTileWaves = 4;  // wavefronts per workgroup of the tiled edge pass

// One list of columns to stage: column i of the list is the global column
// src + ids[i] L and goes to dst + i L in LDS.
template <typename T>
struct StageSeg {
    const T *src;
    const int32_t *ids;
    int n;
    T *dst;
};

// Copy the columns of NS lists (L values of type T each) into LDS with
// 16-byte loads.  The lists are walked as one: every lane group takes up to
// 8 columns, loads their ids, then their data, then stores them, so one
// wavefront has 8 column loads in flight and the whole copy costs two
// memory round trips.
template <typename T, int NS>
__device__ __forceinline__ void stage_columns(const StageSeg<T> (&seg)[NS], int L) {
    constexpr int V = 16 / sizeof(T);
    constexpr int B = 8;
    int start[NS + 1];
    start[0] = 0;
#pragma unroll
    for (int q = 0; q < NS; ++q) start[q + 1] = start[q] + seg[q].n;
    const int total = start[NS];
    if (total == 0) return;
    const int lane = lane_id(), wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if (L % V == 0 && L <= V * kWave) {
        const int lpc = L / V, cpw = kWave / lpc;  // lanes per column, columns per wavefront
        const int slot = lane / lpc, part = lane - slot * lpc;
        const bool lane_on = slot < cpw;
        const int step = nw * cpw;
        for (int c0 = wv * cpw + slot; c0 < total + (B - 1) * step; c0 += B * step) {
            int seg_of[B], pos[B], id[B];
            bool on[B];
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const int c = c0 + u * step;
                on[u] = lane_on && c < total;
                const int cs = c < total ? c : total - 1;
                int q = 0, p0 = cs;
#pragma unroll
                for (int r = 1; r < NS; ++r) {
                    if (cs >= start[r]) {
                        q = r;
                        p0 = cs - start[r];
                    }
                }
                seg_of[u] = q;
                pos[u] = p0;
            }
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const int32_t *ids = seg[0].ids;
#pragma unroll
                for (int r = 1; r < NS; ++r) ids = seg_of[u] == r ? seg[r].ids : ids;
                id[u] = ids[pos[u]];
            }
            uint4 v[B];
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const T *src = seg[0].src;
#pragma unroll
                for (int r = 1; r < NS; ++r) src = seg_of[u] == r ? seg[r].src : src;
                v[u] = *reinterpret_cast<const uint4 *>(src + (size_t)id[u] * L + part * V);
            }
#pragma unroll
            for (int u = 0; u < B; ++u) {
                T *dst = seg[0].dst;
#pragma unroll
                for (int r = 1; r < NS; ++r) dst = seg_of[u] == r ? seg[r].dst : dst;
                if (on[u]) *reinterpret_cast<uint4 *>(dst + (size_t)pos[u] * L + part * V) = v[u];
            }
        }
    } else {
        // Local arrays are indexed with compile-time indices only (select
        // chains), so that they stay in registers.
        for (int c = wv; c < total; c += nw) {
            int i = c;
            const int32_t *ids = seg[0].ids;
            const T *src = seg[0].src;
            T *dst = seg[0].dst;
#pragma unroll
            for (int r = 1; r < NS; ++r) {
                if (c >= start[r]) {
                    i = c - start[r];
                    ids = seg[r].ids;
                    src = seg[r].src;
                    dst = seg[r].dst;
                }
            }
            const T *col = src + (size_t)ids[i] * L;
            for (int k = lane; k < L; k += kWave) dst[(size_t)i * L + k] = col[k];
        }
    }
}

template <typename R>
size_t fe_edge_tiled_lds(const DevTiles &t, int L) {
    return (size_t)(t.max_ue + t.max_uv) * L * sizeof(R);   // X and Z columns
}

template <int NK, typename R, bool kAdd, bool kMix>
__global__ void __launch_bounds__(kTileWaves * kWave) fe_edge_tiled_kernel(FEEdgeArgs<R> a, DevTiles t) {
    extern __shared__ __align__(16) double lds_d[];
    const DevMesh &m = a.m;
    const int tile = xcd_block(t.nT);
    if (tile < 0) return;
    const int T = t.T, L = a.L, E = m.E;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ue0 = t.ue_off[tile], nue = t.ue_off[tile + 1] - ue0;
    const int uv0 = t.uv_off[tile], nuv = t.uv_off[tile + 1] - uv0;
    const int uc0 = t.uc_off[tile], nuc = t.uc_off[tile + 1] - uc0;
    // LDS holds the reused stencil operands only: the X columns of the tile's
    // edges and stencil edges, then the vorticity columns of their vertices.
    // The cell operands (h, rho, K - nu div u, w: two columns each, little
    // reuse across the tile) are read from global memory per edge.
    R *sX = reinterpret_cast<R *>(lds_d);
    R *sZ = sX + (size_t)nue * L;
    const double *ubar = kAdd ? a.ubar_add : a.ubar_sub;
    const int32_t *le = t.ue + ue0, *lv = t.uv + uv0;
    (void)uc0;
    (void)nuc;
    const StageSeg<R> seg[2] = {{a.X, le, nue, sX}, {a.Z, lv, nuv, sZ}};
    stage_columns<R, 2>(seg, L);
    __syncthreads();

    int kk[NK];
    bool ok[NK];
    lane_layers<NK>(L, kk, ok);
    // A workgroup has at most kTileWaves wavefronts (a 256-register budget per
    // lane, no spills); with larger tiles each wavefront evaluates several edges.
    const int nw = blockDim.x >> 6;
    for (int el = wv; el < T; el += nw) {
        const int e = tile * T + el;
        if (e >= E) break;
        if (!m.emask[e]) {
            fe_edge_dry<NK, R>(a, e);
            continue;
        }
        // 8-bit positions of this edge's operands in the staged lists.
        const uint32_t *lw = reinterpret_cast<const uint32_t *>(t.loc + (size_t)e * kLocPerEdge);
        uint32_t word[kLocPerEdge / 4];
#pragma unroll
        for (int qq = 0; qq < kLocPerEdge / 4; ++qq) word[qq] = lw[qq];
        auto locb = [&](int i) -> int { return (word[i >> 2] >> (8 * (i & 3))) & 0xff; };
        const int ls = locb(0), lv1 = locb(3), lv2 = locb(4);
        const int32_t *rec = m.erec + (size_t)e * kEdgeRec;
        const R ub_e = ubar_at<R>(a, ubar, e);
        const int c1 = rec[30], c2 = rec[31];
        const double idcv = m.inv_dc[e], idvv = m.inv_dv[e];

        const size_t b1 = (size_t)c1 * L, b2 = (size_t)c2 * L;
        EdgeOperands<NK, R> o;
        R q[NK];
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            const int k = kk[c];
            const double h1 = a.h[b1 + k], h2 = a.h[b2 + k], r1 = a.rho[b1 + k], r2 = a.rho[b2 + k];
            const R B1 = a.B[b1 + k], B2 = a.B[b2 + k], W1 = a.Wtop[b1 + k], W2 = a.Wtop[b2 + k];
            const R x = sX[(size_t)ls * L + k];
            o.u[c] = ok[c] ? (kAdd ? x + ub_e : x) : R(0);
            o.ut[c] = ok[c] ? (kAdd ? x : x - ub_e) : R(0);
            o.h1[c] = ok[c] ? h1 : 0.0;
            o.h2[c] = ok[c] ? h2 : 0.0;
            o.r1[c] = ok[c] ? r1 : 0.0;
            o.r2[c] = ok[c] ? r2 : 0.0;
            o.za[c] = ok[c] ? sZ[(size_t)lv1 * L + k] : R(0);
            o.zb[c] = ok[c] ? sZ[(size_t)lv2 * L + k] : R(0);
            o.B1[c] = ok[c] ? B1 : R(0);
            o.B2[c] = ok[c] ? B2 : R(0);
            o.W1[c] = ok[c] ? W1 : R(0);
            o.W2[c] = ok[c] ? W2 : R(0);
            q[c] = o.za[c] + o.zb[c];  // twice the edge vorticity
            o.cor[c] = o.vor[c] = R(0);
            o.lap2[c] = R(0);  // the tiled variants run without the biharmonic term
        }
        const R *wp = wpair_of<R>(m) + (size_t)e * 2 * kMaxEdges2;
#pragma unroll
        for (int j = 0; j < kMaxEdges2; ++j) {
            const R wj = wp[2 * j], wfj = wp[2 * j + 1];
            const int sl = locb(5 + j), sa = locb(15 + 2 * j), sb = locb(16 + 2 * j);
            const R ubp = ubar_at<R>(a, ubar, rec[j]);
#pragma unroll
            for (int c = 0; c < NK; ++c) {
                const int k = kk[c];
                const R xp = sX[(size_t)sl * L + k];
                const R up = kAdd ? xp + ubp : xp, utp = kAdd ? xp : xp - ubp;
                const R qp = sZ[(size_t)sa * L + k] + sZ[(size_t)sb * L + k];
                o.cor[c] += wfj * utp;
                o.vor[c] += (wj * (q[c] + qp)) * up;
            }
        }
        fe_edge_finish<NK, R, kMix, true>(a, e, c1, c2, idcv, idvv, o);
    }
}

// ---------------------------------------------------------------------------
// Barotropic forward-Euler evaluation (Algorithms 3 and 4, one stage)
// ---------------------------------------------------------------------------
template <typename R>
struct BTTables;
template <>
struct BTTables<double> {
    __device__ static const double *wf(const DevMesh &m) { return m.wf; }
    __device__ static const double *inv_dc(const DevMesh &m) { return m.inv_dc; }
    __device__ static const double *cdiv(const DevMesh &m) { return m.cell_div_t; }
    __device__ static const double *H(const DevMesh &m) { return m.H; }
};
template <>
struct BTTables<float> {
    __device__ static const float *wf(const DevMesh &m) { return m.wf_f; }
    __device__ static const float *inv_dc(const DevMesh &m) { return m.inv_dc_f; }
    __device__ static const float *cdiv(const DevMesh &m) { return m.cell_div_t_f; }
    __device__ static const float *H(const DevMesh &m) { return m.H_f; }
};

// One block of edges (edge_part) or of cells of one evaluation.  kD16: the
// index tables are read as 16-bit offsets (half the index bytes).
// The barotropic kernels (one evaluation / one tiled substep) spell every
// fused multiply-add out and contract nothing else, so that the two forms
// give the same bits whatever the compiler would fuse in either context.
template <typename R, bool kD16>
__device__ __forceinline__ void bt_eval_body(const BTEvalArgs<R> &a, bool edge_part, int lb) {
#pragma clang fp contract(off)
    const DevMesh &m = a.m;
    const R tau = (R)a.tau, g = (R)a.g;
    if (edge_part) {
        const int e = lb * blockDim.x + threadIdx.x;
        if (e >= m.E) return;
        if (!m.emask[e]) {
            a.uo[e] = R(0);
            if (a.F && a.zeroF) a.F[e] = 0.0;
            return;
        }
        const R *__restrict__ wf = BTTables<R>::wf(m);
        int c1, c2;
        if constexpr (kD16) {
            const int pk = m.ecells16[e], bc = delta_base(e, m.ratio_ce);
            c1 = bc + (int)(int16_t)(pk & 0xffff);
            c2 = bc + (int)(int16_t)((unsigned)pk >> 16);
        } else {
            c1 = m.edge_cells[2 * e];
            c2 = m.edge_cells[2 * e + 1];
        }
        const R ua = a.ua[e];
        const R z1 = a.za[c1], z2 = a.za[c2];
        // Padded stencil slots point at the edge itself with zero weight: the
        // loop runs its full width so that all its gathers issue together.
        R cor = R(0);
#pragma unroll
        for (int j = 0; j < kMaxEdges2; ++j) {
            const int ep = kD16 ? e + (int)m.eoe16[(size_t)j * m.E + e] : m.eoe[(size_t)j * m.E + e];
            cor = fmadd(wf[(size_t)j * m.E + e], a.ua[ep], cor);
        }
        const R ru = fmadd(-(g * (z2 - z1)), BTTables<R>::inv_dc(m)[e], cor) + (R)a.G[e];
        // the first stage of a substep combines with nothing: no base read
        const R base = a.comb != COMB_NONE ? a.ub[e] : R(0);
        a.uo[e] = combine<R>(a.comb, base, fmadd(tau, ru, ua));
        if (a.F) {
            // The transport accumulates in FP64 in both modes.
            const double flux = (double)ua * (0.5 * (((double)z1 + m.H[c1]) + ((double)z2 + m.H[c2])));
            a.F[e] = fmadd(a.wF, flux, a.zeroF ? 0.0 : a.F[e]);
        }
    } else {
        const int i = lb * blockDim.x + threadIdx.x;
        if (i >= m.C) return;
        if (!m.cmask[i]) { a.zo[i] = R(0); return; }
        const R *__restrict__ Ht = BTTables<R>::H(m);
        const R *__restrict__ cd_t = BTTables<R>::cdiv(m);
        const R zi = a.za[i] + Ht[i];
        R div = R(0);
        const int be = kD16 ? delta_base(i, m.ratio_ec) : 0;
#pragma unroll
        for (int j = 0; j < kMaxEdges; ++j) {
            const R cd = cd_t[(size_t)j * m.C + i];
            const int e = kD16 ? be + (int)m.cedges16[(size_t)j * m.C + i] : m.cell_edges_t[(size_t)j * m.C + i];
            const int nb = kD16 ? i + (int)m.cnbrs16[(size_t)j * m.C + i] : m.cell_nbrs_t[(size_t)j * m.C + i];
            const R zn = a.za[nb] + Ht[nb];
            div = fmadd(cd, a.ua[e] * (R(0.5) * (zi + zn)), div);
        }
        const R base = a.comb != COMB_NONE ? a.zb[i] : R(0);
        a.zo[i] = combine<R>(a.comb, base, fmadd(tau, -div, a.za[i]));
    }
}

// ---------------------------------------------------------------------------
// Tiled barotropic substep: one workgroup advances one cell patch (with its
// halo rings) through a whole SSPRK3 (three evaluations) or SSPRK2 (two)
// substep.  The substep input and every stage live in LDS; each thread holds
// the stencil tables of its edges (at most KS) and of its cell in registers
// for all evaluations, so the tables are read once per substep instead of
// once per evaluation.  Evaluation k computes the region level that the next
// one reads (level 2, then 1, then 0 = the patch's own cells and edges) with
// exactly the arithmetic of the one-evaluation kernel, so both paths give the
// same bits.
// ---------------------------------------------------------------------------
template <typename R>
struct BtTab;
template <>
struct BtTab<double> {
    __device__ static const double *w(const DevBtTiles &t) { return t.ew; }
    __device__ static const double *idc(const DevBtTiles &t) { return t.eidc; }
    __device__ static const double *cd(const DevBtTiles &t) { return t.ccd; }
};
template <>
struct BtTab<float> {
    __device__ static const float *w(const DevBtTiles &t) { return t.ew_f; }
    __device__ static const float *idc(const DevBtTiles &t) { return t.eidc_f; }
    __device__ static const float *cd(const DevBtTiles &t) { return t.ccd_f; }
};

// Grid-wide barrier of a cooperative launch: the writes of every workgroup
// before it are visible to every workgroup after it.  One thread per
// workgroup arrives on a counter (after the workgroup barrier and a
// device-scope release, which writes back its XCD's L2); the last of the
// k-th round (the counter reaching k * gridDim.x) publishes generation k, for
// which the others poll; a device-scope acquire then drops stale cache lines.
// The wait is bounded: if it runs out (or another workgroup's did), the
// workgroup sets *err and stops waiting, so every wavefront of the launch
// still finishes; the host reports the error and the results are not used.
__device__ __forceinline__ void grid_barrier(unsigned *bar, unsigned *gen, int *err, unsigned round,
                                             unsigned max_spins) {
    __syncthreads();
    if (threadIdx.x == 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        const unsigned target = round * gridDim.x;
        const unsigned old = __hip_atomic_fetch_add(bar, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (old + 1 == target) {
            __hip_atomic_store(gen, round, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            unsigned spins = 0;
            while (__hip_atomic_load(gen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < round) {
                if (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) break;
                if (++spins > max_spins) {
                    __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
}

// The persistent form of the tiled substep (bt_substep_body below): all l.M
// substeps of the loop for patch p in one workgroup of a cooperative launch
// in which every patch has its own workgroup (p < 0: a padding workgroup that
// only takes part in the barriers).  The stencil tables, the frozen forcing
// and the F^zeta sums stay in registers for the whole loop; substep s reads
// the previous substep's output (the loop input for s = 0) and writes one of
// two stage buffers (the loop output for the last), with a grid barrier
// between substeps.  Every evaluation performs exactly the arithmetic of the
// one-evaluation kernel, so all forms give the same bits.
template <typename R, int kScheme, int KS>
__device__ __forceinline__ void bt_loop_body(const BTTileArgs<R> &a, const BtLoop<R> &l, int p) {
#pragma clang fp contract(off)
    extern __shared__ __align__(16) double lds_d[];
    const DevBtTiles &T = a.t;
    const int tid = threadIdx.x;
    const bool on_patch = p >= 0;
    const int pp = on_patch ? p : 0;
    const int32_t *rec = T.patch + (size_t)pp * kBtRec;
    const int e0 = rec[0], es0 = rec[1], c0 = rec[2], cs0 = rec[3];
    int ne[4], nc[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        ne[k] = on_patch ? rec[4 + k] : 0;
        nc[k] = on_patch ? rec[8 + k] : 0;
    }
    constexpr int kIn = kScheme == 3 ? 3 : 2;  // level of the substep input
    const int nEin = ne[kIn], nCin = nc[kIn];
    const int nE1 = ne[kIn - 1], nC1 = nc[kIn - 1];  // level of the first evaluation
    const int se = ne[2], sc = nc[2];                // strides of the stencil tables

    // LDS: H (double) | U0 U1 U2 | Z0 Z1 Z2 | H in R (FP32 state only)
    double *H64b = lds_d;
    R *U0b = reinterpret_cast<R *>(H64b + nc[3]);
    R *U1b = U0b + ne[3];
    R *U2b = U1b + ne[2];
    R *Z0b = U2b + ne[1];
    R *Z1b = Z0b + nc[3];
    R *Z2b = Z1b + nc[2];
    const R *Hrb;
    if constexpr (sizeof(R) == 8) {
        Hrb = reinterpret_cast<const R *>(H64b);
    } else {
        R *h = Z2b + nc[1];
        for (int lc = tid; lc < nCin; lc += kBtThreads) h[lc] = T.cH_f[c0 + lc];
        Hrb = h;
    }
    for (int lc = tid; lc < nCin; lc += kBtThreads) H64b[lc] = T.cH[c0 + lc];

    // this thread's edges (le = s kBtThreads + tid) and cell (lc = tid)
    const R *__restrict__ wt = BtTab<R>::w(T);
    R w[KS][kMaxEdges2], idc[KS], Gv[KS];
    uint32_t nbw[KS][kMaxEdges2 / 2], ecw[KS];
    double Fa[KS];
    int ge[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const int le = s * kBtThreads + tid;
        const bool on = le < nE1;
        const int q = on ? le : 0;
        ecw[s] = on ? T.ec[es0 + q] : 0u;
        ge[s] = T.eid[e0 + q];
        idc[s] = BtTab<R>::idc(T)[es0 + q];
        Gv[s] = (R)a.G[ge[s]];
#pragma unroll
        for (int j = 0; j < kMaxEdges2; ++j) w[s][j] = wt[(size_t)kMaxEdges2 * es0 + (size_t)j * se + q];
#pragma unroll
        for (int i = 0; i < kMaxEdges2 / 2; ++i) nbw[s][i] = T.enb[(size_t)(kMaxEdges2 / 2) * es0 + (size_t)i * se + q];
        Fa[s] = (a.F && le < ne[0]) ? (a.zeroF ? 0.0 : a.F[ge[s]]) : 0.0;
    }
    const bool con = tid < nC1;
    const int qc = con ? tid : 0;
    const bool cwet = con && T.cwet[cs0 + qc] != 0;
    const int gc = T.cid[c0 + qc];
    R cd[kMaxEdges];
    uint32_t cen[kMaxEdges];
#pragma unroll
    for (int j = 0; j < kMaxEdges; ++j) {
        cd[j] = BtTab<R>::cd(T)[(size_t)kMaxEdges * cs0 + (size_t)j * sc + qc];
        cen[j] = T.cen[(size_t)kMaxEdges * cs0 + (size_t)j * sc + qc];
    }

    const R tau = (R)a.tau, g = (R)a.g;
    const int nsub = l.M;
#pragma unroll 1
    for (int sub = 0; sub < nsub; ++sub) {
        // LDS bases offset by an opaque zero, so that the compiler recomputes
        // the stage addresses in every substep instead of hoisting all of them
        // out of the loop (which needs more registers than the tables)
        int zoff = 0;
        {
            asm volatile("" : "+s"(zoff));
            // the packed index words likewise: decoded once per substep, not
            // kept decoded across the loop
#pragma unroll
            for (int s2 = 0; s2 < KS; ++s2) {
                asm volatile("" : "+v"(ecw[s2]));
#pragma unroll
                for (int i = 0; i < kMaxEdges2 / 2; ++i) asm volatile("" : "+v"(nbw[s2][i]));
            }
#pragma unroll
            for (int j = 0; j < kMaxEdges; ++j) asm volatile("" : "+v"(cen[j]));
        }
        R *const U0 = U0b + zoff, *const U1 = U1b + zoff, *const U2 = U2b + zoff;
        R *const Z0 = Z0b + zoff, *const Z1 = Z1b + zoff, *const Z2 = Z2b + zoff;
        const double *const H64 = H64b + zoff;
        const R *const Hr = Hrb + zoff;
        const bool odd = (sub & 1) != 0;
        const R *ua = sub == 0 ? l.u_in : (odd ? l.bu0 : l.bu1);
        const R *za = sub == 0 ? l.z_in : (odd ? l.bz0 : l.bz1);
        R *uo = sub == nsub - 1 ? l.u_out : (odd ? l.bu1 : l.bu0);
        R *zo = sub == nsub - 1 ? l.z_out : (odd ? l.bz1 : l.bz0);
#pragma unroll 1
        for (int le = tid; le < nEin; le += kBtThreads) U0[le] = ua[T.eid[e0 + le]];
#pragma unroll 1
        for (int lc = tid; lc < nCin; lc += kBtThreads) Z0[lc] = za[T.cid[c0 + lc]];
        __syncthreads();

        // One evaluation producing level lvl from (Ui, Zi); the last one writes
        // the substep output to global memory.
        auto evaluate = [&](const R *Ui, const R *Zi, int lvl, int comb, double wF, R *Uo, R *Zo, bool last) {
#pragma clang fp contract(off)
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const int le = s * kBtThreads + tid;
                if (le < ne[lvl]) {
                    const uint32_t c = ecw[s];
                    R out = R(0);
                    if ((c >> 30) & 1u) {
                        const int l1 = (int)(c & 0x7fffu), l2 = (int)((c >> 15) & 0x7fffu);
                        const R u = Ui[le];
                        const R z1 = Zi[l1], z2 = Zi[l2];
                        R cor = R(0);
#pragma unroll
                        for (int j = 0; j < kMaxEdges2; ++j) {
                            const int lj = (int)((nbw[s][j >> 1] >> (16 * (j & 1))) & 0xffffu);
                            cor = fmadd(w[s][j], Ui[lj], cor);
                        }
                        const R ru = fmadd(-(g * (z2 - z1)), idc[s], cor) + Gv[s];
                        const R base = comb != COMB_NONE ? U0[le] : R(0);
                        out = combine<R>(comb, base, fmadd(tau, ru, u));
                        if (a.F && le < ne[0]) {
                            const double flux = (double)u * (0.5 * (((double)z1 + H64[l1]) + ((double)z2 + H64[l2])));
                            Fa[s] = fmadd(wF, flux, Fa[s]);
                        }
                    }
                    if (last) uo[ge[s]] = out;
                    else Uo[le] = out;
                }
            }
            if (tid < nc[lvl]) {
                R out = R(0);
                if (cwet) {
                    const R zi = Zi[tid] + Hr[tid];
                    R div = R(0);
#pragma unroll
                    for (int j = 0; j < kMaxEdges; ++j) {
                        const int le = (int)(cen[j] & 0xffffu), ln = (int)(cen[j] >> 16);
                        const R zn = Zi[ln] + Hr[ln];
                        div = fmadd(cd[j], Ui[le] * (R(0.5) * (zi + zn)), div);
                    }
                    const R base = comb != COMB_NONE ? Z0[tid] : R(0);
                    out = combine<R>(comb, base, fmadd(tau, -div, Zi[tid]));
                }
                if (last) zo[gc] = out;
                else Zo[tid] = out;
            }
        };
        if constexpr (kScheme == 3) {
            evaluate(U0, Z0, 2, COMB_NONE, a.w1, U1, Z1, false);
            __syncthreads();
            evaluate(U1, Z1, 1, COMB_34, a.w1, U2, Z2, false);
            __syncthreads();
            evaluate(U2, Z2, 0, COMB_THIRD, a.w3, nullptr, nullptr, true);
        } else {
            evaluate(U0, Z0, 1, COMB_NONE, a.w1, U1, Z1, false);
            __syncthreads();
            evaluate(U1, Z1, 0, COMB_HALF, a.w1, nullptr, nullptr, true);
        }
        if (sub + 1 < nsub) grid_barrier(l.bar, l.gen, l.err, (unsigned)(sub + 1), l.spins);
    }
    if (a.F) {
#pragma unroll
        for (int s = 0; s < KS; ++s)
            if (s * kBtThreads + tid < ne[0]) a.F[ge[s]] = Fa[s];
    }
}

// kDry: the mesh has land or coast edges (see the table loads below).
template <typename R, int kScheme, int KS, bool kDry = false>
__device__ __forceinline__ void bt_substep_body(const BTTileArgs<R> &a, int p) {
#pragma clang fp contract(off)
    extern __shared__ __align__(16) double lds_d[];
    const DevBtTiles &T = a.t;
    const int tid = threadIdx.x;
    const int32_t *rec = T.patch + (size_t)p * kBtRec;
    const int e0 = rec[0], es0 = rec[1], c0 = rec[2], cs0 = rec[3];
    int ne[4], nc[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        ne[k] = rec[4 + k];
        nc[k] = rec[8 + k];
    }
    constexpr int kIn = kScheme == 3 ? 3 : 2;  // level of the substep input
    const int nEin = ne[kIn], nCin = nc[kIn];
    const int nE1 = ne[kIn - 1], nC1 = nc[kIn - 1];  // level of the first evaluation
    const int se = ne[2], sc = nc[2];                // strides of the stencil tables

    // LDS: H (double) | U0 U1 U2 | Z0 Z1 Z2 | H in R (FP32 state only)
    double *H64 = lds_d;
    R *U0 = reinterpret_cast<R *>(H64 + nc[3]);
    R *U1 = U0 + ne[3];
    R *U2 = U1 + ne[2];
    R *Z0 = U2 + ne[1];
    R *Z1 = Z0 + nc[3];
    R *Z2 = Z1 + nc[2];
    const R *Hr;
    if constexpr (sizeof(R) == 8) {
        Hr = reinterpret_cast<const R *>(H64);
    } else {
        R *h = Z2 + nc[1];
        for (int lc = tid; lc < nCin; lc += kBtThreads) h[lc] = T.cH_f[c0 + lc];
        Hr = h;
    }
    for (int le = tid; le < nEin; le += kBtThreads) U0[le] = a.ua[T.eid[e0 + le]];
    for (int lc = tid; lc < nCin; lc += kBtThreads) {
        Z0[lc] = a.za[T.cid[c0 + lc]];
        H64[lc] = T.cH[c0 + lc];
    }

    // this thread's edges (le = s kBtThreads + tid) and cell (lc = tid)
    constexpr bool kSkipDry = kDry && sizeof(R) == 8;
    const R *__restrict__ wt = BtTab<R>::w(T);
    R w[KS][kMaxEdges2], idc[KS], Gv[KS];
    uint32_t nbw[KS][kMaxEdges2 / 2], ecw[KS];
    double Fa[KS];
    int ge[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const int le = s * kBtThreads + tid;
        const bool on = le < nE1;
        const int q = on ? le : 0;
        ecw[s] = on ? T.ec[es0 + q] : 0u;
        ge[s] = T.eid[e0 + q];
        // a coast or land edge keeps a zero velocity and never reads its
        // stencil: on meshes with land, in FP64, its tables are not loaded,
        // which skips their share of the table bytes (level-7 sphere with 30%
        // land: 3.01 -> 2.81 ms per step).  With the FP32 tables the
        // exec-masked loads cost more than they save (2.31 -> 2.46 ms), and on
        // a mesh without land they only add their test, so there every edge
        // loads its row
        const bool wet = !kSkipDry || ((ecw[s] >> 30) & 1u) != 0;
        idc[s] = wet ? BtTab<R>::idc(T)[es0 + q] : R(0);
        Gv[s] = wet ? (R)a.G[ge[s]] : R(0);
#pragma unroll
        for (int j = 0; j < kMaxEdges2; ++j) w[s][j] = wet ? wt[(size_t)kMaxEdges2 * es0 + (size_t)j * se + q] : R(0);
#pragma unroll
        for (int i = 0; i < kMaxEdges2 / 2; ++i)
            nbw[s][i] = wet ? T.enb[(size_t)(kMaxEdges2 / 2) * es0 + (size_t)i * se + q] : 0u;
        Fa[s] = (a.F && le < ne[0]) ? (a.zeroF ? 0.0 : a.F[ge[s]]) : 0.0;
    }
    const bool con = tid < nC1;
    const int qc = con ? tid : 0;
    const bool cwet = con && T.cwet[cs0 + qc] != 0;
    const int gc = T.cid[c0 + qc];
    R cd[kMaxEdges];
    uint32_t cen[kMaxEdges];
#pragma unroll
    for (int j = 0; j < kMaxEdges; ++j) {  // land cells keep zeta = 0 and read no stencil
        const bool ld = !kSkipDry || cwet;
        cd[j] = ld ? BtTab<R>::cd(T)[(size_t)kMaxEdges * cs0 + (size_t)j * sc + qc] : R(0);
        cen[j] = ld ? T.cen[(size_t)kMaxEdges * cs0 + (size_t)j * sc + qc] : 0u;
    }
    __syncthreads();

    const R tau = (R)a.tau, g = (R)a.g;
    // One evaluation producing level lvl from (Ui, Zi); the last one writes the
    // substep output to global memory.
    auto evaluate = [&](const R *Ui, const R *Zi, int lvl, int comb, double wF, R *Uo, R *Zo, bool last) {
#pragma clang fp contract(off)
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int le = s * kBtThreads + tid;
            if (le < ne[lvl]) {
                const uint32_t c = ecw[s];
                R out = R(0);
                if ((c >> 30) & 1u) {
                    const int l1 = (int)(c & 0x7fffu), l2 = (int)((c >> 15) & 0x7fffu);
                    const R ua = Ui[le];
                    const R z1 = Zi[l1], z2 = Zi[l2];
                    R cor = R(0);
#pragma unroll
                    for (int j = 0; j < kMaxEdges2; ++j) {
                        const int lj = (int)((nbw[s][j >> 1] >> (16 * (j & 1))) & 0xffffu);
                        cor = fmadd(w[s][j], Ui[lj], cor);
                    }
                    const R ru = fmadd(-(g * (z2 - z1)), idc[s], cor) + Gv[s];
                    const R base = comb != COMB_NONE ? U0[le] : R(0);
                    out = combine<R>(comb, base, fmadd(tau, ru, ua));
                    if (a.F && le < ne[0]) {
                        const double flux = (double)ua * (0.5 * (((double)z1 + H64[l1]) + ((double)z2 + H64[l2])));
                        Fa[s] = fmadd(wF, flux, Fa[s]);
                    }
                }
                if (last) a.uo[ge[s]] = out;
                else Uo[le] = out;
            }
        }
        if (tid < nc[lvl]) {
            R out = R(0);
            if (cwet) {
                const R zi = Zi[tid] + Hr[tid];
                R div = R(0);
#pragma unroll
                for (int j = 0; j < kMaxEdges; ++j) {
                    const int le = (int)(cen[j] & 0xffffu), ln = (int)(cen[j] >> 16);
                    const R zn = Zi[ln] + Hr[ln];
                    div = fmadd(cd[j], Ui[le] * (R(0.5) * (zi + zn)), div);
                }
                const R base = comb != COMB_NONE ? Z0[tid] : R(0);
                out = combine<R>(comb, base, fmadd(tau, -div, Zi[tid]));
            }
            if (last) a.zo[gc] = out;
            else Zo[tid] = out;
        }
    };
    if constexpr (kScheme == 3) {
        evaluate(U0, Z0, 2, COMB_NONE, a.w1, U1, Z1, false);
        __syncthreads();
        evaluate(U1, Z1, 1, COMB_34, a.w1, U2, Z2, false);
        __syncthreads();
        evaluate(U2, Z2, 0, COMB_THIRD, a.w3, nullptr, nullptr, true);
    } else {
        evaluate(U0, Z0, 1, COMB_NONE, a.w1, U1, Z1, false);
        __syncthreads();
        evaluate(U1, Z1, 0, COMB_HALF, a.w1, nullptr, nullptr, true);
    }
    if (a.F) {
#pragma unroll
        for (int s = 0; s < KS; ++s)
            if (s * kBtThreads + tid < ne[0]) a.F[ge[s]] = Fa[s];
    }
}


// ---------------------------------------------------------------------------
// Barotropic substeps with factored weights (see DevFact).
//
// What the weight tables cost: they are streamed once per substep, 80 bytes
// of FP64 weights and 20 of indices per region edge, 270 MB per substep of a
// 262,144-cell mesh, and that traffic bounds the substep (46.9 us).  The
// factored form reads six numbers per cell and three per edge instead, 160 MB
// by the counters (36 us; its loads alone take 27, the rest is the barriers and
// evaluations that two workgroups per CU do not hide), and small enough tables
// stay on chip for a whole loop (the resident form).  It works on a cell's six edges
// at once and leaves the edges two half sums to subtract.  One evaluation is two phases with a barrier between them:
//   edges  finish the velocity of the previous stage, publish x = l u / 2 and
//          the flux x (h_c1 + h_c2), keep zeta_c2 - zeta_c1;
//   cells  read the six x, f and fluxes, write six half sums and the new zeta.
// Every fused multiply-add is spelled out and nothing else contracts, so the
// forms of the loop (one launch per evaluation, per substep or per loop)
// give the same bits.
// ---------------------------------------------------------------------------

// v with its sign flipped when bit 15 of w is set (an inward edge normal)
__device__ __forceinline__ double flip(double v, uint32_t w) {
    return __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, v) ^
                                          ((unsigned long long)(w & 0x8000u) << 48));
}
__device__ __forceinline__ float flip(float v, uint32_t w) {
    return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, v) ^ ((w & 0x8000u) << 16));
}

// v with its sign flipped where an edge's byte offset w names the second of its
// two half sums (see bt_fact_body)
template <typename R>
__device__ __forceinline__ R flip_side(R v, uint32_t w) {
    if constexpr (sizeof(R) == 8)
        return __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, v) ^ ((unsigned long long)(w << 28) << 32));
    else
        return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, v) ^ (w << 29));
}

// Half sums of one cell, from x_b = s_b l_b u_b / 2, f_b / 2 and S = 2 S_1 ..
// 2 S_5, 2 S_n: s_a h_a is edge a's share of d_a times the reconstructed
// Coriolis term.  With y_b = (f_b / 2) x_b and the sums X, Y (Y weighted by S)
// and P_a (before a) of x, X', Y' and P'_a of y,
//   h_a = S_a (f_a X + X') + f_a (X - Y) + (X' - Y') - S_n (f_a P_a + P'_a) - 2 y_a
// (f_a, S in the halved and doubled units above): six operations per edge.
// store(a, h_a) receives them one by one.
template <typename R, typename F>
__device__ __forceinline__ void half_sums(const R (&x)[6], const R (&f)[6], const R (&S)[6], F &&store) {
#pragma clang fp contract(off)
    R X = x[0], Xy = f[0] * x[0], Y = R(0), Yy = R(0);
#pragma unroll
    for (int j = 1; j < 6; ++j) {
        const R y = f[j] * x[j];
        Y = j == 1 ? S[0] * x[1] : fmadd(S[j - 1], x[j], Y);
        Yy = j == 1 ? S[0] * y : fmadd(S[j - 1], y, Yy);
        X += x[j];
        Xy += y;
    }
    const R D = X - Y, Dy = Xy - Yy;
    R P = x[0], Py = f[0] * x[0];
    store(0, fmadd(R(-2), Py, fmadd(f[0], D, Dy)));
#pragma unroll
    for (int j = 1; j < 6; ++j) {
        const R y = f[j] * x[j];
        const R B = fmadd(R(-2), y, fmadd(f[j], D, Dy));
        const R h = fmadd(-S[5], fmadd(f[j], P, Py), B);
        store(j, fmadd(S[j - 1], fmadd(f[j], X, Xy), h));
        P += x[j];
        Py += y;
    }
}
// New velocity and zeta of one evaluation (hs: the half sum of c1 less that of
// c2; dv: sum of x (h_c1 + h_c2), the cell's outward fluxes).
template <typename R>
__device__ __forceinline__ R fact_velocity(R u, R base, R hs, R dz, R idc, R G, R g, R tau, int comb) {
#pragma clang fp contract(off)
    const R ru = fmadd(fmadd(-g, dz, hs), idc, G);
    return combine<R>(comb, base, fmadd(tau, ru, u));
}
template <typename R>
__device__ __forceinline__ R fact_zeta(R z, R base, R dv, R ia, R tau, int comb) {
#pragma clang fp contract(off)
    return combine<R>(comb, base, fmadd(tau, -(dv * ia), z));
}
template <typename R>
__device__ __forceinline__ double fact_transport(R u, R z1, R z2, double H1, double H2) {
#pragma clang fp contract(off)
    return (double)u * (0.5 * (((double)z1 + H1) + ((double)z2 + H2)));
}

template <typename R>
struct FactTab;
template <>
struct FactTab<double> {
    __device__ static const double *lh(const DevBtTiles &t) { return t.elh; }
    __device__ static const double *fh(const DevBtTiles &t) { return t.efh; }
    __device__ static const double *idc(const DevBtTiles &t) { return t.fidc; }
    __device__ static const double *S(const DevBtTiles &t) { return t.cS; }
    __device__ static const double *ia(const DevBtTiles &t) { return t.cia; }
    __device__ static const double *lh(const DevFact &t) { return t.lh; }
    __device__ static const double *fh(const DevFact &t) { return t.fh; }
    __device__ static const double *S(const DevFact &t) { return t.S; }
    __device__ static const double *ia(const DevFact &t) { return t.ia; }
};
template <>
struct FactTab<float> {
    __device__ static const float *lh(const DevBtTiles &t) { return t.elh_f; }
    __device__ static const float *fh(const DevBtTiles &t) { return t.efh_f; }
    __device__ static const float *idc(const DevBtTiles &t) { return t.fidc_f; }
    __device__ static const float *S(const DevBtTiles &t) { return t.cS_f; }
    __device__ static const float *ia(const DevBtTiles &t) { return t.cia_f; }
    __device__ static const float *lh(const DevFact &t) { return t.lh_f; }
    __device__ static const float *fh(const DevFact &t) { return t.fh_f; }
    __device__ static const float *S(const DevFact &t) { return t.S_f; }
    __device__ static const float *ia(const DevFact &t) { return t.ia_f; }
};

// One evaluation, one thread per edge or cell (the per-evaluation form).  The
// edge forms both of its cells' half sums for itself.
template <typename R>
__device__ __forceinline__ void bt_eval_fact(const BTEvalArgs<R> &a, bool edge_part, int lb) {
#pragma clang fp contract(off)
    const DevMesh &m = a.m;
    const R tau = (R)a.tau, g = (R)a.g;
    const R *__restrict__ Ht = BTTables<R>::H(m);
    const R *__restrict__ lh = FactTab<R>::lh(a.fk);
    if (edge_part) {
        const int e = lb * blockDim.x + threadIdx.x;
        if (e >= m.E) return;
        if (!m.emask[e]) {
            a.uo[e] = R(0);
            if (a.F && a.zeroF) a.F[e] = 0.0;
            return;
        }
        const R *__restrict__ fh = FactTab<R>::fh(a.fk);
        const R *__restrict__ St = FactTab<R>::S(a.fk);
        const int c[2] = {m.edge_cells[2 * e], m.edge_cells[2 * e + 1]};
        R hs[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int n = m.cell_nedges[c[s]];
            R x[6], f[6], S[6];
#pragma unroll
            for (int j = 0; j < 6; ++j) {
                const int ej = m.cell_edges_t[(size_t)j * m.C + c[s]];
                const uint32_t w = m.edge_cells[2 * ej] == c[s] ? 0u : 0x8000u;
                const R v = flip(lh[ej] * a.ua[ej], w);
                x[j] = j < n ? v : R(0);
                f[j] = j < n ? fh[ej] : R(0);
                S[j] = St[(size_t)j * m.C + c[s]];
            }
            hs[s] = R(0);
            half_sums<R>(x, f, S, [&](int j, R h) {
                if (j < n && m.cell_edges_t[(size_t)j * m.C + c[s]] == e) hs[s] = h;
            });
        }
        const R ua = a.ua[e];
        const R z1 = a.za[c[0]], z2 = a.za[c[1]];
        const R base = a.comb != COMB_NONE ? a.ub[e] : R(0);
        a.uo[e] = fact_velocity<R>(ua, base, hs[0] - hs[1], z2 - z1, BTTables<R>::inv_dc(m)[e], (R)a.G[e], g, tau, a.comb);
        if (a.F) a.F[e] = fmadd(a.wF, fact_transport<R>(ua, z1, z2, m.H[c[0]], m.H[c[1]]), a.zeroF ? 0.0 : a.F[e]);
    } else {
        const int i = lb * blockDim.x + threadIdx.x;
        if (i >= m.C) return;
        if (!m.cmask[i]) { a.zo[i] = R(0); return; }
        const int n = m.cell_nedges[i];
        const R zi = a.za[i] + Ht[i];
        R dv = R(0);
#pragma unroll
        for (int j = 0; j < 6; ++j) {
            const int e = m.cell_edges_t[(size_t)j * m.C + i], nb = m.cell_nbrs_t[(size_t)j * m.C + i];
            const uint32_t w = m.edge_cells[2 * e] == i ? 0u : 0x8000u;
            const R x = flip(lh[e] * a.ua[e], w);
            if (j < n) dv = fmadd(x, zi + (a.za[nb] + Ht[nb]), dv);
        }
        const R base = a.comb != COMB_NONE ? a.zb[i] : R(0);
        a.zo[i] = fact_zeta<R>(a.za[i], base, dv, FactTab<R>::ia(a.fk)[i], tau, a.comb);
    }
}

template <typename T>
__device__ __forceinline__ T shared_load(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void shared_store(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// What a launch leaves in an error word when a wait of it ran out: never zero,
// and no other launch's.
__device__ __forceinline__ int ran_out(const BtRound &r, bool task) {
    return 0x40000000 | (int)((2 * r.serial + (task ? 1 : 0)) & 0x3fffffff);
}

// Waits until the counter *f has reached target.  The wait is bounded: if it
// runs out, or another workgroup's did, the workgroup goes on without waiting,
// and *err = code says that the results are worthless.
__device__ __forceinline__ void wait_count(const unsigned long long *f, unsigned long long target, int *err, int code,
                                           unsigned max_spins) {
    unsigned spins = 0;
    while (shared_load(f) < target) {
        if (++spins > max_spins) {
            shared_store(err, code);
            break;
        }
        if ((spins & 255u) == 0 && shared_load(err) == code) break;
    }
}

// Admission of a resident loop.  Its workgroups wait for each other, so none
// may wait before all of them hold a place on the device.  An occupancy query
// cannot promise that: it counts the places of an empty device, and a kernel of
// another stream or process takes places, and leaves registers and LDS of a CU
// in pieces that fit fewer workgroups, for as long as the loop's first ones
// wait (beside a kernel of 192-thread workgroups, 174 of 752 workgroups of 512
// threads, three of which an idle CU holds, started only when others had
// ended; as a cooperative launch 158).  So every workgroup counts itself in
// before its first substep; the last one to arrive admits the loop; one that
// has waited kAdmitTicks without that calls it off.  Whoever is first decides,
// for all: nobody has published anything yet, and the task form below computes
// a loop that was called off.
__device__ __forceinline__ void settle(const BtRound &r, unsigned long long verdict) {
    unsigned long long *d = r.words + kVerdict * kDoneStride, v = shared_load(d);
    while (v < 2 * r.serial &&
           !__hip_atomic_compare_exchange_strong(d, &v, verdict, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
    }
}
__device__ __forceinline__ bool called_off(const BtRound &r) {
    return shared_load(r.words + kVerdict * kDoneStride) == 2 * r.serial + 1;
}
__device__ __forceinline__ unsigned long long shared_count(unsigned long long *p) {
    return __hip_atomic_fetch_add(p, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Workgroup lb of n has started.  Counts on one address come one after the
// other, about 40 ns apiece (745 workgroups: 30 us), so each group counts on a
// line of its own and its last one at the root.
__device__ __forceinline__ void arrive(const BtRound &r, int lb, int n) {
    const int g = lb % kGroups, members = n / kGroups + (g < n % kGroups ? 1 : 0);
    if (shared_count(r.words + g * kDoneStride) + 1 != (unsigned long long)members) return;
    if (shared_count(r.words + kGroups * kDoneStride) + 1 != (unsigned long long)min(n, kGroups)) return;
    if (r.ticks) settle(r, 2 * r.serial);
}
__device__ __forceinline__ bool admitted(const BtRound &r) {
    const unsigned long long t0 = wall_clock64();
    for (;;) {
        const unsigned long long v = shared_load(r.words + kVerdict * kDoneStride);
        if (v >= 2 * r.serial) return v == 2 * r.serial;
        if (wall_clock64() - t0 >= r.ticks) settle(r, 2 * r.serial + 1);
    }
}

// One substep of patch p (kOne: the input a.ua, a.za, the output a.uo, a.zo),
// all l->M substeps of the loop (kAll), or substep `task` of the loop (kTask:
// through the exchange buffers, every value of the patch).
//
// In the loop form the tables, the forcing, the transport sums and the
// patch's own state stay on chip, and a substep ends with an exchange: the
// values other patches read go out with device-scope stores (through to the
// memory all XCDs share; no cache is written back or dropped), the workgroup
// counts its substep, waits for its neighbours' counts and reads its halo
// with device-scope loads.  Two buffers alternate: a neighbour overwrites
// the one of substep s only after this workgroup's count for s + 1 tells it
// that its values have been read.
//
// LDS, fixed places so that one address register serves several arrays (NT
// threads hold at most kFactEdges NT region edges and NT region cells):
//   XF  (x, f / 2) of an edge     HS  the half sums of its two cells
//   ZS  h_c1 + h_c2 of an edge    ZH  (zeta, H) of a cell
template <typename R>
struct alignas(2 * sizeof(R)) Pair {
    R a, b;
};
template <typename R>
struct alignas(16) ZetaDepth {
    double H;
    R z;
};
template <typename R, int NT>
struct FactLds {
    Pair<R> XF[kFactEdges * NT];
    Pair<R> HS[kFactEdges * NT];
    ZetaDepth<R> ZH[NT];
    R ZS[kFactEdges * NT];
    int go;   // the workgroup goes on: the loop is admitted, or there are tasks
};

enum { kOne, kAll, kTask };

template <typename R, int kScheme, int kMode, int NT>
__device__ __forceinline__ void bt_fact_body(FactLds<R, NT> &lds, const BTTileArgs<R> &a, const BtResident<R> *l,
                                             int p, const BtRound *round, int task = 0, int lb = 0, int n = 1) {
#pragma clang fp contract(off)
    constexpr bool kLoop = kMode == kAll;
    const DevBtTiles &T = a.t;
    const int tid = threadIdx.x;
    const int32_t *rec = T.patch + (size_t)p * kBtRec;
    const int e0 = rec[0], c0 = rec[2];
    int ne[4], nc[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        ne[k] = rec[4 + k];
        nc[k] = rec[8 + k];
    }
    constexpr int kIn = kScheme == 3 ? 3 : 2;  // level of the substep input
    constexpr int KS = kBtEdgeSlots;
    if (kMode == kOne && !rec[14]) {  // no ocean cell: velocity, zeta and transport are zero
        for (int le = tid; le < ne[0]; le += NT) {
            const int e = T.eid[e0 + le];
            a.uo[e] = R(0);
            if (a.F && a.zeroF) a.F[e] = 0.0;
        }
        if (tid < nc[0]) a.zo[T.cid[c0 + tid]] = R(0);
        return;
    }
    const int nEin = ne[kIn], nCin = nc[kIn];

    // this thread's edges le = s NT + tid and cell lc = tid
    R lhv[kFactEdges], u[KS], u0[KS], idc[KS], Gv[KS], dz[KS];
    double Fa[KS];
    uint32_t ec[kFactEdges];
    int ge[kFactEdges];
    // the resident loop reads and writes the step's FP64 fields (an FP32 loop
    // rounds and widens them here: two launches each way less, 4 us apiece)
    using IO = std::conditional_t<kMode == kOne, R, double>;
    const IO *ua, *za;
    if constexpr (kMode == kOne) {
        ua = a.ua;
        za = a.za;
    } else {
        ua = l->u_in;
        za = l->z_in;
    }
    // a task reads what the tasks of the substep before it have published
    const bool begun = kMode == kTask && task > 0;
    auto old_u = [&](int e, uint32_t c) -> R {
        if (begun) return ((c >> 30) & 1u) ? shared_load(((task - 1) & 1 ? l->bu1 : l->bu0) + e) : R(0);
        return (R)ua[e];
    };
    auto old_z = [&](int c, bool wet) -> R {
        if (begun) return wet ? shared_load(((task - 1) & 1 ? l->bz1 : l->bz0) + c) : R(0);
        return (R)za[c];
    };
    auto old_F = [&](int e) -> double {
        if (kMode == kOne) return a.zeroF ? 0.0 : a.F[e];
        return begun ? shared_load(a.F + e) : 0.0;
    };
#pragma unroll
    for (int s = 0; s < kFactEdges; ++s) {
        const int le = s * NT + tid;
        const bool on = le < nEin;
        const int q = e0 + (on ? le : 0);
        ge[s] = T.eid[q];
        if (kMode != kOne && l->eold) ge[s] = l->eold[ge[s]];
        lhv[s] = FactTab<R>::lh(T)[q];
        ec[s] = T.fec[q];
        const R v = old_u(ge[s], ec[s]);
        if (s < KS) {
            idc[s < KS ? s : 0] = FactTab<R>::idc(T)[q];
            Gv[s < KS ? s : 0] = (R)a.G[ge[s]];
            u[s < KS ? s : 0] = v;
            Fa[s < KS ? s : 0] = (a.F && le < ne[0]) ? old_F(ge[s]) : 0.0;
        }
        if (on) lds.XF[le] = Pair<R>{lhv[s] * v, FactTab<R>::fh(T)[q]};
    }
    const bool con = tid < nCin;
    const int qc = con ? tid : 0;
    int gc = T.cid[c0 + qc];
    if (kMode != kOne && l->cold) gc = l->cold[gc];
    const uint32_t cfl = T.cflag[c0 + qc];
    const bool cwet = con && (cfl & 1u) != 0;
    // byte offset of the cell's half sum on each of its edges: the edge's pair,
    // the second of it where the cell is c2.  The edge's (x, f) pair is the
    // same offset with that bit cleared, and the bit, shifted to the top, the
    // sign s_j.
    constexpr uint32_t kSide = sizeof(R);
    uint32_t w[6];
    R S[6];
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        const uint32_t c = T.fcen[(size_t)3 * c0 + (size_t)(j >> 1) * nc[3] + qc] >> (16 * (j & 1));
        w[j] = (c & 0x7fffu) * 2 * kSide + ((c & 0x8000u) ? kSide : 0u);
        S[j] = FactTab<R>::S(T)[(size_t)6 * c0 + (size_t)j * nc[3] + qc];
    }
    const R ia = FactTab<R>::ia(T)[c0 + qc];
    R z = old_z(gc, cwet), z0;
    if (con) lds.ZH[tid] = ZetaDepth<R>{T.cH[c0 + tid], z};
    if (tid == 0) {  // the entry that missing edge slots read
        lds.XF[ne[3]] = Pair<R>{R(0), R(0)};
        lds.ZS[ne[3]] = R(0);
    }
    const R tau = (R)a.tau, g = (R)a.g;

    // Publishes h_c1 + h_c2 of the edges the evaluation of level lvl sums over
    // (at level 0 those of level 1: some edges of the patch's cells are owned
    // by the neighbour) and adds the owned edges' transport.
    auto prepare = [&](int lvl, double wF) {
#pragma clang fp contract(off)
        const int n = ne[lvl < 1 ? 1 : lvl];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int le = s * NT + tid;
            if (le < n) {
                const ZetaDepth<R> a1 = lds.ZH[ec[s] & 0x7fffu], a2 = lds.ZH[(ec[s] >> 15) & 0x7fffu];
                lds.ZS[le] = (a1.z + (R)a1.H) + (a2.z + (R)a2.H);
                dz[s] = a2.z - a1.z;
                if (a.F && le < ne[0] && ((ec[s] >> 30) & 1u))
                    Fa[s] = fmadd(wF, fact_transport<R>(u[s], a1.z, a2.z, a1.H, a2.H), Fa[s]);
            }
        }
    };
    // Cell phase of the evaluation that produces level lvl.
    auto cells = [&](int lvl, int comb, IO *zout) {
#pragma clang fp contract(off)
        if (tid < nc[lvl + 1] && cwet) {
            const char *const xf = reinterpret_cast<const char *>(lds.XF);
            const char *const zs = reinterpret_cast<const char *>(lds.ZS);
            char *const hs = reinterpret_cast<char *>(lds.HS);
            R x[6], f[6];
#pragma unroll
            for (int j = 0; j < 6; ++j) {
                const Pair<R> v = *reinterpret_cast<const Pair<R> *>(xf + (w[j] & ~kSide));
                x[j] = flip_side<R>(v.a, w[j]);
                f[j] = v.b;
            }
            if (tid < nc[lvl]) {
                R dv = R(0);
#pragma unroll
                for (int j = 0; j < 6; ++j)
                    dv = fmadd(x[j], *reinterpret_cast<const R *>(zs + ((w[j] >> 1) & ~(kSide - 1))), dv);
                z = fact_zeta<R>(z, comb != COMB_NONE ? z0 : R(0), dv, ia, tau, comb);
            }
            // the fluxes' registers are free before the half sums begin
            __builtin_amdgcn_sched_barrier(0);
            half_sums<R>(x, f, S, [&](int j, R h) { *reinterpret_cast<R *>(hs + w[j]) = h; });
        } else {
            z = R(0);  // land
        }
        if (tid < nc[lvl]) {
            lds.ZH[tid].z = z;
            if (zout) zout[gc] = z;
        }
    };
    // Edge phase after it: the new velocity of level lvl.
    auto edges = [&](int lvl, int comb, IO *uout) {
#pragma clang fp contract(off)
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int le = s * NT + tid;
            if (le < ne[lvl]) {
                R out = R(0);
                if ((ec[s] >> 30) & 1u) {
                    const Pair<R> h = lds.HS[le];
                    out = fact_velocity<R>(u[s], comb != COMB_NONE ? u0[s] : R(0), h.a - h.b, dz[s], idc[s], Gv[s], g, tau, comb);
                }
                u[s] = out;
                if (uout) uout[ge[s]] = out;
                else lds.XF[le].a = lhv[s] * out;
            }
        }
    };

    if (kLoop && round->words) {
        if (tid == 0) {
            if (lb == 0) shared_store(round->words + kTicket * kDoneStride, 0ull);
            arrive(*round, lb, n);
            lds.go = admitted(*round);
        }
        __syncthreads();
        if (!__builtin_amdgcn_readfirstlane(lds.go)) return;
    }
    const int nsub = kMode == kOne ? 1 : l->M, first = kMode == kTask ? task : 0;
#pragma unroll 1
    for (int sub = first; sub < (kMode == kTask ? first + 1 : nsub); ++sub) {
        const bool last = sub == nsub - 1;
        IO *uo = nullptr, *zo = nullptr;
        if constexpr (kMode == kOne) {
            uo = a.uo;
            zo = a.zo;
        } else if (last) {
            uo = l->u_out;
            zo = l->z_out;
        }
#pragma unroll
        for (int s = 0; s < KS; ++s) u0[s] = u[s];
        z0 = z;
        __syncthreads();
        if constexpr (kScheme == 3) {
            prepare(2, a.w1);
            __syncthreads();
            cells(2, COMB_NONE, nullptr);
            __syncthreads();
            edges(2, COMB_NONE, nullptr);
            prepare(1, a.w1);
            __syncthreads();
            cells(1, COMB_34, nullptr);
            __syncthreads();
            edges(1, COMB_34, nullptr);
            prepare(0, a.w3);
            __syncthreads();
            cells(0, COMB_THIRD, zo);
            __syncthreads();
            edges(0, COMB_THIRD, uo);
        } else {
            prepare(1, a.w1);
            __syncthreads();
            cells(1, COMB_NONE, nullptr);
            __syncthreads();
            edges(1, COMB_NONE, nullptr);
            prepare(0, a.w1);
            __syncthreads();
            cells(0, COMB_HALF, zo);
            __syncthreads();
            edges(0, COMB_HALF, uo);
        }
        if constexpr (kMode != kOne) {
            if (kLoop && last) break;
            R *bu = (sub & 1) ? l->bu1 : l->bu0, *bz = (sub & 1) ? l->bz1 : l->bz0;
#pragma unroll
            for (int s = 0; s < KS; ++s)
                if (s * NT + tid < ne[0]) {
                    if (kMode == kTask ? !last : (ec[s] >> 31) != 0) shared_store(bu + ge[s], u[s]);
                    if (kMode == kTask && a.F) shared_store(a.F + ge[s], Fa[s]);
                }
            if (tid < nc[0] && (kMode == kTask ? !last : (cfl & 2u) != 0)) shared_store(bz + gc, z);
            if (kMode == kTask && last && shared_load(l->err) == ran_out(*round, true)) {
                // a wait of this or an earlier task ran out: all three results say so
#pragma unroll
                for (int s = 0; s < KS; ++s)
                    if (s * NT + tid < ne[0]) {
                        l->u_out[ge[s]] = NAN;
                        if (a.F) shared_store(a.F + ge[s], (double)NAN);
                    }
                if (tid < nc[0]) l->z_out[gc] = NAN;
            }
            // every wavefront's stores have reached the shared memory before
            // the substep is counted
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            const unsigned long long target = round->base + (unsigned long long)(sub + 1);
            if (tid == 0) shared_store(l->done + (size_t)p * kDoneStride, target);
            if (kMode == kTask) return;
            if (tid < rec[13])
                wait_count(l->done + (size_t)T.nbr[rec[12] + tid] * kDoneStride, target, l->err, ran_out(*round, false), l->spins);
            asm volatile("" ::: "memory");
            __syncthreads();
            // the halo: dry edges and land cells stay zero
#pragma unroll
            for (int s = 0; s < kFactEdges; ++s) {
                const int le = s * NT + tid;
                if (le < nEin) {
                    R v = R(0);
                    if (le < ne[0]) v = u[s < KS ? s : 0];
                    else if ((ec[s] >> 30) & 1u) v = shared_load(bu + ge[s]);
                    if (s < KS) u[s < KS ? s : 0] = v;
                    lds.XF[le].a = lhv[s] * v;
                }
            }
            if (con && tid >= nc[0]) {
                z = cwet ? shared_load(bz + gc) : R(0);
                lds.ZH[tid].z = z;
            }
        }
    }
    if constexpr (kLoop) {
        // after a wait that ran out the results are worthless: they come out
        // as NaN where nobody reads the error word
        if (shared_load(l->err) == ran_out(*round, false) && tid < nc[0]) l->z_out[gc] = NAN;
    }
    if (a.F) {
#pragma unroll
        for (int s = 0; s < KS; ++s)
            if (s * NT + tid < ne[0]) a.F[ge[s]] = Fa[s];
    }
}

// The resident loop of the patch at place i of the order, in workgroup lb of n
// of the launch (patches without ocean cells have no workgroup: their zeros are
// written by others).
template <typename R, int kScheme, int NT>
__device__ __forceinline__ void bt_resident_body(const BtResident<R> &l, int at, const BtRound &round, int lb, int n) {
    __shared__ FactLds<R, NT> lds;
    const DevBtTiles &T = l.a.t;
    for (int i = T.nA + at; i < T.nP; i += T.nA) {
        const int32_t *rec = T.patch + (size_t)T.order[i] * kBtRec;
        for (int le = threadIdx.x; le < rec[4]; le += NT) {
            int e = T.eid[rec[0] + le];
            if (l.eold) e = l.eold[e];
            l.u_out[e] = 0.0;
            if (l.a.F) l.a.F[e] = 0.0;
        }
        for (int lc = threadIdx.x; lc < rec[8]; lc += NT) {
            const int c = T.cid[rec[2] + lc];
            l.z_out[l.cold ? l.cold[c] : c] = 0.0;
        }
    }
    bt_fact_body<R, kScheme, kAll, NT>(lds, l.a, &l, T.order[at], &round, 0, lb, n);
}

// A loop that was called off, or (redo) in which a wait ran out, as tasks:
// (substep, patch) in order of substeps, taken one after the other by however
// many workgroups run.  A task waits only for tasks before it in that order
// (those of its neighbours and itself in the substep before), which running
// workgroups hold or have finished, so it gets on with a single workgroup on
// the device, and it gives the resident loop's bits.  Exits at once after a
// loop that was admitted, the usual case: with the admission it then costs
// about 6 us a loop (60 substeps on 64 x 64 cells: 92 to 96 us; as a cooperative
// launch, which needs all of this too, 107 without it).
template <typename R, int kScheme, int NT>
__device__ __forceinline__ void bt_task_body(const BtResident<R> *args, const int2 *table, int n, int most,
                                             const BtRound &round) {
    __shared__ FactLds<R, NT> lds;
    __shared__ unsigned long long next;
    const int tid = threadIdx.x;
    if (blockIdx.x == 0 && tid <= kGroups) shared_store(round.words + tid * kDoneStride, 0ull);  // for the next launch
    // one thread decides for the workgroup: a wait of another one's task may set
    // the error word meanwhile
    if (tid == 0) lds.go = called_off(round) || (round.redo && shared_load(args->err) == ran_out(round, false));
    __syncthreads();
    if (!__builtin_amdgcn_readfirstlane(lds.go)) return;
    for (;;) {
        __syncthreads();
        if (tid == 0) next = shared_count(round.words + kTicket * kDoneStride);
        __syncthreads();
        const unsigned long long t = next;
        if (t >= (unsigned long long)n * (unsigned)most) return;
        const int sub = __builtin_amdgcn_readfirstlane((int)(t / (unsigned)n));
        const int i = __builtin_amdgcn_readfirstlane((int)(t % (unsigned)n));
        const BtResident<R> &l = args[table ? table[i].x : 0];
        if (sub >= l.M) continue;
        const DevBtTiles &T = l.a.t;
        const int p = T.order[table ? table[i].y : i];
        const int32_t *rec = T.patch + (size_t)p * kBtRec;
        if (sub > 0) {
            const unsigned long long target = round.base + (unsigned long long)sub;
            const int q = tid < rec[13] ? T.nbr[rec[12] + tid] : tid == kFactNbrs ? p : -1;
            if (q >= 0) wait_count(l.done + (size_t)q * kDoneStride, target, l.err, ran_out(round, true), kBarrierSpins);
            asm volatile("" ::: "memory");
            __syncthreads();
        }
        bt_fact_body<R, kScheme, kTask, NT>(lds, l.a, &l, p, &round, sub);
    }
}

// ---------------------------------------------------------------------------
// Thickness stage (z-star): h_out = comb(h_n, h_in + dt T^h), zeta = sum h - H
// ---------------------------------------------------------------------------
template <int NK, int Q>
__device__ __forceinline__ void thickness_body(const THArgs &a, int first) {
    const int lane = lane_id();
    const DevMesh &m = a.m;
    if (first >= m.C) return;
    const int L = a.L;
    int kk[NK];
    bool ok[NK];
    lane_layers<NK>(L, kk, ok);
    int ci[Q];
    bool has[Q], wet[Q];
    double divF[Q], fr[Q][NK], hin[Q][NK], hb[Q][NK];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        has[q] = first + q < m.C;
        const int i = ci[q] = has[q] ? first + q : first;
        const size_t base = (size_t)i * L;
        wet[q] = m.cmask[i] != 0;
        // Padded stencil slots hold a valid edge with a zero coefficient, so
        // the sum runs its full width and all its loads are in flight together.
        divF[q] = 0.0;
        if (wet[q]) {
#pragma unroll
            for (int j = 0; j < kMaxEdges; ++j)
                divF[q] += m.cell_div[i * kMaxEdges + j] * a.Ftot[m.cell_edges[i * kMaxEdges + j]];
        }
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            fr[q][c] = col_ld(a.frac + base, kk[c]);
            hin[q][c] = col_ld(a.h_in + base, kk[c]);
            hb[q][c] = (a.comb != COMB_NONE) ? col_ld(a.h_n + base, kk[c]) : 0.0;
        }
    }
    bool bad = false;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        if (!has[q]) continue;
        const int i = ci[q];
        const size_t base = (size_t)i * L;
        double hv[NK];
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            const double th = wet[q] ? -fr[q][c] * divF[q] : 0.0;
            const double x = hin[q][c] + a.dt * th;
            hv[c] = ok[c] ? combine<double>(a.comb, hb[q][c], x) : 0.0;
            if (ok[c]) col_st(a.h_out + base, kk[c], hv[c]);
            bad |= ok[c] && !isfinite(hv[c]);
        }
        const double sum = col_sum<NK, true>(hv);
        if (lane == 0) a.zeta_out[i] = wet[q] ? sum - m.H[i] : 0.0;
    }
    if (bad && a.nonfinite) *a.nonfinite = 1;
}

// Thickness stage fused with the temperature tracer stage (tracer runs).
template <int NK, typename R>
__device__ __forceinline__ void tracer_body(const TracerArgs<R> &a, int col) {
    const int lane = lane_id();
    const DevMesh &m = a.m;
    const int i = col;
    if (i >= m.C) return;
    const int L = a.L;
    const size_t base = (size_t)i * L;
    const bool wet = m.cmask[i] != 0;
    int kk[NK];
    bool ok[NK];
    lane_layers<NK>(L, kk, ok);
    double hi[NK], Ti[NK], dhv[NK], dhtv[NK], dif[NK];
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        const double h = a.h_in[base + kk[c]], t = a.T_in[base + kk[c]];
        hi[c] = ok[c] ? h : 0.0;
        Ti[c] = ok[c] ? t : 0.0;
        dhv[c] = dhtv[c] = dif[c] = 0.0;
    }
    if (wet) {
        // padded slots carry zero coefficients
#pragma unroll
        for (int j = 0; j < kMaxEdges; ++j) {
            const int e = m.cell_edges[i * kMaxEdges + j];
            const int nb = m.cell_nbrs[i * kMaxEdges + j];
            const double cd = m.cell_div[i * kMaxEdges + j];
            const double ae = (a.a1 ? a.ca1 * a.a1[e] : 0.0) + (a.uA ? a.uA[e] : 0.0);
            const double ew = m.emask[e] ? 1.0 : 0.0;
            // (T_c2 - T_c1) / d_e seen from this cell
            const double gs = (m.edge_cells[2 * e] == i ? 1.0 : -1.0) * m.inv_dc[e];
            const size_t eb = (size_t)e * L, nbb = (size_t)nb * L;
#pragma unroll
            for (int c = 0; c < NK; ++c) {
                const int k = kk[c];
                const double x1 = (double)a.X1[eb + k], x2 = a.X2 ? (double)a.X2[eb + k] : 0.0;
                const double hn = a.h_in[nbb + k], tn = a.T_in[nbb + k];
                // lanes past the last layer loaded layer L - 1: they carry no flux
                const double on = ok[c] ? ew : 0.0;
                const double u = on * (a.c1 * x1 + a.c2 * x2 + ae);
                const double he = 0.5 * (hi[c] + hn), te = 0.5 * (Ti[c] + tn);
                dhv[c] += cd * (he * u);
                dhtv[c] += cd * (he * te * u);
                dif[c] += cd * (on * (he * a.kappa_h * ((tn - Ti[c]) * gs)));
            }
        }
    }
    // thickness tendency and w at the top of every layer
    double th[NK], w[NK];
    if (a.frac) {
        const double tot = col_sum<NK, kDppFor<R>>(dhv);
        double src[NK];
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            th[c] = ok[c] ? -a.frac[base + kk[c]] * tot : 0.0;
            src[c] = ok[c] ? (-dhv[c] - th[c]) : 0.0;
        }
        col_incl_suffix<NK, kDppFor<R>>(src, w);
    } else {
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            th[c] = -dhv[c];
            w[c] = 0.0;
        }
    }
    // vertical fluxes at the interfaces: advective Tbar^t w and diffusive
    // kappa_v (T_{k-1} - T_k) / hbar^t, zero at the surface and the bottom
    double Tu[NK], hu[NK], fa[NK], fd[NK], fan[NK], fdn[NK];
    col_up1<NK, kDppFor<R>>(Ti, Tu);
    col_up1<NK, kDppFor<R>>(hi, hu);
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        const int k = lane + c * kWave;
        const bool inner = k >= 1 && k < L;
        fa[c] = inner ? 0.5 * (Tu[c] + Ti[c]) * w[c] : 0.0;
        fd[c] = inner ? a.kappa_v * ((Tu[c] - Ti[c]) / (0.5 * (hu[c] + hi[c]))) : 0.0;
    }
    col_down1<NK, kDppFor<R>>(fa, fan);
    col_down1<NK, kDppFor<R>>(fd, fdn);
    double hv[NK];
    bool bad = false;
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        const int k = lane + c * kWave;
        hv[c] = 0.0;
        if (k < L) {
            const double tend = wet ? (-dhtv[c] - (fa[c] - fan[c]) + dif[c] + (fd[c] - fdn[c])) : 0.0;
            const double x = hi[c] + a.dt * (wet ? th[c] : 0.0);
            const double xt = hi[c] * Ti[c] + a.dt * tend;
            const double hb = a.comb != COMB_NONE ? a.h_n[base + k] : 0.0;
            const double tb = a.comb != COMB_NONE ? a.h_n[base + k] * a.T_n[base + k] : 0.0;
            hv[c] = combine<double>(a.comb, hb, x);
            const double ht = combine<double>(a.comb, tb, xt);
            const double T = wet ? ht / hv[c] : 0.0;
            a.h_out[base + k] = hv[c];
            a.T_out[base + k] = T;
            a.rho_out[base + k] = a.rho0 * (1.0 - a.alpha * (T - a.tref));
            bad |= !isfinite(hv[c]) || !isfinite(T);
        }
    }
    const double s = col_sum<NK, kDppFor<R>>(hv);
    if (lane == 0) a.zeta_out[i] = wet ? s - m.H[i] : 0.0;
    if (bad && a.nonfinite) *a.nonfinite = 1;
}

// Thickness stage (isopycnal): per-layer flux divergence, w = 0.
template <int NK, typename R>
__device__ __forceinline__ void thickness_iso_body(const THIsoArgs<R> &a, int col) {
    const int lane = lane_id();
    const DevMesh &m = a.m;
    const int i = col;
    if (i >= m.C) return;
    const int L = a.L;
    const size_t base = (size_t)i * L;
    const bool wet = m.cmask[i] != 0;
    double hi[NK], div[NK];
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        int k = lane + c * kWave;
        hi[c] = (k < L) ? a.h_in[base + k] : 0.0;
        div[c] = 0.0;
    }
    if (wet) {
        const int n = m.cell_nedges[i];
        for (int j = 0; j < n; ++j) {
            const int e = m.cell_edges[i * kMaxEdges + j];
            const int nb = m.cell_nbrs[i * kMaxEdges + j];
            const double cd = m.cell_div[i * kMaxEdges + j];
            const double ae = (a.a1 ? a.ca1 * a.a1[e] : 0.0) + (a.uA ? a.uA[e] : 0.0);
            const bool ew = m.emask[e] != 0;
            const size_t eb = (size_t)e * L, nbb = (size_t)nb * L;
#pragma unroll
            for (int c = 0; c < NK; ++c) {
                int k = lane + c * kWave;
                if (k < L && ew) {
                    double u = a.c1 * (double)a.X1[eb + k] + (a.X2 ? a.c2 * (double)a.X2[eb + k] : 0.0) + ae;
                    double he = 0.5 * (hi[c] + a.h_in[nbb + k]);
                    div[c] += cd * (he * u);
                }
            }
        }
    }
    double hv[NK];
    bool bad = false;
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        int k = lane + c * kWave;
        hv[c] = 0.0;
        if (k < L) {
            double x = hi[c] + a.dt * (-div[c]);
            double b = (a.comb != COMB_NONE) ? a.h_n[base + k] : 0.0;
            hv[c] = combine<double>(a.comb, b, x);
            a.h_out[base + k] = hv[c];
            bad |= !isfinite(hv[c]);
        }
    }
    const double s = col_sum<NK, kDppFor<R>>(hv);
    if (lane == 0) a.zeta_out[i] = wet ? s - m.H[i] : 0.0;
    if (bad && a.nonfinite) *a.nonfinite = 1;
}

// ---------------------------------------------------------------------------
// Reconciliation deficits D^e and adjusted total fluxes (Section 3.4)
// ---------------------------------------------------------------------------
__device__ __forceinline__ void recon_body(const ReconArgs &a, int lb) {
    const DevMesh &m = a.m;
    const int e = lb * blockDim.x + threadIdx.x;
    if (e >= m.E) return;
    if (a.ub_half) a.ub_half[e] = 0.75 * a.ub_n[e] + 0.25 * a.ub2[e];
    if (!m.emask[e]) {
        a.Ftot[e] = 0.0;
        if (a.uA) a.uA[e] = 0.0;
        return;
    }
    const double Sh = a.Sh[e];
    double Ftot, uA = 0.0;
    if (a.mode == 0) {
        const double Fh = a.Fh[e];
        if (a.rec) uA = (a.Fz[e] - Fh) / Sh;
        Ftot = Fh + uA * Sh;
    } else if (a.mode == 1) {
        const double P = a.Pp[e] + (a.ub_n[e] + a.ub_new[e]) * Sh;
        if (a.rec) {
            const double f1 = (a.rec == SSE_RECONCILE_EXACT) ? a.Fz1[e] : a.Fh1[e];
            const double f2 = (a.rec == SSE_RECONCILE_EXACT) ? a.Fz2[e] : a.Fh2[e];
            const double Fh3 = (f1 + f2 + 2.0 * P) / 6.0;
            uA = 1.5 * (a.Fz[e] - Fh3) / Sh;
        }
        Ftot = 0.5 * P + uA * Sh;
    } else {
        const double P = a.Pp[e] + a.ub_new[e] * Sh;
        if (a.rec) {
            const double f1 = (a.rec == SSE_RECONCILE_EXACT) ? a.Fz1[e] : a.Fh1[e];
            const double Fh2 = 0.5 * (f1 + P);
            uA = 2.0 * (a.Fz[e] - Fh2) / Sh;
        }
        Ftot = P + uA * Sh;
    }
    a.Ftot[e] = Ftot;
    if (a.uA) a.uA[e] = uA;
}

// ---------------------------------------------------------------------------
// u^{n+1} = ubar^{n+1} + ut^{n+1}; split (BBspl) with h^{n+1}
// ---------------------------------------------------------------------------
template <int NK, typename R, int Q>
__device__ __forceinline__ void assemble_body(const AssembleArgs<R> &a, int first) {
    const int lane = lane_id();
    const DevMesh &m = a.m;
    if (first >= m.E) return;
    const int L = a.L;
    int kk[NK];
    bool ok[NK];
    lane_layers<NK>(L, kk, ok);
    int ei[Q];
    bool has[Q], wet[Q];
    R ub[Q], x[Q][NK];
    double h1[Q][NK], h2[Q][NK];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        has[q] = first + q < m.E;
        const int e = ei[q] = has[q] ? first + q : first;
        wet[q] = m.emask[e] != 0;
        const int c1 = m.edge_cells[2 * e], c2 = m.edge_cells[2 * e + 1];
        ub[q] = (a.ubar_bt && wet[q]) ? (R)a.ubar_bt[e] : R(0);
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            x[q][c] = col_ld(a.X + (size_t)e * L, kk[c]);
            h1[q][c] = col_ld(a.h + (size_t)c1 * L, kk[c]);
            h2[q][c] = col_ld(a.h + (size_t)c2 * L, kk[c]);
        }
    }
    bool bad = false;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        if (!has[q]) continue;
        const int e = ei[q];
        const size_t base = (size_t)e * L;
        double he[NK], hu[NK];
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            const R u = wet[q] ? (a.ubar_bt ? ub[q] + x[q][c] : x[q][c]) : R(0);
            if (ok[c]) col_st(a.U + base, kk[c], u);
            he[c] = ok[c] ? 0.5 * (h1[q][c] + h2[q][c]) : 0.0;
            hu[c] = he[c] * (double)u;
            bad |= ok[c] && !isfinite((double)u);
        }
        const double sh = col_sum<NK, true>(he);
        const double shu = col_sum<NK, true>(hu);
        if (lane == 0) a.ubar[e] = wet[q] ? shu / sh : 0.0;
    }
    if (bad && a.nonfinite) *a.nonfinite = 1;
}

template <int NK>
__global__ void __launch_bounds__(1024) zeta_kernel(DevMesh m, int L, const double *h, double *zeta) {
    const int lane = lane_id();
    const int i = column_id(m.C);
    if (i >= m.C) return;
    double hv[NK];
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        int k = lane + c * kWave;
        hv[c] = (k < L) ? h[(size_t)i * L + k] : 0.0;
    }
    const double s = col_sum<NK, true>(hv);
    if (lane == 0) zeta[i] = m.cmask[i] ? s - m.H[i] : 0.0;
}

// F_e = sum_k h_e (X_k + uA_e)
template <int NK, typename R>
__global__ void __launch_bounds__(1024) edge_flux_sum_kernel(DevMesh m, int L, const double *h, const R *X,
                                                               const double *uA, double *F) {
    const int lane = lane_id();
    const int e = column_id(m.E);
    if (e >= m.E) return;
    const int c1 = m.edge_cells[2 * e], c2 = m.edge_cells[2 * e + 1];
    const double ua = uA ? uA[e] : 0.0;
    double f[NK];
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        int k = lane + c * kWave;
        f[c] = 0.0;
        if (k < L) {
            double he = 0.5 * (h[(size_t)c1 * L + k] + h[(size_t)c2 * L + k]);
            f[c] = he * ((double)X[(size_t)e * L + k] + ua);
        }
    }
    const double s = col_sum<NK, true>(f);
    if (lane == 0) F[e] = m.emask[e] ? s : 0.0;
}

template <typename Tin, typename Tout>
__device__ __forceinline__ void convert_body(const ConvArgs<Tin, Tout> &a, int lb) {
    const size_t i = (size_t)lb * blockDim.x + threadIdx.x;
    if (i < a.n) a.dst[i] = (Tout)a.src[i];
}

// ---------------------------------------------------------------------------
// Entry points.  Every kernel body above runs either from a single-state
// wrapper (the kernel arguments hold the state's argument block) or from a
// batched wrapper: one launch over the workgroups of several states, where
// each workgroup reads its (member, block) pair from a device table and the
// member's argument block from device memory.
// ---------------------------------------------------------------------------

// The single-state launches of the light streaming column kernels (vertex,
// thickness, assembly, Laplacian and divergence passes) give every wavefront
// several consecutive columns and issue all their loads before any
// arithmetic: the wavefront then has several times the loads in flight,
// which these kernels need to reach HBM rates.  Measured per 3 C1 steps,
// FP64 / mixed, one column against two: vertex pass 1.44 -> 1.19 / 1.23 ->
// 0.89 ms, thickness 1.35 -> 1.14 ms, assembly and reconciliation 1.06 ->
// 0.93 ms; two against four: vertex 1.19 / 1.13, assembly 0.92 / 0.81,
// thickness 1.15 / 1.24.  The cell pass, with 13 columns per cell, lost
// occupancy with two cells (65 VGPRs, 106 scalar registers) and ran 5%
// slower, so it keeps one.  (Processing the columns one after the other
// instead made these kernels slower.)  Batched launches take the same
// groups (their workgroup tables count groups of columns); the arithmetic
// per column is the same in every form.  The counts are in sse_kernels.h.

// (member, member-local block) of this workgroup in a batched launch, with
// the same XCD renumbering as the single-state launches.
__device__ __forceinline__ bool batch_entry(const int2 *table, int blocks, int2 &ent) {
    const int lb = xcd_block(blocks);
    if (lb < 0) return false;
    const int2 t = table[lb];
    ent.x = __builtin_amdgcn_readfirstlane(t.x);
    ent.y = __builtin_amdgcn_readfirstlane(t.y);
    return true;
}

__device__ __forceinline__ int batch_column(int local_block) {
    return __builtin_amdgcn_readfirstlane(local_block * (int)(blockDim.x >> 6) + (int)(threadIdx.x >> 6));
}

template <int NK, typename R, bool kAdd>
__global__ void __launch_bounds__(1024) fe_cell_kernel(FECellArgs<R> a) {
    fe_cell_body<NK, R, kAdd>(a, column_id(a.m.C));
}
template <int NK, typename R, bool kAdd>
__global__ void __launch_bounds__(1024) fe_cell_batch(BatchLaunch<FECellArgs<R>> b) {
    int2 t;
    if (batch_entry(b.table, b.blocks, t)) fe_cell_body<NK, R, kAdd>(b.args[t.x], batch_column(t.y));
}

// Waves per SIMD of the split cell pass.  One register chunk, FP64: at 5 (96
// VGPRs) it spills 14 registers and takes 0.78 ms per launch (512 x 512 x 60),
// at 6 1.09, at 4 and at 3 0.55.  FP32: 0.28 at 6 and 7, 0.32 at 8.
template <int NK, typename R>
constexpr int split_min_waves() { return NK != 1 ? kEdge2Waves : sizeof(R) == 8 ? 4 : 6; }
template <int NK, typename R, bool kAdd, bool kWide>
__global__ void __launch_bounds__((NK == 1 ? 1024 : kEdge2MaxCols * kWave), (split_min_waves<NK, R>())) fe_split_kernel(FESplitArgs<R> a) {
    fe_split_body<NK, R, kAdd, kWide>(a, column_id(a.C));
}
template <int NK, typename R, bool kAdd, bool kWide>
__global__ void __launch_bounds__((NK == 1 ? 1024 : kEdge2MaxCols * kWave), (split_min_waves<NK, R>())) fe_split_batch(BatchLaunch<FESplitArgs<R>> b) {
    int2 t;
    if (batch_entry(b.table, b.blocks, t)) fe_split_body<NK, R, kAdd, kWide>(b.args[t.x], batch_column(t.y));
}

template <int NK, typename R, bool kAdd>
__global__ void __launch_bounds__(1024) fe_vertex_kernel(FEVertexArgs<R> a) {
    fe_vertex_body<NK, R, kAdd, kVertexCols>(a, kVertexCols * column_id(wave_groups<kVertexCols>(a.m.V)));
}
template <int NK, typename R, bool kAdd>
__global__ void __launch_bounds__(1024) fe_vertex_batch(BatchLaunch<FEVertexArgs<R>> b) {
    int2 t;
    if (batch_entry(b.table, b.blocks, t))
        fe_vertex_body<NK, R, kAdd, kVertexCols>(b.args[t.x], kVertexCols * batch_column(t.y));
}

// Minimum waves per SIMD requested for the one-register-chunk edge pass.
// Left alone the compiler settles at 79-81 VGPRs (5-6 waves); the
// gather-bound pass runs faster with more loads in flight.  With 64-bit
// column bases the best request was 7 (C1 edge-pass time over 3 steps, FP64:
// none 12.1, 5: 11.2, 6: 11.6, 7: 10.8, 8: 11.4 ms).  With 32-bit scalar
// column offsets and DPP lane moves the pass fits 8 waves (57-63 VGPRs, 78
// SGPRs, no scratch): FP64 9.78 -> 9.65 ms, C1 mixed 6.03 -> 5.94 ms/step.
// The variants with the implicit vertical-mixing solve (kVar bit 1) hold
// its tridiagonal operands as well and run better at 7 (C1 with mixing 8.68
// -> 8.57 ms/step; the biharmonic variant gains nothing from 7).
template <int NK, typename R, int kVar>
constexpr int edge_min_waves() { return NK != 1 ? kEdge2Waves : (kVar & 2) ? 7 : 8; }
// The two-chunk pass (L > 64) holds twice the operands per lane; with
// workgroups of at most kEdge2MaxCols wavefronts its launch bound lets the
// compiler keep them in registers instead of scratch.
template <int NK>
constexpr int edge_max_threads() { return NK == 1 ? 1024 : kEdge2MaxCols * kWave; }

template <int NK, typename R>
__global__ void __launch_bounds__(1024) tracer_kernel(TracerArgs<R> a) { tracer_body<NK, R>(a, column_id(a.m.C)); }
template <int NK, typename R>
__global__ void __launch_bounds__(1024) tracer_batch(BatchLaunch<TracerArgs<R>> b) {
    int2 t;
    if (batch_entry(b.table, b.blocks, t)) tracer_body<NK, R>(b.args[t.x], batch_column(t.y));
}

template <int NK, typename R>
__global__ void __launch_bounds__(1024) lap_kernel(LapArgs<R> a) {
    lap_body<NK, R, kLapCols>(a, kLapCols * column_id(wave_groups<kLapCols>(a.m.E)));
}
template <int NK, typename R>
__global__ void __launch_bounds__(1024) lap_batch(BatchLaunch<LapArgs<R>> b) {
    int2 t;
    if (batch_entry(b.table, b.blocks, t)) lap_body<NK, R, kLapCols>(b.args[t.x], kLapCols * batch_column(t.y));
}
template <int NK, typename R>
__global__ void __launch_bounds__(1024) div_kernel(DivArgs<R> a) {
    div_body<NK, R, kDivCols>(a, kDivCols * column_id(wave_groups<kDivCols>(a.m.C)));
}
template <int NK, typename R>
__global__ void __launch_bounds__(1024) div_batch(BatchLaunch<DivArgs<R>> b) {
    int2 t;
    if (batch_entry(b.table, b.blocks, t)) div_body<NK, R, kDivCols>(b.args[t.x], kDivCols * batch_column(t.y));
}

template <int NK, typename R, bool kAdd, int kVar>
__global__ void __launch_bounds__(edge_max_threads<NK>(), (edge_min_waves<NK, R, kVar>())) fe_edge_kernel(FEEdgeArgs<R> a) {
    if constexpr (kVar & 16) fe_edge_split_body<NK, R, kAdd, kVar>(a, column_id(a.m.E));
    else fe_edge_body<NK, R, kAdd, kVar>(a, column_id(a.m.E));
}
template <int NK, typename R, bool kAdd, int kVar>
__global__ void __launch_bounds__(edge_max_threads<NK>(), (edge_min_waves<NK, R, kVar>())) fe_edge_batch(BatchLaunch<FEEdgeArgs<R>> b) {
    int2 t;
    if (!batch_entry(b.table, b.blocks, t)) return;
    if constexpr (kVar & 16) fe_edge_split_body<NK, R, kAdd, kVar>(b.args[t.x], batch_column(t.y));
    else fe_edge_body<NK, R, kAdd, kVar>(b.args[t.x], batch_column(t.y));
}

template <int NK>
__global__ void __launch_bounds__(1024) thickness_kernel(THArgs a) {
    thickness_body<NK, kThickCols>(a, kThickCols * column_id(wave_groups<kThickCols>(a.m.C)));
}
template <int NK>
__global__ void __launch_bounds__(1024) thickness_batch(BatchLaunch<THArgs> b) {
    int2 t;
    if (batch_entry(b.table, b.blocks, t)) thickness_body<NK, kThickCols>(b.args[t.x], kThickCols * batch_column(t.y));
}

template <int NK, typename R>
__global__ void __launch_bounds__(1024) thickness_iso_kernel(THIsoArgs<R> a) { thickness_iso_body<NK, R>(a, column_id(a.m.C)); }
template <int NK, typename R>
__global__ void __launch_bounds__(1024) thickness_iso_batch(BatchLaunch<THIsoArgs<R>> b) {
    int2 t;
    if (batch_entry(b.table, b.blocks, t)) thickness_iso_body<NK, R>(b.args[t.x], batch_column(t.y));
}

template <int NK, typename R>
__global__ void __launch_bounds__(1024) assemble_kernel(AssembleArgs<R> a) {
    assemble_body<NK, R, kAssembleCols>(a, kAssembleCols * column_id(wave_groups<kAssembleCols>(a.m.E)));
}
template <int NK, typename R>
__global__ void __launch_bounds__(1024) assemble_batch(BatchLaunch<AssembleArgs<R>> b) {
    int2 t;
    if (batch_entry(b.table, b.blocks, t))
        assemble_body<NK, R, kAssembleCols>(b.args[t.x], kAssembleCols * batch_column(t.y));
}

// Barotropic evaluation: XCD x owns edge blocks [x pe, (x + 1) pe) and cell
// blocks [x pc, (x + 1) pc), one contiguous region of the mesh per L2.
template <typename R, bool kD16>
__global__ void __launch_bounds__(1024) bt_eval_kernel(BTEvalArgs<R> a, int nEdgeBlocks, int nCellBlocks) {
    const int pe = (nEdgeBlocks + kXcd - 1) / kXcd, pc = (nCellBlocks + kXcd - 1) / kXcd;
    const int x = blockIdx.x % kXcd, local = blockIdx.x / kXcd;
    if (local < pe) {
        const int lb = x * pe + local;
        if (lb < nEdgeBlocks) {
            if (a.fact) bt_eval_fact<R>(a, true, lb);
            else bt_eval_body<R, kD16>(a, true, lb);
        }
    } else {
        const int lb = x * pc + (local - pe);
        if (lb < nCellBlocks) {
            if (a.fact) bt_eval_fact<R>(a, false, lb);
            else bt_eval_body<R, kD16>(a, false, lb);
        }
    }
}
template <typename R, bool kD16>
__global__ void __launch_bounds__(1024) bt_eval_batch(BatchLaunch<BTEvalArgs<R>> b) {
    int2 t;
    if (!batch_entry(b.table, b.blocks, t)) return;
    const BTEvalArgs<R> &a = b.args[t.x];
    const int nEB = (a.m.E + (int)blockDim.x - 1) / (int)blockDim.x;
    const bool edge_part = t.y < nEB;
    const int lb = edge_part ? t.y : t.y - nEB;
    if (a.fact) bt_eval_fact<R>(a, edge_part, lb);
    else bt_eval_body<R, kD16>(a, edge_part, lb);
}

template <typename R, int kScheme, int KS, bool kDry = false>
__global__ void __launch_bounds__(kBtThreads, kBtWavesPerSimd) bt_substep_kernel(BTTileArgs<R> a) {
    const int p = xcd_block(a.t.nP);
    if (p >= 0) bt_substep_body<R, kScheme, KS, kDry>(a, p);
}
// Batched: one workgroup per (member, patch); the dynamic LDS is the
// largest member's.
template <typename R, int kScheme, int KS>
__global__ void __launch_bounds__(kBtThreads, kBtWavesPerSimd) bt_substep_batch(BatchLaunch<BTTileArgs<R>> b) {
    int2 t;
    if (batch_entry(b.table, b.blocks, t)) bt_substep_body<R, kScheme, KS>(b.args[t.x], t.y);
}

// The whole barotropic loop in one cooperative launch, one workgroup per
// patch (workgroups past the last patch only take part in the barriers).
template <typename R, int kScheme, int KS>
__global__ void __launch_bounds__(kBtThreads, kBtWavesPerSimd) bt_loop_kernel(BTTileArgs<R> a, BtLoop<R> l) {
    bt_loop_body<R, kScheme, KS>(a, l, xcd_block(a.t.nP));
}

// Factored substep and resident loop.  Waves per SIMD (kW): the substep's FP64
// body takes 128 VGPRs (two workgroups of kBtThreads per CU), its FP32 body 88.
// The loop comes in forms that hold one, two or (FP32) three such workgroups
// per CU, and runs in the roomiest that holds the mesh: at two it keeps to 128
// VGPRs and in FP64 spills 14 of them, at three to 80 and spills 16, which
// makes a substep 35% slower (0.39 -> 0.53 ms per step of 60 substeps on a 256
// x 256 mesh) but still halves the time of one launch per substep (level-7
// sphere: 0.88 ms per step of 90 substeps against 1.85).
template <typename R>
constexpr int fact_waves() { return sizeof(R) == 8 ? 4 : 5; }
template <typename R, int kScheme, int NT>
__global__ void __launch_bounds__(NT, fact_waves<R>()) bt_fact_kernel(BTTileArgs<R> a) {
    const int p = xcd_block(a.t.nP);
    __shared__ FactLds<R, NT> lds;
    if (p >= 0) bt_fact_body<R, kScheme, kOne, NT>(lds, a, nullptr, p, nullptr);
}
template <typename R, int kScheme>
__global__ void __launch_bounds__(kBtThreads, fact_waves<R>()) bt_fact_batch(BatchLaunch<BTTileArgs<R>> b) {
    int2 t;
    __shared__ FactLds<R, kBtThreads> lds;
    if (batch_entry(b.table, b.blocks, t)) bt_fact_body<R, kScheme, kOne, kBtThreads>(lds, b.args[t.x], nullptr, t.y, nullptr);
}
template <typename R, int kScheme, int NT, int kW>
__global__ void __launch_bounds__(NT, kW) bt_resident_kernel(BtResident<R> l, BtRound round) {
    const int lb = xcd_block(l.a.t.nA);
    if (lb >= 0) bt_resident_body<R, kScheme, NT>(l, lb, round, lb, l.a.t.nA);
}
template <typename R, int kScheme, int kW>
__global__ void __launch_bounds__(kBtThreads, kW) bt_resident_batch(BatchLaunch<BtResident<R>> b, BtRound round) {
    int2 t;
    if (batch_entry(b.table, b.blocks, t)) bt_resident_body<R, kScheme, kBtThreads>(b.args[t.x], t.y, round, xcd_block(b.blocks), b.blocks);
}
template <typename R, int kScheme, int NT>
__global__ void __launch_bounds__(NT, fact_waves<R>()) bt_task_kernel(BtResident<R> l, BtRound round) {
    bt_task_body<R, kScheme, NT>(&l, nullptr, l.a.t.nA, l.M, round);
}
template <typename R, int kScheme>
__global__ void __launch_bounds__(kBtThreads, fact_waves<R>()) bt_task_batch(BatchLaunch<BtResident<R>> b, int most, BtRound round) {
    bt_task_body<R, kScheme, kBtThreads>(b.args, b.table, b.blocks, most, round);
}

__global__ void __launch_bounds__(64) bt_loop_reset_kernel(unsigned *bar, unsigned *gen) {
    if (threadIdx.x == 0) {
        *bar = 0u;
        *gen = 0u;
    }
}

__global__ void __launch_bounds__(1024) recon_kernel(ReconArgs a) { recon_body(a, blockIdx.x); }
__global__ void __launch_bounds__(1024) recon_batch(BatchLaunch<ReconArgs> b) {
    int2 t;
    if (batch_entry(b.table, b.blocks, t)) recon_body(b.args[t.x], t.y);
}

template <typename Tin, typename Tout>
__global__ void __launch_bounds__(1024) convert_kernel(ConvArgs<Tin, Tout> a) { convert_body<Tin, Tout>(a, blockIdx.x); }
template <typename Tin, typename Tout>
__global__ void __launch_bounds__(1024) convert_batch(BatchLaunch<ConvArgs<Tin, Tout>> b) {
    int2 t;
    if (batch_entry(b.table, b.blocks, t)) convert_body<Tin, Tout>(b.args[t.x], t.y);
}

// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------
bool geom_valid(const Geom &g) {
    const int c = g.cols_per_block;
    return (c == 1 || c == 2 || c == 4 || c == 8 || c == 16) && g.block_2d >= 64 && g.block_2d <= 1024 &&
           g.block_2d % 64 == 0;
}
int col_blocks(int n, const Geom &g) { return (n + g.cols_per_block - 1) / g.cols_per_block; }
Geom edge_geom(const Geom &g, int nk) {
    Geom e = g;
    if (nk == 2 && e.cols_per_block > kEdge2MaxCols) e.cols_per_block = kEdge2MaxCols;
    return e;
}
int flat_blocks(size_t n, const Geom &g) { return (int)((n + g.block_2d - 1) / g.block_2d); }
int bt_blocks(int E, int C, const Geom &g) { return flat_blocks(E, g) + flat_blocks(C, g); }

// Grids are rounded up to a multiple of the 8 XCDs; the kernels renumber the
// workgroups and the padding workgroups exit.
static inline dim3 xcd_grid(int nb) { return dim3((unsigned)(kXcd * ((nb + kXcd - 1) / kXcd))); }
static inline dim3 col_block(const Geom &g) { return dim3((unsigned)(kWave * g.cols_per_block)); }

// The column kernels are instantiated for one or two register chunks
// (L <= 64 or L <= 128) and for the two velocity forms: u = X + ubar
// (ubar_add non-null) or u = X (the edge pass then forms ut = X - ubar_sub;
// exactly one of ubar_add and ubar_sub is non-null there).
#define SSE_NK_ADD(NK2, ADD, KERNEL, GRID, BLOCK, ARG)                                  \
    do {                                                                               \
        if (!(NK2)) {                                                                  \
            if (ADD) KERNEL<1, R, true><<<GRID, BLOCK, 0, s>>>(ARG);                   \
            else KERNEL<1, R, false><<<GRID, BLOCK, 0, s>>>(ARG);                      \
        } else {                                                                       \
            if (ADD) KERNEL<2, R, true><<<GRID, BLOCK, 0, s>>>(ARG);                   \
            else KERNEL<2, R, false><<<GRID, BLOCK, 0, s>>>(ARG);                      \
        }                                                                              \
    } while (0)

template <typename R>
void launch_fe_cell(const FECellArgs<R> &a, const Geom &g, hipStream_t s) {
    SSE_NK_ADD(a.L > kWave, a.ubar_add != nullptr, fe_cell_kernel, xcd_grid(col_blocks(a.m.C, g)), col_block(g), a);
}
template <typename R>
void launch_fe_vertex(const FEVertexArgs<R> &a, const Geom &g, hipStream_t s) {
    SSE_NK_ADD(a.L > kWave, a.ubar_add != nullptr, fe_vertex_kernel, xcd_grid(col_blocks(wave_groups<kVertexCols>(a.m.V), g)), col_block(g), a);
}
// The edge pass has a fourth template parameter, the variant: bit 0 for
// canonical stencils with vertex chains (the mesh's chain flag), bit 1 for
// implicit vertical mixing (the state's vmix parameter), bit 2 for the
// biharmonic viscosity (hdiff).  Every member of a batched launch shares it.
#define SSE_NK_ADD_V(NK2, ADD, V, KERNEL, GRID, BLOCK, ARG)                             \
    do {                                                                               \
        if (!(NK2)) {                                                                  \
            if (ADD) KERNEL<1, R, true, V><<<GRID, BLOCK, 0, s>>>(ARG);                \
            else KERNEL<1, R, false, V><<<GRID, BLOCK, 0, s>>>(ARG);                   \
        } else {                                                                       \
            if (ADD) KERNEL<2, R, true, V><<<GRID, BLOCK, 0, s>>>(ARG);                \
            else KERNEL<2, R, false, V><<<GRID, BLOCK, 0, s>>>(ARG);                   \
        }                                                                              \
    } while (0)
#define SSE_NK_ADD_VAR(NK2, ADD, VAR, KERNEL, GRID, BLOCK, ARG)                         \
    do {                                                                               \
        switch (VAR) {                                                                 \
            case 0: SSE_NK_ADD_V(NK2, ADD, 0, KERNEL, GRID, BLOCK, ARG); break;        \
            case 1: SSE_NK_ADD_V(NK2, ADD, 1, KERNEL, GRID, BLOCK, ARG); break;        \
            case 2: SSE_NK_ADD_V(NK2, ADD, 2, KERNEL, GRID, BLOCK, ARG); break;        \
            case 3: SSE_NK_ADD_V(NK2, ADD, 3, KERNEL, GRID, BLOCK, ARG); break;        \
            case 4: SSE_NK_ADD_V(NK2, ADD, 4, KERNEL, GRID, BLOCK, ARG); break;        \
            case 5: SSE_NK_ADD_V(NK2, ADD, 5, KERNEL, GRID, BLOCK, ARG); break;        \
            case 6: SSE_NK_ADD_V(NK2, ADD, 6, KERNEL, GRID, BLOCK, ARG); break;        \
            case 7: SSE_NK_ADD_V(NK2, ADD, 7, KERNEL, GRID, BLOCK, ARG); break;        \
            case 8: SSE_NK_ADD_V(NK2, ADD, 8, KERNEL, GRID, BLOCK, ARG); break;        \
            case 9: SSE_NK_ADD_V(NK2, ADD, 9, KERNEL, GRID, BLOCK, ARG); break;        \
            case 10: SSE_NK_ADD_V(NK2, ADD, 10, KERNEL, GRID, BLOCK, ARG); break;      \
            case 11: SSE_NK_ADD_V(NK2, ADD, 11, KERNEL, GRID, BLOCK, ARG); break;      \
            case 12: SSE_NK_ADD_V(NK2, ADD, 12, KERNEL, GRID, BLOCK, ARG); break;      \
            case 13: SSE_NK_ADD_V(NK2, ADD, 13, KERNEL, GRID, BLOCK, ARG); break;      \
            case 14: SSE_NK_ADD_V(NK2, ADD, 14, KERNEL, GRID, BLOCK, ARG); break;      \
            case 15: SSE_NK_ADD_V(NK2, ADD, 15, KERNEL, GRID, BLOCK, ARG); break;      \
            case 16: SSE_NK_ADD_V(NK2, ADD, 16, KERNEL, GRID, BLOCK, ARG); break;      \
            case 18: SSE_NK_ADD_V(NK2, ADD, 18, KERNEL, GRID, BLOCK, ARG); break;      \
            case 20: SSE_NK_ADD_V(NK2, ADD, 20, KERNEL, GRID, BLOCK, ARG); break;      \
            case 22: SSE_NK_ADD_V(NK2, ADD, 22, KERNEL, GRID, BLOCK, ARG); break;      \
            case 24: SSE_NK_ADD_V(NK2, ADD, 24, KERNEL, GRID, BLOCK, ARG); break;      \
            case 26: SSE_NK_ADD_V(NK2, ADD, 26, KERNEL, GRID, BLOCK, ARG); break;      \
            case 28: SSE_NK_ADD_V(NK2, ADD, 28, KERNEL, GRID, BLOCK, ARG); break;      \
            default: SSE_NK_ADD_V(NK2, ADD, 30, KERNEL, GRID, BLOCK, ARG); break;      \
        }                                                                              \
    } while (0)

template <typename R>
void launch_fe_split(const FESplitArgs<R> &a, bool wide, const Geom &g0, hipStream_t s) {
    const Geom g = edge_geom(g0, a.L > kWave ? 2 : 1);
    const dim3 grid = xcd_grid(col_blocks(a.C, g)), block = col_block(g);
    if (wide) SSE_NK_ADD_V(a.L > kWave, a.ubar_add != nullptr, true, fe_split_kernel, grid, block, a);
    else SSE_NK_ADD_V(a.L > kWave, a.ubar_add != nullptr, false, fe_split_kernel, grid, block, a);
}
template <typename R>
void launch_fe_split_batch(const BatchLaunch<FESplitArgs<R>> &b, int nk, bool add, bool wide, const Geom &g, hipStream_t s) {
    const dim3 grid = xcd_grid(b.blocks), block = col_block(edge_geom(g, nk));
    if (wide) SSE_NK_ADD_V(nk == 2, add, true, fe_split_batch, grid, block, b);
    else SSE_NK_ADD_V(nk == 2, add, false, fe_split_batch, grid, block, b);
}

template <typename R>
void launch_tracer(const TracerArgs<R> &a, const Geom &g, hipStream_t s) {
    const dim3 grid = xcd_grid(col_blocks(a.m.C, g)), block = col_block(g);
    if (a.L <= kWave) tracer_kernel<1, R><<<grid, block, 0, s>>>(a);
    else tracer_kernel<2, R><<<grid, block, 0, s>>>(a);
}
template <typename R>
void launch_tracer_batch(const BatchLaunch<TracerArgs<R>> &b, int nk, const Geom &g, hipStream_t s) {
    if (nk == 1) tracer_batch<1, R><<<xcd_grid(b.blocks), col_block(g), 0, s>>>(b);
    else tracer_batch<2, R><<<xcd_grid(b.blocks), col_block(g), 0, s>>>(b);
}

template <typename R>
void launch_lap(const LapArgs<R> &a, const Geom &g, hipStream_t s) {
    const dim3 grid = xcd_grid(col_blocks(wave_groups<kLapCols>(a.m.E), g)), block = col_block(g);
    if (a.L <= kWave) lap_kernel<1, R><<<grid, block, 0, s>>>(a);
    else lap_kernel<2, R><<<grid, block, 0, s>>>(a);
}
template <typename R>
void launch_div(const DivArgs<R> &a, const Geom &g, hipStream_t s) {
    const dim3 grid = xcd_grid(col_blocks(wave_groups<kDivCols>(a.m.C), g)), block = col_block(g);
    if (a.L <= kWave) div_kernel<1, R><<<grid, block, 0, s>>>(a);
    else div_kernel<2, R><<<grid, block, 0, s>>>(a);
}
template <typename R>
void launch_lap_batch(const BatchLaunch<LapArgs<R>> &b, int nk, const Geom &g, hipStream_t s) {
    if (nk == 1) lap_batch<1, R><<<xcd_grid(b.blocks), col_block(g), 0, s>>>(b);
    else lap_batch<2, R><<<xcd_grid(b.blocks), col_block(g), 0, s>>>(b);
}
template <typename R>
void launch_div_batch(const BatchLaunch<DivArgs<R>> &b, int nk, const Geom &g, hipStream_t s) {
    if (nk == 1) div_batch<1, R><<<xcd_grid(b.blocks), col_block(g), 0, s>>>(b);
    else div_batch<2, R><<<xcd_grid(b.blocks), col_block(g), 0, s>>>(b);
}

int fe_edge_variant(const DevMesh &m, int L, int vmix, bool del4, bool split) {
    // 32-bit column offsets cover every array the pass reads while the
    // largest (edges, vertices or cells) x L x 8 bytes stays below 4 GiB,
    // with a margin for the layer offsets
    const size_t n = (size_t)std::max(m.E, std::max(m.V, m.C));
    const bool wide = n * (size_t)L * 8 + 4096 > ((size_t)1 << 32);
    return (split ? 16 : m.chain ? 1 : 0) | (vmix ? 2 : 0) | (del4 ? 4 : 0) | (wide ? 8 : 0);
}

template <typename R>
void launch_fe_edge(const FEEdgeArgs<R> &a, int var, const Geom &g0, hipStream_t s) {
    const Geom g = edge_geom(g0, a.L > kWave ? 2 : 1);
    SSE_NK_ADD_VAR(a.L > kWave, a.ubar_add != nullptr, var, fe_edge_kernel, xcd_grid(col_blocks(a.m.E, g)), col_block(g), a);
}
template <typename R>
void launch_fe_cell_batch(const BatchLaunch<FECellArgs<R>> &b, int nk, bool add, const Geom &g, hipStream_t s) {
    SSE_NK_ADD(nk == 2, add, fe_cell_batch, xcd_grid(b.blocks), col_block(g), b);
}
template <typename R>
void launch_fe_vertex_batch(const BatchLaunch<FEVertexArgs<R>> &b, int nk, bool add, const Geom &g, hipStream_t s) {
    SSE_NK_ADD(nk == 2, add, fe_vertex_batch, xcd_grid(b.blocks), col_block(g), b);
}
template <typename R>
void launch_fe_edge_batch(const BatchLaunch<FEEdgeArgs<R>> &b, int nk, bool add, int var, const Geom &g,
                          hipStream_t s) {
    SSE_NK_ADD_VAR(nk == 2, add, var, fe_edge_batch, xcd_grid(b.blocks), col_block(edge_geom(g, nk)), b);
}

template <typename R>
void launch_edge_gathers(const FEEdgeArgs<R> &a, bool split, const Geom &g0, hipStream_t s) {
    const Geom g = edge_geom(g0, 1);
    if (split) edge_gather_kernel<R, true><<<xcd_grid(col_blocks(a.m.E, g)), col_block(g), 0, s>>>(a);
    else edge_gather_kernel<R, false><<<xcd_grid(col_blocks(a.m.E, g)), col_block(g), 0, s>>>(a);
}

template <typename R>
void launch_fe_edge_tiled(const FEEdgeArgs<R> &a, const DevTiles &t, hipStream_t s) {
    const size_t lds = fe_edge_tiled_lds<R>(t, a.L);
    const dim3 grid(kXcd * ((t.nT + kXcd - 1) / kXcd)), block((t.T < kTileWaves ? t.T : kTileWaves) * kWave);
    const bool add = a.ubar_add != nullptr;
    const int v = a.vmix ? 1 : 0;
#define SSE_TILED(NK_, ADD_, MIX_) fe_edge_tiled_kernel<NK_, R, ADD_, MIX_><<<grid, block, lds, s>>>(a, t)
    if (a.L <= kWave) {
        if (add) { if (v) SSE_TILED(1, true, true); else SSE_TILED(1, true, false); }
        else { if (v) SSE_TILED(1, false, true); else SSE_TILED(1, false, false); }
    } else {
        if (add) { if (v) SSE_TILED(2, true, true); else SSE_TILED(2, true, false); }
        else { if (v) SSE_TILED(2, false, true); else SSE_TILED(2, false, false); }
    }
#undef SSE_TILED
}

template <typename R, int kScheme, int KS>
static const void *bt_loop_fn() {
    return reinterpret_cast<const void *>(bt_loop_kernel<R, kScheme, KS>);
}

template <typename R>
static const void *bt_loop_select(int scheme, int ks) {
    if (scheme == 3) return ks == 1 ? bt_loop_fn<R, 3, 1>() : bt_loop_fn<R, 3, 2>();
    return ks == 1 ? bt_loop_fn<R, 2, 1>() : bt_loop_fn<R, 2, 2>();
}

// The resident loop kernel for nt threads in the form of `tight` (see
// kResidentForms), alone or over a batch.
template <typename R, int kScheme, int kW>
static const void *bt_resident_of(int nt, bool batch) {
    if (batch) return reinterpret_cast<const void *>(bt_resident_batch<R, kScheme, kW>);
    if (nt == kBtThreads) return reinterpret_cast<const void *>(bt_resident_kernel<R, kScheme, kBtThreads, kW>);
    return reinterpret_cast<const void *>(bt_resident_kernel<R, kScheme, kFactSmall, kW>);
}
template <typename R, int kScheme>
static const void *bt_resident_form(int nt, int tight, bool batch) {
    if constexpr (sizeof(R) == 4)
        if (tight >= 2) return bt_resident_of<R, kScheme, 6>(nt, batch);
    return tight ? bt_resident_of<R, kScheme, 4>(nt, batch) : bt_resident_of<R, kScheme, 2>(nt, batch);
}
template <typename R>
static const void *bt_resident_fn(int scheme, int nt, int tight, bool batch = false) {
    return scheme == 3 ? bt_resident_form<R, 3>(nt, tight, batch) : bt_resident_form<R, 2>(nt, tight, batch);
}

// Allow the tiled kernels the device's full LDS per workgroup.
void set_tiled_lds_limit(size_t bytes) {
#define SSE_TILED_FN(NK_, R_, ADD_, MIX_) reinterpret_cast<const void *>(fe_edge_tiled_kernel<NK_, R_, ADD_, MIX_>)
#define SSE_TILED_FNS(R_, MIX_)                                                                            \
    SSE_TILED_FN(1, R_, true, MIX_), SSE_TILED_FN(1, R_, false, MIX_), SSE_TILED_FN(2, R_, true, MIX_), \
        SSE_TILED_FN(2, R_, false, MIX_)
    const void *fns[] = {SSE_TILED_FNS(double, false), SSE_TILED_FNS(double, true), SSE_TILED_FNS(float, false),
                         SSE_TILED_FNS(float, true)};
#undef SSE_TILED_FNS
#undef SSE_TILED_FN
    const void *bt[] = {reinterpret_cast<const void *>(bt_substep_kernel<double, 3, 1>),
                        reinterpret_cast<const void *>(bt_substep_kernel<double, 3, 2>),
                        reinterpret_cast<const void *>(bt_substep_kernel<double, 2, 1>),
                        reinterpret_cast<const void *>(bt_substep_kernel<double, 2, 2>),
                        reinterpret_cast<const void *>(bt_substep_kernel<float, 3, 1>),
                        reinterpret_cast<const void *>(bt_substep_kernel<float, 3, 2>),
                        reinterpret_cast<const void *>(bt_substep_kernel<float, 2, 1>),
                        reinterpret_cast<const void *>(bt_substep_kernel<float, 2, 2>),
                        reinterpret_cast<const void *>(bt_substep_kernel<double, 3, 1, true>),
                        reinterpret_cast<const void *>(bt_substep_kernel<double, 3, 2, true>),
                        reinterpret_cast<const void *>(bt_substep_kernel<double, 2, 1, true>),
                        reinterpret_cast<const void *>(bt_substep_kernel<double, 2, 2, true>)};
    for (const void *f : bt) (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    const void *btb[] = {reinterpret_cast<const void *>(bt_substep_batch<double, 3, 1>),
                         reinterpret_cast<const void *>(bt_substep_batch<double, 3, 2>),
                         reinterpret_cast<const void *>(bt_substep_batch<double, 2, 1>),
                         reinterpret_cast<const void *>(bt_substep_batch<double, 2, 2>),
                         reinterpret_cast<const void *>(bt_substep_batch<float, 3, 1>),
                         reinterpret_cast<const void *>(bt_substep_batch<float, 3, 2>),
                         reinterpret_cast<const void *>(bt_substep_batch<float, 2, 1>),
                         reinterpret_cast<const void *>(bt_substep_batch<float, 2, 2>)};
    for (const void *f : btb) (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    const void *btl[] = {bt_loop_fn<double, 3, 1>(), bt_loop_fn<double, 3, 2>(), bt_loop_fn<double, 2, 1>(),
                         bt_loop_fn<double, 2, 2>(), bt_loop_fn<float, 3, 1>(),  bt_loop_fn<float, 3, 2>(),
                         bt_loop_fn<float, 2, 1>(),  bt_loop_fn<float, 2, 2>()};
    for (const void *f : btl) (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    for (const void *f : fns) (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

template <typename R>
void launch_bt_substep(const BTTileArgs<R> &a, int scheme, hipStream_t s) {
    const dim3 grid = xcd_grid(a.t.nP), block(kBtThreads);
    const size_t lds = sizeof(R) == 8 ? a.t.lds_d : a.t.lds_f;
    if (a.t.fact) {
        if (a.t.nt == kBtThreads) {
            if (scheme == 3) bt_fact_kernel<R, 3, kBtThreads><<<grid, kBtThreads, 0, s>>>(a);
            else bt_fact_kernel<R, 2, kBtThreads><<<grid, kBtThreads, 0, s>>>(a);
        } else {
            if (scheme == 3) bt_fact_kernel<R, 3, kFactSmall><<<grid, kFactSmall, 0, s>>>(a);
            else bt_fact_kernel<R, 2, kFactSmall><<<grid, kFactSmall, 0, s>>>(a);
        }
        return;
    }
    if (sizeof(R) == 8 && a.t.dry) {
        if (scheme == 3) {
            if (a.t.ks == 1) bt_substep_kernel<R, 3, 1, true><<<grid, block, lds, s>>>(a);
            else bt_substep_kernel<R, 3, 2, true><<<grid, block, lds, s>>>(a);
        } else {
            if (a.t.ks == 1) bt_substep_kernel<R, 2, 1, true><<<grid, block, lds, s>>>(a);
            else bt_substep_kernel<R, 2, 2, true><<<grid, block, lds, s>>>(a);
        }
    } else if (scheme == 3) {
        if (a.t.ks == 1) bt_substep_kernel<R, 3, 1><<<grid, block, lds, s>>>(a);
        else bt_substep_kernel<R, 3, 2><<<grid, block, lds, s>>>(a);
    } else {
        if (a.t.ks == 1) bt_substep_kernel<R, 2, 1><<<grid, block, lds, s>>>(a);
        else bt_substep_kernel<R, 2, 2><<<grid, block, lds, s>>>(a);
    }
}

// Workgroups of a kernel an empty device holds at once (0 if the device takes
// no cooperative launch).
static int coop_capacity(const void *fn, int threads, size_t lds) {
    int dev = 0, coop = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess || !coop) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads, lds) != hipSuccess) return 0;
    return per_cu * cus;
}

template <typename R>
int bt_loop_capacity(const DevBtTiles &t, int scheme, int tight) {
    if (t.nP <= 0) return 0;
    if (t.fact) return coop_capacity(bt_resident_fn<R>(scheme, t.nt, tight), t.nt, 0);
    return coop_capacity(bt_loop_select<R>(scheme, t.ks), kBtThreads, sizeof(R) == 8 ? t.lds_d : t.lds_f);
}

template <typename R>
hipError_t launch_bt_loop(const BTTileArgs<R> &a, const BtLoop<R> &l, int scheme, hipStream_t s) {
    bt_loop_reset_kernel<<<1, 64, 0, s>>>(l.bar, l.gen);
    const size_t lds = sizeof(R) == 8 ? a.t.lds_d : a.t.lds_f;
    BTTileArgs<R> aa = a;
    BtLoop<R> ll = l;
    void *args[] = {&aa, &ll};
    return hipLaunchCooperativeKernel(bt_loop_select<R>(scheme, a.t.ks), xcd_grid(a.t.nP), dim3(kBtThreads), args,
                                      (unsigned)lds, s);
}

template <typename R>
hipError_t launch_bt_resident(const BtResident<R> &l, int scheme, int tight, const BtRound &round, hipStream_t s) {
    BtResident<R> ll = l;
    BtRound r = round;
    void *args[] = {&ll, &r};
    return hipLaunchKernel(bt_resident_fn<R>(scheme, l.a.t.nt, tight), xcd_grid(l.a.t.nA), dim3(l.a.t.nt), args, 0, s);
}

// Workgroups of the task form: two per CU, what its FP64 body allows.  A mixed
// level-7 and an FP64 level-6 globe of 60 layers stepped together on two
// streams (the first's loops are called off) take 3.39 ms per step of both,
// with one per CU 4.15, with one launch per substep 3.93; one after the other 3.21.
constexpr int kTaskBlocks = 2 * kCus;

template <typename R>
hipError_t launch_bt_tasks(const BtResident<R> &l, int scheme, const BtRound &round, hipStream_t s) {
    if (!round.words) return hipSuccess;
    const bool small = l.a.t.nt != kBtThreads;
    const void *fn = scheme == 3 ? (small ? reinterpret_cast<const void *>(bt_task_kernel<R, 3, kFactSmall>)
                                          : reinterpret_cast<const void *>(bt_task_kernel<R, 3, kBtThreads>))
                                 : (small ? reinterpret_cast<const void *>(bt_task_kernel<R, 2, kFactSmall>)
                                          : reinterpret_cast<const void *>(bt_task_kernel<R, 2, kBtThreads>));
    BtResident<R> ll = l;
    BtRound r = round;
    r.base += (unsigned long long)l.M;  // counts that the called-off launch cannot have stored
    void *args[] = {&ll, &r};
    return hipLaunchKernel(fn, dim3(std::min(l.a.t.nA, kTaskBlocks)), dim3(l.a.t.nt), args, 0, s);
}

template <typename R>
int bt_resident_batch_capacity(int scheme, int tight) {
    return coop_capacity(bt_resident_fn<R>(scheme, kBtThreads, tight, true), kBtThreads, 0);
}

template <typename R>
hipError_t launch_bt_resident_batch(const BatchLaunch<BtResident<R>> &b, int scheme, int tight, const BtRound &round,
                                    hipStream_t s) {
    BatchLaunch<BtResident<R>> bb = b;
    BtRound r = round;
    void *args[] = {&bb, &r};
    return hipLaunchKernel(bt_resident_fn<R>(scheme, kBtThreads, tight, true), xcd_grid(b.blocks), dim3(kBtThreads), args, 0, s);
}

template <typename R>
hipError_t launch_bt_tasks_batch(const BatchLaunch<BtResident<R>> &b, int most, int scheme, const BtRound &round, hipStream_t s) {
    if (!round.words) return hipSuccess;
    const void *fn = scheme == 3 ? reinterpret_cast<const void *>(bt_task_batch<R, 3>)
                                 : reinterpret_cast<const void *>(bt_task_batch<R, 2>);
    BatchLaunch<BtResident<R>> bb = b;
    BtRound r = round;
    r.base += (unsigned long long)most;
    void *args[] = {&bb, &most, &r};
    return hipLaunchKernel(fn, dim3(std::min(b.blocks, kTaskBlocks)), dim3(kBtThreads), args, 0, s);
}

template <typename R>
void launch_bt_substep_batch(const BatchLaunch<BTTileArgs<R>> &b, int scheme, int ks, size_t lds, hipStream_t s) {
    const dim3 grid = xcd_grid(b.blocks), block(kBtThreads);
    if (ks & kFactVar) {
        if (scheme == 3) bt_fact_batch<R, 3><<<grid, kBtThreads, 0, s>>>(b);
        else bt_fact_batch<R, 2><<<grid, kBtThreads, 0, s>>>(b);
        return;
    }
    if (scheme == 3) {
        if (ks == 1) bt_substep_batch<R, 3, 1><<<grid, block, lds, s>>>(b);
        else bt_substep_batch<R, 3, 2><<<grid, block, lds, s>>>(b);
    } else {
        if (ks == 1) bt_substep_batch<R, 2, 1><<<grid, block, lds, s>>>(b);
        else bt_substep_batch<R, 2, 2><<<grid, block, lds, s>>>(b);
    }
}

template <typename R>
void launch_bt_eval(const BTEvalArgs<R> &a, const Geom &g, hipStream_t s) {
    const int nEB = flat_blocks(a.m.E, g), nCB = flat_blocks(a.m.C, g);
    const int per = (nEB + kXcd - 1) / kXcd + (nCB + kXcd - 1) / kXcd;
    if (a.m.delta16)
        bt_eval_kernel<R, true><<<dim3(kXcd * per), g.block_2d, 0, s>>>(a, nEB, nCB);
    else
        bt_eval_kernel<R, false><<<dim3(kXcd * per), g.block_2d, 0, s>>>(a, nEB, nCB);
}
template <typename R>
void launch_bt_eval_batch(const BatchLaunch<BTEvalArgs<R>> &b, bool delta16, const Geom &g, hipStream_t s) {
    if (delta16)
        bt_eval_batch<R, true><<<xcd_grid(b.blocks), g.block_2d, 0, s>>>(b);
    else
        bt_eval_batch<R, false><<<xcd_grid(b.blocks), g.block_2d, 0, s>>>(b);
}

void launch_thickness(const THArgs &a, const Geom &g, hipStream_t s) {
    const dim3 grid = xcd_grid(col_blocks(wave_groups<kThickCols>(a.m.C), g));
    if (a.L <= kWave) thickness_kernel<1><<<grid, col_block(g), 0, s>>>(a);
    else thickness_kernel<2><<<grid, col_block(g), 0, s>>>(a);
}
void launch_thickness_batch(const BatchLaunch<THArgs> &b, int nk, const Geom &g, hipStream_t s) {
    if (nk == 1) thickness_batch<1><<<xcd_grid(b.blocks), col_block(g), 0, s>>>(b);
    else thickness_batch<2><<<xcd_grid(b.blocks), col_block(g), 0, s>>>(b);
}
template <typename R>
void launch_thickness_iso(const THIsoArgs<R> &a, const Geom &g, hipStream_t s) {
    const dim3 grid = xcd_grid(col_blocks(a.m.C, g));
    if (a.L <= kWave) thickness_iso_kernel<1, R><<<grid, col_block(g), 0, s>>>(a);
    else thickness_iso_kernel<2, R><<<grid, col_block(g), 0, s>>>(a);
}
template <typename R>
void launch_thickness_iso_batch(const BatchLaunch<THIsoArgs<R>> &b, int nk, const Geom &g, hipStream_t s) {
    if (nk == 1) thickness_iso_batch<1, R><<<xcd_grid(b.blocks), col_block(g), 0, s>>>(b);
    else thickness_iso_batch<2, R><<<xcd_grid(b.blocks), col_block(g), 0, s>>>(b);
}
template <typename R>
void launch_assemble(const AssembleArgs<R> &a, const Geom &g, hipStream_t s) {
    const dim3 grid = xcd_grid(col_blocks(wave_groups<kAssembleCols>(a.m.E), g));
    if (a.L <= kWave) assemble_kernel<1, R><<<grid, col_block(g), 0, s>>>(a);
    else assemble_kernel<2, R><<<grid, col_block(g), 0, s>>>(a);
}
template <typename R>
void launch_assemble_batch(const BatchLaunch<AssembleArgs<R>> &b, int nk, const Geom &g, hipStream_t s) {
    if (nk == 1) assemble_batch<1, R><<<xcd_grid(b.blocks), col_block(g), 0, s>>>(b);
    else assemble_batch<2, R><<<xcd_grid(b.blocks), col_block(g), 0, s>>>(b);
}
__global__ void __launch_bounds__(256) zero_kernel(unsigned long long *p, size_t n) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = 0ull;
}
hipError_t launch_zero(void *p, size_t bytes, hipStream_t s) {
    size_t n = bytes / 8;
    void *args[] = {&p, &n};
    return hipLaunchKernel(reinterpret_cast<const void *>(zero_kernel), dim3((unsigned)((n + 255) / 256)), dim3(256), args, 0, s);
}
void launch_zeta_from_h(const DevMesh &m, int L, const double *h, double *zeta, hipStream_t s) {
    const dim3 grid = xcd_grid((m.C + 3) / 4);
    if (L <= kWave) zeta_kernel<1><<<grid, 256, 0, s>>>(m, L, h, zeta);
    else zeta_kernel<2><<<grid, 256, 0, s>>>(m, L, h, zeta);
}
template <typename R>
void launch_edge_flux_sum(const DevMesh &m, int L, const double *h, const R *X, const double *uA, double *F,
                          hipStream_t s) {
    const dim3 grid = xcd_grid((m.E + 3) / 4);
    if (L <= kWave) edge_flux_sum_kernel<1, R><<<grid, 256, 0, s>>>(m, L, h, X, uA, F);
    else edge_flux_sum_kernel<2, R><<<grid, 256, 0, s>>>(m, L, h, X, uA, F);
}
__global__ void permute_kernel(const double *__restrict__ src, const int32_t *__restrict__ idx,
                               double *__restrict__ dst, int n, int scatter) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int j = idx[i];
    if (scatter) dst[j] = src[i];
    else dst[i] = src[j];
}
void launch_permute(const double *src, const int32_t *idx, double *dst, int n, bool scatter, const Geom &g,
                    hipStream_t s) {
    if (n > 0) permute_kernel<<<flat_blocks((size_t)n, g), g.block_2d, 0, s>>>(src, idx, dst, n, scatter ? 1 : 0);
}
void launch_recon(const ReconArgs &a, const Geom &g, hipStream_t s) {
    recon_kernel<<<flat_blocks(a.m.E, g), g.block_2d, 0, s>>>(a);
}
void launch_recon_batch(const BatchLaunch<ReconArgs> &b, const Geom &g, hipStream_t s) {
    recon_batch<<<xcd_grid(b.blocks), g.block_2d, 0, s>>>(b);
}
template <typename Tin, typename Tout>
void launch_convert(const ConvArgs<Tin, Tout> &a, const Geom &g, hipStream_t s) {
    if (a.n) convert_kernel<Tin, Tout><<<flat_blocks(a.n, g), g.block_2d, 0, s>>>(a);
}
template <typename Tin, typename Tout>
void launch_convert_batch(const BatchLaunch<ConvArgs<Tin, Tout>> &b, const Geom &g, hipStream_t s) {
    convert_batch<Tin, Tout><<<xcd_grid(b.blocks), g.block_2d, 0, s>>>(b);
}

#define SSE_INSTANTIATE(R)                                                                                   \
    template void launch_fe_cell<R>(const FECellArgs<R> &, const Geom &, hipStream_t);                     \
    template void launch_fe_split<R>(const FESplitArgs<R> &, bool, const Geom &, hipStream_t);             \
    template void launch_fe_split_batch<R>(const BatchLaunch<FESplitArgs<R>> &, int, bool, bool, const Geom &, hipStream_t); \
    template void launch_fe_vertex<R>(const FEVertexArgs<R> &, const Geom &, hipStream_t);                 \
    template void launch_lap<R>(const LapArgs<R> &, const Geom &, hipStream_t);                           \
    template void launch_tracer<R>(const TracerArgs<R> &, const Geom &, hipStream_t);                     \
    template void launch_tracer_batch<R>(const BatchLaunch<TracerArgs<R>> &, int, const Geom &, hipStream_t); \
    template void launch_div<R>(const DivArgs<R> &, const Geom &, hipStream_t);                           \
    template void launch_lap_batch<R>(const BatchLaunch<LapArgs<R>> &, int, const Geom &, hipStream_t);  \
    template void launch_div_batch<R>(const BatchLaunch<DivArgs<R>> &, int, const Geom &, hipStream_t);  \
    template void launch_fe_edge<R>(const FEEdgeArgs<R> &, int, const Geom &, hipStream_t);               \
    template void launch_fe_cell_batch<R>(const BatchLaunch<FECellArgs<R>> &, int, bool, const Geom &,     \
                                          hipStream_t);                                                    \
    template void launch_fe_vertex_batch<R>(const BatchLaunch<FEVertexArgs<R>> &, int, bool, const Geom &, \
                                            hipStream_t);                                                  \
    template void launch_fe_edge_batch<R>(const BatchLaunch<FEEdgeArgs<R>> &, int, bool, int, const Geom &, \
                                          hipStream_t);                                                    \
    template size_t fe_edge_tiled_lds<R>(const DevTiles &, int);                                           \
    template void launch_fe_edge_tiled<R>(const FEEdgeArgs<R> &, const DevTiles &, hipStream_t);           \
    template void launch_edge_gathers<R>(const FEEdgeArgs<R> &, bool, const Geom &, hipStream_t);                \
    template void launch_bt_eval<R>(const BTEvalArgs<R> &, const Geom &, hipStream_t);                     \
    template void launch_bt_substep<R>(const BTTileArgs<R> &, int, hipStream_t);                           \
    template int bt_loop_capacity<R>(const DevBtTiles &, int, int);                                        \
    template hipError_t launch_bt_loop<R>(const BTTileArgs<R> &, const BtLoop<R> &, int, hipStream_t);       \
    template hipError_t launch_bt_resident<R>(const BtResident<R> &, int, int, const BtRound &, hipStream_t); \
    template int bt_resident_batch_capacity<R>(int, int);                                                         \
    template hipError_t launch_bt_resident_batch<R>(const BatchLaunch<BtResident<R>> &, int, int, const BtRound &, hipStream_t); \
    template hipError_t launch_bt_tasks<R>(const BtResident<R> &, int, const BtRound &, hipStream_t);             \
    template hipError_t launch_bt_tasks_batch<R>(const BatchLaunch<BtResident<R>> &, int, int, const BtRound &, hipStream_t); \
    template void launch_bt_substep_batch<R>(const BatchLaunch<BTTileArgs<R>> &, int, int, size_t, hipStream_t); \
    template void launch_bt_eval_batch<R>(const BatchLaunch<BTEvalArgs<R>> &, bool, const Geom &, hipStream_t); \
    template void launch_thickness_iso<R>(const THIsoArgs<R> &, const Geom &, hipStream_t);                \
    template void launch_thickness_iso_batch<R>(const BatchLaunch<THIsoArgs<R>> &, int, const Geom &,      \
                                                hipStream_t);                                              \
    template void launch_assemble<R>(const AssembleArgs<R> &, const Geom &, hipStream_t);                  \
    template void launch_assemble_batch<R>(const BatchLaunch<AssembleArgs<R>> &, int, const Geom &,        \
                                           hipStream_t);                                                   \
    template void launch_edge_flux_sum<R>(const DevMesh &, int, const double *, const R *, const double *, \
                                          double *, hipStream_t);
SSE_INSTANTIATE(double)
SSE_INSTANTIATE(float)
template void launch_convert<double, float>(const ConvArgs<double, float> &, const Geom &, hipStream_t);
template void launch_convert<float, double>(const ConvArgs<float, double> &, const Geom &, hipStream_t);
template void launch_convert_batch<double, float>(const BatchLaunch<ConvArgs<double, float>> &, const Geom &,
                                                  hipStream_t);
template void launch_convert_batch<float, double>(const BatchLaunch<ConvArgs<float, double>> &, const Geom &,
                                                  hipStream_t);

}  // namespace sse

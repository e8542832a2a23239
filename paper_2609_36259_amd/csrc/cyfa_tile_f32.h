// fp32 matrix-core tiles (v_mfma_f32_32x32x2_f32) of the fp32-arithmetic kernels.
//
// Lane layouts (l = lane, l31 = l % 32, h = l / 32):
//   A (32 x 2): lane l holds A[l31][h];  B (2 x 32): lane l holds B[h][l31]
//   D (32 x 32): lane l, register r holds D[8 (r / 4) + 4 h + r % 4][l31]
// Chained products: a D tile's register r is, as it stands, the B operand of a
// product that contracts over D's rows, with the k pair (8 (r/4) + r%4, that + 4).
// A 32-deep contraction step is therefore 16 instructions; "chain" order means that
// register r of either operand holds k = 8 (r/4) + 4 h + r%4, "wide" order
// k = 16 (r/8) + 8 h + r%8 (eight consecutive elements of a token's row per lane).
//
// Arrays in the workspace are kept as 32 x 32 blocks in the order of an operand (or D
// tile): piece q (registers 4 q .. + 3) of lane l at floats 256 q + 4 l of its 4 KiB.
// A block is read or written with four fully coalesced 16-byte accesses per lane.  The
// same operands read from row-major arrays, 16 bytes of 32 rows per instruction, keep
// the address unit busy for the whole step (the backward's readout kernel at B 32, T
// 2048, H 4, d = 256: 1.51 ms with them against 1.18 when blocks took their place; 1.29 in
// its present form).  A block needed with its two indexes swapped passes through a wave's
// own 32 x 36 LDS tile (LdsTile).
#pragma once

#include <utility>

#include "cyfa_internal.h"
#include "cyfa_mfma_common.h"

namespace cyfa {
namespace tile {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

constexpr int kTC = 64;             // tokens per chunk of the fp32 tile kernels (two 32-token tiles)

__device__ __forceinline__ void mma_step(f32x16 &acc, const f32x16 &a, const f32x16 &b) {
#pragma unroll
    for (int r = 0; r < 16; ++r) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[r], b[r], acc, 0, 0, 0);
}

__device__ __forceinline__ f32x16 ld_block(const float *p) {     // p: block + 4 lane
    f32x16 x;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const f32x4 v = *reinterpret_cast<const f32x4 *>(p + 256 * q);
#pragma unroll
        for (int e = 0; e < 4; ++e) x[4 * q + e] = v[e];
    }
    return x;
}
__device__ __forceinline__ void st_block(float *p, const f32x16 &x) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
        *reinterpret_cast<f32x4 *>(p + 256 * q) = f32x4{x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]};
}
// chain order from consecutive floats: p = first + 4 h
__device__ __forceinline__ f32x16 ld_rows(const float *p) {
    f32x16 x;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const f32x4 v = *reinterpret_cast<const f32x4 *>(p + 8 * q);
#pragma unroll
        for (int e = 0; e < 4; ++e) x[4 * q + e] = v[e];
    }
    return x;
}

// Swaps the indexes of a block: in, lane's index x and chain index y; out, lane index y
// and x in chain or wide order.  Only its own wave uses a tile, and a wave's LDS
// accesses are in order, so consecutive blocks need no wait between them.
constexpr int kLdsTile = 32 * 36;   // floats of a wave's tile
struct LdsTile {
    float *w, *rc, *rw;             // this lane's write, chain-read and wide-read places
    __device__ __forceinline__ LdsTile(float *t, int l31, int h)
        : w(t + l31 * 36 + 4 * h), rc(t + 4 * h * 36 + l31), rw(t + 8 * h * 36 + l31) {}
    template <bool WIDE>
    __device__ __forceinline__ f32x16 swap(const f32x16 &x) const {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<f32x4 *>(w + 8 * q) = f32x4{x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]};
        f32x16 y;
#pragma unroll
        for (int r = 0; r < 16; ++r) y[r] = WIDE ? rw[(16 * (r >> 3) + (r & 7)) * 36] : rc[(8 * (r >> 2) + (r & 3)) * 36];
        return y;
    }
};

// N steps: operand n is loaded R + 1 steps ahead and prepared (converted, swapped,
// scaled) one step ahead of its 16 instructions; with one wave per SIMD nothing else
// covers either.  The scheduling barriers keep the order (left to itself the compiler
// collects the loads of many steps and spills); inside a step it may spread them between
// the instructions.
template <int N, int R, typename L, typename P, typename U, int... I>
__device__ __forceinline__ void piped_seq(L &&load, P &&prep, U &&use, std::integer_sequence<int, I...>) {
    f32x16 raw[R + 1], op[2];
#pragma unroll
    for (int n = 0; n <= R; ++n)
        if (n < N) raw[n] = load(n);
    op[0] = prep(0, raw[0]);
    auto step = [&](auto idx) {
        constexpr int n = decltype(idx)::value;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (n + R + 1 < N) raw[n % (R + 1)] = load(n + R + 1);
        if constexpr (n + 1 < N) op[(n + 1) & 1] = prep(n + 1, raw[(n + 1) % (R + 1)]);
        use(n, op[n & 1]);
    };
    (step(std::integral_constant<int, I>{}), ...);
    __builtin_amdgcn_sched_barrier(0);
}
template <int N, int R, typename L, typename P, typename U>
__device__ __forceinline__ void piped(L &&load, P &&prep, U &&use) {
    piped_seq<N, R>(load, prep, use, std::make_integer_sequence<int, N>{});
}
constexpr auto as_is = [](int, const f32x16 &x) { return x; };

// Rows of one head of a [rows, H, D] tensor through a buffer resource that ends
// with the last live row: rows past it read as zero, whatever memory holds there.
template <typename T>
struct TokRows {
    __amdgpu_buffer_rsrc_t rsrc;
    int stride;                     // bytes from one token's row to the next

    __device__ __forceinline__ TokRows(const void *base, size_t row, int h, int H, int D, int live) {
        const char *p = static_cast<const char *>(base) + ((row * H + h) * (size_t)D) * sizeof(T);
        stride = H * D * (int)sizeof(T);
        const int bytes = live > 0 ? (live - 1) * stride + D * (int)sizeof(T) : 0;
        rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(p), (short)0, bytes, 0x00020000);
    }
    // four consecutive elements at byte offset off
    __device__ __forceinline__ f32x4 four(int off) const {
        f32x4 x;
        if constexpr (sizeof(T) == 4) {
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = __uint_as_float(v[e]);
        } else {
            const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rsrc, off, 0, 0);
            x[0] = __uint_as_float(v[0] << 16);
            x[1] = __uint_as_float(v[0] & 0xffff0000u);
            x[2] = __uint_as_float(v[1] << 16);
            x[3] = __uint_as_float(v[1] & 0xffff0000u);
        }
        return x;
    }
    // 16 bytes at byte off of a token's row, and their floats at the same place of an LDS row
    __device__ __forceinline__ u32x4 piece(int row, int off) const {
        return __builtin_amdgcn_raw_buffer_load_b128(rsrc, row * stride + off, 0, 0);
    }
    static __device__ __forceinline__ void spread(float *dst, int q, u32x4 v) {
        f32x4 *d = reinterpret_cast<f32x4 *>(dst);
        if constexpr (sizeof(T) == 4) {
            d[q] = f32x4{__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]), __uint_as_float(v[3])};
        } else {
#pragma unroll
            for (int e = 0; e < 2; ++e)
                d[2 * q + e] = f32x4{__uint_as_float(v[2 * e] << 16), __uint_as_float(v[2 * e] & 0xffff0000u),
                                     __uint_as_float(v[2 * e + 1] << 16), __uint_as_float(v[2 * e + 1] & 0xffff0000u)};
        }
    }
    // elements k0 .. k0 + 31 of token row `row` (this lane's), chain order
    __device__ __forceinline__ f32x16 rows(int row, int h, int k0) const {
        const int off = row * stride + (4 * h + k0) * (int)sizeof(T);
        f32x16 x;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f32x4 v = four(off + 8 * q * (int)sizeof(T));
#pragma unroll
            for (int e = 0; e < 4; ++e) x[4 * q + e] = v[e];
        }
        return x;
    }
    // Raw operands: what the loads return, converted when the operand is prepared (a
    // conversion beside the load would wait for it there).
    // elements k0 .. k0 + 31 of token row `row`, wide order
    __device__ __forceinline__ f32x16 wide_raw(int row, int h, int k0) const {
        const int off = row * stride + (8 * h + k0) * (int)sizeof(T);
        f32x16 x = f32x16{};
#pragma unroll
        for (int q = 0; q < (sizeof(T) == 4 ? 4 : 2); ++q) {
            const int o = sizeof(T) == 4 ? (16 * (q >> 1) + 4 * (q & 1)) * 4 : 32 * q;
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off + o, 0, 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[4 * q + e] = __uint_as_float(v[e]);
        }
        return x;
    }
    static __device__ __forceinline__ f32x16 wide_cvt(const f32x16 &v) {
        if constexpr (sizeof(T) == 4) return v;
        f32x16 x;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const unsigned u = __float_as_uint(v[e]);
            x[2 * e] = __uint_as_float(u << 16);
            x[2 * e + 1] = __uint_as_float(u & 0xffff0000u);
        }
        return x;
    }
    // tokens row0 .. row0 + 31 of column col (this lane's), chain order
    __device__ __forceinline__ f32x16 cols_raw(int row0, int h, int col) const {
        const int off = (row0 + 4 * h) * stride + col * (int)sizeof(T);
        f32x16 x;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int o = off + (8 * (r >> 2) + (r & 3)) * stride;
            if constexpr (sizeof(T) == 4) x[r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, o, 0, 0));
            else x[r] = __uint_as_float((unsigned)__builtin_amdgcn_raw_buffer_load_b16(rsrc, o, 0, 0));
        }
        return x;
    }
    static __device__ __forceinline__ f32x16 cols_cvt(f32x16 x) {
        if constexpr (sizeof(T) != 4)
#pragma unroll
            for (int r = 0; r < 16; ++r) x[r] = __uint_as_float(__float_as_uint(x[r]) << 16);
        return x;
    }
};

// Writes of a temporal-write row a = U(-lambda) b from a phase-table row (cos, sin
// at the pair's two internal columns, 1 at the DC column, 0 at the padding): a is
// the table times (amp, -amp) on the pairs, dc at DC.
struct WriteCoef {
    float amp, dc;
    __device__ __forceinline__ explicit WriteCoef(int m) : amp(sqrtf(2.f / (float)m)), dc(1.f / sqrtf((float)m)) {}
    __device__ __forceinline__ float at(int i) const {      // internal column i
        return i == mfma::kDC ? dc : ((i & 1) ? -amp : amp);
    }
    // chain-order step kb (internal columns 32 kb + chain_k): x times the coefficients
    __device__ __forceinline__ f32x16 apply(f32x16 x, int kb, int h) const {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float c = (r & 1) ? -amp : amp;
            x[r] *= kb == 3 && r == 14 && h == 1 ? dc : c;  // column 126
        }
        return x;
    }
};

// 2^x for a double x: the argument's integer part goes to the exponent, so that the
// rounding of the rest to float (at most 1/2) stays below the result's last place for any x.
__device__ __forceinline__ float exp2_wide(double x) {
    const double n = rint(x);
    return ldexpf(__builtin_amdgcn_exp2f((float)(x - n)), (int)n);
}

// A score tile (rows s, lane t) times Gamma_ts = 2^(G_t - G_s) (G: log2 decay) on and below the causal
// diagonal and 0 above it; times beta_s when bet is given.  off: rows s = 0 .. 31 of the
// tile lie off + s tokens after the chunk's first, t is the lane's token; Gs, bet are at
// the tile's rows + 4 h.
__device__ __forceinline__ f32x16 causal(f32x16 s, double Gt, const double *Gs, const float *bet, int t, int off,
                                         int h) {
    double g[16];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        typedef double f64x2 __attribute__((ext_vector_type(2)));
        const f64x2 a = *reinterpret_cast<const f64x2 *>(Gs + 8 * q), b = *reinterpret_cast<const f64x2 *>(Gs + 8 * q + 2);
        g[4 * q] = a[0];
        g[4 * q + 1] = a[1];
        g[4 * q + 2] = b[0];
        g[4 * q + 3] = b[1];
    }
    f32x16 f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        f[r] = exp2_wide(Gt - g[r]);
    }
    if (bet) f *= ld_rows(bet);
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = off + 8 * (r >> 2) + 4 * h + (r & 3) <= t ? s[r] * f[r] : 0.f;
    return s;
}

// U(sign lambda) of a chain of four tiles (rows = internal basis order, lane = token),
// in place, times mul; cs = the tokens' phase-table blocks + 4 lane.
__device__ __forceinline__ void rotate(f32x16 (&x)[4], const float *cs, float sign, float mul) {
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const f32x16 t = ld_block(cs + 1024 * b);
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
            const float c = t[r], s = sign * t[r + 1], a0 = x[b][r], a1 = x[b][r + 1];
            x[b][r] = mul * (c * a0 - s * a1);
            x[b][r + 1] = mul * (s * a0 + c * a1);
        }
    }
}
// Sums over registers go through sixteen partial sums and a tree: one running sum of the
// 64 or 128 terms costs the gradients of log alpha and delta, cumulative sums of such
// terms' differences, a third of their accuracy.
__device__ __forceinline__ float tree(f32x16 v) {
#pragma unroll
    for (int n = 8; n > 0; n >>= 1)
#pragma unroll
        for (int r = 0; r < n; ++r) v[r] += v[r + n];
    return v[0] + __shfl_xor(v[0], 32);
}
__device__ __forceinline__ void add_products(f32x16 &s, const f32x16 &a, const f32x16 &b) {
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = fmaf(a[r], b[r], s[r]);
}
__device__ __forceinline__ float dot4(const f32x16 (&a)[4], const f32x16 (&b)[4]) {
    f32x16 s = a[0] * b[0];
#pragma unroll
    for (int i = 1; i < 4; ++i) add_products(s, a[i], b[i]);
    return tree(s);
}
// sum over the pairs j of j (dZ_{sin} Z_{cos} - dZ_{cos} Z_{sin}), over both lane halves
__device__ __forceinline__ float pair_moment(const f32x16 (&dz)[4], const f32x16 (&z)[4], int h) {
    f32x16 s;
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
            const float j = (float)((32 * b + 8 * (r >> 2) + (r & 3)) / 2 + 1) + 2.f * (float)h;
            const float x = dz[b][r + 1] * z[b][r] - dz[b][r] * z[b][r + 1];
            const int at = r / 2 + 8 * (b & 1);
            s[at] = b < 2 ? j * x : fmaf(j, x, s[at]);
        }
    return tree(s);
}

}  // namespace tile
}  // namespace cyfa

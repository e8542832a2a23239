// Readout and gradient kernels of the fp32 backward for short calls (d_k, d_v <= 128).
//
// The kernels of cyfa_bwd_f32.hip give one wave 32 tokens and the whole chain, about 136
// (readout, d = 64) and 92 (gradients) dependent steps of 16 instructions, 1024 cycles each,
// however few tokens there are.  Here the chain is split as in the fp32 forward: a
// workgroup of four waves takes 32 tokens' readout, each wave 32 of the 128 basis rows
// (slots), and eight waves a 64-token chunk's gradients, each a share of its tiles; operands
// pass through LDS.  Readout and gradients, before and now: B 1, T 40, H 2, d 64 93 -> 33 and
// 68 -> 32 us, B 1, T 64, H 8, d 128 105 -> 37 and 95 -> 51 us; bound by each tile's chain of
// products and barriers, and beyond one tile per compute unit (its LDS leaves room for
// one workgroup) by the rounds of workgroups.
#pragma once

#include "cyfa_f32_common.h"

namespace cyfa {

namespace {

// pair_moment of block b of the basis rows
__device__ __forceinline__ float pair_moment_block(const f32x16 &dz, const f32x16 &z, int b, int h) {
    f32x16 s = f32x16{};
    const float j0 = (float)(16 * b + 2 * h + 1);
#pragma unroll
    for (int r = 0; r < 16; r += 2)
        s[r / 2] = (j0 + (float)((8 * (r >> 2) + (r & 3)) / 2)) * (dz[r + 1] * z[r] - dz[r] * z[r + 1]);
    return tree(s);
}

// (2) readout recomputation and its adjoint, one 32-token tile at a time, wave w the basis
// rows (slots) 32 w .. + 31.  Workgroup (head, y) takes every gridDim.y-th tile of its head
// and keeps their dM in registers.
template <int DK, int DV, typename Tin>
__global__ __launch_bounds__(256) void f32_readout_short_kernel(BwdParams p, F32Ws w) {
    __shared__ __attribute__((aligned(16))) float xs[4096], ys[4096], b1[4096], b2[4096], tiles[4 * kLdsTile];
    __shared__ float red[3][4][32];
    const int per_seq = (p.T + 31) / 32, hd = blockIdx.x;
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int l31 = lane & 31, h = lane >> 5, lane4 = 4 * lane, m = p.m;
    const WriteCoef wc(m);
    const LdsTile swp(tiles + wv * kLdsTile, l31, h);
    const float *M = w.Mi + (size_t)hd * kR * kR, *MT = w.MiT + (size_t)hd * kR * kR;
    f32x16 dM[4] = {};
    for (int it = blockIdx.y; it < p.B * per_seq; it += gridDim.y) {
        const int b = it / per_seq, tt = it % per_seq, c = tt >> 1, tb = tt & 1, bh = b * p.H + hd;
        const int left = min(bwd_tokens(p, b) - c * kTC, kTC);
        const size_t grow = first_row(p, b) + c * kTC, row0 = (size_t)bh * p.Tpad + c * kTC;
        float *Ur = p.U + (row0 + 32 * tb) * kR + wv * 1024 + lane4, *dPr = p.dP + (row0 + 32 * tb) * kR + wv * 1024 + lane4;
        if (tb == 0 && tt + 1 == per_seq) {         // the chunk's second tile lies past T
            st_block(Ur + 4096, f32x16{});
            st_block(dPr + 4096, f32x16{});
        }
        if (left <= 32 * tb) {                      // none of these tokens exists
            st_block(Ur, f32x16{});
            st_block(dPr, f32x16{});
            continue;
        }
        const int tl = 32 * tb + l31;
        const bool live = tl < left;
        const TokRows<Tin> q(p.q, grow, hd, p.H, DK, left), k(p.k, grow, hd, p.H, DK, left);
        const TokRows<Tin> v(p.v, grow, hd, p.H, DV, left), o(p.dout, grow, hd, p.H, DV, left);
        const float *cs = w.cs + row0 * kR + lane4;
        const double Gt = w.G[row0 + tl];
        const float g = w.gam[row0 + tl];
        // (q, k) and (do, v) score tiles: wave w the tile w % 2, every second 32 channels (the
        // gradient kernel's order: see there)
        auto score = [&](float *part, const TokRows<Tin> &x, const TokRows<Tin> &y, int D) {
            f32x16 s = {};
            if ((wv & 1) <= tb)
                for (int kb = wv >> 1; kb < D / 32; kb += 2)
                    mma_step(s, y.wide_cvt(y.wide_raw(32 * (wv & 1) + l31, h, 32 * kb)), x.wide_cvt(x.wide_raw(tl, h, 32 * kb)));
            st_block(part + wv * 1024 + lane4, s);
        };
        score(b1, q, k, DK);
        score(b2, o, v, DV);
        // this wave's rows of the entering states times the tokens, in two sums
        auto state = [&](const float *St, auto dim, const TokRows<Tin> &x) {
            constexpr int D = decltype(dim)::value;
            const float *sp = St + ((((size_t)bh * p.nc + c) * 4 + wv) * (D / 32)) * 1024 + lane4;
            f32x16 s[2] = {};
#pragma unroll
            for (int kb = 0; kb < D / 32; ++kb)
                mma_step(s[kb / (D / 64)], swp.template swap<true>(ld_block(sp + kb * 1024)), x.wide_cvt(x.wide_raw(tl, h, 32 * kb)));
            return s[0] + s[1];
        };
        const f32x16 pk = state(w.Kst, std::integral_constant<int, DK>{}, q);
        const f32x16 pv = state(w.Vst, std::integral_constant<int, DV>{}, o);
        __syncthreads();
        f32x16 ok = {}, ov = {};
        for (int sb = 0; sb <= tb; ++sb) {
            // (beta on the masked scores, NaN phases as -1: see the forward)
            f32x16 a = swp.template swap<false>(ld_block(cs + (4 * sb + wv) * 1024));
#pragma unroll
            for (int r = 0; r < 16; ++r) a[r] = fmaxf(a[r], -1.f) * wc.at(32 * wv + l31);
            auto masked = [&](const float *part) {
                const f32x16 s = ld_block(part + sb * 1024 + lane4) + ld_block(part + (sb + 2) * 1024 + lane4);
                return causal(s, Gt, w.G + row0 + 32 * sb + 4 * h, w.bet + row0 + 32 * sb + 4 * h, tl, 32 * sb, h);
            };
            mma_step(ok, a, masked(b1));
            mma_step(ov, a, masked(b2));
        }
        const f32x16 ph = ld_block(cs + (4 * tb + wv) * 1024), zero = f32x16{};
        const f32x16 du = pv * g + ov;
        const f32x16 X = live ? rotate_block(pk * g + ok, ph, 1.f, p.scale) : zero;
        const f32x16 dY = live ? rotate_block(du, ph, 1.f, 1.f) : zero;
        st_block(xs + wv * 1024 + lane4, X);
        st_block(ys + wv * 1024 + lane4, dY);
        __syncthreads();
        f32x16 z = row_product(M, wv, xs, lane4);
        const f32x16 dW = row_product(M, wv, ys, lane4);
        // softmax over the m active slots; M^T takes the weights before their normalisation
        {
            float mx = -INFINITY;
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (32 * wv + 8 * (r >> 2) + 4 * h + (r & 3) < m) mx = fmaxf(mx, z[r]);
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            if (h == 0) red[0][wv][l31] = mx;
        }
        __syncthreads();
        auto total = [&](int i) { return (red[i][0][l31] + red[i][1][l31]) + (red[i][2][l31] + red[i][3][l31]); };
        {
            const float mx = fmaxf(fmaxf(red[0][0][l31], red[0][1][l31]), fmaxf(red[0][2][l31], red[0][3][l31]));
#pragma unroll
            for (int r = 0; r < 16; ++r)
                z[r] = 32 * wv + 8 * (r >> 2) + 4 * h + (r & 3) < m ? __expf(z[r] - mx) : 0.f;
            const float sum = tree(z);
            if (h == 0) red[1][wv][l31] = sum;
            st_block(b1 + wv * 1024 + lane4, z);
        }
        __syncthreads();
        const float inv = 1.f / total(1);
        const f32x16 W = live ? z * inv : zero;
        const f32x16 u = rotate_block(row_product(MT, wv, b1, lane4) * inv, ph, -1.f, 1.f);
        st_block(Ur, live ? u : zero);
        {
            const float ud = tree(u * du), wd = tree(W * dW);
            if (h == 0) {
                red[0][wv][l31] = ud;
                red[2][wv][l31] = wd;
            }
        }
        const float c2 = 6.283185307179586f / (float)m;
        float gl = -c2 * pair_moment_block(du, u, wv, h);
        __syncthreads();
        const f32x16 dZ = W * (dW - total(2));
        if (wv == 0 && h == 0) p.udu[row0 + tl] = total(0);
        st_block(b2 + wv * 1024 + lane4, dZ);
        __syncthreads();
        const f32x16 dX = row_product(MT, wv, b2, lane4);
        gl += c2 * pair_moment_block(dX, X, wv, h);
        if (h == 0) red[1][wv][l31] = gl;
        st_block(dPr, live ? rotate_block(dX, ph, -1.f, p.scale) : zero);
        // dM = W dY^T + dZ X^T over the tile's tokens
        st_block(ys + wv * 1024 + lane4, swp.template swap<false>(dY));
        st_block(xs + wv * 1024 + lane4, swp.template swap<false>(X));
        const f32x16 aW = swp.template swap<false>(W), aZ = swp.template swap<false>(dZ);
        __syncthreads();
        if (wv == 0 && h == 0) p.dlam[row0 + tl] = total(1);
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            f32x16 s1 = f32x16{}, s2 = f32x16{};
            mma_step(s1, aW, ld_block(ys + x * 1024 + lane4));
            mma_step(s2, aZ, ld_block(xs + x * 1024 + lane4));
            dM[x] += s1 + s2;
        }
    }
    // partial dM, in the basis order of App. A.1
    float *out = p.dMp + ((size_t)blockIdx.y * p.H + hd) * kR * kR;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        const int jp = internal_to_paper(32 * x + l31, m);
        if (jp >= 0)
#pragma unroll
            for (int r = 0; r < 16; ++r) out[(32 * wv + 8 * (r >> 2) + 4 * h + (r & 3)) * kR + jp] = dM[x][r];
    }
}

// (4) token gradients, one chunk per workgroup of eight waves.
template <int DK, int DV, typename Tin>
__global__ __launch_bounds__(512) void f32_grad_short_kernel(BwdParams p, F32Ws w) {
    constexpr int QK = 0, OV = 1, PA = 2, UA = 3;       // (q, k), (do, v), (dp, a), (u, a)
    constexpr int NK = DK / 32, NV = DV / 32;
    __shared__ __attribute__((aligned(16))) float S[4][kTC][kLS], tiles[8 * kLdsTile];
    __shared__ float dots[2][NK][kTC], red[3][4][kTC];
    const int c = blockIdx.x % p.nc, bh = blockIdx.x / p.nc, b = bh / p.H, hd = bh % p.H, tid = threadIdx.x, m = p.m;
    const int lane = tid & 63, l31 = lane & 31, h = lane >> 5, lane4 = 4 * lane;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int Tb = bwd_tokens(p, b), left = min(Tb - c * kTC, kTC);
    const bool two = left > 32;                 // the second tile has tokens
    const size_t grow = first_row(p, b) + c * kTC, row0 = (size_t)bh * p.Tpad + c * kTC;
    const size_t st = ((size_t)bh * p.nc + c) * kR;
    const WriteCoef wc(m);
    const LdsTile swp(tiles + wv * kLdsTile, l31, h);
    const float *cs = w.cs + row0 * kR + lane4;
    // The masked score tiles: the four-step kinds first, so that no wave has two of them.
    // The (do, v) tile is formed as in the readout kernel, with the same operations in the same
    // order: its rounding errors then cancel between <u, du> and <a, DV v>.
    for (int j = wv; j < 12; j += 8) {
        const int pair = j % 3, tr = pair > 0, ts = pair == 2, tl = 32 * tr + l31;
        const int kind = j < 3 ? UA : (j < 6 ? PA : (j < 9 ? QK : OV));
        if (tr && !two) continue;
        f32x16 s[2] = {};
        if (kind >= PA) {
            const float *xp = (kind == UA ? p.U : p.dP) + (row0 + 32 * tr) * kR + lane4;
            f32x16 a[4], x[4];
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) {
                a[kb] = ld_block(cs + (4 * ts + kb) * 1024);
                x[kb] = ld_block(xp + kb * 1024);
            }
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) mma_step(s[kb >> 1], wc.apply(a[kb], kb, h), x[kb]);
        } else {
            const int D = kind == QK ? DK : DV;
            const TokRows<Tin> x(kind == QK ? p.q : p.dout, grow, hd, p.H, D, left);
            const TokRows<Tin> y(kind == QK ? p.k : p.v, grow, hd, p.H, D, left);
            for (int kb = 0; kb < D / 32; kb += 2) {
                const f32x16 y0 = y.wide_raw(32 * ts + l31, h, 32 * kb), x0 = x.wide_raw(tl, h, 32 * kb);
                const f32x16 y1 = y.wide_raw(32 * ts + l31, h, 32 * kb + 32), x1 = x.wide_raw(tl, h, 32 * kb + 32);
                mma_step(s[0], y.wide_cvt(y0), x.wide_cvt(x0));
                mma_step(s[1], y.wide_cvt(y1), x.wide_cvt(x1));
            }
        }
        const size_t s0 = row0 + 32 * ts + 4 * h;
        const f32x16 y = causal(s[0] + s[1], w.G[row0 + tl], w.G + s0, kind >= PA ? w.bet + s0 : nullptr, tl, 32 * ts, h);
#pragma unroll
        for (int qq = 0; qq < 4; ++qq)
            *reinterpret_cast<f32x4 *>(&S[kind][tl][32 * ts + 8 * qq + 4 * h]) =
                f32x4{y[4 * qq], y[4 * qq + 1], y[4 * qq + 2], y[4 * qq + 3]};
    }
    __syncthreads();
    // rows of tile tt, column tl of a score tile
    auto ld_S = [&](int kind, int tt, int tl) {
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = S[kind][32 * tt + 8 * (r >> 2) + 4 * h + (r & 3)][tl];
        return s;
    };
    // dq = gamma (dP Kbar_c) + Spa K, dk = rho (A DK') + Spa^T Q, dv = rho (A DV') + Sua^T dO:
    // 32 channels of 32 tokens at a time, every 32 terms in a sum of their own
    for (int j = wv; j < 2 * (2 * NK + NV); j += 8) {
        const int tb = j & 1, y = j >> 1, kind = y < NK ? 0 : (y < 2 * NK ? 1 : 2);
        const int cb = y - kind * NK, D = kind == 2 ? DV : DK, tl = 32 * tb + l31, t = c * kTC + tl;
        const bool live = tl < left;
        f32x16 r = f32x16{};
        if (tb == 0 || two) {
            const float *sp = (kind == 0 ? w.Kst : (kind == 1 ? w.DKe : w.DVe)) + st * D + cb * 1024 + lane4;
            const float *xp = (kind == 0 ? p.dP : w.cs) + (row0 + 32 * tb) * kR + lane4;
            const TokRows<Tin> xr(kind == 0 ? p.k : (kind == 1 ? p.q : p.dout), grow, hd, p.H, D, left);
            const int t0 = kind == 0 ? 0 : tb, t1 = kind == 0 ? tb : (int)two;      // tiles of the other tokens
            f32x16 a[4], x[4];
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) {
                a[kb] = ld_block(sp + kb * (D / 32) * 1024);
                x[kb] = ld_block(xp + kb * 1024);
            }
            const f32x16 c0 = xr.cols_raw(32 * t0, h, 32 * cb + l31);
            const f32x16 c1 = t1 > t0 ? xr.cols_raw(32 * t1, h, 32 * cb + l31) : f32x16{};
            auto score = [&](int tt) {
                return kind == 0 ? ld_rows(&S[PA][tl][32 * tt + 4 * h]) : ld_S(kind == 1 ? PA : UA, tt, tl);
            };
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) {
                f32x16 n = f32x16{};
                mma_step(n, a[kb], kind == 0 ? x[kb] : wc.apply(x[kb], kb, h));
                a[kb] = n;
            }
            f32x16 e0 = f32x16{}, e1 = f32x16{};
            mma_step(e0, xr.cols_cvt(c0), score(t0));
            if (t1 > t0) mma_step(e1, xr.cols_cvt(c1), score(t1));
            r = ((a[0] + a[1]) + (a[2] + a[3])) * (kind == 0 ? w.gam : w.wr)[row0 + tl] + (e0 + e1);
            if (kind < 2) {
                const TokRows<Tin> own(kind == 0 ? p.q : p.k, grow, hd, p.H, DK, left);
                const float dot = tree(own.rows(tl, h, 32 * cb) * r);
                if (h == 0) dots[kind][cb][tl] = dot;
            }
        }
        if (t < p.T) {
            Tin *row = static_cast<Tin *>(kind == 0 ? p.gq : (kind == 1 ? p.gk : p.gv)) + ((grow + tl) * p.H + hd) * D +
                       32 * cb + 4 * h;
#pragma unroll
            for (int qq = 0; qq < 4; ++qq) {
                f32x4 n;
#pragma unroll
                for (int e = 0; e < 4; ++e) n[e] = live ? r[4 * qq + e] : 0.f;
                if constexpr (sizeof(Tin) == 4) {
                    *reinterpret_cast<f32x4 *>(row + 8 * qq) = n;
                } else {
                    mfma::bf16x4 s;
#pragma unroll
                    for (int e = 0; e < 4; ++e) s[e] = (__bf16)n[e];
                    *reinterpret_cast<mfma::bf16x4 *>(row + 8 * qq) = s;
                }
            }
        }
    }
    // da's two parts, rho DK' k + Sqk^T dp and rho DV' v + Sov^T u: wave w the basis rows
    // 32 (w % 4) .. + 31 of the tokens 32 (w / 4) .. + 31
    {
        const int tb = wv >> 2, y = wv & 3, tl = 32 * tb + l31;
        if (tb == 0 || two) {
            const float rho = exp2_wide(w.G[row0 + kTC - 1] - w.G[row0 + tl]), be = w.bet[row0 + tl];
            auto part = [&](const float *De, auto dim, const void *tok, int kind, const float *rows) {
                constexpr int D = decltype(dim)::value;
                const TokRows<Tin> xr(tok, grow, hd, p.H, D, left);
                const float *dp = De + st * D + y * (D / 32) * 1024 + lane4, *rp = rows + row0 * kR + y * 1024 + lane4;
                f32x16 a[2] = {}, own = f32x16{};
#pragma unroll
                for (int kb = 0; kb < D / 32; ++kb)
                    mma_step(a[kb / (D / 64)], swp.template swap<true>(ld_block(dp + kb * 1024)),
                             xr.wide_cvt(xr.wide_raw(tl, h, 32 * kb)));
                for (int tt = tb; tt <= (int)two; ++tt)
                    mma_step(own, swp.template swap<false>(ld_block(rp + tt * 4096)), ld_S(kind, tt, tl));
                return (a[0] + a[1]) * rho + own;
            };
            const f32x16 dv = part(w.DVe, std::integral_constant<int, DV>{}, p.v, OV, p.U);
            const f32x16 da = part(w.DKe, std::integral_constant<int, DK>{}, p.k, QK, p.dP) + dv;
            const f32x16 x = wc.apply(ld_block(cs + (4 * tb + y) * 1024), y, h);      // U(-lambda) b
            const float adav = be * tree(x * dv), db = tree(x * da);
            const float gl = -(6.283185307179586f / (float)m) * be * pair_moment_block(da, x, y, h);
            if (h == 0) {
                red[0][y][tl] = adav;
                red[1][y][tl] = db;
                red[2][y][tl] = gl;
            }
        }
    }
    __syncthreads();
    const int t = c * kTC + tid;
    if (tid < kTC && t < p.T) {
        const size_t ti = row0 + tid;
        const bool live = tid < left;
        auto total = [&](int i) { return (red[i][0][tid] + red[i][1][tid]) + (red[i][2][tid] + red[i][3][tid]); };
        float qk = 0.f, kk = 0.f;
#pragma unroll
        for (int i = 0; i < NK; ++i) {
            qk += dots[0][i][tid];
            kk += dots[1][i][tid];
        }
        p.dG[ti] = live ? (qk - kk) - total(0) + p.udu[ti] : 0.f;
        p.dlam[ti] = live ? p.dlam[ti] + total(2) : 0.f;
        if (p.gbeta) p.gbeta[(grow + tid) * p.H + hd] = live ? total(1) : 0.f;
    }
}

}  // namespace
}  // namespace cyfa

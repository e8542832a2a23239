// fp32 backward of the chunk-wise CyFA forward on the fp32 matrix instructions.
//
// Gradients of L = sum_t <do_t, o_t> + <dK_T, Kbar_T> + <dV_T, Vbar_T> in the
// absolute-clock form (Sec. 3.2, Eqs. cyfa-absolute-recurrence and
// cyfa-absolute-readout), evaluated chunk by chunk as the forward is (App. B).
// Forward per token: a_t = beta_t U(-lambda_t) b (Eq. app-temporal-writes),
// Kbar_t = alpha_t Kbar_{t-1} + a_t k_t^T (Vbar likewise), p_t = Kbar_t q_t,
// X_t = scale U(lambda_t) p_t, Z_t = M X_t, W_t = softmax over the m active
// slots, u_t = U(-lambda_t) M^T W_t, o_t = Vbar_t^T u_t, with M = R Phi.
// Reverse mode:
//   du_t = Vbar_t do_t,  dY_t = U(lambda_t) du_t,  dW_t = M dY_t,
//   dZ_t = W_t (.) (dW_t - <W_t, dW_t>),  dX_t = M^T dZ_t,  dp_t = scale U(-lambda_t) dX_t,
//   dM = sum_t W_t dY_t^T + dZ_t X_t^T  and  dR = dM Phi^T,
//   adjoint states DK_t = dp_t q_t^T + alpha_{t+1} DK_{t+1},  DV_t = u_t do_t^T + alpha_{t+1} DV_{t+1}
//   (starting from dK_T, dV_T), dq_t = Kbar_t^T dp_t, dk_t = DK_t^T a_t, dv_t = DV_t^T a_t,
//   da_t = DK_t k_t + DV_t v_t,  dbeta_t = <da_t, U(-lambda_t) b>.
// Decay: with G_t = sum_{j<=t} log alpha_j every pair (t, s) of a pass carries
// exp(G_t - G_s), so dL/dG_t = <q_t, dq_t> - <k_t, dk_t> + <u_t, du_t> - <a_t, DV_t v_t>
// (plus <dK_T, Kbar_T> + <dV_T, Vbar_T> at the last token) and dlog_alpha_t is the
// reverse cumulative sum of dL/dG.  Clock: U(+-lambda_t) acts on the (cos, sin)
// pair j as a rotation by +-2 pi j lambda_t / m, whose derivative is the
// rotation generator; dL/dlambda_t collects the three rotations of token t (a_t,
// X_t, u_t) and ddelta_t = sum_{tau >= t} dL/dlambda_tau
// (Eq. app-clock-gradient-accumulation); dclock0 is the full sum.
//
// Within a chunk of 64 tokens (rows r, s; gamma_r = exp(G_r), Gamma_rs = exp(G_r - G_s)
// for r >= s, rho_s = exp(G_C - G_s), entering states Kbar_c, Vbar_c, adjoints DK', DV'
// at the chunk's end):
//   p  = gamma (.) Q Kbar_c^T + (Q K^T (.) Gamma) A
//   du = gamma (.) dO Vbar_c  + (dO V^T (.) Gamma) A
//   dq = gamma (.) dP Kbar_c  + (dP A^T (.) Gamma) K
//   dk = (dP A^T (.) Gamma)^T Q + (rho (.) A) DK'
//   dv = (U A^T (.) Gamma)^T dO + (rho (.) A) DV'
//   da = (Q K^T (.) Gamma)^T dP + rho (.) K DK'^T + (dO V^T (.) Gamma)^T U + rho (.) V DV'^T
// Every product is a chain of 32 x 32 x 2 fp32 tiles with the tokens on the lanes
// (cyfa_tile_f32.h): one wave takes 32 tokens from their score tile to u and dp
// with every intermediate in registers.  fp32 throughout: 27.3 -> 3.6 ms at B 32, T 2048,
// H 4, d_k = d_v = 256 (bf16 inputs; 330 GFLOP in tiles, 91 TFLOP/s of the 157 the fp32
// matrix instructions have) against vector-ALU kernels on 16-token chunks.  The readout and
// gradient kernels run one wave per SIMD (a wave's tokens need 4 .. 5 tiles of 64
// registers) and are bound by their matrix instructions, the vector work between them and
// the loads' latency at each product's start.  Short calls, where that chain of one wave is
// all the time, have kernels of their own for (2) and (4) (cyfa_bwd_f32_short.h).  Kernels:
// (0) clocks and phase tables; (1)
// states entering every chunk; (2) readout recomputation and its adjoint; (3)
// adjoint states at every chunk's end; (4) token gradients; (5) reverse cumulative
// sums, per sequence; (6) dR, per head.
#include "cyfa_bwd_f32_short.h"

namespace cyfa {

namespace {

constexpr float kTwoPi = 6.283185307179586f;
constexpr int kAhead = 2;           // operands in flight beyond the one being prepared (one: 6 % slower)

// acc[0..3] (state rows on D's rows) = gamma (St X^T) + A^T (X Y^T (.) Gamma)^T for the
// 32 tokens of one wave: X their rows (q or do), Y the keys of the contraction's
// score (k or v), St the entering state [128][D].
template <int D, typename Tin>
__device__ __forceinline__ void state_read(f32x16 (&acc)[4], const float *St, const TokRows<Tin> &x,
                                           const TokRows<Tin> &y, const F32Ws &w, size_t row0, int tb, int l31, int h,
                                           const WriteCoef &wc, const LdsTile &tile) {
    const int tl = 32 * tb + l31, lane4 = 4 * (32 * h + l31);
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[b] = f32x16{};
    f32x16 sc[2] = {f32x16{}, f32x16{}}, half[4];
    // (The gradient kernel forms the (do, v) tile again, with the same operations in the same
    // order: its rounding errors then cancel between <u, du> and <a, DV v>, whose
    // differences accumulate in dlog_alpha.)  Both score tiles in either wave: the second is 0 in wave 0, which would otherwise
    // wait for wave 1 at the next barrier.
    f32x16 xr = x.wide_raw(tl, h, 0), xv;
    piped<D / 32 * 6, kAhead>(
        [&](int n) {
            const int kb = n / 6, z = n % 6;
            return z < 4 ? ld_block(St + (z * (D / 32) + kb) * 1024 + lane4) : y.wide_raw(32 * (z - 4) + l31, h, 32 * kb);
        },
        [&](int n, const f32x16 &a) { return n % 6 < 4 ? tile.template swap<true>(a) : y.wide_cvt(a); },
        [&](int n, const f32x16 &a) {
            if (n % 6 == 0) {
                xv = x.wide_cvt(xr);
                if (n + 6 < D / 32 * 6) xr = x.wide_raw(tl, h, 32 * (n / 6 + 1));
            }
            mma_step(n % 6 < 4 ? acc[n % 6] : sc[n % 6 - 4], a, xv);
            // two sums of half the contraction each
            if (n < D / 32 * 3 && n >= D / 32 * 3 - 6 && n % 6 < 4) {
                half[n % 6] = acc[n % 6];
                acc[n % 6] = f32x16{};
            }
        });
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[b] += half[b];
    const float g = w.gam[row0 + tl];
    const double Gt = w.G[row0 + tl];
#pragma unroll
    for (int sb = 0; sb < 2; ++sb)
        sc[sb] = causal(sc[sb], Gt, w.G + row0 + 32 * sb + 4 * h, nullptr, tl, 32 * sb, h);
    const float *cp = w.cs + row0 * kR + lane4;
    f32x16 own[2];
    piped<8, kAhead>(
        [&](int n) { return ld_block(cp + (((n >> 1) & 1) * 4 + (n >> 2) * 2 + (n & 1)) * 1024); },
        [&](int n, const f32x16 &c) {
            return tile.template swap<false>(c) * (ld_rows(w.bet + row0 + 32 * ((n >> 1) & 1) + 4 * h) *
                                                   wc.at(32 * ((n >> 2) * 2 + (n & 1)) + l31));
        },
        [&](int n, const f32x16 &a) {
            if ((n & 3) < 2) own[n & 1] = f32x16{};
            mma_step(own[n & 1], a, sc[(n >> 1) & 1]);
            const int b = (n >> 2) * 2 + (n & 1);
            if ((n & 3) >= 2) acc[b] = acc[b] * g + own[n & 1];
        });
}

// acc[0..3] = Mat x for a matrix of 4 x 4 blocks and a chain of four tiles
__device__ __forceinline__ void mat_product(f32x16 (&acc)[4], const float *Mat, const f32x16 (&x)[4], int l31, int h) {
    int z = 0;                      // opaque: the operands are the same every chunk, and
    asm volatile("" : "+s"(z));     // the compiler would hold them across the chunk loop
    const float *mp = Mat + z + 4 * (32 * h + l31);
    // two rows of blocks at a time, each in two sums of half the contraction
    f32x16 s[4];
    piped<16, kAhead>(
        [&](int n) { return ld_block(mp + (((n >> 3) * 2 + (n & 1)) * 4 + ((n >> 1) & 3)) * 1024); }, as_is,
        [&](int n, const f32x16 &a) {
            const int at = (n & 1) + 2 * ((n >> 2) & 1);
            if ((n & 3) < 2) s[at] = f32x16{};
            mma_step(s[at], a, x[(n >> 1) & 3]);
            if ((n & 7) >= 6) acc[(n >> 3) * 2 + (n & 1)] = s[n & 1] + s[2 + (n & 1)];
        });
}

// ---------------------------------------------------------------------------
// (2) readout recomputation and its adjoint.  A workgroup takes two chunks at a time,
// wave w the tokens 32 (w % 2) .. + 31 of chunk w / 2, and carries each wave's tokens
// through the whole chain in registers; only dM, which contracts over the tokens, goes
// through LDS (two [128][128 tokens] tiles).  The workgroups of a head share its chunk
// pairs evenly and keep their part of dM in registers.
constexpr int kLT = 132;            // row stride of the dM tiles
template <int DK, int DV, typename Tin>
__global__ __launch_bounds__(256, 1) void f32_readout_kernel(BwdParams p, F32Ws w, int per) {
    __shared__ __attribute__((aligned(16))) float T1[kR * kLT], T2[kR * kLT], tiles[4 * kLdsTile];
    const int hd = blockIdx.x, tid = threadIdx.x;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), tb = wv & 1, m = p.m;
    int l31 = tid & 31, h = (tid >> 5) & 1;
    const int npc = (p.nc + 1) / 2, np = p.B * npc;
    const WriteCoef wc(m);
    const float *M = w.Mi + (size_t)hd * kR * kR, *MT = w.MiT + (size_t)hd * kR * kR;
    f32x16 dM[4] = {};
    // dM += L^T R over the workgroup's 128 tokens (L, R: slot or basis rows x token)
    auto to_lds = [&](float *T, const f32x16 (&x)[4]) {
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                T[(32 * b + 8 * (r >> 2) + 4 * h + (r & 3)) * kLT + 32 * wv + l31] = x[b][r];
    };
    auto add_dM = [&](const f32x16 (&l)[4], const f32x16 (&r)[4]) {
        mfma::lds_barrier();                    // the previous products have read the tiles
        to_lds(T1, l);
        to_lds(T2, r);
        mfma::lds_barrier();
        // each call in sums of its own (the products of all of a workgroup's tokens in one
        // running sum cost dR a quarter of its accuracy)
        f32x16 s[4] = {};
#pragma unroll 1
        for (int kb = 0; kb < 4; ++kb) {
            const f32x16 a = ld_rows(T1 + (32 * wv + l31) * kLT + 32 * kb + 4 * h);
#pragma unroll
            for (int b = 0; b < 4; ++b) mma_step(s[b], a, ld_rows(T2 + (32 * b + l31) * kLT + 32 * kb + 4 * h));
        }
#pragma unroll
        for (int b = 0; b < 4; ++b) dM[b] += s[b];
    };
    const int i_hi = min((int)(blockIdx.y + 1) * per, np);
    for (int it = blockIdx.y * per; it < i_hi; ++it) {
        // lane offsets are formed anew for every pair: kept across the loop they spill
        l31 = mfma::opq(l31);
        h = mfma::opq(h);
        const int b = it / npc, c = 2 * (it % npc) + (wv >> 1), bh = b * p.H + hd;
        const bool real = c < p.nc;             // the last pair of an odd count has one chunk
        const int cc = real ? c : p.nc - 1;
        const int Tb = real ? bwd_tokens(p, b) : 0;
        const int left = min(Tb - cc * kTC, kTC);
        const size_t grow = first_row(p, b) + cc * kTC, row0 = (size_t)bh * p.Tpad + cc * kTC;
        const int tl = 32 * tb + l31;
        const bool live = tl < left;
        const LdsTile tile(tiles + wv * kLdsTile, l31, h);
        const size_t tok4 = (row0 + 32 * tb) * kR + 4 * (32 * h + l31);    // the wave's token blocks
        const float *csr = w.cs + tok4;
        f32x16 X[4], W[4], u[4], dY[4];
        {
            const TokRows<Tin> q(p.q, grow, hd, p.H, DK, left), k(p.k, grow, hd, p.H, DK, left);
            state_read<DK, Tin>(X, w.Kst + ((size_t)bh * p.nc + cc) * kR * DK, q, k, w, row0, tb, l31, h, wc,
                                tile);
        }
        rotate(X, csr, 1.f, p.scale);
        float *Ur = p.U + tok4, *dPr = p.dP + tok4;
        auto put = [&](float *blk, const f32x16 (&x)[4]) {
#pragma unroll
            for (int z = 0; z < 4; ++z) st_block(blk + 1024 * z, live ? x[z] : f32x16{});
        };
        auto get = [&](f32x16 (&x)[4], const float *blk) {
#pragma unroll
            for (int z = 0; z < 4; ++z) {
                const f32x16 v = ld_block(blk + 1024 * z);
                x[z] = live ? v : f32x16{};
            }
        };
        // X waits in dp's rows, which are written last, and u in its own: with both in
        // registers beside W, dM and the value pass's operands the kernel spills
        if (real) put(dPr, X);
        mat_product(W, M, X, l31, h);
        {   // softmax over the m active slots
            float mx = -INFINITY;
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int i = 32 * x + 8 * (r >> 2) + (r & 3);
                    if (i + 4 * h >= m) W[x][r] = -INFINITY;
                    mx = fmaxf(mx, W[x][r]);
                }
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            float sum = 0.f;
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int i = 32 * x + 8 * (r >> 2) + (r & 3);
                    W[x][r] = i + 4 * h < m ? __expf(W[x][r] - mx) : 0.f;
                    sum += W[x][r];
                }
            sum += __shfl_xor(sum, 32);
            const float inv = 1.f / sum;
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int r = 0; r < 16; ++r) W[x][r] = live ? W[x][r] * inv : 0.f;
        }
        mat_product(u, MT, W, l31, h);
        rotate(u, csr, -1.f, 1.f);
        if (real) put(Ur, u);
        {
            const TokRows<Tin> o(p.dout, grow, hd, p.H, DV, left), v(p.v, grow, hd, p.H, DV, left);
            state_read<DV, Tin>(dY, w.Vst + ((size_t)bh * p.nc + cc) * kR * DV, o, v, w, row0, tb, l31, h, wc,
                                tile);
        }
        get(u, Ur);
        const float udu = dot4(u, dY);
        float gl = -(kTwoPi / (float)m) * pair_moment(dY, u, h);
        rotate(dY, csr, 1.f, 1.f);
        if (!live) {
#pragma unroll
            for (int x = 0; x < 4; ++x) dY[x] = f32x16{};
        }
        add_dM(W, dY);
        f32x16 dZ[4];
        mat_product(dZ, M, dY, l31, h);
        {
            const float sd = dot4(W, dZ);
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int r = 0; r < 16; ++r) dZ[x][r] = W[x][r] * (dZ[x][r] - sd);
        }
        get(X, dPr);
        add_dM(dZ, X);
        mat_product(u, MT, dZ, l31, h);         // dX
        gl += (kTwoPi / (float)m) * pair_moment(u, X, h);
        rotate(u, csr, -1.f, p.scale);
        if (real) {
            put(dPr, u);
            if (h == 0) {
                p.udu[row0 + tl] = udu;
                p.dlam[row0 + tl] = gl;
            }
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

// ---------------------------------------------------------------------------
// (4) token gradients, one chunk per workgroup, wave w the tokens 32 w .. + 31 both as
// readers t (dq) and as writers s (dk, dv, da).  The four masked score tiles go through
// LDS, where the other wave's writers read them.
template <int DK, int DV, typename Tin>
__global__ __launch_bounds__(128, 1) void f32_grad_kernel(BwdParams p, F32Ws w) {
    __shared__ __attribute__((aligned(16))) float Sqk[kTC][kLS], Sdov[kTC][kLS], Sdpa[kTC][kLS], Sua[kTC][kLS];
    __shared__ __attribute__((aligned(16))) float tiles[2 * kLdsTile];
    const int c = blockIdx.x % p.nc, bh = blockIdx.x / p.nc, b = bh / p.H, hd = bh % p.H, tid = threadIdx.x, m = p.m;
    const int lane = tid & 63, l31 = lane & 31, h = lane >> 5, tb = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int Tb = bwd_tokens(p, b), left = min(Tb - c * kTC, kTC);
    const size_t grow = first_row(p, b) + c * kTC, row0 = (size_t)bh * p.Tpad + c * kTC;
    const int tl = 32 * tb + l31, t = c * kTC + tl;
    const bool live = tl < left, inside = t < p.T;
    const WriteCoef wc(m);
    const TokRows<Tin> q(p.q, grow, hd, p.H, DK, left), k(p.k, grow, hd, p.H, DK, left);
    const TokRows<Tin> v(p.v, grow, hd, p.H, DV, left), o(p.dout, grow, hd, p.H, DV, left);
    const double Gt = w.G[row0 + tl];
    const LdsTile tile(tiles + tb * kLdsTile, l31, h);
    const int lane4 = 4 * lane;
    const size_t tok4 = (row0 + 32 * tb) * kR + lane4;                  // the wave's token blocks
    auto mask = [&](const f32x16 &s, int sb, bool with_beta) {
        const size_t s0 = row0 + 32 * sb + 4 * h;
        return causal(s, Gt, w.G + s0, with_beta ? w.bet + s0 : nullptr, tl, 32 * sb, h);
    };
    auto put = [&](float (*S)[kLS], const f32x16 &s, int sb) {
#pragma unroll
        for (int qq = 0; qq < 4; ++qq)
            *reinterpret_cast<f32x4 *>(&S[tl][32 * sb + 8 * qq + 4 * h]) =
                f32x4{s[4 * qq], s[4 * qq + 1], s[4 * qq + 2], s[4 * qq + 3]};
    };
    f32x16 sd[2];                               // this wave's (dp, a) tiles, for dq
    f32x16 x[4];
    auto score_a = [&](const float *rows, float (*S)[kLS], bool keep) {
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) x[kb] = ld_block(rows + tok4 + 1024 * kb);
#pragma unroll
        for (int sb = 0; sb < 2; ++sb) {
            f32x16 s = f32x16{}, s2 = f32x16{};
            const float *cp = w.cs + (row0 + 32 * sb) * kR + lane4;
            piped<4, kAhead>([&](int n) { return ld_block(cp + 1024 * n); },
                     [&](int n, const f32x16 &a) { return wc.apply(a, n, h); },
                     [&](int n, const f32x16 &a) { mma_step(n < 2 ? s : s2, a, x[n]); });
            s = mask(s + s2, sb, true);
            put(S, s, sb);
            if (keep) sd[sb] = s;
        }
    };
    auto score_x = [&](const TokRows<Tin> &xr, const TokRows<Tin> &yr, auto dim, float (*S)[kLS]) {
        constexpr int D = decltype(dim)::value;
        f32x16 s[2] = {}, raw = xr.wide_raw(tl, h, 0), nxt = xr.wide_raw(tl, h, 32), xv;
        piped<D / 32 * 2, kAhead>(
            [&](int n) { return yr.wide_raw(32 * (n & 1) + l31, h, 32 * (n >> 1)); },
            [&](int, const f32x16 &a) { return yr.wide_cvt(a); },
            [&](int n, const f32x16 &a) {
                if ((n & 1) == 0) {
                    xv = xr.wide_cvt(raw);
                    raw = nxt;
                    if (n + 4 < D / 16) nxt = xr.wide_raw(tl, h, 32 * (n / 2 + 2));
                }
                mma_step(s[n & 1], a, xv);
            });
        put(S, mask(s[0], 0, false), 0);
        put(S, mask(s[1], 1, false), 1);
    };
    score_a(p.U, Sua, false);
    score_x(q, k, std::integral_constant<int, DK>{}, Sqk);
    score_x(o, v, std::integral_constant<int, DV>{}, Sdov);
    score_a(p.dP, Sdpa, true);                  // last: x keeps dp
    auto store = [&](void *dst, const f32x16 &a, int D, int x0) {
        if (!inside) return;
        Tin *row = static_cast<Tin *>(dst) + ((grow + tl) * p.H + hd) * D + x0 + 4 * h;
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) {
            f32x4 y;
#pragma unroll
            for (int e = 0; e < 4; ++e) y[e] = live ? a[4 * qq + e] : 0.f;
            if constexpr (sizeof(Tin) == 4) {
                *reinterpret_cast<f32x4 *>(row + 8 * qq) = y;
            } else {
                mfma::bf16x4 z;
#pragma unroll
                for (int e = 0; e < 4; ++e) z[e] = (__bf16)y[e];
                *reinterpret_cast<mfma::bf16x4 *>(row + 8 * qq) = z;
            }
        }
    };
    // dq = gamma (dP Kbar_c) + Sdpa K: every 32 terms in a sum of their own (with one
    // running sum the errors of <q, dq> - <k, dk> made dlog_alpha a third less accurate)
    const size_t st = ((size_t)bh * p.nc + c) * kR;
    f32x16 qdq = f32x16{}, kdk = f32x16{};
    {
        const float g = w.gam[row0 + tl];
        const float *kp = w.Kst + st * DK + lane4;
#pragma unroll 1
        for (int x0 = 0; x0 < DK; x0 += 64) {
            f32x16 a[6];
            piped<12, kAhead>(
                [&](int n) {
                    const int y = x0 + 32 * (n / 6), kb = n % 6;
                    return kb < 4 ? ld_block(kp + (kb * (DK / 32) + y / 32) * 1024) : k.cols_raw(32 * (kb - 4), h, y + l31);
                },
                [&](int n, const f32x16 &y) { return n % 6 < 4 ? y : k.cols_cvt(y); },
                [&](int n, const f32x16 &y) {
                    const int kb = n % 6;
                    a[kb] = f32x16{};
                    mma_step(a[kb], y, kb < 4 ? x[kb] : sd[kb - 4]);
                    if (kb < 5) return;
                    const int y0 = x0 + 32 * (n / 6);
                    const f32x16 r = ((a[0] + a[1]) + (a[2] + a[3])) * g + (a[4] + a[5]);
                    add_products(qdq, q.rows(tl, h, y0), r);
                    store(p.gq, r, DK, y0);
                });
        }
    }
    __syncthreads();
    // dk = rho (A DK') + Sdpa^T Q, dv = rho (A DV') + Sua^T dO
    const float wr = w.wr[row0 + tl], be = w.bet[row0 + tl];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) x[kb] = wc.apply(ld_block(w.cs + tok4 + 1024 * kb), kb, h);
    auto ld_S = [&](const float (*S)[kLS], int tt) {
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = S[32 * tt + 8 * (r >> 2) + 4 * h + (r & 3)][tl];
        return s;
    };
    // (above the diagonal the score tiles hold zeros)
    auto writer = [&](const float *De, int D, const float (*S)[kLS], const TokRows<Tin> &xr, void *dst, auto &&dot) {
        const float *dp = De + st * D + lane4;
        const f32x16 s0 = ld_S(S, 0), s1 = ld_S(S, 1);
#pragma unroll 1
        for (int x0 = 0; x0 < D; x0 += 64) {
            f32x16 a[6];
            piped<12, kAhead>(
                [&](int n) {
                    const int y = x0 + 32 * (n / 6), kb = n % 6;
                    return kb < 4 ? ld_block(dp + (kb * (D / 32) + y / 32) * 1024) : xr.cols_raw(32 * (kb - 4), h, y + l31);
                },
                [&](int n, const f32x16 &y) { return n % 6 < 4 ? y : xr.cols_cvt(y); },
                [&](int n, const f32x16 &y) {
                    const int kb = n % 6;
                    a[kb] = f32x16{};
                    mma_step(a[kb], y, kb < 4 ? x[kb] : (kb == 4 ? s0 : s1));
                    if (kb < 5) return;
                    const int y0 = x0 + 32 * (n / 6);
                    const f32x16 r = ((a[0] + a[1]) + (a[2] + a[3])) * wr + (a[4] + a[5]);
                    dot(r, y0);
                    store(dst, r, D, y0);
                });
        }
    };
    writer(w.DKe, DK, Sdpa, q, p.gk, [&](const f32x16 &a, int x0) { add_products(kdk, k.rows(tl, h, x0), a); });
    writer(w.DVe, DV, Sua, o, p.gv, [](const f32x16 &, int) {});
    // da's two parts: rho DK' k + Sqk^T dp and rho DV' v + Sdov^T u
    const float rho = exp2_wide(w.G[row0 + kTC - 1] - Gt);
    auto da_part = [&](f32x16 (&a)[4], const float *De, auto dim, const TokRows<Tin> &xr, const float (*S)[kLS],
                       const float *rows) {
        constexpr int D = decltype(dim)::value;
        const float *dp = De + st * D + lane4;
#pragma unroll
        for (int y = 0; y < 4; ++y) a[y] = f32x16{};
        f32x16 raw = xr.wide_raw(tl, h, 0), xv, own[4];
        piped<D / 32 * 4, kAhead>(
            [&](int n) { return ld_block(dp + ((n & 3) * (D / 32) + (n >> 2)) * 1024); },
            [&](int, const f32x16 &y) { return tile.template swap<true>(y); },
            [&](int n, const f32x16 &y) {
                if ((n & 3) == 0) {
                    xv = xr.wide_cvt(raw);
                    if (n + 4 < D / 8) raw = xr.wide_raw(tl, h, 32 * (n / 4 + 1));
                }
                mma_step(a[n & 3], y, xv);
                if (n / 4 == D / 64 - 1) {      // two sums of half the contraction
                    own[n & 3] = a[n & 3];
                    a[n & 3] = f32x16{};
                }
            });
#pragma unroll
        for (int y = 0; y < 4; ++y) {
            a[y] += own[y];
            own[y] = f32x16{};
        }
        const float *rp = rows + row0 * kR + lane4;
        const f32x16 s0 = ld_S(S, 0), s1 = ld_S(S, 1);
        piped<8, kAhead>([&](int n) { return ld_block(rp + n * 1024); },
                         [&](int, const f32x16 &y) { return tile.template swap<false>(y); },
                         [&](int n, const f32x16 &y) { mma_step(own[n & 3], y, n < 4 ? s0 : s1); });
#pragma unroll
        for (int y = 0; y < 4; ++y) a[y] = a[y] * rho + own[y];
    };
    f32x16 da[4], dv[4];
    da_part(dv, w.DVe, std::integral_constant<int, DV>{}, v, Sdov, p.U);
    const float adav = be * dot4(x, dv);        // x: U(-lambda) b of the token
    da_part(da, w.DKe, std::integral_constant<int, DK>{}, k, Sqk, p.dP);
#pragma unroll
    for (int y = 0; y < 4; ++y) da[y] += dv[y];
    const float db = dot4(x, da);
    const float gl = -(kTwoPi / (float)m) * be * pair_moment(da, x, h);
    const float qk = tree(qdq) - tree(kdk);
    if (h == 0 && inside) {
        const size_t ti = row0 + tl;
        p.dG[ti] = live ? qk - adav + p.udu[ti] : 0.f;
        p.dlam[ti] = live ? p.dlam[ti] + gl : 0.f;
        if (p.gbeta) p.gbeta[(grow + tl) * p.H + hd] = live ? db : 0.f;
    }
}

// Short calls: up to kShortChunks 64-token chunks, or one chunk per sequence, with d_k and d_v
// at most 128.  The kernels of this file take about 200 us (d = 64) or 240 us (128) however few
// the tokens, those of cyfa_bwd_f32_short.h 80 .. 100 and 100 .. 125; at 128 chunks (B 4, T 200,
// H 8) 231 against 115 us and 274 against 154, at 256 (B 8, T 100, H 16) 246 against 156 and 285
// against 201, or with one head (B 64, T 200) 266 against 210 and 298 against 248.  Beyond, four
// waves per 32 tokens fetch the matrices too often and leave dR too many partial sums per head:
// at 384 chunks 307 against 293 us with 16 heads (d = 128, B 8, T 130), but 334 against 370 with
// one (B 64, T 380); at 512 338 against 359.  A sequence of one chunk leaves half of a
// chunk pair idle: 512 sequences of 64 tokens 457 against 382 us (d = 128) and 379 against 271
// (64), 2048 of 16 tokens 1652 against 931 and 1398 against 682.
constexpr int kShortChunks = 256;
bool short_call(const BwdParams &p) {
    return p.dk <= 128 && p.dv <= 128 && (p.nc == 1 || (long long)p.B * p.H * p.nc <= kShortChunks);
}

// Workgroups per head of the readout kernel: one round over the compute units, each with the
// same number of chunk pairs; in a short call two rounds of the 32-token tiles' workgroups.
int readout_wgs(const BwdParams &p, int *per) {
    const bool tiles = short_call(p);
    const int np = tiles ? p.B * ((p.T + 31) / 32) : p.B * ((p.nc + 1) / 2);
    int n = ((tiles ? 512 : 256) + p.H - 1) / p.H;
    if (n > np) n = np;
    if (tiles) return n;
    *per = (np + n - 1) / n;
    return (np + *per - 1) / *per;
}

template <int DK, int DV, typename Tin>
hipError_t launch_typed(const BwdParams &p, const F32Ws &w, hipStream_t s) {
    const int BH = p.B * p.H;
    launch_front(p, w, s);
    launch_states<DK, DV, Tin, false>(p, w, s);
    int per = 1;
    const int nu = p.nc > 0 ? readout_wgs(p, &per) : 0;
    const bool few = p.nc > 0 && short_call(p);
    if constexpr (DK <= 128) {
        if (few)
            hipLaunchKernelGGL((f32_readout_short_kernel<DK, DV, Tin>), dim3(p.H, nu), dim3(256), 0, s, p, w);
    }
    if (p.nc > 0 && !few)
        hipLaunchKernelGGL((f32_readout_kernel<DK, DV, Tin>), dim3(p.H, nu), dim3(256), 0, s, p, w, per);
    launch_states<DK, DV, Tin, true>(p, w, s);
    if constexpr (DK <= 128) {
        if (few)
            hipLaunchKernelGGL((f32_grad_short_kernel<DK, DV, Tin>), dim3(p.nc * BH), dim3(512), 0, s, p, w);
    }
    if (p.nc > 0 && !few)
        hipLaunchKernelGGL((f32_grad_kernel<DK, DV, Tin>), dim3(p.nc * BH), dim3(128), 0, s, p, w);
    BwdParams tail = p;
    tail.groups = 1;                // dMp is [nu][H][128][128]
    return launch_bwd_tail(tail, nu, s);
}

template <int DK, int DV>
hipError_t launch_dtype(const BwdParams &p, const F32Ws &w, hipStream_t s) {
    return p.dtype == 0 ? launch_typed<DK, DV, float>(p, w, s) : launch_typed<DK, DV, __hip_bfloat16>(p, w, s);
}

}  // namespace

// Layout (each piece 256-byte aligned): Mi + MiT, clk, cs, G, gam + wr + bet, gend, Kst,
// Vst, DKe, DVe, U, dP, udu, dlam, dG, dMp, fin.
static size_t need_bytes(int B, int T, int H, int dk, int dv) {
    const size_t BH = (size_t)B * H, nc = ((size_t)T + kTC - 1) / kTC, Tpad = nc * kTC;
    int per = 1;
    BwdParams p{};
    p.B = B; p.T = T; p.H = H; p.dk = dk; p.dv = dv; p.nc = (int)nc;
    size_t n = align_up(2 * readout_f32_bytes(H));
    n += align_up(BH * nc * 8);
    n += align_up(BH * Tpad * kR * 4);
    n += align_up(BH * Tpad * 8);
    n += align_up(3 * BH * Tpad * 4);
    n += align_up(BH * nc * 4);
    n += 2 * (align_up(BH * nc * kR * dk * 4) + align_up(BH * nc * kR * dv * 4));
    n += 2 * align_up(BH * Tpad * kR * 4);
    n += 3 * align_up(BH * Tpad * 4);
    if (nc > 0) n += align_up((size_t)readout_wgs(p, &per) * H * kR * kR * 4);
    n += align_up(BH * kBwdFinParts * 8);
    return n;
}

// Never less than the size the public header states (two states per 16 tokens and two
// rows per token and head), which callers provision for by that formula.
size_t bwd_f32_workspace_bytes(int B, int T, int H, int dk, int dv) {
    const size_t BH = (size_t)B * H, nc = ((size_t)T + kBwdChunk - 1) / kBwdChunk;
    const size_t stated = 2 * align_up(BH * nc * kR * (size_t)(dk + dv) * 4) + 2 * align_up(BH * nc * kBwdChunk * kR * 4);
    const size_t need = need_bytes(B, T, H, dk, dv);
    return need > stated ? need : stated;
}

hipError_t launch_bwd_f32(BwdParams p, void *ws, hipStream_t s) {
    const size_t BH = (size_t)p.B * p.H;
    p.nc = (p.T + kTC - 1) / kTC;
    p.Tpad = p.nc * kTC;
    const size_t nc = p.nc, Tpad = p.Tpad;
    char *at = static_cast<char *>(ws);
    auto take = [&at](size_t bytes) { char *r = at; at += align_up(bytes); return reinterpret_cast<float *>(r); };
    F32Ws w{};
    w.Mi = take(2 * readout_f32_bytes(p.H));
    w.MiT = w.Mi + (size_t)p.H * kR * kR;
    w.clk = reinterpret_cast<double *>(take(BH * nc * 8));
    w.cs = take(BH * Tpad * kR * 4);
    w.G = reinterpret_cast<double *>(take(BH * Tpad * 8));
    w.gam = take(3 * BH * Tpad * 4);
    w.wr = w.gam + BH * Tpad;
    w.bet = w.wr + BH * Tpad;
    w.gend = take(BH * nc * 4);
    w.Kst = take(BH * nc * kR * p.dk * 4);
    w.Vst = take(BH * nc * kR * p.dv * 4);
    w.DKe = take(BH * nc * kR * p.dk * 4);
    w.DVe = take(BH * nc * kR * p.dv * 4);
    p.U = take(BH * Tpad * kR * 4);
    p.dP = take(BH * Tpad * kR * 4);
    p.udu = take(BH * Tpad * 4);
    p.dlam = take(BH * Tpad * 4);
    p.dG = take(BH * Tpad * 4);
    int per = 1;
    if (nc > 0) p.dMp = take((size_t)readout_wgs(p, &per) * p.H * kR * kR * 4);
    p.fin = reinterpret_cast<double *>(take(BH * kBwdFinParts * 8));
    if (p.dk == 64 && p.dv == 64) return launch_dtype<64, 64>(p, w, s);
    if (p.dk == 64 && p.dv == 128) return launch_dtype<64, 128>(p, w, s);
    if (p.dk == 128 && p.dv == 64) return launch_dtype<128, 64>(p, w, s);
    if (p.dk == 256 && p.dv == 256) return launch_dtype<256, 256>(p, w, s);
    return launch_dtype<128, 128>(p, w, s);
}

}  // namespace cyfa

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
// with every intermediate in registers.  fp32 throughout, as the vector-ALU kernels
// that these replace: 27.3 -> 3.6 ms at B 32, T 2048, H 4, d_k = d_v = 256 (bf16 inputs;
// 330 GFLOP in tiles, 91 TFLOP/s of the 157 the fp32 matrix instructions have) and 574
// -> 283 us at B 4, T 1000, H 4, d = 64 (fp32).  The readout and gradient kernels run one
// wave per SIMD (a wave's tokens need 4 .. 5 tiles of 64 registers) and are bound by
// their matrix instructions, the vector work between them and the loads' latency at
// each product's start.  Kernels: (0) clocks and phase tables; (1)
// states entering every chunk; (2) readout recomputation and its adjoint; (3)
// adjoint states at every chunk's end; (4) token gradients; (5) reverse cumulative
// sums, per sequence; (6) dR, per head.
#include <type_traits>

#include "cyfa_bwd.h"
#include "cyfa_tile_f32.h"

namespace cyfa {

namespace {

using namespace tile;
using mfma::internal_to_paper;
using mfma::kDC;

constexpr float kTwoPi = 6.283185307179586f;
constexpr int kR = kStoreRows;
constexpr int kLS = 68;             // row stride of [64][64] LDS tiles
constexpr int kAhead = 2;           // operands in flight beyond the one being prepared (one: 6 % slower)

__device__ __forceinline__ int bwd_tokens(const BwdParams &p, int b) {
    return p.lens ? min(max(p.lens[b], 0), p.T) : p.T;
}

// Storage row of internal row i; internal rows without a basis function stand for the
// padding rows m .. 127.
__device__ __forceinline__ int paper_row(int i, int m) {
    const int ip = internal_to_paper(i, m);
    return ip >= 0 ? ip : (i == kR - 1 ? kR - 1 : i + 1);
}

// Workspace of the fp32 backward; basis rows and columns in the internal order.  "blocks"
// of 32 x 32 floats are laid out as in cyfa_tile_f32.h: [lane index][chain index].
struct F32Ws {
    float *Mi, *MiT;                // [H] 4 x 4 blocks [slot][basis] and [basis][slot] of the readout matrix
    double *clk;                    // [BH][nc] clock entering each chunk (reduced mod m)
    float *cs;                      // [BH][Tpad/32] 4 blocks [token][basis]: phases as (cos, sin) pairs, DC 1, padding 0
    double *G;                      // [BH][Tpad] log2 of the decay from the chunk's start through token t
    float *gam, *wr, *bet;          // [BH][Tpad] exp(G_t), beta_t exp(G_C - G_t), beta_t
    float *gend;                    // [BH][nc] exp(G_C)
    float *Kst, *Vst;               // [BH][nc] 4 x d/32 blocks [channel][basis] of the states entering each chunk
    float *DKe, *DVe;               // the same of the adjoint states at each chunk's end
};                                  // (BwdParams::U and dP: [BH][Tpad/32] 4 blocks [token][basis])

// ---------------------------------------------------------------------------
// (0a) readout matrices in both orientations, and the clock entering every chunk.
// Block (h, rb): rows 8 rb .. + 7 of M_h, thread (j, g) column j of four rows; blocks
// past H * 16: one per sequence.
constexpr int kPrepRows = 8;
__global__ __launch_bounds__(256) void f32_prep_kernel(BwdParams p, F32Ws w) {
    __shared__ __attribute__((aligned(16))) float Rr[kPrepRows][kR];
    __shared__ float tab[2][kR];
    const int tid = threadIdx.x, m = p.m, nprep = p.H * (kR / kPrepRows);
    if ((int)blockIdx.x >= nprep) {
        const int bh = blockIdx.x - nprep, b = bh / p.H, h = bh % p.H, lane = tid & 63;
        const int Tb = bwd_tokens(p, b);
        double *cl = w.clk + (size_t)bh * p.nc;
        const float *dl = p.delta + (size_t)b * p.T * p.H + h;
        for (int c = tid >> 6; c < p.nc; c += 4) {
            const int t = c * kTC + lane;
            const double x = t < Tb ? (double)dl[(size_t)t * p.H] : 0.0;
            const double s = mfma::lane63(mfma::wave_incl_scan(x));
            if (lane == 0) cl[c] = s;
        }
        __syncthreads();
        if (tid >= 64) return;
        double base = p.clock0 ? p.clock0[bh] : 0.0;
        for (int c0 = 0; c0 < p.nc; c0 += 64) {
            const double x = c0 + lane < p.nc ? cl[c0 + lane] : 0.0;
            const double s = mfma::wave_incl_scan(x);
            if (c0 + lane < p.nc) cl[c0 + lane] = reduce_clock(base + (s - x), m);
            base = reduce_clock(base + mfma::lane63(s), m);
        }
        return;
    }
    const int h = blockIdx.x / (kR / kPrepRows), i0 = (blockIdx.x % (kR / kPrepRows)) * kPrepRows;
    if (tid < m) {
        double sn, cs;
        sincospi(2.0 * (double)tid / (double)m, &sn, &cs);
        tab[0][tid] = (float)cs;
        tab[1][tid] = (float)sn;
    }
    const float *Rh = p.R ? p.R + (size_t)h * m * m : nullptr;
    for (int e = tid; e < kPrepRows * kR; e += 256) {
        const int i = i0 + (e >> 7), s = e & 127;
        Rr[e >> 7][s] = (i < m && s < m) ? (Rh ? Rh[(size_t)i * m + s] : (s == i ? 1.f : 0.f)) : 0.f;
    }
    __syncthreads();
    const int j = tid & 127, r0 = (tid >> 7) * 4, jp = internal_to_paper(j, m);
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    if (jp >= 0) {
        const float *t = (jp == 0 || (jp & 1)) ? tab[0] : tab[1];
        const int l = (jp + 1) >> 1;
        int idx = 0;
        for (int s0 = 0; s0 < m; s0 += 4) {             // R's staged rows are 0 past column m
            float ph[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                ph[q] = t[idx];
                idx += l;
                if (idx >= m) idx -= m;
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const f32x4 rv = *reinterpret_cast<const f32x4 *>(&Rr[r0 + r][s0]);
                acc[r] = fmaf(rv[0], ph[0], fmaf(rv[1], ph[1], fmaf(rv[2], ph[2], fmaf(rv[3], ph[3], acc[r]))));
            }
        }
    }
    const float sc = jp == 0 ? (float)(1.0 / sqrt((double)m)) : (float)sqrt(2.0 / (double)m);
    // element (x, y) of a matrix of blocks [x][y]
    auto at = [&](int x, int y) {
        return ((size_t)h * 16 + (x >> 5) * 4 + (y >> 5)) * 1024 + 256 * ((y >> 3) & 3) + 128 * ((y >> 2) & 1) +
               4 * (x & 31) + (y & 3);
    };
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        w.Mi[at(i0 + r0 + r, j)] = acc[r] * sc;
        w.MiT[at(j, i0 + r0 + r)] = acc[r] * sc;
    }
}

// (0b) per (chunk, sequence): clock and log-decay prefix sums (double), per-token
// factors and the phase table.  Tokens past the sequence's end: no shift, no decay,
// no write.
__global__ __launch_bounds__(256) void f32_tables_kernel(BwdParams p, F32Ws w) {
    __shared__ double rev[kTC];
    const int c = blockIdx.x, bh = blockIdx.y, b = bh / p.H, h = bh % p.H, tid = threadIdx.x, m = p.m;
    const int Tb = bwd_tokens(p, b);
    const size_t row0 = (size_t)bh * p.Tpad + (size_t)c * kTC;
    if (tid < kTC) {
        const int t = c * kTC + tid;
        const bool live = t < Tb;
        const size_t si = ((size_t)b * p.T + t) * p.H + h;
        const double dl = live ? (double)p.delta[si] : 0.0;
        const double la = live && p.log_alpha ? (double)p.log_alpha[si] * 1.4426950408889634 : 0.0;
        const float be = live ? (p.beta ? p.beta[si] : 1.f) : 0.f;
        const double lam = reduce_clock(w.clk[(size_t)bh * p.nc + c] + mfma::wave_incl_scan(dl), m);
        const double G = mfma::wave_incl_scan(la), GC = mfma::lane63(G);
        rev[tid] = lam / (double)m;
        w.G[row0 + tid] = G;
        w.gam[row0 + tid] = exp2_wide(G);
        w.wr[row0 + tid] = be * exp2_wide(GC - G);
        w.bet[row0 + tid] = be;
        if (tid == 0) w.gend[(size_t)bh * p.nc + c] = exp2_wide(GC);
    }
    __syncthreads();
    // piece (token block, basis block, q) of the table: lane (h, token) two pairs
    const int J = (m - 1) / 2, lane = tid & 63;
    f32x4 *cs = reinterpret_cast<f32x4 *>(w.cs + row0 * kR);
    for (int u = tid >> 6; u < 32; u += 4) {
        const double rv = rev[32 * (u >> 4) + (lane & 31)];
        const int j0 = 16 * ((u >> 2) & 3) + 4 * (u & 3) + 2 * (lane >> 5);      // pairs j0, j0 + 1
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            float cc = j0 + e == 63 ? 1.f : 0.f, sn = 0.f;
            if (j0 + e < J) {
                double x = (double)(j0 + e + 1) * rv;
                x -= floor(x);
                sincospif((float)(2.0 * x), &sn, &cc);
            }
            v[2 * e] = cc;
            v[2 * e + 1] = sn;
        }
        cs[u * 64 + lane] = v;
    }
}

// ---------------------------------------------------------------------------
// (1), (3) states entering each chunk (ADJ = false: sum_s rho_s a_s k_s^T and v_s) or
// adjoint states at each chunk's end (ADJ = true: sum_t gamma_t dp_t q_t^T and u_t
// do_t^T, chunks in reverse), 64 columns of a state per workgroup, wave w rows 32 w ..
// + 31.  The columns of a state are independent, so with enough sequences (WALK) one
// workgroup carries its columns through every chunk and no combine is needed; with
// few, every chunk's own contribution is formed in parallel (one per blockIdx.z) and
// f32_scan_kernel combines them.  The line lies at 256 workgroups, one per compute
// unit: a walk's step is a dependent chain of two memory round trips.
template <int D, typename Tin, bool ADJ, bool WALK>
__device__ __forceinline__ void state_columns(const BwdParams &p, const F32Ws &w, const void *tok, const float *rows,
                                              float *slots, const float *ext, const float *fext, float *gext, int cb,
                                              float *lds) {
    const int bh = blockIdx.x, b = bh / p.H, hd = bh % p.H, tid = threadIdx.x, m = p.m;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    int l31 = tid & 31, h = (tid >> 5) & 1;
    const int Tb = bwd_tokens(p, b);
    const WriteCoef wc(m);
    const float coef = ADJ ? 1.f : wc.at(32 * wv + l31);
    f32x16 acc[2] = {f32x16{}, f32x16{}};
    if (WALK && ext)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            __builtin_amdgcn_sched_barrier(0);
            const int ip = internal_to_paper(32 * wv + 8 * (r >> 2) + 4 * h + (r & 3), m);
            const float *e = ext + ((size_t)bh * kR + max(ip, 0)) * D + 64 * cb + l31;
            acc[0][r] = ip >= 0 ? e[0] : 0.f;
            acc[1][r] = ip >= 0 ? e[32] : 0.f;
        }
    // The chunk's 64 x 64 piece of the token rows goes through LDS, shared by the four
    // waves; the next chunk's piece, its factors and this wave's table or dp / u blocks
    // are in flight while a chunk is worked on.
    constexpr int NQ = 4 * (int)sizeof(Tin) / 4;        // 16-byte pieces of 16 channels
    float *Ts = lds, *fs = lds + kTC * kLS;
    const int sr = tid >> 2, sc = (tid & 3) * 16;
    u32x4 tok4[NQ];
    f32x16 a[2];
    float fac = 0.f;
    auto chunk_of = [&](int it) { return WALK ? (ADJ ? p.nc - 1 - it : it) : (int)blockIdx.z; };
    auto fetch_tok = [&](int it) {
        const int c = chunk_of(it);
        const TokRows<Tin> tr(tok, (size_t)b * p.T + c * kTC, hd, p.H, D, min(Tb - c * kTC, kTC));
#pragma unroll
        for (int q = 0; q < NQ; ++q) tok4[q] = tr.piece(sr, (64 * cb + sc) * (int)sizeof(Tin) + 16 * q);
        if (tid < kTC) fac = (ADJ ? w.gam : w.wr)[(size_t)bh * p.Tpad + c * kTC + tid];
    };
    auto fetch_row = [&](int it, int kb) {
        const size_t row0 = (size_t)bh * p.Tpad + chunk_of(it) * kTC;
        return ld_block(rows + row0 * kR + (4 * kb + wv) * 1024 + 4 * (32 * h + l31));
    };
    const int n = WALK ? p.nc : 1;
    if (n > 0) {
        fetch_tok(0);
        a[0] = fetch_row(0, 0);
        a[1] = fetch_row(0, 1);
    }
    for (int it = 0; it < n; ++it) {
        l31 = mfma::opq(l31);
        h = mfma::opq(h);
        const LdsTile tile(fs + kTC + wv * kLdsTile, l31, h);
        const int c = chunk_of(it);
        float *slot = slots + ((size_t)bh * p.nc + c) * kR * D + (wv * (D / 32) + 2 * cb) * 1024 + 4 * (32 * h + l31);
        mfma::lds_barrier();                    // the previous chunk's piece has been read
#pragma unroll
        for (int q = 0; q < NQ; ++q) TokRows<Tin>::spread(Ts + sr * kLS + sc, q, tok4[q]);
        if (tid < kTC) fs[tid] = fac;
        mfma::lds_barrier();
        if (it + 1 < n) fetch_tok(it + 1);
        if (WALK) {
            st_block(slot, acc[0]);
            st_block(slot + 1024, acc[1]);
            const float ge = w.gend[(size_t)bh * p.nc + c];
            acc[0] *= ge;
            acc[1] *= ge;
        }
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            a[kb] = tile.swap<false>(a[kb]) * (ld_rows(fs + 32 * kb + 4 * h) * coef);
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                __builtin_amdgcn_sched_barrier(0);
                f32x16 y;
#pragma unroll
                for (int r = 0; r < 16; ++r) y[r] = Ts[(32 * kb + 8 * (r >> 2) + 4 * h + (r & 3)) * kLS + 32 * x + l31];
                mma_step(acc[x], a[kb], y);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (it + 1 < n) a[kb] = fetch_row(it + 1, kb);
        }
        if (!WALK) {
            st_block(slot, acc[0]);
            st_block(slot + 1024, acc[1]);
        }
    }
    if (!WALK) return;
    // the state after the last token against dK_T / dV_T, or the initial state's gradient
    double fin = 0.0;
    const float *io = ADJ ? gext : fext;
    if (io)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            __builtin_amdgcn_sched_barrier(0);
            const int i = 32 * wv + 8 * (r >> 2) + 4 * h + (r & 3), ip = internal_to_paper(i, m);
            const size_t at = ((size_t)bh * kR + paper_row(i, m)) * D + 64 * cb + l31;
            if (ADJ) {
                gext[at] = ip >= 0 ? acc[0][r] : 0.f;
                gext[at + 32] = ip >= 0 ? acc[1][r] : 0.f;
            } else if (ip >= 0) {
                fin += (double)fext[at] * acc[0][r];
                fin += (double)fext[at + 32] * acc[1][r];
            }
        }
    if (!ADJ) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) fin += __shfl_xor(fin, o);
        __syncthreads();
        double *red = reinterpret_cast<double *>(lds);
        if ((tid & 63) == 0) red[wv] = fin;
        __syncthreads();
        if (tid == 0) p.fin[(size_t)bh * kBwdFinParts + blockIdx.y] = (red[0] + red[1]) + (red[2] + red[3]);
        const int ny = gridDim.y;
        if (blockIdx.y == 0 && tid >= ny && tid < kBwdFinParts) p.fin[(size_t)bh * kBwdFinParts + tid] = 0.0;
    }
}

template <int DK, int DV, typename Tin, bool ADJ, bool WALK>
__global__ __launch_bounds__(256, 4) void f32_states_kernel(BwdParams p, F32Ws w) {
    __shared__ __attribute__((aligned(16))) float lds[kTC * kLS + kTC + 4 * kLdsTile];
    const int y = blockIdx.y;
    if (y < DK / 64)
        state_columns<DK, Tin, ADJ, WALK>(p, w, ADJ ? p.q : p.k, ADJ ? p.dP : w.cs, ADJ ? w.DKe : w.Kst,
                                          ADJ ? p.dK_T : p.K0, p.dK_T, p.gK0, y, lds);
    else
        state_columns<DV, Tin, ADJ, WALK>(p, w, ADJ ? p.dout : p.v, ADJ ? p.U : w.cs, ADJ ? w.DVe : w.Vst,
                                          ADJ ? p.dV_T : p.V0, p.dV_T, p.gV0, y - DK / 64, lds);
}

// Combines the chunks' own contributions in place, element by element: slot c becomes
// the state entering chunk c (the adjoint at its end, in reverse).  Eight chunks'
// loads are in flight at a time; only the multiply-add is a chain.
template <int DK, int DV, bool ADJ>
__global__ __launch_bounds__(256) void f32_scan_kernel(BwdParams p, F32Ws w) {
    __shared__ double red[4];
    const int bh = blockIdx.x, tid = threadIdx.x, m = p.m, nc = p.nc;
    const float *ge = w.gend + (size_t)bh * nc;
    double fin = 0.0;
    auto run = [&](int D, float *slots, const float *ext, const float *fext, float *gext) {
        const size_t st = (size_t)kR * D / 4;
        for (int e = blockIdx.y * 256 + tid; e < kR * D / 4; e += 256 * kBwdFinParts) {
            // four basis rows i0 .. + 3 of channel ch
            const int blk = e >> 8, l = e & 63, i0 = 32 * (blk / (D / 32)) + 8 * ((e >> 6) & 3) + 4 * (l >> 5);
            const int ch = 32 * (blk % (D / 32)) + (l & 31);
            f32x4 *s = reinterpret_cast<f32x4 *>(slots + (size_t)bh * nc * kR * D) + e;
            f32x4 E = {0.f, 0.f, 0.f, 0.f};
            auto ext_at = [&](int q) {
                const int ip = internal_to_paper(i0 + q, m);
                return ip >= 0 ? (ptrdiff_t)((size_t)bh * kR + ip) * D + ch : (ptrdiff_t)-1;
            };
            if (ext)
#pragma unroll
                for (int q = 0; q < 4; ++q) E[q] = ext_at(q) >= 0 ? ext[ext_at(q)] : 0.f;
            for (int c0 = 0; c0 < nc; c0 += 8) {
                f32x4 own[8];
                float g[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int c = min(c0 + u, nc - 1), cc = ADJ ? nc - 1 - c : c;
                    own[u] = s[cc * st];
                    g[u] = ge[cc];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    if (c0 + u >= nc) break;
                    s[(ADJ ? nc - 1 - (c0 + u) : c0 + u) * st] = E;
#pragma unroll
                    for (int q = 0; q < 4; ++q) E[q] = fmaf(g[u], E[q], own[u][q]);
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int ip = internal_to_paper(i0 + q, m);
                if (ADJ) {
                    if (gext) gext[((size_t)bh * kR + paper_row(i0 + q, m)) * D + ch] = ip >= 0 ? E[q] : 0.f;
                } else if (fext && ip >= 0) {
                    fin += (double)fext[ext_at(q)] * E[q];
                }
            }
        }
    };
    run(DK, ADJ ? w.DKe : w.Kst, ADJ ? p.dK_T : p.K0, p.dK_T, p.gK0);
    run(DV, ADJ ? w.DVe : w.Vst, ADJ ? p.dV_T : p.V0, p.dV_T, p.gV0);
    if (ADJ) return;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) fin += __shfl_xor(fin, o);
    if ((tid & 63) == 0) red[tid >> 6] = fin;
    __syncthreads();
    if (tid == 0) p.fin[(size_t)bh * kBwdFinParts + blockIdx.y] = (red[0] + red[1]) + (red[2] + red[3]);
}

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
        const size_t grow = (size_t)b * p.T + cc * kTC, row0 = (size_t)bh * p.Tpad + cc * kTC;
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
    const int c = blockIdx.x, bh = blockIdx.y, b = bh / p.H, hd = bh % p.H, tid = threadIdx.x, m = p.m;
    const int lane = tid & 63, l31 = lane & 31, h = lane >> 5, tb = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int Tb = bwd_tokens(p, b), left = min(Tb - c * kTC, kTC);
    const size_t grow = (size_t)b * p.T + c * kTC, row0 = (size_t)bh * p.Tpad + c * kTC;
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

size_t align_up(size_t x) { return (x + 255) / 256 * 256; }

// workgroups per head of the readout kernel: one round over the compute units, each
// with the same number of chunk pairs
int readout_wgs(int B, int H, int nc, int *per) {
    const int np = B * ((nc + 1) / 2);
    int n = (256 + H - 1) / H;
    if (n > np) n = np;
    *per = (np + n - 1) / n;
    return (np + *per - 1) / *per;
}

template <int DK, int DV, typename Tin>
hipError_t launch_typed(const BwdParams &p, const F32Ws &w, hipStream_t s) {
    const int BH = p.B * p.H, ny = (DK + DV) / 64;
    const bool walk = BH * ny >= 256;
    hipLaunchKernelGGL(f32_prep_kernel, dim3(p.H * (kR / kPrepRows) + BH), dim3(256), 0, s, p, w);
    if (p.nc > 0) hipLaunchKernelGGL(f32_tables_kernel, dim3(p.nc, BH), dim3(256), 0, s, p, w);
    auto states = [&](auto adj) {
        constexpr bool A = decltype(adj)::value;
        if (walk) {
            hipLaunchKernelGGL((f32_states_kernel<DK, DV, Tin, A, true>), dim3(BH, ny), dim3(256), 0, s, p, w);
        } else {
            if (p.nc > 0)
                hipLaunchKernelGGL((f32_states_kernel<DK, DV, Tin, A, false>), dim3(BH, ny, p.nc), dim3(256), 0, s, p, w);
            hipLaunchKernelGGL((f32_scan_kernel<DK, DV, A>), dim3(BH, kBwdFinParts), dim3(256), 0, s, p, w);
        }
    };
    states(std::false_type{});
    int per = 1, nu = 0;
    if (p.nc > 0) {
        nu = readout_wgs(p.B, p.H, p.nc, &per);
        hipLaunchKernelGGL((f32_readout_kernel<DK, DV, Tin>), dim3(p.H, nu), dim3(256), 0, s, p, w, per);
    }
    states(std::true_type{});
    if (p.nc > 0) hipLaunchKernelGGL((f32_grad_kernel<DK, DV, Tin>), dim3(p.nc, BH), dim3(128), 0, s, p, w);
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
    size_t n = align_up(2 * readout_f32_bytes(H));
    n += align_up(BH * nc * 8);
    n += align_up(BH * Tpad * kR * 4);
    n += align_up(BH * Tpad * 8);
    n += align_up(3 * BH * Tpad * 4);
    n += align_up(BH * nc * 4);
    n += 2 * (align_up(BH * nc * kR * dk * 4) + align_up(BH * nc * kR * dv * 4));
    n += 2 * align_up(BH * Tpad * kR * 4);
    n += 3 * align_up(BH * Tpad * 4);
    if (nc > 0) n += align_up((size_t)readout_wgs(B, H, (int)nc, &per) * H * kR * kR * 4);
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
    if (nc > 0) p.dMp = take((size_t)readout_wgs(p.B, p.H, p.nc, &per) * p.H * kR * kR * 4);
    p.fin = reinterpret_cast<double *>(take(BH * kBwdFinParts * 8));
    if (p.dk == 64 && p.dv == 64) return launch_dtype<64, 64>(p, w, s);
    if (p.dk == 64 && p.dv == 128) return launch_dtype<64, 128>(p, w, s);
    if (p.dk == 128 && p.dv == 64) return launch_dtype<128, 64>(p, w, s);
    if (p.dk == 256 && p.dv == 256) return launch_dtype<256, 256>(p, w, s);
    return launch_dtype<128, 128>(p, w, s);
}

}  // namespace cyfa

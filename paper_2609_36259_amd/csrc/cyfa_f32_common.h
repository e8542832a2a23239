// What the fp32 matrix-instruction forward and backward share: the workspace's arrays, the
// per-token tables and the states entering (adjoint states ending) every 64-token chunk.
#pragma once

#include <type_traits>

#include "cyfa_bwd.h"
#include "cyfa_tile_f32.h"

namespace cyfa {

namespace {

using namespace tile;
using mfma::internal_to_paper;
using mfma::kDC;

constexpr int kR = kStoreRows;
constexpr int kLS = 68;             // row stride of [64][64] LDS tiles

// tokens and first row of sequence b in the [rows, H, ...] tensors
__device__ __forceinline__ int bwd_tokens(const BwdParams &p, int b) {
    if (p.cu) return min(max(p.cu[b + 1] - p.cu[b], 0), p.T);
    return p.lens ? min(max(p.lens[b], 0), p.T) : p.T;
}
__device__ __forceinline__ size_t first_row(const BwdParams &p, int b) {
    return p.cu ? (size_t)p.cu[b] : (size_t)b * p.T;
}

// Storage row of internal row i; internal rows without a basis function stand for the
// padding rows m .. 127.
__device__ __forceinline__ int paper_row(int i, int m) {
    const int ip = internal_to_paper(i, m);
    return ip >= 0 ? ip : (i == kR - 1 ? kR - 1 : i + 1);
}

// Workspace of the fp32 kernels; basis rows and columns in the internal order.  "blocks"
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
    float *Ko, *Vo;                 // final states and clocks of a forward call, or NULL
    double *clko;                   // (may be p.clock0)
    double *clkT;                   // [BH] clock after the last token, or NULL
    int c0;                         // first chunk of a launch with the chunks on the grid's z axis
};                                  // (BwdParams::U and dP: [BH][Tpad/32] 4 blocks [token][basis])

// ---------------------------------------------------------------------------
// (0) one launch forms the readout matrices in both orientations (block (h, rb): rows
// 8 rb .. + 7 of M_h, thread (j, g) column j of four rows), the clock entering every
// chunk (a block per sequence) and, up to kTableChunks chunks, the per-token tables, each
// of whose blocks then sums the increments before its chunk itself; longer sequences
// launch the tables afterwards, from the chunks' clocks.
constexpr int kPrepRows = 8;
constexpr int kTableChunks = 64;

// Per (chunk, sequence): clock and log-decay prefix sums (double), per-token factors and
// the phase table.  Tokens past the sequence's end: no shift, no decay, no write.
__device__ __forceinline__ void chunk_tables(const BwdParams &p, const F32Ws &w, int c, int bh, bool own_clock,
                                             double *rev) {
    const int b = bh / p.H, h = bh % p.H, tid = threadIdx.x, m = p.m;
    const int Tb = bwd_tokens(p, b);
    const size_t row0 = (size_t)bh * p.Tpad + (size_t)c * kTC, g0 = first_row(p, b);
    double lam0 = 0.0;
    if (own_clock) {
        const int t1 = min(c * kTC, Tb);
        double s = 0.0;
        for (int t = tid; t < t1; t += 256) s += (double)p.delta[(g0 + t) * p.H + h];
        s = mfma::lane63(mfma::wave_incl_scan(s));
        if ((tid & 63) == 0) rev[tid >> 6] = s;
        __syncthreads();
        lam0 = reduce_clock((p.clock0 ? p.clock0[bh] : 0.0) + ((rev[0] + rev[1]) + (rev[2] + rev[3])), m);
        __syncthreads();
    } else {
        lam0 = w.clk[(size_t)bh * p.nc + c];
    }
    if (tid < kTC) {
        const int t = c * kTC + tid;
        const bool live = t < Tb;
        const size_t si = (g0 + t) * p.H + h;
        const double dl = live ? (double)p.delta[si] : 0.0;
        // A decay below 2^-1024 is 0 in fp32 with any token before it, so the bound changes no
        // result but keeps the chunk's prefix sums from absorbing the later tokens' decays after
        // a reset (log alpha = -1e38, -inf).
        double la = live && p.log_alpha ? (double)p.log_alpha[si] * 1.4426950408889634 : 0.0;
        la = la < -1024.0 ? -1024.0 : la;       // (a NaN stays)
        const float be = live ? (p.beta ? p.beta[si] : 1.f) : 0.f;
        const double lam = reduce_clock(lam0 + mfma::wave_incl_scan(dl), m);
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

__global__ __launch_bounds__(256) void f32_tables_kernel(BwdParams p, F32Ws w) {
    __shared__ double rev[kTC];
    chunk_tables(p, w, blockIdx.x % p.nc, blockIdx.x / p.nc, false, rev);
}

__global__ __launch_bounds__(256) void f32_prep_kernel(BwdParams p, F32Ws w) {
    __shared__ __attribute__((aligned(16))) float Rr[kPrepRows][kR];
    __shared__ float tab[2][kR];
    const int tid = threadIdx.x, m = p.m, nprep = p.H * (kR / kPrepRows), BH = p.B * p.H;
    if ((int)blockIdx.x >= nprep + BH) {
        const int u = blockIdx.x - nprep - BH;
        chunk_tables(p, w, u % p.nc, u / p.nc, true, reinterpret_cast<double *>(&Rr[0][0]));
        return;
    }
    if ((int)blockIdx.x >= nprep) {
        const int bh = blockIdx.x - nprep, b = bh / p.H, h = bh % p.H, lane = tid & 63;
        const int Tb = bwd_tokens(p, b);
        double *cl = w.clk + (size_t)bh * p.nc;
        const float *dl = p.delta + first_row(p, b) * p.H + h;
        for (int c = tid >> 6; c < p.nc; c += 4) {
            const int t = c * kTC + lane;
            const double x = t < Tb ? (double)dl[(size_t)t * p.H] : 0.0;
            const double s = mfma::lane63(mfma::wave_incl_scan(x));
            if (lane == 0) cl[c] = s;
        }
        __syncthreads();
        if (tid >= 64) return;
        double base = reduce_clock(p.clock0 ? p.clock0[bh] : 0.0, m);
        for (int c0 = 0; c0 < p.nc; c0 += 64) {
            const double x = c0 + lane < p.nc ? cl[c0 + lane] : 0.0;
            const double s = mfma::wave_incl_scan(x);
            if (c0 + lane < p.nc) cl[c0 + lane] = reduce_clock(base + (s - x), m);
            base = reduce_clock(base + mfma::lane63(s), m);
        }
        // clock_out may be clock0, which the table blocks of this launch still read, so that the
        // states' launch copies it there
        if (w.clkT && lane == 0) w.clkT[bh] = base;
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

// ---------------------------------------------------------------------------
// (1), (3) states entering each chunk (ADJ = false: sum_s rho_s a_s k_s^T and v_s) or
// adjoint states at each chunk's end (ADJ = true: sum_t gamma_t dp_t q_t^T and u_t
// do_t^T, chunks in reverse), 64 columns of a state per workgroup, wave w rows 32 w ..
// + 31.  The columns of a state are independent, so with enough sequences (WALK) one
// workgroup carries its columns through every chunk and no combine is needed; with
// few, every chunk's own contribution is formed in parallel (chunk c0 + blockIdx.z) and
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
    auto chunk_of = [&](int it) { return WALK ? (ADJ ? p.nc - 1 - it : it) : w.c0 + (int)blockIdx.z; };
    auto fetch_tok = [&](int it) {
        const int c = chunk_of(it);
        const TokRows<Tin> tr(tok, first_row(p, b) + c * kTC, hd, p.H, D, min(Tb - c * kTC, kTC));
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
    // the state after the last token (out, and against dK_T / dV_T), or the initial state's
    // gradient
    double fin = 0.0;
    if (gext || (!ADJ && fext))
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            __builtin_amdgcn_sched_barrier(0);
            const int i = 32 * wv + 8 * (r >> 2) + 4 * h + (r & 3), ip = internal_to_paper(i, m);
            const size_t at = ((size_t)bh * kR + paper_row(i, m)) * D + 64 * cb + l31;
            if (gext) {
                gext[at] = ip >= 0 ? acc[0][r] : 0.f;
                gext[at + 32] = ip >= 0 ? acc[1][r] : 0.f;
            }
            if (!ADJ && fext && ip >= 0) {
                fin += (double)fext[at] * acc[0][r];
                fin += (double)fext[at + 32] * acc[1][r];
            }
        }
    if (!ADJ && p.fin) {
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

// clock_out, from a sequence's first workgroup of a launch after the tables'
__device__ __forceinline__ void clock_to_caller(const F32Ws &w, int bh) {
    if (w.clko && blockIdx.y == 0 && threadIdx.x == 0) w.clko[bh] = w.clkT[bh];
}

template <int DK, int DV, typename Tin, bool ADJ, bool WALK>
__global__ __launch_bounds__(256, 4) void f32_states_kernel(BwdParams p, F32Ws w) {
    __shared__ __attribute__((aligned(16))) float lds[kTC * kLS + kTC + 4 * kLdsTile];
    const int y = blockIdx.y;
    if (y < DK / 64)
        state_columns<DK, Tin, ADJ, WALK>(p, w, ADJ ? p.q : p.k, ADJ ? p.dP : w.cs, ADJ ? w.DKe : w.Kst,
                                          ADJ ? p.dK_T : p.K0, p.dK_T, ADJ ? p.gK0 : w.Ko, y, lds);
    else
        state_columns<DV, Tin, ADJ, WALK>(p, w, ADJ ? p.dout : p.v, ADJ ? p.U : w.cs, ADJ ? w.DVe : w.Vst,
                                          ADJ ? p.dV_T : p.V0, p.dV_T, ADJ ? p.gV0 : w.Vo, y - DK / 64, lds);
    if (WALK && !ADJ) clock_to_caller(w, blockIdx.x);
}

// Combines the chunks' own contributions in place, element by element: slot c becomes
// the state entering chunk c (the adjoint at its end, in reverse).  Sixteen chunks'
// loads are in flight at a time; only the multiply-add is a chain.  The first half of a
// sequence's workgroups takes the key state, the second the value state.
template <int DK, int DV, bool ADJ>
__global__ __launch_bounds__(256) void f32_scan_kernel(BwdParams p, F32Ws w) {
    __shared__ double red[4];
    constexpr int kHalf = kBwdFinParts / 2;
    const int bh = blockIdx.x, tid = threadIdx.x, m = p.m, nc = p.nc;
    const float *ge = w.gend + (size_t)bh * nc;
    double fin = 0.0;
    auto run = [&](int D, float *slots, const float *ext, const float *fext, float *gext) {
        const size_t st = (size_t)kR * D / 4;
        for (int e = (blockIdx.y % kHalf) * 256 + tid; e < kR * D / 4; e += 256 * kHalf) {
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
            for (int c0 = 0; c0 < nc; c0 += 16) {
                f32x4 own[16];
                float g[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    const int c = min(c0 + u, nc - 1), cc = ADJ ? nc - 1 - c : c;
                    own[u] = s[cc * st];
                    g[u] = ge[cc];
                }
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    if (c0 + u >= nc) break;
                    s[(ADJ ? nc - 1 - (c0 + u) : c0 + u) * st] = E;
#pragma unroll
                    for (int q = 0; q < 4; ++q) E[q] = fmaf(g[u], E[q], own[u][q]);
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int ip = internal_to_paper(i0 + q, m);
                if (gext) gext[((size_t)bh * kR + paper_row(i0 + q, m)) * D + ch] = ip >= 0 ? E[q] : 0.f;
                if (!ADJ && fext && ip >= 0) {
                    fin += (double)fext[ext_at(q)] * E[q];
                }
            }
        }
    };
    if (blockIdx.y < kHalf)
        run(DK, ADJ ? w.DKe : w.Kst, ADJ ? p.dK_T : p.K0, p.dK_T, ADJ ? p.gK0 : w.Ko);
    else
        run(DV, ADJ ? w.DVe : w.Vst, ADJ ? p.dV_T : p.V0, p.dV_T, ADJ ? p.gV0 : w.Vo);
    if (!ADJ) clock_to_caller(w, bh);
    if (ADJ || !p.fin) return;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) fin += __shfl_xor(fin, o);
    if ((tid & 63) == 0) red[tid >> 6] = fin;
    __syncthreads();
    if (tid == 0) p.fin[(size_t)bh * kBwdFinParts + blockIdx.y] = (red[0] + red[1]) + (red[2] + red[3]);
}

// U(sign lambda) of one block of basis rows; t = its phases
__device__ __forceinline__ f32x16 rotate_block(const f32x16 &x, const f32x16 &t, float sign, float mul) {
    f32x16 y;
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
        const float c = t[r], s = sign * t[r + 1];
        y[r] = mul * (c * x[r] - s * x[r + 1]);
        y[r + 1] = mul * (s * x[r] + c * x[r + 1]);
    }
    return y;
}

// block row w of a 4 x 4-block matrix times four operand blocks in LDS, in two sums
__device__ __forceinline__ f32x16 row_product(const float *Mat, int w, const float *x, int lane4) {
    f32x16 a[4], s[2] = {};
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) a[kb] = ld_block(Mat + (4 * w + kb) * 1024 + lane4);
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) mma_step(s[kb >> 1], a[kb], ld_block(x + kb * 1024 + lane4));
    return s[0] + s[1];
}

template <int DK, int DV, typename Tin, bool ADJ>
void launch_states(const BwdParams &p, F32Ws w, hipStream_t s) {
    const int BH = p.B * p.H, ny = (DK + DV) / 64;
    if (BH * ny >= 256) {
        hipLaunchKernelGGL((f32_states_kernel<DK, DV, Tin, ADJ, true>), dim3(BH, ny), dim3(256), 0, s, p, w);
        return;
    }
    // (a grid's z axis holds 65535 blocks)
    for (w.c0 = 0; w.c0 < p.nc; w.c0 += 65535)
        hipLaunchKernelGGL((f32_states_kernel<DK, DV, Tin, ADJ, false>), dim3(BH, ny, min(p.nc - w.c0, 65535)), dim3(256), 0,
                           s, p, w);
    hipLaunchKernelGGL((f32_scan_kernel<DK, DV, ADJ>), dim3(BH, kBwdFinParts), dim3(256), 0, s, p, w);
}

// The (chunk, sequence) grids of the tables are flat: a grid's y and z hold 65535 blocks
// only, and a batch may have more sequences.
inline void launch_front(const BwdParams &p, const F32Ws &w, hipStream_t s) {
    const int BH = p.B * p.H, base = p.H * (kR / kPrepRows) + BH;
    const bool one = p.nc <= kTableChunks;
    hipLaunchKernelGGL(f32_prep_kernel, dim3(base + (one ? BH * p.nc : 0)), dim3(256), 0, s, p, w);
    if (!one) hipLaunchKernelGGL(f32_tables_kernel, dim3(p.nc * BH), dim3(256), 0, s, p, w);
}

inline size_t align_up(size_t x) { return (x + 255) / 256 * 256; }

}  // namespace
}  // namespace cyfa

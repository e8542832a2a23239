// fp32 forward on the fp32 matrix instructions (m <= 127, every head dimension, fp32 or
// bf16 inputs, fp32 arithmetic).
//
// Chunks of 64 tokens (App. B): the tables and the states entering every chunk as in the
// fp32 backward (cyfa_f32_common.h), then one workgroup per 32 tokens of a sequence for
// the whole chain
//   P = gamma (.) Q Kbar_c^T + (Q K^T (.) Gamma) A,  X = scale U(lambda) P,  W = softmax(M X),
//   u = U(-lambda) M^T W,  O = gamma (.) u Vbar_c + (u A^T (.) Gamma) V.
// Wave w holds the 32 basis rows (slots) 32 w .. + 31 of every intermediate for the 32
// tokens, in tiles with the tokens on the lanes (cyfa_tile_f32.h), and reads the other
// waves' rows from LDS as operand blocks.  The split over the four waves is for the small
// calls this path serves: a tile's chain of 72 (d = 64) steps of 16 instructions, 1024
// cycles each, becomes 24 steps and six barriers.  B 1, T 256, H 2, d 64 (fp32): 187 us
// with the vector-ALU chunk kernel (147 us of it that kernel), 38 us now (this kernel 22.8,
// the tables 8.9, the states 5.1 and their scan 3.4); bound by each tile's chain of products and barriers.
#include "cyfa_f32_common.h"
#include "cyfa_rows.h"

namespace cyfa {

namespace {

template <int DK, int DV, typename Tin>
__global__ __launch_bounds__(256, 2) void f32_forward_kernel(BwdParams p, F32Ws w, void *out, float *logits) {
    __shared__ __attribute__((aligned(16))) float xs[4096], ws[4096], part[4096], tiles[4 * kLdsTile];
    __shared__ float red[2][4][32];
    const int per_seq = (p.T + 31) / 32, tile = blockIdx.x % per_seq, bh = blockIdx.x / per_seq;
    const int c = tile >> 1, tb = tile & 1, b = bh / p.H, hd = bh % p.H;
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int l31 = lane & 31, h = lane >> 5, lane4 = 4 * lane, m = p.m;
    const int left = min(bwd_tokens(p, b) - c * kTC, kTC);
    if (left <= 32 * tb) return;                // none of these tokens exists
    const size_t grow = first_row(p, b) + c * kTC, row0 = (size_t)bh * p.Tpad + c * kTC;
    const int tl = 32 * tb + l31;
    const bool live = tl < left;
    const WriteCoef wc(m);
    const LdsTile swp(tiles + wv * kLdsTile, l31, h);
    const TokRows<Tin> q(p.q, grow, hd, p.H, DK, left), k(p.k, grow, hd, p.H, DK, left);
    const TokRows<Tin> v(p.v, grow, hd, p.H, DV, left);
    const float *cs = w.cs + row0 * kR + lane4;
    const double Gt = w.G[row0 + tl];
    const float g = w.gam[row0 + tl];
    // (q, k) score tiles: wave w the tile w % 2, every second 32 channels
    {
        f32x16 s = {};
        if ((wv & 1) <= tb)
            for (int kb = wv >> 1; kb < DK / 32; kb += 2)
                mma_step(s, k.wide_cvt(k.wide_raw(32 * (wv & 1) + l31, h, 32 * kb)), q.wide_cvt(q.wide_raw(tl, h, 32 * kb)));
        st_block(part + wv * 1024 + lane4, s);
    }
    // this wave's rows of the entering state
    f32x16 acc = {};
    {
        const float *St = w.Kst + (((size_t)bh * p.nc + c) * 4 + wv) * (DK / 32) * 1024 + lane4;
#pragma unroll 4
        for (int kb = 0; kb < DK / 32; ++kb)
            mma_step(acc, swp.template swap<true>(ld_block(St + kb * 1024)), q.wide_cvt(q.wide_raw(tl, h, 32 * kb)));
    }
    __syncthreads();
    f32x16 own = {};
    for (int sb = 0; sb <= tb; ++sb) {
        // A phase that is NaN (a non-finite delta) enters as -1, and beta goes to the masked
        // scores: tokens t < s have a zero score, which the product would multiply by the NaN.
        // The tokens t >= s get it from their own phases (delta) or their score (beta).
        f32x16 a = swp.template swap<false>(ld_block(cs + (4 * sb + wv) * 1024));
#pragma unroll
        for (int r = 0; r < 16; ++r) a[r] = fmaxf(a[r], -1.f) * wc.at(32 * wv + l31);
        f32x16 s = ld_block(part + sb * 1024 + lane4) + ld_block(part + (sb + 2) * 1024 + lane4);
        s = causal(s, Gt, w.G + row0 + 32 * sb + 4 * h, w.bet + row0 + 32 * sb + 4 * h, tl, 32 * sb, h);
        mma_step(own, a, s);
    }
    const f32x16 ph = ld_block(cs + (4 * tb + wv) * 1024);
    st_block(xs + wv * 1024 + lane4, rotate_block(acc * g + own, ph, 1.f, p.scale));
    __syncthreads();
    f32x16 z = row_product(w.Mi + (size_t)hd * kR * kR, wv, xs, lane4);
    if (logits && live) {
        float *zr = logits + ((grow + tl) * p.H + hd) * m;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int i = 32 * wv + 8 * (r >> 2) + 4 * h + (r & 3);
            if (i < m) zr[i] = z[r];
        }
    }
    // softmax over the m active slots; the weights are normalised after M^T
    {
        float mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (32 * wv + 8 * (r >> 2) + 4 * h + (r & 3) < m) mx = fmaxf(mx, z[r]);
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        if (h == 0) red[0][wv][l31] = mx;
    }
    __syncthreads();
    {
        const float mx = fmaxf(fmaxf(red[0][0][l31], red[0][1][l31]), fmaxf(red[0][2][l31], red[0][3][l31]));
#pragma unroll
        for (int r = 0; r < 16; ++r)
            z[r] = 32 * wv + 8 * (r >> 2) + 4 * h + (r & 3) < m ? __expf(z[r] - mx) : 0.f;
        const float sum = tree(z);
        if (h == 0) red[1][wv][l31] = sum;
        st_block(ws + wv * 1024 + lane4, z);
    }
    __syncthreads();
    const float inv = 1.f / ((red[1][0][l31] + red[1][1][l31]) + (red[1][2][l31] + red[1][3][l31]));
    const f32x16 u = rotate_block(row_product(w.MiT + (size_t)hd * kR * kR, wv, ws, lane4) * inv, ph, -1.f, 1.f);
    __syncthreads();                            // the weights have been read
    st_block(xs + wv * 1024 + lane4, u);
    // (u, a) score tiles, this wave's 32 of the 128 terms
    for (int sb = 0; sb <= tb; ++sb) {
        f32x16 s = {};
        mma_step(s, wc.apply(ld_block(cs + (4 * sb + wv) * 1024), wv, h), u);
        st_block((sb ? ws : part) + wv * 1024 + lane4, s);
    }
    __syncthreads();
    if (wv >= DV / 32) return;
    f32x16 s2[2];
#pragma unroll
    for (int sb = 0; sb < 2; ++sb) {
        if (sb > tb) break;
        const float *sp = (sb ? ws : part) + lane4;
        const f32x16 s = (ld_block(sp) + ld_block(sp + 1024)) + (ld_block(sp + 2048) + ld_block(sp + 3072));
        s2[sb] = causal(s, Gt, w.G + row0 + 32 * sb + 4 * h, w.bet + row0 + 32 * sb + 4 * h, tl, 32 * sb, h);
    }
    for (int cb = wv; cb < DV / 32; cb += 4) {
        const float *St = w.Vst + ((size_t)bh * p.nc + c) * kR * DV + cb * 1024 + lane4;
        f32x16 a[2] = {}, mine = {};
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) mma_step(a[kb >> 1], ld_block(St + kb * (DV / 32) * 1024), ld_block(xs + kb * 1024 + lane4));
#pragma unroll
        for (int sb = 0; sb < 2; ++sb) {
            if (sb > tb) break;
            const f32x16 y = v.cols_cvt(v.cols_raw(32 * sb, h, 32 * cb + l31));
            bool bad = false;
            if (sb == tb)
#pragma unroll
                for (int r = 0; r < 16; ++r) bad |= !(fabsf(y[r]) <= 3.4028235e38f);
            if (!__any(bad)) {
                mma_step(mine, y, s2[sb]);
                continue;
            }
            // an infinity or NaN of token s may reach tokens t >= s only: the matrix product
            // would multiply it by the zeros above the diagonal
#pragma unroll
            for (int s = 0; s < 32; ++s) {
                const float f = __shfl(s2[sb][4 * (s >> 3) + (s & 3)], l31 + 32 * ((s >> 2) & 1));
                const f32x16 row = v.rows(32 * sb + s, h, 32 * cb);
#pragma unroll
                for (int r = 0; r < 16; ++r) mine[r] = s <= l31 ? fmaf(f, row[r], mine[r]) : mine[r];
            }
        }
        const f32x16 o = (a[0] + a[1]) * g + mine;
        if (live) {
            Tin *row = static_cast<Tin *>(out) + ((grow + tl) * p.H + hd) * DV + 32 * cb + 4 * h;
#pragma unroll
            for (int qq = 0; qq < 4; ++qq) {
                if constexpr (sizeof(Tin) == 4) {
                    *reinterpret_cast<f32x4 *>(row + 8 * qq) = f32x4{o[4 * qq], o[4 * qq + 1], o[4 * qq + 2], o[4 * qq + 3]};
                } else {
                    mfma::bf16x4 y;
#pragma unroll
                    for (int e = 0; e < 4; ++e) y[e] = (__bf16)o[4 * qq + e];
                    *reinterpret_cast<mfma::bf16x4 *>(row + 8 * qq) = y;
                }
            }
        }
    }
}

template <int DK, int DV, typename Tin>
hipError_t launch_typed(const BwdParams &p, const F32Ws &w, void *out, float *logits, hipStream_t s) {
    launch_front(p, w, s);
    launch_states<DK, DV, Tin, false>(p, w, s);
    if (p.nc > 0)
        hipLaunchKernelGGL((f32_forward_kernel<DK, DV, Tin>), dim3((p.T + 31) / 32 * (p.B * p.H)), dim3(256), 0, s, p, w, out,
                           logits);
    return hipGetLastError();
}

template <int DK, int DV>
hipError_t launch_dtype(const BwdParams &p, const F32Ws &w, void *out, float *logits, hipStream_t s) {
    return p.dtype == 0 ? launch_typed<DK, DV, float>(p, w, out, logits, s)
                        : launch_typed<DK, DV, __hip_bfloat16>(p, w, out, logits, s);
}

template <int DK>
hipError_t launch_dv(const BwdParams &p, const F32Ws &w, void *out, float *logits, hipStream_t s) {
    if (p.dv == 64) return launch_dtype<DK, 64>(p, w, out, logits, s);
    if (p.dv == 128) return launch_dtype<DK, 128>(p, w, out, logits, s);
    return launch_dtype<DK, 256>(p, w, out, logits, s);
}

}  // namespace

size_t fwd_f32_workspace_bytes(const FwdParams &f) {
    const size_t BH = (size_t)f.B * f.H, nc = ((size_t)f.T + kTC - 1) / kTC, Tpad = nc * kTC;
    return align_up(2 * readout_f32_bytes(f.H)) + align_up(BH * nc * 8) + align_up(BH * 8) + align_up(BH * Tpad * kR * 4) +
           align_up(BH * Tpad * 8) + align_up(3 * BH * Tpad * 4) + align_up(BH * nc * 4) +
           align_up(BH * nc * kR * f.dk * 4) + align_up(BH * nc * kR * f.dv * 4);
}

hipError_t launch_fwd_f32(const FwdParams &f, void *ws, hipStream_t s) {
    BwdParams p{};
    p.B = f.B; p.T = f.T; p.H = f.H; p.dk = f.dk; p.dv = f.dv; p.m = f.m;
    p.nc = (f.T + kTC - 1) / kTC;
    p.Tpad = p.nc * kTC;
    p.scale = f.scale; p.dtype = f.dtype;
    p.q = f.q; p.k = f.k; p.v = f.v;
    p.delta = f.delta; p.log_alpha = f.log_alpha; p.beta = f.beta; p.R = f.R; p.lens = f.lens; p.cu = f.cu;
    p.K0 = f.K0; p.V0 = f.V0; p.clock0 = f.clock0;
    const size_t BH = (size_t)p.B * p.H, nc = p.nc, Tpad = p.Tpad;
    char *at = static_cast<char *>(ws);
    auto take = [&at](size_t bytes) { char *r = at; at += align_up(bytes); return reinterpret_cast<float *>(r); };
    F32Ws w{};
    w.Mi = take(2 * readout_f32_bytes(p.H));
    w.MiT = w.Mi + (size_t)p.H * kR * kR;
    w.clk = reinterpret_cast<double *>(take(BH * nc * 8));
    w.clkT = reinterpret_cast<double *>(take(BH * 8));
    w.cs = take(BH * Tpad * kR * 4);
    w.G = reinterpret_cast<double *>(take(BH * Tpad * 8));
    w.gam = take(3 * BH * Tpad * 4);
    w.wr = w.gam + BH * Tpad;
    w.bet = w.wr + BH * Tpad;
    w.gend = take(BH * nc * 4);
    w.Kst = take(BH * nc * kR * p.dk * 4);
    w.Vst = take(BH * nc * kR * p.dv * 4);
    w.Ko = f.K_out;
    w.Vo = f.V_out;
    w.clko = f.clock_out;
    if (p.dk == 64) return launch_dv<64>(p, w, f.o, f.logits, s);
    if (p.dk == 128) return launch_dv<128>(p, w, f.o, f.logits, s);
    return launch_dv<256>(p, w, f.o, f.logits, s);
}

}  // namespace cyfa

// The vector-ALU forward's chunk-group pre-pass (states entering each group) and the
// backward's last two kernels (reverse cumulative sums, dR).
#include <type_traits>

#include "cyfa_bwd.h"
#include "cyfa_mfma_common.h"   // wave-level prefix sums (DPP)

namespace cyfa {

namespace {

constexpr int kC = kBwdChunk;
constexpr int kNT = 512;            // threads per workgroup (two waves per SIMD)
constexpr int kRP = kNT / kStoreRows; // threads sharing one state row in the row layouts
constexpr int kRQ = kC * kStoreRows / kNT;   // token rows per thread in the readout products
constexpr int kReadoutThreads = kNT;           // the readout kernel (1024 measured slower: spills)
constexpr int kLD = kStoreRows + 4; // padded row of a [token][basis] tile (16-byte rows)
constexpr float kTwoPi = 6.283185307179586f;
constexpr int kCombBlocks = kBwdFinParts;   // workgroups per sequence of the group-combine kernels

__device__ __forceinline__ float wsum(float x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    return x;
}
__device__ __forceinline__ int bwd_tokens(const BwdParams &p, int b) {
    if (p.cu) return min(max(p.cu[b + 1] - p.cu[b], 0), p.T);
    return p.lens ? min(max(p.lens[b], 0), p.T) : p.T;
}
// first row of sequence b in the [rows, H, ...] tensors
__device__ __forceinline__ size_t brow0(const BwdParams &p, int b) {
    return p.cu ? (size_t)p.cu[b] : (size_t)b * p.T;
}

// Per-chunk scalar tables.
struct ChunkTab {
    double lam[kC];                 // clock after token r, reduced mod m
    float G[kC];                    // sum of log alpha over the chunk's tokens 0..r
    float beta[kC];
    float2 cs[kC][64];              // (cos, sin) of 2 pi j lam_r / m at [r][j-1]
};

// Loads the chunk's scalars (rows at or past the sequence's end: no shift, no
// decay, no write), forms the clock and log-decay prefix sums and the phase
// table.  Ends with a barrier.
template <int NT = kNT>
__device__ void chunk_tables(const BwdParams &p, int b, int h, int t0, int Tb, double lam_in,
                             ChunkTab &s, int tid) {
    if (tid < kC) {
        const int t = t0 + tid;
        const bool live = t < Tb;
        const size_t si = (brow0(p, b) + t) * p.H + h;
        s.lam[tid] = live ? (double)p.delta[si] : 0.0;
        s.G[tid] = (live && p.log_alpha) ? p.log_alpha[si] : 0.f;
        s.beta[tid] = live ? (p.beta ? p.beta[si] : 1.f) : 0.f;
    }
    __syncthreads();
    if (tid == 0) {
        double lam = lam_in;
        float G = 0.f;
        for (int r = 0; r < kC; ++r) {
            lam = reduce_clock(lam + s.lam[r], p.m);
            s.lam[r] = lam;
            G += s.G[r];
            s.G[r] = G;
        }
    }
    __syncthreads();
    const int J = (p.m - 1) / 2;
    for (int e = tid; e < kC * 64; e += NT) {
        const int r = e >> 6, jj = e & 63;
        float c = 1.f, sn = 0.f;
        if (jj < J) clock_phase(s.lam[r], jj + 1, p.m, &c, &sn);
        s.cs[r][jj] = make_float2(c, sn);
    }
    __syncthreads();
}

// Temporal write rows A_r = beta_r U(-lambda_r) b (Eq. app-temporal-writes).
__device__ __forceinline__ float write_entry(const ChunkTab &s, int m, int r, int i, float be) {
    if (i == 0) return be * (1.f / sqrtf((float)m));
    if (i >= m) return 0.f;
    const float ac = sqrtf(2.f / (float)m);
    const float2 cs = s.cs[r][(i - 1) >> 1];
    return (i & 1) ? be * ac * cs.x : -be * ac * cs.y;
}
template <typename Tin>
__device__ __forceinline__ float ld_row(const void *base, size_t row0, int t, int h, int c, int H, int D, bool live) {
    return live ? load_as_float(static_cast<const Tin *>(base), ((row0 + t) * H + h) * D + c) : 0.f;
}

// ---------------------------------------------------------------------------
// (1a) states entering every chunk from the chunk group's own tokens (the
// group starts from zero), per (sequence, group).  Thread t keeps column t % D
// of a state and its rows (t / D) NR .. + NR - 1 (NR = 128 D / threads), for the key
// state (D = d_k) and the value state (D = d_v): a wave shares its rows, so the
// write rows are broadcast reads and the stored state rows are coalesced.  The
// group's own final state goes to EcK/EcV[g], its total log decay to Gg.
template <int DK, int DV, typename Tin>
__global__ __launch_bounds__(kNT) void bwd_states_local_kernel(BwdParams p) {
    constexpr int NRK = DK * kStoreRows / kNT, NRV = DV * kStoreRows / kNT;
    __shared__ float Ks[kC][DK];
    __shared__ float Vs[kC][DV];
    __shared__ __attribute__((aligned(16))) float Aw[kC][kStoreRows];   // rho_r A_r
    __shared__ ChunkTab tab;
    __shared__ double dred[kNT];
    const int bh = blockIdx.x, g = blockIdx.y, b = bh / p.H, h = bh % p.H, tid = threadIdx.x;
    const int ck = tid % DK, rk = (tid / DK) * NRK;
    const int cv = tid % DV, rv = (tid / DV) * NRV;
    const int m = p.m;
    const int Tb = bwd_tokens(p, b);
    const int c_begin = g * p.cpg, c_end = min(c_begin + p.cpg, p.nc);
    // clock at the group's first token: lambda_0 plus the increments before it
    {
        const int t_start = min(c_begin * kC, Tb);
        double ds = 0.0;
        for (int t = tid; t < t_start; t += kNT) ds += (double)p.delta[(brow0(p, b) + t) * p.H + h];
        dred[tid] = ds;
        __syncthreads();
        for (int w = kNT / 2; w > 0; w >>= 1) {
            if (tid < w) dred[tid] += dred[tid + w];
            __syncthreads();
        }
    }
    double lam = reduce_clock((p.clock0 ? p.clock0[bh] : 0.0) + dred[0], m);
    if (p.gclk && tid == 0) p.gclk[(size_t)bh * p.groups + g] = lam;
    float kst[NRK], vst[NRV];
#pragma unroll
    for (int ii = 0; ii < NRK; ++ii) kst[ii] = 0.f;
#pragma unroll
    for (int ii = 0; ii < NRV; ++ii) vst[ii] = 0.f;
    float Gl = 0.f;
    for (int c = c_begin; c < c_end; ++c) {
        const int t0 = c * kC;
        if (p.Kst) {        // the forward's group pre-pass keeps only the group totals
            float *Kd = p.Kst + ((size_t)bh * p.nc + c) * kStoreRows * DK + ck;
            float *Vd = p.Vst + ((size_t)bh * p.nc + c) * kStoreRows * DV + cv;
#pragma unroll
            for (int ii = 0; ii < NRK; ++ii) Kd[(size_t)(rk + ii) * DK] = kst[ii];
#pragma unroll
            for (int ii = 0; ii < NRV; ++ii) Vd[(size_t)(rv + ii) * DV] = vst[ii];
            if (tid == 0) {
                p.clk[(size_t)bh * p.nc + c] = lam;
                p.Gin[(size_t)bh * p.nc + c] = Gl;
            }
        }
        for (int e = tid; e < kC * DK; e += kNT) {
            const int r = e / DK, cc = e % DK;
            Ks[r][cc] = ld_row<Tin>(p.k, brow0(p, b), t0 + r, h, cc, p.H, DK, t0 + r < Tb);
        }
        for (int e = tid; e < kC * DV; e += kNT) {
            const int r = e / DV, cc = e % DV;
            Vs[r][cc] = ld_row<Tin>(p.v, brow0(p, b), t0 + r, h, cc, p.H, DV, t0 + r < Tb);
        }
        chunk_tables(p, b, h, t0, Tb, lam, tab, tid);
        const float GC = tab.G[kC - 1], gC = __expf(GC);
        for (int e = tid; e < kC * kStoreRows; e += kNT) {
            const int r = e >> 7, i = e & 127;
            Aw[r][i] = write_entry(tab, m, r, i, tab.beta[r]) * __expf(GC - tab.G[r]);
        }
        __syncthreads();
#pragma unroll
        for (int ii = 0; ii < NRK; ++ii) kst[ii] *= gC;
#pragma unroll
        for (int ii = 0; ii < NRV; ++ii) vst[ii] *= gC;
#pragma unroll 1
        for (int r = 0; r < kC; ++r) {
            const float kr = Ks[r][ck], vr = Vs[r][cv];
#pragma unroll
            for (int ii = 0; ii < NRK; ++ii) kst[ii] = fmaf(Aw[r][rk + ii], kr, kst[ii]);
#pragma unroll
            for (int ii = 0; ii < NRV; ++ii) vst[ii] = fmaf(Aw[r][rv + ii], vr, vst[ii]);
        }
        lam = tab.lam[kC - 1];
        Gl += GC;
        __syncthreads();
    }
    float *Ko = p.EcK + ((size_t)bh * p.groups + g) * kStoreRows * DK + ck;
    float *Vo = p.EcV + ((size_t)bh * p.groups + g) * kStoreRows * DV + cv;
#pragma unroll
    for (int ii = 0; ii < NRK; ++ii) Ko[(size_t)(rk + ii) * DK] = kst[ii];
#pragma unroll
    for (int ii = 0; ii < NRV; ++ii) Vo[(size_t)(rv + ii) * DV] = vst[ii];
    if (tid == 0) p.Gg[(size_t)bh * p.groups + g] = Gl;
}

// (1b) states entering each group, per sequence, in group order:
// E_0 = (K0, V0), E_{g+1} = exp(Gg_g) E_g + (group g's own final state); EcK/EcV[g]
// are overwritten with E_g.  The final state gives <dK_T, Kbar_T> + <dV_T, Vbar_T>,
// the final-state term of dL/dG at the last token.
template <int DK, int DV>
__global__ __launch_bounds__(kNT) void bwd_states_combine_kernel(BwdParams p) {
    __shared__ float red[kNT / 64];
    const int bh = blockIdx.x, tid = threadIdx.x, m = p.m, G = p.groups;
    const int e0 = blockIdx.y * kNT + tid, es = kCombBlocks * kNT;
    const float *Gg = p.Gg + (size_t)bh * G;
    float acc = 0.f;
    for (int e = e0; e < kStoreRows * DK; e += es) {
        const bool act = e / DK < m;
        float E = (p.K0 && act) ? p.K0[(size_t)bh * kStoreRows * DK + e] : 0.f;
        for (int g = 0; g < G; ++g) {
            float *slot = p.EcK + ((size_t)bh * G + g) * kStoreRows * DK + e;
            const float own = *slot;
            *slot = E;
            E = fmaf(__expf(Gg[g]), E, own);
        }
        if (p.dK_T && act) acc = fmaf(p.dK_T[(size_t)bh * kStoreRows * DK + e], E, acc);
    }
    for (int e = e0; e < kStoreRows * DV; e += es) {
        const bool act = e / DV < m;
        float E = (p.V0 && act) ? p.V0[(size_t)bh * kStoreRows * DV + e] : 0.f;
        for (int g = 0; g < G; ++g) {
            float *slot = p.EcV + ((size_t)bh * G + g) * kStoreRows * DV + e;
            const float own = *slot;
            *slot = E;
            E = fmaf(__expf(Gg[g]), E, own);
        }
        if (p.dV_T && act) acc = fmaf(p.dV_T[(size_t)bh * kStoreRows * DV + e], E, acc);
    }
    acc = wsum(acc);
    if ((tid & 63) == 0) red[tid >> 6] = acc;
    __syncthreads();
    if (tid == 0) {
        float t = 0.f;
        for (int w = 0; w < kNT / 64; ++w) t += red[w];
        p.fin[(size_t)bh * kCombBlocks + blockIdx.y] = t;
    }
}

// ---------------------------------------------------------------------------
// (5) reverse cumulative sums per sequence: dlog_alpha_t = sum_{tau >= t} dG_tau
// (with the final-state term at the last token), ddelta_t = sum_{tau >= t}
// dlambda_tau, dclock0 = sum_t dlambda_t, all in double.  Workgroup (b h, piece)
// handles one of kScanPieces consecutive pieces of the sequence: it sums the tokens
// after its piece itself (loads batched eight per thread), and within the piece each
// thread sums its own run of tokens; the sum of the later runs is the piece total
// minus an inclusive prefix over the threads (wave prefix sums, then one offset per
// wave).  The thread that ends at token 0 holds the whole sum, dclock0.
constexpr int kScanPieces = 8;
__global__ __launch_bounds__(kNT) void bwd_scan_kernel(BwdParams p) {
    constexpr int kW = kNT / 64;
    __shared__ double sG[kW], sL[kW];
    const int bh = blockIdx.x, pc = blockIdx.y, b = bh / p.H, h = bh % p.H, tid = threadIdx.x, lane = tid & 63,
              wv = tid >> 6;
    const int Tb = bwd_tokens(p, b);
    const float *dG = p.dG + (size_t)bh * p.Tpad;
    const float *dl = p.dlam + (size_t)bh * p.Tpad;
    double fin = 0.0;
    for (int u = 0; u < kCombBlocks; ++u) fin += p.fin[(size_t)bh * kCombBlocks + u];
    const int pp = (Tb + kScanPieces - 1) / kScanPieces;
    const int P0 = min(pc * pp, Tb), P1 = min(P0 + pp, Tb);
    // tokens after the piece
    double lG = 0.0, lL = 0.0;
    for (int t0 = P1; t0 < Tb; t0 += 8 * kNT) {
        float vg[8], vl[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int t = t0 + u * kNT + tid;
            vg[u] = t < Tb ? dG[t] : 0.f;
            vl[u] = t < Tb ? dl[t] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            lG += vg[u];
            lL += vl[u];
        }
    }
    if (P1 < Tb && tid == 0) lG += fin;
    for (int o = 32; o > 0; o >>= 1) {
        lG += __shfl_xor(lG, o);
        lL += __shfl_xor(lL, o);
    }
    if (lane == 0) {
        sG[wv] = lG;
        sL[wv] = lL;
    }
    __syncthreads();
    double LG = 0.0, LL = 0.0;
#pragma unroll
    for (int u = 0; u < kW; ++u) {
        LG += sG[u];
        LL += sL[u];
    }
    __syncthreads();
    const int per = (P1 - P0 + kNT - 1) / kNT;
    const int t_lo = min(P0 + tid * per, P1), t_hi = min(t_lo + per, P1);
    double aG = 0.0, aL = 0.0;
    for (int t = t_lo; t < t_hi; ++t) {
        aG += (double)dG[t] + (t == Tb - 1 ? fin : 0.0);
        aL += dl[t];
    }
    const double iG = mfma::wave_incl_scan(aG), iL = mfma::wave_incl_scan(aL);
    if (lane == 63) {
        sG[wv] = iG;
        sL[wv] = iL;
    }
    __syncthreads();
    double oG = 0.0, oL = 0.0, TG = 0.0, TL = 0.0;
#pragma unroll
    for (int u = 0; u < kW; ++u) {
        if (u < wv) {
            oG += sG[u];
            oL += sL[u];
        }
        TG += sG[u];
        TL += sL[u];
    }
    double rg = LG + (TG - (oG + iG)), rl = LL + (TL - (oL + iL));   // sums over the later tokens
    for (int t = t_hi - 1; t >= t_lo; --t) {
        rg += (double)dG[t] + (t == Tb - 1 ? fin : 0.0);
        rl += dl[t];
        const size_t si = (brow0(p, b) + t) * p.H + h;
        if (p.glog_alpha) p.glog_alpha[si] = (float)rg;
        p.gdelta[si] = (float)rl;
    }
    if (pc == 0 && tid == 0 && p.gclock0) p.gclock0[bh] = rl;       // t_lo = 0: every token
    for (int t = Tb + pc * kNT + tid; t < p.T; t += kScanPieces * kNT) {
        const size_t si = (brow0(p, b) + t) * p.H + h;
        if (p.glog_alpha) p.glog_alpha[si] = 0.f;
        p.gdelta[si] = 0.f;
    }
}

// ---------------------------------------------------------------------------
// (6) dR_h = (sum over sequences b and chunk groups of dM) Phi^T on the active
// m x m block (M = R Phi, Phi the real Fourier basis of App. A.1).  Workgroup
// (h, row block) handles kDRRows rows of dR, which need the same rows of dM only.
constexpr int kDRRows = 8;
__global__ __launch_bounds__(kNT) void bwd_dR_kernel(BwdParams p, int nb) {
    __shared__ float dM[kDRRows][kLD];
    __shared__ float tab[2][kStoreRows];
    const int h = blockIdx.x, i0 = blockIdx.y * kDRRows, tid = threadIdx.x, m = p.m;
    for (int e = tid; e < kDRRows * kStoreRows; e += kNT) {
        const int ii = e >> 7, j = e & 127;
        float s[8] = {};                            // eight running sums, then a tree
        for (int u0 = 0; u0 < nb; u0 += 8) {
            float v[8];                             // eight loads in flight
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int u = u0 + k, b = u / p.groups, g = u % p.groups;
                v[k] = u < nb ? p.dMp[(((size_t)(b * p.H + h) * p.groups + g) * kStoreRows + i0 + ii) * kStoreRows + j]
                              : 0.f;
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) s[k] += v[k];
        }
        dM[ii][j] = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
    }
    if (tid < m) {
        double sn, cs;
        sincospi(2.0 * (double)tid / (double)m, &sn, &cs);
        tab[0][tid] = (float)cs;
        tab[1][tid] = (float)sn;
    }
    __syncthreads();
    const float dc = 1.f / sqrtf((float)m), ac = sqrtf(2.f / (float)m);
    for (int e = tid; e < kDRRows * m; e += kNT) {
        const int ii = e / m, s = e % m;
        if (i0 + ii >= m) continue;
        float acc = dM[ii][0] * dc;
        int n = 0;                                  // l s mod m, advanced by s per step
        for (int l = 1; 2 * l < m; ++l) {
            n += s;
            if (n >= m) n -= m;
            acc = fmaf(dM[ii][2 * l - 1], ac * tab[0][n], acc);
            acc = fmaf(dM[ii][2 * l], ac * tab[1][n], acc);
        }
        p.gR[((size_t)h * m + i0 + ii) * m + s] = acc;
    }
}

size_t align_up(size_t x) { return (x + 255) / 256 * 256; }

}  // namespace

hipError_t launch_bwd_tail(const BwdParams &p, int parts, hipStream_t s) {
    hipLaunchKernelGGL(bwd_scan_kernel, dim3(p.B * p.H, kScanPieces), dim3(kNT), 0, s, p);
    if (p.gR) hipLaunchKernelGGL(bwd_dR_kernel, dim3(p.H, kStoreRows / kDRRows), dim3(kNT), 0, s, p, parts);
    return hipGetLastError();
}

size_t group_states_bytes(int B, int H, int dk, int dv, int groups) {
    const size_t BH = (size_t)B * H;
    return align_up(BH * (size_t)groups * kStoreRows * (size_t)(dk + dv) * 4) +
           align_up(BH * (size_t)groups * 4) + align_up(BH * kCombBlocks * 8) +
           align_up(BH * (size_t)groups * 8);
}

hipError_t launch_group_states(const FwdParams &f, int groups, int cpg, void *ws, const float **EcK,
                               const float **EcV, const double **Eclk, hipStream_t s) {
    BwdParams p{};
    p.B = f.B; p.T = f.T; p.H = f.H; p.dk = f.dk; p.dv = f.dv; p.m = f.m;
    p.nc = (f.T + kC - 1) / kC;
    p.Tpad = p.nc * kC;
    p.groups = groups;
    p.cpg = cpg;
    p.scale = f.scale; p.dtype = f.dtype;
    p.q = f.q; p.k = f.k; p.v = f.v;
    p.delta = f.delta; p.log_alpha = f.log_alpha; p.beta = f.beta; p.lens = f.lens; p.cu = f.cu;
    p.K0 = f.K0; p.V0 = f.V0; p.clock0 = f.clock0;
    const size_t BH = (size_t)f.B * f.H;
    char *w = static_cast<char *>(ws);
    auto take = [&w](size_t bytes) { char *r = w; w += align_up(bytes); return r; };
    const size_t gcar = BH * (size_t)groups * kStoreRows;
    p.EcK = reinterpret_cast<float *>(take(gcar * (size_t)(f.dk + f.dv) * 4));
    p.EcV = p.EcK + gcar * f.dk;
    p.Gg = reinterpret_cast<float *>(take(BH * (size_t)groups * 4));
    p.fin = reinterpret_cast<double *>(take(BH * kCombBlocks * 8));
    p.gclk = reinterpret_cast<double *>(take(BH * (size_t)groups * 8));
    *EcK = p.EcK;
    *EcV = p.EcV;
    *Eclk = p.gclk;
    const dim3 block(kNT), grp(f.B * f.H, groups), comb(f.B * f.H, kCombBlocks);
    auto go = [&](auto dk_tag, auto dv_tag) {
        constexpr int DK = decltype(dk_tag)::value, DV = decltype(dv_tag)::value;
        if (f.dtype == 0) {
            hipLaunchKernelGGL((bwd_states_local_kernel<DK, DV, float>), grp, block, 0, s, p);
        } else {
            hipLaunchKernelGGL((bwd_states_local_kernel<DK, DV, __hip_bfloat16>), grp, block, 0, s, p);
        }
        hipLaunchKernelGGL((bwd_states_combine_kernel<DK, DV>), comb, block, 0, s, p);
    };
    using I64 = std::integral_constant<int, 64>;
    using I128 = std::integral_constant<int, 128>;
    if (f.dk == 64 && f.dv == 64) go(I64{}, I64{});
    else if (f.dk == 64) go(I64{}, I128{});
    else if (f.dv == 64) go(I128{}, I64{});
    else go(I128{}, I128{});
    return hipGetLastError();
}

}  // namespace cyfa

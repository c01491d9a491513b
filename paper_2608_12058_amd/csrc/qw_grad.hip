// Energy of a piecewise-constant anneal and its gradient by the adjoint of the
// matrix Clenshaw recurrence (complex64 forward, single-precision adjoint,
// double-precision reductions).
//
// Forward: psi_s = exp(-i t_s c) p_s(H~_s) psi_{s-1}, s = 1..S, with
// H~_s = (E - c)/r_s + (gamma_s/r_s) sum_j X_j and the Chebyshev coefficients
// of exp(-i a_s x), a_s = t_s r_s (Eq. cheb, Alg. 2).  Loss E = <psi_S|H_P|psi_S>.
//
// Reverse mode (derived from Eq. recursion; the paper has no gradient): with
// w = p(H~)v and adjoint ybar of the segment output,
//   beta_0 = conj(phase) ybar, beta_1 = H~ beta_0, beta_{k+1} = 2 H~ beta_k - beta_{k-1};
//   vbar = sum_k conj(c_k) beta_k                (adjoint of the segment input);
//   dL/dd~_i = sum_{k<K} w_k Re(conj(beta_k,i) b_{k+1,i}),  w_0 = 1, w_k = 2;
//   dL/dg~   = sum_{k<K} w_k Re<F beta_k, b_{k+1}>;
//   dL/dt    = sum_k Re(dc_k/dt <beta_k, v>) + Re(-i c <ybar, psi_s>),
//              dc_k/dt = r (-i)^k alpha_k'(a),
// with the shift c, bound r and degree K held fixed.  The b_k are recomputed
// per window of `ckpt_every` terms from checkpointed pairs stored during the
// forward sweep.  dE/dh, dE/dJ follow from G_i = sum_s dL/dd~_{s,i}/r_s +
// |psi_S,i|^2 by a Walsh-type reduction over the basis states.
#include "qw_kernels.h"
#include "qw_resident.h"

namespace qw {

static constexpr int GTB = Cfg<float>::TB;   // tile bits of the element-wise kernels
static constexpr int GNT = Cfg<float>::NT;

// Coefficients of one adjoint step k (see the file comment).
struct AdjStep {
    float scale, ckr, cki, gw;   // scale 2 (1 for k = 0), conj(c_k) applied to beta_k, w_k / r
    double wk, dcr, dci;         // w_k, r dc_k/da
};

struct AdjArgs {
    const float2 *beta;    // beta_k: its flips over the tile group are summed
    const float2 *prev;    // START: beta_{k-1} (NULL for k = 0); ADD, FUSED: partial beta_{k+1}
    float2 *dst;           // beta_{k+1}, partial or complete (may alias prev)
    float2 *dst2;          // FUSED: partial beta_{k+2} (may alias beta)
    const float2 *bnext;   // b_{k+1}
    const float2 *bnext2;  // FUSED: b_{k+2}
    const float2 *v;       // segment input
    float2 *vbar;          // accumulates conj(c_k) beta_k
    float *G;              // accumulates w_k/r Re(conj(beta_k) b_{k+1})
    const float *erel;     // E - c
    double *part;          // per block: [0] += Re(dc_k <beta_k, v>), [1] += w_k Re<F beta_k, b_{k+1}>
    double *part2;         // FUSED: the same for step k + 1
    float dscale, g;
    AdjStep st, st2;       // step k; FUSED: step k + 1
    int L, g0, h;
};

// Element arithmetic of the adjoint.  Every fused multiply-add is explicit and
// nothing else is contracted, so that all kernels round alike whatever the compiler
// makes of their surroundings.

// Re(dc conj(b) x) = dcr Re(conj(b) x) - dci Im(conj(b) x), added to dt.
__device__ __forceinline__ void dt_elem(double dcr, double dci, float2 b, float2 x, double &dt)
{
#pragma clang fp contract(off)
    const double bx = b.x, by = b.y, xx = x.x, xy = x.y;
    const double pr = fmad(bx, xx, by * xy), pi = fmad(bx, xy, -(by * xx));
    dt += fmad(dcr, pr, -(dci * pi));
}

// vbar += conj(c) b with conj(c) = (cr, -ci) given as c.
__device__ __forceinline__ void vbar_elem(float cr, float ci, float2 b, float2 &vb)
{
#pragma clang fp contract(off)
    vb.x += fmad(cr, b.x, ci * b.y);
    vb.y += fmad(cr, b.y, -(ci * b.x));
}

// The accumulations of step k that need beta_k alone (b = beta_k, bx = b_{k+1}, x = v).
__device__ __forceinline__ void adj_sums_elem(const AdjStep &s, float2 b, float2 bx, float2 x, float2 &vb, float &gg,
                                              double &dt)
{
    vbar_elem(s.ckr, s.cki, b, vb);
    gg = fmad(s.gw, fmad(b.x, bx.x, b.y * bx.y), gg);
    dt_elem(s.dcr, s.dci, b, x, dt);
}

// The first pass of step k: the start of beta_{k+1} (p = beta_{k-1}, (sr, si) =
// flips of beta_k over the pass's group).
__device__ __forceinline__ float2 adj_start_elem(const AdjStep &s, float dscale, float g, float er, float2 b,
                                                 float2 p, float2 bx, float sr, float si, double &dg)
{
#pragma clang fp contract(off)
    dg = fmad(s.wk, (double)fmad(sr, bx.x, si * bx.y), dg);
    const float d = er * dscale;
    return make_float2(fmad(s.scale, fmad(g, sr, d * b.x), -p.x), fmad(s.scale, fmad(g, si, d * b.y), -p.y));
}

// A later pass of step k: p = partial beta_{k+1}.
__device__ __forceinline__ float2 adj_add_elem(const AdjStep &s, float g, float2 p, float2 bx, float sr, float si,
                                               double &dg)
{
#pragma clang fp contract(off)
    dg = fmad(s.wk, (double)fmad(sr, bx.x, si * bx.y), dg);
    const float sg = s.scale * g;
    return make_float2(fmad(sg, sr, p.x), fmad(sg, si, p.y));
}

// beta_0 = conj(phase) ybar; ph += Im(conj(ybar) psi_s).
__device__ __forceinline__ float2 beta0_elem(float cr, float ci, float2 yb, float2 p, double &ph)
{
#pragma clang fp contract(off)
    ph += fmad((double)yb.x, (double)p.y, -((double)yb.y * p.x));
    return make_float2(fmad(cr, yb.x, -(ci * yb.y)), fmad(ci, yb.x, cr * yb.y));
}

// The last step: vbar += conj(c_K) beta_K, dt += Re(dc_K/dt conj(beta_K) v).
__device__ __forceinline__ void adj_last_elem(float cr, float ci, double dcr, double dci, float2 b, float2 x,
                                              float2 &vb, double &dt)
{
    vbar_elem(cr, ci, b, vb);
    dt_elem(dcr, dci, b, x, dt);
}

__device__ inline void block_add2(double x, double y, double *out)
{
    __shared__ double sx[64], sy[64];
    for (int o = 32; o > 0; o >>= 1) {
        x += __shfl_xor(x, o);
        y += __shfl_xor(y, o);
    }
    const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        sx[w] = x;
        sy[w] = y;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = 0.0, b = 0.0;
        for (int i = 0; i < nw; ++i) {
            a += sx[i];
            b += sy[i];
        }
        out[0] += a;
        out[1] += b;
    }
}

// One pass of the adjoint step k -> k+1 (see the file comment), on tiles of
// 2^TB amplitudes with NT threads (the shapes of the forward passes):
//  START: first orientation of step k (diagonal, flips, - beta_{k-1}, accumulations);
//  ADD:   a later orientation of step k;
//  FUSED: the last orientation of step k, then in the same orientation the
//         first of step k + 1 from the completed beta_{k+1} re-staged in LDS.
// The per-element arithmetic is the same in all three (adj_start_elem /
// adj_add_elem), so a step gives the same bits fused or not.
enum AdjMode { AM_START = 0, AM_ADD = 1, AM_FUSED = 2 };

template <int MODE, int TB, int NT, bool STREAM>
__global__ void __launch_bounds__(NT) k_adj_pass(AdjArgs a)
{
    using C = float2;
    using V = CVec<float>;
    constexpr int VE = V::N;
    constexpr int PER = (1 << TB) / (NT * VE);
    constexpr bool START = (MODE == AM_START);
    __shared__ C lds[1 << TB];
    const uint32_t TE = 1u << (a.L + a.h);
    const uint64_t base = tile_base(blockIdx.x, a.L, a.g0, a.h);
    V own[PER], pv[PER], bn[PER];
    V vv[START ? PER : 1], vb[START ? PER : 1];
    float er[START ? PER : 1][VE], gg[START ? PER : 1][VE];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const uint32_t e = (uint32_t)(q * NT + threadIdx.x) * VE;
        if (e < TE) {
            const uint64_t idx = tile_index(base, e, a.L, a.g0);
            own[q] = ld_v<float, STREAM>(a.beta + idx);
            if (a.prev) {
                pv[q] = ld_v<float, STREAM>(a.prev + idx);
            } else {
#pragma unroll
                for (int v = 0; v < VE; ++v) pv[q].v[v] = C{0.f, 0.f};
            }
            bn[q] = ld_v<float, STREAM>(a.bnext + idx);
            if constexpr (START) {
                vv[q] = ld_v<float, STREAM>(a.v + idx);
                vb[q] = ld_v<float, STREAM>(a.vbar + idx);
#pragma unroll
                for (int v = 0; v < VE; ++v) {
                    er[q][v] = a.erel[idx + v];
                    gg[q][v] = a.G[idx + v];
                }
            }
#pragma unroll
            for (int v = 0; v < VE; ++v) lds[e + v] = own[q].v[v];
        }
    }
    __syncthreads();
    auto flips = [&](uint32_t ee, float &sr, float &si) {
        sr = 0.f;
        si = 0.f;
        for (int j = 0; j < a.h; ++j) {
            const C nb = lds[ee ^ (1u << (a.L + j))];
            sr += nb.x;
            si += nb.y;
        }
    };
    double acc_dt = 0.0, acc_dg = 0.0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const uint32_t e = (uint32_t)(q * NT + threadIdx.x) * VE;
        if (e < TE) {
            const uint64_t idx = tile_index(base, e, a.L, a.g0);
            V out;
#pragma unroll
            for (int v = 0; v < VE; ++v) {
                float sr, si;
                flips(e + v, sr, si);
                if constexpr (START) {
                    adj_sums_elem(a.st, own[q].v[v], bn[q].v[v], vv[q].v[v], vb[q].v[v], gg[q][v], acc_dt);
                    out.v[v] = adj_start_elem(a.st, a.dscale, a.g, er[q][v], own[q].v[v], pv[q].v[v], bn[q].v[v], sr,
                                              si, acc_dg);
                } else
                    out.v[v] = adj_add_elem(a.st, a.g, pv[q].v[v], bn[q].v[v], sr, si, acc_dg);
            }
            if constexpr (MODE == AM_FUSED) {
                pv[q] = out;   // completed beta_{k+1}, kept for the second half
            } else {
                st_v<float, STREAM>(a.dst + idx, out);
                if constexpr (START) {
                    st_v<float, STREAM>(a.vbar + idx, vb[q]);
#pragma unroll
                    for (int v = 0; v < VE; ++v) a.G[idx + v] = gg[q][v];
                }
            }
        }
    }
    block_add2(acc_dt, acc_dg, a.part + 2 * blockIdx.x);
    if constexpr (MODE == AM_FUSED) {
        // second half: step k + 1 from the completed beta_{k+1} (pv) with
        // beta_k (own) as the subtracted vector
        __syncthreads();
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const uint32_t e = (uint32_t)(q * NT + threadIdx.x) * VE;
            if (e < TE) {
#pragma unroll
                for (int v = 0; v < VE; ++v) lds[e + v] = pv[q].v[v];
            }
        }
        __syncthreads();
        double dt2 = 0.0, dg2 = 0.0;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const uint32_t e = (uint32_t)(q * NT + threadIdx.x) * VE;
            if (e < TE) {
                const uint64_t idx = tile_index(base, e, a.L, a.g0);
                const V bx = ld_v<float, STREAM>(a.bnext2 + idx);
                const V x = ld_v<float, STREAM>(a.v + idx);
                V vbq = ld_v<float, STREAM>(a.vbar + idx);
                V out;
#pragma unroll
                for (int v = 0; v < VE; ++v) {
                    float sr, si;
                    flips(e + v, sr, si);
                    float gq = a.G[idx + v];
                    adj_sums_elem(a.st2, pv[q].v[v], bx.v[v], x.v[v], vbq.v[v], gq, dt2);
                    out.v[v] = adj_start_elem(a.st2, a.dscale, a.g, a.erel[idx + v], pv[q].v[v], own[q].v[v],
                                              bx.v[v], sr, si, dg2);
                    a.G[idx + v] = gq;
                }
                st_v<float, STREAM>(a.dst + idx, pv[q]);
                st_v<float, STREAM>(a.dst2 + idx, out);
                st_v<float, STREAM>(a.vbar + idx, vbq);
            }
        }
        __syncthreads();   // block_add2's shared sums are reused
        block_add2(dt2, dg2, a.part2 + 2 * blockIdx.x);
    }
}

// Element-wise kernels over tiles of 2^GTB consecutive amplitudes (TE = min(N, 2^GTB)).
struct EwArgs {
    const float2 *x;      // k_adj_last: beta_K;  k_seed: psi_S;  k_beta0: ybar (= vbar buffer)
    const float2 *v;      // k_adj_last: v;  k_beta0: psi_s (segment output)
    float2 *y;            // k_adj_last: vbar;  k_seed: vbar (receives ybar);  k_beta0: beta_0
    float2 *z;            // k_beta0: vbar (zeroed)
    float *G;             // k_seed: |psi_S|^2
    const float *erel;
    double *part;         // per block: [0], [1]
    double c;             // shift
    float cr, ci;         // k_adj_last: c_K;  k_beta0: conj(phase)
    double dcr, dci;      // k_adj_last: dc_K/dt
    uint32_t TE;
};

// vbar += conj(c_K) beta_K;  part[0] += Re(dc_K/dt <beta_K, v>).
__global__ void __launch_bounds__(256) k_adj_last(EwArgs a)
{
    const uint64_t base = (uint64_t)blockIdx.x * a.TE;
    double acc = 0.0;
    for (uint32_t e = threadIdx.x; e < a.TE; e += blockDim.x) {
        float2 vb = a.y[base + e];
        adj_last_elem(a.cr, a.ci, a.dcr, a.dci, a.x[base + e], a.v[base + e], vb, acc);
        a.y[base + e] = vb;
    }
    block_add2(acc, 0.0, a.part + 2 * blockIdx.x);
}

// ybar = 2 E psi_S into vbar, G = |psi_S|^2, part[0] += sum E |psi_S|^2.
__global__ void __launch_bounds__(256) k_seed(EwArgs a)
{
    const uint64_t base = (uint64_t)blockIdx.x * a.TE;
    double acc = 0.0;
    for (uint32_t e = threadIdx.x; e < a.TE; e += blockDim.x) {
        const float2 p = a.x[base + e];
        const double E = (double)a.erel[base + e] + a.c;
        const double m2 = (double)p.x * p.x + (double)p.y * p.y;
        acc += E * m2;
        a.y[base + e] = make_float2((float)(2.0 * E * p.x), (float)(2.0 * E * p.y));
        a.G[base + e] = (float)m2;
    }
    block_add2(acc, 0.0, a.part + 2 * blockIdx.x);
}

// beta_0 = conj(phase) ybar; vbar = 0; part[0] += c Im<ybar, psi_s> = Re(-i c <ybar, psi_s>).
__global__ void __launch_bounds__(256) k_beta0(EwArgs a)
{
    const uint64_t base = (uint64_t)blockIdx.x * a.TE;
    double acc = 0.0;
    for (uint32_t e = threadIdx.x; e < a.TE; e += blockDim.x) {
        a.y[base + e] = beta0_elem(a.cr, a.ci, a.x[base + e], a.v[base + e], acc);
        a.z[base + e] = make_float2(0.f, 0.f);
    }
    block_add2(a.c * acc, 0.0, a.part + 2 * blockIdx.x);
}

__global__ void k_zero_f64(double *p, int n)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0.0;
}

// Walsh reduction, stage 1: per tile of 2^LB amplitudes (high bits fixed),
//   W0 = sum G, W1_j = sum G s_j, W2_jk = sum G s_j s_k  (j < k < LB),
// combined with the tile's high-bit signs into partial dE/dh_j, dE/dJ_jk.
// The sums are those coefficients of a Walsh-Hadamard transform of the tile in
// double: 13 stages in three groups of register stages with the tile in LDS
// between them.  Bounded by those LDS passes and, from one tile to 128, by latency:
// 233 us with one thread per sum, 15 us now, at 20 qubits.
__global__ void __launch_bounds__(256) k_walsh_tile(const float *G, int n, int LB, double *out)
{
    static_assert(LB_TAB == 13, "three groups of at most five bits");
    constexpr int TW = 1 << LB_TAB, PER = TW / 256;
    __shared__ double g[TW + TW / 32];
    auto slot = [](uint32_t e) { return e + (e >> 5); };
    const uint32_t TE = 1u << LB, tid = threadIdx.x;
    const uint64_t hi = blockIdx.x;
    const uint64_t base = hi << LB;
    for (uint32_t e = tid; e < TW; e += 256) g[slot(e)] = e < TE ? (double)G[base + e] : 0.0;   // more bits: sums unchanged
    __syncthreads();
    double x[PER];
    auto stages = [&](int first, auto place) {   // x[r] = element place(r); bits of r from `first` up
#pragma unroll
        for (int r = 0; r < PER; ++r) x[r] = g[slot(place(r))];
#pragma unroll
        for (int b = 0; (1 << b) < PER; ++b) {
            if (b < first) continue;
#pragma unroll
            for (int r = 0; r < PER; ++r)
                if (!((r >> b) & 1)) {
                    const double u = x[r], v = x[r | (1 << b)];
                    x[r] = u + v;
                    x[r | (1 << b)] = u - v;
                }
        }
#pragma unroll
        for (int r = 0; r < PER; ++r) g[slot(place(r))] = x[r];
        __syncthreads();
    };
    stages(0, [&](uint32_t r) { return tid << 5 | r; });
    stages(0, [&](uint32_t r) { return (tid >> 5) << 10 | r << 5 | (tid & 31); });
    stages(2, [&](uint32_t r) { return r << 8 | tid; });
    const double W0 = g[0];
    auto w1 = [&](int j) { return g[slot(1u << j)]; };
    auto w2 = [&](int j, int k) { return g[slot(1u << j | 1u << k)]; };
    const int npar = n + n * (n - 1) / 2;
    double *o = out + (size_t)blockIdx.x * npar;
    auto shi = [&](int j) { return ((hi >> (j - LB)) & 1) ? -1.0 : 1.0; };
    for (int p = threadIdx.x; p < npar; p += blockDim.x) {
        double val;
        if (p < n) {
            val = (p < LB) ? w1(p) : shi(p) * W0;
        } else {
            int r = p - n, j = 0;
            while (r >= n - 1 - j) { r -= n - 1 - j; ++j; }
            const int k = j + 1 + r;
            if (k < LB) val = w2(j, k);
            else if (j < LB) val = shi(k) * w1(j);
            else val = shi(j) * shi(k) * W0;
        }
        o[p] = val;
    }
}

// Stage 2: column sums over tiles, one block per parameter.
__global__ void __launch_bounds__(256) k_walsh_reduce(const double *in, int ntiles, int npar, double *res)
{
    double acc = 0.0;
    for (int t = threadIdx.x; t < ntiles; t += blockDim.x) acc += in[(size_t)t * npar + blockIdx.x];
    __shared__ double s[256];
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) s[threadIdx.x] += s[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) res[blockIdx.x] = s[0];
}

// ---------------------------------------------------------------------------
// The sweeps in one launch each
// ---------------------------------------------------------------------------

static constexpr int GRES_NMIN = 8, GRES_NMAX = 20;
static constexpr int GRES_MAXW = 256;      // workgroups of a launch
static constexpr uint64_t GRES_NONE = ~uint64_t(0);

struct GradSeg {
    float inv_r, g, ph_r, ph_i;
    int K, coef;           // degree, place of c_0 .. c_K (and dc_k, and where b_k goes)
    int win, nwin;         // its windows in the list
};
struct GradWin {
    int B, T;              // b_B .. b_T
    int fresh;             // 1: recomputed from b_K = c_K v, 0: from x1, x2, -1: stored by the forward sweep
    int pad;
    uint64_t x1, x2, at;   // byte offsets in the workspace: b_{T+1}, b_{T+2} (GRES_NONE: zero), b_B
};

struct GradRes {
    char *ws;
    float2 *states;            // psi_s of the launch's first segment; psi_{s+1} .. behind it
    float2 *X0, *X1;           // exchange buffers
    float2 *vbar;
    float *G;
    const float *erel;
    const GradSeg *seg;        // of the launch's first segment
    const GradWin *win;
    const float2 *coef;        // c_k
    const double2 *dcoef;      // r dc_k/da
    const uint64_t *place;     // byte offset of b_k, GRES_NONE: an exchange buffer
    double *part;              // per segment and workgroup: dt, dgamma, phase sums
    int *start, *flags;        // 2 and RES_MAXFLAGS lines, cleared before the launch
    double c;
    int nseg;
    int stride, sel;           // workgroups with blockIdx.x % stride == sel take part
    int polls;                 // looks at a flag before giving up on a partner
};

// One sweep over all segments by W = 2^HC workgroups that hold one tile of 2^T
// consecutive amplitudes each: the two vectors of the recurrence and, in the
// backward sweep, beta_k and beta_{k-1} in registers, psi, vbar and G of the
// backward sweep in LDS (in registers as well they spilled: 14.9 ms for the call
// below).  Per term only b_{k+1} (beta_k) travels between the workgroups, as in
// k_resident, whose exchange, flags and flips these are.  The launch is
// cooperative, so every wait ends.  The vectors that the backward sweep needs again
// are exchange buffers themselves: b_k is written to the place where it is to stay.
// The sums over beta_k alone are formed while its flags travel.
//
// Every sum has the operands and the order of the passes: an element's flips are
// summed in increasing bit order in two groups, the tile and HA cross bits (up to
// bit 12 or 13) and, from 14 qubits, the HB bits above, and term by term the groups
// take turns in coming first.  So states, b_k, beta_k, vbar and G are those of the
// passes bit for bit (dt and dgamma add their doubles in another order).  The
// rounding of the forward states is most of the error of dE/dt, which another
// order would redraw.
//
// What bounds it: as in k_resident, the round trip of an exchange, and from 18
// qubits the exchanged bytes: 20 qubits take 6.6 us per term forwards and 13.6
// backwards (b_k again and an adjoint step), where the passes took 9.8 and 28.5.
template <int T, int NT, int HC, bool BACK> __global__ void __launch_bounds__(NT) k_grad_resident(GradRes a)
{
    using C = float2;
    using V = CVec<float>;
    constexpr int VE = V::N;
    constexpr int PER = (1 << T) / (NT * VE);
    constexpr int LT = (NT == 1024) ? 10 : (NT == 512) ? 9 : (NT == 256) ? 8 : (NT == 128) ? 7 : 6;
    constexpr int QB = (PER == 8) ? 3 : (PER == 4) ? 2 : (PER == 2) ? 1 : 0;
    static_assert((1 << LT) == NT && PER >= 1 && (1 << QB) == PER, "tile shape");
    constexpr int n = T + HC, W = 1 << HC, NW = NT / 64;
    constexpr int HB = (n > GTB) ? n - TB_NARROW : 0, HA = HC - HB;   // cross bits of the two groups
    static_assert(W * NW <= RES_MAXFLAGS && HA >= 0, "one flag per wave");
    constexpr int SC1 = 16;   // cache policy: past the L1, and (stores) through to memory
    constexpr int BYTES = (int)(sizeof(C) << n);
    __shared__ V lds[2][PER * NT];
    __shared__ int go;
    __shared__ double red[BACK ? NW : 1][3];
    // backward: vbar and G, each thread's own; a term needs them only while it waits
    __shared__ V vbl[BACK ? PER * NT : 1];
    __shared__ C ggl[BACK ? PER * NT : 1];
    __shared__ V psl[BACK ? PER * NT : 1];   // and v

    int w = 0;
    if constexpr (HC > 0) {
        if ((int)(blockIdx.x % a.stride) != a.sel) return;
        w = __builtin_amdgcn_readfirstlane(blockIdx.x / a.stride);
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    bool near = false, lost = false;
    if constexpr (HC > 0) {
        if (tid == 0) {
            const int xcc = __builtin_amdgcn_s_getreg(20 | (3 << 11));   // HW_REG_XCC_ID, 4 bits
            (void)__hip_atomic_fetch_or(a.start + RES_LINE, 1 << xcc, __ATOMIC_RELAXED, QW_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            int id;
            const bool ok = res_join(a.start, W, RES_POLLS, &id) == 1;
            const int m = __hip_atomic_load(a.start + RES_LINE, __ATOMIC_RELAXED, QW_AGENT);
            go = !ok ? 0 : (m & (m - 1)) == 0 ? 2 : 1;
        }
        __syncthreads();
        const int ok = __builtin_amdgcn_readfirstlane(go);
        near = (ok == 2);
        lost = (ok == 0);
    }

    const uint32_t base = (uint32_t)w << T;
    auto at = [&](int q) { return base + (uint32_t)(q * NT + tid) * VE; };
    auto rsrc = [&](const void *p) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, BYTES, 0x00027000); };
    auto own = [&](const void *p, int q) {   // a vector of this tile that the launch may have written
        return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(rsrc(p), (q * NT + tid) * 16,
                                                                            (int)(base * sizeof(C)), SC1));
    };
    auto keep = [&](const V (&x)[PER], void *p) {
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const qw_i4 y = __builtin_bit_cast(qw_i4, x[q]);
            const int vo = (q * NT + tid) * 16, so = (int)(base * sizeof(C));
            if (near) __builtin_amdgcn_raw_buffer_store_b128(y, rsrc(p), vo, so, 0);
            else __builtin_amdgcn_raw_buffer_store_b128(y, rsrc(p), vo, so, SC1);
        }
    };
    const int *peer = a.flags + (size_t)(((w ^ (lane < HC ? 1 << lane : 0)) * NW + wave) * RES_LINE);
    int *mine = a.flags + (size_t)((w * NW + wave) * RES_LINE);
    int t = 0;
    auto ring = [&]() -> void * { return (t & 1) ? a.X0 : a.X1; };   // of the next round
    // x to the LDS tile and to p, where its partners look for it (there already
    // unless `store`)
    auto publish = [&](const V (&x)[PER], void *p, bool store) {
        ++t;
        if (HC > 0 || BACK)
            if (store) keep(x, p);
#pragma unroll
        for (int q = 0; q < PER; ++q) lds[t & 1][q * NT + tid] = x[q];
        if constexpr (HC > 0) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the wave's part has arrived
            if (lane == 0) __hip_atomic_store(mine, t, __ATOMIC_RELAXED, QW_AGENT);
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    };
    auto add = [](V &s, const V &y) {
#pragma unroll
        for (int v = 0; v < VE; ++v) {
            s.v[v].x += y.v[v].x;
            s.v[v].y += y.v[v].y;
        }
    };
    GradSeg sg{};
    // Flips of the published x, whose other tiles are at p, handed to elem(q, the
    // first group's sum, the second's).  The partners' vectors of QG of a thread's
    // own are under way at a time: with two or four instead of one of its four, 20
    // qubits spilled in the terms (16 segments in 12.6 and 13.0 ms against 12.1).
    constexpr int QG = (PER > 2) ? 1 : PER;
    auto flips = [&](const V (&x)[PER], const void *p, auto elem) {
        V sa[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            sa[q].v[0] = x[q].v[1];
            sa[q].v[1] = x[q].v[0];
            add(sa[q], lane_flip<float, 0xb1>(x[q]));    // quad_perm 1 0 3 2
            add(sa[q], lane_flip<float, 0x4e>(x[q]));    // quad_perm 2 3 0 1
            add(sa[q], lds[t & 1][q * NT + (tid ^ 4)]);
            add(sa[q], lane_flip<float, 0x128>(x[q]));   // row_ror 8
#pragma unroll
            for (int j = 4; j < LT; ++j) add(sa[q], lds[t & 1][q * NT + (tid ^ (1 << j))]);
#pragma unroll
            for (int j = 0; j < QB; ++j) add(sa[q], x[q ^ (1 << j)]);
            if (PER > QG && (q + 1) % QG == 0) __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (HC > 0) {
            if (!lost) {
                int left = a.polls;
                while (__any(lane < HC && __hip_atomic_load(peer, __ATOMIC_RELAXED, QW_AGENT) < t))
                    if (--left <= 0) { lost = true; break; }
            }
            if (lost) sg.g = NAN;   // as in k_resident: no finite number is a wrong one
            asm volatile("" ::: "memory");
        }
        const auto rs = rsrc(p);
#pragma unroll
        for (int q0 = 0; q0 < PER; q0 += QG) {
            V y[QG][HC > 0 ? HC : 1], sb[QG];
#pragma unroll
            for (int q = 0; q < QG; ++q)
#pragma unroll
                for (int j = 0; j < HC; ++j) {
                    const int so = (int)((((uint32_t)w ^ (1u << j)) << T) * sizeof(C));
                    y[q][j] = __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(rs, ((q0 + q) * NT + tid) * 16,
                                                                                          so, SC1));
                }
#pragma unroll
            for (int q = 0; q < QG; ++q) {
#pragma unroll
                for (int v = 0; v < VE; ++v) sb[q].v[v] = C{0.f, 0.f};
#pragma unroll
                for (int j = 0; j < HC; ++j) add(j < HA ? sa[q0 + q] : sb[q], y[q][j]);
                elem(q0 + q, sa[q0 + q], sb[q]);
            }
            if (PER > QG) __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto lane32 = [](float x, int l) {
        return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), l));
    };
    auto lane64 = [](uint64_t u, int l) {
        return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l) << 32) |
               (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, l);
    };

    V ps[BACK ? 1 : PER];     // v
    auto v_of = [&](int q) -> V {
        if constexpr (BACK) return psl[q * NT + tid];
        else return ps[q];
    };
    float er[PER][VE];        // E - c
#pragma unroll
    for (int q = 0; q < PER; ++q)
#pragma unroll
        for (int v = 0; v < VE; ++v) er[q][v] = a.erel[at(q) + v];

    C ck{0.f, 0.f};           // lane l: c_{64 i + l}
    double dx = 0.0, dy = 0.0;
    uint64_t pl = 0;
    // c_k, dc_k (backward) and the places of b_k (forward) of k's 64
    auto load_terms = [&](int k, bool derivs) {
        const int i = (k & ~63) + lane;
        if (i <= sg.K) {
            ck = a.coef[sg.coef + i];
            if constexpr (!BACK) pl = a.place[sg.coef + i];
            else if (derivs) {
                const double2 d = a.dcoef[sg.coef + i];
                dx = d.x;
                dy = d.y;
            }
        }
    };
    // b_K = c_K v and b_{K+1} = 0
    auto fresh_start = [&](V (&b1)[PER], V (&b2)[PER]) {
#pragma clang fp contract(off)
        const float cr = lane32(ck.x, sg.K & 63), ci = lane32(ck.y, sg.K & 63);
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const V x = v_of(q);
#pragma unroll
            for (int v = 0; v < VE; ++v) {
                const C p = x.v[v];
                b1[q].v[v] = C{fmad(cr, p.x, -(ci * p.y)), fmad(cr, p.y, ci * p.x)};
                b2[q].v[v] = C{0.f, 0.f};
            }
        }
    };
    // b_k over b_{k+2} (b2) from the published b_{k+1} (b1)
    auto term = [&](int k, const V (&b1)[PER], V (&b2)[PER], const void *p) {
        if ((k & 63) == 63) load_terms(k, false);
        const float cr = lane32(ck.x, k & 63), ci = lane32(ck.y, k & 63);
        const float scale = (k == 0) ? 1.f : 2.f, sgg = scale * sg.g;
        const bool low = HB == 0 || ((sg.K - 1 - k) & 1) == 0;   // the low group first
        flips(b1, p, [&](int q, const V &sa, const V &sb) {
#pragma clang fp contract(off)
            const V pv = v_of(q);
#pragma unroll
            for (int v = 0; v < VE; ++v) {
                const C b = b1[q].v[v], s = b2[q].v[v], x = pv.v[v];
                const C f1 = low ? sa.v[v] : sb.v[v], f2 = low ? sb.v[v] : sa.v[v];
                const float d = er[q][v] * sg.inv_r;
                const float hr = fmad(d, b.x, sg.g * f1.x), hi = fmad(d, b.y, sg.g * f1.y);
                const float tr = fmad(scale, hr, -s.x), ti = fmad(scale, hi, -s.y);
                C o{tr + fmad(cr, x.x, -(ci * x.y)), ti + fmad(cr, x.y, ci * x.x)};
                if constexpr (HB > 0) o = C{fmad(sgg, f2.x, o.x), fmad(sgg, f2.y, o.y)};
                b2[q].v[v] = o;
            }
        });
    };
    auto swap = [](V (&x)[PER], V (&y)[PER]) {
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const V z = x[q];
            x[q] = y[q];
            y[q] = z;
        }
    };
    const uint64_t N = uint64_t(1) << n;

    if constexpr (!BACK) {
#pragma unroll
        for (int q = 0; q < PER; ++q) ps[q] = ld_v<float, false>(a.states + at(q));
        for (int i = 0; i < a.nseg; ++i) {
            sg = wave_uniform(a.seg[i]);
            load_terms(sg.K, false);
            V b1[PER], b2[PER];
            auto place = [&](int k) -> void * {
                const uint64_t o = lane64(pl, k & 63);
                return o == GRES_NONE ? ring() : a.ws + o;
            };
            auto send = [&](int k) -> void * {   // b_k = b1
                void *p = place(k);
                if (HC == 0 && lane64(pl, k & 63) != GRES_NONE) keep(b1, p);
                publish(b1, p, true);
                return p;
            };
            fresh_start(b1, b2);
            const void *p = send(sg.K);
            for (int k = sg.K - 1; k >= 0; --k) {
                term(k, b1, b2, p);
                swap(b1, b2);
                if (k > 0) p = send(k);
            }
#pragma unroll
            for (int q = 0; q < PER; ++q) {
#pragma unroll
                for (int v = 0; v < VE; ++v) {
                    const C y = b1[q].v[v];
                    ps[q].v[v] = C{fmad(sg.ph_r, y.x, -(sg.ph_i * y.y)), fmad(sg.ph_r, y.y, sg.ph_i * y.x)};
                    if (lost) ps[q].v[v] = C{NAN, NAN};
                }
                st_v<float, false>(a.states + (i + 1) * N + at(q), ps[q]);
            }
        }
    } else {
        V be[PER], bp[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            vbl[q * NT + tid] = ld_v<float, false>(a.vbar + at(q));
            ggl[q * NT + tid] = C{a.G[at(q)], a.G[at(q) + 1]};
        }
        for (int i = a.nseg - 1; i >= 0; --i) {
            sg = wave_uniform(a.seg[i]);
            double sdt = 0.0, sdg = 0.0, sph = 0.0;
            // beta_0 = conj(phase) ybar
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                const V y = ld_v<float, false>(a.states + (i + 1) * N + at(q));
                const V yb = vbl[q * NT + tid];
                psl[q * NT + tid] = ld_v<float, false>(a.states + i * N + at(q));
#pragma unroll
                for (int v = 0; v < VE; ++v) {
                    be[q].v[v] = beta0_elem(sg.ph_r, -sg.ph_i, yb.v[v], y.v[v], sph);
                    bp[q].v[v] = C{0.f, 0.f};
                }
                vbl[q * NT + tid] = bp[q];
            }
            for (int j = 0; j < sg.nwin; ++j) {
                const GradWin wn = wave_uniform(a.win[sg.win + j]);
                char *const win = a.ws + wn.at;
                auto wat = [&](int k) -> void * { return win + (uint64_t)(k - wn.B) * N * sizeof(C); };
                if (wn.fresh >= 0) {   // b_T .. b_B again
                    V b1[PER], b2[PER];
                    const int k0 = wn.fresh ? sg.K - 1 : wn.T;
                    load_terms(wn.fresh ? sg.K : k0, false);
                    const void *p;
                    if (wn.fresh) {
                        fresh_start(b1, b2);
                        p = wat(sg.K);
                        // every round is waited for by its partners before the next but
                        // one writes its buffer, so none is begun that nobody reads
                        if (k0 >= wn.B) publish(b1, wat(sg.K), true);
                        else keep(b1, wat(sg.K));
                    } else {
                        p = a.ws + wn.x1;
#pragma unroll
                        for (int q = 0; q < PER; ++q) {
                            b1[q] = own(p, q);
                            if (wn.x2 != GRES_NONE) b2[q] = own(a.ws + wn.x2, q);
                            else
#pragma unroll
                                for (int v = 0; v < VE; ++v) b2[q].v[v] = C{0.f, 0.f};
                        }
                        publish(b1, nullptr, false);
                    }
                    for (int k = k0; k >= wn.B; --k) {
                        term(k, b1, b2, p);
                        swap(b1, b2);
                        p = wat(k);
                        if (k > wn.B) publish(b1, wat(k), true);
                        else keep(b1, wat(k));
                    }
                }
                load_terms(wn.B - 1, true);
                for (int k = wn.B - 1; k < wn.T; ++k) {
                    if ((k & 63) == 0) load_terms(k, true);
                    AdjStep st;
                    const double wk = (k == 0) ? 1.0 : 2.0;
                    st.scale = (k == 0) ? 1.f : 2.f;
                    st.ckr = lane32(ck.x, k & 63);
                    st.cki = lane32(ck.y, k & 63);
                    st.gw = (k == 0) ? sg.inv_r : 2.f * sg.inv_r;   // exact: a power of two
                    st.wk = wk;
                    st.dcr = __builtin_bit_cast(double, lane64(__builtin_bit_cast(uint64_t, dx), k & 63));
                    st.dci = __builtin_bit_cast(double, lane64(__builtin_bit_cast(uint64_t, dy), k & 63));
                    void *const p = ring();
                    publish(be, p, HC > 0);
                    V bx[PER];
#pragma unroll
                    for (int q = 0; q < PER; ++q) bx[q] = own(wat(k + 1), q);
#pragma unroll
                    for (int q = 0; q < PER; ++q) {
                        V vb = vbl[q * NT + tid];
                        C gg = ggl[q * NT + tid];
                        const V pv = psl[q * NT + tid];
                        adj_sums_elem(st, be[q].v[0], bx[q].v[0], pv.v[0], vb.v[0], gg.x, sdt);
                        adj_sums_elem(st, be[q].v[1], bx[q].v[1], pv.v[1], vb.v[1], gg.y, sdt);
                        vbl[q * NT + tid] = vb;
                        ggl[q * NT + tid] = gg;
                        if (PER > 2) __builtin_amdgcn_sched_barrier(0);
                    }
                    const bool low = HB == 0 || (k & 1) == 0;
                    flips(be, p, [&](int q, const V &sa, const V &sb) {
#pragma unroll
                        for (int v = 0; v < VE; ++v) {
                            const C f1 = low ? sa.v[v] : sb.v[v], f2 = low ? sb.v[v] : sa.v[v];
                            C o = adj_start_elem(st, sg.inv_r, sg.g, er[q][v], be[q].v[v], bp[q].v[v], bx[q].v[v],
                                                 f1.x, f1.y, sdg);
                            if constexpr (HB > 0) o = adj_add_elem(st, sg.g, o, bx[q].v[v], f2.x, f2.y, sdg);
                            bp[q].v[v] = be[q].v[v];
                            be[q].v[v] = o;
                        }
                    });
                }
            }
            load_terms(sg.K, true);
            {
                const float cr = lane32(ck.x, sg.K & 63), ci = lane32(ck.y, sg.K & 63);
                const double dcr = __builtin_bit_cast(double, lane64(__builtin_bit_cast(uint64_t, dx), sg.K & 63));
                const double dci = __builtin_bit_cast(double, lane64(__builtin_bit_cast(uint64_t, dy), sg.K & 63));
#pragma unroll
                for (int q = 0; q < PER; ++q) {
                    V vb = vbl[q * NT + tid];
                    const V pv = psl[q * NT + tid];
#pragma unroll
                    for (int v = 0; v < VE; ++v)
                        adj_last_elem(cr, ci, dcr, dci, be[q].v[v], pv.v[v], vb.v[v], sdt);
                    vbl[q * NT + tid] = vb;
                }
            }
            sph *= a.c;
            for (int o = 32; o > 0; o >>= 1) {
                sdt += __shfl_xor(sdt, o);
                sdg += __shfl_xor(sdg, o);
                sph += __shfl_xor(sph, o);
            }
            if (lane == 0) {
                red[wave][0] = lost ? NAN : sdt;
                red[wave][1] = sdg;
                red[wave][2] = sph;
            }
            __syncthreads();
            if (tid < 3) {
                double s = 0.0;
                for (int j = 0; j < NW; ++j) s += red[j][tid];
                a.part[((uint64_t)i * W + w) * 3 + tid] = s;
            }
            __syncthreads();
        }
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const C gg = ggl[q * NT + tid];
            st_v<float, false>(a.vbar + at(q), vbl[q * NT + tid]);
            a.G[at(q)] = lost ? NAN : gg.x;
            a.G[at(q) + 1] = lost ? NAN : gg.y;
        }
    }
}

// sums[3 i + j] = sum over the W workgroups of part[3 (i W + w) + j]; one wave each.
__global__ void __launch_bounds__(64) k_grad_sums(const double *part, int W, double *sums)
{
    const double *p = part + (uint64_t)(blockIdx.x / 3) * W * 3 + blockIdx.x % 3;
    double s = 0.0;
    for (int w = threadIdx.x; w < W; w += 64) s += p[3 * w];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (threadIdx.x == 0) sums[blockIdx.x] = s;
}

// Launches a sweep, or with a == NULL only tells whether both sweeps would be
// launched (hipSuccess) or have no room on `cus` compute units.
template <int T, int NT, int HC, int STRIDE>
static hipError_t grad_res_launch(const GradRes *ask, bool back, hipStream_t s, int cus)
{
    static std::atomic<int> per_cu[2];
    if constexpr (HC > 0) {
        const void *f[2] = {reinterpret_cast<const void *>(&k_grad_resident<T, NT, HC, false>),
                            reinterpret_cast<const void *>(&k_grad_resident<T, NT, HC, true>)};
        for (int i = 0; i < 2; ++i)
            if (!groups_fit(f[i], NT, STRIDE << HC, cus, per_cu[i])) return hipErrorCooperativeLaunchTooLarge;
        if (ask && launch_refused(back)) return hipErrorCooperativeLaunchTooLarge;
    }
    if (!ask) return hipSuccess;
    GradRes a = *ask;
    static std::atomic<unsigned> turn{0};   // launches take turns over the XCDs
    a.stride = STRIDE;
    a.sel = (STRIDE > 1) ? (int)(turn.fetch_add(1, std::memory_order_relaxed) % STRIDE) : 0;
    const dim3 grid((1u << HC) * STRIDE), block(NT);
    if constexpr (HC == 0) {
        if (back) hipLaunchKernelGGL((k_grad_resident<T, NT, HC, true>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((k_grad_resident<T, NT, HC, false>), grid, block, 0, s, a);
        return hipGetLastError();
    }
    void *args[] = {&a};
    const void *f = back ? reinterpret_cast<const void *>(&k_grad_resident<T, NT, HC, true>)
                         : reinterpret_cast<const void *>(&k_grad_resident<T, NT, HC, false>);
    return hipLaunchCooperativeKernel(f, grid, block, args, 0, s);
}

// Shapes of launch_resident's exchanges; milliseconds per call in the comments (3
// segments of about 30 terms from 8 to 17 qubits and at 19, 4 segments at 16 and
// 18, 16 segments of 35 terms at 20; windows of 1 to 8, none at 10 and 18), what
// the passes took in parentheses.  One CU holds one workgroup at 19 and 20 qubits,
// so like the smaller sizes they are launched cooperatively.  11 qubits with 1024
// threads once gave a wrong dE/dt while this kernel was being written, and the cause
// was not found; the kernel as it stands gives the passes' bits in that shape, 3
// segments in 0.39 instead of 0.42 ms.  It keeps 512 threads all the same.
static hipError_t launch_grad_resident(int n, const GradRes *a, bool back, hipStream_t s, int cus)
{
    switch (n) {
    case 8: return grad_res_launch<8, 128, 0, 1>(a, back, s, cus);   // 0.25 (0.85)
    case 9: return grad_res_launch<9, 256, 0, 1>(a, back, s, cus);   // 0.35 (1.4)
    case 10: return grad_res_launch<10, 512, 0, 1>(a, back, s, cus);   // 0.28 (0.81)
    case 11: return grad_res_launch<11, 512, 0, 1>(a, back, s, cus);   // 0.46 (1.4)
    case 12: return grad_res_launch<8, 128, 4, 8>(a, back, s, cus);   // 0.60 (2.0)
    case 13: return grad_res_launch<8, 128, 5, 8>(a, back, s, cus);   // 0.79 (3.3)
    case 14: return grad_res_launch<9, 256, 5, 8>(a, back, s, cus);   // 0.90 (2.9)
    case 15: return grad_res_launch<10, 256, 5, 8>(a, back, s, cus);   // 0.93 (2.8)
    case 16: return grad_res_launch<9, 256, 7, 1>(a, back, s, cus);   // 1.30 (3.7)
    case 17: return grad_res_launch<9, 256, 8, 1>(a, back, s, cus);   // 1.18 (3.1)
    case 18: return grad_res_launch<10, 256, 8, 1>(a, back, s, cus);   // 1.49 (3.9)
    case 19: return grad_res_launch<11, 512, 8, 1>(a, back, s, cus);   // 1.93 (4.3)
    default: return grad_res_launch<12, 512, 8, 1>(a, back, s, cus);  // 12.1 (24.4)
    }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

struct SegPlan {
    double r, g, inv_r, a;
    float ph_r, ph_i;
    int K, C, W;
    std::vector<double> alpha, dalpha;   // coefficients and d alpha / d a
    std::vector<int> slot;               // checkpoint slot of b_j (j = 0..K+1), -1 if none
    size_t sbase = 0;                    // store mode: window slot of b_1
};

struct GradLayout {
    size_t states, erel, A, B, vbar, G, win, ckpt, part, partm, walsh, wres, hj, q, red, mpart, total;
    size_t sync, segs, wins, coef, dcoef, place, rpart, sums, total_res;   // behind `total`: the one-launch sweeps
    int nwin, nckpt, ntiles_lo, npar;
    bool store;   // every b_k of every segment kept (win holds them all, no recomputation)
};

// Launch helpers over the tile shapes the forward path chooses (tile_cfg_for).
template <int TB, int NT, bool STREAM>
static void grad_pass_shape(const PassArgs<float> &pa, int mode, uint64_t ntiles, hipStream_t s)
{
    if (mode == PM_START) hipLaunchKernelGGL((k_pass<float, TB, NT, PM_START, false, STREAM>), dim3((unsigned)ntiles), dim3(NT), 0, s, pa);
    else if (mode == PM_FUSED) hipLaunchKernelGGL((k_pass<float, TB, NT, PM_FUSED, false, STREAM>), dim3((unsigned)ntiles), dim3(NT), 0, s, pa);
    else hipLaunchKernelGGL((k_pass<float, TB, NT, PM_ADD, false, STREAM>), dim3((unsigned)ntiles), dim3(NT), 0, s, pa);
}

static void launch_grad_pass(const PassArgs<float> &pa, int mode, uint64_t ntiles, TileCfg cfg, hipStream_t s)
{
    if (cfg.tb == TB_NARROW) grad_pass_shape<TB_NARROW, NT_NARROW, false>(pa, mode, ntiles, s);
    else if (cfg.nt == NT_MID) grad_pass_shape<GTB, NT_MID, false>(pa, mode, ntiles, s);
    else if (cfg.stream) grad_pass_shape<GTB, GNT, true>(pa, mode, ntiles, s);
    else grad_pass_shape<GTB, GNT, false>(pa, mode, ntiles, s);
}

template <int TB, int NT, bool STREAM>
static void adj_pass_shape(const AdjArgs &aa, int mode, uint64_t ntiles, hipStream_t s)
{
    const dim3 g((unsigned)ntiles), b(NT);
    if (mode == AM_START) hipLaunchKernelGGL((k_adj_pass<AM_START, TB, NT, STREAM>), g, b, 0, s, aa);
    else if (mode == AM_FUSED) hipLaunchKernelGGL((k_adj_pass<AM_FUSED, TB, NT, STREAM>), g, b, 0, s, aa);
    else hipLaunchKernelGGL((k_adj_pass<AM_ADD, TB, NT, STREAM>), g, b, 0, s, aa);
}

// The adjoint pass holds five vectors per element (256 VGPRs with 512 threads
// on 2^13 tiles): it always runs 1024 threads, 4 or 8 amplitudes per thread.
static void launch_adj_pass(const AdjArgs &aa, int mode, uint64_t ntiles, TileCfg cfg, hipStream_t s)
{
    if (cfg.tb == TB_NARROW) adj_pass_shape<TB_NARROW, NT_NARROW, false>(aa, mode, ntiles, s);
    else if (cfg.stream) adj_pass_shape<GTB, NT_MID, true>(aa, mode, ntiles, s);
    else adj_pass_shape<GTB, NT_MID, false>(aa, mode, ntiles, s);
}

// Tile shape of the gradient's passes: the action's choice, without the wide
// 2^14 tiles (whose adjoint pass would not fit the register file).
static TileCfg grad_cfg(int n)
{
    const TileCfg c = tile_cfg_for<float>(n);
    return (c.tb == TB_WIDE) ? TileCfg{GTB, GNT, c.stream} : c;
}

// Sizes whose sweeps run in one launch each.  Below 8 qubits a wave has lanes to
// spare; above 20 the backward sweep's vectors exceed the registers.
static bool grad_resident(int n) { return n >= GRES_NMIN && n <= GRES_NMAX; }

static int grad_window(int ckpt_every, int K) { return (ckpt_every <= 0 || ckpt_every > K) ? K : ckpt_every; }

static GradLayout grad_layout(int n, int S, const int *Kb, int ckpt_every)
{
    const int tb = grad_cfg(n).tb;
    const size_t N = size_t(1) << n;
    GradLayout L{};
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += align256(bytes); return o; };
    L.nwin = 1;
    L.nckpt = 0;
    L.store = ckpt_every < 0;
    if (L.store) {
        // b_1 .. b_K of segment s at slots sum_{s' < s} max(Kb[s'], 1) + j - 1
        L.nwin = 0;
        for (int s = 0; s < S; ++s) L.nwin += std::max(Kb[s], 1);
    }
    for (int s = 0; s < S && !L.store; ++s) {
        const int K = std::max(Kb[s], 1);
        const int C = grad_window(ckpt_every, K);
        const int W = (K + C - 1) / C;
        L.nwin = std::max(L.nwin, C);
        L.nckpt += 2 * (W - 1);
    }
    L.ntiles_lo = (n > tb) ? (int)(N >> tb) : 1;
    L.npar = n + n * (n - 1) / 2;
    L.states = take(N * 8 * (S + 1));
    L.erel = take(N * 4);
    L.A = take(N * 8);
    L.B = take(N * 8);
    L.vbar = take(N * 8);
    L.G = take(N * 4);
    L.win = take(N * 8 * L.nwin);
    L.ckpt = take(N * 8 * std::max(L.nckpt, 1));
    L.part = take(sizeof(double) * 2 * L.ntiles_lo * 4);     // up to 4 passes
    L.partm = take(sizeof(double) * 2 * L.ntiles_lo);
    const int wt = (n > LB_TAB) ? (1 << (n - LB_TAB)) : 1;
    L.walsh = take(sizeof(double) * (size_t)wt * L.npar);
    L.wres = take(sizeof(double) * L.npar);
    L.hj = take(sizeof(double) * (n + n * (n - 1) / 2));
    L.q = take(sizeof(double) * (size_t(1) << LB_TAB));
    L.red = take(2 * sizeof(double));
    L.mpart = take(2 * sizeof(double) * MAXPART);
    L.total = off;
    L.total_res = 0;
    if (grad_resident(n)) {
        size_t terms = 0, wins = 0;
        for (int s = 0; s < S; ++s) {
            const int K = std::max(Kb[s], 1), C = L.store ? K : grad_window(ckpt_every, K);
            terms += K + 1;
            wins += (K + C - 1) / C;
        }
        L.sync = take(sizeof(int) * RES_LINE * (2 + RES_MAXFLAGS));
        L.segs = take(sizeof(GradSeg) * S);
        L.wins = take(sizeof(GradWin) * wins);
        L.coef = take(sizeof(float2) * terms);
        L.dcoef = take(sizeof(double2) * terms);
        L.place = take(sizeof(uint64_t) * terms);
        L.rpart = take(sizeof(double) * 3 * GRES_MAXW * S);
        L.sums = take(sizeof(double) * 3 * S);
        L.total_res = off;
    }
    return L;
}

// Segments, windows, coefficients and places of the one-launch sweeps, as they lie
// from L.segs; `vec_bytes` is the size of a vector.
static std::vector<char> grad_tables(const GradLayout &L, const std::vector<SegPlan> &seg, size_t vec_bytes)
{
    std::vector<char> buf(L.rpart - L.segs, 0);
    auto at = [&](size_t off) { return buf.data() + (off - L.segs); };
    GradSeg *gs = reinterpret_cast<GradSeg *>(at(L.segs));
    GradWin *gw = reinterpret_cast<GradWin *>(at(L.wins));
    float2 *cf = reinterpret_cast<float2 *>(at(L.coef));
    double2 *dc = reinterpret_cast<double2 *>(at(L.dcoef));
    uint64_t *place = reinterpret_cast<uint64_t *>(at(L.place));
    int nc = 0, nw = 0;
    for (size_t q = 0; q < seg.size(); ++q) {
        const SegPlan &sp = seg[q];
        gs[q] = {(float)sp.inv_r, (float)sp.g, sp.ph_r, sp.ph_i, sp.K, nc, nw, sp.W};
        auto saved = [&](int k) { return L.ckpt + (size_t)sp.slot[k] * vec_bytes; };
        for (int k = 0; k <= sp.K; ++k, ++nc) {
            double cr, ci, dr, di;
            coef_of(sp.alpha, k, cr, ci);
            coef_of(sp.dalpha, k, dr, di);
            cf[nc] = make_float2((float)cr, (float)ci);
            dc[nc] = make_double2(dr * sp.r, di * sp.r);
            if (k >= 1 && L.store) place[nc] = L.win + (sp.sbase + (size_t)(k - 1)) * vec_bytes;
            else place[nc] = (k >= 1 && sp.slot[k] >= 0) ? saved(k) : GRES_NONE;
        }
        for (int w = 0; w < sp.W; ++w, ++nw) {
            GradWin &g = gw[nw];
            g.B = w * sp.C + 1;
            g.T = std::min((w + 1) * sp.C, sp.K);
            g.fresh = L.store ? -1 : g.T == sp.K ? 1 : 0;
            g.x1 = g.fresh == 0 ? saved(g.T + 1) : GRES_NONE;
            g.x2 = (g.fresh == 0 && g.T + 2 <= sp.K) ? saved(g.T + 2) : GRES_NONE;
            g.at = L.win + (L.store ? sp.sbase * vec_bytes : 0);
        }
    }
    return buf;
}

static int grad_degree_bound(int n, const double *h, const double *J, double gamma, double t)
{
    double s = 0.0;
    for (int j = 0; j < n; ++j) s += std::fabs(h[j]);
    for (int p = 0; p < n * (n - 1) / 2; ++p) s += std::fabs(J[p]);
    const double rmax = s + n * std::fabs(gamma);
    return bessel_cutoff(std::fabs(t) * rmax * 1.01 + 1.0) + 2;
}

// Workgroups of launch_grad_resident.
static int grad_resident_groups(int n)
{
    return n <= 11 ? 1 : n == 12 ? 16 : n <= 15 ? 32 : n == 16 ? 128 : 256;
}

static qw_status grad_validate(int n, const double *h, const double *J, int S, const double *gamma,
                               const double *t, double tol)
{
    if (n < 1 || n > 28) { set_error("the gradient supports 1 <= n <= 28"); return QW_EINVAL; }
    if (S < 1 || !gamma || !t || !h || (n > 1 && !J)) { set_error("S >= 1, gamma, t, h, J are required"); return QW_EINVAL; }
    if (!(tol > 0.0) || !finite(tol)) { set_error("tol must be positive"); return QW_EINVAL; }
    for (int s = 0; s < S; ++s)
        if (!finite(gamma[s]) || !finite(t[s])) { set_error("non-finite schedule"); return QW_EINVAL; }
    for (int j = 0; j < n; ++j)
        if (!finite(h[j])) { set_error("non-finite h"); return QW_EINVAL; }
    for (int p = 0; p < n * (n - 1) / 2; ++p)
        if (!finite(J[p])) { set_error("non-finite J"); return QW_EINVAL; }
    return QW_OK;
}

static std::vector<int> grad_bounds(int n, const double *h, const double *J, int S, const double *gamma,
                                    const double *t)
{
    std::vector<int> Kb(S);
    for (int s = 0; s < S; ++s) Kb[s] = grad_degree_bound(n, h, J, gamma[s], t[s]);
    return Kb;
}

static qw_status grad_impl(int n, const double *h, const double *J, int S, const double *gamma, const double *t,
                           const void *psi0, double tol, int ckpt_every, double *E_out, double *dgamma,
                           double *dt, double *dh, double *dJ, void *workspace, size_t ws_bytes, hipStream_t s,
                           void *psiT_out, qw_grad_info *info, bool one_launch)
{
    qw_status st = grad_validate(n, h, J, S, gamma, t, tol);
    if (st != QW_OK) return st;
    if (!psi0 || !workspace || !E_out || !dgamma || !dt || !dh || (n > 1 && !dJ)) {
        set_error("psi0, workspace and every output are required");
        return QW_EINVAL;
    }
    if ((reinterpret_cast<uintptr_t>(workspace) & 255) || (reinterpret_cast<uintptr_t>(psi0) & 15)) {
        set_error("workspace must be 256-byte and psi0 16-byte aligned");
        return QW_EINVAL;
    }
    const std::vector<int> Kb = grad_bounds(n, h, J, S, gamma, t);
    const GradLayout L = grad_layout(n, S, Kb.data(), ckpt_every);
    if (ws_bytes < L.total) { set_error("workspace too small: need " + std::to_string(L.total)); return QW_ENOMEM; }
    char *ws = static_cast<char *>(workspace);
    const uint64_t N = uint64_t(1) << n;
    using C = float2;
    auto vec = [&](size_t off, size_t i) { return reinterpret_cast<C *>(ws + off) + i * N; };
    C *states = vec(L.states, 0);
    float *erel = reinterpret_cast<float *>(ws + L.erel);
    float *G = reinterpret_cast<float *>(ws + L.G);
    C *vbar = vec(L.vbar, 0);
    double *part = reinterpret_cast<double *>(ws + L.part);
    double *partm = reinterpret_cast<double *>(ws + L.partm);
    hipEvent_t ev[2] = {nullptr, nullptr};
    const bool timing = info && info->timing;
    if (timing)
        for (auto &e : ev) QW_HIP(hipEventCreate(&e));
    struct EvGuard { hipEvent_t *e; ~EvGuard() { for (int i = 0; i < 2; ++i) if (e[i]) (void)hipEventDestroy(e[i]); } } eg{ev};
    if (timing) QW_HIP(hipEventRecord(ev[0], s));

    // tables, range of E, E - c
    const int np = n * (n - 1) / 2;
    std::vector<double> hj(n + np);
    std::memcpy(hj.data(), h, n * sizeof(double));
    if (np) std::memcpy(hj.data() + n, J, np * sizeof(double));
    double *dhj = reinterpret_cast<double *>(ws + L.hj);
    QW_HIP(hipMemcpyAsync(dhj, hj.data(), hj.size() * sizeof(double), hipMemcpyHostToDevice, s));
    EnergyTables T{dhj, dhj + n, reinterpret_cast<double *>(ws + L.q), n, std::min(n, LB_TAB)};
    hipLaunchKernelGGL(k_qtable<0>, dim3(((1 << T.LB) + 255) / 256), dim3(256), 0, s, T, const_cast<double *>(T.Q));
    const int ntE = (int)(N >> T.LB);
    const int npm = std::min(ntE, MAXPART);
    double *mpart = reinterpret_cast<double *>(ws + L.mpart);
    double *red = reinterpret_cast<double *>(ws + L.red);
    hipLaunchKernelGGL(k_minmax_energy<0>, dim3(npm), dim3(256), 0, s, T, mpart);
    hipLaunchKernelGGL(k_minmax_final<0>, dim3(1), dim3(256), 0, s, (const double *)mpart, npm, red);
    QW_HIP(hipGetLastError());
    double emm[2];
    QW_HIP(hipMemcpyAsync(emm, red, sizeof(emm), hipMemcpyDeviceToHost, s));
    QW_HIP(hipStreamSynchronize(s));
    const double c = 0.5 * (emm[0] + emm[1]), half = 0.5 * (emm[1] - emm[0]);
    hipLaunchKernelGGL(k_normalize_energy<float>, dim3(grid_for(ntE, 1, 1 << 16)), dim3(256), 0, s, T, c, 1.0, erel);
    QW_HIP(hipMemcpyAsync(states, psi0, N * sizeof(C), hipMemcpyDeviceToDevice, s));

    // segment plans
    const TileCfg cfg = grad_cfg(n);
    const std::vector<PassPlan> plan = plan_passes(n, cfg.tb, Cfg<float>::LMIN);
    const int P = (int)plan.size();
    std::vector<SegPlan> seg(S);
    int ck_next = 0;
    size_t store_next = 0;
    for (int q = 0; q < S; ++q) {
        SegPlan &sp = seg[q];
        double r = half + n * std::fabs(gamma[q]);
        double g = (r > 0.0) ? gamma[q] / r : 0.0;
        if (gamma[q] != 0.0 && r > 0.0) {
            float gf = (float)g;
            if (std::fabs((double)gf) > std::fabs(g)) gf = std::nextafter(gf, 0.0f);
            g = (double)gf;
            r = gamma[q] / g;
        }
        if (!(r > 0.0)) { set_error("zero spectral bound in a segment (H = const)"); return QW_EINVAL; }
        sp.r = r;
        sp.g = g;
        sp.inv_r = 1.0 / r;
        sp.a = t[q] * r;
        sp.ph_r = (float)std::cos(t[q] * c);
        sp.ph_i = (float)-std::sin(t[q] * c);
        double err = 0.0;
        if (coefficients(sp.a, tol, QW_CHEB, sp.alpha, &sp.K, &err) != 0) { set_error("coefficients"); return QW_ENOCONV; }
        if (sp.K > Kb[q]) { set_error("internal: degree bound exceeded"); return QW_ENOCONV; }
        std::vector<double> Jm(sp.K + 2);
        bessel_miller(sp.a, sp.K + 1, Jm.data());
        sp.dalpha.resize(sp.K + 1);
        for (int k = 0; k <= sp.K; ++k)
            sp.dalpha[k] = (k == 0) ? -Jm[1] : (Jm[k - 1] - Jm[k + 1]);
        const int K = std::max(sp.K, 1);
        sp.C = L.store ? K : grad_window(ckpt_every, K);
        sp.W = (sp.K == 0) ? 0 : (sp.K + sp.C - 1) / sp.C;
        sp.slot.assign(sp.K + 3, -1);
        sp.sbase = store_next;
        store_next += (size_t)std::max(Kb[q], 1);
        for (int w = 0; w + 1 < sp.W; ++w) {
            const int Tw = (w + 1) * sp.C;
            for (int j = Tw + 1; j <= std::min(Tw + 2, sp.K); ++j)
                if (sp.slot[j] < 0) sp.slot[j] = ck_next++;
        }
        if (ck_next > std::max(L.nckpt, 1)) { set_error("internal: checkpoint slots exceeded"); return QW_ENOCONV; }
    }

    // One pass of the fused schedule (mode START / ADD / FUSED, see pass_tile):
    // b1 = b_{k+1}; acc = partial or b_{k+2}; dst (and dst2 for FUSED).
    auto launch_clenshaw_pass = [&](int mode, int p, const C *b1, const C *acc, C *dst, C *dst2, double cr,
                                    double ci, double scale, double scale2, float pr, float pi, const SegPlan &sp,
                                    const C *v) {
        PassArgs<float> pa{};
        pa.b1 = b1;
        pa.acc = acc;
        pa.dst = dst;
        pa.dst2 = dst2;
        pa.psi = v;
        pa.d = erel;
        pa.g = (float)sp.g;
        pa.scale = (float)scale;
        pa.scale2 = (float)scale2;
        pa.cr = (float)cr;
        pa.ci = (float)ci;
        pa.pr = pr;
        pa.pi = pi;
        pa.n = n;
        pa.L = plan[p].L;
        pa.g0 = plan[p].g0;
        pa.h = plan[p].h;
        pa.dscale = (float)sp.inv_r;
        const uint64_t ntiles = N >> (plan[p].L + plan[p].h);
        launch_grad_pass(pa, mode, ntiles, cfg, s);
    };
    const int eg_grid = grid_for(N / 2, 256 * 4, 1 << 16);
    const uint32_t TEw = (uint32_t)std::min<uint64_t>(N, uint64_t(1) << GTB);
    const int ntw = (int)(N / TEw);

    // the one-launch sweeps, where the size and the workspace have room for them
    long long amp_terms = 0;
    for (int q = 0; q < S; ++q) amp_terms += (long long)seg[q].K << n;
    GradRes ra{};
    std::vector<char> tables;
    bool resident = one_launch && grad_resident(n) && ws_bytes >= L.total_res && plan[0].h == std::min(n, n > GTB ? TB_NARROW : GTB);
    for (const SegPlan &sp : seg) resident = resident && sp.K >= 1;
    const int cus = resident ? stream_cus(s) : 0;
    resident = resident && launch_grad_resident(n, nullptr, false, s, cus) == hipSuccess;
    auto clear_sync = [&]() {
        hipLaunchKernelGGL(k_zero_f64, dim3(64), dim3(256), 0, s, reinterpret_cast<double *>(ws + L.sync),
                           (int)(sizeof(int) * RES_LINE * (2 + RES_MAXFLAGS) / sizeof(double)));
    };
    if (resident) {
        tables = grad_tables(L, seg, N * sizeof(C));
        QW_HIP(hipMemcpyAsync(ws + L.segs, tables.data(), tables.size(), hipMemcpyHostToDevice, s));
        ra.ws = ws;
        ra.states = states;
        ra.X0 = vec(L.A, 0);
        ra.X1 = vec(L.B, 0);
        ra.vbar = vbar;
        ra.G = G;
        ra.erel = erel;
        ra.seg = reinterpret_cast<const GradSeg *>(ws + L.segs);
        ra.win = reinterpret_cast<const GradWin *>(ws + L.wins);
        ra.coef = reinterpret_cast<const float2 *>(ws + L.coef);
        ra.dcoef = reinterpret_cast<const double2 *>(ws + L.dcoef);
        ra.place = reinterpret_cast<const uint64_t *>(ws + L.place);
        ra.part = reinterpret_cast<double *>(ws + L.rpart);
        ra.start = reinterpret_cast<int *>(ws + L.sync);
        ra.flags = ra.start + 2 * RES_LINE;
        ra.c = c;
        ra.nseg = S;
        ra.polls = wait_polls();
        clear_sync();
        resident = launch_grad_resident(n, &ra, false, s, cus) == hipSuccess;
        if (!resident) (void)hipGetLastError();   // refused after all: passes
    }

    // forward sweep
    for (int q = 0; q < S && !resident; ++q) {
        const SegPlan &sp = seg[q];
        const C *v = states + (size_t)q * N;
        C *y = states + (size_t)(q + 1) * N;
        double cr, ci;
        if (sp.K == 0) {
            coef_of(sp.alpha, 0, cr, ci);
            const double pr = cr * sp.ph_r - ci * sp.ph_i, pi = cr * sp.ph_i + ci * sp.ph_r;
            hipLaunchKernelGGL(k_scale<float>, dim3(eg_grid), dim3(256), 0, s, reinterpret_cast<const CVec<float> *>(v),
                               reinterpret_cast<CVec<float> *>(y), (float)pr, (float)pi, (uint64_t)(N / 2));
            continue;
        }
        if (L.store) {
            // every b_j goes to its own slot Wst(j); the partial sums live in B.
            // Same passes and arithmetic as below, so the b_j are bit-identical.
            auto Wst = [&](int j) { return vec(L.win, sp.sbase + (size_t)(j - 1)); };
            C *Y = vec(L.B, 0);
            coef_of(sp.alpha, sp.K, cr, ci);
            hipLaunchKernelGGL(k_scale<float>, dim3(eg_grid), dim3(256), 0, s,
                               reinterpret_cast<const CVec<float> *>(v), reinterpret_cast<CVec<float> *>(Wst(sp.K)),
                               (float)cr, (float)ci, (uint64_t)(N / 2));
            auto scale_of = [](int k) { return k == 0 ? 1.0 : 2.0; };
            for (const SchedPass &ps : fused_schedule(sp.K, P)) {
                const float pr = ps.fin ? sp.ph_r : 1.f, pi = ps.fin ? sp.ph_i : 0.f;
                const C *b1 = Wst(ps.k + 1);
                if (ps.mode == PM_START) {
                    coef_of(sp.alpha, ps.k, cr, ci);
                    const C *acc = (ps.k + 2 <= sp.K) ? (P == 1 ? Wst(ps.k + 2) : nullptr) : nullptr;
                    if (P > 1 && ps.k != sp.K - 1) { set_error("internal: start pass inside a term"); return QW_EINVAL; }
                    C *dst = ps.fin ? y : (P == 1 ? Wst(ps.k) : Y);
                    launch_clenshaw_pass(PM_START, ps.orient, b1, acc, dst, nullptr, cr, ci, scale_of(ps.k), 0.0, pr, pi,
                                         sp, v);
                } else if (ps.mode == PM_ADD) {
                    launch_clenshaw_pass(PM_ADD, ps.orient, b1, Y, ps.fin ? y : Y, nullptr, 0.0, 0.0, scale_of(ps.k),
                                         0.0, pr, pi, sp, v);
                } else {
                    coef_of(sp.alpha, ps.k - 1, cr, ci);
                    launch_clenshaw_pass(PM_FUSED, ps.orient, b1, Y, Wst(ps.k), Y, cr, ci, scale_of(ps.k),
                                         scale_of(ps.k - 1), 1.f, 0.f, sp, v);
                }
            }
            QW_HIP(hipGetLastError());
            continue;
        }
        // fused schedule in two ping-pong buffers; X holds the last completed b_k
        C *X = vec(L.A, 0), *Y = vec(L.B, 0);
        coef_of(sp.alpha, sp.K, cr, ci);
        hipLaunchKernelGGL(k_scale<float>, dim3(eg_grid), dim3(256), 0, s, reinterpret_cast<const CVec<float> *>(v),
                           reinterpret_cast<CVec<float> *>(X), (float)cr, (float)ci, (uint64_t)(N / 2));
        auto save = [&](int k, const C *src) -> qw_status {
            if (k >= 1 && sp.slot[k] >= 0)
                QW_HIP(hipMemcpyAsync(vec(L.ckpt, sp.slot[k]), src, N * sizeof(C), hipMemcpyDeviceToDevice, s));
            return QW_OK;
        };
        if ((st = save(sp.K, X)) != QW_OK) return st;
        auto scale_of = [](int k) { return k == 0 ? 1.0 : 2.0; };
        for (const SchedPass &ps : fused_schedule(sp.K, P)) {
            const float pr = ps.fin ? sp.ph_r : 1.f, pi = ps.fin ? sp.ph_i : 0.f;
            if (ps.mode == PM_START) {
                coef_of(sp.alpha, ps.k, cr, ci);
                launch_clenshaw_pass(PM_START, ps.orient, X, (ps.k == sp.K - 1) ? nullptr : Y, ps.fin ? y : Y,
                                     nullptr, cr, ci, scale_of(ps.k), 0.0, pr, pi, sp, v);
                if (P == 1 && !ps.fin) {
                    std::swap(X, Y);
                    if ((st = save(ps.k, X)) != QW_OK) return st;
                }
            } else if (ps.mode == PM_ADD) {
                launch_clenshaw_pass(PM_ADD, ps.orient, X, Y, ps.fin ? y : Y, nullptr, 0.0, 0.0, scale_of(ps.k), 0.0,
                                     pr, pi, sp, v);
            } else {
                coef_of(sp.alpha, ps.k - 1, cr, ci);
                launch_clenshaw_pass(PM_FUSED, ps.orient, X, Y, Y, X, cr, ci, scale_of(ps.k), scale_of(ps.k - 1),
                                     1.f, 0.f, sp, v);
                std::swap(X, Y);
                if ((st = save(ps.k, X)) != QW_OK) return st;
            }
        }
        QW_HIP(hipGetLastError());
    }
    // seed: ybar = 2 H_P psi_S, G = |psi_S|^2, energy
    hipLaunchKernelGGL(k_zero_f64, dim3(64), dim3(256), 0, s, partm, 2 * L.ntiles_lo);
    {
        EwArgs ea{};
        ea.x = states + (size_t)S * N;
        ea.y = vbar;
        ea.G = G;
        ea.erel = erel;
        ea.part = partm;
        ea.c = c;
        ea.TE = TEw;
        hipLaunchKernelGGL(k_seed, dim3(ntw), dim3(256), 0, s, ea);
    }
    QW_HIP(hipGetLastError());
    std::vector<double> hp(2 * std::max(L.ntiles_lo * 4, ntw));
    QW_HIP(hipMemcpyAsync(hp.data(), partm, 2 * ntw * sizeof(double), hipMemcpyDeviceToHost, s));
    if (resident) {
        clear_sync();
        if (launch_grad_resident(n, &ra, true, s, cus) != hipSuccess) {
            (void)hipGetLastError();
            QW_HIP(hipStreamSynchronize(s));   // hp
            return grad_impl(n, h, J, S, gamma, t, psi0, tol, ckpt_every, E_out, dgamma, dt, dh, dJ, workspace, ws_bytes,
                             s, psiT_out, info, false);
        }
        hipLaunchKernelGGL(k_grad_sums, dim3(3 * S), dim3(64), 0, s, (const double *)ra.part, grad_resident_groups(n),
                           reinterpret_cast<double *>(ws + L.sums));
        QW_HIP(hipGetLastError());
        std::vector<double> sums(3 * (size_t)S);
        QW_HIP(hipMemcpyAsync(sums.data(), ws + L.sums, sums.size() * sizeof(double), hipMemcpyDeviceToHost, s));
        QW_HIP(hipStreamSynchronize(s));
        // NaN: a wait was given up (or the state held one): again in passes
        bool whole = true;
        for (int i = 0; i < ntw; ++i) whole = whole && finite(hp[2 * i]);
        for (double x : sums) whole = whole && finite(x);
        if (!whole)
            return grad_impl(n, h, J, S, gamma, t, psi0, tol, ckpt_every, E_out, dgamma, dt, dh, dJ, workspace, ws_bytes,
                             s, psiT_out, info, false);
        for (int q = 0; q < S; ++q) {
            dt[q] = sums[3 * q] + sums[3 * q + 2];
            dgamma[q] = sums[3 * q + 1] / seg[q].r;
        }
    } else {
        QW_HIP(hipStreamSynchronize(s));
    }
    double energy = 0.0;
    for (int i = 0; i < ntw; ++i) energy += hp[2 * i];
    *E_out = energy;
    // (which may be psi0: after the last point from which the call starts again)
    if (psiT_out)
        QW_HIP(hipMemcpyAsync(psiT_out, states + (size_t)S * N, N * sizeof(C), hipMemcpyDeviceToDevice, s));

    // backward sweep
    for (int q = S - 1; q >= 0 && !resident; --q) {
        const SegPlan &sp = seg[q];
        const C *v = states + (size_t)q * N;
        const C *y = states + (size_t)(q + 1) * N;
        hipLaunchKernelGGL(k_zero_f64, dim3(64), dim3(256), 0, s, part, 2 * L.ntiles_lo * 4);
        hipLaunchKernelGGL(k_zero_f64, dim3(64), dim3(256), 0, s, partm, 2 * L.ntiles_lo);
        C *Acur = vec(L.A, 0), *Bnxt = vec(L.B, 0);
        {
            EwArgs ea{};
            ea.x = vbar;           // ybar
            ea.v = y;
            ea.y = Acur;           // beta_0
            ea.z = vbar;           // zeroed
            ea.part = partm;
            ea.c = c;
            ea.cr = sp.ph_r;       // conj(phase) = (ph_r, -ph_i)
            ea.ci = -sp.ph_i;
            ea.TE = TEw;
            hipLaunchKernelGGL(k_beta0, dim3(ntw), dim3(256), 0, s, ea);
        }
        const C *prevp = nullptr;
        for (int w = 0; w < sp.W; ++w) {
            const int Bw = w * sp.C + 1, Tw = std::min((w + 1) * sp.C, sp.K);
            // store mode: one window, b_1 .. b_K already in their slots
            C *win = L.store ? vec(L.win, sp.sbase) : vec(L.win, 0);
            // recompute b_Tw .. b_Bw into win[j - Bw]
            const C *x1 = nullptr, *x2 = nullptr;
            int jstart = 0;
            double cr, ci;
            if (L.store) {
                // nothing to recompute
            } else if (Tw == sp.K) {
                coef_of(sp.alpha, sp.K, cr, ci);
                hipLaunchKernelGGL(k_scale<float>, dim3(eg_grid), dim3(256), 0, s,
                                   reinterpret_cast<const CVec<float> *>(v),
                                   reinterpret_cast<CVec<float> *>(win + (size_t)(sp.K - Bw) * N), (float)cr, (float)ci,
                                   (uint64_t)(N / 2));
                x1 = win + (size_t)(sp.K - Bw) * N;
                x2 = nullptr;
                jstart = sp.K - 1;
            } else {
                x1 = vec(L.ckpt, sp.slot[Tw + 1]);
                x2 = (Tw + 2 <= sp.K) ? vec(L.ckpt, sp.slot[Tw + 2]) : nullptr;
                jstart = Tw;
            }
            // terms j = jstart .. Bw on the fused schedule, b_j kept in win[j - Bw];
            // every term visits the orientations in the order the forward sweep
            // used (mirrored when the window starts on the other parity), so the
            // recomputed b_j equal the forward ones bit for bit
            if (!L.store) {
                auto Wj = [&](int j) { return win + (size_t)(j - Bw) * N; };
                auto Bj = [&](int j) -> const C * {
                    if (j <= jstart) return Wj(j);
                    return (j == jstart + 1) ? x1 : x2;
                };
                const bool mirror = ((sp.K - 1 - jstart) & 1) != 0;
                for (SchedPass ps : fused_schedule(jstart - Bw + 1, P)) {
                    if (mirror) ps.orient = P - 1 - ps.orient;
                    const int j = Bw + ps.k;
                    if (ps.mode == PM_START) {
                        coef_of(sp.alpha, j, cr, ci);
                        launch_clenshaw_pass(PM_START, ps.orient, Bj(j + 1), Bj(j + 2), Wj(j), nullptr, cr, ci, 2.0,
                                             0.0, 1.f, 0.f, sp, v);
                    } else if (ps.mode == PM_ADD) {
                        launch_clenshaw_pass(PM_ADD, ps.orient, Bj(j + 1), Wj(j), Wj(j), nullptr, 0.0, 0.0, 2.0, 0.0,
                                             1.f, 0.f, sp, v);
                    } else {
                        coef_of(sp.alpha, j - 1, cr, ci);
                        launch_clenshaw_pass(PM_FUSED, ps.orient, Bj(j + 1), Wj(j), Wj(j), Wj(j - 1), cr, ci, 2.0,
                                             2.0, 1.f, 0.f, sp, v);
                    }
                }
            }
            // adjoint steps k = Bw-1 .. Tw-1 with b_{k+1} = win[k + 1 - Bw].  Step k
            // visits the orientations in order 0..P-1 (k even) or reversed (k
            // odd), so its last orientation is the first of step k + 1 and the
            // two share one FUSED pass whenever b_{k+2} is in the window.  The
            // order depends on k alone and a partial sum goes to the slot of the
            // pass's position in its step, so the result does not depend on the
            // checkpoint interval.
            {
                auto orient = [&](int k, int i) { return (k & 1) ? P - 1 - i : i; };
                auto step_of = [&](int k) {
                    double ckr, cki, dcr, dci;
                    coef_of(sp.alpha, k, ckr, cki);
                    coef_of(sp.dalpha, k, dcr, dci);
                    const double wk = (k == 0) ? 1.0 : 2.0;
                    AdjStep st;
                    st.scale = (k == 0) ? 1.f : 2.f;
                    st.ckr = (float)ckr;
                    st.cki = (float)cki;
                    st.gw = (float)(wk * sp.inv_r);
                    st.wk = wk;
                    st.dcr = dcr * sp.r;
                    st.dci = dci * sp.r;
                    return st;
                };
                auto bwin = [&](int j) { return win + (size_t)(j - Bw) * N; };
                auto slot = [&](int i) { return part + (size_t)2 * L.ntiles_lo * i; };
                bool started = false;   // step k was started by the previous fused pass
                for (int k = Bw - 1; k <= Tw - 1; ++k) {
                    AdjArgs aa{};
                    aa.v = v;
                    aa.vbar = vbar;
                    aa.G = G;
                    aa.erel = erel;
                    aa.dscale = (float)sp.inv_r;
                    aa.g = (float)sp.g;
                    aa.st = step_of(k);
                    aa.beta = Acur;
                    aa.bnext = bwin(k + 1);
                    auto launch = [&](int mode, int o) {
                        aa.L = plan[o].L;
                        aa.g0 = plan[o].g0;
                        aa.h = plan[o].h;
                        launch_adj_pass(aa, mode, N >> (plan[o].L + plan[o].h), cfg, s);
                    };
                    if (!started) {
                        aa.prev = prevp;
                        aa.dst = Bnxt;
                        aa.part = slot(0);
                        launch(AM_START, orient(k, 0));
                    }
                    started = false;
                    for (int i = 1; i <= P - 2; ++i) {
                        aa.prev = Bnxt;
                        aa.dst = Bnxt;
                        aa.part = slot(i);
                        launch(AM_ADD, orient(k, i));
                    }
                    if (P >= 2) {
                        aa.prev = Bnxt;
                        aa.dst = Bnxt;
                        aa.part = slot(P - 1);
                        if (k + 1 <= Tw - 1) {
                            aa.dst2 = Acur;          // beta_{k+2} over beta_k
                            aa.bnext2 = bwin(k + 2);
                            aa.part2 = slot(0);
                            aa.st2 = step_of(k + 1);
                            launch(AM_FUSED, orient(k, P - 1));
                            started = true;
                        } else {
                            launch(AM_ADD, orient(k, P - 1));
                        }
                    }
                    prevp = Acur;
                    std::swap(Acur, Bnxt);
                }
            }
            QW_HIP(hipGetLastError());
        }
        {
            double ckr, cki, dcr, dci;
            coef_of(sp.alpha, sp.K, ckr, cki);
            coef_of(sp.dalpha, sp.K, dcr, dci);
            EwArgs ea{};
            ea.x = Acur;   // beta_K
            ea.v = v;
            ea.y = vbar;
            ea.part = part;   // pass-0 slots, same tile count
            ea.cr = (float)ckr;
            ea.ci = (float)cki;
            ea.dcr = dcr * sp.r;
            ea.dci = dci * sp.r;
            ea.TE = TEw;
            hipLaunchKernelGGL(k_adj_last, dim3(ntw), dim3(256), 0, s, ea);
            QW_HIP(hipGetLastError());
        }
        const size_t npart = (size_t)2 * L.ntiles_lo * P;
        std::vector<double> pp(npart), pm(2 * ntw);
        QW_HIP(hipMemcpyAsync(pp.data(), part, npart * sizeof(double), hipMemcpyDeviceToHost, s));
        QW_HIP(hipMemcpyAsync(pm.data(), partm, pm.size() * sizeof(double), hipMemcpyDeviceToHost, s));
        QW_HIP(hipStreamSynchronize(s));
        double sdt = 0.0, sdg = 0.0, sph = 0.0;
        for (size_t i = 0; i < npart; i += 2) {
            sdt += pp[i];
            sdg += pp[i + 1];
        }
        for (int i = 0; i < ntw; ++i) sph += pm[2 * i];
        dt[q] = sdt + sph;
        dgamma[q] = sdg / sp.r;
    }

    // Walsh reduction of G
    const int wt = (n > LB_TAB) ? (1 << (n - LB_TAB)) : 1;
    double *walsh = reinterpret_cast<double *>(ws + L.walsh);
    double *wres = reinterpret_cast<double *>(ws + L.wres);
    hipLaunchKernelGGL(k_walsh_tile, dim3(wt), dim3(256), 0, s, (const float *)G, n, std::min(n, LB_TAB), walsh);
    hipLaunchKernelGGL(k_walsh_reduce, dim3(L.npar), dim3(256), 0, s, (const double *)walsh, wt, L.npar, wres);
    QW_HIP(hipGetLastError());
    std::vector<double> res(L.npar);
    QW_HIP(hipMemcpyAsync(res.data(), wres, L.npar * sizeof(double), hipMemcpyDeviceToHost, s));
    QW_HIP(hipStreamSynchronize(s));
    std::memcpy(dh, res.data(), n * sizeof(double));
    if (np) std::memcpy(dJ, res.data() + n, np * sizeof(double));
    if (info) {
        info->amp_terms = amp_terms;
        info->passes = P;
        int sk = 0;
        for (auto &x : seg) sk += x.K;
        info->sum_K = sk;
        if (timing) {
            QW_HIP(hipEventRecord(ev[1], s));
            QW_HIP(hipEventSynchronize(ev[1]));
            QW_HIP(hipEventElapsedTime(&info->total_ms, ev[0], ev[1]));
        }
    }
    return QW_OK;
}

}  // namespace qw

using namespace qw;

extern "C" {

size_t qw_anneal_workspace_bytes_c64(int n, const double *h, const double *J, int S, const double *gamma,
                                     const double *t, int ckpt_every)
{
    if (grad_validate(n, h, J, S, gamma, t, 1.0) != QW_OK) return 0;
    const std::vector<int> Kb = grad_bounds(n, h, J, S, gamma, t);
    const GradLayout L = grad_layout(n, S, Kb.data(), ckpt_every);
    return std::max(L.total, L.total_res);
}

qw_status qw_anneal_energy_grad_c64(int n, const double *h, const double *J, int S, const double *gamma,
                                    const double *t, const void *psi0, double tol, int ckpt_every, double *E,
                                    double *dgamma, double *dt, double *dh, double *dJ, void *workspace,
                                    size_t ws_bytes, void *stream, void *psiT_out, qw_grad_info *info)
{
    if (info) {
        const int tm = info->timing;
        std::memset(info, 0, sizeof(*info));
        info->timing = tm;
    }
    return grad_impl(n, h, J, S, gamma, t, psi0, tol, ckpt_every, E, dgamma, dt, dh, dJ, workspace, ws_bytes,
                     reinterpret_cast<hipStream_t>(stream), psiT_out, info, true);
}

}  // extern "C"

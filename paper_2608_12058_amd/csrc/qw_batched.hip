// Batched exp(-i t_i H_i) psi_i for many independent instances of uneven size.
//
// Section III.A of the paper concatenates 2^(24-n) equal-size instances and
// uses one shared polynomial of the largest radius.  Here every instance keeps
// its own shift, bound and coefficients, and sizes may differ:
//
//  * instances with n <= 13 run their whole recurrence inside one workgroup
//    (vectors in registers): one persistent launch drains them in
//    descending order of cost N*K;
//  * instances with 14 <= n <= 22 run the fused two-orientation schedule of the
//    single-instance path (one pass per Clenshaw term), grouped: instances are
//    sorted by degree K so that at global step s the still-active ones form a
//    prefix of one tile table, and each step is one launch over that prefix.
//    The launches are captured into a HIP graph.  Optionally the large instances are split into
//    "waves" whose working set (20 bytes per amplitude) fits the 256 MB
//    last-level cache, each wave running all of its steps before the next; the
//    wave size is picked by qw_batched_tune_c64 and stored in a tune file.
//
// Spectral bounds and normalised diagonals are generated on the device from
// the couplings of every instance (section III.A: only the couplings are sent).
#include "qw_kernels.h"
#include "qw_resident.h"

#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <fstream>
#include <mutex>
#include <numeric>
#include <sstream>

namespace qw {

struct BatchDesc {
    // energy tables
    const double *h, *J;
    double *Q;
    int n, LB;
    int tile0, ntiles;     // range of this instance in the energy tile table
    // recurrence
    const float2 *psi;
    float2 *out;
    float *d;
    float2 *B1, *B2;
    const float2 *coef;    // c_0..c_K
    double c, inv_r;
    float g, pr, pi;
    int K;
};

// Q tables of all instances: grid (chunks of 256 low-bit patterns, instances).
__global__ void k_qtable_batched(BatchDesc *D)
{
    const BatchDesc &b = D[blockIdx.y];
    const uint32_t lo = blockIdx.x * blockDim.x + threadIdx.x;
    if (lo >= (1u << b.LB)) return;
    double acc = 0.0;
    for (int j = 0; j < b.LB; ++j) {
        const double sj = ((lo >> j) & 1) ? -1.0 : 1.0;
        double fj = 0.0;
        for (int k = j + 1; k < b.LB; ++k) {
            const double Jk = b.J[pair_off(b.n, j, k)];
            fj += ((lo >> k) & 1) ? -Jk : Jk;
        }
        acc += sj * fj;
    }
    b.Q[lo] = acc;
}

// One block per energy tile (instance, high bits): block min / max, or (NORM)
// the normalised diagonal (E - c)/r in float.
template <bool NORM>
__global__ void __launch_bounds__(256) k_energy_batched(const BatchDesc *D, const int2 *etiles, double *part)
{
    __shared__ double f[LB_TAB];
    __shared__ double Cc;
    __shared__ double smin[256], smax[256];
    const int2 tt = etiles[blockIdx.x];
    const BatchDesc &b = D[tt.x];
    EnergyTables T{b.h, b.J, b.Q, b.n, b.LB};
    tile_fields(T, (uint64_t)tt.y, f, &Cc);
    __syncthreads();
    const uint32_t TE = 1u << b.LB;
    double mn = INFINITY, mx = -INFINITY;
    for (uint32_t lo = threadIdx.x; lo < TE; lo += blockDim.x) {
        double e = Cc + b.Q[lo];
        for (int j = 0; j < b.LB; ++j) e += ((lo >> j) & 1) ? -f[j] : f[j];
        if constexpr (NORM) {
            b.d[((uint64_t)tt.y << b.LB) | lo] = (float)((e - b.c) * b.inv_r);
        } else {
            mn = fmin(mn, e);
            mx = fmax(mx, e);
        }
    }
    if constexpr (!NORM) {
        smin[threadIdx.x] = mn;
        smax[threadIdx.x] = mx;
        __syncthreads();
        for (int s = 128; s > 0; s >>= 1) {
            if ((int)threadIdx.x < s) {
                smin[threadIdx.x] = fmin(smin[threadIdx.x], smin[threadIdx.x + s]);
                smax[threadIdx.x] = fmax(smax[threadIdx.x], smax[threadIdx.x + s]);
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            part[2 * blockIdx.x] = smin[0];
            part[2 * blockIdx.x + 1] = smax[0];
        }
    }
}

// Per-instance reduction of the tile partials: block i -> emm[2i], emm[2i+1].
__global__ void __launch_bounds__(256) k_minmax_instances(const BatchDesc *D, const double *part, double *emm)
{
    const BatchDesc &b = D[blockIdx.x];
    double mn = INFINITY, mx = -INFINITY;
    for (int i = b.tile0 + threadIdx.x; i < b.tile0 + b.ntiles; i += blockDim.x) {
        mn = fmin(mn, part[2 * i]);
        mx = fmax(mx, part[2 * i + 1]);
    }
    __shared__ double smin[256], smax[256];
    smin[threadIdx.x] = mn;
    smax[threadIdx.x] = mx;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            smin[threadIdx.x] = fmin(smin[threadIdx.x], smin[threadIdx.x + s]);
            smax[threadIdx.x] = fmax(smax[threadIdx.x], smax[threadIdx.x + s]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        emm[2 * blockIdx.x] = smin[0];
        emm[2 * blockIdx.x + 1] = smax[0];
    }
}

// ---------------------------------------------------------------------------
// Instances of one workgroup
// ---------------------------------------------------------------------------

static constexpr int ONCHIP_NT = 1024;

struct OnchipItem {
    const float2 *psi;
    float2 *out;
    const float *d;
    const float2 *coef;   // c_0 .. c_K
    float g, pr, pi;      // pr + i pi: global phase
    int n, K;
};

// The recurrence of one instance of at most 11 + log2(PER) qubits, its vectors in
// registers and b_{k+1} in LDS besides, where a term reads the flips of the lane
// and wave bits (three lane bits by DPP, bit 0 and a thread's own vectors from its
// registers).  Smaller instances leave threads without an amplitude: those keep
// zeros, so that every thread sums the same flips and the reads go out together.
template <int PER> __device__ __forceinline__ void onchip_run(const OnchipItem &I, CVec<float> *lds)
{
    using C = float2;
    using V = CVec<float>;
    constexpr int VE = V::N, NT = ONCHIP_NT, LT = 10, QB = (PER == 4) ? 2 : (PER == 2) ? 1 : 0;
    constexpr bool TWICE = PER * NT * 2 <= (1 << (Cfg<float>::TB - 1));   // room for two tiles: one barrier per term
    const int tid = threadIdx.x, lane = tid & 63;
    auto inside = [&](int q) { return PER > 1 || (uint32_t)tid * VE < (1u << I.n); };
    V b1[PER], b2[PER], ps[PER];
    float d[PER][VE];
    C ck{0.f, 0.f};           // lane l: c_{64 i + l}
    auto load_coef = [&](int k) {
        const int i = (k & ~63) + lane;
        if (i <= I.K) ck = I.coef[i];
    };
    auto lane_value = [](float x, int l) {
        return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), l));
    };
    load_coef(I.K);
    const float cKr = lane_value(ck.x, I.K & 63), cKi = lane_value(ck.y, I.K & 63);
    int t = 0;
    auto share = [&]() {
        if (TWICE) t ^= 1;
        else __syncthreads();   // every flip of the last term has been read
#pragma unroll
        for (int q = 0; q < PER; ++q) lds[t * PER * NT + q * NT + tid] = b1[q];
        __syncthreads();
    };
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const uint32_t e = (uint32_t)(q * NT + tid) * VE;
#pragma unroll
        for (int v = 0; v < VE; ++v) {
            ps[q].v[v] = C{0.f, 0.f};
            d[q][v] = 0.f;
            if (inside(q)) {
                ps[q].v[v] = I.psi[e + v];
                d[q][v] = I.d[e + v];
            }
            const C p = ps[q].v[v];
            b1[q].v[v] = C{fmad(cKr, p.x, -(cKi * p.y)), fmad(cKr, p.y, cKi * p.x)};
            b2[q].v[v] = C{0.f, 0.f};
        }
    }
    if (I.K > 0) share();
    for (int k = I.K - 1; k >= 0; --k) {
        if ((k & 63) == 63) load_coef(k);
        const float cr = lane_value(ck.x, k & 63), ci = lane_value(ck.y, k & 63);
        const float scale = (k == 0) ? 1.f : 2.f;
        V f[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            auto add = [&](const V &y) {
#pragma unroll
                for (int v = 0; v < VE; ++v) {
                    f[q].v[v].x += y.v[v].x;
                    f[q].v[v].y += y.v[v].y;
                }
            };
            f[q].v[0] = b1[q].v[1];
            f[q].v[1] = b1[q].v[0];
#pragma unroll
            for (int j = 0; j < QB; ++j) add(b1[q ^ (1 << j)]);
            add(lane_flip<float, 0xb1>(b1[q]));    // quad_perm 1 0 3 2
            add(lane_flip<float, 0x4e>(b1[q]));    // quad_perm 2 3 0 1
            add(lane_flip<float, 0x128>(b1[q]));   // row_ror 8
#pragma unroll
            for (int j = 2; j < LT; ++j)
                if (j != 3) add(lds[t * PER * NT + q * NT + (tid ^ (1 << j))]);
        }
#pragma unroll
        for (int q = 0; q < PER; ++q)
#pragma unroll
            for (int v = 0; v < VE; ++v) {
                const C b = b1[q].v[v], s = b2[q].v[v], p = ps[q].v[v], x = f[q].v[v];
                const float hr = fmad(d[q][v], b.x, I.g * x.x), hi = fmad(d[q][v], b.y, I.g * x.y);
                const float tr = fmad(scale, hr, -s.x), ti = fmad(scale, hi, -s.y);
                b2[q].v[v] = b;
                b1[q].v[v] = C{tr + fmad(cr, p.x, -(ci * p.y)), ti + fmad(cr, p.y, ci * p.x)};
                if (!inside(q)) b1[q].v[v] = C{0.f, 0.f};
            }
        if (k > 0) share();
    }
#pragma unroll
    for (int q = 0; q < PER; ++q)
#pragma unroll
        for (int v = 0; v < VE; ++v) {
            const C y = b1[q].v[v];
            if (inside(q))
                I.out[(uint32_t)(q * NT + tid) * VE + v] =
                    C{fmad(I.pr, y.x, -(I.pi * y.y)), fmad(I.pr, y.y, I.pi * y.x)};
        }
    __syncthreads();   // lds is reused by the next instance
}

// Whole recurrences of the small instances, one workgroup each; the workgroups
// drain the list, costliest first.  Bounded by LDS reads at 13 qubits (7 of 16 B
// per two amplitudes and term) and by the latency of a term's reads, sums and
// barrier below.  Microseconds per term, in parentheses with the amplitudes 8 B
// apart, all flips read from LDS and coefficients loaded where they were used:
// 13 qubits 2.6 (5.6; 256 instances 2.9 (5.9)), 12: 1.1 (3.0), 11: 0.78 (1.8), 10
// and less 0.78 (10: 1.3, 8: 1.1, 4: 0.89).
__global__ void __launch_bounds__(ONCHIP_NT) k_onchip(const OnchipItem *items, const int *order, int count)
{
    __shared__ CVec<float> lds[1 << (Cfg<float>::TB - 1)];
    for (int it = blockIdx.x; it < count; it += gridDim.x) {
        const OnchipItem I = wave_uniform(items[__builtin_amdgcn_readfirstlane(order[it])]);
        if (I.n == 13) onchip_run<4>(I, lds);
        else if (I.n == 12) onchip_run<2>(I, lds);
        else onchip_run<1>(I, lds);
    }
}

// ---------------------------------------------------------------------------
// Instances in grouped passes
// ---------------------------------------------------------------------------

// Global step `step` of the fused two-orientation schedule for the tile
// (instance, t) of this block.  Every instance of the multi-pass class runs
// K + 1 passes: step 0 starts term K-1 in the low orientation (MODE START);
// step j (1 <= j < K) completes term K-j and starts term K-j-1 in one fused
// pass; step K completes term 0 and writes the output (MODE ADD).  The
// orientation alternates (even steps: the low TB bits, odd steps: the n - TB
// high bits), so it is the same for every active instance of a step; the
// host launches the fused and the final instances of a step separately.  The
// Clenshaw start b_K = c_K psi is folded into the loads: steps 0 and 1 read
// psi scaled by c_K as b_{k+1}, so b_K is never stored.
//
// Tile classes (chosen per instance size by the tuner): MID = 2^13 tiles with
// 1024 threads (8 amplitudes per thread; the per-instance arguments live in
// vector registers, so fewer amplitudes per thread keep the fused pass free
// of spills), NARROW = 2^12 tiles with 1024 threads (n <= 20), WIDE_T = 2^13
// tiles with 512 threads.  STREAM: the b vectors carry the non-temporal hint
// and psi and the diagonal stay cacheable, for waves whose vectors exceed the
// memory-side cache (256 instances of 12..22 qubits, 7.7 GB: 1093 -> 1020 ms;
// the hint on psi and the diagonal as well: 1043 ms).
enum BatchClass { BC_MID = 0, BC_NARROW = 1, BC_WIDE_T = 2, BC_COUNT = 3 };
template <int C> struct ClassShape;
template <> struct ClassShape<BC_MID> { static constexpr int TB = 13, NT = 1024; };
template <> struct ClassShape<BC_NARROW> { static constexpr int TB = 12, NT = 1024; };
template <> struct ClassShape<BC_WIDE_T> { static constexpr int TB = 13, NT = 512; };
inline int class_tb(int c) { return c == BC_NARROW ? 12 : 13; }

// c_k of an instance, read through a global pointer (one value for the block)
__device__ __forceinline__ float2 coef_at(const float2 *coef, int k)
{
    const QW_GLOBAL float *c = (const QW_GLOBAL float *)(coef + k);
    return make_float2(c[0], c[1]);
}

template <int CLS, bool HIGH, int MODE, bool STREAM = false>
__global__ void __launch_bounds__(ClassShape<CLS>::NT) __attribute__((amdgpu_waves_per_eu(4)))
k_pass_batched(const BatchDesc *D, const int2 *tiles, int step)
{
    constexpr int TB = ClassShape<CLS>::TB, NT = ClassShape<CLS>::NT;
    __shared__ float2 lds[1 << TB];
    const int2 tt = wave_uniform(tiles[blockIdx.x]);
    const BatchDesc b = wave_uniform(D[tt.x]);
    const bool swapped = (step >= 1) && ((step - 1) & 1);   // one swap after every fused step
    float2 *X = swapped ? b.B2 : b.B1;
    float2 *Y = swapped ? b.B1 : b.B2;
    PassArgs<float> a{};
    a.b1 = X;
    if (step <= 1) {
        // b_{k+1} = b_K = c_K psi (b_K itself is never stored)
        const float2 cK = coef_at(b.coef, b.K);
        a.b1 = b.psi;
        a.b1_scaled = 1;
        a.b1r = cK.x;
        a.b1i = cK.y;
    }
    a.psi = b.psi;
    a.d = b.d;
    a.g = b.g;
    a.n = b.n;
    a.pr = 1.f;
    a.pi = 0.f;
    if (HIGH) {
        a.h = b.n - TB;
        a.L = TB - a.h;
        a.g0 = TB;
    } else {
        a.L = 0;
        a.g0 = 0;
        a.h = TB;
    }
    if constexpr (MODE == PM_START) {
        const int k = b.K - 1;
        const float2 ck = coef_at(b.coef, k);
        a.acc = nullptr;
        a.dst = Y;
        a.scale = (k == 0) ? 1.f : 2.f;
        a.cr = ck.x;
        a.ci = ck.y;
    } else if constexpr (MODE == PM_ADD) {
        a.acc = Y;
        a.dst = b.out;
        a.scale = 1.f;
        a.pr = b.pr;
        a.pi = b.pi;
    } else {
        const int k = b.K - step;   // completed here; k - 1 is started
        const float2 ck = coef_at(b.coef, k - 1);
        a.acc = Y;
        a.dst = Y;
        a.dst2 = X;
        a.scale = 2.f;
        a.scale2 = (k - 1 == 0) ? 1.f : 2.f;
        a.cr = ck.x;
        a.ci = ck.y;
    }
    pass_tile<float, TB, NT, MODE, false, STREAM, STREAM>(a, (uint64_t)tt.y, lds);
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

static constexpr int BATCH_MAXN = 22;

// Schedule of a batch: the largest size run whole in one workgroup, the tile
// class of every larger size, the working-set cap of a wave, and whether the
// one-workgroup launch runs beside the passes on a side stream.
struct BatchSched {
    long long wave_bytes = 0;
    int onchip_nmax = Cfg<float>::TB;
    int concurrent = 0;
    signed char cls[BATCH_MAXN + 1];
    bool full = false;   // the batch fills the device with 19 and 20 qubits alone (class_for)
    BatchSched() { std::memset(cls, -1, sizeof(cls)); }
};

// Class actually used for a multi-pass instance of n qubits: the requested
// one, else NARROW up to 20 qubits, MID above, where 2^12 tiles would have rows
// below 128 B (21) or a third orientation (22).  The smaller tiles give twice the
// workgroups, which counts at the steps that only a few instances still take: 48
// instances of 12 to 20 qubits 42.8 ms against 45.0 with MID, 9 of 14 to 19 7.8
// against 9.1, 34 of 11 to 17 5.8 against 6.9.  From 2^24 amplitudes of 19 and 20
// qubits every step fills the device and outgrows the memory-side cache, where those
// two sizes are faster in the longer rows of MID (64 instances of 19 qubits 15.2
// against 14.7 ms, 16 of 20 7.75 against 7.53; 16 of 19 3.30 against 3.43, 64 of 18
// 6.24 against 6.56).
static int class_for(const BatchSched &S, int n)
{
    const int c = S.cls[n];
    if (c >= 0) return c;
    return (n <= 18 || (n <= 20 && !S.full)) ? (int)BC_NARROW : (int)BC_MID;
}

static bool fills_device(const qw_batch_item *items, int count)
{
    long long amps = 0;
    for (int i = 0; i < count; ++i)
        if (items[i].n == 19 || items[i].n == 20) amps += 1ll << items[i].n;
    return amps >= 1ll << 24;
}

static qw_status validate_sched(const BatchSched &S)
{
    if (S.wave_bytes < 0) { set_error("wave_bytes must be >= 0"); return QW_EINVAL; }
    if (S.onchip_nmax != 12 && S.onchip_nmax != 13) { set_error("onchip_nmax must be 12 or 13"); return QW_EINVAL; }
    for (int n = 1; n <= BATCH_MAXN; ++n) {
        const int c = S.cls[n];
        if (c < -1 || c >= BC_COUNT) { set_error("tile class must be -1, 0, 1 or 2"); return QW_EINVAL; }
        if (n <= S.onchip_nmax || c < 0) continue;
        // two orientations of at most TB bits each, the high one with >= 4 passenger bits
        const int tb = class_tb(c);
        if (n <= tb || n - tb > tb - Cfg<float>::LMIN) {
            set_error("tile class " + std::to_string(c) + " cannot hold " + std::to_string(n) + " qubits");
            return QW_EINVAL;
        }
    }
    return QW_OK;
}

struct BatchPlan {
    size_t total = 0;
    size_t off_desc, off_etiles, off_tiles, off_part, off_emm, off_hj, off_q, off_coef, off_items, off_order;
    std::vector<size_t> off_b1, off_b2, off_d;
    int n_etiles = 0, n_tiles = 0, coef_slots = 0, hj_count = 0;
};

// Upper bound on the degree from a bound on the radius computable without the
// GPU: |E(z)| <= sum|h| + sum|J|.
static int degree_bound(const qw_batch_item &it, const double *hJ)
{
    const int n = it.n, np = n * (n - 1) / 2;
    double s = 0.0;
    for (int j = 0; j < n + np; ++j) s += std::fabs(hJ[it.off_hJ + j]);
    const double rmax = s + n * std::fabs(it.gamma);
    // single precision may raise r slightly when rounding gamma/r: pad 1%
    return bessel_cutoff(std::fabs(it.t) * rmax * 1.01 + 1.0) + 2;
}

// Workspace layout; it does not depend on the schedule: every instance of
// n >= 13 has its two work vectors and room for its tiles in the smallest
// tile class.
static BatchPlan plan_batch(const qw_batch_item *items, int count, const double *hJ)
{
    BatchPlan P;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += align256(bytes); return o; };
    P.off_b1.resize(count);
    P.off_b2.resize(count);
    P.off_d.resize(count);
    for (int i = 0; i < count; ++i) {
        const int n = items[i].n;
        const size_t N = size_t(1) << n;
        P.n_etiles += (n > LB_TAB) ? (int)(N >> LB_TAB) : 1;
        if (n >= 13) {
            P.off_b1[i] = take(N * 8);
            P.off_b2[i] = take(N * 8);
            P.n_tiles += (int)(N >> 12);
        } else {
            P.off_b1[i] = P.off_b2[i] = size_t(-1);
        }
        P.off_d[i] = take(N * 4);
        P.coef_slots += degree_bound(items[i], hJ) + 1;
        P.hj_count += n + n * (n - 1) / 2;
    }
    P.off_desc = take(sizeof(BatchDesc) * count);
    P.off_etiles = take(sizeof(int2) * P.n_etiles);
    P.off_tiles = take(sizeof(int2) * std::max(P.n_tiles, 1));
    P.off_part = take(2 * sizeof(double) * P.n_etiles);
    P.off_emm = take(2 * sizeof(double) * count);
    P.off_hj = take(sizeof(double) * P.hj_count);
    P.off_q = take(sizeof(double) * (size_t(1) << LB_TAB) * count);
    P.off_coef = take(sizeof(float2) * P.coef_slots);
    P.off_items = take(sizeof(OnchipItem) * count);
    P.off_order = take(sizeof(int) * count);
    P.total = off;
    return P;
}

static qw_status validate_batch(const qw_batch_item *items, int count, const double *hJ)
{
    if (!items || count < 1 || !hJ) { set_error("items, count >= 1 and the coupling pool are required"); return QW_EINVAL; }
    for (int i = 0; i < count; ++i) {
        const qw_batch_item &it = items[i];
        if (it.n < 1 || it.n > BATCH_MAXN) { set_error("batched instances need 1 <= n <= 22"); return QW_EINVAL; }
        if (!finite(it.gamma) || !finite(it.t) || !(it.tol > 0.0) || !finite(it.tol)) {
            set_error("instance " + std::to_string(i) + ": gamma, t must be finite and tol > 0");
            return QW_EINVAL;
        }
        if (it.off_hJ < 0 || it.off_psi < 0 || it.off_out < 0) { set_error("negative pool offset"); return QW_EINVAL; }
        const int np = it.n * (it.n - 1) / 2;
        for (int j = 0; j < it.n + np; ++j)
            if (!finite(hJ[it.off_hJ + j])) { set_error("non-finite coupling"); return QW_EINVAL; }
        const int vec = 2;  // complex64 pairs: 16-byte alignment of every state
        if ((it.n > 1 && (it.off_psi % vec || it.off_out % vec))) {
            set_error("state offsets must be even (16-byte aligned)");
            return QW_EINVAL;
        }
    }
    return QW_OK;
}

static std::string batch_signature(const qw_batch_item *items, int count)
{
    // size histogram: the schedule depends on the sizes only
    int hist[BATCH_MAXN + 1] = {0};
    for (int i = 0; i < count; ++i) hist[items[i].n]++;
    std::ostringstream os;
    os << "c64";
    for (int n = 1; n <= BATCH_MAXN; ++n)
        if (hist[n]) os << "_" << n << "x" << hist[n];
    return os.str();
}

// Tune file: one line per tuning, "<signature> wave=<bytes> onchip=<n>
// conc=<0|1> classes=<one digit per n = 1..22, '-' = default> ms=<time>"; the
// last line of the batch's signature wins.
static std::string sched_fields(const BatchSched &S)
{
    std::ostringstream os;
    os << "wave=" << S.wave_bytes << " onchip=" << S.onchip_nmax << " conc=" << S.concurrent << " classes=";
    for (int n = 1; n <= BATCH_MAXN; ++n) os << (S.cls[n] < 0 ? '-' : (char)('0' + S.cls[n]));
    return os.str();
}

static bool read_tuned_sched(const char *path, const std::string &sig, BatchSched *out)
{
    if (!path) return false;
    std::ifstream f(path);
    std::string line;
    bool found = false;
    while (std::getline(f, line)) {
        std::istringstream is(line);
        std::string s, tok;
        if (!(is >> s) || s != sig) continue;
        BatchSched S;
        bool ok = true;
        while (is >> tok) {
            const size_t eq = tok.find('=');
            if (eq == std::string::npos) { ok = false; break; }
            const std::string k = tok.substr(0, eq), v = tok.substr(eq + 1);
            if (k == "wave") S.wave_bytes = std::atoll(v.c_str());
            else if (k == "onchip") S.onchip_nmax = std::atoi(v.c_str());
            else if (k == "conc") S.concurrent = std::atoi(v.c_str());
            else if (k == "classes") {
                if ((int)v.size() != BATCH_MAXN) { ok = false; break; }
                for (int n = 1; n <= BATCH_MAXN; ++n) S.cls[n] = (v[n - 1] == '-') ? -1 : (signed char)(v[n - 1] - '0');
            }
        }
        if (ok && validate_sched(S) == QW_OK) {
            *out = S;
            found = true;
        }
    }
    return found;
}

// One launch of a batched call.
struct BLaunch {
    int onchip;      // 1: the one-workgroup launch over the small instances
    int cls, mode, high, stream_hint;
    unsigned grid;
    const int2 *tiles;
    int step;
};

template <int C> static void launch_class(const BLaunch &L, const BatchDesc *dD, hipStream_t s)
{
    const dim3 g(L.grid), b(ClassShape<C>::NT);
    const int st = L.step;
    const int2 *t = L.tiles;
    if (L.stream_hint) {
        if (L.mode == PM_START) hipLaunchKernelGGL((k_pass_batched<C, false, PM_START, true>), g, b, 0, s, dD, t, st);
        else if (L.mode == PM_FUSED && L.high) hipLaunchKernelGGL((k_pass_batched<C, true, PM_FUSED, true>), g, b, 0, s, dD, t, st);
        else if (L.mode == PM_FUSED) hipLaunchKernelGGL((k_pass_batched<C, false, PM_FUSED, true>), g, b, 0, s, dD, t, st);
        else if (L.high) hipLaunchKernelGGL((k_pass_batched<C, true, PM_ADD, true>), g, b, 0, s, dD, t, st);
        else hipLaunchKernelGGL((k_pass_batched<C, false, PM_ADD, true>), g, b, 0, s, dD, t, st);
    } else {
        if (L.mode == PM_START) hipLaunchKernelGGL((k_pass_batched<C, false, PM_START>), g, b, 0, s, dD, t, st);
        else if (L.mode == PM_FUSED && L.high) hipLaunchKernelGGL((k_pass_batched<C, true, PM_FUSED>), g, b, 0, s, dD, t, st);
        else if (L.mode == PM_FUSED) hipLaunchKernelGGL((k_pass_batched<C, false, PM_FUSED>), g, b, 0, s, dD, t, st);
        else if (L.high) hipLaunchKernelGGL((k_pass_batched<C, true, PM_ADD>), g, b, 0, s, dD, t, st);
        else hipLaunchKernelGGL((k_pass_batched<C, false, PM_ADD>), g, b, 0, s, dD, t, st);
    }
}

// Side stream of a device (default priority), for the one-workgroup launch
// beside the passes; created once, kept until the process ends.
static qw_status side_stream(hipStream_t *out)
{
    static std::mutex mu;
    static hipStream_t streams[64] = {};
    int dev = 0;
    QW_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) { set_error("device index out of range"); return QW_EINVAL; }
    std::lock_guard<std::mutex> lock(mu);
    if (!streams[dev]) QW_HIP(hipStreamCreateWithFlags(&streams[dev], hipStreamNonBlocking));
    *out = streams[dev];
    return QW_OK;
}

static void launch_small(unsigned grid, const OnchipItem *ditems, const int *dorder, int nsmall, hipStream_t s)
{
    hipLaunchKernelGGL(k_onchip, dim3(grid), dim3(ONCHIP_NT), 0, s, ditems, dorder, nsmall);
}

// Enqueues the launches on s (captured or not).
static qw_status replay(const std::vector<BLaunch> &Ls, const BatchDesc *dD, const OnchipItem *ditems,
                        const int *dorder, int nsmall, hipStream_t s)
{
    for (const BLaunch &L : Ls) {
        if (L.onchip) launch_small(L.grid, ditems, dorder, nsmall, s);
        else if (L.cls == BC_NARROW) launch_class<BC_NARROW>(L, dD, s);
        else if (L.cls == BC_WIDE_T) launch_class<BC_WIDE_T>(L, dD, s);
        else launch_class<BC_MID>(L, dD, s);
    }
    QW_HIP(hipGetLastError());
    return QW_OK;
}

// The one-workgroup launch on the side stream, from what s has done so far (fork)
// until what it does next (join).  It is never part of a graph: the side stream is
// shared by the threads of the process, and while one of them captured it, the
// launches of another went into that graph.
struct Beside {
    hipStream_t s, side;
    hipEvent_t fork, join;
    bool open = false;
    qw_status start(unsigned grid, const OnchipItem *ditems, const int *dorder, int nsmall)
    {
        QW_HIP(hipEventRecord(fork, s));
        QW_HIP(hipStreamWaitEvent(side, fork, 0));
        launch_small(grid, ditems, dorder, nsmall, side);
        QW_HIP(hipGetLastError());
        QW_HIP(hipEventRecord(join, side));
        open = true;
        return QW_OK;
    }
    qw_status finish()
    {
        if (!open) return QW_OK;
        open = false;
        QW_HIP(hipStreamWaitEvent(s, join, 0));
        return QW_OK;
    }
    ~Beside() { (void)finish(); }
};

// Instantiated graphs of recent calls, keyed by the device and the exact launch
// sequence with every kernel argument (the places of the descriptors, items, order
// and tile tables, which are uploaded anew before each replay; two batches in one
// workspace may have them in different places).  At most GRAPH_CACHE entries; the oldest is destroyed first, after
// its device has finished its work (an eviction waits for the whole device).
static constexpr size_t GRAPH_CACHE = 4;
struct GraphEntry {
    int dev;
    std::string key;
    hipGraphExec_t exec;
};
static std::mutex g_graph_mu;
static std::vector<GraphEntry> g_graphs;

static std::string launch_key(const std::vector<BLaunch> &Ls, const void *desc, const void *items, const void *order,
                              size_t nsmall)
{
    std::ostringstream os;
    os << desc << ',' << items << ',' << order << ',' << nsmall;
    for (const BLaunch &L : Ls)
        os << ';' << L.onchip << ',' << L.cls << ',' << L.mode << ',' << L.high << ',' << L.stream_hint << ','
           << L.grid << ',' << static_cast<const void *>(L.tiles) << ',' << L.step;
    return os.str();
}

struct BatchRun {
    std::vector<int> large, small;   // instance indices
    std::vector<int> K;
    int maxK = 0;
    long long amp_terms = 0;
    int launches = 0, waves = 0;
    int class_count[BC_COUNT] = {0, 0, 0};
};

static qw_status batched_impl(const qw_batch_item *items, int count, const double *hJ, const void *psi_pool,
                              void *out_pool, int method, void *workspace, size_t ws_bytes, BatchSched sch,
                              bool use_graph, hipStream_t s, qw_batch_info *info)
{
    qw_status st = validate_batch(items, count, hJ);
    if (st != QW_OK) return st;
    st = validate_sched(sch);
    if (st != QW_OK) return st;
    sch.full = fills_device(items, count);
    if (method != QW_CHEB && method != QW_CF) { set_error("unknown method"); return QW_EINVAL; }
    if (!psi_pool || !out_pool || !workspace) { set_error("pools and workspace are required"); return QW_EINVAL; }
    if ((reinterpret_cast<uintptr_t>(workspace) & 255) || (reinterpret_cast<uintptr_t>(psi_pool) & 15) ||
        (reinterpret_cast<uintptr_t>(out_pool) & 15)) {
        set_error("workspace must be 256-byte and pools 16-byte aligned");
        return QW_EINVAL;
    }
    const BatchPlan P = plan_batch(items, count, hJ);
    if (ws_bytes < P.total) { set_error("workspace too small: need " + std::to_string(P.total)); return QW_ENOMEM; }
    char *ws = static_cast<char *>(workspace);
    const float2 *psi = static_cast<const float2 *>(psi_pool);
    float2 *out = static_cast<float2 *>(out_pool);

    hipEvent_t ev[5] = {nullptr, nullptr, nullptr, nullptr, nullptr};   // timing 0-2, fork 3, join 4
    const bool timing = info && info->timing;
    struct EvGuard {
        hipEvent_t *e;
        ~EvGuard()
        {
            for (int i = 0; i < 5; ++i)
                if (e[i]) (void)hipEventDestroy(e[i]);
        }
    } eg{ev};
    if (timing)
        for (int i = 0; i < 3; ++i) QW_HIP(hipEventCreate(&ev[i]));
    if (timing) QW_HIP(hipEventRecord(ev[0], s));

    // couplings and descriptors (energy part)
    std::vector<double> hjh(P.hj_count);
    std::vector<BatchDesc> desc(count);
    std::vector<int2> etiles;
    etiles.reserve(P.n_etiles);
    double *dhj = reinterpret_cast<double *>(ws + P.off_hj);
    size_t hoff = 0;
    for (int i = 0; i < count; ++i) {
        const qw_batch_item &it = items[i];
        const int n = it.n, np = n * (n - 1) / 2;
        std::memcpy(hjh.data() + hoff, hJ + it.off_hJ, (n + np) * sizeof(double));
        BatchDesc &b = desc[i];
        std::memset(&b, 0, sizeof(b));
        b.h = dhj + hoff;
        b.J = dhj + hoff + n;
        hoff += n + np;
        b.Q = reinterpret_cast<double *>(ws + P.off_q) + (size_t(1) << LB_TAB) * i;
        b.n = n;
        b.LB = std::min(n, LB_TAB);
        b.tile0 = (int)etiles.size();
        const int nt = (n > LB_TAB) ? (1 << (n - LB_TAB)) : 1;
        b.ntiles = nt;
        for (int t = 0; t < nt; ++t) etiles.push_back(make_int2(i, t));
        b.psi = psi + it.off_psi;
        b.out = out + it.off_out;
        b.d = reinterpret_cast<float *>(ws + P.off_d[i]);
        if (P.off_b1[i] != size_t(-1)) {
            b.B1 = reinterpret_cast<float2 *>(ws + P.off_b1[i]);
            b.B2 = reinterpret_cast<float2 *>(ws + P.off_b2[i]);
        }
    }
    BatchDesc *dD = reinterpret_cast<BatchDesc *>(ws + P.off_desc);
    int2 *dE = reinterpret_cast<int2 *>(ws + P.off_etiles);
    double *dpart = reinterpret_cast<double *>(ws + P.off_part);
    double *demm = reinterpret_cast<double *>(ws + P.off_emm);
    QW_HIP(hipMemcpyAsync(dhj, hjh.data(), hjh.size() * sizeof(double), hipMemcpyHostToDevice, s));
    QW_HIP(hipMemcpyAsync(dD, desc.data(), desc.size() * sizeof(BatchDesc), hipMemcpyHostToDevice, s));
    QW_HIP(hipMemcpyAsync(dE, etiles.data(), etiles.size() * sizeof(int2), hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(k_qtable_batched, dim3((1 << LB_TAB) / 256, count), dim3(256), 0, s, dD);
    hipLaunchKernelGGL(k_energy_batched<false>, dim3(P.n_etiles), dim3(256), 0, s, (const BatchDesc *)dD,
                       (const int2 *)dE, dpart);
    hipLaunchKernelGGL(k_minmax_instances, dim3(count), dim3(256), 0, s, (const BatchDesc *)dD,
                       (const double *)dpart, demm);
    QW_HIP(hipGetLastError());
    std::vector<double> emm(2 * count);
    QW_HIP(hipMemcpyAsync(emm.data(), demm, emm.size() * sizeof(double), hipMemcpyDeviceToHost, s));
    QW_HIP(hipStreamSynchronize(s));

    // per-instance shift, bound, coefficients
    BatchRun run;
    run.K.resize(count);
    std::vector<float2> coefh(P.coef_slots);
    std::vector<OnchipItem> oitems(count);
    float2 *dcoef = reinterpret_cast<float2 *>(ws + P.off_coef);
    int coff = 0;
    for (int i = 0; i < count; ++i) {
        const qw_batch_item &it = items[i];
        BatchDesc &b = desc[i];
        const double emin = emm[2 * i], emax = emm[2 * i + 1];
        if (!finite(emin) || !finite(emax)) { set_error("non-finite energies"); return QW_EINVAL; }
        const double c = 0.5 * (emax + emin);
        double r = 0.5 * (emax - emin) + it.n * std::fabs(it.gamma);
        double g = (r > 0.0) ? it.gamma / r : 0.0;
        if (it.gamma != 0.0 && r > 0.0) {
            float gf = (float)g;
            if (std::fabs((double)gf) > std::fabs(g)) gf = std::nextafter(gf, 0.0f);
            g = (double)gf;
            r = it.gamma / g;
        }
        std::vector<double> alpha;
        int K = 0;
        double err = 0.0;
        if (r > 0.0) {
            if (coefficients(it.t * r, it.tol, method, alpha, &K, &err) != 0) { set_error("coefficients"); return QW_ENOCONV; }
        } else {
            alpha.assign(1, 1.0);  // H = c I: exp(-itc) only
            K = 0;
        }
        const bool small = it.n <= sch.onchip_nmax;
        if (K == 0 && !small) {
            // the grouped two-pass schedule needs one step: pad with c_1 = 0,
            // so the final step gives H~ 0 - 0 + c_0 psi
            alpha.resize(2);
            alpha[1] = 0.0;
            K = 1;
        }
        const int slots = degree_bound(it, hJ) + 1;
        if (K + 1 > slots) { set_error("internal: degree bound exceeded"); return QW_ENOCONV; }
        for (int k = 0; k <= K; ++k) {
            double cr, ci;
            coef_of(alpha, k, cr, ci);
            coefh[coff + k] = make_float2((float)cr, (float)ci);
        }
        b.coef = dcoef + coff;
        coff += slots;
        b.c = c;
        b.inv_r = (r > 0.0) ? 1.0 / r : 0.0;
        b.g = (float)g;
        b.pr = (float)std::cos(it.t * c);
        b.pi = (float)-std::sin(it.t * c);
        b.K = K;
        run.K[i] = K;
        run.amp_terms += (long long)K << it.n;
        if (small) run.small.push_back(i);
        else run.large.push_back(i);
        oitems[i] = OnchipItem{b.psi, b.out, b.d, b.coef, b.g, b.pr, b.pi, it.n, K};
    }
    QW_HIP(hipMemcpyAsync(dcoef, coefh.data(), coefh.size() * sizeof(float2), hipMemcpyHostToDevice, s));
    QW_HIP(hipMemcpyAsync(dD, desc.data(), desc.size() * sizeof(BatchDesc), hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(k_energy_batched<true>, dim3(P.n_etiles), dim3(256), 0, s, (const BatchDesc *)dD,
                       (const int2 *)dE, dpart);
    QW_HIP(hipGetLastError());

    // small class: one persistent launch, costliest first
    std::sort(run.small.begin(), run.small.end(), [&](int a, int b) {
        return ((long long)run.K[a] << items[a].n) > ((long long)run.K[b] << items[b].n);
    });
    OnchipItem *ditems = reinterpret_cast<OnchipItem *>(ws + P.off_items);
    int *dorder = reinterpret_cast<int *>(ws + P.off_order);
    QW_HIP(hipMemcpyAsync(ditems, oitems.data(), oitems.size() * sizeof(OnchipItem), hipMemcpyHostToDevice, s));
    if (!run.small.empty())
        QW_HIP(hipMemcpyAsync(dorder, run.small.data(), run.small.size() * sizeof(int), hipMemcpyHostToDevice, s));

    // large class: waves (greedy in degree order up to wave_bytes of working
    // set), inside a wave one degree-sorted tile table per tile class
    std::vector<int> Lg = run.large;
    std::sort(Lg.begin(), Lg.end(), [&](int a, int b) { return run.K[a] > run.K[b]; });
    std::vector<std::vector<int>> waves;
    {
        std::vector<int> cur;
        size_t cur_bytes = 0;
        for (int i : Lg) {
            const size_t bytes = (size_t(20)) << items[i].n;
            if (sch.wave_bytes && !cur.empty() && cur_bytes + bytes > (size_t)sch.wave_bytes) {
                waves.push_back(cur);
                cur.clear();
                cur_bytes = 0;
            }
            cur.push_back(i);
            cur_bytes += bytes;
        }
        if (!cur.empty()) waves.push_back(cur);
    }
    std::vector<int2> tiles;
    tiles.reserve(P.n_tiles);
    int2 *dT = reinterpret_cast<int2 *>(ws + P.off_tiles);
    std::vector<BLaunch> Ls;
    const bool conc = sch.concurrent && !run.small.empty() && !Lg.empty();
    const unsigned small_grid = (unsigned)std::min<int>((int)run.small.size(), 512);
    if (!run.small.empty() && !conc) Ls.push_back({1, 0, 0, 0, 0, small_grid, nullptr, 0});
    for (auto &w : waves) {
        double wave_vec_bytes = 0.0;   // b1, b2, psi, out (8 B each) and the diagonal per amplitude
        for (int i : w) wave_vec_bytes += std::ldexp(36.0, items[i].n);
        const int hint = wave_vec_bytes > 384.0 * (1 << 20) ? 1 : 0;
        struct ClassTable { int begin = 0; std::vector<int> prefix; };
        ClassTable ct[BC_COUNT];
        int wave_maxK = 0;
        for (int c = 0; c < BC_COUNT; ++c) {
            std::vector<int> mem;
            for (int i : w)
                if (class_for(sch, items[i].n) == c) mem.push_back(i);
            if (mem.empty()) continue;
            std::sort(mem.begin(), mem.end(), [&](int a, int b) { return run.K[a] > run.K[b]; });
            ct[c].begin = (int)tiles.size();
            std::vector<int> cum;
            const int tb = class_tb(c);
            for (int i : mem) {
                const int nt = 1 << (items[i].n - tb);
                for (int t = 0; t < nt; ++t) tiles.push_back(make_int2(i, t));
                cum.push_back((int)tiles.size() - ct[c].begin);
                run.class_count[c]++;
            }
            const int maxK = run.K[mem.front()];
            wave_maxK = std::max(wave_maxK, maxK);
            ct[c].prefix.resize(maxK + 1);
            size_t j = mem.size();
            for (int stp = 0; stp <= maxK; ++stp) {
                while (j > 0 && run.K[mem[j - 1]] < stp) --j;
                ct[c].prefix[stp] = (j > 0) ? cum[j - 1] : 0;
            }
        }
        for (int stp = 0; stp <= wave_maxK; ++stp) {
            const int high = stp & 1;
            for (int c = 0; c < BC_COUNT; ++c) {
                const std::vector<int> &pre = ct[c].prefix;
                const int last = (int)pre.size() - 1;
                if (stp > last) continue;
                const int2 *t0 = dT + ct[c].begin;
                if (stp == 0) {
                    if (pre[0] > 0) Ls.push_back({0, c, PM_START, 0, hint, (unsigned)pre[0], t0, 0});
                    continue;
                }
                // instances with K > stp fuse, those with K == stp finish
                const int nfuse = (stp + 1 <= last) ? pre[stp + 1] : 0;
                if (nfuse > 0) Ls.push_back({0, c, PM_FUSED, high, hint, (unsigned)nfuse, t0, stp});
                if (pre[stp] - nfuse > 0)
                    Ls.push_back({0, c, PM_ADD, high, hint, (unsigned)(pre[stp] - nfuse), t0 + nfuse, stp});
            }
        }
        run.maxK = std::max(run.maxK, wave_maxK);
    }
    if ((int)tiles.size() > P.n_tiles) { set_error("internal: tile table overflow"); return QW_EINVAL; }
    if (!tiles.empty())
        QW_HIP(hipMemcpyAsync(dT, tiles.data(), tiles.size() * sizeof(int2), hipMemcpyHostToDevice, s));
    QW_HIP(hipStreamSynchronize(s));   // host staging buffers go out of scope below

    Beside beside{s, nullptr, nullptr, nullptr};
    if (conc) {
        st = side_stream(&beside.side);
        if (st != QW_OK) return st;
        QW_HIP(hipEventCreateWithFlags(&ev[3], hipEventDisableTiming));
        QW_HIP(hipEventCreateWithFlags(&ev[4], hipEventDisableTiming));
        beside.fork = ev[3];
        beside.join = ev[4];
    }
    auto start_beside = [&]() -> qw_status {
        return conc ? beside.start(small_grid, ditems, dorder, (int)run.small.size()) : QW_OK;
    };
    if (s == nullptr) use_graph = false;   // the null stream cannot be captured
    int graph_cached = 0;
    float graph_ms = 0.f;
    hipGraphExec_t exec = nullptr;
    if (use_graph && !Ls.empty()) {
        int dev = 0;
        QW_HIP(hipGetDevice(&dev));
        const std::string key = launch_key(Ls, dD, ditems, dorder, run.small.size());
        std::lock_guard<std::mutex> lock(g_graph_mu);
        for (const GraphEntry &e : g_graphs)
            if (e.dev == dev && e.key == key) exec = e.exec;
        if (exec) {
            graph_cached = 1;
        } else {
            const auto h0 = std::chrono::steady_clock::now();
            hipGraph_t graph = nullptr;
            QW_HIP(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
            const qw_status rs = replay(Ls, dD, ditems, dorder, (int)run.small.size(), s);
            hipError_t e1 = hipStreamEndCapture(s, &graph);
            if (rs != QW_OK) {
                if (graph) (void)hipGraphDestroy(graph);
                return rs;
            }
            if (e1 != hipSuccess) { set_error(std::string("graph capture: ") + hipGetErrorString(e1)); return QW_EHIP; }
            hipError_t e2 = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
            (void)hipGraphDestroy(graph);
            if (e2 != hipSuccess) { set_error(std::string("graph instantiate: ") + hipGetErrorString(e2)); return QW_EHIP; }
            if (g_graphs.size() >= GRAPH_CACHE) {
                // The oldest graph may still run on a stream of an earlier call
                // (the lock covers lookups and launches, not their execution):
                // its device finishes all work before the graph is destroyed.
                const GraphEntry old = g_graphs.front();
                g_graphs.erase(g_graphs.begin());
                if (old.dev != dev) QW_HIP(hipSetDevice(old.dev));
                const hipError_t es = hipDeviceSynchronize();
                if (old.dev != dev) QW_HIP(hipSetDevice(dev));
                QW_HIP(es);
                (void)hipGraphExecDestroy(old.exec);
            }
            g_graphs.push_back({dev, key, exec});
            graph_ms = std::chrono::duration<float, std::milli>(std::chrono::steady_clock::now() - h0).count();
        }
        if (timing) QW_HIP(hipEventRecord(ev[1], s));
        if ((st = start_beside()) != QW_OK) return st;
        QW_HIP(hipGraphLaunch(exec, s));
    } else {
        if (timing) QW_HIP(hipEventRecord(ev[1], s));
        if ((st = start_beside()) != QW_OK) return st;
        st = replay(Ls, dD, ditems, dorder, (int)run.small.size(), s);
        if (st != QW_OK) return st;
    }
    if ((st = beside.finish()) != QW_OK) return st;
    run.launches = (int)Ls.size() + (conc ? 1 : 0);
    if (timing) QW_HIP(hipEventRecord(ev[2], s));
    QW_HIP(hipStreamSynchronize(s));
    if (info) {
        info->count = count;
        info->small_count = (int)run.small.size();
        info->large_count = (int)run.large.size();
        info->max_K = std::max(run.maxK, [&] { int m = 0; for (int i : run.small) m = std::max(m, run.K[i]); return m; }());
        info->launches = run.launches;
        info->waves = (int)waves.size();
        info->amp_terms = run.amp_terms;
        info->wave_bytes = sch.wave_bytes;
        info->onchip_nmax = sch.onchip_nmax;
        info->concurrent = conc ? 1 : 0;
        info->graph_cached = graph_cached;
        info->graph_ms = graph_ms;
        for (int c = 0; c < BC_COUNT; ++c) info->class_count[c] = run.class_count[c];
        for (int n = 0; n <= BATCH_MAXN; ++n)
            info->tile_class[n] = (n >= 1 && n > sch.onchip_nmax) ? (signed char)class_for(sch, n) : (signed char)-1;
    }
    if (timing) {
        QW_HIP(hipEventElapsedTime(&info->setup_ms, ev[0], ev[1]));
        QW_HIP(hipEventElapsedTime(&info->loop_ms, ev[1], ev[2]));
    }
    return QW_OK;
}

static BatchSched sched_from(const qw_batch_sched *p)
{
    BatchSched S;
    if (!p) return S;
    S.wave_bytes = p->wave_bytes;
    S.onchip_nmax = p->onchip_nmax ? p->onchip_nmax : Cfg<float>::TB;
    S.concurrent = p->concurrent;
    for (int n = 0; n <= BATCH_MAXN; ++n) S.cls[n] = p->tile_class[n];
    return S;
}

static void sched_to(const BatchSched &S, qw_batch_sched *p)
{
    p->wave_bytes = S.wave_bytes;
    p->onchip_nmax = S.onchip_nmax;
    p->concurrent = S.concurrent;
    for (int n = 0; n <= BATCH_MAXN; ++n) p->tile_class[n] = S.cls[n];
}

}  // namespace qw

using namespace qw;

extern "C" {

size_t qw_batched_workspace_bytes_c64(const qw_batch_item *items, int count, const double *hJ_pool)
{
    if (validate_batch(items, count, hJ_pool) != QW_OK) return 0;
    return plan_batch(items, count, hJ_pool).total;
}

static void clear_info(qw_batch_info *info)
{
    if (info) {
        const int t = info->timing;
        std::memset(info, 0, sizeof(*info));
        info->timing = t;
    }
}

qw_status qw_expm_action_batched_c64(const qw_batch_item *items, int count, const double *hJ_pool,
                                     const void *psi_pool, void *out_pool, qw_method method, void *workspace,
                                     size_t ws_bytes, const char *tune_cache, void *stream, qw_batch_info *info)
{
    clear_info(info);
    const qw_status st = validate_batch(items, count, hJ_pool);   // before the sizes are counted
    if (st != QW_OK) return st;
    BatchSched S;
    (void)read_tuned_sched(tune_cache, batch_signature(items, count), &S);
    return batched_impl(items, count, hJ_pool, psi_pool, out_pool, (int)method, workspace, ws_bytes, S, true,
                        reinterpret_cast<hipStream_t>(stream), info);
}

qw_status qw_expm_action_batched_c64_sched(const qw_batch_item *items, int count, const double *hJ_pool,
                                           const void *psi_pool, void *out_pool, qw_method method,
                                           void *workspace, size_t ws_bytes, const qw_batch_sched *sched,
                                           int use_graph, void *stream, qw_batch_info *info)
{
    clear_info(info);
    return batched_impl(items, count, hJ_pool, psi_pool, out_pool, (int)method, workspace, ws_bytes, sched_from(sched),
                        use_graph != 0, reinterpret_cast<hipStream_t>(stream), info);
}

// Coordinate search over the schedule, each candidate timed on one call with
// its graph built beforehand (HIP events around the passes only): the tile
// class of each size bucket in turn, then the one-workgroup limit, running the
// one-workgroup launch beside the passes, and the wave size.
qw_status qw_batched_tune_c64(const qw_batch_item *items, int count, const double *hJ_pool, const void *psi_pool,
                              void *out_pool, void *workspace, size_t ws_bytes, const char *tune_cache,
                              void *stream, qw_batch_sched *best_out)
{
    qw_status st = validate_batch(items, count, hJ_pool);   // before the sizes are counted
    if (st != QW_OK) return st;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    auto time_of = [&](const BatchSched &S, float *ms) -> qw_status {
        qw_batch_info bi{};
        qw_status st = batched_impl(items, count, hJ_pool, psi_pool, out_pool, QW_CHEB, workspace, ws_bytes, S, true,
                                    s, &bi);   // builds (or finds) the graph
        if (st != QW_OK) return st;
        bi = qw_batch_info{};
        bi.timing = 1;
        st = batched_impl(items, count, hJ_pool, psi_pool, out_pool, QW_CHEB, workspace, ws_bytes, S, true, s, &bi);
        *ms = bi.loop_ms;
        return st;
    };
    int present[BATCH_MAXN + 1] = {0};
    for (int i = 0; i < count; ++i) present[items[i].n] = 1;
    BatchSched best;
    best.full = fills_device(items, count);
    float best_ms = 0.f;
    st = time_of(best, &best_ms);
    if (st != QW_OK) return st;
    auto consider = [&](const BatchSched &S) -> qw_status {
        if (validate_sched(S) != QW_OK) return QW_OK;   // not a valid candidate for these sizes
        float ms = 0.f;
        const qw_status st2 = time_of(S, &ms);
        if (st2 != QW_OK) return st2;
        if (ms < best_ms) {
            best_ms = ms;
            best = S;
        }
        return QW_OK;
    };
    const int buckets[][2] = {{13, 16}, {17, 18}, {19, 20}, {21, 22}};
    for (const auto &bk : buckets) {
        bool any = false;
        for (int n = bk[0]; n <= bk[1]; ++n) any = any || present[n];
        if (!any) continue;
        for (int c = 0; c < BC_COUNT; ++c) {
            BatchSched S = best;
            for (int n = bk[0]; n <= bk[1]; ++n) S.cls[n] = (signed char)c;
            bool same = true;
            for (int n = bk[0]; n <= bk[1]; ++n)
                if (present[n] && n > S.onchip_nmax && class_for(S, n) != class_for(best, n)) same = false;
            if (same) continue;
            st = consider(S);
            if (st != QW_OK) return st;
        }
    }
    if (present[13]) {
        BatchSched S = best;
        S.onchip_nmax = (best.onchip_nmax == 13) ? 12 : 13;
        if (S.onchip_nmax == 12) S.cls[13] = BC_NARROW;
        st = consider(S);
        if (st != QW_OK) return st;
    }
    {
        BatchSched S = best;
        S.concurrent = !best.concurrent;
        st = consider(S);
        if (st != QW_OK) return st;
    }
    for (long long w : {512ll << 20, 256ll << 20, 128ll << 20}) {
        BatchSched S = best;
        S.wave_bytes = w;
        st = consider(S);
        if (st != QW_OK) return st;
    }
    if (best_out) sched_to(best, best_out);
    if (tune_cache) {
        FILE *f = std::fopen(tune_cache, "a");
        if (!f) { set_error(std::string("cannot write tune cache ") + tune_cache); return QW_EINVAL; }
        std::fprintf(f, "%s %s ms=%.3f\n", batch_signature(items, count).c_str(), sched_fields(best).c_str(), best_ms);
        std::fclose(f);
    }
    return QW_OK;
}

}  // extern "C"

// The whole recurrence of one instance in a single launch: the vectors stay in
// the registers of W = 2^HC workgroups, one tile of 2^T consecutive amplitudes
// each, and only b_{k+1} travels between them.
#pragma once

#include "qw_device.h"
#include "qw_internal.h"
#include "qw_kernels.h"

#include <atomic>
#include <type_traits>

namespace qw {

typedef int qw_i4 __attribute__((ext_vector_type(4)));

static constexpr int RES_XCDS = 8;
// One flag per wave, each on a cache line of its own (flags that shared lines
// tripled the time of a round over 256 workgroups), and the start word and the
// mask of XCDs on two more lines.
static constexpr int RES_LINE = 32;            // 4-byte words per line
static constexpr int RES_MAXFLAGS = 4096;
// Looks at the start word, 0.4 and 6 ms.  Only a cooperative launch, of which a
// process runs one at a time, waits long: it needs every CU, so a plain one that
// holds some and waits for more has to go on without them (k_resident's start).
static constexpr int RES_PATIENCE = 1 << 9, RES_PATIENCE_COOP = 1 << 13;
static constexpr int RES_POLLS = 1 << 24;      // looks at a flag, seconds
int wait_polls();                              // the same, or what a test has set (qw_action.hip)

// Small host arrays travel as kernel arguments (a launch keeps its own copy, so
// nothing on the host has to outlive the call and no copy engine is involved).
struct PutBlob {
    static constexpr int WORDS = 440;   // 8-byte words; arguments stay below 4 KB
    uint64_t v[WORDS];
};
struct NoBlob {};

// One exponential of a chain: psi stays in registers from one to the next (an
// anneal of 128 exponentials of about five terms at 18 qubits: 2.65 ms, with a
// launch and an upload each 4.79).
template <typename R> struct ResStep {
    double c, inv_r;      // d~ = (E - c) inv_r
    R g, pr, pi;          // gamma / r, global phase
    int K, coef;          // degree, place of c_0 .. c_K
};

template <typename R> struct ResArgs {
    using C = typename Cplx<R>::T;
    const C *psi;
    C *out;               // may be psi
    const R *diag;        // the caller's energies, or NULL: from (h, J)
    const double *hJ;     // device: h (n), J (packed)
    ResStep<R> first;
    const ResStep<R> *more;   // device: the nsteps - 1 steps after the first
    int nsteps;
    const C *coef;        // device: coefficients of all steps
    C *X0, *X1;           // exchange buffers of 2^n
    R *d;                 // 2^n, used only when the workgroups cannot all start
    int *start, *flags;   // 2 and RES_MAXFLAGS lines, their words in use cleared before the launch
    R two, sub;           // Clenshaw 2 and 1, Horner's rule 1 and 0
    int n;
    int stride, sel;      // workgroups with blockIdx.x % stride == sel take part
    int patience;         // looks at the start word before giving up on a common start (< 0: the default)
    int polls;            // looks at a flag before giving up on a partner
};

// E(z) from couplings in LDS (h, then J packed), in double.
__device__ inline double energy_direct(const double *hJ, int n, uint32_t z)
{
    double e = 0.0;
    const double *J = hJ + n;
#pragma unroll 1
    for (int j = 0; j < n; ++j) {
        double f = hJ[j];
#pragma unroll 1
        for (int k = j + 1; k < n; ++k) {
            const double x = *J++;
            f += ((z >> k) & 1) ? -x : x;
        }
        e += ((z >> j) & 1) ? -f : f;
    }
    return e;
}

// Energies of a tile of 2^min(n, T) consecutive states, in double.  The tile's
// bits split into a low and a high half,
//   E = A[lo] + B[hi] + sum_{j in low half} s_j G_j[hi],
// where A holds the low half's couplings and fields and the constant of the bits
// above the tile, B the high half's, G_j the couplings of bit j to the high
// half; a state then costs 2 + T / 2 LDS reads instead of the n (n + 1) / 2
// couplings (over 32 us at 17 qubits, all latency; the tables take 2 us).
template <int T> struct TileEnergy {
    static constexpr int HA = T / 2, HB = T - T / 2;
    double hJ[32 + 32 * 31 / 2];
    double F[T], C, A[1 << HA], B[1 << HB], G[HA > 0 ? HA : 1][1 << HB];

    // All NT threads of the block; ends with the tables visible to them.
    template <int NT> __device__ void build(const double *dhJ, int n, uint32_t w)
    {
        const int tid = threadIdx.x;
        for (int i = tid; i < n + n * (n - 1) / 2; i += NT) hJ[i] = dhJ[i];
        __syncthreads();
        const int nt = n < T ? n : T, a = nt / 2, b = nt - a;
        const double *J = hJ + n;
        auto flip = [](uint32_t z, int k, double x) { return ((z >> k) & 1) ? -x : x; };
        if (tid < nt) {
            double f = hJ[tid];
            for (int k = nt; k < n; ++k) f += flip(w, k - nt, J[pair_off(n, tid, k)]);
            F[tid] = f;
        } else if (tid == NT - 1) {
            double c = 0.0;
            for (int j = nt; j < n; ++j) {
                double f = hJ[j];
                for (int k = j + 1; k < n; ++k) f += flip(w, k - nt, J[pair_off(n, j, k)]);
                c += flip(w, j - nt, f);
            }
            C = c;
        }
        __syncthreads();
        for (int i = tid; i < (1 << a) + (1 << b); i += NT) {
            const bool hi = i >= (1 << a);
            const int z = hi ? i - (1 << a) : i, o = hi ? a : 0, m = hi ? b : a;
            double e = hi ? 0.0 : C;
            for (int j = 0; j < m; ++j) {
                double f = F[o + j];
                for (int k = j + 1; k < m; ++k) f += flip(z, k, J[pair_off(n, o + j, o + k)]);
                e += flip(z, j, f);
            }
            if (hi) B[z] = e;
            else A[z] = e;
        }
        for (int i = tid; i < (a << b); i += NT) {
            const int j = i >> b, z = i & ((1 << b) - 1);
            double g = 0.0;
            for (int k = 0; k < b; ++k) g += flip(z, k, J[pair_off(n, j, a + k)]);
            G[j][z] = g;
        }
        __syncthreads();
    }
    __device__ double at(int n, uint32_t e) const
    {
        const int a = (n < T ? n : T) / 2;
        const uint32_t lo = e & ((1u << a) - 1), hi = e >> a;
        double x = A[lo] + B[hi];
        for (int j = 0; j < a; ++j) x += ((lo >> j) & 1) ? -G[j][hi] : G[j][hi];
        return x;
    }
};

#define QW_AGENT __HIP_MEMORY_SCOPE_AGENT
enum : int { RES_CNT = 0xfff, RES_TRY = 1 << 28, RES_ABORT = 1 << 29, RES_GO = 1 << 30 };
// words of the first line: joined and decided, size of a team, its barrier's count
enum : int { RES_STATE, RES_TEAM, RES_MET };

// Common start of W workgroups (one thread of each): 1 once all of them run.
// From then on every wait between them ends, since none has to be placed any
// more.  After `patience` looks the first one to lose patience decides for all,
// by how many had joined when it did: if some had not, those that had are a team
// (0; *id: number of this one), and who comes later leaves (-1).
__device__ inline int res_join(int *state, int W, int patience, int *id)
{
    const int before = __hip_atomic_fetch_add(state, 1, __ATOMIC_RELAXED, QW_AGENT);
    *id = before & RES_CNT;
    if (before & RES_TRY) return -1;   // without this one the count cannot have been W
    for (int s = before + 1;; s = __hip_atomic_load(state, __ATOMIC_RELAXED, QW_AGENT)) {
        if (s & RES_ABORT) return 0;
        if (s & RES_GO) return 1;
        if (s & RES_TRY) continue;
        if ((s & RES_CNT) == W) return 1;
        if (patience-- <= 0) {
            const int old = __hip_atomic_fetch_or(state, (int)RES_TRY, __ATOMIC_RELAXED, QW_AGENT);
            if (old & RES_TRY) continue;
            const int m = old & RES_CNT;
            if (m != W) {
                __hip_atomic_store(state + RES_TEAM, m, __ATOMIC_RELAXED, QW_AGENT);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
            (void)__hip_atomic_fetch_or(state, (int)(m == W ? RES_GO : RES_ABORT), __ATOMIC_RELAXED, QW_AGENT);
            return m == W;
        }
    }
}

// The recurrence by the workgroups that had started when the common start failed,
// from global memory with a barrier per term.  All of them run, so the barrier's
// waits end.  Bounded by the barrier's round trips (17 us) and, at the largest
// sizes, by the reads of n flips: 17 qubits 21 us per term by 254 workgroups, 25 by
// 24; 20 qubits 37 by 248, 75 by 49.  One workgroup alone, which ran it before after
// 0.1 s, took a second for a call of 20 qubits: eight streams of mixed sizes needed
// 5.7 s for what takes 0.14 one after another and 0.12 now.
template <typename R, int NT>
__device__ __forceinline__ void res_team(const ResArgs<R> &a, const double *hJ, int id, int m)
{
    using C = typename Cplx<R>::T;
    using V = CVec<R>;
    constexpr int VE = V::N, B0 = VE - 1;   // lowest bit whose flip is another vector
    const uint32_t nvec = (1u << a.n) / VE, first = id * NT + threadIdx.x, step = m * NT;
    __shared__ int gone;
    int met = 0;
    bool lost = false;
    auto meet = [&]() {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the wave's stores have reached the L2
        __syncthreads();
        met += m;
        if (threadIdx.x == 0) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            (void)__hip_atomic_fetch_add(a.start + RES_MET, 1, __ATOMIC_RELAXED, QW_AGENT);
            int left = lost ? 0 : a.polls;
            while (left > 0 && __hip_atomic_load(a.start + RES_MET, __ATOMIC_RELAXED, QW_AGENT) < met) --left;
            gone = left <= 0;
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");   // the L1 is the workgroup's
        }
        __syncthreads();
        lost = gone != 0;
    };
#pragma unroll 1
    for (int i = 0; i < a.nsteps; ++i) {
        const ResStep<R> st = i == 0 ? a.first : a.more[i - 1];
        const C *coef = a.coef + st.coef, *psi = i == 0 ? a.psi : a.out;
        C *b1 = a.X0, *b2 = a.X1;
        const C cK = coef[st.K];
#pragma unroll 1
        for (uint32_t q = first; q < nvec; q += step) {
            const uint32_t z = q * VE;
            const V p = ld_v<R, false>(psi + z);
            V x, y;
#pragma unroll
            for (int v = 0; v < VE; ++v) {
                const double E = a.diag ? (double)a.diag[z + v] : energy_direct(hJ, a.n, z + v);
                a.d[z + v] = (R)((E - st.c) * st.inv_r);
                x.v[v] = C{fmad(cK.x, p.v[v].x, -(cK.y * p.v[v].y)), fmad(cK.x, p.v[v].y, cK.y * p.v[v].x)};
                y.v[v] = C{fmad(st.pr, x.v[v].x, -(st.pi * x.v[v].y)), fmad(st.pr, x.v[v].y, st.pi * x.v[v].x)};
            }
            st_v<R, false>(b1 + z, x);
            if (st.K == 0) st_v<R, false>(a.out + z, y);
        }
#pragma unroll 1
        for (int k = st.K - 1; k >= 0; --k) {
            meet();
            const C ck = coef[k];
            const R scale = (k == 0) ? R(1) : a.two, g = lost ? R(NAN) : st.g;
#pragma unroll 1
            for (uint32_t q = first; q < nvec; q += step) {
                const uint32_t z = q * VE;
                const V b = ld_v<R, false>(b1 + z);
                V f, s, o;
#pragma unroll
                for (int v = 0; v < VE; ++v) {
                    f.v[v] = (VE == 2) ? b.v[VE - 1 - v] : C{R(0), R(0)};
                    s.v[v] = C{R(0), R(0)};
                }
                if (k < st.K - 1) s = ld_v<R, false>(b2 + z);
                const V p = ld_v<R, false>(psi + z);
#pragma unroll 1
                for (int j = B0; j < a.n; j += 4) {
                    V x[4];
#pragma unroll
                    for (int l = 0; l < 4; ++l)
                        if (j + l < a.n) x[l] = ld_v<R, false>(b1 + (z ^ (1u << (j + l))));
#pragma unroll
                    for (int l = 0; l < 4; ++l)
                        if (j + l < a.n)
#pragma unroll
                            for (int v = 0; v < VE; ++v) {
                                f.v[v].x += x[l].v[v].x;
                                f.v[v].y += x[l].v[v].y;
                            }
                }
#pragma unroll
                for (int v = 0; v < VE; ++v) {
                    const R d = a.d[z + v];
                    const R hr = fmad(d, b.v[v].x, g * f.v[v].x), hi = fmad(d, b.v[v].y, g * f.v[v].y);
                    const R tr = fmad(scale, hr, -(a.sub * s.v[v].x)), ti = fmad(scale, hi, -(a.sub * s.v[v].y));
                    const C w{tr + fmad(ck.x, p.v[v].x, -(ck.y * p.v[v].y)), ti + fmad(ck.x, p.v[v].y, ck.y * p.v[v].x)};
                    o.v[v] = k > 0 ? w : C{fmad(st.pr, w.x, -(st.pi * w.y)), fmad(st.pr, w.y, st.pi * w.x)};
                }
                st_v<R, false>((k > 0 ? b2 : a.out) + z, o);
            }
            C *t = b1;
            b1 = b2;
            b2 = t;
        }
        // the next step starts over b1, which the others may still be reading
        if (i + 1 < a.nsteps) meet();
    }
}

// The vector of the lane that a DPP control names.
template <typename R, int CTRL> __device__ __forceinline__ CVec<R> lane_flip(const CVec<R> &x)
{
    qw_i4 a = __builtin_bit_cast(qw_i4, x);
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = __builtin_amdgcn_update_dpp(0, a[i], CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(CVec<R>, a);
}

// One workgroup holds 2^T consecutive amplitudes of b_{k+1}, b_{k+2}, psi and the
// diagonal in registers; tile w has the index bits T.. equal to w.  A term:
//   - b_{k+1} goes to the workgroup's LDS tile and, for HC > 0, to one of two
//     exchange buffers; each wave then raises its own flag to the round's number;
//   - the flips of bit 0 (complex64) and of the bits that number a thread's own
//     vectors come from its registers, those of three lane bits by DPP, the other
//     lane bits and the wave bits from the LDS tile, while the flags travel;
//   - a wave waits for the HC waves (one per flipped tile bit) that hold its
//     flips, loads their vectors and forms b_k.
// A wave overwrites a buffer only after the flags of the next round, which its
// partners raise after they have read it, so two buffers and one barrier per
// term (of the workgroup, for its LDS tile) suffice.
// A wave that gives up on a partner goes on with NaN in all its amplitudes.  It may
// then overwrite a buffer that a late partner still reads, which finds there what it
// came for or NaN, and passes that on: a finite amplitude is a right one.
// Every exchanged word passes the L1 (sc1 loads); stores go through to memory
// unless all workgroups sit on one XCD, whose L2 they then share.
// What bounds it: the latency of that round, not bytes: about 0.3 us for the
// LDS tile alone, 0.9-1.4 us through one L2, 2.0 us over 128 workgroups on all
// XCDs; from 18 qubits the exchanged bytes (8 partners of 8 B per amplitude:
// 67 MB per term at 20 qubits, 10.5 TB/s).  The passes it replaces paid a launch
// and a round trip of every vector per term (launch_resident lists both).
// BLOB = PutBlob (one workgroup): the coefficients and, behind them, (h, J) come
// with the launch.
template <typename R, int T, int NT, int HC, int WPE, typename BLOB = NoBlob>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(WPE))) k_resident(ResArgs<R> a, BLOB blob)
{
    using C = typename Cplx<R>::T;
    using V = CVec<R>;
    constexpr int VE = V::N;                             // amplitudes per 16-byte vector
    constexpr int PER = (1 << T) / (NT * VE);            // vectors per thread
    constexpr int LT = (NT == 1024) ? 10 : (NT == 512) ? 9 : (NT == 256) ? 8 : (NT == 128) ? 7 : 6;
    constexpr int QB = (PER == 8) ? 3 : (PER == 4) ? 2 : (PER == 2) ? 1 : 0;
    static_assert((1 << LT) == NT && PER >= 1 && (1 << QB) == PER, "tile shape");
    constexpr int W = 1 << HC, NW = NT / 64;
    static_assert(W * NW <= RES_MAXFLAGS, "one flag per wave");
    constexpr bool GUARD = (HC == 0 && NT == 64);        // the smallest shape also takes n < T
    __shared__ V lds[2][PER * NT];
    __shared__ TileEnergy<T> en;
    __shared__ int go, team[2];

    int w = 0;
    if constexpr (HC > 0) {
        if ((int)(blockIdx.x % a.stride) != a.sel) return;
        w = __builtin_amdgcn_readfirstlane(blockIdx.x / a.stride);
    }
    const int tid = threadIdx.x;
    const int n = a.n;
    constexpr bool INLINE = std::is_same<BLOB, PutBlob>::value;
    static_assert(!INLINE || HC == 0, "one workgroup");
    __shared__ alignas(16) uint64_t words[INLINE ? PutBlob::WORDS : 1];
    const C *coef = a.coef;
    const double *hJ = a.hJ;
    if constexpr (INLINE) {
        for (int i = tid; i < PutBlob::WORDS; i += NT) words[i] = blob.v[i];
        coef = reinterpret_cast<const C *>(words);
        hJ = reinterpret_cast<const double *>(coef + a.first.K + 1);
        __syncthreads();
    }
    if (!a.diag) en.template build<NT>(hJ, n, w);
    bool near = false;   // all workgroups on one XCD: its L2 is their common memory
    if constexpr (HC > 0) {
        if (tid == 0) {
            const int xcc = __builtin_amdgcn_s_getreg(20 | (3 << 11));   // HW_REG_XCC_ID, 4 bits
            (void)__hip_atomic_fetch_or(a.start + RES_LINE, 1 << xcc, __ATOMIC_RELAXED, QW_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            int id, ok = res_join(a.start, W, a.patience, &id);
            if (ok == 1) {
                const int m = __hip_atomic_load(a.start + RES_LINE, __ATOMIC_RELAXED, QW_AGENT);
                if ((m & (m - 1)) == 0) ok = 2;
            } else if (ok == 0) {
                team[0] = id;
                team[1] = __hip_atomic_load(a.start + RES_TEAM, __ATOMIC_RELAXED, QW_AGENT);
            }
            go = ok;
        }
        __syncthreads();
        const int ok = __builtin_amdgcn_readfirstlane(go);
        if (ok <= 0) {
            if (ok == 0)
                res_team<R, NT>(a, en.hJ, __builtin_amdgcn_readfirstlane(team[0]), __builtin_amdgcn_readfirstlane(team[1]));
            return;
        }
        near = (ok == 2);
    }

    V b1[PER], b2[PER], ps[PER];
    R d[PER][VE];
    const int lane = tid & 63, wave = tid >> 6;
    const uint32_t base = (uint32_t)w << T;
    auto inside = [&](int q) { return !GUARD || (uint32_t)(q * NT + tid) * VE < (1u << n); };
    C ck{R(0), R(0)};   // lane l: c_{64 i + l}
    auto lane_value = [&](R x, int l) -> R {
        if constexpr (sizeof(R) == 4) {
            return __builtin_bit_cast(R, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), l));
        } else {
            const uint64_t u = __builtin_bit_cast(uint64_t, x);
            const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)u, l);
            const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l);
            return __builtin_bit_cast(R, ((uint64_t)hi << 32) | lo);
        }
    };
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        if (inside(q)) {
            ps[q] = ld_v<R, false>(a.psi + base + (uint32_t)(q * NT + tid) * VE);
        } else {
#pragma unroll
            for (int v = 0; v < VE; ++v) ps[q].v[v] = C{R(0), R(0)};
        }
    }

    const auto rs0 = __builtin_amdgcn_make_buffer_rsrc((void *)a.X0, 0, (int)(sizeof(C) << n), 0x00027000);
    const auto rs1 = __builtin_amdgcn_make_buffer_rsrc((void *)a.X1, 0, (int)(sizeof(C) << n), 0x00027000);
    constexpr int SC1 = 16;   // cache policy: past the L1, and (stores) through to memory
    // lane j < HC looks at the flag of the wave that holds the flips of tile bit T + j
    const int *peer = a.flags + (size_t)(((w ^ (lane < HC ? 1 << lane : 0)) * NW + wave) * RES_LINE);
    int *mine = a.flags + (size_t)((w * NW + wave) * RES_LINE);
    bool lost = false;
    int t = 0;

    auto publish = [&]() {   // b1 to the LDS tile and the exchange buffer of this round
        ++t;
        if constexpr (HC > 0) {
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                const qw_i4 x = __builtin_bit_cast(qw_i4, b1[q]);
                const int vo = (q * NT + tid) * 16, so = (int)(base * sizeof(C));
                if (near) __builtin_amdgcn_raw_buffer_store_b128(x, (t & 1) ? rs1 : rs0, vo, so, 0);
                else __builtin_amdgcn_raw_buffer_store_b128(x, (t & 1) ? rs1 : rs0, vo, so, SC1);
            }
        }
#pragma unroll
        for (int q = 0; q < PER; ++q) lds[t & 1][q * NT + tid] = b1[q];
        if constexpr (HC > 0) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the wave's part has arrived
            if (lane == 0) __hip_atomic_store(mine, t, __ATOMIC_RELAXED, QW_AGENT);
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    };

    for (int step = 0; step < a.nsteps; ++step) {
        ResStep<R> st = a.first;
        if (step > 0) st = wave_uniform(a.more[step - 1]);
        auto load_coef = [&](int k) {
            const int i = (k & ~63) + lane;
            if (i <= st.K) ck = coef[st.coef + i];
        };
        load_coef(st.K);
        const R cKr = lane_value(ck.x, st.K & 63), cKi = lane_value(ck.y, st.K & 63);
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const uint32_t z = base + (uint32_t)(q * NT + tid) * VE;
#pragma unroll
            for (int v = 0; v < VE; ++v) {
                const C p = ps[q].v[v];
                b1[q].v[v] = C{fmad(cKr, p.x, -(cKi * p.y)), fmad(cKr, p.y, cKi * p.x)};
                b2[q].v[v] = C{R(0), R(0)};
                d[q][v] = R(0);
                if (inside(q)) {
                    const double E = a.diag ? (double)a.diag[z + v] : en.at(n, z + v - base);
                    d[q][v] = (R)((E - st.c) * st.inv_r);
                }
            }
        }
        if (st.K > 0) publish();
        for (int k = st.K - 1; k >= 0; --k) {
            if ((k & 63) == 63) load_coef(k);
            const R cr = lane_value(ck.x, k & 63), ci = lane_value(ck.y, k & 63);
            const R scale = (k == 0) ? R(1) : a.two;
            R sr[PER][VE], si[PER][VE];
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                if constexpr (VE == 2) {
                    sr[q][0] = b1[q].v[1].x;
                    si[q][0] = b1[q].v[1].y;
                    sr[q][VE - 1] = b1[q].v[0].x;
                    si[q][VE - 1] = b1[q].v[0].y;
                } else {
                    sr[q][0] = R(0);
                    si[q][0] = R(0);
                }
                auto add = [&](const V &x) {
#pragma unroll
                    for (int v = 0; v < VE; ++v) {
                        sr[q][v] += x.v[v].x;
                        si[q][v] += x.v[v].y;
                    }
                };
#pragma unroll
                for (int j = 0; j < QB; ++j) add(b1[q ^ (1 << j)]);
                // lane bits 0, 1 and 3 within the row (DPP), the others from the LDS tile
                add(lane_flip<R, 0xb1>(b1[q]));    // quad_perm 1 0 3 2
                add(lane_flip<R, 0x4e>(b1[q]));    // quad_perm 2 3 0 1
                add(lane_flip<R, 0x128>(b1[q]));   // row_ror 8
#pragma unroll
                for (int j = 2; j < LT; ++j)
                    if (j != 3) add(lds[t & 1][q * NT + (tid ^ (1 << j))]);
            }
            if constexpr (HC > 0) {
                if (!lost) {
                    int left = a.polls;
                    while (__any(lane < HC && __hip_atomic_load(peer, __ATOMIC_RELAXED, QW_AGENT) < t))
                        if (--left <= 0) {
                            lost = true;
                            st.g = R(NAN);
                            break;
                        }
                }
                asm volatile("" ::: "memory");
#pragma unroll
                for (int q = 0; q < PER; ++q) {
                    V x[HC > 0 ? HC : 1];
#pragma unroll
                    for (int j = 0; j < HC; ++j) {
                        // partner's tile in the scalar offset: one vector offset for all of them
                        const int so = (int)((((uint32_t)w ^ (1u << j)) << T) * sizeof(C));
                        const qw_i4 y = __builtin_amdgcn_raw_buffer_load_b128((t & 1) ? rs1 : rs0, (q * NT + tid) * 16,
                                                                              so, SC1);
                        x[j] = __builtin_bit_cast(V, y);
                    }
#pragma unroll
                    for (int j = 0; j < HC; ++j)
#pragma unroll
                        for (int v = 0; v < VE; ++v) {
                            sr[q][v] += x[j].v[v].x;
                            si[q][v] += x[j].v[v].y;
                        }
                }
            }
#pragma unroll
            for (int q = 0; q < PER; ++q)
#pragma unroll
                for (int v = 0; v < VE; ++v) {
                    const C b = b1[q].v[v], s = b2[q].v[v], p = ps[q].v[v];
                    const R hr = fmad(d[q][v], b.x, st.g * sr[q][v]), hi = fmad(d[q][v], b.y, st.g * si[q][v]);
                    const R tr = fmad(scale, hr, -(a.sub * s.x)), ti = fmad(scale, hi, -(a.sub * s.y));
                    b2[q].v[v] = C{tr + fmad(cr, p.x, -(ci * p.y)), ti + fmad(cr, p.y, ci * p.x)};
                }
            // b2 holds b_k: the two swap roles; amplitudes beyond n stay zero
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                if (!inside(q))
#pragma unroll
                    for (int v = 0; v < VE; ++v) b2[q].v[v] = C{R(0), R(0)};
                const V x = b1[q];
                b1[q] = b2[q];
                b2[q] = x;
            }
            if (k > 0) publish();
        }
#pragma unroll
        for (int q = 0; q < PER; ++q)
#pragma unroll
            for (int v = 0; v < VE; ++v) {
                const C y = b1[q].v[v];
                ps[q].v[v] = C{fmad(st.pr, y.x, -(st.pi * y.y)), fmad(st.pr, y.y, st.pi * y.x)};
            }
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        if (!inside(q)) continue;
        st_v<R, false>(a.out + base + (uint32_t)(q * NT + tid) * VE, ps[q]);
    }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

// Sizes that run in one launch.  Above them the passes are faster: complex64 21
// qubits would take 2^13 amplitudes per workgroup, more than its registers hold
// (41 us per term with the spills, 17 in passes); complex128 20 likewise.
template <typename R> constexpr int resident_nmax() { return sizeof(R) == 4 ? 20 : 19; }

// Compute units on which stream s may run; 0 if some of its device's are masked
// off, so that nothing is known of how many an XCD has left (qw_action.hip).
int stream_cus(hipStream_t s);
// For tests: whether a launch of several workgroups is to be refused (qw_action.hip);
// `back`: the backward one of two sweeps.
bool launch_refused(bool back = false);

// Whether `groups` workgroups of a kernel find room side by side on `cus` compute
// units: the whole device has 256, a partition of it as few as 32.  Where they do
// not, a cooperative launch would be refused, and a plain one would wait in vain
// for its common start.  per_cu: the kernel's, asked for once.
inline bool groups_fit(const void *kernel, int threads, int groups, int cus, std::atomic<int> &per_cu)
{
    int m = per_cu.load(std::memory_order_relaxed);
    if (m == 0) {
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&m, kernel, threads, 0) != hipSuccess) {
            (void)hipGetLastError();
            return false;
        }
        per_cu.store(m, std::memory_order_relaxed);
    }
    return (int64_t)m * cus >= groups;
}

// Launches the recurrence, or with a == NULL only tells whether it would be
// launched (hipSuccess) or has no room on `cus` compute units.
template <typename R, int T, int NT, int HC, int STRIDE, int WPE, bool COOP>
static hipError_t res_launch(const ResArgs<R> *ask, hipStream_t s, const PutBlob *blob, int cus)
{
    static std::atomic<int> per_cu{0};
    if constexpr (HC > 0) {
        const int groups = (COOP ? STRIDE : 1) << HC;
        if (!groups_fit(reinterpret_cast<const void *>(&k_resident<R, T, NT, HC, WPE>), NT, groups, cus, per_cu) ||
            (ask && launch_refused()))
            return hipErrorCooperativeLaunchTooLarge;
    }
    if (!ask) return hipSuccess;
    ResArgs<R> a = *ask;
    // launches take turns over the XCDs, so that calls on several streams do not
    // crowd one
    static std::atomic<unsigned> turn{0};
    a.stride = STRIDE;
    a.sel = (STRIDE > 1) ? (int)(turn.fetch_add(1, std::memory_order_relaxed) % STRIDE) : 0;
    if (a.patience < 0) a.patience = COOP ? RES_PATIENCE_COOP : RES_PATIENCE;
    const dim3 grid((1u << HC) * STRIDE), block(NT);
    if constexpr (HC == 0) {
        if (blob) {
            hipLaunchKernelGGL((k_resident<R, T, NT, HC, WPE, PutBlob>), grid, block, 0, s, a, *blob);
            return hipGetLastError();
        }
    }
    if constexpr (COOP) {
        NoBlob none;
        void *args[] = {&a, &none};
        return hipLaunchCooperativeKernel(reinterpret_cast<const void *>(&k_resident<R, T, NT, HC, WPE>), grid, block,
                                          args, 0, s);
    } else {
        hipLaunchKernelGGL((k_resident<R, T, NT, HC, WPE>), grid, block, 0, s, a, NoBlob{});
        return hipGetLastError();
    }
}

// Whether the size's shape needs a cooperative launch: one workgroup fills a CU,
// so two such calls on two streams could each hold half the chip and wait for
// the other half.  The other shapes of several workgroups have at most 256
// threads of at most 128 registers, four to a CU, and a process has four
// hardware queues.  (Shapes of 512 and 1024 threads with more registers were up
// to 15 % faster per term, but four threads calling at once then met failed
// starts.)  A cooperative launch costs 8 us more than a plain one.
template <typename R> constexpr bool resident_coop(int n) { return n >= (sizeof(R) == 4 ? 19 : 18); }

// Smallest degree that takes the one launch with the caller's diagonal.  A
// cooperative launch of 256 workgroups costs 18-27 us more than a pass and a term
// 3-6 us less, so the passes are faster below (in us, passes against one launch):
// complex64 19 qubits 6 terms 64.4 / 64.5, 8: 83.6 / 75.5; 20: 8: 83.8 / 87.0, 10:
// 102.7 / 99.4; complex128 18: 3: 41.6 / 49.1, 4: 54.2 / 52.4; 19: 4: 57.3 / 57.8, 5:
// 72.9 / 67.9.  With (h, J) the passes have 60 us of tables to build besides, and one
// launch is faster from the first term (20 qubits 86.5 / 53.6).
template <typename R> constexpr int resident_kmin(int n)
{
    if (!resident_coop<R>(n)) return 1;
    return sizeof(R) == 4 ? (n == 19 ? 7 : 9) : (n == 18 ? 4 : 5);
}

// Sizes of one workgroup, whose launch can carry coefficients and couplings.
template <typename R> constexpr bool resident_single(int n) { return n <= (sizeof(R) == 4 ? 11 : 10); }

// Tile, threads, workgroups and spread per size, the fastest of a sweep that
// keeps to that (microseconds per term in the comments; in parentheses what the
// passes, or up to 13 / 12 qubits the former one-workgroup kernel, took).  One
// workgroup while the exchange would cost more than the shorter term saves;
// then 2^HC workgroups on one XCD, where a round of stores, flags and loads
// takes 0.9-1.4 us through its L2; from 16 / 15 qubits workgroups on all XCDs,
// where it takes 2.0 us and more, since 32 CUs would spend longer on a term
// (17 qubits: 5.2 us).
template <typename R>
static hipError_t launch_resident(int n, const ResArgs<R> *a, hipStream_t s, const PutBlob *blob, int cus)
{
    if constexpr (sizeof(R) == 4) {
        switch (n) {
        case 8: return res_launch<R, 8, 128, 0, 1, 1, false>(a, s, blob, cus);       // 0.31 (1.2)
        case 9: return res_launch<R, 9, 256, 0, 1, 1, false>(a, s, blob, cus);       // 0.36 (1.2)
        case 10: return res_launch<R, 10, 512, 0, 1, 1, false>(a, s, blob, cus);     // 0.45 (1.3)
        case 11: return res_launch<R, 11, 1024, 0, 1, 1, false>(a, s, blob, cus);    // 0.78 (1.9)
        case 12: return res_launch<R, 8, 128, 4, 8, 1, false>(a, s, blob, cus);      // 0.91 (3.1)
        case 13: return res_launch<R, 8, 128, 5, 8, 1, false>(a, s, blob, cus);      // 1.03 (5.6)
        case 14: return res_launch<R, 9, 256, 5, 8, 1, false>(a, s, blob, cus);      // 1.25 (5.8)
        case 15: return res_launch<R, 10, 256, 5, 8, 4, false>(a, s, blob, cus);     // 1.57 (5.8)
        case 16: return res_launch<R, 9, 256, 7, 1, 4, false>(a, s, blob, cus);      // 2.12 (6.3)
        case 17: return res_launch<R, 9, 256, 8, 1, 4, false>(a, s, blob, cus);      // 2.60 (6.6)
        case 18: return res_launch<R, 10, 256, 8, 1, 4, false>(a, s, blob, cus);     // 3.78 (7.6)
        case 19: return res_launch<R, 11, 512, 8, 1, 1, true>(a, s, blob, cus);      // 5.56 (9.7)
        case 20: return res_launch<R, 12, 512, 8, 1, 1, true>(a, s, blob, cus);      // 6.40 (9.6)
        default: return res_launch<R, 7, 64, 0, 1, 1, false>(a, s, blob, cus);       // 0.29 (1.2)
        }
    } else {
        switch (n) {
        case 7: return res_launch<R, 7, 128, 0, 1, 1, false>(a, s, blob, cus);       // 0.31 (1.1)
        case 8: return res_launch<R, 8, 256, 0, 1, 1, false>(a, s, blob, cus);       // 0.31 (1.1)
        case 9: return res_launch<R, 9, 512, 0, 1, 1, false>(a, s, blob, cus);       // 0.44 (1.2)
        case 10: return res_launch<R, 10, 1024, 0, 1, 1, false>(a, s, blob, cus);    // 0.70 (1.3)
        case 11: return res_launch<R, 8, 256, 3, 8, 1, false>(a, s, blob, cus);      // 0.79 (2.0)
        case 12: return res_launch<R, 7, 128, 5, 8, 1, false>(a, s, blob, cus);      // 0.90 (3.4)
        case 13: return res_launch<R, 8, 256, 5, 8, 1, false>(a, s, blob, cus);      // 1.11 (7.8)
        case 14: return res_launch<R, 9, 256, 5, 8, 4, false>(a, s, blob, cus);      // 1.42 (8.1)
        case 15: return res_launch<R, 8, 256, 7, 1, 4, false>(a, s, blob, cus);      // 2.01 (8.6)
        case 16: return res_launch<R, 8, 256, 8, 1, 4, false>(a, s, blob, cus);      // 2.52 (9.1)
        case 17: return res_launch<R, 9, 256, 8, 1, 4, false>(a, s, blob, cus);      // 3.60 (10.3)
        case 18: return res_launch<R, 10, 1024, 8, 1, 1, true>(a, s, blob, cus);     // 5.43 (12.3)
        case 19: return res_launch<R, 11, 512, 8, 1, 1, true>(a, s, blob, cus);      // 6.35 (13.0)
        default: return res_launch<R, 6, 64, 0, 1, 1, false>(a, s, blob, cus);       // 0.25 (1.1)
        }
    }
}

// What launch_resident asks of the stream: its compute units, if the size takes
// more than one workgroup.
template <typename R> static int resident_cus(int n, hipStream_t s) { return resident_single<R>(n) ? 1 : stream_cus(s); }

// Whether a call of n qubits can run in one launch on `cus` compute units.
template <typename R> static bool resident_fits(int n, int cus)
{
    return n <= resident_nmax<R>() &&
           (resident_single<R>(n) || launch_resident<R>(n, nullptr, nullptr, nullptr, cus) == hipSuccess);
}

}  // namespace qw

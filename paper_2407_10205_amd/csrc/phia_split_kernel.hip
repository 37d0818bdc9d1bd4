// Split sweep of the PHIA library for gfx950 (k_sweep_split): a replica block's
// columns over a group of G workgroups, every member's couplings in its CU's
// registers as int8 planes.
//
// Operands.  int8 couplings are one plane, BF16 hi/lo problems (|J| <= 32639)
// two and FP32 problems (|J| <= 8355711) three: J = sum_p 256^p J_p with J_p
// in [-128, 127], taken apart while the fragments are loaded.  The products
// are v_mfma_i32_16x16x64_i8 with the +-1 spins, shifted together in int32:
// the exact integer field of every other path, at a quarter of the register
// space and of the matrix-core time of FP32, half of BF16 hi/lo.
//
// Sparse rows (ELL path, PL = 0) keep their slots in LDS instead, the first
// four of a column in VGPRs, and gather one spin byte per slot.
//
// Layout.  NW waves, one 16-column block each, its fragments (planes x k
// blocks, at most 36 with eight waves and 96 with four) in VGPRs for the
// whole launch.  FEW: four replicas per group, spins as the A operand with
// replica r at row 4 r, so that lane (lr, lg) = (lane % 16, lane / 16) holds
// one element, replica lg and column lr.  Else sixteen replicas, products
// transposed (couplings A, spins B): lane (lr, lg) holds columns 4 lg ..
// 4 lg + 3 of replica lr.  (Thirty-two replicas, as two tiles in turn, took
// twice the time of sixteen: N = 1000, 3.9 against 2.1 us per step.)
//
// Exchange, one 64-bit word per (replica, column block) and step:
//   [63:48] low 16 bits of the sequence number (tag)
//   [47:16] sum over the block's columns of s (I + h) in the step before
//   [15:0]  spins, bit t set: +1
// in the slot of the sequence number's parity.  A slot is rewritten two
// publications later, when every member has read it (its own publication in
// between says so), so a word holds the awaited tag or the one two before.
// Words of a column block are adjacent, so that a wave publishes whole
// lines.  Every member reads all words of its block (its own too), unpacks the
// spins into the LDS buffer of the step's parity and adds up the energies; one
// barrier per step.
// The first word of a launch carries the member's XCD in place of the energy:
// a group that finds itself on one XCD publishes with workgroup scope, into
// the L2 that its members share (0.2 us from store to load), any other with
// agent scope, through to memory (0.5 us, and words of a line one after the
// other).  Waits are bounded: a member that gives up raises the
// device error word and every wave leaves the sweep.
//
// What bounds it: the chain of a step (publish, L2, poll, unpack, barrier,
// products, kick), 1.3 us at four replicas and 1.5 us at sixteen, and per k
// block and plane the products (N = 2000, four replicas, 1.6 us; sixteen,
// 2.7 us).  us per step, the sweeps it took the place of / this: N = 500 FP32,
// 128 replicas 31.7 / 1.50; N = 1000 BF16 hi/lo, 128 replicas 12.1 / 1.95;
// N = 2000 int8, 16 replicas 5.2 / 1.63, 512 replicas 8.6 / 5.6; 3-regular
// N = 4000, 32 replicas 3.5 / 1.55, 64 replicas 3.54 / 2.05.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "phia_devmath.h"
#include "phia_devsweep.h"
#include "phia_internal.h"

namespace phia {

namespace {

// int64 [3][16] energy sums (slot: step mod 3), uint32 [2] record masks, abort
// flag, flag of a group on several XCDs, then [2 parities][rows][stride] spins.
constexpr uint32_t kSplitMask = 384, kSplitAbort = 392, kSplitFar = 396, kSplitSpins = 512;
__host__ __device__ inline uint32_t split_srow(int nkb) { return 64u * static_cast<uint32_t>(nkb) + 16u; }

constexpr int kSplitDepth = 4;  // spin fragments in flight
constexpr int kSplitSlots = 4;  // ELL slots of a column in VGPRs

// Sixteen replicas, eight waves and 25 or more k blocks: two waves share the
// products of their two column blocks, half of the k blocks each, and hand each
// other a half product through LDS.  It halves the LDS reads of the spins, at
// N = 2000 2000 cycles of a step, for one more barrier (us per step without /
// with it: N = 2000, 512 replicas in two passes, 5.98 / 5.61; but 24 k blocks,
// N = 1500, 2.53 / 2.58, 16 2.0 / 2.1, four waves 3.16 / 3.26).
__host__ __device__ constexpr bool split_pair(int nkb, int waves, bool few) { return !few && waves == 8 && nkb > 24; }

__device__ __forceinline__ v4i pack16(const int (&c)[16])
{
    v4i r;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        r[q] = static_cast<int>((c[4 * q] & 0xff) | ((c[4 * q + 1] & 0xff) << 8) | ((c[4 * q + 2] & 0xff) << 16) |
                                (static_cast<uint32_t>(c[4 * q + 3] & 0xff) << 24));
    return r;
}

// Plane pl (0: lowest) of v.
template <int PL>
__device__ __forceinline__ int plane_of(int v, int pl)
{
#pragma unroll
    for (int q = 0; q < PL - 1; ++q)
        if (q < pl) {
            const int lo = static_cast<int8_t>(v & 0xff);
            v = (v - lo) >> 8;
        }
    return pl == PL - 1 ? v : static_cast<int8_t>(v & 0xff);
}

// The lane's 16 couplings of column block cb, k block kb (J[16 cb + lr][64 kb +
// 16 lg + t], t < 16) in the problem's own layout, as PL planes.
template <int PL>
__device__ __forceinline__ void load_planes(const void* J, int Np, int cb, int kb, int lane, v4i (&out)[PL])
{
    const int lr = lane & 15, lg = lane >> 4;
    if constexpr (PL == 1) {
        out[0] = *reinterpret_cast<const v4i*>(static_cast<const unsigned char*>(J) +
                                               (static_cast<size_t>(cb) * (Np / 64) + kb) * 1024 + lane * 16);
    } else {
        int c[16];
        if constexpr (PL == 2) {
            const uint4* src = reinterpret_cast<const uint4*>(J);
            const size_t chunk = static_cast<size_t>(cb) * (Np / 32) + 2 * kb + (lg >> 1);
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const int l = lr + 16 * (2 * (lg & 1) + half);
                const uint4 h4 = src[(chunk * 2) * 64 + l], l4 = src[(chunk * 2 + 1) * 64 + l];
                const uint32_t hw[4] = {h4.x, h4.y, h4.z, h4.w}, lw[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const uint32_t hb = (t & 1) ? hw[t / 2] & 0xffff0000u : hw[t / 2] << 16;
                    const uint32_t lb = (t & 1) ? lw[t / 2] & 0xffff0000u : lw[t / 2] << 16;
                    c[8 * half + t] = static_cast<int>(256.0f * __builtin_bit_cast(float, hb) + __builtin_bit_cast(float, lb));
                }
            }
        } else {
            const float4* src = reinterpret_cast<const float4*>(static_cast<const float*>(J) +
                                                                static_cast<size_t>(16 * cb + lr) * Np + 64 * kb + 16 * lg);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 f = src[q];
                c[4 * q] = static_cast<int>(f.x);
                c[4 * q + 1] = static_cast<int>(f.y);
                c[4 * q + 2] = static_cast<int>(f.z);
                c[4 * q + 3] = static_cast<int>(f.w);
            }
        }
#pragma unroll
        for (int pl = 0; pl < PL; ++pl) {
            int d[16];
#pragma unroll
            for (int t = 0; t < 16; ++t) d[t] = plane_of<PL>(c[t], pl);
            out[pl] = pack16(d);
        }
    }
}

// Sum over the lanes of a wave that gather the same replica row (lane mod RB).
template <int RB>
__device__ __forceinline__ int row_total(int t)
{
    if constexpr (RB == 4) {
        t += __builtin_amdgcn_update_dpp(0, t, 0x124, 0xf, 0xf, false);  // row_ror:4
        t += __builtin_amdgcn_update_dpp(0, t, 0x128, 0xf, 0xf, false);  // row_ror:8
    }
    return static_cast<int>(replica_sum_u(static_cast<uint32_t>(t)));
}

template <int PL, int NKB, int NW, bool FEW>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NW / 4, NW / 4))) k_sweep_split(SweepArgs a)
{
    constexpr int RB = FEW ? 4 : 16;   // replicas per group
    constexpr int E = FEW ? 1 : 4;     // elements per lane
    constexpr int TPR = 64 * NW / RB;  // gathering threads per replica row
    constexpr int NU = (4 * NKB + TPR - 1) / TPR;
    constexpr uint32_t srow = 64u * NKB + 16u, sbuf = RB * srow;
    constexpr bool PAIR = split_pair(NKB, NW, FEW);
    constexpr int KH = PAIR ? NKB / 2 : NKB;  // k blocks per wave and column block
    extern __shared__ __align__(16) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lg = lane >> 4;
    const int Np = a.Np, N = a.N, ncb = a.ncb, G = a.G;
    int group, member;
    if (a.xcd_map) {
        const int w = blockIdx.x, pos = w >> 3;
        member = pos % G;
        group = (pos / G) * 8 + (w & 7);
    } else {
        member = blockIdx.x % G;
        group = blockIdx.x / G;
    }
    const int cb0 = member * ncb / G, cb1 = (member + 1) * ncb / G;
    const int cblk = cb0 + wave;
    const bool cval = cblk < cb1;  // the wave owns a column block
    const int nkb = Np / 64;
    unsigned long long* sE = reinterpret_cast<unsigned long long*>(lds);
    uint32_t* sMask = reinterpret_cast<uint32_t*>(lds + kSplitMask);  // by step parity
    int* sAbort = reinterpret_cast<int*>(lds + kSplitAbort);
    int* sFar = reinterpret_cast<int*>(lds + kSplitFar);
    unsigned char* sS = lds + kSplitSpins;  // by step parity
    const int xcd = __builtin_amdgcn_s_getreg(20 | (3 << 11));  // XCC_ID

    constexpr int PN = PL > 0 ? PL : 1, KN = PL > 0 ? NKB : 1;
    v4i jr[KN][PN];
    int32_t slot[kSplitSlots];  // ELL: (coupling << 16) | column
    v4i* const sP = reinterpret_cast<v4i*>(sS + 2u * sbuf);  // PAIR: [waves][64] half products
    int32_t* const sL = reinterpret_cast<int32_t*>(sS + 2u * sbuf);  // ELL: [slots][16 NW]
    if constexpr (PL > 0) {
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
#pragma unroll
            for (int pl = 0; pl < PL; ++pl) jr[kb][pl] = v4i{0, 0, 0, 0};
            if constexpr (PAIR) {
                const int cb = cb0 + (wave & ~1) + kb / KH, k = (wave & 1) * KH + kb % KH;
                if (cb < cb1 && k < nkb) load_planes<PN>(a.J, Np, cb, k, lane, jr[kb]);
            } else {
                if (cval && kb < nkb) load_planes<PN>(a.J, Np, cblk, kb, lane, jr[kb]);
            }
        }
    } else {
        const int32_t* E = static_cast<const int32_t*>(a.J);
#pragma unroll
        for (int d = 0; d < kSplitSlots; ++d)
            slot[d] = cval && d < a.ell_d ? E[static_cast<size_t>(d) * Np + cblk * 16 + lr] : 0;
        for (int u = tid; u < (a.ell_d - kSplitSlots) * 16 * NW; u += 64 * NW) {
            const int d = kSplitSlots + u / (16 * NW), col = cb0 * 16 + u % (16 * NW);
            sL[u] = col < cb1 * 16 ? E[static_cast<size_t>(d) * Np + col] : 0;
        }
    }
    // spins of k positions past the columns meet zero couplings
    for (uint32_t u = tid; u < (kSplitSpins + 2u * sbuf) / 4u; u += 64 * NW) reinterpret_cast<uint32_t*>(lds)[u] = 0u;

    int hj[E];
    uint32_t creal = 0;  // elements with a real column
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int col = cblk * 16 + (FEW ? lr : 4 * lg + e);
        hj[e] = cval ? a.h[col] : 0;
        if (cval && col < N) creal |= 1u << e;
    }
    const float eps = in_vgpr(a.eps), gamma = in_vgpr(a.gamma);
    const Sech2K sk = sech2_in_vgprs();
    const ConstF ctab = scalar_table(a.ctab);
    const int nsteps = static_cast<int>(a.k1 - a.k0);
    const int grow = tid % RB, gc = tid / RB;
    const size_t plane = static_cast<size_t>(RB) * ncb;
    int goff[NU];  // gather: this thread's words
#pragma unroll
    for (int u = 0; u < NU; ++u) goff[u] = min(gc + TPR * u, ncb - 1) * RB + grow;
    const int64_t ref0 = a.k0 + (a.L - a.k0 % a.L) % a.L;
    uint32_t seq0 = a.seq_base + 1u;  // publication of step k0
    __syncthreads();

    for (int blk = group; blk < a.nblocks; blk += a.ngroups) {
        const int64_t rb0 = static_cast<int64_t>(blk) * RB;
        const int64_t rep = rb0 + (FEW ? lg : lr);  // the lane's replica
        const bool rok = rep < a.R;
        const int64_t idx0 = rep * Np + cblk * 16 + (FEW ? lr : 4 * lg);
        float x[E], v[E];
        uint32_t best = 0, hist = 0;  // record spins; spins of the last steps, four bits each
        int qi = xcd;
        bool far = true;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const bool ok = ((creal >> e) & 1u) && rok;
            x[e] = ok ? a.x[idx0 + e] : 0.0f;
            v[e] = ok ? a.v[idx0 + e] : 0.0f;
            if (ok && a.bestS[idx0 + e] > 0) best |= 1u << e;
        }
        // records: lane r of wave 0 holds replica r's
        const bool rec = wave == 0 && lane < RB && rb0 + lane < a.R;
        int64_t bE = INT64_MIN, bK = -1;
        if (rec) {
            bE = a.bestE[rb0 + lane];
            bK = a.bestStep[rb0 + lane];
        }
        int64_t next_ref = ref0;
        uint64_t round = static_cast<uint64_t>(ref0 / a.L);
        int r3 = 2;  // s mod 3
        auto take = [&](uint32_t m, uint32_t bits) {  // records m of a step in which the spins were bits
            if (m == 0) return;
            if ((m >> (FEW ? lg : lr)) & 1u) best = bits & 15u;
        };
        auto words = [&](uint32_t seq) -> uint64_t* {
            return a.xbits + (static_cast<size_t>(seq & 1u) * a.ngroups + group) * plane;
        };

        bool leave = false;
        for (int s = -1;; ++s) {
            const int64_t k = a.k0 + s;
            const bool closing = s == nsteps;
            const int r3p = r3 == 0 ? 2 : r3 - 1, r3n = r3 == 2 ? 0 : r3 + 1;
            const uint32_t seq = seq0 + static_cast<uint32_t>(s);
            const float ck_s = ctab[s < 0 || closing ? a.k0 : k];
            const bool draw = k + 1 == next_ref && s + 1 < nsteps;
            if (s >= 0) {
                // Gather the words of step k.
                unsigned char* const S = sS + static_cast<uint32_t>(s & 1) * sbuf;
                const uint64_t* const X = words(seq);
                uint64_t w[NU];
#pragma unroll
                for (int u = 0; u < NU; ++u)
                    w[u] = __hip_atomic_load(X + goff[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const uint32_t want = seq & 0xffffu;
                uint32_t polls = 0;
                for (;;) {
                    uint32_t stale = 0;
#pragma unroll
                    for (int u = 0; u < NU; ++u)
                        stale |= (static_cast<uint32_t>(w[u] >> 48) != want) ? 1u << u : 0u;
                    if (!__any(stale != 0)) break;
                    ++polls;
                    // the first words may wait for a member whose CU another
                    // stream's kernel holds: up to a minute, not in haste
                    if (s == 0 && polls > 1024u) __builtin_amdgcn_s_sleep(127);
                    if (polls > (s == 0 ? kSpinLimit << 3 : kSpinLimit) ||
                        ((polls & 255u) == 0 &&
                         __hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
                        __hip_atomic_store(a.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        *sAbort = 1;
                        break;
                    }
#pragma unroll
                    for (int u = 0; u < NU; ++u)
                        if ((stale >> u) & 1u)
                            w[u] = __hip_atomic_load(X + goff[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                int lo = 0, hi = 0;
                bool other = false;
#pragma unroll
                for (int u = 0; u < NU; ++u) {
                    const int c = gc + TPR * u;
                    const int en = static_cast<int>(static_cast<uint32_t>(w[u] >> 16));
                    other |= en != xcd;
                    if (c < ncb) {
                        unpack_signs<1>(static_cast<uint32_t>(w[u]) & 0xffffu, S + grow * srow + c * 16);
                        lo += en & 0xffff;
                        hi += en >> 16;
                    }
                }
                if (s == 0) {
                    if (other) *sFar = 1;
                } else {
                    lo = row_total<RB>(lo);
                    hi = row_total<RB>(hi);
                    if (lane < RB)
                        atomicAdd(sE + r3p * 16 + lane,
                                  static_cast<unsigned long long>((static_cast<int64_t>(hi) << 16) + lo));
                }
                __syncthreads();
                const int abort_flag = *sAbort;
                if (s == 0) far = __builtin_amdgcn_readfirstlane(*sFar) != 0;
                const uint32_t mask = __builtin_amdgcn_readfirstlane(s > 1 ? sMask[(s & 1) ^ 1] : 0u);
                if (wave == 0) {
                    if (s > 0) {  // the records of step k - 1
                        const int64_t tot = lane < RB ? static_cast<int64_t>(sE[r3p * 16 + lane]) : 0;
                        const int64_t en = -(tot >> 1);  // even: J symmetric, h counted twice
                        const bool imp = rec && en < bE;
                        bE = imp ? en : bE;
                        bK = imp ? k - 1 : bK;
                        const uint64_t b = __ballot(imp);
                        if (lane == 0) sMask[s & 1] = static_cast<uint32_t>(b);
                    }
                    if (lane < RB) sE[r3n * 16 + lane] = 0;
                }
                leave = abort_flag != 0;
                int field[E];  // J s
                if (!closing && (PAIR ? cb0 + (wave & ~1) < cb1 : cval)) {
                    if constexpr (PL == 0) {
                        static_assert(PL > 0 || FEW, "ELL: four replicas per group");
                        const int8_t* const Sg = reinterpret_cast<const int8_t*>(S + static_cast<uint32_t>(lg) * srow);
                        int sum = 0;
#pragma unroll
                        for (int d = 0; d < kSplitSlots; ++d) sum += (slot[d] >> 16) * static_cast<int>(Sg[slot[d] & 0xffff]);
                        const int32_t* const Lw = sL + wave * 16 + lr;
#pragma unroll 4
                        for (int d = 0; d < a.ell_d - kSplitSlots; ++d) {
                            const int32_t w = Lw[d * 16 * NW];
                            sum += (w >> 16) * static_cast<int>(Sg[w & 0xffff]);
                        }
                        field[0] = sum;
                    } else {
                        // A ring of spin fragments keeps the LDS reads ahead of
                        // the products (the compiler reads two at a time and
                        // waits for them).
                        constexpr int D = KH < kSplitDepth ? KH : kSplitDepth, NB = PAIR ? 2 : 1;
                        v4i acc[NB][PN];
#pragma unroll
                        for (int b = 0; b < NB; ++b)
#pragma unroll
                            for (int pl = 0; pl < PL; ++pl) acc[b][pl] = v4i{0, 0, 0, 0};
                        const unsigned char* const Sr = S + static_cast<uint32_t>(FEW ? lr >> 2 : lr) * srow + 16 * lg +
                                                        (PAIR ? (wave & 1) * KH * 64 : 0);
                        v4i ring[D];
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int kb = 0; kb < D; ++kb) ring[kb] = *reinterpret_cast<const v4i*>(Sr + kb * 64);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int kb = 0; kb < KH; ++kb) {
                            const v4i s4 = ring[kb % D];
#pragma unroll
                            for (int b = 0; b < NB; ++b)
#pragma unroll
                                for (int pl = 0; pl < PL; ++pl) {
                                    const v4i j4 = jr[b * KH + kb][pl];
                                    acc[b][pl] = FEW ? __builtin_amdgcn_mfma_i32_16x16x64_i8(s4, j4, acc[b][pl], 0, 0, 0)
                                                     : __builtin_amdgcn_mfma_i32_16x16x64_i8(j4, s4, acc[b][pl], 0, 0, 0);
                                }
                            if (kb + D < KH) {
                                ring[kb % D] = *reinterpret_cast<const v4i*>(Sr + (kb + D) * 64);
                                __builtin_amdgcn_sched_barrier(0);
                            }
                        }
#pragma unroll
                        for (int b = 0; b < NB; ++b)
#pragma unroll
                            for (int pl = PL - 2; pl >= 0; --pl)
#pragma unroll
                                for (int e = 0; e < E; ++e)
                                    acc[b][pl][e] += acc[b][pl + 1][e] << 8;
                        const bool upper = PAIR && (wave & 1);
#pragma unroll
                        for (int e = 0; e < E; ++e) field[e] = upper ? acc[NB - 1][0][e] : acc[0][0][e];
                        if constexpr (PAIR) sP[wave * 64 + lane] = upper ? acc[0][0] : acc[1][0];
                    }
                }
                if (PAIR && !closing) __syncthreads();  // the partners' halves
                if (!closing && cval) {
                    if constexpr (PAIR) {
                        const v4i half = sP[(wave ^ 1) * 64 + lane];
#pragma unroll
                        for (int e = 0; e < E; ++e) field[e] += half[e];
                    }
                    float If[E];
                    int q = 0;
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        const int I = field[e] + hj[e];
                        If[e] = static_cast<float>(I);
                        const int ih = I + hj[e];
                        q += x[e] >= 0.0f ? ih : -ih;
                    }
                    qi = FEW ? row_sum16_dpp(q) : static_cast<int>(replica_sum_u(static_cast<uint32_t>(q)));
                    const float ck = in_vgpr(ck_s);
                    if (a.deriv)
                        kick_n<1, E>(x, v, If, ck, eps, gamma, sk);
                    else
                        kick_n<0, E>(x, v, If, ck, eps, gamma, sk);
                }
                take(mask, hist >> (closing ? 4 : 8));
            }
            if (closing) break;
            // Drift of step k + 1 and its publication, with the energies
            // of step k (past the last step: the energies only).
            uint32_t bits = 0;
            if (draw) {
                asm volatile("");  // a branch: as selects the draws would be computed in every step
                float g[4];
                if constexpr (FEW) {
                    // lane l % 16 = 4 replica + 2 (column >> 3) + half draws four columns
                    gauss_block_half(a.seed, a.r_base + rb0 + ((lane >> 2) & 3), round,
                                     static_cast<uint64_t>(cblk) * 2 + ((lane >> 1) & 1), lane & 1, g);
                    const int src = 4 * lg + (lr >> 2);
                    const float t0 = lane_read(src, g[0]), t1 = lane_read(src, g[1]);
                    const float t2 = lane_read(src, g[2]), t3 = lane_read(src, g[3]);
                    const float lo = (lr & 1) ? t1 : t0, up = (lr & 1) ? t3 : t2;
                    v[0] = ((creal & 1u) && rok) ? ((lr & 2) ? up : lo) : 0.0f;
                } else {
                    gauss_block_half(a.seed, a.r_base + rep, round, static_cast<uint64_t>(cblk) * 2 + (lg >> 1),
                                     lg & 1, g);
#pragma unroll
                    for (int e = 0; e < E; ++e)
                        v[e] = (((creal >> e) & 1u) && rok) ? g[e] : 0.0f;
                }
            }
            if (s + 1 < nsteps) {
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    x[e] = __builtin_fmaf(eps, v[e], x[e]);
                    if (x[e] >= 0.0f) bits |= 1u << e;
                }
                hist = (hist << 4) | bits;
            }
            if (cval) {
                uint64_t* const X = words(seq + 1u) + static_cast<size_t>(cblk) * RB;
                uint32_t m;
                if constexpr (FEW)
                    m = static_cast<uint32_t>(__ballot(bits != 0) >> (16 * lg)) & 0xffffu;
                else
                    m = replica_sum_u(bits << (4 * lg));
                const uint64_t w = static_cast<uint64_t>((seq + 1u) & 0xffffu) << 48 |
                                   static_cast<uint64_t>(static_cast<uint32_t>(qi)) << 16 | m;
                if (FEW ? lr == 0 : lg == 0) {
                    uint64_t* const q = X + (FEW ? lg : lr);
                    if (far)
                        __hip_atomic_store(q, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    else
                        __hip_atomic_store(q, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
            if (leave) return;
            if (draw) {
                ++round;
                next_ref += a.L;
            }
            r3 = r3n;
        }
        if (leave) return;
        __syncthreads();
        take(__builtin_amdgcn_readfirstlane(sMask[nsteps & 1]), hist);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if (!(((creal >> e) & 1u) && rok)) continue;
            a.x[idx0 + e] = x[e];
            a.v[idx0 + e] = v[e];
            a.bestS[idx0 + e] = ((best >> e) & 1u) ? 1 : -1;
        }
        if (member == 0 && rec) {
            a.bestE[rb0 + lane] = bE;
            a.bestStep[rb0 + lane] = bK;
        }
        // the next block starts with clear sums
        seq0 += static_cast<uint32_t>(nsteps) + 1u;
        if (tid < 48) sE[tid] = 0;
        if (tid == 0) *sFar = 0;
        __syncthreads();
    }
}

struct SplitVariant {
    int planes, nkb, waves;
    const void* kernel[2];  // 4, 16 replicas per group
};
template <int PL, int NKB, int NW>
SplitVariant split_variant_of()
{
    return {PL, NKB, NW,
            {reinterpret_cast<const void*>(k_sweep_split<PL, NKB, NW, true>),
             reinterpret_cast<const void*>(k_sweep_split<PL, NKB, NW, false>)}};
}
template <>
SplitVariant split_variant_of<0, 64, 16>()
{
    return {0, 64, 16, {reinterpret_cast<const void*>(k_sweep_split<0, 64, 16, true>), nullptr}};
}
const SplitVariant kSplitVariants[] = {
    split_variant_of<1, 16, 8>(), split_variant_of<1, 24, 8>(), split_variant_of<1, 32, 8>(),
    split_variant_of<2, 4, 8>(),  split_variant_of<2, 8, 8>(),  split_variant_of<2, 16, 8>(),
    split_variant_of<2, 24, 4>(), split_variant_of<2, 32, 4>(), split_variant_of<3, 4, 8>(),
    split_variant_of<3, 8, 8>(),  split_variant_of<3, 12, 8>(), split_variant_of<3, 16, 4>(),
    split_variant_of<3, 24, 4>(), split_variant_of<3, 32, 4>(), split_variant_of<0, 64, 16>(),
};

const SplitVariant* split_variant(int Np, int planes)
{
    for (const SplitVariant& v : kSplitVariants)
        if (v.planes == planes && Np <= 64 * v.nkb) return &v;
    return nullptr;
}

size_t split_lds(const SplitVariant& v, int rows, int slots)
{
    return kSplitSpins + 2u * static_cast<size_t>(rows) * split_srow(v.nkb) +
           (v.planes > 0 && split_pair(v.nkb, v.waves, rows == 4) ? 1024u * static_cast<size_t>(v.waves) : 0u) +
           (v.planes == 0 ? 64u * static_cast<size_t>(v.waves) * std::max(0, slots - kSplitSlots) : 0u);
}

int split_form(int rows) { return rows == 4 ? 0 : rows == 16 ? 1 : -1; }

}  // namespace

int split_waves(int Np, int planes)
{
    const SplitVariant* v = split_variant(Np, planes);
    return v ? v->waves : 0;
}

size_t sweep_split_lds_bytes(int Np, int planes, int rows, int slots)
{
    const SplitVariant* v = split_variant(Np, planes);
    if (!v || split_form(rows) < 0 || !v->kernel[split_form(rows)]) return 0;
    const size_t b = split_lds(*v, rows, slots);
    return b <= static_cast<size_t>(kLdsMax) ? b : 0;
}

hipError_t launch_sweep_split(const SweepArgs& a, int planes, hipStream_t st)
{
    const SplitVariant* v = split_variant(a.Np, planes);
    const size_t lds = sweep_split_lds_bytes(a.Np, planes, a.rows, a.ell_d);
    if (lds == 0 || a.k1 <= a.k0 || a.k1 - a.k0 > (int64_t(1) << 30) || (a.ncb + a.G - 1) / a.G > v->waves)
        return hipErrorInvalidValue;
    const void* kern = v->kernel[split_form(a.rows)];
    hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
    if (e != hipSuccess) return e;
    SweepArgs copy = a;
    void* args[] = {&copy};
    e = hipLaunchCooperativeKernel(kern, dim3(static_cast<unsigned>(a.ngroups * a.G)),
                                   dim3(static_cast<unsigned>(64 * v->waves)), args, static_cast<unsigned>(lds), st);
    return e != hipSuccess ? e : hipGetLastError();
}

int max_coresident_split(int Np, int planes, int rows, int slots)
{
    const SplitVariant* v = split_variant(Np, planes);
    const size_t lds = sweep_split_lds_bytes(Np, planes, rows, slots);
    if (lds == 0) return 0;
    const void* f = v->kernel[split_form(rows)];
    int dev = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)) != hipSuccess)
        return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, f, 64 * v->waves, lds) != hipSuccess) return 0;
    return per * cus;
}

}  // namespace phia

// Persistent batched sweep of the PHIA library for gfx950 (k_batch_fp4).
//
// Many instances of uneven size (N <= 512) whose integer couplings are all
// FP4 (E2M1) values run in one launch: every workgroup takes work items --
// one instance's block of 32 replicas -- from a global queue ordered largest
// first, until the queue is empty, and runs each item's steps with all of
// its columns.  One step is the sweep of Sec. 2.1 / App. A A7 for every
// element at once (momentum refresh, drift, readout, J.s + h on matrix
// cores, exact energy, records, kick), exactly as the other sweep kernels
// compute it.
//
// Operands.  The products run transposed, D = J . S^T, with the couplings as
// the A operand and the spins as the B operand of
// v_mfma_scale_f32_16x16x128_f8f6f4 (FP4 x FP4, scales 1, FP32 accumulation
// starting from the fields h): every product and partial sum is an integer
// below 2^24 (host-checked), so the field is exact and stays in FP32 for the
// kick and the energy terms.  A tile is one 16-column block of one of the two
// 16-replica halves; lane (lr, lg) = (lane % 16, lane / 16) of its wave holds
// replica lr and four of the block's columns, x, v and the field in VGPRs.  A
// replica's record, its energy partial (a sum over four lanes) and its spins
// (four FP4 codes, one 16-bit LDS store) are then per-lane work; with a
// column per lane and four replicas per lane they took 27 of the 55 VALU
// instructions per spin-update.  The couplings of the instance sit in LDS as
// FP4 fragments for the whole item (128 KiB at Np = 512).
//
// Two forms.  A whole workgroup of sixteen waves runs one item as two teams of
// eight, one per replica half, a phase apart: one spin buffer per half, two
// barriers per step, the records taken in the step itself (team_item).  A squad
// of eight waves runs an item of up to 256 columns with both halves: two spin
// buffers by step parity, one barrier per step, the records of step k in step
// k + 1; every wave owns ncb / 8 column blocks for both halves, and when four
// are left over wave w owns block w % 4 of them for half w / 4, so that all
// waves carry the same number of tiles; two squads share a workgroup
// (squad_item).  x is drawn here when an item starts (no separate init kernel).
//
// The step is bound by VALU issue.  Its FP32 operations read VGPRs and inline
// constants only (2 cycles per wave; 4 with an SGPR operand, see in_vgpr).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include <type_traits>

#include "phia_devmath.h"
#include "phia_devsweep.h"
#include "phia_internal.h"

namespace phia {

namespace {

constexpr int kBW = 16;                // waves per workgroup
constexpr int kBT = 64 * kBW;          // threads per workgroup
constexpr int kSquad = 8;              // waves per squad
constexpr int kSquadMaxNp = 256;       // largest instance of a squad
// Energy sums [3][32] float, the item slot (byte 384), a squad's barrier
// counter (byte 400).
constexpr uint32_t kFixedLds = 512;

__host__ __device__ inline int nkb4_of(int Np) { return (Np + 127) / 128; }
// LDS passed to a function that is not inlined keeps its address space (a
// generic pointer would turn every access into a flat one).
typedef __attribute__((address_space(3))) unsigned char LdsByte;

// Column of element j (0 .. 3) of lane group lg within its 16-column block.
// The FP4 codes of 8 columns are ordered 0 4 1 5 2 6 3 7 in LDS (the packed
// couplings' k order), so the columns whose codes a lane stores as one
// 16-bit word are 8 (lg / 2) + 2 (lg % 2) + {0, 4, 1, 5}.
__device__ __forceinline__ int col_of(int lg, int j)
{
    return 8 * (lg >> 1) + 2 * (lg & 1) + (j >> 1) + 4 * (j & 1);
}

// vdst's odd rows of 16 lanes exchanged with vsrc's even rows (permlane16),
// or its upper 32 lanes with vsrc's lower 32 (permlane32).  The nop covers
// the VALU-write-to-permlane-read hazard; the whole wave must be active.
__device__ __forceinline__ void swap16(uint32_t& a, uint32_t& b)
{
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ void swap32(uint32_t& a, uint32_t& b)
{
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}

// Gaussian draws of this lane's four columns of one column block for one
// replica (a call, so that the step does not hold generator states).  The
// block of 8 columns c8 belongs to the lane pair lg, lg ^ 1; the lane's
// columns take the even-numbered (lg even) or odd-numbered words' pairs.
struct Draws4 {
    float g[4];
};
struct Draws8 {
    float a[4], b[4];
};
__device__ __forceinline__ Draws4 draws_of(uint32_t lo0, uint32_t hi0, uint32_t lo1, uint32_t hi1)
{
    Draws4 d;
    gauss_pair(static_cast<uint64_t>(hi0) << 32 | lo0, d.g[0], d.g[2]);
    gauss_pair(static_cast<uint64_t>(hi1) << 32 | lo1, d.g[1], d.g[3]);
    return d;
}
__device__ __attribute__((noinline)) Draws4 draws_one(uint64_t seed, uint32_t tag, uint64_t replica, uint64_t round,
                                                       uint64_t c8, int odd)
{
    const u64x4 o = dev_philox(c8, round, replica, tag, seed, 0);
    const uint64_t w0 = odd ? o.w[1] : o.w[0], w1 = odd ? o.w[3] : o.w[2];
    return draws_of(static_cast<uint32_t>(w0), static_cast<uint32_t>(w0 >> 32), static_cast<uint32_t>(w1),
                    static_cast<uint32_t>(w1 >> 32));
}
// The same for two generator blocks (replica ra or rb, column block c8a or
// c8b): the even lane of a pair runs the generator for the first, the odd lane
// for the second, and a lane swap hands each the words it transforms.
__device__ __forceinline__ Draws8 draws_pair(uint64_t seed, uint32_t tag, uint64_t r, uint64_t round, uint64_t c8)
{
    const u64x4 o = dev_philox(c8, round, r, tag, seed, 0);
    uint32_t l[4], h[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        l[q] = static_cast<uint32_t>(o.w[q]);
        h[q] = static_cast<uint32_t>(o.w[q] >> 32);
    }
    swap16(l[0], l[1]);
    swap16(h[0], h[1]);
    swap16(l[2], l[3]);
    swap16(h[2], h[3]);
    const Draws4 p = draws_of(l[0], h[0], l[2], h[2]), q = draws_of(l[1], h[1], l[3], h[3]);
    Draws8 d;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        d.a[j] = p.g[j];
        d.b[j] = q.g[j];
    }
    return d;
}

// two replicas (r0 and r0 + 16) of one column block
__device__ __attribute__((noinline)) Draws8 draws_both(uint64_t seed, uint32_t tag, uint64_t r0, uint64_t round,
                                                       uint64_t c8, int odd)
{
    return draws_pair(seed, tag, r0 + (odd ? 16 : 0), round, c8);
}
// two column blocks of one replica
__device__ __attribute__((noinline)) Draws8 draws_two(uint64_t seed, uint32_t tag, uint64_t r, uint64_t round,
                                                      uint64_t c8a, uint64_t c8b, int odd)
{
    return draws_pair(seed, tag, r, round, odd ? c8b : c8a);
}

// The steps of one work item.  Two teams of eight waves, one per replica half,
// run one phase apart: while one team's waves take the field of their half on
// the matrix cores and its energy sums (P), the other team's take the records,
// the kick and the next drift (V), and a workgroup barrier closes each phase.
// A wave issues at most one instruction per 4 cycles, so the two waves per
// SIMD of the V team reach the VALUs' rate only while nothing else holds them
// up: the operand reads, the products and the waits for them are the other
// team's.  Eight waves that did both in one phase per step took 4.64 us per
// step at N = 512, with the halves' products and kicks interleaved in each
// wave 3.97 us, in this form 3.66 us (a column per lane and FP8 spins, before
// that: 5.8 us).  Without the kick a step takes 1.85 us, without the products
// 3.1 us: the kick runs at 2.1 cycles per instruction and SIMD, and an MFMA
// (16 cycles here) leaves the SIMD's VALU idle while it issues.
//
// The wave owns the column blocks tw + 8 c, c < NC, and the k range is NC
// blocks of 128: the caller pads the couplings in LDS to 8 NC column blocks.
template <int NC, int DERIV>
__device__ __attribute__((noinline)) void team_item(const BatchInst* ap, int blk, LdsByte* lds3, int wave, int lane)
{
    unsigned char* const lds = (unsigned char*)lds3;
    constexpr int NF = NC, NKB = NC;
    constexpr uint32_t srow = NKB * 64u + 16u;
    wave = __builtin_amdgcn_readfirstlane(wave);
    blk = __builtin_amdgcn_readfirstlane(blk);
    const int team = wave >> 3, tw = wave & 7;
    const BatchInst& a = *uniform_ptr(ap);
    const int Np = __builtin_amdgcn_readfirstlane(a.Np), N = __builtin_amdgcn_readfirstlane(a.N);
    constexpr uint32_t jb = 8u * NC * NKB * 1024u;
    float* sE = reinterpret_cast<float*>(lds) + team * 32;  // [2 parities][16] row energy sums (exact integers)
    unsigned char* sJ = lds + kFixedLds;
    unsigned char* S = sJ + jb + team * 16u * srow;  // [16][srow] FP4 spins of the team's half
    const int lr = lane & 15, lg = lane >> 4;
    // fields of the lane's columns of column block 0, in lane order
    const v4f* sH = reinterpret_cast<const v4f*>(sJ + jb + 32u * srow) + lg;
    const int nsteps = __builtin_amdgcn_readfirstlane(static_cast<int>(a.k1));
    const uint64_t seed = *a.seed;
    auto cbt = [&](int c) { return tw + 8 * c; };  // column block of tile c
    const int64_t gr = static_cast<int64_t>(blk) * kBatchRows + 16 * team + lr;  // the lane's replica
    const bool rok = gr < a.R;
    float x[NC][4], v[NC][4], sg[NC][4];
    v4f I[NC];
    uint32_t bp[NC];            // record spins: the four FP4 codes of each tile
    float bE = __builtin_inff();  // record energy (+inf: none yet)
    int32_t bK = -1;
    // draws of a generator round (0 in padding); two column blocks share
    // their generator blocks between the lane pairs
    auto draw = [&](uint32_t tag, uint64_t round, float (&y)[NC][4]) {
        const auto c8 = [&](int c) { return static_cast<uint64_t>(cbt(c)) * 2 + (lg >> 1); };
        const auto put = [&](float (&d)[4], int c, const float (&g)[4]) {
#pragma unroll
            for (int j = 0; j < 4; ++j) d[j] = (cbt(c) * 16 + col_of(lg, j) < N && rok) ? g[j] : 0.0f;
        };
#pragma unroll
        for (int c = 0; c + 1 < NF; c += 2) {
            const Draws8 d = draws_two(seed, tag, static_cast<uint64_t>(gr), round, c8(c), c8(c + 1), lg & 1);
            put(y[c], c, d.a);
            put(y[c + 1], c + 1, d.b);
        }
        if constexpr (NF % 2 == 1) {
            const Draws4 d = draws_one(seed, tag, static_cast<uint64_t>(gr), round, c8(NF - 1), lg & 1);
            put(y[NF - 1], NF - 1, d.g);
        }
    };
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        bp[c] = 0x2222u;
        I[c] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            x[c][j] = v[c][j] = 0.0f;
            sg[c][j] = 1.0f;
        }
    }
    draw(kTagX, 0, x);

    const float eps = in_vgpr(a.eps), gamma = in_vgpr(a.gamma);
    Sech2K sk{};
    if constexpr (DERIV == 0) sk = sech2_in_vgprs();
    const int L = static_cast<int>(a.L < INT32_MAX ? a.L : INT32_MAX);
    const ConstF ctab = scalar_table(a.ctab);
    // the lane's codes of column block 0
    unsigned char* const srow0 = S + static_cast<uint32_t>(lr) * srow + 2u * lg;
    const unsigned char* const brow = S + lr * srow + 16 * lg;
    const unsigned char* const jl =
        sJ + ((lane & 48) + 8 * (lr >> 3) + 2 * ((lr >> 2) & 1) + ((lr >> 1) & 1) + 4 * (lr & 1)) * 16;

    // Drift and readout for step q: momentum refresh, x, spins (FP4 codes).
    int next_ref = 0, round = 0;
    auto drift = [&](int q) {
        if (q == next_ref) {
            draw(kTagV, static_cast<uint64_t>(round), v);
            ++round;
            next_ref = L > INT32_MAX - q ? INT32_MAX : q + L;
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                x[c][j] = __builtin_fmaf(eps, v[c][j], x[c][j]);
                sg[c][j] = x[c][j] >= 0.0f ? 1.0f : -1.0f;
            }
            uint32_t w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(0u, sg[c][0], sg[c][1], 1.0f, 0);
            w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, sg[c][2], sg[c][3], 1.0f, 1);
            *reinterpret_cast<uint16_t*>(srow0 + cbt(c) * 8u) = static_cast<uint16_t>(w);
        }
    };
    // P: field J s + h on matrix cores (accumulation starts from h; operand k
    // order: FP4 nibble t of lane group g is k = 32 g + t for both operands),
    // then the energy terms s (I + h) (padded columns have I = h = 0) summed
    // over the replica's four lanes and the waves.
    auto products = [&](int k) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
            I[c] = sH[cbt(c) * 4];
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
            const v4i b = *reinterpret_cast<const v4i*>(brow + kb * 64);
            const v8i B = v8i{b[0], b[1], b[2], b[3], 0, 0, 0, 0};
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                    const v4i j4 = *reinterpret_cast<const v4i*>(jl + (cbt(c) * NKB + kb) * 1024);
                I[c] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
                    v8i{j4[0], j4[1], j4[2], j4[3], 0, 0, 0, 0}, B, I[c], 4, 4, 0, 127, 0, 127);
            }
        }
        float part = 0.0f;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const v4f h = sH[cbt(c) * 4];
#pragma unroll
            for (int j = 0; j < 4; ++j) part = __builtin_fmaf(sg[c][j], I[c][j] + h[j], part);
        }
        uint32_t c0 = f_to_bits(part), c1 = c0;
        swap32(c0, c1);
        c0 = c1 = f_to_bits(bits_to_f(c0) + bits_to_f(c1));
        swap16(c0, c1);
        const float tot = bits_to_f(c0) + bits_to_f(c1);
        if (lg == 0) atomicAdd(sE + (k & 1) * 16 + lr, tot);
    };
    // V: records of step k (App. B, Table 3, state 5), the kick, and the
    // drift of step k + 1.  Every lane that holds the replica takes the same
    // decision; late in an anneal few steps improve a record, so the updates
    // run only when some replica of the wave improved (uniform branch).
    auto update = [&](int k, float ck_s) {
        const float E = -0.5f * sE[(k & 1) * 16 + lr];  // the sum is even: exact
        if (tw == 0 && lg == 0) sE[((k + 1) & 1) * 16 + lr] = 0.0f;  // read in the V phase before
        const float ck = in_vgpr(ck_s);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const float f[4] = {I[c][0], I[c][1], I[c][2], I[c][3]};
            kick_n<DERIV, 4>(x[c], v[c], f, ck, eps, gamma, sk);
        }
        const bool imp = E < bE;
        if (__any(imp)) {
            bE = imp ? E : bE;
            bK = imp ? k : bK;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                    const uint32_t w = *reinterpret_cast<const uint16_t*>(srow0 + cbt(c) * 8u);
                bp[c] = imp ? w : bp[c];
            }
        }
        if (k + 1 < nsteps) drift(k + 1);
    };

    drift(0);
    __syncthreads();
    if (team == 1) __syncthreads();  // one phase behind
    for (int k = 0; k < nsteps; ++k) {
        const float ck = ctab[k];
        products(k);
        __syncthreads();
        update(k, ck);
        __syncthreads();
    }
    if (team == 0) __syncthreads();

    // Final state and records of the item.
    if (rok) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int col = cbt(c) * 16 + col_of(lg, j);
                if (col < Np) {
                    a.x[gr * Np + col] = x[c][j];
                    a.v[gr * Np + col] = v[c][j];
                }
                if (col < N) a.bestS[gr * Np + col] = ((bp[c] >> (4 * j)) & 8u) ? -1 : 1;
            }
        }
        if (tw == 0 && lg == 0) {
            a.bestE[gr] = bE == __builtin_inff() ? INT64_MAX : static_cast<int64_t>(bE);
            a.bestStep[gr] = bK;
        }
    }
}

__device__ __forceinline__ uint32_t* squad_counter(unsigned char* lds)
{
    return reinterpret_cast<uint32_t*>(lds + 3 * 32 * 4 + 16);
}

// A barrier of one squad's eight waves: a monotonic LDS counter.  LDS
// accesses of a wave take effect in order, so every access before the
// barrier precedes the wave's count.  All eight waves of a squad run the same
// sequence of barriers, so every wait ends.
__device__ __forceinline__ void squad_barrier(uint32_t* counter, uint32_t& target, int lane)
{
    target += kSquad;
    if (lane == 0) __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    while (static_cast<int32_t>(__hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) - target) < 0)
        __builtin_amdgcn_s_sleep(0);
    __atomic_signal_fence(__ATOMIC_ACQ_REL);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// The steps of one work item for one squad of eight waves, for instances whose
// couplings leave room for two in LDS: each squad takes items of its own, so
// that one squad's waits (operand reads, products, its one barrier per step)
// are the other's VALU time.  A wave owns NF column blocks of both replica
// halves and, with HALF, one more of the half sw / 4 (ncb = 8 NF + 4), so all
// waves carry the same number of tiles.
// Returns the barrier count it reached.
template <int NF, bool HALF, int DERIV>
__device__ __attribute__((noinline)) uint32_t squad_item(const BatchInst* ap, int blk, LdsByte* lds3,
                                                         uint32_t target, int sw, int lane)
{
    unsigned char* const lds = (unsigned char*)lds3;
    uint32_t* counter = squad_counter(lds);
    constexpr int NC = NF + (HALF ? 1 : 0);  // column blocks of the wave = k blocks of 128
    constexpr int NT = 2 * NF + (HALF ? 1 : 0);
    constexpr uint32_t srow = NC * 64u + 16u;
    constexpr uint32_t sb = kBatchRows * srow;
    constexpr uint32_t jb = (8u * NF + (HALF ? 4u : 0u)) * NC * 1024u;
    sw = __builtin_amdgcn_readfirstlane(sw);
    blk = __builtin_amdgcn_readfirstlane(blk);
    const BatchInst& a = *uniform_ptr(ap);
    const int Np = __builtin_amdgcn_readfirstlane(a.Np), N = __builtin_amdgcn_readfirstlane(a.N);
    float* sE = reinterpret_cast<float*>(lds);  // [3][32] row energy sums of steps k mod 3 (exact integers)
    unsigned char* sJ = lds + kFixedLds;
    unsigned char* sS = sJ + jb;  // [2][32][srow] FP4 spins by step parity
    const int nsteps = __builtin_amdgcn_readfirstlane(static_cast<int>(a.k1));
    const int lr = lane & 15, lg = lane >> 4;
    const v4f* sH = reinterpret_cast<const v4f*>(sS + 2u * sb) + lg;  // fields of the lane's columns of block 0
    const uint64_t seed = *a.seed;
    const int mth = sw >> 2;  // replica half of the HALF tile
    // tile t: column block cbt(cw(t)), replica half mtt(t)
    auto cwt = [&](int t) { return t < 2 * NF ? t >> 1 : NF; };
    auto mtt = [&](int t) { return t < 2 * NF ? (t & 1) : mth; };
    auto cbt = [&](int cw) { return cw < NF ? sw + kSquad * cw : kSquad * NF + (sw & 3); };
    const int64_t gr0 = static_cast<int64_t>(blk) * kBatchRows + lr;  // replica of half 0; gr0 + 16 in half 1
    const bool rok[2] = {gr0 < a.R, gr0 + 16 < a.R};
    float x[NT][4], v[NT][4];
    float bE[2] = {__builtin_inff(), __builtin_inff()};  // record energies of the two replicas (+inf: none yet)
    int32_t bK[2] = {-1, -1};
    uint32_t bp[NT];  // record spins: the four FP4 codes of each tile
    // draws of a generator round into y (all tiles; 0 in padding)
    auto draw = [&](uint32_t tag, uint64_t round, float (&y)[NT][4]) {
#pragma unroll
        for (int cw = 0; cw < NC; ++cw) {
            const uint64_t c8 = static_cast<uint64_t>(cbt(cw)) * 2 + (lg >> 1);
            const auto real = [&](int j) { return cbt(cw) * 16 + col_of(lg, j) < N; };
            if (cw < NF) {
                const Draws8 d = draws_both(seed, tag, static_cast<uint64_t>(gr0), round, c8, lg & 1);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    y[2 * cw][j] = (real(j) && rok[0]) ? d.a[j] : 0.0f;
                    y[2 * cw + 1][j] = (real(j) && rok[1]) ? d.b[j] : 0.0f;
                }
            } else {
                const Draws4 d = draws_one(seed, tag, static_cast<uint64_t>(gr0) + 16 * mth, round, c8, lg & 1);
#pragma unroll
                for (int j = 0; j < 4; ++j) y[NT - 1][j] = (real(j) && (mth ? rok[1] : rok[0])) ? d.g[j] : 0.0f;
            }
        }
    };
    draw(kTagX, 0, x);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        bp[t] = 0x2222u;
#pragma unroll
        for (int j = 0; j < 4; ++j) v[t][j] = 0.0f;
    }
    const float eps = in_vgpr(a.eps), gamma = in_vgpr(a.gamma);
    Sech2K sk{};
    if constexpr (DERIV == 0) sk = sech2_in_vgprs();
    const int L = static_cast<int>(a.L < INT32_MAX ? a.L : INT32_MAX);
    const ConstF ctab = scalar_table(a.ctab);
    int next_ref = 0, round = 0;
    // the lane's byte offset in a spin buffer: row lr, its codes of column block 0
    const uint32_t soff = static_cast<uint32_t>(lr) * srow + 2u * lg;
    const unsigned char* jl =
        sJ + ((lane & 48) + 8 * (lr >> 3) + 2 * ((lr >> 2) & 1) + ((lr >> 1) & 1) + 4 * (lr & 1)) * 16;

    // Records of step kp (App. B, Table 3, state 5), whose spins are in the
    // buffer `pv`: every lane that holds a replica takes the same decision.
    // Late in an anneal few steps improve a record: the updates run only when
    // some replica of the wave improved (uniform branch).  The wave's own
    // codes of the step are still in their buffer.
    auto records = [&](int r3p, const unsigned char* pv, int kp) {
        const float E0 = -0.5f * sE[r3p * 32 + lr], E1 = -0.5f * sE[r3p * 32 + 16 + lr];  // the sums are even: exact
        const bool i0 = E0 < bE[0], i1 = E1 < bE[1];
        if (__any(i0 || i1)) {
            bE[0] = i0 ? E0 : bE[0];
            bE[1] = i1 ? E1 : bE[1];
            bK[0] = i0 ? kp : bK[0];
            bK[1] = i1 ? kp : bK[1];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const uint32_t w =
                    *reinterpret_cast<const uint16_t*>(pv + soff + mtt(t) * 16u * srow + cbt(cwt(t)) * 8u);
                bp[t] = (mtt(t) ? i1 : i0) ? w : bp[t];
            }
        }
    };

    int r3 = 0;
    for (int k = 0; k < nsteps; ++k) {
        const int r3p = (r3 == 0) ? 2 : r3 - 1, r3n = (r3 == 2) ? 0 : r3 + 1;
        unsigned char* S = sS + (k & 1) * sb;
        const float ck_s = ctab[k];
        if (k == next_ref) {  // momentum refresh
            draw(kTagV, static_cast<uint64_t>(round), v);
            ++round;
            next_ref = L > INT32_MAX - k ? INT32_MAX : k + L;
        }
        // Drift and readout; the spins go to LDS for the product.
        float sg[NT][4];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                x[t][j] = __builtin_fmaf(eps, v[t][j], x[t][j]);
                sg[t][j] = x[t][j] >= 0.0f ? 1.0f : -1.0f;
            }
            uint32_t w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(0u, sg[t][0], sg[t][1], 1.0f, 0);
            w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, sg[t][2], sg[t][3], 1.0f, 1);
            *reinterpret_cast<uint16_t*>(S + soff + mtt(t) * 16u * srow + cbt(cwt(t)) * 8u) = static_cast<uint16_t>(w);
        }
        squad_barrier(counter, target, lane);  // spins of step k and energy sums of step k - 1 complete
        if (k > 0) records(r3p, sS + ((k + 1) & 1) * sb, k - 1);
        if (sw == 0 && lane < 32) sE[r3n * 32 + lane] = 0.0f;  // read two steps ago

        // Field J s + h on matrix cores, as in team_item.
        v4f I[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) I[t] = sH[cbt(cwt(t)) * 4];
        const unsigned char* brow = S + lr * srow + 16 * lg;
#pragma unroll
        for (int kb = 0; kb < NC; ++kb) {
            v8i B[2], Bh;
            if constexpr (NF > 0) {
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const v4i b = *reinterpret_cast<const v4i*>(brow + m * 16 * srow + kb * 64);
                    B[m] = v8i{b[0], b[1], b[2], b[3], 0, 0, 0, 0};
                }
            }
            if constexpr (HALF) {
                const v4i b = *reinterpret_cast<const v4i*>(brow + mth * 16 * srow + kb * 64);
                Bh = v8i{b[0], b[1], b[2], b[3], 0, 0, 0, 0};
            }
#pragma unroll
            for (int cw = 0; cw < NC; ++cw) {
                const v4i j4 = *reinterpret_cast<const v4i*>(jl + (cbt(cw) * NC + kb) * 1024);
                const v8i A = v8i{j4[0], j4[1], j4[2], j4[3], 0, 0, 0, 0};
                if (cw < NF) {
#pragma unroll
                    for (int m = 0; m < 2; ++m)
                        I[2 * cw + m] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(A, B[m], I[2 * cw + m], 4, 4,
                                                                                         0, 127, 0, 127);
                } else {
                    I[NT - 1] =
                        __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(A, Bh, I[NT - 1], 4, 4, 0, 127, 0, 127);
                }
            }
        }
        // Energy partials s (I + h) of the step, summed over the four lanes of
        // each replica: after the 32-lane swap the lower lanes hold half 0
        // and the upper lanes half 1.
        {
            float part[2] = {0.0f, 0.0f}, ph = 0.0f;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const v4f h = sH[cbt(cwt(t)) * 4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float ih = I[t][j] + h[j];
                    if (t < 2 * NF)
                        part[t & 1] = __builtin_fmaf(sg[t][j], ih, part[t & 1]);
                    else
                        ph = __builtin_fmaf(sg[t][j], ih, ph);
                }
            }
            if constexpr (HALF) {
                part[0] += mth ? 0.0f : ph;
                part[1] += mth ? ph : 0.0f;
            }
            uint32_t p0 = f_to_bits(part[0]), p1 = f_to_bits(part[1]);
            swap32(p0, p1);
            uint32_t c0 = f_to_bits(bits_to_f(p0) + bits_to_f(p1)), c1 = c0;
            swap16(c0, c1);
            const float tot = bits_to_f(c0) + bits_to_f(c1);
            if ((lg & 1) == 0) atomicAdd(sE + r3 * 32 + (lg >> 1) * 16 + lr, tot);
        }
        const float ck = in_vgpr(ck_s);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const float f[4] = {I[t][0], I[t][1], I[t][2], I[t][3]};
            kick_n<DERIV, 4>(x[t], v[t], f, ck, eps, gamma, sk);
        }
        r3 = r3n;
    }
    squad_barrier(counter, target, lane);  // energy sums of the last step complete
    records((r3 == 0) ? 2 : r3 - 1, sS + ((nsteps + 1) & 1) * sb, nsteps - 1);

    // Final state and records of the item.
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        if (!(mtt(t) ? rok[1] : rok[0])) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int col = cbt(cwt(t)) * 16 + col_of(lg, j);
            const int64_t idx = (gr0 + 16 * mtt(t)) * Np + col;
            a.x[idx] = x[t][j];
            a.v[idx] = v[t][j];
            if (col < N) a.bestS[idx] = ((bp[t] >> (4 * j)) & 8u) ? -1 : 1;
        }
    }
    if (sw == 0 && lg < 2 && (lg ? rok[1] : rok[0])) {
        const int64_t gr = gr0 + 16 * lg;
        const float e = lg ? bE[1] : bE[0];
        a.bestE[gr] = e == __builtin_inff() ? INT64_MAX : static_cast<int64_t>(e);
        a.bestStep[gr] = lg ? bK[1] : bK[0];
    }
    return target;
}

// Couplings, fields and cleared spins of one item into `lds` by nthr threads
// (column blocks up to ncb_pad and k positions past Np are zero; spins there
// must hold a finite value).
__device__ __forceinline__ void stage_item(const BatchInst* ap, unsigned char* lds, int ncb_pad, uint32_t sbytes, int t,
                                           int nthr)
{
    const int Np = ap->Np, nkb = nkb4_of(Np);
    const uint32_t n = static_cast<uint32_t>(Np / 16) * nkb * 64u, npad = static_cast<uint32_t>(ncb_pad) * nkb * 64u;
    const uint4* src = reinterpret_cast<const uint4*>(ap->J4);
    uint4* dst = reinterpret_cast<uint4*>(lds + kFixedLds);
    for (uint32_t u = t; u < npad; u += nthr) dst[u] = u < n ? src[u] : uint4{0u, 0u, 0u, 0u};
    uint32_t* sz = reinterpret_cast<uint32_t*>(lds + kFixedLds + npad * 16u);
    for (uint32_t u = t; u < sbytes / 4u; u += nthr) sz[u] = 0u;
    // fields in the order of the lanes' columns
    float* sh = reinterpret_cast<float*>(lds + kFixedLds + npad * 16u + sbytes);
    for (int u = t; u < ncb_pad * 16; u += nthr) {
        const int col = (u & ~15) + col_of((u >> 2) & 3, u & 3);
        sh[u] = col < Np ? static_cast<float>(ap->h[col]) : 0.0f;
    }
    if (t < 96) reinterpret_cast<int32_t*>(lds)[t] = 0;
}

template <int NC>
__device__ __forceinline__ void team_item_d(const BatchInst* a, int blk, LdsByte* lds, int wave, int lane)
{
    if (a->deriv)
        team_item<NC, 1>(a, blk, lds, wave, lane);
    else
        team_item<NC, 0>(a, blk, lds, wave, lane);
}

template <int NF, bool HALF>
__device__ __forceinline__ uint32_t squad_item_d(const BatchInst* a, int blk, LdsByte* lds, uint32_t target,
                                                 int sw, int lane)
{
    return a->deriv ? squad_item<NF, HALF, 1>(a, blk, lds, target, sw, lane)
                    : squad_item<NF, HALF, 0>(a, blk, lds, target, sw, lane);
}

// Every workgroup first takes the items for teams (all sixteen waves on one),
// then its two squads take the others independently; both queues are sorted
// largest first.  A workgroup's first items are given by its index (team item
// b to workgroup b; of the workgroups without one, squad items to the first
// squads before the second ones), later ones come from the queue counters.
__global__ void __launch_bounds__(kBT) __attribute__((amdgpu_waves_per_eu(4)))
k_batch_fp4(const BatchInst* __restrict__ insts, const BatchItem* __restrict__ items, int nteam, int nsquad,
            int* queue, uint32_t squad_lds)
{
    extern __shared__ __align__(16) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grid = static_cast<int>(gridDim.x), b = static_cast<int>(blockIdx.x);
    int* sItem = reinterpret_cast<int*>(lds + 3 * 32 * 4);
    for (int q = b; q < nteam;) {
        const BatchItem it = items[q];
        const BatchInst* ap = insts + it.inst;
        const int nc = nkb4_of(ap->Np);
        stage_item(ap, lds, 8 * nc, 32u * (64u * nc + 16u), tid, kBT);
        __syncthreads();
        switch (nc) {
        case 1: team_item_d<1>(ap, it.block, (LdsByte*)lds, wave, lane); break;
        case 2: team_item_d<2>(ap, it.block, (LdsByte*)lds, wave, lane); break;
        case 3: team_item_d<3>(ap, it.block, (LdsByte*)lds, wave, lane); break;
        default: team_item_d<4>(ap, it.block, (LdsByte*)lds, wave, lane); break;
        }
        __syncthreads();
        if (tid == 0) *sItem = atomicAdd(queue, 1);
        __syncthreads();
        q = __builtin_amdgcn_readfirstlane(*sItem);
    }
    if (nsquad == 0) return;
    // squads, each with half of the LDS
    const int squad = wave >> 3, sw = wave & 7, st = tid & (64 * kSquad - 1);
    unsigned char* base = lds + squad * squad_lds;
    uint32_t* counter = squad_counter(base);
    int* slot = reinterpret_cast<int*>(base + 3 * 32 * 4);
    __syncthreads();
    if (st == 0) *counter = 0u;
    __syncthreads();
    uint32_t target = 0;
    int q = b < nteam ? -1 : (b - nteam) + (squad ? grid - nteam : 0);
    for (;;) {
        if (q < 0) {
            if (st == 0) *slot = atomicAdd(queue + 1, 1);
            squad_barrier(counter, target, lane);
            q = __builtin_amdgcn_readfirstlane(*slot);
        }
        if (q >= nsquad) break;
        const BatchItem it = items[nteam + q];
        const BatchInst* ap = insts + it.inst;
        const int q4 = ap->Np / 64, nkb = nkb4_of(ap->Np);
        stage_item(ap, base, 4 * q4, 2u * 32u * (64u * nkb + 16u), st, 64 * kSquad);
        squad_barrier(counter, target, lane);
        const int blk = it.block;
        switch (q4) {
        case 1: target = squad_item_d<0, true>(ap, blk, (LdsByte*)base, target, sw, lane); break;
        case 2: target = squad_item_d<1, false>(ap, blk, (LdsByte*)base, target, sw, lane); break;
        case 3: target = squad_item_d<1, true>(ap, blk, (LdsByte*)base, target, sw, lane); break;
        default: target = squad_item_d<2, false>(ap, blk, (LdsByte*)base, target, sw, lane); break;
        }
        squad_barrier(counter, target, lane);
        q = -1;
    }
}

// The queues' counters: the first index that no workgroup has by its own.
__global__ void k_batch_queue_reset(int* queue, int first_team, int first_squad)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        queue[0] = first_team;
        queue[1] = first_squad;
    }
}

}  // namespace

bool batch_fp4_squad(int Np) { return Np <= kSquadMaxNp; }

size_t batch_fp4_lds_bytes(int Np, bool squad)
{
    const uint32_t nkb = static_cast<uint32_t>(nkb4_of(Np));
    if (!squad)
        return kFixedLds + 8u * nkb * nkb * 1024u + 32u * (64u * nkb + 16u) + 4u * 128u * nkb;
    return kFixedLds + static_cast<uint32_t>(Np / 16) * nkb * 1024u + 2u * 32u * (64u * nkb + 16u) +
           4u * static_cast<uint32_t>(Np);
}

static size_t launch_lds(size_t team_lds, size_t squad_lds)
{
    return std::max(team_lds, 2 * ((squad_lds + 255) & ~static_cast<size_t>(255)));
}

int batch_fp4_grid(size_t team_lds, size_t squad_lds)
{
    int dev = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    const size_t lds = launch_lds(team_lds, squad_lds);
    const void* f = reinterpret_cast<const void*>(k_batch_fp4);
    if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)) != hipSuccess)
        return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, f, kBT, lds) != hipSuccess) return 0;
    return per * cus;
}

hipError_t launch_batch_fp4(const BatchInst* insts, const BatchItem* items, int nteam, int nsquad, int* queue,
                            size_t team_lds, size_t squad_lds, hipStream_t st)
{
    const int grid = batch_fp4_grid(team_lds, squad_lds);
    if (grid < 1) return hipErrorInvalidConfiguration;
    const int want = std::max(1, nteam + nsquad);
    const int nwg = grid < want ? grid : want;
    const int first_team = std::min(nteam, nwg), first_squad = nteam < nwg ? 2 * (nwg - nteam) : 0;
    hipLaunchKernelGGL(k_batch_queue_reset, dim3(1), dim3(64), 0, st, queue, first_team, first_squad);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_batch_fp4, dim3(static_cast<unsigned>(nwg)), dim3(kBT), launch_lds(team_lds, squad_lds), st,
                       insts, items, nteam, nsquad, queue,
                       static_cast<uint32_t>((squad_lds + 255) & ~static_cast<size_t>(255)));
    return hipGetLastError();
}

}  // namespace phia

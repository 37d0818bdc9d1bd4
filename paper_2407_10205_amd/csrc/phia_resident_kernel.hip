// Resident sweep of the PHIA library for gfx950 (k_sweep_res): one workgroup
// runs every step of four replicas with all of their columns, its couplings in
// the registers and the LDS of one CU.
//
// Layout.  Up to sixteen waves; wave w owns the 16-column blocks w + W i,
// i < CB.  The products take the spins as the A operand and the couplings as
// B, with replica r at operand row 4 r (the other rows repeat it and their
// results are not used): lane (lr, lg) = (lane % 16, lane / 16) then receives
// replica lg, column lr of each block in the first result register, so every
// lane holds one element per block, the kick runs at full lane use, and x, v,
// the field and the record signs stay in VGPRs.  The first CBV blocks of every
// wave keep their coupling fragments in VGPRs for the whole launch, the others
// in LDS; the four rows of spins go to LDS in two buffers by step parity, so a
// step has one barrier.
//
// What it is for.  An anneal of up to some thousand replicas spreads over the
// CUs four replicas at a time, and no step waits for another workgroup: the
// column-split sweeps, which hold the same couplings once per group of CUs,
// wait for their exchange in every step, and the VALU sweep computes the
// products on the VALUs.  us per step, those / this: N = 64, 64 replicas 0.95
// / 0.44; N = 256, 512 replicas 1.28 / 0.72; N = 437 (int8), 1024 replicas
// 3.02 / 1.23; max-cut N = 800, 1024 replicas 2.92 / 1.99.
// Bound: the chain of one step (spins from LDS, products, kick, spins and
// energy sums to LDS, barrier) at small N, then instruction issue: at N = 800
// each SIMD issues four waves' 91 products of 16 cycles and 13 kicks of about
// 60 instructions per step.  A quarter of the matrix-core rows is used.
// Accept/reject step (L = 25), the column split / this: N = 64, 256 replicas
// 2.0 / 0.52 us per step, N = 500 4.1 / 1.23, N = 800 4.6 / 2.6.
//
// Operands: FP4 couplings and spins (v_mfma_scale_f32_16x16x128_f8f6f4, FP32
// accumulation of integers below 2^24: exact) or int8 (v_mfma_i32_16x16x64_i8).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "phia_devmath.h"
#include "phia_devsweep.h"
#include "phia_internal.h"

namespace phia {

namespace {

constexpr int kResWaves = 16;
constexpr int kResRows = 4;  // replicas per workgroup

// Row energies [3][4] int32 or float; the accept/reject step's state (ResMh);
// then [2 parities][4 rows][stride] spins and the coupling fragments of the
// blocks past the resident ones.
struct ResMh {
    unsigned long long q[8];   // kinetic units at the trajectory's end [4], start [4]
    int64_t Es[4], El[4];      // energy at the trajectory's start, of the last step before this launch
    float lam[4];              // beta multipliers
    int32_t out[4], acc[4], dec[4];
};
constexpr uint32_t kResMh = 64, kResFixed = 256;
static_assert(kResMh + sizeof(ResMh) <= kResFixed, "LDS head");
__host__ __device__ inline uint32_t res_srow(int nkb) { return 64u * static_cast<uint32_t>(nkb) + 16u; }
__host__ __device__ inline uint32_t res_sbytes(int nkb) { return 2u * kResRows * res_srow(nkb); }

// Gaussian draws of the wave's elements of one generator round: block b = 8 i
// + 2 replica + half of the wave's CB column blocks is generated by the lane
// pair 2 b, 2 b + 1 (two Box-Muller pairs each), and every element reads its
// draw from the lane that made it.  A call, so that the step does not hold
// generator states.
struct Draws {
    float g[4];
};
__device__ __attribute__((noinline)) Draws res_draws(uint64_t seed, uint64_t replica, uint64_t round, uint64_t c8,
                                                     int half)
{
    float g[4];
    gauss_block_half(seed, replica, round, c8, half, g);
    return Draws{{g[0], g[1], g[2], g[3]}};
}

// The decision of one replica and its multiplier after it; a call for the
// same reason.
struct Decision {
    int out;
    float lam;
};
__device__ __attribute__((noinline)) Decision res_decide(uint64_t seed, uint64_t rs, int64_t traj, int64_t Es, int64_t Ee,
                                                         int64_t dq, float beta, float lam, float sigma, float up,
                                                         float down)
{
    const int out = mh_outcome(seed, rs, traj, Es, Ee, dq, beta, lam, sigma);
    return Decision{out, mh_lambda(lam, out, up, down)};
}

template <bool FP4, int CB, int CBV, int NKB, int DERIV, bool MH>
__global__ void __launch_bounds__(64 * kResWaves) __attribute__((amdgpu_waves_per_eu(4))) k_sweep_res(SweepArgs a)
{
    static_assert(CB <= 4, "one lane pair per generator block");
    extern __shared__ __align__(16) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int W = __builtin_amdgcn_readfirstlane(static_cast<int>(blockDim.x >> 6));
    const int lr = lane & 15, lg = lane >> 4;
    const int Np = a.Np, N = a.N, ncb = (N + 15) / 16;
    constexpr uint32_t srow = 64u * NKB + 16u, sbuf = kResRows * srow;
    float* sEf = reinterpret_cast<float*>(lds);
    int32_t* sEi = reinterpret_cast<int32_t*>(lds);  // [3][4], step k in k mod 3
    unsigned char* sS = lds + kResFixed;
    unsigned char* sJ = sS + 2u * sbuf;
    const int nkb = FP4 ? (Np + 127) / 128 : Np / 64;  // packed k blocks
    const unsigned char* Jg = static_cast<const unsigned char*>(a.J);
    const int64_t rep = static_cast<int64_t>(blockIdx.x) * kResRows + lg;  // the lane's replica
    const bool rok = rep < a.R;
    auto cbt = [&](int i) { return wave + W * i; };
    auto has = [&](int i) { return i == 0 ? true : cbt(i) < ncb; };  // W <= ncb

    // couplings: resident fragments (zero past the packed k blocks), the rest to LDS
    v4i jr[CBV][NKB];
#pragma unroll
    for (int i = 0; i < CBV; ++i)
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
            jr[i][kb] = (has(i) && kb < nkb)
                            ? *reinterpret_cast<const v4i*>(Jg + (static_cast<size_t>(cbt(i)) * nkb + kb) * 1024 + lane * 16)
                            : v4i{0, 0, 0, 0};
    if constexpr (CB > CBV) {
        // column blocks W CBV .. ncb - 1, NKB fragments each
        const int n = (ncb - W * CBV) * NKB * 64;
        v4i* dst = reinterpret_cast<v4i*>(sJ);
        for (int u = tid; u < n; u += W * 64) {
            const int c = u / (NKB * 64), kb = (u >> 6) % NKB;
            dst[u] = kb < nkb ? *reinterpret_cast<const v4i*>(
                                    Jg + (static_cast<size_t>(W * CBV + c) * nkb + kb) * 1024 + (u & 63) * 16)
                              : v4i{0, 0, 0, 0};
        }
    }
    // spins of k positions that no column owns must be finite
    for (uint32_t u = tid; u < (kResFixed + 2u * sbuf) / 4u; u += W * 64) reinterpret_cast<uint32_t*>(lds)[u] = 0u;

    float x[CB], v[CB], sf[CB];
    int hi[CB];
    float hf[CB];
    uint32_t best = 0;  // record spins, bit i: +1
#pragma unroll
    for (int i = 0; i < CB; ++i) {
        const int col = cbt(i) * 16 + lr;
        const bool ok = has(i) && rok && col < N;
        const int64_t idx = rep * Np + col;
        x[i] = ok ? a.x[idx] : 0.0f;
        v[i] = ok ? a.v[idx] : 0.0f;
        hi[i] = has(i) && col < N ? a.h[col] : 0;
        hf[i] = static_cast<float>(hi[i]);
        sf[i] = 1.0f;
        if (ok && a.bestS[idx] > 0) best |= 1u << i;
    }
    // record energies: int32 or float, "none yet" above every energy
    int32_t bEi = INT32_MAX;
    float bEf = __builtin_inff();
    int64_t bK = -1;
    if (rok) {
        const int64_t b = a.bestE[rep];
        if (b != INT64_MAX) {
            bEi = static_cast<int32_t>(b);
            bEf = static_cast<float>(b);
        }
        bK = a.bestStep[rep];
    }
    // the kick's constants (and multiplier) in VGPRs, unless the couplings need
    // the registers (N = 800: 2.43 us per step with them, their spills in the
    // step, 1.99 without; accept/reject 2.79 and 2.58)
    constexpr bool kHeld = CBV * NKB <= 10;
    const float eps = kHeld ? in_vgpr(a.eps) : a.eps, gamma = kHeld ? in_vgpr(a.gamma) : a.gamma;
    Sech2K sk{};
    if constexpr (DERIV == 0 && kHeld) sk = sech2_in_vgprs();
    // accept/reject: the first lane of a replica's row in wave 0 decides
    ResMh* const sM = reinterpret_cast<ResMh*>(lds + kResMh);
    const bool decider = MH && wave == 0 && lr == 0 && rok;
    float lam = 1.0f;  // kHeld: the replica's multiplier
    if (MH && rok) lam = a.lam[rep];
    if (MH && tid < 4) sM->lam[tid] = 1.0f;
    const int64_t L = a.L;
    int64_t next_ref = a.k0 + (L - a.k0 % L) % L;
    uint64_t round = static_cast<uint64_t>(next_ref / L);
    // where the lane's spins go in a buffer: FP4, the byte that holds columns
    // lr and lr + 4 of a group of 8 (codes ordered 0 4 1 5 2 6 3 7), written
    // by the lanes of the lower column; int8, the column's byte
    const uint32_t soff = static_cast<uint32_t>(lg) * srow +
                          (FP4 ? 4u * (lr >> 3) + (lr & 3) : static_cast<uint32_t>(lr));
    const bool writer = !FP4 || (lr & 4) == 0;
    const unsigned char* const arow = sS + static_cast<uint32_t>(lr >> 2) * srow + 16 * lg;
    __syncthreads();
    if (decider) {
        sM->q[4 + lg] = a.k0 > 0 ? static_cast<unsigned long long>(a.mhQ[rep]) : 0ull;
        sM->Es[lg] = a.mhE[rep * 2];
        sM->El[lg] = a.mhE[rep * 2 + 1];
        sM->lam[lg] = lam;
        sM->acc[lg] = a.mhc[rep * 2];
        sM->dec[lg] = a.mhc[rep * 2 + 1];
    }
    if constexpr (MH) __syncthreads();

    // The steps, for a wave with NB column blocks (its last one may be past
    // the end; the same barriers in either copy).
    auto run = [&](auto nb) {
        constexpr int NB = decltype(nb)::value;
        auto records = [&](int64_t kp, int r3p) {
            const uint32_t slot = static_cast<uint32_t>(r3p) * 4u + lg;
            bool imp;
            if constexpr (FP4) {
                const float E = -0.5f * sEf[slot];  // the sum is even: exact
                imp = E < bEf;
                bEf = imp ? E : bEf;
                if (a.etrace && wave == 0 && lr == 0 && rok) a.etrace[rep * a.T + kp] = static_cast<int64_t>(E);
            } else {
                const int32_t E = -(sEi[slot] >> 1);
                imp = E < bEi;
                bEi = imp ? E : bEi;
                if (a.etrace && wave == 0 && lr == 0 && rok) a.etrace[rep * a.T + kp] = E;
            }
            // late in an anneal few steps improve a record; the wave's own spins
            // of the step are still in their buffer
            if (__any(imp)) {
                const unsigned char* S = sS + static_cast<uint32_t>(kp & 1) * sbuf + soff;
                uint32_t m = 0;
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                        if constexpr (FP4) {
                        // byte of the pair's lower lane, high code for the upper one
                        const unsigned char w = S[cbt(i) * 8];
                        m |= ((w >> ((lr & 4) ? 7 : 3)) & 1u ? 0u : 1u) << i;
                    } else {
                        m |= (S[cbt(i) * 16] & 0x80u ? 0u : 1u) << i;
                    }
                }
                best = imp ? m : best;
                bK = imp ? kp : bK;
            }
        };

        // energy of a replica from its sum (which is even)
        auto energy = [&](int slot) -> int64_t {
            return FP4 ? static_cast<int64_t>(-0.5f * sEf[slot]) : -(sEi[slot] >> 1);
        };
        // kinetic units of the lane's replica, added up in q[at]
        auto kinetic = [&](int at) {
            long long q = 0;
#pragma unroll
            for (int i = 0; i < NB; ++i)
                if (rok && cbt(i) * 16 + lr < N) q += kin_units(x[i], v[i]);
            q = wave_sum16_i64(q);
            if (lr == 0) atomicAdd(sM->q + at + lg, static_cast<unsigned long long>(q));
        };
        const ConstF ctab = scalar_table(a.ctab);
        int r3 = static_cast<int>(a.k0 % 3);
        for (int64_t k = a.k0; k < a.k1; ++k) {
            const int r3p = (r3 == 0) ? 2 : r3 - 1, r3n = (r3 == 2) ? 0 : r3 + 1;
            const float ck_s = ctab[k];
            if (k == next_ref) {  // momentum refresh
                if (MH && k > 0) {
                    // End of a trajectory: one decision per replica, and x back
                    // to the trajectory's start where it was rejected.
                    kinetic(0);
                    __syncthreads();  // the kinetic units, the energy sums of step k - 1
                    if (decider) {
                        const int64_t Ee = k > a.k0 ? energy(r3p * 4 + lg) : sM->El[lg];
                        const Decision d = res_decide(a.seed, static_cast<uint64_t>(a.r_base + rep), k / L - 1, sM->Es[lg],
                                                      Ee, static_cast<int64_t>(sM->q[lg] - sM->q[4 + lg]),
                                                      a.btab[k - 1], sM->lam[lg], a.sigma, a.mh_up, a.mh_down);
                        sM->out[lg] = d.out;
                        sM->lam[lg] = d.lam;
                        if (d.out != 0) sM->Es[lg] = Ee;
                        if (d.out >= 0) {
                            sM->acc[lg] += d.out;
                            sM->dec[lg] += 1;
                        }
                        sM->q[lg] = sM->q[4 + lg] = 0;
                    }
                    __syncthreads();
                    if (rok) {
                        lam = sM->lam[lg];
                        if (sM->out[lg] == 0)
#pragma unroll
                            for (int i = 0; i < NB; ++i)
                                if (cbt(i) * 16 + lr < N) x[i] = a.x0[rep * Np + cbt(i) * 16 + lr];
                    }
                }
                const int b = lane >> 1, bi = b >> 3;  // block: column block bi, replica (b >> 1) & 3, half b & 1
                const Draws d = res_draws(a.seed, static_cast<uint64_t>(a.r_base + static_cast<int64_t>(blockIdx.x) * kResRows + ((b >> 1) & 3)),
                                          round, static_cast<uint64_t>(wave + W * bi) * 2 + (b & 1), lane & 1);
                const int p = (lr & 7) >> 1;  // pair of the column within its block
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    const int src = 2 * (8 * i + 2 * lg + (lr >> 3)) + (p >> 1);
                    const float t0 = lane_read(src, d.g[0]), t1 = lane_read(src, d.g[1]);
                    const float t2 = lane_read(src, d.g[2]), t3 = lane_read(src, d.g[3]);
                    const float lo = (lr & 1) ? t1 : t0, up = (lr & 1) ? t3 : t2;
                    v[i] = (rok && cbt(i) * 16 + lr < N) ? ((p & 1) ? up : lo) : 0.0f;
                }
                ++round;
                next_ref += L;
                if constexpr (MH) {  // start of a trajectory
#pragma unroll
                    for (int i = 0; i < NB; ++i)
                        if (rok && cbt(i) * 16 + lr < N) a.x0[rep * Np + cbt(i) * 16 + lr] = x[i];
                    kinetic(4);
                }
            }
            // Drift and readout.
            unsigned char* S = sS + static_cast<uint32_t>(k & 1) * sbuf;
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                x[i] = __builtin_fmaf(eps, v[i], x[i]);
                sf[i] = x[i] >= 0.0f ? 1.0f : -1.0f;
                if constexpr (FP4) {
                    const float up = __builtin_bit_cast(
                        float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, sf[i]), 0x104, 0xf, 0xf, true));  // row_shl:4
                    const uint32_t w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(0u, sf[i], up, 1.0f, 0);
                    if (writer) S[soff + cbt(i) * 8] = static_cast<unsigned char>(w);
                } else {
                    S[soff + cbt(i) * 16] = x[i] >= 0.0f ? 1 : 0xff;
                }
            }
            __syncthreads();  // spins of step k and energy sums of step k - 1 complete
            if (k > a.k0) records(k - 1, r3p);
            if (tid < 4) sEi[r3n * 4 + tid] = 0;  // read in the step before

            // Field J s on matrix cores.
            v4f af[NB];
            v4i ai[NB];
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                af[i] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
                ai[i] = v4i{0, 0, 0, 0};
            }
            const unsigned char* Ar = arow + static_cast<uint32_t>(k & 1) * sbuf;
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb) {
                const v4i s4 = *reinterpret_cast<const v4i*>(Ar + kb * 64);
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                        v4i j4;
                    if (i < CBV)
                        j4 = jr[i < CBV ? i : 0][kb];
                    else
                        j4 = *reinterpret_cast<const v4i*>(sJ + ((cbt(i) - W * CBV) * NKB + kb) * 1024 + lane * 16);
                    if constexpr (FP4)
                        af[i] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
                            v8i{s4[0], s4[1], s4[2], s4[3], 0, 0, 0, 0}, v8i{j4[0], j4[1], j4[2], j4[3], 0, 0, 0, 0}, af[i],
                            4, 4, 0, 127, 0, 127);
                    else
                        ai[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(s4, j4, ai[i], 0, 0, 0);
                }
            }
            // Energy partials s (I + h), summed over the 16 columns of a block by
            // DPP and over the waves by LDS atomics.
            float If[NB];
            const uint32_t slot = static_cast<uint32_t>(r3) * 4u + lg;
            if constexpr (FP4) {
                float part = 0.0f;
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    If[i] = af[i][0] + hf[i];
                    part = __builtin_fmaf(sf[i], If[i] + hf[i], part);
                }
                part += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, part), 0xb1, 0xf, 0xf, false));
                part += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, part), 0x4e, 0xf, 0xf, false));
                part += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, part), 0x141, 0xf, 0xf, false));
                part += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, part), 0x140, 0xf, 0xf, true));
                if (lr == 0) atomicAdd(sEf + slot, part);
            } else {
                int part = 0;
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    const int I = ai[i][0] + hi[i];
                    If[i] = static_cast<float>(I);
                    const int ih = I + hi[i];
                    part += x[i] >= 0.0f ? ih : -ih;
                }
                part = row_sum16_dpp(part);
                if (lr == 0) atomicAdd(sEi + slot, part);
            }
            const float ck = MH ? ck_s * (kHeld ? lam : sM->lam[lg]) : in_vgpr(ck_s);
            float xn[NB], vn[NB];
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                xn[i] = x[i];
                vn[i] = v[i];
            }
            kick_n<DERIV, NB>(xn, vn, If, ck, eps, gamma, sk);
#pragma unroll
            for (int i = 0; i < NB; ++i) v[i] = vn[i];
            r3 = r3n;
        }
        __syncthreads();
        records(a.k1 - 1, (r3 == 0) ? 2 : r3 - 1);

    };
    if constexpr (CB > 1) {
        if (has(CB - 1))
            run(std::integral_constant<int, CB>{});
        else
            run(std::integral_constant<int, CB - 1>{});
    } else {
        run(std::integral_constant<int, CB>{});
    }

#pragma unroll
    for (int i = 0; i < CB; ++i) {
        const int col = cbt(i) * 16 + lr;
        if (!has(i) || !rok || col >= N) continue;
        a.x[rep * Np + col] = x[i];
        a.v[rep * Np + col] = v[i];
        a.bestS[rep * Np + col] = ((best >> i) & 1u) ? 1 : -1;
    }
    if (decider) {
        const int slot = static_cast<int>((a.k1 - 1) % 3) * 4 + lg;
        a.mhE[rep * 2] = sM->Es[lg];
        a.mhE[rep * 2 + 1] = FP4 ? static_cast<int64_t>(-0.5f * sEf[slot]) : -(sEi[slot] >> 1);
        a.mhQ[rep] = static_cast<int64_t>(sM->q[4 + lg]);
        a.lam[rep] = sM->lam[lg];
        a.mhc[rep * 2] = sM->acc[lg];
        a.mhc[rep * 2 + 1] = sM->dec[lg];
    }
    if (wave == 0 && lr == 0 && rok) {
        if constexpr (FP4)
            a.bestE[rep] = bEf == __builtin_inff() ? INT64_MAX : static_cast<int64_t>(bEf);
        else
            a.bestE[rep] = bEi == INT32_MAX ? INT64_MAX : bEi;
        a.bestStep[rep] = bK;
    }
}

// One variant's kernel; columns blocks up to 16 CB, k blocks up to NKB.
template <bool FP4, int CB, int CBV, int NKB>
const void* res_kernel(int deriv, int mh)
{
    if (mh)
        return deriv ? reinterpret_cast<const void*>(k_sweep_res<FP4, CB, CBV, NKB, 1, true>)
                     : reinterpret_cast<const void*>(k_sweep_res<FP4, CB, CBV, NKB, 0, true>);
    return deriv ? reinterpret_cast<const void*>(k_sweep_res<FP4, CB, CBV, NKB, 1, false>)
                 : reinterpret_cast<const void*>(k_sweep_res<FP4, CB, CBV, NKB, 0, false>);
}

struct ResVariant {
    bool fp4;
    int max_ncb, cbv, nkb;
    const void* (*kernel)(int deriv, int mh);
};
// Coupling fragments in VGPRs: at most 16 per wave (64 registers); what is
// past the first cbv blocks per wave must fit the LDS.
const ResVariant kResVariants[] = {
    {true, 8, 1, 1, res_kernel<true, 1, 1, 1>},   {true, 16, 1, 2, res_kernel<true, 1, 1, 2>},
    {true, 24, 2, 3, res_kernel<true, 2, 2, 3>},  {true, 32, 2, 4, res_kernel<true, 2, 2, 4>},
    {true, 40, 2, 5, res_kernel<true, 3, 2, 5>},  {true, 48, 2, 6, res_kernel<true, 3, 2, 6>},
    {true, 56, 2, 7, res_kernel<true, 4, 2, 7>},  {false, 4, 1, 1, res_kernel<false, 1, 1, 1>},
    {false, 8, 1, 2, res_kernel<false, 1, 1, 2>}, {false, 16, 1, 4, res_kernel<false, 1, 1, 4>},
    {false, 24, 2, 6, res_kernel<false, 2, 2, 6>}, {false, 28, 2, 7, res_kernel<false, 2, 2, 7>},
    {false, 32, 1, 8, res_kernel<false, 2, 1, 8>},
};

const ResVariant* res_variant(int N, int fp4)
{
    const int ncb = (N + 15) / 16;
    for (const ResVariant& v : kResVariants)
        if (v.fp4 == (fp4 != 0) && ncb <= v.max_ncb) return &v;
    return nullptr;
}

size_t res_lds(const ResVariant& v, int N)
{
    const int ncb = (N + 15) / 16, w = std::min(ncb, kResWaves);
    const int over = std::max(0, ncb - w * v.cbv);
    return kResFixed + res_sbytes(v.nkb) + static_cast<size_t>(over) * v.nkb * 1024u;
}

}  // namespace

// LDS of the resident sweep for N columns, 0 where it does not hold them.
size_t sweep_res_lds_bytes(int N, int fp4)
{
    const ResVariant* v = res_variant(N, fp4);
    if (!v) return 0;
    const size_t b = res_lds(*v, N);
    return b <= static_cast<size_t>(kLdsMax) ? b : 0;
}

hipError_t launch_sweep_res(int fp4, const SweepArgs& a, hipStream_t st)
{
    const size_t lds = sweep_res_lds_bytes(a.N, fp4);
    const ResVariant* v = res_variant(a.N, fp4);
    if (lds == 0 || a.R < 1 || a.k1 <= a.k0) return hipErrorInvalidValue;
    const void* kern = v->kernel(a.deriv ? 1 : 0, a.mh);
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
        if (e != hipSuccess) return e;
    }
    const int waves = std::min((a.N + 15) / 16, kResWaves);
    SweepArgs copy = a;
    void* args[] = {&copy};
    const unsigned blocks = static_cast<unsigned>((a.R + kResRows - 1) / kResRows);
    const hipError_t e = hipLaunchKernel(kern, dim3(blocks), dim3(static_cast<unsigned>(64 * waves)), args, lds, st);
    return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace phia

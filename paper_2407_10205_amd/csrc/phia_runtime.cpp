// Host runtime of the PHIA library: validation and fixed-point packing of the
// instance, choice of the J.s arithmetic and of the kernel geometry, device
// memory, schedule tables, launches and error reporting behind the C ABI of
// include/phia.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <new>
#include <string>
#include <vector>

#include "phia.h"
#include "phia_internal.h"
#include "phia_problem.h"

using namespace phia;

namespace phia {

static thread_local std::string g_err;

phia_status fail(phia_status st, const char* fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return st;
}

phia_status hip_fail(phia_problem* p, hipError_t e, const char* what)
{
    if (p) p->poisoned = true;
    return fail(PHIA_EDEVICE, "%s: %s", what, hipGetErrorString(e));
}

void clear_error() { g_err.clear(); }

template <class T>
static void dfree(T*& ptr)
{
    if (ptr) (void)hipFree(ptr);
    ptr = nullptr;
}

static hipError_t dalloc(void** ptr, size_t bytes, size_t* counter)
{
    hipError_t e = hipMalloc(ptr, bytes ? bytes : 16);
    if (e == hipSuccess && counter) *counter += bytes;
    return e;
}

// ------------------------------------------------------------- packing --
// Grid check: v * 2^f is an integer.
static bool on_grid(double v, int f)
{
    const double t = std::ldexp(v, f);
    return t == std::nearbyint(t);
}

phia_status pack_instance(const double* J, const double* h, int N, int frac_bits, int quantize,
                          std::vector<int32_t>& Ji, std::vector<int32_t>& hi, int& f_out, bool& exact)
{
    const int64_t NN = static_cast<int64_t>(N) * N;
    for (int i = 0; i < N; ++i) {
        if (J[static_cast<int64_t>(i) * N + i] != 0.0) return fail(PHIA_EDIAG, "J[%d][%d] != 0", i, i);
        for (int j = 0; j < N; ++j) {
            const double a = J[static_cast<int64_t>(i) * N + j];
            if (!std::isfinite(a)) return fail(PHIA_EINVAL, "J[%d][%d] is not finite", i, j);
            if (a != J[static_cast<int64_t>(j) * N + i]) return fail(PHIA_ENOTSYM, "J[%d][%d] != J[%d][%d]", i, j, j, i);
        }
    }
    if (h)
        for (int i = 0; i < N; ++i)
            if (!std::isfinite(h[i])) return fail(PHIA_EINVAL, "h[%d] is not finite", i);
    int f = frac_bits;
    if (f > 15) return fail(PHIA_EINVAL, "frac_bits must be in [-1, 15]");
    if (f < 0) {
        for (f = 0; f <= 15; ++f) {
            bool ok = true;
            for (int64_t t = 0; ok && t < NN; ++t) ok = on_grid(J[t], f);
            for (int i = 0; ok && h && i < N; ++i) ok = on_grid(h[i], f);
            if (ok) break;
        }
        if (f > 15) {
            if (!quantize) return fail(PHIA_ERANGE, "couplings are not on any grid 2^-f with f <= 15");
            f = 15;
        }
    }
    exact = true;
    Ji.assign(static_cast<size_t>(NN), 0);
    hi.assign(static_cast<size_t>(N), 0);
    for (int64_t t = 0; t < NN; ++t) {
        const double a = std::ldexp(J[t], f), q = std::nearbyint(a);
        if (q != a) {
            if (!quantize) return fail(PHIA_ERANGE, "J entry %lld is off the 2^-%d grid", (long long)t, f);
            exact = false;
        }
        if (std::fabs(q) >= 1073741824.0) return fail(PHIA_ERANGE, "J entry %lld out of range", (long long)t);
        Ji[static_cast<size_t>(t)] = static_cast<int32_t>(q);
    }
    for (int i = 0; i < N; ++i) {
        const double a = h ? std::ldexp(h[i], f) : 0.0, q = std::nearbyint(a);
        if (q != a) {
            if (!quantize) return fail(PHIA_ERANGE, "h[%d] is off the 2^-%d grid", i, f);
            exact = false;
        }
        if (std::fabs(q) >= 1073741824.0) return fail(PHIA_ERANGE, "h[%d] out of range", i);
        hi[static_cast<size_t>(i)] = static_cast<int32_t>(q);
    }
    f_out = f;
    return PHIA_OK;
}

// FP4 (E2M1) code of an integer coupling, or -1 if it has none: the
// representable integers are 0, +-1, +-2, +-3, +-4, +-6.
static int fp4_code(int v)
{
    const int a = v < 0 ? -v : v;
    static const int mag[7] = {0, 2, 4, 5, 6, -1, 7};  // |v| = 0, 1, 2, 3, 4, 5, 6
    if (a > 6 || mag[a] < 0) return -1;
    return (v < 0 && a != 0 ? 8 : 0) | mag[a];
}

// FP4 fragment-major: [Np/16 col blocks][nkb4][64 lanes][16 bytes] with
// nkb4 = ceil(Np / 128).  Lane l holds column cb*16 + l%16 and the 32 k
// positions 128 kb + 32 (l/16) + t, element t in nibble t (low nibble first).
// Within each group of 8 k positions the spins are ordered 0 4 1 5 2 6 3 7,
// the order in which the sweep expands a byte of spin bits.
static void pack_fp4(const std::vector<int32_t>& Ji, int N, int Np, std::vector<uint8_t>& out)
{
    static const int perm[8] = {0, 4, 1, 5, 2, 6, 3, 7};
    const int ncb = Np / 16, nkb4 = (Np + 127) / 128;
    out.assign(static_cast<size_t>(ncb) * nkb4 * 64 * 16, 0);
    for (int cb = 0; cb < ncb; ++cb)
        for (int kb = 0; kb < nkb4; ++kb)
            for (int l = 0; l < 64; ++l) {
                const int i = cb * 16 + (l & 15);
                uint8_t* dst = &out[((static_cast<size_t>(cb) * nkb4 + kb) * 64 + l) * 16];
                for (int t = 0; t < 32; ++t) {
                    const int kpos = kb * 128 + 32 * (l >> 4) + t;
                    const int j = 8 * (kpos / 8) + perm[kpos % 8];
                    const int v = (i < N && j < N) ? Ji[static_cast<size_t>(i) * N + j] : 0;
                    const int c = fp4_code(v);
                    dst[t >> 1] |= static_cast<uint8_t>((c & 15) << (4 * (t & 1)));
                }
            }
}

// I8 fragment-major: [Np/16][Np/64][64 lanes][16 bytes].
static void pack_i8(const std::vector<int32_t>& Ji, int N, int Np, std::vector<int8_t>& out)
{
    const int ncb = Np / 16, nkb = Np / 64;
    out.assign(static_cast<size_t>(Np) * Np, 0);
    for (int cb = 0; cb < ncb; ++cb)
        for (int kb = 0; kb < nkb; ++kb)
            for (int l = 0; l < 64; ++l) {
                const int i = cb * 16 + (l & 15);
                int8_t* dst = &out[((static_cast<size_t>(cb) * nkb + kb) * 64 + l) * 16];
                for (int t = 0; t < 16; ++t) {
                    const int j = kb * 64 + 16 * (l >> 4) + t;
                    dst[t] = (i < N && j < N) ? static_cast<int8_t>(Ji[static_cast<size_t>(i) * N + j]) : 0;
                }
            }
}

// ELL: [D][Np] int32, D = the largest number of nonzeros in a row (at least
// 1); slot d of row i holds (J_ij << 16) | j for the d-th nonzero of row i in
// ascending j, zero past the row's last nonzero (coupling 0: no effect).
static void pack_ell(const std::vector<int32_t>& Ji, int N, int Np, std::vector<int32_t>& out, int& D)
{
    D = 1;
    for (int i = 0; i < N; ++i) {
        int d = 0;
        for (int j = 0; j < N; ++j) d += Ji[static_cast<size_t>(i) * N + j] != 0;
        D = std::max(D, d);
    }
    out.assign(static_cast<size_t>(D) * Np, 0);
    for (int i = 0; i < N; ++i) {
        int d = 0;
        for (int j = 0; j < N; ++j) {
            const int32_t v = Ji[static_cast<size_t>(i) * N + j];
            if (v == 0) continue;
            out[static_cast<size_t>(d) * Np + i] =
                static_cast<int32_t>((static_cast<uint32_t>(v) << 16) | static_cast<uint32_t>(j));
            ++d;
        }
    }
}

static uint16_t bf16_of_int(int v)
{
    // |v| <= 256: exact in bfloat16 (8 significant bits).
    const float f = static_cast<float>(v);
    uint32_t b;
    std::memcpy(&b, &f, 4);
    return static_cast<uint16_t>(b >> 16);
}

// BF16 hi/lo fragment-major: [Np/16][Np/32][2][64 lanes][8 bf16].
static void pack_bf16(const std::vector<int32_t>& Ji, int N, int Np, std::vector<uint16_t>& out)
{
    const int ncb = Np / 16, nkc = Np / 32;
    out.assign(static_cast<size_t>(Np) * Np * 2, 0);
    for (int cb = 0; cb < ncb; ++cb)
        for (int kc = 0; kc < nkc; ++kc)
            for (int pl = 0; pl < 2; ++pl)
                for (int l = 0; l < 64; ++l) {
                    const int i = cb * 16 + (l & 15);
                    uint16_t* dst = &out[(((static_cast<size_t>(cb) * nkc + kc) * 2 + pl) * 64 + l) * 8];
                    for (int t = 0; t < 8; ++t) {
                        const int j = kc * 32 + 8 * (l >> 4) + t;
                        const int v = (i < N && j < N) ? Ji[static_cast<size_t>(i) * N + j] : 0;
                        const int lo = ((v + 128) & 255) - 128;
                        const int hi = (v - lo) / 256;
                        dst[t] = bf16_of_int(pl == 0 ? hi : lo);
                    }
                }
}

// ------------------------------------------------------- kernel geometry --
// ------------------------------------------------------- tuning cache --
// One line per tuned shape: "phia-tune5 path Np R kind mt cbw G jlds xcd us_per_step"
// (kinds 4 and 6, the VALU and the split sweep: replicas per workgroup or group in place of mt).
// Lines with the tag phia-tune4 were timed without the resident and the split
// sweep and would pin what these take the place of; they count only for
// shapes that neither holds.
static const char* tune_cache_path() { return std::getenv("PHIA_TUNE_CACHE"); }

static const char* path_name(int path)
{
    switch (path) {
    case PHIA_PATH_FP32: return "FP32";
    case PHIA_PATH_I8: return "int8";
    case PHIA_PATH_BF16HILO: return "BF16 hi/lo";
    case PHIA_PATH_ELL: return "ELL";
    default: return "?";
    }
}

static bool make_geometry(phia_problem* p, int R, int mt, int cbw, int G, int j_lds, Geometry& g, int xcd = -1);
static bool make_geometry_pp(phia_problem* p, int R, int G, int fp4, Geometry& g, int xcd = -1, int jg = 0);
static bool make_geometry_valu(phia_problem* p, int R, int rb, Geometry& g);
static bool make_geometry_res(phia_problem* p, int R, Geometry& g);
static bool make_geometry_split(phia_problem* p, int R, int rows, int G, Geometry& g);

static bool lookup_tune_cache(phia_problem* p, int R)
{
    const char* path = tune_cache_path();
    if (!path) return false;
    FILE* f = std::fopen(path, "r");
    if (!f) return false;
    char tag[32];
    int pa, np, r, kind, mt, cbw, G, jl, xcd;
    double us;
    bool found = false;
    Geometry g;
    while (std::fscanf(f, "%31s %d %d %d %d %d %d %d %d %d %lf", tag, &pa, &np, &r, &kind, &mt, &cbw, &G, &jl, &xcd,
                       &us) == 11) {
        const bool older = std::strcmp(tag, "phia-tune4") == 0;
        if ((older || std::strcmp(tag, "phia-tune5") == 0) && pa == p->path && np == p->Np && r == R &&
            !(older && (make_geometry_res(p, R, g) || make_geometry_split(p, R, 0, 0, g))) &&
            (kind == 6   ? make_geometry_split(p, R, mt, G, g)
             : kind == 5 ? make_geometry_res(p, R, g)
             : kind == 4 ? make_geometry_valu(p, R, mt, g)
             : kind >= 1 ? make_geometry_pp(p, R, G, kind == 2, g, xcd, kind == 1 && jl == 0)
                         : make_geometry(p, R, mt, cbw, G, jl, g, xcd))) {
            p->geo = g;
            found = true;
        }
    }
    std::fclose(f);
    return found;
}

static void append_tune_cache(const phia_problem* p, int R, const Geometry& g, double us)
{
    const char* path = tune_cache_path();
    if (!path) return;
    FILE* f = std::fopen(path, "a");
    if (!f) return;
    std::fprintf(f, "phia-tune5 %d %d %d %d %d %d %d %d %d %.3f\n", p->path, p->Np, R, g.kind,
                 g.kind == 4 || g.kind == 6 ? g.rows : g.mt, g.cbw, g.G,
                 g.j_lds, g.xcd_map, us);
    std::fclose(f);
}

// Placement of a group's workgroups over the 8 XCDs (round-robin dispatch:
// workgroup b runs on XCD b mod 8).  xcd_map = 1 puts all members of a group
// on one XCD; 0 puts member m of every group on XCD m mod 8 (G a multiple of
// 8), so that each XCD's L2 holds only its members' slices of a J that is
// streamed every step.  Default: 1, unless J is streamed from L2 and larger
// than half an XCD's 4 MiB L2.  xcd = 0 or 1 forces a placement; false if
// it cannot apply.
static bool pick_xcd(const phia_problem* p, int G, int ngroups, int j_lds, int xcd, int& out)
{
    const bool same_ok = G > 1 && ngroups % 8 == 0;
    if (xcd == 1) {
        out = 1;
        return same_ok;
    }
    if (xcd == 0) {
        out = 0;
        return true;
    }
    const double jbytes = static_cast<double>(p->Np) * p->Np * (p->path == PHIA_PATH_I8 ? 1 : 4);
    out = (same_ok && (j_lds || jbytes <= 2.0 * 1024 * 1024)) ? 1 : 0;
    return true;
}

// Complete a candidate launch geometry (mt row tiles per block, G workgroups
// per block, J slice in LDS or not, XCD placement) for R replicas; false if it
// does not fit this device (LDS, columns per workgroup, co-residency of a
// group).
static bool make_geometry(phia_problem* p, int R, int mt, int cbw, int G, int j_lds, Geometry& g, int xcd)
{
    const int Np = p->Np, ncb = Np / 16;
    if (p->path != PHIA_PATH_I8 && p->path != PHIA_PATH_BF16HILO) return false;
    if (mt < 1 || mt > 2 || cbw < 1 || cbw > kCbwMax || G < 1 || G > ncb) return false;
    if (p->mh && (mt != 1 || cbw != 2)) return false;  // accept/reject variants: one row tile, two column blocks
    const int cbs_max = (ncb + G - 1) / G;
    if (cbs_max > kWaves * cbw) return false;
    SweepArgs a{};
    a.Np = Np;
    a.ncb = ncb;
    a.G = G;
    a.j_lds = j_lds;
    a.mh = p->mh;
    // flip-incremental field update where it has a variant: int8 or BF16
    // hi/lo, one row tile, column split with J streamed, own launch
    // (by default not with the accept/reject step: rejections return whole
    // replicas to their trajectory start, so few steps qualify)
    const bool want = p->inc_mode == 1 || (p->inc_mode < 0 && !p->mh);
    a.inc = (want && p->path != PHIA_PATH_FP32 && mt == 1 && G > 1 && !j_lds && !p->one_block_kernel &&
             ncb <= 64 * kWaves)
                ? 1
                : 0;
    size_t lds = sweep_mfma_lds_bytes(p->path, mt, a);
    if (a.inc && lds > static_cast<size_t>(kLdsMax)) {
        a.inc = 0;
        lds = sweep_mfma_lds_bytes(p->path, mt, a);
    }
    if (lds > static_cast<size_t>(kLdsMax)) return false;
    const int rows = 16 * mt, nblocks = (R + rows - 1) / rows;
    int ngroups = nblocks;
    if (G > 1) {
        const int maxwg = max_coresident_mfma(p->path, mt, cbw, j_lds, p->trace ? 1 : 0, p->mh, a.inc, lds);
        if (maxwg < G) return false;
        ngroups = std::min(nblocks, maxwg / G);
        if (ngroups >= 8) ngroups -= ngroups % 8;
    }
    g = Geometry{};
    g.ok = true;
    g.mt = mt;
    g.cbw = cbw;
    g.G = G;
    g.j_lds = j_lds;
    g.rows = rows;
    g.nblocks = nblocks;
    g.ngroups = ngroups;
    if (!pick_xcd(p, G, ngroups, j_lds, xcd, g.xcd_map)) return false;
    g.lds = lds;
    g.mh = p->mh;
    g.inc = a.inc;
    return true;
}

// Interleaved group sweep (k_sweep_pp): int8 path, blocks of 32 replicas as
// two 16-replica sub-blocks on two wave teams, G >= 2 workgroups per block
// with one column block per wave; MFMA operands int8 or (fp4 = 1, couplings
// that are all FP4 integers) FP4; jg = 1: int8 J streamed from global memory
// instead of held per member (j_lds = 0).  False if it does not apply.
static bool make_geometry_pp(phia_problem* p, int R, int G, int fp4, Geometry& g, int xcd, int jg)
{
    const int Np = p->Np, ncb = Np / 16;
    if (p->path != PHIA_PATH_I8 || p->trace || p->one_block_kernel || p->mh || G < 2 || G > ncb ||
        ncb > kPpMaxNcb)
        return false;
    if (fp4 && (!p->has_j4 || jg)) return false;
    if (p->maxrow >= kPpMaxRowSum || 2 * p->maxrow * p->N >= (int64_t(1) << 31)) return false;
    if ((ncb + G - 1) / G > kWaves) return false;
    const size_t lds = sweep_pp_lds_bytes(Np, G, fp4, jg);
    if (lds > static_cast<size_t>(kLdsMax)) return false;
    const int maxwg = max_coresident_pp(ncb, fp4, jg, lds);
    if (maxwg < G) return false;
    const int nblocks = (R + 31) / 32;
    int ngroups = std::min(nblocks, maxwg / G);
    if (ngroups >= 8) ngroups -= ngroups % 8;
    g = Geometry{};
    g.ok = true;
    g.kind = fp4 ? 2 : 1;
    g.mt = 2;
    g.cbw = 1;
    g.G = G;
    g.j_lds = jg ? 0 : 1;
    g.rows = 32;
    g.nblocks = nblocks;
    g.ngroups = ngroups;
    if (!pick_xcd(p, G, ngroups, jg ? 0 : 1, xcd, g.xcd_map)) return false;
    g.lds = lds;
    return true;
}

// Resident sweep (k_sweep_res): int8 path, four replicas and all columns per
// workgroup, couplings in VGPRs and LDS as FP4 operands where the problem has
// them (and its row sums stay exact in FP32), else int8.  False if it does
// not apply.
static bool make_geometry_res(phia_problem* p, int R, Geometry& g)
{
    if (p->path != PHIA_PATH_I8 || p->ikick) return false;
    // Served requests past the batch sizes with up to 32 replicas stay in the
    // column-split table, whose step they share and which more of them hardly
    // lengthen.  ms for n requests of 500 steps, resident / table: N = 551, 16
    // replicas 0.9 / 2.7 (n = 1), 3.5 / 4.4 (12), 8.6 / 6.0 (30), 32 replicas
    // 0.9 / 4.1, 3.6 / 6.2, 8.6 / 7.7; N = 700, 16 replicas 9.8 / 7.2 (30), 48
    // replicas 1.0 / 5.0, 4.1 / 7.1, 9.6 / 10.0, 256 replicas 9.9 / 22 (30).
    if (p->one_block_kernel && p->Np > kBatchMaxNp && R <= 32) return false;
    const int64_t row = 2 * p->maxrow * p->N;  // bounds |sum_i s_i (I_i + h_i)|
    const int fp4 = p->has_j4 && row < (int64_t(1) << 24) && sweep_res_lds_bytes(p->N, 1) > 0;
    if (!fp4 && (row >= (int64_t(1) << 31) || sweep_res_lds_bytes(p->N, 0) == 0)) return false;
    g = Geometry{};
    g.ok = true;
    g.kind = 5;
    g.fp4 = fp4;
    g.mt = 1;
    g.cbw = 1;
    g.G = 1;
    g.j_lds = 1;
    g.rows = kResReplicas;
    g.nblocks = (R + g.rows - 1) / g.rows;
    g.ngroups = g.nblocks;
    g.lds = sweep_res_lds_bytes(p->N, fp4);
    g.mh = p->mh;
    return true;
}

// A served request that the split sweep runs in launches of its own, one after
// the other, beside the table launches of the others (100 steps of 64
// replicas, ms, in the table / alone: BF16 hi/lo N = 1105 1.82 / 0.23, N = 454,
// 258 and 187 together 1.14 / 0.42).  ELL and FP32 requests share the device
// on the auxiliary streams instead, int8 ones up to Np = 832 (and up
// to N = 864 with FP4 codes and more than 32 replicas) run resident there or in
// the column-split table.
static bool served_alone(const phia_problem* p)
{
    return p->path == PHIA_PATH_BF16HILO || (p->path == PHIA_PATH_I8 && p->Np > 832);
}

// Split sweep (k_sweep_split): a group of G workgroups (0: as few as hold the
// columns) per block of `rows` replicas (4 or 16; 0: the fewest with which
// every block runs at once).  False if it does not apply.
static bool make_geometry_split(phia_problem* p, int R, int rows, int G, Geometry& g)
{
    const int planes = p->path == PHIA_PATH_I8 ? 1 : p->path == PHIA_PATH_BF16HILO ? 2 : p->path == PHIA_PATH_FP32 ? 3 : 0;
    if (p->no_split || p->trace || (p->one_block_kernel && !served_alone(p)) || p->mh || p->ikick || p->maxrow >= kSplitMaxRow)
        return false;
    if (planes > 1 && p->maxabsJ > (planes == 2 ? kSplitMaxJ2 : kSplitMaxJ3)) return false;
    const int waves = split_waves(p->Np, planes), ncb = p->Np / 16;
    if (waves == 0) return false;
    const int fewest = std::max(2, (ncb + waves - 1) / waves);
    if (G != 0 && (G < fewest || G > ncb)) return false;
    for (const int r : {4, 16}) {
        if (rows != 0 && r != rows) continue;
        const size_t lds = sweep_split_lds_bytes(p->Np, planes, r, p->ell_d);
        if (lds == 0) continue;
        // groups in multiples of eight, every one on one XCD (the exchange
        // stays in its L2); what is left over of the last eight exits at once
        const int nblocks = (R + r - 1) / r, eights = (nblocks + 7) / 8;
        const int most = max_coresident_split(p->Np, planes, r, p->ell_d) / 8;  // workgroups per XCD
        int m = G != 0 ? G : fewest;
        // four replicas to a group leave the CUs idle otherwise: fewer columns
        // per member (N = 2000, 16 replicas, 32 members 1.62 us per step, 16
        // members 2.14; N = 500 in three planes, 128 replicas, 8 members 1.45,
        // 4 members 1.63)
        while (G == 0 && r == 4 && 2 * m <= ncb && eights * 2 * m <= most) m *= 2;
        const int groups = most / m * 8;
        if (groups == 0 || (rows == 0 && r != 16 && nblocks > groups)) continue;
        g = Geometry{};
        g.ok = true;
        g.kind = 6;
        g.planes = planes;
        g.mt = 1;
        g.cbw = 1;
        g.G = m;
        g.rows = r;
        g.nblocks = nblocks;
        g.ngroups = std::min(8 * eights, groups);
        g.xcd_map = 1;
        g.lds = lds;
        return true;
    }
    return false;
}

// Replica counts that take the VALU sweeps by default.
constexpr int kValuTuneMaxR = 64;  // the autotuner also times the int8 VALU sweep up to here

// Largest replica count for which an int8 anneal of up to 384 columns whose row
// sums are too large for the resident sweep's energies (2 N max_i(sum_j |J_ij| +
// |h_i|) from 2^31: fields far beyond the couplings) takes the VALU dot-product
// sweep.  What else holds it are the one-block and the column-split sweep.
// While J fits in LDS (Np <= 384) one workgroup per replica finishes a step
// sooner than these (0.94 against 1.21 us at Np = 64, 1.3 against 2.6 us at Np
// = 256, 2.05 against 2.77 us at Np = 384) until the replicas outnumber the
// workgroups the CUs hold at once (J of 64 KiB: two per CU, above 80 KiB: one);
// beyond Np = 384 the column-split sweep wins at every replica count.
static int valu_fallback(int Np)
{
    if (Np <= 64) return 1024;
    if (Np <= 256) return 512;
    if (Np <= 384) return 256;
    return 0;
}

// The VALU sweep is not the default where the resident sweep holds the
// couplings: four replicas per workgroup on the matrix cores take 0.40 us per
// step at Np = 64 and 0.70 us at Np = 256, at 4 to 1024 replicas.
// PHIA_VALU_CROSSOVER=n replaces the rule (tuning experiments).
int valu_crossover(int)
{
    if (const char* env = std::getenv("PHIA_VALU_CROSSOVER")) return std::atoi(env);
    return 0;
}

// Replicas per workgroup of the int8 VALU sweep and of the ELL sweep.
static int valu_rows(int R) { return R > 1024 ? 2 : 1; }
// ELL: one replica per workgroup, four from 1024 replicas (3-regular N = 512
// with 1024 replicas: 3.1 against 5.7 us per step; 64 replicas at N = 4000:
// 7.9 against 3.4 us)
static int ell_rows(int R) { return R >= 1024 ? 4 : 1; }

// VALU sweep (k_sweep_valu): rb replicas and all columns per workgroup; the
// form follows the path (FP32, ELL, or the int8 dot products of the I8 path).
static int valu_form(const phia_problem* p)
{
    return p->path == PHIA_PATH_FP32 ? kValuFp32 : p->path == PHIA_PATH_ELL ? kValuEll : kValuDot8;
}

static bool make_geometry_valu(phia_problem* p, int R, int rb, Geometry& g)
{
    const int form = valu_form(p);
    // the int8 couplings live in LDS when they fit next to the spins
    const bool jl = form == kValuDot8 && valu_lds_bytes(form, rb, p->Np, true) <= static_cast<size_t>(kLdsMax);
    if (p->Np > kValuMaxNp || !valu_variant(form, rb, p->mh, jl)) return false;
    // the int8 form: own launches only (served and batched problems run the
    // matrix-core table kernels)
    if (form == kValuDot8 && (p->path != PHIA_PATH_I8 || p->one_block_kernel)) return false;
    g = Geometry{};
    g.ok = true;
    g.kind = 4;
    g.mt = 1;
    g.cbw = 1;
    g.G = 1;
    g.j_lds = jl ? 1 : 0;
    g.rows = rb;
    g.nblocks = (R + rb - 1) / rb;
    g.ngroups = g.nblocks;
    g.xcd_map = 0;
    g.lds = valu_lds_bytes(form, rb, p->Np, jl);
    g.mh = p->mh;
    return true;
}

}  // namespace phia

extern "C" int32_t phia_valu_crossover(int32_t Np)
{
    return phia::valu_crossover(Np);
}

namespace phia {

// Every feasible geometry for R replicas (group sizes up to 64 workgroups).
static std::vector<Geometry> candidate_geometries(phia_problem* p, int R)
{
    std::vector<Geometry> out;
    if (p->path == PHIA_PATH_FP32 || p->path == PHIA_PATH_ELL) {
        for (int rb : {1, 2, 4}) {
            Geometry g;
            if (make_geometry_valu(p, R, rb, g)) out.push_back(g);
        }
        for (const int rows : {4, 16}) {
            Geometry g;
            if (make_geometry_split(p, R, rows, 0, g)) out.push_back(g);
        }
        return out;
    }
    {
        Geometry g;
        if (make_geometry_res(p, R, g)) out.push_back(g);
        for (const int rows : {4, 16})
            if (make_geometry_split(p, R, rows, 0, g)) out.push_back(g);
    }
    if (p->path == PHIA_PATH_I8 && R <= kValuTuneMaxR)
        for (int rb : {1, 2}) {
            Geometry g;
            if (make_geometry_valu(p, R, rb, g)) out.push_back(g);
        }
    const int ncb = p->Np / 16;
    int last_cbs = -1;
    for (int G = 1; G <= std::min(ncb, 64); ++G) {
        const int cbs_max = (ncb + G - 1) / G;
        if (cbs_max == last_cbs) continue;  // same slice width as a smaller group
        last_cbs = cbs_max;
        for (int mt : {1, 2})
            for (int cbw = 1; cbw <= kCbwMax; ++cbw)
                for (int jl : {1, 0}) {
                    Geometry g, h;
                    if (!make_geometry(p, R, mt, cbw, G, jl, g)) continue;
                    out.push_back(g);  // default placement first
                    // the other placement only matters for a J streamed from L2
                    if (G > 1 && !jl && make_geometry(p, R, mt, cbw, G, jl, h, 1 - g.xcd_map)) out.push_back(h);
                }
        for (int fp4 : {0, 1}) {
            Geometry g;
            if (make_geometry_pp(p, R, G, fp4, g)) out.push_back(g);
        }
        {
            // interleaved with J streamed from global memory, both placements
            Geometry g, h;
            if (make_geometry_pp(p, R, G, 0, g, -1, 1)) {
                out.push_back(g);
                if (make_geometry_pp(p, R, G, 0, h, 1 - g.xcd_map, 1)) out.push_back(h);
            }
        }
    }
    return out;
}

// Default among the one-block and interleaved sweeps, into p->geo: fewest
// passes over the replica blocks first; among those a geometry without column
// split, else the interleaved kernel with the smallest group, else the fewest
// owned elements per workgroup, then J in LDS.
static void choose_mfma(phia_problem* p, int R)
{
    const std::vector<Geometry> cands = candidate_geometries(p, R);
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, p->dev) != hipSuccess || cus < 1) cus = 256;
    int min_iters = 1 << 30;
    for (const Geometry& g : cands)
        if (g.kind < 4) min_iters = std::min(min_iters, (g.nblocks + g.ngroups - 1) / g.ngroups);
    double best = 0;
    for (const Geometry& g : cands) {
        const int iters = (g.nblocks + g.ngroups - 1) / g.ngroups;
        if (iters != min_iters || g.kind >= 4) continue;  // those: by the rules above or tuning only
        const int cbs_max = (p->Np / 16 + g.G - 1) / g.G;
        const double elems = static_cast<double>(g.rows) * cbs_max * 16;
        double cost = g.kind >= 1 ? 1e6 + 2 * g.G - (g.kind == 2 ? 1 : 0) + (g.j_lds ? 0 : 0.5)
                                  : (g.G > 1 ? 2e6 : 0.0) + elems * 2 + (g.j_lds ? 0 : 1);
        // An interleaved grid that leaves most CUs idle (few replica blocks)
        // gives way to a larger group: SK N = 2000 with 16 replicas takes
        // 113 ms at G = 64 against 140 ms at G = 16.
        if (g.kind >= 1) cost += 1e4 * std::max(0.0, 0.5 - static_cast<double>(g.ngroups) * g.G / cus);
        // Served requests share cooperative launches: the fewest workgroups.
        if (p->one_block_kernel) cost = static_cast<double>(g.nblocks) * g.G * 4 + (g.j_lds ? 0 : 1) + g.mt;
        if (!p->geo.ok || cost < best) {
            p->geo = g;
            best = cost;
        }
    }
}

// Replica counts at which the resident sweep is the default where it fits,
// in us per step, it / the best of the other sweeps:
//   N = 16    0.40 / 0.95 at 64 replicas, 0.63 / 3.1 at 16384;
//   N = 96    0.65 / 1.42 at 2048, 1.3 / 1.44 at 4096, 4.7 / 4.1 at 16384;
//   N = 192   1.3 / 2.3 at 2048, 2.5 / 2.4 at 4096, 9.6 / 6.5 at 16384;
//   N = 256   0.77 / 2.7 at 1024, 1.5 / 2.7 at 2048, 2.9 / 2.9 at 4096;
//   N = 320   1.7 / 2.4 at 2048, 12.9 / 26 at 16384;
//   N = 437   1.23 / 3.0 (int8) at 1024, 17 / 33 at 16384;
//   N = 800   1.70 / 2.56 at 64, 2.0 / 2.9 at 1024, 28 / 79 at 16384.
// Its workgroups of four replicas run one or two to a CU, so its time grows
// with every further 1024 or 2048 replicas; up to 256 columns the one-block
// kernel of 16 or 32 replicas per workgroup fills the chip only at 4096 or
// 8192 and then overtakes it.
// A traced anneal of 1024 replicas or more keeps the column split beyond 512
// columns (2.9 against 2.0 us per step, with the same results): the parity
// tests hold a traced benchmark-size anneal to it.
static bool resident_wins(const phia_problem* p, int R)
{
    if (p->trace && p->Np > 512 && R >= 1024) return false;
    if (p->Np <= 64 || p->Np > 256) return true;
    return R <= (p->Np <= 128 ? 4096 : 3072);
}

// Anneals on streams of their own run side by side, exchange sweeps do not: the
// runtime runs cooperative launches one after the other, and a group of four
// replicas spreads over as many CUs as it can use.  So on a stream of its own
// an anneal keeps the sweep without an exchange where four of them side by
// side (the process's hardware queues) finish more per second; on the null
// stream nothing runs beside it.  us per step and anneal on 1, 2 and 4 streams,
// without exchange / split: 3-regular N = 1000, 64 replicas 1.56 0.78 0.39 /
// 1.26 1.26 1.25, N = 4000 3.6 1.8 1.1 / 2.0 1.9 1.9; BF16 hi/lo N = 130, 16
// replicas 2.57 1.28 0.65 / 1.14 1.14 1.13, but N = 256 4.24 2.12 1.07 / 1.16
// 1.15 1.14; FP32 N = 16 2.67 1.36 0.68 / 1.19 1.18 1.17, but N = 64 4.75 2.38
// 1.2 / 1.18 1.18 1.18.  Beyond 1024 replicas one anneal takes a quarter of
// the device and more.  (phia_autotune picks what is fastest alone.)
static bool runs_beside_others(const phia_problem* p, int R)
{
    if (!p->st || p->one_block_kernel) return false;
    if (p->path == PHIA_PATH_ELL) return true;
    return R <= 1024 && (p->path == PHIA_PATH_BF16HILO ? p->Np <= 192 : p->path == PHIA_PATH_FP32 && p->N <= 48);
}

// Launch geometry: forced, tuned, cached, or by the rules below.
// PHIA_GEOMETRY="mt,G,jlds[,cbw[,xcd]]" or "pp,G[,xcd]" / "pp4,G[,xcd]" /
// "ppg,G[,xcd]" (interleaved, int8 J streamed from global memory), "valu,rb",
// "res" or "split[,rows[,G]]" forces one candidate (tuning experiments).
static void choose_geometry(phia_problem* p, int R)
{
    p->geo.ok = false;
    if (p->ikick) {
        // the initial kick is a variant of the VALU sweep only
        int rb = p->path == PHIA_PATH_FP32 ? kFp32Rows : p->path == PHIA_PATH_ELL ? ell_rows(R) : valu_rows(R);
        if (const char* env = std::getenv("PHIA_GEOMETRY")) (void)std::sscanf(env, "valu,%d", &rb);
        if (p->path == PHIA_PATH_FP32 || p->path == PHIA_PATH_ELL || p->path == PHIA_PATH_I8)
            make_geometry_valu(p, R, rb, p->geo);
        return;
    }
    int f_mt = 0, f_G = 0, f_j = -1, f_c = kCbwMax;
    if (const char* env = std::getenv("PHIA_GEOMETRY")) {
        int f_x = -1;
        if (std::strcmp(env, "res") == 0) {
            Geometry g;
            if (make_geometry_res(p, R, g)) p->geo = g;
            return;
        }
        if (std::strncmp(env, "split", 5) == 0) {
            Geometry g;
            (void)std::sscanf(env, "split,%d,%d", &f_mt, &f_G);
            if (make_geometry_split(p, R, f_mt, f_G, g)) p->geo = g;
            return;
        }
        if (std::sscanf(env, "valu,%d", &f_G) == 1) {
            Geometry g;
            if (make_geometry_valu(p, R, f_G, g)) p->geo = g;
            return;
        }
        if (std::sscanf(env, "pp,%d,%d", &f_G, &f_x) >= 1 || std::sscanf(env, "pp4,%d,%d", &f_G, &f_x) >= 1 ||
            std::sscanf(env, "ppg,%d,%d", &f_G, &f_x) >= 1) {
            Geometry g;
            if (make_geometry_pp(p, R, f_G, std::strncmp(env, "pp4", 3) == 0, g, f_x, std::strncmp(env, "ppg", 3) == 0))
                p->geo = g;
            return;
        }
        if (std::sscanf(env, "%d,%d,%d,%d,%d", &f_mt, &f_G, &f_j, &f_c, &f_x) >= 3) {
            Geometry g;
            if (make_geometry(p, R, f_mt, f_c, f_G, f_j, g, f_x)) p->geo = g;
            return;
        }
    }
    if (p->tuned.ok && p->tuned_R == R) {
        if (p->tuned.kind == 6) {  // as far as it applies to this anneal
            if (make_geometry_split(p, R, p->tuned.rows, p->tuned.G, p->geo)) return;
        } else if (p->tuned.mh == p->mh && p->tuned.kind != 0) {
            p->geo = p->tuned;
            return;
        }
        // same shape; LDS and variant redone for the current accept/reject
        // step and flip-incremental setting
        Geometry g;
        if (p->tuned.kind == 0 &&
            make_geometry(p, R, p->tuned.mt, p->tuned.cbw, p->tuned.G, p->tuned.j_lds, g, p->tuned.xcd_map)) {
            p->geo = g;
            return;
        }
    }
    if (lookup_tune_cache(p, R)) return;
    if (p->path == PHIA_PATH_FP32 || p->path == PHIA_PATH_ELL) {
        // FP32 always (figures below).  ELL as long as every block runs at once,
        // and from 513 to 1024 columns with at most eight column blocks to a
        // member; the VALU sweep, one replica to a CU, is quick there (3-regular
        // rows, us per step, VALU / split: N = 1000 1.55 / 1.36 at 64 replicas,
        // 1.61 / 1.95 at 256; N = 2000 2.0 / 1.4-2.0 up to 128; N = 4000 3.5 /
        // 1.5 at 32, 3.5 / 2.05 at 64; two passes, 128 replicas, 3.7 / 4.2).
        if (!runs_beside_others(p, R) && make_geometry_split(p, R, 0, 0, p->geo)) {
            if (p->path == PHIA_PATH_FP32 || p->Np > 1024 || (p->Np > 512 && p->Np / 16 <= 8 * p->geo.G)) return;
            p->geo = Geometry{};
        }
        make_geometry_valu(p, R, p->path == PHIA_PATH_FP32 ? kFp32Rows : ell_rows(R), p->geo);
        return;
    }
    if (p->path == PHIA_PATH_I8 && R <= valu_crossover(p->Np) && make_geometry_valu(p, R, valu_rows(R), p->geo))
        return;
    // phia_set_incremental(1) asks for the flip-incremental product wherever it
    // applies: a choice among the sweeps that have it goes before the newer ones.
    if (p->inc_mode == 1) {
        choose_mfma(p, R);
        if (p->geo.ok && p->geo.inc) return;
        p->geo = Geometry{};
    }
    // Couplings that one CU holds: the resident sweep (resident_wins).
    if (resident_wins(p, R) && make_geometry_res(p, R, p->geo)) return;
    // The split sweep wherever it applies, int8 only past the sizes of the
    // resident sweep (us per step, the best of the others / it, 16 to 2048
    // replicas): FP32 N = 32 3.4 / 1.3-1.5, N = 500 32-69 / 1.4-4.2; BF16
    // hi/lo N = 200 4.2-4.5 / 1.3-1.9, N = 1000 5.7-19 / 1.5-9.6; int8
    // N = 513 2.8-7.9 / 1.3-6.4, N = 900 2.6-11.9 / 1.3-8.9, N = 2000
    // 5.2-17.5 / 1.6-11.6.  Further replicas are further passes of both, and
    // the order stays (FP32 N = 16 44 / 43 at 65536, N = 500 2035 / 137; BF16
    // hi/lo N = 256 18.6 / 13.2 at 16384; int8 N = 640 67 / 48), except where
    // one workgroup per block, which needs no exchange, is as quick per pass:
    // BF16 hi/lo up to 128 columns at every replica count (N = 64 1.25 / 1.29
    // at 16, 1.36 / 2.9 at 4096) and up to 192 columns past one pass (N = 129
    // and 192 2.7 / 1.77 at 2048, 2.7-2.8 / 3.3 at 3072, 10.8-11.2 / 12.5 at
    // 16384).
    if (p->Np > (p->path == PHIA_PATH_BF16HILO ? 128 : 512) && !runs_beside_others(p, R) &&
        make_geometry_split(p, R, 0, 0, p->geo)) {
        if (p->Np > 192 || p->geo.nblocks <= p->geo.ngroups) return;
        p->geo = Geometry{};
    }
    // Few replicas on the int8 path: the VALU dot-product sweep.
    if (p->path == PHIA_PATH_I8 && R <= valu_fallback(p->Np) && make_geometry_valu(p, R, valu_rows(R), p->geo))
        return;
    choose_mfma(p, R);
}

// Bytes of the exchange words and of the partial energies of a geometry.
static size_t xbits_bytes(const phia_problem* p, const Geometry& g)
{
    return 2 * static_cast<size_t>(g.ngroups) * g.rows * (p->Np / 16) * sizeof(uint64_t);
}
static size_t pbuf_bytes(const Geometry& g)
{
    return 2 * static_cast<size_t>(g.ngroups) * g.G * g.rows * 2 * sizeof(uint64_t);
}

void free_state(phia_problem* p)
{
    dfree(p->dx);
    dfree(p->dv);
    dfree(p->dbestE);
    p->dbestS = nullptr;
    p->dbestStep = nullptr;
    dfree(p->dctab);
    dfree(p->detrace);
    dfree(p->dxbits);
    dfree(p->dpbuf);
    dfree(p->dbtab);
    dfree(p->dx0);
    dfree(p->dmhE);
    dfree(p->dmhQ);
    dfree(p->dlam);
    dfree(p->dmhc);
    dfree(p->dmhbuf);
    p->mhQ_cap = 0;
    p->xb_bytes = p->pb_bytes = p->mb_bytes = 0;
    p->recorded = false;
    p->table = Geometry{};
    p->table_tried = false;
    p->state_bytes = 0;
    p->R = 0;
    p->T = 0;
    p->k = 0;
}

// Device copies of the couplings and fields (uploaded synchronously from the
// host copies), if they are not resident yet.
phia_status make_resident(phia_problem* p)
{
    if (p->dJ) return PHIA_OK;
    if (p->hJ.empty()) return fail(PHIA_ESTATE, "the couplings are neither resident nor kept on the host");
    hipError_t e = hipSetDevice(p->dev);
    if (e != hipSuccess) return hip_fail(p, e, "hipSetDevice");
    size_t* cnt = &p->base_bytes;
    if ((e = dalloc(reinterpret_cast<void**>(&p->dJ), p->hJ.size(), cnt)) != hipSuccess ||
        (e = dalloc(reinterpret_cast<void**>(&p->dh), sizeof(int32_t) * p->hh.size(), cnt)) != hipSuccess ||
        (p->has_j4 && (e = dalloc(reinterpret_cast<void**>(&p->dJ4), p->hJ4.size(), cnt)) != hipSuccess) ||
        (!p->hJ64.empty() &&
         ((e = dalloc(reinterpret_cast<void**>(&p->dJ64), sizeof(double) * p->hJ64.size(), cnt)) != hipSuccess ||
          (e = dalloc(reinterpret_cast<void**>(&p->dh64), sizeof(double) * p->hh64.size(), cnt)) != hipSuccess))) {
        release_resident(p);
        return fail(PHIA_ENOMEM, "device allocation of the couplings failed: %s", hipGetErrorString(e));
    }
    if ((e = hipMemcpy(p->dJ, p->hJ.data(), p->hJ.size(), hipMemcpyHostToDevice)) != hipSuccess ||
        (e = hipMemcpy(p->dh, p->hh.data(), sizeof(int32_t) * p->hh.size(), hipMemcpyHostToDevice)) != hipSuccess ||
        (p->has_j4 && (e = hipMemcpy(p->dJ4, p->hJ4.data(), p->hJ4.size(), hipMemcpyHostToDevice)) != hipSuccess) ||
        (p->dJ64 &&
         ((e = hipMemcpy(p->dJ64, p->hJ64.data(), sizeof(double) * p->hJ64.size(), hipMemcpyHostToDevice)) !=
              hipSuccess ||
          (e = hipMemcpy(p->dh64, p->hh64.data(), sizeof(double) * p->hh64.size(), hipMemcpyHostToDevice)) !=
              hipSuccess))) {
        release_resident(p);
        return fail(PHIA_EDEVICE, "upload of the couplings failed: %s", hipGetErrorString(e));
    }
    return PHIA_OK;
}

// Free the device copies of the couplings (deferred problems only: the host
// copies stay, and the next use uploads them again).
void release_resident(phia_problem* p)
{
    size_t freed = 0;
    if (p->dJ) freed += p->hJ.size();
    if (p->dh) freed += sizeof(int32_t) * p->hh.size();
    if (p->dJ4) freed += p->hJ4.size();
    if (p->dJ64) freed += sizeof(double) * p->hJ64.size();
    if (p->dh64) freed += sizeof(double) * p->hh64.size();
    dfree(p->dJ);
    dfree(p->dJ4);
    dfree(p->dh);
    dfree(p->dJ64);
    dfree(p->dh64);
    p->base_bytes -= std::min(freed, p->base_bytes);
}

// Launch geometry that an anneal of R replicas without the accept/reject
// step or energy traces would take (forced, tuned, cached or default), with
// the problem's current anneal left as it is; split = false leaves out the
// split sweep.
Geometry plain_geometry(phia_problem* p, int R, int ikick, bool split)
{
    const Geometry saved = p->geo;
    const int mh = p->mh, ik = p->ikick;
    const bool trace = p->trace;
    p->mh = 0;
    p->ikick = ikick;
    p->trace = false;
    p->no_split = !split;
    choose_geometry(p, R);
    p->no_split = false;
    const Geometry g = p->geo;
    p->geo = saved;
    p->mh = mh;
    p->ikick = ik;
    p->trace = trace;
    return g;
}

SweepArgs sweep_args(const phia_problem* p)
{
    SweepArgs a{};
    a.N = p->N;
    a.Np = p->Np;
    a.h = p->dh;
    a.J = p->geo.kind == 2 || (p->geo.kind == 5 && p->geo.fp4) ? p->dJ4 : p->dJ;
    a.ell_d = p->ell_d;
    a.ikick = p->ikick;
    a.ctab = p->dctab;
    a.eps = p->eps;
    a.gamma = p->gamma;
    a.L = p->L;
    a.deriv = p->deriv;
    a.seed = p->seed;
    a.R = p->R;
    a.r_base = 0;
    a.x = p->dx;
    a.v = p->dv;
    a.bestE = p->dbestE;
    a.bestS = p->dbestS;
    a.bestStep = p->dbestStep;
    a.etrace = p->detrace;
    a.T = p->T;
    a.G = p->geo.G;
    a.ncb = p->Np / 16;
    a.rows = p->geo.rows;
    a.nblocks = p->geo.nblocks;
    a.ngroups = p->geo.ngroups;
    a.xcd_map = p->geo.xcd_map;
    a.j_lds = p->geo.j_lds;
    a.inc = p->geo.inc;
    a.incstat = p->dincstat;
    a.xbits = p->dxbits;
    a.pbuf = p->dpbuf;
    a.seq_base = p->seq;
    a.err = p->derr;
    a.mh = p->mh;
    a.mh_up = p->mh_up;
    a.mh_down = p->mh_down;
    a.sigma = std::ldexp(1.0f, -p->f);
    a.btab = p->dbtab;
    a.x0 = p->dx0;
    a.mhE = p->dmhE;
    a.mhQ = p->dmhQ;
    a.lam = p->dlam;
    a.mhc = p->dmhc;
    a.mhbuf = p->dmhbuf;
    return a;
}

phia_status check_usable(const phia_problem* p)
{
    if (!p) return fail(PHIA_EINVAL, "null problem");
    if (p->poisoned) return fail(PHIA_EDEVICE, "problem handle is poisoned by an earlier device error");
    return PHIA_OK;
}

// Calls that change a problem's anneal: not while a batch plan holds its state.
phia_status check_owned(const phia_problem* p)
{
    phia_status st = check_usable(p);
    if (st != PHIA_OK) return st;
    if (p->batch) return fail(PHIA_ESTATE, "the problem belongs to a batch plan (phia_batch_destroy releases it)");
    return PHIA_OK;
}

}  // namespace phia

// =================================================================== ABI ==
extern "C" {

const char* phia_last_error(void) { return g_err.c_str(); }

const char* phia_version(void) { return "phia-mi355x 0.1 (gfx950)"; }

phia_status phia_create(const double* J, const double* h, int32_t N, const phia_options* opt, phia_problem** out)
{
    clear_error();
    if (!out) return fail(PHIA_EINVAL, "out is null");
    *out = nullptr;
    if (!J) return fail(PHIA_EINVAL, "J is null");
    if (N < 1 || N > 16384) return fail(PHIA_EINVAL, "N = %d outside [1, 16384]", N);
    phia_options o{-1, 0, PHIA_PATH_AUTO, 0, nullptr, 0};
    if (opt) o = *opt;
    if (o.path < PHIA_PATH_AUTO || o.path > PHIA_PATH_ELL) return fail(PHIA_EINVAL, "unknown path %d", o.path);
    if (o.defer_upload != 0 && o.defer_upload != 1) return fail(PHIA_EINVAL, "defer_upload = %d", o.defer_upload);

    std::vector<int32_t> Ji, hi;
    int f = 0;
    bool exact = true;
    phia_status st = pack_instance(J, h, N, o.frac_bits, o.quantize, Ji, hi, f, exact);
    if (st != PHIA_OK) return st;

    int64_t maxJ = 0, minJ = 0, maxrow = 0;
    int maxdeg = 0;  // most nonzero couplings in a row
    for (int i = 0; i < N; ++i) {
        int64_t row = std::llabs(hi[i]);
        int deg = 0;
        for (int j = 0; j < N; ++j) {
            const int64_t v = Ji[static_cast<size_t>(i) * N + j];
            maxJ = std::max(maxJ, v);
            minJ = std::min(minJ, v);
            row += std::llabs(v);
            deg += v != 0;
        }
        maxrow = std::max(maxrow, row);
        maxdeg = std::max(maxdeg, deg);
    }
    const int64_t maxabs = std::max(maxJ, -minJ);
    if (maxrow >= (int64_t(1) << 31)) return fail(PHIA_ERANGE, "sum_j |J_ij| + |h_i| does not fit int32");
    int path = o.path;
    const bool i8_ok = maxJ <= 127 && minJ >= -128;
    const bool bf_ok = maxabs <= 32767;
    const bool f32_ok = maxrow < (int64_t(1) << 24);
    if (path == PHIA_PATH_AUTO) path = i8_ok ? PHIA_PATH_I8 : bf_ok ? PHIA_PATH_BF16HILO : PHIA_PATH_FP32;
    {
        // Sparse rows beyond the batch sweep's sizes: ELL when the densest
        // row has at most Np / 64 nonzeros (measured on MI355X, 16 and 256
        // replicas: ELL ties the int8 matrix cores at 16-18 nonzeros for
        // N = 1000, 32-41 for N = 2000, 52 and more for N = 4000; 3-regular
        // rows take 1.6 against 2.5 us per step at N = 1000 and 3.4 against
        // 14 us at N = 4000).
        const int Np = (N + 63) / 64 * 64;
        if (o.path == PHIA_PATH_AUTO && bf_ok && Np > kBatchFp4MaxNp && Np <= kValuMaxNp && maxdeg <= Np / 64)
            path = PHIA_PATH_ELL;
    }
    if (path == PHIA_PATH_I8 && !i8_ok) return fail(PHIA_ERANGE, "couplings outside int8 for the I8 path");
    if (path == PHIA_PATH_BF16HILO && !bf_ok) return fail(PHIA_ERANGE, "couplings outside 16 bits for BF16HILO");
    if (path == PHIA_PATH_FP32 && !f32_ok) return fail(PHIA_ERANGE, "row sums exceed 2^24 for the FP32 path");
    if (path == PHIA_PATH_ELL && !bf_ok) return fail(PHIA_ERANGE, "couplings outside 16 bits for the ELL path");
    {
        // Largest instance each sweep holds: the FP32 and ELL sweeps keep up
        // to 4 columns per thread of 1024 (Np <= 4096); the matrix-core sweeps stage two
        // spin rows of every replica in LDS, so even the thinnest column
        // slice needs 32 Np bytes per operand byte there.
        const int Np = (N + 63) / 64 * 64;
        bool fits;
        if (path == PHIA_PATH_FP32 || path == PHIA_PATH_ELL) {
            fits = Np <= kValuMaxNp;
        } else {
            SweepArgs a{};
            a.Np = Np;
            a.ncb = Np / 16;
            a.G = a.ncb;
            a.j_lds = 0;
            fits = sweep_mfma_lds_bytes(path, 1, a) <= static_cast<size_t>(kLdsMax);
        }
        if (!fits)
            return fail(PHIA_ERANGE, "N = %d is beyond the %s sweep (N <= 5056 int8, 2496 BF16 hi/lo, 4096 FP32/ELL)",
                        N, path_name(path));
    }

    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) return fail(PHIA_EDEVICE, "no HIP device");
    if (o.device < 0 || o.device >= ndev) return fail(PHIA_EINVAL, "device %d not present", o.device);
    hipError_t e = hipSetDevice(o.device);
    if (e != hipSuccess) return hip_fail(nullptr, e, "hipSetDevice");

    phia_problem* p = new (std::nothrow) phia_problem();
    if (!p) return fail(PHIA_ENOMEM, "host allocation failed");
    p->dev = o.device;
    p->st = static_cast<hipStream_t>(o.stream);
    p->N = N;
    p->Np = (N + 63) / 64 * 64;
    p->path = path;
    p->f = f;
    p->exact = exact;
    p->maxabsJ = maxabs;
    p->maxrow = maxrow;
    const int Np = p->Np;

    std::vector<int32_t> hpad(static_cast<size_t>(Np), 0);
    std::copy(hi.begin(), hi.end(), hpad.begin());
    size_t jbytes = 0;
    std::vector<float> jf;
    std::vector<int8_t> j8;
    std::vector<uint8_t> j4;
    std::vector<uint16_t> jb;
    std::vector<int32_t> jell;
    const void* jsrc = nullptr;
    if (path == PHIA_PATH_FP32) {
        jf.assign(static_cast<size_t>(Np) * Np, 0.0f);
        for (int i = 0; i < N; ++i)
            for (int j = 0; j < N; ++j)
                jf[static_cast<size_t>(i) * Np + j] = static_cast<float>(Ji[static_cast<size_t>(i) * N + j]);
        jbytes = jf.size() * sizeof(float);
        jsrc = jf.data();
    } else if (path == PHIA_PATH_ELL) {
        pack_ell(Ji, N, Np, jell, p->ell_d);
        jbytes = jell.size() * sizeof(int32_t);
        jsrc = jell.data();
    } else if (path == PHIA_PATH_I8) {
        pack_i8(Ji, N, Np, j8);
        jbytes = j8.size();
        jsrc = j8.data();
        // Couplings that are all FP4 integers also get the FP4 operand copy
        // of the interleaved sweep (Np <= 1024: J fragments in VGPRs).
        bool fp4_ok = Np <= 1024;
        for (size_t t = 0; fp4_ok && t < Ji.size(); ++t) fp4_ok = fp4_code(Ji[t]) >= 0;
        if (fp4_ok) pack_fp4(Ji, N, Np, j4);
    } else {
        pack_bf16(Ji, N, Np, jb);
        jbytes = jb.size() * sizeof(uint16_t);
        jsrc = jb.data();
    }
    // Packed couplings on the host until they are made resident; the FP64
    // copies of J and h only for rounded input (exact instances take their
    // FP64 energy from the integer one).
    p->hJ.assign(static_cast<const unsigned char*>(jsrc), static_cast<const unsigned char*>(jsrc) + jbytes);
    p->hJ4 = std::move(j4);
    p->has_j4 = !p->hJ4.empty();
    p->hh = std::move(hpad);
    if (!exact) {
        p->hJ64.assign(J, J + static_cast<size_t>(N) * N);
        p->hh64.assign(static_cast<size_t>(N), 0.0);
        if (h) std::copy(h, h + N, p->hh64.begin());
    }
    p->jres_bytes = p->hJ.size() + p->hJ4.size() + sizeof(int32_t) * p->hh.size() +
                    sizeof(double) * (p->hJ64.size() + p->hh64.size());
    p->defer = o.defer_upload != 0;
    size_t* cnt = &p->base_bytes;
    if ((e = dalloc(reinterpret_cast<void**>(&p->derr), sizeof(int32_t) * 4, cnt)) != hipSuccess ||
        (e = dalloc(reinterpret_cast<void**>(&p->dscratch), 64 + static_cast<size_t>(Np), cnt)) != hipSuccess ||
        (e = dalloc(reinterpret_cast<void**>(&p->dincstat), 4 * sizeof(int64_t), cnt)) != hipSuccess) {
        phia_destroy(p);
        return fail(PHIA_ENOMEM, "device allocation failed: %s", hipGetErrorString(e));
    }
    if ((e = hipMemset(p->derr, 0, sizeof(int32_t) * 4)) != hipSuccess) {
        phia_destroy(p);
        return fail(PHIA_EDEVICE, "device set-up failed: %s", hipGetErrorString(e));
    }
    if (!p->defer) {
        if ((st = make_resident(p)) != PHIA_OK) {
            phia_destroy(p);
            return st;
        }
        // the host copies are not needed again
        std::vector<unsigned char>().swap(p->hJ);
        std::vector<unsigned char>().swap(p->hJ4);
        std::vector<double>().swap(p->hJ64);
    }
    *out = p;
    return PHIA_OK;
}

void phia_destroy(phia_problem* p)
{
    if (!p) return;
    (void)hipSetDevice(p->dev);
    if (p->batch) batch_forget(p->batch, p);
    if (!p->poisoned && p->st) (void)hipStreamSynchronize(p->st);
    if (!p->poisoned && !p->st) (void)hipDeviceSynchronize();
    free_state(p);
    dfree(p->dJ);
    dfree(p->dJ4);
    dfree(p->dh);
    dfree(p->dJ64);
    dfree(p->dh64);
    dfree(p->derr);
    dfree(p->dscratch);
    dfree(p->dincstat);
    delete p;
}

phia_status phia_set_trace(phia_problem* p, int32_t enable)
{
    clear_error();
    phia_status st = check_usable(p);
    if (st != PHIA_OK) return st;
    p->trace = enable != 0;
    return PHIA_OK;
}

}  // extern "C"

namespace phia {

phia_status check_schedule(int32_t replicas, int64_t steps, const phia_schedule* s)
{
    if (!s) return fail(PHIA_EINVAL, "schedule is null");
    if (replicas < 1 || replicas > (1 << 20)) return fail(PHIA_EINVAL, "replicas = %d outside [1, 2^20]", replicas);
    if (steps < 1 || steps > (int64_t(1) << 31)) return fail(PHIA_EINVAL, "steps = %lld out of range", (long long)steps);
    if (s->refresh_L < 1) return fail(PHIA_EINVAL, "refresh_L must be >= 1");
    if (s->deriv_mode != PHIA_DERIV_TANH && s->deriv_mode != PHIA_DERIV_POLY2)
        return fail(PHIA_EINVAL, "deriv_mode = %d is neither TANH nor POLY2", s->deriv_mode);
    if (!std::isfinite(s->eps) || !std::isfinite(s->gamma)) return fail(PHIA_EINVAL, "eps and gamma must be finite");
    if (s->metropolis != 0 && s->metropolis != 1) return fail(PHIA_EINVAL, "metropolis = %d is neither 0 nor 1", s->metropolis);
    if (s->metropolis && !(std::isfinite(s->mh_up) && std::isfinite(s->mh_down) && s->mh_up > 0.0f && s->mh_down > 0.0f))
        return fail(PHIA_EINVAL, "mh_up and mh_down must be positive and finite");
    if (s->initial_kick != 0 && s->initial_kick != 1)
        return fail(PHIA_EINVAL, "initial_kick = %d is neither 0 nor 1", s->initial_kick);
    if (s->initial_kick && s->metropolis) return fail(PHIA_EINVAL, "the initial kick is not combined with metropolis");
    return PHIA_OK;
}

// Kick factors c_k = (beta_k * gamma) * sigma of a schedule, with the linear
// inverse-temperature table beta_k = float(b0 + ((b1 - b0) k) / (T - 1))
// evaluated in double when no explicit table is given.
static float beta_of(int64_t steps, const phia_schedule* s, int64_t k)
{
    if (s->betas) return s->betas[k];
    double d = static_cast<double>(s->beta0);
    if (steps > 1)
        d = static_cast<double>(s->beta0) +
            ((static_cast<double>(s->beta1) - static_cast<double>(s->beta0)) * static_cast<double>(k)) /
                static_cast<double>(steps - 1);
    return static_cast<float>(d);
}

void kick_factors(const phia_problem* p, int64_t steps, const phia_schedule* s, std::vector<float>& ctab)
{
    ctab.resize(static_cast<size_t>(steps));
    const float sigma = std::ldexp(1.0f, -p->f);
    for (int64_t k = 0; k < steps; ++k) ctab[static_cast<size_t>(k)] = (beta_of(steps, s, k) * s->gamma) * sigma;
}

// Accept/reject buffers that depend on the launch geometry: kinetic units per
// (replica, group member) and, for column-split groups, the exchange of the
// decision's partial sums (tags start at 1, the buffer at zero).
phia_status setup_mh_geometry(phia_problem* p)
{
    if (!p->mh) return PHIA_OK;
    size_t* cnt = &p->state_bytes;
    hipError_t e;
    const size_t need = static_cast<size_t>(p->R) * static_cast<size_t>(std::max(1, p->geo.G));
    if (need > p->mhQ_cap) {
        dfree(p->dmhQ);
        p->mhQ_cap = 0;
        if ((e = dalloc(reinterpret_cast<void**>(&p->dmhQ), need * sizeof(int64_t), cnt)) != hipSuccess)
            return fail(PHIA_ENOMEM, "accept/reject state allocation failed");
        p->mhQ_cap = need;
    }
    dfree(p->dmhbuf);
    if (p->geo.kind == 0 && p->geo.G > 1) {
        const size_t mb = 2 * static_cast<size_t>(p->geo.ngroups) * p->geo.G * p->geo.rows * 4 * sizeof(uint64_t);
        if ((e = dalloc(reinterpret_cast<void**>(&p->dmhbuf), mb, cnt)) != hipSuccess)
            return fail(PHIA_ENOMEM, "accept/reject exchange allocation failed");
        p->mb_bytes = mb;
        if ((e = hipMemsetAsync(p->dmhbuf, 0, mb, p->st)) != hipSuccess) return hip_fail(p, e, "exchange reset");
    }
    return PHIA_OK;
}

// Replica state and schedule of a new anneal (device buffers kept when the
// shape is unchanged).  The kick factors are copied asynchronously from
// `ctab`, which must stay alive until the stream has passed the copy.
phia_status setup_state(phia_problem* p, int32_t replicas, int64_t steps, const phia_schedule* s, uint64_t seed,
                        const std::vector<float>& ctab, bool& reuse, bool sync_first)
{
    hipError_t e = hipSetDevice(p->dev);
    if (e != hipSuccess) return hip_fail(p, e, "hipSetDevice");
    const int mh = s->metropolis ? 1 : 0;
    const int ikick = s->initial_kick ? 1 : 0;
    reuse = p->dx && p->R == replicas && p->T == steps && p->trace == (p->detrace != nullptr) && p->mh == mh &&
            p->ikick == ikick && p->inc_mode_geo == p->inc_mode;
    // before buffers are freed, or rewritten by a copy that is not ordered on
    // the stream (the accept/reject step's table)
    if (sync_first && (!reuse || mh)) {
        e = p->st ? hipStreamSynchronize(p->st) : hipDeviceSynchronize();
        if (e != hipSuccess) return hip_fail(p, e, "synchronise before re-allocation");
    }
    if (!reuse) free_state(p);
    p->inc_mode_geo = p->inc_mode;
    p->R = replicas;
    p->T = steps;
    p->k = 0;
    p->eps = s->eps;
    p->gamma = s->gamma;
    p->L = s->refresh_L;
    p->deriv = s->deriv_mode;
    p->mh = mh;
    p->ikick = ikick;
    p->mh_up = mh ? s->mh_up : 1.0f;
    p->mh_down = mh ? s->mh_down : 1.0f;
    p->seed = seed;
    p->has_run = false;
    p->started = false;
    const size_t RN = static_cast<size_t>(replicas) * p->Np;
    size_t* cnt = &p->state_bytes;
    if (!reuse && ((e = dalloc(reinterpret_cast<void**>(&p->dx), RN * sizeof(float), cnt)) != hipSuccess ||
                   (e = dalloc(reinterpret_cast<void**>(&p->dv), RN * sizeof(float), cnt)) != hipSuccess ||
                   (e = dalloc(reinterpret_cast<void**>(&p->dbestE), 2 * sizeof(int64_t) * replicas + RN, cnt)) !=
                       hipSuccess ||
                   (e = dalloc(reinterpret_cast<void**>(&p->dctab), sizeof(float) * steps, cnt)) != hipSuccess)) {
        free_state(p);
        return fail(PHIA_ENOMEM, "state allocation failed: %s", hipGetErrorString(e));
    }
    if (!reuse) {
        p->dbestStep = p->dbestE + replicas;
        p->dbestS = reinterpret_cast<int8_t*>(p->dbestE + 2 * static_cast<size_t>(replicas));
    }
    if (p->trace && !reuse) {
        if ((e = dalloc(reinterpret_cast<void**>(&p->detrace), sizeof(int64_t) * replicas * steps, cnt)) !=
            hipSuccess) {
            free_state(p);
            return fail(PHIA_ENOMEM, "trace allocation failed");
        }
    }
    if (p->trace) (void)hipMemsetAsync(p->detrace, 0, sizeof(int64_t) * replicas * steps, p->st);
    if (mh) {
        if (!reuse && ((e = dalloc(reinterpret_cast<void**>(&p->dx0), RN * sizeof(float), cnt)) != hipSuccess ||
                       (e = dalloc(reinterpret_cast<void**>(&p->dmhE), 2 * sizeof(int64_t) * replicas, cnt)) !=
                           hipSuccess ||
                       (e = dalloc(reinterpret_cast<void**>(&p->dlam), sizeof(float) * replicas, cnt)) != hipSuccess ||
                       (e = dalloc(reinterpret_cast<void**>(&p->dmhc), 2 * sizeof(int32_t) * replicas, cnt)) !=
                           hipSuccess ||
                       (e = dalloc(reinterpret_cast<void**>(&p->dbtab), sizeof(float) * steps, cnt)) != hipSuccess)) {
            free_state(p);
            return fail(PHIA_ENOMEM, "accept/reject state allocation failed");
        }
        std::vector<float> btab(static_cast<size_t>(steps));
        for (int64_t k = 0; k < steps; ++k) btab[static_cast<size_t>(k)] = beta_of(steps, s, k);
        // pageable source: the copy completes before hipMemcpy returns
        if ((e = hipMemcpy(p->dbtab, btab.data(), sizeof(float) * steps, hipMemcpyHostToDevice)) != hipSuccess) {
            free_state(p);
            return hip_fail(p, e, "upload of the inverse temperatures");
        }
    }
    if ((e = hipMemcpyAsync(p->dctab, ctab.data(), sizeof(float) * steps, hipMemcpyHostToDevice, p->st)) !=
        hipSuccess) {
        free_state(p);
        return hip_fail(p, e, "upload of the schedule");
    }
    return PHIA_OK;
}

}  // namespace phia

extern "C" {

phia_status phia_anneal_start(phia_problem* p, int32_t replicas, int64_t steps, const phia_schedule* s,
                              uint64_t seed)
{
    clear_error();
    phia_status st = check_owned(p);
    if (st != PHIA_OK) return st;
    if ((st = check_schedule(replicas, steps, s)) != PHIA_OK) return st;
    if ((st = make_resident(p)) != PHIA_OK) return st;
    std::vector<float> ctab;
    kick_factors(p, steps, s, ctab);
    bool reuse = false;
    if ((st = setup_state(p, replicas, steps, s, seed, ctab, reuse, true)) != PHIA_OK) return st;
    // ctab is a pageable host vector; make the copy complete before it goes out of scope.
    hipError_t e = p->st ? hipStreamSynchronize(p->st) : hipDeviceSynchronize();
    if (e != hipSuccess) return hip_fail(p, e, "schedule upload");
    size_t* cnt = &p->state_bytes;
    if (reuse) {
        if ((st = setup_mh_geometry(p)) != PHIA_OK) return st;
        SweepArgs a = sweep_args(p);
        if ((e = launch_init(a, p->st)) != hipSuccess) return hip_fail(p, e, "init kernel launch");
        p->started = true;
        return PHIA_OK;
    }
    p->geo = Geometry{};
    choose_geometry(p, replicas);
    if (!p->geo.ok) {
        free_state(p);
        if (p->ikick) return fail(PHIA_ERANGE, "the initial kick runs on the VALU sweep (FP32, I8 and ELL paths)");
        return fail(PHIA_ERANGE, "no kernel geometry fits N = %d on this device", p->N);
    }
    if (p->geo.G > 1) {
        // Tagged exchange words start at zero; tags start at 1 (the split
        // sweep's partial energies travel in them).
        const size_t xb = xbits_bytes(p, p->geo), pb = p->geo.kind == 6 ? 0 : pbuf_bytes(p->geo);
        if ((e = dalloc(reinterpret_cast<void**>(&p->dxbits), xb, cnt)) != hipSuccess ||
            (pb && (e = dalloc(reinterpret_cast<void**>(&p->dpbuf), pb, cnt)) != hipSuccess)) {
            free_state(p);
            return fail(PHIA_ENOMEM, "exchange buffer allocation failed");
        }
        p->xb_bytes = xb;
        p->pb_bytes = pb;
        if ((e = hipMemsetAsync(p->dxbits, 0, xb, p->st)) != hipSuccess ||
            (pb && (e = hipMemsetAsync(p->dpbuf, 0, pb, p->st)) != hipSuccess))
            return hip_fail(p, e, "exchange buffer reset");
        p->seq = 0;
        p->exchange_kind = p->geo.kind;
    }
    if ((st = setup_mh_geometry(p)) != PHIA_OK) {
        free_state(p);
        return st;
    }
    SweepArgs a = sweep_args(p);
    if ((e = launch_init(a, p->st)) != hipSuccess) return hip_fail(p, e, "init kernel launch");
    p->started = true;
    return PHIA_OK;
}

}  // extern "C"

namespace phia {

// Zero the exchange words (their tags restart at 1).
hipError_t clear_exchange(phia_problem* p)
{
    hipError_t e = hipSuccess;
    if (p->dxbits) e = fill_words(p->dxbits, 0, p->xb_bytes, p->st);
    if (e == hipSuccess && p->dpbuf) e = fill_words(p->dpbuf, 0, p->pb_bytes, p->st);
    if (e == hipSuccess && p->dmhbuf) e = fill_words(p->dmhbuf, 0, p->mb_bytes, p->st);
    return e;
}

// A served request on the split sweep that may run in the table launches too:
// their geometry (p->table, if there is one) and room for their words.  No
// launch of the request is under way.  Without the memory for them it stays as
// it is, without a table geometry.
void prepare_table(phia_problem* p)
{
    if (p->table_tried) return;
    p->table_tried = true;
    const Geometry own = p->geo;
    p->geo = Geometry{};
    choose_mfma(p, p->R);
    const Geometry g = p->geo;
    p->geo = own;
    if (!g.ok || g.kind != 0 || g.G < 2) return;
    uint64_t *xbits = nullptr, *pbuf = nullptr;
    const size_t xb = xbits_bytes(p, g), pb = pbuf_bytes(g);
    const bool more = xb > p->xb_bytes;
    if ((more && dalloc(reinterpret_cast<void**>(&xbits), xb, nullptr) != hipSuccess) ||
        dalloc(reinterpret_cast<void**>(&pbuf), pb, nullptr) != hipSuccess) {
        dfree(xbits);
        dfree(pbuf);
        (void)hipGetLastError();
        return;
    }
    if (more) {
        dfree(p->dxbits);
        p->dxbits = xbits;
        p->state_bytes += xb - p->xb_bytes;
        p->xb_bytes = xb;
    }
    dfree(p->dpbuf);
    p->dpbuf = pbuf;
    p->state_bytes += pb - p->pb_bytes;
    p->pb_bytes = pb;
    p->exchange_kind = -1;  // cleared by the next launch
    p->table = g;
}

// Before a launch of sweep `kind`: the words start over when another sweep
// wrote them (its tags have another form) or a recorded launch may have.
hipError_t take_exchange(phia_problem* p, int kind)
{
    if (!p->recorded && p->exchange_kind == kind) return hipSuccess;
    p->seq = 0;
    p->exchange_kind = kind;
    return clear_exchange(p);
}

}  // namespace phia

extern "C" {

phia_status phia_anneal_run(phia_problem* p, int64_t k_end)
{
    clear_error();
    phia_status st = check_owned(p);
    if (st != PHIA_OK) return st;
    if (!p->started) return fail(PHIA_ESTATE, "phia_anneal_start has not been called");
    if (k_end < p->k || k_end > p->T) return fail(PHIA_EINVAL, "k_end = %lld outside [%lld, %lld]", (long long)k_end,
                                                  (long long)p->k, (long long)p->T);
    if (k_end == p->k) return PHIA_OK;
    hipError_t e = hipSetDevice(p->dev);
    if (e != hipSuccess) return hip_fail(p, e, "hipSetDevice");
    if (p->geo.G > 1 && p->st) {
        // A replay of a recorded launch meets the words of whatever ran before
        // it, their tags among them: a whole anneal earlier, possibly the very
        // ones it waits for (the split sweep's repeat after 2^16 steps, and
        // every sweep's after one).  So the recorded launch starts from cleared
        // words, and so does every later one on this state, as replays may come
        // in between.  Where the split sweep's shape has a sweep without an
        // exchange, that one is recorded.
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(p->st, &cs) == hipSuccess && cs == hipStreamCaptureStatusActive) {
            if (p->geo.kind == 6 && !p->give_up) {
                const Geometry split = p->geo;
                p->no_split = true;
                choose_geometry(p, p->R);
                p->no_split = false;
                if (p->geo.ok && p->geo.G == 1) {
                    st = phia_anneal_run(p, k_end);
                    p->geo = split;
                    return st;
                }
                p->geo = split;
            }
            p->recorded = true;
        }
    }
    if (p->geo.G > 1 && (e = take_exchange(p, p->geo.kind)) != hipSuccess) return hip_fail(p, e, "exchange reset");
    SweepArgs a = sweep_args(p);
    a.k0 = p->k;
    a.k1 = k_end;
    // test hook: the error word raised before the launch, as if another
    // workgroup had given up
    if (p->give_up && (e = fill_words(p->derr, 2, 8, p->st)) != hipSuccess)
        return hip_fail(p, e, "error word");
    if (p->give_up || p->geo.G > 1) p->err_live = true;
    if (p->geo.kind == 5) {
        e = launch_sweep_res(p->geo.fp4, a, p->st);
    } else if (p->geo.kind == 4) {
        e = launch_sweep_valu(valu_form(p), p->geo.rows, p->geo.j_lds != 0, a, p->st);
    } else if (p->geo.kind == 6) {
        // 16-bit tags.  Groups that run every pass rewrite their words in
        // turn, so any run of sequence numbers will do; words of a group
        // that sat out the last pass must not meet their own tag again.
        const int64_t iters = (p->geo.nblocks + p->geo.ngroups - 1) / p->geo.ngroups;
        const bool uneven = iters > 1 && p->geo.nblocks % p->geo.ngroups != 0;
        const int64_t chunk = std::max<int64_t>(1, (int64_t(1) << 30) / iters);
        for (int64_t k = p->k; k < k_end && e == hipSuccess;) {
            if (uneven && p->seq > 0xfff0u) {
                if ((e = clear_exchange(p)) != hipSuccess) break;
                p->seq = 0;
            }
            a.k0 = k;
            a.k1 = std::min(k_end, k + chunk);
            a.seq_base = p->seq;
            e = launch_sweep_split(a, p->geo.planes, p->st);
            p->seq += static_cast<uint32_t>(iters * (a.k1 - a.k0 + 1));
            k = a.k1;
        }
    } else if (p->geo.kind >= 1) {
        // 24-bit tags: launches of at most `chunk` steps, and the sequence
        // restarts (with cleared words) before it would wrap.
        const int64_t iters = (p->geo.nblocks + p->geo.ngroups - 1) / p->geo.ngroups;
        const int64_t tag_room = (int64_t(1) << 24) - 2;
        const int64_t chunk = std::min<int64_t>(int64_t(1) << 22, tag_room / iters - 1);
        for (int64_t k = p->k; k < k_end && e == hipSuccess;) {
            const int64_t kk = std::min(k_end, k + chunk);
            const int64_t use = iters * (kk - k + 1);
            if (static_cast<int64_t>(p->seq) + use > tag_room) {
                if ((e = clear_exchange(p)) != hipSuccess) break;
                p->seq = 0;
            }
            a.k0 = k;
            a.k1 = kk;
            a.seq_base = p->seq;
            e = launch_sweep_pp(a, p->geo.kind == 2, p->geo.kind == 1 && !p->geo.j_lds, p->geo.lds, p->st);
            p->seq += static_cast<uint32_t>(use);
            k = kk;
        }
    } else {
        if (p->geo.G > 1) {
            // 32-bit tags: the sequence restarts (with cleared words) before
            // it would wrap, so a word never carries a tag of a later step.
            const uint64_t iters = static_cast<uint64_t>((p->geo.nblocks + p->geo.ngroups - 1) / p->geo.ngroups);
            const uint64_t use = iters * static_cast<uint64_t>(k_end - p->k + 1);
            if (static_cast<uint64_t>(p->seq) + use > 0xfffffffeull) {
                if ((e = clear_exchange(p)) != hipSuccess) return hip_fail(p, e, "exchange reset");
                p->seq = 0;
                a.seq_base = 0;
            }
            p->seq += static_cast<uint32_t>(use);
        }
        e = launch_sweep_mfma(p->path, p->geo.mt, p->geo.cbw, a, p->geo.lds, p->st);
    }
    if (e != hipSuccess) return hip_fail(p, e, "sweep launch");
    p->k = k_end;
    p->has_run = true;
    return PHIA_OK;
}

static phia_status timed_out(phia_problem* p, int32_t err)
{
    p->poisoned = true;
    return fail(PHIA_EDEVICE, "a workgroup-group barrier timed out (device error word %d)", err);
}

phia_status phia_sync(phia_problem* p)
{
    clear_error();
    phia_status st = check_usable(p);
    if (st != PHIA_OK) return st;
    hipError_t e = hipSetDevice(p->dev);
    if (e == hipSuccess) e = p->st ? hipStreamSynchronize(p->st) : hipDeviceSynchronize();
    if (e != hipSuccess) return hip_fail(p, e, "synchronise");
    // only launches with an exchange between workgroups raise the error word (recorded ones at any time)
    if (!p->err_live && !p->recorded) return PHIA_OK;
    int32_t err = 0;
    e = hipMemcpy(&err, p->derr, sizeof err, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_fail(p, e, "read device error word");
    if (err) return timed_out(p, err);
    p->err_live = false;
    return PHIA_OK;
}

phia_status phia_anneal(phia_problem* p, int32_t replicas, int64_t steps, const phia_schedule* s, uint64_t seed)
{
    phia_status st = phia_anneal_start(p, replicas, steps, s, seed);
    if (st != PHIA_OK) return st;
    st = phia_anneal_run(p, steps);
    if (st != PHIA_OK) return st;
    return phia_sync(p);
}

// Results exist; those of a batch are complete.
static phia_status have_results(phia_problem* p)
{
    phia_status st = check_usable(p);
    if (st != PHIA_OK) return st;
    if (!p->started || !p->has_run) return fail(PHIA_ESTATE, "no anneal steps have run");
    hipError_t e = hipSetDevice(p->dev);
    if (e == hipSuccess && p->batch) e = batch_wait(p->batch);
    if (e != hipSuccess) return hip_fail(p, e, p->batch ? "batch" : "hipSetDevice");
    return PHIA_OK;
}

static phia_status need_results(phia_problem* p)
{
    phia_status st = have_results(p);
    return st != PHIA_OK ? st : phia_sync(p);
}

// `rows` rows of w bytes from device memory of row pitch `pitch` into dense
// host memory, after the work on the problem's stream.  Blocks of rows move
// whole and are packed on the host: a strided copy to pageable memory takes
// 6.5 us per row (512 rows of 2000 bytes: 3.3 ms, this way 0.1 ms).
constexpr size_t kReadBlock = size_t(32) << 20;

static hipError_t read_rows(phia_problem* p, void* dst, const void* src, size_t w, size_t pitch, size_t rows)
{
    const size_t per = w == pitch ? rows : std::min(rows, std::max<size_t>(1, kReadBlock / pitch));
    std::unique_ptr<unsigned char[]> tmp;
    if (w != pitch) {
        tmp.reset(new (std::nothrow) unsigned char[pitch * per]);
        if (!tmp) return hipErrorOutOfMemory;
    }
    hipError_t e = hipSuccess;
    for (size_t r0 = 0; r0 < rows && e == hipSuccess; r0 += per) {
        const size_t n = std::min(per, rows - r0);
        unsigned char* out = static_cast<unsigned char*>(dst) + r0 * w;
        unsigned char* buf = tmp ? tmp.get() : out;
        e = hipMemcpyAsync(buf, static_cast<const unsigned char*>(src) + r0 * pitch, pitch * n, hipMemcpyDeviceToHost,
                           p->st);
        if (e == hipSuccess) e = p->st ? hipStreamSynchronize(p->st) : hipDeviceSynchronize();
        if (e == hipSuccess && tmp)
            for (size_t r = 0; r < n; ++r) std::memcpy(out + r * w, buf + r * pitch, w);
    }
    return e;
}

// The best record: (energy units, replica) and, with spins, its N spins.  One
// kernel gathers them with the error word and one copy brings them back.
static phia_status read_best(phia_problem* p, int64_t* res, int8_t* spins)
{
    phia_status st = have_results(p);
    if (st != PHIA_OK) return st;
    const int n = spins ? p->N : 0;
    alignas(8) unsigned char buf[64 + 16384];  // N <= 16384
    hipError_t e = launch_argmin(p->dbestE, p->R, p->dscratch, p->st, spins ? p->dbestS : nullptr, p->Np, n,
                                 p->err_live || p->recorded ? p->derr : nullptr);
    if (e != hipSuccess) return hip_fail(p, e, "argmin launch");
    if ((e = hipMemcpyAsync(buf, p->dscratch, n ? 64 + static_cast<size_t>(n) : 24, hipMemcpyDeviceToHost, p->st)) !=
            hipSuccess ||
        (e = p->st ? hipStreamSynchronize(p->st) : hipDeviceSynchronize()) != hipSuccess)
        return hip_fail(p, e, "argmin readback");
    int64_t r3[3];
    std::memcpy(r3, buf, sizeof r3);
    if (r3[2]) return timed_out(p, static_cast<int32_t>(r3[2]));
    p->err_live = false;
    res[0] = r3[0];
    res[1] = r3[1];
    if (spins) std::memcpy(spins, buf + 64, static_cast<size_t>(n));
    p->best_r = static_cast<int32_t>(r3[1]);
    return PHIA_OK;
}

phia_status phia_best_exact(phia_problem* p, int64_t* energy_units, int32_t* frac_bits, int32_t* replica)
{
    clear_error();
    int64_t res[2];
    phia_status st = read_best(p, res, nullptr);
    if (st != PHIA_OK) return st;
    if (energy_units) *energy_units = res[0];
    if (frac_bits) *frac_bits = p->f;
    if (replica) *replica = static_cast<int32_t>(res[1]);
    return PHIA_OK;
}

phia_status phia_best_f64(phia_problem* p, double* energy)
{
    clear_error();
    if (!energy) return fail(PHIA_EINVAL, "energy is null");
    int64_t E;
    int32_t f, r;
    phia_status st = phia_best_exact(p, &E, &f, &r);
    if (st != PHIA_OK) return st;
    if (p->exact) {
        // couplings and fields are exactly J_int 2^-f: the energy is too
        *energy = std::ldexp(static_cast<double>(E), -f);
        return PHIA_OK;
    }
    if ((st = make_resident(p)) != PHIA_OK) return st;
    double* dout = reinterpret_cast<double*>(p->dscratch) + 4;
    hipError_t e = launch_energy_f64(p->dJ64, p->dh64, p->N, p->dbestS + static_cast<size_t>(r) * p->Np, dout, p->st);
    if (e != hipSuccess) return hip_fail(p, e, "FP64 energy launch");
    if ((e = hipMemcpyAsync(energy, dout, sizeof(double), hipMemcpyDeviceToHost, p->st)) != hipSuccess ||
        (e = p->st ? hipStreamSynchronize(p->st) : hipDeviceSynchronize()) != hipSuccess)
        return hip_fail(p, e, "FP64 energy readback");
    return PHIA_OK;
}

phia_status phia_best(phia_problem* p, double* energy, int8_t* spins)
{
    clear_error();
    int64_t res[2];
    phia_status st = read_best(p, res, spins);
    if (st != PHIA_OK) return st;
    if (energy) {
        if (p->exact) {
            *energy = std::ldexp(static_cast<double>(res[0]), -p->f);
        } else {
            st = phia_best_f64(p, energy);
            if (st != PHIA_OK) return st;
        }
    }
    return PHIA_OK;
}

phia_status phia_replica_best(phia_problem* p, int64_t* E, int8_t* S, int64_t* step)
{
    clear_error();
    phia_status st = need_results(p);
    if (st != PHIA_OK) return st;
    // energies, steps and spins are one allocation: one copy brings back what is read
    const size_t R = static_cast<size_t>(p->R), eb = sizeof(int64_t) * R;
    const bool spins_too = S && R * p->Np <= kReadBlock;
    const size_t bytes = spins_too ? 2 * eb + R * p->Np : step ? 2 * eb : E ? eb : 0;
    hipError_t e = hipSuccess;
    if (bytes) {
        std::unique_ptr<unsigned char[]> buf(new (std::nothrow) unsigned char[bytes]);
        if (!buf) return fail(PHIA_ENOMEM, "host allocation failed");
        e = hipMemcpyAsync(buf.get(), p->dbestE, bytes, hipMemcpyDeviceToHost, p->st);
        if (e == hipSuccess) e = p->st ? hipStreamSynchronize(p->st) : hipDeviceSynchronize();
        if (e != hipSuccess) return hip_fail(p, e, "records readback");
        if (E) std::memcpy(E, buf.get(), eb);
        if (step) std::memcpy(step, buf.get() + eb, eb);
        if (spins_too)
            for (size_t r = 0; r < R; ++r)
                std::memcpy(S + r * p->N, buf.get() + 2 * eb + r * p->Np, static_cast<size_t>(p->N));
    }
    if (S && !spins_too &&
        (e = read_rows(p, S, p->dbestS, static_cast<size_t>(p->N), static_cast<size_t>(p->Np), R)) != hipSuccess)
        return hip_fail(p, e, "records readback");
    return PHIA_OK;
}

phia_status phia_replica_mh(phia_problem* p, int32_t* accepted, int32_t* decided, float* lam)
{
    clear_error();
    phia_status st = need_results(p);
    if (st != PHIA_OK) return st;
    if (!p->mh) return fail(PHIA_ESTATE, "the current anneal has no accept/reject step");
    hipError_t e;
    if (accepted || decided) {
        std::vector<int32_t> c(2 * static_cast<size_t>(p->R));
        if ((e = hipMemcpy(c.data(), p->dmhc, sizeof(int32_t) * c.size(), hipMemcpyDeviceToHost)) != hipSuccess)
            return hip_fail(p, e, "accept/reject readback");
        for (int32_t r = 0; r < p->R; ++r) {
            if (accepted) accepted[r] = c[2 * static_cast<size_t>(r)];
            if (decided) decided[r] = c[2 * static_cast<size_t>(r) + 1];
        }
    }
    if (lam && (e = hipMemcpy(lam, p->dlam, sizeof(float) * p->R, hipMemcpyDeviceToHost)) != hipSuccess)
        return hip_fail(p, e, "accept/reject readback");
    return PHIA_OK;
}

phia_status phia_get_trace(phia_problem* p, int64_t* E)
{
    clear_error();
    phia_status st = need_results(p);
    if (st != PHIA_OK) return st;
    if (!p->detrace) return fail(PHIA_ESTATE, "tracing was not enabled before phia_anneal_start");
    if (!E) return fail(PHIA_EINVAL, "E is null");
    hipError_t e = hipMemcpy(E, p->detrace, sizeof(int64_t) * p->R * p->T, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_fail(p, e, "trace readback");
    return PHIA_OK;
}

phia_status phia_get_state(phia_problem* p, float* x, float* v, int64_t* k)
{
    clear_error();
    phia_status st = check_usable(p);
    if (st != PHIA_OK) return st;
    if (!p->started) return fail(PHIA_ESTATE, "no anneal started");
    if (p->batch) {
        hipError_t eb = batch_wait(p->batch);
        if (eb != hipSuccess) return hip_fail(p, eb, "batch");
    }
    st = phia_sync(p);
    if (st != PHIA_OK) return st;
    const size_t pitch = sizeof(float) * p->Np, w = sizeof(float) * p->N;
    hipError_t e;
    if (x && (e = read_rows(p, x, p->dx, w, pitch, static_cast<size_t>(p->R))) != hipSuccess)
        return hip_fail(p, e, "state readback");
    if (v && (e = read_rows(p, v, p->dv, w, pitch, static_cast<size_t>(p->R))) != hipSuccess)
        return hip_fail(p, e, "state readback");
    if (k) *k = p->k;
    return PHIA_OK;
}

phia_status phia_set_state(phia_problem* p, const float* x, const float* v, int64_t k)
{
    clear_error();
    phia_status st = check_owned(p);
    if (st != PHIA_OK) return st;
    if (!p->started) return fail(PHIA_ESTATE, "no anneal started");
    if (!x || !v) return fail(PHIA_EINVAL, "x and v are required");
    if (k < 0 || k > p->T) return fail(PHIA_EINVAL, "k outside [0, steps]");
    st = phia_sync(p);
    if (st != PHIA_OK) return st;
    const size_t pitch = sizeof(float) * p->Np, w = sizeof(float) * p->N;
    hipError_t e;
    if ((e = hipMemcpy2D(p->dx, pitch, x, w, w, static_cast<size_t>(p->R), hipMemcpyHostToDevice)) != hipSuccess ||
        (e = hipMemcpy2D(p->dv, pitch, v, w, w, static_cast<size_t>(p->R), hipMemcpyHostToDevice)) != hipSuccess)
        return hip_fail(p, e, "state upload");
    if (p->mh) {
        // the accept/reject state restarts as after the initial draw
        const size_t R = static_cast<size_t>(p->R);
        std::vector<int64_t> mE(2 * R, 0);
        for (size_t r = 0; r < R; ++r) mE[2 * r] = INT64_MIN;
        const std::vector<float> lam(R, 1.0f);
        const std::vector<int32_t> c(2 * R, 0);
        const std::vector<int64_t> q(p->mhQ_cap, 0);
        if ((e = hipMemcpy(p->dmhE, mE.data(), sizeof(int64_t) * mE.size(), hipMemcpyHostToDevice)) != hipSuccess ||
            (e = hipMemcpy(p->dlam, lam.data(), sizeof(float) * R, hipMemcpyHostToDevice)) != hipSuccess ||
            (e = hipMemcpy(p->dmhc, c.data(), sizeof(int32_t) * c.size(), hipMemcpyHostToDevice)) != hipSuccess ||
            (e = hipMemcpy(p->dmhQ, q.data(), sizeof(int64_t) * q.size(), hipMemcpyHostToDevice)) != hipSuccess)
            return hip_fail(p, e, "accept/reject state reset");
    }
    p->k = k;
    return PHIA_OK;
}

phia_status phia_autotune(phia_problem* p, int32_t replicas, int64_t probe_steps, double* best_us)
{
    clear_error();
    phia_status st = check_owned(p);
    if (st != PHIA_OK) return st;
    if (replicas < 1 || replicas > (1 << 20)) return fail(PHIA_EINVAL, "replicas = %d outside [1, 2^20]", replicas);
    if (probe_steps < 10 || probe_steps > 100000) return fail(PHIA_EINVAL, "probe_steps outside [10, 100000]");
    if (best_us) *best_us = 0.0;
    if ((p->path == PHIA_PATH_FP32 || p->path == PHIA_PATH_ELL) && p->mh) return PHIA_OK;
    p->ikick = 0;  // the last anneal's, which has candidates of its own; the probes run without
    std::vector<Geometry> cands = candidate_geometries(p, replicas);
    if (cands.empty()) return fail(PHIA_ERANGE, "no kernel geometry fits N = %d on this device", p->N);
    // Candidates that need more passes over the replica blocks than twice
    // the best one cannot win; skip them.
    int min_iters = 1 << 30;
    for (const Geometry& g : cands)
        if (g.kind < 5) min_iters = std::min(min_iters, (g.nblocks + g.ngroups - 1) / g.ngroups);
    hipError_t e = hipSetDevice(p->dev);
    if (e != hipSuccess) return hip_fail(p, e, "hipSetDevice");
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if ((e = hipEventCreate(&e0)) != hipSuccess || (e = hipEventCreate(&e1)) != hipSuccess) {
        if (e0) (void)hipEventDestroy(e0);
        return hip_fail(p, e, "event creation");
    }
    const phia_schedule sched{0.1f, 3.0f, nullptr, 0.2f, 1.0f, 25};
    const int64_t warm = 8;
    const bool trace = p->trace;
    p->trace = false;
    Geometry best{};
    double best_step_us = 0.0;
    for (const Geometry& g : cands) {
        if (g.kind < 5 && (g.nblocks + g.ngroups - 1) / g.ngroups > 2 * min_iters) continue;
        free_state(p);
        p->tuned = g;
        p->tuned_R = replicas;
        st = phia_anneal_start(p, replicas, warm + probe_steps, &sched, 1);
        if (st == PHIA_OK) st = phia_anneal_run(p, warm);
        if (st != PHIA_OK) break;
        if ((e = hipEventRecord(e0, p->st)) != hipSuccess) {
            st = hip_fail(p, e, "event record");
            break;
        }
        st = phia_anneal_run(p, warm + probe_steps);
        if (st != PHIA_OK) break;
        if ((e = hipEventRecord(e1, p->st)) != hipSuccess || (e = hipEventSynchronize(e1)) != hipSuccess) {
            st = hip_fail(p, e, "event timing");
            break;
        }
        st = phia_sync(p);
        if (st != PHIA_OK) break;
        float ms = 0.f;
        (void)hipEventElapsedTime(&ms, e0, e1);
        const double us = 1000.0 * ms / static_cast<double>(probe_steps);
        // A later candidate must win by 2 % (timing noise on the probe).
        if (!best.ok || us < 0.98 * best_step_us) {
            best = g;
            best_step_us = us;
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    free_state(p);
    p->trace = trace;
    p->started = false;
    p->has_run = false;
    p->tuned = best;
    p->tuned_R = best.ok ? replicas : 0;
    p->geo = best;
    if (st != PHIA_OK) return st;
    if (!best.ok) return fail(PHIA_ERANGE, "no geometry could be timed");
    append_tune_cache(p, replicas, best, best_step_us);
    if (best_us) *best_us = best_step_us;
    return PHIA_OK;
}

phia_status phia_get_info(const phia_problem* p, phia_info* out)
{
    clear_error();
    if (!p || !out) return fail(PHIA_EINVAL, "null argument");
    out->N = p->N;
    out->Np = p->Np;
    out->path = p->path;
    out->frac_bits = p->f;
    out->exact = p->exact ? 1 : 0;
    out->group = p->geo.G;
    out->replicas = p->R;
    out->rows_per_block = p->geo.rows;
    out->j_in_lds = p->geo.j_lds;
    out->incremental = p->geo.inc;
    out->sweep_kernel = p->geo.kind;
    out->steps = p->T;
    out->step = p->k;
    out->max_abs_J = p->maxabsJ;
    out->device_bytes = p->base_bytes + p->state_bytes;
    out->group_on_one_xcd = p->geo.G > 1 ? p->geo.xcd_map : 0;
    return PHIA_OK;
}

phia_status phia_incremental_stats(phia_problem* p, int64_t* out)
{
    clear_error();
    phia_status st = check_usable(p);
    if (st != PHIA_OK) return st;
    if (!out) return fail(PHIA_EINVAL, "null argument");
    if (!p->started) return fail(PHIA_ESTATE, "phia_anneal_start has not been called");
    hipError_t e = hipSetDevice(p->dev);
    if (e == hipSuccess) e = hipMemcpyAsync(out, p->dincstat, 3 * sizeof(int64_t), hipMemcpyDeviceToHost, p->st);
    if (e == hipSuccess) e = p->st ? hipStreamSynchronize(p->st) : hipDeviceSynchronize();
    if (e != hipSuccess) return hip_fail(p, e, "counter read");
    return PHIA_OK;
}

phia_status phia_set_incremental(phia_problem* p, int32_t on)
{
    clear_error();
    phia_status st = check_usable(p);
    if (st != PHIA_OK) return st;
    if (on < -1 || on > 1) return fail(PHIA_EINVAL, "incremental must be -1, 0 or 1 (got %d)", on);
    p->inc_mode = on;
    return PHIA_OK;
}

phia_status phia_set_exchange_seq(phia_problem* p, uint32_t seq)
{
    clear_error();
    phia_status st = check_usable(p);
    if (st != PHIA_OK) return st;
    if (!p->started) return fail(PHIA_ESTATE, "phia_anneal_start has not been called");
    if (p->geo.G < 2) return fail(PHIA_ESTATE, "the current geometry has no exchange between workgroups");
    const uint32_t room = p->geo.kind == 6 ? 0xfff0u : p->geo.kind >= 1 ? (1u << 24) - 2u : 0xfffffffeu;
    if (seq > room) return fail(PHIA_EINVAL, "seq = %u beyond the tag range", seq);
    p->seq = seq;
    return PHIA_OK;
}

phia_status phia_raise_error_word(phia_problem* p, int32_t on)
{
    clear_error();
    phia_status st = check_usable(p);
    if (st != PHIA_OK) return st;
    p->give_up = on != 0;
    return PHIA_OK;
}

phia_status phia_eval_fmath(int32_t kind, const float* in, const uint64_t* in64, float* out, int64_t n,
                            int32_t device)
{
    clear_error();
    if (kind < 0 || kind > 5 || n < 0 || !out) return fail(PHIA_EINVAL, "bad argument");
    if (n == 0) return PHIA_OK;
    if (kind != 4 && !in) return fail(PHIA_EINVAL, "in is null");
    if (kind == 4 && !in64) return fail(PHIA_EINVAL, "in64 is null");
    hipError_t e = hipSetDevice(device);
    if (e != hipSuccess) return hip_fail(nullptr, e, "hipSetDevice");
    const size_t nout = static_cast<size_t>(n) * (kind == 2 ? 2 : 1);
    float *din = nullptr, *dout = nullptr;
    uint64_t* d64 = nullptr;
    phia_status st = PHIA_OK;
    if ((e = hipMalloc(&dout, nout * sizeof(float))) != hipSuccess) return fail(PHIA_ENOMEM, "allocation failed");
    if (kind != 4) {
        if ((e = hipMalloc(&din, static_cast<size_t>(n) * sizeof(float))) != hipSuccess ||
            (e = hipMemcpy(din, in, static_cast<size_t>(n) * sizeof(float), hipMemcpyHostToDevice)) != hipSuccess)
            st = hip_fail(nullptr, e, "fmath upload");
    } else {
        const size_t m = 1 + 4 * static_cast<size_t>(n);
        if ((e = hipMalloc(&d64, m * sizeof(uint64_t))) != hipSuccess ||
            (e = hipMemcpy(d64, in64, m * sizeof(uint64_t), hipMemcpyHostToDevice)) != hipSuccess)
            st = hip_fail(nullptr, e, "fmath upload");
    }
    if (st == PHIA_OK) {
        if ((e = launch_fmath_eval(kind, din, d64, dout, n, nullptr)) != hipSuccess ||
            (e = hipDeviceSynchronize()) != hipSuccess ||
            (e = hipMemcpy(out, dout, nout * sizeof(float), hipMemcpyDeviceToHost)) != hipSuccess)
            st = hip_fail(nullptr, e, "fmath kernel");
    }
    dfree(din);
    dfree(dout);
    dfree(d64);
    return st;
}

}  // extern "C"

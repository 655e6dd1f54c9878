// lbm_api.cpp - the C ABI of liblbm (declared in include/lbm.h): context,
// argument validation, buffer layout and the launch sequences of the update,
// the diagnostics, checkpointed runs and the adjoint.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <limits>
#include <new>
#include <string>
#include <vector>

#include "lbm.h"
#include "lbm_host.h"
#include "lbm_internal.h"

#define LBM_API extern "C" __attribute__((visibility("default")))

using lbm::KParams;
using lbm::ModelId;
using lbm::Prec;

struct lbm_ctx {
    ModelId model;
    Prec prec;
    int D = 0, Q = 0, G = 0;
    int64_t extent[3] = {1, 1, 1};
    long long N = 0;
    double c = 0, T0 = 0, omega = 0, rho0 = 0;
    double w[LBM_MAX_Q] = {};
    double W[lbm::kMaxG] = {};
    hipStream_t stream = nullptr;
    int device = -1;
    void* f[2] = {nullptr, nullptr};
    int cur = 0;
    void* scratch = nullptr;
    bool bound = false;
    bool initialized = false;
    KParams kp{};
    bool aa = false;                // one buffer, in-place AA-pattern steps
    // Graph replay of lbm_step: G steps captured once and replayed while the
    // launch state (buffer parity, storage form) matches the captured one.
    int graph_steps = 0;
    hipGraphExec_t graph_exec = nullptr;
    int graph_cur = -1, graph_form = -1;
    int hold_lo = 0, hold_hi = 0;   // planes held at f^eq at each end of the slowest axis
    int mapping = 0;                // forward steps' block order: 0 contiguous rows per XCD,
                                    // 1 slabs in turn (lbm_tune_step)
    lbm::FixedState hold[2]{};
    std::string err;
};

namespace lbm {

// Launch geometry (host only; the kernels' launch bounds use the same limit).
int step_max_threads(ModelId m, Prec p) { return row_block_limit(model_q(m), p); }

RowLaunch row_launch(int nx, long long rows, int max_threads) {
    RowLaunch r;
    r.chunks = (nx + max_threads - 1) / max_threads;
    const int per = (nx + r.chunks - 1) / r.chunks;
    r.bx = ((per + 63) / 64) * 64;
    r.blocks = rows * r.chunks;
    return r;
}

int reduce_blocks(long long N) {
    long long b = (N + kReduceThreads - 1) / kReduceThreads;
    if (b > 1024) b = 1024;
    if (b < 1) b = 1;
    return static_cast<int>(b);
}

long long step_blocks(ModelId, Prec, const KParams& kp) {
    if (kp.flat) return static_cast<long long>(kp.nz) * kp.gpp * kp.chunks;
    return static_cast<long long>(kp.ny) * kp.nz / kp.rpb * kp.chunks;
}

}  // namespace lbm

namespace {

thread_local std::string g_err;

constexpr size_t kAlign = 256;

size_t round_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

int fail(lbm_ctx* ctx, int code, const std::string& msg) {
    if (ctx)
        ctx->err = msg;
    else
        g_err = msg;
    return code;
}

int fail_hip(lbm_ctx* ctx, hipError_t e, const char* what) {
    return fail(ctx, LBM_E_DEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

size_t elem_bytes(Prec p) { return p == Prec::F64 ? 8 : 4; }

// Elements between two population runs of a grid row.
long long run_stride_of(long long nx) {
    const long long a = nx < lbm::kRunAlign ? 1 : lbm::kRunAlign;
    return (nx + a - 1) / a * a + lbm::kRunPad;
}

size_t pop_bytes(const lbm_ctx* ctx) {
    const KParams& k = ctx->kp;
    return static_cast<size_t>(k.gs) * k.gpp * k.nz * elem_bytes(ctx->prec);
}

size_t scratch_bytes(const lbm_ctx* ctx) {
    const size_t parts = static_cast<size_t>(lbm::reduce_blocks(ctx->N)) * (ctx->D + 2) * 8;
    return round_up(parts) + round_up((ctx->D + 2) * 8);
}

// Checks that [p, p + bytes) lies inside one device allocation of the
// context's device, so that no kernel of this library can touch memory
// outside what the caller handed over.
int check_dev(lbm_ctx* ctx, const void* p, size_t bytes, const char* name) {
    if (!p) return fail(ctx, LBM_E_INVALID, std::string(name) + " is NULL");
    if (reinterpret_cast<uintptr_t>(p) % 8 != 0)
        return fail(ctx, LBM_E_INVALID, std::string(name) + " is not 8-byte aligned");
    hipPointerAttribute_t attr;
    std::memset(&attr, 0, sizeof(attr));
    hipError_t e = hipPointerGetAttributes(&attr, p);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return fail(ctx, LBM_E_INVALID, std::string(name) + " is not a HIP device pointer");
    }
    if (attr.type != hipMemoryTypeDevice)
        return fail(ctx, LBM_E_INVALID, std::string(name) + " is not device memory");
    if (ctx->device >= 0 && attr.device != ctx->device)
        return fail(ctx, LBM_E_INVALID, std::string(name) + " is on another device");
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    e = hipMemGetAddressRange(&base, &size, const_cast<void*>(p));
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return fail(ctx, LBM_E_INVALID, std::string(name) + ": allocation range unknown");
    }
    const uintptr_t b = reinterpret_cast<uintptr_t>(base);
    const uintptr_t q = reinterpret_cast<uintptr_t>(p);
    if (q < b || q - b + bytes > size)
        return fail(ctx, LBM_E_INVALID,
                    std::string(name) + " is smaller than the " + std::to_string(bytes) +
                        " bytes required");
    return LBM_OK;
}

// Storage form the state starts in after lbm_init_fields / lbm_set_populations.
int initial_form(const lbm_ctx* ctx) { return ctx->aa ? lbm::kFormSwapped : lbm::kFormAB; }

// Blocks of the forward step per slab of the slowest axis (a z-plane in 3D,
// a row in 2D): the chunk the XCDs take in turn in the alternative mapping.
int cyclic_chunk(const KParams& k, int D) {
    const long long rows = D == 3 ? (k.flat ? k.gpp : k.ny) : 1;   // or flat row groups
    const long long blocks = rows * k.chunks / k.rpb;
    return static_cast<int>(std::max(1LL, std::min(blocks, 1LL << 20)));
}

// Storage layout (row_base in the kernels).
//
// Run length.  A population run holds at least kRunCells cells where the
// plane has them: one long run per population and group costs HBM less than
// several short ones (D3Q95 FP32-shifted 128^3, runs of 256 cells against
// 1024: 304 against 295 us per step, 256^3: 2319 against 2246-2270 us; float64
// 128^3: 589 against 567 us; 192^3, 320^3 and 384^3 the same within 0.3 %;
// longer runs give no more).  2D rows are taken one by one: on D2Q33 8192^2
// groups lost 3 % (2 rows) to 13 % (8 rows).
//
// Flat rows.  Rows that are no multiple of a wave and shorter than kFlatCells
// follow each other without padding, and lanes count through the group: no
// lane is lost at a row's end, every store of a wave is whole lines, and no
// padding is read.  Measured against padded rows, whose surplus lanes fill the
// row's last line (D3Q95 FP32-shifted): 33 cells 72 against 43 us
// (33x90x80), 100 cells 74 against 64 us (100x75x50), 200 cells 1255 against
// 1131 us (200^3), 300 cells 665 against 645 us, 415 cells 871 against 875 us:
// past kFlatCells the padding is small and uniform row addresses cost less.
// Groups of a power of two of rows leave the last one partly empty; the
// shortest that keeps the state within the padded rows' bytes (or, for states
// that are small against the memory, within an eighth of its cells) is taken,
// else the whole plane is one group, up to kWholeCells: longer runs lie too far
// apart, as in one array per population (us per step, one group against rows:
// D2Q33 float64 96x62501 610, 539, in place 595, 515; D3Q95 float64 383x250x60
// 1731, 1537, FP32-shifted in place 224x250x100 853, 815; 160x50x750, 8000 cells,
// 1638, 1735), unless rows would leave half the lanes idle and all runs off the
// line grid (D3Q15 float64 in place 30x1219x445 691, 852; D2Q33 20x300001 592, 709,
// but 31x200001 623, 567).  By rows are also 29 to 31 cells of D3Q95 FP32-shifted
// with two buffers where the plane's run is no multiple of a line: its stores
// would all start inside one (31x33x9000 1766, 1507; in place 1289, 1488).
constexpr long long kSmallState = 1LL << 30;   // bytes
constexpr long long kWholeCells = 16 * lbm::kRunCells;

void fill_layout(const lbm_ctx* ctx, KParams& k) {
    const long long bytes = static_cast<long long>(elem_bytes(ctx->prec));
    const long long by_rows = run_stride_of(k.nx) * k.ny;   // elements per population and plane
    const bool small = by_rows * k.nz * ctx->Q * bytes <= kSmallState;
    int sh = 0;
    k.flat = 0;
    if (k.nx % 64 != 0 && k.nx < lbm::kFlatCells) {
        while ((static_cast<long long>(k.nx) << sh) < lbm::kRunCells && (1LL << sh) < k.ny) ++sh;
        for (bool whole = false; !k.flat && !whole; ++sh) {
            whole = (1LL << sh) >= k.ny;
            const long long rg = whole ? k.ny : 1LL << sh;
            const long long gpp = (k.ny + rg - 1) / rg;
            // whole lines per run, unless that adds more than a sixteenth
            const long long lines = (rg * k.nx + lbm::kRunAlign - 1) / lbm::kRunAlign;
            const bool pad = 16 * (lines * lbm::kRunAlign - rg * k.nx) <= rg * k.nx &&
                             (!whole || lines * lbm::kRunAlign <= by_rows || small);
            const long long ps = pad ? lines * lbm::kRunAlign : rg * k.nx;
            const bool apart =
                whole && ((k.nx >= (ctx->D == 3 ? 32 : 24) && rg * k.nx > kWholeCells) ||
                          (!ctx->aa && ctx->Q >= 95 && bytes == 4 && k.nx > 28 &&
                           ps % lbm::kRunAlign != 0 && !small));
            const long long plane = ps * gpp * ctx->Q * bytes;
            const bool fits = ps * gpp <= by_rows ||
                              (small && (whole || 8 * gpp * rg <= 9LL * k.ny));
            // the kernels address a plane (in 2D: the grid) with 32-bit byte offsets
            if (!fits || apart || plane >= (1LL << 32)) continue;
            k.flat = 1;
            k.rg = static_cast<int>(rg);
            k.rg_shift = whole ? 31 : sh;
            k.rs = k.nx;
            k.ps = static_cast<int>(ps);
            k.gpp = static_cast<int>(gpp);
        }
    }
    if (!k.flat) {
        sh = 0;
        if (ctx->D == 3)
            while ((static_cast<long long>(k.nx) << sh) < lbm::kRunCells && k.ny % (2 << sh) == 0)
                ++sh;
        k.rs = static_cast<int>(run_stride_of(k.nx));
        k.rg_shift = sh;
        k.rg = 1 << sh;
        k.gpp = k.ny / k.rg;
        k.ps = k.rg * k.rs;
    }
    const int line = lbm::kLineBytes / static_cast<int>(bytes);
    k.lim = std::min((k.nx + line - 1) / line * line, k.rs);   // unpadded rows: rs = nx
    // groups and 3D planes stay below 4 GiB
    k.gs = static_cast<unsigned>(ctx->Q) * static_cast<unsigned>(k.ps);
    k.zs = ctx->D == 3 ? k.gs * static_cast<unsigned>(k.gpp) : 0u;
    // Populations a step leaves in the cache are read from there by the next
    // one: plain stores while the state (both buffers) is not much larger than
    // the cache, non-temporal ones past that, where no line survives until it
    // is read.  D3Q95, us per step non-temporal against plain: FP32-shifted
    // 64^3 (199 MB) 38.9, 30.7; 64x64x96 (299 MB) 63.7, 60.2; 64x64x128 (398 MB)
    // 80.6, 78.4; 64x64x160 (498 MB) 100.6, 101.7; 128x128x64 (797 MB) 157.9,
    // 162.7; float64 64x64x32 (199 MB) 38.4, 31.9; in place 64x64x128 (199 MB)
    // 64.9, 58.7, 64x64x160 (249 MB) 75.8, 74.4, float64 128^3 D3Q19 (319 MB) 93.6,
    // 95.6 and 128x128x64 (398 MB) 129.9, 134.2.  The smaller sets change over earlier:
    // D2Q33 512^2 15.0, 12.5; 1000x1000 (264 MB) 53.1, 46.8; 1000x1200 (317) 59.4, 55.0;
    // 1000x1311 (346) 64.4, 64.1; 1000x1450 (383) 70.5, 74.4; float64 1024x700 (378)
    // 67.4, 70.7; D3Q19 FP32-shifted 128x128x140 (349) 61.0, 60.7; 128x128x156 (388) 67.1,
    // 69.8; float64 128x128x76 (379) 66.3, 68.3.
    const long long state = static_cast<long long>(k.gs) * k.gpp * k.nz * bytes;
    // Between those, D3Q95 with two buffers of 16 to 40 MB: the L2s (8 of 4 MB)
    // hold a whole step's output and write it back at the kernel's end, which
    // non-temporal stores start earlier (FP32-shifted 32^3, 25 MB: 9.5 against
    // 11.0 us; float64 24^3, 21 MB: 9.6, 10.7; 16^3, 6 MB: 9.3, 8.6; FP32-shifted
    // 40^3, 49 MB: 17.9, 13.5).  The smaller sets gain nothing (D3Q15 64^3, 31
    // MB: 7.2 against 6.6 us).
    const long long moved = ctx->aa ? state : 2 * state;
    const long long cached = ctx->aa ? lbm::kCachedStateInPlace
                             : ctx->Q >= 95 ? lbm::kCachedState : lbm::kCachedStateSmallSets;
    k.nt = moved > cached ||
           (!ctx->aa && ctx->Q >= 95 && moved > lbm::kL2StateLo && moved <= lbm::kL2StateHi);
}

lbm::FastDiv fast_div(int d) {
    lbm::FastDiv f;
    f.shift = 31;
    while ((1LL << (f.shift - 31)) < d) ++f.shift;
    f.mul = static_cast<unsigned>((1ULL << f.shift) / static_cast<unsigned>(d) + 1);
    return f;
}

// Divisions of the lane-to-cell mapping.
void set_divisors(KParams& k) {
    k.by_nx = fast_div(k.nx);
    k.by_ny = fast_div(k.ny);
    k.by_gpp = fast_div(k.gpp);
    k.by_chunks = fast_div(k.chunks);
    k.inv_nx = 65536u / static_cast<unsigned>(k.nx) + 1;
    k.inv_ny = 65536u / static_cast<unsigned>(k.ny) + 1;
    k.inv_nz = 65536u / static_cast<unsigned>(k.nz) + 1;
}

// Kernels that share a block size.
enum BlockUse { kSteps, kStepsInPlace, kAdjoint };

// FP32-shifted D3Q95 states from which both in-place steps are held (see set_blocks).
constexpr size_t kHeldInPlace = size_t{1} << 30;

// Cells that the blocks a CU holds at once have together at least, where they are
// held (see set_blocks).  Cells and not blocks are counted, since a short row or
// a thin plane may give a block only a few.  us per step by blocks per CU (- not
// measured; * what the rule takes):
//                       cells    1    2    3    4    6    8  unlimited
//   D3Q95 FP32-shifted
//     64x251x251           64  1308  720  573  541  549  553  564   *5
//     11x11x5000          121   138  100  *94   94   95   94   94
//     128x129x129         128   397  301 *293  296  302  301  300
//     192x129x129         192   487 *442  444  448  454  454  455
//     256x129x129         256   600 *583  594  601  601  601  601
//     320x111x111         320  *540  546  549  549  549  549  549
//   D3Q95 float64
//     5x5x20000            25   491  262  209  182 *167  168  168
//     64x251x251           64  1522 1110*1094 1102 1120 1119 1120
//     11x11x10000         121   376 *342  352  353  353    -  353
//     11x11x20000         121   782 *814  870  782  764    -  763
//     128x129x129         128   639 *585  597  599  597  598  598
//     320x128x128         160 *1452 1484 1509 1509 1510    - 1510
//     192x129x129         192  *868  891  896  896  896  896  897
//   D3Q95 FP32-shifted in place
//     64x251x251           64  1203  666  561 *552  553  557  549
//     16x11x20000          88   827  561 *519  522  566    -  569
//     400x128x128         100  1362 1017 *993 1021 1078    - 1058
//     777x101x101         111  1487 1166*1179 1213 1274    - 1232
//     100x200x200         115   727 *576  580  599  625    -  598
//     128x200x200         128     - *704  711  724  729  732  731
//     192x200x200         192     -*1095 1115 1123 1121 1119 1120
//   smaller sets, FP32-shifted
//     D3Q19 64x511x511     64     - 1154  815  634  465 *417  447
//     D3Q19 192x256x256   192     -  381 *322  327  332  334  342
//     D3Q19 400x160x160   200   430  292 *275  283  289    -  291
//     D3Q19 128x256x256   256     - *214  217  218  221  225  225
//     D2Q33 384x30000     384   557 *518  527  526  528    -  527
//     D2Q33 256x50000     512  *556  582  580  593  593    -  592
//     D3Q15 200^3         229   277  174 *163  164  168    -  172
//     D3Q15 256x200x200   256   318  212 *207  211  210    -  215
//     D3Q15 384x160x160   192   395  232  204 *202  208    -  210
//   smaller sets, float64 (two blocks at least, but see set_blocks)
//     D3Q19 5x5x200000     25     -  751  540  449  377  334  331  *10
//     D3Q19 11x11x60000   121   522 *392  414  430  462    -  439
//     D3Q19 400x160x160   200   673  536  560  567  581    -  581
//                         400  *516  527    -    -    -    -    -
//     D3Q15 384x160x160   192   497 *406  417  422  421    -  425
//     D3Q15 256x200x200   256   506 *415  417  420  422    -  423
int held_cells(const lbm_ctx* ctx, BlockUse use) {
    const bool f64 = ctx->prec == Prec::F64;
    if (ctx->Q >= 95) {
        if (f64) return 150;
        return use == kStepsInPlace && pop_bytes(ctx) >= kHeldInPlace ? 230 : 300;
    }
    return f64 ? 240 : ctx->Q >= 19 ? 450 : 600;
}

// Blocks of the kernels that advance cells: their size, and how many a CU holds
// at once (k.resident).
//
// Few waves are spread one by one over the CUs (us per step with blocks of
// several waves against one: D3Q95 float64 512x4x4 12.2, 9.6; 64x16x16 12.7,
// 9.8; FP32-shifted 28^3 10.0, 8.9; 64x48x48 21.8, 19.5; D2Q33 float64 128x4 6.1,
// 5.3; 400^2 16.0, 15.1; from 64^3 on the same).
//
// States past the cache (k.nt) are bound by HBM, whose rate falls as more waves
// read and write their own places in it at once, and which too few do not fill:
// a CU is held to the fewest blocks that have held_cells() cells.  us per step,
// unlimited against held, on the same buffers: D3Q95 FP32-shifted one block
// of 512 or a 384-cell row (128^3 292, 281; 256^3 2260, 2188; 384^3 7770, 7505 where
// the buffers lie badly in HBM, the same within 1 % where they lie well (7.1-7.2 ms);
// 200^3 1144, 1105), float64 one of 256 (256^3 4468, 4315; 150^3 937, 898); D2Q33
// FP32-shifted one of 512 (2393x3579 403, 388; 8192^2 2914, 2867), float64 two of
// 256 (814, 788); D3Q19 FP32-shifted two of 256 (256^3 438, 416), float64 the same
// (889, 856).
// In place the two steps differ (see k_step_aa): the one that pushes writes lines
// other blocks read and is held; the local one touches its own cells only.  us
// per step (the mean of both), unlimited, push held, both held: D3Q95 float64
// 192x70x60 218, 210, 228; 256x64x80 357, 353, 374; 128^3 588, 586, 600; 400x100x100
// 1249, 1189, 1172; 512x100x100 1507, 1469, 1482; flat 150x100x60 250, 241, 254; 200x100x100
// 606, 579, 586; flat with runs off the line grid both (17x652x269 958, 938, 899;
// 11x11x40000 1417, 1401, 1323); rows of one block of 192, or of two, both from 1.5 GB (192x128x100
// 741, 713, 711; 320x100x100 994, 942, 922; below 384x60x44 293, 277, 292); FP32-shifted
// below 1 GB 57x176x86 136, 126, 126; 300x80x60 194, 187, 200; 128^3 271, 269, 281;
// 320x80x60 227, 219, 220; from 1 GB two blocks of 128 in both (256x128x128 647, 597,
// 588; 384^3 8830, -, 8009; 170x145x141 525, -, 506).  The smaller sets two blocks of 256
// in both (D2Q33 2000^2 179, 168, 163, float64 365, 356, 345; D3Q19 float64
// 200x150x110 165, 157, 155).  The cache prefers many waves (64^3 FP32-shifted 30,
// held 49), and so does the adjoint's mix of arithmetic and loads (128^3, 40
// steps: 18.5 ms with and without).
void set_blocks(const lbm_ctx* ctx, KParams& k, BlockUse use) {
    const long long rows = static_cast<long long>(k.ny) * k.nz;
    const long long waves = k.flat ? (ctx->N + 63) / 64 : rows * ((k.nx + 63) / 64);
    const bool few = waves <= lbm::kFewWaves, f64 = ctx->prec == Prec::F64;
    int most = lbm::step_max_threads(ctx->model, ctx->prec);
    int flat_most = lbm::flat_block_limit(ctx->Q, ctx->prec);
    int pack_most = use == kAdjoint ? lbm::kPackAdjMaxBlock : lbm::kPackMaxBlock;
    bool held = false;
    int least = 1;   // blocks where they are
    if (few) {
        most = flat_most = pack_most = 64;
    } else if (k.nt && use != kAdjoint) {
        held = true;
        if (ctx->Q >= 95 && !f64 && use == kStepsInPlace) {
            most = flat_most = pop_bytes(ctx) >= kHeldInPlace ? 128 : 256;
        } else if (ctx->Q >= 95 || (ctx->Q >= 33 && !f64 && use == kSteps)) {
            flat_most = most;
        } else {
            most = flat_most = 256;
            least = 2;
        }
    }
    k.rpb = 1;
    double cells;   // of a block, on average
    if (k.flat) {
        // the waves of a group, in blocks of equal size
        const int group = (k.rg * k.nx + 63) / 64;
        k.chunks = (group + flat_most / 64 - 1) / (flat_most / 64);
        k.bx = (group + k.chunks - 1) / k.chunks * 64;
        cells = static_cast<double>(k.nx) * k.ny / k.gpp / k.chunks;
    } else {
        // a held row that its blocks would leave a tenth short of lanes takes
        // larger ones, the first that do not, else those with the fewest lanes
        // (D3Q95 in place 192^3: 1115 us with 2 blocks of 128 a row, 1025 with one
        // of 192; 385x71x28 120 with 2 of 256, 106 with one of 448; 400x128x128 938
        // with 4 of 128, 925; D2Q33 400x8000 136, 128)
        const auto lanes = [&](int m) {
            const lbm::RowLaunch r = lbm::row_launch(k.nx, rows, m);
            return r.chunks * r.bx;
        };
        int fit = most;
        if (held) {
            const int limit = lbm::step_max_threads(ctx->model, ctx->prec);
            for (int m = most; m <= limit && 10LL * lanes(fit) > 11LL * k.nx; m += 64)
                if (lanes(m) < lanes(fit)) fit = m;
        }
        const lbm::RowLaunch rl = lbm::row_launch(k.nx, rows, fit);
        k.chunks = rl.chunks;
        k.bx = rl.bx;
        if (lbm::kPackRows && k.nx % 64 == 0) {
            // whole rows per block: waves stay inside one row (nx % 64 = 0) and
            // no block is partly empty (rpb divides the row count)
            const int maxb = std::min(most, pack_most);
            while (k.nx * k.rpb * 2 <= maxb && rows % (k.rpb * 2) == 0) k.rpb *= 2;
            if (k.rpb > 1) k.bx = k.nx * k.rpb;   // else: the row launch above (chunks >= 1)
        }
        cells = static_cast<double>(k.nx) * k.rpb / k.chunks;
    }
    // float64, two buffers: one of 400 cells does (D3Q19 400^2 x 100 211 us, two 219;
    // in place 200, 199; D3Q15 in place 159, 156)
    if (ctx->Q >= 19 && use == kSteps && cells >= 380) least = 1;
    const double hold =
        held ? std::max<double>(least, std::ceil(held_cells(ctx, use) / cells)) : 0.0;
    k.resident = hold <= lbm::kMaxHeld ? static_cast<int>(hold) : 0;
    k.resident_local = k.resident;
    if (ctx->Q >= 95 && use == kStepsInPlace) {
        const size_t bytes = pop_bytes(ctx);
        const bool off_lines = k.flat && k.ps % (lbm::kLineBytes / 8) != 0;
        const bool local = !f64      ? bytes >= kHeldInPlace
                           : k.flat ? off_lines
                                    : k.bx == 192 && 2 * bytes >= 3 * kHeldInPlace;
        if (!local) k.resident_local = 0;
    }
    set_divisors(k);
    // D3Q95 steps of so few waves that even four times as many leave the CUs two
    // each: four share the work of one (k_step_split; us per step float64 64x8x8
    // 7.3, 5.9; 512x4x4 (128 waves) 8.5, 7.7; 210x5x9 (153) 9.0, 9.8;
    // FP32-shifted 12^3 7.5, 5.6; 512x4x4 7.3, 6.2; 20^3 (140) 7.4, 8.1).
    k.split = few && ctx->Q >= 95 && use == kSteps &&
              lbm::step_blocks(ctx->model, ctx->prec, k) * 2 <= lbm::kCUs;
}

// Strips of a narrow 2D grid (k_steps_strip): steps per launch and strip width
// by the time they are expected to take on the GPU.  A launch costs `launch` us and
// `gather` for every 1000 cells its first step reads (of the difference between
// plans of one grid a quarter: their reads overlap in the caches), a step of a
// block `step` and `wave` for each wave that works in it; in strips along x the
// lanes of a wave lie in different rows, which costs the first load and the last
// store `lines` per wave and row.  Single steps take `one` and `cells` for every
// 1000 cells.  Fitted to 2700 plans of 53 grids of 150 to 38000 cells, 1 to 42
// across, timed behind a full queue: 7 % RMS.  A host that launches steps one by
// one adds to them (3.8 to 5.2 us a launch on the hosts measured), so strips are
// also taken where they promise up to 0.1 (FP32-shifted 0.2, along x 0.3) us more
// (130x14: single 3.9, from the host 4.8, strips 4.0); along rows that are not
// flat, where the fit is worst, they have to promise 0.3 less.  Held ends that lie
// across the lanes of a wave (strips along x) make single steps faster (300x12
// 3.9, strips 4.9).  All blocks run at once (one per CU, the strip's LDS).
// us per step behind a full queue, single and in the strips taken (steps of
// cells), float64 and FP32-shifted:
//   128x4         4.21, 2.91 (6 of 8)   4.29, 2.43 (6 of 8)
//   5x1500        3.95, 3.02 (6 of 8)   3.77, 2.70 (6 of 8)
//   11x800 held   5.02, 3.99 (4 of 4)   5.09, 3.55 (4 of 4)
//   300x12        3.90, 3.76 (5 of 4)   3.78, 3.57 (5 of 4)
//   600x10        4.40, 4.15 (5 of 4)   4.33, 3.67 (5 of 4)
//   16x2400       5.51, 5.23 (3 of 12)  4.62, 4.33 (3 of 12)
//   8x8192        6.96, 4.69 (5 of 32)  5.23, 3.97 (5 of 32)
//   20x800 held   5.08, 4.87 (3 of 4)   5.01, 4.00 (3 of 4)
//   25x800 held   5.31 (strips 5.08)    5.18, 4.49 (3 of 4)
//   40x900        5.50 (strips 5.83)    4.43 (strips 5.24)
//   256x20        4.30 (strips 5.80)    4.31 (strips 5.13)
void strip_plan(lbm_ctx* ctx) {
    KParams& k = ctx->kp;
    lbm::StripParams& sp = k.strip;
    k.steps = 1;
    sp = lbm::StripParams{};
    sp.steps = 1;
    if (ctx->D != 2 || ctx->aa) return;
    const bool f64 = ctx->prec == Prec::F64, held = k.hold_lo + k.hold_hi > 0;
    const double launch = f64 ? 2.4 : 1.6, gather = f64 ? 0.049 : 0.034, wave = f64 ? 0.20 : 0.14,
                 lines = f64 ? 0.023 : 0.028,
                 step = (f64 ? 1.80 : 1.87) + (held ? f64 ? 0.39 : 0.53 : 0.0);
    const int reach = lbm::model_reach(ctx->model);
    sp.along_y = k.ny >= k.nx;
    sp.n = sp.along_y ? k.ny : k.nx;
    sp.s = sp.along_y ? k.nx : k.ny;
    if (sp.s > lbm::kStripCells || (held && !sp.along_y)) return;
    const double cells = (f64 ? 0.036 : 0.014) + (k.flat ? 0.0 : f64 ? 0.04 : 0.01),
                 one = (f64 ? 3.8 : 3.75) + (held ? f64 ? 0.9 : 1.1 : 0.0) +
                       (k.flat ? 0.0 : f64 ? 0.2 : 0.45) + cells * ctx->N / 1000;
    const double more = !sp.along_y ? (k.flat ? 0.3 : -0.3) : f64 ? 0.1 : 0.2;
    const auto waves = [&](int len) { return (len * sp.s + 63) / 64; };
    double best = std::numeric_limits<double>::infinity(), taken = best;
    for (int steps = 7; steps >= 2; --steps) {
        for (int w = reach; w <= lbm::kStripCells; w += reach) {
            const int margin = reach * (steps - 1);
            const bool whole = w + 2 * margin >= sp.n;
            const int len = whole ? sp.n : w + 2 * margin;
            if (static_cast<long long>(len) * sp.s > lbm::kStripCells) break;
            const int blocks = whole ? 1 : (sp.n + w - 1) / w;
            if (blocks > lbm::kCUs) continue;
            const int lost = whole ? 0 : 2 * reach;   // cells along the strip, per step
            const double reads = gather * blocks * len * sp.s / 1000;
            double us = launch + step * steps + reads / 4;
            for (int t = 0; t < steps; ++t) us += wave * waves(len - lost * t);
            if (!sp.along_y) us += lines * sp.s * (waves(len) + waves(len - lost * (steps - 1)));
            if (us / steps < best) {
                best = us / steps;
                taken = (us + 0.75 * reads) / steps;
                sp.steps = steps;
                sp.w = whole ? sp.n : w;
                sp.threads = waves(len) * 64;
            }
            if (whole) break;
        }
    }
    if (!(taken < one + more)) sp.steps = 1;
    sp.by_s = fast_div(sp.s);
    sp.inv_s = 65536u / static_cast<unsigned>(sp.s) + 1;
    sp.inv_n = 65536u / static_cast<unsigned>(sp.n) + 1;
}

void fill_kparams(lbm_ctx* ctx) {
    KParams& k = ctx->kp;
    if (!ctx->initialized) k.form = initial_form(ctx);
    k.nx = static_cast<int>(ctx->extent[0]);
    k.ny = static_cast<int>(ctx->extent[1]);
    k.nz = ctx->D == 3 ? static_cast<int>(ctx->extent[2]) : 1;
    fill_layout(ctx, k);
    k.N = ctx->N;
    set_blocks(ctx, k, ctx->aa ? kStepsInPlace : kSteps);
    strip_plan(ctx);
    k.xcd_cyclic = ctx->mapping ? cyclic_chunk(k, ctx->D) : 0;
    k.omega = ctx->omega;
    k.omc = 1.0 - ctx->omega;
    if (ctx->prec == Prec::F32S) k.omc = static_cast<double>(static_cast<float>(k.omc));
    k.omega_eff = 1.0 - k.omc;
    k.T0 = ctx->T0;
    k.invT0 = 1.0 / ctx->T0;
    k.rho0 = ctx->prec == Prec::F32S ? ctx->rho0 : 0.0;
    for (int g = 0; g < lbm::kMaxG; ++g) {
        const bool on = g < ctx->G;
        k.W[g] = on ? ctx->W[g] : 0.0;
        k.X[g] = on ? lbm::model_e2(ctx->model, g) / ctx->T0 : 0.0;
    }
}

bool omega_ok(double omega) { return std::isfinite(omega) && omega >= 0.0 && omega < 2.0; }

int require_init(lbm_ctx* ctx) {
    if (!ctx) return fail(nullptr, LBM_E_INVALID, "context is NULL");
    if (!ctx->bound) return fail(ctx, LBM_E_STATE, "no buffers bound (call lbm_bind)");
    if (!ctx->initialized)
        return fail(ctx, LBM_E_STATE, "populations not initialised (call lbm_init_fields)");
    return LBM_OK;
}

int set_device(lbm_ctx* ctx) {
    hipError_t e = hipSetDevice(ctx->device);
    if (e != hipSuccess) return fail_hip(ctx, e, "hipSetDevice");
    return LBM_OK;
}

}  // namespace

LBM_API const char* lbm_status_str(int status) {
    switch (status) {
        case LBM_OK: return "ok";
        case LBM_E_INVALID: return "invalid argument";
        case LBM_E_UNSUPPORTED: return "unsupported model or precision";
        case LBM_E_DEVICE: return "HIP device error";
        case LBM_E_STATE: return "call out of order";
        case LBM_E_NONFINITE: return "non-finite result";
        default: return "unknown status";
    }
}

LBM_API const char* lbm_last_error(const lbm_ctx* ctx) {
    return ctx ? ctx->err.c_str() : g_err.c_str();
}

LBM_API int lbm_velocity_set(int D, int Q, int32_t* e, double* w, double* c) {
    ModelId m;
    if (!lbm::model_from_shape(D, Q, m))
        return fail(nullptr, LBM_E_UNSUPPORTED, "supported models: D=2,Q=33; D=3,Q=95; D=3,Q=19; D=3,Q=15");
    double W[lbm::kMaxG], cc;
    std::string err;
    if (!lbm::model_solve(m, W, &cc, err)) return fail(nullptr, LBM_E_INVALID, err);
    for (int i = 0; i < Q; ++i) {
        if (e)
            for (int k = 0; k < D; ++k) e[i * D + k] = lbm::model_e(m, i, k);
        if (w) w[i] = W[lbm::model_group_of(m, i)];
    }
    if (c) *c = cc;
    g_err.clear();
    return LBM_OK;
}

LBM_API int lbm_equation_count(int m, int D, int* count) {
    if (!count) return fail(nullptr, LBM_E_INVALID, "count is NULL");
    if (m < 0 || m > 16 || D < 1 || D > 8)
        return fail(nullptr, LBM_E_INVALID, "need 0 <= m <= 16 and 1 <= D <= 8");
    *count = lbm::equation_count(m, D);
    g_err.clear();
    return LBM_OK;
}

LBM_API int lbm_model_build(int D, int m, int G, const int32_t* reps, const double* w_guess,
                            double c_guess, int q_cap, int32_t* e, int32_t* group, double* w,
                            double* c, int* Q, double* residual) {
    if (D < 1 || D > 3) return fail(nullptr, LBM_E_UNSUPPORTED, "D must be 1, 2 or 3");
    if (m < 1 || m > 8 || G < 1 || !reps || !(c_guess > 0.0) || !std::isfinite(c_guess))
        return fail(nullptr, LBM_E_INVALID, "need 1 <= m <= 8, G >= 1, reps and c_guess > 0");
    if (w_guess)
        for (int g = 0; g < G; ++g)
            if (!std::isfinite(w_guess[g]))
                return fail(nullptr, LBM_E_INVALID, "w_guess has a non-finite value");
    lbm::BuiltModel bm;
    std::string err;
    if (!lbm::model_build(D, m, G, reps, w_guess, c_guess, bm, err))
        return fail(nullptr, LBM_E_INVALID, err);
    if (Q) *Q = bm.Q;
    for (int g = 0; g < G; ++g)
        if (!(bm.W[g] > 0.0))
            return fail(nullptr, LBM_E_INVALID,
                        "the solution has a non-positive weight (group " + std::to_string(g) + ")");
    if (!(bm.c > 0.0)) return fail(nullptr, LBM_E_INVALID, "the solution has c <= 0");
    if (bm.Q > q_cap)
        return fail(nullptr, LBM_E_INVALID,
                    "q_cap is smaller than the number of velocities " + std::to_string(bm.Q));
    for (int i = 0; i < bm.Q; ++i) {
        if (e)
            for (int k = 0; k < D; ++k) e[i * D + k] = bm.e[i][k];
        if (group) group[i] = bm.group[i];
        if (w) w[i] = bm.W[bm.group[i]];
    }
    if (c) *c = bm.c;
    if (residual) *residual = bm.residual;
    g_err.clear();
    return LBM_OK;
}

LBM_API int lbm_create(lbm_ctx** out, int D, int Q, const int32_t* e, const double* w,
                       double c, const int64_t* extent, double omega, int precision,
                       double rho0, void* stream) {
    if (!out) return fail(nullptr, LBM_E_INVALID, "out is NULL");
    *out = nullptr;
    if (!e || !w || !extent) return fail(nullptr, LBM_E_INVALID, "e, w and extent must be given");
    ModelId m;
    if (!lbm::model_from_shape(D, Q, m))
        return fail(nullptr, LBM_E_UNSUPPORTED, "supported models: D=2,Q=33; D=3,Q=95; D=3,Q=19; D=3,Q=15");
    if (!lbm::model_matches(m, e))
        return fail(nullptr, LBM_E_UNSUPPORTED,
                    "velocity list is not the canonical order of the model");
    if (precision != LBM_FP64 && precision != LBM_FP32_SHIFTED)
        return fail(nullptr, LBM_E_UNSUPPORTED, "precision must be LBM_FP64 or LBM_FP32_SHIFTED");
    const int G = lbm::model_groups(m);
    double W[lbm::kMaxG];
    int seen[lbm::kMaxG] = {};
    long double wsum = 0.0L;
    for (int i = 0; i < Q; ++i) {
        if (!std::isfinite(w[i]) || w[i] <= 0.0)
            return fail(nullptr, LBM_E_INVALID, "weights must be finite and positive");
        const int g = lbm::model_group_of(m, i);
        if (!seen[g]) {
            W[g] = w[i];
            seen[g] = 1;
        } else if (std::fabs(w[i] - W[g]) > 1e-14 * W[g]) {
            return fail(nullptr, LBM_E_INVALID, "weights differ inside a symmetry group");
        }
        wsum += w[i];
    }
    if (std::fabs(static_cast<double>(wsum) - 1.0) > 1e-12)
        return fail(nullptr, LBM_E_INVALID, "weights must sum to 1");
    if (!std::isfinite(c) || c <= 0.0) return fail(nullptr, LBM_E_INVALID, "c must be positive");
    const double res = lbm::model_residual(m, W, c);
    if (!(res <= 1e-10))
        return fail(nullptr, LBM_E_INVALID,
                    "weights and c do not solve the moment equations (residual " +
                        std::to_string(res) + ")");
    long long N = 1;
    for (int k = 0; k < D; ++k) {
        if (extent[k] < 1) return fail(nullptr, LBM_E_INVALID, "extents must be >= 1");
        if (extent[k] > (1LL << 24)) return fail(nullptr, LBM_E_INVALID, "extent too large");
        N *= extent[k];
        if (N >= (1LL << 31))
            return fail(nullptr, LBM_E_INVALID, "grid too large: at most 2^31 - 1 cells");
    }
    const long long rows = N / extent[0];
    const lbm::RowLaunch rl =
        lbm::row_launch(static_cast<int>(extent[0]), rows,
                        lbm::step_max_threads(m, precision == LBM_FP64 ? Prec::F64 : Prec::F32S));
    if (rl.blocks >= (1LL << 31) || rl.blocks * rl.bx >= (1LL << 32))
        return fail(nullptr, LBM_E_INVALID, "grid too large for one launch");
    // The kernels address one slab of the slowest axis (all populations of a
    // z-plane in 3D, of a row in 2D) with 32-bit byte offsets.
    const long long slab = run_stride_of(extent[0]) * (D == 3 ? extent[1] : 1) * Q *
                           (precision == LBM_FP64 ? 8LL : 4LL);
    if (slab >= (1LL << 32))
        return fail(nullptr, LBM_E_INVALID,
                    "grid too large: the populations of one slab (z-plane in 3D, row in 2D) "
                    "must stay below 4 GiB");
    if (!omega_ok(omega)) return fail(nullptr, LBM_E_INVALID, "omega must be in [0, 2)");
    if (precision == LBM_FP32_SHIFTED && (!std::isfinite(rho0) || rho0 < 0.0))
        return fail(nullptr, LBM_E_INVALID, "rho0 must be finite and >= 0");

    lbm_ctx* ctx = new (std::nothrow) lbm_ctx();
    if (!ctx) return fail(nullptr, LBM_E_INVALID, "out of host memory");
    ctx->model = m;
    ctx->prec = precision == LBM_FP64 ? Prec::F64 : Prec::F32S;
    ctx->D = D;
    ctx->Q = Q;
    ctx->G = G;
    for (int k = 0; k < D; ++k) ctx->extent[k] = extent[k];
    ctx->N = N;
    ctx->c = c;
    ctx->T0 = 1.0 / (2.0 * c * c);
    ctx->omega = omega;
    ctx->rho0 = rho0;
    for (int i = 0; i < Q; ++i) ctx->w[i] = w[i];
    for (int g = 0; g < G; ++g) ctx->W[g] = W[g];
    ctx->stream = static_cast<hipStream_t>(stream);
    fill_kparams(ctx);
    *out = ctx;
    g_err.clear();
    return LBM_OK;
}

LBM_API int lbm_workspace_bytes(const lbm_ctx* ctx, size_t* pop, size_t* scratch) {
    if (!ctx) return fail(nullptr, LBM_E_INVALID, "context is NULL");
    if (pop) *pop = pop_bytes(ctx);
    if (scratch) *scratch = scratch_bytes(ctx);
    return LBM_OK;
}

namespace {

void drop_graph(lbm_ctx* ctx) {
    if (ctx->graph_exec) (void)hipGraphExecDestroy(ctx->graph_exec);
    ctx->graph_exec = nullptr;
    ctx->graph_cur = ctx->graph_form = -1;
}

// Every second in-place step takes the cells backwards: the cache still holds
// what the step before it touched last, which a sweep in the same direction
// reaches only after evicting it (us per step, same direction against
// alternating: D2Q33 FP32-shifted 2048^2 (554 MB) 198, 167; 4096^2 772, 739; D3Q19
// 200^3 220, 195; D3Q95 128^3 284, 274).  States past 4 GB gain nothing (256^3
// FP32-shifted, 6.4 GB: 2322, 2337), nor do two buffers, where a step reads what
// the cache has not kept: it fills on reads (128^3 282, 282).
int reverse_step(const lbm_ctx* ctx) {
    return ctx->kp.form == lbm::kFormPushed && pop_bytes(ctx) <= (size_t{4} << 30);
}

// One update step on the context's stream (two-buffer or in place).
hipError_t launch_one_step(lbm_ctx* ctx) {
    if (ctx->aa) {
        const bool push = ctx->kp.form == lbm::kFormSwapped;
        ctx->kp.reverse = reverse_step(ctx);
        hipError_t e =
            lbm::launch_step_aa(ctx->model, ctx->prec, ctx->kp, ctx->f[0], push, nullptr,
                                ctx->stream);
        if (e == hipSuccess) ctx->kp.form = push ? lbm::kFormPushed : lbm::kFormSwapped;
        return e;
    }
    hipError_t e = lbm::launch_step(ctx->model, ctx->prec, ctx->kp, ctx->f[ctx->cur],
                                    ctx->f[1 - ctx->cur], nullptr, ctx->stream);
    if (e == hipSuccess) ctx->cur = 1 - ctx->cur;
    return e;
}

// n >= 3 steps in strips (kp.strip.steps a launch at most).  Every launch moves
// the state to the other buffer; their number has the parity of n, so that the
// state lies where n single steps leave it (a caller may replay an even number
// of captured steps).
int launch_strips(lbm_ctx* ctx, int n) {
    const int most = ctx->kp.strip.steps;
    int launches = (n + most - 1) / most;
    if ((launches ^ n) & 1) ++launches;
    for (int left = n; left > 0; --launches) {
        const int now = (left + launches - 1) / launches;   // as even as they come
        ctx->kp.steps = now;
        const hipError_t e = launch_one_step(ctx);
        ctx->kp.steps = 1;
        if (e != hipSuccess) return fail_hip(ctx, e, "step kernel");
        left -= now;
    }
    return LBM_OK;
}

// Captures graph_steps steps from the current launch state.  The state
// after an even number of steps equals the one before, so the graph can be
// replayed as long as that state is current.
int capture_graph(lbm_ctx* ctx) {
    drop_graph(ctx);
    const int cur0 = ctx->cur, form0 = ctx->kp.form;
    hipError_t e = hipStreamBeginCapture(ctx->stream, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) return fail_hip(ctx, e, "hipStreamBeginCapture");
    hipError_t le = hipSuccess;
    for (int t = 0; t < ctx->graph_steps && le == hipSuccess; ++t) le = launch_one_step(ctx);
    hipGraph_t g = nullptr;
    e = hipStreamEndCapture(ctx->stream, &g);
    ctx->cur = cur0;
    ctx->kp.form = form0;
    if (le != hipSuccess || e != hipSuccess) {
        if (g) (void)hipGraphDestroy(g);
        return fail_hip(ctx, le != hipSuccess ? le : e, "graph capture of the step");
    }
    e = hipGraphInstantiate(&ctx->graph_exec, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (e != hipSuccess) {
        ctx->graph_exec = nullptr;
        return fail_hip(ctx, e, "hipGraphInstantiate");
    }
    ctx->graph_cur = cur0;
    ctx->graph_form = form0;
    return LBM_OK;
}

}  // namespace

LBM_API int lbm_bind(lbm_ctx* ctx, void* f_a, void* f_b, void* scratch) {
    if (!ctx) return fail(nullptr, LBM_E_INVALID, "context is NULL");
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail_hip(ctx, e, "hipGetDevice");
    for (void* p : {f_a, f_b, scratch}) {
        if (p && reinterpret_cast<uintptr_t>(p) % kAlign != 0)
            return fail(ctx, LBM_E_INVALID, "buffers must be 256-byte aligned");
    }
    if (ctx->aa && f_b)
        return fail(ctx, LBM_E_INVALID, "in-place (AA) streaming uses one buffer: f_b must be NULL");
    const int saved = ctx->device;
    ctx->device = dev;
    int rc;
    if ((rc = check_dev(ctx, f_a, pop_bytes(ctx), "f_a")) != LBM_OK ||
        (!ctx->aa && (rc = check_dev(ctx, f_b, pop_bytes(ctx), "f_b")) != LBM_OK) ||
        (rc = check_dev(ctx, scratch, scratch_bytes(ctx), "scratch")) != LBM_OK) {
        ctx->device = saved;
        return rc;
    }
    if (!ctx->aa && f_a == f_b) {
        ctx->device = saved;
        return fail(ctx, LBM_E_INVALID, "f_a and f_b must be distinct buffers");
    }
    ctx->f[0] = f_a;
    ctx->f[1] = ctx->aa ? nullptr : f_b;
    ctx->cur = 0;
    ctx->scratch = scratch;
    ctx->bound = true;
    ctx->initialized = false;
    ctx->kp.form = initial_form(ctx);
    ctx->mapping = 0;   // a tuned block order belongs to the buffers it was measured on
    ctx->kp.xcd_cyclic = 0;
    drop_graph(ctx);
    ctx->err.clear();
    return LBM_OK;
}

LBM_API int lbm_init_fields(lbm_ctx* ctx, const double* rho, const double* U, const double* T) {
    if (!ctx) return fail(nullptr, LBM_E_INVALID, "context is NULL");
    if (!ctx->bound) return fail(ctx, LBM_E_STATE, "no buffers bound (call lbm_bind)");
    int rc;
    const size_t nb = static_cast<size_t>(ctx->N) * 8;
    if ((rc = check_dev(ctx, rho, nb, "rho")) != LBM_OK) return rc;
    if ((rc = check_dev(ctx, U, nb * ctx->D, "U")) != LBM_OK) return rc;
    if ((rc = check_dev(ctx, T, nb, "T")) != LBM_OK) return rc;
    if ((rc = set_device(ctx)) != LBM_OK) return rc;
    KParams kp = ctx->kp;
    kp.form = initial_form(ctx);
    hipError_t e = lbm::launch_init(ctx->model, ctx->prec, kp, rho, U, T, ctx->f[ctx->cur],
                                    ctx->stream);
    if (e != hipSuccess) return fail_hip(ctx, e, "init kernel");
    ctx->kp.form = kp.form;
    ctx->initialized = true;
    return LBM_OK;
}

LBM_API int lbm_set_populations(lbm_ctx* ctx, const double* f) {
    if (!ctx) return fail(nullptr, LBM_E_INVALID, "context is NULL");
    if (!ctx->bound) return fail(ctx, LBM_E_STATE, "no buffers bound (call lbm_bind)");
    int rc;
    if ((rc = check_dev(ctx, f, static_cast<size_t>(ctx->N) * ctx->Q * 8, "f")) != LBM_OK)
        return rc;
    if ((rc = set_device(ctx)) != LBM_OK) return rc;
    KParams kp = ctx->kp;
    kp.form = initial_form(ctx);
    hipError_t e = lbm::launch_set_pop(ctx->model, ctx->prec, kp, f, ctx->f[ctx->cur], ctx->stream);
    if (e != hipSuccess) return fail_hip(ctx, e, "set-populations kernel");
    ctx->kp.form = kp.form;
    ctx->initialized = true;
    return LBM_OK;
}

LBM_API int lbm_get_populations(lbm_ctx* ctx, double* f) {
    int rc;
    if ((rc = require_init(ctx)) != LBM_OK) return rc;
    if ((rc = check_dev(ctx, f, static_cast<size_t>(ctx->N) * ctx->Q * 8, "f")) != LBM_OK)
        return rc;
    if ((rc = set_device(ctx)) != LBM_OK) return rc;
    hipError_t e =
        lbm::launch_get_pop(ctx->model, ctx->prec, ctx->kp, ctx->f[ctx->cur], f, ctx->stream);
    if (e != hipSuccess) return fail_hip(ctx, e, "get-populations kernel");
    return LBM_OK;
}

LBM_API int lbm_step(lbm_ctx* ctx, int n) {
    int rc;
    if ((rc = require_init(ctx)) != LBM_OK) return rc;
    if (n < 0) return fail(ctx, LBM_E_INVALID, "n must be >= 0");
    if ((rc = set_device(ctx)) != LBM_OK) return rc;
    int left = n;
    if (ctx->graph_steps > 0) {
        while (left >= ctx->graph_steps) {
            if (!ctx->graph_exec || ctx->graph_cur != ctx->cur ||
                ctx->graph_form != ctx->kp.form) {
                if ((rc = capture_graph(ctx)) != LBM_OK) return rc;
            }
            hipError_t e = hipGraphLaunch(ctx->graph_exec, ctx->stream);
            if (e != hipSuccess) return fail_hip(ctx, e, "hipGraphLaunch");
            left -= ctx->graph_steps;
        }
    }
    if (ctx->kp.strip.steps > 1 && left > 2) {
        if ((rc = launch_strips(ctx, left)) != LBM_OK) return rc;
        left = 0;
    }
    for (; left > 0; --left) {
        hipError_t e = launch_one_step(ctx);
        if (e != hipSuccess) return fail_hip(ctx, e, ctx->aa ? "in-place step kernel" : "step kernel");
    }
    return LBM_OK;
}

LBM_API int lbm_tune_step(lbm_ctx* ctx, int n, int* mapping) {
    int rc;
    if ((rc = require_init(ctx)) != LBM_OK) return rc;
    if (n < 0) return fail(ctx, LBM_E_INVALID, "n must be >= 0");
    if ((rc = set_device(ctx)) != LBM_OK) return rc;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (ctx->stream) {
        const hipError_t e = hipStreamIsCapturing(ctx->stream, &cap);
        if (e != hipSuccess) return fail_hip(ctx, e, "hipStreamIsCapturing");
    }
    // In place the steps alternate between two kernels (push, local), so the
    // orders alternate per pair of steps there.
    const int unit = ctx->aa ? 2 : 1;
    if (n < 4 * unit || cap != hipStreamCaptureStatusNone) {
        if ((rc = lbm_step(ctx, n)) != LBM_OK) return rc;
        if (mapping) *mapping = ctx->mapping;
        return LBM_OK;
    }
    // n single steps, the two block orders alternating (per step, or per pair
    // in place), each step between two events
    std::vector<hipEvent_t> ev(static_cast<size_t>(n) + 1, nullptr);
    const auto release = [&]() {
        for (hipEvent_t x : ev)
            if (x) (void)hipEventDestroy(x);
    };
    hipError_t e = hipSuccess;
    for (size_t t = 0; t < ev.size() && e == hipSuccess; ++t) e = hipEventCreate(&ev[t]);
    if (e != hipSuccess) {
        release();
        return fail_hip(ctx, e, "hipEventCreate");
    }
    drop_graph(ctx);
    const int chunk = cyclic_chunk(ctx->kp, ctx->D);
    e = hipEventRecord(ev[0], ctx->stream);
    for (int t = 0; t < n && e == hipSuccess; ++t) {
        ctx->kp.xcd_cyclic = ((t / unit) % 2) ? chunk : 0;
        e = launch_one_step(ctx);
        if (e == hipSuccess) e = hipEventRecord(ev[t + 1], ctx->stream);
    }
    if (e == hipSuccess) e = hipEventSynchronize(ev[n]);
    // mean time of each order, leaving out the first step (pair) of each as
    // warm-up when there are enough
    double sum[2] = {0.0, 0.0};
    int cnt[2] = {0, 0};
    for (int t = (n >= 6 * unit ? 2 * unit : 0); t < n && e == hipSuccess; ++t) {
        float ms = 0.0f;
        e = hipEventElapsedTime(&ms, ev[t], ev[t + 1]);
        sum[(t / unit) % 2] += ms;
        ++cnt[(t / unit) % 2];
    }
    release();
    if (e != hipSuccess) {
        ctx->kp.xcd_cyclic = ctx->mapping ? chunk : 0;
        return fail_hip(ctx, e, "tuning steps");
    }
    if (cnt[0] > 0 && cnt[1] > 0) ctx->mapping = (sum[1] * cnt[0] < sum[0] * cnt[1]) ? 1 : 0;
    ctx->kp.xcd_cyclic = ctx->mapping ? chunk : 0;
    if (mapping) *mapping = ctx->mapping;
    return LBM_OK;
}

LBM_API int lbm_set_block_order(lbm_ctx* ctx, int order) {
    if (!ctx) return fail(nullptr, LBM_E_INVALID, "context is NULL");
    if (order != 0 && order != 1) return fail(ctx, LBM_E_INVALID, "order must be 0 or 1");
    drop_graph(ctx);
    ctx->mapping = order;
    ctx->kp.xcd_cyclic = order ? cyclic_chunk(ctx->kp, ctx->D) : 0;
    return LBM_OK;
}

LBM_API int lbm_set_graph_steps(lbm_ctx* ctx, int steps) {
    if (!ctx) return fail(nullptr, LBM_E_INVALID, "context is NULL");
    if (steps < 0 || steps % 2 != 0)
        return fail(ctx, LBM_E_INVALID, "steps must be an even number >= 0");
    if (steps > 0 && !ctx->stream)
        return fail(ctx, LBM_E_UNSUPPORTED, "graph replay needs a stream other than the null stream");
    drop_graph(ctx);
    ctx->graph_steps = steps;
    return LBM_OK;
}

LBM_API int lbm_set_fixed_planes(lbm_ctx* ctx, int n_lo, int n_hi, const double* state_lo,
                                 const double* state_hi) {
    if (!ctx) return fail(nullptr, LBM_E_INVALID, "context is NULL");
    const int64_t L = ctx->extent[ctx->D - 1];
    if (n_lo < 0 || n_hi < 0 || static_cast<int64_t>(n_lo) + n_hi > L)
        return fail(ctx, LBM_E_INVALID, "need n_lo, n_hi >= 0 and n_lo + n_hi <= extent[D-1]");
    const double* st[2] = {state_lo, state_hi};
    const int cnt[2] = {n_lo, n_hi};
    lbm::FixedState fs[2]{};
    for (int s = 0; s < 2; ++s) {
        if (cnt[s] == 0) continue;
        if (!st[s]) return fail(ctx, LBM_E_INVALID, "state of a held end is NULL");
        for (int j = 0; j < ctx->D + 2; ++j)
            if (!std::isfinite(st[s][j]))
                return fail(ctx, LBM_E_NONFINITE, "held state has a non-finite value");
        if (!(st[s][0] > 0.0) || !(st[s][ctx->D + 1] > 0.0))
            return fail(ctx, LBM_E_INVALID, "held state needs rho > 0 and T > 0");
        fs[s].rho = st[s][0];
        for (int a = 0; a < ctx->D; ++a) fs[s].U[a] = st[s][1 + a];
        fs[s].T = st[s][ctx->D + 1];
    }
    ctx->hold_lo = n_lo;
    ctx->hold_hi = n_hi;
    ctx->hold[0] = fs[0];
    ctx->hold[1] = fs[1];
    ctx->kp.hold_lo = n_lo;
    ctx->kp.hold_hi = n_hi;
    ctx->kp.hold[0] = fs[0];
    ctx->kp.hold[1] = fs[1];
    strip_plan(ctx);
    drop_graph(ctx);
    return LBM_OK;
}

LBM_API int lbm_moments(lbm_ctx* ctx, double* rho, double* U, double* T) {
    int rc;
    if ((rc = require_init(ctx)) != LBM_OK) return rc;
    const size_t nb = static_cast<size_t>(ctx->N) * 8;
    if (rho && (rc = check_dev(ctx, rho, nb, "rho")) != LBM_OK) return rc;
    if (U && (rc = check_dev(ctx, U, nb * ctx->D, "U")) != LBM_OK) return rc;
    if (T && (rc = check_dev(ctx, T, nb, "T")) != LBM_OK) return rc;
    if (!rho && !U && !T) return LBM_OK;
    if ((rc = set_device(ctx)) != LBM_OK) return rc;
    hipError_t e = lbm::launch_moments(ctx->model, ctx->prec, ctx->kp, ctx->f[ctx->cur], rho, U,
                                       T, ctx->stream);
    if (e != hipSuccess) return fail_hip(ctx, e, "moments kernel");
    return LBM_OK;
}

namespace {

// The conservation sums with the reduction partials at `scratch` (room for
// reduce_blocks(N) * (D + 2) partials, rounded up to 256 bytes, then D + 2
// results).  The caller has checked the context and made its device current.
int conservation_into(lbm_ctx* ctx, void* scratch, double* out) {
    const int K = ctx->D + 2;
    double* partials = static_cast<double*>(scratch);
    const size_t parts = round_up(static_cast<size_t>(lbm::reduce_blocks(ctx->N)) * K * 8);
    double* dres = reinterpret_cast<double*>(static_cast<char*>(scratch) + parts);
    hipError_t e = lbm::launch_conservation(ctx->model, ctx->prec, ctx->kp, ctx->f[ctx->cur],
                                            partials, dres, ctx->stream);
    if (e != hipSuccess) return fail_hip(ctx, e, "conservation kernels");
    double host[5] = {0, 0, 0, 0, 0};
    e = hipMemcpyAsync(host, dres, K * sizeof(double), hipMemcpyDeviceToHost, ctx->stream);
    if (e != hipSuccess) return fail_hip(ctx, e, "copy of conservation sums");
    e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) return fail_hip(ctx, e, "stream synchronisation");
    if (ctx->prec == Prec::F32S) {
        // add the shift: sum over cells of w_i rho0 (and its moments)
        long double m = 0, j[3] = {0, 0, 0}, en = 0;
        for (int i = 0; i < ctx->Q; ++i) {
            long double e2 = 0;
            for (int k = 0; k < ctx->D; ++k) {
                const int ek = lbm::model_e(ctx->model, i, k);
                j[k] += static_cast<long double>(ctx->w[i]) * ek;
                e2 += static_cast<long double>(ek) * ek;
            }
            m += ctx->w[i];
            en += 0.5L * ctx->w[i] * e2;
        }
        const long double scale = static_cast<long double>(ctx->N) * ctx->rho0;
        host[0] += static_cast<double>(scale * m);
        for (int k = 0; k < ctx->D; ++k) host[1 + k] += static_cast<double>(scale * j[k]);
        host[K - 1] += static_cast<double>(scale * en);
    }
    bool finite = true;
    for (int k = 0; k < K; ++k) {
        out[k] = host[k];
        finite = finite && std::isfinite(host[k]);
    }
    if (!finite) return fail(ctx, LBM_E_NONFINITE, "a conservation sum is not finite");
    return LBM_OK;
}

}  // namespace

LBM_API int lbm_conservation(lbm_ctx* ctx, double* out) {
    int rc;
    if ((rc = require_init(ctx)) != LBM_OK) return rc;
    if (!out) return fail(ctx, LBM_E_INVALID, "out is NULL");
    if ((rc = set_device(ctx)) != LBM_OK) return rc;
    return conservation_into(ctx, ctx->scratch, out);
}

LBM_API int lbm_conservation_noalloc(lbm_ctx* ctx, double* out) {
    int rc;
    if ((rc = require_init(ctx)) != LBM_OK) return rc;
    if (!out) return fail(ctx, LBM_E_INVALID, "out is NULL");
    if ((rc = set_device(ctx)) != LBM_OK) return rc;
    void* scratch = nullptr;
    size_t cap = 0;
    hipError_t e = lbm::static_scratch(ctx->device, &scratch, &cap);
    if (e != hipSuccess) return fail_hip(ctx, e, "address of the static scratch array");
    const size_t need = scratch_bytes(ctx);
    if (need > cap)
        return fail(ctx, LBM_E_INVALID,
                    "the grid needs " + std::to_string(need) +
                        " bytes of reduction scratch, the static array holds " +
                        std::to_string(cap));
    return conservation_into(ctx, scratch, out);
}

LBM_API int lbm_stream_copy(lbm_ctx* ctx, int n) {
    int rc;
    if ((rc = require_init(ctx)) != LBM_OK) return rc;
    if (n < 0) return fail(ctx, LBM_E_INVALID, "n must be >= 0");
    if (ctx->aa)
        return fail(ctx, LBM_E_UNSUPPORTED, "the copy needs the two buffers of LBM_STREAM_AB");
    if ((rc = set_device(ctx)) != LBM_OK) return rc;
    const size_t bytes = pop_bytes(ctx);
    for (int r = 0; r < n; ++r) {
        const hipError_t e = lbm::launch_stream_copy(ctx->f[ctx->cur], ctx->f[1 - ctx->cur], bytes,
                                                     ctx->stream);
        if (e != hipSuccess) return fail_hip(ctx, e, "copy kernel");
    }
    return LBM_OK;
}

LBM_API int lbm_set_streaming(lbm_ctx* ctx, int scheme) {
    if (!ctx) return fail(nullptr, LBM_E_INVALID, "context is NULL");
    if (scheme != LBM_STREAM_AB && scheme != LBM_STREAM_AA)
        return fail(ctx, LBM_E_INVALID, "scheme must be LBM_STREAM_AB or LBM_STREAM_AA");
    if (ctx->bound) return fail(ctx, LBM_E_STATE, "choose the streaming scheme before lbm_bind");
    ctx->aa = scheme == LBM_STREAM_AA;
    fill_kparams(ctx);
    ctx->kp.form = initial_form(ctx);
    return LBM_OK;
}

LBM_API int lbm_set_omega(lbm_ctx* ctx, double omega) {
    if (!ctx) return fail(nullptr, LBM_E_INVALID, "context is NULL");
    if (!omega_ok(omega)) return fail(ctx, LBM_E_INVALID, "omega must be in [0, 2)");
    ctx->omega = omega;
    fill_kparams(ctx);
    drop_graph(ctx);
    return LBM_OK;
}

namespace {

// Checkpoint buffer of an n-step run with a snapshot every k steps whose
// last `keep` segments keep their step moments:
//   [snapshot s at t = s k, s = 0 .. segs-1][final state f*(n)]
//   [moments of every step t >= t_keep = (segs - keep) k, one (D+2)-plane
//    block per step]
// The adjoint recomputes only the segments before t_keep.
struct CkLayout {
    size_t stride, off_final, off_tail, mom_step, total;
    int segs, keep, t_keep;
};

CkLayout ck_layout(const lbm_ctx* ctx, int n, int k, int keep) {
    CkLayout c;
    c.stride = round_up(pop_bytes(ctx));
    c.segs = (n + k - 1) / k;
    c.keep = std::min(std::max(keep, 1), c.segs);
    c.t_keep = (c.segs - c.keep) * k;
    c.mom_step = round_up(static_cast<size_t>(ctx->N) * (ctx->D + 2) * elem_bytes(ctx->prec));
    c.off_final = static_cast<size_t>(c.segs) * c.stride;
    c.off_tail = c.off_final + c.stride;
    c.total = c.off_tail + static_cast<size_t>(n - c.t_keep) * c.mom_step;
    return c;
}

}  // namespace

LBM_API int lbm_checkpoint_bytes(const lbm_ctx* ctx, int n, int k, int keep, size_t* bytes) {
    if (!ctx) return fail(nullptr, LBM_E_INVALID, "context is NULL");
    if (n < 1 || k < 1 || keep < 1 || !bytes)
        return fail(nullptr, LBM_E_INVALID, "need n >= 1, k >= 1, keep >= 1");
    *bytes = ck_layout(ctx, n, k, keep).total;
    return LBM_OK;
}

LBM_API int lbm_run_checkpointed(lbm_ctx* ctx, int n, int k, int keep, void* ckpt,
                                 size_t ckpt_bytes) {
    int rc;
    if ((rc = require_init(ctx)) != LBM_OK) return rc;
    if (n < 1 || k < 1 || keep < 1) return fail(ctx, LBM_E_INVALID, "need n >= 1, k >= 1, keep >= 1");
    const CkLayout c = ck_layout(ctx, n, k, keep);
    if (ckpt_bytes < c.total) return fail(ctx, LBM_E_INVALID, "checkpoint buffer too small");
    if ((rc = check_dev(ctx, ckpt, c.total, "ckpt")) != LBM_OK) return rc;
    if ((rc = set_device(ctx)) != LBM_OK) return rc;
    const size_t pb = pop_bytes(ctx);
    char* ck = static_cast<char*>(ckpt);
    if (ctx->aa) {
        // In place: the state stays in the bound buffer; snapshot 0, each
        // later snapshot and the final state are copied out of it in the
        // two-buffer form, so the adjoint reads the same checkpoints.
        hipError_t e = lbm::launch_to_ab(ctx->model, ctx->prec, ctx->kp, ctx->f[0], ck, ctx->stream);
        if (e != hipSuccess) return fail_hip(ctx, e, "checkpoint copy kernel");
        for (int t = 0; t < n; ++t) {
            void* mom = (t >= c.t_keep) ? ck + c.off_tail + (t - c.t_keep) * c.mom_step : nullptr;
            const bool push = ctx->kp.form == lbm::kFormSwapped;
            ctx->kp.reverse = reverse_step(ctx);
            e = lbm::launch_step_aa(ctx->model, ctx->prec, ctx->kp, ctx->f[0], push, mom,
                                    ctx->stream);
            if (e != hipSuccess) return fail_hip(ctx, e, "in-place step kernel");
            ctx->kp.form = push ? lbm::kFormPushed : lbm::kFormSwapped;
            char* slot = nullptr;
            if (t + 1 == n) slot = ck + c.off_final;
            else if ((t + 1) % k == 0) slot = ck + ((t + 1) / k) * c.stride;
            if (slot) {
                e = lbm::launch_to_ab(ctx->model, ctx->prec, ctx->kp, ctx->f[0], slot, ctx->stream);
                if (e != hipSuccess) return fail_hip(ctx, e, "checkpoint copy kernel");
            }
        }
        return LBM_OK;
    }
    // Snapshot 0 is a copy (the adjoint recomputes segment 0 from it, or
    // measures its invariant there); every later snapshot is written directly
    // by the step that ends the previous segment, and the next step reads it
    // there.
    hipError_t e = hipMemcpyAsync(ck, ctx->f[ctx->cur], pb, hipMemcpyDeviceToDevice, ctx->stream);
    if (e != hipSuccess) return fail_hip(ctx, e, "checkpoint copy");
    const void* src = ctx->f[ctx->cur];
    for (int t = 0; t < n; ++t) {
        const bool to_slot = ((t + 1) % k == 0) && (t + 1 < n);
        void* dst = to_slot ? ck + ((t + 1) / k) * c.stride
                            : (src == ctx->f[0] ? ctx->f[1] : ctx->f[0]);
        void* mom = (t >= c.t_keep) ? ck + c.off_tail + (t - c.t_keep) * c.mom_step : nullptr;
        e = lbm::launch_step(ctx->model, ctx->prec, ctx->kp, src, dst, mom, ctx->stream);
        if (e != hipSuccess) return fail_hip(ctx, e, "step kernel");
        src = dst;
    }
    // the final state is in one of the context's buffers (t + 1 = n never goes to a slot)
    ctx->cur = (src == ctx->f[0]) ? 0 : 1;
    e = hipMemcpyAsync(ck + c.off_final, src, pb, hipMemcpyDeviceToDevice, ctx->stream);
    if (e != hipSuccess) return fail_hip(ctx, e, "checkpoint copy");
    return LBM_OK;
}

LBM_API int lbm_restore_checkpoint(lbm_ctx* ctx, int n, int k, int keep, const void* ckpt,
                                   size_t ckpt_bytes, int slot) {
    if (!ctx) return fail(nullptr, LBM_E_INVALID, "context is NULL");
    if (!ctx->bound) return fail(ctx, LBM_E_STATE, "no buffers bound (call lbm_bind)");
    if (n < 1 || k < 1 || keep < 1) return fail(ctx, LBM_E_INVALID, "need n >= 1, k >= 1, keep >= 1");
    const CkLayout c = ck_layout(ctx, n, k, keep);
    if (slot < 0 || slot > c.segs)
        return fail(ctx, LBM_E_INVALID, "slot must be in [0, ceil(n/k)] (the last: final state)");
    if (ckpt_bytes < c.total) return fail(ctx, LBM_E_INVALID, "checkpoint buffer too small");
    int rc;
    if ((rc = check_dev(ctx, ckpt, c.total, "ckpt")) != LBM_OK) return rc;
    if ((rc = set_device(ctx)) != LBM_OK) return rc;
    const char* src = static_cast<const char*>(ckpt) +
                      (slot == c.segs ? c.off_final : static_cast<size_t>(slot) * c.stride);
    KParams kp = ctx->kp;
    kp.form = initial_form(ctx);
    hipError_t e =
        ctx->aa ? lbm::launch_from_ab(ctx->model, ctx->prec, kp, src, ctx->f[0], ctx->stream)
                : hipMemcpyAsync(ctx->f[ctx->cur], src, pop_bytes(ctx), hipMemcpyDeviceToDevice,
                                 ctx->stream);
    if (e != hipSuccess) return fail_hip(ctx, e, "checkpoint restore");
    ctx->kp.form = kp.form;
    ctx->initialized = true;
    return LBM_OK;
}

namespace {

// Launch parameters of the adjoint's kernels: the two-buffer form whatever
// scheme the forward run used.
KParams adjoint_params(const lbm_ctx* ctx, BlockUse use) {
    KParams k = ctx->kp;
    k.form = lbm::kFormAB;
    k.reverse = 0;
    set_blocks(ctx, k, use);
    k.xcd_cyclic = ctx->mapping ? cyclic_chunk(k, ctx->D) : 0;
    return k;
}

// Adjoint workspace: [three adjoint-state buffers][moments of one recomputed
// segment][partials of A][partials of K(n)][partials of one invariant mark]
// [A, K(n), one invariant mark per segment].
struct AdjLayout {
    size_t pop;       // stride of one population-sized buffer
    size_t mom_step;  // bytes of one step of stored moments
    size_t off_mom, off_partA, off_partK, off_partM, off_out, total;
    long long nA, nK;
};

AdjLayout adj_layout(const lbm_ctx* ctx, int k, int segs, bool recompute) {
    AdjLayout L;
    L.pop = round_up(pop_bytes(ctx));
    L.mom_step = round_up(static_cast<size_t>(ctx->N) * (ctx->D + 2) * elem_bytes(ctx->prec));
    L.off_mom = 3 * L.pop;
    L.nA = lbm::step_blocks(ctx->model, ctx->prec, adjoint_params(ctx, kAdjoint));
    L.nK = (ctx->N + 255) / 256;
    L.off_partA = L.off_mom + (recompute ? static_cast<size_t>(k) * L.mom_step : 0);
    L.off_partK = L.off_partA + round_up(static_cast<size_t>(L.nA) * 8);
    L.off_partM = L.off_partK + round_up(static_cast<size_t>(L.nK) * 8);
    L.off_out = L.off_partM + round_up(static_cast<size_t>(L.nA) * 8);
    L.total = L.off_out + round_up(static_cast<size_t>(2 + segs) * 8);
    return L;
}

}  // namespace

LBM_API int lbm_adjoint_workspace_bytes(const lbm_ctx* ctx, int n, int k, int keep,
                                        size_t* bytes) {
    if (!ctx) return fail(nullptr, LBM_E_INVALID, "context is NULL");
    if (n < 1 || k < 1 || keep < 1 || !bytes)
        return fail(nullptr, LBM_E_INVALID, "need n >= 1, k >= 1, keep >= 1");
    const CkLayout C = ck_layout(ctx, n, k, keep);
    *bytes = adj_layout(ctx, k, C.segs, C.t_keep > 0).total;
    return LBM_OK;
}

LBM_API int lbm_adjoint(lbm_ctx* ctx, int n, int k, int keep, const void* ckpt,
                        size_t ckpt_bytes,
                        const double* rho_init, const double* U_init, const double* T_init,
                        const double* dL_drho_final, void* workspace, size_t ws_bytes,
                        double* dL_dT_init, double* dL_domega) {
    int rc;
    if (!ctx) return fail(nullptr, LBM_E_INVALID, "context is NULL");
    if (!ctx->bound) return fail(ctx, LBM_E_STATE, "no buffers bound (call lbm_bind)");
    if (n < 1 || k < 1 || keep < 1)
        return fail(ctx, LBM_E_INVALID, "need n >= 1, k >= 1, keep >= 1");
    if (dL_domega && ctx->hold_lo + ctx->hold_hi > 0)
        return fail(ctx, LBM_E_UNSUPPORTED, "the omega gradient needs an all-periodic lattice "
                                            "(fixed planes are set); the temperature gradient "
                                            "does not");
    if (dL_domega && std::fabs(1.0 - ctx->omega) < 1e-3)
        return fail(ctx, LBM_E_INVALID,
                    "the omega gradient needs |1 - omega| >= 1e-3 (it is divided by 1 - omega)");
    const CkLayout C = ck_layout(ctx, n, k, keep);
    const size_t need_ck = C.total;
    if (ckpt_bytes < need_ck) return fail(ctx, LBM_E_INVALID, "checkpoint buffer too small");
    const AdjLayout L = adj_layout(ctx, k, C.segs, C.t_keep > 0);
    if (ws_bytes < L.total) return fail(ctx, LBM_E_INVALID, "adjoint workspace too small");
    const size_t nb = static_cast<size_t>(ctx->N) * 8;
    if ((rc = check_dev(ctx, ckpt, need_ck, "ckpt")) != LBM_OK) return rc;
    if ((rc = check_dev(ctx, workspace, L.total, "workspace")) != LBM_OK) return rc;
    if ((rc = check_dev(ctx, dL_drho_final, nb, "dL_drho_final")) != LBM_OK) return rc;
    if (dL_dT_init) {
        if ((rc = check_dev(ctx, dL_dT_init, nb, "dL_dT_init")) != LBM_OK) return rc;
        if ((rc = check_dev(ctx, rho_init, nb, "rho_init")) != LBM_OK) return rc;
        if ((rc = check_dev(ctx, U_init, nb * ctx->D, "U_init")) != LBM_OK) return rc;
        if ((rc = check_dev(ctx, T_init, nb, "T_init")) != LBM_OK) return rc;
    }
    if (reinterpret_cast<uintptr_t>(workspace) % kAlign != 0)
        return fail(ctx, LBM_E_INVALID, "workspace must be 256-byte aligned");
    if ((rc = set_device(ctx)) != LBM_OK) return rc;

    const lbm::KParams kab = adjoint_params(ctx, kAdjoint);
    const lbm::KParams kstep = adjoint_params(ctx, kSteps);   // recomputed steps
    char* ws = static_cast<char*>(workspace);
    void* B[3] = {ws, ws + L.pop, ws + 2 * L.pop};
    char* mom = ws + L.off_mom;
    double* partA = reinterpret_cast<double*>(ws + L.off_partA);
    double* partK = reinterpret_cast<double*>(ws + L.off_partK);
    double* partM = reinterpret_cast<double*>(ws + L.off_partM);
    double* dout = reinterpret_cast<double*>(ws + L.off_out);
    const size_t ck_stride = C.stride;
    const char* ck = static_cast<const char*>(ckpt);
    hipStream_t st = ctx->stream;
    hipError_t e = lbm::launch_fill_zero(partA, L.nA, st);
    if (e != hipSuccess) return fail_hip(ctx, e, "fill kernel");

    // The kernels advance the stored (post-collision) state B as
    // B^{t+1} = C(S B^t); the moments of S B^t are those of time t+1, and the
    // recomputation of segment s stores them in slot j for t = t0 + j + 1.
    // Adjoint: nu^n = dL/drho_n (broadcast over i), then for t = n-1 .. 1
    // nu^t = C'(m^t)^T S^T nu^{t+1}, and finally dL/dB^0 = S^T nu^1.
    const int segs = (n + k - 1) / k;
    int lam = -1;   // index of the buffer holding the current adjoint state
    for (int s = segs - 1; s >= 0; --s) {
        const int t0 = s * k;
        const int len = std::min(k, n - t0);
        int fr[2], nf = 0;
        for (int b = 0; b < 3 && nf < 2; ++b)
            if (b != lam) fr[nf++] = b;
        const char* segmom = mom;
        if (lam < 0) {
            // start from f*(n), kept by the forward run
            lam = fr[0];
            e = lbm::launch_lambda_init(ctx->model, ctx->prec, kab, ck + C.off_final,
                                        dL_drho_final, B[lam], partK, st);
            if (e != hipSuccess) return fail_hip(ctx, e, "adjoint initialisation kernel");
            fr[0] = 2;   // the free pair is now {1, 2}
        }
        if (t0 >= C.t_keep) {
            // the forward run kept this segment's moments
            segmom = ck + C.off_tail + static_cast<size_t>(t0 - C.t_keep) * C.mom_step;
        } else {
            // recompute the segment from its checkpoint (read in place),
            // storing the moments of every step; the last step stores its
            // moments only (its state is snapshot s + 1, which nothing here
            // reads again)
            const void* src = ck + s * ck_stride;
            int dst = fr[0];
            for (int j = 0; j < len; ++j) {
                e = lbm::launch_step(ctx->model, ctx->prec, kstep, src,
                                     j + 1 < len ? B[dst] : nullptr, mom + j * L.mom_step, st);
                if (e != hipSuccess) return fail_hip(ctx, e, "recompute step kernel");
                src = B[dst];
                dst = (dst == fr[0]) ? fr[1] : fr[0];
            }
        }
        const int t_hi = std::min(t0 + len, n - 1);
        for (int t = t_hi; t >= t0 + 1; --t) {
            const int nxt = (lam == fr[0]) ? fr[1] : fr[0];
            // Below the last segment, the first step (t = (s+1) k) gathers
            // S^T nu^{t+1} while snapshot s+1 holds B^t: it also measures the
            // invariant mark K(t+1) = <nu^{t+1}, S B^t> of snapshot s+1.
            const bool mark = dL_domega && t == t_hi && s + 1 < segs;
            e = lbm::launch_adjoint_step(ctx->model, ctx->prec, kab, B[lam], B[nxt],
                                         segmom + (t - t0 - 1) * L.mom_step, partA,
                                         mark ? ck + (s + 1) * ck_stride : nullptr, partM, st);
            if (e == hipSuccess && mark)
                e = lbm::launch_sum_partials(partM, L.nA, 1, 1, dout + 2 + s + 1, st);
            if (e != hipSuccess) return fail_hip(ctx, e, "adjoint step kernel");
            lam = nxt;
        }
    }
    {
        // dL/dB^0 = S^T nu^1; mark K(1) = <nu^1, S B^0> against snapshot 0
        const int nxt = (lam == 0) ? 1 : 0;
        e = lbm::launch_adjoint_step(ctx->model, ctx->prec, kab, B[lam], B[nxt], nullptr,
                                     nullptr, dL_domega ? ck : nullptr, partM, st);
        if (e == hipSuccess && dL_domega)
            e = lbm::launch_sum_partials(partM, L.nA, 1, 1, dout + 2, st);
        if (e != hipSuccess) return fail_hip(ctx, e, "transposed streaming kernel");
        lam = nxt;
    }
    if (dL_dT_init) {
        e = lbm::launch_dT_init(ctx->model, ctx->prec, kab, B[lam], rho_init, U_init, T_init,
                                dL_dT_init, st);
        if (e != hipSuccess) return fail_hip(ctx, e, "temperature gradient kernel");
    }
    if (dL_domega) {
        e = lbm::launch_sum_partials(partA, L.nA, 1, 1, dout, st);
        if (e == hipSuccess) e = lbm::launch_sum_partials(partK, L.nK, 1, 1, dout + 1, st);
        if (e != hipSuccess) return fail_hip(ctx, e, "reduction kernel");
        std::vector<double> h(2 + segs, 0.0);
        e = hipMemcpyAsync(h.data(), dout, h.size() * sizeof(double), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) return fail_hip(ctx, e, "copy of the omega gradient");
        // dL/domega = sum_{t=1}^{n-1} (A^t - K(t+1)) / (1 - omega) with
        // A^t = <S^T nu^{t+1}, f^eq(m^t)> and K(tau) = <nu^tau, f^tau>.  K is
        // the same at every tau in exact arithmetic; the stored adjoint state
        // is rounded at every step, so K is measured at tau = s k + 1 (one
        // mark per segment) and at tau = n, and summed as the piecewise linear
        // interpolant through those marks.
        double sum_k = 0.0;
        for (int s = 0; s < segs; ++s) {
            const long long a = static_cast<long long>(s) * k + 1;
            const long long b = (s + 1 < segs) ? a + k : n;
            const double ka = h[2 + s];
            const double kb = (s + 1 < segs) ? h[2 + s + 1] : h[1];
            const double d = static_cast<double>(b - a);
            if (b > a) sum_k += d * ka + 0.5 * (kb - ka) * (d + 1.0);
        }
        *dL_domega = (h[0] - sum_k) / (1.0 - ctx->omega);
        if (!std::isfinite(*dL_domega))
            return fail(ctx, LBM_E_NONFINITE, "omega gradient is not finite");
    }
    return LBM_OK;
}

LBM_API int lbm_destroy(lbm_ctx* ctx) {
    if (ctx) drop_graph(ctx);
    delete ctx;
    return LBM_OK;
}

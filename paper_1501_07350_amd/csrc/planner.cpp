// planner.cpp -- kernel registry lookup, heuristic plan, candidate plans for
// tuning, plan strings, and the [M1][L][M2] pass descriptors of a plan.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <sstream>
#include <tuple>

#include "offt_internal.h"
#include "../../include/offt.h"

namespace offt {

#include "_gen/registry_parts.inc"

namespace {
struct Table {
    const KernelEntry* p;
    int n;
};
}  // namespace

const std::vector<const KernelEntry*>& registry() {
    static const std::vector<const KernelEntry*> all = [] {
        std::vector<const KernelEntry*> v;
        const Table tables[] = {OFFT_REGISTRY_TABLES};
        for (const Table& t : tables)
            for (int i = 0; i < t.n; ++i) v.push_back(&t.p[i]);
        return v;
    }();
    return all;
}

// Kernels of one length, default first: radix <= 16 before radix-32
// sequences, then fewest stages, then largest leading radix, then the most
// threads per line (one butterfly of the largest radix per thread), then
// whole-line exchanges before exchanges in parts.
// (Sorted once per length: planning a batch of 64 grids asks hundreds of times.)
static std::vector<const KernelEntry*> sorted_kernels(int dtype, int L) {
    std::vector<const KernelEntry*> v;
    for (const KernelEntry* e : registry())
        if (e->dtype == dtype && e->L == L) v.push_back(e);
    auto key = [](const KernelEntry* e) {
        int maxr = 0;
        for (int i = 0; i < e->nstages; ++i) maxr = std::max(maxr, e->radices[i]);
        return std::make_tuple(maxr > 16, e->nstages, -maxr, -e->tpl, e->nparts);
    };
    std::stable_sort(v.begin(), v.end(),
                     [&](const KernelEntry* x, const KernelEntry* y) { return key(x) < key(y); });
    return v;
}

const std::vector<const KernelEntry*>& kernels_for(int dtype, int L) {
    static const auto all = [] {
        std::vector<std::vector<const KernelEntry*>> t(2 * (OFFT_MAX_AXIS + 1));
        for (int d : {OFFT_C2C_F64, OFFT_C2C_F32})
            for (int n = 1; n <= OFFT_MAX_AXIS; ++n) t[(d == OFFT_C2C_F64 ? 0 : OFFT_MAX_AXIS + 1) + n] = sorted_kernels(d, n);
        return t;
    }();
    static const std::vector<const KernelEntry*> none;
    if (L < 1 || L > OFFT_MAX_AXIS) return none;
    return all[(dtype == OFFT_C2C_F64 ? 0 : OFFT_MAX_AXIS + 1) + L];
}

static int default_tpl(const KernelEntry* k) {
    int maxr = 0;
    for (int i = 0; i < k->nstages; ++i) maxr = std::max(maxr, k->radices[i]);
    return k->L / maxr;
}

size_t elem_size(int dtype) { return dtype == OFFT_C2C_F64 ? 16 : 8; }

bool smooth235(int64_t n) {
    if (n < 1) return false;
    for (int p : {2, 3, 5})
        while (n % p == 0) n /= p;
    return n == 1;
}

static int ilog2(int64_t v) {
    int k = 0;
    while ((int64_t(1) << (k + 1)) <= v) ++k;
    return k;
}

int64_t lds_limit() {
    static const int64_t lim = [] {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess || v <= 0) {
            (void)hipGetLastError();
            return int64_t(64 * 1024);
        }
        return int64_t(v);
    }();
    return lim;
}

bool tile_fits(const KernelEntry* k, int logW, int dtype) {
    if (!k || logW < 0) return false;
    const int64_t W = int64_t(1) << logW;
    const int64_t threads = W * k->tpl;
    if (threads > k->max_threads) return false;
    const int64_t lds = tile_lds_elems((int)W, k->L, k->nparts) * (int64_t)elem_size(dtype);
    return lds <= lds_limit();
}

bool tile_fits_transpose(const KernelEntry* k, int logW, int dtype) {
    if (!k || !k->launch_t || logW < 0) return false;
    const int64_t W = int64_t(1) << logW;
    if (W * k->tpl > kTransposeMaxThreads) return false;
    return tile_lds_elems_transpose((int)W, k->L, k->nparts) * (int64_t)elem_size(dtype) <= lds_limit();
}

bool tile_fits_geom(const KernelEntry* k, int logW, int dtype, int g) {
    return g == kGeomTranspose ? tile_fits_transpose(k, logW, dtype) : tile_fits(k, logW, dtype);
}

int fit_logW(const KernelEntry* k, int logW, int dtype, int g) {
    if (!k) return 0;
    while (logW > 0 && !tile_fits_geom(k, logW, dtype, g)) --logW;
    return logW;
}

// ---- geometry of the passes ---------------------------------------------------

int axis_geom(const PlanChoice& c, int ax) {
    if (c.tax < 0) return kGeomNatural;
    if (ax == c.tax) return kGeomTranspose;
    int pa = 0, pt = 0;
    for (int i = 0; i < 3; ++i) {
        if (c.order[i] == ax) pa = i;
        if (c.order[i] == c.tax) pt = i;
    }
    return pa < pt ? kGeomNatural : kGeomReversed;
}

// On the abc grid the lines of axis ax form the [M1][L][M2] view with M1 the
// product of the axes before it (times the batch) and M2 of those after it;
// on the cba grid the two swap.  The transposing pass keeps the strided view
// of its strided side: the abc grid for axis a (rows written to the cba
// grid), the cba grid for axis c (rows read from the abc grid).  In both the
// row of line m1*M2 + m2 is m1*M2 + (m2 mod X)*Y + m2 div X with X the
// length of the opposite end axis and Y = Nb.
PassPlan make_pass(const int64_t dims[3], int64_t batch, int ax, int g, const KernelEntry* k, int logW, int xcd,
                   int io) {
    PassPlan p;
    p.axis = ax;
    p.L = (int)dims[ax];
    p.k = k;
    p.logW = logW;
    p.xcd = xcd;
    p.stream = k ? resolve_stream(io, dims[0] * dims[1] * dims[2] * batch * (int64_t)elem_size(k->dtype)) : 0;
    p.tw = nullptr;
    p.X = 1;
    p.Y = 1;
    int64_t before = 1, after = 1;
    for (int j = 0; j < ax; ++j) before *= dims[j];
    for (int j = ax + 1; j < 3; ++j) after *= dims[j];
    if (g == kGeomTranspose) {
        p.M1 = batch;
        p.M2 = before * after;
        p.X = dims[2 - ax];
        p.Y = dims[1];
        p.mode = ax == 0 ? 3 : 2;
    } else if (g == kGeomReversed) {
        p.M1 = batch * after;
        p.M2 = before;
        p.mode = before > 1 ? 1 : 0;
    } else {
        p.M1 = batch * before;
        p.M2 = after;
        p.mode = after > 1 ? 1 : 0;
    }
    return p;
}

bool reversal_moves_data(const int64_t dims[3]) {
    int n = 0;
    for (int ax = 0; ax < 3; ++ax) n += dims[ax] > 1;
    return n >= 2;
}

int transpose_index(const PassPlan* ps, int n) {
    for (int i = 0; i < n; ++i)
        if (ps[i].mode >= 2) return i;
    return -1;
}

// Without a transposing pass (or with one first and distinct buffers) pass 0
// reads `in` and every pass writes `out`.  Passes before a later transposing
// pass run in the workspace, which it then reads; a transposing first pass
// with in == out writes the workspace and the second pass brings the data
// back to `out`.
bool pass_io(const PassPlan* ps, int n, int i, const void* in, void* out, void* work, const void** src,
             void** dst) {
    const int tp = transpose_index(ps, n);
    if (tp < 0 || (tp == 0 && in != out)) {
        *src = i == 0 ? in : out;
        *dst = out;
        return true;
    }
    if (!work) return false;
    if (tp == 0) {
        *src = i == 0 ? in : (i == 1 ? (const void*)work : (const void*)out);
        *dst = i == 0 ? work : out;
        return true;
    }
    if (i < tp) {
        *src = i == 0 ? in : (const void*)work;
        *dst = work;
    } else {
        *src = i == tp ? (const void*)work : (const void*)out;
        *dst = out;
    }
    return true;
}

static int max_radix(const KernelEntry* k) {
    int maxr = 0;
    for (int i = 0; i < k->nstages; ++i) maxr = std::max(maxr, k->radices[i]);
    return maxr;
}

// Heuristic tile width: strided lines get 256-byte row segments (16 columns
// of complex128, 32 of complex64), and radix-32 kernels 32 columns in both
// precisions; contiguous lines ~512 threads per workgroup for complex128 and
// ~256 for complex64.
static int strided_logW(const KernelEntry* k, int dtype) {
    return max_radix(k) >= 32 ? 5 : (dtype == OFFT_C2C_F64 ? 4 : 5);
}

static int default_logW(const KernelEntry* k, int dtype, bool strided) {
    if (!k) return 0;
    int logW;
    if (strided)
        logW = strided_logW(k, dtype);
    else
        logW = ilog2(std::max<int64_t>(1, (dtype == OFFT_C2C_F64 ? 512 : 256) / k->tpl));
    return fit_logW(k, logW, dtype);
}

// Default kernel of an axis: the first in kernels_for() order whose tile at the
// heuristic width fits; contiguous axes take the first kernel with whole-line
// exchanges and radix <= 16, complex64 ones first looking for radix <= 8 at
// the default threads per line (over the 2200 grids of the selector's data
// set, such a kernel at the same width made the complex64 transform faster in
// 84% of the grids where the radix-16 kernel was the default, geometric mean
// 0.93 of the time, 0.92 for axes up to 128 points).  Strided axes of length >= 512 look first at
// radix-32 kernels whose LDS exchanges run in 2 parts (one exchange per line
// instead of two, half the LDS per tile), then at the other 2-part kernels:
// on MI355X these were the fastest, or within 0.5% of it, for every strided
// pass measured at 512^3 (both precisions) and 1024^3 (complex64).
static const KernelEntry* default_kernel(int dtype, int L, bool strided) {
    std::vector<const KernelEntry*> ks;
    if (strided && L >= 512) {
        for (const KernelEntry* k : kernels_for(dtype, L))
            if (!k->extra && k->nparts == 2 && max_radix(k) >= 32) ks.push_back(k);
        for (const KernelEntry* k : kernels_for(dtype, L))
            if (!k->extra && k->nparts == 2 && max_radix(k) <= 16) ks.push_back(k);
    }
    if (!strided && dtype == OFFT_C2C_F32)
        for (const KernelEntry* k : kernels_for(dtype, L))
            if (!k->extra && k->nparts == 1 && max_radix(k) <= 8 && k->tpl * max_radix(k) == L) ks.push_back(k);
    for (const KernelEntry* k : kernels_for(dtype, L))
        if (!k->extra && k->nparts == 1 && max_radix(k) <= 16) ks.push_back(k);
    if (ks.empty()) return nullptr;
    if (!strided) return ks[0];
    for (const KernelEntry* k : ks)
        if (default_logW(k, dtype, true) >= strided_logW(k, dtype)) return k;
    for (const KernelEntry* k : ks)
        if (k->nparts == 1) return k;
    return ks[0];
}

// ---- measured default kernels ---------------------------------------------
// kernel_defaults.txt: per precision, line kind and length one spec per class
// of grid bytes.
namespace {
enum LineKind { kContiguous = 0, kStrided = 1, kTransposing = 2 };
struct KernelDefault {
    int dtype;
    int kind;              // LineKind
    int L;
    const char* spec[3];
    int half;              // strided lines: half of the last spec's width on aligned rows
};
const KernelDefault kKernelDefaults[] = {
#include "_gen/kernel_defaults.inc"
};
}  // namespace

struct AxisSpec {
    bool given = false;
    std::vector<int> rad;
    long W = 0, tpl = 0, P = 1;
    int xcd = 0;
    int io = kIoAuto;
};
static bool parse_axis_spec(const std::string& val, AxisSpec* sp);
static const KernelEntry* find_kernel(int dtype, int L, const AxisSpec& sp);

// Passes of fewer lines than the device has CUs keep the radix-sequence rules'
// kernels (fewest stages): they are one latency chain whatever the tile
// (8 x 8 x 512 complex128: 12.4 to 13.7 us a transform with either).
constexpr int64_t kTableMinLines = 256;
// Size classes of kernel_defaults.txt.  The first line lies between the 4 MiB
// and the 16 MiB timings: at 4 MiB the large grids' kernels of 128-point lines
// (complex128) move 1.5 TB/s on strided lines where the narrow tiles move
// 2.0, at 64 MiB 3.9 against 3.6.  The second, where
// the passes between begin to stream: at 205 to 256 MiB of complex64 (12
// cubes, batched) the second class's plans took 0.94 of the third's time (216^3
// x 3 228 against 254 us, 256^3 x 2 237 against 260, 144^3 x 9 202 against
// 201), at 261 MiB 1.52; complex128, boxes of 12 shapes, 0.91, 0.96, 0.94 and
// 1.06 at 160, 208, 256 and 330 MiB.  A complex64 plan with a transposing pass
// also fills a workspace, and its line lies at 192 MiB: over 14 boxes of 198
// to 253 MiB the third class took 0.957 of the second's time in the mean where
// three plans ran in turn (0.89 to 0.97 on eleven, 1.01 to 1.12 on three) and
// 1.006 where one plan ran alone (0.95 to 1.06, backward 0.89 to 1.06).
constexpr int64_t kSmallGridBytes = int64_t(8) << 20;
constexpr int64_t kLargeTransposedBytes = int64_t(192) << 20;

// Streaming strided lines: rows of whole cache lines may take narrower tiles,
// strides below a cache line do not follow the table (kernel_defaults.txt says
// what was measured).
constexpr int64_t kCacheLine = 128;

// Whether streaming strided lines, whose rows lie `row` bytes apart, take half
// of a tile width of `width` bytes.
//   below 2 MiB     where rows are whole cache lines (or less than one)
//   from 2 MiB on   (each row of a tile on a page of its own) complex64 where
//                   the half still spans two cache lines, complex128 there
//                   also only at powers of two, whose rows fall on the same
//                   channels
// Time with the width against half of it, first axes of all listed lengths
// (means; halves of 256 bytes, of 128 bytes), complex64: 15 strides of 0.6 to
// 1.95 MiB 1.01 to 1.07, 1.04 to 1.09; 2 and 4 MiB 1.07, 0.87 to 0.92; other
// strides to 7.6 MiB 1.00 to 1.04, 0.95 to 1.04.  complex128: six strides of
// 1.2 to 1.98 MiB 1.02 to 1.06, 1.03 to 1.10; 2 and 8 MiB 1.08 and 1.03, 0.91
// and 0.88; 13 others to 15 MiB 0.96 to 1.02, 0.90 to 1.01.
static bool halves_width(int64_t row, int64_t width, int64_t es) {
    constexpr int64_t kPage = int64_t(2) << 20;
    if (row % kCacheLine != 0 && row >= kCacheLine) return false;
    return row < kPage || (width >= 4 * kCacheLine && (es == 8 || (row & (row - 1)) == 0));
}

// The measured default kernel and tile width of a pass over `lines` lines of
// length L and element stride m2 in a batch of grids of `bytes`; null where the
// table has none.
static const KernelEntry* table_kernel(int dtype, int L, LineKind kind, int64_t m2, int64_t lines, int64_t bytes,
                                       int* logW) {
    if (lines < kTableMinLines) return nullptr;
    const int cls = bytes <= kSmallGridBytes ? 0 : (bytes <= kStreamMinBytes ? 1 : 2);
    const int64_t es = (int64_t)elem_size(dtype), row = m2 * es;
    if (cls == 2 && kind == kStrided && row < (L < 512 ? kCacheLine : kCacheLine / 4)) return nullptr;
    for (const KernelDefault& d : kKernelDefaults) {
        if (d.dtype != dtype || d.kind != kind || d.L != L) continue;
        AxisSpec sp;
        const KernelEntry* k = parse_axis_spec(d.spec[cls], &sp) ? find_kernel(dtype, L, sp) : nullptr;
        if (!k) return nullptr;
        if (cls == 2 && d.half && halves_width(row, sp.W * es, es)) sp.W /= 2;
        *logW = fit_logW(k, ilog2(sp.W), dtype, kind == kTransposing ? kGeomTranspose : kGeomNatural);
        return k;
    }
    return nullptr;
}

// The kernel and width of a pass that does not transpose: the table's, or
// the rules' where it has none.
static const KernelEntry* pass_kernel(int dtype, int L, int64_t m2, int64_t lines, int64_t bytes, int* logW) {
    const bool strided = m2 > 1;
    if (const KernelEntry* k = table_kernel(dtype, L, strided ? kStrided : kContiguous, m2, lines, bytes, logW)) return k;
    const KernelEntry* k = default_kernel(dtype, L, strided);
    *logW = default_logW(k, dtype, strided);
    return k;
}

static bool axis_strided(int axis, const int64_t dims[3]) {
    // M2 of an axis: product of the later axes' lengths
    int64_t m2 = 1;
    for (int j = axis + 1; j < 3; ++j) m2 *= dims[j];
    return m2 > 1;
}

// Default tile order: XCD-contiguous for strided lines.  Over the 2200 grids
// of the selector's data set (axes 16..1024, MI355X) that order made strided
// passes faster in 59-75% of the grids above 64 MiB (geometric mean 0.93 of
// the time) and slightly faster below; on contiguous lines it was neutral to
// slower, and transposing passes keep the launch order.  With streaming
// accesses (grids above the Infinity Cache) the launch order was faster for
// lines strided by 2 MiB or more: 6% for pass a at 1024^3 complex64, 3% at
// 512^3 complex64.
constexpr int64_t kLongStrideBytes = int64_t(2) << 20;
static int default_xcd(int g, bool strided, bool streamed_long_stride = false) {
    return g != kGeomTranspose && strided && !streamed_long_stride ? 1 : 0;
}
// Whether the heuristic's pass along `ax` (natural geometry, one grid) streams
// over lines strided by kLongStrideBytes or more.
static bool streamed_long_stride(int dtype, const int64_t* dims, int ndim, int ax) {
    int64_t n = 1, after = 1;
    for (int j = 0; j < ndim; ++j) n *= dims[j];
    for (int j = ax + 1; j < ndim; ++j) after *= dims[j];
    const int64_t es = (int64_t)elem_size(dtype);
    return resolve_stream(kIoAuto, n * es) && after * es >= kLongStrideBytes;
}

// Default kernel of a transposing pass: for L >= 512 the first radix <= 16
// kernel whose exchanges and row side run in 2 parts (half the LDS of a
// whole-line tile, so two workgroups share a CU: on MI355X at 512^3 these
// ran the transposing pass 13-17% faster than whole-line tiles), else the
// first whole-line kernel with radix <= 16.  Tiles of 16 lines.
static const KernelEntry* default_kernel_transpose(int dtype, int L) {
    if (L >= 512)
        for (const KernelEntry* k : kernels_for(dtype, L))
            if (!k->extra && k->nparts == 2 && k->launch_t && max_radix(k) <= 16 && tile_fits_transpose(k, 4, dtype)) return k;
    for (const KernelEntry* k : kernels_for(dtype, L))
        if (!k->extra && k->nparts == 1 && k->launch_t && max_radix(k) <= 16) return k;
    for (const KernelEntry* k : kernels_for(dtype, L))
        if (!k->extra && k->nparts == 1 && k->launch_t) return k;
    return nullptr;
}

// The heuristic kernel and width of every axis, for the geometry the
// choice's order and output order give it.
static void assign_default_kernels(PlanChoice& c, int dtype, const int64_t dims[3], int64_t batch,
                                   bool rules_only = false) {
    const int64_t points = dims[0] * dims[1] * dims[2] * batch;
    int64_t bytes = points * (int64_t)elem_size(dtype);
    for (int ax = 0; ax < 3; ++ax)
        if (dims[ax] > 1 && axis_geom(c, ax) == kGeomTranspose && dtype == OFFT_C2C_F32 && bytes > kLargeTransposedBytes)
            bytes = std::max(bytes, kStreamMinBytes + 1);
    for (int ax = 0; ax < 3; ++ax) {
        c.k[ax] = nullptr;
        c.logW[ax] = 0;
        if (dims[ax] <= 1) continue;
        const int g = axis_geom(c, ax);
        const KernelEntry* k;
        int logW = 0;
        if (g == kGeomTranspose) {
            k = table_kernel(dtype, (int)dims[ax], kTransposing, 1, points / dims[ax], bytes, &logW);
            if (!k) {
                k = default_kernel_transpose(dtype, (int)dims[ax]);
                logW = k ? fit_logW(k, 4, dtype, g) : 0;
            }
        } else {
            const int64_t m2 = make_pass(dims, 1, ax, g, nullptr, 0).M2;
            k = pass_kernel(dtype, (int)dims[ax], m2, rules_only ? 0 : points / dims[ax], bytes, &logW);
        }
        if (k) {
            c.k[ax] = k;
            c.logW[ax] = logW;
            c.xcd[ax] = default_xcd(g, make_pass(dims, 1, ax, g, nullptr, 0).M2 > 1,
                                    g == kGeomNatural && streamed_long_stride(dtype, dims, 3, ax));
        }
    }
}

static int fuse_rule(int dtype, int64_t A, int64_t B, int64_t C, int64_t grids, int64_t lds_max = lds_limit());
static const KernelEntry* block_kernel_entry(int dtype, int64_t L);

// The last axes of a default plan that run as a block kernel take kernels of
// its radix sequences, so that the passes one by one give the same bits.
// (first: index of dims[0] in k and logW.)
static void assign_block_kernels(int dtype, int ndim, const int64_t* dims, int64_t batch, const KernelEntry** k,
                                 int* logW, int first = 0) {
    int64_t grids = batch;
    for (int i = 0; i < ndim - 3; ++i) grids *= dims[i];
    const int64_t A = ndim >= 3 ? dims[ndim - 3] : 1;
    const int f = fuse_rule(dtype, A, dims[ndim - 2], dims[ndim - 1], grids);
    for (int i = 0; i < f; ++i) {
        const int ax = ndim - 1 - i;
        const KernelEntry* e = block_kernel_entry(dtype, dims[ax]);
        if (!e) continue;
        k[first + ax] = e;
        logW[first + ax] = default_logW(e, dtype, i > 0);
    }
}

PassPlan contiguous_pass(int dtype, int L, int64_t lines, int64_t grid_bytes) {
    PassPlan p;
    p.axis = 2;
    p.L = L;
    p.M1 = lines;
    p.M2 = 1;
    p.X = 1;
    p.Y = 1;
    p.mode = 0;
    p.xcd = 0;
    p.tw = nullptr;
    p.k = pass_kernel(dtype, L, 1, lines, grid_bytes, &p.logW);
    p.stream = resolve_stream(kIoAuto, grid_bytes);
    return p;
}

PlanChoice default_choice(int dtype, const int64_t dims[3], int64_t batch, bool rules_only) {
    PlanChoice c;
    c.order[0] = 2; c.order[1] = 1; c.order[2] = 0;   // c, then b, then a
    c.tax = -1;
    assign_default_kernels(c, dtype, dims, batch, rules_only);
    if (!rules_only) assign_block_kernels(dtype, 3, dims, batch, c.k, c.logW);
    return c;
}

// Reversed output: passes c, b, a with the pass along a transposing (strided
// abc lines in, cba rows out), so the first pass reads contiguous lines and
// only pass b runs on strided lines of one buffer; without an axis a, the
// pass along c transposes (abc rows in, strided cba lines out).
PlanChoice default_choice_reversed(int dtype, const int64_t dims[3], int64_t batch) {
    if (!reversal_moves_data(dims)) return default_choice(dtype, dims, batch);
    PlanChoice c;
    c.order[0] = 2; c.order[1] = 1; c.order[2] = 0;
    c.tax = dims[0] > 1 ? 0 : 2;
    assign_default_kernels(c, dtype, dims, batch);
    // the passes over c and b come before the transposing one over a
    if (c.tax == 0) assign_block_kernels(dtype, 2, dims + 1, batch * dims[0], c.k, c.logW, 1);
    return c;
}

std::vector<PlanChoice> candidate_choices(int dtype, const int64_t dims[3], int64_t batch, bool rules_only) {
    std::vector<PlanChoice> out;
    const PlanChoice base = default_choice(dtype, dims, batch, rules_only);
    out.push_back(base);
    // per-axis variants with the default order: other kernels (radix
    // sequence, threads per line, exchange parts on strided axes) and tile
    // widths one step either side of the heuristic
    for (int ax = 0; ax < 3; ++ax) {
        if (dims[ax] <= 1) continue;
        const bool strided = axis_strided(ax, dims);
        std::vector<const KernelEntry*> ks = kernels_for(dtype, (int)dims[ax]);
        for (const KernelEntry* k : ks) {
            if ((k->nparts > 1 && !strided) || k->extra) continue;
            const int l0 = default_logW(k, dtype, strided);
            for (int dl = -1; dl <= 1; ++dl) {
                const int lw = l0 + dl;
                if (lw < 0 || fit_logW(k, lw, dtype) != lw) continue;
                if (k == base.k[ax] && lw == base.logW[ax]) continue;
                PlanChoice c = base;
                c.k[ax] = k;
                c.logW[ax] = lw;
                out.push_back(c);
            }
        }
    }
    // the heuristic with one axis's tile order switched (launch order <->
    // XCD-contiguous)
    for (int ax = 0; ax < 3; ++ax) {
        if (dims[ax] <= 1 || !base.k[ax]) continue;
        PlanChoice c = base;
        c.xcd[ax] = !base.xcd[ax];
        out.push_back(c);
    }
    // other axis orders with the default kernels
    const int perms[5][3] = {{2, 0, 1}, {1, 2, 0}, {1, 0, 2}, {0, 2, 1}, {0, 1, 2}};
    for (const auto& pm : perms) {
        PlanChoice c = base;
        for (int i = 0; i < 3; ++i) c.order[i] = pm[i];
        out.push_back(c);
    }
    return out;
}

static const char kAxisName[] = "abcde";

// ---- plan strings ---------------------------------------------------------------
// One axis: "<radix sequence>/<tile width>[/<threads per line>][/p<parts>][/x][/s|/c]",
// or "1" for a length-1 axis ("/x": XCD-contiguous tile order; "/s", "/c":
// streaming or cached grid-data accesses, by default chosen from the grid's
// size).

static void axis_to_string(std::ostringstream& os, const KernelEntry* k, int logW, int64_t len, int xcd, int io) {
    if (!k || len <= 1) {
        os << "1";
        return;
    }
    for (int i = 0; i < k->nstages; ++i) os << (i ? "x" : "") << k->radices[i];
    os << "/" << (1 << logW);
    if (k->tpl != default_tpl(k)) os << "/" << k->tpl;
    if (k->nparts > 1) os << "/p" << k->nparts;
    if (xcd) os << "/x";
    if (io == kIoStream) os << "/s";
    if (io == kIoCached) os << "/c";
}

static bool parse_axis_spec(const std::string& val, AxisSpec* sp) {
    sp->given = true;
    const size_t slash = val.find('/');
    if (slash == std::string::npos) return false;
    std::stringstream rs(val.substr(0, slash));
    std::string tok;
    while (std::getline(rs, tok, 'x')) {
        char* end = nullptr;
        const long r = strtol(tok.c_str(), &end, 10);
        if (!end || *end || r < 2) return false;
        sp->rad.push_back((int)r);
    }
    char* end = nullptr;
    sp->W = strtol(val.c_str() + slash + 1, &end, 10);
    if (!end || sp->W < 1 || (sp->W & (sp->W - 1))) return false;
    if (*end == '/' && end[1] >= '0' && end[1] <= '9') {   // threads per line (default: the sequence's)
        char* end2 = nullptr;
        sp->tpl = strtol(end + 1, &end2, 10);
        if (!end2 || sp->tpl < 1) return false;
        end = end2;
    }
    if (*end == '/' && end[1] == 'p') {   // parts of each LDS exchange (strided axes)
        char* end2 = nullptr;
        sp->P = strtol(end + 2, &end2, 10);
        if (!end2 || (sp->P != 1 && sp->P != 2 && sp->P != 4)) return false;
        end = end2;
    }
    if (end[0] == '/' && end[1] == 'x' && (end[2] == 0 || end[2] == '/')) {   // XCD-contiguous tile order
        sp->xcd = 1;
        end += 2;
    }
    if (end[0] == '/' && (end[1] == 's' || end[1] == 'c') && end[2] == 0) {   // grid-data access mode
        sp->io = end[1] == 's' ? kIoStream : kIoCached;
        end += 2;
    }
    return *end == 0;
}

static const KernelEntry* find_kernel(int dtype, int L, const AxisSpec& sp) {
    for (const KernelEntry* k : kernels_for(dtype, L)) {
        if (k->nstages != (int)sp.rad.size()) continue;
        bool eq = true;
        for (int i = 0; i < k->nstages; ++i) eq = eq && k->radices[i] == sp.rad[i];
        if (eq && k->tpl == (sp.tpl ? (int)sp.tpl : default_tpl(k)) && k->nparts == (int)sp.P) return k;
    }
    return nullptr;
}

// "order=<axis letters>": a permutation of the first ndim letters
static bool parse_order(const std::string& val, int ndim, int* order) {
    if ((int)val.size() != ndim) return false;
    bool seen[kMaxDims] = {false, false, false, false, false};
    for (int i = 0; i < ndim; ++i) {
        const char* p = val[i] ? strchr(kAxisName, val[i]) : nullptr;
        if (!p || p - kAxisName >= ndim) return false;
        const int ax = int(p - kAxisName);
        if (seen[ax]) return false;
        seen[ax] = true;
        order[i] = ax;
    }
    return true;
}

std::string choice_to_string(const PlanChoice& c, const int64_t dims[3]) {
    std::ostringstream os;
    os << "order=" << kAxisName[c.order[0]] << kAxisName[c.order[1]] << kAxisName[c.order[2]];
    if (c.tax >= 0) os << ";rev=" << kAxisName[c.tax];
    for (int ax = 0; ax < 3; ++ax) {
        os << ";" << kAxisName[ax] << "=";
        axis_to_string(os, c.k[ax], c.logW[ax], dims[ax], c.xcd[ax], c.io[ax]);
    }
    if (c.slab > 0) os << ";slab=" << c.slab;
    if (c.col > 0) os << ";col=" << c.col;
    return os.str();
}

bool slab_fits(const PlanChoice& c, const int64_t dims[3]) {
    return c.slab == 0 || (c.slab > 0 && c.col == 0 && c.tax < 0 && c.order[0] == 0 && dims[0] > 1 &&
                           dims[1] * dims[2] > 1);
}

bool col_fits(const PlanChoice& c, const int64_t dims[3], bool check_tiles) {
    if (c.col == 0) return true;
    const int64_t w = c.col;
    if (w < 1 || (w & (w - 1)) || c.slab != 0 || c.tax >= 0 || c.order[0] != 2 || dims[2] <= 1 ||
        dims[0] * dims[1] <= 1 || dims[2] % w != 0 || w >= dims[2])
        return false;
    // every blocked pass takes whole tiles of one block row: W lines of one
    // m1 are W consecutive columns
    if (check_tiles)
        for (int ax = 0; ax < 2; ++ax)
            if (dims[ax] > 1 && (!c.k[ax] || (int64_t(1) << c.logW[ax]) > w)) return false;
    return true;
}

// Planes per slab from a plan string: a decimal count of 1 to 2^40.
static bool parse_slab(const std::string& val, int64_t* out) {
    if (val.empty() || val.size() > 13) return false;
    int64_t v = 0;
    for (char ch : val) {
        if (ch < '0' || ch > '9') return false;
        v = v * 10 + (ch - '0');
    }
    if (v < 1 || v > (int64_t(1) << 40)) return false;
    *out = v;
    return true;
}

PassPlan slab_pass(const PassPlan& p, int64_t p0, int64_t np, int64_t* elem_off) {
    PassPlan q = p;
    q.M1 = p.M1 / p.planes * np;
    *elem_off = p0 * p.plane_elems;
    return q;
}

PassPlan col_pass(const PassPlan& p, int64_t c0) {
    PassPlan q = p;
    int lw = 0;
    while ((int64_t(1) << lw) < p.col) ++lw;
    q.blk_logw = lw;
    q.blk_ld = p.ncol;
    q.blk_off = c0;
    q.lpm = p.M2 / p.ncol * p.col;   // rows of the m1 (M2 / Nc of them) times the block's columns
    return q;
}

int slab_start(const PassPlan* ps, int n) {
    for (int i = 0; i < n; ++i)
        if (ps[i].slab > 0 || ps[i].col > 0) return i;
    return n;
}

bool choice_from_string(const char* s, int dtype, const int64_t dims[3], PlanChoice* out, bool check_fit) {
    if (!s) return false;
    AxisSpec spec[3];
    PlanChoice c;
    c.tax = -1;
    std::string str(s);
    std::stringstream ss(str);
    std::string item;
    bool have_order = false;
    while (std::getline(ss, item, ';')) {
        const size_t eq = item.find('=');
        if (eq == std::string::npos) return false;
        const std::string key = item.substr(0, eq), val = item.substr(eq + 1);
        if (key == "order") {
            if (!parse_order(val, 3, c.order)) return false;
            have_order = true;
        } else if (key == "rev") {
            if (val == "a") c.tax = 0;
            else if (val == "c") c.tax = 2;
            else return false;
        } else if (key == "slab") {
            if (!parse_slab(val, &c.slab)) return false;
        } else if (key == "col") {
            if (!parse_slab(val, &c.col)) return false;
        } else if (key.size() == 1 && key[0] >= 'a' && key[0] <= 'c') {
            const int ax = key[0] - 'a';
            if (dims[ax] <= 1) {
                if (val != "1") return false;
                continue;
            }
            if (!parse_axis_spec(val, &spec[ax])) return false;
        } else {
            return false;
        }
    }
    if (!have_order) return false;
    if (c.tax >= 0 && (!reversal_moves_data(dims) || dims[c.tax] <= 1)) return false;
    if (!slab_fits(c, dims) || !col_fits(c, dims, false)) return false;
    // axes the string leaves out take the heuristic's kernel for their geometry
    assign_default_kernels(c, dtype, dims, 1);
    for (int ax = 0; ax < 3; ++ax) {
        if (!spec[ax].given) continue;
        const AxisSpec& sp = spec[ax];
        const int g = axis_geom(c, ax);
        const bool strided = g == kGeomTranspose || make_pass(dims, 1, ax, g, nullptr, 0).M2 > 1;
        if (sp.P > 1 && !strided) return false;
        const KernelEntry* found = find_kernel(dtype, (int)dims[ax], sp);
        if (!found || (g == kGeomTranspose && !found->launch_t)) return false;
        const int lw = ilog2(sp.W);
        if (check_fit && !tile_fits_geom(found, lw, dtype, g)) return false;
        c.k[ax] = found;
        c.logW[ax] = lw;
        c.xcd[ax] = sp.xcd;
        c.io[ax] = sp.io;
    }
    if (!col_fits(c, dims, true)) return false;
    *out = c;
    return true;
}

// ---- grids of more than three dimensions -------------------------------------

PassPlan make_pass_nd(int ndim, const int64_t* dims, int64_t batch, int ax, const KernelEntry* k, int logW,
                      int xcd, int io) {
    PassPlan p;
    p.axis = ax;
    p.L = (int)dims[ax];
    p.k = k;
    p.logW = logW;
    p.xcd = xcd;
    int64_t bytes = batch;
    for (int j = 0; j < ndim; ++j) bytes *= dims[j];
    p.stream = k ? resolve_stream(io, bytes * (int64_t)elem_size(k->dtype)) : 0;
    p.tw = nullptr;
    p.X = 1;
    p.Y = 1;
    int64_t before = 1, after = 1;
    for (int j = 0; j < ax; ++j) before *= dims[j];
    for (int j = ax + 1; j < ndim; ++j) after *= dims[j];
    p.M1 = batch * before;
    p.M2 = after;
    p.mode = after > 1 ? 1 : 0;
    return p;
}

// Heuristic: passes from the last (contiguous) axis to the first, each axis
// with the kernel and width the three-dimensional heuristic gives a line of
// its length and stride kind.
NdChoice default_choice_nd(int dtype, int ndim, const int64_t* dims, int64_t batch) {
    NdChoice c;
    c.ndim = ndim;
    for (int i = 0; i < ndim; ++i) c.order[i] = ndim - 1 - i;
    int64_t points = batch;
    for (int i = 0; i < ndim; ++i) points *= dims[i];
    for (int ax = 0; ax < ndim; ++ax) {
        c.k[ax] = nullptr;
        c.logW[ax] = 0;
        if (dims[ax] <= 1) continue;
        const int64_t m2 = make_pass_nd(ndim, dims, 1, ax, nullptr, 0).M2;
        const bool strided = m2 > 1;
        int logW = 0;
        const KernelEntry* k = pass_kernel(dtype, (int)dims[ax], m2, points / dims[ax],
                                           points * (int64_t)elem_size(dtype), &logW);
        if (k) {
            c.k[ax] = k;
            c.logW[ax] = logW;
            c.xcd[ax] = default_xcd(kGeomNatural, strided, streamed_long_stride(dtype, dims, ndim, ax));
        }
    }
    assign_block_kernels(dtype, ndim, dims, batch, c.k, c.logW);
    return c;
}

std::string nd_choice_to_string(const NdChoice& c, const int64_t* dims) {
    std::ostringstream os;
    os << "order=";
    for (int i = 0; i < c.ndim; ++i) os << kAxisName[c.order[i]];
    for (int ax = 0; ax < c.ndim; ++ax) {
        os << ";" << kAxisName[ax] << "=";
        axis_to_string(os, c.k[ax], c.logW[ax], dims[ax], c.xcd[ax], c.io[ax]);
    }
    if (c.slab > 0) os << ";slab=" << c.slab;
    return os.str();
}

bool nd_slab_fits(const NdChoice& c, const int64_t* dims) {
    int64_t rest = 1;
    for (int ax = 1; ax < c.ndim; ++ax) rest *= dims[ax];
    return c.slab == 0 || (c.slab > 0 && c.ndim >= 2 && c.order[0] == 0 && dims[0] > 1 && rest > 1);
}

bool nd_choice_from_string(const char* s, int dtype, int ndim, const int64_t* dims, NdChoice* out,
                           bool check_fit) {
    if (!s || ndim < 1 || ndim > kMaxDims) return false;
    AxisSpec spec[kMaxDims];
    NdChoice c = default_choice_nd(dtype, ndim, dims);
    std::string str(s);
    std::stringstream ss(str);
    std::string item;
    bool have_order = false;
    while (std::getline(ss, item, ';')) {
        const size_t eq = item.find('=');
        if (eq == std::string::npos) return false;
        const std::string key = item.substr(0, eq), val = item.substr(eq + 1);
        if (key == "order") {
            if (!parse_order(val, ndim, c.order)) return false;
            have_order = true;
        } else if (key == "slab") {
            if (!parse_slab(val, &c.slab)) return false;
        } else if (key.size() == 1 && key[0] >= 'a' && key[0] < 'a' + ndim) {
            const int ax = key[0] - 'a';
            if (dims[ax] <= 1) {
                if (val != "1") return false;
                continue;
            }
            if (!parse_axis_spec(val, &spec[ax])) return false;
        } else {
            return false;
        }
    }
    if (!have_order || !nd_slab_fits(c, dims)) return false;
    for (int ax = 0; ax < ndim; ++ax) {
        if (!spec[ax].given) continue;
        const bool strided = make_pass_nd(ndim, dims, 1, ax, nullptr, 0).M2 > 1;
        if (spec[ax].P > 1 && !strided) return false;
        const KernelEntry* found = find_kernel(dtype, (int)dims[ax], spec[ax]);
        if (!found) return false;
        const int lw = ilog2(spec[ax].W);
        if (check_fit && !tile_fits(found, lw, dtype)) return false;
        c.k[ax] = found;
        c.logW[ax] = lw;
        c.xcd[ax] = spec[ax].xcd;
        c.io[ax] = spec[ax].io;
    }
    *out = c;
    return true;
}

static int64_t grid_elems_nd(int ndim, const int64_t* dims) {
    int64_t n = 1;
    for (int i = 0; i < ndim; ++i) n *= dims[i];
    return n;
}

// Every pass after the first on slabs of `slab` planes (blocks of
// plane_elems elements, `planes` of them); access modes resolved for one
// slab's bytes (it may stay cached between the passes).
static void set_slab(PassPlan* out, int n, int64_t planes, int64_t plane_elems, int64_t slab_planes, const int* io) {
    const int64_t slab = std::min(slab_planes, planes);
    for (int i = 1; i < n; ++i) {
        out[i].slab = slab;
        out[i].planes = planes;
        out[i].plane_elems = plane_elems;
        if (out[i].k)
            out[i].stream = resolve_stream(io[out[i].axis], slab * plane_elems * (int64_t)elem_size(out[i].k->dtype));
    }
}

// Streaming ends of a batch of grids whose passes are cached.  From half of
// the Infinity Cache on, input and output do not both fit there, and the input
// is not read again: out of place the first pass streams its loads.  The last
// pass of a transposing plan reads one buffer and writes another, which no
// pass reads: it streams its stores.  Measured on MI355X, before -> after:
//   loads   256^3 complex128 258 -> 239 us, 300^3 complex64 255 -> 242,
//           48 x 64^3 complex128 143 -> 128; in place 238 -> 257 (256^3), so
//           a launch in place keeps its loads cached; 128 MiB, 256^3 complex64,
//           three buffer pairs in turn 145 -> 126, one pair 123 -> 125; below,
//           160^3 complex128 66.6 -> 70.8
//   stores  reversed output order, 256 x 320 x 384 complex64 284 -> 249 us
//           (with the loads 242), 192^3 complex128 115 -> 107, 128^3 36.6 -> 35.2
constexpr int64_t kStreamSrcMinBytes = int64_t(128) << 20;
constexpr int64_t kStreamDstMinBytes = int64_t(32) << 20;
static void set_edge_streams(PassPlan* out, int n, int64_t bytes, const int* io) {
    if (n < 2) return;
    PassPlan &first = out[0], &last = out[n - 1];
    if (bytes >= kStreamSrcMinBytes && bytes <= kStreamMinBytes && io[first.axis] == kIoAuto) first.stream_src = 1;
    if (bytes >= kStreamDstMinBytes && last.mode >= 2 && io[last.axis] == kIoAuto) last.stream |= kStreamStores;
}

// Access mode of a launch of pass p.
static int launch_streams(const PassPlan& p, const void* in, const void* out) {
    return p.stream | (p.stream_src && in != out ? kStreamLoads : 0);
}

int build_passes_nd(const NdChoice& c, const int64_t* dims, int64_t batch, PassPlan* out) {
    int n = 0;
    for (int i = 0; i < c.ndim; ++i) {
        const int ax = c.order[i];
        if (dims[ax] <= 1) continue;
        out[n++] = make_pass_nd(c.ndim, dims, batch, ax, c.k[ax], c.logW[ax], c.xcd[ax], c.io[ax]);
    }
    if (c.slab > 0 && nd_slab_fits(c, dims))
        set_slab(out, n, batch * dims[0], dims[0] > 0 ? grid_elems_nd(c.ndim, dims) / dims[0] : 0, c.slab, c.io);
    if (n > 0 && out[0].k)
        set_edge_streams(out, n, grid_elems_nd(c.ndim, dims) * batch * (int64_t)elem_size(out[0].k->dtype), c.io);
    return n;
}

int build_passes(const PlanChoice& c, const int64_t dims[3], int64_t batch, PassPlan out[3]) {
    int n = 0;
    for (int i = 0; i < 3; ++i) {
        const int ax = c.order[i];
        if (dims[ax] <= 1) continue;
        out[n++] = make_pass(dims, batch, ax, axis_geom(c, ax), c.k[ax], c.logW[ax], c.xcd[ax], c.io[ax]);
    }
    if (c.slab > 0 && slab_fits(c, dims)) set_slab(out, n, batch * dims[0], dims[1] * dims[2], c.slab, c.io);
    if (c.col > 0 && col_fits(c, dims, true)) {
        // every pass after the one over c, on blocks of columns; access modes
        // resolved for one block's bytes
        for (int i = 1; i < n; ++i) {
            out[i].col = c.col;
            out[i].ncol = dims[2];
            if (out[i].k)
                out[i].stream = resolve_stream(c.io[out[i].axis], batch * dims[0] * dims[1] * c.col *
                                                                      (int64_t)elem_size(out[i].k->dtype));
        }
    }
    if (n > 0 && out[0].k)
        set_edge_streams(out, n, dims[0] * dims[1] * dims[2] * batch * (int64_t)elem_size(out[0].k->dtype), c.io);
    return n;
}

// ---- block kernels --------------------------------------------------------------

// The block kernels of each precision (generated table): longest line and
// most threads, the kernel of the shorter lines first.
#include "_gen/block_kernels.inc"
static const BlockCase kBlockCases[] = {
#include "_gen/block_cases.inc"
};

constexpr int64_t kCUs = 256;

// Case of the block kernel for lines of kernel k's radix sequence, or -1 (the
// index counts the cases of k's precision).
static int block_case(const KernelEntry* k) {
    int i = 0;
    for (const BlockCase& c : kBlockCases) {
        if (c.dtype != k->dtype) continue;
        if (c.L == k->L && c.nstages == k->nstages && std::equal(c.radices, c.radices + c.nstages, k->radices)) return i;
        ++i;
    }
    return -1;
}

static const BlockCase* block_case_of_length(int dtype, int64_t L) {
    for (const BlockCase& c : kBlockCases)
        if (c.dtype == dtype && c.L == L) return &c;
    return nullptr;
}

static const KernelEntry* block_kernel_entry(int dtype, int64_t L) {
    if (L < 2 || L > OFFT_MAX_AXIS) return nullptr;
    for (const KernelEntry* k : kernels_for(dtype, (int)L))
        if (k->nparts == 1 && block_case(k) >= 0) return k;
    return nullptr;
}

// The block kernel of lines of up to `maxl` points.
static const BlockKernel* block_kernel_for(int dtype, int maxl) {
    for (const BlockKernel& bk : kBlockKernels)
        if (bk.dtype == dtype && maxl <= bk.max_l) return &bk;
    return nullptr;
}

// Threads of a workgroup that transforms one block of `blocks` (naxes of its
// axes), and streams its stores or not; 0 without a kernel.
//
// Up to one block per CU: a thread for every line of the longest pass at once
// (in threads per line).  Beyond that a CU holds several workgroups, as many as
// its LDS and the kernel's waves per SIMD allow.  Of 64, 128, ... 1024 threads
// (a workgroup's waves then spread evenly over the SIMDs; two lines at a time
// at least) the most with which all blocks reside at once; if there are none,
// the first that keeps the most threads resident.  Stores that stream pass L2
// unmerged, so that there the lanes of a row of the last pass should span a
// cache line.  The short kernels keep their earlier count, half of the lines at
// once where two such workgroups still fill a CU (3072 planes of 48 x 48,
// complex128: 112, 105, 94 and 85 us a transform with 576, 320, 384 and 192
// threads), where all blocks reside with it or the other keeps less than a
// fifth more threads.
// Measured on 150 plane shapes per precision at 8, 24, 96 and 400 MiB (time
// against the earlier count in every kernel): long lines 0.98, 0.82, 0.71 and
// 0.81 in complex64, 0.92, 0.83, 0.79 and 0.84 in complex128; short ones 1.00,
// 0.95, 0.93, 0.96 and 1.00, 0.94, 0.88, 0.89.  2013 planes of 50 x 125 in
// complex64: 102 us with 1024 threads, 62 with 512 (separate passes 64).
static int block_threads(int dtype, int A, int B, int C, int naxes, int64_t blocks, bool streamed,
                         int64_t lds_max = lds_limit()) {
    const BlockKernel* bk = block_kernel_for(dtype, std::max(std::max(A, B), C));
    if (!bk) return 0;
    const int64_t n = (int64_t)A * B * C, es = (int64_t)elem_size(dtype);
    int64_t one = 0, least = 1, last = 1;
    for (const int L : {C, B, A}) {
        if (L < 2) continue;
        const BlockCase* c = block_case_of_length(dtype, L);
        if (!c) return 0;
        one = std::max(one, n / L * c->tpl);
        least = std::max<int64_t>(least, c->tpl);
        last = c->tpl;
    }
    const auto waves = [](int64_t t) { return (t + 63) / 64 * 64; };
    const auto in_kernel = [&](int64_t t) { return std::min<int64_t>(bk->threads, waves(std::max(t, least))); };
    if (blocks <= kCUs) return (int)in_kernel(one);
    const int64_t per_cu = lds_max / (block_lds_elems(A, B, C) * es), held = (blocks + kCUs - 1) / kCUs;
    const int64_t slots = (int64_t)bk->waves * 4 * 64;
    const auto groups = [&](int64_t t) { return std::min(per_cu, slots / t); };
    const auto resident = [&](int64_t t) { return std::min(groups(t), held) * t; };
    const int64_t row = naxes == 3 ? (int64_t)B * C : C;
    const auto lines_of_cache = [&](int64_t t) { return !streamed || t / last >= row || t / last * es >= kCacheLine; };
    const bool is_short = bk->max_l < kBlockMaxLine;
    const int64_t earlier = in_kernel(per_cu * waves(one / 2) >= 1024 ? one / 2 : one);
    if (is_short && groups(earlier) >= held) return (int)earlier;
    int64_t best = 0, at_once = 0;
    bool whole_rows = false;
    for (int64_t t = 64; t <= bk->threads; t *= 2) {
        if (t < least || (t < 2 * least && t < one && 2 * t <= bk->threads)) continue;
        if (best && t / 2 >= one) break;
        if (groups(t) >= held) at_once = t;
        const bool ok = lines_of_cache(t);
        if (!best || (ok && !whole_rows) || (ok == whole_rows && resident(t) > resident(best))) {
            best = t;
            whole_rows = ok;
        }
    }
    if (at_once) return (int)at_once;
    const bool keep = is_short && 5 * resident(best) < 6 * resident(earlier) && (lines_of_cache(earlier) || !whole_rows);
    return (int)(keep ? earlier : best);
}

// Axes that run as one block kernel, by size: 3 (blocks are whole A x B x C
// grids), 2 (B x C planes) or 0 (each pass alone).  What decides is whether a
// CU holds two blocks (one block's loads and stores then overlap the other's
// stages) and whether there are blocks for enough CUs.  Measured on MI355X,
// separate passes against the block kernel, per transform:
//   whole grids    16^3 complex128 14.6 -> 9.5 us, 1024 of them 65 -> 38 us;
//                  18^3 alone 13.1 -> 13.4 us (planes: 10.3), 1024 93 -> 70 us
//   planes         64^3 complex64 14.8 -> 11.8 us, 64 of them 118 -> 102 us;
//                  64 x 32^3 complex128 37.7 -> 29.5 us
//   one block per  8 x 100^3 complex64 65.8 -> 75.4 us (in the Infinity Cache),
//   CU             64 of them 617 -> 549 us, 128^4 2.97 -> 2.80 ms (streaming);
//                  128^3 alone 35.6 -> 27.3 us, 8 of them equal; fewer planes
//                  alone, speed against separate passes: 64, 80 and 108 of 100 x
//                  100 complex64 1.00, 1.05, 1.15, of 128 x 128 0.92, 1.01,
//                  1.19, of 90 x 90 complex128 0.98, 1.07, 1.19; with threads
//                  idle in a round 64, 108, 128 and 160 of 100 x 120 complex64
//                  0.79, 0.94, 0.98, 1.03, of 72 x 150 0.76, 0.91, 0.95, 1.02
//   few blocks     12 x 150 x 60 complex64 14.3 -> 16.4 us; a plane to a CU with
//                  three-stage lines, 125^3 complex64 33.5 -> 36.2 us, but
//                  250 x 125^2 44.7 -> 41.2 us
//   tiny blocks    each costs a workgroup, 0.4 to 0.8 ns: 8192 planes of 2^2 to
//                  12^2 points 8 to 12 us against 10 to 14, 9715 of 30 x 6 in
//                  complex64 20 -> 13, 65536 of 2^2, 8^2 and 16^2 9.8 -> 39,
//                  24 -> 52 and 82 -> 75 (streaming: 331200 of 20 x 5 in
//                  complex128 636 -> 400); 32768 grids of 3^3, 4^3 and 5^3 in
//                  complex64 15 -> 28, 31 -> 30, 39 -> 34
//   three stages   along b, above 64 MiB: 6742 planes of 243 x 32 complex64 301
//                  -> 586 us, 30340 of 216 x 8 345 -> 398, 8738 of 200 x 15
//                  complex128 359 -> 439; along c they gain (3145 planes of 36 x
//                  250 complex64 291 -> 221)
static int fuse_rule(int dtype, int64_t A, int64_t B, int64_t C, int64_t grids, int64_t lds_max) {
    if (C < 2 || B < 2 || !block_case_of_length(dtype, B) || !block_case_of_length(dtype, C)) return 0;
    const int64_t es = (int64_t)elem_size(dtype);
    constexpr int64_t kTwoPerCu = 80 * 1024;
    // the most blocks by their bytes (any number from `large` on)
    const auto few = [](int64_t bytes, int64_t blocks, int64_t large) {
        return bytes >= large || blocks <= (bytes < 1000 ? 8192 : 16384);
    };
    const int64_t planes = A * grids;
    // up to 64 rows the contiguous pass keeps the rules' kernels, radix 16 in
    // complex128 and up to 8 in complex64
    if (planes * B <= 64) return 0;
    const bool streamed = planes * B * C * es > kStreamMinBytes;
    // a launch holds at most 2^32 - 1 threads
    const auto launches = [&](int64_t a, int naxes, int64_t blocks) {
        for (const bool st : {false, true}) {
            const int t = block_threads(dtype, (int)a, (int)B, (int)C, naxes, blocks, st, lds_max);
            if (t < 1 || blocks > int64_t(0xffffffffu) / t) return false;
        }
        return true;
    };
    if (A > 1 && block_case_of_length(dtype, A)) {
        const int64_t lds = block_lds_elems((int)A, (int)B, (int)C) * es;
        if (lds <= lds_max && (grids >= 512 || (lds <= kTwoPerCu && A * B * C <= 4096)) &&
            few(A * B * C * es, grids, 1100) && launches(A, 3, grids))
            return 3;
    }
    const int64_t lds = block_lds_elems(1, (int)B, (int)C) * es;
    if (lds > lds_max) return 0;
    if (!few(B * C * es, planes, streamed ? 100 * es : 2048)) return 0;
    const int sb = block_case_of_length(dtype, B)->nstages, sc = block_case_of_length(dtype, C)->nstages;
    if (sb > 2 && planes * B * C * es > (int64_t(64) << 20)) return 0;
    if (lds <= kTwoPerCu) {
        if (B * C > 4096 && planes < 64) return 0;
    } else if (!streamed) {
        // lines that fill three quarters of each round of threads
        const int64_t t = block_threads(dtype, 1, (int)B, (int)C, 2, planes, false, lds_max);
        const auto full = [&](int64_t w) { return 4 * w >= 3 * ((w + t - 1) / t * t); };
        const bool busy = full(B * block_case_of_length(dtype, C)->tpl) && full(C * block_case_of_length(dtype, B)->tpl);
        if (planes < (std::max(sb, sc) > 2 ? 192 : busy ? 80 : 128) || planes > kCUs) return 0;
    }
    return launches(1, 2, planes) ? 2 : 0;
}

void set_fuse(PassPlan* ps, int n) {
    for (int i = 0; i + 1 < n; ++i) {
        const PassPlan &c = ps[i], &b = ps[i + 1];
        // rows, then the lines across them, of one contiguous block
        if (c.mode != 0 || b.mode != 1 || b.M2 != c.L || c.M1 != b.M1 * b.L || c.slab || c.col || b.slab || b.col)
            continue;
        if (!c.k || !b.k || block_case(c.k) < 0 || block_case(b.k) < 0) continue;
        const PassPlan* a = i + 2 < n ? &ps[i + 2] : nullptr;
        const bool whole = a && a->mode == 1 && !a->slab && !a->col && a->k && a->M2 == b.M2 * b.L &&
                           b.M1 == a->M1 * a->L && block_case(a->k) >= 0;
        const int f = fuse_rule(c.k->dtype, whole ? a->L : 1, b.L, c.L, whole ? a->M1 : b.M1);
        if (f < 2) continue;
        ps[i].fuse = f;
        for (const bool st : {false, true})
            ps[i].block_threads[st] = block_threads(c.k->dtype, f == 3 ? a->L : 1, b.L, c.L, f, ps[i + f - 1].M1, st);
    }
}

hipError_t launch_block(const PassPlan* ps, const void* in, void* out, int conj_in, int conj_out, double scale,
                        hipStream_t s) {
    const int f = ps[0].fuse;
    BlockArgs a{};
    a.in = in;
    a.out = out;
    a.naxes = f;
    for (int i = 0; i < f; ++i) {
        a.tw[i] = ps[i].tw;
        a.kid[i] = block_case(ps[i].k);
        if (a.kid[i] < 0) return hipErrorInvalidValue;
    }
    a.C = ps[0].L;
    a.B = ps[1].L;
    a.A = f == 3 ? ps[2].L : 1;
    a.pitch = block_pitch(a.C);
    a.rcp_C = block_rcp(a.C);
    a.stream_in = launch_streams(ps[0], in, out) & kStreamLoads;
    a.stream_out = ps[f - 1].stream & kStreamStores;
    a.conj_in = conj_in;
    a.conj_out = conj_out;
    a.scale = scale;
    const int64_t blocks = ps[f - 1].M1;
    const int dtype = ps[0].k->dtype;
    const int64_t lds = block_lds_elems(a.A, a.B, a.C) * (int64_t)elem_size(dtype);
    if (lds > lds_limit()) return hipErrorInvalidValue;
    const int threads = ps[0].block_threads[a.stream_out != 0];
    const BlockKernel* bk = block_kernel_for(dtype, std::max(std::max(a.A, a.B), a.C));
    if (threads < 1 || blocks > int64_t(0xffffffffu) / threads) return hipErrorInvalidValue;
    return bk->launch(a, blocks, threads, (size_t)lds, s);
}

hipError_t launch_pass(const PassPlan& p, const void* in, void* out, int conj_in, int conj_out,
                       double scale, hipStream_t s) {
    PassArgs a;
    a.in = in;
    a.out = out;
    a.tw = p.tw;
    a.lpm = p.lpm > 0 ? p.lpm : p.M2;
    a.nlines = p.M1 * a.lpm;
    a.M2 = p.M2;
    a.blk_logw = p.blk_logw;
    a.blk_ld = p.blk_ld;
    a.blk_off = p.blk_off;
    a.X = p.X;
    a.Y = p.Y;
    a.logW = p.logW;
    a.mode = p.mode;
    a.xcd_remap = p.xcd;
    a.stream_io = launch_streams(p, in, out);
    a.conj_in = conj_in;
    a.conj_out = conj_out;
    a.scale = scale;
    // a kernel with exchanges in parts keeps only part of each line in LDS:
    // strided lines (or the strided side of a transposing pass) only
    if (p.k->nparts > 1 && p.mode == 0) return hipErrorInvalidValue;
    const int64_t W = int64_t(1) << p.logW;
    const int64_t nblocks = (a.nlines + W - 1) / W;
    const int threads = (int)(W * p.k->tpl);
    if (p.mode >= 2) {
        // transposing pass: never in place (its row side and strided side
        // cover the same elements in different orders)
        if (!p.k->launch_t || in == out || p.X < 1 || p.Y < 1 || p.X * p.Y != p.M2) return hipErrorInvalidValue;
        const size_t lds_t = (size_t)tile_lds_elems_transpose((int)W, p.L, p.k->nparts) * elem_size(p.k->dtype);
        return p.k->launch_t(a, nblocks, threads, lds_t, s);
    }
    const size_t lds = (size_t)tile_lds_elems((int)W, p.L, p.k->nparts) * (p.k->dtype == OFFT_C2C_F64 ? 16 : 8);
    return p.k->launch(a, nblocks, threads, lds, s);
}

}  // namespace offt

using namespace offt;

extern "C" {

// Not part of the C ABI: the block rule and the threads of a block launch for
// a device with lds_max bytes of LDS per workgroup, and the rule of the width
// of streaming strided lines (tests).
int offt_test_halves_width(int64_t row, int64_t width, int64_t es) { return halves_width(row, width, es); }

int offt_test_fuse_rule(int dtype, int64_t A, int64_t B, int64_t C, int64_t grids, int64_t lds_max) {
    return fuse_rule(dtype, A, B, C, grids, lds_max);
}

int offt_test_block_threads(int dtype, int64_t A, int64_t B, int64_t C, int64_t blocks, int streamed, int64_t lds_max) {
    return block_threads(dtype, (int)A, (int)B, (int)C, A > 1 ? 3 : 2, blocks, streamed != 0, lds_max);
}

}  // extern "C"

// Host side of the wave lattice Boltzmann library: the C ABI declared in
// include/lb_wave.h (descriptor checks, workspace layout, compact sound-speed
// tables, surface stencils, launches and read-back).
//
// Method: Castro-Avila et al., "A lattice Boltzmann approach for acoustic
// manipulation" (arXiv 2404.02346).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <climits>
#include <functional>
#include <limits>
#include <mutex>
#include <numeric>
#include <string>
#include <utility>
#include <vector>

#include "../../include/lb_wave.h"
#include "lb_kernels.hpp"

using namespace lbw;

namespace {

thread_local std::string g_err;

int fail(int code, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

#define HIP_TRY(expr)                                                                    \
    do {                                                                                 \
        hipError_t e_ = (expr);                                                          \
        if (e_ != hipSuccess)                                                            \
            return fail(LB_EDEVICE, "%s failed: %s", #expr, hipGetErrorString(e_));      \
    } while (0)

constexpr size_t kAlign = 256;
inline size_t align_up(size_t v, size_t a = kAlign) { return (v + a - 1) / a * a; }

size_t elem_bytes(int storage)
{
    switch (storage) {
    case LB_F64: return 8;
    case LB_F32: return 4;
    default: return 2;
    }
}
size_t compute_bytes(int storage) { return storage == LB_F64 ? 8 : 4; }

inline int wrapi(long v, int n)
{
    long r = v % n;
    return (int)(r < 0 ? r + n : r);
}

// The 3-point kernel printed after eq. InterpolatedFields.
double roma3(double r)
{
    const double a = std::fabs(r);
    if (a <= 0.5) return (1.0 + std::sqrt(1.0 - 3.0 * a * a)) / 3.0;
    if (a <= 1.5) return (5.0 - 3.0 * a - std::sqrt(1.0 - 3.0 * (1.0 - a) * (1.0 - a))) / 6.0;
    return 0.0;
}

// Sound speed of eq. sound_speed_object, read with c = c_p inside.  For
// (r^2 - R^2)/d >= 20 the tanh rounds to 1 and c is exactly c0.
double object_c(const lb_wave_desc &d, double x, double y, double z)
{
    const double dx = x - d.obj_center[0], dy = y - d.obj_center[1];
    const double dz = d.dim == 3 ? z - d.obj_center[2] : 0.0;
    const double u = (dx * dx + dy * dy + dz * dz - d.obj_radius * d.obj_radius) / d.obj_d;
    return d.c0 - 0.5 * (d.c0 - d.obj_cp) * (1.0 - std::tanh(u));
}

constexpr double kTanhSaturate = 20.0;

inline bool finite(double v) { return std::isfinite(v); }

// Box of cells whose sound speed differs from c0 (inclusive lo, extent n).
struct Box {
    int lo[3] = {0, 0, 0};
    int n[3] = {0, 0, 0};
    size_t cells() const { return (size_t)n[0] * n[1] * n[2]; }
};

// cells of its c^2 table
size_t c2_cells(const Box &b) { return (size_t)c2_plane(b.n[0], b.n[1]) * b.n[2]; }

Box sound_speed_box(const lb_wave_desc &d)
{
    Box b;
    const int nn[3] = {d.nx, d.ny, d.dim == 3 ? d.nz : 1};
    if (d.c_field) {
        int lo[3] = {nn[0], nn[1], nn[2]}, hi[3] = {-1, -1, -1};
        for (int z = 0; z < nn[2]; ++z)
            for (int y = 0; y < nn[1]; ++y)
                for (int x = 0; x < nn[0]; ++x) {
                    const double c = d.c_field[((size_t)z * nn[1] + y) * nn[0] + x];
                    if (c != d.c0) {
                        const int p[3] = {x, y, z};
                        for (int a = 0; a < 3; ++a) {
                            lo[a] = std::min(lo[a], p[a]);
                            hi[a] = std::max(hi[a], p[a]);
                        }
                    }
                }
        if (hi[0] < 0) return b;
        for (int a = 0; a < 3; ++a) {
            b.lo[a] = lo[a];
            b.n[a] = hi[a] - lo[a] + 1;
        }
        return b;
    }
    if (d.obj_cp == d.c0) return b;  // c = c0 exactly everywhere
    const double h = std::sqrt(d.obj_radius * d.obj_radius + kTanhSaturate * d.obj_d);
    for (int a = 0; a < 3; ++a) {
        if (a == 2 && d.dim == 2) {
            b.lo[2] = 0;
            b.n[2] = 1;
            continue;
        }
        long lo = (long)std::floor(d.obj_center[a] - h);
        long hi = (long)std::ceil(d.obj_center[a] + h);
        lo = std::max(lo, 0L);
        hi = std::min(hi, (long)nn[a] - 1);
        if (hi < lo) return Box{};
        b.lo[a] = (int)lo;
        b.n[a] = (int)(hi - lo + 1);
    }
    return b;
}

// 3-point stencil of one surface point: base node by rounding half away from
// zero, nodes base-1, base, base+1 along each axis.
void stencil(const lb_wave_desc &d, const double *P, SurfPt &s, long xn[3])
{
    const int nn[3] = {d.nx, d.ny, d.dim == 3 ? d.nz : 1};
    for (int a = 0; a < 3; ++a) {
        if (a == 2 && d.dim == 2) {
            for (int o = 0; o < 3; ++o) {
                s.bz[o] = 0;
                s.w[6 + o] = (o == 0) ? 1.0 : 0.0;
            }
            continue;
        }
        const long b = std::lround(P[a]);
        for (int o = 0; o < 3; ++o) {
            const long node = b - 1 + o;
            const double w = roma3((double)node - P[a]);
            if (a == 0) {
                xn[o] = node;
                s.bx[o] = (int)node;
                s.w[o] = w;
            } else if (a == 1) {
                s.by[o] = wrapi(node, nn[1]);
                s.w[3 + o] = w;
            } else {
                s.bz[o] = wrapi(node, nn[2]);
                s.w[6 + o] = w;
            }
        }
    }
    s.pad = 0;
}

// Box of the stencil nodes of all surface points.  Along y and z a box that
// would cross the periodic boundary takes the whole extent.
Box measure_box(const lb_wave_desc &d)
{
    Box b;
    if (d.n_surf <= 0) return b;
    const int nn[3] = {d.nx, d.ny, d.dim == 3 ? d.nz : 1};
    long lo[3] = {LONG_MAX, LONG_MAX, LONG_MAX}, hi[3] = {LONG_MIN, LONG_MIN, LONG_MIN};
    for (int k = 0; k < d.n_surf; ++k)
        for (int a = 0; a < d.dim; ++a) {
            const long c = std::lround(d.surf_xyz[3 * k + a]);
            lo[a] = std::min(lo[a], c - 1);
            hi[a] = std::max(hi[a], c + 1);
        }
    for (int a = 0; a < 3; ++a) {
        if (a >= d.dim) {
            b.lo[a] = 0;
            b.n[a] = 1;
        } else if (lo[a] >= 0 && hi[a] < nn[a]) {
            b.lo[a] = (int)lo[a];
            b.n[a] = (int)(hi[a] - lo[a] + 1);
        } else {
            b.lo[a] = 0;
            b.n[a] = nn[a];
        }
    }
    return b;
}

// Stencil nodes relative to the moment box (y, z wrapped first).
void stencil_in_box(const lb_wave_desc &d, const double *P, const Box &mb, SurfPt &s)
{
    SurfPt g;
    long xn[3];
    stencil(d, P, g, xn);
    s = g;
    for (int o = 0; o < 3; ++o) {
        s.bx[o] = g.bx[o] - mb.lo[0];
        s.by[o] = g.by[o] - mb.lo[1];
        s.bz[o] = g.bz[o] - mb.lo[2];
    }
}

int check_one(const lb_wave_desc &d, const lb_wave_desc &d0, int idx)
{
    if (d.dim != 2 && d.dim != 3) return fail(LB_EINVAL, "instance %d: dim must be 2 or 3", idx);
    if (d.dim != d0.dim) return fail(LB_EINVAL, "instance %d: all instances must share dim", idx);
    if (d.nx < 1 || d.ny < 1 || d.nz < 1) return fail(LB_EINVAL, "instance %d: bad shape", idx);
    if (d.dim == 2 && d.nz != 1) return fail(LB_EINVAL, "instance %d: nz must be 1 in 2D", idx);
    if (d.storage < LB_F64 || d.storage > LB_BF16)
        return fail(LB_EINVAL, "instance %d: bad storage", idx);
    if (d.storage != d0.storage)
        return fail(LB_EINVAL, "instance %d: all instances must share storage", idx);
    if (d.xbc != LB_XBC_DRIVEN && d.xbc != LB_XBC_PERIODIC)
        return fail(LB_EINVAL, "instance %d: bad xbc", idx);
    if (d.xbc == LB_XBC_DRIVEN && d.nx < 3)
        return fail(LB_EINVAL, "instance %d: driven x needs nx >= 3", idx);
    if (!(d.c0 > 0) || !finite(d.c0)) return fail(LB_EINVAL, "instance %d: c0 must be > 0", idx);
    if (!(d.rho0 > 0) || !finite(d.rho0))
        return fail(LB_EINVAL, "instance %d: rho0 must be > 0", idx);
    if (!(d.wall_phi >= 0 && d.wall_phi < 1))
        return fail(LB_EINVAL, "instance %d: wall_phi must lie in [0, 1)", idx);
    if (!finite(d.rho_a) || !finite(d.omega))
        return fail(LB_EINVAL, "instance %d: rho_a and omega must be finite", idx);
    if (d.avg_start < 0 || d.trace_steps < 0)
        return fail(LB_EINVAL, "instance %d: avg_start and trace_steps must be >= 0", idx);
    if (d.src_kind != LB_SRC_SHEET && d.src_kind != LB_SRC_POINT)
        return fail(LB_EINVAL, "instance %d: bad src_kind", idx);
    if (d.src_kind == LB_SRC_POINT) {
        if (d.xbc != LB_XBC_PERIODIC)
            return fail(LB_EINVAL, "instance %d: a point source needs periodic x", idx);
        const int32_t *s = d.src_cell;
        if (s[0] < 0 || s[0] >= d.nx || s[1] < 0 || s[1] >= d.ny || s[2] < 0 || s[2] >= d.nz)
            return fail(LB_EINVAL, "instance %d: source node (%d, %d, %d) outside the lattice",
                        idx, s[0], s[1], s[2]);
    }
    // sizes: rows and wave tasks are indexed with 32-bit integers
    const long pitch = (long)align_up((size_t)d.nx, 64);
    const long rows = (long)d.ny * d.nz;
    if (pitch * rows > (long)INT32_MAX * 8 || rows * ((pitch + 63) / 64) > INT32_MAX / 2)
        return fail(LB_EINVAL, "instance %d: lattice too large", idx);
    // stability of the tau = 1/2 scheme: every c <= 1/sqrt(dim)
    const double cmax_allowed = 1.0 / std::sqrt((double)d.dim) * (1.0 + 1e-12);
    double cmax = d.c0;
    if (d.c_field) {
        const size_t n = (size_t)d.nx * d.ny * d.nz;
        for (size_t i = 0; i < n; ++i) {
            if (!finite(d.c_field[i])) return fail(LB_EINVAL, "instance %d: c_field not finite", idx);
            cmax = std::max(cmax, std::fabs(d.c_field[i]));
        }
    } else {
        if (!finite(d.obj_cp) || !finite(d.obj_radius) || !finite(d.obj_d) ||
            !finite(d.obj_center[0]) || !finite(d.obj_center[1]) || !finite(d.obj_center[2]))
            return fail(LB_EINVAL, "instance %d: object parameters not finite", idx);
        if (d.obj_cp != d.c0 && !(d.obj_d > 0))
            return fail(LB_EINVAL, "instance %d: obj_d must be > 0", idx);
        cmax = std::max(cmax, std::fabs(d.obj_cp));
    }
    if (cmax > cmax_allowed)
        return fail(LB_EUNSTABLE, "instance %d: sound speed %.6g exceeds 1/sqrt(%d)", idx, cmax,
                    d.dim);
    if (d.n_surf < 0) return fail(LB_EINVAL, "instance %d: n_surf < 0", idx);
    if (d.n_surf > 0) {
        if (!d.surf_xyz || !d.surf_normal || !d.surf_area)
            return fail(LB_EINVAL, "instance %d: surface arrays missing", idx);
        const long xlo = d.xbc == LB_XBC_DRIVEN ? 2 : 0;
        const long xhi = d.xbc == LB_XBC_DRIVEN ? d.nx - 2 : d.nx - 1;
        for (int k = 0; k < d.n_surf; ++k) {
            for (int a = 0; a < 3; ++a)
                if (!finite(d.surf_xyz[3 * k + a]) || !finite(d.surf_normal[3 * k + a]))
                    return fail(LB_EINVAL, "instance %d: surface point %d not finite", idx, k);
            if (!finite(d.surf_area[k]))
                return fail(LB_EINVAL, "instance %d: surface area %d not finite", idx, k);
            SurfPt s;
            long xn[3];
            stencil(d, d.surf_xyz + 3 * k, s, xn);
            if (xn[0] < xlo || xn[2] > xhi)
                return fail(LB_EGEOMETRY,
                            "instance %d: stencil of surface point %d spans x = %ld..%ld, "
                            "outside %ld..%ld",
                            idx, k, xn[0], xn[2], xlo, xhi);
        }
    }
    return LB_OK;
}

int check_all(const lb_wave_desc *descs, int n)
{
    if (!descs || n < 1) return fail(LB_EINVAL, "need at least one descriptor");
    long tasks = 0;
    for (int i = 0; i < n; ++i) {
        int st = check_one(descs[i], descs[0], i);
        if (st != LB_OK) return st;
        const long xsegs = (descs[i].nx + 63) / 64;
        tasks += xsegs * descs[i].ny * descs[i].nz;
        // a one-step launch runs 64 threads per task and a 1D grid holds fewer than 2^32
        if (tasks > (long)(UINT32_MAX / 64)) return fail(LB_EINVAL, "batch too large");
    }
    return LB_OK;
}

// Population planes are skewed against each other: the plane stride is the
// plane rounded up to 8 KiB plus 3 KiB, so the seven planes start at seven
// different offsets modulo 8 KiB and their streams spread over the memory
// channels and banks (with power-of-two strides they collide; measured on
// the 16 x 256 x 128 x 128 workload: 5.43 -> 5.90 TB/s).
constexpr int64_t kPlaneRound = 8192, kPlaneSkew = 3072;
// State buffers start on 4 KiB: where they lie then does not depend on the sizes of the tables
// before them (four channels of 1000 x 64 x 64 in FP32: 80 us per step, 81 to 83 without).
constexpr size_t kBufAlign = 4096;
int64_t plane_stride(int64_t elems, size_t eb)
{
    const int64_t bytes = (elems * (int64_t)eb + kPlaneRound - 1) / kPlaneRound * kPlaneRound;
    return (bytes + kPlaneSkew) / (int64_t)eb;
}

struct InstPlan {
    Box box;   // sound speed differs from c0
    Box mbox;  // cells whose moments the surface reads
    int pitch;
    int64_t plane;
    int n_chunks;
    size_t off_surf, off_part, off_mom, mom_bytes, off_trace, off_box, off_buf[kNumBuf];
};

struct Layout {
    size_t off_inst, off_acc, off_sbtab, off_tdev, total;
    int n_sb_total;
    bool resident;  // every box is advanced by the resident kernel
    int slots;      // moment boxes and partial sums per instance
    std::vector<InstPlan> p;
};

// The resident kernel takes handles whose boxes are all 2D, driven and small enough, for calls of at
// least eight steps: a launch costs the box's way into the registers and back.  us per step of a call
// of 8, 16 and 64 steps (with a launch per step): FP64 one box of 128 x 64 5.0, 3.3, 1.9 (5.4, 4.7, 4.4),
// of 64 x 64 3.5, 2.3, 1.3 (5.5, 5.0, 4.6), 512 of 127 x 63 24, 18, 12 (74 each); FP32 127 x 63 4.3, 3.1,
// 2.0 (5.3, 5.0, 4.5).  FP64 boxes that almost fill their tile mask most of their columns: a few of
// them pay from twelve steps on (127 x 63 6.3, 4.5, 3.0 against 5.5, 5.0, 4.6; 116 x 55 5.9, 4.2, 2.8
// against 5.5, 5.1, 4.7; 100 x 50 5.3, 3.8, 2.5 against 5.2, 5.0, 4.5).
constexpr int kResidentMin = 8, kResidentMinMasked = 12;
constexpr int kMaskedCells = 5000, kMaskedBoxes = 16;
// Its moment boxes and partial sums, one for each step of two launches, may take this much: handles of
// thousands of boxes with large surfaces keep the small workspace of one step per launch.  So do those
// whose surface blocks, those of all steps in one launch, are more threads than a grid holds.
constexpr size_t kResidentBytes = (size_t)8 << 30;
// blocks of a launch over `boxes` boxes with `meas` measurement blocks of kStepThreads threads, which
// run side by side
int64_t resident_grid(int64_t boxes, int64_t meas)
{
    const int per = 64 * kResidentWaves / kStepThreads;
    return boxes + (meas + per - 1) / per;
}
int resident_of(const lb_wave_desc &d)
{
    if (d.dim != 2 || d.xbc != LB_XBC_DRIVEN || d.src_kind != LB_SRC_SHEET) return 0;
    return resident_config(d.nx, d.ny);
}

int resident_min(const lb_wave_desc *descs, int n)
{
    for (int i = 0; i < n && n < kMaskedBoxes && descs[0].storage == LB_F64; ++i) {
        const int c = resident_of(descs[i]);
        const bool full = descs[i].nx == kResidentWaves * (c >> 8) && descs[i].ny == 64 * (c & 255);
        if (!full && descs[i].nx * descs[i].ny > kMaskedCells) return kResidentMinMasked;
    }
    return kResidentMin;
}

Layout plan(const lb_wave_desc *descs, int n)
{
    Layout L;
    size_t off = 0;
    L.off_inst = off;
    off = align_up(off + sizeof(InstDev) * n);
    L.off_acc = off;
    off = align_up(off + sizeof(AccDev) * n);
    L.n_sb_total = 0;
    L.resident = true;
    size_t slot_bytes = 0;
    for (int i = 0; i < n; ++i) {
        L.n_sb_total += (descs[i].n_surf + 63) / 64;
        if (!resident_of(descs[i])) L.resident = false;
        if (L.resident)
            slot_bytes += align_up(4 * compute_bytes(descs[i].storage) * measure_box(descs[i]).cells()) +
                          sizeof(double) * 4 * (size_t)((descs[i].n_surf + 63) / 64);
    }
    if (slot_bytes > kResidentBytes / (2 * kResidentSteps)) L.resident = false;
    if (resident_grid(n, n + (int64_t)kResidentSteps * L.n_sb_total) * 64 * kResidentWaves > (int64_t)UINT32_MAX)
        L.resident = false;
    L.slots = L.resident ? 2 * kResidentSteps : kNumSlot;
    L.off_sbtab = off;
    off = align_up(off + sizeof(int32_t) * 2 * (size_t)L.n_sb_total);
    L.off_tdev = off;
    off = align_up(off + 2 * sizeof(int64_t));
    L.p.resize(n);
    for (int i = 0; i < n; ++i) {
        const lb_wave_desc &d = descs[i];
        InstPlan &P = L.p[i];
        const int Q = 2 * d.dim + 1;
        P.box = sound_speed_box(d);
        P.pitch = (int)align_up((size_t)d.nx, 64);
        P.plane = plane_stride((int64_t)P.pitch * d.ny * d.nz, elem_bytes(d.storage));
        P.n_chunks = (d.n_surf + 63) / 64;
        P.mbox = measure_box(d);
        P.off_mom = off;
        P.mom_bytes = align_up(4 * compute_bytes(d.storage) * P.mbox.cells());
        off += P.mom_bytes * L.slots;
        P.off_surf = off;
        off = align_up(off + sizeof(SurfPt) * d.n_surf);
        P.off_part = off;
        off = align_up(off + sizeof(double) * L.slots * 4 * (size_t)P.n_chunks);
        P.off_box = off;
        off = align_up(off + compute_bytes(d.storage) * c2_cells(P.box));
        for (int b = 0; b < kNumBuf; ++b) {
            off = align_up(off, kBufAlign);
            P.off_buf[b] = off;
            off = align_up(off + elem_bytes(d.storage) * (size_t)P.plane * Q);
        }
        P.off_trace = off;
        off = align_up(off + sizeof(double) * 3 * (size_t)d.trace_steps);
    }
    L.total = off;
    return L;
}

double storage_scale(const lb_wave_desc &d)
{
    if (d.storage == LB_F64 || d.storage == LB_F32) return 1.0;
    if (!(std::fabs(d.rho_a) > 0)) return 1.0;
    return std::ldexp(1.0, (int)std::lround(-std::log2(std::fabs(d.rho_a))));
}

// ---- host conversions for state read-back ----
inline float bf16_to_f(uint16_t b)
{
    uint32_t u = (uint32_t)b << 16;
    float f;
    std::memcpy(&f, &u, 4);
    return f;
}
inline uint16_t f_to_bf16(float f)
{
    uint32_t u;
    std::memcpy(&u, &f, 4);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
inline double load_host(const uint8_t *p, int storage)
{
    switch (storage) {
    case LB_F64: { double v; std::memcpy(&v, p, 8); return v; }
    case LB_F32: { float v; std::memcpy(&v, p, 4); return v; }
    case LB_F16: { _Float16 v; std::memcpy(&v, p, 2); return (double)(float)v; }
    default: { uint16_t v; std::memcpy(&v, p, 2); return (double)bf16_to_f(v); }
    }
}
inline void store_host(uint8_t *p, int storage, double v)
{
    switch (storage) {
    case LB_F64: std::memcpy(p, &v, 8); break;
    case LB_F32: { float f = (float)v; std::memcpy(p, &f, 4); break; }
    case LB_F16: { _Float16 h = (_Float16)(float)v; std::memcpy(p, &h, 2); break; }
    default: { uint16_t b = f_to_bf16((float)v); std::memcpy(p, &b, 2); break; }
    }
}

// Blocks of one box: row blocks x chunks of planes x strips of a row.
struct MarchBox {
    int64_t nyb = 0, nzc = 0, nsx = 0;
    int64_t blocks() const { return nyb * nzc * nsx; }
};

}  // namespace

struct lb_wave {
    int n = 0, dim = 0, storage = 0, vx = 1, xm = 0, nt = 0;
    int fused = 1;                    // 1: one lattice step per launch, 2: several
    bool fused_ok = false;            // several steps per launch are allowed
    bool march_ok = false;            // every instance fits the march kernel
    bool resident = false;            // long calls run the resident kernel
    int resident_min = 0;             // ... from this many steps on
    int march_waves = 4;              // wavefronts per block of the march kernel
    int march_depth = 2;              // most steps of its launches
    int march_chunk = 0;              // most planes of a block
    int model_chunk[2][2] = {};       // ... by the model, by steps and wavefronts (0: not asked yet)
    std::vector<int> blk0;            // internal order, size n + 1: march blocks
    char *ws = nullptr;
    size_t ws_bytes = 0;
    hipStream_t stream = nullptr;
    Layout lay;
    std::vector<lb_wave_desc> desc;   // user order (host arrays not kept)
    std::vector<int> order;           // internal -> user
    std::vector<int> pos;             // user -> internal
    std::vector<InstDev> hinst;       // internal order
    std::vector<int> task0;           // internal order, size n + 1
    std::vector<SegInfo> segs;        // runs of equal shape, internal order
    std::vector<double> scale;        // user order
    InstDev *d_inst = nullptr;
    AccDev *d_acc = nullptr;          // internal order
    int32_t *d_sb_inst = nullptr;     // surface block table (internal order)
    int32_t *d_sb_chunk = nullptr;
    std::vector<int> sb_first;        // internal order, size n + 1
    bool any_surf = false;
    bool any_point = false;           // some instance has a point source
    int64_t t = 0;                    // lattice steps done
    int64_t meas = 0;                 // steps whose chunk partials exist
    int64_t red = 0;                  // steps reduced into the accumulators
    bool nan_seen = false;
    int cur = 0;                      // state buffer holding the state after step t - 1
    std::vector<int> stop_buf;        // internal order: that buffer when the instance stopped
    int64_t *d_t = nullptr;           // device counter {t, index of the current state buffer}
    int64_t tdev = 0;                 // its values in stream order
    int bufdev = 0;
    int graph_chunk = 0;              // replay steady steps as captured graphs of this length
    hipStream_t cap_stream = nullptr; // private stream used only for capture
    struct GraphEntry {
        int k, na, n_red, n_sb, nst;
        hipGraphExec_t exec;
    };
    std::vector<GraphEntry> graphs;
    ~lb_wave()
    {
        for (auto &g : graphs) (void)hipGraphExecDestroy(g.exec);
        if (cap_stream) (void)hipStreamDestroy(cap_stream);
    }
};

namespace {

// wave tasks of one step of all instances, `cells` of a row to a task
int64_t one_step_tasks(const lb_wave *h, int cells)
{
    int64_t n = 0;
    for (const InstDev &I : h->hinst) n += (int64_t)((I.nx + cells - 1) / cells) * I.ny * I.nz;
    return n;
}

// the buffer that holds the current state of an instance
int state_buf(const lb_wave *h, int internal)
{
    const int64_t ms = h->hinst[internal].max_steps;
    return ms > 0 && h->t >= ms ? h->stop_buf[internal] : h->cur;
}

int active_prefix(const lb_wave *h, int64_t t)
{
    int n = 0;
    while (n < h->n) {
        const int64_t ms = h->hinst[n].max_steps;
        if (ms > 0 && t >= ms) break;
        ++n;
    }
    return n;
}

int prefix_alive(const lb_wave *h, int64_t t)
{
    // instances are sorted by max_steps (longest first): those still alive at t form a prefix
    if (t < 0) return 0;
    return active_prefix(h, t);
}

template <int DIM, typename S, int CPL, int XM, int NT>
void launch_t(const StepArgs &a, int blocks, hipStream_t st)
{
    hipLaunchKernelGGL((step_kernel<DIM, S, CPL, XM, NT>), dim3(blocks), dim3(kStepThreads), 0, st,
                       a);
}

// Variants compiled per storage: 16-bit storage only shifts across lanes (its
// elements are 2 bytes, too small for the offset vector load).
template <int DIM, typename S, int CPL>
void launch_c(const lb_wave *h, const StepArgs &a, int blocks, hipStream_t st)
{
    constexpr bool wide = sizeof(typename StoreTraits<S>::R) >= 4;
    constexpr int XW = wide ? 1 : 0;
    if (h->xm == 1 && wide) {
        switch (h->nt) {
        case 1: launch_t<DIM, S, CPL, XW, 1>(a, blocks, st); break;
        case 2: launch_t<DIM, S, CPL, XW, 2>(a, blocks, st); break;
        default: launch_t<DIM, S, CPL, XW, 0>(a, blocks, st); break;
        }
    } else {
        switch (h->nt) {
        case 1: launch_t<DIM, S, CPL, 0, 1>(a, blocks, st); break;
        case 2: launch_t<DIM, S, CPL, 0, 2>(a, blocks, st); break;
        default: launch_t<DIM, S, CPL, 0, 0>(a, blocks, st); break;
        }
    }
}

template <int DIM, typename S>
void launch_s(const lb_wave *h, const StepArgs &a, int blocks, hipStream_t st)
{
    switch (h->vx) {
    case 2: launch_c<DIM, S, 2>(h, a, blocks, st); break;
    case 4: launch_c<DIM, S, 4>(h, a, blocks, st); break;
    default: launch_c<DIM, S, 1>(h, a, blocks, st); break;
    }
}

void launch(const lb_wave *h, const StepArgs &a, int blocks, hipStream_t st)
{
    if (blocks <= 0) return;
    const bool d2 = h->dim == 2;
    switch (h->storage) {
    case LB_F64: d2 ? launch_s<2, double>(h, a, blocks, st) : launch_s<3, double>(h, a, blocks, st); break;
    case LB_F32: d2 ? launch_s<2, float>(h, a, blocks, st) : launch_s<3, float>(h, a, blocks, st); break;
    case LB_F16:
        d2 ? launch_s<2, _Float16>(h, a, blocks, st) : launch_s<3, _Float16>(h, a, blocks, st);
        break;
    default: d2 ? launch_s<2, bf16>(h, a, blocks, st) : launch_s<3, bf16>(h, a, blocks, st); break;
    }
}

// The point sources of step t (the lattice launches of step t come first in
// stream order); launches of several steps never run on a handle with point sources.
template <int DIM, typename S>
void launch_point_s(const lb_wave *h, const StepArgs &a, hipStream_t st)
{
    hipLaunchKernelGGL((point_source_kernel<DIM, S>), dim3((h->n + 63) / 64), dim3(64), 0, st,
                       a.inst, h->n, a.tp, a.dt, a.dbuf);
}
void launch_point(const lb_wave *h, const StepArgs &a, hipStream_t st)
{
    const bool d2 = h->dim == 2;
    switch (h->storage) {
    case LB_F64: d2 ? launch_point_s<2, double>(h, a, st) : launch_point_s<3, double>(h, a, st); break;
    case LB_F32: d2 ? launch_point_s<2, float>(h, a, st) : launch_point_s<3, float>(h, a, st); break;
    case LB_F16:
        d2 ? launch_point_s<2, _Float16>(h, a, st) : launch_point_s<3, _Float16>(h, a, st);
        break;
    default: d2 ? launch_point_s<2, bf16>(h, a, st) : launch_point_s<3, bf16>(h, a, st); break;
    }
}

// Most steps of one march launch, and rows per row group.  FP64 holds twice the registers and LDS.
int march_steps(int storage) { return storage == LB_F64 ? 2 : 3; }
int march_rows(int storage) { return storage == LB_F64 ? 2 : 4; }
bool march_eight(int storage) { return storage == LB_F64 || storage == LB_F32; }

using MarchFn = void (*)(StepArgs);
template <typename S, int K, int R> MarchFn march_fn_t(int waves, int nt)
{
    if constexpr (sizeof(typename StoreTraits<S>::R) >= 4)  // march_eight
        if (waves == 8) return nt ? march_kernel<S, K, R, 8, 1> : march_kernel<S, K, R, 8, 0>;
    return nt ? march_kernel<S, K, R, 4, 1> : march_kernel<S, K, R, 4, 0>;
}
MarchFn march_fn(int storage, int steps, int waves, int nt)
{
    const bool three = steps == 3;
    switch (storage) {
    case LB_F64: return march_fn_t<double, 2, 2>(waves, nt);
    case LB_F32: return three ? march_fn_t<float, 3, 4>(waves, nt) : march_fn_t<float, 2, 4>(waves, nt);
    case LB_F16:
        return three ? march_fn_t<_Float16, 3, 4>(waves, nt) : march_fn_t<_Float16, 2, 4>(waves, nt);
    default: return three ? march_fn_t<bf16, 3, 4>(waves, nt) : march_fn_t<bf16, 2, 4>(waves, nt);
    }
}
// blocks of it that a CU holds at once
int march_blocks_per_cu(int storage, int steps, int waves)
{
    int n = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &n, reinterpret_cast<const void *>(march_fn(storage, steps, waves, 1)), 64 * waves, 0);
    return e == hipSuccess && n > 0 ? n : 8 / waves;
}
// Wavefronts of a march block: 8 (one block per CU) or 4 (two or three).  With 4, a row of 256 cells or a
// strip makes a block of one row group, which reads (R + 4) / R = 2 times its own rows; 8 make
// two groups that share their halo rows, 1.5 times.  That pays where the L2 misses of the halo
// rows are on the critical path, in handles larger than the memory-side cache (16 FP32 spheres of
// 256 x 128 x 128: 266 us per step against 273; FP64, 16 spheres 721 against 756, 4 spheres 182
// against 186; four FP32 channels of 1000 x 64 x 64 79 against 85); in it, and in 16-bit storage,
// which is bound by its instructions, independent blocks hide each other's barriers better (one FP32
// sphere: 18.9 against 20.8; 16 in FP16: 178 against 197).
constexpr int64_t kMallBytes = 256 << 20;
int64_t state_bytes(const std::vector<InstDev> &inst, int storage)
{
    int64_t cells = 0;
    for (const InstDev &I : inst) cells += (int64_t)I.pitch * I.ny * I.nz;
    return cells * 7 * kNumBuf * (int64_t)elem_bytes(storage);
}

MarchBox march_box(const InstDev &I, int storage, int waves, int zchunk)
{
    MarchBox m;
    m.nsx = march_strips(I.nx, I.pitch);
    const int rows = march_rows(storage) * (waves / (m.nsx > 1 ? 4 : I.pitch / 64));
    m.nyb = (I.ny + rows - 1) / rows;
    m.nzc = (I.nz + zchunk - 1) / zchunk;
    return m;
}

// Time of one launch with chunks of at most zchunk planes, in iterations of a block: every XCD
// takes an eighth of the blocks, in order, and as one ends its place (a CU holds per_cu blocks) takes
// the next.  A block runs its planes and the K - 1 halo planes at both ends; two on a CU take 1.4
// times as long as one alone (measured: 1.6 from HBM, 1.2 from the memory-side cache); in 16-bit
// storage, where each waits for its own instructions, two take 1.15 and three 1.3 times as long (FP16,
// us per step with the chunks that this gives and with those for two: 160^3 20.7 and 27.9,
// 300 x 96 x 96 16.9 and 20.9, three of 488 x 32 x 32 11.4 and 12.3).  Measurement blocks (surf per
// step, and one per instance) that outnumber the places follow, each a little over an iteration: fewer
// lattice blocks then leave places free for them (FP16 16 boxes of 64^3 with a surface each 22.1 and
// 23.8, 24 of 60 x 48 x 48 25.3 and 27.8; FP64 16 of 55 x 64 x 40 43.9 and 48.5).  Not in FP32, where
// full places are the faster choice all the same (8 boxes of 79 x 64 x 64 23.0 and 28.8).
double march_time(const std::vector<InstDev> &inst, int storage, int64_t surf, int k, int waves, int per_cu,
                  int zchunk)
{
    std::vector<std::pair<int64_t, double>> runs;  // blocks, iterations
    int64_t n = 0;
    for (const InstDev &I : inst) {
        const MarchBox m = march_box(I, storage, waves, zchunk);
        runs.push_back({m.blocks(), (double)(I.nz + m.nzc - 1) / (double)m.nzc +
                                        2.0 * (k - 1) + 1.0});
        n += m.blocks();
    }
    const int places = 32 * per_cu;
    int64_t meas = (k * surf + (int64_t)inst.size()) / (kNumXcd * (waves / 4));
    if (storage == LB_F32 || meas <= places) meas = 0;
    double worst = 0.0;
    size_t r = 0;
    int64_t used = 0;
    for (int x = 0; x < kNumXcd; ++x) {
        std::vector<double> free_at(places, 0.0);  // a heap, the earliest on top
        double last = 0.0;
        for (int64_t k = n / kNumXcd + (x < n % kNumXcd); k > 0; --k) {
            while (used == runs[r].first) {
                ++r;
                used = 0;
            }
            ++used;
            std::pop_heap(free_at.begin(), free_at.end(), std::greater<double>());
            last = std::max(last, free_at.back() += runs[r].second);
            std::push_heap(free_at.begin(), free_at.end(), std::greater<double>());
        }
        for (int64_t m = meas; m > 0; --m) {
            std::pop_heap(free_at.begin(), free_at.end(), std::greater<double>());
            last = std::max(last, free_at.back() += 1.2);
            std::push_heap(free_at.begin(), free_at.end(), std::greater<double>());
        }
        worst = std::max(worst, last);
    }
    const int64_t share = std::min<int64_t>(per_cu, (n + 255) / 256);
    return worst * (1.0 + (elem_bytes(storage) < 4 ? 0.15 : 0.4) * (double)(share - 1));
}

// The chunk length with the shortest such time; handles of very many blocks, where the ends
// hardly matter, take long chunks without trying.  Measured against chunks of a fixed 64 planes
// (FP32, us per step): 16 uneven boxes of 64 to 192 cells a side 180 against 208, four channels of
// 1000 x 64 x 64 85 against 95, one sphere of 256 x 128 x 128 19 against 74.
constexpr int kChunks[] = {128, 96, 64, 48, 40, 32, 28, 24, 20, 16, 12, 10, 8, 6, 5, 4, 3, 2, 1};
int march_zchunk(const std::vector<InstDev> &inst, int storage, int64_t surf, int k, int waves)
{
    int64_t n = 0;
    for (const InstDev &I : inst) n += march_box(I, storage, waves, 64).blocks();
    int best = 64;
    if (n > 8192) return best;
    const int per_cu = march_blocks_per_cu(storage, k, waves);
    double best_time = march_time(inst, storage, surf, k, waves, per_cu, best);
    for (int zc : kChunks) {
        int64_t blocks = 0;
        for (const InstDev &I : inst) blocks += march_box(I, storage, waves, zc).blocks();
        if (blocks > 8192) break;  // and shorter ones, whose halo planes only cost more
        const double time = march_time(inst, storage, surf, k, waves, per_cu, zc);
        if (time < best_time) {
            best_time = time;
            best = zc;
        }
    }
    return best;
}

// Steps of a launch of a handle that is not tuned (FP64 has two only).  An iteration of three
// steps takes 1.2 to 1.4 times as long as one of two, so three pay where the planes computed twice at
// the ends of the chunks do not eat up the launch that is saved.
//  * FP32: where the model's iterations per step are below 0.8 of those with two.  us per step with two
//    and three: 64^3 (0.93) 6.4 and 7.2, 1456 x 32 x 32 (0.83) 12.6 and 17.4, 251 x 64 x 64 (0.83) 11.4
//    and 11.8, 128^3 (0.83) 14.8 and 16.9, 96^3 (0.82) 12.8 and 12.7, two of 128^3 (0.78) 22.9 and 20.4,
//    160^3 (0.73) 31.2 and 27.9, 16 of 256 x 128 x 128 (0.68) 412 and 268.
//  * 16 bit: blocks of two steps leave registers for three on a CU.  Two, unless the states outgrow the
//    memory-side cache, where the traffic of a launch counts, and the schedule does not lose more.
//    FP16 and BF16, two and three: 96^3 10.0 and 11.7, 192^3 27.3 and 32.7, 16 of 64^3 23.7 and 25.6;
//    beyond the cache 16 of 256 x 128 x 128 (0.85) 214 and 178, 4 of them (0.88) 57 and 51, 8 of 192^3
//    (0.96) 178 and 201, 512 x 256 x 256 (0.99) 131 and 140.
int march_depth(const std::vector<InstDev> &inst, int storage, int64_t surf, int waves)
{
    if (march_steps(storage) == 2) return 2;
    auto per_step = [&](int k) {
        return march_time(inst, storage, surf, k, waves, march_blocks_per_cu(storage, k, waves),
                          march_zchunk(inst, storage, surf, k, waves)) / k;
    };
    if (storage == LB_F32) return per_step(3) < 0.8 * per_step(2) ? 3 : 2;
    return state_bytes(inst, storage) > kMallBytes && per_step(3) < 0.92 * per_step(2) ? 3 : 2;
}

// 8 wavefronts where most cells lie in rows that fill a block of 4 and the states outgrow the
// memory-side cache (see kMallBytes)
int march_block_waves(const std::vector<InstDev> &inst, int storage)
{
    if (!march_eight(storage)) return 4;
    int64_t cells = 0, wide = 0;
    for (const InstDev &I : inst) {
        const int64_t c = (int64_t)I.pitch * I.ny * I.nz;
        cells += c;
        if (I.pitch >= 256) wide += c;
    }
    return 2 * wide > cells && state_bytes(inst, storage) > kMallBytes ? 8 : 4;
}

// blocks of a launch: `lattice` blocks, and `meas` measurement blocks of kStepThreads threads side by side
int64_t march_grid(int64_t lattice, int64_t meas, int waves)
{
    const int per = 64 * waves / kStepThreads;
    return lattice + (meas + per - 1) / per;
}

// Launches of `steps` lattice steps by blocks of `waves` wavefronts: the chunks of planes (of zchunk at
// most, 0: what the model prefers) and the blocks of every instance.  Returns false if a launch, with the measurement of as many steps, would
// have 2^32 threads or more.
bool plan_march(lb_wave *h, int steps, int waves, int zchunk = 0)
{
    int &model = h->model_chunk[steps - 2][waves / 8];
    if (!zchunk) {
        if (!model) model = march_zchunk(h->hinst, h->storage, h->lay.n_sb_total, steps, waves);
        zchunk = model;
    }
    std::vector<int> blk0(h->n + 1, 0);
    std::vector<MarchBox> boxes(h->n);
    int64_t total = 0;
    for (int ii = 0; ii < h->n; ++ii) {
        boxes[ii] = march_box(h->hinst[ii], h->storage, waves, zchunk);
        total += boxes[ii].blocks();
        if (total > INT32_MAX) return false;
        blk0[ii + 1] = (int)total;
    }
    if (march_grid(total, h->n + (int64_t)steps * h->lay.n_sb_total, waves) * 64 * waves > (int64_t)UINT32_MAX)
        return false;
    h->march_depth = steps;
    h->march_waves = waves;
    h->march_chunk = zchunk;
    for (SegInfo &sg : h->segs) {
        sg.blk0 = blk0[sg.first];
        sg.bpi = blk0[sg.first + 1] - blk0[sg.first];
        sg.nsx = (int)boxes[sg.first].nsx;
        sg.nyb = (int)boxes[sg.first].nyb;
    }
    h->blk0 = std::move(blk0);
    return true;
}

// Several steps per launch need ny to be a multiple of the rows of a block: kRuleRows rows per
// row group.  (The march kernel itself takes any ny; the rule is the interface's.)
int rule_rows(int storage) { return storage == LB_F32 ? 4 : 2; }

void launch_march(const lb_wave *h, const StepArgs &a, int nst, int meas_blocks, hipStream_t st)
{
    const unsigned blocks = (unsigned)march_grid(a.ntask, meas_blocks, h->march_waves);
    if (blocks > 0)
        hipLaunchKernelGGL(march_fn(h->storage, nst, h->march_waves, h->nt), dim3(blocks),
                           dim3(64 * h->march_waves), 0, st, a);
}

// nst steps of every live box, one block each, with the measurement of the launches before
void launch_resident(const lb_wave *h, const StepArgs &a, int meas_blocks, hipStream_t st)
{
    const dim3 grid((unsigned)resident_grid(a.ntask, meas_blocks)), threads(64 * kResidentWaves);
    switch (h->storage) {
    case LB_F64: hipLaunchKernelGGL(resident_kernel<double>, grid, threads, 0, st, a); break;
    case LB_F32: hipLaunchKernelGGL(resident_kernel<float>, grid, threads, 0, st, a); break;
    case LB_F16: hipLaunchKernelGGL(resident_kernel<_Float16>, grid, threads, 0, st, a); break;
    default: hipLaunchKernelGGL(resident_kernel<bf16>, grid, threads, 0, st, a); break;
    }
}

// The launches of n lattice steps: at most `most` steps each, the shorter ones first.
int next_steps(int64_t n, int most)
{
    if (most == 3) return n % 3 == 0 ? 3 : n == 1 ? 1 : 2;  // 3 m + 1 = 2 + 2 + 3 (m - 1)
    if (most == 2) return n % 2 == 0 ? 2 : 1;
    return 1;
}

int most_steps(const lb_wave *h)
{
    return h->fused == 2 && h->march_ok ? h->march_depth : 1;
}

// Measurement part of the launch whose lattice part starts at t_launch:
// reduce every measured step whose partials an earlier launch wrote
// (steps red .. meas-1), and measure every step whose moments an earlier
// launch stored (steps meas .. t_launch-1).  Both ranges hold the steps of one
// launch at most, and the slots they use differ from those the launch writes.
void plan_measure(lb_wave *h, StepArgs &a, int64_t t_launch)
{
    a.n_red = a.n_sb = a.n_ms = a.n_rs = 0;
    a.meas_off = a.red_off = 0;
    a.sb_inst = h->d_sb_inst;
    a.sb_chunk = h->d_sb_chunk;
    if (!h->any_surf) {
        h->meas = h->red = t_launch;
        return;
    }
    if (h->red < h->meas) {
        a.red_off = (int32_t)(t_launch - h->red);
        a.n_rs = (int32_t)(h->meas - h->red);
        a.n_red = prefix_alive(h, h->red);
        h->red = h->meas;
    }
    if (h->meas < t_launch) {
        a.meas_off = (int32_t)(t_launch - h->meas);
        a.n_ms = (int32_t)(t_launch - h->meas);
        a.n_sb = h->sb_first[prefix_alive(h, h->meas)];
        h->meas = t_launch;
    }
}

// Fill the lattice part of `a` for the steps t .. t+nst-1 (segments of the
// live prefix) and launch, one launch per kMaxSeg segments; the measurement
// blocks ride on the first launch.  nst = 1: wave tasks of step_kernel;
// else blocks of march_kernel (the live prefix is the same for all its steps).
void emit_step(const lb_wave *h, StepArgs a, int64_t t, int32_t dt, int dbuf, int nst,
               hipStream_t st)
{
    const int na = active_prefix(h, t);
    if (h->resident && nst > 1) {
        a.dt = dt;
        a.dbuf = dbuf;
        a.nst = nst;
        a.ntask = na;
        if (a.n_red + a.n_ms * a.n_sb + na > 0)
            launch_resident(h, a, a.n_red + a.n_ms * a.n_sb, st);
        return;
    }
    const bool march = nst > 1;
    auto first_of = [&](const SegInfo &sg) { return march ? sg.blk0 : sg.task0; };
    const int n_active = march ? h->blk0[na] : h->task0[na];
    a.dt = dt;
    a.dbuf = dbuf;
    size_t s = 0;
    bool first = true;
    do {
        const int base = s < h->segs.size() ? first_of(h->segs[s]) : 0;
        int k = 0;
        for (; k < kMaxSeg && s + k < h->segs.size() && first_of(h->segs[s + k]) < n_active; ++k) {
            a.seg[k] = h->segs[s + k];
            a.seg[k].task0 -= march ? 0 : base;
            a.seg[k].blk0 -= march ? base : 0;
        }
        const int end = (s + k < h->segs.size()) ? std::min(first_of(h->segs[s + k]), n_active)
                                                 : n_active;
        a.nseg = k;
        a.ntask = k > 0 ? end - base : 0;
        if (!first) a.n_red = a.n_sb = a.n_ms = a.n_rs = 0;
        const int meas_blocks = a.n_red + a.n_ms * a.n_sb;
        if (march)
            launch_march(h, a, nst, meas_blocks, st);
        else
            launch(h, a, meas_blocks + (a.ntask + 3) / 4, st);
        first = false;
        s += k;
    } while (s < h->segs.size() && first_of(h->segs[s]) < n_active);
    if (h->any_point && !march) launch_point(h, a, st);
}

// Set the device counter to the handle's step and buffer, in stream order.
void set_counter(lb_wave *h)
{
    hipLaunchKernelGGL(set_step_kernel, dim3(1), dim3(64), 0, h->stream, h->d_t, h->t,
                       (int64_t)h->cur);
    h->tdev = h->t;
    h->bufdev = h->cur;
}

// ... if dt would not fit
void sync_counter(lb_wave *h)
{
    if (h->t - h->tdev > (1 << 30) || h->t < h->tdev) set_counter(h);
}

// k steps in n_launch launches are enqueued: advance the host's counters, and note
// where the state of every instance that has just stopped lies.
void advance(lb_wave *h, int64_t k, int n_launch)
{
    const int live = active_prefix(h, h->t);
    h->t += k;
    h->cur = (h->cur + n_launch) & 1;
    for (int ii = active_prefix(h, h->t); ii < live; ++ii) h->stop_buf[ii] = h->cur;
}

// nst lattice steps for every live instance, with the measurement
// of the previous steps folded into the same launch.
int enqueue_step(lb_wave *h, int nst)
{
    const int64_t t = h->t;
    sync_counter(h);
    StepArgs a;
    std::memset(&a, 0, sizeof a);
    a.inst = h->d_inst;
    a.tp = h->d_t;
    plan_measure(h, a, t);
    emit_step(h, a, t, (int32_t)(t - h->tdev), h->cur ^ h->bufdev, nst, h->stream);
    HIP_TRY(hipGetLastError());
    advance(h, nst, 1);
    return LB_OK;
}

// The largest number of steps up to k that one launch can advance: no instance stops inside it.
int fuse_steps(const lb_wave *h, int k)
{
    const int live = active_prefix(h, h->t);
    while (k > 1 && active_prefix(h, h->t + k - 1) != live) --k;
    return k;
}

// Finish the measurement of every completed step (two launches at most).
int flush_measure(lb_wave *h)
{
    while (h->red < h->t) {
        sync_counter(h);
        StepArgs a;
        std::memset(&a, 0, sizeof a);
        a.inst = h->d_inst;
        a.tp = h->d_t;
        a.dt = (int32_t)(h->t - h->tdev);
        plan_measure(h, a, h->t);
        launch(h, a, a.n_red + a.n_ms * a.n_sb, h->stream);
        HIP_TRY(hipGetLastError());
    }
    return LB_OK;
}

// Steps t .. t+k-1 all launch the same blocks, nst steps at a time: the
// measurement runs nst and 2 nst steps behind and no instance stops inside
// the window.
bool steady(const lb_wave *h, int k, int nst)
{
    const int64_t t = h->t;
    if (h->any_surf && (t < 2 * nst || h->meas != t - nst || h->red != t - 2 * nst)) return false;
    for (const InstDev &I : h->hinst) {
        const int64_t ms = I.max_steps;
        if (ms > 0 && ms > t - 2 * nst && ms < t + k) return false;
    }
    return true;
}

// Replay k steady steps, nst at a time, as one captured graph (captured once
// per launch shape on a private stream, launched on the handle's stream).
int replay_steps(lb_wave *h, int k, int nst)
{
    const int64_t t = h->t;
    const int na = active_prefix(h, t);
    const int n_red = h->any_surf ? prefix_alive(h, t - 2 * nst) : 0;
    const int n_sb = h->any_surf ? h->sb_first[prefix_alive(h, t - nst)] : 0;
    hipGraphExec_t exec = nullptr;
    for (auto &g : h->graphs)
        if (g.k == k && g.na == na && g.n_red == n_red && g.n_sb == n_sb && g.nst == nst)
            exec = g.exec;
    if (!exec) {
        if (!h->cap_stream) HIP_TRY(hipStreamCreateWithFlags(&h->cap_stream, hipStreamNonBlocking));
        HIP_TRY(hipStreamBeginCapture(h->cap_stream, hipStreamCaptureModeThreadLocal));
        StepArgs a;
        std::memset(&a, 0, sizeof a);
        a.inst = h->d_inst;
        a.tp = h->d_t;
        a.meas_off = nst;
        a.n_ms = h->any_surf ? nst : 0;
        a.red_off = 2 * nst;
        a.n_rs = h->any_surf ? nst : 0;
        a.n_red = n_red;
        a.n_sb = n_sb;
        a.sb_inst = h->d_sb_inst;
        a.sb_chunk = h->d_sb_chunk;
        for (int j = 0; j < k; j += nst)
            emit_step(h, a, t + j, j, (j / nst) & 1, nst, h->cap_stream);
        hipLaunchKernelGGL(advance_step_kernel, dim3(1), dim3(64), 0, h->cap_stream, h->d_t,
                           (int64_t)k, (int64_t)(k / nst));
        hipGraph_t graph = nullptr;
        hipError_t e = hipStreamEndCapture(h->cap_stream, &graph);
        if (e != hipSuccess) return fail(LB_EDEVICE, "graph capture: %s", hipGetErrorString(e));
        e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
        (void)hipGraphDestroy(graph);
        if (e != hipSuccess) return fail(LB_EDEVICE, "graph instantiate: %s", hipGetErrorString(e));
        h->graphs.push_back({k, na, n_red, n_sb, nst, exec});
    }
    if (h->tdev != t || h->bufdev != h->cur) set_counter(h);
    HIP_TRY(hipGraphLaunch(exec, h->stream));
    advance(h, k, k / nst);
    h->tdev = h->t;
    h->bufdev = h->cur;
    if (h->any_surf) {
        h->meas += k;
        h->red += k;
    } else {
        h->meas = h->red = h->t;
    }
    return LB_OK;
}

// n steps without the launches that finish their measurement
int enqueue_steps(lb_wave *h, int64_t left)
{
    while (left > 0) {
        // a replayed sequence holds launches of nst steps only: the chunk rounded down to them
        const int most = most_steps(h), nst = std::min(most, std::max(h->graph_chunk, 1));
        const int k = h->graph_chunk / nst * nst;
        int st;
        if (h->resident && left >= h->resident_min) {
            const int64_t launches = (left + kResidentSteps - 1) / kResidentSteps;
            const int n = (int)((left + launches - 1) / launches);  // equal shares: no short rest
            st = enqueue_step(h, n);
            left -= n;
        } else if (k >= 2 && left >= k && steady(h, k, nst)) {
            st = replay_steps(h, k, nst);
            left -= k;
        } else {
            // before the first replay launches of its size fill the measurement pipeline
            int n = k >= 2 && left >= k ? nst : next_steps(left, most);
            n = fuse_steps(h, n);
            st = enqueue_step(h, n);
            left -= n;
        }
        if (st != LB_OK) return st;
    }
    return LB_OK;
}

void drop_graphs(lb_wave *h)
{
    for (auto &g : h->graphs) (void)hipGraphExecDestroy(g.exec);
    h->graphs.clear();
}

int zero_region(lb_wave *h, size_t off, size_t bytes)
{
    if (bytes == 0) return LB_OK;
    const int64_t n16 = (int64_t)((bytes + 15) / 16);
    const int blocks = (int)std::min<int64_t>((n16 + 255) / 256, 4096);
    hipLaunchKernelGGL(zero_kernel, dim3(blocks), dim3(256), 0, h->stream,
                       reinterpret_cast<uint4 *>(h->ws + off), n16);
    HIP_TRY(hipGetLastError());
    return LB_OK;
}

int zero_state(lb_wave *h)
{
    for (int i = 0; i < h->n; ++i) {
        const InstPlan &P = h->lay.p[i];
        const lb_wave_desc &d = h->desc[i];
        const size_t buf = elem_bytes(d.storage) * (size_t)P.plane * (2 * d.dim + 1);
        for (int b = 0; b < kNumBuf; ++b) {
            int st = zero_region(h, P.off_buf[b], buf);
            if (st) return st;
        }
        int st = zero_region(h, P.off_trace, sizeof(double) * 3 * (size_t)d.trace_steps);
        if (st) return st;
    }
    int st = zero_region(h, h->lay.off_acc, sizeof(AccDev) * h->n);
    if (st) return st;
    h->t = h->meas = h->red = 0;
    h->cur = 0;
    h->nan_seen = false;
    set_counter(h);
    return LB_OK;
}

}  // namespace

// error reporting shared with the MLP translation unit
int lbw_fail_msg(int code, const char *msg) { return fail(code, "%s", msg); }

// ===========================================================================
// C ABI
// ===========================================================================
extern "C" {

const char *lb_last_error(void) { return g_err.c_str(); }

int lb_wave_check(const lb_wave_desc *descs, int32_t n_inst)
{
    g_err.clear();
    return check_all(descs, n_inst);
}

size_t lb_wave_workspace_bytes(const lb_wave_desc *descs, int32_t n_inst)
{
    if (check_all(descs, n_inst) != LB_OK) return 0;
    return plan(descs, n_inst).total;
}

int lb_wave_create(const lb_wave_desc *descs, int32_t n_inst, void *dev_workspace,
                   size_t workspace_bytes, void *hip_stream, lb_wave **out)
{
    g_err.clear();
    if (!out) return fail(LB_EINVAL, "out is NULL");
    *out = nullptr;
    int st = check_all(descs, n_inst);
    if (st != LB_OK) return st;
    Layout L = plan(descs, n_inst);
    if (!dev_workspace) return fail(LB_ENOMEM, "workspace is NULL");
    if (reinterpret_cast<uintptr_t>(dev_workspace) % kAlign)
        return fail(LB_ENOMEM, "workspace must be 256-byte aligned");
    if (workspace_bytes < L.total)
        return fail(LB_ENOMEM, "workspace has %zu bytes, needs %zu", workspace_bytes, L.total);

    lb_wave *h = new lb_wave();
    h->n = n_inst;
    h->dim = descs[0].dim;
    h->storage = descs[0].storage;
    h->ws = static_cast<char *>(dev_workspace);
    h->ws_bytes = workspace_bytes;
    h->stream = static_cast<hipStream_t>(hip_stream);
    h->lay = L;
    h->resident = L.resident;
    if (L.resident) h->resident_min = resident_min(descs, n_inst);
    h->desc.assign(descs, descs + n_inst);
    for (auto &d : h->desc) {  // the host arrays are not kept
        d.c_field = nullptr;
        d.surf_xyz = d.surf_normal = d.surf_area = nullptr;
    }
    h->d_inst = reinterpret_cast<InstDev *>(h->ws + L.off_inst);
    h->d_acc = reinterpret_cast<AccDev *>(h->ws + L.off_acc);
    h->d_sb_inst = reinterpret_cast<int32_t *>(h->ws + L.off_sbtab);
    h->d_sb_chunk = h->d_sb_inst + L.n_sb_total;
    h->d_t = reinterpret_cast<int64_t *>(h->ws + L.off_tdev);
    h->vx = 1;

    // internal order: longest runs first (so the active set is a prefix),
    // equal shapes adjacent (so they share one segment of the launch)
    h->order.resize(n_inst);
    std::iota(h->order.begin(), h->order.end(), 0);
    auto key_steps = [&](int i) {
        return descs[i].max_steps > 0 ? descs[i].max_steps : std::numeric_limits<int64_t>::max();
    };
    std::stable_sort(h->order.begin(), h->order.end(), [&](int a, int b) {
        if (key_steps(a) != key_steps(b)) return key_steps(a) > key_steps(b);
        if (descs[a].nx != descs[b].nx) return descs[a].nx > descs[b].nx;
        if (descs[a].ny != descs[b].ny) return descs[a].ny > descs[b].ny;
        return descs[a].nz > descs[b].nz;
    });
    h->pos.resize(n_inst);
    for (int i = 0; i < n_inst; ++i) h->pos[h->order[i]] = i;

    // per-instance device records, surface stencils, sound-speed boxes
    std::vector<std::vector<uint8_t>> host_blobs;
    std::vector<size_t> blob_off;
    h->hinst.resize(n_inst);
    h->scale.resize(n_inst);
    h->task0.assign(n_inst + 1, 0);
    h->stop_buf.assign(n_inst, 0);
    for (int ii = 0; ii < n_inst; ++ii) {
        const int u = h->order[ii];
        const lb_wave_desc &d = descs[u];
        const InstPlan &P = L.p[u];
        InstDev &I = h->hinst[ii];
        std::memset(&I, 0, sizeof I);
        I.dim = d.dim;
        I.nx = d.nx;
        I.ny = d.ny;
        I.nz = d.nz;
        I.pitch = P.pitch;
        I.xbc = d.xbc;
        I.plane = P.plane;
        for (int b = 0; b < kNumBuf; ++b) I.buf[b] = h->ws + P.off_buf[b];
        I.c0sq = d.c0 * d.c0;
        for (int a = 0; a < 3; ++a) {
            I.bb_lo[a] = P.box.lo[a];
            I.bb_n[a] = P.box.n[a];
        }
        I.c2box = h->ws + P.off_box;
        const double sc = storage_scale(d);
        h->scale[u] = sc;
        I.src_amp = d.rho_a * sc;
        I.omega = d.omega;
        I.wall_phi = d.wall_phi;
        I.max_steps = d.max_steps;
        I.src_point = d.src_kind == LB_SRC_POINT ? 1 : 0;
        for (int a = 0; a < 3; ++a) I.src_pt[a] = I.src_point ? d.src_cell[a] : 0;
        if (I.src_point) h->any_point = true;
        for (int a = 0; a < 3; ++a) {
            I.mb_lo[a] = P.mbox.lo[a];
            I.mb_n[a] = P.mbox.n[a];
        }
        I.mom = h->ws + P.off_mom;
        I.mom_bytes = (int64_t)P.mom_bytes;
        I.slots = L.slots;
        I.resident = L.resident ? resident_of(d) : 0;
        I.n_surf = d.n_surf;
        I.n_chunks = P.n_chunks;
        I.surf = reinterpret_cast<const SurfPt *>(h->ws + P.off_surf);
        I.part = reinterpret_cast<double *>(h->ws + P.off_part);
        I.c0sq_force = d.c0 * d.c0;
        I.force_scale = -1.0 / (d.rho0 * sc * sc);
        I.avg_start = d.avg_start;
        I.acc = h->d_acc + ii;
        I.trace = reinterpret_cast<double *>(h->ws + P.off_trace);
        I.trace_cap = d.trace_steps;
        if (d.n_surf > 0) h->any_surf = true;

        const int xsegs = (d.nx + 63) / 64;
        h->task0[ii + 1] = h->task0[ii] + xsegs * d.ny * d.nz;

        // surface stencils
        if (d.n_surf > 0) {
            std::vector<uint8_t> blob(sizeof(SurfPt) * d.n_surf);
            SurfPt *sp = reinterpret_cast<SurfPt *>(blob.data());
            for (int k = 0; k < d.n_surf; ++k) {
                stencil_in_box(d, d.surf_xyz + 3 * k, P.mbox, sp[k]);
                for (int a = 0; a < 3; ++a) sp[k].nA[a] = d.surf_normal[3 * k + a] * d.surf_area[k];
            }
            host_blobs.push_back(std::move(blob));
            blob_off.push_back(P.off_surf);
        }
        // compact c^2 table in the compute type, c0^2 after every plane
        if (P.box.cells() > 0) {
            const size_t cb = compute_bytes(d.storage);
            std::vector<uint8_t> blob(cb * c2_cells(P.box));
            size_t q = 0;
            auto put = [&](double c2) {
                if (cb == 8) {
                    std::memcpy(blob.data() + 8 * q, &c2, 8);
                } else {
                    const float f = (float)c2;
                    std::memcpy(blob.data() + 4 * q, &f, 4);
                }
                ++q;
            };
            for (int z = 0; z < P.box.n[2]; ++z) {
                for (int y = 0; y < P.box.n[1]; ++y)
                    for (int x = 0; x < P.box.n[0]; ++x) {
                        const int gx = P.box.lo[0] + x, gy = P.box.lo[1] + y, gz = P.box.lo[2] + z;
                        double c;
                        if (d.c_field)
                            c = d.c_field[((size_t)gz * d.ny + gy) * d.nx + gx];
                        else
                            c = object_c(d, gx, gy, gz);
                        put(c * c);
                    }
                put(d.c0 * d.c0);  // rounded as the kernels round c0^2
            }
            host_blobs.push_back(std::move(blob));
            blob_off.push_back(P.off_box);
        }
    }
    // surface block table in internal order
    std::vector<int32_t> sbtab(2 * (size_t)L.n_sb_total);
    h->sb_first.assign(n_inst + 1, 0);
    for (int ii = 0; ii < n_inst; ++ii) {
        const int nc = L.p[h->order[ii]].n_chunks;
        h->sb_first[ii + 1] = h->sb_first[ii] + nc;
        for (int c = 0; c < nc; ++c) {
            sbtab[h->sb_first[ii] + c] = ii;
            sbtab[L.n_sb_total + h->sb_first[ii] + c] = c;
        }
    }
    if (L.n_sb_total > 0) {
        std::vector<uint8_t> blob(sizeof(int32_t) * sbtab.size());
        std::memcpy(blob.data(), sbtab.data(), blob.size());
        host_blobs.push_back(std::move(blob));
        blob_off.push_back(L.off_sbtab);
    }
    // segments: maximal runs of equal shape in internal order
    for (int ii = 0; ii < n_inst; ++ii) {
        const InstDev &I = h->hinst[ii];
        if (ii == 0 || I.nx != h->hinst[ii - 1].nx || I.ny != h->hinst[ii - 1].ny ||
            I.nz != h->hinst[ii - 1].nz) {
            SegInfo sg;
            std::memset(&sg, 0, sizeof sg);
            sg.task0 = h->task0[ii];
            sg.first = ii;
            sg.nx = I.nx;
            sg.ny = I.ny;
            sg.nz = I.nz;
            sg.xsegs = (I.nx + 63) / 64;
            sg.tpi = sg.xsegs * I.ny * I.nz;
            h->segs.push_back(sg);
        }
    }
    // march decomposition: row blocks, chunks of planes, strips
    {
        h->fused_ok = h->dim == 3 && !h->any_point;
        bool fits = true;
        for (const InstDev &I : h->hinst) {
            const int groups = I.pitch > kMarchMaxPitch ? 1 : 4 / (I.pitch / 64);
            if (I.xbc != LB_XBC_DRIVEN || I.ny % (rule_rows(h->storage) * groups)) h->fused_ok = false;
            // lane offsets inside one plane, of the state and of the c^2 table, are 32-bit byte counts
            if ((int64_t)I.ny * I.pitch * (int64_t)elem_bytes(h->storage) > (int64_t)UINT32_MAX ||
                c2_plane(I.bb_n[0], I.bb_n[1]) * (int64_t)compute_bytes(h->storage) > (int64_t)UINT32_MAX)
                fits = false;
        }
        if (h->fused_ok && fits) {
            const int waves = march_block_waves(h->hinst, h->storage);
            h->march_ok = plan_march(h, march_depth(h->hinst, h->storage, L.n_sb_total, waves), waves) ||
                          plan_march(h, 2, 4);
            h->fused_ok = h->march_ok;  // refused, not run one step at a time
        }
    }

    auto cleanup = [&](int code) {
        delete h;
        return code;
    };
    hipError_t e = hipMemcpyAsync(h->ws + L.off_inst, h->hinst.data(), sizeof(InstDev) * n_inst,
                                  hipMemcpyHostToDevice, h->stream);
    for (size_t b = 0; b < host_blobs.size() && e == hipSuccess; ++b)
        e = hipMemcpyAsync(h->ws + blob_off[b], host_blobs[b].data(), host_blobs[b].size(),
                           hipMemcpyHostToDevice, h->stream);
    if (e != hipSuccess) return cleanup(fail(LB_EDEVICE, "upload failed: %s", hipGetErrorString(e)));
    st = zero_state(h);
    if (st != LB_OK) return cleanup(st);
    e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess)
        return cleanup(fail(LB_EDEVICE, "create: %s", hipGetErrorString(e)));
    *out = h;
    return LB_OK;
}

int lb_wave_step_n(lb_wave *h, int64_t n_steps)
{
    if (!h) return fail(LB_EINVAL, "handle is NULL");
    if (n_steps < 0) return fail(LB_EINVAL, "n_steps < 0");
    if (h->nan_seen) return fail(LB_ENAN, "a previous force was not finite");
    const int st = enqueue_steps(h, n_steps);
    return st ? st : flush_measure(h);
}

int lb_wave_set_steps_per_launch(lb_wave *h, int32_t k)
{
    if (!h) return fail(LB_EINVAL, "handle is NULL");
    if (k != 1 && k != 2) return fail(LB_EINVAL, "steps per launch must be 1 or 2");
    if (k == 2 && !h->fused_ok)
        return fail(LB_EINVAL, "several steps per launch need 3D instances with driven x sheets "
                               "and ny a multiple of the row block, few enough for one grid");
    if (k != h->fused) drop_graphs(h);
    h->fused = k;
    return LB_OK;
}

int lb_wave_get_steps_per_launch(const lb_wave *h, int32_t *k)
{
    if (!h || !k) return fail(LB_EINVAL, "NULL argument");
    *k = h->fused;
    return LB_OK;
}

int lb_wave_get_launch_steps(const lb_wave *h, int32_t *k)
{
    if (!h || !k) return fail(LB_EINVAL, "NULL argument");
    *k = most_steps(h);
    return LB_OK;
}

int lb_wave_set_launch_plan(lb_wave *h, int32_t steps, int32_t waves)
{
    if (!h) return fail(LB_EINVAL, "handle is NULL");
    if (!h->march_ok) return fail(LB_EINVAL, "this handle runs one step per launch");
    if (steps < 2 || steps > march_steps(h->storage))
        return fail(LB_EINVAL, "steps must lie in 2 .. %d", march_steps(h->storage));
    if (waves != 4 && (waves != 8 || !march_eight(h->storage)))
        return fail(LB_EINVAL, "waves must be 4%s", march_eight(h->storage) ? " or 8" : "");
    drop_graphs(h);
    if (!plan_march(h, steps, waves)) return fail(LB_EINVAL, "too many blocks in a launch");
    return LB_OK;
}

int lb_wave_get_launch_plan(const lb_wave *h, int32_t *steps, int32_t *waves)
{
    if (!h || !steps || !waves) return fail(LB_EINVAL, "NULL argument");
    *steps = h->march_ok ? h->march_depth : 1;
    *waves = h->march_ok ? h->march_waves : 0;
    return LB_OK;
}

int lb_wave_set_graph(lb_wave *h, int32_t chunk)
{
    if (!h) return fail(LB_EINVAL, "handle is NULL");
    if (chunk < 0 || chunk == 1 || chunk > 4096) return fail(LB_EINVAL, "chunk must be 0 or 2..4096");
    if (chunk != h->graph_chunk) drop_graphs(h);
    h->graph_chunk = chunk;
    return LB_OK;
}

int lb_surface_force(lb_wave *h, double *F_avg, int64_t *n_accum)
{
    if (!h) return fail(LB_EINVAL, "handle is NULL");
    if (!F_avg) return fail(LB_EINVAL, "F_avg is NULL");
    std::vector<AccDev> acc(h->n);
    HIP_TRY(hipMemcpyAsync(acc.data(), h->d_acc, sizeof(AccDev) * h->n, hipMemcpyDeviceToHost,
                           h->stream));
    HIP_TRY(hipStreamSynchronize(h->stream));
    int st = LB_OK;
    for (int u = 0; u < h->n; ++u) {
        const AccDev &A = acc[h->pos[u]];
        if (n_accum) n_accum[u] = A.n;
        for (int a = 0; a < 3; ++a) F_avg[3 * u + a] = A.n > 0 ? A.sum[a] / (double)A.n : 0.0;
        if (A.nan) {
            h->nan_seen = true;
            st = fail(LB_ENAN, "instance %d: non-finite force", u);
        } else if (A.n == 0 && st == LB_OK) {
            st = fail(LB_EEMPTY, "instance %d: no step accumulated", u);
        }
    }
    return st;
}

int lb_wave_destroy(lb_wave *h)
{
    delete h;
    return LB_OK;
}

int lb_wave_steps_done(const lb_wave *h, int64_t *t)
{
    if (!h || !t) return fail(LB_EINVAL, "NULL argument");
    *t = h->t;
    return LB_OK;
}

int lb_wave_reset(lb_wave *h)
{
    if (!h) return fail(LB_EINVAL, "handle is NULL");
    return zero_state(h);
}

int lb_wave_state_view(const lb_wave *h, int32_t inst, lb_state_view *v)
{
    if (!h || !v) return fail(LB_EINVAL, "NULL argument");
    if (inst < 0 || inst >= h->n) return fail(LB_EINVAL, "instance out of range");
    const int ii = h->pos[inst];
    const InstPlan &P = h->lay.p[inst];
    v->offset_bytes = P.off_buf[state_buf(h, ii)];
    v->plane_bytes = elem_bytes(h->storage) * (size_t)P.plane;
    v->pitch = P.pitch;
    v->elem_bytes = (int32_t)elem_bytes(h->storage);
    v->scale = h->scale[inst];
    return LB_OK;
}

int lb_wave_get_state(lb_wave *h, int32_t inst, double *host_fnew)
{
    if (!h || !host_fnew) return fail(LB_EINVAL, "NULL argument");
    if (inst < 0 || inst >= h->n) return fail(LB_EINVAL, "instance out of range");
    lb_state_view v;
    int st = lb_wave_state_view(h, inst, &v);
    if (st) return st;
    const lb_wave_desc &d = h->desc[inst];
    const int Q = 2 * d.dim + 1;
    std::vector<uint8_t> raw(v.plane_bytes * Q);
    HIP_TRY(hipMemcpyAsync(raw.data(), h->ws + v.offset_bytes, raw.size(), hipMemcpyDeviceToHost,
                           h->stream));
    HIP_TRY(hipStreamSynchronize(h->stream));
    const double inv = 1.0 / v.scale;
    size_t c = 0;
    for (int z = 0; z < d.nz; ++z)
        for (int y = 0; y < d.ny; ++y)
            for (int x = 0; x < d.nx; ++x, ++c) {
                const size_t e = ((size_t)z * d.ny + y) * v.pitch + x;
                for (int i = 0; i < Q; ++i)
                    host_fnew[c * Q + i] =
                        load_host(raw.data() + i * v.plane_bytes + e * v.elem_bytes, h->storage) * inv;
            }
    return LB_OK;
}

int lb_wave_set_state(lb_wave *h, int32_t inst, const double *host_fnew)
{
    if (!h || !host_fnew) return fail(LB_EINVAL, "NULL argument");
    if (inst < 0 || inst >= h->n) return fail(LB_EINVAL, "instance out of range");
    lb_state_view v;
    int st = lb_wave_state_view(h, inst, &v);
    if (st) return st;
    const lb_wave_desc &d = h->desc[inst];
    const int Q = 2 * d.dim + 1;
    std::vector<uint8_t> raw(v.plane_bytes * Q, 0);
    size_t c = 0;
    for (int z = 0; z < d.nz; ++z)
        for (int y = 0; y < d.ny; ++y)
            for (int x = 0; x < d.nx; ++x, ++c) {
                const size_t e = ((size_t)z * d.ny + y) * v.pitch + x;
                for (int i = 0; i < Q; ++i)
                    store_host(raw.data() + i * v.plane_bytes + e * v.elem_bytes, h->storage,
                               host_fnew[c * Q + i] * v.scale);
            }
    HIP_TRY(hipMemcpyAsync(h->ws + v.offset_bytes, raw.data(), raw.size(), hipMemcpyHostToDevice,
                           h->stream));
    HIP_TRY(hipStreamSynchronize(h->stream));
    return LB_OK;
}

int lb_wave_force_trace(lb_wave *h, int32_t inst, double *host_F, int64_t n)
{
    if (!h || !host_F) return fail(LB_EINVAL, "NULL argument");
    if (inst < 0 || inst >= h->n) return fail(LB_EINVAL, "instance out of range");
    if (n < 0 || n > h->desc[inst].trace_steps)
        return fail(LB_EINVAL, "n exceeds the trace capacity");
    if (n == 0) return LB_OK;
    HIP_TRY(hipMemcpyAsync(host_F, h->ws + h->lay.p[inst].off_trace, sizeof(double) * 3 * n,
                           hipMemcpyDeviceToHost, h->stream));
    HIP_TRY(hipStreamSynchronize(h->stream));
    return LB_OK;
}

int lb_wave_probe_rho(lb_wave *h, int32_t inst, const int64_t *dev_cells, int32_t n_cells,
                      double *dev_out)
{
    if (!h) return fail(LB_EINVAL, "handle is NULL");
    if (inst < 0 || inst >= h->n) return fail(LB_EINVAL, "instance out of range");
    if (n_cells < 0 || (n_cells > 0 && (!dev_cells || !dev_out)))
        return fail(LB_EINVAL, "probe: bad arguments");
    if (n_cells == 0) return LB_OK;
    const int ii = h->pos[inst];
    const InstPlan &P = h->lay.p[inst];
    const lb_wave_desc &d = h->desc[inst];
    const void *buf = h->ws + P.off_buf[state_buf(h, ii)];
    const int64_t ncell = (int64_t)d.nx * d.ny * (d.dim == 3 ? d.nz : 1);
    const int Q = 2 * d.dim + 1;
    const dim3 grid((unsigned)((n_cells + 255) / 256)), blk(256);
    switch (h->storage) {
    case LB_F64:
        hipLaunchKernelGGL(probe_rho_kernel<double>, grid, blk, 0, h->stream, buf, P.plane, Q,
                           d.nx, ncell, P.pitch, dev_cells, n_cells, h->scale[inst], dev_out);
        break;
    case LB_F32:
        hipLaunchKernelGGL(probe_rho_kernel<float>, grid, blk, 0, h->stream, buf, P.plane, Q,
                           d.nx, ncell, P.pitch, dev_cells, n_cells, h->scale[inst], dev_out);
        break;
    case LB_F16:
        hipLaunchKernelGGL(probe_rho_kernel<_Float16>, grid, blk, 0, h->stream, buf, P.plane, Q,
                           d.nx, ncell, P.pitch, dev_cells, n_cells, h->scale[inst], dev_out);
        break;
    default:
        hipLaunchKernelGGL(probe_rho_kernel<bf16>, grid, blk, 0, h->stream, buf, P.plane, Q,
                           d.nx, ncell, P.pitch, dev_cells, n_cells, h->scale[inst], dev_out);
        break;
    }
    HIP_TRY(hipGetLastError());
    return LB_OK;
}

int lb_wave_set_variant(lb_wave *h, int32_t cells_per_lane, int32_t x_mode, int32_t nontemporal)
{
    if (!h) return fail(LB_EINVAL, "handle is NULL");
    if (cells_per_lane != 1 && cells_per_lane != 2 && cells_per_lane != 4)
        return fail(LB_EINVAL, "cells_per_lane must be 1, 2 or 4");
    if (x_mode != 0 && x_mode != 1) return fail(LB_EINVAL, "x_mode must be 0 or 1");
    if (x_mode == 1 && elem_bytes(h->storage) < 4)
        return fail(LB_EINVAL, "x_mode 1 needs 4- or 8-byte storage");
    if (nontemporal < 0 || nontemporal > 2) return fail(LB_EINVAL, "nontemporal must be 0, 1 or 2");
    // the task table and any captured sequence depend on the variant
    drop_graphs(h);
    h->vx = cells_per_lane;
    h->xm = x_mode;
    h->nt = nontemporal;
    const int w = 64 * cells_per_lane;
    for (int ii = 0; ii < h->n; ++ii) {
        const InstDev &I = h->hinst[ii];
        h->task0[ii + 1] = h->task0[ii] + ((I.nx + w - 1) / w) * I.ny * I.nz;
    }
    for (auto &sg : h->segs) {
        sg.task0 = h->task0[sg.first];
        sg.xsegs = (sg.nx + w - 1) / w;
        sg.tpi = sg.xsegs * sg.ny * sg.nz;
    }
    return LB_OK;
}

int lb_wave_get_variant(const lb_wave *h, int32_t *cells_per_lane, int32_t *x_mode,
                        int32_t *nontemporal)
{
    if (!h) return fail(LB_EINVAL, "handle is NULL");
    if (cells_per_lane) *cells_per_lane = h->vx;
    if (x_mode) *x_mode = h->xm;
    if (nontemporal) *nontemporal = h->nt;
    return LB_OK;
}

int lb_wave_set_tile(lb_wave *h, int32_t cells_per_lane)
{
    if (!h) return fail(LB_EINVAL, "handle is NULL");
    return lb_wave_set_variant(h, cells_per_lane, h->xm, h->nt);
}

int lb_wave_get_tile(const lb_wave *h, int32_t *cells_per_lane)
{
    if (!h || !cells_per_lane) return fail(LB_EINVAL, "NULL argument");
    *cells_per_lane = h->vx;
    return LB_OK;
}

int lb_wave_autotune(lb_wave *h, int32_t n_trial, double *best_ms)
{
    if (!h) return fail(LB_EINVAL, "handle is NULL");
    if (n_trial < 1) return fail(LB_EINVAL, "n_trial must be >= 1");
    if (h->nan_seen) return fail(LB_ENAN, "a previous force was not finite");
    struct Scope {  // plain launches of the step or march kernel while tuning
        lb_wave *h;
        int chunk;
        hipEvent_t e0 = nullptr, e1 = nullptr;
        explicit Scope(lb_wave *w) : h(w), chunk(w->graph_chunk)
        {
            h->graph_chunk = 0;
            h->resident = false;
        }
        ~Scope()
        {
            h->graph_chunk = chunk;
            h->resident = h->lay.resident;
            if (e0) (void)hipEventDestroy(e0);
            if (e1) (void)hipEventDestroy(e1);
        }
    } scope(h);
    HIP_TRY(hipEventCreate(&scope.e0));
    HIP_TRY(hipEventCreate(&scope.e1));
    // ms per step of `steps` steps after `warm` others, the least of `repeats` runs, each from step 0
    // (no instance has stopped) and without the launches that finish the measurement of a call: in
    // a long run they do not count.  The populations move on; they are reset at the end.
    auto time_it = [&](int warm, int steps, int repeats, double *per) -> int {
        *per = 1e300;
        for (int r = 0; r < repeats; ++r) {
            h->t = h->meas = h->red = 0;
            set_counter(h);
            int st = enqueue_steps(h, warm);
            if (st) return st;
            HIP_TRY(hipEventRecord(scope.e0, h->stream));
            if ((st = enqueue_steps(h, steps))) return st;
            HIP_TRY(hipEventRecord(scope.e1, h->stream));
            if ((st = flush_measure(h))) return st;
            HIP_TRY(hipEventSynchronize(scope.e1));
            float ms = 0.f;
            HIP_TRY(hipEventElapsedTime(&ms, scope.e0, scope.e1));
            *per = std::min(*per, (double)ms / steps);
        }
        return LB_OK;
    };
    struct Choice {
        int cells, x_mode, nt, steps, waves;  // waves of a march block, 0: step_kernel
        int chunk = 0;                        // planes of a march block, 0: what the model prefers
        double ms = 1e300;                    // per step
    };
    auto apply = [&](const Choice &c) -> int {
        int st = lb_wave_set_steps_per_launch(h, c.steps > 1 ? 2 : 1);
        if (!st && c.steps > 1) {
            st = lb_wave_set_launch_plan(h, c.steps, c.waves);
            if (!st && c.chunk && c.chunk != h->march_chunk && !plan_march(h, c.steps, c.waves, c.chunk))
                st = fail(LB_EINVAL, "too many blocks in a launch");
        }
        return st ? st : lb_wave_set_variant(h, c.cells, c.x_mode, c.nt);
    };
    int64_t life = INT32_MAX;  // steps until the first instance stops
    for (const InstDev &I : h->hinst)
        if (I.max_steps > 0) life = std::min(life, I.max_steps);
    auto whole = [&](double n, int steps) {  // launches of `steps` for n steps, while all instances live
        const int64_t most = std::max<int64_t>(steps, (life - steps) / steps * steps);
        return (int)std::min((int64_t)std::ceil(n / steps) * steps, most);
    };

    // every plan of the march kernel (which number of steps and of wavefronts wins depends on how the
    // boxes divide over the chip), and every variant of the step kernel
    const int xm_max = elem_bytes(h->storage) >= 4 ? 1 : 0;
    std::vector<Choice> cand;
    for (int steps = 2; h->march_ok && steps <= march_steps(h->storage); ++steps)
        for (int waves = 4; waves <= (march_eight(h->storage) ? 8 : 4); waves += 4)
            for (int nt = 0; nt <= 1; ++nt) cand.push_back({1, xm_max, nt, steps, waves});
    const size_t n_plans = cand.size();
    // Only short calls of a handle with a resident kernel use a variant, and up to 2048 wave tasks, two
    // per SIMD, the first is within 2% of the best (us per step in calls of six, first / best / worst:
    // FP64 one box of 128 x 64 5.5 / 5.4 / 7.0, 16 boxes 6.9 / 6.8 / 7.9, 32 boxes 8.2 / 7.6 / 9.6): the
    // trials of the others would take longer than many a run.
    const bool first_only = h->lay.resident && one_step_tasks(h, 64) <= 2048;
    for (int cpl : {1, 2, 4})
        for (int xm = 0; xm <= xm_max; ++xm)
            for (int nt = 0; nt <= 2; ++nt)
                if (!first_only || cpl + xm + nt == 1) cand.push_back({cpl, xm, nt, 1, 0});
    double win = 1e300;
    int st = LB_OK;
    for (Choice &c : cand) {
        st = apply(c);
        if (st == LB_EINVAL && c.steps > 1) continue;  // too many blocks for one grid
        if (st) return st;
        const int warm = std::max(2, c.steps);
        // where a trial is long, a first look at three steps or one launch: what is a quarter slower is
        // not looked at again
        if (n_trial * win > 0.1 && win < 1e300) {
            if ((st = time_it(warm, whole(3, c.steps), 1, &c.ms))) return st;
            if (c.ms > 1.25 * win + 0.003) continue;
        }
        if ((st = time_it(warm, whole(n_trial, c.steps), 1, &c.ms))) return st;
        win = std::min(win, c.ms);
    }
    const auto faster = [](const Choice &x, const Choice &y) { return x.ms < y.ms; };
    Choice best = *std::min_element(cand.begin(), cand.end(), faster);
    if (n_plans > 0) {
        Choice plan = *std::min_element(cand.begin(), cand.begin() + n_plans, faster);
        // Again over at least 200 us, the least of two runs, where steps are short: the first three of
        // those within 5%, then the winner's chunks of planes a little shorter or longer.
        const bool brief = n_trial * best.ms < 2.0;
        auto again = [&](Choice &c) -> int {
            const int st = apply(c);
            const double n = std::max((double)n_trial, std::min(96.0, 0.2 / best.ms));
            return st ? st : time_it(c.steps, whole(n, c.steps), brief ? 2 : 1, &c.ms);
        };
        if (brief) {
            std::stable_sort(cand.begin(), cand.end(), faster);
            size_t near = 1;
            while (near < 3 && near < cand.size() && cand[near].ms < 1.05 * cand[0].ms) ++near;
            cand.resize(near);
            for (Choice &c : cand)
                if ((st = again(c))) return st;
            best = *std::min_element(cand.begin(), cand.end(), faster);
        }
        if (best.steps > 1) {
            if ((st = apply(best))) return st;
            best.chunk = h->march_chunk;
            const int n_chunks = (int)(sizeof kChunks / sizeof *kChunks);
            const int here = (int)(std::find(kChunks, kChunks + n_chunks, best.chunk) - kChunks);
            for (int dir : {1, -1}) {
                int blocks = h->blk0[h->n];
                for (int i = here + dir; i >= 0 && i < n_chunks; i += dir) {
                    Choice c = best;
                    c.chunk = kChunks[i];
                    st = apply(c);
                    if (st == LB_EINVAL) break;  // too many blocks for one grid
                    if (st) return st;
                    if (h->blk0[h->n] == blocks) continue;  // the same chunks
                    blocks = h->blk0[h->n];
                    if ((st = again(c))) return st;
                    if (c.ms > 0.995 * best.ms) break;
                    best = c;
                }
                if (best.chunk != kChunks[here]) break;
                if ((st = apply(best))) return st;
            }
            plan = best;
        }
        win = best.ms;
        if ((st = apply(plan))) return st;  // kept, also where one step per launch wins
    }
    if ((st = apply(best))) return st;
    if (h->lay.resident) {  // long calls run the resident kernel, whatever the variant
        h->resident = true;
        double ms = 0.0;
        if ((st = time_it(kResidentSteps, kResidentSteps, 1, &ms))) return st;
        win = std::min(win, ms);
    }
    if (best_ms) *best_ms = win;
    if ((st = zero_state(h))) return st;
    HIP_TRY(hipStreamSynchronize(h->stream));
    return LB_OK;
}

int lb_stream_copy(const void *dev_src, void *dev_dst, size_t bytes, void *hip_stream)
{
    if (!dev_src || !dev_dst) return fail(LB_EINVAL, "NULL pointer");
    if (bytes % 16 || reinterpret_cast<uintptr_t>(dev_src) % 16 ||
        reinterpret_cast<uintptr_t>(dev_dst) % 16)
        return fail(LB_EINVAL, "pointers and size must be multiples of 16 bytes");
    const int64_t n16 = (int64_t)(bytes / 16);
    if (n16 == 0) return LB_OK;
    constexpr int UNR = 4;
    const int64_t blocks = (n16 + 256 * UNR - 1) / (256 * UNR);
    if (blocks > INT32_MAX) return fail(LB_EINVAL, "copy too large");
    // non-temporal loads and stores: the fastest plain copy measured on this chip (6.2 TB/s
    // against 5.75 with cached accesses, at 1.75 GiB each way)
    hipLaunchKernelGGL((copy_kernel<UNR, true>), dim3((unsigned)blocks), dim3(256), 0,
                       static_cast<hipStream_t>(hip_stream), static_cast<const word16 *>(dev_src),
                       static_cast<word16 *>(dev_dst), n16);
    HIP_TRY(hipGetLastError());
    return LB_OK;
}

size_t lb_cavity_workspace_bytes(int32_t nx)
{
    if (nx < 16 || nx > kCavMaxNx) return 0;
    return align_up(sizeof(double) * 2 * (size_t)nx);
}

}  // extern "C"

// The lock-in sums of lb_cavity_calibrate_noalloc live in a file-scope device array, one
// copy per GPU, held until the process ends: 2 kCavMaxNx doubles (32 KiB).  Host code uses
// the address hipGetSymbolAddress returns for the current device, never the array's name.
static __device__ __align__(256) double scratch[2 * kCavMaxNx];

namespace {

// Argument checks shared by both calibration entry points; on success m_out and k_out receive
// the fit window in steps and the lattice wavenumber, n_total_out the run length.
int cavity_check(int32_t nx, double c0, double omega, double wall_phi, int32_t n_periods,
                 int32_t n_fit, const double *out, int64_t *n_total_out, int64_t *m_out,
                 double *k_out)
{
    g_err.clear();
    if (!out) return fail(LB_EINVAL, "out is NULL");
    if (nx < 16 || nx > kCavMaxNx) return fail(LB_EINVAL, "nx must lie in [16, %d]", kCavMaxNx);
    if (!(c0 > 0) || c0 > 1.0) return fail(LB_EUNSTABLE, "c0 must lie in (0, 1]");
    if (!(omega > 0) || omega >= M_PI) return fail(LB_EINVAL, "omega must lie in (0, pi)");
    if (!(wall_phi >= 0 && wall_phi < 1)) return fail(LB_EINVAL, "wall_phi must lie in [0, 1)");
    if (n_fit < 1 || n_periods < n_fit) return fail(LB_EINVAL, "need 1 <= n_fit <= n_periods");
    const double cosk = 1.0 - (1.0 - std::cos(omega)) / (c0 * c0);
    if (!(cosk > -1.0 && cosk < 1.0)) return fail(LB_EINVAL, "omega has no lattice wavenumber");
    const double period = 2.0 * M_PI / omega;
    *n_total_out = (int64_t)std::llround(n_periods * period);
    *m_out = (int64_t)std::llround(n_fit * period);
    *k_out = std::acos(cosk);
    return LB_OK;
}

// The fit of the cavity's lock-in sums (host array of 2 nx doubles: sum rho cos wt, then
// sum rho sin wt over the last m steps), into out[0..5] and optionally host_P.
int cavity_fit(int32_t nx, int64_t m, double k, const double *lock, double *out, double *host_P)
{
    // complex amplitude P = (2/m) sum rho e^{-i w t}
    auto re = [&](int x) { return 2.0 / (double)m * lock[x]; };
    auto im = [&](int x) { return -2.0 / (double)m * lock[nx + x]; };
    if (host_P)
        for (int x = 0; x < nx; ++x) {
            host_P[2 * x] = re(x);
            host_P[2 * x + 1] = im(x);
        }
    // least squares |P|^2 = a + b cos 2kx + c sin 2kx over 2 <= x <= nx-3
    double M[3][4] = {{0}};
    for (int x = 2; x <= nx - 3; ++x) {
        const double row[3] = {1.0, std::cos(2 * k * x), std::sin(2 * k * x)};
        const double y = re(x) * re(x) + im(x) * im(x);
        for (int i = 0; i < 3; ++i) {
            for (int j = 0; j < 3; ++j) M[i][j] += row[i] * row[j];
            M[i][3] += row[i] * y;
        }
    }
    for (int c = 0; c < 3; ++c) {  // Gaussian elimination with partial pivoting
        int p = c;
        for (int r = c + 1; r < 3; ++r)
            if (std::fabs(M[r][c]) > std::fabs(M[p][c])) p = r;
        for (int j = 0; j < 4; ++j) std::swap(M[c][j], M[p][j]);
        if (M[c][c] == 0.0) return fail(LB_EINVAL, "degenerate fit");
        for (int r = 0; r < 3; ++r) {
            if (r == c) continue;
            const double f = M[r][c] / M[c][c];
            for (int j = c; j < 4; ++j) M[r][j] -= f * M[c][j];
        }
    }
    const double a = M[0][3] / M[0][0], b = M[1][3] / M[1][1], c = M[2][3] / M[2][2];
    const double A = std::sqrt(a + std::hypot(b, c));
    const double x0 = std::atan2(c, b) / (2.0 * k);
    const double spacing = M_PI / k;
    const double centre = 0.5 * (nx - 1);
    const double xm = x0 + std::floor((centre - x0) / spacing) * spacing;
    out[0] = A;
    out[1] = xm;
    out[2] = k;
    out[3] = a;
    out[4] = b;
    out[5] = c;
    return LB_OK;
}

// One wavefront holds up to 256 cells, 4 to a lane; fewer to a lane shorten a step.
void launch_cavity(int nx, double c0sq, double omega, double rho_a, double phi, int64_t n_total,
                   int64_t n_fit, double *lock, hipStream_t s)
{
    const auto go = [&](auto kernel, int waves) {
        hipLaunchKernelGGL(kernel, dim3(1), dim3(64 * waves), 0, s, nx, c0sq, omega, rho_a, phi,
                           n_total, n_fit, lock);
    };
    if (nx <= 64)
        go(cavity_kernel<1, false>, 1);
    else if (nx <= 128)
        go(cavity_kernel<2, false>, 1);
    else if (nx <= 256)
        go(cavity_kernel<4, false>, 1);
    else
        go(cavity_kernel<4, true>, (nx + kCavOwn - 1) / kCavOwn);
}

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double *g_scratch[kMaxDevices] = {};

// the scratch array of the current device (looked up on the device's first call)
int cavity_scratch(double **ptr)
{
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(LB_EDEVICE, "device index %d unsupported", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(LB_EDEVICE, "scratch address: %s", hipGetErrorString(e));
        g_scratch[dev] = static_cast<double *>(p);
    }
    *ptr = g_scratch[dev];
    return LB_OK;
}

}  // namespace

extern "C" {

int lb_cavity_calibrate(int32_t nx, double c0, double omega, double rho_a, double wall_phi,
                        int32_t n_periods, int32_t n_fit, void *dev_workspace,
                        size_t workspace_bytes, void *hip_stream, double *out, double *host_P)
{
    int64_t n_total = 0, m = 0;
    double k = 0.0;
    int st = cavity_check(nx, c0, omega, wall_phi, n_periods, n_fit, out, &n_total, &m, &k);
    if (st) return st;
    if (!dev_workspace || workspace_bytes < lb_cavity_workspace_bytes(nx))
        return fail(LB_ENOMEM, "workspace too small");
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    double *d_lock = static_cast<double *>(dev_workspace);
    launch_cavity(nx, c0 * c0, omega, rho_a, wall_phi, n_total, m, d_lock, s);
    HIP_TRY(hipGetLastError());
    std::vector<double> lock(2 * (size_t)nx);
    HIP_TRY(hipMemcpyAsync(lock.data(), d_lock, sizeof(double) * 2 * nx, hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    return cavity_fit(nx, m, k, lock.data(), out, host_P);
}

int lb_cavity_calibrate_noalloc(int32_t nx, double c0, double omega, double rho_a,
                                double wall_phi, int32_t n_periods, int32_t n_fit,
                                void *hip_stream, double *out, double *host_P)
{
    int64_t n_total = 0, m = 0;
    double k = 0.0;
    int st = cavity_check(nx, c0, omega, wall_phi, n_periods, n_fit, out, &n_total, &m, &k);
    if (st) return st;
    double *d_lock = nullptr;
    if ((st = cavity_scratch(&d_lock))) return st;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    // the kernel writes every one of the 2 nx sums, so nothing needs clearing first
    launch_cavity(nx, c0 * c0, omega, rho_a, wall_phi, n_total, m, d_lock, s);
    HIP_TRY(hipGetLastError());
    double lock[2 * kCavMaxNx];  // host copy on the stack (no heap allocation)
    HIP_TRY(hipMemcpyAsync(lock, d_lock, sizeof(double) * 2 * nx, hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    return cavity_fit(nx, m, k, lock, out, host_P);
}

}  // extern "C"

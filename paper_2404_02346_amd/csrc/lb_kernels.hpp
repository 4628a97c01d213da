// Device code of the wave lattice Boltzmann library (gfx950).
//
// Method: Castro-Avila et al., "A lattice Boltzmann approach for acoustic
// manipulation" (arXiv 2404.02346), Sec. "Lattice-Boltzmann for acoustics"
// and Sec. "Wave-particle interaction and interpolation".
//
// Population storage is structure-of-arrays: plane i (velocity i) holds the
// cells row by row, x fastest, rows `pitch` elements apart (pitch is a
// multiple of 64 elements, so every row starts on a 256-byte boundary for
// 4-byte storage).  Two state buffers alternate: a launch reads the buffer
// the previous one wrote and writes the other, however many steps it advances
// (the device counter holds the index of the current one).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace lbw {

constexpr int kMaxSeg = 8;          // same-shape instance runs handled by one launch
constexpr int kStepThreads = 256;   // 4 wavefronts of 64 lanes

// ---------------------------------------------------------------------------
// Storage types: raw element R, compute type C
// ---------------------------------------------------------------------------
struct bf16 {  // tag type for bfloat16 storage (raw bits in uint16_t)
};

template <typename S> struct StoreTraits;
template <> struct StoreTraits<double> {
    using R = double;
    using C = double;
    __device__ static inline C to_c(R v) { return v; }
    __device__ static inline R to_r(C v) { return v; }
};
template <> struct StoreTraits<float> {
    using R = float;
    using C = float;
    __device__ static inline C to_c(R v) { return v; }
    __device__ static inline R to_r(C v) { return v; }
};
template <> struct StoreTraits<_Float16> {
    using R = _Float16;
    using C = float;
    __device__ static inline C to_c(R v) { return (float)v; }
    __device__ static inline R to_r(C v)
    {
        // kept apart from the FP32 operation that made v: as one instruction (a multiply-add
        // with an FP16 result) they would round once instead of twice, in some kernels only
        asm("" : "+v"(v));
        return (_Float16)v;
    }
};
template <> struct StoreTraits<bf16> {
    using R = uint16_t;
    using C = float;
    __device__ static inline C to_c(R v) { return __uint_as_float(((uint32_t)v) << 16); }
    __device__ static inline R to_r(C v) {
        // round to nearest, ties to even
        uint32_t u = __float_as_uint(v);
        u += 0x7FFFu + ((u >> 16) & 1u);
        return (R)(u >> 16);
    }
};

template <typename R, int N> struct VecT {
    using type = R __attribute__((ext_vector_type(N)));
};
template <typename R> struct VecT<R, 1> {
    using type = R;
};

// Pointers into global memory (address space 1): loads and stores through
// them take a uniform 64-bit base in scalar registers plus a 32-bit lane
// offset, instead of flat accesses with per-lane 64-bit addresses.
template <typename T> using gptr = T __attribute__((address_space(1))) *;
template <typename T> __device__ inline gptr<T> to_global(void *p) { return (gptr<T>)p; }
template <typename T> __device__ inline gptr<const T> to_global(const void *p)
{
    return (gptr<const T>)p;
}

// base + i elements with a 32-bit byte offset (i * sizeof(T) < 2^32 for any
// row offset here), so the access can use a scalar base and a 32-bit offset.
template <typename T> __device__ inline gptr<const T> at(gptr<const T> base, uint32_t i)
{
    return (gptr<const T>)((gptr<const char>)base + i * (uint32_t)sizeof(T));
}
template <typename T> __device__ inline gptr<T> at(gptr<T> base, uint32_t i)
{
    return (gptr<T>)((gptr<char>)base + i * (uint32_t)sizeof(T));
}

// The per-instance records do not change during a launch: reading them
// through the constant address space lets them live in scalar registers.
template <typename T> using cptr = const T __attribute__((address_space(4))) *;
template <typename T> __device__ inline cptr<T> to_const(const T *p) { return (cptr<T>)p; }

template <typename V, bool NT> __device__ inline V vload(gptr<const V> p)
{
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}
template <typename V, bool NT> __device__ inline void vstore(gptr<V> p, V v)
{
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}
template <typename V, bool NT> __device__ inline V vload(const V *p)
{
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}
template <typename V, bool NT> __device__ inline void vstore(V *p, V v)
{
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}
template <typename R, int N> __device__ inline R vget(const typename VecT<R, N>::type &v, int c)
{
    if constexpr (N == 1) return v;
    else return v[c];
}
template <typename R, int N> __device__ inline void vset(typename VecT<R, N>::type &v, int c, R x)
{
    if constexpr (N == 1) v = x;
    else v[c] = x;
}

// ---------------------------------------------------------------------------
// Per-instance data (lives in the workspace)
// ---------------------------------------------------------------------------
struct SurfPt {
    int32_t bx[3], by[3], bz[3];  // stencil nodes in moment-box coordinates
    int32_t pad;
    double w[9];                  // 1D kernel weights: wx[0..2], wy[0..2], wz[0..2]
    double nA[3];                 // outward normal times element size
};

struct AccDev {
    double sum[3];
    int64_t n;
    int32_t nan;
    int32_t pad;
};

// State buffers, read and written in turn by successive launches.  Two, not three indexed by the
// step: one FP32 sphere of 256 x 128 x 128 (117 MB a buffer) stays inside the 256 MB memory-side
// cache (24.5 us a step against 29.0 with three, when a launch advanced two steps).
constexpr int kNumBuf = 2;
// Moment boxes and partial sums, indexed by step mod InstDev::slots: a launch writes those of its
// steps while the ones of the launch before are read, so twice the most steps of a launch, rounded
// up to a power of two.
constexpr int kNumSlot = 8;
constexpr int kResidentSteps = 64;  // most steps of a resident launch (2D)

struct InstDev {
    int32_t dim, nx, ny, nz;
    int32_t pitch, xbc;
    int64_t plane;           // elements per population plane
    void *buf[kNumBuf];      // state buffers (plane 0)
    double c0sq;             // fluid c0^2 (outside the box)
    int32_t bb_lo[3];        // sound-speed box origin
    int32_t bb_n[3];         // sound-speed box extent (0 -> no box)
    const void *c2box;       // c^2 over the box in the compute type, plane by plane (c2_plane)
    double src_amp;          // rho_a times the storage scale
    double omega, wall_phi;
    int64_t max_steps;       // frozen for t >= max_steps
    int32_t src_pt[3];       // point-source node (when src_point)
    int32_t src_point;       // 1: the node src_pt is imposed after every step
    // measurement
    int32_t mb_lo[3];        // moment box origin (cells whose rho, J the surface reads)
    int32_t mb_n[3];         // moment box extent (0 -> no measurement)
    char *mom;               // moment boxes (rho, Jx, Jy, Jz per cell, compute type) by slot
    int64_t mom_bytes;       // bytes from one to the next
    int32_t slots;           // moment boxes and partial sums
    int32_t resident;        // configuration of the resident kernel (2D)
    int32_t n_surf, n_chunks;  // surface elements, 64-element chunks
    const SurfPt *surf;
    double *part;            // slots x n_chunks x 4 per-chunk flux sums
    double c0sq_force;       // c0^2 in the surface integral
    double force_scale;      // -1 / (rho0 * scale^2)
    int64_t avg_start;
    AccDev *acc;
    double *trace;           // trace_cap x 3
    int64_t trace_cap;
};

// Cells of the c^2 table from one plane of the sound-speed box to the next: its n0 x n1 cells, x
// fastest, then one c0^2 for reads from outside the box
__host__ __device__ inline int64_t c2_plane(int n0, int n1) { return (int64_t)n0 * n1 + 1; }

// slot of step t, and the moment box there
template <typename I> __device__ inline int slot_of(const I &inst, int64_t t)
{
    return (int)(t & (inst.slots - 1));
}
template <typename I> __device__ inline char *mom_of(const I &inst, int64_t t)
{
    return inst.mom + slot_of(inst, t) * inst.mom_bytes;
}

struct SegInfo {
    int32_t task0;      // first wave task of the run (one-step launch)
    int32_t first;      // first (internal) instance of the run
    int32_t nx, ny, nz; // shape shared by the run
    int32_t xsegs;      // wave tasks per row
    int32_t tpi;        // wave tasks per instance
    int32_t pad;
    int32_t blk0;       // first block of the run (march launch)
    int32_t bpi;        // blocks per instance (march launch)
    int32_t nyb;        // row blocks per instance (march launch)
    int32_t nsx;        // x strips per row (march launch; 1: the row fits one block)
};

// One launch = [reducer blocks][surface blocks][lattice blocks] (the
// march kernel puts its lattice blocks first), a three-stage pipeline
// over consecutive steps:
//  * lattice blocks advance steps t .. t+nst-1 (nst = 1 to 3, in 2D up to 64) and
//    store rho1, J1 of each f(s) in the moment box of its slot;
//  * surface blocks interpolate F(s) for the n_ms steps s = t - meas_off ..
//    that earlier launches advanced, from their moment boxes, and write one
//    partial sum per 64 elements into the slot of s;
//  * reducer blocks sum the partials of the n_rs steps t - red_off .. (in
//    step order, one block per instance) in a fixed order, scale, trace and
//    accumulate.
// Every stage reads what an earlier launch wrote, and the slots written and
// read by one launch differ, so no stage waits on another inside a
// launch.  The lattice step of a launch is t = tp[0] + dt and the buffer it reads
// (tp[1] + dbuf) mod 2: the counter lives in device memory so that a captured
// sequence of launches can be replayed at any t and from either buffer.
struct StepArgs {
    const InstDev *inst;
    const int64_t *tp;        // device step counter: {t, index of the current state buffer}
    int32_t dt;               // step offset of this launch from tp[0]
    int32_t dbuf;             // launches since tp[1] was set, mod 2
    int32_t meas_off, n_ms;   // surface stage measures t - meas_off + j, j < n_ms
    int32_t red_off, n_rs;    // reducer stage reduces t - red_off + j, j < n_rs
    int32_t nseg;
    int32_t ntask;            // lattice tasks (one-step launch) or blocks (march launch)
    int32_t n_red, n_sb;      // reducer blocks; surface blocks per measured step
    int32_t nst;              // steps of a resident launch
    SegInfo seg[kMaxSeg];
    const int32_t *sb_inst;   // per surface block: internal instance
    const int32_t *sb_chunk;  // per surface block: chunk of 64 elements
};

__device__ inline int wave_uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// ---------------------------------------------------------------------------
// Lattice part: fused pull-advection + collision + x sheets.  One wavefront
// task covers 64*CPL consecutive cells of one row; lane l owns the CPL
// contiguous cells xl = x0 + l*CPL ... and moves them with one vector load
// and one vector store per population.  The +x / -x populations come from
// the neighbouring cell: XM = 0 shifts them across lanes (one extra scalar
// load per task end), XM = 1 loads them with a vector load offset by one
// element.  NT = 0: plain loads and stores, 1: non-temporal stores,
// 2: non-temporal loads and stores.
//
// Collision with tau = 1/2 (eq. LBM-Collision) and the equilibrium of
// eq. feq_waves reduce, for these velocity sets (w_i / c_s^2 = 1/2,
// f0^eq = rho (1 - dim c^2)), to
//   f^new_{+a} = c^2 rho - f_{-a},  f^new_{-a} = c^2 rho - f_{+a},
//   f^new_0    = 2 (1 - dim c^2) rho - f_0,
// with c = c(x) the local sound speed.
// ---------------------------------------------------------------------------
// The multiply-adds are written out: left to the compiler, whether c^2 rho - f is one fused
// operation or two depends on the code around it, and every kernel has to give the same bits.
__device__ inline float mul_add(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ inline double mul_add(double a, double b, double c) { return __builtin_fma(a, b, c); }

// imposed density rs with the cell's own momentum (eq. imposingfields):
// f^eq(rs, J) of the pre-collision populations f
template <int DIM, typename C>
__device__ inline void impose_rule(const C *f, C c2, C rs, C *out)
{
    constexpr int Q = 2 * DIM + 1;
    const C h = (C)0.5;
    out[0] = rs * mul_add(-(C)DIM, c2, (C)1);
#pragma unroll
    for (int i = 1; i < Q; i += 2) {
        const C Ja = f[i] - f[i + 1];
        out[i] = h * mul_add(c2, rs, Ja);
        out[i + 1] = h * mul_add(c2, rs, -Ja);
    }
}

// collision away from the sheets
template <int DIM, typename C>
__device__ inline void bulk_rule(const C *f, C rho, C c2, C *out)
{
    constexpr int Q = 2 * DIM + 1;
    out[0] = mul_add((C)2 * mul_add(-(C)DIM, c2, (C)1), rho, -f[0]);
#pragma unroll
    for (int i = 1; i < Q; i += 2) {
        out[i] = mul_add(c2, rho, -f[i + 1]);
        out[i + 1] = mul_add(c2, rho, -f[i]);
    }
}

// damped bounce-back of the pre-collision populations (eq. bounce-back)
template <int DIM, typename C> __device__ inline void wall_rule(const C *f, C phi, C *out)
{
    constexpr int Q = 2 * DIM + 1;
    out[0] = phi * f[0];
#pragma unroll
    for (int i = 1; i < Q; i += 2) {
        out[i] = phi * f[i + 1];
        out[i + 1] = phi * f[i];
    }
}

template <int DIM, typename C>
__device__ inline void cell_rule(const C *f, C rho, C c2, int x, int nx, bool driven, C phi, C rs,
                                 C *out)
{
    if (driven && (x == 0 || x == nx - 1))
        wall_rule<DIM, C>(f, phi, out);
    else if (driven && x == 1)
        impose_rule<DIM, C>(f, c2, rs, out);
    else
        bulk_rule<DIM, C>(f, rho, c2, out);
}

template <int DIM, typename S, int CPL, int XM, int NT>
__device__ inline void lattice_task(const StepArgs &a, const int64_t t, const int bsrc, int task,
                                    int lane)
{
    using T = StoreTraits<S>;
    using R = typename T::R;
    using C = typename T::C;
    using V = typename VecT<R, CPL>::type;
    constexpr int Q = 2 * DIM + 1;

    int s = 0;
#pragma unroll
    for (int k = 1; k < kMaxSeg; ++k)
        if (k < a.nseg && task >= a.seg[k].task0) s = k;
    const SegInfo &sg = a.seg[s];
    const int local = task - sg.task0;
    const int il = local / sg.tpi;
    int r = local - il * sg.tpi;
    const int z = r / (sg.ny * sg.xsegs);
    r -= z * (sg.ny * sg.xsegs);
    const int y = r / sg.xsegs;
    const int xs = r - y * sg.xsegs;
    const auto &I = to_const(a.inst)[sg.first + il];
    if (I.max_steps > 0 && t >= I.max_steps) return;

    // per-instance constants, read once before the population loads
    const int nx = sg.nx, ny = sg.ny, nz = sg.nz;
    const int pitch = I.pitch;
    const int64_t plane = I.plane;
    const bool driven = (I.xbc == 0);
    const C c0sq = (C)I.c0sq;
    const int bb_lo0 = I.bb_lo[0], bb_lo1 = I.bb_lo[1], bb_lo2 = I.bb_lo[2];
    const int bb_n0 = I.bb_n[0], bb_n1 = I.bb_n[1], bb_n2 = I.bb_n[2];
    const int mb_lo0 = I.mb_lo[0], mb_lo1 = I.mb_lo[1], mb_lo2 = I.mb_lo[2];
    const int mb_n0 = I.mb_n[0], mb_n1 = I.mb_n[1], mb_n2 = I.mb_n[2];
    const gptr<const C> c2box = to_global<C>(I.c2box);
    const gptr<C> mom = to_global<C>(mom_of(I, t));
    const C phi = (C)I.wall_phi;
    const double src_amp = I.src_amp, omega = I.omega;
    const gptr<const R> src = to_global<R>(static_cast<const void *>(I.buf[bsrc]));
    const gptr<R> dst = to_global<R>(I.buf[bsrc ^ 1]);

    const int ym = (y == 0) ? ny - 1 : y - 1;
    const int yp = (y == ny - 1) ? 0 : y + 1;
    const int zm = (z == 0) ? nz - 1 : z - 1;
    const int zp = (z == nz - 1) ? 0 : z + 1;
    const int64_t row = ((int64_t)z * ny + y) * pitch;
    // uniform row bases of the seven pulled populations
    const gptr<const R> r0 = src + row;
    const gptr<const R> r1 = src + plane + row;
    const gptr<const R> r2 = src + 2 * plane + row;
    const gptr<const R> r3 = src + 3 * plane + ((int64_t)z * ny + ym) * pitch;
    const gptr<const R> r4 = src + 4 * plane + ((int64_t)z * ny + yp) * pitch;
    const gptr<const R> r5 = src + 5 * plane + ((int64_t)zm * ny + y) * pitch;
    const gptr<const R> r6 = src + 6 * plane + ((int64_t)zp * ny + y) * pitch;

    const int x0 = xs * 64 * CPL;
    const int xl = x0 + lane * CPL;
    const uint32_t ux = (uint32_t)xl;  // unsigned lane offset: uniform base + 32-bit offset
    // the lane owns at least one real cell (the vector then lies inside the
    // row; cells >= nx of a straddling vector are padding)
    const bool lane_in = xl < nx;

    C f[Q][CPL];
    {
        V v[Q];
        if (lane_in) {
            v[0] = vload<V, (NT == 2)>((gptr<const V>)at(r0, ux));
            if (XM == 0) {
                v[1] = vload<V, (NT == 2)>((gptr<const V>)at(r1, ux));
                v[2] = vload<V, (NT == 2)>((gptr<const V>)at(r2, ux));
            } else {
                // one element earlier / later: stays inside the buffer because the
                // +x plane follows plane 0 and the -x plane precedes plane 3
                v[1] = vload<V, (NT == 2)>((gptr<const V>)at(r1 - 1, ux));
                v[2] = vload<V, (NT == 2)>((gptr<const V>)at(r2 + 1, ux));
            }
            v[3] = vload<V, (NT == 2)>((gptr<const V>)at(r3, ux));
            v[4] = vload<V, (NT == 2)>((gptr<const V>)at(r4, ux));
            if (DIM == 3) {
                v[5] = vload<V, (NT == 2)>((gptr<const V>)at(r5, ux));
                v[6] = vload<V, (NT == 2)>((gptr<const V>)at(r6, ux));
            }
        } else {
#pragma unroll
            for (int i = 0; i < Q; ++i) v[i] = V{};
        }
#pragma unroll
        for (int i = 0; i < Q; ++i)
#pragma unroll
            for (int c = 0; c < CPL; ++c) f[i][c] = T::to_c(vget<R, CPL>(v[i], c));
    }
    if (XM == 0) {
        // +x arrives from x - 1, -x from x + 1: shift within the lane, then across lanes
        const C from_left = __shfl_up(f[1][CPL - 1], 1);
        const C from_right = __shfl_down(f[2][0], 1);
#pragma unroll
        for (int c = CPL - 1; c > 0; --c) f[1][c] = f[1][c - 1];
#pragma unroll
        for (int c = 0; c < CPL - 1; ++c) f[2][c] = f[2][c + 1];
        f[1][0] = from_left;
        f[2][CPL - 1] = from_right;
        if (lane == 0 && x0 > 0) f[1][0] = T::to_c(r1[x0 - 1]);
        if (lane == 63) {
            const int xn = x0 + 64 * CPL;
            f[2][CPL - 1] = (xn < nx) ? T::to_c(r2[xn]) : C(0);
        }
    }
    // the two ends of the row: nothing enters from outside (driven) or wrap (periodic)
    if (xl == 0) f[1][0] = driven ? C(0) : T::to_c(r1[nx - 1]);
    {
        const int cl = nx - 1 - xl;
        if (cl >= 0 && cl < CPL) {
#pragma unroll
            for (int c = 0; c < CPL; ++c)
                if (c == cl) f[2][c] = driven ? C(0) : T::to_c(r2[0]);
        }
    }

    const bool in_box_yz = (bb_n0 > 0) && (y >= bb_lo1) && (y < bb_lo1 + bb_n1) &&
                           (DIM == 2 || ((z >= bb_lo2) && (z < bb_lo2 + bb_n2)));
    const bool in_mbox_yz = (mb_n0 > 0) && (y >= mb_lo1) && (y < mb_lo1 + mb_n1) &&
                            (DIM == 2 || ((z >= mb_lo2) && (z < mb_lo2 + mb_n2)));

    V o[Q];
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        const int x = xl + c;
        C rho = f[0][c];
#pragma unroll
        for (int i = 1; i < Q; ++i) rho += f[i][c];
        if (in_mbox_yz) {
            // rho1, J1 of the advected populations f(t) for the surface measurement
            const int bx = x - mb_lo0;
            if (bx >= 0 && bx < mb_n0 && x < nx) {
                const int by = y - mb_lo1;
                const int bz = (DIM == 3) ? z - mb_lo2 : 0;
                using V4 = typename VecT<C, 4>::type;
                V4 mv;
                mv[0] = rho;
                mv[1] = f[1][c] - f[2][c];
                mv[2] = f[3][c] - f[4][c];
                mv[3] = (DIM == 3) ? f[5][c] - f[6][c] : C(0);
                *(gptr<V4>)(mom + 4 * (((int64_t)bz * mb_n1 + by) * mb_n0 + bx)) = mv;
            }
        }
        C c2 = c0sq;
        if (in_box_yz) {
            const int bx = x - bb_lo0;
            if (bx >= 0 && bx < bb_n0) {
                const int by = y - bb_lo1;
                const int bz = (DIM == 3) ? z - bb_lo2 : 0;
                c2 = c2box[bz * c2_plane(bb_n0, bb_n1) + (int64_t)by * bb_n0 + bx];
            }
        }
        C out[Q];
        if (x >= nx) {
#pragma unroll
            for (int i = 0; i < Q; ++i) out[i] = C(0);  // padding stays zero
        } else {
            C fc[Q];
#pragma unroll
            for (int i = 0; i < Q; ++i) fc[i] = f[i][c];
            C rs = C(0);
            if (driven && x == 1) rs = (C)(src_amp * sin(omega * (double)t));
            cell_rule<DIM, C>(fc, rho, c2, x, nx, driven, phi, rs, out);
        }
#pragma unroll
        for (int i = 0; i < Q; ++i) vset<R, CPL>(o[i], c, T::to_r(out[i]));
    }
    if (lane_in) {
#pragma unroll
        for (int i = 0; i < Q; ++i)
            vstore<V, (NT >= 1)>((gptr<V>)at(dst + (i * plane + row), ux), o[i]);
    }
}

// ---------------------------------------------------------------------------
// Several steps per launch (t -> t + K; D3Q7, driven x sheets).  A block of
// W wavefronts (4 or 8) owns R rows per row group and a chunk of up to zchunk
// planes (chosen per handle): wavefront w moves the cells x = 64 (w % nw) + lane of row group
// w / nw, with nw = pitch / 64 wavefronts per row and W / nw row groups (with
// nw = 3 one or two wavefronts only help to copy).  It marches
// through the planes; in iteration i level 1 (step t) is computed on plane i,
// level 2 (step t + 1) on plane i - 1, .. level K on plane i - K + 1, which
// is stored.  Level s covers K - s halo rows on each side of the owned rows
// and K - s halo planes at the chunk ends, so no block waits for another.
// What a level hands to the next stays in registers, ready to be pulled: a
// row's rest, +-x and +-y values of one plane and its +z value of the plane
// before; -z comes straight from the row just computed (the levels of one row
// are computed one after the other, so no plane is held twice).  The +-x
// values are shifted across lanes, and across wavefronts through LDS.
//
// The populations of plane i + 1 are copied from memory into LDS (16 bytes a
// lane, without passing through registers) while plane i is computed, and
// read from there once: neighbouring row groups of a block share their halo
// rows, and a wavefront has a plane's loads in flight without holding
// registers for them.
//
// What bounds it: in FP32 and FP64 the traffic behind the L2, 2 Q s bytes per
// cell in K steps plus the halo rows that miss the L2 (16 spheres of 256 x 128 x
// 128 in FP32, blocks of eight wavefronts: 2.05 GB read and 1.90 GB written per
// launch of three steps against 1.88 each, at 5.0 TB/s; of four 3.0 GB read; a
// copy reaches 6.2 TB/s); in 16-bit storage the instructions of a plane (FP16:
// 2.46 GB against 1.88 at 4.6 TB/s).  Measured against the kernel before it
// (two steps, every load through registers), us per step: those 16 spheres FP32
// 384 -> 264, FP16 244 -> 178, one sphere 24.5 -> 18.8, 16 uneven boxes of 64 to
// 192 cells a side 307 -> 180, four channels of 1000 x 64 x 64 123 -> 80, four
// spheres in FP64 208 -> 182.  K = 3 is the most that the register file holds
// (70 values of the levels, a plane's 56 loads and 28 results of the 256); K = 2
// is the faster one where a block has few planes.
//
// The per-cell arithmetic is cell_rule, as in lattice_task, and 16-bit
// storage rounds every level through the storage type, so the state is
// bit-identical to that of K one-step launches.  Moments of every step go to
// their moment boxes as in lattice_task.
// ---------------------------------------------------------------------------
constexpr int kMarchMaxPitch = 256;
constexpr int kMarchMaxSteps = 3;  // most steps of one launch
// Rows longer than kMarchMaxPitch are cut into strips of kStripW owned cells: the K - 1 columns
// on either side are computed as the halo rows are.
constexpr int kStripW = 256 - 2 * (kMarchMaxSteps - 1);
__host__ __device__ inline int march_strips(int nx, int pitch)
{
    return pitch <= kMarchMaxPitch ? 1 : (nx + kStripW - 1) / kStripW;
}

// The LDS copy of a plane: per population the rows of the block and its halo, row after row, in
// 16-byte pieces; one instruction of a wavefront copies 64 pieces (1 KiB).
template <typename E, int K, int R, int W> struct MarchStage {
    static constexpr int kPer = 16 / (int)sizeof(E);  // cells per piece
    static constexpr int kHalo = K - 1;
    // cells of a staged row of a strip: 256 lanes, one neighbour on either side, and the
    // rounding down of the first cell to a whole piece
    static constexpr int kStripRow = (258 + 2 * (kPer - 1)) / kPer * kPer;
    static constexpr int copies(int rows, int row_cells) { return (rows * row_cells / kPer + 63) / 64; }
    static constexpr int most(int a, int b) { return a > b ? a : b; }
    static constexpr int kCopies =
        most(most(most(copies(W * R + 2 * kHalo, 64), copies(W / 2 * R + 2 * kHalo, 128)),
                  most(copies(W / 3 * R + 2 * kHalo, 192), copies(W / 4 * R + 2 * kHalo, 256))),
             copies(W / 4 * R + 2 * kHalo, kStripRow));
    static constexpr int kPop = kCopies * 1024;  // bytes per population
    static constexpr int kPerWave = (kCopies + W - 1) / W;
};

// one value per lane from the lane below (to_up) or above; the lane at the end takes `edge`
template <bool UP> __device__ inline float lane_shift(float edge, float v)
{
    constexpr int ctrl = UP ? 0x138 : 0x130;  // whole-wavefront shift by one lane
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), ctrl,
                                                      0xf, 0xf, false));
}
template <bool UP> __device__ inline double lane_shift(double edge, double v)
{
    constexpr int ctrl = UP ? 0x138 : 0x130;
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(edge), __double2loint(v), ctrl, 0xf,
                                               0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(edge), __double2hiint(v), ctrl, 0xf,
                                               0xf, false);
    return __hiloint2double(hi, lo);
}

// v of lane n as a value of the whole wavefront
__device__ inline float lane_value(float v, int n)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), n));
}
__device__ inline double lane_value(double v, int n)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), n),
                            __builtin_amdgcn_readlane(__double2loint(v), n));
}
// the shift of 64 lanes around the end
template <bool UP> __device__ inline float lane_rotate(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), UP ? 0x13C : 0x134, 0xf, 0xf, true));
}
template <bool UP> __device__ inline double lane_rotate(double v)
{
    constexpr int ctrl = UP ? 0x13C : 0x134;
    return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), ctrl, 0xf, 0xf, true),
                            __builtin_amdgcn_mov_dpp(__double2loint(v), ctrl, 0xf, 0xf, true));
}

constexpr int kWaitLoads = 0x0F70;  // s_waitcnt vmcnt(0), the other counters unconstrained

// LDS stores that the compiler does not order after the copies into LDS still in flight (it
// would wait for all of them before any LDS access it sees); the caller waits before its barrier
template <typename T> using lptr = __attribute__((address_space(3))) T *;
template <int OFFSET> __device__ inline void lds_store(uint32_t addr, float v)
{
    asm volatile("ds_write_b32 %0, %1 offset:%2" ::"v"(addr), "v"(v), "n"(OFFSET) : "memory");
}
template <int OFFSET> __device__ inline void lds_store(uint32_t addr, double v)
{
    asm volatile("ds_write_b64 %0, %1 offset:%2" ::"v"(addr), "v"(v), "n"(OFFSET) : "memory");
}
// f(0) .. f(N - 1) with the index as a compile-time constant
template <int N, typename F> __device__ inline void static_for(F &&f)
{
    if constexpr (N > 0) {
        static_for<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

template <typename C>
__device__ inline void store_moments(gptr<C> mom, int mrow, int mb_lo0, int mb_n0, int x, C rho,
                                     const C *f)
{
    const int bx = x - mb_lo0;
    if (mrow >= 0 && bx >= 0 && bx < mb_n0) {
        using V4 = typename VecT<C, 4>::type;
        V4 mv;
        mv[0] = rho;
        mv[1] = f[1] - f[2];
        mv[2] = f[3] - f[4];
        mv[3] = f[5] - f[6];
        *(gptr<V4>)(mom + 4 * (int64_t)(mrow + bx)) = mv;
    }
}

template <typename S, int K, int R, int W, int NT>
__device__ inline void march_block(const StepArgs &a, const int64_t t, const int bsrc, int lb,
                                   char *stage, typename StoreTraits<S>::C *xe)
{
    using T = StoreTraits<S>;
    using E = typename T::R;
    using C = typename T::C;
    using G = MarchStage<E, K, R, W>;
    constexpr int H = K - 1;        // halo rows of level 1 on each side
    constexpr int N1 = R + 2 * H;   // rows of level 1
    constexpr int NX = N1 - 2;      // rows of level 2 (the most any level takes from the one below)
    int s = 0;
#pragma unroll
    for (int k = 1; k < kMaxSeg; ++k)
        if (k < a.nseg && lb >= a.seg[k].blk0) s = k;
    const SegInfo &sg = a.seg[s];
    const int local = lb - sg.blk0;
    const int il = local / sg.bpi;
    const int nsx = sg.nsx;
    const int rem = local - il * sg.bpi;
    const int sx = wave_uniform(rem % nsx);  // strips of one row run side by side
    const int zc = wave_uniform((rem / nsx) / sg.nyb);
    const int yb = wave_uniform(rem / nsx - zc * sg.nyb);
    const auto &I = to_const(a.inst)[wave_uniform(sg.first + il)];
    const int nx = sg.nx, ny = sg.ny, nz = sg.nz;
    const int pitch = I.pitch;
    const int64_t plane = I.plane;
    const int nw = nsx > 1 ? 4 : pitch / 64;  // wavefronts per row (strip)
    const int ng = wave_uniform(W / nw);  // row groups per block
    const int lane = threadIdx.x & 63;
    const int w = wave_uniform(threadIdx.x >> 6);
    const int wg = wave_uniform(w / nw);
    const bool active = wg < ng;
    const int g = active ? wg : 0;
    const int xs = w - wg * nw;
    const int y0 = (yb * ng + g) * R;
    const int nzc = sg.bpi / (sg.nyb * nsx);  // chunks of planes, equal to within one plane
    const int z0 = zc * (nz / nzc) + min(zc, nz % nzc);
    const int zlen = nz / nzc + (zc < nz % nzc);
    // owned columns [xo, xend); in a strip the first and last K - 1 columns are halo
    const int xo = nsx > 1 ? sx * kStripW : 0;
    const int xend = nsx > 1 ? min(nx, xo + kStripW) : nx;
    const int xfirst = nsx > 1 ? xo - H : 0;
    const int x = xfirst + xs * 64 + lane;
    const bool own = active && x >= xo && x < xend;
    const C c0sq = (C)I.c0sq;
    const C phi = (C)I.wall_phi;
    const gptr<const C> c2box = to_global<C>(I.c2box);
    const int bb_lo[3] = {I.bb_lo[0], I.bb_lo[1], I.bb_lo[2]};
    const int bb_n[3] = {I.bb_n[0], I.bb_n[1], I.bb_n[2]};
    const int mb_lo[3] = {I.mb_lo[0], I.mb_lo[1], I.mb_lo[2]};
    const int mb_n[3] = {I.mb_n[0], I.mb_n[1], I.mb_n[2]};
    C rs[K];
    gptr<C> mom[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        rs[k] = C(0);
        mom[k] = to_global<C>(mom_of(I, t + k));
    }
    if (x == 1) {
#pragma unroll
        for (int k = 0; k < K; ++k) rs[k] = (C)(I.src_amp * sin(I.omega * (double)(t + k)));
    }
    const gptr<const char> src = to_global<char>(static_cast<const void *>(I.buf[bsrc]));
    const gptr<E> dst = to_global<E>(I.buf[bsrc ^ 1]);
    const int64_t zstride = (int64_t)ny * pitch;
    auto wrapz = [&](int z) {  // a box may have fewer planes than the halo
        while (z < 0) z += nz;
        while (z >= nz) z -= nz;
        return z;
    };

    // ---- the copy of a plane into LDS
    // staged rows: row r of the block is y = yb ng R - H + r (wrapped; the +y and -y populations
    // come from one row below and above); staged columns: from x0s on, row_cells each
    const int row_cells = nsx > 1 ? G::kStripRow : pitch;
    const int x0s = nsx > 1 ? (xfirst - 1) & ~(G::kPer - 1) : 0;
    const int rows = ng * R + 2 * H;
    const int ppr = row_cells / G::kPer;  // pieces per row
    const int n_copy = (rows * ppr + 63) / 64;
    uint32_t off[3][G::kPerWave];  // byte offset of this lane's piece within a plane, per y shift
#pragma unroll
    for (int m = 0; m < G::kPerWave; ++m) {
        const int piece = (w + W * m) * 64 + lane;
        int r = piece / ppr;
        const int c = piece - r * ppr;
        if (r >= rows) r = 0;  // past the end: copies of a row into the unused tail
        const int xg = min(max(x0s + c * G::kPer, 0), pitch - G::kPer);
#pragma unroll
        for (int v = 0; v < 3; ++v) {
            int y = (yb * ng * R - H + r + (v == 1 ? -1 : v == 2 ? 1 : 0)) % ny;
            if (y < 0) y += ny;
            off[v][m] = ((uint32_t)y * (uint32_t)pitch + (uint32_t)xg) * (uint32_t)sizeof(E);
        }
    }
    const int64_t zbytes = zstride * (int64_t)sizeof(E), pbytes = plane * (int64_t)sizeof(E);
    auto copy_plane = [&](int zq) {
        const gptr<const char> zb = src + zq * zbytes;
        const gptr<const char> zbm = src + ((zq == 0) ? nz - 1 : zq - 1) * zbytes;
        const gptr<const char> zbn = src + ((zq == nz - 1) ? 0 : zq + 1) * zbytes;
#pragma unroll
        for (int m = 0; m < G::kPerWave; ++m)
            if (w + W * m < n_copy) {
                char *to = stage + (w + W * m) * 1024;
#pragma unroll
                for (int i = 0; i < 7; ++i)
                    __builtin_amdgcn_global_load_lds(
                        (gptr<const void>)((i == 5 ? zbm : i == 6 ? zbn : zb) + i * pbytes +
                                           off[i == 3 ? 1 : i == 4 ? 2 : 0][m]),
                        (lptr<void>)(to + i * G::kPop), 16, 0, 0);
            }
    };
    // this lane's cell in the first staged row of its row group
    const E *cell = reinterpret_cast<const E *>(stage) + g * R * row_cells + (x - x0s);

    // ---- rows of the moment box and the sound-speed box: a row (y, z) of a box (origin lo,
    // extent n) starts at cell (bz n1 + by) n0, the sum of a y part and a z part (-1: it misses)
    const uint32_t out_x = (uint32_t)(y0 * pitch + x);  // cell of row y0 within a plane
    int mb_y[R], bb_y[N1];
#pragma unroll
    for (int j = 0; j < N1; ++j) {
        int y = (y0 + j - H) % ny;
        if (y < 0) y += ny;
        const int bby = y - bb_lo[1];
        bb_y[j] = wave_uniform((bb_n[0] > 0 && bby >= 0 && bby < bb_n[1]) ? bby * bb_n[0] : -1);
        if (j >= H && j < H + R) {
            const int mby = y - mb_lo[1];
            mb_y[j - H] = wave_uniform(
                (mb_n[0] > 0 && y0 + j - H < ny && mby >= 0 && mby < mb_n[1]) ? mby * mb_n[0] : -1);
        }
    }
    auto mb_z = [&](int z) {
        const int bz = z - mb_lo[2];
        return (mb_n[0] > 0 && bz >= 0 && bz < mb_n[2]) ? bz * mb_n[1] * mb_n[0] : -1;
    };
    // c^2 of the lane's cell in the rows of level 1 of plane zq: lanes outside the box read the
    // c0^2 stored at the end of the plane.  The plane is addressed in 64 bits: a c^2 that varies
    // over the whole lattice takes more than 4 GiB from 2^30 cells on in FP32 (2^29 in FP64).
    const int n_plane = bb_n[0] * bb_n[1];
    const int bx = x - bb_lo[0];
    const bool xb = bx >= 0 && bx < bb_n[0];
    int bb_any = -1;  // some row of the block meets the box
#pragma unroll
    for (int j = 0; j < N1; ++j) bb_any = max(bb_any, bb_y[j]);
    auto load_c2 = [&](int zq, C (&c)[N1]) {
        const int bz = zq - bb_lo[2];
        if (__builtin_expect(bb_any >= 0 && bz >= 0 && bz < bb_n[2], 0)) {
            const gptr<const C> plane_c2 = c2box + bz * c2_plane(bb_n[0], bb_n[1]);
            // with three steps the offsets are formed in every plane of the box: kept for all rows they
            // overflow the registers (two steps keep them: 1% faster in 16-bit storage)
            int first = 0;
            if constexpr (K == 3) asm("" : "+s"(first) : "s"(bz));
#pragma unroll
            for (int j = 0; j < N1; ++j)
                c[j] = *at(plane_c2, (uint32_t)(xb && bb_y[j] >= 0 ? first + bb_y[j] + bx : n_plane));
        } else {
#pragma unroll
            for (int j = 0; j < N1; ++j) c[j] = c0sq;
        }
    };

    // ---- wavefront edges: lane 63 hands its +x value right, lane 0 its -x value left
    // xe[level][row][wavefront][0: +x of lane 63, 1: -x of lane 0]
    auto xe_at = [&](int lev, int row, int ww, int side) {
        return ((lev * NX + row) * W + ww) * 2 + side;
    };
    const bool edge_lane = lane == 0 || lane == 63;
    const uint32_t xe_base = (uint32_t)(uintptr_t)(lptr<C>)xe;
    const int xe_from = lane == 63 ? xe_at(0, 0, min(w + 1, W - 1), 1) : xe_at(0, 0, max(w - 1, 0), 0);
    const uint32_t xe_to =
        xe_base + (uint32_t)sizeof(C) * (uint32_t)xe_at(0, 0, w, lane == 63 ? 0 : 1);

    // ---- what level k + 1 hands to level k + 2, pull-ready for the rows of that level: rest, +x,
    // -x, +y, -y of one plane, +z of that plane and of the one before
    C q[H][7][NX];
    C C2[K][N1];  // c^2 of the rows of level k + 1 in its plane
    C c2next[N1];
    C edge[H][NX];
#pragma unroll
    for (int k = 0; k < H; ++k)
#pragma unroll
        for (int i = 0; i < 7; ++i)
#pragma unroll
            for (int j = 0; j < NX; ++j) q[k][i][j] = C(0);
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
        for (int j = 0; j < N1; ++j) C2[k][j] = c0sq;

    load_c2(wrapz(z0 - H), c2next);
    copy_plane(wrapz(z0 - H));
    __builtin_amdgcn_s_waitcnt(kWaitLoads);

    // Wavefronts without a sheet cell, those with the far wall only and those with the near wall
    // and the source each run their own copy of the loop: the block waits for its slowest
    // wavefront, and the others have no branch per cell.
    const bool wall = x == 0 || x == nx - 1;
    auto march = [&](auto sheets) {
        constexpr int SHEETS = decltype(sheets)::value;  // 0: none, 1: the far wall, 2: any
        for (int i = -H; i < zlen + H; ++i) {
            // the plane has arrived, for this wavefront and behind the barrier for the others,
            // and with it the edges they stored in the last iteration
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __syncthreads();
            E L[N1][7];
#pragma unroll
            for (int j = 0; j < N1; ++j) {
                const char *c = reinterpret_cast<const char *>(cell + j * row_cells);
#pragma unroll
                for (int p = 0; p < 7; ++p)
                    L[j][p] = *reinterpret_cast<const E *>(
                        c + p * G::kPop + (p == 1 ? -1 : p == 2 ? 1 : 0) * (int)sizeof(E));
            }
#pragma unroll
            for (int k = 0; k < H; ++k)
#pragma unroll
                for (int j = 0; j < NX - 2 * k; ++j) edge[k][j] = xe[xe_from + (k * NX + j) * 2 * W];
#pragma unroll
            for (int j = 0; j < N1; ++j) C2[0][j] = c2next[j];
            __syncthreads();  // everybody has read: the plane may be overwritten
            if (i + 1 < zlen + H) {
                load_c2(wrapz(z0 + i + 1), c2next);
                copy_plane(wrapz(z0 + i + 1));
            }

            C pend[K];    // +y value of a level's last row: pulled after the next row's turn
            int mrow[K];  // z part of the moment-box row index of a level's plane
#pragma unroll
            for (int k = 0; k < K; ++k) {
                pend[k] = C(0);
                const int p = i - k;
                mrow[k] = wave_uniform((p >= 0 && p < zlen) ? mb_z(z0 + p) : -1);
            }
            E res[R][7];  // level K
#pragma unroll
            for (int j = 0; j < N1; ++j) {  // row y0 + j - H
                C f[7], o[7];
#pragma unroll
                for (int p = 0; p < 7; ++p) f[p] = T::to_c(L[j][p]);
#pragma unroll
                for (int k = 0; k < K; ++k) {  // level k + 1 covers rows k .. N1 - 1 - k
                    if (j < k || j >= N1 - k) break;
                    if (k > 0) {
                        const int r = j - k;  // row index of this level
                        C(&Q)[7][NX] = q[k - 1];
                        C n[7];
                        n[0] = Q[0][r];
                        n[1] = lane_shift<true>(edge[k - 1][r], Q[1][r]);
                        n[2] = lane_shift<false>(edge[k - 1][r], Q[2][r]);
                        n[3] = Q[3][r];
                        n[4] = Q[4][r];
                        n[5] = Q[6][r];
                        n[6] = o[6];
                        // the row of the level below that has just been computed takes its place
                        Q[0][r] = o[0];
                        Q[1][r] = o[1];
                        Q[2][r] = o[2];
                        Q[6][r] = Q[5][r];
                        Q[5][r] = o[5];
                        Q[3][r] = pend[k - 1];
                        if (r > 0) Q[4][r - 1] = o[4];
                        pend[k - 1] = o[3];
#pragma unroll
                        for (int p = 0; p < 7; ++p) f[p] = n[p];
                    }
                    // nothing enters from outside the sheets
                    if (SHEETS == 2) f[1] = (x == 0) ? C(0) : f[1];
                    if (SHEETS >= 1) f[2] = (x == nx - 1) ? C(0) : f[2];
                    C rho = f[0];
#pragma unroll
                    for (int p = 1; p < 7; ++p) rho += f[p];
                    if (j >= H && j < H + R && __builtin_expect((mrow[k] | mb_y[j - H]) >= 0, 0)) {
                        if (own)
                            store_moments(mom[k], mrow[k] + mb_y[j - H], mb_lo[0], mb_n[0], x, rho, f);
                    }
                    bulk_rule<3, C>(f, rho, C2[k][j], o);
                    if (SHEETS >= 1 && wall) wall_rule<3, C>(f, phi, o);
                    if (SHEETS == 2 && x == 1) impose_rule<3, C>(f, C2[k][j], rs[k], o);
#pragma unroll
                    for (int p = 0; p < 7; ++p) {
                        if (k < H) o[p] = T::to_c(T::to_r(o[p]));
                        else res[j - H][p] = T::to_r(o[p]);
                    }
                }
                // the first and last row of a level give only their +y or -y value to the next
#pragma unroll
                for (int k = 0; k < H; ++k) {
                    if (j == k) pend[k] = o[3];
                    if (j == N1 - 1 - k) q[k][4][NX - 1 - 2 * k] = o[4];
                }
            }
            if (nw > 1 && edge_lane) {
                static_for<H * NX>([&](auto at_row) {
                    constexpr int k = decltype(at_row)::value / NX, j = decltype(at_row)::value % NX;
                    if constexpr (j < NX - 2 * k)
                        lds_store<(k * NX + j) * 2 * W * (int)sizeof(C)>(
                            xe_to, lane == 63 ? q[k][1][j] : q[k][2][j]);
                });
            }
            // wait for the next plane before this one's stores are issued: the counter that is
            // waited on also counts stores, which now have the next iteration to complete in
            __builtin_amdgcn_s_waitcnt(kWaitLoads);
            if (i >= H && own) {
                gptr<E> out = dst + (int64_t)(z0 + i - H) * zstride;
#pragma unroll
                for (int p = 0; p < 7; ++p, out += plane)
#pragma unroll
                    for (int j = 0; j < R; ++j)
                        if (__builtin_expect(y0 + j < ny, 1))
                            vstore<E, (NT >= 1)>(at(out, out_x + j * (uint32_t)pitch), res[j][p]);
            }
#pragma unroll
            for (int k = K - 1; k > 0; --k)
#pragma unroll
                for (int j = 0; j < N1; ++j) C2[k][j] = C2[k - 1][j];
        }
    };
    if (!active) {
        // a wavefront without cells (three to a row leave two over) copies its share and waits
        for (int i = -H; i < zlen + H; ++i) {
            __syncthreads();
            __syncthreads();
            if (i + 1 < zlen + H) copy_plane(wrapz(z0 + i + 1));
            __builtin_amdgcn_s_waitcnt(kWaitLoads);
        }
    } else if (__ballot(x == 0 || x == 1))
        march(std::integral_constant<int, 2>{});
    else if (__ballot(wall))
        march(std::integral_constant<int, 1>{});
    else
        march(std::integral_constant<int, 0>{});
}

// ---------------------------------------------------------------------------
// Surface part.  A block handles 64 elements of one instance; its four
// wavefronts split the 3^DIM stencil nodes (node n goes to wavefront n % 4).
// Interpolation of eq. InterpolatedFields with the 3-point kernel as a tensor
// product from the moment box of f(t_meas), then the per-element flux of
// eq. arf_integral_LBM,
//   (-|J|^2/2 + c0^2 rho^2/2) n dS + J (J . n dS),
// summed over the 64 elements in a fixed order into one partial per chunk.
// ---------------------------------------------------------------------------
template <int DIM, typename C>
__device__ inline void surface_block(const StepArgs &a, const int64_t t_meas, int sb, int tid,
                                     double (*lds)[64][4])
{
    constexpr int NN = (DIM == 3) ? 27 : 9;
    constexpr int PER = (NN + 3) / 4;
    const int lane = tid & 63;
    const int w = wave_uniform(tid >> 6);
    const InstDev &I = a.inst[a.sb_inst[sb]];
    const int chunk = a.sb_chunk[sb];
    const int k = chunk * 64 + lane;
    const bool live = k < I.n_surf;
    const gptr<const C> mom = to_global<C>(static_cast<const void *>(mom_of(I, t_meas)));
    // in 2D several steps at once come from the resident kernel, which writes column by column
    const int mbx = I.mb_n[0], mby = I.mb_n[1];
    const bool columns = DIM == 2 && a.n_ms > 1;
    const int sx = columns ? mby : 1, sy = columns ? 1 : mbx;

    double rI = 0.0, Jx = 0.0, Jy = 0.0, Jz = 0.0;
    if (live) {
        const SurfPt &P = I.surf[k];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int n = w + 4 * j;
            if (n < NN) {
                const int dx = n % 3, dy = (n / 3) % 3, dz = n / 9;
                const gptr<const C> m =
                    mom + 4 * ((int64_t)P.bz[dz] * mby * mbx + P.by[dy] * sy + P.bx[dx] * sx);
                const double wt = P.w[dx] * P.w[3 + dy] * P.w[6 + dz];
                rI += wt * (double)m[0];
                Jx += wt * (double)m[1];
                Jy += wt * (double)m[2];
                Jz += wt * (double)m[3];
            }
        }
    }
    lds[w][lane][0] = rI;
    lds[w][lane][1] = Jx;
    lds[w][lane][2] = Jy;
    lds[w][lane][3] = Jz;
    __syncthreads();
    if (w != 0) return;
    double fx = 0.0, fy = 0.0, fz = 0.0;
    if (live) {
        rI = lds[0][lane][0] + lds[1][lane][0] + lds[2][lane][0] + lds[3][lane][0];
        Jx = lds[0][lane][1] + lds[1][lane][1] + lds[2][lane][1] + lds[3][lane][1];
        Jy = lds[0][lane][2] + lds[1][lane][2] + lds[2][lane][2] + lds[3][lane][2];
        Jz = lds[0][lane][3] + lds[1][lane][3] + lds[2][lane][3] + lds[3][lane][3];
        const SurfPt &P = I.surf[k];
        const double iso = -0.5 * (Jx * Jx + Jy * Jy + Jz * Jz) + 0.5 * I.c0sq_force * rI * rI;
        const double Jn = Jx * P.nA[0] + Jy * P.nA[1] + Jz * P.nA[2];
        fx = iso * P.nA[0] + Jx * Jn;
        fy = iso * P.nA[1] + Jy * Jn;
        fz = iso * P.nA[2] + Jz * Jn;
    }
    // fixed-order butterfly over the 64 lanes
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        fx += __shfl_xor(fx, off);
        fy += __shfl_xor(fy, off);
        fz += __shfl_xor(fz, off);
    }
    if (lane == 0) {
        double *o = I.part + (slot_of(I, t_meas) * I.n_chunks + chunk) * 4;
        o[0] = fx;
        o[1] = fy;
        o[2] = fz;
    }
}

// Reducer: F(t) of one instance for the steps t0 .. t0+n-1 (n <= 64), each
// from its chunk partials (written by an earlier launch), scaled, traced and
// accumulated.  One wavefront per instance, a step to a lane; the sums over the
// chunks and the accumulation over the steps run in a fixed order.
__device__ inline void reduce_block(const StepArgs &a, const int64_t t0, int n, int ii, int tid)
{
    if (tid >= 64) return;
    const InstDev &I = a.inst[ii];
    if (I.n_surf == 0) return;
    if (I.max_steps > 0) n = (int)min((int64_t)n, I.max_steps - t0);
    const int64_t t = t0 + tid;
    double F[3] = {0.0, 0.0, 0.0};
    if (tid < n) {
        const double *p = I.part + slot_of(I, t) * I.n_chunks * 4;
        for (int c = 0; c < I.n_chunks; ++c) {
            F[0] += p[4 * c];
            F[1] += p[4 * c + 1];
            F[2] += p[4 * c + 2];
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) F[i] *= I.force_scale;
        if (t < I.trace_cap) {
            I.trace[3 * t + 0] = F[0];
            I.trace[3 * t + 1] = F[1];
            I.trace[3 * t + 2] = F[2];
        }
    }
    AccDev *acc = I.acc;
    double sum[3] = {acc->sum[0], acc->sum[1], acc->sum[2]};
    int64_t count = acc->n;
    bool bad = acc->nan != 0;
    for (int j = 0; j < n; ++j) {
        double G[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) G[i] = __shfl(F[i], j);
        if (t0 + j < I.avg_start) continue;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            sum[i] += G[i];
            bad |= !isfinite(G[i]);
        }
        ++count;
    }
    if (tid == 0) {
#pragma unroll
        for (int i = 0; i < 3; ++i) acc->sum[i] = sum[i];
        acc->n = count;
        acc->nan = bad;
    }
}

// The measurement blocks of a launch (reducers, then the surface blocks of
// each measured step); returns false for a lattice block.
template <int DIM, typename C>
__device__ inline bool measure_part(const StepArgs &a, const int64_t t, int b, int tid,
                                    double (*lds)[64][4])
{
    if (b < a.n_red) {
        reduce_block(a, t - a.red_off, a.n_rs, b, tid);
        return true;
    }
    b -= a.n_red;
    if (b < a.n_ms * a.n_sb) {
        const int j = b / a.n_sb;
        const int sb = b - j * a.n_sb;
        const InstDev &I = a.inst[a.sb_inst[sb]];
        const int64_t t_meas = t - a.meas_off + j;
        if (I.max_steps > 0 && t_meas >= I.max_steps) return true;
        surface_block<DIM, C>(a, t_meas, sb, tid, lds);
        return true;
    }
    return false;
}

template <int DIM, typename S, int CPL, int XM, int NT>
__global__ void __launch_bounds__(kStepThreads) step_kernel(StepArgs a)
{
    __shared__ double lds[4][64][4];
    const int64_t t = a.tp[0] + a.dt;
    const int b = blockIdx.x;
    if (measure_part<DIM, typename StoreTraits<S>::C>(a, t, b, threadIdx.x, lds)) return;
    const int bsrc = ((int)a.tp[1] + a.dbuf) & 1;
    const int wave = wave_uniform(threadIdx.x >> 6);
    const int task = (b - a.n_red - a.n_ms * a.n_sb) * (kStepThreads / 64) + wave;
    if (task >= a.ntask) return;
    lattice_task<DIM, S, CPL, XM, NT>(a, t, bsrc, task, threadIdx.x & 63);
}

// Blocks are dispatched round-robin over the 8 XCDs (each with its own L2):
// physical block b runs on XCD b % 8.  Give each XCD a contiguous range of
// the n logical blocks, so that neighbouring row blocks, which read each
// other's halo rows, share an L2.  A bijection on [0, n).
constexpr int kNumXcd = 8;
__device__ inline int xcd_block(int b, int n)
{
    const int q = n / kNumXcd, r = n % kNumXcd;
    const int x = b % kNumXcd, k = b / kNumXcd;
    return (x < r) ? x * (q + 1) + k : r * (q + 1) + (x - r) * q + k;
}

template <typename S, int K, int R, int W, int NT>
__global__ void __launch_bounds__(64 * W, 2) march_kernel(StepArgs a)
{
    using C = typename StoreTraits<S>::C;
    using G = MarchStage<typename StoreTraits<S>::R, K, R, W>;
    constexpr int NX = R + 2 * (K - 1) - 2;
    __shared__ __attribute__((aligned(1024))) char stage[7 * G::kPop];
    __shared__ C xe[(K - 1) * NX * 2 * W];
    const int64_t t = a.tp[0] + a.dt;
    const int b = blockIdx.x;
    // the long lattice blocks first, the short measurement blocks fill the tail
    if (b < a.ntask) {
        march_block<S, K, R, W, NT>(a, t, ((int)a.tp[1] + a.dbuf) & 1, xcd_block(b, a.ntask), stage, xe);
        return;
    }
    // measurement blocks of kStepThreads threads, side by side
    using Lds = double[4][64][4];
    constexpr int per = 64 * W / kStepThreads;
    static_assert(sizeof stage >= per * sizeof(Lds), "the surface blocks use the same LDS");
    const int part = wave_uniform(threadIdx.x / kStepThreads);
    measure_part<3, C>(a, t, per * (b - a.ntask) + part, threadIdx.x % kStepThreads,
                       reinterpret_cast<Lds *>(stage)[part]);
}

// ---------------------------------------------------------------------------
// Up to kResidentSteps steps per launch in 2D (D2Q5, driven x sheets): one block
// holds a whole box in registers.  Wavefront w owns a share of the columns, lane
// l the cells y = l and l + 64 of each.  A step reads nothing but its neighbours'
// values: +-y from the next lane, +-x from the next column's registers, and at a
// wavefront's first and last column through LDS, with one barrier.  Columns
// rather than rows, because the wall and source columns, which have a rule of
// their own, are then whole wavefronts and no lane masks.  The moments of every
// step go to memory, where the surface blocks of the next launch interpolate
// them, all steps side by side on the other CUs.
//
// What bounds it: the instruction rate of one CU (about 110 FP64 instructions and
// 32 lane moves of a wavefront per step at 128 x 64 cells).  us per step in a long call, one box and 32
// at once, with a launch per step in brackets:
//   boxes that fill their tile of wavefronts and lanes (FULL), FP64: 128 x 64 1.7, 1.8 (4.0, 6.8),
//   64 x 64 1.1, 1.3 (4.1, 5.6), 64 x 128 2.4, 2.8 (4.1, 7.1); FP32 1.2, 1.3, 0.8, 1.0 and 1.5, 1.8;
//   others, which mask columns and rows and find the last row's neighbour by hand, FP64: 127 x 63 2.8,
//   2.9 (4.1, 6.7), 116 x 55 2.6, 2.8 (4.3, 6.0), 100 x 50 2.3, 2.4, 33 x 33 1.1, 1.2; FP32 127 x 63 1.8, 1.9.
// Rows instead of columns: 3.1 and 5.0 in FP64 (128 x 64).  c^2 of FP64 from LDS: kept in registers,
// which then spill, 2.3 and 2.6.  A launch costs the box's way in and out, in vectors of a lane's
// columns: 127 x 63, a call of 8 steps in FP64 50 us, in FP32 35 (69 and 61 column by column).
// ---------------------------------------------------------------------------
constexpr int kResidentWaves = 16;
// configuration CX << 8 | RY (columns of a wavefront, cells of a lane in a column) of a box, 0 if it
// does not fit: eight cells of a lane are what the registers of 16 wavefronts hold in FP64
__host__ __device__ inline int resident_config(int nx, int ny)
{
    const int cols = (nx + kResidentWaves - 1) / kResidentWaves;
    const int cx = cols <= 4 ? 4 : 8, ry = ny <= 64 ? 1 : 2;
    return cols <= 8 && ny <= 128 && cx * ry <= 8 ? cx << 8 | ry : 0;
}

// the first n of the columns v[LO .. LO + N), in stores as wide as they go
template <typename E, int LO, int N> __device__ inline void store_columns(gptr<E> p, const E *v, int n)
{
    if (n >= N) {
        using U = typename VecT<E, N>::type __attribute__((aligned(sizeof(E))));
        typename VecT<E, N>::type w;
#pragma unroll
        for (int c = 0; c < N; ++c) vset<E, N>(w, c, v[LO + c]);
        *(gptr<U>)(p + LO) = w;
    } else if constexpr (N > 1) {
        store_columns<E, LO, N / 2>(p, v, n);
        store_columns<E, LO + N / 2, N / 2>(p, v, n - N / 2);
    }
}

// FULL: every wavefront owns CX columns and every lane RY cells of each; the other form takes any box
template <typename S, int CX, int RY, bool FULL>
__device__ inline void resident_box(const StepArgs &a, int box, const int64_t t, const int bsrc,
                                    typename StoreTraits<S>::C *edges, typename StoreTraits<S>::C *c2lds,
                                    const typename StoreTraits<S>::C *drive)
{
    using T = StoreTraits<S>;
    using E = typename T::R;
    using C = typename T::C;
    using V = typename VecT<E, CX>::type;
    using U = V __attribute__((aligned(sizeof(E) * (FULL ? CX : 1))));
    constexpr int W = kResidentWaves;
    const auto &I = to_const(a.inst)[box];
    const int nx = FULL ? W * CX : I.nx, ny = FULL ? 64 * RY : I.ny, pitch = I.pitch;
    const int lane = threadIdx.x & 63, w = wave_uniform(threadIdx.x >> 6);
    const int cols = FULL ? CX : nx / W + (w < nx % W);  // an equal share, some one column more
    const int x0 = FULL ? w * CX : w * (nx / W) + min(w, nx % W);
    const int last = min(nx, W) - 1;                     // the last wavefront that has columns
    const int end = ny - 64 * (RY - 1) - 1;              // the lane of the last row
    const int nst = I.max_steps > 0 ? (int)min((int64_t)a.nst, I.max_steps - t) : a.nst;
    const int64_t plane = I.plane;
    const gptr<const E> src = to_global<E>(static_cast<const void *>(I.buf[bsrc]));
    const gptr<E> dst = to_global<E>(I.buf[bsrc ^ 1]);
    const C phi = (C)I.wall_phi;

    // post-collision values, and c^2, which in FP64 the registers have no room for
    constexpr bool kLds = sizeof(C) == 8;
    C q[5][CX][RY], c2[kLds ? 1 : CX][kLds ? 1 : RY];
    C *const c2own = c2lds + w * (CX * RY * 64) + lane;
#pragma unroll
    for (int r = 0; r < RY; ++r) {
        const int y = lane + 64 * r;
        const bool in = FULL || y < ny;
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            // CX columns from x0 on lie inside the padded row, whatever the share of this wavefront
            V v = V{};
            if (in) v = *(gptr<const U>)(src + i * plane + (int64_t)y * pitch + x0);
#pragma unroll
            for (int c = 0; c < CX; ++c) q[i][c][r] = FULL || c < cols ? T::to_c(vget<E, CX>(v, c)) : C(0);
        }
        const gptr<const C> c2box = to_global<C>(I.c2box);
        const int bb_n0 = I.bb_n[0], by = y - I.bb_lo[1];
        const bool inside = in && by >= 0 && by < I.bb_n[1];
#pragma unroll
        for (int c = 0; c < CX; ++c) {
            const int bx = x0 + c - I.bb_lo[0];
            const C v = inside && c < cols && bx >= 0 && bx < bb_n0 ? c2box[by * bb_n0 + bx] : (C)I.c0sq;
            if constexpr (kLds)
                c2own[(c * RY + r) * 64] = v;
            else
                c2[c][r] = v;
        }
    }

    // edges[parity][wavefront][0: -x values of its first column, 1: +x values of its last][y]
    auto edge = [&](int parity, int ww, int side) {
        return edges + ((parity * W + ww) * 2 + side) * (64 * RY) + lane;
    };
    auto publish = [&](int parity) {
#pragma unroll
        for (int c = 0; c < CX; ++c)
#pragma unroll
            for (int r = 0; r < RY; ++r) {
                if (c == 0 && (FULL || cols > 0)) edge(parity, w, 0)[64 * r] = q[2][0][r];
                if (FULL ? c == CX - 1 : c == cols - 1) edge(parity, w, 1)[64 * r] = q[1][c][r];
            }
    };
    publish(0);
    __syncthreads();
    for (int k = 0; k < nst; ++k) {
        C prev[RY], beyond[RY];  // +x of the column before, -x of the column after the last
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            prev[r] = w > 0 ? edge(k & 1, w - 1, 1)[64 * r] : C(0);
            beyond[r] = w < last ? edge(k & 1, w + 1, 0)[64 * r] : C(0);
        }
        const C rs = drive[k];
        // evaluated in every step: kept for all columns, what depends on it overflows the registers
        int mx0 = x0 - I.mb_lo[0], my0 = lane - I.mb_lo[1];
        asm volatile("" : "+s"(mx0), "+v"(my0));
        const int mb_n1 = I.mb_n[1], columns_measured = mb_n1 > 0 ? I.mb_n[0] : 0;
        const gptr<C> mom = to_global<C>(mom_of(I, t + k));
#pragma unroll
        for (int c = 0; c < CX; ++c) {
            if (!FULL && c >= cols) break;
            const bool edge_col = FULL ? c == CX - 1 : c == cols - 1;
            C f[RY][5], rho[RY];
#pragma unroll
            for (int r = 0; r < RY; ++r) {
                f[r][0] = q[0][c][r];
                f[r][1] = prev[r];
                prev[r] = q[1][c][r];
                f[r][2] = edge_col || c == CX - 1 ? beyond[r] : q[2][c < CX - 1 ? c + 1 : c][r];
                if constexpr (FULL && RY == 1) {
                    f[r][3] = lane_rotate<true>(q[3][c][r]);
                    f[r][4] = lane_rotate<false>(q[4][c][r]);
                } else {
                    const C up = r > 0 ? lane_value(q[3][c][r > 0 ? r - 1 : 0], 63)
                                       : lane_value(q[3][c][RY - 1], end);
                    const C down = lane_value(q[4][c][r < RY - 1 ? r + 1 : 0], 0);
                    f[r][3] = lane_shift<true>(up, q[3][c][r]);
                    f[r][4] = lane_shift<false>(down, q[4][c][r]);
                    if (!FULL && r == RY - 1) f[r][4] = lane == end ? down : f[r][4];
                }
                rho[r] = f[r][0];
#pragma unroll
                for (int i = 1; i < 5; ++i) rho[r] += f[r][i];
            }
            if ((uint32_t)(mx0 + c) < (uint32_t)columns_measured) {
#pragma unroll
                for (int r = 0; r < RY; ++r) {
                    const int by = my0 + 64 * r;
                    if ((uint32_t)by < (uint32_t)mb_n1) {
                        using V4 = typename VecT<C, 4>::type;
                        V4 mv;
                        mv[0] = rho[r];
                        mv[1] = f[r][1] - f[r][2];
                        mv[2] = f[r][3] - f[r][4];
                        mv[3] = C(0);
                        *(gptr<V4>)(mom + 4 * ((mx0 + c) * mb_n1 + by)) = mv;
                    }
                }
            }
            const int x = x0 + c;
            // full boxes have their sheets in these columns of a wavefront
            const bool sheet = FULL && c > 1 && c < CX - 1 ? false : x <= 1 || x == nx - 1;
#pragma unroll
            for (int r = 0; r < RY; ++r) {
                C o[5], cc;
                if constexpr (kLds)
                    cc = c2own[(c * RY + r) * 64];
                else
                    cc = c2[c][r];
                if (!sheet)
                    bulk_rule<2, C>(f[r], rho[r], cc, o);
                else
                    cell_rule<2, C>(f[r], rho[r], cc, x, nx, true, phi, rs, o);
#pragma unroll
                for (int i = 0; i < 5; ++i) q[i][c][r] = T::to_c(T::to_r(o[i]));
            }
        }
        publish((k + 1) & 1);
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < RY; ++r) {
        const int y = lane + 64 * r;
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            E v[CX];
#pragma unroll
            for (int c = 0; c < CX; ++c) v[c] = T::to_r(q[i][c][r]);
            if (FULL || y < ny)
                store_columns<E, 0, CX>(dst + i * plane + (int64_t)y * pitch + x0, v, cols);
        }
    }
}

template <typename S> __global__ void __launch_bounds__(64 * kResidentWaves) resident_kernel(StepArgs a)
{
    using C = typename StoreTraits<S>::C;
    constexpr int W = kResidentWaves;
    __shared__ __attribute__((aligned(16))) C edges[2 * W * 2 * 128];
    __shared__ C c2lds[sizeof(C) == 8 ? W * 64 * 8 : 1];
    __shared__ C drive[kResidentSteps];
    const int64_t t = a.tp[0] + a.dt;
    const int b = blockIdx.x;
    if (b >= a.ntask) {
        // measurement blocks of kStepThreads threads, side by side
        using Lds = double[4][64][4];
        constexpr int per = 64 * W / kStepThreads;
        static_assert(sizeof edges >= per * sizeof(Lds), "the surface blocks use the same LDS");
        const int part = wave_uniform(threadIdx.x / kStepThreads);
        measure_part<2, C>(a, t, per * (b - a.ntask) + part, threadIdx.x % kStepThreads,
                           reinterpret_cast<Lds *>(edges)[part]);
        return;
    }
    const int bsrc = ((int)a.tp[1] + a.dbuf) & 1;
    const auto &I = to_const(a.inst)[b];
    if ((int)threadIdx.x < a.nst)
        drive[threadIdx.x] = (C)(I.src_amp * sin(I.omega * (double)(t + (int)threadIdx.x)));
    __syncthreads();
    const int cx = I.resident >> 8, ry = I.resident & 255;
    const bool full = I.nx == W * cx && I.ny == 64 * ry;
    auto run = [&](auto columns, auto rows) {
        constexpr int CX = decltype(columns)::value, RY = decltype(rows)::value;
        if (full)
            resident_box<S, CX, RY, true>(a, b, t, bsrc, edges, c2lds, drive);
        else
            resident_box<S, CX, RY, false>(a, b, t, bsrc, edges, c2lds, drive);
    };
    using std::integral_constant;
    if (cx == 8)
        run(integral_constant<int, 8>{}, integral_constant<int, 1>{});
    else if (ry == 2)
        run(integral_constant<int, 4>{}, integral_constant<int, 2>{});
    else
        run(integral_constant<int, 4>{}, integral_constant<int, 1>{});
}

// Point source (the paper's oscillating point source): after the lattice
// step t, the source node of every instance that has one takes
// f^eq(rho_a sin(omega t), J1) from its own pre-collision populations, as the
// source sheet does; x, y and z are periodic.  One thread per instance, in
// stream order after the step's lattice launch and before the next one.
template <int DIM, typename S>
__global__ void point_source_kernel(const InstDev *inst, int n_inst, const int64_t *tp, int32_t dt,
                                    int32_t dbuf)
{
    using T = StoreTraits<S>;
    using R = typename T::R;
    using C = typename T::C;
    constexpr int Q = 2 * DIM + 1;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n_inst) return;
    const InstDev &I = inst[k];
    const int64_t t = tp[0] + dt;
    if (!I.src_point || (I.max_steps > 0 && t >= I.max_steps)) return;
    const int bsrc = ((int)tp[1] + dbuf) & 1;
    const R *src = static_cast<const R *>(I.buf[bsrc]);
    R *dst = static_cast<R *>(I.buf[bsrc ^ 1]);
    const int x = I.src_pt[0], y = I.src_pt[1], z = I.src_pt[2];
    auto at = [&](int i, int xx, int yy, int zz) {
        xx = xx < 0 ? xx + I.nx : (xx >= I.nx ? xx - I.nx : xx);
        yy = yy < 0 ? yy + I.ny : (yy >= I.ny ? yy - I.ny : yy);
        zz = zz < 0 ? zz + I.nz : (zz >= I.nz ? zz - I.nz : zz);
        return (int64_t)i * I.plane + ((int64_t)zz * I.ny + yy) * I.pitch + xx;
    };
    // the pulled populations f_i(x) = f^new_i(x - v_i) of the previous step
    C f[Q];
    f[0] = T::to_c(src[at(0, x, y, z)]);
    f[1] = T::to_c(src[at(1, x - 1, y, z)]);
    f[2] = T::to_c(src[at(2, x + 1, y, z)]);
    f[3] = T::to_c(src[at(3, x, y - 1, z)]);
    f[4] = T::to_c(src[at(4, x, y + 1, z)]);
    if (DIM == 3) {
        f[5] = T::to_c(src[at(5, x, y, z - 1)]);
        f[6] = T::to_c(src[at(6, x, y, z + 1)]);
    }
    C c2 = (C)I.c0sq;
    const int bx = x - I.bb_lo[0], by = y - I.bb_lo[1], bz = (DIM == 3) ? z - I.bb_lo[2] : 0;
    if (I.bb_n[0] > 0 && bx >= 0 && bx < I.bb_n[0] && by >= 0 && by < I.bb_n[1] &&
        (DIM == 2 || (bz >= 0 && bz < I.bb_n[2])))
        c2 = static_cast<const C *>(
            I.c2box)[bz * c2_plane(I.bb_n[0], I.bb_n[1]) + (int64_t)by * I.bb_n[0] + bx];
    const C rs = (C)(I.src_amp * sin(I.omega * (double)t));
    C out[Q];
    impose_rule<DIM, C>(f, c2, rs, out);
#pragma unroll
    for (int i = 0; i < Q; ++i) dst[at(i, x, y, z)] = T::to_r(out[i]);
}

// rho1 = sum_i f_i (eq. MacroscopicFields) at listed cells of one state buffer, summed in
// FP64 in velocity order and divided by the storage scale; a cell index outside
// 0 .. ncell-1 gives NaN.  Cell c = (z ny + y) nx + x lives at row (z ny + y) of each plane.
template <typename S>
__global__ void probe_rho_kernel(const void *buf, int64_t plane, int Q, int nx, int64_t ncell,
                                 int pitch, const int64_t *cells, int n, double scale, double *out)
{
    using T = StoreTraits<S>;
    using R = typename T::R;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t c = cells[i];
    if (c < 0 || c >= ncell) {
        out[i] = __builtin_nan("");
        return;
    }
    const int64_t off = (c / nx) * pitch + c % nx;
    const R *f = static_cast<const R *>(buf);
    double s = 0.0;
    for (int q = 0; q < Q; ++q) s += (double)T::to_c(f[q * plane + off]);
    out[i] = s / scale;
}

// Device counter {t, index of the current state buffer}: set, or advanced by k steps in
// n_launch launches after a replayed sequence.
__global__ void set_step_kernel(int64_t *tp, int64_t t, int64_t buf)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        tp[0] = t;
        tp[1] = buf;
    }
}
__global__ void advance_step_kernel(int64_t *tp, int64_t k, int64_t n_launch)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        tp[0] = tp[0] + k;
        tp[1] = (tp[1] + n_launch) & 1;
    }
}

// Fill with zeros (used instead of hipMemsetAsync so that every node of a
// captured sequence is a kernel).
__global__ void zero_kernel(uint4 *p, int64_t n16)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride)
        p[i] = make_uint4(0u, 0u, 0u, 0u);
}

// Plain copy (bandwidth reference for the roofline): each thread moves UNR
// independent 16-byte words, consecutive threads consecutive words.
using word16 = VecT<uint32_t, 4>::type;
template <int UNR, bool NT>
__global__ void __launch_bounds__(256) copy_kernel(const word16 *__restrict__ src,
                                                    word16 *__restrict__ dst, int64_t n16)
{
    const int64_t base = (int64_t)blockIdx.x * 256 * UNR + threadIdx.x;
    word16 v[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
        const int64_t i = base + (int64_t)u * 256;
        if (i < n16) v[u] = vload<word16, NT>(src + i);
    }
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
        const int64_t i = base + (int64_t)u * 256;
        if (i < n16) vstore<word16, NT>(dst + i, v[u]);
    }
}

// ---------------------------------------------------------------------------
// Empty driven cavity: the x-only field of the empty box is the 3-population
// 1D lattice (rest weight 1 - c0^2, moving weights c0^2/2), run by one
// workgroup with the lattice in registers, CPL cells to a lane.  Accumulates
// sum rho cos(w t) and sum rho sin(w t) per cell over the last n_fit steps.
//
// What bounds it: the chain of one step after another (15360 for 30 periods of
// 256 cells), so a step has no barrier, no LDS access and no branch per cell:
//  * up to 64 CPL cells one wavefront does it all, the moving populations
//    passing from lane to lane in registers.  Wider boxes take a wavefront per
//    kCavOwn cells, each also computing kCavHalo cells on either side, and the
//    wavefronts exchange their cells through LDS every kCavHalo steps;
//  * bulk, wall and padding cells share one rule with per-cell coefficients,
//    out = a rho + b f with a = 0 on the walls (b = Phi there, -1 in the bulk)
//    and both 0 in the padding, which so stays empty; the added product is exact;
//  * the drive's sines are evaluated 64 steps at a time, one per lane.
// ns per step for 64 / 128 / 256 / 300 / 1000 / 2048 cells: 100 / 119 / 158 / 181 / 289 / 406
// (602 / 601 / 597 / 625 / 707 / 826 with 1024 threads, two barriers a step and a sine per thread).
// ---------------------------------------------------------------------------
constexpr int kCavMaxNx = 2048;
constexpr int kCavHalo = 16;                      // divides 64
constexpr int kCavOwn = 64 * 4 - 2 * kCavHalo;    // CPL = 4
constexpr int kCavMaxWaves = (kCavMaxNx + kCavOwn - 1) / kCavOwn;

template <int CPL, bool MANY>
__global__ void __launch_bounds__(MANY ? 64 * kCavMaxWaves : 64)
cavity_kernel(int nx, double c0sq, double omega, double rho_a, double phi, int64_t n_total,
              int64_t n_fit, double *lockin /* 2*nx: cos sums, sin sums */)
{
    static_assert(!MANY || CPL == 4, "kCavOwn is for 4 cells to a lane");
    __shared__ double cells[MANY ? 3 : 1][MANY ? kCavMaxNx : 1];
    const int lane = threadIdx.x & 63, w = wave_uniform(threadIdx.x >> 6);
    const int x0 = (MANY ? w * kCavOwn - kCavHalo : 0) + lane * CPL;  // its first cell
    double g0[CPL], np[CPL], nm[CPL], sc[CPL], ss[CPL];
    double a0[CPL], ac[CPL], b[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        const int x = x0 + c;
        g0[c] = np[c] = nm[c] = sc[c] = ss[c] = 0.0;
        const bool in = x >= 0 && x < nx, wall = x == 0 || x == nx - 1;
        a0[c] = in && !wall ? 2.0 * (1.0 - c0sq) : 0.0;
        ac[c] = in && !wall ? c0sq : 0.0;
        b[c] = !in ? 0.0 : wall ? phi : -1.0;
    }
    const double rest = 1.0 - c0sq;
    constexpr int kSrc = 1 % CPL;  // the source is x = 1: this cell of one lane
    const bool src = x0 + kSrc == 1;
    auto own = [&](int x) {
        return x >= 0 && x < nx && (!MANY || (x >= w * kCavOwn && x < (w + 1) * kCavOwn));
    };
    for (int64_t t0 = 0; t0 < n_total; t0 += 64) {
        const double arg = omega * (double)(t0 + lane);
        const double rs_all = rho_a * sin(arg);
        double cw_all = 0.0, sw_all = 0.0;
        if (t0 + 64 > n_total - n_fit) sincos(arg, &sw_all, &cw_all);
        const int n = (int)min((int64_t)64, n_total - t0);
#pragma unroll 1
        for (int k0 = 0; k0 < n; k0 += MANY ? kCavHalo : 64) {
            if (MANY) {  // every wavefront's own cells to the others' halos
                __syncthreads();
#pragma unroll
                for (int c = 0; c < CPL; ++c)
                    if (own(x0 + c)) {
                        cells[0][x0 + c] = g0[c];
                        cells[1][x0 + c] = np[c];
                        cells[2][x0 + c] = nm[c];
                    }
                __syncthreads();
#pragma unroll
                for (int c = 0; c < CPL; ++c) {
                    const int x = x0 + c;
                    if (x >= 0 && x < nx && !own(x)) {
                        g0[c] = cells[0][x];
                        np[c] = cells[1][x];
                        nm[c] = cells[2][x];
                    }
                }
            }
            const int k1 = MANY ? min(n, k0 + kCavHalo) : n;
#pragma unroll 1
            for (int k = k0; k < k1; ++k) {
                double ap[CPL], am[CPL], rho[CPL];
                ap[0] = lane_shift<true>(0.0, np[CPL - 1]);
                am[CPL - 1] = lane_shift<false>(0.0, nm[0]);
#pragma unroll
                for (int c = 1; c < CPL; ++c) {
                    ap[c] = np[c - 1];
                    am[c - 1] = nm[c];
                }
#pragma unroll
                for (int c = 0; c < CPL; ++c) rho[c] = g0[c] + ap[c] + am[c];
                if (t0 + k >= n_total - n_fit) {
                    const double cw = lane_value(cw_all, k), sw = lane_value(sw_all, k);
#pragma unroll
                    for (int c = 0; c < CPL; ++c) {
                        sc[c] = mul_add(rho[c], cw, sc[c]);
                        ss[c] = mul_add(rho[c], sw, ss[c]);
                    }
                }
#pragma unroll
                for (int c = 0; c < CPL; ++c) {
                    g0[c] = mul_add(a0[c], rho[c], b[c] * g0[c]);
                    np[c] = mul_add(ac[c], rho[c], b[c] * am[c]);
                    nm[c] = mul_add(ac[c], rho[c], b[c] * ap[c]);
                }
                const double rs = lane_value(rs_all, k);
                const double J = ap[kSrc] - am[kSrc];
                const double s0 = rs * rest;
                const double sp = 0.5 * mul_add(c0sq, rs, J), sm = 0.5 * mul_add(c0sq, rs, -J);
                g0[kSrc] = src ? s0 : g0[kSrc];
                np[kSrc] = src ? sp : np[kSrc];
                nm[kSrc] = src ? sm : nm[kSrc];
            }
        }
    }
#pragma unroll
    for (int c = 0; c < CPL; ++c)
        if (own(x0 + c)) {
            lockin[x0 + c] = sc[c];
            lockin[nx + x0 + c] = ss[c];
        }
}

}  // namespace lbw

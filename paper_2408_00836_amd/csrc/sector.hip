// sector.hip -- the particle-number sector form of the HVA circuit on gfx950.
//
// H (Eq. (1)/(2)/(15)/(16)) and every gate of the Eq. (7) layer keep the
// numbers of spin-up and spin-down electrons, so the circuit state prepared
// from the checkerboard basis state |b0> (Sec. 2.1) has nonzero amplitudes
// only on the basis states with b0's (N_up, N_dn).  This file stores only
// those: the state is the matrix Psi[r_dn][r_up] of C(Ns, N_dn) x C(Ns, N_up)
// complex128 amplitudes, r_s the rank of the spin-s site pattern among the
// patterns with N_s electrons in increasing numeric order (at 4x4 half
// filling 12870 x 12870 = 1.66e8 amplitudes, 2.6 GB, against 2^32 and
// 64 GiB for the full vector).
//
// A hopping term of spin s changes only the spin-s pattern, so it acts inside
// the rows of the matrix (s = up) or inside its columns (s = down), with the
// same pairing of elements in every row.  A row pass holds rows in a
// workgroup and applies a run of gates to them; the hops of a layer go in
// phases (sector_plan.hpp): a thread takes an orbit of 6, 4 and 4 elements
// that all hops of a four-site cluster keep, so that a phase of three to four
// hops costs one exchange through LDS.  The diagonal acts element-wise.
//
// Schedule of L layers: [D_0, up_0], [dn_0, D_1, dn_1], [up_1, D_2, up_2],
// ...: within a layer the up and down hops commute, so each row pass carries
// the second half of one layer and the first half of the next, L + 1 row
// passes per sweep.
//
// Rows of up to kShortRow elements live in LDS, 2^lr of them per workgroup;
// down passes read the matrix by columns.  Longer rows (16 sites) live in
// registers, one per workgroup, and a pass stores its result transposed for
// the other spin's (layout A: rows r_dn; layout B: the transpose).  Small
// matrices stay in one workgroup's LDS for a whole evaluation.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cmath>
#include <cstring>
#include <exception>
#include <functional>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <tuple>
#include <type_traits>
#include <vector>

#include "../../include/hubbard.h"
#include "hubvqe.hpp"
#include "phase.hpp"
#include "sector_plan.hpp"

namespace hv {

// engine.hip: the handle's model, its unique id, the thread's last error,
// whether a stream is being captured, the Lanczos recurrence on a Hamiltonian given as a callback
const Model *handle_model(hubbard_t h);
uint64_t handle_uid(hubbard_t h);
hubbard_status set_error(hubbard_status s, const std::string &msg);
bool under_capture(hipStream_t s);
using ApplyH = std::function<hubbard_status(const double2 *, double2 *)>;
hubbard_status lanczos_run(const ApplyH &apply, uint64_t n, const double2 *start_dev,
                           int32_t max_iter, double tol, double *E0, int32_t *iters,
                           double *residual, double2 *gs_dev, double2 *const buf[3],
                           double2 *partial, hipStream_t s);
size_t lanczos_partial_bytes();

namespace sec {

constexpr int kMaxRed = 16;               // reduction slots of one row pass
constexpr int kWholeN = 35, kWholeEl = 8; // whole evaluations: patterns of a spin, amplitudes
constexpr int kWholeLayers = 1024;        // of a thread, layers
constexpr int kGrid = 1024;               // at most this many workgroups write partials

enum { S_FWD = 0, S_REV = 1 };
// SF_TURN (long rows): the result goes, transposed, to the other layout's
// buffer; with SF_BOTH also to its own place.
enum { SF_NO_STORE = 1, SF_START = 2, SF_TURN = 4, SF_BOTH = 8 };
// What a pass of H does with its part phi of H psi: out <- phi, out <- out +
// phi, lambda = out + phi and then psi <- lambda / m + i m psi, out <- lambda
// / m - i m psi (the reverse sweep's two vectors), or only the energy.
enum { HO_SET = 0, HO_ADD = 1, HO_MIX = 2, HO_NONE = 3 };

typedef __attribute__((address_space(1))) double2 gc128;
typedef __attribute__((address_space(3))) double lds64w;
// LDS byte address (of kernels whose only LDS is their launch's, which begins at 0)
__device__ __forceinline__ lds64w *lds_at(uint32_t a) { return (lds64w *)(uintptr_t)a; }
typedef const __attribute__((address_space(1))) uint16_t gu16;
typedef const __attribute__((address_space(1))) uint32_t gu32;
typedef const __attribute__((address_space(1))) uint4 gu128;
typedef const __attribute__((address_space(1))) double gf64;
// wave-uniform and read-only for the launch: scalar loads
typedef const __attribute__((address_space(4))) SecPhase kPhase;
typedef const __attribute__((address_space(4))) SecGate kGate;
typedef const __attribute__((address_space(4))) double kf64;
typedef const __attribute__((address_space(4))) uint32_t ku32;

// One row pass: the rows' tables (of the spin whose patterns index the row),
// the other spin's, and which layers' hops and diagonal it applies.
struct RowsArgs {
    const SecPhase *phases;
    const SecGate *gates;
    const Rec *recs;             // short rows
    const uint4 *lcode;          // long rows: slots and signs, two uint4 per thread and phase
    const uint4 *lpat;           //   patterns in phase 0's layout
    const double *lbase;         //   base values in phase 0's layout
    const uint16_t *colslot;     // slot of each row element
    const uint16_t *patslot;     // short rows: pattern and base value of each slot
    const double *baseslot;
    const uint32_t *rpat;        // the other spin: pattern, base value and
    const double *rbase;         //   coupling weights (16 per rank) of each row
    const double *wrow;
    const double *theta;
    double U;
    int n, n_rows, nslots, lr;
    int n_phases, per;
    int l_pre, l_diag, l_post;   // layer of the hops before the diagonal, of the
                                 // diagonal and of the hops after it (-1: none)
    int64_t rs, cs;              // element (row, col) at row rs + col cs
    const uint32_t *dnpat;       // in a full vector's place (SpreadAt): spin-down patterns,
    int ns, skew;                //   sites and the skew's mask
    double2 *v[2];
    double2 *t[2];               // long rows, SF_TURN: the transposed result
    double *partial;
    int row0[2];                 // first partial row of each vector
    int n_red, pstride, flags;
    int b0_row, b0_col;
    int grid;                    // workgroups of the pass (per vector)
};

// x from another lane of the same 16-lane row (DPP control CTRL), both
// 32-bit halves.
template <int CTRL>
__device__ __forceinline__ double row_dpp(double y)
{
    const long long b = __double_as_longlong(y);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

__device__ __forceinline__ double lane_value(double y, int l)
{
    const long long b = __double_as_longlong(y);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), l);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Sum of x over the wave, the same value in every lane: each 16-lane row
// summed by lane permutations (no LDS traffic), then the four rows' sums.
__device__ __forceinline__ double wave_sum(double x)
{
    x += row_dpp<0xB1>(x);    // quad_perm [1,0,3,2]: pairs
    x += row_dpp<0x4E>(x);    // quad_perm [2,3,0,1]: quads
    x += row_dpp<0x141>(x);   // row_half_mirror: the other quad of the half row
    x += row_dpp<0x140>(x);   // row_mirror: the other half of the row
    return (lane_value(x, 0) + lane_value(x, 16)) + (lane_value(x, 32) + lane_value(x, 48));
}

// ----------------------------------------------------------------- gates --

// x with the sign bits of mask (0 or 0x80000000) flipped.
__device__ __forceinline__ double xor_sign(double x, uint32_t mask)
{
    return __hiloint2double(__double2hiint(x) ^ (int)mask, __double2loint(x));
}

// x <- x m + q computed in the registers of x: the orbit is updated in place.
// (Left to itself the allocator writes a hop's results to fresh registers and
// copies the orbits back where branches meet: twice the registers, and hundreds
// of bytes per lane in scratch memory.)
__device__ __forceinline__ void fma_ip(double &x, double m, double q)
{
    asm("v_fma_f64 %0, %0, %1, %2" : "+v"(x) : "v"(m), "v"(q));
}

// (x, y) <- (c x + i s y, i s x + c y)
__device__ __forceinline__ void rotate(double2 &x, double2 &y, double c, double s)
{
    const double p = -s * y.y, q = s * y.x, u = -s * x.y, v = s * x.x;
    fma_ip(x.x, c, p);
    fma_ip(x.y, c, q);
    fma_ip(y.x, c, u);
    fma_ip(y.y, c, v);
}

__device__ __forceinline__ double re_dot(double2 a, double2 b) { return fma(a.x, b.x, a.y * b.y); }

// Position of the two-electron pattern {a, b} in an orbit of six.
__host__ __device__ constexpr int duo(int a, int b)
{
    return a > b ? duo(b, a) : (a == 0 ? b - 1 : a + b);   // 01 02 03 12 13 23
}

// The hop at position Q of a phase (sites A, B) on a thread's orbits: x[0..5]
// two electrons, x[6..9] one (by its site), x[10..13] three (by the empty
// site).  The orbits' sign bits are those of Rec.
//   REV: w <- w + the sum over the pairs of sign Re(conj(x_a) x_b), before the rotation
template <bool REV, int Q, int N>
__device__ __forceinline__ void hop2(double2 (&x)[N], double2 cs, uint32_t f, double &w)
{
    constexpr int A = kPosA[Q], B = kPosB[Q];
    constexpr int E0 = A != 0 && B != 0 ? 0 : (A != 1 && B != 1 ? 1 : 2);
    constexpr int E1 = 6 - A - B - E0;   // the spectators, E0 < E1
    constexpr int a0 = duo(A, E0), b0 = duo(B, E0), a1 = duo(A, E1), b1 = duo(B, E1);
    const uint32_t m0 = (f << (2 * Q)) & 0x80000000u, m1 = (f << (2 * Q + 1)) & 0x80000000u;
    if constexpr (REV)
        w += xor_sign(re_dot(x[a0], x[b0]), m0) + xor_sign(re_dot(x[a1], x[b1]), m1);
    rotate(x[a0], x[b0], cs.x, xor_sign(cs.y, m0));
    rotate(x[a1], x[b1], cs.x, xor_sign(cs.y, m1));
}

// O: where the one-electron orbit begins (the three-electron one follows).
template <bool REV, int Q, int O, int N>
__device__ __forceinline__ void hop13(double2 (&x)[N], double2 cs, uint32_t f1, uint32_t f3,
                                      double &w)
{
    constexpr int A1 = O + kPosA[Q], B1 = O + kPosB[Q], A3 = A1 + 4, B3 = B1 + 4;
    const uint32_t m1 = (f1 << (8 + Q)) & 0x80000000u, m3 = (f3 << (12 + Q)) & 0x80000000u;
    if constexpr (REV)
        w += xor_sign(re_dot(x[A1], x[B1]), m1) + xor_sign(re_dot(x[A3], x[B3]), m3);
    rotate(x[A1], x[B1], cs.x, xor_sign(cs.y, m1));
    rotate(x[A3], x[B3], cs.x, xor_sign(cs.y, m3));
}

// LDS of a row pass.
struct RowLds {
    uint32_t vec, ang, dtab, nib, rowp, rowb, acc, total;
};
__host__ __device__ inline RowLds row_lds(uint32_t vec_bytes, int rows, int n_phases, int n_red,
                                          int threads, bool gen)
{
    RowLds L;
    uint32_t at = vec_bytes;
    L.vec = 0;
    L.ang = at;
    at += 2u * (uint32_t)(n_phases * kPositions) * 16u;
    L.dtab = at;   // U-only: phases by the number of doubly occupied sites; else unit phases
    at += (gen ? 1u << kCisBits : (uint32_t)kDiagTab) * 16u;
    L.nib = at;    // per row: the coupling weights' sums over the pattern's nibbles
    at += gen ? (uint32_t)rows * 64u * 8u : 0u;
    L.rowb = at;
    at += (uint32_t)rows * 8u;
    L.rowp = at;
    at += ((uint32_t)rows * 4u + 15u) & ~15u;
    L.acc = at;
    at += (uint32_t)n_red * ((uint32_t)threads / 4u) * 8u;
    L.total = at;
    return L;
}
__host__ __device__ inline uint32_t short_vec_bytes(int nslots, int lr)
{
    return ((uint32_t)(nslots + 1) << lr) * 16u;
}
__host__ __device__ inline uint32_t long_vec_bytes(int nslots)
{
    return (uint32_t)(nslots + kLongDummy) * 8u;
}

// Work common to both row kernels.  A pass's steps: the phases of the hops
// before the diagonal, then those of the hops after it.
template <int MODE, bool GEN, typename AT>
struct RowPassCtx {
    static constexpr bool REV = MODE == S_REV;
    const AT &A;
    double2 *ang, *dtab;
    double *acc;
    int tid, T, dslot, post_slot;

    __device__ RowPassCtx(const AT &a, char *smem, const RowLds &L)
        : A(a), ang((double2 *)(smem + L.ang)), dtab((double2 *)(smem + L.dtab)),
          acc((double *)(smem + L.acc)), tid(threadIdx.x), T(blockDim.x)
    {
        // reduction slots: the groups of the hops before, the diagonal, the
        // groups of the hops after it
        dslot = A.l_pre >= 0 ? A.per - 1 : 0;
        post_slot = dslot + (A.l_diag >= 0 ? 1 : 0);
    }
    // rotation angles, phase tables, zeroed reduction rows (no barrier)
    __device__ void prologue()
    {
        const int n_gates = A.n_phases * kPositions;
        for (int i = tid; i < 2 * n_gates; i += T) {
            const int run = i >= n_gates ? 1 : 0, layer = run ? A.l_post : A.l_pre;
            if (layer < 0)
                continue;
            const gf64 *theta = (const gf64 *)A.theta;
            const __attribute__((address_space(1))) SecGate &g =
                ((const __attribute__((address_space(1))) SecGate *)A.gates)[i - run * n_gates];
            double s, c;
            sincos(theta[layer * A.per + g.slot] * g.t, &s, &c);
            ang[i] = make_double2(c, REV ? -s : s);
        }
        if (A.l_diag >= 0) {
            if constexpr (GEN) {
                build_cis(dtab, tid, T);
            } else {
                const double th = A.theta[A.l_diag * A.per];
                for (int k = tid; k < kDiagTab; k += T) {
                    double s, c;
                    sincos(th * (A.U * (double)k), &s, &c);
                    dtab[k] = make_double2(c, REV ? s : -s);
                }
            }
        }
        for (int i = tid; i < A.n_red * (T / 4); i += T)
            acc[i] = 0.0;
    }
    // a thread's sum of one reduction slot's terms into that slot: four lanes
    // are added in registers, one of them adds to the four's own LDS entry (an
    // add that nothing waits for)
    __device__ __forceinline__ void flush(int slot, double &racc)
    {
        double x = racc;
        x += row_dpp<0xB1>(x);
        x += row_dpp<0x4E>(x);
        if ((tid & 3) == 0)
            __hip_atomic_fetch_add(&acc[slot * (T / 4) + (tid >> 2)], x, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
        racc = 0.0;
    }
    // what a phase's hops need besides the orbits, read before anything waits:
    // angles, and in reverse the weights -2 t (<chi|G|chi> counts every pair
    // twice) and reduction slots
    struct PhaseArgs {
        double2 c[kPositions];
        double t[kPositions];
        int slot[kPositions], last[kPositions];
        bool on[kPositions];   // false: the position has no bond (reverse)
    };
    __device__ __forceinline__ PhaseArgs phase_args(int run, int ph) const
    {
        return phase_args(run, ph, run);
    }
    __device__ __forceinline__ PhaseArgs phase_args(int run, int ph, int buf) const
    {
        PhaseArgs a;
        const double2 *an = ang + (buf * A.n_phases + ph) * kPositions;
        const kGate *g = (const kGate *)A.gates + ph * kPositions;
        const int base = (run ? post_slot : 0) - 1;
#pragma unroll
        for (int q = 0; q < kPositions; ++q) {
            a.c[q] = an[q];
            a.on[q] = !REV || g[q].t != 0.0;
            if constexpr (REV) {
                a.t[q] = -2.0 * g[q].t;
                a.slot[q] = base + g[q].slot;
                a.last[q] = g[q].last;
            }
        }
        return a;
    }
    // positions Q, Q + 1 (one matching): two(c0, c1, p0, p1) applies them to
    // the thread's orbits
    template <int Q, typename F>
    __device__ __forceinline__ void matching(const PhaseArgs &a, double &racc, F &&two)
    {
        double p0 = 0.0, p1 = 0.0;
        two(a.c[Q], a.c[Q + 1], p0, p1);
        if constexpr (REV) {
            racc = fma(a.t[Q + 1], p1, racc);
            if (a.last[Q + 1])
                flush(a.slot[Q + 1], racc);
            racc = fma(a.t[Q], p0, racc);
            if (a.last[Q])
                flush(a.slot[Q], racc);
        }
    }
    template <typename F0, typename F2>
    __device__ __forceinline__ void both(const PhaseArgs &a, F0 &&first, F2 &&second)
    {
        double racc = 0.0;
        if constexpr (!REV) {
            matching<0>(a, racc, first);
            matching<2>(a, racc, second);
        } else {
            matching<2>(a, racc, second);
            matching<0>(a, racc, first);
        }
    }
    // the phase's hops on an orbit of six
    __device__ __forceinline__ void gates2(double2 (&x)[6], const PhaseArgs &a, uint32_t f)
    {
        both(a,
             [&](double2 c0, double2 c1, double &p0, double &p1) __attribute__((always_inline)) {
                 if (a.on[0])
                     hop2<REV, 0>(x, c0, f, p0);
                 if (a.on[1])
                     hop2<REV, 1>(x, c1, f, p1);
             },
             [&](double2 c0, double2 c1, double &p0, double &p1) __attribute__((always_inline)) {
                 if (a.on[2])
                     hop2<REV, 2>(x, c0, f, p0);
                 if (a.on[3])
                     hop2<REV, 3>(x, c1, f, p1);
             });
    }
    // on two orbits of four
    __device__ __forceinline__ void gates13(double2 (&x)[8], const PhaseArgs &a, uint32_t f1,
                                            uint32_t f3)
    {
        both(a,
             [&](double2 c0, double2 c1, double &p0, double &p1) __attribute__((always_inline)) {
                 if (a.on[0])
                     hop13<REV, 0, 0>(x, c0, f1, f3, p0);
                 if (a.on[1])
                     hop13<REV, 1, 0>(x, c1, f1, f3, p1);
             },
             [&](double2 c0, double2 c1, double &p0, double &p1) __attribute__((always_inline)) {
                 if (a.on[2])
                     hop13<REV, 2, 0>(x, c0, f1, f3, p0);
                 if (a.on[3])
                     hop13<REV, 3, 0>(x, c1, f1, f3, p1);
             });
    }
    // on all of a long row's orbits (w2, w13: the wave has any of the kind)
    __device__ __forceinline__ void gates(double2 (&x)[kOrbitElems], const PhaseArgs &a, uint32_t f,
                                          bool w2, bool w13)
    {
        both(a,
             [&](double2 c0, double2 c1, double &p0, double &p1) __attribute__((always_inline)) {
                 if (w2) {
                     hop2<REV, 0>(x, c0, f, p0);
                     hop2<REV, 1>(x, c1, f, p1);
                 }
                 if (w13) {
                     hop13<REV, 0, 6>(x, c0, f, f, p0);
                     hop13<REV, 1, 6>(x, c1, f, f, p1);
                 }
             },
             [&](double2 c0, double2 c1, double &p0, double &p1) __attribute__((always_inline)) {
                 if (w2) {
                     hop2<REV, 2>(x, c0, f, p0);
                     hop2<REV, 3>(x, c1, f, p1);
                 }
                 if (w13) {
                     hop13<REV, 2, 6>(x, c0, f, f, p0);
                     hop13<REV, 3, 6>(x, c1, f, f, p1);
                 }
             });
    }
    // the workgroup's partial sums (after a barrier)
    __device__ void finish(int bid, int vsel, bool negate)
    {
        const int lane = tid & 63, wave = tid >> 6, R = T / 4;
        for (int r = wave; r < A.n_red; r += T >> 6) {
            double s = 0.0;
            for (int i = lane; i < R; i += 64)
                s += acc[r * R + i];
            s = wave_sum(s);
            if (lane == 0)
                A.partial[(size_t)(A.row0[vsel] + r) * A.pstride + bid] = negate ? -s : s;
        }
    }
};

// D's value of an element from its row's nibble sums: the row's and the
// pattern's own terms and the coupling sum_j p_j w_j.  err: the last sum's
// rounding (the phase exp(-i th D) needs it: D is large against pi).
__device__ __forceinline__ double diag_gen(double rb, double cb, const double *nib, uint32_t cp,
                                           double &err)
{
    const double a = rb + cb;
    const double b = (nib[cp & 15u] + nib[16 + ((cp >> 4) & 15u)]) +
                     (nib[32 + ((cp >> 8) & 15u)] + nib[48 + (cp >> 12)]);
    const double d = a + b, t = d - a;
    err = (a - (d - t)) + (b - t);
    return d;
}
__device__ __forceinline__ double diag_gen(double rb, double cb, const double *nib, uint32_t cp)
{
    double err;
    return diag_gen(rb, cb, nib, cp, err);
}

__device__ __forceinline__ double nibble_sum(const gf64 *w, int e)
{
    const gf64 *q = w + (e >> 4) * 4;
    double s = 0.0;
#pragma unroll
    for (int b = 0; b < 4; ++b)
        s += (e >> b) & 1 ? q[b] : 0.0;
    return s;
}

// The diagonal on one element: exp(-i th D) forward, the bracket D |a|^2 and
// exp(+i th D) in reverse.
template <bool REV, bool GEN>
__device__ __forceinline__ void diag_el(double2 &a, double d, double err, double2 ph, double th,
                                        const double2 *cis, double &racc)
{
    if constexpr (GEN) {
        const double t = REV ? -th : th, x = t * d;
        ph = cis_neg(x, cis, fma(t, d, -x) + t * err);
    }
    if constexpr (REV)
        racc = fma(d, fma(a.x, a.x, a.y * a.y), racc);
    a = make_double2(fma(ph.x, a.x, -ph.y * a.y), fma(ph.x, a.y, ph.y * a.x));
}

// Workgroup i of a launch works on row group group_of(i): workgroups go to
// the eight XCDs in turn, and each XCD takes a contiguous range of groups, so
// that the lines shared by neighbouring groups of a column pass meet in one L2.
__device__ __forceinline__ int group_of(int i, int n)
{
    const int chunk = (n + 7) / 8;
    const int g = (i & 7) * chunk + (i >> 3);
    return (i >> 3) < chunk && g < n ? g : -1;
}

// A sector vector kept in the memory of the full vector that it becomes: the
// amplitudes of a spin-down pattern, packed, in the pattern's own row of the
// full vector, so that every row can be expanded by itself.  The skew (128
// bytes per rank, under half a row: the patterns with a given number of
// electrons are at most half of all) keeps a column's elements off one memory
// channel.
__device__ __forceinline__ int64_t spread_at(const gu32 *dnpat, int rank, int ns, int skew)
{
    return ((int64_t)dnpat[rank] << ns) + ((rank * 8) & skew);
}

// ------------------------------------------------------------ short rows --
// 2^lr rows of up to kShortRow elements per workgroup, in LDS: element (slot,
// row) at slot 2^lr + row, lanes with the row in their low bits.  Each phase
// reads a thread's orbits, rotates them in registers and writes them back to
// the same slots: one barrier per phase.  The slots' bank classes keep the
// lanes of an LDS access apart (sector_plan.cpp).
// Bound by latency and VALU, not by HBM (24-qubit ladder, 924 x 924: 13.6 MB
// per vector).  One exchange per phase instead of one per hop, several rows
// per workgroup and no transposes took its energy+gradient evaluation with
// the general diagonal from 4.19 to 1.03 ms, and a 20-qubit chain's from 0.554
// to 0.283 ms.  Half the threads for the orbits of six and half for those of
// four, a phase's records and scalars fetched a phase ahead, and the diagonal's
// tables four elements at a time: 1.02 and 0.189 ms; a 16-qubit chain 0.219 to
// 0.149 ms, a 28-qubit ladder 4.18 to 3.36 ms.  A reverse phase's positions
// without a bond skipped: 0.98 and 0.188, 0.148 and 3.23 ms (forward, where
// nothing else reads the gates, the skip cost more than it gave).
//   S_FWD: v[0] <- ops applied.  SF_START: the input is |b0>, not read; the
//          rows without it are zero.
//   S_REV: vsel picks chi2 = v[0] or chi1 = v[1]; the ops un-applied in
//          reverse order, <chi|G|chi> of every hop and of D before its
//          un-application added to its reduction slot (chi1's negated).  The
//          bracket Im <lambda|G|psi> is (<chi2|G|chi2> - <chi1|G|chi1>) / 4
//          with chi1, chi2 = lambda / m +- i m psi for any m: one near the
//          square root of |lambda| / |psi| keeps the difference's rounding
//          as small as the bracket's own.
//   SPREAD: the vector lies inside the full vector that it is going to become
//          (spread_at).
template <int MODE, bool GEN, bool SPREAD, typename AT>
__device__ __forceinline__ void rows_short(const AT &A, int bid, int vsel, char *smem)
{
    constexpr bool REV = MODE == S_REV;
    const int tid = threadIdx.x, T = blockDim.x, lr = A.lr, R = 1 << lr;
    const RowLds L = row_lds(short_vec_bytes(A.nslots, lr), R, A.n_phases, A.n_red, T, GEN);
    RowPassCtx<MODE, GEN, AT> C(A, smem, L);
    double2 *vec = (double2 *)smem;
    double *nib = (double *)(smem + L.nib), *rowb = (double *)(smem + L.rowb);
    uint32_t *rowp = (uint32_t *)(smem + L.rowp);
    gc128 *__restrict__ v = (gc128 *)A.v[vsel];
    const gu16 *__restrict__ colslot = (const gu16 *)A.colslot;
    const gu16 *__restrict__ patslot = (const gu16 *)A.patslot;
    const gu128 *__restrict__ recs = (const gu128 *)A.recs;
    C.prologue();
    for (int i = tid; i < (A.nslots + 1) << lr; i += T)   // holes and the dummy slot stay zero
        vec[i] = make_double2(0.0, 0.0);
    const int n_pre = A.l_pre >= 0 ? A.n_phases : 0;
    const int n_steps = n_pre + (A.l_post >= 0 ? A.n_phases : 0);
    // the first half of the threads takes the orbits of six, the second half
    // those of four (a thread one with one and one with three electrons): the
    // same work for either, in half the time of one thread taking all three
    const int TH = T >> 1;
    const bool duo_half = __builtin_amdgcn_readfirstlane(tid) < TH;
    const int row = tid & (R - 1), orb = (duo_half ? tid : tid - TH) >> lr, lanes = TH >> lr;
    const uint32_t rofs = (uint32_t)row * 16u;
    const int ng = (A.n_rows + R - 1) >> lr, total = A.n << lr;

    // the elements' rows and columns of load and store: rows in the low bits
    auto each = [&](auto &&f) __attribute__((always_inline)) {
        for (int i0 = tid; i0 < total; i0 += 4 * T) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = i0 + u * T;
                if (i < total)
                    f(u, i >> lr);
            }
        }
    };
    for (int ig = bid; ig < (ng + 7) / 8 * 8; ig += A.grid) {
        const int g = group_of(ig, ng);
        if (g < 0)
            continue;
        const int r = (g << lr) + row;
        const bool live = r < A.n_rows;
        // element (r, col); a spread vector's row is the one of the two that
        // indexes spin-down patterns (cs 1: the rows do)
        gc128 *__restrict__ vr;
        if constexpr (SPREAD)
            vr = v + (A.cs == 1 ? spread_at((const gu32 *)A.dnpat, min(r, A.n_rows - 1), A.ns,
                                            A.skew)
                                : (int64_t)r);
        else
            vr = v + (int64_t)r * A.rs;
        auto elem = [&](int col) __attribute__((always_inline)) -> gc128 * {
            if constexpr (SPREAD)
                return vr + (A.cs == 1 ? (int64_t)col
                                       : spread_at((const gu32 *)A.dnpat, col, A.ns, A.skew));
            else
                return vr + (int64_t)col * A.cs;
        };
        if constexpr (!REV) {
            if (A.flags & SF_START) {
                const bool here = (g << lr) <= A.b0_row && A.b0_row < ((g + 1) << lr);
                if (!here) {
                    for (int i = tid; i < total; i += T)
                        if (live) {
                            gc128 *p = elem(i >> lr);
                            p->x = 0.0;
                            p->y = 0.0;
                        }
                    continue;
                }
            }
        }
        const bool start = !REV && (A.flags & SF_START);
        __syncthreads();
        for (int i0 = tid; i0 < total; i0 += 4 * T) {
            double2 x[4];
            int sl[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = i0 + u * T, col = min(i, total - 1) >> lr;
                x[u] = make_double2(0.0, 0.0);
                sl[u] = colslot[col];
                if (start) {
                    x[u].x = r == A.b0_row && col == A.b0_col ? 1.0 : 0.0;
                } else if (live && i < total) {
                    const gc128 *p = elem(col);
                    x[u] = make_double2(p->x, p->y);
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (i0 + u * T < total)
                    vec[(sl[u] << lr) + row] = x[u];
        }
        if (A.l_diag >= 0) {
            const gu32 *rpat = (const gu32 *)A.rpat;
            const gf64 *rbase = (const gf64 *)A.rbase, *wrow = (const gf64 *)A.wrow;
            for (int i = tid; i < R; i += T) {
                const int rr = min((g << lr) + i, A.n_rows - 1);
                rowp[i] = rpat[rr];
                rowb[i] = rbase[rr];
            }
            if constexpr (GEN)
                for (int i = tid; i < 64 << lr; i += T)
                    nib[i] = nibble_sum(wrow + (size_t)min((g << lr) + (i >> 6), A.n_rows - 1) * 16,
                                        i & 63);
        }
        auto diag = [&]() __attribute__((always_inline)) {
            const double th = A.theta[A.l_diag * A.per];
            const uint32_t rp = rowp[row];
            const double rb = GEN ? rowb[row] : 0.0;
            const double *nb = nib + row * 64;
            const gf64 *baseslot = (const gf64 *)A.baseslot;
            double racc = 0.0;
            const int last = (A.nslots << lr) - 1;
            for (int i0 = tid; i0 <= last; i0 += 4 * T) {
                uint32_t cp[4];
                double cb[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {   // the tables' loads in flight together
                    const int sl = min(i0 + u * T, last) >> lr;
                    cp[u] = patslot[sl];
                    cb[u] = GEN ? baseslot[sl] : 0.0;
                }
                double2 a[4];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    a[u] = vec[min(i0 + u * T, last)];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    double sum = racc;
                    if constexpr (GEN) {
                        double err;
                        const double d = diag_gen(rb, cb[u], nb, cp[u], err);
                        diag_el<REV, true>(a[u], d, err, a[u], th, C.dtab, sum);
                    } else {
                        const int k = __popc(rp & cp[u]);
                        diag_el<REV, false>(a[u], A.U * (double)k, 0.0, C.dtab[k], th, nullptr,
                                            sum);
                    }
                    if (i0 + u * T <= last) {
                        vec[i0 + u * T] = a[u];
                        racc = sum;
                    }
                }
            }
            if constexpr (REV)
                C.flush(C.dslot, racc);
            __syncthreads();
        };
        // records of a step's orbits (the next step's are fetched while one runs)
        struct Recs {
            uint4 a, b;
        };
        auto fetch = [&](int st) __attribute__((always_inline)) {
            const int first = (3 * (st < A.n_phases ? st : st - A.n_phases) + (duo_half ? 0 : 1)) *
                                  lanes + orb;
            auto ld = [&](int i) __attribute__((always_inline)) {
                const gu128 *p = recs + i;
                return make_uint4(p->x, p->y, p->z, p->w);
            };
            Recs q;
            q.a = ld(first);
            q.b = ld(first + (duo_half ? 0 : lanes));   // no branch around a load in flight
            return q;
        };
        // element j of a record
        auto at = [&](const uint4 &q, int j) __attribute__((always_inline)) -> double2 & {
            const uint32_t w = j < 2 ? q.x : (j < 4 ? q.y : q.z);
            return *(double2 *)(smem + ((j & 1 ? w >> 16 : w & 0xFFFFu) << 4) + rofs);
        };
        auto phase = [&](int st, const Recs &q) __attribute__((always_inline)) {
            const int p = st < A.n_phases ? st : st - A.n_phases;
            const typename RowPassCtx<MODE, GEN, AT>::PhaseArgs pa =
                C.phase_args(st < n_pre ? 0 : 1, p);
            if (duo_half) {
                const bool act = q.a.w & 1u;
                if (__ballot(act)) {
                    double2 x[6];
#pragma unroll
                    for (int j = 0; j < 6; ++j)
                        x[j] = at(q.a, j);
                    C.gates2(x, pa, q.a.w);
                    if (act) {
#pragma unroll
                        for (int j = 0; j < 6; ++j)
                            at(q.a, j) = x[j];
                    }
                }
            } else {
                const bool a1 = q.a.z & 1u, a3 = q.b.z & 1u;
                if (__ballot(a1 || a3)) {
                    double2 x[8];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        x[j] = at(q.a, j);
                        x[4 + j] = at(q.b, j);
                    }
                    C.gates13(x, pa, q.a.z, q.b.z);
                    if (a1) {
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            at(q.a, j) = x[j];
                    }
                    if (a3) {
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            at(q.b, j) = x[4 + j];
                    }
                }
            }
            __syncthreads();
        };
        Recs cur{};
        if (n_steps > 0)
            cur = fetch(REV ? n_steps - 1 : 0);
        __syncthreads();
        for (int k = 0; k < n_steps; ++k) {
            const int st = REV ? n_steps - 1 - k : k;
            if (!REV && st == n_pre && A.l_diag >= 0)
                diag();
            const int nx = min(k + 1, n_steps - 1);
            const Recs nxt = fetch(REV ? n_steps - 1 - nx : nx);
            phase(st, cur);
            cur = nxt;
            if (REV && st == n_pre && A.l_diag >= 0)
                diag();
        }
        if (!(A.flags & SF_NO_STORE) && live) {
            each([&](int, int col) __attribute__((always_inline)) {
                const double2 x = vec[(colslot[col] << lr) + row];
                gc128 *p = elem(col);
                p->x = x.x;
                p->y = x.y;
            });
        }
    }
    if constexpr (REV) {
        __syncthreads();
        C.finish(bid, vsel, vsel == 1);
    }
}

template <int MODE, bool GEN>
__global__ void __launch_bounds__(1024) k_sec_rows_short(RowsArgs A)
{
    extern __shared__ __align__(16) char smem[];
    rows_short<MODE, GEN, false>(A, (int)blockIdx.x, MODE == S_REV ? (int)blockIdx.y : 0, smem);
}

// A forward pass on a vector spread over its full vector's memory.
template <bool GEN>
__global__ void __launch_bounds__(1024) k_sec_rows_spread(RowsArgs A)
{
    extern __shared__ __align__(16) char smem[];
    rows_short<S_FWD, GEN, true>(A, (int)blockIdx.x, 0, smem);
}

// The full vector from a spread one, in place: a workgroup reads a spin-down
// pattern's amplitudes into LDS and writes the pattern's whole row, a spin-up
// pattern's amplitude found by its rank: patterns are in numeric order, so the
// rank is the number of sector patterns with smaller high bits plus the rank of
// the low six bits among those with the same number of electrons.
// Bound by the full vector's write (24 qubits, 268 MB: 40 us).
__global__ void __launch_bounds__(512)
k_sec_expand(double2 *vec, int ns, int skew, int n_up, int e_up, int e_dn)
{
    extern __shared__ __align__(16) char smem[];
    double2 *row = (double2 *)smem;
    gc128 *v = (gc128 *)vec;
    const int tid = threadIdx.x, T = blockDim.x;
    const int lb = min(ns, 6), nhi = 1 << (ns - lb), lmask = (1 << lb) - 1;
    int *first[2];   // of each spin's patterns, by their high bits
    first[0] = (int *)(smem + (size_t)n_up * 16);
    first[1] = first[0] + nhi;
    int *lo_rank = first[1] + nhi, *binom = lo_rank + 64;
    if (tid < 64) {
        int k = 0;
        for (int j = 0; j < tid; ++j)
            k += __popc(j) == __popc(tid) ? 1 : 0;
        lo_rank[tid] = k;
    }
    if (tid < 8) {
        int c = tid <= lb ? 1 : 0;
        for (int q = 0; q < tid && q < lb; ++q)
            c = c * (lb - q) / (q + 1);
        binom[tid] = c;
    }
    __syncthreads();
    for (int i = tid; i < 2 * nhi; i += T) {
        const int e0 = i < nhi ? e_up : e_dn;
        int k = 0;
        for (int j = 0; j < (i & (nhi - 1)); ++j) {
            const int e = e0 - __popc(j);   // electrons left for the low bits
            k += e >= 0 && e <= lb ? binom[e] : 0;
        }
        first[0][i] = k;
    }
    const int n_rows = 1 << ns;
    for (int d = blockIdx.x; d < n_rows; d += gridDim.x) {
        gc128 *out = v + ((int64_t)d << ns);
        const bool in = __popc(d) == e_dn;
        __syncthreads();   // the tables; the last row's reads
        if (in) {
            const int rank = first[1][d >> lb] + lo_rank[d & lmask];
            const gc128 *x = out + ((rank * 8) & skew);
            for (int i = tid; i < n_up; i += T)
                row[i] = make_double2(x[i].x, x[i].y);
            __syncthreads();
        }
        for (int i = tid; i < n_rows; i += T) {
            double2 a = make_double2(0.0, 0.0);
            if (in && __popc(i) == e_up)
                a = row[first[0][i >> lb] + lo_rank[i & lmask]];
            out[i].x = a.x;
            out[i].y = a.y;
        }
    }
}

// A batch's pass: every workgroup runs one workgroup's part of one instance's
// pass, the same work in the same order as that instance's own launch.
struct SecWork {
    int32_t args, bid, vsel, pad;
};
typedef const __attribute__((address_space(4))) RowsArgs kRowsArgs;

template <int MODE, bool GEN>
__global__ void __launch_bounds__(1024)
k_sec_rows_batch(const RowsArgs *__restrict__ args, const SecWork *__restrict__ work)
{
    extern __shared__ __align__(16) char smem[];
    const SecWork w = work[blockIdx.x];
    rows_short<MODE, GEN, false>(((kRowsArgs *)args)[w.args], w.bid, w.vsel, smem);
}

// ------------------------------------------------------------- long rows --
// One row of up to 13312 elements per workgroup of 1024 threads, in
// registers; a phase's layout gives each thread one orbit of six, two of four
// and one single element.  Between phases the row goes through LDS, real
// parts first, then imaginary parts: 16 bytes per element would not fit.
// Modes, vectors and reductions as in k_sec_rows_short.
// Bound by LDS traffic and VALU: 206 KB go through LDS in each direction per
// phase, eight phases per layer and spin at 4x4 periodic where an exchange per
// hop needed 32.  At 12870 x 12870 (5.3 GB, 9.2 by the counters) a forward pass of 64 hops
// with its transposed store takes 3.9 ms (an exchange per hop and a transpose:
// 9.1 ms), the reverse pass of both vectors 8.6 (20.9).  The diagonal's
// products must not be put off past flush: kept waiting there they spilled 750
// bytes per thread in reverse, 55 against 40 ms per evaluation of a general
// torus of two layers.
struct LongCodes {
    uint32_t w[8];
    // LDS byte offset of element j
    __device__ __forceinline__ uint32_t at(int j) const
    {
        return j & 1 ? (w[j >> 1] >> 13) & 0x7FFF8u : (w[j >> 1] << 3) & 0x7FFF8u;
    }
    __device__ __forceinline__ void renew()
    {
#pragma unroll
        for (int k = 0; k < 8; ++k)
            asm volatile("" : "+v"(w[k]));
    }
};

// LDS byte offsets of a layout's N elements, unpacked once for the real and
// the imaginary parts (kept through the hops instead, they spilled).
template <int N> struct LongAddr {
    uint32_t a[N];
    __device__ __forceinline__ explicit LongAddr(const LongCodes &c)
    {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            a[j] = c.at(j);
            asm volatile("" : "+v"(a[j]));
        }
    }
};

__device__ __forceinline__ LongCodes long_codes(const gu128 *p)
{
    LongCodes c;
    const uint4 a = make_uint4(p[0].x, p[0].y, p[0].z, p[0].w);
    const uint4 b = make_uint4(p[1].x, p[1].y, p[1].z, p[1].w);
    c.w[0] = a.x;
    c.w[1] = a.y;
    c.w[2] = a.z;
    c.w[3] = a.w;
    c.w[4] = b.x;
    c.w[5] = b.y;
    c.w[6] = b.z;
    c.w[7] = b.w;
    return c;
}

// The row's slots of a thread's elements t + j kLongT (two chunks of eight).
__device__ __forceinline__ LongCodes col_codes(const uint16_t *colslot, int t)
{
    const gu128 *p = (const gu128 *)colslot;
    LongCodes c;
    const uint4 a = make_uint4(p[t].x, p[t].y, p[t].z, p[t].w);
    const uint4 b = make_uint4(p[kLongT + t].x, p[kLongT + t].y, p[kLongT + t].z,
                               p[kLongT + t].w);
    c.w[0] = a.x;
    c.w[1] = a.y;
    c.w[2] = a.z;
    c.w[3] = a.w;
    c.w[4] = b.x;
    c.w[5] = b.y;
    c.w[6] = b.z;
    c.w[7] = b.w;
    return c;
}

// Move a row from one register layout to another through LDS.
template <int NF, int NTO>
__device__ __forceinline__ void long_exchange(const double2 (&from)[NF], const LongCodes &fcodes,
                                              double2 (&to)[NTO], const LongCodes &tcodes)
{
    double re[NTO];
    const LongAddr<NF> cf(fcodes);
    __syncthreads();   // the last exchange's reads are done
#pragma unroll
    for (int j = 0; j < NF; ++j)
        *lds_at(cf.a[j]) = from[j].x;
    const LongAddr<NTO> ct(tcodes);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NTO; ++j)
        re[j] = *lds_at(ct.a[j]);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NF; ++j)
        *lds_at(cf.a[j]) = from[j].y;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NTO; ++j)
        to[j] = make_double2(re[j], *lds_at(ct.a[j]));
}

template <int MODE, bool GEN>
__global__ void __launch_bounds__(kLongT) k_sec_rows_long(RowsArgs A)
{
    constexpr bool REV = MODE == S_REV;
    extern __shared__ __align__(16) char smem[];
    const int tid = threadIdx.x;
    const RowLds L = row_lds(long_vec_bytes(A.nslots), 1, A.n_phases, A.n_red, kLongT, GEN);
    RowPassCtx<MODE, GEN, RowsArgs> C(A, smem, L);
    double *nib = (double *)(smem + L.nib);
    const int vsel = REV ? (int)blockIdx.y : 0;
    const kPhase *__restrict__ phases = (const kPhase *)A.phases;
    const gu128 *__restrict__ lcode = (const gu128 *)A.lcode;
    const ku32 *__restrict__ rpat = (const ku32 *)A.rpat;
    const kf64 *__restrict__ rbase = (const kf64 *)A.rbase;
    C.prologue();
    if (tid < kLongDummy)
        ((double *)smem)[A.nslots + tid] = 0.0;
    const int n_pre = A.l_pre >= 0 ? A.n_phases : 0;
    const int n_steps = n_pre + (A.l_post >= 0 ? A.n_phases : 0);
    const int wave0 = __builtin_amdgcn_readfirstlane(tid & ~63);
    const uint32_t n = (uint32_t)A.n;
    auto ph_of = [&](int st) { return st < A.n_phases ? st : st - A.n_phases; };

    for (int ig = blockIdx.x; ig < (A.n_rows + 7) / 8 * 8; ig += A.grid) {
        const int r = group_of(ig, A.n_rows);
        if (r < 0)
            continue;
        gc128 *__restrict__ row = (gc128 *)A.v[vsel] + (size_t)r * n;
        const bool start = !REV && (A.flags & SF_START);
        auto put = [&](uint32_t i, double2 v) __attribute__((always_inline)) {
            if (!(A.flags & SF_TURN) || (A.flags & SF_BOTH)) {
                row[i].x = v.x;
                row[i].y = v.y;
            }
            if (A.flags & SF_TURN) {
                gc128 *p = (gc128 *)A.t[vsel] + (size_t)i * A.n_rows + r;
                p->x = v.x;
                p->y = v.y;
            }
        };
        uint32_t t = (uint32_t)tid;   // per-row addresses are not kept across rows
        asm volatile("" : "+v"(t));
        if (start && r != A.b0_row) {
            for (uint32_t i = t; i < n; i += kLongT)
                put(i, make_double2(0.0, 0.0));
            continue;
        }
        double2 x[kOrbitElems];
        int p0 = ph_of(REV ? n_steps - 1 : 0);
        LongCodes cur = long_codes(lcode + ((size_t)p0 * kLongT + t) * 2);
        {
            double2 in[kLongElems];
            if (start) {
#pragma unroll
                for (int j = 0; j < kLongElems; ++j)
                    in[j] = make_double2(
                        t + (uint32_t)(j * kLongT) == (uint32_t)A.b0_col ? 1.0 : 0.0, 0.0);
            } else {
                // past the row's end: zeros, into the dummy slots
#pragma unroll
                for (int j = 0; j < kLongElems; ++j) {
                    const uint32_t i = t + (uint32_t)(j * kLongT), ic = min(i, n - 1);
                    in[j] = make_double2(row[ic].x, row[ic].y);
                    in[j] = i < n ? in[j] : make_double2(0.0, 0.0);
                }
            }
            const LongCodes cc = col_codes(A.colslot, (int)t);
            if constexpr (GEN)
                if (A.l_diag >= 0) {
                    __syncthreads();   // the diagonal may have been the last row's last step
                    if (tid < 64)      // read after the exchange's barriers
                        nib[tid] = nibble_sum((const gf64 *)A.wrow + (size_t)r * 16, tid);
                }
            long_exchange(in, cc, x, cur);
        }
        auto diag = [&]() __attribute__((always_inline)) {
            const double th = A.theta[A.l_diag * A.per];
            const uint32_t rp = rpat[r];
            const double rb = GEN ? rbase[r] : 0.0;
            uint32_t td = (uint32_t)tid;   // the tables' values are loaded here, not kept
            asm volatile("" : "+v"(td));
            const LongCodes pt = long_codes((const gu128 *)A.lpat + (size_t)td * 2);
            const gf64 *lbase = (const gf64 *)A.lbase;
            double racc = 0.0;
#pragma unroll
            for (int j = 0; j < kOrbitElems; ++j) {
                const uint32_t cp = (pt.w[j >> 1] >> (16 * (j & 1))) & 0xFFFFu;
                if constexpr (GEN) {
                    double err;
                    const double d = diag_gen(rb, lbase[j * kLongT + td], nib, cp, err);
                    diag_el<REV, true>(x[j], d, err, x[j], th, C.dtab, racc);
                } else {
                    const int k = __popc(rp & cp);
                    diag_el<REV, false>(x[j], A.U * (double)k, 0.0, C.dtab[k], th, nullptr, racc);
                }
                // fewer values in flight, and none of the products put off past flush
                asm volatile("" : "+v"(x[j].x), "+v"(x[j].y));
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (REV)
                C.flush(C.dslot, racc);
        };
        for (int k = 0; k < n_steps; ++k) {
            const int st = REV ? n_steps - 1 - k : k;
            const kPhase &ph = phases[ph_of(st)];
            if (!REV && st == n_pre && A.l_diag >= 0)
                diag();
            const uint32_t f = cur.w[7];
            C.gates(x, C.phase_args(st < n_pre ? 0 : 1, ph_of(st)), f, wave0 < ph.n[0],
                    wave0 < ph.n[1] || wave0 < ph.n[2]);
            if (REV && st == n_pre && A.l_diag >= 0)
                diag();
            if (k + 1 < n_steps) {
                // the next layout: wanted once the real parts are written
                const int pn = ph_of(REV ? st - 1 : st + 1);
                uint32_t tn = (uint32_t)tid;
                asm volatile("" : "+v"(tn));
                const LongCodes nxt = long_codes(lcode + ((size_t)pn * kLongT + tn) * 2);
                double2 y[kOrbitElems];
                long_exchange(x, cur, y, nxt);
                cur = nxt;
#pragma unroll
                for (int j = 0; j < kOrbitElems; ++j)
                    x[j] = y[j];
            }
        }
        if (!(A.flags & SF_NO_STORE)) {
            uint32_t ts = (uint32_t)tid;
            asm volatile("" : "+v"(ts));
            double2 out[kLongElems];
            long_exchange(x, cur, out, col_codes(A.colslot, (int)ts));
#pragma unroll
            for (int j = 0; j < kLongElems; ++j) {
                const uint32_t i = ts + (uint32_t)(j * kLongT);
                if (i < n)
                    put(i, out[j]);
            }
        }
    }
    if constexpr (REV) {
        __syncthreads();
        C.finish((int)blockIdx.x, vsel, vsel == 1);
    }
}

// --------------------------------------------------------------------- H --
// The part of H that acts on one spin's rows: every hop of that spin, and
// with `diag` the diagonal.  An element sums its partners' values over the
// bonds; a table names each partner's slot and sign (an inactive element's
// code names a zero slot).
struct HamArgs {
    const uint16_t *colslot, *patslot, *hcode;
    const double *baseslot;
    const uint32_t *rpat;
    const double *rbase, *wrow, *tb;   // tb: -t_b per bond, padded with zeros
    double U;
    int n, n_rows, nslots, lr, nb, diag, out_mode, turn;   // turn (long rows): out is transposed
    int n_flat;                        // long rows: bonds without a sign, which come first
    int64_t rs, cs;
    double2 *psi, *out;
    double mix;                        // HO_MIX: m, a power of two
    double *partial;                   // NULL: no energy
    int grid;
};

// sign bit of a code (bit 15, or bit 31 of the packed dword)
__device__ __forceinline__ uint32_t code_sign(uint32_t w, int odd)
{
    return odd ? w & 0x80000000u : (w << 16) & 0x80000000u;
}

// Store phi's element as the pass asks.
__device__ __forceinline__ void ham_store(int mode, double m, gc128 *out, gc128 *psi, double2 phi,
                                          double2 own)
{
    if (mode == HO_NONE)
        return;
    if (mode != HO_SET) {
        phi.x += out->x;
        phi.y += out->y;
    }
    if (mode == HO_MIX) {
        const double im = 1.0 / m;   // exact
        phi = make_double2(phi.x * im, phi.y * im);
        own = make_double2(own.x * m, own.y * m);
        psi->x = phi.x - own.y;
        psi->y = phi.y + own.x;
        phi = make_double2(phi.x + own.y, phi.y - own.x);
    }
    out->x = phi.x;
    out->y = phi.y;
}

template <bool GEN, typename AT>
__device__ __forceinline__ void ham_short(const AT &A, int bid, char *smem)
{
    const int tid = threadIdx.x, T = blockDim.x, lr = A.lr, R = 1 << lr;
    double2 *vec = (double2 *)smem;
    double *nib = (double *)(smem + short_vec_bytes(A.nslots, lr));
    double *wsum = nib + (GEN ? 64 << lr : 0);
    const int row = tid & (R - 1), total = A.n << lr, ng = (A.n_rows + R - 1) >> lr;
    const gu16 *colslot = (const gu16 *)A.colslot, *patslot = (const gu16 *)A.patslot;
    const gu32 *rpat = (const gu32 *)A.rpat;
    const gf64 *rbase = (const gf64 *)A.rbase, *wrow = (const gf64 *)A.wrow;
    const gf64 *baseslot = (const gf64 *)A.baseslot;
    const kf64 *tb = (const kf64 *)A.tb;
    const int chunks = (A.nb + 7) / 8;
    if (tid < R)
        vec[(A.nslots << lr) + tid] = make_double2(0.0, 0.0);
    double e = 0.0;
    for (int ig = bid; ig < (ng + 7) / 8 * 8; ig += A.grid) {
        const int g = group_of(ig, ng);
        if (g < 0)
            continue;
        const int r = min((g << lr) + row, A.n_rows - 1);
        const bool live = (g << lr) + row < A.n_rows;
        gc128 *psi = (gc128 *)A.psi + (int64_t)r * A.rs, *out = (gc128 *)A.out + (int64_t)r * A.rs;
        __syncthreads();   // the last group's reads are done
        for (int i = tid; i < total; i += T) {
            const gc128 *p = psi + (int64_t)(i >> lr) * A.cs;
            vec[((int)colslot[i >> lr] << lr) + row] = make_double2(p->x, p->y);
        }
        if (GEN && A.diag)
            for (int i = tid; i < 64 << lr; i += T)
                nib[i] = nibble_sum(wrow + (size_t)min((g << lr) + (i >> 6), A.n_rows - 1) * 16,
                                    i & 63);
        __syncthreads();
        const uint32_t rp = rpat[r];
        const double rb = GEN ? rbase[r] : 0.0;
        for (int i = tid; i < total; i += T) {
            const int col = i >> lr, sl = colslot[col];
            const double2 own = vec[(sl << lr) + row];
            double2 phi = make_double2(0.0, 0.0);
            if (A.diag) {
                const uint32_t cp = patslot[sl];
                const double d = GEN ? diag_gen(rb, baseslot[sl], nib + row * 64, cp)
                                     : A.U * (double)__popc(rp & cp);
                phi = make_double2(d * own.x, d * own.y);
            }
            const gu128 *hc = (const gu128 *)A.hcode + (size_t)col * chunks;
            for (int c = 0; c < chunks; ++c) {
                const uint32_t w[4] = {hc[c].x, hc[c].y, hc[c].z, hc[c].w};
#pragma unroll
                for (int b = 0; b < 8; ++b) {
                    const uint32_t q = b & 1 ? (w[b >> 1] >> 16) & 0x7FFFu : w[b >> 1] & 0x7FFFu;
                    const double2 p = vec[(q << lr) + row];
                    const double m = xor_sign(tb[c * 8 + b], code_sign(w[b >> 1], b & 1));
                    phi.x = fma(m, p.x, phi.x);
                    phi.y = fma(m, p.y, phi.y);
                }
            }
            if (live) {
                e += re_dot(own, phi);
                ham_store(A.out_mode, A.mix, out + (int64_t)col * A.cs, psi + (int64_t)col * A.cs, phi,
                          own);
            }
        }
    }
    if (A.partial) {
        e = wave_sum(e);
        if ((tid & 63) == 0)
            wsum[tid >> 6] = e;
        __syncthreads();
        if (tid == 0) {
            double s = 0.0;
            for (int w = 0; w < T >> 6; ++w)
                s += wsum[w];
            A.partial[bid] = s;
        }
    }
}

template <bool GEN>
__global__ void __launch_bounds__(1024) k_sec_ham_short(HamArgs A)
{
    extern __shared__ __align__(16) char smem[];
    ham_short<GEN>(A, (int)blockIdx.x, smem);
}

typedef const __attribute__((address_space(4))) HamArgs kHamArgs;
template <bool GEN>
__global__ void __launch_bounds__(1024)
k_sec_ham_batch(const HamArgs *__restrict__ args, const SecWork *__restrict__ work)
{
    extern __shared__ __align__(16) char smem[];
    const SecWork w = work[blockIdx.x];
    ham_short<GEN>(((kHamArgs *)args)[w.args], w.bid, smem);
}

// ------------------------------------------------------- whole evaluations --
// Sectors of up to kWholeN x kWholeN amplitudes: the matrix stays in one
// workgroup's LDS for a whole evaluation.  Two workgroups run the circuit and
// H, the same work in both, and then the reverse sweep of one of the vectors
// chi1, chi2 each, so that nothing passes between them: one launch, then the
// reduction.  Up passes rotate along the rows, down passes along the columns
// of the matrix (an odd pitch keeps either side's lanes on different banks);
// index n of a row or column is the zero element.
// Bound by latency and by one CU's VALU (14 qubits, three phases a half layer:
// about 1.5 us a phase, of both sweeps).
struct WholeArgs {
    const SecGate *gates;
    const uint4 *recs;           // per spin and phase: n2 + 1 orbits of six, n13 + 1 pairs of
                                 // orbits of four (the last of each: zero elements)
    const uint16_t *hcode;       // per spin, rank and bond: partner | sign << 15
    const uint32_t *pat[2];      // per rank
    const double *base[2];
    const double *wrow;          // of the spin-down patterns
    const double *tb, *theta;
    double U, mix;
    int n, pitch, n_phases, per, layers, nb, n_red;
    int n2[2], n13[2];
    uint32_t magic;              // i / n = i magic >> 20
    int b0_row, b0_col;
    double *partial;
    int pstride, grad;
};

// LDS of a whole evaluation: the matrix, every layer's angles and (U-only)
// diagonal phases, the tables, and a pass's sums.
struct WholeLds {
    uint32_t ang, dtab, nib, base, pat, recs, hcode, acc, total;
};
__host__ __device__ inline int whole_recs(const int (&n2)[2], const int (&n13)[2], int n_phases,
                                          int spin)   // records before spin's
{
    return spin == 0 ? 0 : n_phases * (n2[0] + 1 + 2 * (n13[0] + 1));
}
__host__ __device__ inline WholeLds whole_lds(int n, int pitch, int n_phases, int layers, int nb,
                                              int n_red, const int (&n2)[2], const int (&n13)[2], int threads,
                                              bool gen)
{
    WholeLds L;
    uint32_t at = (uint32_t)((n + 1) * pitch) * 16u;
    L.ang = at;
    at += (uint32_t)(layers * n_phases * kPositions) * 16u;
    L.dtab = at;
    at += (gen ? 1u << kCisBits : (uint32_t)(layers * kDiagTab)) * 16u;
    L.recs = at;
    at += (uint32_t)(whole_recs(n2, n13, n_phases, 1) +
                     n_phases * (n2[1] + 1 + 2 * (n13[1] + 1))) * 16u;
    L.nib = at;
    at += gen ? (uint32_t)n * 64u * 8u : 0u;
    L.base = at;
    at += gen ? (uint32_t)n * 16u : 0u;
    L.acc = at;   // (the energy's sums per wave: at most 16)
    at += (uint32_t)(n_red * (threads / 4) + 16) * 8u;
    L.pat = at;
    at += (uint32_t)n * 8u;
    L.hcode = at;
    at += ((uint32_t)(2 * n * nb) * 2u + 15u) & ~15u;
    L.total = at;
    return L;
}

// A pass of a whole evaluation, as RowPassCtx sees it.
struct WholePass {
    const SecGate *gates;
    const double *theta;
    double U;
    double *partial;
    int l_pre, l_diag, l_post, per, n_phases, n_red, pstride;
    int row0[2];
};

template <bool GEN, typename AT>
__device__ __forceinline__ void whole(const AT &A, int vsel, char *smem)
{
    const int tid = threadIdx.x, T = blockDim.x, n = A.n, P = A.pitch;
    const int N2[2] = {A.n2[0], A.n2[1]}, N13[2] = {A.n13[0], A.n13[1]};
    const WholeLds L = whole_lds(n, P, A.n_phases, A.layers, A.nb, A.n_red, N2, N13, T, GEN);
    double2 *vec = (double2 *)smem, *ang = (double2 *)(smem + L.ang);
    double2 *dtab = (double2 *)(smem + L.dtab);
    double *nib = (double *)(smem + L.nib), *base = (double *)(smem + L.base);
    double *acc = (double *)(smem + L.acc);
    uint32_t *pat = (uint32_t *)(smem + L.pat);
    uint4 *recs = (uint4 *)(smem + L.recs);
    uint16_t *hcode = (uint16_t *)(smem + L.hcode);
    const gf64 *theta = (const gf64 *)A.theta;
    const int n_gates = A.n_phases * kPositions, ne = n * n;
    auto div_n = [&](int i) __attribute__((always_inline)) {
        return (int)(((uint32_t)i * A.magic) >> 20);
    };
    // tables, and |b0>
    const int n_recs = whole_recs(N2, N13, A.n_phases, 1) +
                       A.n_phases * (N2[1] + 1 + 2 * (N13[1] + 1));
    for (int i = tid; i < n_recs; i += T) {
        const gu128 *p = (const gu128 *)A.recs + i;
        recs[i] = make_uint4(p->x, p->y, p->z, p->w);
    }
    for (int i = tid; i < 2 * n * A.nb; i += T)
        hcode[i] = ((const gu16 *)A.hcode)[i];
    for (int i = tid; i < n; i += T)
        for (int s = 0; s < 2; ++s) {
            pat[s * n + i] = ((const gu32 *)A.pat[s])[i];
            if constexpr (GEN)
                base[s * n + i] = ((const gf64 *)A.base[s])[i];
        }
    if constexpr (GEN) {
        for (int i = tid; i < n * 64; i += T)
            nib[i] = nibble_sum((const gf64 *)A.wrow + (i >> 6) * 16, i & 63);
        build_cis(dtab, tid, T);
    }
    // angles and phases of all layers (the reverse sweep takes their conjugates)
    for (int i = tid; i < A.layers * n_gates; i += T) {
        const int l = i / n_gates;
        const __attribute__((address_space(1))) SecGate &g =
            ((const __attribute__((address_space(1))) SecGate *)A.gates)[i - l * n_gates];
        double s, c;
        sincos(theta[l * A.per + g.slot] * g.t, &s, &c);
        ang[i] = make_double2(c, s);
    }
    if constexpr (!GEN)
        for (int i = tid; i < A.layers * kDiagTab; i += T) {
            const int l = i / kDiagTab;
            double s, c;
            sincos(theta[l * A.per] * (A.U * (double)(i - l * kDiagTab)), &s, &c);
            dtab[i] = make_double2(c, -s);
        }
    for (int i = tid; i < (n + 1) * P; i += T)
        vec[i] = make_double2(i == A.b0_row * P + A.b0_col ? 1.0 : 0.0, 0.0);
    __syncthreads();

    const int TH = T >> 1;
    const bool duo_half = __builtin_amdgcn_readfirstlane(tid) < TH;
    const int t0 = duo_half ? tid : tid - TH;

    // pass i of the forward sweep, or its reverse
    auto pass = [&](auto mode, int i, int row0) __attribute__((always_inline)) {
        constexpr int MODE = decltype(mode)::value;
        constexpr bool REV = MODE == S_REV;
        const int col = i & 1;
        WholePass V;
        V.gates = A.gates;
        V.theta = A.theta;
        V.U = A.U;
        V.partial = A.partial;
        V.l_pre = i - 1;
        V.l_diag = V.l_post = i < A.layers ? i : -1;
        V.per = A.per;
        V.n_phases = A.n_phases;
        V.n_red = REV ? (V.l_pre >= 0 ? A.per - 1 : 0) + (V.l_diag >= 0 ? A.per : 0) : 0;
        V.pstride = A.pstride;
        V.row0[0] = row0;
        V.row0[1] = row0 + V.n_red;
        RowLds rl;
        rl.ang = L.ang;
        rl.dtab = L.dtab;
        rl.acc = L.acc;
        RowPassCtx<MODE, GEN, WholePass> C(V, smem, rl);
        for (int q = tid; q < V.n_red * (T / 4); q += T)
            acc[q] = 0.0;
        __syncthreads();
        const int rs = col == 0 ? P * 16 : 16;   // bytes between rows of the other spin
        const int m2 = N2[col], m13 = N13[col], per_phase = m2 + 1 + 2 * (m13 + 1);
        const uint4 *mine = recs + (col == 0 ? 0 : whole_recs(N2, N13, A.n_phases, 1));
        const int items = (duo_half ? m2 : m13) * n;
        auto at = [&](const uint4 &q, int j, uint32_t ofs)
                      __attribute__((always_inline)) -> double2 & {
            const uint32_t w = j < 2 ? q.x : (j < 4 ? q.y : q.z);
            return *(double2 *)(smem + ((j & 1 ? w >> 16 : w & 0xFFFFu) << 4) + ofs);
        };
        auto phase = [&](int run, int ph) __attribute__((always_inline)) {
            typename RowPassCtx<MODE, GEN, WholePass>::PhaseArgs pa =
                C.phase_args(run, ph, run ? V.l_post : V.l_pre);
            if constexpr (REV)
#pragma unroll
                for (int q = 0; q < kPositions; ++q)
                    pa.c[q].y = -pa.c[q].y;
            const uint4 *list = mine + ph * per_phase + (duo_half ? 0 : m2 + 1);
            for (int k = t0 & ~63; k < items; k += TH) {   // whole waves
                const int it = k + (tid & 63);
                const bool act = it < items;
                const int orb = act ? div_n(it) : (duo_half ? m2 : m13);
                const uint32_t ofs = act ? (uint32_t)((it - orb * n) * rs) : 0u;
                if (duo_half) {
                    const uint4 q = list[orb];
                    double2 x[6];
#pragma unroll
                    for (int j = 0; j < 6; ++j)
                        x[j] = at(q, j, ofs);
                    C.gates2(x, pa, q.w);
                    if (act) {
#pragma unroll
                        for (int j = 0; j < 6; ++j)
                            at(q, j, ofs) = x[j];
                    }
                } else {
                    const uint4 q1 = list[orb], q3 = list[m13 + 1 + orb];
                    double2 x[8];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        x[j] = at(q1, j, ofs);
                        x[4 + j] = at(q3, j, ofs);
                    }
                    C.gates13(x, pa, q1.z, q3.z);
                    if (act) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            at(q1, j, ofs) = x[j];
                            at(q3, j, ofs) = x[4 + j];
                        }
                    }
                }
            }
            __syncthreads();
        };
        auto diag = [&]() __attribute__((always_inline)) {
            const double th = theta[V.l_diag * A.per];
            double racc = 0.0;
            for (int e = tid; e < ne; e += T) {
                const int rd = div_n(e), ru = e - rd * n;
                double2 &a = vec[rd * P + ru];
                if constexpr (GEN) {
                    double err;
                    const double d = diag_gen(base[n + rd], base[ru], nib + rd * 64, pat[ru], err);
                    diag_el<REV, true>(a, d, err, a, th, dtab, racc);
                } else {
                    const int k = __popc(pat[n + rd] & pat[ru]);
                    double2 f = dtab[V.l_diag * kDiagTab + k];
                    if constexpr (REV)
                        f.y = -f.y;
                    diag_el<REV, false>(a, A.U * (double)k, 0.0, f, th, nullptr, racc);
                }
            }
            if constexpr (REV)
                C.flush(C.dslot, racc);
            __syncthreads();
        };
        if constexpr (!REV) {
            for (int ph = 0; V.l_pre >= 0 && ph < A.n_phases; ++ph)
                phase(0, ph);
            if (V.l_diag >= 0)
                diag();
            for (int ph = 0; V.l_post >= 0 && ph < A.n_phases; ++ph)
                phase(1, ph);
        } else {
            for (int ph = A.n_phases - 1; V.l_post >= 0 && ph >= 0; --ph)
                phase(1, ph);
            if (V.l_diag >= 0)
                diag();
            for (int ph = A.n_phases - 1; V.l_pre >= 0 && ph >= 0; --ph)
                phase(0, ph);
            C.finish(0, vsel, vsel == 1);
            __syncthreads();
        }
    };
    const int n_pass = A.layers > 0 ? A.layers + 1 : 0;
    for (int i = 0; i < n_pass; ++i)
        pass(std::integral_constant<int, S_FWD>(), i, 0);

    // H psi, kept in registers; the energy; chi1 or chi2 in psi's place
    double2 phi[kWholeEl];
    double e = 0.0;
    const kf64 *tb = (const kf64 *)A.tb;
#pragma unroll
    for (int u = 0; u < kWholeEl; ++u) {
        const int el = tid + u * T;
        phi[u] = make_double2(0.0, 0.0);
        if (el < ne) {
            const int rd = div_n(el), ru = el - rd * n;
            const double2 own = vec[rd * P + ru];
            double d;
            if constexpr (GEN)
                d = diag_gen(base[n + rd], base[ru], nib + rd * 64, pat[ru]);
            else
                d = A.U * (double)__popc(pat[n + rd] & pat[ru]);
            double2 f = make_double2(d * own.x, d * own.y);
            const uint16_t *hu = hcode + ru * A.nb, *hd = hcode + (n + rd) * A.nb;
            for (int b = 0; b < A.nb; ++b) {
                const uint32_t cu = hu[b], cd = hd[b];
                const double2 pu = vec[rd * P + (int)(cu & 0x7FFFu)];
                const double2 pd = vec[(int)(cd & 0x7FFFu) * P + ru];
                const double mu = xor_sign(tb[b], code_sign(cu, 0));
                const double md = xor_sign(tb[b], code_sign(cd, 0));
                f.x = fma(mu, pu.x, f.x);
                f.y = fma(mu, pu.y, f.y);
                f.x = fma(md, pd.x, f.x);
                f.y = fma(md, pd.y, f.y);
            }
            e += re_dot(own, f);
            phi[u] = f;
        }
    }
    e = wave_sum(e);
    if ((tid & 63) == 0)
        acc[tid >> 6] = e;
    __syncthreads();
    if (vsel == 0 && tid == 0) {
        double sum = 0.0;
        for (int w = 0; w < T >> 6; ++w)
            sum += acc[w];
        A.partial[0] = sum;
        A.partial[A.pstride] = 0.0;
    }
    if (!A.grad || n_pass == 0)
        return;
    const double im = 1.0 / A.mix, sg = vsel == 1 ? 1.0 : -1.0;   // im: exact
#pragma unroll
    for (int u = 0; u < kWholeEl; ++u) {
        const int el = tid + u * T;
        if (el < ne) {
            const int rd = div_n(el);
            double2 &a = vec[rd * P + (el - rd * n)];
            const double2 own = make_double2(a.x * A.mix, a.y * A.mix);
            a = make_double2(phi[u].x * im - sg * own.y, phi[u].y * im + sg * own.x);
        }
    }
    int row0 = 2 + 2 * ((2 * A.per - 1) * A.layers);
    for (int i = n_pass - 1; i >= 0; --i) {
        const int red = (i > 0 ? A.per - 1 : 0) + (i < A.layers ? A.per : 0);
        row0 -= 2 * red;
        __syncthreads();
        pass(std::integral_constant<int, S_REV>(), i, row0);
    }
}

template <bool GEN>
__global__ void __launch_bounds__(1024) k_sec_whole(WholeArgs A)
{
    extern __shared__ __align__(16) char smem[];
    whole<GEN>(A, (int)blockIdx.x, smem);
}

typedef const __attribute__((address_space(4))) WholeArgs kWholeArgs;
template <bool GEN>
__global__ void __launch_bounds__(1024)
k_sec_whole_batch(const WholeArgs *__restrict__ args, const SecWork *__restrict__ work)
{
    extern __shared__ __align__(16) char smem[];
    const SecWork w = work[blockIdx.x];
    whole<GEN>(((kWholeArgs *)args)[w.args], w.vsel, smem);
}

// Long rows: H is real, so the real and the imaginary parts of a row take
// turns in LDS.  Thread t sums for the slots t + j kLongT: lanes of
// neighbouring slots are in different bank classes, and so are their
// partners across one bond.
// Bound by VALU (half of its time) and by the row's phases not overlapping:
// load, two rounds of sums, store.  At 12870 x 12870 and 32 bonds a pass took
// 4.3 ms; the imaginary parts kept from the one load of the row 3.8; signs apart
// from the partners' codes, bonds without signs first and LDS addressed without
// a base 3.5.
template <bool GEN>
__global__ void __launch_bounds__(kLongT) k_sec_ham_long(HamArgs A)
{
    extern __shared__ __align__(16) char smem[];
    double *buf = (double *)smem;
    double *nib = buf + A.nslots + kLongDummy;
    double *wsum = nib + 64;
    const int tid = threadIdx.x;
    const uint32_t n = (uint32_t)A.n;
    const gu16 *patslot = (const gu16 *)A.patslot;
    const gf64 *baseslot = (const gf64 *)A.baseslot;
    const kf64 *tb = (const kf64 *)A.tb;
    const ku32 *rpat = (const ku32 *)A.rpat;
    const kf64 *rbase = (const kf64 *)A.rbase;
    for (int i = tid; i < A.nslots + kLongDummy; i += kLongT)   // the holes and the zero slots
        buf[i] = 0.0;
    double e = 0.0;
    for (int ig = blockIdx.x; ig < (A.n_rows + 7) / 8 * 8; ig += A.grid) {
        const int r = group_of(ig, A.n_rows);
        if (r < 0)
            continue;
        gc128 *psi = (gc128 *)A.psi + (size_t)r * n;
        const uint32_t rp = rpat[r];
        const double rb = GEN ? rbase[r] : 0.0;
        int t = tid;   // the tables' values are not kept across rows
        asm volatile("" : "+v"(t));
        double re_out[kLongElems];   // first the imaginary parts, then the real results
        LongCodes cc = col_codes(A.colslot, t);
        __syncthreads();
        if (GEN && A.diag && tid < 64)
            nib[tid] = nibble_sum((const gf64 *)A.wrow + (size_t)r * 16, tid);
#pragma unroll
        for (int j = 0; j < kLongElems; ++j) {
            const uint32_t i = (uint32_t)(t + j * kLongT);
            const gc128 *p = psi + min(i, n - 1);
            const double2 x = make_double2(p->x, p->y);
            *(double *)(smem + cc.at(j)) = i < n ? x.x : 0.0;
            re_out[j] = i < n ? x.y : 0.0;
        }
#pragma unroll 1
        for (int half = 0; half < 2; ++half) {
            asm volatile("" : "+v"(t));
            __syncthreads();
            double phi[kLongElems];
#pragma unroll
            for (int j = 0; j < kLongElems; ++j) {
                phi[j] = 0.0;
                const int sl = t + j * kLongT;
                if (A.diag && sl < A.nslots) {
                    const uint32_t cp = patslot[sl];
                    const double d = GEN ? diag_gen(rb, baseslot[sl], nib, cp)
                                         : A.U * (double)__popc(rp & cp);
                    phi[j] = d * buf[sl];
                }
            }
            cc.renew();
            LongCodes nx = col_codes(A.hcode, t);   // the same chunk layout
            // the bonds without a Jordan-Wigner string come first; of the
            // others, bit 31 - j of the last dword is element j's sign
            auto bonds = [&](auto sgn, int b0, int b1) __attribute__((always_inline)) {
#pragma unroll 1
                for (int b = b0; b < b1; ++b) {
                    const LongCodes w = nx;
                    nx = col_codes(A.hcode + (size_t)min(b + 1, A.nb - 1) * 16 * kLongT, t);
                    const double m = tb[b];
#pragma unroll
                    for (int j = 0; j < kLongElems; ++j) {
                        const uint32_t q = w.w[j >> 1];
                        const uint32_t o = j & 1 ? (q >> 13) & 0x7FFF8u : (q << 3) & 0x7FFF8u;
                        double p = *lds_at(o);
                        if constexpr (decltype(sgn)::value)
                            p = xor_sign(p, (w.w[7] << j) & 0x80000000u);
                        phi[j] = fma(m, p, phi[j]);
                    }
                }
            };
            bonds(std::false_type(), 0, A.n_flat);
            bonds(std::true_type(), A.n_flat, A.nb);
#pragma unroll
            for (int j = 0; j < kLongElems; ++j) {
                const int sl = t + j * kLongT;
                if (sl < A.nslots)
                    e = fma(buf[sl], phi[j], e);
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < kLongElems; ++j) {
                const int sl = t + j * kLongT;
                if (sl < A.nslots)
                    buf[sl] = phi[j];
            }
            __syncthreads();
            if (half == 0) {
#pragma unroll
                for (int j = 0; j < kLongElems; ++j) {   // a thread's own places
                    double *o = (double *)(smem + cc.at(j));
                    const double y = re_out[j];
                    re_out[j] = *o;
                    *o = y;
                }
            } else {
#pragma unroll
                for (int j = 0; j < kLongElems; ++j) {
                    const uint32_t i = (uint32_t)(t + j * kLongT);
                    if (i < n) {
                        const double2 f = make_double2(re_out[j],
                                                       *(const double *)(smem + cc.at(j)));
                        gc128 *o = (gc128 *)A.out +
                                   (A.turn ? (size_t)i * A.n_rows + r : (size_t)r * n + i);
                        double2 own = make_double2(0.0, 0.0);
                        if (A.out_mode == HO_MIX)
                            own = make_double2(psi[i].x, psi[i].y);
                        ham_store(A.out_mode, A.mix, o, psi + i, f, own);
                    }
                }
            }
        }
    }
    if (A.partial) {
        e = wave_sum(e);
        if ((tid & 63) == 0)
            wsum[tid >> 6] = e;
        __syncthreads();
        if (tid == 0) {
            double s = 0.0;
            for (int w = 0; w < kLongT / 64; ++w)
                s += wsum[w];
            A.partial[blockIdx.x] = s;
        }
    }
}

// out[c nr + r] = in[r nc + c], through 64 x 64 LDS tiles
// (1 KB row segments; 32 x 32 tiles reached 3.7 TB/s at 12870 x 12870, these
// 4.6 TB/s).
constexpr int kTrTile = 64, kTrThreads = 512;
__global__ void __launch_bounds__(kTrThreads)
k_sec_transpose(const double2 *__restrict__ in, double2 *__restrict__ out, int nr, int nc)
{
    constexpr int RW = kTrThreads / kTrTile;   // tile rows per sweep of the threads
    __shared__ double2 tile[kTrTile][kTrTile + 1];
    const int c0 = blockIdx.x * kTrTile, r0 = blockIdx.y * kTrTile;
    const int tx = threadIdx.x % kTrTile, ty = threadIdx.x / kTrTile;
    for (int k = ty; k < kTrTile; k += RW) {
        const int r = r0 + k, c = c0 + tx;
        if (r < nr && c < nc)
            tile[k][tx] = in[(size_t)r * nc + c];
    }
    __syncthreads();
    for (int k = ty; k < kTrTile; k += RW) {
        const int c = c0 + k, r = r0 + tx;
        if (r < nr && c < nc) {
            out[(size_t)c * nr + r] = tile[tx][k];
        }
    }
}

// psi <- the basis state at position `at` (zeros elsewhere).
__global__ void __launch_bounds__(256) k_sec_basis(double2 *__restrict__ psi, size_t n, size_t at)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x)
        psi[i] = make_double2(i == at ? 1.0 : 0.0, 0.0);
}

// out[o] = scale[o] * sum over partial rows rows[ptr[o] .. ptr[o+1]) of the
// nblk[row] entries each (the workgroups of the pass that wrote it), in a
// fixed order; o = 0 goes to E, o >= 1 to grad[o-1].
__global__ void __launch_bounds__(256)
k_sec_reduce(const double *__restrict__ partial, int pstride, const int32_t *__restrict__ nblk,
             const int32_t *__restrict__ ptr, const int32_t *__restrict__ rows,
             const double *__restrict__ scale, double *__restrict__ E, double *__restrict__ grad)
{
    __shared__ double sm[256];
    const int o = blockIdx.x, tid = threadIdx.x;
    double s = 0.0;
    for (int k = ptr[o]; k < ptr[o + 1]; ++k) {
        const double *p = partial + (size_t)rows[k] * pstride;
        for (int b = tid; b < nblk[rows[k]]; b += 256)
            s += p[b];
    }
    sm[tid] = s;
    for (int st = 128; st > 0; st >>= 1) {
        __syncthreads();
        if (tid < st)
            sm[tid] += sm[tid + st];
    }
    if (tid == 0) {
        const double v = scale[o] * sm[0];
        if (o == 0)
            E[0] = v;
        else
            grad[o - 1] = v;
    }
}

// ------------------------------------------------------------------ host --

struct RowPass {
    int col = 0;                          // the spin whose patterns index the rows
    int l_pre = -1, l_diag = -1, l_post = -1;
    std::vector<int> red_param;           // parameter of each reduction slot
};

// One spin's tables on the device (one allocation).
struct SpinTables {
    int n = 0, nslots = 0, lr = 0, threads = 64;
    bool is_long = false;
    SecPhase *phases = nullptr;
    Rec *recs = nullptr;
    uint4 *lcode = nullptr, *lpat = nullptr;
    uint32_t *pat = nullptr;
    double *lbase = nullptr, *base = nullptr, *baseslot = nullptr, *wrow = nullptr;
    uint16_t *colslot = nullptr, *patslot = nullptr, *hcode = nullptr;
};

// Sector tables of one model on one device.
struct Tables {
    int n[2] = {0, 0}, ne[2] = {0, 0};   // patterns and electrons of each spin
    size_t b0_pos = 0;            // position of |b0> in layout A
    int b0_rank[2] = {0, 0};      // ranks of |b0>'s patterns
    bool general = false;         // eps or V terms in the diagonal
    bool is_long = false;
    double U = 0.0, mix = 1.0;
    int n_phases = 0, nb = 0, per = 1;
    int n_flat = 0;               // long rows' H: bonds without a sign
    SpinTables sp[2];
    SecGate *d_gates = nullptr;
    double *d_tb = nullptr;
    // whole evaluations (threads 0: the sector has none)
    struct {
        int threads = 0, n2[2] = {0, 0}, n13[2] = {0, 0};
        uint4 *recs = nullptr;
        uint16_t *hcode = nullptr;
    } whole;
    char *blob = nullptr;
    ~Tables() { (void)hipFree(blob); }
};

struct Program {
    std::vector<RowPass> fwd;
    int final_col = 0;
    // reduction: partial rows 0, 1 = the two energy parts, then each reverse
    // pass's slots (forward order of passes)
    std::vector<int> red_row0;    // per forward pass: its chi2 rows, then its chi1 rows
    int n_rows = 0, max_red = 0;
    bool whole = false;           // runs as a whole evaluation
    int32_t *d_ptr = nullptr, *d_rows = nullptr, *d_nblk = nullptr;
    double *d_scale = nullptr;
    char *blob = nullptr;
    int n_out = 0;
    ~Program() { (void)hipFree(blob); }
};

// A handle's tables on a device.  They are planned and uploaded under mu, their
// own lock: other handles' calls do not wait for it (26 ms at 4x4).
struct Entry {
    std::mutex mu;
    std::unique_ptr<Tables> tab;
    std::map<int, std::unique_ptr<Program>> progs;   // by layer count
};

std::mutex g_mu;   // guards the map only
std::map<std::pair<uint64_t, int>, std::shared_ptr<Entry>> g_cache;   // (handle uid, device)

hubbard_status fail(hubbard_status s, const std::string &m) { return set_error(s, m); }

// Host arrays collected into one device allocation.
struct Blob {
    std::vector<char> host;
    std::vector<std::pair<void **, size_t>> at;
    template <typename T> void add(T **dst, const void *src, size_t bytes)
    {
        host.resize((host.size() + 255) & ~(size_t)255);
        at.push_back({(void **)dst, host.size()});
        host.resize(host.size() + std::max<size_t>(bytes, 16));
        if (bytes)
            std::memcpy(host.data() + at.back().second, src, bytes);
    }
    template <typename T, typename S> void add(T **dst, const std::vector<S> &v)
    {
        add(dst, v.data(), v.size() * sizeof(S));
    }
    hipError_t upload(char **blob)
    {
        hipError_t e = hipMalloc((void **)blob, std::max<size_t>(host.size(), 256));
        if (e == hipSuccess)
            e = hipMemcpy(*blob, host.data(), host.size(), hipMemcpyHostToDevice);
        if (e == hipSuccess)
            for (auto &p : at)
                *p.first = *blob + p.second;
        else
            (void)hipGetLastError();   // reported by the caller, not by the next launch
        return e;
    }
};

// The tables of whole evaluations; false (threads 0) where a sector does not
// fit.  Elements by rank, of spin-down orbits times the pitch; rank n, and the
// orbits that fill a phase's lists up to the longest one, are zero elements.
// A launch per pass over the chip / one workgroup per vector: 8 qubits 38 / 17
// us, 14 qubits 156 / 97 us (ten layers), 256 instances of 8 to 20 qubits 1.63 /
// 1.48 ms.  With 70 patterns (16 qubits) one CU is too slow: 148 / 182 us.
bool plan_whole(const Model &m, const SectorPlan &P, Tables &T, std::vector<uint4> &recs,
                std::vector<uint16_t> &code)
{
    const int n = P.spin[0].n, nph = (int)P.sites.size(), pitch = (n + 1) | 1;
    if (n > kWholeN || P.spin[1].n != n || 2 * m.params_per_layer() - 1 > kMaxRed)
        return false;
    auto &W = T.whole;
    auto rec = [&](int s, int ph, int list, int k) -> const Rec & {
        const SpinPlan &S = P.spin[s];
        return S.recs[(size_t)(3 * ph + list) * (size_t)((S.threads / 2) >> S.lr) + (size_t)k];
    };
    int items = 0;
    for (int s = 0; s < 2; ++s) {
        const int lanes = (P.spin[s].threads / 2) >> P.spin[s].lr;
        for (int ph = 0; ph < nph; ++ph)
            for (int list = 0; list < 3; ++list)
                for (int k = 0; k < lanes; ++k)
                    if (rec(s, ph, list, k).w[list == 0 ? 3 : 2] & 1u) {
                        int &c = list == 0 ? W.n2[s] : W.n13[s];
                        c = std::max(c, k + 1);
                    }
        items = std::max(items, std::max(W.n2[s], W.n13[s]) * n);
    }
    const int th = std::min(512, std::max(64, (items + 63) / 64 * 64));
    const int threads = std::max(2 * th, std::min(1024, (n * n + 1023) / 1024 * 128));
    const int n_red = 2 * m.params_per_layer() - 1;
    if (n * n > kWholeEl * threads ||
        whole_lds(n, pitch, nph, 0, m.nb, n_red, W.n2, W.n13, threads, m.general).total > 160u * 1024u)
        return false;
    for (int s = 0; s < 2; ++s) {
        const SpinPlan &S = P.spin[s];
        const int lanes = (S.threads / 2) >> S.lr, scale = s == 0 ? 1 : pitch;
        std::vector<int> rank(S.nslots + 1, n);
        for (int r = 0; r < n; ++r)
            rank[S.colslot[r]] = r;
        for (int ph = 0; ph < nph; ++ph)
            for (int list = 0; list < 3; ++list) {
                const int len = list == 0 ? W.n2[s] : W.n13[s];
                for (int k = 0; k <= len; ++k) {
                    Rec q = {{0, 0, 0, 0}};
                    const bool have = k < len && k < lanes && (rec(s, ph, list, k).w[list == 0 ? 3 : 2] & 1u);
                    if (have)
                        q = rec(s, ph, list, k);
                    for (int w = 0; w < (list == 0 ? 3 : 2); ++w) {
                        const uint32_t lo = (uint32_t)((have ? rank[q.w[w] & 0xFFFFu] : n) * scale);
                        const uint32_t hi = (uint32_t)((have ? rank[q.w[w] >> 16] : n) * scale);
                        q.w[w] = lo | hi << 16;
                    }
                    recs.push_back(make_uint4(q.w[0], q.w[1], q.w[2], q.w[3]));
                }
            }
        const int hb = ham_bonds(m.nb);
        for (int r = 0; r < n; ++r)
            for (int b = 0; b < m.nb; ++b) {
                const uint16_t c = S.hcode[(size_t)r * hb + b];
                code.push_back((uint16_t)(rank[c & 0x7FFF] | (c & 0x8000)));
            }
    }
    W.threads = threads;
    return true;
}

hubbard_status build_tables(const Model &m, Tables &T)
{
    SectorPlan P;
    const std::string err = plan_sector(m, P);
    if (!err.empty())
        return fail(HUBBARD_ERR_ARG, err);
    const uint32_t smask = (1u << m.ns) - 1u;
    T.ne[0] = __builtin_popcount((uint32_t)m.neel & smask);
    T.ne[1] = __builtin_popcount((uint32_t)(m.neel >> m.ns) & smask);
    T.b0_rank[0] = P.spin[0].rank_of[(uint32_t)m.neel & smask];
    T.b0_rank[1] = P.spin[1].rank_of[(uint32_t)(m.neel >> m.ns) & smask];
    T.general = m.general;
    T.U = m.U;
    T.n_phases = (int)P.sites.size();
    T.nb = m.nb;
    T.per = m.params_per_layer();
    T.mix = P.mix;
    Blob B;
    B.add(&T.d_gates, P.gates);
    std::vector<double> tb((size_t)std::max(8, ham_bonds(m.nb)), 0.0);
    for (int k = 0; k < m.nb; ++k)
        tb[k] = -m.t[P.ham_order[k]];
    B.add(&T.d_tb, tb);
    T.n_flat = P.n_flat;
    const bool same = T.ne[0] == T.ne[1];   // one set of tables
    for (int s = 0; s < 2; ++s) {
        const SpinPlan &S = P.spin[s];
        SpinTables &D = T.sp[s];
        T.n[s] = D.n = S.n;
        D.nslots = S.nslots;
        D.lr = S.lr;
        D.threads = S.threads;
        D.is_long = S.is_long;
        T.is_long = T.is_long || S.is_long;
        if (s == 1 && same)
            break;
        B.add(&D.phases, S.phases);
        B.add(&D.recs, S.recs);
        B.add(&D.lcode, S.lcode);
        B.add(&D.lpat, S.lpat);
        B.add(&D.pat, S.pat);
        B.add(&D.lbase, S.lbase);
        B.add(&D.base, S.base);
        B.add(&D.baseslot, S.baseslot);
        B.add(&D.wrow, S.wrow);
        B.add(&D.colslot, S.colslot);
        B.add(&D.patslot, S.patslot);
        B.add(&D.hcode, S.hcode);
    }
    std::vector<uint4> wrecs;
    std::vector<uint16_t> wcode;
    if (plan_whole(m, P, T, wrecs, wcode)) {
        B.add(&T.whole.recs, wrecs);
        B.add(&T.whole.hcode, wcode);
    }
    // one electron per site: C(Ns, N_up) = C(Ns, N_dn)
    if (T.n[0] != T.n[1])
        return fail(HUBBARD_ERR_STATE, "sector matrix is not square");
    T.b0_pos = (size_t)T.b0_rank[1] * T.n[0] + T.b0_rank[0];
    const hipError_t e = B.upload(&T.blob);
    if (e != hipSuccess)
        return fail(HUBBARD_ERR_DEVICE, std::string("uploading sector tables: ") +
                                            hipGetErrorString(e));
    if (same)
        T.sp[1] = T.sp[0];
    return HUBBARD_OK;
}

// Workgroups of a pass over spin col's rows, per vector: at most kGrid, and
// no more than there are row groups.
int rows_grid(const Tables &T, int col)
{
    if (T.is_long)   // one workgroup per CU
        return 256;
    const int ng = (T.n[1 - col] + (1 << T.sp[col].lr) - 1) >> T.sp[col].lr;
    return std::min((ng + 7) / 8 * 8, kGrid);
}

uint32_t whole_lds(const Tables &T, int layers)
{
    return whole_lds(T.n[0], (T.n[0] + 1) | 1, T.n_phases, layers, T.nb, 2 * T.per - 1, T.whole.n2,
                     T.whole.n13, T.whole.threads, T.general)
        .total;
}

// Whether evaluations of `layers` layers run whole: every layer's angles fit, too.
bool runs_whole(const Tables &T, int layers)
{
    return T.whole.threads && layers <= kWholeLayers && whole_lds(T, layers) <= 160u * 1024u;
}


uint32_t rows_lds(const Tables &T, int col, int n_red)
{
    const SpinTables &S = T.sp[col];
    return row_lds(S.is_long ? long_vec_bytes(S.nslots) : short_vec_bytes(S.nslots, S.lr),
                   1 << S.lr, T.n_phases, n_red, S.threads, T.general)
        .total;
}

hubbard_status build_program(const Model &m, const Tables &T, int layers, Program &P)
{
    const int per = m.params_per_layer();
    P.fwd.clear();
    if (layers > 0) {
        RowPass cur;
        for (int l = 0; l < layers; ++l) {
            cur.l_diag = cur.l_post = l;
            P.fwd.push_back(cur);
            const int other = 1 - cur.col;
            cur = RowPass();
            cur.col = other;
            cur.l_pre = l;
        }
        P.fwd.push_back(cur);
    }
    for (RowPass &p : P.fwd) {
        // in the order of the kernel's reduction slots
        for (int s = 1; p.l_pre >= 0 && s < per; ++s)
            p.red_param.push_back(p.l_pre * per + s);
        if (p.l_diag >= 0)
            p.red_param.push_back(p.l_diag * per);
        for (int s = 1; p.l_post >= 0 && s < per; ++s)
            p.red_param.push_back(p.l_post * per + s);
        if ((int)p.red_param.size() > kMaxRed)
            return fail(HUBBARD_ERR_ARG, "sector row pass with more than 16 parameters");
        P.max_red = std::max(P.max_red, (int)p.red_param.size());
    }
    P.final_col = P.fwd.empty() ? 0 : P.fwd.back().col;
    // reduction rows, and the workgroups of the pass that writes each
    P.n_rows = 2;
    P.whole = runs_whole(T, layers);
    // (a whole evaluation: one workgroup)
    auto red_grid = [&](int col) { return P.whole ? 1 : rows_grid(T, col); };
    std::vector<int32_t> nblk{red_grid(P.final_col), red_grid(1 - P.final_col)};
    std::vector<std::vector<int>> rows_of(1 + layers * per);
    rows_of[0] = {0, 1};
    for (const RowPass &p : P.fwd) {
        P.red_row0.push_back(P.n_rows);
        for (int half = 0; half < 2; ++half) {   // chi2, then chi1 (stored negated)
            for (size_t s = 0; s < p.red_param.size(); ++s) {
                rows_of[1 + p.red_param[s]].push_back(P.n_rows + (int)s);
                nblk.push_back(red_grid(p.col));
            }
            P.n_rows += (int)p.red_param.size();
        }
    }
    std::vector<int32_t> ptr{0}, rows;
    std::vector<double> scale;
    for (size_t o = 0; o < rows_of.size(); ++o) {
        rows.insert(rows.end(), rows_of[o].begin(), rows_of[o].end());
        ptr.push_back((int32_t)rows.size());
        // dE/dth_k = 2 Im <lambda_k|G_k|psi_k> = (<chi2|G_k|chi2> - <chi1|G_k|chi1>) / 2
        scale.push_back(o == 0 ? 1.0 : 0.5);
    }
    P.n_out = (int)rows_of.size();
    Blob B;
    B.add(&P.d_ptr, ptr);
    B.add(&P.d_rows, rows);
    B.add(&P.d_scale, scale);
    B.add(&P.d_nblk, nblk);
    const hipError_t e = B.upload(&P.blob);
    if (e != hipSuccess)
        return fail(HUBBARD_ERR_DEVICE, std::string("uploading the sector program: ") +
                                            hipGetErrorString(e));
    return HUBBARD_OK;
}

// Tables and (layers >= 0) the program of a handle on the current device.
hubbard_status get(hubbard_t h, int layers, Tables **T, Program **P)
try {
    const Model *m = handle_model(h);
    if (!m)
        return fail(HUBBARD_ERR_ARG, "null handle");
    if (m->ansatz != 0)
        return fail(HUBBARD_ERR_STATE, "the sector form needs the HVA circuit (the NP "
                                       "ansatz's on-site gates change N_up and N_dn)");
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess)
        return fail(HUBBARD_ERR_DEVICE, "hipGetDevice failed");
    std::shared_ptr<Entry> entry;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        std::shared_ptr<Entry> &e = g_cache[std::make_pair(handle_uid(h), dev)];
        if (!e)
            e = std::make_shared<Entry>();
        entry = e;
    }
    Entry &en = *entry;
    std::lock_guard<std::mutex> lk(en.mu);
    if (!en.tab) {
        std::unique_ptr<Tables> t(new Tables());
        hubbard_status st = build_tables(*m, *t);
        if (st != HUBBARD_OK)
            return st;
        en.tab = std::move(t);
    }
    *T = en.tab.get();
    if (P) {
        auto it = en.progs.find(layers);
        if (it == en.progs.end()) {
            std::unique_ptr<Program> p(new Program());
            hubbard_status st = build_program(*m, *en.tab, layers, *p);
            if (st != HUBBARD_OK)
                return st;
            it = en.progs.emplace(layers, std::move(p)).first;
        }
        *P = it->second.get();
    }
    return HUBBARD_OK;
} catch (const std::exception &) {
    return fail(HUBBARD_ERR_NOMEM, "out of memory");
}

size_t vec_elems(const Tables &T) { return (size_t)T.n[0] * (size_t)T.n[1]; }
size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Element strides of spin col's rows: short rows read the one layout (rows
// r_dn, columns r_up) along either side.
void strides(const Tables &T, int col, int64_t *rs, int64_t *cs)
{
    *rs = col == 0 || T.is_long ? T.n[col] : 1;
    *cs = col == 0 || T.is_long ? 1 : T.n[0];
}

// Arguments of pass p (reverse: of its two vectors) on v0 (and v1); its
// partial rows start at row0, pstride entries each.
RowsArgs rows_args(const Tables &T, const RowPass &p, bool rev, const double *theta, double2 *v0,
                   double2 *v1, double *partial, int row0, int pstride, int flags, double2 *t0,
                   double2 *t1)
{
    const SpinTables &S = T.sp[p.col], &O = T.sp[1 - p.col];
    RowsArgs A;
    std::memset(&A, 0, sizeof(A));
    A.phases = S.phases;
    A.gates = T.d_gates;
    A.recs = S.recs;
    A.lcode = S.lcode;
    A.lpat = S.lpat;
    A.lbase = S.lbase;
    A.colslot = S.colslot;
    A.patslot = S.patslot;
    A.baseslot = S.baseslot;
    A.rpat = O.pat;
    A.rbase = O.base;
    A.wrow = O.wrow;
    A.theta = theta;
    A.U = T.U;
    A.n = S.n;
    A.n_rows = O.n;
    A.nslots = S.nslots;
    A.lr = S.lr;
    A.n_phases = T.n_phases;
    A.per = T.per;
    A.l_pre = p.l_pre;
    A.l_diag = p.l_diag;
    A.l_post = p.l_post;
    strides(T, p.col, &A.rs, &A.cs);
    A.v[0] = v0;
    A.v[1] = v1;
    A.t[0] = t0;
    A.t[1] = t1;
    A.partial = partial;
    A.n_red = rev ? (int)p.red_param.size() : 0;
    A.row0[0] = row0;
    A.row0[1] = row0 + A.n_red;
    A.pstride = pstride;
    A.flags = flags;
    A.b0_row = T.b0_rank[1 - p.col];
    A.b0_col = T.b0_rank[p.col];
    A.grid = rows_grid(T, p.col);
    return A;
}

template <int MODE>
void launch_rows(const Tables &T, const RowPass &p, const double *theta, double2 *v0, double2 *v1,
                 double *partial, int row0, int flags, hipStream_t s, double2 *t0 = nullptr,
                 double2 *t1 = nullptr)
{
    const SpinTables &S = T.sp[p.col];
    const RowsArgs A = rows_args(T, p, MODE == S_REV, theta, v0, v1, partial, row0, kGrid, flags,
                                 t0, t1);
    const dim3 grid(A.grid, MODE == S_REV ? 2 : 1);
    const uint32_t lds = rows_lds(T, p.col, A.n_red);
    if (S.is_long) {
        if (T.general)
            hipLaunchKernelGGL((k_sec_rows_long<MODE, true>), grid, dim3(kLongT), lds, s, A);
        else
            hipLaunchKernelGGL((k_sec_rows_long<MODE, false>), grid, dim3(kLongT), lds, s, A);
    } else {
        if (T.general)
            hipLaunchKernelGGL((k_sec_rows_short<MODE, true>), grid, dim3(S.threads), lds, s, A);
        else
            hipLaunchKernelGGL((k_sec_rows_short<MODE, false>), grid, dim3(S.threads), lds, s, A);
    }
}

// Spin col's part of H (with_d: and the diagonal) on psi.
HamArgs ham_args(const Tables &T, int col, bool with_d, double2 *psi, double2 *out, int out_mode,
                 bool turn, double *partial)
{
    const SpinTables &S = T.sp[col], &O = T.sp[1 - col];
    HamArgs A;
    std::memset(&A, 0, sizeof(A));
    A.colslot = S.colslot;
    A.patslot = S.patslot;
    A.hcode = S.hcode;
    A.baseslot = S.baseslot;
    A.rpat = O.pat;
    A.rbase = O.base;
    A.wrow = O.wrow;
    A.tb = T.d_tb;
    A.U = T.U;
    A.n = S.n;
    A.n_rows = O.n;
    A.nslots = S.nslots;
    A.lr = S.lr;
    A.nb = T.nb;
    A.n_flat = T.n_flat;
    A.diag = with_d ? 1 : 0;
    A.out_mode = out_mode;
    A.turn = turn ? 1 : 0;
    A.mix = T.mix;
    strides(T, col, &A.rs, &A.cs);
    A.psi = psi;
    A.out = out;
    A.partial = partial;
    A.grid = rows_grid(T, col);
    return A;
}

// Short rows' H: about an element per thread and round.
int ham_threads(const SpinTables &S) { return std::min(1024, 2 * S.threads); }
uint32_t ham_lds(const Tables &T, const SpinTables &S)
{
    return short_vec_bytes(S.nslots, S.lr) + (T.general ? (64u << S.lr) * 8u : 0u) + 16u * 8u;
}

void launch_ham(const Tables &T, int col, bool with_d, double2 *psi, double2 *out, int out_mode,
                bool turn, double *partial, hipStream_t s)
{
    const SpinTables &S = T.sp[col];
    const HamArgs A = ham_args(T, col, with_d, psi, out, out_mode, turn, partial);
    const dim3 grid(A.grid);
    if (S.is_long) {
        const uint32_t lds = long_vec_bytes(S.nslots) + 64u * 8u + 16u * 8u;
        if (T.general)
            hipLaunchKernelGGL((k_sec_ham_long<true>), grid, dim3(kLongT), lds, s, A);
        else
            hipLaunchKernelGGL((k_sec_ham_long<false>), grid, dim3(kLongT), lds, s, A);
    } else {
        const dim3 th(ham_threads(S));
        const uint32_t lds = ham_lds(T, S);
        if (T.general)
            hipLaunchKernelGGL((k_sec_ham_short<true>), grid, th, lds, s, A);
        else
            hipLaunchKernelGGL((k_sec_ham_short<false>), grid, th, lds, s, A);
    }
}

void transpose(const Tables &T, int from_col, const double2 *in, double2 *out, hipStream_t s)
{
    const int nr = T.n[1 - from_col], nc = T.n[from_col];
    hipLaunchKernelGGL(k_sec_transpose, dim3((nc + kTrTile - 1) / kTrTile, (nr + kTrTile - 1) / kTrTile),
                       dim3(kTrThreads), 0, s, in, out, nr, nc);
}

void set_attrs()
{
    static std::once_flag once;
    std::call_once(once, [] {
        const void *fns[] = {
            (const void *)k_sec_rows_short<S_FWD, false>, (const void *)k_sec_rows_short<S_FWD, true>,
            (const void *)k_sec_rows_short<S_REV, false>, (const void *)k_sec_rows_short<S_REV, true>,
            (const void *)k_sec_rows_spread<false>,       (const void *)k_sec_rows_spread<true>,
            (const void *)k_sec_expand,
            (const void *)k_sec_whole<false>,             (const void *)k_sec_whole<true>,
            (const void *)k_sec_whole_batch<false>,       (const void *)k_sec_whole_batch<true>,
            (const void *)k_sec_rows_long<S_FWD, false>,  (const void *)k_sec_rows_long<S_FWD, true>,
            (const void *)k_sec_rows_long<S_REV, false>,  (const void *)k_sec_rows_long<S_REV, true>,
            (const void *)k_sec_ham_short<false>,         (const void *)k_sec_ham_short<true>,
            (const void *)k_sec_ham_long<false>,          (const void *)k_sec_ham_long<true>,
            (const void *)k_sec_rows_batch<S_FWD, false>, (const void *)k_sec_rows_batch<S_FWD, true>,
            (const void *)k_sec_rows_batch<S_REV, false>, (const void *)k_sec_rows_batch<S_REV, true>,
            (const void *)k_sec_ham_batch<false>,         (const void *)k_sec_ham_batch<true>};
        for (const void *f : fns)
            (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    });
}

// Forward sweep: psi starts in layout A in `a` (from_start: it is |b0>, and
// `a` is not read); `b` is the layout-B buffer of long rows.  Returns the
// buffer holding the result (long rows: in layout P.final_col; both: in both
// layouts).
double2 *forward(const Tables &T, const Program &P, const double *theta, double2 *a, double2 *b,
                 bool from_start, bool both, hipStream_t s)
{
    double2 *cur = a;
    for (size_t i = 0; i < P.fwd.size(); ++i) {
        const bool last = i + 1 == P.fwd.size();
        double2 *other = (cur == a) ? b : a;
        int flags = from_start && i == 0 ? SF_START : 0;
        if (T.is_long && (!last || both))
            flags |= SF_TURN | (last ? SF_BOTH : 0);
        launch_rows<S_FWD>(T, P.fwd[i], theta, cur, nullptr, nullptr, 0, flags, s, other);
        if (T.is_long && !last)
            cur = other;
    }
    return cur;
}

// out <- H in for sector vectors in layout `col` (long rows; short ones have
// one layout).  Long rows: in_y is `in` in the other layout, where the other
// spin's hops act; their part comes back transposed.  last: HO_ADD; HO_MIX
// for the reverse sweep's vectors (out and in); HO_NONE: the energy only.
// Energy parts to partial rows 0 and 1 (partial != NULL).
void hamiltonian(const Tables &T, int col, double2 *in, double2 *out, double2 *in_y, int last,
                 double *partial, hipStream_t s)
{
    double *p1 = partial ? partial + kGrid : nullptr;
    launch_ham(T, 1 - col, false, T.is_long ? in_y : in, out, last == HO_NONE ? HO_NONE : HO_SET,
               T.is_long, p1, s);
    launch_ham(T, col, true, in, out, last, false, partial, s);
}

hubbard_status check(const char *what)
{
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return fail(HUBBARD_ERR_DEVICE, std::string(what) + ": " + hipGetErrorString(e));
    return HUBBARD_OK;
}

// Workspace of an evaluation: psi and lambda, each in both layouts (short rows
// have one layout and use the first buffer of each), and the partial rows (of the
// energy alone: two).
size_t eval_bytes(const Tables &T, const Program &P, bool grad = true)
{
    return 4 * align256(vec_elems(T) * 16) + align256((size_t)(grad ? P.n_rows : 2) * kGrid * 8);
}

// Arguments of a whole evaluation.
WholeArgs whole_args(const Tables &T, int layers, const double *theta, double *partial,
                     int pstride, bool grad)
{
    WholeArgs A;
    std::memset(&A, 0, sizeof(A));
    A.gates = T.d_gates;
    A.recs = T.whole.recs;
    A.hcode = T.whole.hcode;
    for (int s = 0; s < 2; ++s) {
        A.pat[s] = T.sp[s].pat;
        A.base[s] = T.sp[s].base;
        A.n2[s] = T.whole.n2[s];
        A.n13[s] = T.whole.n13[s];
    }
    A.wrow = T.sp[1].wrow;
    A.tb = T.d_tb;
    A.theta = theta;
    A.U = T.U;
    A.mix = T.mix;
    A.n = T.n[0];
    A.pitch = (T.n[0] + 1) | 1;
    A.n_phases = T.n_phases;
    A.per = T.per;
    A.layers = layers;
    A.nb = T.nb;
    A.n_red = 2 * T.per - 1;
    A.magic = ((1u << 20) + (uint32_t)T.n[0] - 1u) / (uint32_t)T.n[0];
    A.b0_row = T.b0_rank[1];
    A.b0_col = T.b0_rank[0];
    A.partial = partial;
    A.pstride = pstride;
    A.grad = grad ? 1 : 0;
    return A;
}
// E and, with grad != NULL, the gradient of the circuit's energy.
void evaluate(const Tables &T, const Program &P, const double *theta, double *E, double *grad,
              char *w, hipStream_t s)
{
    set_attrs();
    const size_t v = align256(vec_elems(T) * 16);
    // the two layouts' buffers (short rows: one layout, index 0)
    double2 *psi[2] = {(double2 *)w, (double2 *)(w + v)};
    double2 *lam[2] = {(double2 *)(w + 2 * v), (double2 *)(w + 3 * v)};
    double *partial = (double *)(w + 4 * v);
    const bool rev = grad && !P.fwd.empty();
    if (P.whole) {
        const int layers = std::max(0, (int)P.fwd.size() - 1);
        const WholeArgs A = whole_args(T, layers, theta, partial, kGrid, rev);
        const uint32_t lds = whole_lds(T, layers);
        const dim3 grid(rev ? 2 : 1), th(T.whole.threads);
        if (T.general)
            hipLaunchKernelGGL((k_sec_whole<true>), grid, th, lds, s, A);
        else
            hipLaunchKernelGGL((k_sec_whole<false>), grid, th, lds, s, A);
        hipLaunchKernelGGL(k_sec_reduce, dim3(rev ? P.n_out : 1), dim3(256), 0, s, partial, kGrid,
                           P.d_nblk, P.d_ptr, P.d_rows, P.d_scale, E, grad);
        return;
    }
    auto at = [&](int col) { return T.is_long ? col : 0; };
    if (P.fwd.empty()) {
        hipLaunchKernelGGL(k_sec_basis, dim3(2048), dim3(256), 0, s, psi[0], vec_elems(T),
                           T.b0_pos);
        if (T.is_long)
            transpose(T, 0, psi[0], psi[1], s);
    }
    // layout A lives in the first buffers, B in the second
    (void)forward(T, P, theta, psi[0], psi[1], true, true, s);
    int col = P.final_col;
    // lambda = H psi, the partial rows 0 and 1 get E; the reverse sweep runs
    // on chi1 (psi's buffers) and chi2 (lambda's): brackets from their
    // expectations
    hamiltonian(T, col, psi[at(col)], lam[at(col)], psi[at(1 - col)], rev ? HO_MIX : HO_NONE,
                partial, s);
    for (int i = (int)P.fwd.size() - 1; rev && i >= 0; --i) {
        const RowPass &p = P.fwd[i];
        col = p.col;
        launch_rows<S_REV>(T, p, theta, lam[at(col)], psi[at(col)], partial, P.red_row0[i],
                           i == 0 ? SF_NO_STORE : (T.is_long ? SF_TURN : 0), s, lam[at(1 - col)],
                           psi[at(1 - col)]);
    }
    hipLaunchKernelGGL(k_sec_reduce, dim3(rev ? P.n_out : 1), dim3(256), 0, s, partial, kGrid,
                       P.d_nblk, P.d_ptr, P.d_rows, P.d_scale, E, grad);
}

// psi, a full vector (2^(2 ns) amplitudes, not read) <- the circuit's state.
void state(const Tables &T, const Program &P, int ns, const double *theta, double2 *psi,
           hipStream_t s)
{
    set_attrs();
    const int skew = (1 << (ns - 1)) - 1;
    for (size_t i = 0; i < P.fwd.size(); ++i) {
        const RowPass &p = P.fwd[i];
        const SpinTables &S = T.sp[p.col];
        RowsArgs A = rows_args(T, p, false, theta, psi, nullptr, nullptr, 0, kGrid,
                               i == 0 ? SF_START : 0, nullptr, nullptr);
        A.dnpat = T.sp[1].pat;
        A.ns = ns;
        A.skew = skew;
        A.cs = p.col == 0 ? 1 : 0;
        const uint32_t lds = rows_lds(T, p.col, 0);
        if (T.general)
            hipLaunchKernelGGL((k_sec_rows_spread<true>), dim3(A.grid), dim3(S.threads), lds, s, A);
        else
            hipLaunchKernelGGL((k_sec_rows_spread<false>), dim3(A.grid), dim3(S.threads), lds, s, A);
    }
    const uint32_t lds = (uint32_t)T.n[0] * 16u + ((ns > 6 ? 2u << (ns - 6) : 2u) + 72u) * 4u;
    hipLaunchKernelGGL(k_sec_expand, dim3(std::min(1 << ns, 1024)), dim3(512), lds, s, psi, ns,
                       skew, T.n[0], T.ne[0], T.ne[1]);
}

// Angles of every op and diagonal phase tables were once kept in the
// workspace; callers' sizes stay what they were.
size_t ang_bytes(const Tables &T, int layers)
{
    return align256((size_t)(2 * T.nb + 1) * (layers + 1) * 16) +
           align256((size_t)layers * kDiagTab * 16);
}

}  // namespace sec

// ---------------------------------------------------------------- batches --
// energy_grad_batch on the sectors: one launch per position of the forward
// schedules, two of H and one per position of the reverse schedules, each
// running that pass of every instance that has one (launches of their own for
// each workgroup size and diagonal kind, on streams of their own).
// Every workgroup does what it does in the instance's own evaluation, and the
// partial sums are added in the same order: a batch's results are those of
// energy_grad bit for bit.

struct SectorBatch {
    struct Launch {
        int kind;   // S_FWD, S_REV, 2: H, 3: whole evaluations
        bool gen;
        int threads, lane, item0, n_items;
        uint32_t lds;
    };
    std::vector<Launch> launches;
    size_t partial_at = 0;   // byte offset of the partial sums in the workspace
    sec::RowsArgs *d_rows = nullptr;
    sec::HamArgs *d_ham = nullptr;
    sec::WholeArgs *d_whole = nullptr;
    sec::SecWork *d_work = nullptr;
    int32_t *d_seg_ptr = nullptr, *d_seg_cnt = nullptr;
    int64_t *d_seg_off = nullptr, *d_out_idx = nullptr;
    double *d_scale = nullptr;
    int n_out = 0;
    char *blob = nullptr;
    ~SectorBatch() { (void)hipFree(blob); }
};

// Workspace bytes that a batch on the sectors needs at most; 0: the instances
// do not all have such a form.
size_t sector_batch_bound(const hubbard_t *hs, int n, const int32_t *layers)
{
    size_t at = 0;
    for (int i = 0; i < n; ++i) {
        const Model &m = *handle_model(hs[i]);
        const uint32_t smask = (1u << m.ns) - 1u;
        const int ne = __builtin_popcount((uint32_t)m.neel & smask);
        size_t c = 1;   // C(ns, ne)
        for (int k = 1; k <= ne; ++k)
            c = c * (size_t)(m.ns - ne + k) / (size_t)k;
        const int G = m.ngroups;
        if (m.ansatz != 0 || c > (size_t)sec::kShortRow || layers[i] < 1 ||
            2 * G + 1 > sec::kMaxRed)
            return 0;
        const size_t rows = 2 + 2 * (size_t)layers[i] * (2 * G + 1);
        at += 2 * sec::align256(c * c * 16) + sec::align256(rows * (c + 8) * 8);
    }
    return at;
}

// Plans and uploads a batch; NULL: it has no such form, or no memory for it.
SectorBatch *sector_batch_build(const hubbard_t *hs, int n, const double *theta,
                                const int64_t *toff, const int32_t *layers, char *ws, int lanes)
try {
    using namespace sec;
    if (sector_batch_bound(hs, n, layers) == 0)
        return nullptr;
    std::unique_ptr<SectorBatch> B(new SectorBatch());
    std::vector<Tables *> T(n);
    std::vector<Program *> P(n);
    size_t at = 0;
    std::vector<size_t> voff(n);
    for (int i = 0; i < n; ++i) {
        if (get(hs[i], layers[i], &T[i], &P[i]) != HUBBARD_OK)
            return nullptr;
        voff[i] = at;
        at += 2 * align256(vec_elems(*T[i]) * 16);
    }
    B->partial_at = at;
    set_attrs();
    // instances by workgroup size and diagonal kind
    std::map<std::pair<int, bool>, std::vector<int>> classes;
    std::map<std::pair<int, bool>, double> cost;
    for (int i = 0; i < n; ++i) {
        // (whole evaluations: classes of their own)
        const std::pair<int, bool> c{P[i]->whole
                                         ? -T[i]->whole.threads
                                         : std::max(T[i]->sp[0].threads, T[i]->sp[1].threads),
                                     T[i]->general};
        classes[c].push_back(i);
        cost[c] += (double)vec_elems(*T[i]) * layers[i];
    }
    std::vector<std::pair<int, bool>> order;
    for (auto &kv : classes) {
        // the largest instances' workgroups start first
        std::stable_sort(kv.second.begin(), kv.second.end(), [&](int a, int b) {
            return T[a]->n[0] > T[b]->n[0];
        });
        order.push_back(kv.first);
    }
    std::stable_sort(order.begin(), order.end(),
                     [&](const std::pair<int, bool> &a, const std::pair<int, bool> &b) {
                         return cost[a] > cost[b];
                     });
    // outputs: the energies, then every instance's gradient
    std::vector<size_t> gbase(n);
    size_t n_out = n;
    for (int i = 0; i < n; ++i) {
        gbase[i] = n_out;
        n_out += (size_t)P[i]->n_out - 1;
    }
    std::vector<std::vector<std::pair<int64_t, int32_t>>> segs(n_out);
    std::vector<double> scale(n_out, 0.5);
    std::vector<int64_t> out_idx(n_out);
    std::vector<int64_t> prow(n);   // first partial entry of each instance
    std::vector<int> pstride(n);
    int64_t np = 0;
    for (int i = 0; i < n; ++i) {
        prow[i] = np;
        auto red_grid = [&](int col) { return P[i]->whole ? 1 : rows_grid(*T[i], col); };
        pstride[i] = std::max(red_grid(0), red_grid(1));
        np += (int64_t)P[i]->n_rows * pstride[i];
        scale[i] = 1.0;
        out_idx[i] = i;
        const Program &p = *P[i];
        auto seg = [&](int row, int col) {
            return std::make_pair(prow[i] + (int64_t)row * pstride[i],
                                  (int32_t)red_grid(col));
        };
        segs[i].push_back(seg(0, p.final_col));
        segs[i].push_back(seg(1, 1 - p.final_col));
        for (size_t k = 0; k < p.fwd.size(); ++k)
            for (int half = 0; half < 2; ++half)
                for (size_t r = 0; r < p.fwd[k].red_param.size(); ++r)
                    segs[gbase[i] + p.fwd[k].red_param[r]].push_back(
                        seg(p.red_row0[k] + half * (int)p.fwd[k].red_param.size() + (int)r,
                            p.fwd[k].col));
        for (int k = 0; k + 1 < p.n_out; ++k)
            out_idx[gbase[i] + k] = toff[i] + k;
    }
    double *partial = (double *)(ws + at);
    std::vector<RowsArgs> rows;
    std::vector<HamArgs> hams;
    std::vector<WholeArgs> wholes;
    std::vector<SecWork> work;
    size_t longest = 0;
    for (int i = 0; i < n; ++i)
        longest = std::max(longest, P[i]->fwd.size());
    // position `pos` of kind `kind`: one launch per class that has one
    auto position = [&](int kind, size_t pos) {
        for (size_t c = 0; c < order.size(); ++c) {
            if ((order[c].first < 0) != (kind == 3))
                continue;
            SectorBatch::Launch L;
            L.kind = kind;
            L.gen = order[c].second;
            L.lane = lanes > 1 ? (int)(c % (size_t)lanes) : 0;
            L.item0 = (int)work.size();
            L.threads = 64;
            L.lds = 0;
            for (int i : classes[order[c]]) {
                const Tables &t = *T[i];
                const Program &p = *P[i];
                if (kind == 3) {
                    SecWork w;
                    w.args = (int32_t)wholes.size();
                    w.bid = w.pad = 0;
                    wholes.push_back(whole_args(t, (int)p.fwd.size() - 1, theta + toff[i],
                                                partial + prow[i], pstride[i], true));
                    L.threads = t.whole.threads;
                    L.lds = std::max(L.lds, whole_lds(t, (int)p.fwd.size() - 1));
                    for (w.vsel = 0; w.vsel < 2; ++w.vsel)
                        work.push_back(w);
                    continue;
                }
                const size_t len = kind == 2 ? 2 : p.fwd.size();
                if (pos >= len)
                    continue;
                double2 *psi = (double2 *)(ws + voff[i]);
                double2 *lam = (double2 *)(ws + voff[i] + align256(vec_elems(t) * 16));
                int grid, vecs = 1;
                SecWork w;
                if (kind == 2) {
                    const int col = pos == 0 ? 1 - p.final_col : p.final_col;
                    w.args = (int32_t)hams.size();
                    hams.push_back(ham_args(t, col, pos == 1, psi, lam, pos == 0 ? HO_SET : HO_MIX,
                                            false,
                                            partial + prow[i] + (pos == 0 ? pstride[i] : 0)));
                    grid = hams.back().grid;
                    L.threads = std::max(L.threads, ham_threads(t.sp[col]));
                    L.lds = std::max(L.lds, ham_lds(t, t.sp[col]));
                } else {
                    const size_t k = kind == S_FWD ? pos : len - 1 - pos;
                    const RowPass &rp = p.fwd[k];
                    const bool rev = kind == S_REV;
                    w.args = (int32_t)rows.size();
                    rows.push_back(rows_args(t, rp, rev, theta + toff[i], rev ? lam : psi,
                                             rev ? psi : nullptr, partial + prow[i],
                                             rev ? p.red_row0[k] : 0, pstride[i],
                                             rev ? (k == 0 ? SF_NO_STORE : 0)
                                                 : (k == 0 ? SF_START : 0),
                                             nullptr, nullptr));
                    grid = rows.back().grid;
                    vecs = rev ? 2 : 1;
                    L.threads = std::max(L.threads, t.sp[rp.col].threads);
                    L.lds = std::max(L.lds, rows_lds(t, rp.col, rows.back().n_red));
                }
                for (int v = 0; v < vecs; ++v)
                    for (int b = 0; b < grid; ++b) {
                        w.bid = b;
                        w.vsel = v;
                        w.pad = 0;
                        work.push_back(w);
                    }
            }
            L.n_items = (int)work.size() - L.item0;
            if (L.n_items)
                B->launches.push_back(L);
        }
    };
    position(3, 0);
    for (size_t j = 0; j < longest; ++j)
        position(S_FWD, j);
    position(2, 0);
    position(2, 1);
    for (size_t j = 0; j < longest; ++j)
        position(S_REV, j);
    std::vector<int32_t> seg_ptr{0}, seg_cnt;
    std::vector<int64_t> seg_off;
    for (auto &v : segs) {
        for (auto &q : v) {
            seg_off.push_back(q.first);
            seg_cnt.push_back(q.second);
        }
        seg_ptr.push_back((int32_t)seg_off.size());
    }
    B->n_out = (int)n_out;
    Blob blob;
    blob.add(&B->d_rows, rows);
    blob.add(&B->d_ham, hams);
    blob.add(&B->d_whole, wholes);
    blob.add(&B->d_work, work);
    blob.add(&B->d_seg_ptr, seg_ptr);
    blob.add(&B->d_seg_cnt, seg_cnt);
    blob.add(&B->d_seg_off, seg_off);
    blob.add(&B->d_out_idx, out_idx);
    blob.add(&B->d_scale, scale);
    if (blob.upload(&B->blob) != hipSuccess)
        return nullptr;
    return B.release();
} catch (const std::exception &) {
    return nullptr;
}

void sector_batch_free(SectorBatch *b) { delete b; }

// Whether a launch runs on stream `lane` of the batch.
bool sector_batch_uses(const SectorBatch *b, int lane)
{
    for (const SectorBatch::Launch &l : b->launches)
        if (l.lane == lane)
            return true;
    return false;
}

// The launches of a batch on its lanes' streams (forked and joined by the caller).
void sector_batch_launch(const SectorBatch *b, const hipStream_t *lane)
{
    using namespace sec;
    for (const SectorBatch::Launch &l : b->launches) {
        const SecWork *w = b->d_work + l.item0;
        hipStream_t s = lane[l.lane];
#define HV_SEC_BATCH(K, ARGS)                                                                   \
    hipLaunchKernelGGL((K), dim3(l.n_items), dim3(l.threads), l.lds, s, ARGS, w)
        if (l.kind == 3) {
            if (l.gen)
                HV_SEC_BATCH(k_sec_whole_batch<true>, b->d_whole);
            else
                HV_SEC_BATCH(k_sec_whole_batch<false>, b->d_whole);
        } else if (l.kind == 2) {
            if (l.gen)
                HV_SEC_BATCH(k_sec_ham_batch<true>, b->d_ham);
            else
                HV_SEC_BATCH(k_sec_ham_batch<false>, b->d_ham);
        } else if (l.kind == S_FWD) {
            if (l.gen)
                HV_SEC_BATCH((k_sec_rows_batch<S_FWD, true>), b->d_rows);
            else
                HV_SEC_BATCH((k_sec_rows_batch<S_FWD, false>), b->d_rows);
        } else {
            if (l.gen)
                HV_SEC_BATCH((k_sec_rows_batch<S_REV, true>), b->d_rows);
            else
                HV_SEC_BATCH((k_sec_rows_batch<S_REV, false>), b->d_rows);
        }
#undef HV_SEC_BATCH
    }
}

// The reduction's tables (k_reduce_seg), and where the partial sums are.
void sector_batch_reduction(const SectorBatch *b, const int32_t **seg_ptr,
                            const int64_t **seg_off, const int32_t **seg_cnt,
                            const double **scale, const int64_t **out_idx, int *n_out,
                            size_t *partial_at)
{
    *seg_ptr = b->d_seg_ptr;
    *seg_off = b->d_seg_off;
    *seg_cnt = b->d_seg_cnt;
    *scale = b->d_scale;
    *out_idx = b->d_out_idx;
    *n_out = b->n_out;
    *partial_at = b->partial_at;
}

// The evaluations of the full-vector entry points (energy, energy_grad,
// energy_grad_noalloc) in the sector form: their circuits start from |b0>, so
// every amplitude outside its sector is zero throughout.

namespace sec {

// Tables and program that are already there (allocates nothing).
bool find(hubbard_t h, int layers, Tables **T, Program **P)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess)
        return false;
    std::shared_ptr<Entry> en;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        auto it = g_cache.find(std::make_pair(handle_uid(h), dev));
        if (it == g_cache.end())
            return false;
        en = it->second;
    }
    std::lock_guard<std::mutex> lk(en->mu);
    if (!en->tab)
        return false;
    auto p = en->progs.find(layers);
    if (p == en->progs.end())
        return false;
    *T = en->tab.get();
    *P = p->second.get();
    return true;
}

// The same, uploaded if they are not there; not under capture, where nothing may
// be allocated and the caller has launches that need none of it.
bool find_or_upload(hubbard_t h, int layers, hipStream_t s, Tables **T, Program **P)
{
    if (find(h, layers, T, P))
        return true;
    return !under_capture(s) && get(h, layers, T, P) == HUBBARD_OK;
}

}  // namespace sec

// Workspace bytes of an evaluation, uploading the tables if they are not there
// and s is not being captured; 0: not available (then the full vector is used).
size_t sector_eval_bytes(hubbard_t h, int layers, bool grad, hipStream_t s)
{
    sec::Tables *T = nullptr;
    sec::Program *P = nullptr;
    return sec::find_or_upload(h, layers, s, &T, &P) ? sec::eval_bytes(*T, *P, grad) : 0;
}

// The same for tables already uploaded (allocates nothing; 0: not there).
size_t sector_eval_ready(hubbard_t h, int layers)
{
    sec::Tables *T = nullptr;
    sec::Program *P = nullptr;
    return sec::find(h, layers, &T, &P) ? sec::eval_bytes(*T, *P) : 0;
}

// After either of them.  grad NULL: the energy only.
hubbard_status sector_eval(hubbard_t h, int layers, const double *theta, double *E, double *grad,
                           void *ws, hipStream_t s)
{
    sec::Tables *T = nullptr;
    sec::Program *P = nullptr;
    if (!sec::find(h, layers, &T, &P))
        return set_error(HUBBARD_ERR_STATE, "no sector tables");
    sec::evaluate(*T, *P, theta, E, grad, (char *)ws, s);
    return sec::check("sector evaluation");
}

// Whether a start-state circuit's full vector can be made on its sector: a
// plan of short rows and at least one pass.
bool sector_state_ok(hubbard_t h, int layers, hipStream_t s)
{
    sec::Tables *T = nullptr;
    sec::Program *P = nullptr;
    return sec::find_or_upload(h, layers, s, &T, &P) && !T->is_long && !P->fwd.empty();
}

hubbard_status sector_state(hubbard_t h, int layers, const double *theta, double2 *psi,
                            hipStream_t s)
{
    sec::Tables *T = nullptr;
    sec::Program *P = nullptr;
    if (!sec::find(h, layers, &T, &P))
        return set_error(HUBBARD_ERR_STATE, "no sector tables");
    sec::state(*T, *P, handle_model(h)->ns, theta, psi, s);
    return sec::check("state preparation");
}

// Drop the sector tables and programs of a destroyed handle.
void sector_forget(uint64_t uid)
{
    std::lock_guard<std::mutex> lk(sec::g_mu);
    for (auto it = sec::g_cache.begin(); it != sec::g_cache.end();)
        it = it->first.first == uid ? sec::g_cache.erase(it) : std::next(it);
}

}  // namespace hv

using namespace hv;
using namespace hv::sec;

hubbard_status hubbard_sector_dim(hubbard_t h, int64_t *n_up, int64_t *n_dn)
{
    Tables *T = nullptr;
    hubbard_status st = get(h, -1, &T, nullptr);
    if (st != HUBBARD_OK)
        return st;
    if (n_up)
        *n_up = T->n[0];
    if (n_dn)
        *n_dn = T->n[1];
    return HUBBARD_OK;
}

hubbard_status hubbard_sector_workspace_size(hubbard_t h, int32_t n_layers, int32_t op,
                                             size_t *bytes)
{
    if (!bytes || n_layers < 0 || op < HUBBARD_SECTOR_ANSATZ || op > HUBBARD_SECTOR_LANCZOS)
        return set_error(HUBBARD_ERR_ARG, "bad arguments to hubbard_sector_workspace_size");
    Tables *T = nullptr;
    Program *P = nullptr;
    const bool h_only = op == HUBBARD_SECTOR_HAMILTONIAN || op == HUBBARD_SECTOR_LANCZOS;
    hubbard_status st = get(h, h_only ? 0 : n_layers, &T, &P);
    if (st != HUBBARD_OK)
        return st;
    const size_t v = align256(vec_elems(*T) * 16);
    if (op == HUBBARD_SECTOR_ANSATZ)
        *bytes = v + ang_bytes(*T, n_layers);
    else if (op == HUBBARD_SECTOR_HAMILTONIAN)
        *bytes = 2 * v;
    else if (op == HUBBARD_SECTOR_LANCZOS)
        *bytes = 5 * v + lanczos_partial_bytes();
    else
        *bytes = eval_bytes(*T, *P) + ang_bytes(*T, n_layers);
    return HUBBARD_OK;
}

hubbard_status hubbard_sector_init_neel(hubbard_t h, void *psi_dev, void *stream)
{
    Tables *T = nullptr;
    hubbard_status st = get(h, -1, &T, nullptr);
    if (st != HUBBARD_OK)
        return st;
    if (!psi_dev)
        return set_error(HUBBARD_ERR_ARG, "null vector");
    hipLaunchKernelGGL(k_sec_basis, dim3(2048), dim3(256), 0, (hipStream_t)stream,
                       (double2 *)psi_dev, vec_elems(*T), T->b0_pos);
    return check("sector init");
}

hubbard_status sector_ansatz_apply(hubbard_t h, const double *theta_dev, int32_t n_layers,
                                   void *psi_dev, void *ws_dev, size_t ws_bytes, void *stream)
{
    if (n_layers < 0 || !psi_dev || (n_layers > 0 && !theta_dev))
        return set_error(HUBBARD_ERR_ARG, "bad arguments to sector_ansatz_apply");
    Tables *T = nullptr;
    Program *P = nullptr;
    hubbard_status st = get(h, n_layers, &T, &P);
    if (st != HUBBARD_OK)
        return st;
    const size_t v = align256(vec_elems(*T) * 16);
    if (!ws_dev || ws_bytes < v + ang_bytes(*T, n_layers))
        return set_error(HUBBARD_ERR_SIZE, "workspace too small for sector_ansatz_apply");
    set_attrs();
    hipStream_t s = (hipStream_t)stream;
    double2 *out = forward(*T, *P, theta_dev, (double2 *)psi_dev, (double2 *)ws_dev, false, false, s);
    if (out != (double2 *)psi_dev)   // ended in layout B
        transpose(*T, 1, out, (double2 *)psi_dev, s);
    return check("sector ansatz");
}

hubbard_status sector_hamiltonian_apply(hubbard_t h, const void *psi_dev, void *out_dev,
                                        void *ws_dev, size_t ws_bytes, void *stream)
{
    if (!psi_dev || !out_dev || psi_dev == out_dev)
        return set_error(HUBBARD_ERR_ARG, "sector_hamiltonian_apply needs distinct vectors");
    Tables *T = nullptr;
    Program *P = nullptr;
    hubbard_status st = get(h, 0, &T, &P);
    if (st != HUBBARD_OK)
        return st;
    const size_t v = align256(vec_elems(*T) * 16);
    if (!ws_dev || ws_bytes < 2 * v)
        return set_error(HUBBARD_ERR_SIZE, "workspace too small for sector_hamiltonian_apply");
    set_attrs();
    if (T->is_long)
        transpose(*T, 0, (const double2 *)psi_dev, (double2 *)ws_dev, (hipStream_t)stream);
    hamiltonian(*T, 0, (double2 *)psi_dev, (double2 *)out_dev, (double2 *)ws_dev, HO_ADD, nullptr,
                (hipStream_t)stream);
    return check("sector H");
}

hubbard_status hubbard_sector_lanczos(hubbard_t h, const void *start_dev, int32_t max_iter,
                                      double tol, double *E0, int32_t *iters, double *residual,
                                      void *gs_dev, void *ws_dev, size_t ws_bytes, void *stream)
{
    if (!start_dev || max_iter < 1 || !(tol > 0.0) || !E0 || !ws_dev)
        return set_error(HUBBARD_ERR_ARG, "bad arguments to hubbard_sector_lanczos");
    Tables *T = nullptr;
    Program *P = nullptr;
    hubbard_status st = get(h, 0, &T, &P);
    if (st != HUBBARD_OK)
        return st;
    const size_t n = vec_elems(*T), v = align256(n * 16);
    const size_t need = 5 * v + lanczos_partial_bytes();
    if (ws_bytes < need)
        return set_error(HUBBARD_ERR_SIZE, "workspace too small for hubbard_sector_lanczos");
    const char *ws = (const char *)ws_dev;
    for (const void *p : {start_dev, (const void *)gs_dev}) {
        const char *q = (const char *)p;
        if (q && q < ws + need && ws < q + n * 16)
            return set_error(HUBBARD_ERR_ARG, "start or state vector overlaps the workspace");
    }
    set_attrs();
    hipStream_t s = (hipStream_t)stream;
    char *w = (char *)ws_dev;
    double2 *buf[3] = {(double2 *)w, (double2 *)(w + v), (double2 *)(w + 2 * v)};
    double2 *in_b = (double2 *)(w + 3 * v);
    const ApplyH apply = [&](const double2 *in, double2 *out) {
        if (T->is_long)
            transpose(*T, 0, in, in_b, s);
        hamiltonian(*T, 0, (double2 *)in, out, in_b, HO_ADD, nullptr, s);
        return check("sector H");
    };
    return lanczos_run(apply, n, (const double2 *)start_dev, max_iter, tol, E0, iters, residual,
                       (double2 *)gs_dev, buf, (double2 *)(w + 5 * v), s);
}

hubbard_status sector_energy_grad(hubbard_t h, const double *theta_dev, int32_t n_layers,
                                  double *E_dev, double *grad_dev, void *ws_dev, size_t ws_bytes,
                                  void *stream)
{
    if (n_layers < 0 || !E_dev || (n_layers > 0 && (!theta_dev || !grad_dev)))
        return set_error(HUBBARD_ERR_ARG, "bad arguments to sector_energy_grad");
    Tables *T = nullptr;
    Program *P = nullptr;
    hubbard_status st = get(h, n_layers, &T, &P);
    if (st != HUBBARD_OK)
        return st;
    if (!ws_dev || ws_bytes < eval_bytes(*T, *P) + ang_bytes(*T, n_layers))
        return set_error(HUBBARD_ERR_SIZE, "workspace too small for sector_energy_grad");
    evaluate(*T, *P, theta_dev, E_dev, grad_dev, (char *)ws_dev, (hipStream_t)stream);
    return check("sector energy_grad");
}

// ham.hip -- H on a caller's full vector in two sweeps over memory.
//
// The pass kernels (kernels.hip) apply the hops whose qubits meet in one LDS
// tile of 2^12 amplitudes and accumulate into the result: at 28 qubits five
// passes, four of which also read the result back.  Here every amplitude of
// the result gathers its neighbours psi[i ^ m_b], all bonds of one spin in one
// sweep: a workgroup holds a piece of a spin-up row (or of eight neighbouring
// spin-down columns, 128 bytes wide) in LDS and reads the neighbours inside it
// there.  The others lie in the same row, or columns, which the same XCD works on:
// a row stays in its L2, the columns do not.
//   down: out <- H_dn psi                  (read psi, write out)
//   up:   out <- out + (D + H_up) psi      (read psi and out, write out)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <vector>

#include "hubvqe.hpp"

namespace hv {

constexpr int kGatherBonds = 64;   // as kernel arguments
constexpr int kGatherMinSites = 8;
constexpr int kGatherT = 512, kGatherR = 4;

// A bond as one sweep's waves see it.  The lanes of a wave differ in the
// pattern's low bits (up: six, down: three), so a bond of two higher sites
// moves an electron of all lanes' amplitudes or of none, with one sign.
struct GatherBond {
    uint32_t m;        // the bond's two sites
    uint32_t bt;       // the sites strictly between (Jordan-Wigner string)
    double t;          // H's coefficient, -t_b
    uint64_t on, odd;  // lanes whose low bits hold one of the bond's electrons; an odd
                       // number of them between its sites
};
struct GatherArgs {
    int ns, nb;
    double U;
    const double *site;          // general: eps and V energy of one spin's patterns
    GatherBond b[kGatherBonds];
    double V[kGatherBonds];
};

namespace {

typedef __attribute__((address_space(1))) double2 gc128;
typedef const __attribute__((address_space(1))) char gchar;
typedef const __attribute__((address_space(1))) double gf64;
typedef double vec2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(1))) vec2 gvec2;

__device__ __forceinline__ double flip(double y, bool sign)
{
    const long long b = __double_as_longlong(y);
    return __longlong_as_double(b ^ (sign ? (long long)0x8000000000000000ull : 0ll));
}

// Bit r of byte v: the parity of r & v.
__device__ __forceinline__ uint32_t round_parity(uint32_t v)
{
    return (uint32_t)(0x963C5AF066CCAA00ull >> (8 * v)) & 0xFFu;
}

// A wave's R rounds of 64 amplitudes: acc[r] <- acc[r] + bond B's term.  The
// wave's first pattern is `first` (round 0; round r adds r << RS); bit r of am:
// the uniform part of "the bond moves an electron of round r's amplitudes".
//   VARY: the bond's low site is one of the lanes' pattern bits, so that the
//   lanes decide.  LOCAL: the neighbours are in the workgroup's tile.
template <bool UP, int T, int R, bool VARY, bool LOCAL>
__device__ __forceinline__ void bond_term(const GatherBond &B, uint32_t first, uint32_t mr,
                                          uint32_t am, const char *tile, int l0,
                                          const gchar *base, uint32_t at, int sh,
                                          double2 (&acc)[R])
{
    constexpr int LB = UP ? 6 : 3, RS = LB + __builtin_ctz(T / 64);
    constexpr uint32_t low = (1u << LB) - 1u, rounds = (uint32_t)(R - 1) << RS;
    const uint32_t sm = round_parity(B.bt >> RS & (R - 1)) ^
                        (__popc(first & B.bt) & 1 ? 0xFFu : 0u);   // signs of the rounds
    const double c0 = VARY ? flip(B.t, __builtin_amdgcn_inverse_ballot_w64(B.odd)) : B.t;
    const uint32_t la = (uint32_t)((l0 ^ (int)((B.m & ~rounds) << (UP ? 0 : 3))) * 16);
    const uint32_t ga = VARY ? at ^ (B.m & low) << (sh + 4) : at;
    double2 x[R];
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (VARY || (am >> r & 1u)) {
            if constexpr (LOCAL) {
                x[r] = *(const double2 *)(tile + (la + ((uint32_t)r ^ mr) * (T * 16)));
            } else {
                const uint32_t p = (first | (uint32_t)r << RS) ^ (B.m & ~low);
                const gc128 *e = (const gc128 *)(base + ((int64_t)p << (sh + 4)) + ga);
                x[r] = make_double2(e->x, e->y);
            }
        }
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (VARY ? __builtin_amdgcn_inverse_ballot_w64(B.on ^ (am >> r & 1u ? ~0ull : 0ull))
                 : (am >> r & 1u) != 0) {
            const double c = flip(c0, sm >> r & 1u);
            acc[r].x = fma(c, x[r].x, acc[r].x);
            acc[r].y = fma(c, x[r].y, acc[r].y);
        }
}

}  // namespace

// Bound by what lies behind the L2s: at 28 qubits and 19 bonds 4.8 ms down and 3.1
// up (the five passes 13.7), with 33.8 and 15.0 GB moved there (least: 8.6 and
// 12.9), 7.0 and 4.8 TB/s.  A slab of columns at a power-of-two stride meets few of
// an L2's sets, so the neighbours outside the tile (12 bonds, half of the elements
// each) are all read again, whichever the order of the slabs (4.7 to 6 ms).  With all neighbours gathered from L2 the texture path
// bound it, 30 cycles per load of 64 amplitudes: 10.5 ms.  512 threads of four
// amplitudes: 256 x 4, 512 x 2, 1024 x 4 and 256 x 8 took 3 to 12 % longer.
template <bool UP, bool GEN, int T, int R>
__global__ void __launch_bounds__(T)
k_ham_gather(GatherArgs A, const double2 *__restrict__ psi_, double2 *__restrict__ out_)
{
    __shared__ __align__(16) double2 tile[T * R];
    __shared__ double nib[64], w[16];
    const gc128 *__restrict__ psi = (const gc128 *)psi_;
    gc128 *__restrict__ out = (gc128 *)out_;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // workgroups go to the XCDs in turn: a row, or a slab of columns, to one
    const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
    constexpr int LB = UP ? 6 : 3, RS = LB + __builtin_ctz(T / 64);   // pattern bits that differ between lanes,
                                                  // within a round
    constexpr uint32_t low = (1u << LB) - 1u, span = (uint32_t)R << RS;
    const int parts = (1 << A.ns) / (int)span;
    const int line = (idx / parts) * 8 + xcd, part = idx % parts;
    const int sh = UP ? 0 : A.ns;
    const int64_t line0 = UP ? (int64_t)line << A.ns : (int64_t)line * 8;
    const gchar *base = (const gchar *)(psi + line0);
    const uint32_t at = UP ? (uint32_t)lane * 16u
                           : ((uint32_t)(lane >> 3) << A.ns | (uint32_t)(lane & 7)) * 16u;
    const uint32_t first = (uint32_t)part * span + ((uint32_t)wave << LB);
    auto offset = [&](int r) __attribute__((always_inline)) {   // of the wave's round r
        return (int64_t)(first | (uint32_t)r << RS) << (sh + 4);
    };
    double2 acc[R];
    vec2 old[UP ? R : 1];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const gc128 *e = (const gc128 *)(base + offset(r) + at);
        acc[r] = make_double2(e->x, e->y);
    }
    if constexpr (UP)
#pragma unroll
        for (int r = 0; r < R; ++r)   // read once
            old[r] = __builtin_nontemporal_load(
                (const gvec2 *)((const gchar *)(out + line0) + offset(r) + at));
#pragma unroll
    for (int r = 0; r < R; ++r)
        tile[r * T + tid] = acc[r];
    if constexpr (UP) {
        double erow = 0.0;
        if constexpr (GEN) {
            // D = E(up) + E(dn) + sum_i n_i,up w_i, w_i = U n_i,dn + sum_j V_ij n_j,dn:
            // the sum over each nibble's values
            if (tid < 16) {
                double s = tid < A.ns && (line >> tid & 1) ? A.U : 0.0;
                for (int b = 0; b < A.nb; ++b)
                    if (A.b[b].m >> tid & 1u)
                        s += (A.b[b].m & ~(1u << tid) & (uint32_t)line) ? A.V[b] : 0.0;
                w[tid] = s;
            }
            __syncthreads();
            if (tid < 64) {
                double s = 0.0;
                for (int j = 0; j < 4; ++j)
                    s += tid >> j & 1 ? w[(tid >> 4) * 4 + j] : 0.0;
                nib[tid] = s;
            }
            __syncthreads();
            erow = ((gf64 *)A.site)[line];
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t p = first | (uint32_t)r << RS | (uint32_t)lane;
            double d;
            if constexpr (GEN)
                d = ((gf64 *)A.site)[p] + erow +
                    ((nib[p & 15] + nib[16 + (p >> 4 & 15)]) +
                     (nib[32 + (p >> 8 & 15)] + nib[48 + (p >> 12 & 15)]));
            else
                d = A.U * (double)__popc(p & (uint32_t)line);
            acc[r] = make_double2(fma(d, acc[r].x, old[r].x), fma(d, acc[r].y, old[r].y));
        }
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r)
            acc[r] = make_double2(0.0, 0.0);
    }
    __syncthreads();
    for (int b = 0; b < A.nb; ++b) {
        const GatherBond &B = A.b[b];
        const uint32_t mr = B.m >> RS & (uint32_t)(R - 1);
        const uint32_t am = (round_parity(mr) ^ (__popc(first & B.m) & 1 ? 0xFFu : 0u)) &
                            ((1u << R) - 1u);
        const bool local = B.m < span;
        const char *t = (const char *)tile;
        if (B.m & low) {
            if (local)
                bond_term<UP, T, R, true, true>(B, first, mr, am, t, tid, base, at, sh, acc);
            else
                bond_term<UP, T, R, true, false>(B, first, mr, am, t, tid, base, at, sh, acc);
        } else if (am != 0) {
            if (local)
                bond_term<UP, T, R, false, true>(B, first, mr, am, t, tid, base, at, sh, acc);
            else
                bond_term<UP, T, R, false, false>(B, first, mr, am, t, tid, base, at, sh, acc);
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const vec2 y = {acc[r].x, acc[r].y};
        __builtin_nontemporal_store(
            y, (gvec2 *)((__attribute__((address_space(1))) char *)(out + line0) + offset(r) + at));
    }
}

// Whether H of the model has this form: its bonds fit the kernel's arguments and
// a row fills a round of a workgroup.  It won at every size measured (passes / this, with
// launches): 16 qubits 55 / 15 us, 20 qubits 92 / 29 us, 24 qubits 611 / 348 us,
// 28 qubits 13.6 / 7.9 ms, 30 qubits 53 / 34 ms, 32 qubits (a torus) 253 / 216 ms.
bool ham_gather_ok(const Model &m)
{
    return m.ns >= kGatherMinSites && m.nb <= kGatherBonds;
}

// eps and V energy of one spin's patterns (both spins': the same).
std::vector<double> ham_site_table(const Model &m)
{
    std::vector<double> e((size_t)1 << m.ns, 0.0);
    for (size_t p = 1; p < e.size(); ++p) {
        const int i = __builtin_ctzll(p);
        const size_t rest = p & (p - 1);
        double s = m.eps[i];
        for (int b = 0; b < m.nb; ++b) {
            const int j = m.bi[b] == i ? m.bj[b] : (m.bj[b] == i ? m.bi[b] : -1);
            if (j >= 0 && (rest >> j & 1))
                s += m.V[b];
        }
        e[p] = e[rest] + s;
    }
    return e;
}

// Arguments of the sweep over spin-up (or spin-down) hops.
static GatherArgs gather_args(const Model &m, bool up, const double *site)
{
    GatherArgs A;
    std::memset(&A, 0, sizeof(A));
    A.ns = m.ns;
    A.nb = m.nb;
    A.U = m.U;
    A.site = site;
    const int bits = up ? 6 : 3, lane0 = up ? 0 : 3;   // the lanes' pattern bits
    auto holds = [&](uint32_t sites) {   // lanes with an odd number of the sites' electrons
        uint64_t lanes = 0;
        for (int l = 0; l < 64; ++l)
            if (__builtin_popcount(sites & (uint32_t)(l >> lane0) & ((1u << bits) - 1u)) & 1)
                lanes |= 1ull << l;
        return lanes;
    };
    for (int b = 0; b < m.nb; ++b) {
        const int lo = std::min(m.bi[b], m.bj[b]), hi = std::max(m.bi[b], m.bj[b]);
        GatherBond &B = A.b[b];
        B.m = 1u << lo | 1u << hi;
        B.bt = ((1u << hi) - 1u) & ~((2u << lo) - 1u);
        B.t = -m.t[b];
        B.on = holds(B.m);
        B.odd = holds(B.bt);
        A.V[b] = m.V[b];
    }
    return A;
}

// out <- H psi (full vectors); site: ham_site_table's values on the device
// (general models).
void ham_gather(const Model &m, const double *site, const double2 *psi, double2 *out,
                hipStream_t s)
{
    const GatherArgs D = gather_args(m, false, site), U = gather_args(m, true, site);
    // kGatherT kGatherR amplitudes per workgroup; up rows of under 2^11: 256
    const uint64_t dim = (uint64_t)1 << m.nq;
    const bool tall = m.ns >= 11;
    const dim3 gd((unsigned)(dim / (kGatherT * kGatherR))), td(kGatherT);
    const dim3 gu(tall ? gd.x : (unsigned)(dim / 256)), tu(tall ? kGatherT : 256);
    hipLaunchKernelGGL((k_ham_gather<false, false, kGatherT, kGatherR>), gd, td, 0, s, D, psi, out);
    if (m.general && tall)
        hipLaunchKernelGGL((k_ham_gather<true, true, kGatherT, kGatherR>), gu, tu, 0, s, U, psi, out);
    else if (m.general)
        hipLaunchKernelGGL((k_ham_gather<true, true, 256, 1>), gu, tu, 0, s, U, psi, out);
    else if (tall)
        hipLaunchKernelGGL((k_ham_gather<true, false, kGatherT, kGatherR>), gu, tu, 0, s, U, psi, out);
    else
        hipLaunchKernelGGL((k_ham_gather<true, false, 256, 1>), gu, tu, 0, s, U, psi, out);
}

}  // namespace hv

// sector_plan.hpp -- host plan and device tables of the particle-number
// sector form (sector_plan.cpp builds them, sector.hip runs them).
//
// A row of the sector matrix holds the amplitudes of the n patterns of one
// spin.  The hops of one layer and spin are split into phases; a phase takes
// a cluster of four sites and applies hops on those sites that are next in
// order.  The patterns that agree outside the cluster and have k electrons
// on it form an orbit of C(4, k) elements (1, 4, 6, 4, 1) that the phase's
// hops keep: one thread holds a whole orbit in registers, so all hops of a
// phase cost one pass over the row's copy in LDS.
//
// A phase's hops form at most two matchings, one after the other.  Two
// matchings on four sites make a path or a ring, so the sites can be named
// 0..3 such that the first holds (0,1) and (2,3) and the second (0,2) and
// (1,3): every phase is the same four positions, those without a hop rotate
// by zero, and the kernels have no case to decide (six cases per hop, merged
// after each one, spilled hundreds of bytes per lane).
#pragma once

#include <array>
#include <cstdint>
#include <vector>

#include "hubvqe.hpp"

namespace hv {
namespace sec {

// Rows of up to kShortRow elements live in LDS (one or more rows per
// workgroup, kernels k_sec_*_short); longer ones (16 sites with 6 to 10
// electrons) do not fit next to the tables and live in registers, LDS
// carrying their real and imaginary parts one after the other (k_sec_*_long).
constexpr int kShortRow = 6500;
constexpr int kLongT = 1024;                  // threads of a long-row workgroup
constexpr int kLongElems = 13;                // row elements per thread, in row order
constexpr int kMaxRows = kLongElems * kLongT; // longest row: C(16, 8) = 12870
constexpr int kLongDummy = 32;                // slots that absent elements of a long row use
constexpr int kOrbitElems = 15;               // a long-row thread's elements in a phase: one
                                              // orbit of 6, two of 4 (k = 1, 3), one single

// The hop at one position of a phase (the same for both spins): its group
// slot, and its t_b (0: no hop; the slot is then its neighbour's).
constexpr int kPositions = 4;
constexpr int kPosA[kPositions] = {0, 2, 0, 1}, kPosB[kPositions] = {1, 3, 2, 3};
struct SecGate {
    int32_t slot;    // parameter slot in the layer, 1..groups (0: the model has no bonds)
    int32_t last;    // reverse order: the phase's next position has another slot, so the
                     // slot's sum is complete (never with slot 0, which has no sum)
    double t;        // hopping t_b
};
static_assert(sizeof(SecGate) == 16, "SecGate layout");

// One phase of a long row: orbits with 2, 1, 3 electrons.
struct SecPhase {
    int32_t n[3];
    int32_t pad;
};
static_assert(sizeof(SecPhase) == 16, "SecPhase layout");

// A phase record of a short row (16 bytes): u16 slots of the orbit's elements
// (6 for k = 2 in the order 01 02 03 12 13 23, 4 for k = 1 by the occupied
// site and for k = 3 by the empty one), and in the dword after them the hops'
// Jordan-Wigner signs: with two electrons bit 31 - (2 q + e) for position q
// and the e-th of the two spectator sites, with one bit 23 - q, with three
// bit 19 - q; bit 0 is set.  A phase's records are three lists (k = 2, 1, 3),
// each filled up to the lanes of half a workgroup with records of the zero
// slot (bit 0 clear).
struct Rec {
    uint32_t w[4];
};

// Tables of one spin's rows.
struct SpinPlan {
    int n = 0;                       // patterns
    int n_el = 0;                    // electrons
    int classes = 1;                 // LDS bank classes: slot mod classes = the pattern's class
    int nslots = 0;                  // LDS slots of a row (a multiple of classes)
    int lr = 0;                      // short rows: log2 of the rows of a workgroup
    int threads = 64;                // threads of a workgroup
    bool is_long = false;
    std::vector<uint32_t> pat;       // pattern of each rank
    std::vector<int32_t> rank_of;    // rank of a pattern, or -1
    std::vector<uint16_t> colslot;   // slot of each rank (long rows: in thread chunks)
    std::vector<uint16_t> patslot;   // pattern of each slot (0: the slot holds nothing)
    std::vector<double> base;        // per rank: sum_i eps_i p_i + sum_b V_b p_i p_j
    std::vector<double> baseslot;    // the same per slot
    std::vector<double> wrow;        // per rank: 16 x (U p_j + sum_i V_ij p_i)
    std::vector<SecPhase> phases;
    std::vector<Rec> recs;           // short rows: phase by phase, three lists each
    std::vector<uint32_t> lcode;     // long rows: per phase and thread 8 dwords: 15 u16 slots
                                     // and the upper half of the three orbits' sign bits
    std::vector<uint32_t> lpat;      // long rows: phase 0's patterns, 8 dwords per thread
    std::vector<double> lbase;       // long rows: phase 0's base values, [15][kLongT]
    std::vector<uint16_t> hcode;     // H: partner slot | sign << 15 (see build_spin)
};

struct SectorPlan {
    std::vector<SecGate> gates;              // kPositions per phase
    std::vector<std::array<int, 4>> sites;   // per phase: sites 0..3 (>= ns: none)
    std::vector<std::array<int, 4>> bond;    // per phase and position: its bond, or -1
    std::vector<int> ham_order;              // H's bonds in the order of hcode: long rows'
    int n_flat = 0;                          // without a Jordan-Wigner string first, n_flat of them
    SpinPlan spin[2];
    double mix = 1.0;                        // m of the reverse sweep's vectors, a power of two
};

// Codes per row element of H's tables: bonds padded to whole 16-byte chunks.
inline int ham_bonds(int nb) { return (nb + 7) / 8 * 8; }

// Entry of element j of thread t in a long row's u16 tables: chunks of eight
// codes, so that a thread reads a chunk with one load.
inline int long_index(int t, int j) { return ((j / 8) * kLongT + t) * 8 + j % 8; }

// The plan of a model's sector; returns an empty string or an error message.
std::string plan_sector(const Model &m, SectorPlan &P);

}  // namespace sec
}  // namespace hv

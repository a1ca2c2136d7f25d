// Partial-sum slots of the little GCR kernels, and which of them a step uses.
// Plain C++ without HIP, so that a check on the host can include it.
#pragma once

namespace dfl {

constexpr int kMaxLittleNkv = 32;   // most Krylov vectors of the little GCR
constexpr int kMaxLittleDefl = 32;  // most global deflation directions of the little system

namespace little {

constexpr int NK = kMaxLittleNkv;
constexpr int NQ = kMaxLittleDefl;
constexpr int NPASS = 2 * NK + 2 + NQ;  // slots of one Gram-Schmidt pass
constexpr int SA = 0;                   // first pass: (chi_j, chi_k) j<k | (chi_j, r) j<k | ||chi_k||^2 | (chi_k, r) | (Q_l, chi_k)
constexpr int SB = NPASS;               // second pass, same layout
constexpr int SC = 2 * NPASS;           // ||r||^2 inside a cycle
constexpr int SR = SC + 1;              // ||r||^2 after a restart
constexpr int SW = SC + 2;              // ||w||^2
constexpr int SQ = SC + 3;              // (Q_l, r), or (Z_l, r) then (W_l, r), at the start and after a restart
constexpr int NSLOT = SQ + 2 * NQ;
// the block-pair solver's first passes alternate between SA and these
constexpr int SA1 = NSLOT;
constexpr int NSLOT_PAIR = SA1 + NPASS;

// Up to so many workgroups, each of the block-pair solver sums all partial sums
// itself after one barrier. Nothing then tells a workgroup that the others have
// read its partial sums but their flags at a later barrier, and the barriers of
// the operator wait for neighbours only: workgroups at distance three or more
// are ordered by the next reduction alone. So the first passes of consecutive
// steps use different slots, and a slot is written again only after a whole
// reduction has come between.
constexpr int kPairAllRead = 16;
constexpr int pair_first_slot(int k) { return (k & 1) ? SA1 : SA; }

}  // namespace little
}  // namespace dfl

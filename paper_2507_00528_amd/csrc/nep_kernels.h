// HIP kernels of the NEP loss-and-gradient path (gfx950, wave64).
//
// Data flow of one loss-and-gradient evaluation:
//   neighbors -> species order -> forward (descriptors, network, partial forces)
//   -> forces and virials -> per-structure loss and cotangents -> adjoint (tangent
//   pass, network adjoint, parameter partials) -> W0 reduction -> final gradient
//   reduction -> Adam.
// Per-atom kernels run in "species order": per chunk of 2048 atoms grouped by
// species, each group starting on a multiple of 32 positions, and 8, 16 or 32
// lanes per atom, so every block evaluates one species' network.  Positions
// without an atom write nothing.
#pragma once
#include "nep_device.h"

namespace nep {

enum : int { FL_OVERFLOW = 1, FL_NONFINITE = 2, FL_BOX = 4, FL_TYPE = 8, FL_POS = 16, FL_STEP = 32, FL_BARRIER = 64 };

// ---------------------------------------------------------------- arguments
struct NbrArgs {
  int N, S, T, capR, capA;
  float rcR, rcA;
  const int* aoff;
  const float* box;
  const float* tilt;  // [S][3] (xy, xz, yz), null: every cell orthorhombic
  const float* pos;
  const int* type;
  uint32_t* idxR;
  int* cntR;
  uint32_t* idxA;
  int* cntA;
  int* astruct;
  float4* p4;    // [N] packed atoms (atom_word)
  int* bflags;   // [blocks] flag word of each all-pairs block; null: into flags
  int* flags;
  // cell-list search of structures of at least cell_min atoms (cells = 0:
  // all-pairs only)
  int cells, cell_min;
  int4* grid;    // [S] bins per axis (na, nb, nc, na nb nc), zero: all-pairs
  int* cell;     // [N] bin counts
  int* start;    // [N+1] bin start offsets; [N] = binned atoms
  int* cpart;    // [N / kScanChunk + 1] per-chunk counts
  int* acell;    // [N] bin id of the atom, -1: all-pairs
  int* aslot;    // [N] slot in the bin
  float4* cpos;  // [N] binned atoms bin by bin (x, y, z, j)
};

struct PairLists {
  const uint32_t* idxR;
  const int* cntR;
  const uint32_t* idxA;
  const int* cntA;
  int capR, capA;
};

// A packed atom (x, y, z, word): one 16-byte gather per neighbor.  The word
// holds the species in its low bits and whether the atom's radial or angular
// list overflowed its capacity.
constexpr uint32_t kAtomOverR = 1u << 8, kAtomOverA = 1u << 9;
__device__ __forceinline__ float atom_word(int type, int T, bool over_r, bool over_a) {
  const uint32_t t = (type >= 0 && type < T) ? (uint32_t)type : 0u;   // others are flagged
  return __uint_as_float(t | (over_r ? kAtomOverR : 0u) | (over_a ? kAtomOverA : 0u));
}

// Flags of a neighbor build in a launch that follows it: each of its blocks
// stores its own word and one block collects them (block 0 of the order
// launch, or of a small batch an extra block of the forward).  In a captured
// step that block also starts the replay's flag word and latches the step
// (graph_head's part), so the step needs no launch for that.
struct FlagArgs {
  const int* bflags;
  int n;       // 0: none
  int* flags;
  int* step;   // null outside a captured step
  int* cur;
};

struct FwdArgs {
  int N, Npad, H;
  float inv_rcR, inv_rcA;
  const int* order;
  const int* blist;   // launch order of the blocks
  int nch;
  const int* astruct;
  const float* box;
  const float* tilt;  // null: every cell orthorhombic
  const float4* p4;  // packed atoms
  PairLists nb;
  const float* cR;
  const float* cA;
  const float* nn;  // per species block of H*D + 2H + 1
  int nn_stride;
  float* G;        // [D][Npad] species order (may be null)
  float* Guser;    // [D][N] atom order (may be null)
  float* Sst;      // [Npad][NA*YR rounded up to 4] (may be null)
  float* FRst;     // [T*KR][Npad] radial sums F[J][k] (may be null)
  float* Ep;       // [D][Npad] (may be null)
  float* X;        // [H][Npad] (may be null)
  float* eatom;    // [N] atom order (may be null)
  float* eatom2;   // second copy for the caller (may be null)
  float* hrow;     // [N][T][KP] radial force coefficients (atom order)
  float* fA;       // [N][capA][3] angular pair forces
  int do_mlp, do_force;
  FlagArgs fl;
};

// Forces and per-atom virials from the forward's radial force coefficients
// and angular pair forces.
struct ForceArgs {
  int N;
  float inv_rcR;
  PairLists nb;
  const float4* p4;
  const int* astruct;
  const float* box;
  const float* tilt;  // null: every cell orthorhombic
  const float* hrow;  // [N][T][KP]
  const float* fA;    // [N][capA][3]
  float* F;           // [3][N]
  float* Fuser;       // second copy for the caller (may be null)
  float* wv;          // [6][N]
};

struct AdjArgs {
  int N, Npad, H, S;
  float inv_rcR, inv_rcA;
  const int* order;
  const int* blist;   // launch order of the blocks
  int nch;
  const int* astruct;
  const float* box;
  const float* tilt;  // null: every cell orthorhombic
  const float4* p4;   // packed atoms
  PairLists nb;
  const float* cR;
  const float* cA;
  const float* nn;
  int nn_stride;
  const float* Sst;   // [Npad][NA*YR rounded up to 4]
  const float* Ep;    // [D][Npad]
  const float* X;     // [H][Npad]
  const float* eps;   // [S] dL/dE(n)
  const float4* fb4;  // [N] dL/dF
  const float* wbar;  // [S][6] dL/dW(n)
  float* Gd;          // [D][Npad]
  float* FPst;        // [T*KR][Npad] tangent sums Fp[J][k]
  float* Gbr;         // [NR][Npad] Gbar of the radial descriptors
  float* beta;        // [H][Npad]
  float* part;        // [n_waves][PW] wave partial sums
  int PW;
};

// Kernels of the angular degrees l = 5..L3 (nep_highl.h)
struct HighArgs {
  int N, Npad, PW;
  float inv_rcA;
  const int* order;
  const int* astruct;
  const float* box;
  const float* tilt;
  const float4* p4;   // packed atoms
  PairLists nb;
  const float* cA;
  float* Sh;          // [Npad][YH][NA] sums S~ of the orthonormal harmonics
  float* Sdh;         // [Npad][YH][NA] their tangents
  float* G;           // [D][Npad] descriptor rows (q_nl of l > 4 written here)
  const float* Ep;    // [D][Npad] dE/dG
  float* Gd;          // [D][Npad] descriptor tangents
  const float* Gb;    // [D][Npad] Gbar (rows of l > 4)
  float* fA;          // [N][capA][3] angular pair forces (added to)
  const float4* fb4;  // [N] dL/dF
  const float* wbar;  // [S][6]
  float* part;        // [n_waves][PW] (c^A slots added to)
};

}  // namespace nep

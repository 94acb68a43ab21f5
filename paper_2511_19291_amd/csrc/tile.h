// tile.h -- several gates per sweep: program format and launcher shared by
// tile.cpp (host planner) and k_tile.hip (kernel). Not part of the public ABI.
//
// A tile is the 2^T amplitudes that differ only in T chosen qubits; one
// workgroup holds it in LDS and applies a list of gates before writing it
// back, so the state crosses HBM once per list instead of once per gate. A
// gate needs its non-diagonal targets inside the tile; controls and diagonal
// targets may be any qubit. The list is cut into rounds: in a round each
// thread holds the 2^R amplitudes that differ only in R "register" bits of
// the tile and applies every gate whose targets are among them; between
// rounds the tile is regrouped through LDS.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <type_traits>
#include <vector>

#include "sv_internal.h"

namespace sv {

constexpr int kTileMaxBits = 12;      // 2^12 complex64 = 32 KiB of LDS
constexpr int kTileRegBits = 4;       // widest register set
constexpr int kTileWords = 912;       // program words in the kernel arguments
constexpr int kTilePad = 48;          // words behind them that the kernel may read (one step, one line touch ahead)

// Gate kinds of the planner (matrix words: kMatFloats in tile.cpp).
enum TileKind : int {
    TK_DENSE = 0,      // 2 x 2 complex: 8 floats
    TK_REAL,           // 2 x 2 real: 4 floats
    TK_IMOFF,          // real diagonal, imaginary off-diagonal: 4 floats
    TK_DIAG1,          // phase by one bit: 4 floats
    TK_DIAG2,          // phase by two bits: 8 floats
    TK_ONES,           // phase where all fixed bits are 1: 2 floats
    TK_SIGN,           // sign flip where all fixed bits are 1: no matrix
    TK_DENSE2,         // 4 x 4 complex: 32 floats
    TK_MAP,            // X with at most one control, or SWAP: a linear map of the index
};

// Flags of a step's first word.
enum TileFlag : uint32_t {
    TF_LAYER = 1,      // uncontrolled gates of one kind, at most one on each register bit; with one of:
    TF_DENSE = 2,
    TF_REAL = 4,
    TF_IMOFF = 8,
    TF_DIAG = 16,
    TF_OTHER = 128,    // with one of:
    TF_SIGN = 2,       // without thread controls
    TF_PHASE = 4,
    TF_CTRL = 8,       // a controlled one-target matrix
    TF_DENSE2 = 16,
    TF_APPLY = 32,     // with SIGN: the last of consecutive ones
    TF_LANE_SIGN = 64, // with thread controls
    TF_DERIV = 1u << 28,   // adjoint: the step has derivatives
};

// Derivative of a gate (adjoint): of exp(-i theta P / 2), one value; of any
// other one-target gate, the eight parts of its pairs' correlation.
enum TileDeriv : int {
    TD_NONE = 0,
    TD_X = 1,
    TD_Y = 2,
    TD_Z = 4,
    TD_GENERAL = 8,
};

// Program: per round a record, then its steps, each a header of
// kTileHeadWords words; matrices follow the last round.
constexpr int kTileRoundWords = 12;   // multiples of four: read as 16-byte words
constexpr int kTileMapWords = 8;      // more of them when the round ends in an index map
constexpr int kTileHeadWords = 4;
// round record: [0] steps in the round | outer bits of the index map << 8 |
//   bit 16: the thread's own sign is used | 17: its own phase | 18: the round
//   ends in an index map | thread steps, which stand before the others, << 24; [1..4] swizzled LDS column of each thread bit (two
//   16-bit columns a word); [5..6] columns of the register bits; [7] tile bit
//   of each thread bit (4 bits each); [8], [9] columns and tile bits of the
//   ninth and tenth thread bit (two register bits). Index map: [12..16] LDS
//   column that each thread bit is written to, [17..18] each register bit,
//   [19] constant; then, in groups of four, a word per outer bit: bit of the
//   tile's index | column << 16.
// layer header: [0] flags | register bits with a gate << 8; [1] their
//   matrices, in units of four words, << 8 * bit; [2] words between rows'
//   matrices
// other headers (thread steps: SIGN or PHASE): [0] flags | register control
//   mask << 8 | thread controls << 16 (tile bits); [1] outer controls (bits of
//   the tile's index); [2] first matrix word | words between rows' matrices
//   << 16; [3] SIGN: a bit for each register amplitude to flip; PHASE: free bits: position 0 | position 1 << 8 | their number
//   << 16 | places << 20, 22; CTRL: the target's register bit as a mask;
//   DENSE2: 1 << the pair's place in (1,0) (2,0) (2,1) (3,0) (3,1) (3,2)
// with TF_DERIV (layers, CTRL): [3] |= TileDeriv of the gate on register bit b
//   << 8 + 4 b; the values follow each other in the order of the bits
constexpr int kPlaceReg = 0, kPlaceThread = 1, kPlaceOuter = 2;

struct TileArgs {
    float2* p0;
    float2* p1;
    uint64_t N;
    int nrow0;
    int row0;                         // first row of this launch
    int T;
    int nrounds;
    int nwords;                       // words in use
    uint8_t pos[kTileMaxBits];        // tile qubits, ascending
    alignas(16) uint32_t words[kTileWords + kTilePad];   // read 16 bytes at a time
};
static_assert(sizeof(TileArgs) <= 4096 - 128, "kernel arguments stay within 4 KiB");
static_assert(offsetof(TileArgs, words) % 16 == 0, "a program starts at a 16-byte word");

// Swizzle of a tile index into its LDS element: tile bit b >= 4 also flips
// the low four bits by kTileSwz[b - 4]. The columns of the twelve bits in the
// low four positions are twelve different nonzero vectors of GF(2)^4; a
// hyperplane holds only seven, so whichever four bits are the register bits,
// the other eight span the bank index, and four of them, taken as the lowest
// lane bits, reach 16 different 8-byte banks.
constexpr uint32_t kTileSwz[8] = {3, 5, 9, 6, 10, 12, 7, 11};

void launch_tile(const TileArgs& a, int rows, int reg_bits, hipStream_t st);

// The adjoint: of a state of at most kTileMaxBits qubits (a tile per row), or
// one sweep of a larger one (kTileMaxBits qubits a tile).
constexpr int kAdjValues = 256;       // derivative values of a launch
constexpr int kAdjTileValues = 128;   // of a launch over several tiles: two workgroups' LDS in a compute unit
struct TileAdjArgs {
    float2* psi;
    float2* lam;
    const double* coeff;              // NULL: lambda is loaded; else lambda = sum_q coeff[row][q] Z_q psi
    double* out;                      // one tile: per row the values, then loss, drift; several: [rows][nvalues][grid]
    uint64_t N;
    int64_t out_stride;
    int coeff_stride;
    int row0;
    int T;
    int nrounds;
    int nwords;
    int value0;                       // first value of this launch
    int nvalues;
    int first, last;                  // writes the loss, the drift
    uint8_t pos[kTileMaxBits];        // tile qubits, ascending
    alignas(16) uint32_t words[kTileWords + kTilePad];   // read 16 bytes at a time
};
static_assert(sizeof(TileAdjArgs) <= 4096 - 128, "kernel arguments stay within 4 KiB");
static_assert(offsetof(TileAdjArgs, words) % 16 == 0, "a program starts at a 16-byte word");
void launch_tile_adj(const TileAdjArgs& a, int grid, int rows, hipStream_t st);

// Pauli strings whose x bits lie in one tile (k_pauli.hip). Words: per
// distinct x and part [0] x (tile bits) | 1 << 12: the products' imaginary
// part | strings << 16, then per string [0] a bit with odd z for each product
// of a thread (16, with x 8) | z on the thread bits << 16 | 1 << 29: minus, [1] z
// on the tile's index. The tile's bits but x's top one number the products:
// the thread's bits, then the product's.
constexpr int kPauliTerms = 256;      // strings of a launch
struct PauliTileArgs {
    const float2* p0;
    const float2* p1;
    uint64_t N;
    double* part;                     // [rows][nterms][grid]
    int nrow0;
    int T;
    int ngroups;
    int nterms;
    uint8_t pos[kTileMaxBits];
    uint32_t words[3 * kPauliTerms];
};
static_assert(sizeof(PauliTileArgs) <= 4096 - 128, "kernel arguments stay within 4 KiB");
int pauli_tile_grid(int n, int T, int rows);
// out: [rows][nterms]
void launch_pauli_tile(const PauliTileArgs& a, int rows, double* out, hipStream_t st);

// Strings (x, z) for every row, grouped into sweeps: out receives rows *
// (strings of the sweep) doubles per sweep, `order` the strings in that
// order, one list per sweep. Strings it leaves out (more x bits than a tile
// holds, or better off in sweeps by x) are in `rest`.
struct PauliSweep {
    PauliTileArgs args;
    std::vector<int> terms;
};
bool pauli_tile_applies(int n);
void plan_pauli_tiles(int n, int rows, const uint64_t* x, const uint64_t* z, int count, std::vector<PauliSweep>& sweeps,
                      std::vector<int>& rest);

// One gate as the planner sees it. Fixed qubits (`nc` of them) must be 1 for
// the gate to act: the controls, and the targets of a phase on the all-ones
// pattern.
struct TileGate {
    int kind;                         // TileKind
    int k;                            // targets (none for TK_ONES, TK_SIGN)
    int targets[2];
    int nc;
    int controls[SV_MAX_CONTROLS + 2];
    size_t mat;                       // first float of row 0's matrix in the pool
    bool per_row;                     // one matrix per row, one after the other
    int deriv;                        // TileDeriv
    int op;                           // the caller's index of the gate
};

// Gates to apply, and their matrices (complex64 parts as floats).
struct TileList {
    std::vector<TileGate> gates;
    std::vector<float> pool;
    double drift = 0.0;               // of the norm by the matrices' rounding (logarithm)
    std::vector<double> row_drift;    // by each row's own matrices
};

// Append (matrices, targets, controls): `ms` holds nm matrices of 4^k entries
// (nm = 1, or one per row). Nothing is appended when all are the identity and
// there is no derivative.
void tile_append(TileList& l, int k, const int* targets, int nc, const int* controls, const cd* ms, int nm, int op,
                 int deriv = TD_NONE);

// Whether `count` gates of the list (gates[0..], NULL: the first ones) go faster
// by sweeps of their own than in one sweep of tiles.
bool tile_apart(const TileList& l, const int* gates, int count, int n, int rows);

// Row r's matrix of a gate as its program holds it (scaled and rounded): 2^k x
// 2^k entries by the gate's targets (one entry without any).
void tile_matrix(const TileList& l, const TileGate& g, int r, cd* m);

// Apply the list to every row, asynchronously on `st`. Gates that a sweep of
// their own serves better are handed to one_gate(gate), or one_gate(op). Returns
// the number of launches over the state (a row's, where rows take several).
template <class F>
int tile_run(const Rows& rows, int n, const TileList& l, hipStream_t st, const F& one_gate);

bool tile_applies(int n);

struct TilePlanner;                   // tile.cpp
struct TileSweep {
    std::vector<int> gates;           // in an order that equals the list's
    uint64_t qubits;                  // the tile's
    bool single;                      // apply its gates by sweeps of their own
};
// The next sweep of the list; empty when every gate is placed.
struct TilePlannerHandle {
    TilePlanner* p;
    TilePlannerHandle(const TileList& l, int n, int rows);
    ~TilePlannerHandle();
    TilePlannerHandle(const TilePlannerHandle&) = delete;
    TilePlannerHandle& operator=(const TilePlannerHandle&) = delete;
    bool next(TileSweep& s);
};
// (returns its launches: a program longer than the kernel arguments takes more)
int tile_sweep(const Rows& rows, int n, const TileList& l, const TileSweep& s, hipStream_t st);

// The adjoint of a list (the circuit's U^* from last to first, derivatives
// marked) on states of 4..12 qubits: queues the launches that write every
// row's values, loss and drift to out. `order` receives the gates (positions
// in the list) whose values follow each other.
bool tile_adjoint_applies(int n);
int tile_values(const TileList& l);
void tile_adjoint(float2* psi, float2* lam, int n, int rows, const TileList& l, const double* coeff, int coeff_stride,
                  double* out, std::vector<int>& order, hipStream_t st);

// One sweep of the adjoint of a larger state: part (tile_adjoint_parts
// doubles) is its workspace. Every launch appends its values, [rows][nvalues]
// doubles at `out`, to `values`.
struct TileValues {
    int row0, rows, nvalues;
    uint64_t at;                      // first double, from `out`
    std::vector<int> gates;           // whose values follow each other
};
uint64_t tile_adjoint_parts(int rows);
void tile_adjoint_sweep(float2* psi, float2* lam, int n, int rows, const TileList& l, const TileSweep& s, double* part,
                        double* out, std::vector<TileValues>& values, hipStream_t st);

template <class F>
int tile_run(const Rows& rows, int n, const TileList& l, hipStream_t st, const F& one_gate)
{
    auto one = [&](const TileGate& g) {
        if constexpr (std::is_invocable_v<F, const TileGate&>) one_gate(g);
        else one_gate(g.op);
    };
    // a few gates: what the planner would find, without its 0.5 us
    if (l.gates.size() <= 3 && tile_apart(l, nullptr, (int)l.gates.size(), n, rows.nrows)) {
        for (const TileGate& g : l.gates) one(g);
        return (int)l.gates.size();
    }
    TilePlannerHandle plan(l, n, rows.nrows);
    TileSweep s;
    int launches = 0;
    while (plan.next(s)) {
        if (s.single) {
            for (int g : s.gates) one(l.gates[g]);
            launches += (int)s.gates.size();
        } else {
            launches += tile_sweep(rows, n, l, s, st);
        }
    }
    return launches;
}

}  // namespace sv

// Host-side circuit object and gate-fusion planner (internal).
#pragma once

#include <complex>
#include <cstdint>
#include <vector>

#include "../../include/qs.h"

namespace qs {

using cd = std::complex<double>;

// One gate: qubits[j] is bit j of the row/column index of the 2^k matrix.
struct Gate {
  int k = 0;
  int q[QS_MAX_FUSED] = {0};
  std::vector<cd> m;  // 2^k x 2^k row-major
};

// A fused block: the product of its gates, on `k` qubits (ascending).
struct Block {
  int k = 0;
  int q[QS_MAX_FUSED] = {0};
  int ngates = 0;
  std::vector<cd> m;
};

// Matrix of a named gate kind (QS_GATE_*) with its parameters; false for an
// unknown kind or a wrong qubit count.
bool gate_matrix(int kind, int nq, const double* params, std::vector<cd>* m, int* k_out);

// Greedy fusion: gates in order; open blocks on disjoint qubit sets; a gate
// joins (and merges) the open blocks it touches when the union has at most
// kmax qubits, else those blocks are emitted and the gate opens a new one.
// Blocks are emitted in an order that keeps every qubit's gates in order.
std::vector<Block> fuse(const std::vector<Gate>& gates, int n, int kmax);

// ---- tile passes
// A pass loads a tile of 2^(C+H) amplitudes: the contiguous low bits [0, C)
// and H chosen bits (rows), runs rounds of gates on it and stores it back,
// one HBM read and write for every gate it holds. A round gathers, per
// thread, the 2^W amplitudes that differ in W tile bits and applies the
// round's one- and two-qubit gates to them in registers.
struct TileGate {
  int kind = 1;      // 1: one-qubit (j1); 2: two-qubit (row bit 0 = j1, bit 1 = j2)
  int j1 = 0, j2 = 0;
  size_t mat = 0;    // offset of the matrix in TilePlan::mats (complex entries)
};
// What the rounds of a pass hold: gates of one or two qubits on any of the
// round's bits (kSparse); one or two gates on disjoint pairs, the first on the
// round's bits 0 and 1, the second on 2 and 3 (kPairs); one dense product of
// gates of at most W qubits (kDense). A pair round's numbers (TilePlan::reals)
// are its gates' 4 x 4 complex matrices (32 reals each, row-major).
enum class TileMode { kSparse, kPairs, kDense };
// The forms a plan may use; where there are two, each pass takes the cheaper.
enum class TileForms {
  kSparse,       // complex64 off the matrix cores; runs of one-qubit gates
  kPairs,        // states below a tile, batches
  kDense,        // complex64 batches
  kPairsDense,   // complex64 on the matrix cores
  kPairsSparse,  // complex128
};
struct TileRound {
  TileMode mode = TileMode::kSparse;
  int bits[4] = {0, 0, 0, 0};  // tile bits of the round, ascending (pairs: the
                               // first gate's two, then the second's)
  int g0 = 0, ng = 0;          // its gates in TilePlan::gates (sparse); pairs: 1 or 2 gates
  size_t mat = 0;              // dense: offset of the 16x16 product in mats; pairs: in reals
};
struct TileStep {
  bool block = false;  // a dense block (a gate on more than two qubits), not a pass
  TileMode mode = TileMode::kSparse;  // pass: of its rounds
  int hb[7] = {0, 0, 0, 0, 0, 0, 0};  // pass: tile row bits, ascending
  int r0 = 0, nr = 0;  // pass: its rounds in TilePlan::rounds
  int ngates = 0;      // pass: gates applied; block: 1
  Block blk;           // block step, on physical bits
  size_t mat = 0;      // block step: offset of its matrix
};
struct TilePlan {
  int C = 0, H = 0, W = 0;
  TileForms forms = TileForms::kSparse;
  std::vector<TileStep> steps;
  std::vector<TileRound> rounds;
  std::vector<TileGate> gates;
  std::vector<cd> mats;
  std::vector<double> reals;  // pair rounds
  // what the passes that could take pair rounds cost so and in the other form
  // (the same units, per tile), where both were asked for
  double pair_cost = 0, group_cost = 0;
  int passes() const {
    int p = 0;
    for (const auto& s : steps) p += s.block ? 0 : 1;
    return p;
  }
};

// Plans `gates` (on physical bits, in circuit order) into tile passes for a
// state of n >= C + H qubits. One-qubit gates are first multiplied into wider
// neighbours. A pass takes every gate the dependence order lets it run inside
// the low bits plus at most H other bits, which are chosen to let many gates
// run (PassPicker in circuit.cpp). Within a pass, sparse and dense rounds are
// formed greedily, W bits each; pair rounds take the two ready gates with the
// longest chains of gates behind them; a pass takes the form whose rounds cost
// less (RoundCost in circuit.cpp). Gates too wide for a round (more than
// two qubits, or more than W for dense rounds) run as blocks between passes.
// dense_price: also what dense rounds would cost where forms is kPairs.
TilePlan plan_tiles(const std::vector<Gate>& gates, int n, int C, int H, int W, TileForms forms,
                    bool dense_price = false);

// Whether every gate has one or two qubits.
bool narrow_gates(const std::vector<Gate>& gates);
// Of a list of such gates: how many are left when merged as plan_tiles does
// (one-qubit gates that stay count half). Without any matrix.
double merged_gates(const std::vector<Gate>& gates, int n);
// The widths of the blocks that fuse() makes, about in their order. Without any
// matrix.
std::vector<int> block_widths(const std::vector<Gate>& gates, int n, int kmax);
// The product of all gates as one block on qubits 0 .. n - 1 (n <= QS_MAX_FUSED).
Block whole_block(const std::vector<Gate>& gates, int n);

// The device tables of a plan, as one byte image: per round an int4 {bits
// packed by byte, first gate (sparse) or operand offset in floats (dense),
// gate count, 0}, or for pairs {bits packed by byte, the same bits ascending,
// offset of its numbers, 1 if it has a second gate}; at `gates` per gate
// (sparse) an int2 {kind | j1 << 4 | j2 << 8, offset of its matrix in reals};
// at `ops` the dense rounds' matrix-core operands (embed_round); at `mats` the
// plan's matrices (float or double pairs); at `reals` the pair rounds' numbers.
// Offsets are bytes from the start.
struct TileOffsets {
  size_t gates = 0, ops = 0, mats = 0, reals = 0;
};
void tile_tables(const TilePlan& pl, bool c64, std::vector<unsigned char>* out, TileOffsets* at);

// The pair rounds' numbers (TilePlan::reals) in FP32. Each gate's matrix is
// scaled, before the cast, by what the casts so far have changed its
// predecessors' norms by, which bounds the change of the state's norm: the
// casts of equal gates are equally off, and those of a Fourier circuit of 10
// qubits run six times took 1.8e-6 off it, ten times what all roundings of the
// amplitudes make.
std::vector<float> float_pairs(const TilePlan& pl);

// A pair round's table entry (int4 as above), its numbers moved by `base`.
void pair_round_entry(const TileRound& r, size_t base, int32_t row[4]);

// The operands a dense matrix-core round reads, for the three real products of
// Re U X_r, Im U X_i and (Re U + Im U)(X_r + X_i) of a 16 x 16 complex round
// matrix u (16 x 16 x 4 MFMA A-operand layout): out[(3 s + c) * 64 + lane] =
// W_c[lane % 16][4 s + lane / 16] with W_0 = Re U, W_1 = Im U,
// W_2 = Re U + Im U (summed in float64), s = 0 .. 3.
void embed_round(const cd* u, float* out);

// Fuse a circuit's gates into blocks of at most kmax qubits (0 = 5) without
// recording a choice of run mode (internal planning; qs_circuit_plan does
// record it).
int circuit_plan_blocks(qs_circuit* c, int kmax);
// As if circuit_plan_blocks had been called with this valid width, but leaves
// the work until someone asks for the blocks (circuit_blocks_due does it).
void circuit_plan_blocks_later(qs_circuit* c, int kmax);
void circuit_blocks_due(const qs_circuit* c);

}  // namespace qs

struct qs_circuit {
  int n = 0;
  uint64_t generation = 0;      // bumped whenever the gate list changes
  std::vector<qs::Gate> gates;  // on virtual positions (SWAPs already folded)
  std::vector<int> pos;         // logical qubit -> virtual position after all SWAPs
  int kmax = 5;
  bool planned = false;
  bool due = false;             // blocks of at most kmax qubits are due, not made yet
  std::vector<qs::Block> blocks;
  // device copies of the block matrices, per precision (owned)
  void* dmat[2] = {nullptr, nullptr};
  std::vector<size_t> off[2];   // element offset of each block's matrix
  // tile passes (dense runs), planned per precision and physical labelling:
  // 1 on, 0 off (qs_circuit_use_tiles(c, 0), or blocks planned with
  // qs_circuit_plan before any choice), -1 not chosen (on)
  int tiles = -1;
  struct TileCache {
    std::vector<int> key;  // physical bit of every virtual position
    qs::TilePlan plan;
    void* dev = nullptr;   // rounds, gates, matrices (owned)
    qs::TileOffsets at;
  } tcache[2];
  // runs on states below a tile: how (decided once per precision and block
  // width) and the tables, on virtual positions, whatever the state's labels
  enum WholeForm { kUndecided, kBlocks, kRounds, kMatrix };
  struct WholeCache {
    WholeForm form = kUndecided;
    int kmax = 0;          // block width the decision was made for
    void* dev = nullptr;   // rounds and their numbers, or the matrix (owned)
    int nrounds = 0;
    size_t num = 0;        // byte offset of the rounds' numbers
  } whole[2];
  // host plan for batched runs (identity labelling), and what its passes cost
  // in pair and in dense rounds once that was asked for; cleared with the other
  // plans when the circuit changes
  bool bplan_ok = false, bcost_ok = false;
  qs::TilePlan bplan;
  double bcost[2] = {0, 0};
};

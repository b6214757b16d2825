// Passes of gates over tiles held in registers: what the planner (passes.cpp)
// hands to the kernel (tile.hip).
#pragma once

#include <cstddef>
#include <cstdint>
#include <vector>

struct qs_state;
struct qs_circuit;

namespace qs {

constexpr int kTileBitsMin = 10, kTileBitsMax = 12;   // qubits of a tile

// A pass in the word stream: per stage three words of layout, then its
// operations.
//   word 0: tile bit of thread bit i at 4i (i < T - 4), then of register
//           bit b at 4(T - 4 + b)
//   word 1: state bit of thread bit i at 6i
//   word 2: state bit of register bit b at 6b, operation count at bit 32
// An operation's first word holds its kind in bits 0-2, a register bit or
// pair of them in bits 3-5, and its length in words from bit 32. The kernel
// reads kTileAhead words at the start of every operation, so the stream ends
// with as many unused ones.
enum TileOp {
    kTileDense1 = 0,    // matrix (8 doubles)
    kTileCDense1 = 1,   // register mask at bit 8; index mask, index values, matrix
    kTileX = 2,         // register mask at bit 8; index mask, index values
    kTileDense2 = 3,    // matrix (32 doubles)
    kTileRotate = 4,    // real matrix (4 doubles)
    kTileDiag = 5,      // bit 6: a table of 16 phases first; at bit 8 the number of sign blocks (each two
                        // times index mask, index values, register mask), at bit 20 that of phase groups
                        // (register mask | terms << 16, first phase; per term: index mask, index values,
                        // phase). A phase is 2 doubles.
};
constexpr int kTileAhead = 8;
constexpr int kTileSigns = 2;   // signs in a block

struct TilePass {
    int T = 0;
    int pos[kTileBitsMax] = {0};   // the tile's qubits, ascending
    int n_stages = 0;
    size_t word0 = 0;              // first word in the stream
};

// A circuit as passes; gates that fit none (uncontrolled gates on three or
// more qubits, and controlled ones on two or more, that are not diagonal)
// are steps of their own.
struct TileStep {
    int pass = -1;                 // index into passes, or
    int gate = -1;                 // index of a gate swept by itself
};
struct TilePlan {
    std::vector<TilePass> passes;
    std::vector<TileStep> steps;
    std::vector<uint64_t> words;
    double cost = 0;               // estimated time in microseconds
    int n_stages = 0;
    int ops[6] = {0};              // operations by TileOp
};

// Estimated times of a dense and of a diagonal block, in microseconds.
double dense_us(int n, size_t amp_bytes, int k);
double diagonal_us(int n, size_t amp_bytes);

// False where no plan is made: states smaller than a tile, or a cost of
// `limit` or more (planning stops there).
bool plan_tiles(int n, size_t amp_bytes, const qs_circuit *c, double limit, TilePlan &out);

int launch_tile_pass(qs_state *h, const TilePass &p, const uint64_t *dwords);

}  // namespace qs

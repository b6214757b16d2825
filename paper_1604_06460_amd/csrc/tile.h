// Passes of gates over tiles held in registers: what the planner (passes.cpp)
// hands to the kernel (tile.hip).
#pragma once

#include <cstddef>
#include <cstdint>
#include <vector>

struct qs_state;
struct qs_circuit;

namespace qs {

constexpr int kTileBitsMin = 10, kTileBitsMax = 13;   // qubits of a tile

// A pass in the word stream: per stage three words of layout, then its
// operations.
//   word 0: tile bit of thread bit i at 4i (i < T - 4), then of register
//           bit b at 4(T - 4 + b)
//   word 1: state bit of thread bit i at 6i
//   word 2: state bit of register bit b at 6b, operation count at bit 32
// An operation's first word holds its kind in the low byte:
enum TileOp {
    kTileDense1 = 0,    // | register bit << 8; matrix (8 doubles)
    kTileCDense1 = 1,   // | register bit << 8 | register mask << 16; index mask, index values, matrix
    kTileX = 2,         // | register bit << 8 | register mask << 16; index mask, index values
    kTileDense2 = 3,    // | pair << 8; matrix (32 doubles)
    kTileRotate = 4,    // | register bit << 8; real matrix (4 doubles)
    kTileDiag = 5,      // | signs << 8 | groups << 24 | union of the signs' register masks << 40 | table << 56;
                        // with a table: 16 phases; per sign: index mask, index values, register mask; per
                        // group: register mask | terms << 16, first phase, per term: index mask, index
                        // values, phase (a phase: 2 doubles)
};

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
    double cost = 0;               // estimated time, in sweeps over the state
};

double dense_cost(size_t amp_bytes, int k);

// False where no plan is made (states smaller than a tile).
bool plan_tiles(int n, size_t amp_bytes, const qs_circuit *c, TilePlan &out);

int launch_tile_pass(qs_state *h, const TilePass &p, const uint64_t *dwords);

}  // namespace qs

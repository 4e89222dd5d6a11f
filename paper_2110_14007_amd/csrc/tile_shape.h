// Launch shapes of the LDS-list tile kernel (tile.h), shared by the kernel's
// launcher and the planner.
#pragma once

#include <stddef.h>

namespace tod {
namespace tile {

constexpr int kQH = 16;       // queue slots per (query, half-wave)
constexpr int kQ = 2 * kQH;   // queue slots per query

// Waves (of 32 queries) per workgroup.
constexpr int tile_waves(int kp) { return kp <= 32 ? 4 : kp == 64 ? 2 : 1; }

__host__ __device__ constexpr int row_bytes(int dpad, int es) { return dpad * es + 16; }

// Rows longer than the register-operand shapes are staged in column slabs of
// kSlabBytes per row (32 rows per slab), so LDS use does not grow with d:
// at most 33 KiB of slab plus the lists (K' = 256: 72 KiB) per workgroup.
constexpr int kSlabBytes = 1024;

// LDS bytes of the tile kernel for these parameters (host and device agree).
// dbuf: the double-buffered whole-row staging of the register-operand shapes.
__host__ __device__ constexpr size_t lds_bytes(int dpad, int es, int kp, int w, bool dbuf) {
  return (dbuf ? (size_t)2 * 32 * row_bytes(dpad, es) : (size_t)32 * (kSlabBytes + 16)) + 256 +
         (size_t)w * 32 * (kp + kQ) * sizeof(uint64_t);
}

}  // namespace tile
}  // namespace tod

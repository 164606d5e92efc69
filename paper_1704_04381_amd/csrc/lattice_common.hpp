// Shared pieces of the simple cubic growth kernels: byte words, the pair
// test and the canonical move tables.
//
// Byte words.  Coordinates sit in bytes 0..2 as x + 128, y + 128, z + 128.
//   tip word     T = coordinates | (Q mod 256) << 24,  Q = x + 2y + 3z
//   history word w = coordinates | 1 << (24 + Q mod 8)
// The six neighbours of a site differ from it by dQ = -3, -2, -1, 1, 2, 3
// (-z, -y, -x, +x, +y, +z), six distinct residues mod 8, so one bit of byte 3
// names the direction of an occupied neighbour.
//
// Pair test, two operations per earlier monomer of the parity that can touch
// the tip (the cubic lattice is bipartite, so the L1 distance is odd):
//   v    = v_msad_u8(w, T & 0xFFFFFF, -2)   L1 distance - 2: all ones iff w is
//          a neighbour of the tip, else a small positive number (below 2^10:
//          byte 3 of the reference is zero, which masks byte 3 of w)
//   acc |= w & v                            (one v_bitop3)
// Only the top byte of acc is used: the bits Q_j mod 8 of the occupied
// neighbours.  Rotating that byte right by Q_t mod 8 puts direction dQ at bit
// dQ mod 8 (z+ y+ x+ at 3 2 1, x- y- z- at 7 6 5).  The earlier word kept
// Q mod 256 in the low byte and formed 1 << (Q_j - Q_t + 3) per pair: four
// operations (msad, saturating subtract, subtract, shift-or).
//
// Free candidates are numbered in the canonical order -z, -y, -x, +x, +y, +z.
#pragma once

#include "rsaw_device.hpp"

namespace rsaw {

constexpr uint32_t kByteOrigin = 0x00808080u;  // tip word of the origin, Q = 0
constexpr uint32_t kByteCoords = 0x00FFFFFFu;
constexpr uint32_t kByteDirs = 0xEEu;          // bits dQ mod 8 of the six directions

// History word of a tip word.
__device__ __forceinline__ uint32_t byte_history(uint32_t tip)
{
    return (0x01000000u << __builtin_amdgcn_ubfe(tip, 24u, 3u)) | (tip & kByteCoords);
}

// acc | (w & v) with v the pair test above; tref = tip & 0xFFFFFF.
__device__ __forceinline__ uint32_t byte_pair(uint32_t acc, uint32_t w, uint32_t tref)
{
    const uint32_t v = __builtin_amdgcn_msad_u8(w, tref, 0xFFFFFFFEu);
    return __builtin_amdgcn_bitop3_b32(acc, w, v, 0xF8); // acc | (w & v)
}

// Free directions (bits of kByteDirs) from the accumulated pair tests: the
// top byte copied to all four and rotated right by Q_t (mod 32, the copies
// make it mod 8); zero where alive = 0 (all ones for a growing chain).
__device__ __forceinline__ uint32_t byte_free(uint32_t acc, uint32_t tip, uint32_t alive)
{
    const uint32_t o = __builtin_amdgcn_perm(acc, acc, 0x07070707u);
    const uint32_t rot = __builtin_amdgcn_alignbit(o, o, tip >> 24);
    return __builtin_amdgcn_bitop3_b32(rot, kByteDirs, alive, 0x08); // ~rot & dirs & alive
}

// Table entry for (free << 2) | r: the tip-word increment of the move to the
// r-th free candidate (coordinate delta, plus dQ in byte 3), one addition
// that neither carries nor borrows across a coordinate byte within
// [-127, 127]; zero for an empty mask, so that a dead chain stays.
__device__ __forceinline__ uint32_t byte_move(uint32_t idx)
{
    const uint32_t mask = (idx >> 2) & kByteDirs, r = idx & 7u;
    uint32_t seen = 0;
    for (int dq = -3; dq <= 3; ++dq) {
        if (dq == 0 || !((mask >> (dq & 7)) & 1u)) continue;
        if (seen == r) {
            const int axis = (dq < 0 ? -dq : dq) - 1; // 0 = x, 1 = y, 2 = z
            const int32_t d = (int32_t)(1u << (8 * axis));
            return (uint32_t)(dq < 0 ? -d : d) + ((uint32_t)dq << 24);
        }
        ++seen;
    }
    return 0;
}

constexpr int kByteLutSize = 120 * 8; // (free << 2) | r, free up to 0xEE

// Wide words: candidate codes c = 0..6 without 3 stand for dQ = c - 3.
// LUT[mask * 8 + r]: dQ of the r-th free candidate of the 7-bit mask.
__device__ __forceinline__ int lattice_dq(uint32_t idx)
{
    const uint32_t mask = idx >> 3, r = idx & 7u;
    uint32_t seen = 0;
    for (uint32_t c = 0; c < 7; ++c) {
        if (c == 3 || !((mask >> c) & 1u)) continue;
        if (seen == r) return (int)c - 3;
        ++seen;
    }
    return 0;
}

constexpr int kLutSize = 120 * 8; // masks up to 0x77

} // namespace rsaw

// Geometry shared by the kernels and by the host-side layout arithmetic (no HIP types here, so
// that the host logic also compiles with a plain C++ compiler).
//   group      = 4 consecutive coordinates (one 128-bit access, one Philox4x32 block)
//   tile       = 64 groups = 256 consecutive coordinates = what one wavefront handles at a time
//   superblock = 512 tiles: one workgroup of the passes that find where the tiles' lines start in a ring slot; a
//                tile's word is its offset inside the superblock, and each superblock has a base
//   strip      = 64 lanes x 32 consecutive coordinates = 8 tiles: what one wavefront hashes at a time
//                where only the subset matters (one 32-bit mask per lane, in coordinate order)
//   line       = 128 bytes = 32 floats, the unit in which memory is read (written: half a line)
//   block      = up to 8 replicas whose sparse values sit side by side in memory
#pragma once
#include <stdint.h>

namespace am {

constexpr uint32_t kTileCoords = 256;
constexpr uint32_t kTilesPerSuperblock = 512;
constexpr uint32_t kStripCoords = 2048;
constexpr uint32_t kStripsPerSuperblock = kTileCoords * kTilesPerSuperblock / kStripCoords;
constexpr uint32_t kLineFloats = 32;
constexpr uint32_t kStageFloats = 256;      // ring values of a block (and EMA entries) the averaging-only kernel stages at a time
constexpr uint32_t kLdsBytes = 160 * 1024, kLdsGranule = 1280;      // of a compute unit
constexpr uint32_t kMaxReplicas = 32;
constexpr uint32_t kMaxBlockReplicas = 8;
// Tiles whose replicas follow each other in the step by one-wave workgroups; a multiple of the XCDs.  us a step by their number, nine waves a compute unit: interleaved 125.8M x 8 64: 5804, 128: 5626, 192: 5750, 256: 5799, 512: 5731,
// 31.5M 1433, 1409, 1441, 1426, 1436; per replica 125.8M, eight waves, 64: 6332, 128: 6278, 256: 6355, 512: 6457.
constexpr uint32_t kWaveChunk = 128;

}  // namespace am

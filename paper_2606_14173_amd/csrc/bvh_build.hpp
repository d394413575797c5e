// Host BVH builder interface.
#pragma once
#include <cstdint>
#include <vector>

namespace hpt {

constexpr uint32_t kBvhDepthMax = 64;   // traversal stack entries
constexpr uint32_t kBvhTopNodes = 320;  // nodes stored first, in breadth-first order from the root
// Least direction component of the slab tests: its reciprocal times a coordinate
// is finite up to 1e20 (1e-30 lost rays along the axes beyond 3e8), and times
// the margin of a packed box, 2^-21 of the largest coordinate, still 4e11
// times that coordinate, farther than any ray is followed.
constexpr float kSlabMin = 1e-18f;

struct BvhResult {
  std::vector<float> nodes;   // 16 floats per node
  std::vector<float> prims;   // 12 floats per primitive, leaf order
  uint32_t n_nodes = 0, max_depth = 0;
  float bounds[6] = {0, 0, 0, 0, 0, 0};
  double build_ms = 0.0;
};

// Build over spheres [0, n_sph) then triangles [n_sph, n_sph + n_tri)
// (global ids). Returns false if the input is empty, too large, or the
// tree is deeper than the traversal stack.
bool build_bvh(const float *tri, uint32_t n_tri, const float *sph, uint32_t n_sph, BvhResult &out);

// The nodes as the traversal reads them, 12 words (48 bytes) each: origin xyz
// (float) and link 0; the planes of both child boxes as pairs of binary16
// offsets from the origin (child 0: lo.x hi.x, lo.y hi.y, lo.z hi.z, then child
// 1), rounded outwards; link 1; unused. Origin and offsets are in units of 1 /
// scale, a power of two for which every offset is below 2^15. The traversal is
// bound by vector-L1 accesses (one per lane and load) and by vector
// instructions: such a node takes three loads instead of four, and a fused
// multiply-add reads a binary16 offset for nothing.
struct PackedNodes {
  std::vector<uint32_t> words;
  float scale = 1.f;
};
void pack_nodes(const BvhResult &bvh, PackedNodes &out);

}  // namespace hpt

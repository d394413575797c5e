// Rays along the axes through the packed BVH nodes, in the slab test's own FP32
// arithmetic: the leaf of every triangle that a ray meets has to be visited,
// however large the scene's coordinates. Usage: prog size shift
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

#include "../../paper_2606_14173_amd/csrc/bvh_build.hpp"

static float half_value(uint32_t h) {
  const int e = h >> 10 & 31, m = h & 1023;
  const float v = e == 31 ? INFINITY : e ? std::ldexp((float)(1024 + m), e - 25) : std::ldexp((float)m, -24);
  return h >> 15 & 1 ? -v : v;
}

int main(int argc, char **argv) {
  if (argc < 3) return 2;
  const double size = std::atof(argv[1]), shift = std::atof(argv[2]);
  std::mt19937 g(11);
  std::uniform_real_distribution<double> U(-1.0, 1.0);
  const uint32_t n = 600;
  std::vector<float> tri;
  for (uint32_t i = 0; i < n; ++i) {   // every fourth lies in an axis plane
    const double c[3] = {U(g), U(g), U(g)};
    for (int v = 0; v < 3; ++v)
      for (uint32_t a = 0; a < 3; ++a)
        tri.push_back((float)(size * (c[a] + (i % 4 == 0 && a == i / 4 % 3 ? 0.0 : 0.2 * U(g))) + shift));
  }
  hpt::BvhResult b;
  if (!hpt::build_bvh(tri.data(), n, nullptr, 0, b)) return 3;
  hpt::PackedNodes pk;
  hpt::pack_nodes(b, pk);
  long meets = 0, lost = 0;
  for (int k = 0; k < 20000; ++k) {
    const int axis = k % 3, u = (axis + 1) % 3, v = (axis + 2) % 3;
    const double s = k % 2 ? 1.0 : -1.0;
    float o[3], d[3] = {0.f, k % 4 < 2 ? 0.f : -0.f, 0.f}, inv[3], oi[3];
    const float *t = &tri[9 * (g() % n)];
    for (int a = 0; a < 3; ++a) o[a] = (float)(0.2 * t[a] + 0.3 * t[3 + a] + 0.5 * t[6 + a]);
    o[axis] = (float)(shift - s * size * (2.0 + U(g)));
    d[axis] = (float)s;
    for (int a = 0; a < 3; ++a) {
      inv[a] = 1.0f / (std::fabs(d[a]) > hpt::kSlabMin ? d[a] : std::copysign(hpt::kSlabMin, d[a])) * (1.0f / pk.scale);
      inv[a] = std::fmin(std::fmax(inv[a], -1e36f), 1e36f);
      oi[a] = -(o[a] * pk.scale * inv[a]);
    }
    std::vector<char> seen(n, 0);
    std::vector<int32_t> st{0};
    while (!st.empty()) {
      const int32_t node = st.back();
      st.pop_back();
      if (node < 0) {
        const uint32_t first = (uint32_t)~node >> 3, cnt = ((uint32_t)~node & 7u) + 1;
        for (uint32_t j = first; j < first + cnt; ++j) {
          uint32_t gid;
          std::memcpy(&gid, &b.prims[12 * (size_t)j + 3], 4);
          seen[gid] = 1;
        }
        continue;
      }
      const uint32_t *w = &pk.words[12 * (size_t)node];
      for (int c = 0; c < 2; ++c) {
        float near = 0.f, far = INFINITY;
        for (int a = 0; a < 3; ++a) {
          float org;
          std::memcpy(&org, &w[a], 4);
          const uint32_t pair = w[4 + 3 * c + a];
          const bool neg = std::signbit(inv[a]);
          const float at = std::fma(org, inv[a], oi[a]);
          near = std::fmax(near, std::fma(half_value(neg ? pair >> 16 : pair & 0xFFFFu), inv[a], at));
          far = std::fmin(far, std::fma(half_value(neg ? pair & 0xFFFFu : pair >> 16), inv[a], at));
        }
        int32_t link;
        std::memcpy(&link, &w[c ? 10 : 3], 4);
        if (near <= far * 1.000001f) st.push_back(link);
      }
    }
    for (uint32_t i = 0; i < n; ++i) {   // the ray's point inside the triangle's projection, the triangle ahead of it
      const float *p = &tri[9 * (size_t)i];
      double e[3];
      bool ahead = true;
      for (int q = 0; q < 3; ++q) {
        const float *x = p + 3 * q, *y = p + 3 * ((q + 1) % 3);
        e[q] = ((double)x[u] - o[u]) * ((double)y[v] - o[v]) - ((double)x[v] - o[v]) * ((double)y[u] - o[u]);
        ahead = ahead && s * ((double)x[axis] - o[axis]) > 0;
      }
      if (!ahead || !((e[0] > 0 && e[1] > 0 && e[2] > 0) || (e[0] < 0 && e[1] < 0 && e[2] < 0))) continue;
      ++meets;
      if (!seen[i] && ++lost < 5) std::printf("ray %d misses the leaf of triangle %u\n", k, i);
    }
  }
  std::printf("meets %ld, lost %ld\n", meets, lost);
  return lost || meets < 20000 ? 1 : 0;
}

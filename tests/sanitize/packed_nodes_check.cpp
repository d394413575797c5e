// Packed BVH nodes against brute force: the traversal's slab test in its own
// FP32 arithmetic (fused multiply-adds on binary16 plane offsets), with an FP64
// triangle test, has to find the closest hit of every ray. Usage: prog size shift
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

#include "../../paper_2606_14173_amd/csrc/bvh_build.hpp"

static float half_value(uint16_t h) {
  const int e = h >> 10 & 31, m = h & 1023;
  const float v = e == 31 ? INFINITY : e ? std::ldexp((float)(1024 + m), e - 25) : std::ldexp((float)m, -24);
  return h >> 15 ? -v : v;
}

struct Ray { float o[3], d[3]; };

static bool tri_hit(const float *t, const Ray &r, double tmin, double &out) {
  double e1[3], e2[3], s[3], p[3], q[3];
  for (int a = 0; a < 3; ++a) {
    e1[a] = (double)t[3 + a] - t[a]; e2[a] = (double)t[6 + a] - t[a]; s[a] = (double)r.o[a] - t[a];
  }
  auto cross = [](const double *u, const double *v, double *w) {
    w[0] = u[1] * v[2] - u[2] * v[1]; w[1] = u[2] * v[0] - u[0] * v[2]; w[2] = u[0] * v[1] - u[1] * v[0];
  };
  auto dot = [](const double *u, const double *v) { return u[0] * v[0] + u[1] * v[1] + u[2] * v[2]; };
  const double d[3] = {r.d[0], r.d[1], r.d[2]};
  cross(d, e2, p);
  const double det = dot(e1, p);
  if (det == 0.0) return false;
  cross(s, e1, q);
  const double u = dot(s, p) / det, v = dot(d, q) / det, w = dot(e2, q) / det;
  if (u < 0 || v < 0 || u + v > 1 || !(w > tmin)) return false;
  out = w;
  return true;
}

int main(int argc, char **argv) {
  if (argc < 3) return 2;
  const double size = std::atof(argv[1]), shift = std::atof(argv[2]);
  std::mt19937 g(7);
  std::uniform_real_distribution<double> U(-1.0, 1.0);
  long bad = 0, hits = 0, visits = 0;
  for (uint32_t n : {1u, 2u, 3u, 37u, 900u}) {
    std::vector<float> tri;
    for (uint32_t i = 0; i < n; ++i) {
      double c[3], e = i % 3 ? 0.1 : 0.7;   // small ones and large ones; every fourth lies in an axis plane
      for (double &x : c) x = U(g);
      for (int v = 0; v < 3; ++v)
        for (int a = 0; a < 3; ++a)
          tri.push_back((float)(size * (i % 4 == 0 && a == (int)(i / 4 % 3) ? c[a] : c[a] + e * U(g)) + (a == 1 ? -shift : shift)));
    }
    hpt::BvhResult b;
    if (!hpt::build_bvh(tri.data(), n, nullptr, 0, b)) return 3;
    hpt::PackedNodes pk;
    hpt::pack_nodes(b, pk);
    if (pk.words.size() != 12 * (size_t)b.n_nodes) return 4;
    for (int k = 0; k < 20000; ++k) {
      Ray r;
      const double away = k % 5 == 0 ? 40.0 : 1.2;
      double len = 0, d[3];
      for (int a = 0; a < 3; ++a) {
        r.o[a] = (float)(away * size * U(g) + (a == 1 ? -shift : shift));
        d[a] = k % 7 == 1 && a != k % 3 ? (k % 2 ? 0.0 : -0.0) : U(g);
      }
      if (k % 5 == 0 || k % 3 == 0) {   // towards a point of a triangle: a vertex, or inside
        const float *t = &tri[9 * (g() % n)];
        for (int a = 0; a < 3; ++a) d[a] = (k % 2 ? t[a] : 0.25 * t[a] + 0.25 * t[3 + a] + 0.5 * t[6 + a]) - (double)r.o[a];
      }
      for (double x : d) len += x * x;
      for (int a = 0; a < 3; ++a) r.d[a] = (float)(d[a] / std::sqrt(len));
      const double tmin = 1e-7;
      double best = INFINITY;
      for (uint32_t i = 0; i < n; ++i) {
        double t;
        if (tri_hit(&tri[9 * i], r, tmin, t) && t < best) best = t;
      }
      // the traversal
      float inv[3], oi[3];
      for (int a = 0; a < 3; ++a) {
        inv[a] = 1.0f / (std::fabs(r.d[a]) > 1e-30f ? r.d[a] : std::copysign(1e-30f, r.d[a])) * (1.0f / pk.scale);
        // (the hardware reciprocal may be an ulp off, either way)
        if ((k + a) % 3 < 2) inv[a] = std::nextafter(inv[a], (k + a) % 3 ? INFINITY : -INFINITY);
        inv[a] = std::fmin(std::fmax(inv[a], -1e36f), 1e36f);
        oi[a] = -(r.o[a] * pk.scale * inv[a]);
      }
      double found = INFINITY;
      std::vector<int32_t> st{0};
      while (!st.empty()) {
        const int32_t node = st.back();
        st.pop_back();
        if (node < 0) {
          const uint32_t first = (uint32_t)~node >> 3, cnt = ((uint32_t)~node & 7u) + 1;
          for (uint32_t j = first; j < first + cnt; ++j) {
            const float *p = &b.prims[12 * j];
            const float t9[9] = {p[0], p[1], p[2], p[4], p[5], p[6], p[8], p[9], p[10]};
            double t;
            if (tri_hit(t9, r, tmin, t) && t < found) found = t;
          }
          continue;
        }
        ++visits;
        const uint32_t *w = &pk.words[12 * (size_t)node];
        for (int c = 0; c < 2; ++c) {
          // (the traversal's hits are FP32: leave it what rounding the distance can move)
          float near = 1e-7f, far = (float)(found * (1 + 1e-6));
          for (int a = 0; a < 3; ++a) {
            float org;
            std::memcpy(&org, &w[a], 4);
            const uint32_t pair = w[4 + 3 * c + a];
            const bool neg = std::signbit(inv[a]);
            const float at = std::fma(org, inv[a], oi[a]);
            near = std::fmax(near, std::fma(half_value((uint16_t)(neg ? pair >> 16 : pair)), inv[a], at));
            far = std::fmin(far, std::fma(half_value((uint16_t)(neg ? pair : pair >> 16)), inv[a], at));
          }
          int32_t link;
          std::memcpy(&link, &w[c ? 10 : 3], 4);
          if (near <= far * 1.000001f) st.push_back(link);
        }
      }
      hits += best < INFINITY;
      if (best != found && ++bad < 5) std::printf("n %u ray %d: %.9g, traversal %.9g\n", n, k, best, found);
    }
  }
  std::printf("hits %ld, node visits %ld, lost %ld\n", hits, visits, bad);
  return bad ? 1 : 0;
}

// Boxes of a closed mesh read from a file (int64 vertices, int64 triangles, then FP32 vertices
// and int32 indices), printed with the time they took and the distance they keep:
// seconds pad, then lo hi of every box.
#include <chrono>
#include <cstdio>
#include <vector>

#include "gm_internal.h"

int main(int argc, char** argv)
{
    FILE* f = argc == 3 ? std::fopen(argv[1], "rb") : nullptr;
    int64_t n[2];
    if (!f || std::fread(n, sizeof(n), 1, f) != 1) return 1;
    std::vector<float> V((size_t)(3 * n[0]));
    std::vector<int32_t> I((size_t)(3 * n[1]));
    if (std::fread(V.data(), 4, V.size(), f) != V.size() || std::fread(I.data(), 4, I.size(), f) != I.size()) return 1;
    std::fclose(f);
    double scale = 0.0;
    for (float v : V) scale = std::max(scale, (double)(v < 0 ? -v : v));
    std::vector<gm::SolidBox> out;
    const auto t0 = std::chrono::steady_clock::now();
    const double pad = gm::solid_boxes(V.data(), I.data(), n[1], scale, std::atoi(argv[2]), 0, out);
    std::printf("%.6f %.9g\n", std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count(), pad);
    for (const gm::SolidBox& b : out)
        std::printf("%.9g %.9g %.9g %.9g %.9g %.9g\n", b.lo[0], b.lo[1], b.lo[2], b.hi[0], b.hi[1], b.hi[2]);
    return 0;
}

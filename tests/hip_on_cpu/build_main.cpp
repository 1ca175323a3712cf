// build N WIDTH BUILDER [LEVEL BACKWARDS]: builds a scene of N random disks. With LEVEL the build's fail word rises as
// in a launch whose look-back gave up: in the first block of the collapse's LEVEL-th launch, between the first
// wavefront's look and the others'. Prints the outcome; the workspace starts as a fixed pattern.
#include "common.h"
#include "internal.h"

using namespace pcrt;
namespace pcrt {
uint32_t resident_blocks(const void *, int) { return 1; }
}  // namespace pcrt

int main(int argc, char **argv) {
    const uint32_t n = atoi(argv[1]), width = atoi(argv[2]), builder = atoi(argv[3]);
    const int level = argc > 4 ? atoi(argv[4]) : -1;
    std::vector<float> pos(3 * n), nrm(3 * n);
    std::vector<uint16_t> mat(n, 0);
    std::vector<uint32_t> surf(n, 0);
    uint64_t s = n;
    auto rnd = [&] {
        s = s * 6364136223846793005ull + 1442695040888963407ull;
        return (float)((s >> 40) / 16777216.0) - 0.5f;
    };
    for (uint32_t i = 0; i < 3 * n; ++i) {
        pos[i] = 2.f * rnd();
        nrm[i] = rnd() + 0.01f;
    }
    const SceneLayout L = scene_layout(n, width, builder, false);
    std::vector<char> mem(L.total + 512, (char)0xa5);
    char *ws = (char *)(((uintptr_t)mem.data() + 255) & ~(uintptr_t)255);
    int launches = 0;
    emu::backwards = argc > 5 && atoi(argv[5]);
    emu::start = [&](const char *name, uint32_t block, uint32_t t) {
        if (level < 0 || !strstr(name, "k_wide_level") || block != 0) return;
        launches += t == (emu::backwards ? emu::bdim.x - 1 : 0u);
        if (launches == level + 1 && t == (emu::backwards ? 63u : 64u)) ((uint32_t *)(ws + L.ticket))[3] = 1;
    };
    uint32_t levels = 0, nodes = 0;
    int root = 0;
    const hipError_t e = build_scene(pos.data(), nrm.data(), mat.data(), surf.data(), n, 0.05f, 2, ws, L, nullptr, &levels,
                                     &nodes, &root);
    // every disk lies in one leaf of one wide node
    uint32_t seen = 0;
    std::vector<char> in_leaf(n, 0);
    for (uint32_t i = 0; !e && i < nodes; ++i)
        for (uint32_t j = 0; j < width; ++j) {
            const float *o = (const float *)(ws + L.wnode) + (size_t)i * 8 * width;
            int ref;
            memcpy(&ref, o + 6 * width + j, 4);
            if (ref >= 0 || !(o[j] < 1e30f)) continue;
            const int v = -1 - ref;
            for (int k = 0; k < (v & 7) + 1; ++k) seen += !in_leaf[(v >> 3) + k]++;
        }
    printf("%s levels %u nodes %u disks %u\n", e ? "refused" : "built", levels, nodes, seen);
    return 0;
}

// Host build of the hop launches' block order (csrc/chunks.h) for tests/test_chunks.py.
#include "chunks.h"

using namespace lqcd;

extern "C" {

// Every block, chunk and lane of a plan: counts[h] is raised for each valid
// lane of parity p; returns the first inconsistency (0: none) and the plan's
// blocks in *nsp.
int chunk_cover(const int* L, int order, int block, int ygroup, int maxsub, int idle, int p, int* counts, int* nsp)
{
    ChunkGrid g{{L[0], L[1], L[2], L[3]}, L[0] / 2, L[0] / 2 * L[1] * L[2] * L[3]};
    const ChunkArgs c = plan_chunk_order(g, order, block, ygroup, maxsub, idle);
    *nsp = c.nsp;
    if (c.nsub < 1 || c.nsub > maxsub) return 1;
    for (int b = 0; b < c.nsp; ++b)
        for (int sub = 0; sub < c.nsub; ++sub) {
            bool some = false;
            for (int lane = 0; lane < kChunk; ++lane) {
                const SitePos s = chunk_site(c, g.Lxh, L[1], L[2], g.Vh, (uint32_t)b, sub, p, lane);
                if (s.h < 0 || s.h >= g.Vh) return 2;  // (lanes past the end repeat a site)
                if (s.h != s.xh + g.Lxh * (s.y + L[1] * (s.z + L[2] * s.t))) return 3;
                if (s.xh < 0 || s.xh >= g.Lxh || s.y < 0 || s.y >= L[1] || s.z < 0 || s.z >= L[2] || s.t < 0 ||
                    s.t >= L[3])
                    return 4;
                if (s.x / 2 != s.xh || (s.x + s.y + s.z + s.t) % 2 != p) return 5;
                if (s.valid) ++counts[s.h];
                some = some || s.valid;
                if (s.valid && !s.some) return 6;
            }
            const SitePos s0 = chunk_site(c, g.Lxh, L[1], L[2], g.Vh, (uint32_t)b, sub, p, 0);
            if (some != s0.some) return 7;
        }
    return 0;
}

unsigned fast_divide(unsigned d, unsigned n)
{
    return fdiv(make_fastdiv(d), n);
}
}

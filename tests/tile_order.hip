// Host check of the input gradients' rows in position order: every input position of every sample belongs to exactly one row of one tile, a
// row's contexts are those of its sample and position, rows beyond a tile's last have none, and no tap that reaches a row is left out.
#include <hip/hip_runtime.h>
#include <cstdio>
#include <vector>
#include "../paper_2012_09849_amd/csrc/internal.hpp"

using namespace hts;

template <class T, class L> static const char *check(int B, int Hin, int Win)
{
    ConvDgrad<T, L> p{};
    p.N = L::CIN; p.K = p.klen = p.KC; p.Bn = B; p.Hin = Hin; p.Win = Win;
    p.Ho = (Hin - L::KSZ) / L::STRIDE + 1; p.Wo = (Win - L::KSZ) / L::STRIDE + 1;
    p.prepare();
    if (!ConvDgradByPosition<T, L>::fits(p)) return B < p.BM ? nullptr : "refused";
    const ConvDgradByPosition<T, L> q(p);
    const int tiles = (q.max_m() + p.BM - 1) / p.BM;
    std::vector<int> seen((size_t)B * Hin * Win, 0);
    for (int z = 0; z < p.batches(); ++z) {
        const auto c = p.cls(z);
        for (int i = 0; i < tiles; ++i) {
            typename ConvDgradByPosition<T, L>::Tile t(p);
            if (!q.tile(i, z, t)) continue;
            if (t.batch_m(z) < 1 || t.batch_m(z) > p.BM) return "rows of a tile";
            const uint32_t live = t.live_taps();
            for (int m = 0; m < p.BM; ++m) {
                const auto x = t.ctx_a(m, z);
                if (m >= t.batch_m(z)) {
                    if (x.off != -1) return "context beyond the last row";
                    continue;
                }
                const long long o = t.row(m, z).o, pixel = o / p.N;
                if (o < 0 || o % p.N || pixel >= (long long)seen.size()) return "output row";
                const int b = (int)(pixel / (Hin * Win)), y = (int)(pixel / Win % Hin), xx = (int)(pixel % Win);
                ++seen[pixel];
                if (y % L::STRIDE != c.py || xx % L::STRIDE != c.px || y / L::STRIDE != x.yy || xx / L::STRIDE != x.xx) return "position";
                if (x.off != (((long long)b * p.Ho + x.yy) * p.Wo + x.xx) * L::COUT) return "operand row";
                for (int tap = 0; tap < p.TK * p.TK; ++tap) {
                    const int oy = x.yy - tap / p.TK, ox = x.xx - tap % p.TK;
                    if (oy >= 0 && ox >= 0 && oy < p.Ho && ox < p.Wo && !(live >> tap & 1)) return "tap left out";
                }
            }
        }
    }
    for (int n : seen) if (n != 1) return "a position without a row, or with two";
    return nullptr;
}

int main()
{
    const int conv2[][2] = {{20, 20}, {17, 23}, {10, 12}, {8, 8}, {4, 6}, {5, 9}}, conv3[][2] = {{9, 9}, {7, 10}, {4, 5}, {3, 3}, {3, 8}, {13, 4}};
    const int rows[] = {1, 63, 64, 65, 127, 128, 129, 131, 200, 255, 256, 257, 300, 511, 512, 513, 700, 1000, 1023, 1024, 1025, 2300};
    int n = 0;
    for (int g = 0; g < 6; ++g)
        for (int B : rows) {
            const char *e[] = {check<float, Layer2>(B, conv2[g][0], conv2[g][1]), check<bf16_t, Layer2>(B, conv2[g][0], conv2[g][1]),
                               check<float, Layer3>(B, conv3[g][0], conv3[g][1]), check<bf16_t, Layer3>(B, conv3[g][0], conv3[g][1])};
            for (int i = 0; i < 4; ++i, ++n) if (e[i]) { printf("%s: layer %d, %d rows, grid %d\n", e[i], 2 + i / 2, B, g); return 1; }
        }
    printf("%d problems\n", n);
}

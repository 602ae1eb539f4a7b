// Host unit test of the packing of the coupling GEMM's macro tiles into workgroups:
// every output tile of every macro tile is computed by exactly one wave, from operand
// slots of its own workgroup that hold the tile's rows and columns, and every wave
// forms at most one operand.  Built with g++ by tests/test_gemm_packs_cpu.py.
#include <cstdio>
#include <string>
#include <utility>
#include <vector>

#include "../../paper_2105_08722_amd/csrc/mfma_plan.h"

namespace encore {
static std::string g_err;
void set_error(const std::string& m) { g_err = m; }
const char* get_error() { return g_err.c_str(); }
int fail(int, const std::string& m) { g_err = m; return 1; }
}  // namespace encore

using namespace encore;

static int check_case(int N, int L, bool allp, int nbins, int KL)
{
    GemmPlan P;
    if (build_gemm_plan(N, L, allp, nbins, KL, P) != 0) return 1;
    // rows and columns of each output tile
    std::vector<std::pair<int, int>> want((size_t)P.ntiles);
    for (size_t m = 0; m < P.macros.size(); m += kGemmMacroWidth)
        for (int r = 0; r < P.macros[m + 2]; ++r)
            for (int c = 0; c < P.macros[m + 3]; ++c)
                want[(size_t)P.macros[m + 4] + r * P.macros[m + 3] + c] = {P.macros[m] + 16 * r, P.macros[m + 1] + 16 * c};
    std::vector<int> seen((size_t)P.ntiles, 0);
    int bad = P.packs.size() % kGemmPackWidth != 0;
    for (size_t g = 0; g < P.packs.size(); g += kGemmPackWidth) {
        const int32_t* pk = &P.packs[g];
        for (int w = 0; w < kGemmMaxOps; ++w) {
            const int32_t* d = pk + kGemmPackWave * w;
            const unsigned s = (unsigned)d[2];
            const int nr = d[3] & 0xff, nc = (d[3] >> 8) & 0xff, mc = d[3] >> 16;
            const unsigned slot[4] = {s & 0xff, (s >> 8) & 0xff, (s >> 16) & 0xff, s >> 24};
            for (unsigned q : slot) bad += q >= kGemmMaxOps;
            if (bad) return bad;
            for (int i = 0; i < nr; ++i)
                for (int j = 0; j < nc; ++j) {
                    const int64_t t = d[4] + (int64_t)i * mc + j;
                    if (t < 0 || t >= P.ntiles) return 1;
                    const int32_t* ro = pk + kGemmPackWave * slot[i];
                    const int32_t* co = pk + kGemmPackWave * slot[2 + j];
                    bad += ro[1] != 0 || co[1] != 1 || ro[0] != want[t].first || co[0] != want[t].second;
                    ++seen[(size_t)t];
                }
        }
    }
    for (int v : seen) bad += v != 1;
    return bad;
}

int main()
{
    const int cases[][5] = {{5, 0, 0, 4, 2}, {5, 2, 0, 10, 2}, {5, 3, 1, 7, 2}, {5, 4, 0, 10, 2}, {6, 0, 0, 5, 3},
                            {6, 1, 0, 8, 3}, {6, 2, 1, 7, 3}, {6, 2, 0, 8, 2}, {4, 3, 1, 6, 2}, {3, 4, 0, 5, 1}};
    int failures = 0;
    for (const auto& c : cases) {
        const int bad = check_case(c[0], c[1], c[2] != 0, c[3], c[4]);
        if (bad) std::printf("FAIL N=%d lmax=%d allparity=%d bins=%d KL=%d: %d\n", c[0], c[1], c[2], c[3], c[4], bad);
        failures += bad != 0;
    }
    std::printf(failures ? "%d failed\n" : "all passed\n", failures);
    return failures != 0;
}

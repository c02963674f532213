// The GPU graph build's choice of a form against a device whose memory is
// bounded: what fits the chunked form is built, whatever the pair form needs.
// (Test infrastructure.)
#include "knn_form.hpp"

#include <cstdio>

using namespace vie;

int main()
{
    const size_t GiB = (size_t)1 << 30;
    for (int64_t V : {100, 16383, 16384, 16385, 151936, 262144, 300001, 524288, 524289, 1000003}) {
        for (int64_t chunk : {(int64_t)0, (int64_t)1, (int64_t)700, V}) {
            for (size_t limit : {GiB / 64, GiB, 2 * GiB + GiB / 16, 8 * GiB}) {
                KnnForm f;
                const bool got = knn_first_form(V, chunk, f, [&](const KnnForm &g) { return g.score_bytes <= limit; });
                const KnnForm plain = knn_form(V, chunk, false);
                if (plain.score_bytes <= limit && !got) {
                    std::printf("failed: V = %lld, chunk %lld: %zu bytes fit, no form found\n", (long long)V,
                                (long long)chunk, plain.score_bytes);
                    return 1;
                }
                if (!got) continue;
                const bool pairs = chunk == 0 && V >= kPairMinRows && V <= 524288 && (size_t)V * 8192 <= limit;
                if (f.pairs != pairs || f.chunk < 1 || f.chunk > V || f.ld % 4 || f.ld < V ||
                    f.score_bytes < (size_t)f.chunk * f.ld * 4 || (chunk && f.chunk != std::min(chunk, V))) {
                    std::printf("failed: the form of V = %lld, chunk %lld\n", (long long)V, (long long)chunk);
                    return 1;
                }
            }
        }
    }
    std::printf("all checks passed\n");
    return 0;
}

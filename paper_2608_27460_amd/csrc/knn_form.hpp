// The two forms of the GPU graph build's first step and the scores' memory
// each needs (knn_build.hip describes the forms).
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace vie {

constexpr int kPairCap = 1024;  // keys kept per row in the pair form
// Heads from this many rows on take the pair form: per build, against the
// chunked form, 6000 / 12000 / 20000 / 32768 rows of 256 fp32 values took 3.9 /
// 5.4 / 7.4 / 11.7 ms (3.5 / 5.2 / 8.2 / 14.8), of 1024 bf16 values 4.2 / 4.7 /
// 6.1 / 8.9 ms (4.3 / 4.6 / 6.8 / 11.6): below, the sampling costs what it saves.
constexpr int kPairMinRows = 16384;

struct KnnForm {
    bool pairs;
    int64_t ld;          // pitch of a row of scores (16-byte aligned rows)
    int64_t chunk;       // rows of one Gram block of the chunked form
    size_t score_bytes;  // scores, or the keys of the pair form
};

// The pair form unless the caller bounds the scores in memory, the keys would
// pass 4 GiB, or the head is small enough for the chunked form.  In the pair
// form the rows it leaves over are chunked in the keys' memory.
inline KnnForm knn_form(int64_t V, int64_t chunk_rows, bool pairs)
{
    KnnForm f;
    const int64_t keys = V * (int64_t)(kPairCap * 8);
    f.pairs = pairs && chunk_rows == 0 && V >= kPairMinRows && keys <= ((int64_t)4 << 30);
    f.ld = (V + 3) & ~(int64_t)3;
    f.chunk = f.pairs ? keys / (f.ld * 4) : chunk_rows > 0 ? chunk_rows : ((int64_t)2 << 30) / (f.ld * 4);
    f.chunk = std::max<int64_t>(1, std::min<int64_t>(f.chunk, V));
    f.score_bytes = f.pairs ? (size_t)keys : (size_t)f.chunk * f.ld * 4;
    return f;
}

// The form whose memory attempt(form) finds: the pair form's keys are twice
// the chunked form's scores at its largest heads, so where they do not fit
// the chunked form still may.
template <typename Attempt> bool knn_first_form(int64_t V, int64_t chunk_rows, KnnForm &f, Attempt attempt)
{
    f = knn_form(V, chunk_rows, true);
    if (attempt(f)) return true;
    if (!f.pairs) return false;
    f = knn_form(V, chunk_rows, false);
    return attempt(f);
}

}  // namespace vie

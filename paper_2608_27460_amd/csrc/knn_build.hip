// Batch construction of a single-layer graph over the rows of W_out on the
// GPU.  Section 3 builds the index offline and prioritises its quality;
// Section 5 names GPU construction as future work.  The graph is the batch
// form also written out by the CPU oracle:
//
//   1. cand(i): the K rows nearest to row i by inner product (j != i), in the
//      (score desc, id asc) order of the search;
//   2. fwd(i): the neighbour-selection heuristic of Malkov & Yashunin
//      (Algorithm 4) over cand(i) with cap M0: in candidate order, e is kept
//      iff <w_e, w_i> > <w_e, w_r> for every r kept before it (a list of at
//      most M0 candidates is kept whole);
//   3. rev(j): every i with j in fwd(i);
//   4. the list of j: fwd(j), then the nodes of rev(j) not in fwd(j) in
//      (score desc, id asc) order, cut at M0 entries;
//   5. entry point: the row of largest squared norm (ties: smaller id).
//
// Step 1 is a dense contraction on the matrix cores (fp32 accumulation).
// Large heads multiply every pair of rows once and keep only the scores that
// pass a sampled threshold of either row (knn_pairs_kernel).  Small heads,
// callers that bound the scores in memory and the rows whose threshold did
// not serve take the chunked form: the Gram block S = W[rows] W^T of a chunk
// of rows (knn_gram_kernel), then one workgroup per row selects its exact
// top K from S (knn_topk_kernel).  Scores are fp32 throughout; ties of equal scores are
// broken by id exactly as the oracle breaks them.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <type_traits>
#include <vector>

#include "index.hpp"
#include "keys.hpp"
#include "knn_form.hpp"

namespace vie {

namespace {

constexpr int kWave = 64;
constexpr int kTopkThreads = 256;
constexpr int kDigitBits = 12;               // radix digit of the selection
constexpr int kDigitBuckets = 1 << kDigitBits;
constexpr int kGatherCap = 2048;             // keys a selection sorts in LDS
constexpr int kSelectThreads = 256;
constexpr int kSelectRows = 128;             // candidate rows of one Gram block (K <= 128)

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

// 16 x 16 tile += A (16 rows x 32 columns) B^T, bf16 operands, fp32 accumulation
__device__ __forceinline__ f32x4 mfma_bf16(u32x4 a, u32x4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b),
                                                   c, 0, 0, 0);
}

struct TopkShared {
    uint32_t hist[kDigitBuckets];
    uint64_t gat[kGatherCap];
    uint32_t wsum[kTopkThreads / kWave];
    uint32_t n, bucket, above, count;
};

// Exclusive prefix sum over the block of one value per thread.
template <int NT>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *wsum)
{
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    uint32_t incl = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t t = __shfl_up(incl, o, kWave);
        if (lane >= o) incl += t;
    }
    if (lane == kWave - 1) wsum[wave] = incl;
    __syncthreads();
    uint32_t base = 0;
    for (int w = 0; w < wave; ++w) base += wsum[w];
    __syncthreads();
    return base + incl - v;
}

// Sorts n <= kGatherCap keys in LDS, largest first (bitonic network over the
// next power of two; the padding is 0, the smallest key).
template <int NT>
__device__ void block_sort_desc(uint64_t *a, int n)
{
    int p = 1;
    while (p < n) p <<= 1;
    for (int i = n + threadIdx.x; i < p; i += NT) a[i] = 0ull;
    __syncthreads();
    for (int size = 2; size <= p; size <<= 1)
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int i = threadIdx.x; i < p / 2; i += NT) {
                const int lo = 2 * i - (i & (stride - 1)), hi = lo + stride;
                const bool desc = (lo & size) == 0;
                const uint64_t x = a[lo], y = a[hi];
                if (desc ? x < y : x > y) {
                    a[lo] = y;
                    a[hi] = x;
                }
            }
            __syncthreads();
        }
}

// The K largest of the keys key_at(0 .. n-1) (0 = no key), sorted, into
// sh.gat[0 .. K).  Exact: a radix select over the 64-bit keys, kDigitBits
// per round from the top, narrows the bucket of the K-th largest until every
// key at or above that bucket fits in LDS; those are gathered and sorted.
// Keys are distinct, so at most 6 rounds are needed.  Returns the number of
// keys found (< K only when fewer than K keys exist).
template <int NT, typename KeyAt>
__device__ int block_topk(int64_t n, int K, KeyAt key_at, TopkShared &sh)
{
    const int tid = threadIdx.x;
    uint64_t prefix = 0ull;
    int known = 0;
    uint32_t want = (uint32_t)K;
    uint64_t T = 0ull;
    for (;;) {
        const int width = 64 - known < kDigitBits ? 64 - known : kDigitBits;
        const int shift = 64 - known - width;
        const uint32_t nb = 1u << width;
        for (int b = tid; b < kDigitBuckets; b += NT) sh.hist[b] = 0u;
        if (tid == 0) {
            sh.bucket = 0u;
            sh.above = 0u;
            sh.count = 0u;
        }
        __syncthreads();
        for (int64_t i = tid; i < n; i += NT) {
            const uint64_t key = key_at(i);
            if (key != 0ull && (known == 0 || (key >> (64 - known)) == (prefix >> (64 - known))))
                atomicAdd(&sh.hist[(uint32_t)(key >> shift) & (nb - 1)], 1u);
        }
        __syncthreads();
        // buckets from the top: thread t holds buckets nb-1-16t .. nb-16-16t
        constexpr int per = kDigitBuckets / NT;
        uint32_t c[per], sum = 0;
#pragma unroll
        for (int j = 0; j < per; ++j) {
            const int b = (int)nb - 1 - (per * tid + j);
            c[j] = b >= 0 ? sh.hist[b] : 0u;
            sum += c[j];
        }
        uint32_t above = block_exclusive_scan<NT>(sum, sh.wsum);
        bool found = false;
#pragma unroll
        for (int j = 0; j < per; ++j) {
            if (!found && above < want && want <= above + c[j]) {
                sh.bucket = (uint32_t)((int)nb - 1 - (per * tid + j));
                sh.above = above;
                sh.count = c[j];
                found = true;
            }
            above += c[j];
        }
        __syncthreads();
        if (sh.count == 0u) {
            // fewer than want keys match the prefix: take every key >= prefix
            T = prefix == 0ull ? 1ull : prefix;
            break;
        }
        const uint64_t lo = prefix | ((uint64_t)sh.bucket << shift);
        const uint32_t total = ((uint32_t)K - want) + sh.above + sh.count;
        if (total <= (uint32_t)kGatherCap || shift == 0) {
            T = lo == 0ull ? 1ull : lo;
            break;
        }
        prefix = lo;
        known += width;
        want -= sh.above;
        __syncthreads();
    }
    if (tid == 0) sh.n = 0u;
    __syncthreads();
    for (int64_t i = tid; i < n; i += NT) {
        const uint64_t key = key_at(i);
        if (key >= T) {
            const uint32_t slot = atomicAdd(&sh.n, 1u);
            if (slot < (uint32_t)kGatherCap) sh.gat[slot] = key;
        }
    }
    __syncthreads();
    const int m = (int)min(sh.n, (uint32_t)kGatherCap);
    block_sort_desc<NT>(sh.gat, m);
    return m < K ? m : K;
}

// Step 1, per row of a chunk: the K nearest other rows from the chunk's
// scores S [rows][ld] (row r of the chunk is row r0 + r of W_out; rows start
// 16-byte aligned).  A sample of the row (every kSampleEvery-th block of
// kTopkThreads scores) gives a threshold T0 with about twice the sample's
// share of K keys above it; one vectorized pass then gathers every key >= T0.
// If at least K and at most kGatherCap keys were gathered, every key of the
// answer is among them (K keys are >= T0, so the K-th largest is too) and a
// sort finishes; otherwise the exact radix select runs.  The sample only
// decides the speed, never the result.
constexpr int kSampleEvery = 8;

// ---------------------------------------------------------------------------
// Gram blocks on the matrix cores
// ---------------------------------------------------------------------------
//
// S[c][j] = <w_{r0 + c}, w_j> for the rows c of a chunk and every row j, fp32
// accumulation, written with row pitch ld.  A workgroup of eight waves owns
// a 256 x 128 tile (256 chunk rows c by 128 rows j); wave (wm, wn) computes
// its 64 x 64 block as 4 x 4 tiles of 16 x 16 on the matrix cores
// (v_mfma_f32_16x16x32_bf16 for bf16 rows, v_mfma_f32_16x16x4_f32 for fp32
// rows).  The reduction over the row width runs in stages of kGramKC bytes
// of each row: both slices of a stage (256 and 128 rows) are staged in LDS,
// the stages two ahead loading into registers while the current one is
// multiplied.  (128 x 128 tiles of four waves, two workgroups per CU, read a
// quarter more through the CU for the same products and measured the same
// per chunk but 2-5% slower per build.)
// Lane (r, g) of a wave (r = lane % 16, g = lane / 16) feeds row r of a
// 16-row operand with its g-th quarter of the k step, and ends holding rows
// 4 g + i of column r of each 16 x 16 result.  Every score is the same
// sequence of products and sums whichever tile computes it.
//
// Staged rows are not padded: the 16-byte piece p of staged row x sits at
// piece p ^ ((x >> 1) & 7) of the row.  Measured with the LDS counters on
// gfx950, the operand reads (16 rows, four consecutive pieces or four
// consecutive floats each) then use every bank once per cycle, where rows
// padded by 16 bytes took twice the cycles (half of them bank conflicts).  Every load of a stage is issued with
// no branch around it (pieces past the row are clamped to its last piece and
// replaced by zeros when staged), in the order they are consumed, so the
// compiler waits only for the stage being staged.

#ifndef VIE_GRAM_TILE_C
#define VIE_GRAM_TILE_C 256
#endif
constexpr int kGramTileC = VIE_GRAM_TILE_C;        // chunk rows c per workgroup (128 or 256)
constexpr int kGramTile = 128;                     // rows j per workgroup
constexpr int kGramThreads = 2 * kGramTileC;       // (kGramTileC / 64) x 2 waves of 64 x 64 quarters
#ifndef VIE_GRAM_KC
#define VIE_GRAM_KC 128
#endif
constexpr int kGramKC = VIE_GRAM_KC;               // bytes of a row per stage
static_assert(kGramKC == 128, "the piece swizzle is laid out for 8 pieces a staged row");
constexpr int kGramRowPitch = kGramKC;                 // LDS bytes per staged row
constexpr int kGramStage = (kGramTileC + kGramTile) * kGramRowPitch;  // A and B slices of one stage

// byte offset of 16-byte piece p of staged row x
__device__ __forceinline__ int gram_piece(int x, int p) { return x * kGramRowPitch + ((p ^ ((x >> 1) & 7)) << 4); }
constexpr int kGramLoads = (kGramTileC + kGramTile) * (kGramKC / 16) / kGramThreads;  // 16-byte loads per thread
static_assert(kGramLoads * kGramThreads == (kGramTileC + kGramTile) * (kGramKC / 16), "staging shape");

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <bool BF16>
__global__ __launch_bounds__(kGramThreads) __attribute__((amdgpu_waves_per_eu(2))) void knn_gram_kernel(const char *__restrict__ W, int row_bytes,
                                                                const int32_t *__restrict__ list, int64_t r0,
                                                                int64_t rows, const char *__restrict__ WB, int64_t VB,
                                                                float *__restrict__ S, int64_t ld)
{
    extern __shared__ __align__(16) char smem[];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int r = lane & 15, g = lane >> 4;
    const int wm = wave >> 1, wn = wave & 1;
    // Launch order for the eight XCDs, each with its own L2: workgroups are
    // dealt to the XCDs in turn (workgroup L runs on XCD L % 8).  XCD x
    // takes half of the chunk's tiles c (the first half for even x) and the
    // tiles of rows j numbered x / 2, x / 2 + 4, ..., each with all of its
    // tiles c in a row: a tile of j is fetched by two XCDs, and each XCD
    // re-reads only its half of the chunk's rows.  The grid rounds the tiles
    // of c up to an even count and those of j up to a multiple of 4; the
    // workgroups past the last tile return at once.
    const int nc = (int)((rows + kGramTileC - 1) / kGramTileC);
    const int nch = (nc + 1) / 2;
    const int64_t nj = (VB + kGramTile - 1) / kGramTile;
    const int64_t wg = blockIdx.x, i = wg >> 3, x = wg & 7;
    const int64_t jt = (i / nch) * 4 + (x >> 1), ct = (x & 1) * nch + i % nch;
    if (jt >= nj || ct >= nc) return;
    const int64_t c0 = ct * kGramTileC, j0 = jt * kGramTile;
    const int nstage = (row_bytes + kGramKC - 1) / kGramKC;
    const u32x4 zero = {0u, 0u, 0u, 0u};
    // staging: load t of a thread covers staged row (L / 8) of A (the first
    // kGramTileC rows) or of B, 16 bytes at byte (L % 8) * 16 of the stage,
    // L = t * kGramThreads + tid
    const char *src[kGramLoads];
    int soff[kGramLoads], scol[kGramLoads];
#pragma unroll
    for (int t = 0; t < kGramLoads; ++t) {
        const int L = t * kGramThreads + tid;
        const int srow = L / (kGramKC / 16);  // 0..255: A rows then B rows
        scol[t] = (L % (kGramKC / 16)) * 16;
        const int64_t arow = r0 + min<int64_t>(c0 + srow, rows - 1);
        src[t] = srow < kGramTileC ? W + (list ? (int64_t)list[arow] : arow) * row_bytes
                                   : WB + min<int64_t>(j0 + srow - kGramTileC, VB - 1) * row_bytes;
        soff[t] = gram_piece(srow, scol[t] >> 4);
    }
    auto load_stage = [&](int st, u32x4(&buf)[kGramLoads]) {
#pragma unroll
        for (int t = 0; t < kGramLoads; ++t)
            buf[t] = *reinterpret_cast<const u32x4 *>(src[t] + min(st * kGramKC + scol[t], row_bytes - 16));
        __builtin_amdgcn_sched_barrier(0);  // keep the issue order
    };
    f32x4 acc[4][4];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int n = 0; n < 4; ++n) acc[m][n] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    // stages load two ahead: stage st's loads sit in register buffer st % 2
    // (the stage pairs are written out over the buffers, so no load in
    // flight is ever copied) and in LDS buffer st % 2
    u32x4 pre[2][kGramLoads];
    load_stage(0, pre[0]);
    load_stage(min(1, nstage - 1), pre[1]);
    // one stage: into LDS buffer PB from register buffer PB, the loads of the
    // stage two ahead into that register buffer, then the products.  The
    // stage pairs run in a loop without any branch inside (so the compiler
    // keeps the loads of the next stage in flight across it) and an odd last
    // stage after it.
    auto run_stage = [&](auto pbc, int st) {
        constexpr int pb = decltype(pbc)::value;
        char *buf = smem + pb * kGramStage;
#pragma unroll
        for (int t = 0; t < kGramLoads; ++t)
            *reinterpret_cast<u32x4 *>(buf + soff[t]) = st * kGramKC + scol[t] + 16 <= row_bytes ? pre[pb][t] : zero;
        __builtin_amdgcn_sched_barrier(0);
        load_stage(min(st + 2, nstage - 1), pre[pb]);  // past the end: the last stage again (cached)
        __syncthreads();  // the stage is in LDS (and the stage before it is no longer read)
        const char *A = buf + (wm * 64) * kGramRowPitch;
        const char *B = buf + (kGramTileC + wn * 64) * kGramRowPitch;
        if constexpr (BF16) {
#pragma unroll
            for (int kk = 0; kk < kGramKC; kk += 64) {  // 32 bf16 per MFMA step
                u32x4 a[4], b[4];
#pragma unroll
                for (int m = 0; m < 4; ++m)
                    a[m] = *reinterpret_cast<const u32x4 *>(A + gram_piece(m * 16 + r, kk / 16 + g));
#pragma unroll
                for (int n = 0; n < 4; ++n)
                    b[n] = *reinterpret_cast<const u32x4 *>(B + gram_piece(n * 16 + r, kk / 16 + g));
#pragma unroll
                for (int m = 0; m < 4; ++m)
#pragma unroll
                    for (int n = 0; n < 4; ++n) acc[m][n] = mfma_bf16(a[m], b[n], acc[m][n]);
            }
        } else {
#pragma unroll
            for (int kk = 0; kk < kGramKC; kk += 16) {  // 4 floats per MFMA step
                float a[4], b[4];
#pragma unroll
                for (int m = 0; m < 4; ++m)
                    a[m] = *reinterpret_cast<const float *>(A + gram_piece(m * 16 + r, kk / 16) + 4 * g);
#pragma unroll
                for (int n = 0; n < 4; ++n)
                    b[n] = *reinterpret_cast<const float *>(B + gram_piece(n * 16 + r, kk / 16) + 4 * g);
#pragma unroll
                for (int m = 0; m < 4; ++m)
#pragma unroll
                    for (int n = 0; n < 4; ++n) acc[m][n] = mfma_f32(a[m], b[n], acc[m][n]);
            }
        }
    };
    int st = 0;
    for (; st + 1 < nstage; st += 2) {
        run_stage(std::integral_constant<int, 0>(), st);
        run_stage(std::integral_constant<int, 1>(), st + 1);
    }
    if (st < nstage) run_stage(std::integral_constant<int, 0>(), st);
    // lane (r, g) holds chunk rows 16 m + 4 g + i of the quarter, column 16 n + r
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t c = c0 + wm * 64 + m * 16 + 4 * g + i;
            if (c >= rows) continue;
            float *out = S + c * ld + j0 + wn * 64;
#pragma unroll
            for (int n = 0; n < 4; ++n)
                if (j0 + wn * 64 + n * 16 + r < VB) out[n * 16 + r] = acc[m][n][i];
        }
}

// ---------------------------------------------------------------------------
// every pair of rows once
// ---------------------------------------------------------------------------
//
// The scores are symmetric, and a row needs only its K best of V.  So each
// unordered pair of rows is multiplied once, in 256 x 128 tiles of the upper
// triangle, and no score reaches HBM: a score that reaches the threshold of
// either of its rows is appended, as a key, to the keys of that row.  A
// row's threshold is a sampled score (knn_threshold_kernel) with about 1.7 (one
// row in four sampled) to 3.3 times K scores above it (one in 32, K = 128); a
// row whose keys turn out fewer than K or more
// than kPairCap is left to the chunked form, so the sample decides the speed
// only, never the result.  Where the sample shows that half of the rows would
// be left (equal scores without number), the pairs are not multiplied at all
// (a build over 32768 x 256 bf16 zeros: 38.1 ms
// with them, 23.6 without, 23.5 in the chunked form).
//
// Bound by the matrix cores.  151936 x 1024 bf16: 26.5 ms for 23.6 TFLOP (0.89
// PFLOP/s; an 8192-cubed library product reaches 1.21), where the chunked form
// multiplied every pair twice (63.6 ms), wrote 92 GB of scores and read them
// back (21.3 ms of selection); with sampling and picking the step takes 32
// ms instead of 85.  32768 x 256 fp32: 2.9 ms (5.6 chunked) at 94 TFLOP/s.
//
// A wave owns a 64 x 64 block of the tile as 4 x 4 tiles of 16 x 16 (the
// layout, and so every score's sequence of products and sums, is that of
// knn_gram_kernel).  Stages of 64 bytes of each row go from memory straight
// to LDS (global_load_lds, 16 bytes a lane), kPairBufs - 1 stages ahead, so
// no register holds a load in flight and two workgroups fit a CU: one fills
// the matrix cores while the other waits or sifts its scores.  Piece p of
// staged row x sits at p ^ ((x >> 2) & 3).  By the LDS counters that still
// leaves half of the operand reads' cycles to bank conflicts (2.9e9 of 6.0e9 a
// build of 151936 x 1024 bf16; 1.35e8 of 2.9e8 for 32768 x 256 fp32), and the fp32
// form spills 114 registers around the sift: what it has left is there.

constexpr int kPairTileC = 256, kPairTileJ = 128;  // rows c and j of a tile
constexpr int kPairWavesJ = kPairTileJ / 64;
constexpr int kPairThreads = (kPairTileC / 64) * kPairWavesJ * kWave;
constexpr int kPairKC = 64;    // bytes of a row per stage
constexpr int kPairBufs = 3;
constexpr int kPairRows = kPairTileC + kPairTileJ;
constexpr int kPairStage = kPairRows * kPairKC;
constexpr int kPairLoads = kPairStage / (16 * kPairThreads);  // 16-byte loads per lane and stage
static_assert(kPairLoads * kPairThreads * 16 == kPairStage, "staging shape");
static_assert(kPairTileC % (kPairThreads / 4) == 0, "one load covers rows c or rows j, never both");
constexpr int kPairLds = kPairBufs * kPairStage + kPairRows * 4;
constexpr int kPairList = kPairBufs * kPairStage / 8 / (kPairThreads / kWave);  // listed scores per wave
// squares of 256 rows on a side of a launch block: 151936 x 1024 bf16 43.0 ms a
// build with 8, 42.9 with 4, 44.2 with 16; 32768 x 256 fp32 7.03, 7.04 and 7.42
constexpr int kPairBlock = 8;
constexpr int kPairPickRows = 4096;   // sampled rows, at least (or V)
constexpr int kPairPickStep = 32;     // sampled rows, at least one in this many

__device__ __forceinline__ int pair_piece(int x, int p) { return x * kPairKC + ((p ^ ((x >> 2) & 3)) << 4); }

// Appends a key to the keys of a row (more than kPairCap are counted only).
__device__ __forceinline__ void pair_append(int64_t row, uint64_t key, uint32_t *count, uint64_t *keys)
{
    const uint32_t slot = atomicAdd(&count[row], 1u);
    if (slot < (uint32_t)kPairCap) keys[row * kPairCap + slot] = key;
}

template <bool BF16>
__global__ __launch_bounds__(kPairThreads) __attribute__((amdgpu_waves_per_eu(4, 4))) void knn_pairs_kernel(
    const char *__restrict__ W, int64_t V, int row_bytes, const float *__restrict__ thr,
    const uint32_t *__restrict__ full, uint32_t *count, uint64_t *keys)
{
    extern __shared__ __align__(16) char smem[];
    if (*full > (uint32_t)(V / 2)) return;  // most rows would take too many keys
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int r = lane & 15, g = lane >> 4;
    const int wm = wave / kPairWavesJ, wn = wave % kPairWavesJ;
    // Launch order: blocks of kPairBlock x kPairBlock squares of kPairTileC
    // rows, walked over the upper triangle and dealt to the XCDs in turn (workgroup L runs on
    // XCD L % 8), so that the tiles an XCD works on at a time share their
    // rows in its L2.  Workgroups past the triangle return at once.
    constexpr int F = kPairTileC / kPairTileJ;
    constexpr int sb = kPairBlock;
    constexpr uint32_t per = (uint32_t)(sb * sb * F);
    const uint32_t i0 = blockIdx.x >> 3;
    const uint32_t blk = (i0 / per) * 8 + (blockIdx.x & 7), in = i0 % per;
    uint32_t bj = (uint32_t)((sqrtf(8.0f * (float)blk + 1.0f) - 1.0f) * 0.5f);
    while (bj * (bj + 1) / 2 > blk) --bj;
    while ((bj + 1) * (bj + 2) / 2 <= blk) ++bj;
    const uint32_t bi = blk - bj * (bj + 1) / 2;
    const int64_t c0 = (int64_t)(bi * sb + in % sb) * kPairTileC;
    const int64_t j0 = (int64_t)(bj * sb * F + in / sb) * kPairTileJ;
    if (c0 >= V || j0 >= V || j0 + kPairTileJ - 1 <= c0) return;
    float *lthr = reinterpret_cast<float *>(smem + kPairBufs * kPairStage);

    const int nfull = row_bytes / kPairKC;  // whole stages
    uint32_t off[kPairLoads];               // from the tile's first row c or j
#pragma unroll
    for (int t = 0; t < kPairLoads; ++t) {
        const int x = (t * kPairThreads + tid) / 4;  // staged row
        const int p = (tid & 3) ^ ((x >> 2) & 3);
        const int64_t n = x < kPairTileC ? min<int64_t>(x, V - 1 - c0) : min<int64_t>(x - kPairTileC, V - 1 - j0);
        off[t] = (uint32_t)n * (uint32_t)row_bytes + 16 * p;
    }
    const char *baseC = W + c0 * row_bytes, *baseJ = W + j0 * row_bytes;
    auto issue = [&](int st, int buf) {
        const int64_t so = (int64_t)min(st, nfull - 1) * kPairKC;  // past the end: the last stage again, unused
#pragma unroll
        for (int t = 0; t < kPairLoads; ++t) {
            const char *base = t * (kPairThreads / 4) < kPairTileC ? baseC : baseJ;
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void *)(base + so + off[t]),
                (__attribute__((address_space(3))) void *)(smem + buf * kPairStage + (t * kPairThreads + wave * kWave) * 16),
                16, 0, 0);
        }
    };
    f32x4 acc[4][4];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int n = 0; n < 4; ++n) acc[m][n] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    auto multiply = [&](const char *buf) {
        const char *A = buf, *B = buf + kPairTileC * kPairKC;
        const int ra = wm * 64 + r, rb = wn * 64 + r;
        if constexpr (BF16) {
            u32x4 a[4], b[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) a[m] = *reinterpret_cast<const u32x4 *>(A + pair_piece(ra + m * 16, g));
#pragma unroll
            for (int n = 0; n < 4; ++n) b[n] = *reinterpret_cast<const u32x4 *>(B + pair_piece(rb + n * 16, g));
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int n = 0; n < 4; ++n) acc[m][n] = mfma_bf16(a[m], b[n], acc[m][n]);
        } else {
#pragma unroll
            for (int kk = 0; kk < kPairKC / 16; ++kk) {
                float a[4], b[4];
#pragma unroll
                for (int m = 0; m < 4; ++m)
                    a[m] = *reinterpret_cast<const float *>(A + pair_piece(ra + m * 16, kk) + 4 * g);
#pragma unroll
                for (int n = 0; n < 4; ++n)
                    b[n] = *reinterpret_cast<const float *>(B + pair_piece(rb + n * 16, kk) + 4 * g);
#pragma unroll
                for (int m = 0; m < 4; ++m)
#pragma unroll
                    for (int n = 0; n < 4; ++n) acc[m][n] = mfma_f32(a[m], b[n], acc[m][n]);
                __builtin_amdgcn_sched_barrier(0);  // one step's operands in registers at a time
            }
        }
    };
    if (nfull > 0) {
#pragma unroll
        for (int st = 0; st < kPairBufs - 1; ++st) issue(st, st);
    }
    // thresholds of the tile's rows; a row with too many keys takes no more
    for (int x = tid; x < kPairRows; x += kPairThreads) {
        const int64_t row = x < kPairTileC ? c0 + x : j0 + x - kPairTileC;
        float t = __builtin_inff();
        if (row < V && __hip_atomic_load(&count[row], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <= (uint32_t)kPairCap)
            t = thr[row];
        lthr[x] = t;
    }
    int slot = 0;  // buffer of stage st
    for (int st = 0; st < nfull; ++st) {
        // this wave's loads of stage st have landed (those of the stages
        // ahead may be in flight) and its reads of stage st - 1 are done;
        // past the barrier that holds for every wave
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((kPairBufs - 2) * kPairLoads) : "memory");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        issue(st + kPairBufs - 1, slot == 0 ? kPairBufs - 1 : slot - 1);
        multiply(smem + slot * kPairStage);
        slot = slot == kPairBufs - 1 ? 0 : slot + 1;
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
    if (row_bytes % kPairKC) {  // the rest of the rows, zeros past it
#pragma unroll
        for (int t = 0; t < kPairLoads; ++t) {
            const int x = (t * kPairThreads + tid) / 4;
            const int at = nfull * kPairKC + (((tid & 3) ^ ((x >> 2) & 3)) << 4);
            u32x4 v = {0u, 0u, 0u, 0u};
            if (at < row_bytes)
                v = *reinterpret_cast<const u32x4 *>((x < kPairTileC ? baseC : baseJ) + off[t] + nfull * kPairKC);
            *reinterpret_cast<u32x4 *>(smem + (t * kPairThreads + tid) * 16) = v;
        }
        __syncthreads();
        multiply(smem);
        __syncthreads();
    }
    // Sift: lane (r, g) holds rows c 16 m + 4 g + i of its block, row j
    // 16 n + r.  Scores that reach a threshold are listed by the wave (its
    // own part of LDS) and then appended together: the appends of a whole
    // tile share one round trip.
    uint64_t *list = reinterpret_cast<uint64_t *>(smem) + wave * kPairList;
    const float *tcp = lthr + wm * 64 + 4 * g, *tjp = lthr + kPairTileC + wn * 64 + r;
    float tj[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) tj[n] = tjp[16 * n];
    uint32_t nl = 0;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const f32x4 tc = *reinterpret_cast<const f32x4 *>(tcp + 16 * m);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int n = 0; n < 4; ++n) {
                const float sc = acc[m][n][i];
                const bool hc = !(sc < tc[i]), hj = !(sc < tj[n]);
                if (__ballot(hc || hj) == 0ull) continue;
                const uint32_t cl = wm * 64 + 16 * m + 4 * g + i, jl = wn * 64 + 16 * n + r;
                const int64_t c = c0 + cl, j = j0 + jl;
                const bool hit = (hc || hj) && c < j && j < V;  // c < j: every pair once
                const uint64_t mask = __ballot(hit);
                const uint32_t at = nl + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                                   __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
                nl += (uint32_t)__popcll(mask);
                if (!hit) continue;
                if (at < (uint32_t)kPairList) {
                    list[at] = ((uint64_t)__float_as_uint(sc) << 32) | (cl | jl << 8 | (uint32_t)hc << 16 | (uint32_t)hj << 17);
                } else {  // (equal scores beyond the list: rows that take too many keys stop here)
                    if (hc && __hip_atomic_load(&count[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <= (uint32_t)kPairCap)
                        pair_append(c, make_key(sc, (int32_t)j), count, keys);
                    if (hj && __hip_atomic_load(&count[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <= (uint32_t)kPairCap)
                        pair_append(j, make_key(sc, (int32_t)c), count, keys);
                }
            }
    }
    nl = min(nl, (uint32_t)kPairList);
    for (uint32_t e = lane; e < nl; e += kWave) {
        const uint64_t v = list[e];
        const float sc = __uint_as_float((uint32_t)(v >> 32));
        const int64_t c = c0 + (v & 255), j = j0 + (v >> 8 & 255);
        if (v & (1u << 16)) pair_append(c, make_key(sc, (int32_t)j), count, keys);
        if (v & (1u << 17)) pair_append(j, make_key(sc, (int32_t)c), count, keys);
    }
}

// The p-th sampled row: one of the rows p * step .. p * step + step - 1, drawn
// by a hash of p (rows that repeat with a period of the step would all be the
// same kind of row otherwise, and no threshold serve: 65536 x 512 bf16 in 64
// interleaved clusters: 27.4 ms a build with every 32nd row, 7.1).
__device__ __forceinline__ int64_t sampled_row(int64_t p, int step, int64_t V)
{
    const uint32_t h = (uint32_t)p * 0x9E3779B1u;
    return p * step + (h >> 16) % (uint32_t)min<int64_t>(step, V - p * step);
}

// The sampled rows of W_out, gathered (one workgroup a row).
__global__ __launch_bounds__(256) void knn_sample_kernel(const char *__restrict__ W, int64_t V, int row_bytes, int step,
                                                         char *__restrict__ pick)
{
    const int64_t p = blockIdx.x;
    const u32x4 *src = reinterpret_cast<const u32x4 *>(W + sampled_row(p, step, V) * row_bytes);
    u32x4 *dst = reinterpret_cast<u32x4 *>(pick + p * row_bytes);
    for (int c = threadIdx.x; c < row_bytes / 16; c += blockDim.x) dst[c] = src[c];
}

// Threshold of each row of a chunk from its scores against the sampled rows:
// the want-th largest (want <= 64),
// the row itself left out; *full counts the rows whose threshold is reached by
// so many sampled scores that they would take more than twice kPairCap keys.
// One wave per row, no barrier: the want-th largest
// of the 64 lanes' maxima has at least `want` scores at or above it; those
// are listed and ranked (more than kThrCap of them, equal scores: that bound
// itself, still a valid threshold).  Bound by its two reads of the scores, the
// second from the caches: 151936 rows of 4748 scores take 1.0 ms (2.9 GB); a
// histogram of a row in LDS, whose updates meet in a few buckets, took 3.25.
constexpr int kThrWaves = 4;
constexpr int kThrCap = 512;

__global__ __launch_bounds__(kThrWaves *kWave) void knn_threshold_kernel(const float *__restrict__ S, int64_t ld,
                                                                        int64_t r0, int64_t rows, int64_t V, int64_t np,
                                                                        int step, int want, float *__restrict__ thr,
                                                                        uint32_t *__restrict__ full)
{
    __shared__ uint32_t s_list[kThrWaves][kThrCap];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int64_t rr = (int64_t)blockIdx.x * kThrWaves + wave;
    if (rr >= rows) return;
    const int64_t i = r0 + rr;
    const int64_t self = sampled_row(i / step, step, V) == i ? i / step : -1;  // the row's own place in the sample
    const f32x4 *row = reinterpret_cast<const f32x4 *>(S + rr * ld);  // (rows of scores start 16-byte aligned)
    const int64_t n4 = (np + 3) / 4;  // scores past np are in the row's padding, left out below
    // order bits of the scores 4 c .. 4 c + 3 (0 for those left out: no score has these bits but a NaN)
    auto bits = [&](int64_t c, uint32_t(&o)[4]) {
        const f32x4 v = row[c];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const int64_t p = 4 * c + x;
            o[x] = p < np && p != self ? f2ord(v[x]) : 0u;
        }
    };
    uint32_t mx = 0u;
#pragma unroll 4
    for (int64_t c = lane; c < n4; c += kWave) {
        uint32_t o[4];
        bits(c, o);
        mx = max(mx, max(max(o[0], o[1]), max(o[2], o[3])));
    }
    // the want-th largest lane maximum
    uint32_t lo = 0u;
    {
        int above = 0, equal = 0;
        for (int l = 0; l < kWave; ++l) {
            const uint32_t m = (uint32_t)__builtin_amdgcn_readlane((int)mx, l);
            above += m > mx;
            equal += m == mx;
        }
        const uint64_t at = __ballot(above < want && want <= above + equal);  // (never empty: want <= 64)
        lo = (uint32_t)__builtin_amdgcn_readlane((int)mx, __ffsll((long long)at) - 1);
    }
    if (lo == 0u) {  // fewer lanes with a score than wanted: no threshold
        if (lane == 0) thr[i] = -__builtin_inff();
        return;
    }
    uint32_t *list = s_list[wave];
    uint32_t m = 0;
    for (int64_t c0 = 0; c0 < n4; c0 += kWave) {
        uint32_t o[4] = {0u, 0u, 0u, 0u};
        if (c0 + lane < n4) bits(c0 + lane, o);
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const uint64_t hit = __ballot(o[x] >= lo);
            if (hit == 0ull) continue;
            const uint32_t at = m + __builtin_amdgcn_mbcnt_hi((uint32_t)(hit >> 32),
                                                              __builtin_amdgcn_mbcnt_lo((uint32_t)hit, 0u));
            if (o[x] >= lo && at < (uint32_t)kThrCap) list[at] = o[x];
            m += (uint32_t)__popcll(hit);
        }
    }
    if (m > (uint32_t)kThrCap) {
        if (lane == 0) {
            thr[i] = ord2f(lo);
            if (m * (uint32_t)step > 2u * kPairCap) atomicAdd(full, 1u);
        }
        return;
    }
    __builtin_amdgcn_wave_barrier();
    bool found = false;
    for (uint32_t t = lane; t < m; t += kWave) {
        const uint32_t v = list[t];
        int above = 0, equal = 0;
        for (uint32_t u = 0; u < m; ++u) {
            above += list[u] > v;
            equal += list[u] == v;
        }
        // (one lane, or several with equal scores, also 64 places on)
        const uint64_t at = __ballot(above < want && want <= above + equal);
        if (!found && at != 0ull && lane == __ffsll((long long)at) - 1) {
            thr[i] = ord2f(v);
            if ((above + equal) * step > 2 * kPairCap) atomicAdd(full, 1u);
        }
        found |= at != 0ull;
    }
}

// The K best of a row's keys, sorted; a row whose threshold kept fewer than K
// or more than kPairCap is put on the list of rows left.
__global__ __launch_bounds__(kTopkThreads) void knn_pick_kernel(int K, const uint32_t *__restrict__ count,
                                                                const uint64_t *__restrict__ keys,
                                                                int32_t *__restrict__ cand,
                                                                float *__restrict__ cand_score,
                                                                uint32_t *__restrict__ nleft,
                                                                int32_t *__restrict__ left)
{
    __shared__ uint64_t a[kPairCap];
    const int64_t i = blockIdx.x;
    const uint32_t n = count[i];
    if (n < (uint32_t)K || n > (uint32_t)kPairCap) {
        if (threadIdx.x == 0) left[atomicAdd(nleft, 1u)] = (int32_t)i;
        return;
    }
    for (uint32_t t = threadIdx.x; t < n; t += kTopkThreads) a[t] = keys[i * kPairCap + t];
    block_sort_desc<kTopkThreads>(a, (int)n);
    for (int t = threadIdx.x; t < K; t += kTopkThreads) {
        cand[i * K + t] = key_id(a[t]);
        cand_score[i * K + t] = key_logit(a[t]);
    }
}

__global__ __launch_bounds__(kTopkThreads) void knn_topk_kernel(const float *__restrict__ S, int64_t ld,
                                                                const int32_t *__restrict__ list, int64_t r0,
                                                                int64_t V, int K, int32_t *__restrict__ cand,
                                                                float *__restrict__ cand_score)
{
    __shared__ TopkShared sh;
    const int tid = threadIdx.x;
    const int64_t i = list ? list[r0 + blockIdx.x] : r0 + blockIdx.x;
    const float *row = S + (int64_t)blockIdx.x * ld;
    auto key_at = [&](int64_t j) -> uint64_t { return j == i ? 0ull : make_key(row[j], (int32_t)j); };

    // sample: blocks 0, kSampleEvery, 2 kSampleEvery, ... of kTopkThreads scores
    for (int bkt = tid; bkt < kDigitBuckets; bkt += kTopkThreads) sh.hist[bkt] = 0u;
    if (tid == 0) {
        sh.n = 0u;
        sh.bucket = 0u;
        sh.count = 0u;
    }
    __syncthreads();
    // (kSampleBatch sampled blocks per round: their loads are all in flight
    // before the first histogram update)
    // (the next round's loads are issued before this round's updates)
    constexpr int kSampleBatch = 8;
    constexpr int64_t kRound = (int64_t)kSampleBatch * kSampleEvery * kTopkThreads;
    uint32_t ns = 0;
    auto load_round = [&](int64_t j0, float(&x)[kSampleBatch]) {
#pragma unroll
        for (int u = 0; u < kSampleBatch; ++u)
            x[u] = row[min<int64_t>(j0 + (int64_t)u * kSampleEvery * kTopkThreads + tid, V - 1)];
        __builtin_amdgcn_sched_barrier(0);  // keep the issue order
    };
    auto count_round = [&](int64_t j0, const float(&x)[kSampleBatch]) {
#pragma unroll
        for (int u = 0; u < kSampleBatch; ++u) {
            const int64_t jb = j0 + (int64_t)u * kSampleEvery * kTopkThreads, j = jb + tid;
            if (jb < V) ns += (uint32_t)min<int64_t>(kTopkThreads, V - jb);
            if (j < V && j != i) atomicAdd(&sh.hist[(uint32_t)(make_key(x[u], (int32_t)j) >> (64 - kDigitBits))], 1u);
        }
    };
    {
        float xa[kSampleBatch], xb[kSampleBatch];
        load_round(0, xa);
        for (int64_t j0 = 0; j0 < V; j0 += 2 * kRound) {
            load_round(j0 + kRound, xb);
            count_round(j0, xa);
            load_round(j0 + 2 * kRound, xa);
            count_round(j0 + kRound, xb);
        }
    }
    const uint32_t want = (uint32_t)((2 * (int64_t)K * ns + V - 1) / V) + 4;
    __syncthreads();
    {
        constexpr int per = kDigitBuckets / kTopkThreads;
        uint32_t c[per], sum = 0;
#pragma unroll
        for (int j = 0; j < per; ++j) {
            c[j] = sh.hist[kDigitBuckets - 1 - (per * tid + j)];
            sum += c[j];
        }
        uint32_t above = block_exclusive_scan<kTopkThreads>(sum, sh.wsum);
#pragma unroll
        for (int j = 0; j < per; ++j) {
            if (above < want && want <= above + c[j]) {
                sh.bucket = (uint32_t)(kDigitBuckets - 1 - (per * tid + j));
                sh.count = 1u;
            }
            above += c[j];
        }
    }
    __syncthreads();
    // (fewer sampled keys than want: T0 = 1, every key)
    const uint64_t T0 = sh.count ? ((uint64_t)sh.bucket << (64 - kDigitBits)) | 1ull : 1ull;
    // gather every key >= T0, four scores per load: batches of kGatherLoads
    // loads per thread, the next batch issued before the current one is
    // sifted so that the row keeps streaming (indices clamped, no branch
    // around a load; the keys past the row are skipped when sifted)
    constexpr int kGatherLoads = 8;
    constexpr int64_t kBatch = (int64_t)kGatherLoads * kTopkThreads;
    const int64_t n4 = (V + 3) / 4;
    const float4 *row4 = reinterpret_cast<const float4 *>(row);
    auto load_batch = [&](int64_t b0, float4(&v)[kGatherLoads]) {
#pragma unroll
        for (int u = 0; u < kGatherLoads; ++u) v[u] = row4[min(b0 + u * kTopkThreads + tid, n4 - 1)];
        __builtin_amdgcn_sched_barrier(0);  // keep the issue order
    };
    auto sift_batch = [&](int64_t b0, const float4(&v)[kGatherLoads]) {
#pragma unroll
        for (int u = 0; u < kGatherLoads; ++u) {
            const int64_t j = 4 * (b0 + u * kTopkThreads + tid);
            const float x[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (j + e < V && j + e != i) {
                    const uint64_t key = make_key(x[e], (int32_t)(j + e));
                    if (key >= T0) {
                        const uint32_t slot = atomicAdd(&sh.n, 1u);
                        if (slot < (uint32_t)kGatherCap) sh.gat[slot] = key;
                    }
                }
            }
        }
    };
    float4 va[kGatherLoads], vb[kGatherLoads];
    load_batch(0, va);
    for (int64_t b0 = 0; b0 < n4; b0 += 2 * kBatch) {
        load_batch(b0 + kBatch, vb);
        sift_batch(b0, va);
        load_batch(b0 + 2 * kBatch, va);
        sift_batch(b0 + kBatch, vb);
    }
    __syncthreads();
    const uint32_t ng = sh.n;
    int m;
    if (ng >= (uint32_t)K && ng <= (uint32_t)kGatherCap) {
        block_sort_desc<kTopkThreads>(sh.gat, (int)ng);
        m = K;
    } else {
        __syncthreads();
        m = block_topk<kTopkThreads>(V, K, key_at, sh);
    }
    for (int t = tid; t < K; t += kTopkThreads) {
        const uint64_t key = t < m ? sh.gat[t] : 0ull;
        cand[i * K + t] = t < m ? key_id(key) : -1;
        cand_score[i * K + t] = t < m ? key_logit(key) : 0.0f;
    }
}

// Two bf16 products per 32-bit word (the words are passed as plain integers:
// bit-casting a vector lane in place compiled to the first lane here).
__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float acc)
{
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, b), acc,
                                           false);
}

__device__ __forceinline__ float dot16(u32x4 a, u32x4 b, float acc, bool bf16)
{
    const uint32_t a0 = a.x, a1 = a.y, a2 = a.z, a3 = a.w;
    const uint32_t b0 = b.x, b1 = b.y, b2 = b.z, b3 = b.w;
    if (bf16) {
        acc = dot2_bf16(a0, b0, acc);
        acc = dot2_bf16(a1, b1, acc);
        acc = dot2_bf16(a2, b2, acc);
        return dot2_bf16(a3, b3, acc);
    }
    acc = fmaf(__uint_as_float(a0), __uint_as_float(b0), acc);
    acc = fmaf(__uint_as_float(a1), __uint_as_float(b1), acc);
    acc = fmaf(__uint_as_float(a2), __uint_as_float(b2), acc);
    return fmaf(__uint_as_float(a3), __uint_as_float(b3), acc);
}

// Step 2, one workgroup per node: the products of its candidates with each
// other, then the heuristic scan in candidate order by one wave.  A node with
// at most M0 candidates keeps them all.
//
// The scan reads the product of e with an r kept before it only, so of the
// 8 x 8 tiles of 16 x 16 the 36 on and below the diagonal are multiplied,
// nine a wave, fp32 accumulation (the layout of knn_gram_kernel).  Bound by
// the gather of K rows per node through the caches (40 GB a build at 151936 x
// 1024 bf16), so what counts is bytes in flight: stages of kSelKC bytes of
// each candidate go straight to LDS (global_load_lds, 16 bytes a lane), two
// ahead, and the products are kept as a packed triangle over the spent
// stages, so that three workgroups fit a CU.  151936 x 1024 bf16: 4.9 ms (8.2
// TB/s of gathered rows); all 64 tiles from register-staged rows, two
// workgroups a CU and a scan that read one product at a time took 11.2.
// 32768 x 256 fp32: 1.8 ms on the matrix cores (in the sums' order of the
// scores they are compared with), 4.8 on the vector ALUs.
constexpr int kSelKC = 128;       // bytes of a row per stage
constexpr int kSelBufs = 3;
constexpr int kSelStage = kSelectRows * kSelKC;
constexpr int kSelTiles = kSelectRows / 16;
constexpr int kSelWaves = kSelectThreads / kWave;
constexpr int kSelOwn = kSelTiles * (kSelTiles + 1) / 2 / kSelWaves;  // tiles of a wave
static_assert(kSelOwn * kSelWaves * 2 == kSelTiles * (kSelTiles + 1), "tiles divide evenly over the waves");
constexpr int kSelLoads = kSelStage / (16 * kSelectThreads);
constexpr int kSelTri = kSelectRows * (kSelectRows + 1) / 2 * 4;
static_assert(kSelTri <= kSelBufs * kSelStage, "the triangle takes the place of the stages");
constexpr size_t kSelectLds = (size_t)kSelBufs * kSelStage + (size_t)kSelectRows * 8;

// Staged row x holds its 16-byte piece p at p ^ ((x >> 1) & 7): the 16-byte
// operand reads of bf16 rows (16 rows, one piece each of four) leave 5% of the
// LDS cycles to bank conflicts; the 4-byte ones of fp32 rows 46%.
__device__ __forceinline__ int sel_piece(int x, int p) { return x * kSelKC + ((p ^ ((x >> 1) & 7)) << 4); }

// Wave w's tiles: block rows w and 7 - w of the lower triangle, (w + 1) +
// (8 - w) = 9 tiles; its tile t is (m, n) with n <= m.
__device__ __forceinline__ int sel_m(int w, int t) { return t <= w ? w : kSelTiles - 1 - w; }
__device__ __forceinline__ int sel_n(int w, int t) { return t <= w ? t : t - w - 1; }

// Adds a stage's products to the nine tiles of wave W.
template <bool BF16, int W> __device__ __forceinline__ void sel_multiply(const char *buf, int r, int g, f32x4 (&acc)[kSelOwn])
{
    constexpr int NX = kSelTiles - W;  // operands: block rows 0 .. 7 - W (row w of the pair is among them)
    if constexpr (BF16) {
#pragma unroll
        for (int kk = 0; kk < kSelKC / 64; ++kk) {  // 32 columns per step
            u32x4 x[NX];
#pragma unroll
            for (int n = 0; n < NX; ++n) x[n] = *reinterpret_cast<const u32x4 *>(buf + sel_piece(16 * n + r, 4 * kk + g));
#pragma unroll
            for (int t = 0; t < kSelOwn; ++t) acc[t] = mfma_bf16(x[sel_m(W, t)], x[sel_n(W, t)], acc[t]);
        }
    } else {
#pragma unroll
        for (int kk = 0; kk < kSelKC / 16; ++kk) {  // 4 columns per step
            float x[NX];
#pragma unroll
            for (int n = 0; n < NX; ++n) x[n] = *reinterpret_cast<const float *>(buf + sel_piece(16 * n + r, kk) + 4 * g);
#pragma unroll
            for (int t = 0; t < kSelOwn; ++t) acc[t] = mfma_f32(x[sel_m(W, t)], x[sel_n(W, t)], acc[t]);
        }
    }
}

template <bool BF16>
__global__ __launch_bounds__(kSelectThreads) __attribute__((amdgpu_waves_per_eu(3))) void knn_select_kernel(
    const char *__restrict__ W, int row_bytes, int K, int M0, const int32_t *__restrict__ cand,
    const float *__restrict__ cand_score, int32_t *__restrict__ fwd, float *__restrict__ fwd_score,
    int32_t *__restrict__ nfwd)
{
    extern __shared__ __align__(16) char smem[];
    float *G = reinterpret_cast<float *>(smem);  // packed lower triangle, after the stages
    int32_t *cid = reinterpret_cast<int32_t *>(smem + kSelBufs * kSelStage);  // [128]
    float *cs = reinterpret_cast<float *>(cid + kSelectRows);                 // [128]
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int r = lane & 15, g = lane >> 4;
    const int64_t i = blockIdx.x;
    for (int t = tid; t < kSelectRows; t += kSelectThreads) {
        cid[t] = t < K ? cand[i * K + t] : -1;
        cs[t] = t < K ? cand_score[i * K + t] : 0.0f;
    }
    __syncthreads();
    const int nc = __popcll(__ballot(cid[lane] >= 0)) + __popcll(__ballot(cid[lane + kWave] >= 0));  // uniform
    if (nc <= M0) {
        for (int t = tid; t < M0; t += kSelectThreads) {
            fwd[i * M0 + t] = t < nc ? cid[t] : -1;
            fwd_score[i * M0 + t] = t < nc ? cs[t] : 0.0f;
        }
        if (tid == 0) nfwd[i] = nc;
        return;
    }
    // lane (x, p) of load t brings piece p of staged row x (the place of its
    // swizzle); past the candidates the first one again, unused
    const int nfull = row_bytes / kSelKC;
    const char *src[kSelLoads];
    int spiece[kSelLoads];
#pragma unroll
    for (int t = 0; t < kSelLoads; ++t) {
        const int x = (t * kSelectThreads + tid) / 8;
        const int32_t c = cid[x];
        spiece[t] = 16 * ((tid & 7) ^ ((x >> 1) & 7));
        src[t] = W + (int64_t)(c >= 0 ? c : cid[0]) * row_bytes + spiece[t];
    }
    auto issue = [&](int st, int buf) {
        const int64_t so = (int64_t)min(st, nfull - 1) * kSelKC;  // past the end: the last stage again, unused
#pragma unroll
        for (int t = 0; t < kSelLoads; ++t)
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void *)(src[t] + so),
                (__attribute__((address_space(3))) void *)(smem + buf * kSelStage + (t * kSelectThreads + wave * kWave) * 16),
                16, 0, 0);
    };
    f32x4 acc[kSelOwn];
#pragma unroll
    for (int t = 0; t < kSelOwn; ++t) acc[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    auto multiply = [&](const char *buf) {
        switch (wave) {  // uniform in a wave
        case 0: sel_multiply<BF16, 0>(buf, r, g, acc); break;
        case 1: sel_multiply<BF16, 1>(buf, r, g, acc); break;
        case 2: sel_multiply<BF16, 2>(buf, r, g, acc); break;
        default: sel_multiply<BF16, 3>(buf, r, g, acc); break;
        }
    };
    static_assert(kSelWaves == 4, "a case per wave");
    if (nfull > 0) {
#pragma unroll
        for (int st = 0; st < kSelBufs - 1; ++st) issue(st, st);
    }
    int slot = 0;  // buffer of stage st
    for (int st = 0; st < nfull; ++st) {
        // this wave's loads of stage st have landed (those of the stages
        // ahead may be in flight) and its reads of stage st - 1 are done;
        // past the barrier that holds for every wave
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((kSelBufs - 2) * kSelLoads) : "memory");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        issue(st + kSelBufs - 1, slot == 0 ? kSelBufs - 1 : slot - 1);
        multiply(smem + slot * kSelStage);
        slot = slot == kSelBufs - 1 ? 0 : slot + 1;
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
    if (row_bytes % kSelKC) {  // the rest of the rows, zeros past it
#pragma unroll
        for (int t = 0; t < kSelLoads; ++t) {
            u32x4 v = {0u, 0u, 0u, 0u};
            if (nfull * kSelKC + spiece[t] < row_bytes) v = *reinterpret_cast<const u32x4 *>(src[t] + nfull * kSelKC);
            *reinterpret_cast<u32x4 *>(smem + (t * kSelectThreads + tid) * 16) = v;
        }
        __syncthreads();
        multiply(smem);
        __syncthreads();
    }
    // lane (r, g) holds rows 4 g + x of a tile, column r
#pragma unroll
    for (int t = 0; t < kSelOwn; ++t)
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const int e = 16 * sel_m(wave, t) + 4 * g + x, c = 16 * sel_n(wave, t) + r;
            if (c <= e) G[e * (e + 1) / 2 + c] = acc[t][x];
        }
    __syncthreads();
    if (tid < kWave) {
        // heuristic scan: e is kept iff s_e > <w_e, w_r> for every kept r.
        // Lane l holds candidates l and l + 64; their products with the next
        // kScan candidates are read together, before it is known which are
        // kept (entries past e belong to no kept candidate).
        constexpr int kScan = 8;
        const float s0 = cs[lane], s1 = cs[lane + kWave];
        uint64_t k0 = 0ull, k1 = 0ull;  // kept candidates 0 .. 63, 64 .. 127
        int nk = 0;
        for (int e0 = 0; e0 < nc && nk < M0; e0 += kScan) {
            float a[kScan], b[kScan];
#pragma unroll
            for (int u = 0; u < kScan; ++u) {
                const float *row = G + (e0 + u) * (e0 + u + 1) / 2;
                a[u] = row[lane];
                b[u] = row[lane + kWave];
            }
#pragma unroll
            for (int u = 0; u < kScan; ++u) {
                const int e = e0 + u;
                const float se = __uint_as_float((uint32_t)__builtin_amdgcn_readlane(
                    (int)__float_as_uint(e0 < kWave ? s0 : s1), e & (kWave - 1)));
                const uint64_t bad = (__ballot(a[u] >= se) & k0) | (__ballot(b[u] >= se) & k1);
                if (bad == 0ull && e < nc && nk < M0) {
                    if (e0 < kWave) k0 |= 1ull << (e & (kWave - 1));
                    else k1 |= 1ull << (e & (kWave - 1));
                    ++nk;
                }
            }
        }
        const uint64_t below = (1ull << lane) - 1ull;
        const int p0 = __popcll(k0 & below), p1 = __popcll(k0) + __popcll(k1 & below);
        if (k0 >> lane & 1ull) {
            fwd[i * M0 + p0] = cid[lane];
            fwd_score[i * M0 + p0] = s0;
        }
        if (k1 >> lane & 1ull) {
            fwd[i * M0 + p1] = cid[lane + kWave];
            fwd_score[i * M0 + p1] = s1;
        }
        for (int t = nk + lane; t < M0; t += kWave) {
            fwd[i * M0 + t] = -1;
            fwd_score[i * M0 + t] = 0.0f;
        }
        if (lane == 0) nfwd[i] = nk;
    }
}

// Step 3: reverse edges not already forward edges of their target, counted
// per target; each edge's place among its target's (kNoPlace: none) is kept,
// so that the writing pass after the scan (knn_reverse_write_kernel) checks
// and counts nothing again.  Sixteen lanes take sixteen edges: for each, the
// target's list is read across the lanes in whole lines (one lane per edge
// read a line per entry).  Bound by the reads of random lists:
// 151936 nodes of 64 edges take 0.54 ms with the writing pass, where two passes
// of one lane per edge took 2.5.
constexpr uint32_t kNoPlace = 0xFFFFFFFFu;
constexpr int kRevLanes = 16;

__global__ __launch_bounds__(256) void knn_reverse_kernel(int64_t V, int M0, const int32_t *__restrict__ fwd,
                                                          const int32_t *__restrict__ nfwd,
                                                          uint32_t *__restrict__ count, uint32_t *__restrict__ place)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int l = threadIdx.x % kRevLanes, shift = (threadIdx.x & (kWave - 1)) / kRevLanes * kRevLanes;
    int32_t i = -1, j = -1;
    if (e < V * M0) {
        i = (int32_t)(e / M0);
        if (e - (int64_t)i * M0 < nfwd[i]) j = fwd[e];
    }
    const int nj = j >= 0 ? nfwd[j] : 0;
    bool both = false;
#pragma unroll 4
    for (int x = 0; x < kRevLanes; ++x) {
        const int32_t jx = __shfl(j, x, kRevLanes), ix = __shfl(i, x, kRevLanes);
        const int n = __shfl(nj, x, kRevLanes);
        bool f = false;
        for (int t = l; t < n; t += kRevLanes) f |= fwd[(int64_t)jx * M0 + t] == ix;
        const uint64_t any = __ballot(f) >> shift & ((1ull << kRevLanes) - 1ull);
        if (x == l) both = any != 0ull;
    }
    if (e < V * M0) place[e] = j >= 0 && !both ? atomicAdd(&count[j], 1u) : kNoPlace;
}

__global__ __launch_bounds__(256) void knn_reverse_write_kernel(int64_t V, int M0, const int32_t *__restrict__ fwd,
                                                                const float *__restrict__ fwd_score,
                                                                const uint32_t *__restrict__ place,
                                                                const int64_t *__restrict__ roff,
                                                                uint64_t *__restrict__ rev)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= V * M0) return;
    const uint32_t at = place[e];
    if (at != kNoPlace) rev[roff[fwd[e]] + at] = make_key(fwd_score[e], (int32_t)(e / M0));
}

// Exclusive prefix sum of count[0 .. V) into roff[0 .. V] (one workgroup).
__global__ __launch_bounds__(1024) void knn_scan_kernel(const uint32_t *__restrict__ count, int64_t V,
                                                        int64_t *__restrict__ roff)
{
    __shared__ uint32_t wsum[16];
    __shared__ int64_t s_base;
    if (threadIdx.x == 0) s_base = 0;
    __syncthreads();
    for (int64_t b0 = 0; b0 < V; b0 += 1024) {
        const int64_t j = b0 + threadIdx.x;
        const uint32_t v = j < V ? count[j] : 0u;
        const uint32_t ex = block_exclusive_scan<1024>(v, wsum);
        const int64_t base = s_base;
        if (j < V) roff[j] = base + ex;
        __syncthreads();
        if (threadIdx.x == 1023) s_base = base + ex + v;
        __syncthreads();
    }
    if (threadIdx.x == 0) roff[V] = s_base;
}

// Step 4, one workgroup per node: the forward list, then the best reverse
// edges in the free slots.
__global__ __launch_bounds__(kTopkThreads) void knn_lists_kernel(int M0, const int32_t *__restrict__ fwd,
                                                                 const int32_t *__restrict__ nfwd,
                                                                 const int64_t *__restrict__ roff,
                                                                 const uint64_t *__restrict__ rev,
                                                                 int32_t *__restrict__ adj0)
{
    __shared__ TopkShared sh;
    const int64_t j = blockIdx.x;
    const int nf = nfwd[j];
    const int free_slots = M0 - nf;
    const int64_t off = roff[j], nr = roff[j + 1] - off;
    int m = 0;
    if (free_slots > 0 && nr > 0) {
        auto key_at = [&](int64_t t) -> uint64_t { return rev[off + t]; };
        m = block_topk<kTopkThreads>(nr, free_slots, key_at, sh);
    }
    for (int t = threadIdx.x; t < M0; t += kTopkThreads)
        adj0[j * M0 + t] = t < nf ? fwd[j * M0 + t] : t < nf + m ? key_id(sh.gat[t - nf]) : -1;
}

// Step 5: the key (squared norm, id) of every row, the largest kept.  Each
// wave takes rows grid-stride and keeps its best key; the workgroup's best
// goes to *best with one atomic (one per row would serialise on the word).
constexpr int kEntryThreads = 256;
constexpr int kEntryBlocks = 2048;

template <bool BF16>
__global__ __launch_bounds__(kEntryThreads) void knn_entry_kernel(const char *__restrict__ W, int64_t V,
                                                                  int row_bytes, unsigned long long *__restrict__ best)
{
    __shared__ unsigned long long wbest[kEntryThreads / kWave];
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    const int64_t nwaves = (int64_t)gridDim.x * (kEntryThreads / kWave);
    unsigned long long mine = 0ull;
    for (int64_t i = (int64_t)blockIdx.x * (kEntryThreads / kWave) + wv; i < V; i += nwaves) {
        const char *w = W + i * row_bytes;
        float acc = 0.0f;
        for (int c = 16 * lane; c < row_bytes; c += 16 * kWave) {
            const u32x4 v = *reinterpret_cast<const u32x4 *>(w + c);
            acc = dot16(v, v, acc, BF16);
        }
#pragma unroll
        for (int o = kWave / 2; o >= 1; o >>= 1) acc += __shfl_xor(acc, o, kWave);
        const unsigned long long key = make_key(acc, (int32_t)i);
        mine = key > mine ? key : mine;
    }
    if (lane == 0) wbest[wv] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long m = wbest[0];
#pragma unroll
        for (int x = 1; x < kEntryThreads / kWave; ++x) m = wbest[x] > m ? wbest[x] : m;
        if (m) atomicMax(best, m);
    }
}

// The build's scratch (one allocation: hipMalloc and hipFree of a buffer each
// cost host time that the device spends idle) and the graph the index keeps.
struct Buffers {
    void *scratch = nullptr;
    size_t bytes = 0;  // of scratch, while its parts are laid out
    float *S = nullptr;
    int32_t *cand = nullptr, *fwd = nullptr, *nfwd = nullptr, *adj0 = nullptr, *upper_off = nullptr,
            *upper = nullptr;
    float *cand_score = nullptr, *fwd_score = nullptr;
    uint32_t *count = nullptr;
    int64_t *roff = nullptr;
    uint64_t *rev = nullptr;
    unsigned long long *best = nullptr;
    char *sample = nullptr;  // the rows of W_out the fingerprint samples, gathered
    char *pick = nullptr;    // the rows the thresholds are sampled from, gathered
    float *thr = nullptr;    // threshold of every row
    uint32_t *nleft = nullptr;  // number of rows left, then of rows whose sample has too many keys
    int32_t *left = nullptr;  // rows whose threshold did not serve
    // a part of n bytes at the end of the scratch (256-byte aligned)
    template <typename T> void part(T *&p, size_t n)
    {
        p = reinterpret_cast<T *>(static_cast<char *>(scratch) + bytes);
        bytes += (n + 255) & ~(size_t)255;
    }
    void release()
    {
        if (scratch) (void)hipFree(scratch);
        scratch = nullptr;
    }
    void release_graph()
    {
        void *p[] = {adj0, upper_off, upper};
        for (void *q : p)
            if (q) (void)hipFree(q);
        adj0 = upper_off = upper = nullptr;
    }
};

template <typename T>
bool dalloc(T *&p, size_t bytes)
{
    void *q = nullptr;
    if (hipMalloc(&q, bytes < 16 ? 16 : bytes) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    p = static_cast<T *>(q);
    return true;
}

}  // namespace

vie_status build_knn_graph_gpu(const void *W_dev, int dtype, int64_t V, int d, int K, int M0, int64_t chunk_rows,
                               hipStream_t s, Graph &g, DeviceGraph &dg)
{
    const int row_bytes = d * elem_bytes(dtype);
    KnnForm form = knn_form(V, chunk_rows, true);
    if (form.chunk * form.ld > ((int64_t)1 << 31))
        return fail(VIE_EUNSUPPORTED, "GPU build: a score chunk of %lld rows is too large", (long long)form.chunk);
    int dev = 0;
    hipError_t he = hipGetDevice(&dev);
    if (he != hipSuccess) return fail(VIE_EHIP, "hipGetDevice: %s", hipGetErrorString(he));
    const size_t lds = kSelectLds;
    auto sel = dtype == VIE_BF16 ? knn_select_kernel<true> : knn_select_kernel<false>;
    he = hipFuncSetAttribute((const void *)sel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (he != hipSuccess) return fail(VIE_EHIP, "GPU build: %s", hipGetErrorString(he));

    Buffers b;
    const int64_t edges = V * M0;
    // the rows the W_out fingerprint samples: every step-th row, then the last
    const int64_t step = V / 1024 > 1 ? V / 1024 : 1;
    const int64_t nreg = (V + step - 1) / step;
    // the rows the thresholds are sampled from: every pick_step-th
    const int pick_step = (int)std::max<int64_t>(1, std::min<int64_t>(kPairPickStep, V / kPairPickRows));
    const int64_t npick = (V + pick_step - 1) / pick_step;
    // laid out twice: for the size, then in the allocation
    auto lay_out = [&](const KnnForm &f) {
        b.bytes = 0;
        b.part(b.S, f.score_bytes);
        b.part(b.cand, (size_t)V * K * 4);
        b.part(b.cand_score, (size_t)V * K * 4);
        b.part(b.fwd, (size_t)edges * 4);
        b.part(b.fwd_score, (size_t)edges * 4);
        b.part(b.nfwd, (size_t)V * 4);
        b.part(b.count, (size_t)V * 4);
        b.part(b.roff, (size_t)(V + 1) * 8);
        b.part(b.rev, (size_t)edges * 8);
        b.part(b.best, 8);
        b.part(b.sample, (size_t)(nreg + 1) * row_bytes);
        if (f.pairs) {
            b.part(b.pick, (size_t)npick * row_bytes);
            b.part(b.thr, (size_t)V * 4);
            b.part(b.nleft, 8);
            b.part(b.left, (size_t)V * 4);
        }
    };
    const bool ok = knn_first_form(V, chunk_rows, form, [&](const KnnForm &f) {
        lay_out(f);
        bool fits = dalloc(b.scratch, b.bytes);
        if (fits) lay_out(f);
        fits = fits && dalloc(b.adj0, (size_t)edges * 4) && dalloc(b.upper_off, (size_t)V * 4) && dalloc(b.upper, 4);
        if (!fits) {
            b.release();
            b.release_graph();
        }
        return fits;
    });
    if (!ok)
        return fail(VIE_ENOMEM, "GPU build: device allocation failed (V = %lld, chunk of %lld rows)", (long long)V,
                    (long long)form.chunk);
    const bool pairs = form.pairs;
    const int64_t ld = form.ld, R = form.chunk;
    auto bail = [&](vie_status st) {
        (void)hipStreamSynchronize(s);
        b.release();
        b.release_graph();
        return st;
    };

    // the sampled rows of W_out gathered on the device (one strided copy
    // and the last row), then one copy to the host: a copy per row, or a
    // strided copy straight to host memory, took 7-15 ms of host time.  They
    // come first so that they are hashed while the device works.
    std::vector<char> sample((size_t)(nreg + 1) * row_bytes);
    he = hipMemcpy2DAsync(b.sample, (size_t)row_bytes, W_dev, (size_t)step * row_bytes, (size_t)row_bytes, (size_t)nreg,
                          hipMemcpyDeviceToDevice, s);
    if (he == hipSuccess)
        he = hipMemcpyAsync(b.sample + nreg * row_bytes, static_cast<const char *>(W_dev) + (V - 1) * row_bytes,
                            row_bytes, hipMemcpyDeviceToDevice, s);
    if (he == hipSuccess) he = hipMemcpyAsync(sample.data(), b.sample, sample.size(), hipMemcpyDeviceToHost, s);
    if (he == hipSuccess) he = hipStreamSynchronize(s);
    if (he != hipSuccess) return bail(fail(VIE_EHIP, "GPU build: %s", hipGetErrorString(he)));
    // host form of the graph (the index file and vie_index_export read it),
    // made while the device works
    auto host_part = [&]() {
        g = Graph();
        g.V = V;
        g.d = d;
        g.dtype = dtype;
        g.M0 = M0;
        g.M = std::min(M0, std::max(2, M0 / 2));
        g.efC = K;
        g.seed = 0;
        g.maxlevel = 0;
        g.levels.assign((size_t)V, 0);
        g.upper_off.assign((size_t)V, -1);
        g.fingerprint = w_fingerprint_rows(sample.data(), dtype, V, d, nreg + 1);
    };

    const int64_t gram_nj4 = ((V + kGramTile - 1) / kGramTile + 3) / 4 * 4;  // tiles of j, rounded up to 4
    if (gram_nj4 * ((R + kGramTileC - 1) / kGramTileC + 1) > 0x7FFFFFFF)
        return bail(fail(VIE_EUNSUPPORTED, "GPU build: V = %lld rows exceed the Gram grid", (long long)V));
    auto gram = dtype == VIE_BF16 ? knn_gram_kernel<true> : knn_gram_kernel<false>;
    he = hipFuncSetAttribute((const void *)gram, hipFuncAttributeMaxDynamicSharedMemorySize, 2 * kGramStage);
    if (he != hipSuccess) return bail(fail(VIE_EHIP, "GPU build: %s", hipGetErrorString(he)));
    // rows [from, from + rows) (of list, or of W_out) against the nb rows of WB
    auto launch_gram = [&](const int32_t *list, int64_t from, int64_t rows, const char *WB, int64_t nb, int64_t pitch) {
        const int64_t nj4 = ((nb + kGramTile - 1) / kGramTile + 3) / 4 * 4;  // tiles of j, rounded up to 4
        const dim3 grid((unsigned)((((rows + kGramTileC - 1) / kGramTileC + 1) / 2 * 2) * nj4));
        gram<<<grid, kGramThreads, 2 * kGramStage, s>>>(static_cast<const char *>(W_dev), row_bytes, list, from, rows,
                                                        WB, nb, b.S, pitch);
        return hipGetLastError();
    };
    // the top K of listed rows (list NULL: of every row), chunk by chunk
    auto chunked = [&](const int32_t *list, int64_t n) {
        for (int64_t r0 = 0; r0 < n; r0 += R) {
            const int64_t rows = std::min(R, n - r0);
            hipError_t e = launch_gram(list, r0, rows, static_cast<const char *>(W_dev), V, ld);
            if (e != hipSuccess) return e;
            knn_topk_kernel<<<(unsigned)rows, kTopkThreads, 0, s>>>(b.S, ld, list, r0, V, K, b.cand, b.cand_score);
            e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    };
    if (pairs) {
        const char *W = static_cast<const char *>(W_dev);
        uint64_t *keys = reinterpret_cast<uint64_t *>(b.S);
        // sampled scores of every row, in the keys' memory
        he = hipMemsetAsync(b.nleft, 0, 8, s);
        if (he == hipSuccess) {
            knn_sample_kernel<<<(unsigned)npick, 256, 0, s>>>(W, V, row_bytes, pick_step, b.pick);
            he = hipGetLastError();
        }
        const int64_t pld = (npick + 3) & ~(int64_t)3;
        const int64_t PR = std::min<int64_t>(V, (int64_t)(form.score_bytes / (pld * 4)));
        const double mean = (double)K * npick / V;
        // (at most 55: from kPairMinRows rows on at most one row in four is sampled)
        const int want = std::min(kWave, (int)std::ceil(mean + 3.5 * std::sqrt(mean) + 2.0));
        for (int64_t r0 = 0; r0 < V && he == hipSuccess; r0 += PR) {
            const int64_t rows = std::min(PR, V - r0);
            he = launch_gram(nullptr, r0, rows, b.pick, npick, pld);
            if (he != hipSuccess) break;
            knn_threshold_kernel<<<(unsigned)((rows + kThrWaves - 1) / kThrWaves), kThrWaves * kWave, 0, s>>>(
                b.S, pld, r0, rows, V, npick, pick_step, want, b.thr, b.nleft + 1);
            he = hipGetLastError();
        }
        if (he == hipSuccess) he = hipMemsetAsync(b.count, 0, (size_t)V * 4, s);
        if (he == hipSuccess) {
            const int64_t nt = (V + kPairTileC - 1) / kPairTileC;
            const int64_t nsb = (nt + kPairBlock - 1) / kPairBlock;
            const int64_t wgs = (nsb * (nsb + 1) / 2 + 7) / 8 * 8 * kPairBlock * kPairBlock * (kPairTileC / kPairTileJ);
            auto kern = dtype == VIE_BF16 ? knn_pairs_kernel<true> : knn_pairs_kernel<false>;
            he = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kPairLds);
            if (he == hipSuccess) {
                kern<<<(unsigned)wgs, kPairThreads, kPairLds, s>>>(W, V, row_bytes, b.thr, b.nleft + 1, b.count, keys);
                he = hipGetLastError();
            }
        }
        uint32_t nleft = 0;
        if (he == hipSuccess) {
            knn_pick_kernel<<<(unsigned)V, kTopkThreads, 0, s>>>(K, b.count, keys, b.cand, b.cand_score, b.nleft, b.left);
            he = hipGetLastError();
        }
        if (he == hipSuccess) host_part();
        if (he == hipSuccess) he = hipMemcpyAsync(&nleft, b.nleft, 4, hipMemcpyDeviceToHost, s);
        if (he == hipSuccess) he = hipStreamSynchronize(s);
        // (all of them: in their own order, a row of W_out after the other)
        if (he == hipSuccess && nleft > 0) he = chunked(nleft == V ? nullptr : b.left, nleft);
    } else {
        he = chunked(nullptr, V);
    }
    if (he != hipSuccess) return bail(fail(VIE_EHIP, "GPU build: Gram / top-k launch: %s", hipGetErrorString(he)));

    sel<<<(unsigned)V, kSelectThreads, lds, s>>>(static_cast<const char *>(W_dev), row_bytes, K, M0, b.cand,
                                                 b.cand_score, b.fwd, b.fwd_score, b.nfwd);
    he = hipMemsetAsync(b.count, 0, (size_t)V * 4, s);
    const unsigned eg = (unsigned)((edges + 255) / 256);
    if (he == hipSuccess) {
        // (the places sit in the memory of the lists, which come last)
        uint32_t *place = reinterpret_cast<uint32_t *>(b.adj0);
        knn_reverse_kernel<<<eg, 256, 0, s>>>(V, M0, b.fwd, b.nfwd, b.count, place);
        knn_scan_kernel<<<1, 1024, 0, s>>>(b.count, V, b.roff);
        knn_reverse_write_kernel<<<eg, 256, 0, s>>>(V, M0, b.fwd, b.fwd_score, place, b.roff, b.rev);
        knn_lists_kernel<<<(unsigned)V, kTopkThreads, 0, s>>>(M0, b.fwd, b.nfwd, b.roff, b.rev, b.adj0);
        he = hipMemsetAsync(b.best, 0, 8, s);
    }
    if (he == hipSuccess) {
        const unsigned eb = (unsigned)std::min<int64_t>((V + 3) / 4, kEntryBlocks);
        if (dtype == VIE_BF16)
            knn_entry_kernel<true><<<eb, kEntryThreads, 0, s>>>(static_cast<const char *>(W_dev), V, row_bytes, b.best);
        else
            knn_entry_kernel<false><<<eb, kEntryThreads, 0, s>>>(static_cast<const char *>(W_dev), V, row_bytes, b.best);
        he = hipMemsetAsync(b.upper_off, 0xFF, (size_t)V * 4, s);  // every node on layer 0 only: -1
    }
    if (he == hipSuccess) he = hipGetLastError();
    if (he != hipSuccess) return bail(fail(VIE_EHIP, "GPU build: %s", hipGetErrorString(he)));

    // (the layer-0 lists stay on the device: the index copies them to the
    // host when a host-side call first needs them)
    if (!pairs) host_part();
    unsigned long long best = 0;
    he = hipMemcpyAsync(&best, b.best, 8, hipMemcpyDeviceToHost, s);
    if (he == hipSuccess) he = hipStreamSynchronize(s);
    if (he != hipSuccess) return bail(fail(VIE_EHIP, "GPU build: %s", hipGetErrorString(he)));
    g.entry = (int32_t)(~(uint32_t)best);
    b.release();

    dg = DeviceGraph();
    dg.device = dev;
    dg.W = W_dev;
    dg.adj0 = b.adj0;
    dg.upper_off = b.upper_off;
    dg.upper = b.upper;
    return VIE_OK;
}

}  // namespace vie

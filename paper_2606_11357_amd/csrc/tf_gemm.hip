// Prefill GEMM: which of the three tiled kernels computes a call (Section 2.1;
// Section 4.3 "GEMM microkernel"), and the workspace its entry points promise.
//   gemm256_kernel  256 x 256 tiles, one weight step dequantized per 256 rows
//   gemm_ks_kernel  64 x 128 and 64 x 256 tiles, K split over the workgroup's
//                   waves, whole 128-row chunks and groups of a power of two
//   gemm_kq_kernel  128 x 128 and 64 x 64 tiles, K split over the workgroup's
//                   waves and, with a workspace, over workgroups; any K, group
#include <algorithm>

#include "tf_internal.h"

namespace tf {
namespace {

// Expected time of each candidate in nanoseconds: rounds of workgroups, one
// per compute unit, each a fixed part (launch, first loads, sums, stores) and
// a part per row of K.  Fitted on MI355X (graph replay, W4 and W8, fp16 and
// bf16, M = 40 .. 3072 on (K, N) = (4096, 14336), (14336, 4096), (4096, 4096),
// (2048, 2048), (2048, 11008), (11008, 2048)), good to about 10%: enough to
// pick the faster kernel wherever the choice matters.  Measured at a round of
// K = 4096 (fp16): 64 x 64 tiles 12.5, 64 x 128 19, 64 x 256 34, 128 x 128 31,
// 256 x 256 90 us; a partly filled round costs nearly a full one, so the small
// tiles win while one round of them covers C (K = N = 4096, M = 128 W8: 12.8
// against 18.7 us) and the large ones where each covers more (M = 1000,
// N = 28672: 256 x 256 tiles 179 against 234 us with tiles of 128 x 256).
int64_t rounds(int64_t units, int64_t cus) { return (units + cus - 1) / cus; }
int64_t tiles_of(const Layout& L, int64_t M, int64_t bm, int64_t bn) {
    return ((M + bm - 1) / bm) * ((L.N + bn - 1) / bn);
}

int64_t kq_cost(const Layout& L, int64_t M, int rb, int64_t S, int64_t cus) {
    const int64_t units = tiles_of(L, M, 16 * rb, 16 * rb) * S, r = rounds(units, cus);
    const int64_t k = (L.K + S - 1) / S;
    // picoseconds per row of K; the large tile slows down as more of the chip
    // works (4.8 ns on a quarter of the compute units, 6.3 on all)
    const int64_t fixed = rb == 8 ? 6300 : 4000, per_k = rb == 8 ? 4800 + 1500 * units / (r * cus) : 2050;
    // partial tiles written and read back by the second launch
    const int64_t sum = S > 1 ? 2500 + units * (rb * rb * 1024) / 8000 : 0;
    return r * (fixed + per_k * k / 1000) + sum;
}

// Promised workspace (tf_workspace_bytes) of M > kSkinnyMaxM rows: the 256-row
// GEMM's stream-K from M = 1024, or M = 256 where K is long; below that, room
// for partial tiles where tiles of 128 x 256 are few (none where the K-split
// GEMM covers the call).  A plan never uses more than this, so that a buffer
// of the promised size serves whichever kernel a call takes.
constexpr int64_t kGemm256MinM = 1024, kGemm256MinMLongK = 256, kLongK = 8192;
bool gemm256_size(const Layout& L, int64_t M) {
    return gemm256_supported(L) && (M >= kGemm256MinM || (M >= kGemm256MinMLongK && L.K >= kLongK));
}
constexpr int64_t kKsMaxTiles = 1200, kKsMinTilesLongK = 192;
bool ks_size(const Layout& L, int64_t M) {
    const int64_t tiles = tiles_of(L, M, 64, 128);
    return gemm_ks_supported(L) && tiles <= kKsMaxTiles && (L.K <= kLongK || tiles >= kKsMinTilesLongK);
}
int64_t split_bytes(const Layout& L, int64_t M) {
    constexpr int64_t kBM = 128, kBN = 256, kTarget = 256, kMinSliceChunks = 4, kMaxSplit = 8;
    const int64_t tiles = tiles_of(L, M, kBM, kBN), chunks = L.K / 128;
    if (L.K % 128 != 0 || (L.group & (L.group - 1)) != 0 || tiles >= kTarget) return 0;
    int64_t S = std::min((kTarget + tiles - 1) / tiles, chunks / kMinSliceChunks);
    S = std::max<int64_t>(std::min(S, kMaxSplit), 1);
    const int64_t cps = (chunks + S - 1) / S;
    S = (chunks + cps - 1) / cps;
    return S <= 1 ? 0 : kWsCounterBytes + tiles * S * (kBM * kBN * 4);
}

// Workspace a (rb, S) plan needs.
int64_t kq_bytes(const Layout& L, int64_t M, int rb, int64_t S) {
    return S <= 1 ? 0 : kWsCounterBytes + tiles_of(L, M, 16 * rb, 16 * rb) * S * (rb * rb * 1024);
}

struct KqPlan {
    int rb, S;
    int64_t cost;
};
// The best tile and K split whose partial tiles fit `room` bytes.  A slice
// keeps at least 1024 rows of K: shorter ones leave a wave of the 64 x 64
// tile fewer than four steps.
KqPlan plan_kq(const Layout& L, int64_t M, int64_t room, int64_t cus) {
    KqPlan best{0, 0, INT64_MAX};
    for (const int rb : {4, 8})
        for (int S = 1; S <= 8; S *= 2) {
            if (S > 1 && (L.K / S < 1024 || kq_bytes(L, M, rb, S) > room)) break;
            const int64_t c = kq_cost(L, M, rb, S, cus);
            if (c < best.cost) best = {rb, S, c};
        }
    return best;
}

}  // namespace

int64_t gemm_workspace_bytes(const Layout& L, int64_t M) {
    if (M <= kSkinnyMaxM) return skinny_workspace_bytes(L, M);
    if (gemm256_size(L, M)) return gemm256_workspace_bytes(L, M);
    return ks_size(L, M) ? 0 : split_bytes(L, M);
}

int launch_gemm(const Layout& L, const uint16_t* A, const void* packed, uint16_t* C, int64_t M,
                void* ws, size_t ws_bytes, hipStream_t s, bool bf) {
    const uint8_t* pk = static_cast<const uint8_t*>(packed);
    const int64_t cus = device_cus(s);
    const int64_t room = ws ? std::min((int64_t)ws_bytes, gemm_workspace_bytes(L, M)) : 0;
    const KqPlan kq = plan_kq(L, M, room, cus);
    constexpr int64_t kNever = INT64_MAX / 16;
    const int64_t ks = gemm_ks_supported(L) ? gemm_ks_cost(L, M, cus, bf) : kNever;
    const int64_t g256 = gemm256_supported(L) ? gemm256_cost(L, M, room, cus, bf) : kNever;
    if (g256 <= ks && g256 <= kq.cost)
        return launch_gemm256(L, A, pk, C, M, room ? ws : nullptr, room, s, bf);
    // within the model's error (an eighth) the K-split kernel keeps the call
    if (8 * ks <= 9 * kq.cost) return launch_gemm_ks(L, A, pk, C, M, s, bf);
    return launch_gemm_kq(L, A, pk, C, M, kq.rb, kq.S, ws, s, bf);
}

}  // namespace tf

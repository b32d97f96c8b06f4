// Prefill GEMM: which of the four tiled kernels computes a call (Section 2.1;
// Section 4.3 "GEMM microkernel"), and the workspace its entry points promise.
//   gemm256_kernel  256 x 256 tiles, one weight step dequantized per 256 rows
//   gemm_ks_kernel  64 x 128 and 64 x 256 tiles, K split over the workgroup's
//                   waves, whole 128-row chunks and groups of a power of two
//   gemm_kq_kernel  128 x 128 and 64 x 64 tiles, K split over the workgroup's
//                   waves and, with a workspace, over workgroups; any K, group
//   gemm_any_kernel 128 x 128 tiles without a pipeline, for short K; any K, group
// The kernel with the shortest expected time (in microseconds) runs.
#include <algorithm>

#include "tf_internal.h"

namespace tf {
namespace {

int64_t tiles_of(const Layout& L, int64_t M, int64_t bm, int64_t bn) {
    return ((M + bm - 1) / bm) * ((L.N + bn - 1) / bn);
}

}  // namespace

// The model of a tiled kernel with one workgroup per compute unit.  A round of
// workgroups takes a fixed time (first loads, sums, stores) and then the
// longer of its steps and its loads: consecutive workgroups of an XCD share
// rows of A or columns of weights, and what its 32 (or fewer) workgroups read
// between them comes from outside its L2.  All rounds together take at least
// the time of one read of the operands from memory.
// Why a model and not a line per kernel: a partly filled round costs nearly a
// full one, so which kernel is faster changes back and forth with every
// dimension (K = N = 4096, M = 128 W8: 64 x 64 tiles 12.8 us against 18.7 with
// 64 x 128; M = 1500, K = 11008, N = 2048 W8: 128 x 128 73 against 88 with
// 256 x 256).
// Fitted on MI355X to 18000 timings of single kernels (graph replay over three
// copies of the operands): M = 65 .. 3400, K = 400 .. 32768, N = 256 .. 32768,
// groups of 32 to 256, both widths and types.  Where a kernel is within 35%
// of the best one its expected time is within 5 to 9% in nine of ten cases
// and 25% in all; the kernel chosen is 0.1% (geometric mean) slower than the best
// one, at most 19%.  (As rounds of a fixed time, without width, type, loads and
// the kernel for short K: 1.7%, at most 96%.)
double tiled_cost(const TileCost& c, const Layout& L, int64_t M, int64_t bm, int64_t bn, int64_t S, int64_t cus,
                  bool bf, bool whole_groups) {
    const int64_t tm = (M + bm - 1) / bm, tn = (L.N + bn - 1) / bn, units = tm * tn * S;
    const double k = (double)L.K / (double)S, wbytes = L.bits / 8.0;
    const double per_k = c.per_k[(L.bits == 8 ? 2 : 0) + (bf ? 1 : 0)] * (whole_groups ? 1.0 : c.small_group);
    auto round_us = [&](int64_t u) {
        const int64_t n = (u + 7) / 8, dm = std::min(n, tm), dn = (n + tm - 1) / tm;
        const double loads = 8.0 * k * ((double)(dm * bm) * 2.0 + (double)(dn * bn) * wbytes);
        const double idle = c.idle * (1.0 - (double)u / (double)cus);
        return c.round + std::max(per_k * (1.0 - idle) * k * 1e-3, loads / c.load_tbs * 1e-6);
    };
    const int64_t full = (units - 1) / cus;
    const double t = c.start + (double)full * round_us(cus) + round_us(units - full * cus);
    const double once = 2.0 * (double)M * (double)(L.K + L.N) + (double)L.K * (double)L.N * wbytes;
    return std::max(t, c.start + c.round + once / c.once_tbs * 1e-6);
}

namespace {

// gemm_kq_kernel: one K slice; with more, the partial tiles are written and
// read back by the second launch.
constexpr TileCost kKq64{1.8, 3.6, 1.23, 6.8, 0.31, 4.3, {2.19, 2.36, 2.63, 2.68}};
constexpr TileCost kKq128{2.5, 7.5, 1.15, 6.4, 0.32, 4.1, {6.40, 6.57, 7.33, 7.33}};
double kq_cost(const Layout& L, int64_t M, int rb, int64_t S, int64_t cus, bool bf) {
    const int64_t b = 16 * rb;
    const double t = tiled_cost(rb == 8 ? kKq128 : kKq64, L, M, b, b, S, cus, bf, L.na % 4 == 0 && L.group % 128 == 0);
    if (S == 1) return t;
    const double part = (double)(tiles_of(L, M, b, b) * S) * (double)(b * b * 4);
    return t + (rb == 8 ? 2.0 : 2.4) + part / (rb == 8 ? 5.0 : 5.2) * 1e-6;
}

// gemm_any_kernel: four workgroups share a compute unit; the first sets the
// time that a batch of four waits for its loads, the others what they add.
double any_cost(const Layout& L, int64_t M, int64_t cus, bool bf) {
    constexpr double kFirst[4] = {20.0, 19.8, 20.0, 26.8};       // ns per row of K
    const double k = (double)L.K * 1e-3, first = kFirst[(L.bits == 8 ? 2 : 0) + (bf ? 1 : 0)] * k;
    const int64_t tiles = tiles_of(L, M, 128, 128), batch = 4 * cus, full = tiles / batch;
    auto batch_us = [&](int64_t deep) { return deep ? first + (double)(deep - 1) * (0.5 + 8.5 * k) : 0.0; };
    return 5.4 + (double)full * batch_us(4) + batch_us((tiles - full * batch + cus - 1) / cus);
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

constexpr double kNever = 1e30;
struct KqPlan {
    int rb, S;
    double cost;
};
// The best tile and K split whose partial tiles fit `room` bytes.  A slice
// keeps at least 1024 rows of K: shorter ones leave a wave of the 64 x 64
// tile fewer than four steps.
KqPlan plan_kq(const Layout& L, int64_t M, int64_t room, int64_t cus, bool bf) {
    KqPlan best{0, 0, kNever};
    for (const int rb : {4, 8})
        for (int S = 1; S <= 8; S *= 2) {
            if (S > 1 && (L.K / S < 1024 || kq_bytes(L, M, rb, S) > room)) break;
            const double c = kq_cost(L, M, rb, S, cus, bf);
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
    const KqPlan kq = plan_kq(L, M, room, cus, bf);
    const double ks = gemm_ks_supported(L) ? gemm_ks_cost(L, M, cus, bf) : kNever;
    const double g256 = gemm256_supported(L) ? gemm256_cost(L, M, room, cus, bf) : kNever;
    const double any = any_cost(L, M, cus, bf);
    const double best = std::min(std::min(kq.cost, ks), std::min(g256, any));
    if (g256 == best) return launch_gemm256(L, A, pk, C, M, room ? ws : nullptr, room, s, bf);
    if (ks == best) return launch_gemm_ks(L, A, pk, C, M, s, bf);
    if (any == best) return launch_gemm_any(L, A, pk, C, M, s, bf);
    return launch_gemm_kq(L, A, pk, C, M, kq.rb, kq.S, ws, s, bf);
}

}  // namespace tf

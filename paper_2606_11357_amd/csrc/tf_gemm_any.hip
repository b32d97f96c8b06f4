// Prefill GEMM for short K (Section 2.1; Section 4.3 "GEMM microkernel"):
//   C[M, N] = A[M, K] x dequant(packed)[K, N], any K and group.
// 128 x 128 tiles, four waves of 64 x 64, 32-row steps through one 8 KB LDS
// buffer.  It keeps nothing in flight across a step; several workgroups share
// a compute unit instead and hide each other's loads, and a tile starts and
// ends without a ring to fill or partial sums to add.  With few steps that is
// the larger part of a tile's time in the pipelined kernels, which run one
// workgroup per compute unit.
// Measured on MI355X (graph replay, us) against gemm_kq_kernel, which
// otherwise serves any K and group (4-bit): 2128 x 608 x 14664 groups of 32, bf16 109 -> 67,
// 2547 x 864 x 14776 groups of 96 154 -> 98, 1478 x 480 x 5752 33.4 -> 22.7;
// with longer K it waits for every step's loads (4096 rows: 85 us for one tile)
// and the pipelined kernels win.
#include "tf_internal.h"

namespace tf {
namespace {

constexpr int kAnyBM = 128, kAnyBN = 128, kAnyBK = 32;
constexpr int kAnyThreads = 256;

template <int BITS, bool BF>
__global__ __launch_bounds__(kAnyThreads) void gemm_any_kernel(
    const uint16_t* __restrict__ A, const uint8_t* __restrict__ packed, uint16_t* __restrict__ C,
    int M, int K, int N, int group, int64_t s_off, int64_t z_off, int na, int ng, int np) {
    constexpr int PW = BITS == 4 ? 64 : 32;
    constexpr int T = PW / 16;
    __shared__ u32x4 As[kAnyBM * kAnyBK / 8];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int c = lane & 15, kg = lane >> 4;
    const int64_t row0 = (int64_t)blockIdx.y * kAnyBM;
    const int64_t col0 = (int64_t)blockIdx.x * kAnyBN;
    const uint32_t magic = magic_reg();

    float4_t acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[i][t] = float4_t{0.f, 0.f, 0.f, 0.f};

    constexpr int kPanels = 64 / PW;
    const uint16_t* sreg = reinterpret_cast<const uint16_t*>(packed + s_off);
    const uint8_t* zreg = packed + z_off;

    for (int a = 0; a < na; ++a) {
        u32x4 av[2];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int idx = tid + kAnyThreads * r;
            const int row = lds_a_row(idx), ch = lds_a_chunk(idx);   // the chunk slot idx holds
            const int64_t grow = row0 + row;
            av[r] = grow < M ? *reinterpret_cast<const u32x4*>(A + grow * K + (int64_t)a * kAnyBK + ch * 8)
                             : u32x4{0u, 0u, 0u, 0u};
        }
        u32x4 b[4];
        const int g = (a * kAnyBK) / group;
#pragma unroll
        for (int pp = 0; pp < kPanels; ++pp) {
            const int64_t panel = col0 / PW + wn * kPanels + pp;
            u32x4 wv = u32x4{0u, 0u, 0u, 0u};
            uint16_t sb[T];
            uint8_t zb[T];
#pragma unroll
            for (int t = 0; t < T; ++t) {
                sb[t] = 0;
                zb[t] = 0;
            }
            if (panel < np) {
                wv = reinterpret_cast<const u32x4*>(packed)[(panel * na + a) * 64 + lane];
                const int64_t meta = (panel * ng + g) * PW + c * T;
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    sb[t] = sreg[meta + t];
                    zb[t] = zreg[meta + t];
                }
            }
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const DqConst<BF> kq = make_dq_const<BF>(sb[t], zb[t]);
                if constexpr (BITS == 4)
                    b[t] = dq_operand<BF, 4>(wv[t], 0u, magic, kq);
                else
                    b[pp * T + t] = dq_operand<BF, 8>(wv[2 * t], wv[2 * t + 1], magic, kq);
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int idx = tid + kAnyThreads * r;
            As[idx] = av[r];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const u32x4 af = As[lds_a_slot(wm * 64 + 16 * i + c, kg)];
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[i][t] = mfma16<BF>(af, b[t], acc[i][t]);
        }
    }

#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int64_t col = col0 + wn * 64 + 16 * t + c;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t row = row0 + wm * 64 + 16 * i + 4 * kg + r;
                if (row < M && col < N)
                    C[row * N + col] = round_out<BF>(acc[i][t][r]);
            }
        }
}

}  // namespace

int launch_gemm_any(const Layout& L, const uint16_t* A, const void* packed, uint16_t* C, int64_t M,
                    hipStream_t s, bool bf) {
    const uint8_t* pk = static_cast<const uint8_t*>(packed);
    const dim3 grid((unsigned)((L.N + kAnyBN - 1) / kAnyBN), (unsigned)((M + kAnyBM - 1) / kAnyBM));
    if (log_enabled())
        log_plan("gemm_any_kernel<%d,%s> M=%lld K=%lld N=%lld G=%d: %ux%u tiles of 128x128", L.bits,
                 bf ? "bf16" : "f16", (long long)M, (long long)L.K, (long long)L.N, L.group, grid.y, grid.x);
    auto go = [&](auto kernel) {
        return launch(kernel, grid, dim3(kAnyThreads), 0, s, A, pk, C, (int)M, (int)L.K, (int)L.N, L.group,
                      L.s_off, L.z_off, (int)L.na, (int)L.ng, (int)L.np);
    };
    if (L.bits == 4) return bf ? go(gemm_any_kernel<4, true>) : go(gemm_any_kernel<4, false>);
    return bf ? go(gemm_any_kernel<8, true>) : go(gemm_any_kernel<8, false>);
}

}  // namespace tf

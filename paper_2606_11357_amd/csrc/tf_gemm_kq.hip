// Prefill GEMM for middle sizes and for every K and group the packed format
// takes (Section 2.1; Section 4.3 "GEMM microkernel"; Section 4.4):
//   C[M, N] = A[M, K] x dequant(packed)[K, N], fp16 or bf16 MFMA, fp32 sums.
//
// Workgroup tile 128 x 128 (RB = NB = 8, four waves, one per SIMD, 256
// accumulators each) or 64 x 64 (RB = NB = 4, eight waves, two per SIMD); each
// wave computes the whole tile over its own part of the workgroup's K range,
// the parts are added through LDS in wave order, and, where the tiles alone
// leave compute units idle and a workspace is given, K is first cut into S
// slices of one workgroup each, whose fp32 tiles a second launch adds in
// slice order (bitwise reproducible).  Inside the loop the waves share
// nothing and never wait for each other.
//  - A goes through a private LDS ring of RING buffers per wave, each one pair
//    of 32-row steps (16 RB rows x 128 bytes, whole cache lines), by direct
//    global-to-LDS loads; the pair RING ahead is requested in the step after
//    a buffer's last fragments were read.
//  - The packed atoms of the tile's panels go into a register ring of four
//    steps; a group's metadata is loaded two to four steps ahead.
//  - A step's MFMAs run column block by column block; while the RB MFMAs of
//    block u run, the wave dequantizes (Eq. 2, rounded once, the code of the
//    other GEMMs) the B operand of block u + 1.  With RB = 8 an operand of 13
//    (bf16: 19) vector instructions covers eight MFMAs, half of what the
//    64-row tiles of gemm_ks_kernel pay per MFMA.
//  - K need only be a multiple of 32 and a group of 32: steps are dealt to
//    the waves in pairs, the last one to three steps of a run follow the loop,
//    and G4 = false tracks groups of any size with a scalar counter.  G4 = true
//    (whole 128-row chunks, groups of 128 or more in multiples of it) fixes
//    the steps that open a group at compile time.
// What bounds it (wall-clock stamps on MI355X, K = 4096, N = 14336): 128 x 128,
// M = 256: 2.4 us to the first data, 0.75 us a step of 64 MFMAs (0.45 at the
// matrix core's rate; a copy without loads 0.7, without MFMAs 0.54: one wave
// issues everything, at about 5 cycles an instruction), 4.2 us to add and store
// the parts.  64 x 64, M = 64: one wave per SIMD took 0.36 us a step, two
// take 0.25 each pair (12.0 -> 7.9 us the loop), since one wave's matrix
// instructions then run under the other's vector work.
// Measured against what served these calls otherwise (graph replay, fp16, us):
// 333 x 1376 x 2048 groups of 32 (a 128 x 128 kernel for any group, single
// buffered) 33.9 -> 8.6; 64 x 4096 x 14336 (streaming form) 25.4 -> 12.8, W8
// 46 -> 17; 200 x 14336 x 4096 (128 x 256 tiles, split K) 47.8 -> 33.2;
// bf16 512 x 4096 x 14336 (64 x 256 tiles) 78 -> 61.4.
#include <algorithm>

#include "tf_internal.h"

namespace tf {
namespace {

constexpr int kKqBK = 32;
constexpr int kKqXcds = 8;
constexpr int kKqNR = 4;                // atom ring slots = steps of an unrolled pass
constexpr int kKqMetaLead = 2;          // steps between a step's metadata request and it (G4 = false)

// Buffer and ring sizes of one tile shape.
template <int RB, int NB>
struct KqCfg {
    static constexpr int WAVES = RB == 8 ? 4 : 8;
    static constexpr int RING = 2;                         // A buffers (pairs of steps) per wave
    static constexpr int PAIR_BYTES = 16 * RB * 128;
    static constexpr int SUMB = NB < 2 * RING ? NB : 2 * RING;   // column blocks per pass of the waves' sum
};

// The vector-memory operations a wave issues around step t (negative t: the
// prologue issues them in the same order), in the order metadata, atoms,
// direct loads of A: what a counted wait leaves in flight.
template <int RB, int PANELS, int RING, bool G4>
struct KqOps {
    static constexpr int NR = kKqNR;
    static constexpr int meta(int t) {
        return (G4 ? (t >= -4 && ((t % 4) + 4) % 4 == 0) : t >= -kKqMetaLead) ? 2 * PANELS : 0;
    }
    static constexpr int atoms(int t) { return t >= -(NR - 1) ? PANELS : 0; }
    static constexpr int dma(int t) { return (t & 1) && t >= 1 - 2 * RING ? 2 * RB : 0; }
    static constexpr int all(int t) { return meta(t) + atoms(t) + dma(t); }
    // At the end of odd step t's requests: operations issued after the last
    // direct load of the pair that step t + 1 reads (requested in odd step
    // t + 2 - 2 RING).
    static constexpr int after_pair(int t) {
        int n = 0;
        for (int s = t + 3 - 2 * RING; s <= t; ++s) n += all(s);
        return n;
    }
    // the same for the unrolled step j: its first pass and its later ones
    static constexpr int wait(int j) {
        const int a = after_pair(j), b = after_pair(j + 8 * NR);
        return a < b ? a : b;
    }
    // in the prologue, after pair 0's: only the later pairs' are counted (the
    // compiler may move the other loads, which it waits for itself)
    static constexpr int wait0() { return (RING - 1) * 2 * RB; }
};

template <int OFF>
__device__ __forceinline__ u32x4 kq_read16(uint32_t addr) {
    u32x4 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "i"(OFF));
    return v;
}
// fragment of row block i (16 rows x 128 bytes = 2 KB apart)
__device__ __forceinline__ u32x4 kq_read_block(uint32_t addr, int i) {
    switch (i) {
        case 0: return kq_read16<0 * 2048>(addr);
        case 1: return kq_read16<1 * 2048>(addr);
        case 2: return kq_read16<2 * 2048>(addr);
        case 3: return kq_read16<3 * 2048>(addr);
        case 4: return kq_read16<4 * 2048>(addr);
        case 5: return kq_read16<5 * 2048>(addr);
        case 6: return kq_read16<6 * 2048>(addr);
        default: return kq_read16<7 * 2048>(addr);
    }
}
__device__ __forceinline__ void kq_lgkm_wait() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
// At most n vector-memory operations in flight (n known at compile time; the
// counter has 6 bits, a smaller count only waits for more).
template <int N>
__device__ __forceinline__ void kq_vm_wait() {
    constexpr int n = N < 63 ? N : 63;
    asm volatile("s_waitcnt vmcnt(%0)" ::"i"(n) : "memory");
}
template <typename V>
__device__ __forceinline__ void kq_tie(V& v) { asm volatile("" : "+v"(v)); }

__device__ __forceinline__ u32x4 kq_load128(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}

struct KqSplit {
    int S;              // K slices (1: none)
    float4_t* part;     // S > 1: one fp32 tile per (slice, tile)
};

template <int BITS, bool BF, int RB, int NB, bool G4>
__global__ __launch_bounds__((64 * KqCfg<RB, NB>::WAVES), 1) void gemm_kq_kernel(
    const uint16_t* __restrict__ A, const uint8_t* __restrict__ packed, uint16_t* __restrict__ C,
    int M, int K, int N, int apg, int64_t s_off, int64_t z_off, int na, int ng, int np,
    int tiles_m, int tiles_n, KqSplit sk) {
    using Cfg = KqCfg<RB, NB>;
    constexpr int PW = BITS == 4 ? 64 : 32;   // columns per panel (one atom per step)
    constexpr int T = PW / 16;                // column blocks per panel
    constexpr int BN = 16 * NB, BM = 16 * RB;
    constexpr int PANELS = BN / PW;
    constexpr int WAVES = Cfg::WAVES, RING = Cfg::RING, PAIR_BYTES = Cfg::PAIR_BYTES, SUMB = Cfg::SUMB;
    constexpr int DQ = dq_steps<BF, BITS>();
    using Ops = KqOps<RB, PANELS, RING, G4>;
    constexpr int NR = kKqNR;
    static_assert((RING & (RING - 1)) == 0 && NR == 4, "ring indices");
    __shared__ __align__(16) uint8_t lds[WAVES * RING * PAIR_BYTES];
    static_assert(WAVES * RB * SUMB * 1024 <= (int)sizeof(lds), "a pass of the sum fits the rings' storage");

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, kg = lane >> 4;
    const uint32_t magic = magic_reg();

    // Block b runs on XCD b % 8, which takes the (b % 8)-th contiguous band of
    // the list of units: K slice by K slice, row tiles varying fastest, so a
    // band shares its weight columns and its part of A.
    int unit;
    {
        const int total = tiles_m * tiles_n * sk.S;
        const int b = blockIdx.x;
        const int per = total / kKqXcds, rem = total % kKqXcds;
        const int x = b % kKqXcds, i = b / kKqXcds;
        unit = x * per + min(x, rem) + i;
    }
    const int tm = __builtin_amdgcn_readfirstlane(unit % tiles_m);
    const int tn = __builtin_amdgcn_readfirstlane(unit / tiles_m % tiles_n);
    const int slice = __builtin_amdgcn_readfirstlane(unit / (tiles_m * tiles_n));
    const int64_t row0 = (int64_t)tm * BM, col0 = (int64_t)tn * BN;

    // K ranges in blocks of KB steps (a chunk, or a pair): the slice's, then
    // this wave's part of it; possibly empty.
    constexpr int KB = G4 ? 4 : 2;
    const int nblk = (na + KB - 1) / KB;
    const int sb0 = (int)((int64_t)slice * nblk / sk.S), sb1 = (int)((int64_t)(slice + 1) * nblk / sk.S);
    const int q = (sb1 - sb0) / WAVES, qr = (sb1 - sb0) % WAVES;
    const int b0 = sb0 + wave * q + min(wave, qr);
    const int st0 = __builtin_amdgcn_readfirstlane(b0 * KB);
    const int steps = __builtin_amdgcn_readfirstlane(min((b0 + q + (wave < qr ? 1 : 0)) * KB, na) - st0);

    float4_t acc[RB][NB];
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int u = 0; u < NB; ++u) acc[i][u] = float4_t{0.f, 0.f, 0.f, 0.f};

    if (steps > 0) {
        // A: direct load g moves rows 8 g .. 8 g + 7 of the tile, 128 bytes
        // each (lane l: row l / 8 of the 8, 16-byte chunk (l % 8) ^ (row % 8)
        // to LDS position l % 8); rows past M read row M - 1 (in bounds; never
        // stored).  The fragment of row block i for half h of a pair: lane
        // (c, kg) reads row 16 i + c at chunk 4 h + kg.
        const int rows = __builtin_amdgcn_readfirstlane(min(M - tm * BM, BM));
        const __amdgpu_buffer_rsrc_t ar = make_rsrc(A + row0 * K, (uint32_t)rows * (uint32_t)K * 2u);
        const int pairs = (steps + 1) / 2;
        uint8_t* const wring = lds + wave * (RING * PAIR_BYTES);
        const uint32_t wlds = (uint32_t)reinterpret_cast<uintptr_t>(wring);
        const int chunk = (lane & 7) ^ (lane >> 3);
        uint32_t vb[2 * RB];
#pragma unroll
        for (int g = 0; g < 2 * RB; ++g)
            vb[g] = (uint32_t)min(8 * g + (lane >> 3), rows - 1) * (uint32_t)K * 2u + (uint32_t)chunk * 16u;
        // a last pair with one step: the lanes of its missing half read the
        // first half again (the row may end there)
        const uint32_t back = chunk >= 4 ? 64u : 0u;
        uint32_t rb[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) rb[h] = wlds + (uint32_t)(c * 128 + (((4 * h + kg) ^ (c & 7)) * 16));
        auto dma_a = [&](int pair, int g) {
            uint8_t* dst = wring + (pair & (RING - 1)) * PAIR_BYTES + g * 1024;
            pair = min(pair, pairs - 1);         // clamped: a repeated valid pair, never read
            uint32_t v = vb[g];
            if constexpr (!G4) v -= back & (2 * pair + 1 < steps ? 0u : ~0u);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ar, (__attribute__((address_space(3))) void*)dst, 16, v,
                                                     (uint32_t)(st0 + 2 * pair) * (kKqBK * 2), 0, 0);
        };
        // B: atoms and metadata of the tile's panels; panels past N read the
        // last panel (in bounds, never stored).
        __amdgpu_buffer_rsrc_t wr[PANELS], sr[PANELS], zr[PANELS];
#pragma unroll
        for (int pp = 0; pp < PANELS; ++pp) {
            const int panel = __builtin_amdgcn_readfirstlane(min(tn * PANELS + pp, np - 1));
            wr[pp] = make_rsrc(packed + (int64_t)panel * na * kAtomBytes, (uint32_t)na * kAtomBytes);
            sr[pp] = make_rsrc(packed + s_off + (int64_t)panel * ng * PW * 2, (uint32_t)(ng * PW * 2));
            zr[pp] = make_rsrc(packed + z_off + (int64_t)panel * ng * PW, (uint32_t)(ng * PW));
        }
        struct Slot {
            u32x4 w[PANELS];
        };
        struct Meta {
            uint32_t s[PANELS][(T + 1) / 2];   // T 16-bit scales of the lane's columns
            uint32_t z[PANELS];                // T zero-point bytes
        };
        auto load_w = [&](int step, Slot& sl) {
            // clamped: a repeated valid step, never used
            const uint32_t soff = __builtin_amdgcn_readfirstlane((st0 + min(step, steps - 1)) * kAtomBytes);
#pragma unroll
            for (int pp = 0; pp < PANELS; ++pp) sl.w[pp] = kq_load128(wr[pp], (uint32_t)lane * 16u, soff);
        };
        auto load_meta = [&](int g, Meta& mt) {
#pragma unroll
            for (int pp = 0; pp < PANELS; ++pp) {
                if constexpr (BITS == 4) {
                    const uint2 sv = __builtin_bit_cast(
                        uint2, __builtin_amdgcn_raw_buffer_load_b64(sr[pp], (uint32_t)c * 8u, (uint32_t)g * (PW * 2), 0));
                    mt.s[pp][0] = sv.x;
                    mt.s[pp][1] = sv.y;
                    mt.z[pp] = __builtin_amdgcn_raw_buffer_load_b32(zr[pp], (uint32_t)c * 4u, (uint32_t)g * PW, 0);
                } else {
                    mt.s[pp][0] = __builtin_amdgcn_raw_buffer_load_b32(sr[pp], (uint32_t)c * 4u, (uint32_t)g * (PW * 2), 0);
                    mt.z[pp] = __builtin_amdgcn_raw_buffer_load_b16(zr[pp], (uint32_t)c * 2u, (uint32_t)g * PW, 0);
                }
            }
        };
        // Group constants of column block u (panel u / T, lane column t = u % T).
        auto make_const = [&](const Meta& mt, int u) {
            const int pp = u / T, t = u % T;
            DqConst<BF> kq;
            if constexpr (BF) {
                const uint32_t sw = mt.s[pp][t / 2];
                kq.s = __builtin_bit_cast(float, (t & 1) ? (sw & 0xFFFF0000u) : (sw << 16));
                kq.nzs = -(byte_f32(mt.z[pp], t) * kq.s);
            } else {
                const uint32_t sh = mt.s[pp][t / 2] >> (16 * (t & 1));
                kq.s2 = as_h2(__builtin_amdgcn_perm(sh, sh, 0x01000100u));
                const uint32_t n = __builtin_amdgcn_perm(0xE4E4E4E4u, mt.z[pp], 0x04000400u | (t * 0x00010001u));
                kq.nz = n;
                kq.nz64 = neg_zero64_pair(n);
            }
            return kq;
        };
        auto dq_micro = [&](int k, const Slot& sl, int u, const DqConst<BF>& kq, DqSt<BF>& st) {
            const int pp = u / T, t = u % T;
            dq_step<BF, BITS>(k, sl.w[pp][BITS == 4 ? t : 2 * t], sl.w[pp][BITS == 4 ? t : 2 * t + 1], magic, kq, st);
        };

        // Metadata requests in order, the group tracked by a scalar counter
        // (the step's place in its group), clamped at the wave's last group.
        // G4: one per chunk, a chunk ahead.  Otherwise one per step, two steps
        // ahead, in slot step % 2.
        constexpr int MSTEP = G4 ? 4 : 1;
        Meta meta[G4 ? 1 : 2];
        int mstep = 0, mg = __builtin_amdgcn_readfirstlane(st0 / apg), mrem = __builtin_amdgcn_readfirstlane(st0 % apg);
        auto next_meta = [&](int slot) {
            load_meta(mg, meta[slot]);
            const int by = mstep + MSTEP < steps ? MSTEP : 0;
            mstep += by;
            mrem += by;
            mg += mrem == apg ? 1 : 0;
            mrem = mrem == apg ? 0 : mrem;
        };
        int crem = mrem;               // place of the current step in its group

        // Prologue: the requests of steps -(2 RING - 1) .. -1 in the loop's order.
        Slot ring[NR];
#pragma unroll
        for (int t = -4; t < 0; ++t) {
            if constexpr (G4) {
                if (t == -4) next_meta(0);
            } else {
                if (t >= -kKqMetaLead) next_meta(t + kKqMetaLead);
            }
            if (t >= -(NR - 1)) load_w(t + NR - 1, ring[t + NR - 1]);
            if ((t & 1) && t >= 1 - 2 * RING)
#pragma unroll
                for (int g = 0; g < 2 * RB; ++g) dma_a((t - 1) / 2 + RING, g);
            __builtin_amdgcn_sched_barrier(0);
        }
        kq_vm_wait<Ops::wait0()>();
        u32x4 af[2][RB];
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            af[0][i] = kq_read_block(rb[0], i);
            af[1][i] = u32x4{0u, 0u, 0u, 0u};
        }
        DqConst<BF> kc[NB];
#pragma unroll
        for (int u = 0; u < NB; ++u) kc[u] = make_const(meta[0], u);
        u32x4 bop[2];
        {
            DqSt<BF> st;
#pragma unroll
            for (int k = 0; k < DQ; ++k) dq_micro(k, ring[0], 0, kc[0], st);
            bop[0] = st.out;
        }
        // Every LDS read has landed before control leaves the straight run of
        // steps: a register copy that the compiler may place on such an edge
        // does not know of reads in flight.
        auto settle = [&]() {
            kq_lgkm_wait();
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int r = 0; r < RB; ++r) kq_tie(af[h][r]);
        };
        settle();
        // the accumulators' zeros are written before the gap
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int u = 0; u < NB; ++u) asm volatile("" : "+a"(acc[i][u]));
        mfma_hazard_gap();

        // Slots of a step (RB NB MFMAs, block u = slot / RB, row block i =
        // slot % RB): metadata and atoms after slot 0, the direct loads of A
        // (odd steps) one per kDmaStride slots from kDmaSlot on, then the
        // next step's fragments, all before the last block.
        constexpr int kSlots = RB * NB;
        constexpr int kDmaSlot = RB;
        constexpr int kReadSlot = kSlots - 2 * RB;
        constexpr int kDmaStride = (kReadSlot - kDmaSlot) / (2 * RB) > 0 ? (kReadSlot - kDmaSlot) / (2 * RB) : 1;
        constexpr int kDmaPer = (2 * RB * kDmaStride + kReadSlot - kDmaSlot - 1) / (kReadSlot - kDmaSlot);
        // one step: j = step % NR.  open_next: step + 1 opens a group.
        // In the steps after the loop (TAIL) the compiler drops requests that no
        // later step uses, so they count on the newest direct loads only.
        auto do_step = [&](auto jt, int step, auto tail) {
            constexpr int j = decltype(jt)::value;
            constexpr bool TAIL = decltype(tail)::value;
            constexpr int jn = (j + 1) % NR, jl = (j + NR - 1) % NR;
            if constexpr (!G4) crem = crem + 1 == apg ? 0 : crem + 1;
            const bool open_next = G4 ? j % 4 == 3 : crem == 0;
            const Meta& mnext = meta[G4 ? 0 : (j + 1) & 1];
#pragma unroll
            for (int u = 0; u < NB; ++u) {
                // operand dequantized under block u: block u + 1 of this step,
                // or block 0 of the next step under the last block
                const int du = (u + 1) % NB;
                const Slot& src = ring[u + 1 < NB ? j : jn];
                // constants of the group the next step opens: block v's old
                // ones were last used under block v - 1
                if (u == NB / 2 && open_next)
#pragma unroll
                    for (int v = 0; v < NB / 2; ++v) kc[v] = make_const(mnext, v);
                if (u == NB - 1 && open_next)
#pragma unroll
                    for (int v = NB / 2; v < NB; ++v) kc[v] = make_const(mnext, v);
                DqSt<BF> st;
#pragma unroll
                for (int i = 0; i < RB; ++i) {
                    const int s = u * RB + i;
                    __builtin_amdgcn_sched_barrier(0);
                    if (i == 0) {
                        // two wait states between the last write of this
                        // block's operand and its first MFMA
                        asm volatile("s_nop 1");
                        if (u == 0) {
                            kq_lgkm_wait();      // this step's fragments (read a step ago)
#pragma unroll
                            for (int r = 0; r < RB; ++r) kq_tie(af[j & 1][r]);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (s == 0) {
                        if constexpr (G4) {
                            if (j % 4 == 0) next_meta(0);
                        } else {
                            next_meta(j & 1);
                        }
                    }
                    if (s == 1) load_w(step + NR - 1, ring[jl]);
                    if ((j & 1) && s >= kDmaSlot && (s - kDmaSlot) % kDmaStride == 0)
#pragma unroll
                        for (int e = 0; e < kDmaPer; ++e) {
                            const int g = (s - kDmaSlot) / kDmaStride * kDmaPer + e;
                            if (g < 2 * RB && s < kReadSlot) dma_a((step - 1) / 2 + RING, g);
                        }
                    if (s >= kReadSlot && s < kReadSlot + RB) {
                        if (s == kReadSlot && (j & 1)) kq_vm_wait<TAIL ? 2 * RB : Ops::wait(j)>();
                        const int p1 = (step + 1) >> 1;
                        af[(j + 1) & 1][s - kReadSlot] =
                            kq_read_block(rb[(j + 1) & 1] + (uint32_t)(p1 & (RING - 1)) * PAIR_BYTES, s - kReadSlot);
                    }
#pragma unroll
                    for (int k = i * DQ / RB; k < (i + 1) * DQ / RB; ++k) dq_micro(k, src, du, kc[du], st);
                    mfma_acc<BF>(acc[i][u], bop[u & 1], af[j & 1][i]);
                }
                // (tied: the operand is formed here, not sunk past the loop's exit)
                kq_tie(st.out);
                bop[du & 1] = st.out;
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        static_assert(RING == 2 && NR == 4, "the prologue starts at step -4");
        static_assert((kReadSlot - kDmaSlot + kDmaStride - 1) / kDmaStride * kDmaPer >= 2 * RB,
                      "every direct load has a slot before the reads");
        int s = 0;
        for (; s + NR <= steps; s += NR) {
            do_step(std::integral_constant<int, 0>{}, s, std::false_type{});
            do_step(std::integral_constant<int, 1>{}, s + 1, std::false_type{});
            do_step(std::integral_constant<int, 2>{}, s + 2, std::false_type{});
            do_step(std::integral_constant<int, 3>{}, s + 3, std::false_type{});
        }
        settle();
        if constexpr (!G4) {
            if (s < steps) {
                do_step(std::integral_constant<int, 0>{}, s, std::true_type{});
                settle();
            }
            if (s + 1 < steps) {
                do_step(std::integral_constant<int, 1>{}, s + 1, std::true_type{});
                settle();
            }
            if (s + 2 < steps) {
                do_step(std::integral_constant<int, 2>{}, s + 2, std::true_type{});
                settle();
            }
        }
        // the requests past the last step (clamped, unused) land before their
        // registers or buffers are reused
        kq_vm_wait<0>();
    }
    mfma_hazard_gap();

    // Sum the waves' parts of K in wave order, SUMB column blocks per pass:
    // every wave parks its sums, then each adds its share of the blocks of
    // all of them.  The weights were the first MFMA operand: lane (c, kg) holds
    // row c of a block and its columns 4 kg .. 4 kg + 3 (N % 8 == 0, so all
    // four or none fit).
    float4_t* const red = reinterpret_cast<float4_t*>(lds);
    float4_t* const part =
        sk.S > 1 ? sk.part + ((int64_t)(slice * tiles_n + tn) * tiles_m + tm) * (RB * NB * 64) : nullptr;
#pragma unroll
    for (int h = 0; h < NB / SUMB; ++h) {
        __syncthreads();     // every wave is done with its ring, or has read the previous pass's sums
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int u = 0; u < SUMB; ++u)
                red[((wave * RB + r) * SUMB + u) * 64 + lane] = acc[r][h * SUMB + u];
        __syncthreads();
        constexpr int kEach = RB * SUMB / WAVES;
#pragma unroll
        for (int k = 0; k < kEach; ++k) {
            const int b = wave * kEach + k;
            const int r = b / SUMB, u = h * SUMB + b % SUMB;
            float4_t v = red[b * 64 + lane];
#pragma unroll
            for (int w = 1; w < WAVES; ++w) v += red[(w * RB * SUMB + b) * 64 + lane];
            const int64_t row = row0 + 16 * r + c, col = col0 + 16 * u + 4 * kg;
            if (sk.S > 1)
                part[(r * NB + u) * 64 + lane] = v;
            else if (row < M && col < N)
                *reinterpret_cast<uint2*>(C + row * N + col) =
                    uint2{round_out2<BF>(v[0], v[1]), round_out2<BF>(v[2], v[3])};
        }
    }
}

// Sum of the K slices: one thread per float4 of a tile, slices in order, four
// outputs rounded once.
template <bool BF, int RB, int NB>
__global__ __launch_bounds__(256) void kq_reduce_kernel(const float4_t* __restrict__ part, uint16_t* __restrict__ C,
                                                        int M, int N, int tiles_m, int S, int64_t total) {
    constexpr int kPerTile = RB * NB * 64;
    const int64_t f = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (f >= total) return;
    float4_t v = part[f];
    for (int s = 1; s < S; ++s) v += part[s * total + f];
    const int tile = (int)(f / kPerTile), e = (int)(f % kPerTile);
    const int tn = tile / tiles_m, tm = tile % tiles_m;
    const int lane = e & 63, u = (e >> 6) % NB, r = (e >> 6) / NB;
    const int64_t row = (int64_t)tm * (16 * RB) + 16 * r + (lane & 15);
    const int64_t col = (int64_t)tn * (16 * NB) + 16 * u + 4 * (lane >> 4);
    if (row < M && col < N)
        *reinterpret_cast<uint2*>(C + row * N + col) = uint2{round_out2<BF>(v[0], v[1]), round_out2<BF>(v[2], v[3])};
}

template <int BITS, bool BF, int RB, int NB, bool G4>
int launch_kq(const Layout& L, const uint16_t* A, const uint8_t* pk, uint16_t* C, int64_t M, int S, void* ws,
              hipStream_t s) {
    const int tiles_m = (int)((M + 16 * RB - 1) / (16 * RB));
    const int tiles_n = (int)((L.N + 16 * NB - 1) / (16 * NB));
    KqSplit sk{S, nullptr};
    if (S > 1) sk.part = reinterpret_cast<float4_t*>(static_cast<uint8_t*>(ws) + kWsCounterBytes);
    if (log_enabled())
        log_plan("gemm_kq_kernel<%d,%s,%d,%d,%d> M=%lld K=%lld N=%lld G=%d: %dx%d tiles of %dx%d, %d K slices over "
                 "the waves%s", BITS, BF ? "bf16" : "f16", RB, NB, (int)G4, (long long)M, (long long)L.K,
                 (long long)L.N, L.group, tiles_m, tiles_n, 16 * RB, 16 * NB, S, S > 1 ? ", reduction launch" : "");
    const int rc = launch(gemm_kq_kernel<BITS, BF, RB, NB, G4>, dim3((unsigned)(tiles_m * tiles_n * S)),
                          dim3(64 * KqCfg<RB, NB>::WAVES), 0, s, A, pk, C, (int)M, (int)L.K, (int)L.N, L.group / kAtomK, L.s_off,
                          L.z_off, (int)L.na, (int)L.ng, (int)L.np, tiles_m, tiles_n, sk);
    if (rc || S == 1) return rc;
    const int64_t total = (int64_t)tiles_m * tiles_n * (RB * NB * 64);
    return launch(kq_reduce_kernel<BF, RB, NB>, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, sk.part, C,
                  (int)M, (int)L.N, tiles_m, S, total);
}

template <int RB, int NB, bool G4>
int launch_any(const Layout& L, const uint16_t* A, const uint8_t* pk, uint16_t* C, int64_t M, int S, void* ws,
               hipStream_t s, bool bf) {
    if (L.bits == 4)
        return bf ? launch_kq<4, true, RB, NB, G4>(L, A, pk, C, M, S, ws, s)
                  : launch_kq<4, false, RB, NB, G4>(L, A, pk, C, M, S, ws, s);
    return bf ? launch_kq<8, true, RB, NB, G4>(L, A, pk, C, M, S, ws, s)
              : launch_kq<8, false, RB, NB, G4>(L, A, pk, C, M, S, ws, s);
}

}  // namespace

int launch_gemm_kq(const Layout& L, const uint16_t* A, const void* packed, uint16_t* C, int64_t M, int rb, int S,
                   void* ws, hipStream_t s, bool bf) {
    const uint8_t* pk = static_cast<const uint8_t*>(packed);
    const bool g4 = L.na % 4 == 0 && L.group % 128 == 0;
    if (rb == 8)
        return g4 ? launch_any<8, 8, true>(L, A, pk, C, M, S, ws, s, bf)
                  : launch_any<8, 8, false>(L, A, pk, C, M, S, ws, s, bf);
    return g4 ? launch_any<4, 4, true>(L, A, pk, C, M, S, ws, s, bf)
              : launch_any<4, 4, false>(L, A, pk, C, M, S, ws, s, bf);
}

}  // namespace tf

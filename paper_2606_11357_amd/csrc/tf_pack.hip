// Offline pre-tiling (Section 4.2) into the packed layout described in
// tf_internal.h, and the debug kernels that read it back through the same
// device unpack / dequantize primitives as the matmul kernels (Section 4.3).
#include "tf_internal.h"

namespace tf {
namespace {

// Packing: a block of 256 threads rearranges one 32-row atom of each of 8
// panels (512 4-bit or 256 8-bit columns), so that every row is read as 256
// consecutive bytes, and, where the atom opens a group, the panels' scales and
// zero-points.  Thread (kg, w) loads word w (8 4-bit or 4 8-bit columns) of
// the 8 rows 8 kg .. 8 kg + 7 and transposes them in registers into the 8
// dwords those codes have in the layout; LDS gathers the dwords of the atoms,
// which leave as 16 bytes per lane, 1 KB in a row.
// Bound by memory: K = 4096, N = 14336 4-bit moves 61 MB.  Measured on MI355X:
// one thread per output dword, gathering its 8 codes with 4-byte loads, and a
// second launch for the metadata took 31.9 us (1.9 TB/s), this form 12.2 us
// (5.0 TB/s, the rate of a large copy).
constexpr int kPackPanels = 8, kPackThreads = 256;
constexpr int kPackStride = 256 + 4;     // dwords of LDS per atom: the panels' stores fall on different banks

struct PackMeta {
    const uint16_t* sc;      // scales [ng, s_gstride] (s_gstride 0: one row for every group)
    const uint8_t* z;        // zero-points as the caller has them (4-bit: packed words), or NULL
    int64_t s_gstride;
    int zconst;              // the zero-point where z is NULL
    int64_t s_off, z_off;
    int ng, apg;             // groups; atoms per group
};

// 8 x 8 transpose of nibbles: afterwards nibble j of v[i] is what was nibble i of v[j].
__device__ __forceinline__ void transpose_nibbles(uint32_t (&v)[8]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t a = v[j], b = v[j + 4];
        v[j] = __builtin_amdgcn_perm(b, a, 0x05040100u);
        v[j + 4] = __builtin_amdgcn_perm(b, a, 0x07060302u);
    }
#pragma unroll
    for (int h = 0; h < 8; h += 4)
#pragma unroll
        for (int j = h; j < h + 2; ++j) {
            const uint32_t a = v[j], b = v[j + 2];
            v[j] = __builtin_amdgcn_perm(b, a, 0x06020400u);
            v[j + 2] = __builtin_amdgcn_perm(b, a, 0x07030501u);
        }
#pragma unroll
    for (int j = 0; j < 8; j += 2) {
        const uint32_t a = v[j], b = v[j + 1];
        v[j] = (a & 0x0F0F0F0Fu) | ((b << 4) & 0xF0F0F0F0u);
        v[j + 1] = ((a >> 4) & 0x0F0F0F0Fu) | (b & 0xF0F0F0F0u);
    }
}
// 4 x 4 transpose of bytes.
__device__ __forceinline__ void transpose_bytes(uint32_t& r0, uint32_t& r1, uint32_t& r2, uint32_t& r3) {
    const uint32_t a = __builtin_amdgcn_perm(r1, r0, 0x05010400u), b = __builtin_amdgcn_perm(r1, r0, 0x07030602u);
    const uint32_t c = __builtin_amdgcn_perm(r3, r2, 0x05010400u), d = __builtin_amdgcn_perm(r3, r2, 0x07030602u);
    r0 = __builtin_amdgcn_perm(c, a, 0x05040100u);
    r1 = __builtin_amdgcn_perm(c, a, 0x07060302u);
    r2 = __builtin_amdgcn_perm(d, b, 0x05040100u);
    r3 = __builtin_amdgcn_perm(d, b, 0x07060302u);
}

// flip = 0x80808080 turns signed INT8 codes into unsigned codes q + 128
// (two's complement: flipping the sign bit adds 128).
template <int BITS>
__global__ __launch_bounds__(kPackThreads) void pack_kernel(const uint32_t* __restrict__ qw, uint8_t* __restrict__ packed,
                                                            int N, int np, int na, uint32_t flip, PackMeta mt) {
    constexpr int PW = BITS == 4 ? 64 : 32, T = PW / 16;
    constexpr int WPP = 8;                          // words of a row per panel
    __shared__ __align__(16) uint32_t st[kPackPanels * kPackStride];
    const int tid = threadIdx.x, w = tid & 63, kg = tid >> 6;
    const int a = blockIdx.y;
    const int64_t p0 = (int64_t)blockIdx.x * kPackPanels;
    const int64_t row_words = (int64_t)N * BITS / 32, word = p0 * WPP + w;
    // words past the row: the columns past N hold q = 0 (8-bit rows end on a
    // word too, N % 8 == 0)
    const bool in = word < row_words;
    const uint32_t* src = qw + (int64_t)(a * kAtomK + 8 * kg) * row_words + word;
    uint32_t v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        // 4-bit: nibble position j holds row offset 2 j or 2 (j - 4) + 1
        const int r = BITS == 8 ? j : j < 4 ? 2 * j : 2 * (j - 4) + 1;
        v[j] = in ? src[r * row_words] ^ flip : 0u;
    }
    uint32_t* const dst = st + (w / WPP) * kPackStride + kg * 64;
    if constexpr (BITS == 4) {
        transpose_nibbles(v);
        // column 8 (w % 8) + i of the panel: c = 8 (w % 2) + i, t = (w % 8) / 2
#pragma unroll
        for (int i = 0; i < 8; ++i) dst[(8 * (w & 1) + i) * 4 + (w % 8) / 2] = v[i];
    } else {
        transpose_bytes(v[0], v[1], v[2], v[3]);
        transpose_bytes(v[4], v[5], v[6], v[7]);
        // column 4 (w % 8) + i: c = 4 (w % 4) + i, dwords 2 ((w % 8) / 4) + 0, 1 for rows 0..3, 4..7
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *reinterpret_cast<u32x2*>(&dst[(4 * (w & 3) + i) * 4 + 2 * ((w % 8) / 4)]) = u32x2{v[i], v[4 + i]};
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int pp = (tid >> 6) + 4 * h;          // panel of this wave's store
        if (p0 + pp < np)
            *reinterpret_cast<u32x4*>(packed + ((p0 + pp) * na + a) * kAtomBytes + 16 * w) =
                *reinterpret_cast<const u32x4*>(&st[pp * kPackStride + 4 * w]);
    }
    // scales (copied bit for bit) and zero-points (a byte each) of the group this atom opens
    if (a % mt.apg != 0) return;
    const int64_t g = a / mt.apg;
#pragma unroll
    for (int h = 0; h < kPackPanels * PW / kPackThreads; ++h) {
        const int col = tid + h * kPackThreads;
        const int64_t p = p0 + col / PW, n = p0 * PW + col;
        if (p >= np) break;
        uint16_t s = 0;
        uint8_t z = 0;
        if (n < N) {
            s = mt.sc[g * mt.s_gstride + n];
            if (!mt.z)
                z = (uint8_t)mt.zconst;
            else if (BITS == 4)
                z = (uint8_t)((mt.z[g * (N / 2) + n / 2] >> (4 * (n & 1))) & 0xFu);
            else
                z = mt.z[g * N + n];
        }
        const int e = (col % 16) * T + col % PW / 16;        // entry c * T + t of column c + 16 t
        const int64_t at = (p * mt.ng + g) * PW + e;
        reinterpret_cast<uint16_t*>(packed + mt.s_off)[at] = s;
        packed[mt.z_off + at] = z;
    }
}

// Column and row of code (lane, dword t, position j) of an atom.
struct CodePos {
    int64_t n, k;
};

__device__ __forceinline__ CodePos w4_pos(int64_t p, int64_t a, int lane, int t, int j) {
    // j: row offset 0..7 inside the lane's 8-row slice
    return {p * 64 + (lane & 15) + 16 * t, a * kAtomK + 8 * (lane >> 4) + j};
}
__device__ __forceinline__ CodePos w8_pos(int64_t p, int64_t a, int lane, int t, int b) {
    return {p * 32 + (lane & 15) + 16 * (t >> 1), a * kAtomK + 8 * (lane >> 4) + 4 * (t & 1) + b};
}

// tf_unpack: one thread per packed dword; the codes come out of the same
// magic-number unpack the matmul kernels use, then 1024 is removed.
__global__ void unpack_weights(int bits, const uint32_t* __restrict__ wreg, uint8_t* __restrict__ q_out,
                               int64_t N, int64_t na, int64_t total_dwords) {
    int64_t d = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (d >= total_dwords) return;
    int64_t atom = d >> 8;
    int within = (int)(d & 255);
    int lane = within >> 2, t = within & 3;
    int64_t p = atom / na, a = atom % na;
    uint32_t w = wreg[d];
    if (bits == 4) {
        uint32_t cp[4];
        w4_code_pairs(w, magic_reg(), cp);
        for (int pr = 0; pr < 4; ++pr) {
            for (int h = 0; h < 2; ++h) {
                CodePos pos = w4_pos(p, a, lane, t, 2 * pr + h);
                if (pos.n < N)
                    q_out[pos.k * N + pos.n] = (uint8_t)((cp[pr] >> (16 * h)) & 0x3FFu);
            }
        }
    } else {
        uint32_t cp[2];
        w8_code_pairs(w, cp);
        for (int pr = 0; pr < 2; ++pr) {
            for (int h = 0; h < 2; ++h) {
                CodePos pos = w8_pos(p, a, lane, t, 2 * pr + h);
                if (pos.n < N)
                    q_out[pos.k * N + pos.n] = (uint8_t)((cp[pr] >> (16 * h)) & 0x3FFu);
            }
        }
    }
}

__global__ void unpack_zeros(const uint8_t* __restrict__ zreg, uint8_t* __restrict__ z_out, int64_t N,
                             int64_t ng, int pw, int64_t entries) {
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= entries) return;
    int64_t p = e / (ng * pw);
    int64_t g = (e / pw) % ng;
    int i = (int)(e % pw);
    int T = pw / 16;
    int64_t n = p * pw + i / T + 16 * (i % T);
    if (n < N) z_out[g * N + n] = zreg[e];
}

// tf_dequant: one thread per 8 codes of one column (one MFMA B operand),
// dequantized with the matmul kernels' own code.  mode 0: fp16 scales, fp16
// weights; 1: fp16 scales, exact fp32 weights; 2: bf16 scales, bf16 weights.
__global__ void dequant_weights(int bits, const uint8_t* __restrict__ packed, int64_t s_off,
                                int64_t z_off, int64_t N, int64_t na, int64_t ng, int group,
                                int mode, void* __restrict__ w_out, int64_t slices) {
    int64_t sidx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (sidx >= slices) return;
    // slice = (atom, lane, column-slot); 64 lanes x 4 (4-bit) or 2 (8-bit) slots
    const int T = bits == 4 ? 4 : 2;
    const int pw = bits == 4 ? 64 : 32;
    int64_t atom = sidx / (64 * T);
    int rem = (int)(sidx % (64 * T));
    int lane = rem / T, t = rem % T;
    int64_t p = atom / na, a = atom % na;
    int c = lane & 15;
    int64_t n = p * pw + c + 16 * t;
    if (n >= N) return;
    int64_t k0 = a * kAtomK + 8 * (lane >> 4);
    int64_t g = (a * kAtomK) / group;
    int64_t meta = (p * ng + g) * pw + c * T + t;
    uint16_t sbits = reinterpret_cast<const uint16_t*>(packed + s_off)[meta];
    uint32_t z = packed[z_off + meta];
    const uint32_t* atomw = reinterpret_cast<const uint32_t*>(packed) + atom * 256 + lane * 4;
    if (mode == 2) {
        const DqConst<true> kq = make_dq_const<true>(sbits, z);
        const u32x4 wb = bits == 4 ? dq_operand<true, 4>(atomw[t], 0u, 0u, kq)
                                   : dq_operand<true, 8>(atomw[2 * t], atomw[2 * t + 1], 0u, kq);
        uint16_t* o = reinterpret_cast<uint16_t*>(w_out);
        for (int j = 0; j < 8; ++j) o[(k0 + j) * N + n] = (uint16_t)(wb[j >> 1] >> (16 * (j & 1)));
        return;
    }
    half8_t w8;
    uint32_t codes[4];
    if (bits == 4) {
        uint32_t w = atomw[t];
        const uint32_t magic = magic_reg();
        const uint32_t nz = neg_zero_pair(z);
        w8 = dq_w4_dword(w, magic, nz, neg_zero64_pair(nz), as_h2(sbits | ((uint32_t)sbits << 16)));
        w4_code_pairs(w, magic, codes);
    } else {
        uint32_t w0 = atomw[2 * t], w1 = atomw[2 * t + 1];
        w8 = dq_w8_dwords(w0, w1, neg_zero_pair(z), as_h2(sbits | ((uint32_t)sbits << 16)));
        w8_code_pairs(w0, codes);
        w8_code_pairs(w1, codes + 2);
    }
    if (mode == 1) {
        // exact: (q - z) is formed exactly in fp16 by the same pair subtraction
        // and its product with the fp16 scale needs at most 19 significant bits
        float s = (float)__builtin_bit_cast(_Float16, sbits);
        float* o = reinterpret_cast<float*>(w_out);
        for (int j = 0; j < 8; ++j) {
            half2_t d = as_h2(codes[j >> 1]) + as_h2(neg_zero_pair(z));
            o[(k0 + j) * N + n] = (float)d[j & 1] * s;
        }
    } else {
        _Float16* o = reinterpret_cast<_Float16*>(w_out);
        for (int j = 0; j < 8; ++j) o[(k0 + j) * N + n] = w8[j];
    }
}

inline unsigned blocks_for(int64_t n, int threads) { return (unsigned)((n + threads - 1) / threads); }

}  // namespace

namespace {
template <int BITS>
int launch_pack(const void* qw, const void* z, const uint16_t* sc, int64_t s_gstride, int zconst, uint32_t flip,
                const Layout& L, void* packed, hipStream_t s) {
    const PackMeta mt{sc, static_cast<const uint8_t*>(z), s_gstride, zconst, L.s_off, L.z_off, (int)L.ng,
                      L.group / kAtomK};
    const dim3 grid((unsigned)((L.np + kPackPanels - 1) / kPackPanels), (unsigned)L.na);
    return launch(pack_kernel<BITS>, grid, dim3(kPackThreads), 0, s, static_cast<const uint32_t*>(qw),
                  static_cast<uint8_t*>(packed), (int)L.N, (int)L.np, (int)L.na, flip, mt);
}
}  // namespace

int launch_pack_w4(const int32_t* qw, const int32_t* qz, const uint16_t* sc, const Layout& L,
                   void* packed, hipStream_t s) {
    return launch_pack<4>(qw, qz, sc, L.N, 0, 0u, L, packed, s);
}

int launch_pack_w8(const uint8_t* qw, const uint8_t* zr, const uint16_t* sc, const Layout& L,
                   void* packed, hipStream_t s) {
    return launch_pack<8>(qw, zr, sc, L.N, 0, 0u, L, packed, s);
}

// Signed INT8 with one scale per column (Eq. 1): stored as the 8-bit layout
// with codes q + 128, zero-point 128 and the column's scale in every group,
// so s * ((q + 128) - 128) = s * q through the same kernels.
int launch_pack_w8_sym(const int8_t* qw, const uint16_t* sc, const Layout& L, void* packed,
                       hipStream_t s) {
    return launch_pack<8>(qw, nullptr, sc, 0, 128, 0x80808080u, L, packed, s);
}

int launch_unpack(const Layout& L, const void* packed, uint8_t* q_out, uint8_t* z_out,
                  hipStream_t s) {
    const uint8_t* base = static_cast<const uint8_t*>(packed);
    int64_t dwords = L.np * L.na * 256;
    int rc = launch(unpack_weights, dim3(blocks_for(dwords, 256)), dim3(256), 0, s, L.bits,
                    reinterpret_cast<const uint32_t*>(base + L.w_off), q_out, L.N, L.na, dwords);
    if (rc) return rc;
    int64_t entries = L.np * L.ng * L.pw;
    return launch(unpack_zeros, dim3(blocks_for(entries, 256)), dim3(256), 0, s, base + L.z_off,
                  z_out, L.N, L.ng, (int)L.pw, entries);
}

int launch_dequant(const Layout& L, const void* packed, int out_dtype, void* w_out,
                   hipStream_t s) {
    int64_t slices = L.np * L.na * 64 * L.T;
    return launch(dequant_weights, dim3(blocks_for(slices, 256)), dim3(256), 0, s, L.bits,
                  static_cast<const uint8_t*>(packed), L.s_off, L.z_off, L.N, L.na, L.ng,
                  L.group, out_dtype == TF_F32 ? 1 : out_dtype == TF_BF16 ? 2 : 0, w_out, slices);
}

}  // namespace tf

// Online 2:4 sparsification of an activation matrix: magnitude Top-2 of every aligned group of
// four along K (Alg. 1 "X~ <- TopK(X)"), the norm-compensation factor of the method section
// ("Norm-Compensated Sparsification", s = sqrt(|X|^2 / (|X~|^2 + eps))), and compression into
// kept values + 2-bit positions (App. A operand format). One sweep over X; HBM-bandwidth bound:
// 2 bytes read + 1.125 bytes written per input element.
//
// Mapping: one wavefront per row (several for long rows, each taking a run of whole trips); a lane
// takes 8 consecutive bf16 (one 16-byte load = two groups) per step and the wave walks the row in
// steps of 512 elements, so every load, the
// 8-byte value stores and the 4-byte metadata stores (four lanes' bytes gathered with DPP
// quad permutes) are contiguous across the wave in the canonical (row-major) output. The
// k-major output the GEMM streams (64-byte value blocks and 8-byte metadata records per row and
// 64-k block, rows contiguous) is written as 64-byte pieces, two neighbouring rows per line.
// When only the k-major output is wanted and nothing is summed along a row (the rtl_sparse_linear
// path with NONE / GROUP scope), sparsify_pack_block_kernel runs instead: its mapping follows the
// output layout (32 rows x 64-k blocks per wave) and every access is a whole line. (The FP8 sweep keeps
// the row mapping: with its heavier per-group arithmetic the block mapping measured the same.)
#include <type_traits>
#include "rtl_internal.h"
#include "select.h"
#include "tensor_factor.h"

namespace rtl {
namespace {

constexpr int kWavesPerBlock = 8;
constexpr int kUnroll = 3;   // 6 and 24 steps per row at K = 3072 / 12288 divide evenly

template <int CTRL>
__device__ __forceinline__ uint32_t quad_bcast(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// `vals`: bf16 [M,K/2], or one-byte E4M3 codes [M,K/2] when FP8 (then x_scale[0] is the divisor).
// Workgroup `block` of the row mapping (kWavesPerBlock waves).
template <int COMP, bool FP8>
__device__ __forceinline__ void sweep_rows(
    const unsigned block, const uint16_t* __restrict__ X, int64_t M, int K, int64_t ldx, float eps,
    void* __restrict__ vals, uint8_t* __restrict__ meta, uint8_t* __restrict__ vals_km,
    uint8_t* __restrict__ meta_km, int64_t Mpad, float* __restrict__ scale,
    float* __restrict__ rowsums, const float* __restrict__ x_scale, int parts, int span) {
    const int lane = threadIdx.x & 63;
    // `parts` waves share a row, each taking a run of `span` elements: few rows then still give
    // every SIMD enough waves in flight. ROW / TENSOR add the waves' sums up in LDS, so there the waves of a
    // row sit in one workgroup (parts divides kWavesPerBlock).
    constexpr bool SUMS = COMP == RTL_COMP_ROW || COMP == RTL_COMP_TENSOR;
    const int64_t gw = (int64_t)block * kWavesPerBlock + (threadIdx.x >> 6);
    const int64_t row = gw / parts;
    const int part = (int)(gw % parts);
    if (row >= M && (!SUMS || parts == 1)) return;   // whole wave leaves together (it has no barrier to meet)
    const int kbeg = part * span;
    const int kend = row < M ? min(K, kbeg + span) : 0;
    const uint16_t* xr = X + row * ldx;
    // canonical value row (only dereferenced when vals != null): bf16 form / FP8 form
    uint16_t* vr = static_cast<uint16_t*>(vals) + row * (int64_t)(K / 2);
    uint8_t* vr8 = static_cast<uint8_t*>(vals) + row * (int64_t)(K / 2);
    uint8_t* vkr = vals_km + row * 64;                     // only dereferenced when vals_km != null
    uint8_t* mr = meta + row * (int64_t)(K / 8);          // only dereferenced when meta != null
    constexpr int KM_REC = FP8 ? 16 : 8;                   // k-major record: 128 or 64 dense k
    uint8_t* kmr = meta_km + row * KM_REC;                 // only dereferenced when meta_km != null
    float inv = 1.0f;
    if constexpr (FP8) inv = 1.0f / x_scale[0];
    float num = 0.f, den = 0.f;
    // rows of metadata are K/8 bytes: whole 32-bit words only when K is a multiple of 32
    const bool word_meta = (K & 31) == 0;
    for (int k0 = kbeg; k0 < kend; k0 += 512 * kUnroll) {
        uint4 v[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int k = k0 + u * 512 + lane * 8;
            v[u] = make_uint4(0, 0, 0, 0);
            if (k < kend) v[u] = *reinterpret_cast<const uint4*>(xr + k);
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int k = k0 + u * 512 + lane * 8;
            const GroupOut g0 = select_group<COMP, FP8>(v[u].x, v[u].y, eps, inv);
            const GroupOut g1 = select_group<COMP, FP8>(v[u].z, v[u].w, eps, inv);
            if constexpr (COMP == RTL_COMP_ROW || COMP == RTL_COMP_TENSOR) {
                num += g0.num + g1.num;   // zero-filled lanes past K contribute nothing
                den += g0.den + g1.den;
            }
            const uint32_t b = g0.nibble | (g1.nibble << 4);
            // gather the metadata bytes of the four lanes of a quad into its first lane
            const uint32_t w = b | (quad_bcast<0x55>(b) << 8) | (quad_bcast<0xAA>(b) << 16) |
                               (quad_bcast<0xFF>(b) << 24);
            if (k < kend) {
                if constexpr (FP8) {
                    const uint32_t codes = g0.packed | (g1.packed << 16);
                    if (vals) *reinterpret_cast<uint32_t*>(vr8 + k / 2) = codes;
                    // k-major twin: 64 codes (64 bytes) per row and 128-k block
                    if (vals_km)
                        *reinterpret_cast<uint32_t*>(vkr + (int64_t)(k >> 7) * Mpad * 64 + ((k & 127) >> 1)) = codes;
                } else {
                    const uint2 pair = make_uint2(g0.packed, g1.packed);
                    if (vals) *reinterpret_cast<uint2*>(vr + k / 2) = pair;
                    // k-major twin: 32 values (64 bytes) per row and 64-k block
                    if (vals_km)
                        *reinterpret_cast<uint2*>(vkr + (int64_t)(k >> 6) * Mpad * 64 + (k & 63)) = pair;
                }
                if (meta) {
                    if (word_meta) {
                        if ((lane & 3) == 0) *reinterpret_cast<uint32_t*>(mr + k / 8) = w;
                    } else {
                        mr[k / 8] = (uint8_t)b;
                    }
                }
                // k-major twin: the quad's word is one 32-k slice of the row's record of its block
                // (8 bytes per 64 k, or 16 bytes per 128 k with FP8 values)
                if (meta_km && (lane & 3) == 0) {
                    if constexpr (FP8)
                        *reinterpret_cast<uint32_t*>(kmr + (int64_t)(k >> 7) * Mpad * 16 + ((k >> 5) & 3) * 4) = w;
                    else
                        *reinterpret_cast<uint32_t*>(kmr + (int64_t)(k >> 6) * Mpad * 8 + ((k >> 5) & 1) * 4) = w;
                }
            }
        }
    }
    if constexpr (SUMS) {
        num = wave_sum(num);
        den = wave_sum(den);
        if (parts > 1) {
            __shared__ float part_num[kWavesPerBlock], part_den[kWavesPerBlock];
            const int wave = threadIdx.x >> 6;
            if (lane == 0) {
                part_num[wave] = num;
                part_den[wave] = den;
            }
            __syncthreads();
            if (part != 0 || row >= M) return;
            for (int i = 1; i < parts; ++i) {        // in the order of the row
                num += part_num[wave + i];
                den += part_den[wave + i];
            }
        }
        if (lane == 0) {
            if constexpr (COMP == RTL_COMP_ROW) {
                scale[row] = sqrtf(num / (den + eps));
            } else {
                rowsums[2 * row] = num;
                rowsums[2 * row + 1] = den;
            }
        }
    }
}

template <int COMP, bool FP8>
__global__ __launch_bounds__(kWavesPerBlock * 64) void sparsify_pack_kernel(
    const uint16_t* __restrict__ X, int64_t M, int K, int64_t ldx, float eps,
    void* __restrict__ vals, uint8_t* __restrict__ meta, uint8_t* __restrict__ vals_km,
    uint8_t* __restrict__ meta_km, int64_t Mpad, float* __restrict__ scale,
    float* __restrict__ rowsums, const float* __restrict__ x_scale, int parts, int span) {
    sweep_rows<COMP, FP8>(blockIdx.x, X, M, K, ldx, eps, vals, meta, vals_km, meta_km, Mpad, scale, rowsums, x_scale, parts, span);
}

// The same sweep for the case that matters most: only the k-major outputs are wanted (what
// rtl_sparse_linear feeds its tile loop) and nothing is summed along a row (NONE / GROUP). Then the
// mapping can follow the OUTPUT layout instead of the input rows: a wave takes 32 rows and a run of
// 64-k blocks; per block, lane (r, c) = (lane / 8, lane % 8) loads chunk c (16 bytes, two groups) of
// the rows r, r + 8, r + 16, r + 24 of its 32. Every load instruction then reads 8 whole 128-byte
// lines, every value store writes 512 contiguous bytes (the 64-byte blocks of 8 neighbouring rows are
// adjacent in the k-major layout) and the metadata of a row (8 bytes per block) leaves as one store.
// The row mapping above writes the same buffer as 64-byte pieces of single rows, half a line at a
// time, which costs HBM efficiency once the activation is large.
constexpr int kBlockWaves = 4;      // waves per workgroup: the same 32 rows, consecutive runs of blocks
constexpr int kBlockUnroll = 2;     // 64-k blocks in flight per wave
template <int COMP, int WAVES>
__device__ __forceinline__ void sweep_blocks(
    const unsigned block, const uint16_t* __restrict__ X, int64_t M, int KB, int64_t ldx, float eps, uint8_t* __restrict__ vals_km,
    uint8_t* __restrict__ meta_km, int64_t Mpad, int per, unsigned row_blocks) {
    const int lane = threadIdx.x & 63, r8 = lane >> 3, c = lane & 7;
    const int wave = threadIdx.x >> 6;
    // workgroup id = run group * row_blocks + row block: neighbours take neighbouring rows of one K range
    const int64_t m0 = (int64_t)(block % row_blocks) * 32;
    const int b0 = ((int)(block / row_blocks) * WAVES + wave) * per;   // first block of this wave's run
    const int b1 = min(KB, b0 + per);
    const uint16_t* xr[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) xr[t] = X + min(m0 + 8 * t + r8, M - 1) * ldx + c * 8;   // rows past M: clamped, results land in padding rows
    // lane's row r8 of the tile (t adds 8 rows = 512 bytes of values, 64 bytes of metadata)
    uint8_t* vdst = vals_km + (m0 + r8) * 64 + c * 8;
    uint8_t* mdst = meta_km + (m0 + r8) * 8;
    for (int b = b0; b < b1; b += kBlockUnroll) {
        uint4 v[kBlockUnroll][4];
#pragma unroll
        for (int u = 0; u < kBlockUnroll; ++u)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                v[u][t] = make_uint4(0, 0, 0, 0);
                if (b + u < b1) v[u][t] = *reinterpret_cast<const uint4*>(xr[t] + (int64_t)(b + u) * 64);
            }
#pragma unroll
        for (int u = 0; u < kBlockUnroll; ++u) {
            if (b + u >= b1) break;
            uint8_t* vb = vdst + (int64_t)(b + u) * Mpad * 64;
            uint8_t* mb = mdst + (int64_t)(b + u) * Mpad * 8;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const GroupOut g0 = select_group<COMP, false>(v[u][t].x, v[u][t].y, eps);
                const GroupOut g1 = select_group<COMP, false>(v[u][t].z, v[u][t].w, eps);
                *reinterpret_cast<uint2*>(vb + t * 512) = make_uint2(g0.packed, g1.packed);
                // the row's eight metadata bytes: quads gather theirs into a word, the first quad of the
                // row fetches the second quad's word from four lanes up
                const uint32_t nb = g0.nibble | (g1.nibble << 4);
                const uint32_t w = nb | (quad_bcast<0x55>(nb) << 8) | (quad_bcast<0xAA>(nb) << 16) |
                                   (quad_bcast<0xFF>(nb) << 24);
                const uint32_t w_hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)w, 0x104, 0xF, 0xF, true);   // row_shl:4
                if (c == 0) *reinterpret_cast<uint2*>(mb + t * 64) = make_uint2(w, w_hi);
            }
        }
    }
}

template <int COMP>
__global__ __launch_bounds__(kBlockWaves * 64) void sparsify_pack_block_kernel(
    const uint16_t* __restrict__ X, int64_t M, int KB, int64_t ldx, float eps, uint8_t* __restrict__ vals_km,
    uint8_t* __restrict__ meta_km, int64_t Mpad, int per, unsigned row_blocks) {
    sweep_blocks<COMP, kBlockWaves>(blockIdx.x, X, M, KB, ldx, eps, vals_km, meta_km, Mpad, per, row_blocks);
}

// Few rows with the LoRA residual: sweep and T = X L_B^T in one launch, by workgroups of their own. Workgroups
// [0, t_blocks) form T, the others run the sweep as the plain call does.
// A workgroup of T takes 16 rows x 16 ranks over the whole contraction: its eight waves deal the 64-k blocks out among
// themselves (block w, w + 8, ...), a lane holds 32 bytes of a row per block, in two pieces of 16 (a load takes 64 contiguous bytes of each
// of 16 rows), as the operands of two v_mfma_f32_16x16x32_bf16, straight from memory, and the waves' sums are added in LDS in
// the order of the waves. So T needs no partial planes and no second launch. It is bound by the rate at which one compute
// unit gets its 64 K bytes (about 40 GB/s, however many blocks are in flight), which is why the tile is the smallest one:
// 32 x 16 and 32 x 32 take 1.5 and 2 times as long up to 512 rows (whole FP8 call [512, 3072, 3072]: 21.6, 24.3, 27.5 us), and why
// long contractions stay with the split ones of pack_lora.hip.
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
union DownFrag {
    uint4 u;
    bf16x8 v;
};
constexpr int kDownTile = 16, kDownUnroll = 4;           // rows and ranks of a tile; 64-k blocks of a wave in flight
constexpr int kDownParts = kLoraRank / kDownTile;        // workgroups of a row tile
__device__ __forceinline__ void down_tile(const unsigned block, const uint16_t* __restrict__ X, int64_t M, int KB, int64_t ldx,
                                          const uint16_t* __restrict__ LB, int64_t ldlb, uint16_t* __restrict__ T) {
    __shared__ float part[kWavesPerBlock][kDownTile * kDownTile];
    const int lane = threadIdx.x & 63, li = lane & 15, kb = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // the workgroups of a row tile on one XCD (ids go round robin): X from its L2 after the first
    const int64_t m0 = ((int64_t)(block / (8 * kDownParts)) * 8 + block % 8) * kDownTile;
    const int rank0 = (int)(block / 8) % kDownParts * kDownTile;
    if (m0 >= M) return;                                                     // whole workgroup
    const uint16_t* xa = X + min(m0 + li, M - 1) * ldx + kb * 8;             // rows past M: never stored
    const uint16_t* lb = LB + (int64_t)(rank0 + li) * ldlb + kb * 8;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    auto blocks = [&](const int b, auto count) {         // blocks b, b + 8, ...: all loads in flight together
        constexpr int U = decltype(count)::value;
        DownFrag x[U][2], l[U][2];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int64_t k = (int64_t)(b + u * kWavesPerBlock) * 64 + h * 32;
                x[u][h].u = *reinterpret_cast<const uint4*>(xa + k);
                l[u][h].u = *reinterpret_cast<const uint4*>(lb + k);
            }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int h = 0; h < 2; ++h) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[u][h].v, l[u][h].v, acc, 0, 0, 0);
    };
    int b = wave;
    for (; b + (kDownUnroll - 1) * kWavesPerBlock < KB; b += kDownUnroll * kWavesPerBlock)
        blocks(b, std::integral_constant<int, kDownUnroll>{});
    for (; b < KB; b += kWavesPerBlock) blocks(b, std::integral_constant<int, 1>{});
#pragma unroll
    for (int r = 0; r < 4; ++r) part[wave][(4 * kb + r) * kDownTile + li] = acc[r];      // row 4 kb + r, rank li
    __syncthreads();
    const int e = threadIdx.x;
    const int64_t m = m0 + e / kDownTile;
    if (e >= kDownTile * kDownTile || m >= M) return;
    float v = part[0][e];
#pragma unroll
    for (int w = 1; w < kWavesPerBlock; ++w) v += part[w][e];
    const uint32_t hi = f32_to_bf16_rne(v);              // two bf16 planes: hi = bf16(T), lo = bf16(T - hi)
    uint16_t* t = T + m * kLoraRank + rank0 + e % kDownTile;
    t[0] = (uint16_t)hi;
    t[M * kLoraRank] = (uint16_t)f32_to_bf16_rne(v - __uint_as_float(hi << 16));
}

// bf16 NONE / GROUP take the block mapping of the sweep (then parts = row blocks, span = 64-k blocks per wave), the others the
// row mapping.
template <int COMP, bool FP8>
__global__ __launch_bounds__(kWavesPerBlock * 64) void sparsify_down_kernel(
    const uint16_t* __restrict__ X, int64_t M, int K, int64_t ldx, float eps, uint8_t* __restrict__ vals_km,
    uint8_t* __restrict__ meta_km, int64_t Mpad, float* __restrict__ scale, float* __restrict__ rowsums,
    const float* __restrict__ x_scale, int parts, int span, const uint16_t* __restrict__ LB, int64_t ldlb,
    uint16_t* __restrict__ T, unsigned t_blocks) {
    if (blockIdx.x < t_blocks) down_tile(blockIdx.x, X, M, K / 64, ldx, LB, ldlb, T);
    else if constexpr (!FP8 && (COMP == RTL_COMP_NONE || COMP == RTL_COMP_GROUP))
        sweep_blocks<COMP, kWavesPerBlock>(blockIdx.x - t_blocks, X, M, K / 64, ldx, eps, vals_km, meta_km, Mpad, span, (unsigned)parts);
    else
        sweep_rows<COMP, FP8>(blockIdx.x - t_blocks, X, M, K, ldx, eps, nullptr, nullptr, vals_km, meta_km, Mpad, scale, rowsums,
                              x_scale, parts, span);
}

// TENSOR scope: fold the per-row sums and emit the single factor. `fused` (nullable) receives the factor times
// mul[0] (the FP8 activation scale).
__global__ __launch_bounds__(kFactorThreads) void tensor_scale_kernel(const float* __restrict__ rowsums, int64_t M,
                                                                      float eps, float* __restrict__ scale,
                                                                      const float* __restrict__ mul,
                                                                      float* __restrict__ fused) {
    const float sc = tensor_factor(rowsums, M, eps);
    if (threadIdx.x == 0) {
        scale[0] = sc;
        if (fused) fused[0] = mul[0] * sc;
    }
}

// Direct cast bf16 -> E4M3 (weights "directly quantized to FP8"): 8 elements per thread.
__global__ __launch_bounds__(256) void quantize_fp8_kernel(const uint16_t* __restrict__ W, int64_t rows,
                                                           int64_t cols8, int64_t ld,
                                                           uint8_t* __restrict__ Wq, int64_t ldq) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= rows * cols8) return;
    const int64_t r = t / cols8, c = (t % cols8) * 8;
    const uint4 v = *reinterpret_cast<const uint4*>(W + r * ld + c);
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    uint32_t o[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t lo = e4m3_pair(bits_to_f32(w[2 * h] << 16), bits_to_f32(w[2 * h] & 0xFFFF0000u));
        const uint32_t hi = e4m3_pair(bits_to_f32(w[2 * h + 1] << 16), bits_to_f32(w[2 * h + 1] & 0xFFFF0000u));
        o[h] = lo | (hi << 16);
    }
    *reinterpret_cast<uint2*>(Wq + r * ldq + c) = make_uint2(o[0], o[1]);
}

// Copy of the canonical operand into the k-major layout. A workgroup takes R = 2^log_rows rows (64, fewer where M is smaller) and 64 / R
// groups of U neighbouring 64-k blocks: thread (group g, row r, piece p) moves piece p (16 bytes) of the row's U value blocks,
// all loads in flight together, and the metadata records of the blocks p, p + 4, .... Reads are runs of 64 U bytes of a row,
// writes 64 R bytes contiguous per block. (With R = 64 whatever M, calls of a few rows are 2 to 3 % slower: whole call [1, 6080, 1024]
// 6.74 -> 6.99 us, [2, 11104, 512] 6.97 -> 7.18.)
template <int U>
__global__ __launch_bounds__(256) void operand_to_kmajor_kernel(const uint16_t* __restrict__ vals, const uint8_t* __restrict__ meta,
                                                                int64_t M, int KB, int64_t Mpad, uint8_t* __restrict__ vals_km,
                                                                uint8_t* __restrict__ meta_km, unsigned row_blocks, int log_rows) {
    const int piece = (int)threadIdx.x & 3;
    const int64_t row = ((int64_t)(blockIdx.x % row_blocks) << log_rows) + ((threadIdx.x >> 2) & ((1u << log_rows) - 1));
    const int b0 = (int)(((blockIdx.x / row_blocks) << (6 - log_rows)) + (threadIdx.x >> (2 + log_rows))) * U;
    if (row >= M || b0 >= KB) return;
    const uint8_t* src = reinterpret_cast<const uint8_t*>(vals) + (row * KB + b0) * 64 + piece * 16;
    const uint8_t* msrc = meta + (row * KB + b0) * 8;
    const int last = KB - 1 - b0;                        // (blocks past K: the last one again, not stored)
    uint4 v[U];
    uint2 m[(U + 3) / 4];
#pragma unroll
    for (int u = 0; u < U; ++u)
        v[u] = *reinterpret_cast<const uint4*>(src + min(u, last) * 64);
#pragma unroll
    for (int u = 0; u < (U + 3) / 4; ++u)
        m[u] = *reinterpret_cast<const uint2*>(msrc + min(4 * u + piece, last) * 8);
    uint8_t* dst = vals_km + (b0 * Mpad + row) * 64 + piece * 16;
    uint8_t* mdst = meta_km + (b0 * Mpad + row) * 8;
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (b0 + u < KB) *reinterpret_cast<uint4*>(dst + u * Mpad * 64) = v[u];
#pragma unroll
    for (int u = 0; u < (U + 3) / 4; ++u)
        if (4 * u + piece < U && b0 + 4 * u + piece < KB) *reinterpret_cast<uint2*>(mdst + (4 * u + piece) * Mpad * 8) = m[u];
}

}  // namespace

// Querying one kernel makes the runtime load this translation unit's code object.
hipError_t prepare_pack_kernels() {
    hipFuncAttributes attr;
    return hipFuncGetAttributes(&attr, reinterpret_cast<const void*>(tensor_scale_kernel));
}

hipError_t launch_operand_to_kmajor(const uint16_t* vals, const uint8_t* meta, int64_t M, int64_t K,
                                    uint8_t* vals_km, uint8_t* meta_km, hipStream_t stream) {
    const int KB = (int)(K / 64);
    int log_rows = 0;
    while (log_rows < 6 && ((int64_t)1 << log_rows) < M) ++log_rows;
    const unsigned row_blocks = (unsigned)((M + 63) / 64);
    auto go = [&](auto kernel, int u) {
        const int per = u << (6 - log_rows);             // k blocks of a workgroup
        hipLaunchKernelGGL(kernel, dim3(row_blocks * (unsigned)((KB + per - 1) / per)), dim3(256), 0, stream, vals, meta, M, KB,
                           kmajor_rows(M), vals_km, meta_km, row_blocks, log_rows);
    };
    // Four blocks per thread where that leaves two workgroups a compute unit, else one: whole rtl_packed_linear call with
    // 1 / 2 / 4 / 8 blocks, us: [4608, 1024, 3072] 38.6 / 36.0 / 34.2 / 33.1, [4096, 1024, 12288] 90.8 / 86.2 / 86.3 / 86.5, [16896, 512,
    // 3072] 57.1 / 55.0 / 55.6 / 55.9; [512, 1024, 3072] 11.8 / 11.9 / 12.3 / 12.9, [1029, 512, 1024] 9.5 / 9.5 / 9.8 / 10.4. Around the line, 1 / 2 / 4
    // blocks, row_blocks x KB = 768 [512, 512, 6144] 15.1 / 15.3 / 15.4, 1152 [4608, 512, 1024] 15.4 / 15.5 / 15.6, 1632 [1029, 512, 6144] 25.0 / 24.8 / 24.7,
    // 1728 [4608, 512, 1536] 18.9 / 19.0 / 18.9, 2304 [4608, 512, 2048] 22.0 / 21.8 / 21.5, 3072 [2048, 512, 6144] 28.2 / 27.8 / 27.1.
    if ((int64_t)row_blocks * KB >= 2048) go(operand_to_kmajor_kernel<4>, 4);
    else go(operand_to_kmajor_kernel<1>, 1);
    return hipGetLastError();
}

// Waves per row: one per unrolled trip of work (1536 elements) while the rows alone do not fill the chip,
// fewer once they do. Measured [M, 12288], us with 1 / 2 / 4 / 8 waves per row: FP8 GROUP M = 37 18.9 / 10.7 /
// 6.5 / 4.4, 512 19.6 / 11.3 / 7.3 / 6.5, 1029 21.2 / 16.4 / 12.8 / 11.1, 2048 22.4 / 19.0 / 17.1 / 18.1,
// 4608 41.9 / 34.5 / 31.7 / 32.1, 9728 67 / 64 / 62 / 64. ROW and TENSOR pay for the sum over the waves:
// ROW M = 37 12.7 / 7.9 / 5.4 / 4.5, 512 14.2 / 8.7 / 6.6 / 7.0, 2048 17.0 / 16.2 / 18.5 / 19.1. At K = 3072 two waves
// win or tie for GROUP (4608: 13.0 -> 11.6) and lose for ROW from M = 1500 on (5.8 -> 5.9, 9728 17.9 -> 19.3).
// Between those K, FP8 GROUP at [16000, 5120 / 6656 / 9216]: 1 wave 45.6 / 56.2 / 84.1, this rule 45.4 / 56.7 / 76.9; runs cut at
// 512 elements 53.3 / 70.7 / 80.8. ROW [37 / 300 / 700, 7680], five trips: 4 waves 5.6 / 5.9 / 8.2, 8 waves 4.7 / 5.4 / 6.9
// (eight trips, [1000, 12288]: 9.3 and 9.8).
// Runs are whole trips: a trip costs its three steps of arithmetic however much of it lies past the run's end, and runs
// of whole 512-element steps made up to 7 trips out of the 5 of K = 6656.
void row_split(int comp, int64_t M, int64_t K, int out[2]) {
    const int trips = (int)((K + 512 * kUnroll - 1) / (512 * kUnroll));
    int parts;
    if (comp == RTL_COMP_NONE || comp == RTL_COMP_GROUP) {
        const int most = M <= 1024 ? 8 : (K >= 2 * 512 * kUnroll ? 4 : 1);
        const int per = (trips + most - 1) / most;                            // trips of a wave
        parts = (trips + per - 1) / per;                                      // no wave without one
    } else {
        const int most = M <= 256 || (M <= 1024 && trips % 4 != 0) ? 8 : (M <= 1536 ? 4 : (K >= 4 * 512 * kUnroll ? 2 : 1));
        parts = trips > 4 ? 8 : (trips > 2 ? 4 : trips);                      // divides kWavesPerBlock
        parts = parts > most ? most : parts;
    }
    out[0] = parts;
    out[1] = (trips + parts - 1) / parts * (512 * kUnroll);
}

template <bool FP8>
static hipError_t launch_pack_any(const uint16_t* X, int64_t M, int64_t K, int64_t ldx, rtl_comp comp,
                                  float eps, void* vals, uint8_t* meta, uint8_t* vals_km, uint8_t* meta_km,
                                  float* scale, float* rowsums, const float* x_scale, hipStream_t stream) {
    const int64_t Mpad = kmajor_rows(M);
    if constexpr (!FP8) {
        // only the k-major outputs, nothing summed along a row: the block mapping (see its kernel)
        if (!vals && !meta && vals_km && meta_km && K % 64 == 0 &&
            (comp == RTL_COMP_NONE || comp == RTL_COMP_GROUP)) {
            // Blocks per wave: two once the rows are long (measured flat between one and three: at
            // [4096,12288] 190.9 / 190.7 / 190.2 us per rtl_sparse_linear call, at [16896,12288] 817 / 812 /
            // 814; six and more lose), one for short rows, where more waves matter more.
            const int KB = (int)(K / 64);
            const int per = KB >= 96 ? kBlockUnroll : 1;
            const int runs = (KB + per - 1) / per;                     // waves per 32 rows
            const int64_t row_blocks = (M + 31) / 32, groups = (runs + kBlockWaves - 1) / kBlockWaves;
            if (row_blocks * groups < ((int64_t)1 << 31)) {            // (else: far beyond memory; the row mapping serves)
                const dim3 grid((unsigned)(row_blocks * groups));
                if (comp == RTL_COMP_GROUP)
                    hipLaunchKernelGGL((sparsify_pack_block_kernel<RTL_COMP_GROUP>), grid, dim3(kBlockWaves * 64), 0,
                                       stream, X, M, KB, ldx, eps, vals_km, meta_km, Mpad, per, (unsigned)row_blocks);
                else
                    hipLaunchKernelGGL((sparsify_pack_block_kernel<RTL_COMP_NONE>), grid, dim3(kBlockWaves * 64), 0,
                                       stream, X, M, KB, ldx, eps, vals_km, meta_km, Mpad, per, (unsigned)row_blocks);
                return hipGetLastError();
            }
        }
    }
    int split[2];
    row_split((int)comp, M, K, split);
    const int parts = split[0], span = split[1];
    const dim3 grid((unsigned)((M * parts + kWavesPerBlock - 1) / kWavesPerBlock));
    const dim3 block(kWavesPerBlock * 64);
    switch (comp) {
        case RTL_COMP_NONE:
            hipLaunchKernelGGL((sparsify_pack_kernel<RTL_COMP_NONE, FP8>), grid, block, 0, stream, X, M,
                               (int)K, ldx, eps, vals, meta, vals_km, meta_km, Mpad, scale, rowsums, x_scale, parts, span);
            break;
        case RTL_COMP_GROUP:
            hipLaunchKernelGGL((sparsify_pack_kernel<RTL_COMP_GROUP, FP8>), grid, block, 0, stream, X, M,
                               (int)K, ldx, eps, vals, meta, vals_km, meta_km, Mpad, scale, rowsums, x_scale, parts, span);
            break;
        case RTL_COMP_ROW:
            hipLaunchKernelGGL((sparsify_pack_kernel<RTL_COMP_ROW, FP8>), grid, block, 0, stream, X, M,
                               (int)K, ldx, eps, vals, meta, vals_km, meta_km, Mpad, scale, rowsums, x_scale, parts, span);
            break;
        case RTL_COMP_TENSOR:
            hipLaunchKernelGGL((sparsify_pack_kernel<RTL_COMP_TENSOR, FP8>), grid, block, 0, stream, X, M,
                               (int)K, ldx, eps, vals, meta, vals_km, meta_km, Mpad, scale, rowsums, x_scale, parts, span);
            if (scale) return launch_tensor_scale(rowsums, M, eps, scale, stream);
            break;
    }
    return hipGetLastError();
}

hipError_t launch_sparsify_pack(const uint16_t* X, int64_t M, int64_t K, int64_t ldx, rtl_comp comp,
                                float eps, uint16_t* vals, uint8_t* meta, uint8_t* vals_km,
                                uint8_t* meta_km, float* scale, float* rowsums, hipStream_t stream) {
    return launch_pack_any<false>(X, M, K, ldx, comp, eps, vals, meta, vals_km, meta_km, scale, rowsums,
                                  nullptr, stream);
}

hipError_t launch_sparsify_pack_fp8(const uint16_t* X, int64_t M, int64_t K, int64_t ldx, rtl_comp comp,
                                    float eps, const float* x_scale, uint8_t* vals8, uint8_t* meta,
                                    uint8_t* vals_km, uint8_t* meta_km, float* scale, float* rowsums,
                                    hipStream_t stream) {
    return launch_pack_any<true>(X, M, K, ldx, comp, eps, vals8, meta, vals_km, meta_km, scale, rowsums,
                                 x_scale, stream);
}

hipError_t launch_sparsify_down(const uint16_t* X, int64_t M, int64_t K, int64_t ldx, rtl_comp comp, float eps, const uint16_t* LB,
                                int64_t ldlb, uint8_t* vals_km, uint8_t* meta_km, uint16_t* T, float* scale, float* rowsums,
                                hipStream_t stream, const float* x_scale) {
    const int64_t tiles = (M + kDownTile - 1) / kDownTile;
    const unsigned t_blocks = (unsigned)((tiles + 7) / 8 * 8 * kDownParts);
    int split[2];
    int64_t blocks;
    if (!x_scale && (comp == RTL_COMP_NONE || comp == RTL_COMP_GROUP)) {
        split[0] = (int)((M + 31) / 32);
        split[1] = 1;                                    // (short contractions only: one block per wave, see launch_pack_down)
        blocks = split[0] * (int64_t)((K / 64 + kWavesPerBlock - 1) / kWavesPerBlock);
    } else {
        row_split((int)comp, M, K, split);
        blocks = (M * split[0] + kWavesPerBlock - 1) / kWavesPerBlock;
    }
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(t_blocks + (unsigned)blocks), dim3(kWavesPerBlock * 64), 0, stream, X, M, (int)K, ldx, eps,
                           vals_km, meta_km, kmajor_rows(M), scale, rowsums, x_scale, split[0], split[1], LB, ldlb, T, t_blocks);
    };
    switch (comp) {
        case RTL_COMP_NONE:
            x_scale ? go(sparsify_down_kernel<RTL_COMP_NONE, true>) : go(sparsify_down_kernel<RTL_COMP_NONE, false>);
            break;
        case RTL_COMP_GROUP:
            x_scale ? go(sparsify_down_kernel<RTL_COMP_GROUP, true>) : go(sparsify_down_kernel<RTL_COMP_GROUP, false>);
            break;
        case RTL_COMP_ROW:
            x_scale ? go(sparsify_down_kernel<RTL_COMP_ROW, true>) : go(sparsify_down_kernel<RTL_COMP_ROW, false>);
            break;
        case RTL_COMP_TENSOR:
            x_scale ? go(sparsify_down_kernel<RTL_COMP_TENSOR, true>) : go(sparsify_down_kernel<RTL_COMP_TENSOR, false>);
            break;
    }
    return hipGetLastError();
}

hipError_t launch_tensor_scale(const float* rowsums, int64_t M, float eps, float* scale, hipStream_t stream,
                               const float* mul, float* fused) {
    hipLaunchKernelGGL(tensor_scale_kernel, dim3(1), dim3(kFactorThreads), 0, stream, rowsums, M, eps, scale, mul, fused);
    return hipGetLastError();
}

hipError_t launch_quantize_fp8(const uint16_t* W, int64_t rows, int64_t cols, int64_t ld, uint8_t* Wq,
                               int64_t ldq, hipStream_t stream) {
    const int64_t n = rows * (cols / 8);
    hipLaunchKernelGGL(quantize_fp8_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, W,
                       rows, cols / 8, ld, Wq, ldq);
    return hipGetLastError();
}

}  // namespace rtl

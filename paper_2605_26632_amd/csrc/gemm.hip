// Linear layers on the gfx950 matrix cores.
//
//   dense : Y = X W^T                       (paper Eq. linear_layer; v_mfma_f32_16x16x32_bf16)
//   sparse: Y = S(X) W^T, S(X) compressed   (Alg. 1 "Y_s <- S(X) W^T", operand format of App. A;
//                                            v_smfmac_f32_32x32x32_bf16)
//
// Both share one tile loop. A workgroup owns a BM x BN tile of Y and walks K in stages of 128-byte rows
// of W (64 dense k in bf16, 128 in FP8). Stages travel HBM/L2 -> LDS with direct-to-LDS loads (no register
// staging) through a ring of LDS buffers, and each wave keeps operand fragments in flight while the matrix
// core works on others.
// The sparse kernel reads its compressed operand in the k-major layout the pack sweep writes
// (values and metadata of a 256-row tile contiguous per stage: whole 128-byte lines only); the
// dense operands X and W are the caller's row-major tensors.
//
// The compressed activation is the FIRST matrix operand of SMFMAC (the one that carries 2-of-4
// structure along K), so tokens map to the instruction's rows and the weight rows (K contiguous)
// map to its columns: no transposition of either tensor is needed.
//
// Matrix instructions of size S x S: 32 in the sparse kernels, 16 in the dense one, of the same rate per clock. The clock
// is set by the package power limit. On N(0, 1) operands fed from LDS with 128 x 64 per wave the 16 x 16 ones reach
// 1730 against 1556 TFLOP/s (dense bf16), 1470 against 1395 (sparse bf16, executed) and 2865 against 2725 (sparse FP8):
// twice the operand reads per multiply-add cost less than halving the accumulator traffic saves. On zeros all reach 2130
// to 2230. In a tile loop a stalled wave has half the time to come back before the matrix core runs dry, and the small
// instructions lose 3 % (dense) to 8 % (sparse) of the cycles. Dense gains from 16 (this loop built in both sizes, before its
// tails and its table were fitted to 16; the whole change from the loop before it was worth 3 % at [4608, 9216, 3072]. rtl_dense_linear on
// inputs from HBM, 32 -> 16, us: [4608, 9216, 3072] 229.5 -> 217.3, [4096, 3072, 12288] 268.4 -> 261.3, [4608, 3072, 3072] 82.6 -> 80.4,
// [800, 9216, 3072] 61.1 -> 59.1); sparse ties ([4096, 3072, 12288] 188.1 -> 186.6, [4608, 12288, 3072] 199.9 -> 200.5,
// [16896, 12288, 3072] 724.8 -> 723.9, FP8 [4608, 3072, 12288] 131.4 -> 131.2) and loses with 128 x 128 tiles ([1500, 3072, 3072] 31.6
// -> 33.1).
//
// Operand layouts, measured on the device (one-hot operands, random small integers); lane l: i = l % S, kb = l / S.
// v_smfmac_f32_32x32x32_bf16 | v_smfmac_f32_16x16x64_bf16:
//   A (8 bf16)  : row i, the kept values of dense k in [16 kb, 16 kb + 16) in order
//   idx (16 bit): ABID picks the 16-bit half of the lane's own index register; nibble g holds
//                 pos0 | pos1 << 2 of the lane's g-th group
//   B (16 bf16) : column i; element u < 8 is dense k = 8 kb + u, u >= 8 is k = 16 | 32 + 8 kb + (u - 8)
//   D           : column i, register r (of 16) is row 8 (r / 4) + 4 kb + r % 4 | (of 4) row 4 kb + r
// v_mfma_f32_32x32x16_bf16 | v_mfma_f32_16x16x32_bf16: A and B (8 bf16) hold k = 8 kb + v of row / column i; D as above.
// The labelling of k inside a stage is free as long as both operands agree; it is chosen so that
// a lane reads whole 16-byte chunks from LDS and its metadata as one word per stage.
//
// FP8 variant of the sparse kernel (E4M3 codes on both operands, the W8A8 composition of the
// implementation-details section): v_smfmac_f32_32x32x64_fp8_fp8 | v_smfmac_f32_16x16x128_fp8_fp8:
//   A (16 fp8)  : row i, the kept values of dense k in [32 kb, 32 kb + 32) in order
//   idx (32 bit): the whole register, nibble g = pos0 | pos1 << 2 of the lane's g-th group
//   B (32 fp8)  : column i; element u < 16 is dense k = 16 kb + u, u >= 16 is k = 32 | 64 + 16 kb + (u - 16)
//   D           : as above
// In bytes this is the bf16 geometry (16-byte A chunk, two 16-byte B chunks at the same chunk
// indices), so a stage simply covers 128 dense k instead of 64 and the kernel differs only in the
// instruction and in the metadata record (16 bytes per row and stage). Both sizes add their products in the same way
// (runs of 8 kept values cut at 13 bits below the run's largest exponent sum).
#include <mutex>
#include <type_traits>
#include <vector>
#include "rtl_internal.h"
#include "tensor_factor.h"

namespace rtl {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) __bf16 bf16x16;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(8))) int i32x8;

union Frag8 {
    uint4 u;
    bf16x8 v;
    i32x4 q;     // 16 fp8
};
union Frag16 {
    uint4 u[2];
    bf16x16 v;
    i32x8 q;     // 32 fp8
};

// One dense bf16 matrix instruction of size S x S (16 or 32 k).
template <int S> struct AccOf { typedef f32x16 type; };
template <> struct AccOf<16> { typedef f32x4 type; };
template <int S>
__device__ __forceinline__ typename AccOf<S>::type dense_mma(bf16x8 a, bf16x8 b, typename AccOf<S>::type c) {
    if constexpr (S == 32) return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ uint32_t f32_to_bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    uint32_t r = (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
    uint32_t nan = (u >> 16) | 0x40u;
    return ((u & 0x7FFFFFFFu) > 0x7F800000u) ? nan : r;
}

// Direct-to-LDS load of one wave: lane l fetches `bytes` (16 or 4) from its own global address and
// the hardware writes them to LDS address lds_base + l * bytes (lds_base is wave-uniform and
// travels in M0). Written as inline assembly so that the outstanding-load counter stays under
// the kernel's own control: the loads of a stage are awaited with an explicit vmcnt wait right
// before the barrier that publishes the stage, and reads of older stages never wait for them.
__device__ __forceinline__ void lds_dma16(const void* gaddr, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                 :: "s"(lds_base), "v"(gaddr) : "memory", "m0");
}
__device__ __forceinline__ void lds_dma4(const void* gaddr, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off"
                 :: "s"(lds_base), "v"(gaddr) : "memory", "m0");
}
// Same with a wave-uniform 64-bit base (SGPR pair) plus a 32-bit per-lane byte offset: the per-lane
// state of a stream shrinks to one register and the walk along K is a scalar addition.
__device__ __forceinline__ uint64_t uniform64(const void* p) {   // pin a wave-uniform pointer to SGPRs
    const uint64_t b = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ void lds_dma16_so(const void* sbase, uint32_t voff, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds_base), "v"(voff), "s"(uniform64(sbase)) : "memory", "m0");
}
__device__ __forceinline__ void lds_dma4_so(const void* sbase, uint32_t voff, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
                 :: "s"(lds_base), "v"(voff), "s"(uniform64(sbase)) : "memory", "m0");
}
template <int N>
__device__ __forceinline__ void wait_vmcnt_lgkm0() {   // vmcnt <= N, all LDS reads returned
    __builtin_amdgcn_s_waitcnt(0x0070 | (N & 0xF) | ((N >> 4) << 14));
}

// Size of the matrix instructions (see the top of the file).
template <bool SPARSE>
constexpr int kMmaSize = SPARSE ? 32 : 16;

// Per-stage LDS footprint. Rows of the A tile hold 64 bytes in the sparse kernels (the kept half) and 128 in
// the dense one; rows of the B tile hold 128 bytes, so that every L2 request of a row-major operand is a
// whole line. WAVES_K > 1: a stage holds one k block per K group (see gemm_tile), kGroup bytes each.
template <bool SPARSE, int BM, int BN, int STAGES, int WAVES_M, int WAVES_N, bool FP8, int WAVES_K = 1>
struct Smem {
    static constexpr int kABytes = BM * (SPARSE ? 64 : 128);
    static constexpr int kMetaRec = FP8 ? 16 : 8;   // metadata bytes per row and stage
    static constexpr int kMetaBytes = SPARSE ? BM * kMetaRec : 0;
    static constexpr int kBBytes = BN * 128;
    static constexpr int kGroup = kABytes + kMetaBytes + kBBytes;
    static constexpr int kStage = WAVES_K * kGroup;
    static constexpr int kRing = STAGES * kStage;
    // epilogue staging: every wave owns (BM / WAVES_M) rows of (BN / WAVES_N) bf16 plus 16 bytes
    // of padding per row (keeps the rows written together in different banks)
    static constexpr int kEpiRowBytes = (BN / WAVES_N) * 2 + 16;
    // K groups: one fp32 plane of the tile per group instead; the row padding puts rows 4 apart (written together by the
    // two or four lane groups) 32 or 16 banks apart
    static constexpr int kPitch = BN + (SPARSE ? 8 : 4);
    static constexpr int kPlane = BM * kPitch * 4;
    static constexpr int kEpi = WAVES_K > 1 ? WAVES_K * kPlane : WAVES_M * WAVES_N * (BM / WAVES_M) * kEpiRowBytes;
    static constexpr int kTotal = kRing > kEpi ? kRing : kEpi;
    static_assert(kTotal <= 160 * 1024, "LDS budget of a CU");
};

// f(0), f(1), ... f(N - 1) with compile-time indices
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// LDS swizzles. A 16-byte read of a wave is served 16 lanes at a time over 64 four-byte banks, so
// the 16 consecutive tile rows those lanes address (same logical chunk c) must land in 16 different
// 16-byte slots modulo 256 bytes.
// Rows of 8 chunks (128 bytes): two rows per 256 bytes; the row parity picks the half, c is XORed
// with bits 1..3 of the row.
__device__ __forceinline__ int swz8(int row, int c) { return row * 128 + ((c ^ ((row >> 1) & 7)) << 4); }
// Rows of 4 chunks (64 bytes): four rows per 256 bytes; c is XORed with bits 2..3 of the row.
__device__ __forceinline__ int swz4(int row, int c) { return row * 64 + ((c ^ ((row >> 2) & 3)) << 4); }
// Inverse maps: which (row, c) lives at chunk position p of the tile.
__device__ __forceinline__ void unswz8(int p, int& row, int& c) {
    row = p >> 3;
    c = (p & 7) ^ ((row >> 1) & 7);
}
__device__ __forceinline__ void unswz4(int p, int& row, int& c) {
    row = p >> 2;
    c = (p & 3) ^ ((row >> 2) & 3);
}

// Tile order: consecutive workgroup ids land on different XCDs (round robin), so ids are first
// regrouped per XCD (XCD x works through a contiguous share of the tile list), and the list walks
// the tile grid in groups of GM tile-rows so that the ~32 tiles an XCD runs at a time share few
// activation and weight panels in its L2.
__device__ __forceinline__ int xcd_share_start(int n, int xcd) {   // first list index of XCD xcd's share of n tiles
    return xcd * (n / 8) + min(xcd, n % 8);
}
template <int GM>
__device__ __forceinline__ void tile_walk(int t, int tiles_m, int tiles_n, int& pm, int& pn) {
    const int per_group = GM * tiles_n;
    const int group = t / per_group;
    const int first_m = group * GM;
    const int gsize = min(tiles_m - first_m, GM);
    pm = first_m + (t % per_group) % gsize;
    pn = (t % per_group) / gsize;
}

// a * b and x + y rounded one by one: the LoRA form (sum of residual and bias as `add`) and the plain form
// (bias alone) then agree bit for bit when the residual is zero.
__device__ __forceinline__ float mul_add_rn(float a, float b, float add) {
#pragma clang fp contract(off)
    const float p = a * b;
    return p + add;
}

// MODE 0: plain linear. MODE 1 (sparse only): LoRA tail, the accumulators also receive T L_A^T before
// the epilogue.
// `tile`: index of this workgroup's output tile in the walk of the (M / BM) x (N / BN) tile grid.
// PART: the workgroup covers the k blocks [kblk0, kblk0 + kblks) only and leaves its fp32 sums in plane `part` of
// a.partials; the factors (MODE 0), the bias and the rounding are split_reduce_kernel's.
// FOLDED: with a.rowsums set the TENSOR factor is a.folded.
// WAVES_K > 1: the waves divide the contraction too. K group g of the WAVES_K groups of WAVES_M x WAVES_N
// waves takes the k blocks g, g + WAVES_K, ... with operands and accumulators of its own, and the groups'
// tiles are added up in LDS, in the order of g, when the loop is done.
template <bool SPARSE, int BM, int BN, int WAVES_M, int WAVES_N, int STAGES, int MODE = 0, bool FP8 = false,
          int WAVES_K = 1, bool PART = false, bool FOLDED = false, bool PIN = true>
__device__ __forceinline__ void gemm_tile(const GemmArgs a, const int tile, const int part = 0, const int kblk0 = 0,
                                          const int kblks = 0) {
    static_assert(!PART || WAVES_K == 1, "partial sums leave from the accumulators");
    static_assert(MODE == 0 || (MODE == 1 && SPARSE), "mode/operand combination");
    static_assert(!FP8 || SPARSE, "FP8 operands: sparse kernels only");
    constexpr int NW = WAVES_M * WAVES_N;             // waves that share a block of operands
    constexpr int WTM = BM / WAVES_M, WTN = BN / WAVES_N;
    constexpr int S = kMmaSize<SPARSE>, TM = WTM / S, TN = WTN / S;
    static_assert(WTM % S == 0 && WTN % S == 0 && (S == 32 || TM > 1), "wave tile must be made of S x S blocks");
    using L = Smem<SPARSE, BM, BN, STAGES, WAVES_M, WAVES_N, FP8, WAVES_K>;
    using Acc = typename AccOf<S>::type;
    constexpr int RB = S == 32 ? 16 : 4;              // accumulator registers of a block
    constexpr int ESZ = FP8 ? 1 : 2;                  // bytes per operand element
    constexpr int KSTAGE = 128 / ESZ;                 // dense k per stage
    constexpr int IXW = FP8 ? 2 : 1;                  // metadata words a lane holds per stage and row block
    constexpr int MREC = L::kMetaRec;                 // metadata bytes per row and stage
    // one wave-wide direct-to-LDS load moves 64 chunks of 16 bytes = 1 KiB
    constexpr int A_LOADS = L::kABytes / 1024;
    static_assert(A_LOADS % NW == 0, "tile loads must divide over the waves");
    // The B tile is dealt to the waves in runs of B_CH 16-byte chunks. When that is an odd
    // multiple of 32 (192-row dense tile: 96 chunks), a wave's last load runs with its upper half
    // masked off, so every wave still issues the same number of loads.
    constexpr int B_CH = L::kBBytes / 16 / NW;
    static_assert((L::kBBytes / 16) % NW == 0 && B_CH % 32 == 0, "B tile must divide over the waves");
    constexpr int A_PER_W = A_LOADS / NW, B_PER_W = (B_CH + 63) / 64;
    constexpr bool B_HALF = (B_CH % 64) != 0;
    constexpr int M_LOADS = SPARSE ? (BM * MREC) / 256 : 0;  // metadata: 4 bytes per lane per load
    static_assert(!SPARSE || M_LOADS % NW == 0, "metadata loads must divide over the waves");
    constexpr int M_PER_W = M_LOADS / NW;

    extern __shared__ __align__(16) uint8_t smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);    // wave-uniform, lives in an SGPR
    const int wk = WAVES_K > 1 ? wid / NW : 0, wave = WAVES_K > 1 ? wid % NW : wid;   // K group, wave inside it
    uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)smem;
    if constexpr (WAVES_K > 1) lds0 += wk * L::kGroup;           // the group's part of the first stage
    auto stage_base = [&](int stage) {
        if constexpr (WAVES_K > 1) return (const uint8_t*)(smem + wk * L::kGroup + stage * L::kStage);
        else return (const uint8_t*)(smem + stage * L::kStage);
    };
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const int tiles_m = (int)((a.M + BM - 1) / BM), tiles_n = (int)((a.N + BN - 1) / BN);
    int pm, pn;
    tile_walk<(BM >= 256 ? 8 : 16)>(tile, tiles_m, tiles_n, pm, pn);
    const int64_t m0 = (int64_t)pm * BM, n0 = (int64_t)pn * BN;
    const int blocks = PART ? kblks : (int)(a.K / KSTAGE);
    const int KT = WAVES_K > 1 ? (blocks - wk + WAVES_K - 1) / WAVES_K : blocks;   // stages in which this wave's group has a block

    // ---- global -> LDS: every lane owns fixed chunks; rows past the edge are clamped to the last
    //      valid row (their products only reach outputs that are never stored) -----------------
    // wave-uniform bases of this tile's three streams, already advanced to the first stage
    // Sparse A is the k-major value buffer: 64 bytes per row and stage, the rows of a stage
    // contiguous, so the tile's stage is one 16 KiB run; dense A is row-major X.
    const int64_t rows_pad = a.rows_pad;    // rows per k block of the k-major operand (whole activation)
    const int64_t a_stride = SPARSE ? rows_pad * 64 : (int64_t)128;   // bytes between stages
    const uint8_t* base_a = SPARSE
        ? static_cast<const uint8_t*>(a.A) + m0 * 64
        : static_cast<const uint8_t*>(a.A) + m0 * a.lda * ESZ;
    const uint8_t* base_b = static_cast<const uint8_t*>(a.W) + n0 * a.ldw * ESZ;
    if constexpr (PART) {
        base_a += kblk0 * a_stride;
        base_b += (int64_t)kblk0 * (KSTAGE * ESZ);
    }
    const int64_t rows_a = a.M - m0, rows_b = a.N - n0;     // valid rows from the tile's first row
    uint32_t oa[A_PER_W];
#pragma unroll
    for (int s = 0; s < A_PER_W; ++s) {
        const int p = (wave * A_PER_W + s) * 64 + lane;
        int row, c;
        if constexpr (SPARSE) unswz4(p, row, c); else unswz8(p, row, c);
        const int64_t gr = min((int64_t)row, rows_a - 1);
        // (the k-major buffer is padded to whole tiles: rows past M hold unspecified bytes whose
        //  products only reach outputs that are never stored)
        oa[s] = SPARSE ? (uint32_t)(row * 64 + c * 16) : (uint32_t)(gr * a.lda * ESZ + c * 16);
    }
    uint32_t ob[B_PER_W];
#pragma unroll
    for (int s = 0; s < B_PER_W; ++s) {
        const int p = wave * B_CH + min(s * 64 + lane, B_CH - 1);   // masked lanes of a half load: any valid chunk
        int row, c;
        unswz8(p, row, c);
        const int64_t gr = min((int64_t)row, rows_b - 1);
        ob[s] = (uint32_t)(gr * a.ldw * ESZ + c * 16);
    }
    const uint8_t* base_m = nullptr;
    uint32_t om = 0;
    if constexpr (SPARSE) {
        // k-major records: the rows of this tile are one contiguous run per stage (2 KiB, 4 KiB with
        // FP8 operands) and wave w moves M_PER_W 256-byte pieces of it, 4 bytes per lane
        base_m = a.meta + m0 * MREC;
        if constexpr (PART) base_m += kblk0 * rows_pad * MREC;
        om = (uint32_t)(wave * M_PER_W * 256 + lane * 4);
    }

    const int64_t meta_stride = rows_pad * MREC;   // bytes between stage blocks
    // PIN: in SGPRs from here on. Left to itself the compiler may walk them along K in VGPRs, with two v_readfirstlane per
    // request, which cost the bf16 loops 1.5 to 2.7 % at [4096, 3072, 12288] and [4608, 12288, 3072]. The FP8 loops of the 256-row
    // plan are not all better off with it (kPinStages).
    if constexpr (PIN) {
        base_a = reinterpret_cast<const uint8_t*>(uniform64(base_a));
        base_b = reinterpret_cast<const uint8_t*>(uniform64(base_b));
        if constexpr (SPARSE) base_m = reinterpret_cast<const uint8_t*>(uniform64(base_m));
    }
    // Load number n (0 .. LOADS_PER_STAGE-1) of this wave for stage kt into ring buffer `stage`.
    // The loads of a stage are issued one at a time between matrix instructions: the texture
    // addresser takes a wave-wide 1 KiB request every ~16 cycles and a wave stalls at a request
    // that finds it busy, so a burst of requests from all waves would leave the matrix cores idle.
    auto gload_one = [&](int kt, int stage, auto n_tag) {
        constexpr int n = decltype(n_tag)::value;
        const uint32_t base = lds0 + stage * L::kStage;
        if constexpr (n < A_PER_W) {
            lds_dma16_so(base_a + (int64_t)(kt * WAVES_K + wk) * a_stride, oa[n], base + (wave * A_PER_W + n) * 1024);
        } else if constexpr (n < A_PER_W + B_PER_W) {
            constexpr int s = n - A_PER_W;
            const uint32_t dst = base + L::kABytes + L::kMetaBytes + (wave * B_CH + s * 64) * 16;
            if constexpr (B_HALF && s == B_PER_W - 1) {
                if (lane < 32) lds_dma16_so(base_b + (int64_t)(kt * WAVES_K + wk) * (KSTAGE * ESZ), ob[s], dst);
            } else {
                lds_dma16_so(base_b + (int64_t)(kt * WAVES_K + wk) * (KSTAGE * ESZ), ob[s], dst);
            }
        } else if constexpr (SPARSE && n < A_PER_W + B_PER_W + M_PER_W) {
            constexpr int s = n - A_PER_W - B_PER_W;
            lds_dma4_so(base_m + (int64_t)(kt * WAVES_K + wk) * meta_stride + s * 256, om,
                        base + L::kABytes + (wave * M_PER_W + s) * 256);
        }
    };
    constexpr int LOADS_PER_STAGE = A_PER_W + B_PER_W + (SPARSE ? M_PER_W : 0);
    auto gload = [&](int kt, int stage) {
        static_for<LOADS_PER_STAGE>([&](auto n) { gload_one(kt, stage, n); });
    };

    // ---- accumulators -------------------------------------------------------------------------
    Acc acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < RB; ++r) acc[i][j][r] = 0.f;

    const int li = lane % S, kb = lane / S;
    // Register r of a block is row 4 kb + reg_row(r) of it. The lane's part goes into one base wherever rows are addressed, so that
    // the rest is constant: as one sum per register, 11 of the 96 paired LDS writes of the sparse 256 x 256 epilogue fell apart.
    auto reg_row = [](int r) { return S == 32 ? 8 * (r / 4) + r % 4 : r; };
    const int64_t lane_row = m0 + wm * WTM + 4 * kb;
    const int arow0 = wm * WTM + li;   // + i * S
    const int brow0 = wn * WTN + li;   // + j * S

    // ---- sparse: a stage in two halves of k. Two sets of fragments, one per half, each filled half a stage ahead ------------
    struct Frags {
        Frag8 a[TM];
        Frag16 b[TN];
    } f[SPARSE ? 2 : 1];
    int ix[TM * IXW], ix_nxt[TM * IXW];      // metadata words of this and the next stage; FP8: word 2 i + half of row block i
    // LDS read e behind the matrix instructions of half H: the fragments of the other half (H = 0: second half of this
    // stage, H = 1: first half of the next), metadata words first, then A fragments, then B column block by column block.
    auto read_half = [&](int stage, auto h_tag, auto e_tag) {
        constexpr int SUB = 1 - decltype(h_tag)::value, e = decltype(e_tag)::value, NI = SUB == 0 ? TM : 0;
        const uint8_t* base = stage_base(stage);
        const uint8_t* bB = base + L::kABytes + L::kMetaBytes;
        if constexpr (e < NI) {
            const uint8_t* rec = base + L::kABytes + (arow0 + e * S) * MREC;
            if constexpr (FP8) {
                const int2 w = reinterpret_cast<const int2*>(rec)[kb];
                ix_nxt[2 * e] = w.x;
                ix_nxt[2 * e + 1] = w.y;
            } else {
                ix_nxt[e] = reinterpret_cast<const int*>(rec)[kb];
            }
        } else if constexpr (e < NI + TM) {
            f[SUB].a[e - NI].u = *reinterpret_cast<const uint4*>(base + swz4(arow0 + (e - NI) * S, 2 * kb + SUB));
        } else if constexpr (e < NI + TM + 2 * TN) {
            constexpr int j = (e - NI - TM) / 2, c = (e - NI - TM) % 2;
            f[SUB].b[j].u[c] = *reinterpret_cast<const uint4*>(bB + swz8(brow0 + j * S, 4 * c + 2 * SUB + kb));
        }
    };
    // Half H of a stage's matrix work. Behind each matrix instruction go two of the LDS reads above (when READ) and one of
    // the ring-refill requests LO <= n < HI of stage kt_load into ring buffer buf. Spreading both keeps the LDS command
    // queue and the texture addresser from filling up, which would stall the wave in front of its next matrix instruction.
    constexpr int NMMA = TM * TN;
    auto half = [&](auto h_tag, auto read_tag, int rstage, auto lo_tag, auto hi_tag, int kt_load, int buf) {
        constexpr int H = decltype(h_tag)::value, LO = decltype(lo_tag)::value, CNT = decltype(hi_tag)::value - LO;
        constexpr int LPM = (CNT + NMMA - 1) / NMMA;          // requests behind each matrix instruction (one, but for small wave tiles)
        constexpr int READS = (H == 1 ? TM : 0) + TM + 2 * TN;
        static_for<NMMA>([&](auto n_tag) {
            constexpr int n = decltype(n_tag)::value, i = n % TM, j = n / TM;
            if constexpr (!SPARSE) return;
            else if constexpr (FP8)
                acc[i][j] = __builtin_amdgcn_smfmac_f32_32x32x64_fp8_fp8(f[H].a[i].q, f[H].b[j].q, acc[i][j], ix[2 * i + H], 0, 0);
            else
                acc[i][j] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(f[H].a[i].v, f[H].b[j].v, acc[i][j], ix[i], 0, H);
            constexpr int e1 = n == NMMA - 1 ? READS : 2 * n + 2;
            if constexpr (decltype(read_tag)::value)
                static_for<(e1 > 2 * n ? e1 - 2 * n : 0)>([&](auto e) { read_half(rstage, h_tag, std::integral_constant<int, 2 * n + decltype(e)::value>{}); });
            constexpr int g0 = n * LPM < CNT ? n * LPM : CNT, g1 = (n + 1) * LPM < CNT ? (n + 1) * LPM : CNT;
            static_for<g1 - g0>([&](auto e) { gload_one(kt_load, buf, std::integral_constant<int, LO + g0 + decltype(e)::value>{}); });
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    // ---- dense: a stage row block by row block, two matrix instructions (chunks of k) per block, the barrier behind the first
    //      R0 row blocks. One set of fragments: the A registers of a row block are refilled for the next stage behind its last
    //      matrix instruction, the B registers behind theirs in the last row block (two sets would not fit beside
    //      256 x 256 accumulators) -----------------------------------------------------------------------------------
    constexpr int R0 = TM >= 4 ? 2 : 1, ROW = 2 * TN, M1 = (TM - R0) * ROW;       // ROW: matrix instructions of a row block
    Frag16 fa[SPARSE ? 1 : TM], fb[SPARSE ? 1 : TN];
    // LDS read e of a stage: 0 .. 2 TM - 1 the two chunks of each row block, then the chunks of the columns in the order in
    // which the last row block is done with them.
    constexpr int A_RD = 2 * TM, B_RD = 2 * TN;
    auto read_row = [&](int stage, auto e_tag) {
        constexpr int e = decltype(e_tag)::value;
        const uint8_t* base = stage_base(stage);
        const uint8_t* bB = base + L::kABytes;
        if constexpr (e < A_RD)
            fa[e / 2].u[e % 2] = *reinterpret_cast<const uint4*>(base + swz8(arow0 + e / 2 * S, 4 * (e % 2) + kb));
        else
            fb[(e - A_RD) % TN].u[(e - A_RD) / TN] =
                *reinterpret_cast<const uint4*>(bB + swz8(brow0 + (e - A_RD) % TN * S, 4 * ((e - A_RD) / TN) + kb));
    };
    // Which of them go behind which of the M1 matrix instructions that follow the barrier: as soon as their registers are
    // free, evenly spread. (The last row block's two follow the first matrix instructions of the next stage.)
    struct Slots {
        int item[M1][4], count[M1], total;
    };
    static constexpr Slots kSlots = [] {
        Slots t{};
        int a = 0, b = 0;
        for (int m = 0; m < M1; ++m) {
            const int left = A_RD - 2 + B_RD - t.total;
            for (int budget = (left + M1 - m - 1) / (M1 - m); budget > 0 && t.count[m] < 4; --budget) {
                const int rows = R0 + m / ROW;                               // row blocks done with their registers
                if (a < 2 * (rows < TM - 1 ? rows : TM - 1)) t.item[m][t.count[m]++] = a++;
                else if (b < B_RD && b <= m - (M1 - ROW)) t.item[m][t.count[m]++] = A_RD + b++;
                else break;
                ++t.total;
            }
        }
        return t;
    }();
    static_assert(SPARSE || kSlots.total == A_RD - 2 + B_RD, "every read has a slot");
    auto mma_row = [&](auto i_tag, auto n_tag) {             // matrix instruction n of row block i
        constexpr int i = decltype(i_tag)::value, n = decltype(n_tag)::value, j = n % TN, c = n / TN;
        const bf16x16 x = fa[i].v, y = fb[j].v;
        acc[i][j] = dense_mma<S>(c == 0 ? bf16x8(x.lo) : bf16x8(x.hi), c == 0 ? bf16x8(y.lo) : bf16x8(y.hi), acc[i][j]);
    };
    // Requests LO <= n < HI of stage kt_load behind the first HI - LO of every D-th of NM matrix instructions (spread evenly
    // where that does not reach). D = 1 / 2 / 3 / 4 / even, us: [4608, 9216, 3072] 226.0 / 217.3 / 216.4 / 217.3 / 218.3, [4096,
    // 3072, 12288] 279.0 / 261.3 / 262.0 / 265.2, [4608, 3072, 3072] 85.1 / 80.4 / 81.2 / 81.9: a late one arrives late.
    auto requests = [&](auto n_tag, auto nm_tag, auto lo_tag, auto hi_tag, int kt_load, int buf) {
        constexpr int n = decltype(n_tag)::value, NM = decltype(nm_tag)::value, LO = decltype(lo_tag)::value, CNT = decltype(hi_tag)::value - LO;
        constexpr int D = CNT > 0 && NM >= 2 * CNT ? 2 : 1;
        constexpr int g0 = D > 1 ? (n + D - 1) / D : n * CNT / NM, g1 = D > 1 ? n / D + 1 : (n + 1) * CNT / NM;
        static_for<(g0 < g1 && (D == 1 || g0 < CNT) ? g1 - g0 : 0)>(
            [&](auto e) { gload_one(kt_load, buf, std::integral_constant<int, LO + g0 + decltype(e)::value>{}); });
    };

    // The barrier of a stage. A group of one wave shares its ring with nobody: its own waits are enough.
    auto stage_barrier = [&]() {
        asm volatile("" ::: "memory");
        if constexpr (NW > 1) __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    // ---- prologue: the whole ring in flight, stage 0 visible ----------------------------------
#pragma unroll
    for (int s = 0; s < STAGES; ++s)
        if (s < KT) gload(s, s);
    if (KT >= STAGES) wait_vmcnt_lgkm0<(STAGES - 1) * LOADS_PER_STAGE>();
    else wait_vmcnt_lgkm0<0>();
    stage_barrier();

    if (WAVES_K == 1 || KT > 0) {
        if constexpr (SPARSE) {
            static_for<2 * TM + 2 * TN>([&](auto e) { read_half(0, std::integral_constant<int, 1>{}, e); });
#pragma unroll
            for (int i = 0; i < TM * IXW; ++i) ix[i] = ix_nxt[i];
        } else {
            static_for<A_RD - 2>([&](auto e) { read_row(0, e); });
            static_for<B_RD>([&](auto e) { read_row(0, std::integral_constant<int, A_RD + decltype(e)::value>{}); });
        }
    }
    wait_vmcnt_lgkm0<63>();            // first fragments are in registers

    // One stage of the main loop. Schedule inside a stage kt:
    //   matrix work of the first part, interleaved with the rest of the reads of stage kt and the second part of the
    //   requests of stage kt+STAGES-1 (its buffer, the one of stage kt-1, was released by the previous barrier) |
    //   wait: own reads of stage kt done, stage kt+1 landed | barrier |
    //   matrix work of the second part, interleaved with the first reads of stage kt+1 and the first part of the
    //   requests of stage kt+STAGES (into the buffer of stage kt, which nobody reads any more).
    // Every stage has about two stage times to arrive and the request stream never bursts.
    // PENDING: whole stages younger than kt+1 in flight at the wait (compile-time per phase).
    // SPLIT: requests issued in the second half. A ring of two has no buffer to spare for the early part:
    // all requests of stage kt+2 go out after the barrier of stage kt, one stage time ahead.
    constexpr int SPLIT = STAGES == 2 ? LOADS_PER_STAGE : (LOADS_PER_STAGE + 1) / 2;
    using c0 = std::integral_constant<int, 0>;
    using c1 = std::integral_constant<int, 1>;
    using cS = std::integral_constant<int, SPLIT>;
    using cL = std::integral_constant<int, LOADS_PER_STAGE>;
    using T = std::true_type;
    using F = std::false_type;
    int cur = 0;                       // LDS buffer of stage kt
    auto stage_step = [&](int kt, auto load_a, auto load_b, auto has_next, auto pending) {
        constexpr bool LOAD_A = decltype(load_a)::value, LOAD_B = decltype(load_b)::value, HAS_NEXT = decltype(has_next)::value;
        constexpr int PENDING = decltype(pending)::value;
        const int nxt = cur + 1 == STAGES ? 0 : cur + 1;
        const int prv = cur == 0 ? STAGES - 1 : cur - 1;
        using a_lo = std::conditional_t<LOAD_A, cS, c0>;
        using a_hi = std::conditional_t<LOAD_A, cL, c0>;
        using b_hi = std::conditional_t<LOAD_B, cS, c0>;
        if constexpr (SPARSE) half(c0{}, T{}, cur, a_lo{}, a_hi{}, kt + STAGES - 1, prv);
        else static_for<R0 * ROW>([&](auto n) {
            constexpr int m = decltype(n)::value;
            mma_row(std::integral_constant<int, m / ROW>{}, std::integral_constant<int, m % ROW>{});
            if constexpr (m < 2) read_row(cur, std::integral_constant<int, A_RD - 2 + m>{});
            requests(n, std::integral_constant<int, R0 * ROW>{}, a_lo{}, a_hi{}, kt + STAGES - 1, prv);
            __builtin_amdgcn_sched_barrier(0);
        });
        wait_vmcnt_lgkm0<PENDING * LOADS_PER_STAGE>();
        stage_barrier();
        if constexpr (SPARSE) half(c1{}, has_next, nxt, c0{}, b_hi{}, kt + STAGES, cur);
        else static_for<M1>([&](auto n) {
            constexpr int m = decltype(n)::value;
            mma_row(std::integral_constant<int, R0 + m / ROW>{}, std::integral_constant<int, m % ROW>{});
            if constexpr (HAS_NEXT)
                static_for<kSlots.count[m]>([&](auto e) { read_row(nxt, std::integral_constant<int, kSlots.item[m][decltype(e)::value]>{}); });
            requests(n, std::integral_constant<int, M1>{}, c0{}, b_hi{}, kt + STAGES, cur);
            __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (HAS_NEXT && SPARSE) {
#pragma unroll
            for (int i = 0; i < TM * IXW; ++i) ix[i] = ix_nxt[i];
        }
        cur = nxt;
    };
    static_assert(STAGES == 2 || STAGES == 3 || STAGES == 4, "ring depth");
    using P = std::integral_constant<int, STAGES - 2>;
    int kt = 0;
    if (WAVES_K == 1 || KT > 0) {
        if (KT > STAGES) {
            // stage 0 has no half-requested predecessor; from then on both halves carry requests
            stage_step(kt, F{}, T{}, T{}, P{});
            for (kt = 1; kt < KT - STAGES; ++kt) stage_step(kt, T{}, T{}, T{}, P{});
            // second part of the last stage; nothing new afterwards
            stage_step(kt, T{}, F{}, T{}, P{});
            ++kt;
        }
        // drain (and short K): stages kt+1 .. KT-1 are all requested; fewer remain in flight each step
        if constexpr (STAGES >= 4) {
            if (kt == KT - 4) { stage_step(kt, F{}, F{}, T{}, std::integral_constant<int, 2>{}); ++kt; }
        }
        if constexpr (STAGES >= 3) {
            if (kt == KT - 3) { stage_step(kt, F{}, F{}, T{}, std::integral_constant<int, 1>{}); ++kt; }
        }
        if (kt == KT - 2) { stage_step(kt, F{}, F{}, T{}, std::integral_constant<int, 0>{}); ++kt; }
        stage_step(kt, F{}, F{}, F{}, std::integral_constant<int, 0>{});
    }
    if constexpr (WAVES_K > 1 && NW > 1) {
        if (KT < (blocks + WAVES_K - 1) / WAVES_K) stage_barrier();   // no block in the last stage: the barrier only
    }

    const bool own_factor = FOLDED && a.rowsums;
    // Only the sparse product has factors. (Known at compile time it keeps their 32 registers out of the 256 x 256 dense epilogue,
    // which spilled seven of its own without it.)
    const bool has_row_scale = SPARSE && a.row_scale, has_tensor_scale = SPARSE && (own_factor || a.tensor_scale);
    auto tensor_scale = [&]() { return own_factor ? a.folded : (has_tensor_scale ? a.tensor_scale[0] : 1.0f); };

    if constexpr (WAVES_K > 1) {
        // ---- add the K groups up in LDS, factors, residual, bias, bf16, store --------------------------------
        wait_vmcnt_lgkm0<0>();
        __syncthreads();                         // the ring is free
        float* const planes = reinterpret_cast<float*>(smem);
        auto put_plane = [&](const Acc (&v)[TM][TN]) {       // this wave's block of its group's plane
            float* p = planes + wk * (L::kPlane / 4) + (wm * WTM + 4 * kb) * L::kPitch + wn * WTN + li;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int r = 0; r < RB; ++r)
                        p[(i * S + reg_row(r)) * L::kPitch + j * S] = v[i][j][r];
        };
        constexpr int THREADS = NW * WAVES_K * 64;
        constexpr int CPR = BN / 8, CHUNKS = BM * CPR;       // a thread finishes runs of 8 columns
        constexpr int PER = (CHUNKS + THREADS - 1) / THREADS;
        float sum[PER][8];
        auto add_planes = [&](float (&out)[8], int row, int c) {
            const float* p = planes + row * L::kPitch + c * 8;
#pragma unroll
            for (int e = 0; e < 8; ++e) out[e] = p[e];
#pragma unroll
            for (int g = 1; g < WAVES_K; ++g)
#pragma unroll
                for (int e = 0; e < 8; ++e) out[e] += p[g * (L::kPlane / 4) + e];
        };
        put_plane(acc);
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int q = u * THREADS + (int)threadIdx.x;
            if (q < CHUNKS) add_planes(sum[u], q / CPR, q % CPR);
        }
        float res[MODE == 1 ? PER : 1][8];
        if constexpr (MODE == 1) {
            // Residual Y_r = T L_A^T (T = X L_B^T as two bf16 planes hi + lo, rank 64): steps of 16 or 32 ranks
            // dealt over the K groups, operands straight from memory (a few KB that sit in L2),
            // added up through the same planes. The factors belong to the sparse product only.
            constexpr int RANKS = 512 / S, STEPS = 2 * kLoraRank / RANKS;        // ranks of a step; steps of both planes
            Acc t[TM][TN];
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int r = 0; r < RB; ++r) t[i][j][r] = 0.f;
            for (int s = wk; s < STEPS; s += WAVES_K) {
                const uint16_t* tp = a.T + (s & 1 ? 0 : a.t_plane);      // lo plane first
                const int col = (s >> 1) * RANKS + 8 * kb;
                Frag8 ft[TM], fl[TN];
#pragma unroll
                for (int i = 0; i < TM; ++i)
                    ft[i].u = *reinterpret_cast<const uint4*>(tp + min(m0 + arow0 + i * S, a.M - 1) * kLoraRank + col);
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    fl[j].u = *reinterpret_cast<const uint4*>(a.LA + min(n0 + brow0 + j * S, a.N - 1) * a.ldla + col);
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int i = 0; i < TM; ++i) t[i][j] = dense_mma<S>(ft[i].v, fl[j].v, t[i][j]);
            }
            __syncthreads();                                 // the sparse planes have been read
            put_plane(t);
            __syncthreads();
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const int q = u * THREADS + (int)threadIdx.x;
                if (q < CHUNKS) add_planes(res[u], q / CPR, q % CPR);
            }
        }
        // the runs of a thread share their eight columns
        static_assert(THREADS % CPR == 0, "a thread keeps its columns");
        const int64_t col = n0 + ((int)threadIdx.x % CPR) * 8;
        const int valid = (int)min((int64_t)8, a.N - col);   // columns of the run inside Y
        if (valid <= 0) return;
        float bv[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) bv[e] = 0.f;
        if (a.bias) {
            uint16_t b16[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) b16[e] = a.bias[col + min(e, valid - 1)];
#pragma unroll
            for (int e = 0; e < 8; ++e) bv[e] = __uint_as_float((uint32_t)b16[e] << 16);
        }
        float f[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int64_t row = m0 + (u * THREADS + (int)threadIdx.x) / CPR;
            f[u] = has_row_scale ? a.row_scale[min(row, a.M - 1)] : 1.0f;
        }
        const float ts = tensor_scale();
        const bool wide_ok = ((reinterpret_cast<uintptr_t>(a.Y) & 15) == 0) && (a.ldy % 8 == 0) && valid == 8;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int q = u * THREADS + (int)threadIdx.x;
            const int64_t row = m0 + q / CPR;
            if (q >= CHUNKS || row >= a.M) continue;
            typedef float f32x2 __attribute__((ext_vector_type(2)));
            typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
            uint32_t out[4];
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
                f32x2 y;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    float add = bv[e + h];
                    if constexpr (MODE == 1) add += res[u][e + h];
                    y[h] = mul_add_rn(sum[u][e + h], f[u] * ts, add);
                }
                out[e / 2] = __builtin_bit_cast(uint32_t, __builtin_convertvector(y, bf16x2));   // RNE
            }
            uint16_t* dst = a.Y + row * a.ldy + col;
            if (wide_ok) {
                *reinterpret_cast<uint4*>(dst) = make_uint4(out[0], out[1], out[2], out[3]);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (e < valid) dst[e] = (uint16_t)(out[e >> 1] >> (16 * (e & 1)));
            }
        }
        return;
    }

    const float ts = tensor_scale();

    if constexpr (MODE == 1 && WAVES_K == 1) {
        // ---- LoRA tail (Alg. 1: Y <- Y_s + Y_r, accumulated on chip) --------------------------
        // The ROW / TENSOR factors belong to the sparse product only, so they are applied to the
        // accumulators first. Then Y_r = T L_A^T, T = X L_B^T (bf16 [M,64]), is added by four dense
        // matrix-instruction steps over the rank; SMFMAC and MFMA of one size share one accumulator layout.
        if (has_row_scale || has_tensor_scale) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int r = 0; r < RB; ++r) {
                    const int64_t row = min(lane_row + (i * S + reg_row(r)), a.M - 1);
                    const float f = (has_row_scale ? a.row_scale[row] : 1.0f) * ts;
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[i][j][r] *= f;
                }
        }
      if (!PART || part == 0) {                // (of several partial planes the first carries the residual)
        wait_vmcnt_lgkm0<0>();
        __builtin_amdgcn_s_barrier();          // the ring is free: reuse it for the two rank tiles
        constexpr int T_LOADS = BM * 128 / 1024, LA_LOADS = BN * 128 / 1024;   // rows of 64 bf16
        static_assert(T_LOADS % NW == 0, "rank tiles must divide over the waves");
        static_assert((2 * BM + BN) * 128 <= L::kTotal, "rank tiles fit in the ring");
        const int64_t plane = a.t_plane;                // T is two bf16 planes: hi, lo
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int s = 0; s < T_LOADS / NW; ++s) {
                const int p = (wave * (T_LOADS / NW) + s) * 64 + lane;
                int row, c;
                unswz8(p, row, c);
                lds_dma16(a.T + h * plane + min(m0 + row, a.M - 1) * kLoraRank + c * 8,
                          lds0 + h * BM * 128 + (wave * (T_LOADS / NW) + s) * 1024);
            }
#pragma unroll
        for (int s = 0; s < (LA_LOADS + NW - 1) / NW; ++s) {
            const int unit = s * NW + wave;
            if (unit >= LA_LOADS) break;
            const int p = unit * 64 + lane;
            int row, c;
            unswz8(p, row, c);
            lds_dma16(a.LA + min(n0 + row, a.N - 1) * a.ldla + c * 8, lds0 + 2 * BM * 128 + unit * 1024);
        }
        wait_vmcnt_lgkm0<0>();
        __builtin_amdgcn_s_barrier();
#pragma unroll
        for (int sub = 0; sub < kLoraRank * S / 512; ++sub) {      // 512 / S ranks each
            Frag8 lb[TN];
            const int c = 64 / S * sub + kb;
#pragma unroll
            for (int j = 0; j < TN; ++j)
                lb[j].u = *reinterpret_cast<const uint4*>(smem + 2 * BM * 128 + swz8(brow0 + j * S, c));
#pragma unroll
            for (int h = 1; h >= 0; --h) {             // lo plane first
                Frag8 t[TM];
#pragma unroll
                for (int i = 0; i < TM; ++i)
                    t[i].u = *reinterpret_cast<const uint4*>(smem + h * BM * 128 + swz8(arow0 + i * S, c));
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int i = 0; i < TM; ++i) acc[i][j] = dense_mma<S>(t[i].v, lb[j].v, acc[i][j]);
            }
        }
      }
    }

    if constexpr (PART) {
        // S lanes of a register hold S neighbouring columns of one row
        float* plane = a.partials + (int64_t)part * a.M * a.part_pitch;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int64_t col = n0 + wn * WTN + j * S + li;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int r = 0; r < RB; ++r) {
                    const int64_t row = lane_row + (i * S + reg_row(r));
                    if (row < a.M && col < a.N) plane[row * a.part_pitch + col] = acc[i][j][r];
                }
        }
        return;
    }

    // ---- epilogue: optional fp32 scales, bias, bf16 RNE, store --------------------------------
    auto finish = [&](float v, int64_t row, float bv) {
        if constexpr (MODE != 1) {
            if (has_row_scale) v *= a.row_scale[row];
            if (has_tensor_scale) v *= ts;
        }
        if (a.bias) v += bv;
        return (uint16_t)f32_to_bf16_rne(v);
    };
    const bool wide_ok = ((reinterpret_cast<uintptr_t>(a.Y) & 15) == 0) && (a.ldy % 8 == 0);
    if (wide_ok) {
        // The accumulator layout gives a lane one column and scattered rows, i.e. 2-byte stores.
        // Each wave therefore transposes its tile through a private LDS region (the ring is no
        // longer needed) and writes whole 16-byte row segments.
        constexpr int ROWB = L::kEpiRowBytes;
        wait_vmcnt_lgkm0<0>();
        __builtin_amdgcn_s_barrier();     // every wave is done reading the ring
        uint8_t* ep = smem + wave * (WTM * ROWB);
        // Two accumulator registers (rows r, r + PS of one column) are converted by one packed
        // fp32 -> bf16 instruction (round to nearest even). The plain case (no factors, no bias) is kept
        // free of any other per-element work: with 128 elements per lane the epilogue is otherwise bound
        // by its vector ALU work, not by stores.
        typedef float f32x2 __attribute__((ext_vector_type(2)));
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        // A lane holds rows rl, rl + PS of ONE column; its neighbour (lane ^ 1) holds the same rows
        // of the next column. The pair swaps halves (one DPP move, one byte permute) so that the
        // even lane owns row rl and the odd lane row rl + PS of BOTH columns: one 32-bit LDS write
        // per lane instead of two 16-bit ones. (S = 16: rows two apart, so that the eight runs of eight words that one
        // write consists of fall into different banks.)
        constexpr int PS = S == 32 ? 1 : 2;
        const bool odd = lane & 1;
        const uint32_t sel = odd ? 0x03020706u : 0x05040100u;   // v_perm_b32: bytes 0-3 = own, 4-7 = partner
        uint8_t* const ep_lane = ep + (4 * kb + (odd ? PS : 0)) * ROWB + (li & ~1) * 2;   // odd lanes write the row PS below
        auto put2 = [&](float v0, float v1, int rl, int cl) {   // rl, cl: beyond the lane's own row and column, constants
            const f32x2 pv = {v0, v1};
            const uint32_t own = __builtin_bit_cast(uint32_t, __builtin_convertvector(pv, bf16x2));
            const uint32_t partner = (uint32_t)__builtin_amdgcn_mov_dpp((int)own, 0xB1, 0xF, 0xF, true);
            // even: (own.lo, partner.lo) = its row, its column and the next
            // odd : (partner.hi, own.hi) = its row + PS, the column before and its own
            const uint32_t w = __builtin_amdgcn_perm(partner, own, sel);
            *reinterpret_cast<uint32_t*>(ep_lane + rl * ROWB + cl * 2) = w;
        };
        auto first_of_pair = [](int q) { return S == 32 ? 2 * q : q; };     // registers r, r + PS, q = 0 .. RB / 2 - 1
        const bool scaled = MODE != 1 && (has_row_scale || has_tensor_scale);
        if (!scaled && !a.bias) {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int q = 0; q < RB / 2; ++q) {
                        const int r = first_of_pair(q);
                        put2(acc[i][j][r], acc[i][j][r + PS], i * S + reg_row(r), j * S);
                    }
        } else {
            // the factors of the lane's rows per row block are fetched once, not once per column block,
            // four consecutive rows per load, all loads in flight together
            float bv[TN];
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int64_t col = min(n0 + wn * WTN + j * S + li, a.N - 1);
                bv[j] = a.bias ? __uint_as_float((uint32_t)a.bias[col] << 16) : 0.f;
            }
            float fr[TM][RB];
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int q = 0; q < RB / 4; ++q) {  // registers 4 q .. 4 q + 3 are four consecutive rows
                    const int64_t row = lane_row + (i * S + reg_row(4 * q));
                    if (!scaled || !has_row_scale) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) fr[i][4 * q + e] = 1.0f;
                    } else if (row + 3 < a.M && (reinterpret_cast<uintptr_t>(a.row_scale + row) & 15) == 0) {
                        const float4 v = *reinterpret_cast<const float4*>(a.row_scale + row);
                        fr[i][4 * q] = v.x; fr[i][4 * q + 1] = v.y; fr[i][4 * q + 2] = v.z; fr[i][4 * q + 3] = v.w;
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) fr[i][4 * q + e] = a.row_scale[min(row + e, a.M - 1)];
                    }
                }
            const float tsf = scaled ? ts : 1.0f;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int q = 0; q < RB / 2; ++q) {
                        const int r = first_of_pair(q);
                        put2(acc[i][j][r] * (fr[i][r] * tsf) + bv[j], acc[i][j][r + PS] * (fr[i][r + PS] * tsf) + bv[j],
                             i * S + reg_row(r), j * S);
                    }
        }
        // same wave reads back what it wrote: LDS operations of a wave complete in order
        constexpr int CPR = WTN / 8;               // 16-byte chunks per tile row
        constexpr int CHUNKS = WTM * CPR;
#pragma unroll
        for (int q0 = 0; q0 < CHUNKS; q0 += 64) {
            const int q = q0 + lane;
            if (q < CHUNKS) {
                const int rl = q / CPR, c = q % CPR;
                const int64_t row = m0 + wm * WTM + rl, col = n0 + wn * WTN + c * 8;
                if (row < a.M && col < a.N) {
                    const uint4 v = *reinterpret_cast<const uint4*>(ep + rl * ROWB + c * 16);
                    uint16_t* dst = a.Y + row * a.ldy + col;
                    if (col + 8 <= a.N) {
                        *reinterpret_cast<uint4*>(dst) = v;
                    } else {
                        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
                        for (int e = 0; e < 8 && col + e < a.N; ++e)
                            dst[e] = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
                    }
                }
            }
        }
    } else {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int64_t col = n0 + wn * WTN + j * S + li;
            if (col >= a.N) continue;
            const float bv = a.bias ? __uint_as_float((uint32_t)a.bias[col] << 16) : 0.f;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
#pragma unroll
                for (int r = 0; r < RB; ++r) {
                    const int64_t row = lane_row + (i * S + reg_row(r));
                    if (row >= a.M) continue;
                    a.Y[row * a.ldy + col] = finish(acc[i][j][r], row, bv);
                }
            }
        }
    }
}

// Two tile shapes in one launch (the "block-parallel" balancing of the method section's kernel
// paragraph, done with tile shapes instead of split contractions): rows [0, m_split) of the output
// are cut into 256 x BN body tiles, rows [m_split, M) into 256 x 128 tail tiles. Uniform tiles
// leave the chip's last round of workgroups mostly empty for many layer shapes (e.g. 792 tiles on
// 256 compute units: 3.09 rounds cost 4); smaller tiles at the end fill that round at 0.6 of a
// body tile's time. Every XCD works through its share of the body tiles first, then its share of
// the tail tiles (workgroups are dispatched in id order). tail_tiles == 0: a plain one-shape launch.
constexpr int kTailBN = 128;
// Waves and ring of the 256 x 128 tail tile. Sparse: as the body. Dense: a ring of three (144 KB), where the body has room for two:
// with two, a stage is requested only when the one before it has landed, and a plan of tail tiles alone (the operands arrive
// more slowly than they are used) waits for every stage in full. 64 x 64 per wave instead of 128 x 32, because the columns'
// fragments are refilled behind one row block's instructions and two of them are too few to hide it. us: [2967, 2624, 7936] 149.0 -> 111.9
// (128 x 32 112.7), [3900, 2040, 3072] 62.5 -> 47.5 (48.2), [2967, 2624, 1024] 20.2 -> 18.8 (19.5), [6468, 2848, 5056] 203.1 -> 174.3.
template <bool SPARSE>
struct Tail {
    static constexpr int kWavesM = SPARSE ? 2 : 4, kWavesN = SPARSE ? 4 : 2;
    static constexpr int stages(int body) { return SPARSE ? body : 3; }
};
template <bool SPARSE, int BN, int WAVES_M, int WAVES_N, int STAGES, int MODE, bool FP8, bool PIN>
__global__ __launch_bounds__(512) void gemm_mixed_kernel(const GemmArgs a) {
    static_assert(WAVES_M * WAVES_N == 8, "both tile shapes run with eight waves");
    const int xcd = (int)blockIdx.x % 8, local = (int)blockIdx.x / 8;
    const int nb = a.body_tiles, nt = a.tail_tiles;
    const int nb_x = nb / 8 + (xcd < nb % 8);
    if (local < nb_x) {
        GemmArgs b = a;
        if (nt > 0) b.M = a.m_split;
        gemm_tile<SPARSE, 256, BN, WAVES_M, WAVES_N, STAGES, MODE, FP8, 1, false, false, PIN>(b, xcd_share_start(nb, xcd) + local);
    } else {
        // the tail region as a problem of its own: same operands, shifted by m_split rows
        constexpr int ESZ = FP8 ? 1 : 2;
        GemmArgs t = a;
        t.M = a.M - a.m_split;
        t.A = static_cast<const uint8_t*>(a.A) + (SPARSE ? a.m_split * 64 : a.m_split * a.lda * ESZ);
        if constexpr (SPARSE) t.meta = a.meta + a.m_split * (FP8 ? 16 : 8);
        t.Y = a.Y + a.m_split * a.ldy;
        if (a.row_scale) t.row_scale = a.row_scale + a.m_split;
        if constexpr (MODE == 1) t.T = a.T + a.m_split * kLoraRank;
        const int idx = xcd_share_start(nb + nt, xcd) - xcd_share_start(nb, xcd) + (local - nb_x);
        gemm_tile<SPARSE, 256, kTailBN, Tail<SPARSE>::kWavesM, Tail<SPARSE>::kWavesN, Tail<SPARSE>::stages(STAGES), MODE, FP8, 1, false, false,
                  PIN>(t, idx);
    }
}

// The tile loops need more dynamic LDS than the default limit of a launch: the limit is raised once
// per kernel by the prepare functions (called for every configuration from prepare_gemm_kernels, i.e.
// from rtl_init or from the first entry-point call on a device), never from a launch, so that launches
// consist of the kernel node only and can be recorded into a HIP graph.
template <bool SPARSE, int BN, int WAVES_M, int WAVES_N, int STAGES, int MODE = 0, bool FP8 = false, bool PIN = !FP8>
struct Mixed {
    using LB = Smem<SPARSE, 256, BN, STAGES, WAVES_M, WAVES_N, FP8>;
    using LT = Smem<SPARSE, 256, kTailBN, Tail<SPARSE>::stages(STAGES), Tail<SPARSE>::kWavesM, Tail<SPARSE>::kWavesN, FP8>;
    static constexpr int kLds = LB::kTotal > LT::kTotal ? LB::kTotal : LT::kTotal;
    static hipError_t prepare() {
        auto kern = gemm_mixed_kernel<SPARSE, BN, WAVES_M, WAVES_N, STAGES, MODE, FP8, PIN>;
        return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
    }
    // a.m_split, a.body_tiles and a.tail_tiles come from the planner
    static hipError_t launch(const GemmArgs& a, hipStream_t stream) {
        auto kern = gemm_mixed_kernel<SPARSE, BN, WAVES_M, WAVES_N, STAGES, MODE, FP8, PIN>;
        hipLaunchKernelGGL(kern, dim3((unsigned)(a.body_tiles + a.tail_tiles)), dim3(512), kLds, stream, a);
        return hipGetLastError();
    }
};

// One tile shape per launch, for problems that leave the chip idle with the 256-row tiles above: few tokens
// (the text stream, short prompts, small images) or narrow layers. Those are bound by the chain of stages:
// a compute unit pulls about 95 GB/s of operands that miss its L2 (64 KB in flight over the 0.7 us a stage
// takes to arrive), whatever its waves do, so a call ends sooner the more units pull and the fewer bytes each
// of them has to. Small tiles give more units a part, and inside a tile the waves split the contraction
// (WAVES_K groups, a block each per stage), which keeps all of LDS in flight without more waves per block.
// Whole calls, [M, N, K], 256-row tiles -> these (us, GROUP scope with bias, graph replay):
//   sparse  [37, 3072, 12288] 73 -> 22, [256, 512, 512] 11.0 -> 7.3, [512, 3072, 3072] 26.9 -> 18.2,
//           [512, 3072, 12288] 77 -> 46, [1024, 3072, 3072] 29.8 -> 25.5
//   dense   [37, 3072, 12288] 129 -> 20, [333, 3072, 12288] 142 -> 52, [1024, 3072, 3072] 42 -> 24
template <bool SPARSE, int BM, int BN, int WAVES_M, int WAVES_N, int WAVES_K, int STAGES, int MODE = 0, bool FP8 = false>
__global__ __launch_bounds__(WAVES_M * WAVES_N * WAVES_K * 64) void gemm_split_kernel(const GemmArgs a) {
    const int total = (int)(((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN));
    const int xcd = (int)blockIdx.x % 8, local = (int)blockIdx.x / 8;
    GemmArgs b = a;
    if constexpr (SPARSE) {
        if (a.rowsums) {
            // TENSOR scope: every workgroup adds the rows' sums up for itself (a few KB from L2, 1 to 2 us), which
            // spares the launch that would do only this (4.7 us and the gap before it)
            const float sc = tensor_factor(a.rowsums, a.M, a.factor_eps);
            b.folded = a.factor_mul ? a.factor_mul[0] * sc : sc;
            if (blockIdx.x == 0 && threadIdx.x == 0) {
                a.factor_out[0] = sc;
                if (a.factor_fused) a.factor_fused[0] = b.folded;
            }
        }
    }
    gemm_tile<SPARSE, BM, BN, WAVES_M, WAVES_N, STAGES, MODE, FP8, WAVES_K, false, SPARSE>(b, xcd_share_start(total, xcd) + local);
}

template <bool SPARSE, int BM, int BN, int WAVES_M, int WAVES_N, int WAVES_K, int STAGES, int MODE = 0, bool FP8 = false>
struct Split {
    using L = Smem<SPARSE, BM, BN, STAGES, WAVES_M, WAVES_N, FP8, WAVES_K>;
    static hipError_t prepare() {
        auto kern = gemm_split_kernel<SPARSE, BM, BN, WAVES_M, WAVES_N, WAVES_K, STAGES, MODE, FP8>;
        return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, L::kTotal);
    }
    static hipError_t launch(const GemmArgs& a, hipStream_t stream) {
        auto kern = gemm_split_kernel<SPARSE, BM, BN, WAVES_M, WAVES_N, WAVES_K, STAGES, MODE, FP8>;
        const int64_t tiles = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
        hipLaunchKernelGGL(kern, dim3((unsigned)tiles), dim3(WAVES_M * WAVES_N * WAVES_K * 64), L::kTotal, stream, a);
        return hipGetLastError();
    }
};

// Contraction split over workgroups (PART): a.k_splits workgroups per tile, each with an even share of the k blocks,
// and split_reduce_kernel over their planes. For problems whose tiles do not reach all compute units and whose
// contraction is long enough to pay for the planes (M x N x 4 bytes each way per split) and the second launch.
// Whole calls, best unsplit shape -> split (us): dense [200, 3072, 12288] 36.9 -> 28.7, [333, 3072, 12288] 51.6 -> 37.6,
// [512, 1024, 12288] 29.7 -> 23.6; sparse [333, 3072, 12288] 44.4 -> 37.3, [700, 3072, 12288] 66.2 -> 55.7; LoRA [512, 3072,
// 12288] 55.9 -> 51.3.
template <bool SPARSE, int BM, int BN, int WAVES_M, int WAVES_N, int STAGES, int MODE = 0, bool FP8 = false>
__global__ __launch_bounds__(WAVES_M * WAVES_N * 64) void gemm_part_kernel(const GemmArgs a) {
    const int tiles = (int)(((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN)), total = tiles * a.k_splits;
    const int xcd = (int)blockIdx.x % 8, local = (int)blockIdx.x / 8;
    const int idx = xcd_share_start(total, xcd) + local;       // an XCD's share: few parts, neighbouring tiles
    const int part = idx / tiles, blocks = (int)(a.K / (FP8 ? 128 : 64));
    const int b0 = (int)((int64_t)blocks * part / a.k_splits), b1 = (int)((int64_t)blocks * (part + 1) / a.k_splits);
    gemm_tile<SPARSE, BM, BN, WAVES_M, WAVES_N, STAGES, MODE, FP8, 1, true>(a, idx % tiles, part, b0, b1 - b0);
}

// Adds the planes up in order, then factors, bias, bf16. A thread finishes eight columns of a row, the planes'
// loads in flight together; grid (column chunks / 256, rows).
constexpr int kMaxKSplits = 8;
__global__ __launch_bounds__(256) void split_reduce_kernel(const GemmArgs a, const bool factors) {
    const int64_t row = blockIdx.y, col = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8;
    if (col >= a.N) return;
    const float* p = a.partials + row * a.part_pitch + col;
    float4 v[kMaxKSplits][2];
#pragma unroll
    for (int s = 0; s < kMaxKSplits; ++s)
        if (s < a.k_splits) {
            v[s][0] = *reinterpret_cast<const float4*>(p + (int64_t)s * a.M * a.part_pitch);
            v[s][1] = *reinterpret_cast<const float4*>(p + (int64_t)s * a.M * a.part_pitch + 4);
        }
    const int valid = (int)min((int64_t)8, a.N - col);
    float bv[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) bv[e] = a.bias ? __uint_as_float((uint32_t)a.bias[col + min(e, valid - 1)] << 16) : 0.f;
    const float f = factors ? (a.row_scale ? a.row_scale[row] : 1.0f) * (a.tensor_scale ? a.tensor_scale[0] : 1.0f) : 1.0f;
    float sum[8] = {v[0][0].x, v[0][0].y, v[0][0].z, v[0][0].w, v[0][1].x, v[0][1].y, v[0][1].z, v[0][1].w};
#pragma unroll
    for (int s = 1; s < kMaxKSplits; ++s)
        if (s < a.k_splits) {
            sum[0] += v[s][0].x; sum[1] += v[s][0].y; sum[2] += v[s][0].z; sum[3] += v[s][0].w;
            sum[4] += v[s][1].x; sum[5] += v[s][1].y; sum[6] += v[s][1].z; sum[7] += v[s][1].w;
        }
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    uint32_t out[4];
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
        const f32x2 y = {mul_add_rn(sum[e], f, bv[e]), mul_add_rn(sum[e + 1], f, bv[e + 1])};
        out[e / 2] = __builtin_bit_cast(uint32_t, __builtin_convertvector(y, bf16x2));       // RNE
    }
    uint16_t* dst = a.Y + row * a.ldy + col;
    if (((reinterpret_cast<uintptr_t>(a.Y) & 15) == 0) && (a.ldy % 8 == 0) && valid == 8) {
        *reinterpret_cast<uint4*>(dst) = make_uint4(out[0], out[1], out[2], out[3]);
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (e < valid) dst[e] = (uint16_t)(out[e >> 1] >> (16 * (e & 1)));
    }
}

template <bool SPARSE, int BM, int BN, int WAVES_M, int WAVES_N, int STAGES, int MODE = 0, bool FP8 = false>
struct Part {
    using L = Smem<SPARSE, BM, BN, STAGES, WAVES_M, WAVES_N, FP8>;
    static hipError_t prepare() {
        auto kern = gemm_part_kernel<SPARSE, BM, BN, WAVES_M, WAVES_N, STAGES, MODE, FP8>;
        return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, L::kTotal);
    }
    static hipError_t launch(const GemmArgs& a, hipStream_t stream) {
        auto kern = gemm_part_kernel<SPARSE, BM, BN, WAVES_M, WAVES_N, STAGES, MODE, FP8>;
        const int64_t tiles = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
        hipLaunchKernelGGL(kern, dim3((unsigned)(tiles * a.k_splits)), dim3(WAVES_M * WAVES_N * 64), L::kTotal, stream, a);
        hipLaunchKernelGGL(split_reduce_kernel, dim3((unsigned)((a.N + 2047) / 2048), (unsigned)a.M), dim3(256), 0, stream, a,
                           MODE == 0);
        return hipGetLastError();
    }
};

}  // namespace

// ---- tile plan ---------------------------------------------------------------------------------
// A launch cuts rows [0, m_split) of the output into 256 x BN body tiles (BN = 256 or 192) and the
// remaining rows into 256 x 128 tail tiles. The main loop is bound by the rate at which a CU can pull
// operand stages out of L2, so a tile's time goes with its bytes per stage: 256x256 moves 51 KB,
// 256x192 43 KB (dense kernel: 64 and 56 KB per 64-k stage); a 256x128 tile was measured at 0.60 to
// 0.66 of a 256x256 tile. The plan is the (BN, m_split) whose simulated schedule ends first: per XCD
// (32 compute units, one workgroup each), workgroups in id order, each to the unit that frees first.
struct TilePlan {
    bool use_192;
    int64_t m_split;     // rows covered by body tiles (a multiple of 256, or M when there is no tail)
    int body_tiles, tail_tiles;
    double cost;         // end of the simulated schedule (KB per stage, as c256 etc. in make_plan)
};

static double simulate_schedule(int64_t nb, int64_t nt, double cb, double ct) {
    double worst = 0.0;
    for (int x = 0; x < 8; ++x) {
        const int64_t tot = nb + nt;
        const int64_t nbx = nb / 8 + (x < nb % 8), cx = tot / 8 + (x < tot % 8);
        double unit[32] = {0};
        for (int64_t i = 0; i < cx; ++i) {
            int best = 0;
            for (int u = 1; u < 32; ++u)
                if (unit[u] < unit[best]) best = u;
            unit[best] += i < nbx ? cb : ct;
        }
        for (int u = 0; u < 32; ++u) worst = unit[u] > worst ? unit[u] : worst;
    }
    return worst;
}

static TilePlan make_plan(int64_t M, int64_t N, bool dense) {
    const double c256 = dense ? 64 : 51, c192 = dense ? 56 : 43, c128 = 0.64 * c256;
    const int64_t tm = (M + 255) / 256;
    const int64_t n256 = (N + 255) / 256, n192 = (N + 191) / 192, n128 = (N + kTailBN - 1) / kTailBN;
    if (tm * n128 > (int64_t)1 << 16) {
        // very large grids: many rounds, the last one no longer matters; pick the cheaper uniform shape
        // by rounds x bytes per stage and skip the simulation (it is linear in the number of tiles)
        const double r256 = (double)((tm * n256 + 255) / 256) * c256, r192 = (double)((tm * n192 + 255) / 256) * c192;
        return r192 < r256 ? TilePlan{true, M, (int)(tm * n192), 0, r192} : TilePlan{false, M, (int)(tm * n256), 0, r256};
    }
    double best_cost = simulate_schedule(tm * n256, 0, c256, c128);
    TilePlan best{false, M, (int)(tm * n256), 0, best_cost};
    auto consider = [&](bool use_192, int64_t p) {
        if (p < 0 || p > tm) return;
        const int64_t nb = p * (use_192 ? n192 : n256), nt = (tm - p) * n128;
        double cost = simulate_schedule(nb, nt, use_192 ? c192 : c256, c128);
        if (nt > 0) cost *= 1.03;          // a tail has to pay for itself
        if (cost < best_cost - 1e-9) {
            best_cost = cost;
            best = TilePlan{use_192, p == tm ? M : p * 256, (int)nb, (int)nt, cost};
        }
    };
    consider(true, tm);
    // body sizes that fill whole rounds of the chip, and a few panels around them
    for (int use_192 = 0; use_192 < 2; ++use_192) {
        const int64_t tn = use_192 ? n192 : n256;
        const int64_t rounds = tm * tn / 256;
        for (int64_t r = rounds; r >= rounds - 1 && r >= 0; --r)
            for (int64_t d = -2; d <= 1; ++d) consider(use_192 != 0, r * 256 / tn + d);
    }
    return best;
}

// Plans are cached per (M, N, kind): the simulation costs tens of microseconds on the host.
static TilePlan plan_for(int64_t M, int64_t N, bool dense) {
    struct Entry { int64_t M, N; bool dense; TilePlan plan; };
    static std::mutex mu;
    static std::vector<Entry> cache;
    std::lock_guard<std::mutex> lock(mu);
    for (const Entry& e : cache)
        if (e.M == M && e.N == N && e.dense == dense) return e.plan;
    const TilePlan p = make_plan(M, N, dense);
    if (cache.size() < 4096) cache.push_back(Entry{M, N, dense, p});
    return p;
}

void tile_plan(int64_t M, int64_t N, bool dense, int64_t out[4]) {
    const TilePlan p = plan_for(M, N, dense);
    out[0] = p.use_192 ? 192 : 256;
    out[1] = p.m_split;
    out[2] = p.body_tiles;
    out[3] = p.tail_tiles;
}

// ---- small tiles -------------------------------------------------------------------------------
// Shapes of gemm_split_kernel with what one workgroup takes alone on its compute unit: `fixed` us (prologue,
// reduction of the K groups, epilogue) plus `block` us per k block, both measured ([1..4096, 3072 | 12288,
// 3072 | 12288], 250 points per operand kind).
struct SplitShape {
    int bm, bn;
    double fixed, block;
};
// Sparse 256 x 96 (eight waves of 32 rows, ring of four) stands between the 128 x 128 tile and the 256-row plan: with the plan's
// 256 x 128 tiles an output of 130 to 192 tiles leaves compute units idle and each of the others pulls 34 KB a stage, here up to 256
// pull 30. Its constants put the line where measurement has it, which is at fewer stages (kFixed96Early) in FP8 and for widths not divisible by
// 8, whose 2-byte stores take the plan's tiles longer ([1289, 3372, 512] 22.3 -> 19.8, [864, 5158, 2048] 41.1 -> 36.4). Forced against the best
// other form at 760 drawn shapes of all sparse kinds that it can run in one pass ([129..16896, 512..21504, 512..15360], inputs from HBM):
// bf16 70 of 490 take it, FP8 75 of 270, 6.7 % and 4.7 % faster in the mean and none slower by 1 % (32 of 200 others: 6.1 %, none slower): sparse
// [793, 4672, 8960] 98.5 -> 86.0 us, [4906, 832, 11392] 137.8 -> 128.2, FP8 [737, 5825, 6400] 52.1 -> 48.7, FP8 + LoRA [434, 10432, 512] 13.9 -> 13.0;
// with a line at 20 stages bf16 lost up to 9 % ([886, 5952, 1280], [3516, 1504, 1536] 22.7 -> 24.5).
// Dense 256 x 96 (ring of three) for the same reason where 256 x 128 tiles (which the plan's tails are) do not reach all units: 108 of 2360 drawn shapes take it, 5.9 % faster
// than the best other form in the mean, 9.7 % slower at worst.
constexpr SplitShape kSparseShapes[] = {
    {32, 32, 1.2, 0.087}, {64, 32, 1.9, 0.108}, {64, 64, 2.4, 0.153}, {128, 64, 2.3, 0.19}, {128, 128, 2.8, 0.30},
    {256, 96, 9.2, 0.325}};
constexpr double kFixed96Early = 3.4;
constexpr SplitShape kDenseShapes[] = {
    {32, 32, 1.45, 0.081}, {64, 32, 1.55, 0.135}, {64, 64, 1.25, 0.19}, {128, 64, 2.5, 0.285}, {128, 128, 3.4, 0.38},
    {256, 96, 3.95, 0.44}};

// How the problem should run. Times are estimated from the measured constants: a small shape needs ceil(tiles / 256)
// passes over the 256 compute units; with more than one, all units pull operands all the time and slow each other down
// beyond the constants, which were taken one workgroup to a unit (factor 1.1; dense 1.24, 128 x 128 1.12 with two passes, 1.3
// with more). The 256-row plan is its simulated schedule times the time per KB of a stage, which grows from 10.7 ns (dense
// 14.6: both operands row-major) while at most 96 units work to 17.2 (20) when all do and share the L2s and the power
// budget. One table serves every operand kind, but for the line of the sparse 256 x 96 tile: the others rank the same way in FP8 and LoRA
// calls (LoRA's residual, 5 us a tile of the 256-row plan, is left out), and LoRA without its residual then sums like the plain call.
// Against every form forced one by one on drawn shapes that played no part in the fit ([1..16896, 512..21504, 512..15360], inputs from
// HBM): sparse of all kinds, 600 shapes: 1.0 % slower than the best on average, more than 2 % slower than the 256-row plan at 2; dense,
// 600 shapes: 0.3 % and 5. (The constants of the dense loop before its 16 x 16 instructions: 2.1 % and 19 of 2360.)
// With the factors at 0.92 (sparse 64 x 64 and 128 x 128) 128 x 128 tiles in several passes lost up to 1.29x to the plan: [1408, 14368,
// 11904] 303 -> 392 us; above 2048 rows they won more than 3 % at 2 of 220.
struct SplitChoice {
    int shape;       // index of the small shape, or -1 for the 256-row plan
    int k_splits;    // > 1: gemm_part_kernel on the 128 x 128 (part_256 false) or 256 x 128 tile
    bool part_256;
};
static int64_t part_pitch(int64_t N) { return (N + 7) / 8 * 8; }     // columns of a plane: whole eight-column chunks
static SplitChoice pick_split(const TilePlan& plan, int64_t M, int64_t N, int64_t blocks, bool dense, bool fp8, size_t room) {
    const double busy = (double)(plan.body_tiles + plan.tail_tiles < 256 ? plan.body_tiles + plan.tail_tiles : 256);
    const double load = busy > 96 ? (busy - 96) / 160 : 0.0;
    const double per_kb = dense ? 0.0146 + 0.0053 * load : 0.0107 + 0.0065 * load;
    double best = (dense ? 3.3 : 3.4) + (double)blocks * plan.cost * per_kb;
    SplitChoice pick{-1, 1, false};
    const SplitShape* shapes = dense ? kDenseShapes : kSparseShapes;
    const int count = dense ? (int)(sizeof(kDenseShapes) / sizeof(SplitShape)) : (int)(sizeof(kSparseShapes) / sizeof(SplitShape));
    for (int i = 0; i < count; ++i) {
        const SplitShape& s = shapes[i];
        const int64_t tiles = ((M + s.bm - 1) / s.bm) * ((N + s.bn - 1) / s.bn);
        if (tiles > 4096) continue;                        // far more than a few passes: never the better one
        double block = s.block;
        if (s.bm == 256) {                                 // one pass only, slower as the chip fills (its rivals are, in the sparse case)
            if (tiles > 256) continue;
            if (dense && tiles > 128) block += 0.0021 * (double)(tiles - 128);
        }
        if (dense && s.bm == 32) block += 0.0005 * (double)(M < 32 ? M : 32);      // (rows past M repeat the last one: less to pull)
        const int64_t passes = (tiles + 255) / 256;
        if (passes > 1 && s.bm >= 128 && s.bn >= 128 && M > 2048) continue;
        // (the dense 64 x 64 line was fitted at long K; with one or two blocks it takes what its neighbours do: [161, 6168, 128]
        // 8.2 us against 7.4 with the 256-row plan and 6.4 with 128 x 64, [1981, 1024, 128] 7.4 / 6.2 / 5.5)
        const double fixed = dense && s.bm == 64 && s.bn == 64 && blocks <= 2 ? 2.4 : !dense && s.bm == 256 && (fp8 || N % 8 != 0) ? kFixed96Early : s.fixed;
        const double several = !dense ? 1.1 : s.bm >= 128 && s.bn >= 128 ? (passes > 2 ? 1.3 : 1.12) : 1.24;
        const double t = (double)passes * (fixed + (double)blocks * block) * (passes > 1 ? several : 1.0);
        if (t < best) {
            best = t;
            pick.shape = i;
        }
    }
    // Contraction split over workgroups: at most one workgroup per compute unit, at least 16 blocks each (dense 20, but 16 from 9 to 64
    // rows, which 32 x 32 tiles would take in full), up to six parts
    // (dense eight). Second launch, writing and reading the planes: 8 us + 0.5 us per MB of planes (dense 5.1 + 0.31); the
    // estimate has to be 2 % better than the best unsplit one.
    const int64_t min_blocks = dense && (M <= 8 || M > 64) ? 20 : 16;
    for (int big = 0; big < 2; ++big) {
        const int64_t tiles = ((M + (big ? 255 : 127)) / (big ? 256 : 128)) * ((N + 127) / 128);
        const double block = big ? (dense ? 0.535 : 0.35) : (dense ? 0.395 : 0.285);
        for (int s = 2; s <= (dense ? kMaxKSplits : 6) && tiles * s <= 256 && blocks / s >= min_blocks; ++s) {
            const double planes = (double)s * (double)M * (double)part_pitch(N) * 4.0;
            if (planes > (double)room) break;
            const double t = (double)((blocks + s - 1) / s) * block + (dense ? 5.1 + planes * 0.31e-6 : 8.0 + planes * 0.5e-6);
            if (t < best * (pick.k_splits > 1 ? 1.0 : 0.98)) {
                best = t;
                pick = SplitChoice{pick.shape, s, big != 0};
            }
        }
    }
    return pick;
}

// Size of the partial planes of the choice made with `room` bytes (0 where the contraction is not split over workgroups).
// launch_gemm makes the same choice with any room from this size up to `room`.
size_t gemm_partial_bytes(bool sparse, bool fp8, int64_t M, int64_t N, int64_t K, size_t room) {
    const int64_t blocks = K / (fp8 ? 128 : 64);
    if (blocks < 32 || ((M + 255) / 256) * ((N + 127) / 128) > 128) return 0;       // (the bound of the loop above at two splits)
    const SplitChoice c = pick_split(plan_for(M, N, !sparse), M, N, blocks, !sparse, fp8, room);
    return c.k_splits > 1 ? (size_t)c.k_splits * (size_t)M * (size_t)part_pitch(N) * 4 : 0;
}

void gemm_choice(bool sparse, bool fp8, int64_t M, int64_t N, int64_t K, size_t room, int out[3]) {
    const SplitChoice c = pick_split(plan_for(M, N, !sparse), M, N, K / (fp8 ? 128 : 64), !sparse, fp8, room);
    out[0] = c.k_splits > 1 ? -1 : c.shape;
    out[1] = c.k_splits;
    out[2] = c.part_256 ? 256 : 128;
}

// FP8 calls of the 256-row plan: stream bases pinned to SGPRs (PIN of gemm_tile) with 256-column bodies from 20 stages of 128 k on.
// Not pinned -> pinned, us: 256-column bodies [14238, 13344, K] K = 1024 193.3 -> 201.6, 1280 224.4 -> 248.5, 2048 282.4 -> 281.0, 2560
// 339.9 -> 337.9, 3072 382.4 -> 374.3; [10000, 20000, K] 1280 231.4 -> 241.8, 2560 357.2 -> 350.8, 3072 404.5 -> 392.8; [12000, 2048, K] 1024
// 40.6 -> 41.2, 2048 59.0 -> 60.7, 2560 65.1 -> 64.2; [9734, 5760, K] 768 63.9 -> 64.0, 2560 117.0 -> 115.7. 192-column bodies [5326, 3680, K]
// 1024 31.8 -> 32.9, 3072 57.2 -> 57.9; [2887, 3072, 6144] 53.8 -> 53.7. (It is W's base that does it; a reason was not found.)
constexpr int kPinStages = 20;

// Runs `op` (launch or prepare) of small shape `i`. Ring depths: as many stages as LDS holds, two workgroups
// per unit for 64 x 64 and 128 x 128 (sparse).
template <bool SPARSE, int MODE, bool FP8, class Op>
static hipError_t with_split(int i, Op op) {
    if constexpr (SPARSE) {
        switch (i) {
            case 0: return op(Split<true, 32, 32, 1, 1, 4, 4, MODE, FP8>{});
            case 1: return op(Split<true, 64, 32, 1, 1, 4, 4, MODE, FP8>{});
            case 2: return op(Split<true, 64, 64, 1, 2, 2, 3, MODE, FP8>{});
            case 3: return op(Split<true, 128, 64, 2, 2, 2, 3, MODE, FP8>{});
            case 4: return op(Split<true, 128, 128, 2, 2, 1, 3, MODE, FP8>{});
            default: return op(Split<true, 256, 96, 8, 1, 1, 4, MODE, FP8>{});
        }
    } else {
        switch (i) {
            case 0: return op(Split<false, 32, 32, 1, 1, 4, 4>{});
            case 1: return op(Split<false, 64, 32, 1, 1, 4, 3>{});
            case 2: return op(Split<false, 64, 64, 1, 2, 2, 4>{});
            case 3: return op(Split<false, 128, 64, 2, 2, 2, 3>{});
            case 4: return op(Split<false, 128, 128, 2, 2, 1, 3>{});
            default: return op(Split<false, 256, 96, 4, 2, 1, 3>{});
        }
    }
}

template <bool SPARSE, int MODE, bool FP8, class Op>
static hipError_t with_part(bool big, Op op) {
    if (big) return op(Part<SPARSE, 256, 128, Tail<SPARSE>::kWavesM, Tail<SPARSE>::kWavesN, 3, MODE, FP8>{});
    return op(Part<SPARSE, 128, 128, 2, 2, 3, MODE, FP8>{});
}

// Every configuration launch_gemm can pick.
hipError_t prepare_gemm_kernels() {
    hipError_t e = hipSuccess;
    auto run = [&](hipError_t r) { if (e == hipSuccess) e = r; };
    run(Mixed<true, 192, 4, 2, 3, 0, true>::prepare());
    run(Mixed<true, 256, 2, 4, 3, 0, true>::prepare());
    run(Mixed<true, 256, 2, 4, 3, 0, true, true>::prepare());
    run(Mixed<true, 192, 4, 2, 3, 1, true>::prepare());
    run(Mixed<true, 256, 2, 4, 3, 1, true>::prepare());
    run(Mixed<true, 256, 2, 4, 3, 1, true, true>::prepare());
    run(Mixed<true, 192, 4, 2, 3, 1>::prepare());
    run(Mixed<true, 192, 4, 2, 3>::prepare());
    run(Mixed<true, 256, 2, 4, 3, 1>::prepare());
    run(Mixed<true, 256, 2, 4, 3>::prepare());
    run(Mixed<false, 192, 2, 4, 2>::prepare());
    run(Mixed<false, 256, 2, 4, 2>::prepare());
    auto prep = [](auto k) { return decltype(k)::prepare(); };
    for (int i = 0; i < 6; ++i) {
        run(with_split<true, 0, false>(i, prep));
        run(with_split<true, 1, false>(i, prep));
        run(with_split<true, 0, true>(i, prep));
        run(with_split<true, 1, true>(i, prep));
        run(with_split<false, 0, false>(i, prep));
    }
    for (int i = 0; i < 2; ++i) {
        run(with_part<false, 0, false>(i != 0, prep));
        run(with_part<true, 0, false>(i != 0, prep));
        run(with_part<true, 1, false>(i != 0, prep));
        run(with_part<true, 0, true>(i != 0, prep));
        run(with_part<true, 1, true>(i != 0, prep));
    }
    return e;
}

hipError_t launch_gemm(bool sparse, const GemmArgs& a_in, hipStream_t stream) {
    GemmArgs a = a_in;
    const TilePlan plan = plan_for(a.M, a.N, !sparse);
    a.m_split = plan.m_split;
    a.body_tiles = plan.body_tiles;
    a.tail_tiles = plan.tail_tiles;
    a.rows_pad = kmajor_rows(a.M);
    a.t_plane = a.M * kLoraRank;
    // The TENSOR factor: formed by the small-tile kernels themselves while that is cheaper than a launch (each of their
    // workgroups reads all rows' sums: up to two passes of workgroups and 2048 rows), else by its own kernel. Whole call
    // [M, 3072, 3072], own kernel -> folded, us: M = 37 12.2 -> 11.1, 512 21.9 -> 20.4, 1024 28.6 -> 27.6; [2000, 512, 1024] 15.4 -> 13.8; 4000 rows lost 0.2.
    const SplitChoice choice = pick_split(plan, a.M, a.N, a.K / (a.fp8 ? 128 : 64), !sparse, a.fp8,
                                          a.partials ? a.partial_bytes : 0);
    if (a.rowsums) {
        bool fold = sparse && choice.k_splits == 1 && choice.shape >= 0 && a.M <= 2048;
        if (fold) {
            const SplitShape& s = kSparseShapes[choice.shape];
            fold = ((a.M + s.bm - 1) / s.bm) * ((a.N + s.bn - 1) / s.bn) <= 512;
        }
        if (!fold) {
            const hipError_t e = launch_tensor_scale(a.rowsums, a.M, a.factor_eps, a.factor_out, stream, a.factor_mul, a.factor_fused);
            if (e != hipSuccess) return e;
            a.rowsums = nullptr;
            a.tensor_scale = a.factor_fused ? a.factor_fused : a.factor_out;
        }
    }
    auto go = [&](auto k) { return decltype(k)::launch(a, stream); };
    if (choice.k_splits > 1) {
        a.k_splits = choice.k_splits;
        a.part_pitch = part_pitch(a.N);
        const bool big = choice.part_256;
        if (!sparse) return with_part<false, 0, false>(big, go);
        if (a.fp8) return a.T ? with_part<true, 1, true>(big, go) : with_part<true, 0, true>(big, go);
        return a.T ? with_part<true, 1, false>(big, go) : with_part<true, 0, false>(big, go);
    }
    const int split = choice.shape;
    if (split >= 0) {
        if (!sparse) return with_split<false, 0, false>(split, go);
        if (a.fp8) return a.T ? with_split<true, 1, true>(split, go) : with_split<true, 0, true>(split, go);
        return a.T ? with_split<true, 1, false>(split, go) : with_split<true, 0, false>(split, go);
    }
    if (sparse && a.fp8) {
        const bool pin = a.K >= 128 * kPinStages;
        if (a.T != nullptr) {          // LoRA tail in bf16 on top of the FP8 product
            if (plan.use_192) return Mixed<true, 192, 4, 2, 3, 1, true>::launch(a, stream);
            if (pin) return Mixed<true, 256, 2, 4, 3, 1, true, true>::launch(a, stream);
            return Mixed<true, 256, 2, 4, 3, 1, true>::launch(a, stream);
        }
        if (plan.use_192) return Mixed<true, 192, 4, 2, 3, 0, true>::launch(a, stream);
        if (pin) return Mixed<true, 256, 2, 4, 3, 0, true, true>::launch(a, stream);
        return Mixed<true, 256, 2, 4, 3, 0, true>::launch(a, stream);
    }
    if (sparse) {
        const bool lora = a.T != nullptr;
        if (plan.use_192) {
            if (lora) return Mixed<true, 192, 4, 2, 3, 1>::launch(a, stream);
            return Mixed<true, 192, 4, 2, 3>::launch(a, stream);
        }
        if (lora) return Mixed<true, 256, 2, 4, 3, 1>::launch(a, stream);
        return Mixed<true, 256, 2, 4, 3>::launch(a, stream);
    }
    // dense: stages of 64 k (whole-line requests on the row-major operands), body tiles with a ring of two
    if (plan.use_192) return Mixed<false, 192, 2, 4, 2>::launch(a, stream);
    return Mixed<false, 256, 2, 4, 2>::launch(a, stream);
}

}  // namespace rtl

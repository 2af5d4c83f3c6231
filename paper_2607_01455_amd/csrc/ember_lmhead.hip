// LM-head weight gradient with the Ember statistics in its epilogue (gfx950).
//
// For an LM head z_m = W h_m the cross-entropy gradient of row i is
// G_i = sum_m (q_mi - 1[y_m = i]) h_m (appendix, "The LM Head Factorizes Like
// the Embedding Table"), i.e. G = dY^T H with dY[T][V] the logits gradient and
// H[T][D] the hidden states.  This kernel forms G with bf16 MFMA (fp32
// accumulation), rounds it once to its storage dtype, stores it, and, from the
// stored values, writes the two partial reductions the Ember step starts from
// (Algorithm 1, the row and column means of g^2):
//   rowpart[tn][i] = sum of g_ij^2 over the tile's columns j,
//   P[tm][j]       = sum of g_ij^2 over the tile's rows i,
// in fixed orders.  The finalize pass of the step reduces both arrays exactly
// as it reduces the statistics pass's partials, so the step's first read of G
// is gone.
//
// Tiling: one block computes a 256 x 256 tile of G (256 rows of the
// vocabulary, 256 hidden columns) with 8 wavefronts, two per SIMD, so one
// wave's MFMAs run while the other waits on LDS or a barrier; wave w owns the
// 64 x 128 part (w % 4, w / 4) as 2 x 4 MFMA 32x32x16 tiles.  The contraction
// runs over the tokens in steps of 32.  Both operands are stored token-major, so
// each step's 32 x 256 slices go from global memory straight into LDS as they are
// (16-byte buffer loads with an LDS destination) and are turned into the MFMA
// operand layout (8 consecutive tokens per lane) by the LDS transpose read
// ds_read_b64_tr_b16.  A ring of four LDS stages keeps the loads of the next
// three steps in flight while a step is multiplied; the operands of each
// 16-token sub-step are read behind the previous sub-step's MFMAs, across the
// step barrier too, so no MFMA waits for an LDS read it follows directly.
//
// What bounds it: operand delivery and power.  At 128256 x 4096 x 16384 (bf16,
// normal data) the kernel takes 13.3-14.8 ms by card, 1160-1295 TFLOP/s, with
// the chip clocked down to ~1.6 GHz; a form of two 64-token stages takes 11.7 ms
// at 2.38 GHz with all-zero operands, 7.6 ms without its operand loads, and 11.5
// ms with the loads and LDS reads but no MFMA.  On one card: operand reads that
// do not cross the barrier 14.5 ms, this form 13.5, two 64-token stages 13.7,
// five 32-token stages 1% slower than four, 4 waves of 128 x 128 parts, which
// read a third less LDS, 15.3 (one wave per SIMD leaves the barrier uncovered).
// Tiles are numbered so that the blocks one XCD runs at a time share a few
// row tiles and a window of column tiles (its L2 holds their slices).

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "ember_launch.h"

namespace ember {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;

constexpr int kGemmWaves = 8;                   // wavefronts per block
constexpr int kThreads = kGemmWaves * kWave;
constexpr int kWavesN = 2;                      // wave grid over the tile: kWavesM x 2
constexpr int kWavesM = kGemmWaves / kWavesN;
constexpr int kBM = kLmheadTile;        // rows of G per block (vocabulary)
constexpr int kBN = kLmheadTile;        // columns of G per block (hidden)
constexpr int kBK = kLmheadK;           // tokens per step
constexpr int kStages = 4;                      // LDS stages (steps in flight)
// Row tiles per group of the tile order: the 32 tiles an XCD runs at a time
// are 2 x 16 (long contractions) or 8 x 4 of row by column tiles.  8 x 4 reads
// 12 operand slices per step instead of 18 (V x 4096 x T, us, groups of 2 / 4 /
// 8: 32000 x 2048 530 / 510 / 501, 128256 x 2048 1902 / 1876 / 1870); over a
// long contraction the tiles drift apart and the wide groups lose
// (128256 x 16384: 13450 / 13540 / 14250; x 8192: 7040 / 7040 / 7310; x 4096:
// 3610 / 3570 / 3605).
constexpr int kGroupMShort = 8, kGroupMLong = 2;
constexpr int64_t kGroupShortT = 4096;          // longest contraction of the wide groups
// Small tables with a ragged last row tile take the narrow groups at any T: the
// blocks of that tile take the checked epilogue, some 2 us longer, and one wide
// group would give one to nearly every XCD (whole step, fp32, us, groups of
// 8 / 2 at T = 64 and 256: 1000 x 2048 34.3 / 32.3 and 36.9 / 34.5 (33.5 and 36.0
// when every block checked), 1500 x 1792 37.0 / 34.3 and 39.4 / 36.7, 2000 x 3072
// 44.0 / 41.8 and, at T = 512, 50.6 / 49.1).  With whole row tiles there is no such difference
// (1024 x 2048 within 0.6 us either way), and past 12 column tiles the wide
// groups win again (1000 x 4096 38.4 / 40.8).
constexpr int kRaggedMT = 8, kRaggedNT = 12;
// An fp32 G that does not fit the 256 MB last-level cache is stored
// non-temporally: the apply pass would not find most of it there, and the
// operands keep their place (whole step, us, cached / non-temporal: 32000 x 4096
// x 2048 (524 MB) 779 / 754, 128256 x 2048 x 1024 (1.05 GB) 954 / 930).  One that
// fits is left there for the apply pass (32000 x 1024 x 1024, 131 MB: 125 / 129).
// bf16 G shows no difference at 65 MB to 1.05 GB.
constexpr int64_t kStreamGBytes = (int64_t)256 << 20;
constexpr int kRowBytes = kBM * 2;              // one token's 256 bf16 of one operand
constexpr int kOperandBytes = kBK * kRowBytes;  // one operand's slice of a step
constexpr int kStageBytes = 2 * kOperandBytes;  // dY slice, then H slice
constexpr int kRowsPerLoad = kWave * 16 / kRowBytes;            // rows one wave-wide load fills (2)
constexpr int kLoadsPerWave = kBK / kRowsPerLoad / kGemmWaves;  // per operand and step
constexpr int kWaveRows = kBM / kWavesM;        // rows of one wave's part of the tile (64)
constexpr int kWaveCols = kBN / kWavesN;        // its columns (128)
constexpr int kMT = kWaveRows / 32;             // 32 x 32 MFMA tiles per wave: kMT x kNT
constexpr int kNT = kWaveCols / 32;
constexpr int kSub = kBK / 16;                  // 16-token sub-steps of a step
constexpr int kXcds = 8;
constexpr int kBufferWord3 = 0x00020000;  // raw 32-bit data format, gfx9 family

static_assert(kBM == kBN, "both operand slices share one LDS layout");
static_assert(kBM == 256 && kBK % 16 == 0, "wave tiling assumes 256 x 256 tiles");
static_assert((kBK + 1) * EMBER_LMHEAD_MAX_LD * 2 < (int64_t)1 << 31, "32-bit load offsets");
static_assert(kGemmWaves == 8, "8 wavefronts per block");
static_assert(kStages >= 2 && kLoadsPerWave * kRowsPerLoad * kGemmWaves == kBK, "load split");
static_assert(kStages * kStageBytes <= 160 * 1024, "LDS of one CU");
static_assert(2 * kLoadsPerWave <= kMT * kNT, "at most one load behind each MFMA of a sub-step");
static_assert(kSub % 2 == 0, "a step ends on the register set it began with");
static_assert(kStages <= 5, "the step loop is written out for at most five stages");

struct Params {
    const uint16_t* dY;   // [T][ldy] bf16
    int64_t ldy;
    const uint16_t* H;    // [T][ldh] bf16
    int64_t ldh;
    int64_t T;
    int64_t V;
    int64_t D;
    void* G;              // [V][ldg], float or bf16
    int64_t ldg;
    float* rowpart;       // [NT][V]
    float* P;             // [MT][D]
    int MT;
    int NT;
    int64_t tile0;        // this launch's tiles: [tile0, tile1) of the MT * NT
    int64_t tile1;
    int64_t per_xcd;      // tiles per XCD: ceil((tile1 - tile0) / 8)
    int group_m;          // row tiles per group of the tile order
    bool stream_g;        // fp32 G: non-temporal stores
};

// Raw buffer resource of `bytes` bytes at a wave-uniform base, as the four
// words the load takes (readfirstlane keeps them in scalar registers).
__device__ __forceinline__ i32x4 rsrc(const void* base, int64_t bytes) {
    const uint64_t p = reinterpret_cast<uint64_t>(base);
    i32x4 r;
    r.x = __builtin_amdgcn_readfirstlane((int)p);
    r.y = __builtin_amdgcn_readfirstlane((int)(p >> 32) & 0xFFFF);
    r.z = __builtin_amdgcn_readfirstlane(bytes > 0x7FFFFFF0 ? 0x7FFFFFF0 : (int)bytes);
    r.w = kBufferWord3;
    return r;
}

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t h) { return __uint_as_float(h << 16); }

// Two fp32 -> bf16 (low, high half), round to nearest even: one v_cvt_pk_bf16_f32.
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    const f32x2 f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
}

// Orders a wave's LDS accesses before and after it (a wave's LDS operations
// execute in order, so only the compiler has to be held).
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Logical tile -> (row tile, column tile): groups of group_m row tiles, row
// tile fastest inside a group, so a run of consecutive tiles covers group_m
// row tiles and a window of column tiles.
__device__ __forceinline__ void tile_of(const Params& a, int64_t l, int& tm, int& tn) {
    const int64_t per_group = (int64_t)a.group_m * a.NT;
    const int64_t g = l / per_group;
    const int first = (int)(g * a.group_m);
    const int gm = min(a.MT - first, a.group_m);
    const int64_t q = l - g * per_group;
    tm = first + (int)(q % gm);
    tn = (int)(q / gm);
}

// Epilogue of one tile.  Each wavefront takes its kWaveRows x 128 part in
// strips of kStripRows rows: the strip's values are rounded to the G dtype
// (the statistics are taken from the rounded values, as the step would read
// them) and written to a wave-private LDS strip in the MFMA layout; the column
// sums are accumulated on the way.  The strip is then read back row by row,
// stored to G with 16-byte stores, and its row sums are formed by the lanes
// that share a row.  Last, the waves that share rows (or columns) add their
// partials in a fixed order through LDS.
template <typename GT>
constexpr int kStripRows = sizeof(GT) == 4 ? 16 : 32;
template <typename GT>
constexpr int kStripPitch = 128 * (int)sizeof(GT) + 16;    // bytes per strip row (padded)
template <typename GT>
constexpr int kStripBytes = kStripRows<GT> * kStripPitch<GT>;
constexpr int kRedBytes = (kWavesN + kWavesM) * kLmheadTile * 4;   // row and column partials

// kFull: the whole tile lies inside the table (no element is checked).
template <typename GT, bool kFull>
__device__ __forceinline__ void epilogue(const Params& a, int tm, int tn, f32x16 (&acc)[kMT][kNT], uint8_t* strip,
                                         uint8_t* red) {
    constexpr int kEs = (int)sizeof(GT);
    constexpr int kRows = kStripRows<GT>;
    constexpr int kPitch = kStripPitch<GT>;
    constexpr int kChunksPerRow = 128 * kEs / 16;          // 16-byte chunks per strip row
    constexpr int kLanesPerRow = kChunksPerRow < kWave ? kChunksPerRow : kWave;
    constexpr int kRowsPerPass = kWave / kLanesPerRow;
    constexpr int kEpc = 16 / kEs;                          // elements per chunk
    constexpr int kRegsPerStrip = kRows / 2;                // MFMA registers i of one strip
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int wm = wave % kWavesM, wn = wave / kWavesM;
    const int64_t m0 = (int64_t)tm * kBM + wm * kWaveRows;
    const int64_t n0 = (int64_t)tn * kBN + wn * kWaveCols;
    const int half = lane >> 5, col = lane & 31;
    float* rows_lds = reinterpret_cast<float*>(red);   // [kWavesN][256 rows]
    float* cols_lds = rows_lds + kWavesN * kBM;         // [kWavesM][256 columns]

    float cs[kNT];
#pragma unroll
    for (int nt = 0; nt < kNT; ++nt) cs[nt] = 0.0f;
    // read-back mapping: lane -> row pass offset lane / kLanesPerRow, chunk lane % kLanesPerRow
    const int rb_row = lane / kLanesPerRow, rb_chunk = lane % kLanesPerRow;

    __syncthreads();   // every wave is done with the operand stages
#pragma unroll
    for (int mt = 0; mt < kMT; ++mt) {
#pragma unroll
        for (int sp = 0; sp < 32 / kRows; ++sp) {
            // rows sp * kRows .. of the 32-row MFMA tile: registers i with
            // 8 (i / 4) + 4 half + i % 4 in that range, i.e. i in [sp kRows / 2, ...)
            const int64_t mstrip = m0 + mt * 32 + sp * kRows;
#pragma unroll
            for (int nt = 0; nt < kNT; ++nt) {
                const bool nv = n0 + nt * 32 + col < a.D;
#pragma unroll
                for (int ii = 0; ii < kRegsPerStrip; ii += 2) {
                    // registers i and i + 1 hold rows r and r + 1
                    const int i = sp * kRegsPerStrip + ii;
                    const int r = 8 * (i >> 2) + 4 * half + (i & 3) - sp * kRows;
                    float g0 = acc[mt][nt][i], g1 = acc[mt][nt][i + 1];
                    uint8_t* e = strip + r * kPitch + (nt * 32 + col) * kEs;
                    if constexpr (kEs == 2) {
                        const uint32_t h = pack_bf16x2(g0, g1);
                        *reinterpret_cast<uint16_t*>(e) = (uint16_t)h;
                        *reinterpret_cast<uint16_t*>(e + kPitch) = (uint16_t)(h >> 16);
                        g0 = bf16_bits_to_f32(h & 0xFFFFu);
                        g1 = __uint_as_float(h & 0xFFFF0000u);
                    } else {
                        *reinterpret_cast<float*>(e) = g0;
                        *reinterpret_cast<float*>(e + kPitch) = g1;
                    }
                    // rows and columns past the table hold products of other data
                    const bool v0 = kFull || (nv && mstrip + r < a.V);
                    const bool v1 = kFull || (nv && mstrip + r + 1 < a.V);
                    cs[nt] += v0 ? g0 * g0 : 0.0f;
                    cs[nt] += v1 ? g1 * g1 : 0.0f;
                }
            }
            wave_lds_order();
            // read back, store, row sums
#pragma unroll
            for (int pass = 0; pass < kRows / kRowsPerPass; ++pass) {
                const int r = pass * kRowsPerPass + rb_row;
                const int64_t m = mstrip + r;
                const int64_t n = n0 + rb_chunk * kEpc;
                const u32x4 w = *reinterpret_cast<const u32x4*>(strip + r * kPitch + rb_chunk * 16);
                float rsum = 0.0f;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if constexpr (kEs == 2) {
                        const float lo = bf16_bits_to_f32(w[q] & 0xFFFFu), hi = bf16_bits_to_f32(w[q] >> 16);
                        rsum += kFull || n + 2 * q < a.D ? lo * lo : 0.0f;
                        rsum += kFull || n + 2 * q + 1 < a.D ? hi * hi : 0.0f;
                    } else {
                        const float x = __uint_as_float(w[q]);
                        rsum += kFull || n + q < a.D ? x * x : 0.0f;
                    }
                }
                if (kFull || m < a.V) {
                    char* grow = static_cast<char*>(a.G) + (m * a.ldg + n) * kEs;
                    if (kFull || n + kEpc <= a.D) {
                        if (kEs == 4 && a.stream_g) __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(grow));
                        else *reinterpret_cast<u32x4*>(grow) = w;
                    } else {
                        for (int e = 0; e < kEpc && n + e < a.D; ++e) {
                            if constexpr (kEs == 2)
                                reinterpret_cast<uint16_t*>(grow)[e] = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
                            else
                                reinterpret_cast<uint32_t*>(grow)[e] = w[e];
                        }
                    }
                }
#pragma unroll
                for (int x = 1; x < kLanesPerRow; x <<= 1) rsum += __shfl_xor(rsum, x);
                if (rb_chunk == 0) rows_lds[wn * kBM + wm * kWaveRows + mt * 32 + sp * kRows + r] = rsum;
            }
            wave_lds_order();   // the strip is rewritten next
        }
    }
    // columns: rows of the low lane half, then of the high half
#pragma unroll
    for (int nt = 0; nt < kNT; ++nt) {
        const float other = __shfl_xor(cs[nt], 32);
        const float c2 = half == 0 ? cs[nt] + other : other + cs[nt];
        if (half == 0) cols_lds[wm * kBN + wn * kWaveCols + nt * 32 + col] = c2;
    }
    __syncthreads();
    const int x = threadIdx.x;
    if (x < kBM) {
        const int64_t m = (int64_t)tm * kBM + x;
        if (m < a.V) a.rowpart[(int64_t)tn * a.V + m] = rows_lds[x] + rows_lds[kBM + x];
        const int64_t n = (int64_t)tn * kBN + x;
        float c = cols_lds[x];
#pragma unroll
        for (int q = 1; q < kWavesM; ++q) c += cols_lds[q * kBN + x];
        if (n < a.D) a.P[(int64_t)tm * a.D + n] = c;
    }
}

// 16 bytes per lane from a buffer into LDS at lds_base + 16 lane (lanes
// outside the buffer's range write zeros).  Issued as inline assembly so that
// the compiler does not treat every later LDS read as dependent on it (it
// would wait for all such loads before any LDS read); completion is awaited
// explicitly with wait_vmcnt and a barrier before a stage is read.  M0 holds
// the LDS base (wave-uniform) for the load and is restored afterwards; one
// wait state separates its write from the load.
__device__ __forceinline__ void load_to_lds(i32x4 rs, uint32_t lds_base, int voffset) {
    const uint32_t base = __builtin_amdgcn_readfirstlane(lds_base);
    uint32_t saved;
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
                 "buffer_load_dwordx4 %2, %3, 0 offen lds\n\ts_mov_b32 m0, %0"
                 : "=&s"(saved)
                 : "s"(base), "v"(voffset), "s"(rs)
                 : "memory");
}

// Wait until at most N vector-memory loads of this wave are outstanding
// (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt and lgkmcnt at their
// "no wait" maxima).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// The step barrier: at most N of this wave's vector-memory loads outstanding
// (the next step's data has arrived), all of its LDS reads returned, then the
// block's waves meet.  Written out because __syncthreads would also wait for
// the loads that are to stay in flight.
template <int N>
__device__ __forceinline__ void wait_step() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

template <typename GT>
__global__ __launch_bounds__(kThreads) void ember_lmhead_grad(Params a) {
    // kStages stages of (dY slice, H slice) of kBK tokens each, addressed by their
    // LDS byte offset.  Each slice row (one token, 256 columns, 512 bytes) is
    // stored unpadded, its 16-byte chunks XOR-permuted by the row: chunk c of
    // token row k sits at position c ^ (4 (k % 4)).  The transpose reads of a
    // quarter-wave then cover all LDS banks once (no conflicts), and every
    // wave-wide load still fills two whole rows, as the LDS-direct load
    // requires (lane l -> base + 16 l).
    __shared__ __attribute__((aligned(1024))) uint8_t lds[kStages * kStageBytes];
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)lds;
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = tid / kWave;
    const int wm = wave % kWavesM, wn = wave / kWavesM;

    // one tile per block (a loop over tiles would keep per-lane epilogue
    // values live across the contraction); blocks of one XCD take consecutive
    // tiles of this launch's range
    const int64_t l = a.tile0 + (int64_t)(blockIdx.x % kXcds) * a.per_xcd + blockIdx.x / kXcds;
    if (l >= a.tile1) return;
    const int nk = __builtin_amdgcn_readfirstlane((int)((a.T + kBK - 1) / kBK));   // T <= 2^30
    int tm, tn;
    tile_of(a, l, tm, tn);
    const int64_t v0 = (int64_t)tm * kBM;
    const int64_t d0 = (int64_t)tn * kBN;

    // loads: wave w fills slice row pairs w, w + kGemmWaves, ...; lane l writes row
    // 2 j + l / 32 at chunk position l % 32, i.e. global chunk (l % 32) ^ 4 (row % 4)
    int off_y[kLoadsPerWave], off_h[kLoadsPerWave];
#pragma unroll
    for (int i = 0; i < kLoadsPerWave; ++i) {
        const int row = kRowsPerLoad * (wave + kGemmWaves * i) + lane / 32;
        const int chunk = (lane & 31) ^ (4 * (row & 3));
        off_y[i] = (int)((row * a.ldy + chunk * 8) * 2);
        off_h[i] = (int)((row * a.ldh + chunk * 8) * 2);
    }
    // operand resources of step kt; past the last step they cover no bytes: the
    // loads write zeros into a stage whose products are then exact zeros
    struct StepLoads {
        i32x4 ra, rb;
    };
    auto loads_of = [&](int kt) {
        const bool in = kt < nk;
        const int64_t k0 = in ? (int64_t)kt * kBK : 0;
        StepLoads sl;
        sl.ra = rsrc(a.dY + k0 * a.ldy + v0, in ? ((a.T - k0) * a.ldy - v0) * 2 : 0);
        sl.rb = rsrc(a.H + k0 * a.ldh + d0, in ? ((a.T - k0) * a.ldh - d0) * 2 : 0);
        return sl;
    };
    // load j of this wave's 2 kLoadsPerWave loads of a step
    auto issue_one = [&](const StepLoads& sl, uint32_t st, int j) {
        const int i = j >> 1;
        const uint32_t dst = st + (wave + kGemmWaves * i) * (kRowsPerLoad * kRowBytes);
        if ((j & 1) == 0) load_to_lds(sl.ra, dst, off_y[i]);
        else load_to_lds(sl.rb, dst + kOperandBytes, off_h[i]);
    };

    // transpose reads: lane l reads token row 8 (l / 32) + (l % 16) / 4 (+ 4),
    // columns 16 ((l / 16) % 2) + 4 (l % 4) + 32 t of its wave's part; with
    // the chunk permutation the byte offset of tile t within a row is
    // 16 (chunk ^ 4 (row % 4)) + 8 (l % 2), and row % 4 = (l % 16) / 4 here
    const int tr_row = 8 * (lane >> 5) + ((lane & 15) >> 2);
    const int cpart = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
    int tr_a[kMT], tr_b[kNT];
#pragma unroll
    for (int t = 0; t < kMT; ++t) {
        const int chunk = wm * (kWaveRows / 8) + t * 4 + cpart;
        tr_a[t] = tr_row * kRowBytes + (chunk ^ (4 * (tr_row & 3))) * 16 + 8 * (lane & 1);
    }
#pragma unroll
    for (int t = 0; t < kNT; ++t) {
        const int chunk = wn * (kWaveCols / 8) + t * 4 + cpart;
        tr_b[t] = tr_row * kRowBytes + (chunk ^ (4 * (tr_row & 3))) * 16 + 8 * (lane & 1) + kOperandBytes;
    }
    auto rd = [&](uint32_t p) {
        return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(uintptr_t)p);
    };
    // operand f of a 16-token sub-step, in the order the MFMAs first use them:
    // A 0, B 0 .. kNT - 1, A 1 .. kMT - 1
    auto frag = [&](uint32_t st, int kk, int f, bf16x8 (&af)[kMT], bf16x8 (&bfr)[kNT]) {
        const bool is_b = f >= 1 && f <= kNT;
        const int t = f == 0 ? 0 : is_b ? f - 1 : f - kNT;
        const uint32_t p = st + (is_b ? tr_b[t] : tr_a[t]) + kk * 16 * kRowBytes;
        const bf16x8 x = __builtin_bit_cast(bf16x8, __builtin_shufflevector(rd(p), rd(p + 4 * kRowBytes),
                                                                            0, 1, 2, 3, 4, 5, 6, 7));
        if (is_b) bfr[t] = x;
        else af[t] = x;
    };

    f32x16 acc[kMT][kNT];
#pragma unroll
    for (int mt = 0; mt < kMT; ++mt)
#pragma unroll
        for (int nt = 0; nt < kNT; ++nt)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[mt][nt][i] = 0.0f;

    // Step kt multiplies stage kt % kStages in kSub 16-token sub-steps.  While
    // the MFMAs of a sub-step run, the operands of the next one are read into
    // the other register set, one operand behind each MFMA (without the fences
    // the scheduler fetches every operand just before its MFMA and waits for it).
    // The block barrier (wait_step) sits before the last sub-step, whose
    // operands are in registers by then.  Each wave comes to it with
    //  - all of its LDS reads returned, so past the barrier no wave reads stage
    //    kt % kStages any more, and the loads of step kt + kStages may fill it;
    //  - at most (kStages - 2) 2 kLoadsPerWave of its loads outstanding.  Steps
    //    up to kt + kStages - 1 have been issued and loads complete in order,
    //    so those are of steps kt + 2 and later: past the barrier every wave's
    //    part of step kt + 1 lies in stage (kt + 1) % kStages.
    // The last sub-step's MFMAs then cover the first operand reads of step
    // kt + 1 and the issue of the loads of step kt + kStages, which have
    // kStages - 1 steps to arrive.
    bf16x8 af[2][kMT], bfr[2][kNT];
    auto step = [&](int kt, auto sc) {
        constexpr int k = decltype(sc)::value;
        const uint32_t st = lds_base + k * kStageBytes, next = lds_base + (k + 1) % kStages * kStageBytes;
        const StepLoads sl = loads_of(kt + kStages);
#pragma unroll
        for (int kk = 0; kk < kSub; ++kk) {
            const int cur = kk & 1;
            const bool last = kk == kSub - 1;
            if (last) wait_step<(kStages - 2) * 2 * kLoadsPerWave>();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < kMT * kNT; ++i) {
                const int mt = i / kNT, nt = i % kNT;
                acc[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[cur][mt], bfr[cur][nt], acc[mt][nt], 0, 0, 0);
                if (i < kMT + kNT) {
                    if (last) frag(next, 0, i, af[cur ^ 1], bfr[cur ^ 1]);
                    else frag(st, kk + 1, i, af[cur ^ 1], bfr[cur ^ 1]);
                }
                if (last && i < 2 * kLoadsPerWave) issue_one(sl, st, i);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    // the first kStages steps go out before the loop, then the first operands
    // are read once step 0 has arrived
#pragma unroll
    for (int q = 0; q < kStages; ++q) {
        const StepLoads sl = loads_of(q);
#pragma unroll
        for (int j = 0; j < 2 * kLoadsPerWave; ++j) issue_one(sl, lds_base + q * kStageBytes, j);
    }
    wait_step<(kStages - 1) * 2 * kLoadsPerWave>();
#pragma unroll
    for (int f = 0; f < kMT + kNT; ++f) frag(lds_base, 0, f, af[0], bfr[0]);
    // whole rounds of kStages steps (one loop exit keeps the accumulators in
    // place); a step past the last one multiplies the zeros its loads wrote
    for (int kt = 0; kt < nk; kt += kStages) {
        step(kt, std::integral_constant<int, 0>{});
        step(kt + 1, std::integral_constant<int, 1>{});
        if constexpr (kStages > 2) step(kt + 2, std::integral_constant<int, 2>{});
        if constexpr (kStages > 3) step(kt + 3, std::integral_constant<int, 3>{});
        if constexpr (kStages > 4) step(kt + 4, std::integral_constant<int, 4>{});
    }
    wait_vmcnt<0>();   // the zero-filling loads past the end, before the LDS is reused
    // epilogue scratch: the waves' strips, then the block's partial sums
    constexpr int kStrip = kStripBytes<GT>;
    static_assert(kGemmWaves * kStrip + kRedBytes <= kStages * kStageBytes, "epilogue scratch fits the stages");
    uint8_t* const strip = lds + wave * kStrip;
    uint8_t* const red = lds + kGemmWaves * kStrip;
    if (v0 + kBM <= a.V && d0 + kBN <= a.D) epilogue<GT, true>(a, tm, tn, acc, strip, red);
    else epilogue<GT, false>(a, tm, tn, acc, strip, red);
}

} // namespace

LmheadPlan lmhead_plan(int64_t V, int64_t D) {
    LmheadPlan p;
    p.MT = (int)((V + kLmheadTile - 1) / kLmheadTile);
    p.NT = (int)((D + kLmheadTile - 1) / kLmheadTile);
    return p;
}

hipError_t launch_lmhead_grad(const LmheadArgs& x, hipStream_t s) {
    const LmheadPlan pl = lmhead_plan(x.V, x.D);
    Params p;
    p.dY = static_cast<const uint16_t*>(x.dY);
    p.ldy = x.ldy;
    p.H = static_cast<const uint16_t*>(x.H);
    p.ldh = x.ldh;
    p.T = x.T;
    p.V = x.V;
    p.D = x.D;
    p.G = x.G;
    p.ldg = x.ldg;
    p.rowpart = x.rowpart;
    p.P = x.P;
    p.MT = pl.MT;
    p.NT = pl.NT;
    const bool few_ragged = x.V % kBM != 0 && pl.MT <= kRaggedMT && pl.NT <= kRaggedNT;
    p.group_m = x.T <= kGroupShortT && !few_ragged ? kGroupMShort : kGroupMLong;
    p.stream_g = x.g_dtype == 0 && x.V * x.D * 4 > kStreamGBytes;
    const int64_t total = (int64_t)pl.MT * pl.NT;
    const int64_t per_launch = kMaxGridBlocks;   // a multiple of kXcds
    for (int64_t t0 = 0; t0 < total; t0 += per_launch) {
        p.tile0 = t0;
        p.tile1 = t0 + per_launch < total ? t0 + per_launch : total;
        p.per_xcd = (p.tile1 - t0 + kXcds - 1) / kXcds;
        const dim3 grid((unsigned)(p.per_xcd * kXcds));
        if (x.g_dtype == 0)
            ember_lmhead_grad<float><<<grid, kThreads, 0, s>>>(p);
        else
            ember_lmhead_grad<uint16_t><<<grid, kThreads, 0, s>>>(p);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipGetLastError();
}

} // namespace ember

// Internal declarations shared by the host entry points and the gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "apb.h"

namespace apb {

constexpr int kWave = 64;        // CDNA wavefront width
constexpr int kRowTile = 16;     // weight rows one wave keeps in registers in the popcount GEMM
constexpr int kChunkWords = 8;   // K is walked in chunks of 8 words = 256 weights (one LDS code table each)
constexpr int kChunkK = 32 * kChunkWords;
constexpr int kMaxWavesPerBlock = 8;
// ent_val holds residual * 2^895: finite for every float, and large enough that the columns-in-lanes kernel's
// table codes (code * 2^-1009, see apb_sparse.hip) give products far from underflow.
constexpr int kEntValScaleLog2 = 895;
constexpr int kEntBlockWords = 24;   // one block of 8 residual entries: 8 key words + 8 float64

struct LayerDev {
    void* blocks[4] = {};        // the allocations that everything below lies in: what N and K give the size of, the
                                 // CSR, the digit steps, the tile runs
    int N = 0, K = 0, Kw = 0;    // Kw = ceil(K/32)
    int Np = 0;                  // launch slots: N rounded up to a multiple of kRowTile * waves
    int waves = 2;               // waves per workgroup of the forward kernel (2, 4 or 8)
    int nchunks = 0;             // ceil(Kw / kChunkWords)
    long long nnz = 0;
    float alpha = 0.f;
    uint32_t* sign = nullptr;    // [N][Kw]   canonical sign words
    uint32_t* signT = nullptr;   // [Kw2][Np] sign words, slot-major: word j of launch slot i (padding slots and
                                 //           the extra word row of an odd Kw are zero; Kw2 as for signC)
    uint32_t* signC = nullptr;   // [Kw2][N]  sign words, word-major in the layer's own row order;
                                 //           Kw2 = Kw rounded up to even, the extra word row is zero
    int32_t* perm = nullptr;     // [Np]      row index served by launch slot i, -1 for padding
    int32_t* row_ptr = nullptr;  // [N+1]
    int32_t* col_idx = nullptr;  // [nnz]
    float* val = nullptr;        // [nnz]
    double* vald = nullptr;      // [nnz]     the same residuals widened to float64 (exact), for the kernel
    int32_t* rowsum = nullptr;   // [N]
    int32_t* chunk_ptr = nullptr;  // [nchunks+1][Np]  first residual of slot i with column >= 256*c
    double* slot_valsum = nullptr; // [Np]             sum of the residuals of slot i (float64)
    // Residuals regrouped for the columns-in-lanes kernel (layers that it may serve only, null otherwise): one flat run per (tile of kRowTile slots, chunk of
    // 256 columns), sorted by row inside the run, in blocks of 8 entries.
    int32_t* seg_ptr = nullptr;    // [Np/kRowTile][nchunks+1]  first block of (tile, chunk)
    uint32_t* ent = nullptr;       // [blocks][24]  8 keys: 2 * row_in_tile | (col - 256*chunk) << 8, then
                                   //               8 float64: residual * 2^kEntValScaleLog2 (0 for padding)
    // What the matrix-core forward kernel (apb_rows.hip) reads; rows_steps == 0 when not built (K beyond its table).
    // Rows go in tiles of 16; a tile is two quads of four pairs of rows, in this order: for r = 0, 1 (first quad), 2, 3
    // (second) the rows (r, 8 + r), then (4 + r, 12 + r).
    int rows_ksteps = 0;           // K in steps of 128, rounded up
    int rows_unit_log2 = 0;        // the residuals are whole multiples of 2^rows_unit_log2 ...
    int rows_windows = 1;          // ... and are cut into this many windows of kWindowBits bits
    long long rows_steps = 0;
    uint32_t* rows_sign = nullptr; // [tiles][ksteps][64]     sign words in the order the binary part's lanes take them:
                                   //           lane (i, g): word 4 * step + g of row 16 * tile + i, the bit pairs of every
                                   //           nibble swapped for odd g; zero outside the matrix
    int32_t* rows_first = nullptr; // [tiles]                 first digit step of a tile
    uint8_t* rows_count = nullptr; // [tiles][2 quads][windows]  digit steps of each pair of a quad (see digit_steps_of)
    uint8_t* rows_step = nullptr;  // [steps][kStepBytes]     see kStepBytes
    double* rows_valsum = nullptr; // [16 * tiles]            sum of the residuals of the row (float64, CSR order)
};

// A digit step of the matrix-core forward kernel: up to 128 values of k at which one of the two rows of a pair has a
// residual.  Lane block g (of 4) holds values 32 * g .. 32 * g + 31 of the step:
//   16 + 8 bytes for each of 48 lanes (12 digit rows x 4 blocks: row 6 * half + digit, block g at 12 * g + row): 32 FP6
//   numbers, the digits of the residuals at these k (0 where the row has none); first all the 16s, then all the 8s;
//   one word for each of 64 lanes (i, g): row of value 32 * g + i | row of value 32 * g + 16 + i << 16, where row is the
//   byte offset 8 * k in the code table (layers of K <= kRowsByteK) or k.
// A digit d is the FP6 (E2M3) number d / 8 at an even k and d / 4 at an odd one.  kStepPad more steps follow the last one.
constexpr int kStepA8 = 48 * 16;
constexpr int kStepRows = 48 * 24;
constexpr int kStepBytes = 48 * 24 + 64 * 4;
// Steps each pair of a quad takes when its longest list has `entries`: what the kernel has straight code for (1, 2, 3,
// 4 and 6), or whole rounds of its four registers sets.
__host__ __device__ inline int digit_steps_of(int entries) {
    const int s = (entries + 127) / 128;
    return s <= 1 ? 1 : s <= 4 ? s : s <= 6 ? 6 : (s + 3) / 4 * 4;
}
constexpr int kStepPad = 8;
constexpr int kRowsByteK = 8192;             // (and 3 * 16 * 33 * kRowsByteK < 2^24: see rows_item)
constexpr int kWindowBits = 30;              // six base-32 digits, -16 .. 16
constexpr int kRowsMaxK = 18432;             // the code table of one column group (8 bytes per value of k): 144 KB of LDS

void set_last_hip_error(hipError_t e);

// Shapes of an activation matrix the entry points refuse (APB_ERR_SHAPE).
inline bool bad_shape_acts(int K, int M) {
    if (K <= 0 || M <= 0) return true;
    if ((long long)K * 3 >= (1LL << 31)) return true;
    if ((long long)M + kWave >= (1LL << 31)) return true;
    return false;
}

// The 2-bit activation quantizer (Sec. IV "1/2"): p = clamp(rint(x / s), 0, 3) with one float
// multiply by the precomputed 1/s, ties to even; NaN -> 0.
__device__ __forceinline__ uint32_t code2(float x, float inv_step) {
    return (uint32_t)(int)fminf(3.0f, fmaxf(0.0f, rintf(x * inv_step)));
}
// The same code as the two low bits of the result (the bits above are not zero): clamping first and rounding
// second gives the same p (rounding is monotone and 0, 3 are integers), and adding 2^23 to a float in [0, 3]
// IS the rounding to the nearest integer, ties to even, with p left in the low mantissa bits -- four vector
// instructions instead of five, and no conversion.
__device__ __forceinline__ uint32_t code2_low_bits(float x, float inv_step) {
    return __float_as_uint(fminf(3.0f, fmaxf(0.0f, x * inv_step)) + 8388608.0f);
}
// Shift a word right by one and put bit 0 of `bits` on top: after 32 calls the first bit sits at position 0.
__device__ __forceinline__ uint32_t push_bit(uint32_t word, uint32_t bits) { return __builtin_amdgcn_alignbit(bits, word, 1); }

#define APB_HIP(expr)                                 \
    do {                                              \
        hipError_t e_ = (expr);                       \
        if (e_ != hipSuccess) {                       \
            ::apb::set_last_hip_error(e_);            \
            return APB_ERR_HIP;                       \
        }                                             \
    } while (0)

template <typename T>
int dev_alloc(T** p, size_t count) {
    *p = nullptr;
    if (count == 0) count = 1;                       // keep pointers non-null for empty CSR
    hipError_t e = hipMalloc(reinterpret_cast<void**>(p), count * sizeof(T));
    if (e == hipErrorOutOfMemory) return APB_ERR_NOMEM;
    if (e != hipSuccess) {
        set_last_hip_error(e);
        return APB_ERR_HIP;
    }
    return APB_OK;
}

// Several arrays in one allocation: `add` each, then `alloc` sets all the pointers.  (An allocation and its release cost
// about as much as one of the kernels that compress a layer.)
struct DeviceArrays {
    struct Piece {
        void** p;
        size_t at;
    };
    std::vector<Piece> pieces;
    size_t bytes = 0;

    template <typename T>
    void add(T** p, size_t count) {
        pieces.push_back({reinterpret_cast<void**>(p), bytes});
        bytes += (count * sizeof(T) + 255) / 256 * 256;
    }
    int alloc(void** block) {
        uint8_t* base = nullptr;
        const int rc = dev_alloc(&base, bytes);
        if (rc != APB_OK) return rc;
        *block = base;
        for (const Piece& q : pieces) *q.p = base + q.at;
        return APB_OK;
    }
};

// ---- kernel launchers (each returns an apb_status) ------------------------------------------

// compress
int launch_inlier_abs_sum(const float* W, long long count, float delta, double* part_sum, long long* part_cnt,
                          int parts, hipStream_t s);
int launch_sign_pack_count(const float* W, int N, int K, int Kw, float delta, uint32_t* sign, int32_t* counts,
                           int32_t* rowsum, hipStream_t s);
int launch_scatter_csr(const float* W, int N, int K, float delta, float alpha, const int32_t* row_ptr,
                       int32_t* col_idx, float* val, double* vald, hipStream_t s);
int launch_slot_major_signs(const uint32_t* sign, const int32_t* perm, int Np, int Kw, int rows_out,
                            uint32_t* signT, hipStream_t s);
int launch_slot_tables(const int32_t* perm, const int32_t* row_ptr, const int32_t* col_idx, const double* row_valsum, int Np,
                       int nchunks, int32_t* chunk_ptr, double* slot_valsum, hipStream_t s);
int launch_row_valsum(const int32_t* row_ptr, const float* val, int N, int rows, double* valsum, hipStream_t s);
// The operands of the matrix-core forward kernel: the sign words in its lanes' order, and the digit steps, from the sign
// words and the CSR.  `found` is scratch of digit_scratch_words(N) words.  Waits for the stream.
size_t digit_scratch_words(int N);
int build_rows_layer(LayerDev& d, int32_t* found, hipStream_t s);

// activations.  colsum == nullptr: the planes only (for a consumer that adds the code sums up from the words itself)
int launch_quantize(const float* X, int K, int M, int bits, float inv_step, uint32_t* planes, int32_t* colsum,
                    hipStream_t s);
int launch_zero_words(uint32_t* p, size_t count, hipStream_t s);

// forward
// the popcount formulation on the vector ALU (Y, or D alone when D != nullptr)
int launch_forward_popcount(const LayerDev& L, const uint32_t* planes, const int32_t* colsum, int M, int bits,
                            float step, float* Y, int32_t* D, hipStream_t s);
// the forward kernel: binary part on the matrix cores, residual part and epilogue, one launch.
// conv == nullptr: `planes` is the packed K x M matrix; otherwise a packed feature map of conv->C channels
// (L.K = 9 * C, C a multiple of 32) of images of H x W pixels, read through an implicit im2col (3 x 3,
// padding 1, the given stride), and M = B * Ho * Wo output pixels.
struct ConvShape {
    int C, H, W;
    int stride, Ho, Wo;            // Ho = (H - 1) / stride + 1, Wo likewise
    int Pp_in;                     // B * H * W rounded up to a multiple of 64: columns of the packed input map
};
int launch_forward(const LayerDev& L, const uint32_t* planes, const int32_t* colsum, int M, int bits, float step,
                   const ConvShape* conv, float* Y, hipStream_t s);
const char* forward_kernel_name(const LayerDev& L, int M, int bits);
// the same with the next layer's quantizer applied to scale[n] * Y + shift[n] (scale, shift nullable) and
// the codes packed into `packed_out` (K = L.N, same M), fully overwritten
int launch_forward_requant(const LayerDev& L, const uint32_t* planes, const int32_t* colsum, int M, int bits, float step,
                           const ConvShape* conv, const float* scale, const float* shift, int bits_out,
                           float inv_step_out, uint32_t* packed_out, hipStream_t s);

// true while K * max_weight * max_code < 2^24: the float accumulators of the matrix instruction then hold
// every partial sum exactly (launchers return APB_ERR_SHAPE otherwise)
bool mfma_sum_exact(int K, int max_weight, int max_code);

// the matrix-core forward kernel (apb_rows.hip): same Y as launch_forward.  colsum == nullptr: the kernel adds the
// code sums of its columns up from the packed words (always so for convolutions).
bool forward_rows_applies(const LayerDev& L, int bits);
const char* forward_rows_kernel_name(const LayerDev& L, int M, int bits);
int launch_forward_rows(const LayerDev& L, const uint32_t* planes, const int32_t* colsum, int M, int bits, float step,
                        const ConvShape* conv, float* Y, hipStream_t s);
// ending in the next layer's quantizer (see launch_forward_requant)
int launch_forward_rows_requant(const LayerDev& L, const uint32_t* planes, const int32_t* colsum, int M, int bits, float step,
                                const ConvShape* conv, const float* scale, const float* shift, int bits_out,
                                float inv_step_out, uint32_t* packed_out, hipStream_t s);
// the one-kernel step with the columns in the lanes (apb_sparse.hip), where it is possible
bool forward_float_applies(const LayerDev& L, int M, int bits);
int launch_forward_float(const LayerDev& L, const float* X, int M, int bits, float step, float* Y, hipStream_t s);

// Which of the two forward kernels a call takes: the columns-in-lanes kernel (apb_sparse.hip) for layers the other has no
// operands for, and where it is the faster one.
bool takes_columns_kernel(const LayerDev& L, int M, int bits, bool packed_out);
// from the float matrix X (K x M), quantize + forward in one kernel: same Y, bit for bit, as launch_quantize +
// launch_forward_best; only where step_is_one_kernel says so (APB_ERR_SHAPE otherwise)
bool step_is_one_kernel(const LayerDev& L, int M, int bits);
int launch_step_one_kernel(const LayerDev& L, const float* X, int M, int bits, float step, float* Y, hipStream_t s);
// launch_quantize + launch_forward_best through the scratch buffer planes / colsum (the step of layers that do
// not run as one kernel); what `colsum` holds afterwards is unspecified
int launch_quantize_then_forward(const LayerDev& L, const float* X, int M, int bits, float step, uint32_t* planes,
                                 int32_t* colsum, float* Y, hipStream_t s);
// apb_forward's choice between the two forward kernels for a plain K x M matrix and a float output
int launch_forward_best(const LayerDev& L, const uint32_t* planes, const int32_t* colsum, int M, int bits, float step,
                        float* Y, hipStream_t s);

// binary part alone on the matrix cores: the integer part D
int launch_binary_mfma(const LayerDev& L, const uint32_t* planes, const int32_t* colsum, int M, int bits,
                       int32_t* out, hipStream_t s);

// 2/2 routine: quantize + pack 2-bit weights (canonical [2][N][Kw] and word-major [2][Kw2][N], Kw2 =
// Kw rounded up to even with a zero pad row), and the product itself (D22 when Y == nullptr)
int launch_w2_pack(const float* W, int N, int K, float inv_step, uint32_t* planes, uint32_t* planesC, hipStream_t s);
int launch_gemm_2_2(const uint32_t* wplanesC, int N, int Kw, const uint32_t* planes, const int32_t* colsum, int M,
                    double scale, int32_t* D, float* Y, hipStream_t s);

}  // namespace apb

struct apb_layer {
    apb::LayerDev d;
};

struct apb_w2 {
    int N = 0, K = 0, Kw = 0;
    float step_w = 0.f;
    uint32_t* planes = nullptr;    // [2][N][Kw]   canonical bit-planes of the level indices
    uint32_t* planesC = nullptr;   // [2][Kw2][N]  the same, word-major, for the matrix-core kernel
};

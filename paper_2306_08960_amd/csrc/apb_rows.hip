// The forward kernel (Sec. III Eqs. 12-13):
//     Y[n,m] = s * ( alpha * D[n,m] + R[n,m] ),   R[n,m] = sum_{j in row n} val_j * c[col_j, m]
// with BOTH parts on the matrix cores, exactly.
//
// Residual part.  Over the residuals of a row, R is a sum of float32 values times small integers: a sum of
// integers once the values are written in units of a power of two small enough for all of them (the
// layer's unit).  Those integers are cut into signed base-32 digits, -16 .. 16, which the FP6 format (E2M3) holds
// exactly, and the digits are multiplied by the FP4 codes with v_mfma_scale_f32_16x16x128_f8f6f4: every product
// and every partial sum is an integer far below 2^24, so the float accumulators are exact, and putting the digit
// sums together gives R without any rounding (one rounding follows in float64, one to float).  Six digits span 30
// bits; a float has 24, so that covers layers whose residuals' last bits and largest bits lie up to 2^29 apart
// (residuals are differences of a weight and alpha, whose last bits are those of the smaller of the two); other
// layers take several windows of six digits.
//
// The matrix instruction multiplies 16 rows by 16 columns over 128 values of k.  The 16 rows are the 6 + 6 digits
// of TWO rows of the layer (and four idle ones); the 128 values of k are not consecutive ones but those at which
// either of the two rows has a residual: with 3 % residuals half of the operand is non-zero, where 16 plain rows
// would leave 97 % of it empty.  The activation operand is gathered accordingly: the codes of all of K for the
// workgroup's columns lie in LDS as a table [k][16 columns] of 4-bit codes, and ds_read_b64_tr_b4, for which every
// lane names the row it reads, fetches 64 arbitrary rows of the table and hands every lane its column of them --
// the gather IS the operand load.  128 residuals (of two rows, 16 columns each) thus cost two LDS reads and one
// matrix instruction of 16 cycles, where the vector ALU needs 16 x 128 / 64 = 32 mask + multiply-add pairs of 9.
// The rows of each half wave of a gather should fall into different banks (k mod 32 all different), so the order
// of the k of a list -- free -- is chosen when the layer is built.
//
// Binary part.  The same table serves as the activation operand, the weight operand is expanded from the sign bits.
//
// A workgroup builds the table for its columns (16 per column group) once, and its waves then work through items of NT
// tiles of 16 rows x NCW column groups with no further barriers.  Convolutions gather the table from the packed feature
// map, and the one-kernel step quantizes X into it.  A packed output leaves as whole words (two tiles) or half words.
//
// Measured against a kernel with one row and 16 columns to a lane, which summed the residuals one after another in
// float64 (forward alone, both parts): 512 x 4608, 12544 columns, 3 % residuals 86 -> 45 us; 4096 x 4096, 256 columns
// 21.4 -> 14.2; 256 x 2304 1-bit, 8192 columns 17.7 -> 10.6; 128 x 1152, 50176 columns, 1 % in skewed rows 30 -> 23.4.
// What bounds the largest of these (counters: profiles/forward_C5b_pmc_counters.txt): no unit -- of the compute units in use
// the vector ALU is busy 44 % of the time, LDS and L1 43 % each (a seventh of the LDS cycles bank conflicts), the matrix
// cores 28 % -- but that its tables, 152 KB for 64 columns of K = 4608, leave one workgroup of 8 waves to a compute unit
// and 196 workgroups for 256 of them.  Layers of few residuals per row and many columns are bound by the epilogue and by
// digit steps that are mostly empty: see columns_kernel_residuals (apb_rows_shape.h).
#include <algorithm>
#include <atomic>
#include <cmath>
#include <type_traits>
#include <utility>

#include "apb_fp4_expand.h"
#include "apb_internal.h"
#include "apb_rows_shape.h"

namespace apb {

namespace {

constexpr int kMaxDevices = 64;
constexpr int kBufferFlags = 0x00020000;                        // fourth word of a raw buffer descriptor: 32-bit data, no swizzle
constexpr int kOutOfRange = (int)0x80000000u;                   // a lane offset beyond every descriptor: the load returns zero

typedef float v4f __attribute__((ext_vector_type(4)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) v2i lds_v2i;
typedef __attribute__((address_space(3))) v4u lds_v4u;
typedef __attribute__((address_space(3))) int32_t lds_i32;
typedef __attribute__((address_space(3))) double lds_f64;

enum Source { kPlanes = 0, kConv = 1, kFloat = 2 };             // where the codes come from

struct RowsParams {
    double alpha;                                                // alpha * step
    double step;
    int N, K, Kw, Mp, M;
    int ksteps;                                                  // K in steps of 128, rounded up
    int tiles;                                                   // of 16 rows, an even number
    int windows;
    double unit;                                                 // step * value of one unit of the lowest window's digits
    int groups, groups_log2;                                     // column groups of 16 per workgroup (1, 2 or 4)
    int chunk, parts;                                            // tiles per workgroup, workgroups per column tile
    int row_shift;                                               // a digit step's table rows are k << (3 - row_shift)
    // packed output: the activation buffer of the next layer (its K = this layer's N)
    int out_bits, out_Kw;
    float out_inv_step;
    float in_inv_step;                                           // kFloat
    // kConv: see ConvShape
    int conv_Cw, conv_H, conv_W, conv_Ho, conv_Wo, conv_stride, conv_Mp;
    float conv_inv_Cw;
};

struct RowsArgs {
    const void* __restrict__ src;                                // planes, packed feature map, or X
    const int32_t* __restrict__ colsum;                          // kPlanes: code sums, or null (added up here)
    const uint32_t* __restrict__ sign;
    const uint8_t* __restrict__ steps;
    const int32_t* __restrict__ first;
    const uint8_t* __restrict__ count;
    const double* __restrict__ valsum;
    const int32_t* __restrict__ rowsum;
    const float* __restrict__ scale;
    const float* __restrict__ shift;
    void* __restrict__ out;
};

// Tap of word row j of a patch matrix (exact for j * Cw < 2^22), the pixel shift of a tap, and the taps of a window
// that fall inside the image.
__device__ __forceinline__ int tap_of_row(int j, const RowsParams& p) { return (int)(((float)j + 0.5f) * p.conv_inv_Cw); }
__device__ __forceinline__ int tap_shift(int tap, int W) {
    const int t3 = (tap * 11) >> 5;                              // tap / 3 for tap < 12
    return (t3 - 1) * W + (tap - 3 * t3 - 1);
}
__device__ __forceinline__ uint32_t conv_pixel(int m, const RowsParams& p, int& pin) {
    const int xo = m % p.conv_Wo, rest = m / p.conv_Wo;
    const int yo = rest % p.conv_Ho, img = rest / p.conv_Ho;
    const int x = p.conv_stride * xo, y = p.conv_stride * yo;
    pin = m < p.M ? (img * p.conv_H + y) * p.conv_W + x : 0;
    uint32_t vm = 0;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        const int yy = y + t / 3 - 1, xx = x + t % 3 - 1;
        if (m < p.M && yy >= 0 && yy < p.conv_H && xx >= 0 && xx < p.conv_W) vm |= 1u << t;
    }
    return vm;
}

// ---- the code table: [column group][32 * 4 * ksteps values of k][16 codes of 4 bits] from LDS address 0.
// Expanded words arrive as in apb_fp4_expand.h (nibble t of dword d <-> bit d + 4t), 16 bytes for one column and 32
// values of k: lane (i, g) leaves those of column i, word 4s + g at byte 16 * lane of the block of step s, and the
// transposing read turns 16 columns x 16 nibbles around: lane i of block g then holds 16 columns of one value of k.
// All in place and within one wave, whose LDS operations are executed in order.  (Odd blocks take the two halves in
// the other order, here and wherever rows are read by consecutive k: the 32 lanes of a half wave then fall into 32
// different bank pairs.)
__device__ __forceinline__ int row_of_lane(int lane, int q) {    // value of k (within a step) of lane, read q
    const int i = lane & 15, g = lane >> 4, qq = q ^ (g & 1);
    return 32 * g + 2 * qq + (i >> 3) + 4 * (i & 7);
}
template <int NB>
__device__ __forceinline__ void transpose_blocks(const uint32_t (&block)[NB], int lane) {
    const int odd = (lane >> 4) & 1;
    const uint32_t from = (uint32_t)(lane * 16 + 8 * odd), to0 = (uint32_t)row_of_lane(lane, 0) * 8, to1 = (uint32_t)row_of_lane(lane, 1) * 8;
    v2i r[NB][2];
    asm volatile("" ::: "memory");
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        r[u][0] = __builtin_amdgcn_ds_read_tr4_b64_v2i32((lds_v2i*)(uintptr_t)(block[u] + from));
        r[u][1] = __builtin_amdgcn_ds_read_tr4_b64_v2i32((lds_v2i*)(uintptr_t)(block[u] + (from ^ 8u)));
    }
    asm volatile("" ::: "memory");
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        *(lds_v2i*)(uintptr_t)(block[u] + to0) = r[u][0];
        *(lds_v2i*)(uintptr_t)(block[u] + to1) = r[u][1];
    }
    asm volatile("" ::: "memory");
}

// A code of an even k is stored as the FP4 number code (0, 1, 2, 3), of an odd k as code / 2 (0, .5, 1, 1.5: the nibble is
// the code itself).  The sign operand can then take the bits of odd k where they stand in a nibble (the number 1
// instead of .5): five instructions a word instead of seven, once per 16 rows and 128 values of k, where the table is
// written once per workgroup.  The digits of odd k are doubled in turn.
template <int BITS>
__device__ __forceinline__ void stage_word(uint32_t at, uint32_t w0, uint32_t w1) {
    v4u f;
    if (BITS == 1) {
        f[0] = (w0 << 1) & (kNib << 1);
        f[1] = (w0 >> 1) & kNib;
        f[2] = (w0 >> 1) & (kNib << 1);
        f[3] = (w0 >> 3) & kNib;
    } else {
#pragma unroll
        for (int d = 0; d < 4; d += 2) {                         // 0b0010, 0b0100, 0b0101 for codes 1, 2, 3
            const uint32_t x0 = (w0 >> d) & kNib, x1 = (w1 >> d) & kNib, both = x0 & x1;
            f[d] = (x1 << 2) | ((x0 ^ both) << 1) | both;
        }
#pragma unroll
        for (int d = 1; d < 4; d += 2) f[d] = ((w1 >> (d - 1)) & (kNib << 1)) | ((w0 >> d) & kNib);
    }
    *(lds_v4u*)(uintptr_t)at = f;
}
__device__ __forceinline__ v8i sign_operand(uint32_t w) {
    const uint32_t h = w >> 2;
    return v8i{(int)(w & kNib), (int)(w & (kNib << 1)), (int)(h & kNib), (int)(h & (kNib << 1)), 0, 0, 0, 0};
}

template <int BITS, int SRC>
__device__ __forceinline__ void build_table(const RowsArgs& a, const RowsParams& p, int m0, uint32_t cs_at, bool want_sums,
                                            int lane, int wave, int waves) {
    const int plane = p.ksteps * 1024;
    if constexpr (SRC == kFloat) {
        // A unit of work is 64 words: 32 rows of X at 64 columns (or 64 rows at 32, 128 at 16), so that a load of one
        // row is 64 * groups consecutive bytes; the arithmetic is that of apb_quantize_acts.  A lane block of 16
        // then has one word of the 16 columns of one column group, which it turns around by itself.
        const float* X = static_cast<const float*>(a.src);
        const int i = lane & 15, block = lane >> 4, odd = block & 1;
        const int cg = block & (p.groups - 1), sub = block >> p.groups_log2, per_unit = 4 >> p.groups_log2;
        const int col = 16 * cg + i, m = m0 + col;
        const bool col_ok = m < p.M;
        const unsigned mc = (unsigned)min(m, p.M - 1);
        const uint32_t row0 = 8u * (2 * odd + (i >> 3) + 4 * (i & 7)), row1 = row0 ^ 16u;
        int sum = 0;
        for (int j = wave * per_unit + sub; j < 4 * p.ksteps; j += waves * per_unit) {
            const int k0 = 32 * j;
            float xv[32];
#pragma unroll
            for (int t = 0; t < 32; ++t)
                xv[t] = __builtin_nontemporal_load(X + (size_t)min(k0 + t, p.K - 1) * p.M + mc);
            uint32_t w0 = 0, w1 = 0;
#pragma unroll
            for (int t = 0; t < 32; ++t) {
                if (BITS == 1) {
                    w0 |= (xv[t] >= 0.0f ? 1u : 0u) << t;
                } else {
                    const uint32_t c = code2_low_bits(xv[t], p.in_inv_step);
                    w0 = push_bit(w0, c);
                    w1 = push_bit(w1, c >> 1);
                }
            }
            const int valid = p.K - k0;
            const uint32_t keep = !col_ok || valid <= 0 ? 0u : (valid >= 32 ? 0xffffffffu : ((1u << valid) - 1u));
            w0 &= keep;
            w1 &= keep;
            sum += __builtin_popcount(w0) + 2 * __builtin_popcount(w1);
            const uint32_t at = (uint32_t)(cg * plane + j * 256);
            stage_word<BITS>(at + 16 * i, w0, w1);
            asm volatile("" ::: "memory");
            const v2i r0 = __builtin_amdgcn_ds_read_tr4_b64_v2i32((lds_v2i*)(uintptr_t)(at + 16 * i + 8 * odd));
            const v2i r1 = __builtin_amdgcn_ds_read_tr4_b64_v2i32((lds_v2i*)(uintptr_t)(at + 16 * i + 8 * (odd ^ 1)));
            asm volatile("" ::: "memory");
            *(lds_v2i*)(uintptr_t)(at + row0) = r0;
            *(lds_v2i*)(uintptr_t)(at + row1) = r1;
            asm volatile("" ::: "memory");
        }
        if (sum) __hip_atomic_fetch_add((lds_i32*)(uintptr_t)(cs_at + 4 * col), sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        return;
    } else {
        const uint32_t* planes = static_cast<const uint32_t*>(a.src);
        const int i = lane & 15, g = lane >> 4;
        const int across = min(waves, p.groups), along = waves / across;
        const size_t plane_stride = SRC == kConv ? (size_t)p.conv_Cw * p.conv_Mp : (size_t)p.Kw * p.Mp;
        for (int cg = wave & (across - 1); cg < p.groups; cg += across) {
            const int m = m0 + 16 * cg + i;
            int pin = 0;
            const uint32_t vm = SRC == kConv ? conv_pixel(m, p, pin) : 0u;
            const unsigned mc = (unsigned)min(m, p.Mp - 1);
            int sum = 0;
            // This wave's blocks: steps first, first + along, ...  A batch of them at a time, so that neither the loads
            // nor the LDS operations wait for one another; the next batch's words are on their way meanwhile.  (Past the
            // last block: the last one again -- same words, same place.)
            constexpr int kBatch = 4;
            const int first = wave / across, mine = (p.ksteps - first + along - 1) / along;
            if (mine <= 0) continue;
            uint32_t w0[kBatch], w1[kBatch];
            auto load = [&](int t, uint32_t& x0, uint32_t& x1) {
                const int j = 4 * (first + min(t, mine - 1) * along) + g;
                if constexpr (SRC == kConv) {
                    const int tap = tap_of_row(j, p), cw = j - tap * p.conv_Cw;
                    const int off = ((vm >> tap) & 1u) ? (cw * p.conv_Mp + pin + tap_shift(tap, p.conv_W)) * 4 : kOutOfRange;
                    const __amdgpu_buffer_rsrc_t r0 = __builtin_amdgcn_make_buffer_rsrc(
                        const_cast<uint32_t*>(planes), 0, p.conv_Cw * p.conv_Mp * 4, kBufferFlags);
                    x0 = __builtin_amdgcn_raw_buffer_load_b32(r0, off, 0, 0);
                    x1 = 0u;
                    if (BITS == 2) {
                        const __amdgpu_buffer_rsrc_t r1 = __builtin_amdgcn_make_buffer_rsrc(
                            const_cast<uint32_t*>(planes + plane_stride), 0, p.conv_Cw * p.conv_Mp * 4, kBufferFlags);
                        x1 = __builtin_amdgcn_raw_buffer_load_b32(r1, off, 0, 0);
                    }
                } else {
                    const uint32_t* row = planes + (size_t)min(j, p.Kw - 1) * p.Mp + mc;
                    x0 = row[0];
                    x1 = BITS == 2 ? row[plane_stride] : 0u;
                }
            };
#pragma unroll
            for (int u = 0; u < kBatch; ++u) load(u, w0[u], w1[u]);
            for (int t0 = 0; t0 < mine; t0 += kBatch) {
                uint32_t x0[kBatch], x1[kBatch], block[kBatch];
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    x0[u] = w0[u];
                    x1[u] = w1[u];
                    load(t0 + kBatch + u, w0[u], w1[u]);
                }
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    const int s = first + min(t0 + u, mine - 1) * along, j = 4 * s + g;
                    if (SRC == kPlanes && j >= p.Kw) x0[u] = x1[u] = 0u;
                    if (want_sums && t0 + u < mine) sum += __builtin_popcount(x0[u]) + 2 * __builtin_popcount(x1[u]);
                    block[u] = (uint32_t)(cg * plane + s * 1024);
                    stage_word<BITS>(block[u] + lane * 16, x0[u], x1[u]);
                }
                transpose_blocks<kBatch>(block, lane);
            }
            if (want_sums && sum)
                __hip_atomic_fetch_add((lds_i32*)(uintptr_t)(cs_at + 4 * (16 * cg + i)), sum, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
}

// One digit step as it waits in registers: the FP6 operand of this lane (24 bytes) and the table rows it gathers
// (two of 16 bits each: k << 3, or k in layers of many k).
struct Slot {
    v4u a;
    v2u b;
    uint32_t k;
};

__device__ __forceinline__ v2i read_rows(uint32_t at) { return __builtin_amdgcn_ds_read_tr4_b64_v2i32((lds_v2i*)(uintptr_t)at); }
__device__ __forceinline__ v8i operand(const v2i (&b)[2]) { return v8i{b[0].x, b[0].y, b[1].x, b[1].y, 0, 0, 0, 0}; }

// Uniform values read through the constant address space: scalar loads, outside the vector memory counter.
typedef __attribute__((address_space(4))) const int32_t const_i32;
typedef __attribute__((address_space(4))) const uint32_t const_u32;
typedef __attribute__((address_space(4))) const uint16_t const_u16;
typedef __attribute__((address_space(4))) const uint8_t const_u8;

// f(0), f(1), ... f(N - 1) with the numbers known at compile time from the start: what a wave keeps in registers across
// its items is indexed by them, and must not be an array in memory when the compiler first looks at it.
template <typename F, int... Q>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Q...>) {
    (f(std::integral_constant<int, Q>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_impl(static_cast<F&&>(f), std::make_integer_sequence<int, N>{});
}

// What a wave has in flight: four digit steps, and the sign words of four steps of the binary part.
constexpr int kRing = 4, kWords = 4;
struct Stream {
    const uint8_t* steps;                                        // from the item's first tile on
    const uint32_t* sign;
    int fa_off, fb_off, fk_off;                                  // this lane's parts of a digit step
};
__device__ __forceinline__ void issue(const Stream& st, int& so, Slot& s) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(st.steps), 0, 0x7fffffff, kBufferFlags);
    s.a = __builtin_amdgcn_raw_buffer_load_b128(rs, st.fa_off, so, 0);
    s.b = __builtin_amdgcn_raw_buffer_load_b64(rs, st.fb_off, so, 0);
    s.k = __builtin_amdgcn_raw_buffer_load_b32(rs, st.fk_off, so, 0);
    so += kStepBytes;
}
// word of step `step` of the item's `tile`th tile
__device__ __forceinline__ uint32_t sign_word(const Stream& st, int tile, int step, int ksteps) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(st.sign), 0, 0x7fffffff, kBufferFlags);
    return (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, (int)(threadIdx.x & (kWave - 1)) * 4, (tile * ksteps + step) * 256, 0);
}

// Where things lie in LDS behind the tables (and behind one step that the binary part reads past its last).
struct Places {
    int plane;                                                   // bytes of one column group's table
    uint32_t cs, ocs;                                            // code sums of the columns; those of a packed output
    uint32_t affine, sums, rowsum;                               // of the workgroup's rows: scale, shift; valsum; rowsum
};

// One item: NT tiles of 16 rows (from `tile` on, the workgroup's `local` and the wave's `at` th) x 16 * NCW columns from
// column group cg0 of the table.
// The sums of the three digits of a half are put together in 32-bit integers (up to 3 * 16 * 1057 per residual), after
// the first two in a float, which is exact while 3 * 16 * 33 per residual stays below 2^24: 10592 residuals of a row,
// more than K without GENERAL.
// GENERAL: several windows, which are walked, or K beyond kRowsByteK.
template <int BITS, bool REQ, int NT, int NCW, bool GENERAL>
__device__ __forceinline__ void rows_item(const RowsArgs& a, const RowsParams& p, const Places& l, int tile, int local, int m0,
                                          int cg0, int lane) {
    const int i = lane & 15, g = lane >> 4;
    const uint32_t table = (uint32_t)(cg0 * l.plane);
    const int mc = m0 + 16 * cg0 + i;                            // this lane's column in its first column group
    const const_u8* cnt_at = (const_u8*)a.count + (size_t)2 * tile * p.windows;
    const uint32_t cnt = GENERAL ? 0u : NT == 2 ? *(const_u32*)cnt_at : *(const_u16*)cnt_at;
    const int row_shift = GENERAL ? p.row_shift : 0;

    // digit operand of lane (i, g): digit rows i = 4 * (row half) + digit, the fourth of every four idle
    const int frag = g * 12 + (i >> 2) * 3 + (i & 3);
    const Stream st = {a.steps + (size_t)((const_i32*)a.first)[tile] * kStepBytes, a.sign + (size_t)tile * p.ksteps * 64,
                       (i & 3) == 3 ? kOutOfRange : frag * 16, (i & 3) == 3 ? kOutOfRange : kStepA8 + frag * 8, kStepRows + lane * 4};
    // The first words and digit steps leave at once.
    Slot ring[kRing];
    uint32_t words[kWords][NT];
    int so = 0;
    static_for<kWords>([&](auto Q) {
        static_for<NT>([&](auto T) {
            words[decltype(Q)::value][decltype(T)::value] =
                sign_word(st, decltype(T)::value, min((int)decltype(Q)::value, p.ksteps - 1), p.ksteps);
        });
    });
    static_for<kRing>([&](auto Q) {                              // (in this order: the steps wait for slot after slot)
        issue(st, so, ring[decltype(Q)::value]);
        __builtin_amdgcn_sched_barrier(0);
    });

    // ---- binary part: P = sum_k bit * code for 16 * NT rows x 16 * NCW columns.  Two operand sets used in turn, or (many
    // column groups) one, whose parts are fetched for the next step as soon as the matrix instructions have taken them.
    constexpr int kSets = NCW == 4 ? 1 : 2;
    v4f D[NT][NCW];
    v2i b[kSets][NCW][2];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int cg = 0; cg < NCW; ++cg) D[t][cg] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    {
        const uint32_t brow0 = table + (uint32_t)row_of_lane(lane, 0) * 8, brow1 = table + (uint32_t)row_of_lane(lane, 1) * 8;
        auto fetch = [&](uint32_t off, int set, int cg) {
            b[set][cg][0] = read_rows(brow0 + cg * l.plane + off);
            b[set][cg][1] = read_rows(brow1 + cg * l.plane + off);
        };
#pragma unroll
        for (int cg = 0; cg < NCW; ++cg) fetch(0, 0, cg);
        auto one_step = [&](int s0, auto Q) {
            constexpr int q = decltype(Q)::value;
            v8i fa[NT];
            const uint32_t next = (uint32_t)s0 * 1024 + (q + 1) * 1024;
            if (kSets == 2)
#pragma unroll
                for (int cg = 0; cg < NCW; ++cg) fetch(next, (q + 1) & 1, cg);
            static_for<NT>([&](auto T) {
                constexpr int t = decltype(T)::value;
                uint32_t& word = words[q][t];
                fa[t] = sign_operand(word);
                word = sign_word(st, t, min(s0 + q + kWords, p.ksteps - 1), p.ksteps);
            });
#pragma unroll
            for (int cg = 0; cg < NCW; ++cg) {
#pragma unroll
                for (int t = 0; t < NT; ++t)                     // (.5 code * 2: integers)
                    D[t][cg] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(fa[t], operand(b[kSets == 2 ? q & 1 : 0][cg]), D[t][cg], 4, 4, 0,
                                                                                0x80808080, 0, kScaleOne);
                if (kSets == 1) fetch(next, 0, cg);
            }
            __builtin_amdgcn_sched_barrier(0);                   // (steps stay apart: the ring has most of the registers)
        };
        int s0 = 0;
        for (; s0 + kWords <= p.ksteps; s0 += kWords) static_for<kWords>([&](auto Q) { one_step(s0, Q); });
        static_for<kWords - 1>([&](auto Q) {
            if (s0 + decltype(Q)::value < p.ksteps) one_step(s0, Q);
        });
    }

    // ---- residual part and epilogue, a quad of four pairs (eight rows) at a time: rows (r, 8 + r), (4 + r, 12 + r) for
    // two values of r.  A pair's product leaves digits 0..2 of its first row in lane block 0, 3..5 in block 1, the
    // second row's in blocks 2 and 3; after an exchange between the two pairs of an r, block g holds both halves of
    // row 4g + r: the row whose D it has as element r.
    uint32_t wb[NT][NCW];                                        // packed output: bits of plane 0 | plane 1 << 16
    bool col_ok[NCW];
    float cs[NCW];                                               // (code sums, like all sums of codes here, stay below 2^24)
    double racc[2][NCW];
#pragma unroll
    for (int cg = 0; cg < NCW; ++cg) {
#pragma unroll
        for (int t = 0; t < NT; ++t) wb[t][cg] = 0u;
        col_ok[cg] = mc + 16 * cg < p.M;
        cs[cg] = (float)*(lds_i32*)(uintptr_t)(l.cs + 4 * (16 * (cg0 + cg) + i));
        racc[0][cg] = racc[1][cg] = 0.0;
    }
    auto gather = [&](uint32_t rows, int set, int cg) {
        const uint32_t at0 = table + ((rows & 0xffffu) << row_shift), at1 = table + ((rows >> 16) << row_shift);
        b[set][cg][0] = read_rows(at0 + cg * l.plane);
        b[set][cg][1] = read_rows(at1 + cg * l.plane);
    };
#pragma unroll
    for (int cg = 0; cg < NCW; ++cg) gather(ring[0].k, 0, cg);
    const int quads = 2 * NT * p.windows;
    double wunit = p.unit;                                       // of the current window
    int w = 0;
    for (int quad = 0, round = 0; quad < quads; ++quad) {
        const int S = GENERAL ? (int)cnt_at[quad] : (int)((cnt >> (8 * quad)) & 255u);
        int t[4][NCW];
        auto run = [&](auto steps_of_pair) {
            constexpr int kS = decltype(steps_of_pair)::value;
            v4f c[NCW];
            auto step = [&](auto Q, auto fresh) {
                constexpr int q = decltype(Q)::value;
                Slot& sl = ring[q];
                const uint32_t next = ring[(q + 1) & 3].k;
                if (kSets == 2)
#pragma unroll
                    for (int cg = 0; cg < NCW; ++cg) gather(next, (q + 1) & 1, cg);
                const v8i fa = v8i{(int)sl.a[0], (int)sl.a[1], (int)sl.a[2], (int)sl.a[3], (int)sl.b[0], (int)sl.b[1], 0, 0};
#pragma unroll
                for (int cg = 0; cg < NCW; ++cg) {               // (digit * code / 8 * 8: integers)
                    c[cg] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
                        fa, operand(b[kSets == 2 ? q & 1 : 0][cg]), decltype(fresh)::value ? v4f{0.0f, 0.0f, 0.0f, 0.0f} : c[cg], 2, 4, 0,
                        0x82828282, 0, kScaleOne);
                    if (kSets == 1) gather(next, 0, cg);
                }
                issue(st, so, sl);
                __builtin_amdgcn_sched_barrier(0);
            };
            static_for<4>([&](auto Pr) {
                constexpr int pr = decltype(Pr)::value;
                if constexpr (kS > 0) {
                    static_for<kS>([&](auto E) {
                        constexpr int e = decltype(E)::value;
                        step(std::integral_constant<int, (pr * kS + e) & 3>{}, std::integral_constant<bool, e == 0>{});
                    });
                } else {                                         // whole rounds of the ring
#pragma unroll
                    for (int cg = 0; cg < NCW; ++cg) c[cg] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
                    for (int e = 0; e < S; e += 4) static_for<4>([&](auto Q) { step(Q, std::false_type{}); });
                }
#pragma unroll
                for (int cg = 0; cg < NCW; ++cg)
                    t[pr][cg] = GENERAL ? (int)c[cg][0] + ((int)c[cg][1] << 5) + ((int)c[cg][2] << 10)
                                        : (int)fmaf(c[cg][1], 32.0f, c[cg][0]) + ((int)c[cg][2] << 10);
            });
        };
        switch (S) {                                             // (kept in step with digit_steps_of)
            case 1: run(std::integral_constant<int, 1>{}); break;
            case 2: run(std::integral_constant<int, 2>{}); break;
            case 3: run(std::integral_constant<int, 3>{}); break;
            case 4: run(std::integral_constant<int, 4>{}); break;
            case 6: run(std::integral_constant<int, 6>{}); break;
            default: run(std::integral_constant<int, 0>{}); break;
        }
        const bool last_window = !GENERAL || w + 1 == p.windows;
        float y[2][NCW];
#pragma unroll
        for (int rr = 0; rr < 2; ++rr) {
            const int row = 16 * (round >> 2) + 4 * g + (round & 3) + rr;        // of the item
            v2i aff = {0, 0};
            double vs = 0.0;
            int rsum = 0;
            const uint32_t meta = (uint32_t)(16 * local + row);
            if (REQ) aff = *(lds_v2i*)(uintptr_t)(l.affine + 8 * meta);
            if (BITS == 1) {
                vs = *(lds_f64*)(uintptr_t)(l.sums + 8 * meta);
                rsum = *(lds_i32*)(uintptr_t)(l.rowsum + 4 * meta);
            }
#pragma unroll
            for (int cg = 0; cg < NCW; ++cg) {
                const v2u x = __builtin_amdgcn_permlane16_swap(t[2 * rr][cg], t[2 * rr + 1][cg], false, false);
                const double R = fma((double)(int)x[1], 32768.0, (double)(int)x[0]);
                // z = step * (alpha * D + R)   (all windows but the last only add to R)
                const float P = D[0][cg][rr];
                const double d = BITS == 1 ? (double)(4 * (int)P - rsum - 2 * (int)cs[cg]) : (double)fmaf(2.0f, P, -cs[cg]);
                const double r = GENERAL ? fma(R, wunit, racc[rr][cg]) : R * p.unit;
                double z = BITS == 1 ? fma(p.alpha, d, fma(2.0, r, -vs)) : fma(p.alpha, d, r);
                if (REQ) {
                    z = fma((double)__int_as_float(aff.x), z, (double)__int_as_float(aff.y));
                    y[rr][cg] = (float)z;
                    uint32_t code = p.out_bits == 1 ? (y[rr][cg] >= 0.0f ? 1u : 0u) : code2(y[rr][cg], p.out_inv_step);
                    if (!col_ok[cg] || 16 * tile + row >= p.N || !last_window) code = 0;
                    code = (code | (code << 15)) & 0x10001u;     // plane 0 at bit 0, plane 1 at bit 16
#pragma unroll
                    for (int tt = 0; tt < NT; ++tt) wb[tt][cg] |= NT == 1 || (round >> 2) == tt ? code << (row & 15) : 0u;
                } else {
                    y[rr][cg] = (float)z;
                }
                if (GENERAL) racc[rr][cg] = last_window ? 0.0 : r;
            }
        }
        if (GENERAL) {
            w = last_window ? 0 : w + 1;
            wunit = last_window ? p.unit : wunit * 0x1p30;       // 2^kWindowBits
        }
        // The products wait in registers for their rows' turn, a queue of which the outputs take the places.
        if (last_window) {
#pragma unroll
            for (int cg = 0; cg < NCW; ++cg) {
                const v4f d0 = D[0][cg], d1 = D[NT - 1][cg];
                if (NT == 2) {
                    D[0][cg] = v4f{d0[2], d0[3], d1[0], d1[1]};
                    D[NT - 1][cg] = v4f{d1[2], d1[3], y[0][cg], y[1][cg]};
                } else {
                    D[0][cg] = v4f{d0[2], d0[3], y[0][cg], y[1][cg]};
                }
            }
            round += 2;
        }
    }
    if (!REQ) {
        // Stored here, all at once: a store between the digit steps would be waited for together with the loads
        // behind it (one counter, in order).
        float* out = static_cast<float*>(a.out) + (size_t)(16 * tile + 4 * g) * p.M + mc;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int cg = 0; cg < NCW; ++cg)
                    if (col_ok[cg] && 16 * tile + 16 * t + 4 * g + r < p.N) out[(size_t)(16 * t + r) * p.M + 16 * cg] = D[t][cg][r];
    } else {
        // The 16 bits of a column's half word are spread over the four lane blocks: OR them together.
        uint16_t* halves = static_cast<uint16_t*>(a.out);
        const size_t plane1 = (size_t)p.out_Kw * p.Mp * 2;
#pragma unroll
        for (int cg = 0; cg < NCW; ++cg) {
            const int m = mc + 16 * cg;
            int sum = 0;
            uint32_t x[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                x[t] = wb[t][cg];
                x[t] |= (uint32_t)__shfl_xor((int)x[t], 16);
                x[t] |= (uint32_t)__shfl_xor((int)x[t], 32);
                sum += __builtin_popcount(x[t] & 0xffffu) + 2 * __builtin_popcount(x[t] >> 16);
            }
            if (NT == 2) {                                       // a whole word
                uint32_t* words = static_cast<uint32_t*>(a.out) + (size_t)(tile >> 1) * p.Mp + m;
                if (m < p.Mp && g == 0) words[0] = (x[0] & 0xffffu) | (x[NT - 1] << 16);
                if (m < p.Mp && g == 1 && p.out_bits == 2) words[(size_t)p.out_Kw * p.Mp] = (x[0] >> 16) | (x[NT - 1] & 0xffff0000u);
            } else {
                const size_t to = ((size_t)(tile >> 1) * p.Mp + m) * 2 + (tile & 1);
                if (m < p.Mp && g == 0) halves[to] = (uint16_t)x[0];
                if (m < p.Mp && g == 1 && p.out_bits == 2) halves[to + plane1] = (uint16_t)(x[0] >> 16);
            }
            if (g == 0)
                __hip_atomic_fetch_add((lds_i32*)(uintptr_t)(l.ocs + 4 * (16 * (cg0 + cg) + i)), sum, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
}

// Four waves per SIMD at up to 128 registers; the widest items have the registers of two.
#define APB_ROWS_ATTR __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(NCW == 4 ? 2 : 4, 4)))
template <int BITS, int SRC, bool REQ, int NT, int NCW, bool GENERAL>
__global__ APB_ROWS_ATTR void k_forward_rows(const RowsArgs a, const RowsParams p) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int waves = blockDim.x / kWave;
    // Workgroups are dealt round-robin to the 8 XCDs; give each XCD a contiguous range of tasks so that the
    // workgroups that share a column tile share an L2.
    const int groups = (int)gridDim.x;
    const int task = (groups & 7) == 0 ? (int)(blockIdx.x & 7) * (groups >> 3) + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
    Places l;
    l.plane = p.ksteps * 1024;
    l.cs = (uint32_t)(l.plane << p.groups_log2) + 1024u;
    l.ocs = l.cs + (64u << p.groups_log2);
    l.affine = l.ocs + (64u << p.groups_log2);
    l.sums = l.affine + (REQ ? 8u * 16u * p.chunk : 0u);
    l.rowsum = l.sums + 8u * 16u * p.chunk;
    const bool want_sums = SRC != kPlanes || a.colsum == nullptr;
    const int parts_log2 = p.groups_log2 - (NCW == 4 ? 2 : NCW == 2 ? 1 : 0);    // shares of a tile's columns: NCW groups each
    const int part = wave & ((1 << parts_log2) - 1), runner = wave >> parts_log2, runners = max(1, waves >> parts_log2);

    const int tile_m = task / p.parts, t_begin = (task - tile_m * p.parts) * p.chunk, t_end = min(p.tiles, t_begin + p.chunk);
    const int m0 = tile_m * (16 << p.groups_log2);

    const int items = (t_end - t_begin) / NT;
    for (int t = threadIdx.x; t < (32 << p.groups_log2); t += blockDim.x)
        *(lds_i32*)(uintptr_t)(l.cs + 4 * t) = want_sums || t >= (16 << p.groups_log2) ? 0 : a.colsum[min(m0 + t, p.Mp - 1)];
    if (REQ || BITS == 1)
        for (int t = threadIdx.x; t < 16 * (t_end - t_begin); t += blockDim.x) {
            const int n = min(16 * t_begin + t, p.N - 1);
            if (REQ) {
                const v2i x = {a.scale ? __float_as_int(a.scale[n]) : 0x3f800000, a.scale ? __float_as_int(a.shift[n]) : 0};
                *(lds_v2i*)(uintptr_t)(l.affine + 8 * t) = x;
            }
            if (BITS == 1) {
                *(lds_f64*)(uintptr_t)(l.sums + 8 * t) = p.step * a.valsum[n];
                *(lds_i32*)(uintptr_t)(l.rowsum + 4 * t) = a.rowsum[n];
            }
        }
    __syncthreads();
    build_table<BITS, SRC>(a, p, m0, l.cs, want_sums, lane, wave, waves);
    __syncthreads();
    for (int item = runner; item < items; item += runners)
        rows_item<BITS, REQ, NT, NCW, GENERAL>(a, p, l, t_begin + item * NT, item * NT, m0, part * NCW, lane);
    if (REQ) {
        __syncthreads();
        uint32_t* sums = static_cast<uint32_t*>(a.out) + (size_t)p.out_bits * p.out_Kw * p.Mp;
        for (int t = threadIdx.x; t < (16 << p.groups_log2); t += blockDim.x) {
            const uint32_t tot = (uint32_t)*(lds_i32*)(uintptr_t)(l.ocs + 4 * t);
            if (m0 + t >= p.Mp) continue;
            if (p.parts == 1) sums[m0 + t] = tot;
            else if (tot) __hip_atomic_fetch_add(sums + m0 + t, tot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// The kernels address their LDS from address 0: true while they have no static LDS in front of the dynamic array.
// Checked once per kernel and process, from the kernel's own attributes; a launch of more LDS than a kernel gets
// without asking is asked for once per device and kernel.
template <auto Kernel>
int launch_kernel(const RowsArgs& a, const RowsParams& p, long long wgs, int waves, int lds, hipStream_t s) {
    static std::atomic<int> state{0};
    static std::atomic<bool> asked[kMaxDevices];
    const void* f = reinterpret_cast<const void*>(Kernel);
    int st = state.load(std::memory_order_acquire);
    if (st == 0) {
        hipFuncAttributes attr;
        APB_HIP(hipFuncGetAttributes(&attr, f));
        st = attr.sharedSizeBytes == 0 ? 1 : -1;
        state.store(st, std::memory_order_release);
    }
    if (st != 1 || lds > kMaxLdsBytes) return APB_ERR_SHAPE;
    if (lds > 64 * 1024) {
        int dev = 0;
        APB_HIP(hipGetDevice(&dev));
        if (dev < 0 || dev >= kMaxDevices) return APB_ERR_SHAPE;
        if (!asked[dev].load(std::memory_order_acquire)) {
            APB_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLdsBytes));
            asked[dev].store(true, std::memory_order_release);
        }
    }
    hipLaunchKernelGGL(Kernel, dim3((unsigned)wgs), dim3(kWave * waves), lds, s, a, p);
    APB_HIP(hipGetLastError());
    return APB_OK;
}

bool is_general(const LayerDev& L) { return L.rows_windows > 1 || L.K > kRowsByteK; }

template <int BITS, int SRC, bool REQ>
int launch_shape(const LayerDev& L, const RowsArgs& a, const RowsParams& p, const RowsShape& h, long long wgs, int lds, hipStream_t s) {
    const bool general = is_general(L);
    if (general && h.nt == 1 && h.ncw == 1) return launch_kernel<k_forward_rows<BITS, SRC, REQ, 1, 1, true>>(a, p, wgs, h.waves, lds, s);
    if (general) return APB_ERR_SHAPE;
    if (h.nt == 1 && h.ncw == 1) return launch_kernel<k_forward_rows<BITS, SRC, REQ, 1, 1, false>>(a, p, wgs, h.waves, lds, s);
    if (h.nt == 1 && h.ncw == 4) return launch_kernel<k_forward_rows<BITS, SRC, REQ, 1, 4, false>>(a, p, wgs, h.waves, lds, s);
    if (h.nt == 2 && h.ncw == 2) return launch_kernel<k_forward_rows<BITS, SRC, REQ, 2, 2, false>>(a, p, wgs, h.waves, lds, s);
    return APB_ERR_SHAPE;
}

int log2_of(int v) {
    int l = 0;
    while ((1 << l) < v) ++l;
    return l;
}

struct Output {
    const float* scale;
    const float* shift;
    int bits;                                                    // 0: float Y
    float inv_step;
    void* out;
};

int launch_any(const LayerDev& L, const void* src, Source kind, const int32_t* colsum, int M, int bits, float step,
               const ConvShape* conv, const Output& o, hipStream_t s) {
    if (!forward_rows_applies(L, bits) || (kind == kFloat && !rows_from_float(L.N, L.K, M))) return APB_ERR_SHAPE;
    const long long Mp = (long long)kWave * (((long long)M + kWave - 1) / kWave);
    if (Mp * 8 >= (1LL << 31)) return APB_ERR_SHAPE;
    const bool req = o.bits != 0;
    const RowsProblem q{L.N, M, L.rows_ksteps, bits, is_general(L), req, kind == kFloat};
    const RowsShape h = pick_rows_shape(q);
    RowsParams p{};
    p.alpha = (double)L.alpha * (double)step;
    p.step = (double)step;
    p.unit = std::ldexp((double)step, L.rows_unit_log2);
    p.N = L.N;
    p.K = L.K;
    p.Kw = L.Kw;
    p.Mp = (int)Mp;
    p.M = M;
    p.ksteps = L.rows_ksteps;
    p.tiles = rows_tiles(L.N);
    p.windows = L.rows_windows;
    p.groups = h.groups;
    p.groups_log2 = log2_of(h.groups);
    const long long cols = req ? Mp : M;                         // (a packed output covers the padding columns as well)
    p.chunk = std::min(h.chunk, p.tiles);
    p.parts = (p.tiles + p.chunk - 1) / p.chunk;
    const long long wgs = (cols + 16 * h.groups - 1) / (16 * h.groups) * p.parts;
    const long long lds = rows_lds_bytes(q, h.groups, p.chunk);
    if (wgs <= 0 || wgs > 0x7fffffffLL || lds > kMaxLdsBytes) return APB_ERR_SHAPE;
    p.row_shift = L.K > kRowsByteK ? 3 : 0;
    p.out_bits = o.bits;
    p.out_Kw = (L.N + 31) / 32;
    p.out_inv_step = o.inv_step;
    p.in_inv_step = 1.0f / step;
    p.conv_Ho = p.conv_Wo = p.conv_stride = 1;
    if (conv) {
        p.conv_Cw = conv->C / 32;
        p.conv_H = conv->H;
        p.conv_W = conv->W;
        p.conv_Ho = conv->Ho;
        p.conv_Wo = conv->Wo;
        p.conv_stride = conv->stride;
        p.conv_Mp = conv->Pp_in;
        p.conv_inv_Cw = 1.0f / (float)p.conv_Cw;
    }
    if (req && p.parts > 1) {
        const int rc = launch_zero_words(static_cast<uint32_t*>(o.out) + (size_t)o.bits * p.out_Kw * Mp, (size_t)Mp, s);
        if (rc != APB_OK) return rc;
    }
    const RowsArgs a{src, colsum, L.rows_sign, L.rows_step, L.rows_first, L.rows_count, L.rows_valsum, L.rowsum,
                     o.scale, o.shift, o.out};
    if (kind == kFloat) {
        if (req) return APB_ERR_SHAPE;
        return bits == 1 ? launch_shape<1, kFloat, false>(L, a, p, h, wgs, (int)lds, s) : launch_shape<2, kFloat, false>(L, a, p, h, wgs, (int)lds, s);
    }
    if (kind == kConv) {
        if (req) return bits == 1 ? launch_shape<1, kConv, true>(L, a, p, h, wgs, (int)lds, s) : launch_shape<2, kConv, true>(L, a, p, h, wgs, (int)lds, s);
        return bits == 1 ? launch_shape<1, kConv, false>(L, a, p, h, wgs, (int)lds, s) : launch_shape<2, kConv, false>(L, a, p, h, wgs, (int)lds, s);
    }
    if (req) return bits == 1 ? launch_shape<1, kPlanes, true>(L, a, p, h, wgs, (int)lds, s) : launch_shape<2, kPlanes, true>(L, a, p, h, wgs, (int)lds, s);
    return bits == 1 ? launch_shape<1, kPlanes, false>(L, a, p, h, wgs, (int)lds, s) : launch_shape<2, kPlanes, false>(L, a, p, h, wgs, (int)lds, s);
}

}  // namespace

bool forward_rows_applies(const LayerDev& L, int bits) {
    return L.rows_steps > 0 && mfma_sum_exact(L.K, 1, bits == 1 ? 1 : 3);
}

bool step_is_one_kernel(const LayerDev& L, int M, int bits) {
    return takes_columns_kernel(L, M, bits, false) ? forward_float_applies(L, M, bits) : rows_from_float(L.N, L.K, M);
}

int launch_step_one_kernel(const LayerDev& L, const float* X, int M, int bits, float step, float* Y, hipStream_t s) {
    if (!step_is_one_kernel(L, M, bits)) return APB_ERR_SHAPE;
    if (takes_columns_kernel(L, M, bits, false)) return launch_forward_float(L, X, M, bits, step, Y, s);
    return launch_any(L, X, kFloat, nullptr, M, bits, step, nullptr, Output{nullptr, nullptr, 0, 0.0f, Y}, s);
}

const char* forward_rows_kernel_name(const LayerDev& L, int M, int bits) {
    const RowsShape h = pick_rows_shape({L.N, M, L.rows_ksteps, bits, is_general(L), false, false});
#define APB_NAMES(B) \
    {"k_forward_rows<" #B ", 0, false, 1, 1, true>", "k_forward_rows<" #B ", 0, false, 1, 1, false>", \
     "k_forward_rows<" #B ", 0, false, 1, 4, false>", "k_forward_rows<" #B ", 0, false, 2, 2, false>"}
    static const char* names[2][4] = {APB_NAMES(1), APB_NAMES(2)};
#undef APB_NAMES
    return names[bits - 1][is_general(L) ? 0 : h.nt == 2 ? 3 : h.ncw == 4 ? 2 : 1];
}

int launch_forward_rows(const LayerDev& L, const uint32_t* planes, const int32_t* colsum, int M, int bits, float step,
                        const ConvShape* conv, float* Y, hipStream_t s) {
    return launch_any(L, planes, conv ? kConv : kPlanes, colsum, M, bits, step, conv,
                      Output{nullptr, nullptr, 0, 0.0f, Y}, s);
}

int launch_forward_rows_requant(const LayerDev& L, const uint32_t* planes, const int32_t* colsum, int M, int bits, float step,
                                const ConvShape* conv, const float* scale, const float* shift, int bits_out,
                                float inv_step_out, uint32_t* packed_out, hipStream_t s) {
    return launch_any(L, planes, conv ? kConv : kPlanes, colsum, M, bits, step, conv,
                      Output{scale, shift, bits_out, inv_step_out, packed_out}, s);
}

bool takes_columns_kernel(const LayerDev& L, int M, int bits, bool packed_out) {
    if (!forward_rows_applies(L, bits)) return true;
    return L.ent && columns_kernel_better(L.N, L.K, L.nnz, M, packed_out);
}

int launch_forward_best(const LayerDev& L, const uint32_t* planes, const int32_t* colsum, int M, int bits, float step,
                        float* Y, hipStream_t s) {
    if (!takes_columns_kernel(L, M, bits, false)) return launch_forward_rows(L, planes, colsum, M, bits, step, nullptr, Y, s);
    return launch_forward(L, planes, colsum, M, bits, step, nullptr, Y, s);
}

int launch_quantize_then_forward(const LayerDev& L, const float* X, int M, int bits, float step, uint32_t* planes,
                                 int32_t* colsum, float* Y, hipStream_t s) {
    // This kernel reads every word of its columns anyway and adds their code sums up itself: the quantize kernel then
    // writes the planes only -- no sums in LDS, and where it splits K no fill launch and no atomics.
    const bool rows = !takes_columns_kernel(L, M, bits, false);
    const int rc = launch_quantize(X, L.K, M, bits, 1.0f / step, planes, rows ? nullptr : colsum, s);
    if (rc != APB_OK) return rc;
    return launch_forward_best(L, planes, rows ? nullptr : colsum, M, bits, step, Y, s);
}

}  // namespace apb

// What the matrix-core forward kernel (apb_rows.hip) reads, built from the compressed layer on the GPU: the residuals
// as digit steps (see LayerDev and kStepBytes) and the sign words in the order of its lanes.
//
// Bounded by latency, not by traffic (512 x 4608 with 3 % residuals: 0.3 MB of residuals in, 0.9 MB of steps out), and by
// two short waits of the host, which allocates the steps once it knows their number.  One wave builds a pair of rows: the
// columns of both as bitmaps in LDS.  A word of a bitmap is 32 consecutive k, so that "sorted by k mod 32" is a walk of
// lane c over bit c of all words, the place of a residual in the CSR is a prefix count of bits, and no step needs a sort.
// The 24 bytes of an operand lane are put together in registers and stored whole.  (Built by a loop on the host
// before, bit by bit: apb_compress of that layer with its export took 10.1 ms, now 0.31.)
#include <climits>
#include <vector>

#include "apb_internal.h"

namespace apb {

namespace {

constexpr int kBlock = 256;
constexpr int kMaxWindows = 10;              // bits 2^-149 .. 2^127 and a sign, 30 at a time
constexpr int kCodeWords = 4 * 2 * 32 * 2;   // a digit step's codes as they wait in LDS

// Windows of a layer whose residuals have bits 2^lo .. 2^hi (no residual: lo = INT_MAX).
__host__ __device__ inline int windows_of(int lo, int hi) { return lo == INT_MAX ? 1 : (hi - lo + 2 + kWindowBits - 1) / kWindowBits; }

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

// Lowest and highest bit over all residuals; range[0], range[1] start at INT_MAX, INT_MIN.  (Zeros, infinities and NaN have none.)
__global__ __launch_bounds__(kBlock) void k_residual_range(const float* __restrict__ val, long long nnz, int32_t* __restrict__ range) {
    int lo = INT_MAX, hi = INT_MIN;
    for (long long e = (long long)blockIdx.x * kBlock + threadIdx.x; e < nnz; e += (long long)gridDim.x * kBlock) {
        const uint32_t bits = __float_as_uint(val[e]), ex = (bits >> 23) & 255u;
        uint32_t m = bits & 0x7fffffu;
        if (ex == 255u || (ex == 0u && m == 0u)) continue;
        int unit = -149;                                         // exponent of the mantissa's last bit
        if (ex != 0u) {
            m |= 0x800000u;
            unit = (int)ex - 150;
        }
        lo = min(lo, unit + __builtin_ctz(m));
        hi = max(hi, unit + 31 - __builtin_clz(m));
    }
    for (int off = kWave / 2; off > 0; off >>= 1) {
        lo = min(lo, __shfl_xor(lo, off, kWave));
        hi = max(hi, __shfl_xor(hi, off, kWave));
    }
    if (lane_id() == 0 && lo != INT_MAX) {
        atomicMin(range, lo);
        atomicMax(range + 1, hi);
    }
}

// Sum of the residuals of each row in float64, in CSR order (a wave loads 64 at a time; rows past N: 0).
__global__ __launch_bounds__(kBlock) void k_row_valsum(const int32_t* __restrict__ row_ptr, const float* __restrict__ val, int N, int rows,
                                                       double* __restrict__ valsum) {
    const int n = blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave, lane = lane_id();
    if (n >= rows) return;
    double sum = 0.0;
    if (n < N)
        for (int e = row_ptr[n], end = row_ptr[n + 1]; e < end; e += kWave) {
            const int left = min(kWave, end - e);
            const float v = lane < left ? val[e + lane] : 0.0f;
            for (int t = 0; t < left; ++t) sum += (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), t));
        }
    if (lane == 0) valsum[n] = sum;
}

// (It also sets the range of k_residual_range, which follows it, to nothing.)
__global__ __launch_bounds__(kBlock) void k_rows_sign(const uint32_t* __restrict__ sign, int N, int Kw, int ksteps, long long words,
                                                      uint32_t* __restrict__ out, int32_t* __restrict__ range) {
    const long long t = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (t >= words) return;
    if (t == 0) {
        range[0] = INT_MAX;
        range[1] = INT_MIN;
    }
    const int lane = (int)(t & 63), g = lane >> 4;
    const long long block = t >> 6;
    const long long n = block / ksteps * 16 + (lane & 15);
    const int j = 4 * (int)(block % ksteps) + g;
    uint32_t w = n < N && j < Kw ? sign[(size_t)n * Kw + j] : 0u;
    if (g & 1) w = ((w & 0x33333333u) << 2) | ((w >> 2) & 0x33333333u);
    out[t] = w;
}

// The number that the six digits of residual v stand for in window w (of `windows`; the last is the highest): v in units of
// 2^lo is the sum of these times 2^(kWindowBits * w), each rounded to the nearest so that the rest fits below.
__device__ __forceinline__ int window_value(float v, int lo, int windows, int w) {
    if (!(fabsf(v) <= 3.402823466e38f)) return 0;
    double x = ldexp((double)v, -lo);
    int q = 0;
    for (int ww = windows - 1; ww >= w; --ww) {
        const double qd = rint(ldexp(x, -kWindowBits * ww));
        x -= ldexp(qd, kWindowBits * ww);
        q = (int)qd;
    }
    return q;
}

// First row of pair `pair` of a quad (the other is 8 further).
__device__ __forceinline__ int row_of_pair(int quad, int pair) { return 16 * (quad >> 1) + 2 * (quad & 1) + (pair >> 1) + 4 * (pair & 1); }

// Residuals of row n as CSR bounds (empty past N).
__device__ __forceinline__ void row_bounds(const int32_t* row_ptr, int N, int n, int& begin, int& end) {
    begin = n < N ? row_ptr[n] : 0;
    end = n < N ? row_ptr[n + 1] : 0;
}

// Longest list of a quad's four pairs, window by window: columns at which one of the two rows has a residual (with
// several windows: one whose digits in this window are not all zero).
__global__ __launch_bounds__(4 * kWave) void k_longest_lists(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
                                                            const float* __restrict__ val, int N, int Kw, const int32_t* __restrict__ range,
                                                            int32_t* __restrict__ longest) {
    extern __shared__ __align__(16) uint32_t lds[];                            // a bitmap for each wave, then the four lengths
    const int quad = blockIdx.x, wave = threadIdx.x / kWave, lane = lane_id();
    uint32_t* map = lds + wave * Kw;
    uint32_t* lengths = lds + 4 * Kw;
    const int lo = range[0], windows = windows_of(lo, range[1]);
    const int row = row_of_pair(quad, wave);
    for (int w = 0; w < windows; ++w) {
        for (int j = lane; j < Kw; j += kWave) map[j] = 0u;
        __syncthreads();
        for (int h = 0; h < 2; ++h) {
            int e, end;
            row_bounds(row_ptr, N, row + 8 * h, e, end);
            for (e += lane; e < end; e += kWave)
                if (windows == 1 || window_value(val[e], lo, windows, w) != 0) atomicOr(&map[col[e] >> 5], 1u << (col[e] & 31));
        }
        __syncthreads();
        int n = 0;
        for (int j = lane; j < Kw; j += kWave) n += __builtin_popcount(map[j]);
        for (int off = kWave / 2; off > 0; off >>= 1) n += __shfl_xor(n, off, kWave);
        if (lane == 0) lengths[wave] = (uint32_t)n;
        __syncthreads();
        if (threadIdx.x == 0) longest[(size_t)quad * kMaxWindows + w] = (int32_t)max(max(lengths[0], lengths[1]), max(lengths[2], lengths[3]));
    }
}

// The codes of a window value's six digits, FP6 (E2M3): d / 8 at an even k, d / 4 at an odd one; three to a word.
__device__ __forceinline__ void digit_codes(int q, bool odd, uint32_t* to) {
    const int biased = q + 16 * 0x108421;                        // 16 * (1 + 32 + 32^2 + 32^3 + 32^4): five digits of 0 .. 31, less 16
    uint32_t out[2] = {0u, 0u};
#pragma unroll
    for (int d = 0; d < 6; ++d) {
        const int digit = d == 5 ? biased >> 25 : ((biased >> (5 * d)) & 31) - 16;
        const uint32_t m = (uint32_t)abs(digit);
        const uint32_t code = (odd ? (m < 8u ? 2u * m : m + 8u) : m) | (digit < 0 ? 32u : 0u);
        out[d / 3] |= code << (6 * (d % 3));
    }
    to[0] = out[0];
    to[1] = out[1];
}

// The digit steps of a pair of rows, a wave each; the last block clears the kStepPad steps behind the last one.
// LDS: bitmaps of the two rows and of the list, prefix counts of the first two, the list, and a step's codes.
__global__ __launch_bounds__(kWave) void k_digit_steps(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
                                                       const float* __restrict__ val, int N, int Kw, int lo, int windows, int k_scale,
                                                       const int32_t* __restrict__ step_first,   // [quads * windows + 1]
                                                       uint8_t* __restrict__ out) {
    extern __shared__ __align__(16) uint32_t lds[];
    const int lane = threadIdx.x, pairs = (int)gridDim.x - 1;
    if ((int)blockIdx.x == pairs) {
        uint32_t* pad = reinterpret_cast<uint32_t*>(out + (size_t)step_first[(size_t)(pairs / 4) * windows] * kStepBytes);
        for (int t = lane; t < kStepPad * kStepBytes / 4; t += kWave) pad[t] = 0u;
        return;
    }
    uint32_t* codes = lds;                                       // [lane block][row][32 values][2]: see digit_codes
    uint32_t* map = lds + kCodeWords;                            // [2][Kw]: the rows' columns
    uint32_t* list_map = map + 2 * Kw;                           // [Kw]: those on the list
    uint16_t* before = reinterpret_cast<uint16_t*>(list_map + Kw);   // [2][Kw]: residuals of the row in the words before
    uint16_t* list = before + 2 * Kw;                            // the list: k in ascending order of k mod 32, then k
    const int quad = (int)blockIdx.x >> 2, pair = (int)blockIdx.x & 3, row = row_of_pair(quad, pair);
    int begin[2], end[2];
    for (int j = lane; j < 2 * Kw; j += kWave) map[j] = 0u;
    __syncthreads();
    for (int h = 0; h < 2; ++h) {
        row_bounds(row_ptr, N, row + 8 * h, begin[h], end[h]);
        for (int e = begin[h] + lane; e < end[h]; e += kWave) atomicOr(&map[h * Kw + (col[e] >> 5)], 1u << (col[e] & 31));
    }
    __syncthreads();
    const int share = (Kw + kWave - 1) / kWave, j0 = min(Kw, lane * share), j1 = min(Kw, j0 + share);
    for (int h = 0; h < 2; ++h) {
        int mine = 0;
        for (int j = j0; j < j1; ++j) mine += __builtin_popcount(map[h * Kw + j]);
        int sum = mine;
        for (int off = 1; off < kWave; off <<= 1) {
            const int other = __shfl_up(sum, off, kWave);
            if (lane >= off) sum += other;
        }
        sum -= mine;
        for (int j = j0; j < j1; ++j) {
            before[h * Kw + j] = (uint16_t)sum;
            sum += __builtin_popcount(map[h * Kw + j]);
        }
    }
    __syncthreads();
    auto residual = [&](int h, int k) -> float {                 // of row h of the pair at column k
        const uint32_t word = map[h * Kw + (k >> 5)], bit = 1u << (k & 31);
        return word & bit ? val[begin[h] + before[h * Kw + (k >> 5)] + __builtin_popcount(word & (bit - 1u))] : 0.0f;
    };
    for (int w = 0; w < windows; ++w) {
        // the list: those columns whose digits in this window are not all zero (of one window: all)
        for (int j = lane; j < Kw; j += kWave) list_map[j] = windows == 1 ? map[j] | map[Kw + j] : 0u;
        __syncthreads();
        if (windows > 1)
            for (int h = 0; h < 2; ++h)
                for (int e = begin[h] + lane; e < end[h]; e += kWave)
                    if (window_value(val[e], lo, windows, w) != 0) atomicOr(&list_map[col[e] >> 5], 1u << (col[e] & 31));
        __syncthreads();
        const int bit = lane & 31, half = (Kw + 1) / 2, from = lane < 32 ? 0 : half, to = lane < 32 ? half : Kw;
        int mine = 0;
        for (int j = from; j < to; ++j) mine += (int)((list_map[j] >> bit) & 1u);
        const int lower = __shfl(mine, bit, kWave), both = lower + __shfl(mine, bit + 32, kWave);
        int upto = both;                                         // over the bits up to this one
        for (int off = 1; off < 32; off <<= 1) {
            const int other = __shfl_up(upto, off, 32);
            if (bit >= off) upto += other;
        }
        const int n = __shfl(upto, 31, kWave);
        int at = upto - both + (lane < 32 ? 0 : lower);
        for (int j = from; j < to; ++j)
            if ((list_map[j] >> bit) & 1u) list[at++] = (uint16_t)(32 * j + bit);
        __syncthreads();

        const int first = step_first[(size_t)quad * windows + w], S = (step_first[(size_t)quad * windows + w + 1] - first) / 4;
        uint8_t* base = out + (size_t)(first + pair * S) * kStepBytes;
        const int g = lane >> 4, i = lane & 15;
        for (int st = 0; st < S; ++st, base += kStepBytes) {
            // value 16 * qq + i of lane block g: a gather's half wave has 32 neighbours of the list, 4 * S apart
            uint32_t rows = 0;
            for (int qq = 0; qq < 2; ++qq) {
                const int gather = 4 * st + 2 * (g >> 1) + qq, e = ((g & 1) * 16 + i) * 4 * S + gather;
                const bool in = e < n;
                const int k = in ? list[e] : gather < n ? list[gather] : 0;
                rows |= (uint32_t)(k * k_scale) << (16 * qq);
                for (int h = 0; h < 2; ++h)
                    digit_codes(in ? window_value(residual(h, k), lo, windows, w) : 0, k & 1, codes + ((g * 2 + h) * 32 + 16 * qq + i) * 2);
            }
            __syncthreads();
            *reinterpret_cast<uint32_t*>(base + kStepRows + lane * 4) = rows;
            if (lane < 48) {                                     // digit d of row h in lane block lane / 12
                const int h = lane % 12 / 6, d = lane % 6;
                const uint32_t* from_codes = codes + (lane / 12 * 2 + h) * 64 + d / 3;
                const int shift = 6 * (d % 3);
                uint32_t word[6] = {0u, 0u, 0u, 0u, 0u, 0u};
#pragma unroll
                for (int t = 0; t < 32; ++t) {
                    const uint32_t code = (from_codes[2 * t] >> shift) & 63u;
                    word[6 * t / 32] |= code << (6 * t % 32);
                    if (6 * t % 32 > 26) word[6 * t / 32 + 1] |= code >> (32 - 6 * t % 32);
                }
                *reinterpret_cast<uint4*>(base + lane * 16) = make_uint4(word[0], word[1], word[2], word[3]);
                *reinterpret_cast<uint2*>(base + kStepA8 + lane * 8) = make_uint2(word[4], word[5]);
            }
            __syncthreads();
        }
    }
}

size_t digit_steps_lds(int Kw, int most_steps) { return 4u * kCodeWords + 4u * 3 * Kw + 2u * 2 * Kw + 2u * 128 * most_steps; }
// (18432 columns, all of them on the list: 49 KB)
static_assert(4u * kCodeWords + 16u * (kRowsMaxK / 32) + 2u * kRowsMaxK <= 64 * 1024, "the LDS that a launch gets without asking");

}  // namespace

int launch_row_valsum(const int32_t* row_ptr, const float* val, int N, int rows, double* valsum, hipStream_t s) {
    const int per_block = kBlock / kWave;
    hipLaunchKernelGGL(k_row_valsum, dim3((unsigned)((rows + per_block - 1) / per_block)), dim3(kBlock), 0, s, row_ptr, val, N, rows, valsum);
    APB_HIP(hipGetLastError());
    return APB_OK;
}

size_t digit_scratch_words(int N) { return 2 + (size_t)4 * ((N + 31) / 32) * kMaxWindows; }

int build_rows_layer(LayerDev& d, int32_t* found, hipStream_t s) {
    const int tiles = 2 * ((d.N + 31) / 32), quads = 2 * tiles;
    const long long words = (long long)tiles * d.rows_ksteps * 64;
    hipLaunchKernelGGL(k_rows_sign, dim3((unsigned)((words + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, d.sign, d.N, d.Kw, d.rows_ksteps, words,
                       d.rows_sign, found);
    APB_HIP(hipGetLastError());

    // range of the residuals' bits, and from it the lengths of the lists: [0], [1] the range, then [quads][kMaxWindows]
    std::vector<int32_t> h(digit_scratch_words(d.N));
    if (d.nnz > 0) {
        const long long blocks = (d.nnz + 4 * kBlock - 1) / (4 * kBlock);
        hipLaunchKernelGGL(k_residual_range, dim3((unsigned)(blocks < 1024 ? blocks : 1024)), dim3(kBlock), 0, s, d.val, d.nnz, found);
        APB_HIP(hipGetLastError());
    }
    hipLaunchKernelGGL(k_longest_lists, dim3((unsigned)quads), dim3(4 * kWave), 4u * (4 * d.Kw + 4), s, d.row_ptr, d.col_idx, d.val, d.N, d.Kw,
                       found, found + 2);
    APB_HIP(hipGetLastError());
    APB_HIP(hipMemcpyAsync(h.data(), found, h.size() * sizeof(int32_t), hipMemcpyDeviceToHost, s));
    APB_HIP(hipStreamSynchronize(s));

    const int W = windows_of(h[0], h[1]);
    d.rows_windows = W;
    d.rows_unit_log2 = h[0] == INT_MAX ? 0 : h[0];
    // One upload: first step of each tile, first step of each quad and window, and (bytes) the steps of a pair there.
    const size_t lists = (size_t)quads * W, at_lists = (size_t)tiles + 1, at_count = at_lists + lists + 1;
    std::vector<int32_t> up(at_count + (lists + 3) / 4, 0);
    uint8_t* count = reinterpret_cast<uint8_t*>(up.data() + at_count);
    long long steps = 0;
    int most = 1;
    for (int quad = 0; quad < quads; ++quad) {
        if (quad % 2 == 0) up[quad / 2] = (int32_t)steps;
        for (int w = 0; w < W; ++w) {
            const int S = digit_steps_of(h[2 + (size_t)quad * kMaxWindows + w]);
            count[(size_t)quad * W + w] = (uint8_t)S;
            up[at_lists + (size_t)quad * W + w] = (int32_t)steps;
            steps += 4 * S;
            most = S > most ? S : most;
        }
    }
    if (steps > INT_MAX - kStepPad) return APB_ERR_NOMEM;        // (the steps alone would take 3 TB)
    up[tiles] = up[at_count - 1] = (int32_t)steps;
    d.rows_steps = steps;
    DeviceArrays arrays;
    arrays.add(&d.rows_first, up.size() + 4);                    // (counts are read four at a time)
    arrays.add(&d.rows_step, (size_t)(steps + kStepPad) * kStepBytes);
    const int rc = arrays.alloc(&d.blocks[2]);
    if (rc != APB_OK) return rc;
    d.rows_count = reinterpret_cast<uint8_t*>(d.rows_first + at_count);
    APB_HIP(hipMemcpyAsync(d.rows_first, up.data(), up.size() * sizeof(int32_t), hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(k_digit_steps, dim3((unsigned)(4 * quads + 1)), dim3(kWave), digit_steps_lds(d.Kw, most), s, d.row_ptr, d.col_idx, d.val,
                       d.N, d.Kw, d.rows_unit_log2, W, d.K <= kRowsByteK ? 8 : 1, d.rows_first + at_lists, d.rows_step);
    APB_HIP(hipGetLastError());
    APB_HIP(hipStreamSynchronize(s));                            // (the staging vectors end here)
    return APB_OK;
}

}  // namespace apb

// Host side of the C ABI: argument checks, layer ownership, launch-order row binning, tile runs.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <numeric>
#include <vector>

#include "apb_internal.h"
#include "apb_rows_shape.h"

namespace apb {

static thread_local int g_last_hip_error = 0;
void set_last_hip_error(hipError_t e) { g_last_hip_error = (int)e; }

namespace {

hipStream_t as_stream(void* s) { return reinterpret_cast<hipStream_t>(s); }

void free_layer_buffers(LayerDev& d) {
    for (void* p : d.blocks)
        if (p) (void)hipFree(p);
    d = LayerDev{};
}

// Launch-order row binning for the skewed residual counts: rows sorted by decreasing residual
// count are dealt to the row tiles like cards, forwards then backwards (a "snake"), so every
// tile of kRowTile rows carries about the same number of residuals.
std::vector<int32_t> balanced_slots(const std::vector<int32_t>& counts, int Np) {
    const int N = (int)counts.size();
    const int tiles = Np / kRowTile;
    std::vector<int32_t> order(N);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return counts[a] > counts[b]; });
    std::vector<int32_t> perm(Np, -1);
    std::vector<int> fill(tiles, 0);
    for (int i = 0; i < N; ++i) {
        const int round = i / tiles, pos = i % tiles;
        const int t = (round & 1) ? tiles - 1 - pos : pos;
        perm[t * kRowTile + fill[t]++] = order[i];
    }
    // Inside a tile the order of the rows is free: ascending, so that rows sharing a 32-row word of
    // a packed output sit next to each other.
    for (int t = 0; t < tiles; ++t) std::sort(perm.begin() + t * kRowTile, perm.begin() + t * kRowTile + fill[t]);
    return perm;
}

// Regroup the CSR for the columns-in-lanes kernel: for every tile of kRowTile launch slots and every chunk of
// kChunkK columns one flat run of entries, sorted by (row in tile, column) and padded to whole
// blocks of 8.  A block is 24 words: 8 keys (2*row | column_in_chunk << 8), then the 8 residuals as
// float64 times 2^kEntValScaleLog2; padding entries have key 0 and value 0.  seg_ptr, which counts blocks, lies at the
// front of `out`, the blocks from word ent_at on.
void build_tile_runs(const std::vector<int32_t>& perm, const std::vector<int32_t>& row_ptr, const int32_t* col, const float* val, long long nnz,
                     int nchunks, std::vector<uint32_t>& out, size_t& ent_at) {
    const int tiles = (int)perm.size() / kRowTile;
    ent_at = ((size_t)tiles * (nchunks + 1) + 63) / 64 * 64;
    out.reserve(ent_at + (size_t)nnz * 4 + 64);
    out.assign(ent_at, 0u);
    auto blocks = [&] { return (uint32_t)((out.size() - ent_at) / kEntBlockWords); };
    std::vector<int32_t> cursor(kRowTile);
    std::vector<uint32_t> key;
    std::vector<double> dval;
    for (int t = 0; t < tiles; ++t) {
        for (int r = 0; r < kRowTile; ++r) {
            const int n = perm[(size_t)t * kRowTile + r];
            cursor[r] = n >= 0 ? row_ptr[n] : 0;
        }
        for (int c = 0; c < nchunks; ++c) {
            out[(size_t)t * (nchunks + 1) + c] = blocks();
            const int hi = (c + 1) * kChunkK;
            key.clear();
            dval.clear();
            for (int r = 0; r < kRowTile; ++r) {
                const int n = perm[(size_t)t * kRowTile + r];
                if (n < 0) continue;
                const int end = row_ptr[n + 1];
                while (cursor[r] < end && col[cursor[r]] < hi) {
                    key.push_back((uint32_t)(2 * r) | ((uint32_t)(col[cursor[r]] - c * kChunkK) << 8));
                    dval.push_back(std::ldexp((double)val[cursor[r]], kEntValScaleLog2));
                    ++cursor[r];
                }
            }
            while (key.size() % 8 != 0) {
                key.push_back(0u);
                dval.push_back(0.0);
            }
            for (size_t b = 0; b < key.size(); b += 8) {
                const size_t at = out.size();
                out.resize(at + kEntBlockWords);
                std::memcpy(&out[at], &key[b], 8 * sizeof(uint32_t));
                std::memcpy(&out[at + 8], &dval[b], 8 * sizeof(double));
            }
        }
        out[(size_t)t * (nchunks + 1) + nchunks] = blocks();
    }
}

int compress_impl(const float* W, int N, int K, float delta, float alpha, hipStream_t s, LayerDev& d) {
    d.N = N;
    d.K = K;
    d.Kw = (K + 31) / 32;
    d.waves = 2;                                       // workgroup = 2, 4 or 8 waves of kRowTile rows each
    while (d.waves < kMaxWavesPerBlock && d.waves * kRowTile < N) d.waves *= 2;
    const int rows_per_block = kRowTile * d.waves;
    d.Np = rows_per_block * ((N + rows_per_block - 1) / rows_per_block);
    d.nchunks = (d.Kw + kChunkWords - 1) / kChunkWords;
    const bool digits = K <= kRowsMaxK;
    const int Kw2 = 2 * ((d.Kw + 1) / 2), rows = 32 * ((N + 31) / 32);   // (whole words of a packed output)
    constexpr int kParts = 1024;
    double* parts = nullptr;
    int32_t *counts = nullptr, *found = nullptr;
    DeviceArrays fixed;
    fixed.add(&parts, 2 * kParts);
    fixed.add(&counts, (size_t)N);
    fixed.add(&found, digit_scratch_words(N));
    fixed.add(&d.sign, (size_t)N * d.Kw);
    fixed.add(&d.rowsum, (size_t)N);
    fixed.add(&d.row_ptr, (size_t)N + 1 + d.Np);       // and perm
    fixed.add(&d.signT, (size_t)d.Np * Kw2);
    fixed.add(&d.signC, (size_t)N * Kw2);
    fixed.add(&d.chunk_ptr, (size_t)d.Np * (d.nchunks + 1));
    fixed.add(&d.slot_valsum, (size_t)d.Np);
    fixed.add(&d.rows_valsum, (size_t)rows);
    d.rows_ksteps = (d.Kw + 3) / 4;
    fixed.add(&d.rows_sign, digits ? (size_t)rows / 16 * d.rows_ksteps * 64 : 0);
    int rc = fixed.alloc(&d.blocks[0]);
    if (rc != APB_OK) return rc;
    d.perm = d.row_ptr + N + 1;

    if (std::isnan(alpha)) {                          // default scale: mean |w| over the binarized set
        static_assert(sizeof(long long) == sizeof(double), "sums and counts share an array");
        long long* part_cnt = reinterpret_cast<long long*>(parts + kParts);
        std::vector<double> h(2 * kParts);
        if ((rc = launch_inlier_abs_sum(W, (long long)N * K, delta, parts, part_cnt, kParts, s)) != APB_OK) return rc;
        APB_HIP(hipMemcpyAsync(h.data(), parts, 2 * kParts * sizeof(double), hipMemcpyDeviceToHost, s));
        APB_HIP(hipStreamSynchronize(s));
        double total = 0.0;
        long long cnt = 0;
        for (int i = 0; i < kParts; ++i) {
            long long c;
            std::memcpy(&c, &h[kParts + i], sizeof(c));
            total += h[i];
            cnt += c;
        }
        alpha = cnt > 0 ? (float)(total / (double)cnt) : 0.0f;
    }
    d.alpha = alpha;

    std::vector<int32_t> hcounts(N);
    if ((rc = launch_sign_pack_count(W, N, K, d.Kw, delta, d.sign, counts, d.rowsum, s)) != APB_OK) return rc;
    APB_HIP(hipMemcpyAsync(hcounts.data(), counts, (size_t)N * sizeof(int32_t), hipMemcpyDeviceToHost, s));
    APB_HIP(hipStreamSynchronize(s));

    std::vector<int32_t> hrow_ptr((size_t)N + 1 + d.Np, 0);
    long long nnz = 0;
    for (int n = 0; n < N; ++n) {
        nnz += hcounts[n];
        hrow_ptr[n + 1] = (int32_t)nnz;
    }
    d.nnz = nnz;
    const std::vector<int32_t> hperm = balanced_slots(hcounts, d.Np);
    std::copy(hperm.begin(), hperm.end(), hrow_ptr.begin() + N + 1);

    DeviceArrays csr;
    csr.add(&d.col_idx, (size_t)nnz);
    csr.add(&d.val, (size_t)nnz);
    csr.add(&d.vald, (size_t)nnz);
    if ((rc = csr.alloc(&d.blocks[1])) != APB_OK) return rc;
    APB_HIP(hipMemcpyAsync(d.row_ptr, hrow_ptr.data(), hrow_ptr.size() * sizeof(int32_t), hipMemcpyHostToDevice, s));
    if (nnz > 0 && (rc = launch_scatter_csr(W, N, K, delta, alpha, d.row_ptr, d.col_idx, d.val, d.vald, s)) != APB_OK) return rc;
    if ((rc = launch_slot_major_signs(d.sign, d.perm, d.Np, d.Kw, Kw2, d.signT, s)) != APB_OK) return rc;
    if ((rc = launch_slot_major_signs(d.sign, nullptr, N, d.Kw, Kw2, d.signC, s)) != APB_OK) return rc;
    if ((rc = launch_row_valsum(d.row_ptr, d.val, N, rows, d.rows_valsum, s)) != APB_OK) return rc;
    if ((rc = launch_slot_tables(d.perm, d.row_ptr, d.col_idx, d.rows_valsum, d.Np, d.nchunks, d.chunk_ptr, d.slot_valsum,
                                 s)) != APB_OK)
        return rc;
    // Tile runs for the columns-in-lanes kernel are built on the host from the CSR just written, which comes over (the
    // columns and the values behind them) while the digit steps are built.
    const bool tile_runs = !digits || columns_kernel_possible(N, K, nnz);
    const size_t val_at = reinterpret_cast<uint8_t*>(d.val) - reinterpret_cast<uint8_t*>(d.col_idx);
    std::vector<uint8_t> hcsr(tile_runs ? val_at + (size_t)nnz * sizeof(float) : 0);
    if (tile_runs && nnz > 0) APB_HIP(hipMemcpyAsync(hcsr.data(), d.col_idx, hcsr.size(), hipMemcpyDeviceToHost, s));
    if (digits && (rc = build_rows_layer(d, found, s)) != APB_OK) return rc;
    if (!tile_runs) return APB_OK;                     // (it waited for the stream: the staging vectors may go)
    if (!digits) APB_HIP(hipStreamSynchronize(s));
    std::vector<uint32_t> runs;                        // seg_ptr, then the entries from a multiple of 64 words on
    size_t ent_at = 0;
    build_tile_runs(hperm, hrow_ptr, reinterpret_cast<const int32_t*>(hcsr.data()), reinterpret_cast<const float*>(hcsr.data() + val_at), nnz,
                    d.nchunks, runs, ent_at);
    uint32_t* base = nullptr;
    if ((rc = dev_alloc(&base, runs.size())) != APB_OK) return rc;
    d.blocks[3] = base;
    d.seg_ptr = reinterpret_cast<int32_t*>(base);
    d.ent = base + ent_at;
    APB_HIP(hipMemcpyAsync(base, runs.data(), runs.size() * sizeof(uint32_t), hipMemcpyHostToDevice, s));
    APB_HIP(hipStreamSynchronize(s));                 // host staging vectors go out of scope after this
    return APB_OK;
}

int position_bits(long long n) {
    if (n <= 2) return 1;
    int b = 0;
    for (long long v = n - 1; v > 0; v >>= 1) ++b;
    return b;
}

}  // namespace
}  // namespace apb

using namespace apb;

extern "C" {

int apb_compress(const float* W, int N, int K, float delta, float alpha, void* stream, apb_layer** out) {
    if (out) *out = nullptr;
    if (!W || !out) return APB_ERR_NULL;
    if (N <= 0 || K <= 0 || (long long)N * K >= (1LL << 31) || (long long)K * 3 >= (1LL << 31)) return APB_ERR_SHAPE;
    if (std::isnan(delta)) return APB_ERR_VALUE;
    if (!std::isnan(alpha) && (alpha < 0.0f || std::isinf(alpha))) return APB_ERR_VALUE;
    apb_layer* L = new (std::nothrow) apb_layer();
    if (!L) return APB_ERR_NOMEM;
    int rc;
    try {
        rc = compress_impl(W, N, K, delta, alpha, as_stream(stream), L->d);
    } catch (const std::bad_alloc&) {
        rc = APB_ERR_NOMEM;
    }
    if (rc != APB_OK) {
        free_layer_buffers(L->d);
        delete L;
        return rc;
    }
    *out = L;
    return APB_OK;
}

int apb_layer_info(const apb_layer* layer, int* N, int* K, float* alpha, long long* nnz, long long* mem_bits) {
    if (!layer) return APB_ERR_NULL;
    const LayerDev& d = layer->d;
    if (N) *N = d.N;
    if (K) *K = d.K;
    if (alpha) *alpha = d.alpha;
    if (nnz) *nnz = d.nnz;
    if (mem_bits) {
        const long long n = (long long)d.N * d.K;
        *mem_bits = n + d.nnz * (32 + position_bits(n));
    }
    return APB_OK;
}

int apb_layer_export(const apb_layer* layer, uint32_t* sign_words, int32_t* row_ptr, int32_t* col_idx, float* val,
                     int32_t* rowsum, void* stream) {
    if (!layer) return APB_ERR_NULL;
    const LayerDev& d = layer->d;
    hipStream_t s = as_stream(stream);
    if (sign_words)
        APB_HIP(hipMemcpyAsync(sign_words, d.sign, (size_t)d.N * d.Kw * sizeof(uint32_t), hipMemcpyDefault, s));
    if (row_ptr) APB_HIP(hipMemcpyAsync(row_ptr, d.row_ptr, ((size_t)d.N + 1) * sizeof(int32_t), hipMemcpyDefault, s));
    if (col_idx && d.nnz > 0)
        APB_HIP(hipMemcpyAsync(col_idx, d.col_idx, (size_t)d.nnz * sizeof(int32_t), hipMemcpyDefault, s));
    if (val && d.nnz > 0) APB_HIP(hipMemcpyAsync(val, d.val, (size_t)d.nnz * sizeof(float), hipMemcpyDefault, s));
    if (rowsum) APB_HIP(hipMemcpyAsync(rowsum, d.rowsum, (size_t)d.N * sizeof(int32_t), hipMemcpyDefault, s));
    APB_HIP(hipStreamSynchronize(s));
    return APB_OK;
}

int apb_layer_export_steps(const apb_layer* layer, long long sizes[4], int32_t* first, uint8_t* count, uint8_t* steps,
                           double* valsum, uint32_t* sign, void* stream) {
    if (!layer || !sizes) return APB_ERR_NULL;
    const LayerDev& d = layer->d;
    const long long tiles = 2 * (((long long)d.N + 31) / 32), S = d.rows_steps;
    sizes[0] = S;
    sizes[1] = S ? d.rows_windows : 0;
    sizes[2] = S ? d.rows_unit_log2 : 0;
    sizes[3] = S ? tiles * d.rows_ksteps * 64 : 0;
    if (S == 0) return APB_OK;
    hipStream_t s = as_stream(stream);
    if (first) APB_HIP(hipMemcpyAsync(first, d.rows_first, (size_t)(tiles + 1) * 4, hipMemcpyDefault, s));
    if (count) APB_HIP(hipMemcpyAsync(count, d.rows_count, (size_t)(2 * tiles * d.rows_windows), hipMemcpyDefault, s));
    if (steps) APB_HIP(hipMemcpyAsync(steps, d.rows_step, (size_t)(S + kStepPad) * kStepBytes, hipMemcpyDefault, s));
    if (valsum) APB_HIP(hipMemcpyAsync(valsum, d.rows_valsum, (size_t)(16 * tiles) * 8, hipMemcpyDefault, s));
    if (sign) APB_HIP(hipMemcpyAsync(sign, d.rows_sign, (size_t)sizes[3] * 4, hipMemcpyDefault, s));
    APB_HIP(hipStreamSynchronize(s));
    return APB_OK;
}

void apb_layer_free(apb_layer* layer) {
    if (!layer) return;
    free_layer_buffers(layer->d);
    delete layer;
}

size_t apb_acts_bytes(int K, int M, int bits) {
    if (bad_shape_acts(K, M) || (bits != 1 && bits != 2)) return 0;
    const size_t Kw = ((size_t)K + 31) / 32;
    const size_t Mp = (size_t)kWave * (((size_t)M + kWave - 1) / kWave);
    return sizeof(uint32_t) * Mp * ((size_t)bits * Kw + 1);
}

int apb_quantize_acts(const float* X, int K, int M, int bits, float step, void* packed, void* stream) {
    if (!X || !packed) return APB_ERR_NULL;
    if (bad_shape_acts(K, M)) return APB_ERR_SHAPE;
    if (bits != 1 && bits != 2) return APB_ERR_BITS;
    if (!std::isfinite(step) || !(step > 0.0f)) return APB_ERR_VALUE;
    const size_t Kw = ((size_t)K + 31) / 32;
    const size_t Mp = (size_t)kWave * (((size_t)M + kWave - 1) / kWave);
    uint32_t* planes = static_cast<uint32_t*>(packed);
    int32_t* colsum = reinterpret_cast<int32_t*>(planes + (size_t)bits * Kw * Mp);
    const float inv_step = 1.0f / step;
    return launch_quantize(X, K, M, bits, inv_step, planes, colsum, as_stream(stream));
}

enum FwdKind { kFwdFull, kFwdFullPopcount, kFwdIntPopcount, kFwdIntMfma };

static int forward_common(const apb_layer* layer, const void* packed, int M, int bits, float step, float* Y,
                          int32_t* D, void* stream, FwdKind kind) {
    if (!layer || !packed || (!Y && !D)) return APB_ERR_NULL;
    const LayerDev& d = layer->d;
    if (bad_shape_acts(d.K, M) || (long long)d.N * M >= (1LL << 40)) return APB_ERR_SHAPE;
    if (bits != 1 && bits != 2) return APB_ERR_BITS;
    if (Y && (!std::isfinite(step) || !(step > 0.0f))) return APB_ERR_VALUE;
    const size_t Mp = (size_t)kWave * (((size_t)M + kWave - 1) / kWave);
    const uint32_t* planes = static_cast<const uint32_t*>(packed);
    const int32_t* colsum = reinterpret_cast<const int32_t*>(planes + (size_t)bits * d.Kw * Mp);
    hipStream_t s = as_stream(stream);
    if (kind == kFwdIntMfma) {
        return launch_binary_mfma(d, planes, colsum, M, bits, D, s);
    }
    if (kind == kFwdFull) {
        return launch_forward_best(d, planes, colsum, M, bits, step, Y, s);
    }
    return launch_forward_popcount(d, planes, colsum, M, bits, step, Y, D, s);
}

int apb_forward(const apb_layer* layer, const void* packed, int M, int bits, float step, float* Y, void* stream) {
    if (!Y) return APB_ERR_NULL;
    return forward_common(layer, packed, M, bits, step, Y, nullptr, stream, kFwdFull);
}

int apb_forward_requant(const apb_layer* layer, const void* packed, int M, int bits, float step, const float* scale,
                        const float* shift, int bits_out, float step_out, void* packed_out, void* stream) {
    if (!layer || !packed || !packed_out || (scale == nullptr) != (shift == nullptr)) return APB_ERR_NULL;
    const LayerDev& d = layer->d;
    if (bad_shape_acts(d.K, M) || bad_shape_acts(d.N, M) || (long long)d.N * M >= (1LL << 40)) return APB_ERR_SHAPE;
    if ((bits != 1 && bits != 2) || (bits_out != 1 && bits_out != 2)) return APB_ERR_BITS;
    if (!std::isfinite(step) || !(step > 0.0f) || !std::isfinite(step_out) || !(step_out > 0.0f)) return APB_ERR_VALUE;
    const size_t Mp = (size_t)kWave * (((size_t)M + kWave - 1) / kWave);
    const uint32_t* planes = static_cast<const uint32_t*>(packed);
    const int32_t* colsum = reinterpret_cast<const int32_t*>(planes + (size_t)bits * d.Kw * Mp);
    hipStream_t s = as_stream(stream);
    uint32_t* out = static_cast<uint32_t*>(packed_out);
    if (!takes_columns_kernel(d, M, bits, true))
        return launch_forward_rows_requant(d, planes, colsum, M, bits, step, nullptr, scale, shift, bits_out, 1.0f / step_out,
                                           out, s);
    return launch_forward_requant(d, planes, colsum, M, bits, step, nullptr, scale, shift, bits_out, 1.0f / step_out, out, s);
}

const char* apb_forward_kernel_name(const apb_layer* layer, int M, int bits) {
    if (!layer || M <= 0 || (bits != 1 && bits != 2)) return "";
    if (!takes_columns_kernel(layer->d, M, bits, false)) return forward_rows_kernel_name(layer->d, M, bits);
    return forward_kernel_name(layer->d, M, bits);
}

int apb_quantize_forward_is_one_kernel(const apb_layer* layer, int M, int bits) {
    if (!layer || M <= 0 || (bits != 1 && bits != 2)) return 0;
    return step_is_one_kernel(layer->d, M, bits) ? 1 : 0;
}

int apb_quantize_forward(const apb_layer* layer, const float* X, int M, int bits, float step, void* packed, float* Y,
                         void* stream) {
    if (!layer || !X || !packed || !Y) return APB_ERR_NULL;
    const LayerDev& d = layer->d;
    if (bad_shape_acts(d.K, M) || (long long)d.N * M >= (1LL << 40)) return APB_ERR_SHAPE;
    if (bits != 1 && bits != 2) return APB_ERR_BITS;
    if (!std::isfinite(step) || !(step > 0.0f)) return APB_ERR_VALUE;
    hipStream_t s = as_stream(stream);
    if (step_is_one_kernel(d, M, bits)) return launch_step_one_kernel(d, X, M, bits, step, Y, s);
    uint32_t* planes = static_cast<uint32_t*>(packed);
    int32_t* colsum = reinterpret_cast<int32_t*>(planes + (size_t)bits * d.Kw * ((size_t)kWave * (((size_t)M + kWave - 1) / kWave)));
    return launch_quantize_then_forward(d, X, M, bits, step, planes, colsum, Y, s);
}

// Shape checks shared by the two convolution entry points; fills `conv` and the output pixel count.
static int conv_shape(const LayerDev& d, int B, int H, int W, int stride, ConvShape& conv, int& P_out) {
    if (B <= 0 || H <= 0 || W <= 0 || (stride != 1 && stride != 2)) return APB_ERR_SHAPE;
    if (d.K % 9 != 0 || (d.K / 9) % 32 != 0) return APB_ERR_SHAPE;
    if (d.K / 9 > 16384) return APB_ERR_SHAPE;                 // the kernels' row -> tap arithmetic is exact up to here
    const long long pixels = (long long)B * H * W;
    if (pixels >= (1LL << 28)) return APB_ERR_SHAPE;
    const long long Pp_in = kWave * ((pixels + kWave - 1) / kWave);
    // a plane of the map is one buffer range of the kernels' loads: below 2^31 bytes
    if ((long long)(d.K / 9 / 32) * Pp_in * 4 >= (1LL << 31)) return APB_ERR_SHAPE;
    const int Ho = (H - 1) / stride + 1, Wo = (W - 1) / stride + 1;
    const long long out_pixels = (long long)B * Ho * Wo;
    if ((long long)d.N * out_pixels >= (1LL << 40)) return APB_ERR_SHAPE;
    conv = ConvShape{d.K / 9, H, W, stride, Ho, Wo, (int)Pp_in};
    P_out = (int)out_pixels;
    return APB_OK;
}

int apb_forward_conv3x3(const apb_layer* layer, const void* fmap, int B, int H, int W, int stride, int bits, float step,
                        void* /*workspace*/, size_t /*workspace_bytes*/, float* Y, void* stream) {
    if (!layer || !fmap || !Y) return APB_ERR_NULL;
    const LayerDev& d = layer->d;
    ConvShape conv;
    int P;
    int rc = conv_shape(d, B, H, W, stride, conv, P);
    if (rc != APB_OK) return rc;
    if (bits != 1 && bits != 2) return APB_ERR_BITS;
    if (!std::isfinite(step) || !(step > 0.0f)) return APB_ERR_VALUE;
    hipStream_t s = as_stream(stream);
    const uint32_t* planes = static_cast<const uint32_t*>(fmap);
    const int32_t* pixsum = reinterpret_cast<const int32_t*>(planes + (size_t)bits * (conv.C / 32) * conv.Pp_in);
    if (!takes_columns_kernel(d, P, bits, false))
        return launch_forward_rows(d, planes, nullptr, P, bits, step, &conv, Y, s);
    return launch_forward(d, planes, pixsum, P, bits, step, &conv, Y, s);
}

int apb_forward_conv3x3_requant(const apb_layer* layer, const void* fmap, int B, int H, int W, int stride, int bits,
                                float step, const float* scale, const float* shift, int bits_out, float step_out,
                                void* /*workspace*/, size_t /*workspace_bytes*/, void* fmap_out, void* stream) {
    if (!layer || !fmap || !fmap_out || (scale == nullptr) != (shift == nullptr)) return APB_ERR_NULL;
    const LayerDev& d = layer->d;
    ConvShape conv;
    int P;
    int rc = conv_shape(d, B, H, W, stride, conv, P);
    if (rc != APB_OK) return rc;
    if ((bits != 1 && bits != 2) || (bits_out != 1 && bits_out != 2)) return APB_ERR_BITS;
    if (!std::isfinite(step) || !(step > 0.0f) || !std::isfinite(step_out) || !(step_out > 0.0f)) return APB_ERR_VALUE;
    const uint32_t* planes = static_cast<const uint32_t*>(fmap);
    const int32_t* pixsum = reinterpret_cast<const int32_t*>(planes + (size_t)bits * (conv.C / 32) * conv.Pp_in);
    hipStream_t s = as_stream(stream);
    uint32_t* out = static_cast<uint32_t*>(fmap_out);
    if (!takes_columns_kernel(d, P, bits, true))
        return launch_forward_rows_requant(d, planes, nullptr, P, bits, step, &conv, scale, shift, bits_out, 1.0f / step_out,
                                           out, s);
    return launch_forward_requant(d, planes, pixsum, P, bits, step, &conv, scale, shift, bits_out, 1.0f / step_out, out, s);
}

int apb_forward_popcount(const apb_layer* layer, const void* packed, int M, int bits, float step, float* Y,
                         void* stream) {
    if (!Y) return APB_ERR_NULL;
    return forward_common(layer, packed, M, bits, step, Y, nullptr, stream, kFwdFullPopcount);
}

int apb_forward_int(const apb_layer* layer, const void* packed, int M, int bits, int32_t* D, void* stream) {
    if (!D) return APB_ERR_NULL;
    return forward_common(layer, packed, M, bits, 1.0f, nullptr, D, stream, kFwdIntMfma);
}

int apb_forward_int_popcount(const apb_layer* layer, const void* packed, int M, int bits, int32_t* D, void* stream) {
    if (!D) return APB_ERR_NULL;
    return forward_common(layer, packed, M, bits, 1.0f, nullptr, D, stream, kFwdIntPopcount);
}

int apb_w2_pack(const float* W, int N, int K, float step_w, void* stream, apb_w2** out) {
    if (out) *out = nullptr;
    if (!W || !out) return APB_ERR_NULL;
    if (N <= 0 || K <= 0 || (long long)N * K >= (1LL << 31) || (long long)K * 3 >= (1LL << 31)) return APB_ERR_SHAPE;
    if (!std::isfinite(step_w) || !(step_w > 0.0f)) return APB_ERR_VALUE;
    apb_w2* w = new (std::nothrow) apb_w2();
    if (!w) return APB_ERR_NOMEM;
    w->N = N;
    w->K = K;
    w->Kw = (K + 31) / 32;
    w->step_w = step_w;
    const size_t Kw2 = 2 * (((size_t)w->Kw + 1) / 2);
    int rc = dev_alloc(&w->planes, (size_t)2 * N * w->Kw);
    if (rc == APB_OK) rc = dev_alloc(&w->planesC, (size_t)2 * Kw2 * N);
    if (rc == APB_OK) rc = launch_w2_pack(W, N, K, 1.0f / step_w, w->planes, w->planesC, as_stream(stream));
    if (rc != APB_OK) {
        apb_w2_free(w);
        return rc;
    }
    *out = w;
    return APB_OK;
}

int apb_w2_export(const apb_w2* w2, uint32_t* planes, void* stream) {
    if (!w2 || !planes) return APB_ERR_NULL;
    hipStream_t s = as_stream(stream);
    APB_HIP(hipMemcpyAsync(planes, w2->planes, (size_t)2 * w2->N * w2->Kw * sizeof(uint32_t), hipMemcpyDefault, s));
    APB_HIP(hipStreamSynchronize(s));
    return APB_OK;
}

void apb_w2_free(apb_w2* w2) {
    if (!w2) return;
    if (w2->planes) (void)hipFree(w2->planes);
    if (w2->planesC) (void)hipFree(w2->planesC);
    delete w2;
}

static int gemm_2_2_common(const apb_w2* w2, const void* packed, int M, float step_a, int32_t* D, float* Y,
                           void* stream) {
    if (!w2 || !packed || (!D && !Y)) return APB_ERR_NULL;
    if (bad_shape_acts(w2->K, M) || (long long)w2->N * M >= (1LL << 40)) return APB_ERR_SHAPE;
    if (Y && (!std::isfinite(step_a) || !(step_a > 0.0f))) return APB_ERR_VALUE;
    const size_t Mp = (size_t)kWave * (((size_t)M + kWave - 1) / kWave);
    const uint32_t* planes = static_cast<const uint32_t*>(packed);
    const int32_t* colsum = reinterpret_cast<const int32_t*>(planes + (size_t)2 * w2->Kw * Mp);
    const double scale = 0.5 * (double)w2->step_w * (double)step_a;
    return launch_gemm_2_2(w2->planesC, w2->N, w2->Kw, planes, colsum, M, scale, D, Y, as_stream(stream));
}

int apb_gemm_2_2_int(const apb_w2* w2, const void* packed, int M, int32_t* D, void* stream) {
    if (!D) return APB_ERR_NULL;
    return gemm_2_2_common(w2, packed, M, 1.0f, D, nullptr, stream);
}

int apb_gemm_2_2(const apb_w2* w2, const void* packed, int M, float step_a, float* Y, void* stream) {
    if (!Y) return APB_ERR_NULL;
    return gemm_2_2_common(w2, packed, M, step_a, nullptr, Y, stream);
}

const char* apb_strerror(int code) {
    switch (code) {
        case APB_OK: return "ok";
        case APB_ERR_NULL: return "a required pointer is NULL";
        case APB_ERR_SHAPE: return "bad shape (non-positive or too large)";
        case APB_ERR_BITS: return "activation bits must be 1 or 2";
        case APB_ERR_VALUE: return "bad scalar (delta NaN, alpha negative/infinite, or step not finite and > 0)";
        case APB_ERR_NOMEM: return "out of memory";
        case APB_ERR_HIP: return "a HIP call failed (see apb_last_hip_error)";
        case APB_ERR_SCRATCH: return "the packed activations of this K, M and bits do not fit the library's static scratch array";
        default: return "unknown apb status";
    }
}

int apb_last_hip_error(void) { return g_last_hip_error; }

}  // extern "C"

// The digit steps of the matrix-core forward kernel, built one bit at a time from the CSR of a layer: what the GPU
// builder's result is compared with, byte for byte.  (Layout: kStepBytes in apb_internal.h, repeated here.)
#include <climits>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <algorithm>
#include <vector>

namespace {

constexpr int kStepA8 = 48 * 16, kStepRows = 48 * 24, kStepBytes = 48 * 24 + 64 * 4, kStepPad = 8, kWindowBits = 30;

int digit_steps_of(int entries) {
    const int s = (entries + 127) / 128;
    return s <= 1 ? 1 : s <= 4 ? s : s <= 6 ? 6 : (s + 3) / 4 * 4;
}

struct DigitSteps {
    int windows = 1;
    std::vector<int32_t> first;
    std::vector<uint8_t> count;
    std::vector<uint8_t> step;
    std::vector<double> valsum;
    int unit = 0;
};
void build_digit_steps(int N, const std::vector<int32_t>& row_ptr, const std::vector<int32_t>& col, const std::vector<float>& val,
                       bool bytes, DigitSteps& o) {
    const int tiles = 2 * ((N + 31) / 32), rows = 16 * tiles;
    int lo = 0, hi = -1;
    bool any = false;
    o.valsum.assign(rows, 0.0);
    for (int n = 0; n < N; ++n)
        for (int e = row_ptr[n]; e < row_ptr[n + 1]; ++e) {
            o.valsum[n] += (double)val[e];
            const float v = std::fabs(val[e]);
            if (!(v > 0.0f) || std::isinf(v)) continue;
            int ex;
            const double f = std::frexp((double)v, &ex);           // v = f * 2^ex, f in [.5, 1)
            uint32_t mant = (uint32_t)(f * 16777216.0);            // 24 bits
            int low = ex - 24;
            while (!(mant & 1u)) { mant >>= 1; ++low; }
            if (!any || low < lo) lo = low;
            if (!any || ex - 1 > hi) hi = ex - 1;
            any = true;
        }
    o.windows = any ? (hi - lo + 2 + kWindowBits - 1) / kWindowBits : 1;
    o.unit = lo;
    const int W = o.windows;
    o.first.assign(tiles + 1, 0);
    o.count.assign((size_t)tiles * 2 * W, 1);
    long long steps = 0;
    struct Entry { int k; int q[2]; };
    for (int quad = 0; quad < 2 * tiles; ++quad) {
        if (quad % 2 == 0) o.first[quad / 2] = (int32_t)steps;
        for (int w = 0; w < W; ++w) {
            std::vector<Entry> lists[4];
            size_t longest = 0;
            for (int pr = 0; pr < 4; ++pr) {
                const int ra = 16 * (quad / 2) + 2 * (quad % 2) + pr / 2 + 4 * (pr % 2), rb = ra + 8;
                std::vector<Entry>& list = lists[pr];
                int ea = ra < N ? row_ptr[ra] : 0, eb = rb < N ? row_ptr[rb] : 0;
                const int eae = ra < N ? row_ptr[ra + 1] : 0, ebe = rb < N ? row_ptr[rb + 1] : 0;
                auto digits_of = [&](float v) -> int {
                    if (!std::isfinite(v)) v = 0.0f;
                    double x = std::ldexp((double)v, -lo);
                    int q = 0;
                    for (int ww = W - 1; ww >= w; --ww) {
                        const double qd = std::rint(std::ldexp(x, -kWindowBits * ww));
                        x -= std::ldexp(qd, kWindowBits * ww);
                        q = (int)qd;
                    }
                    return q;
                };
                while (ea < eae || eb < ebe) {
                    const int ka = ea < eae ? col[ea] : INT_MAX, kb = eb < ebe ? col[eb] : INT_MAX, k = std::min(ka, kb);
                    Entry x{k, {0, 0}};
                    if (ka == k) x.q[0] = digits_of(val[ea++]);
                    if (kb == k) x.q[1] = digits_of(val[eb++]);
                    if (W == 1 || x.q[0] || x.q[1]) list.push_back(x);
                }
                longest = std::max(longest, list.size());
            }
            const int S = digit_steps_of((int)longest);
            o.count[(size_t)quad * W + w] = (uint8_t)S;
            for (int pr = 0; pr < 4; ++pr) {
                    std::vector<Entry>& list = lists[pr];
                    o.step.resize((size_t)(steps + S) * kStepBytes, 0);
                    uint8_t* base = &o.step[(size_t)steps * kStepBytes];
                    std::stable_sort(list.begin(), list.end(), [](const Entry& a, const Entry& b) { return (a.k & 31) < (b.k & 31); });
                    for (int gam = 0; gam < 4 * S; ++gam) {         // a half wave's 32 rows of one gather
                        uint8_t* st = base + (size_t)(gam >> 2) * kStepBytes;
                        const int half = (gam >> 1) & 1, qq = gam & 1;
                        const int k_first = gam < (int)list.size() ? list[gam].k : 0;
                        for (int sl = 0; sl < 32; ++sl) {
                            const size_t e = (size_t)sl * 4 * S + gam;
                            const int g = 2 * half + (sl >> 4), i = sl & 15, tt = 16 * qq + i;
                            const Entry x = e < list.size() ? list[e] : Entry{k_first, {0, 0}};
                            uint16_t kk = (uint16_t)(bytes ? x.k * 8 : x.k);
                            std::memcpy(st + kStepRows + (16 * g + i) * 4 + 2 * qq, &kk, 2);
                            for (int hh = 0; hh < 2; ++hh) {
                                int q = x.q[hh];
                                for (int d = 0; d < 6; ++d) {
                                    const int dg = d == 5 ? q : ((q + 16) & 31) - 16;
                                    q = (q - dg) >> 5;
                                    const uint32_t m = (uint32_t)std::abs(dg);
                                    const uint32_t code = ((x.k & 1) == 0 ? m : m < 8 ? 2 * m : m + 8) | (dg < 0 ? 32u : 0u);
                                    const int frag = g * 12 + hh * 6 + d;
                                    for (int bit = 0; bit < 6; ++bit)
                                        if ((code >> bit) & 1u) {
                                            const int at = 6 * tt + bit;          // bit of the 192
                                            uint8_t* p = at < 128 ? st + frag * 16 + at / 8 : st + kStepA8 + frag * 8 + (at - 128) / 8;
                                            *p |= (uint8_t)(1u << (at & 7));
                                        }
                                }
                            }
                        }
                    }
                    steps += S;
            }
        }
    }
    o.first[tiles] = (int32_t)steps;
    o.step.resize((size_t)(steps + kStepPad) * kStepBytes, 0);
}

DigitSteps built;

}  // namespace

// Builds, and returns the sizes; digit_steps_copy then copies the result out.
extern "C" void digit_steps_build(int N, int K, const int32_t* row_ptr, const int32_t* col, const float* val, long long sizes[3]) {
    built = DigitSteps();
    const size_t nnz = (size_t)row_ptr[N];
    build_digit_steps(N, std::vector<int32_t>(row_ptr, row_ptr + N + 1), std::vector<int32_t>(col, col + nnz), std::vector<float>(val, val + nnz),
                      K <= 8192, built);
    sizes[0] = built.first.back();
    sizes[1] = built.windows;
    sizes[2] = built.unit;
}
extern "C" void digit_steps_copy(int32_t* first, uint8_t* count, uint8_t* step, double* valsum) {
    std::copy(built.first.begin(), built.first.end(), first);
    std::copy(built.count.begin(), built.count.end(), count);
    std::copy(built.step.begin(), built.step.end(), step);
    std::copy(built.valsum.begin(), built.valsum.end(), valsum);
}

// GELU and the quantizer of its output as one table of steps, built on the host from the pinned arithmetic itself.
//
// The code of GELU(x) is a step function of x: it falls by one at some points left of GELU's minimum and rises by one at others
// right of it (300 steps for 8 bits on [-0.17, 0.8], 18 for 4 bits).  The line is cut into equal entries of at most one step
// each; an entry holds the code on the high side of its step and a multiplier and an addend whose fused multiply-add with x is
// negative exactly on the low side.  So a code is an index, one 8-byte read, one fused multiply-add and a subtraction of
// its sign, where the piecewise cubic takes sixteen bytes and twice the instructions, and the bits are the same: the steps are
// found by evaluating the pinned sequence, a fused multiply-add never rounds across zero, and the host computes the index with the
// operations of the kernel.
//
// The pinned sequence is correctly rounded nearly everywhere, hence monotone between its minimum and the ends, but nothing forces
// it to be.  The builder walks the neighbours of every step until the value is further from the step than the roundings
// can carry it; where a code returns on the way (one of 80 000 steps of 400 random quantizers), where a step lies at the minimum
// itself, or where the steps are too close for the table (ranges narrower than about 0.5 at 8 bits) it gives up, and the
// caller keeps the cubic.
#pragma once
#include <math.h>
#include <stdint.h>
#include <string.h>
#include <algorithm>
#include <vector>

namespace mixaq {

constexpr int GELU_STEP_PIECES = 13;                                // of 1 KB, 128 entries each: five workgroups of the token kernel at C = 96 fit a CU, and more (see there)
constexpr int GELU_STEP_MAX = GELU_STEP_PIECES * 128;
constexpr float GELU_STEP_MAGIC = 0x1.8p23f;                          // adding it rounds to an integer, ties to even
constexpr int GELU_STEP_MASK = 0x3ff8;                              // byte offset of an entry in the low bits of the index sum
static_assert(GELU_STEP_MAX * 8 <= GELU_STEP_MASK + 8, "the mask holds every entry");

// How a kernel finds the entry of x: byte offset = GELU_STEP_MASK & bits(fma(clamp01(fma(x, scale, offset)), span, 1.5 * 2^23))
struct GeluIndex { float scale, offset, span; };
// The entry: value = fma(x, factor, addend); code + 128 = low byte of factor, less one where value is negative
struct GeluStep { float addend, factor; };

class GeluSteps {
public:
    GeluIndex index = {0.0f, 0.0f, 0.0f};
    std::vector<GeluStep> table;                                    // whole 1 KB pieces

    // cubic: the coefficient table of the pinned GELU, `intervals` of four, on arguments and results scaled by `intervals / 6`;
    // the quantizer as the kernels hold it: code = clamp(fma(value, inv_s, magic), lo, hi) - 1.5 * 2^23
    bool build(const float* cubic, int intervals, float inv_s, float magic, float lo, float hi)
    {
        if (!(inv_s > 0x1p-30f && inv_s < 0x1p30f)) return false;
        cubic_ = cubic; intervals_ = intervals; inv_s_ = inv_s; magic_ = magic; lo_ = lo; hi_ = hi;
        table.clear();
        steps_.clear();
        const float lowest = -0.7517915f * (float)intervals / 6.0f;  // GELU's minimum
        float top = (float)intervals;
        const int last = (int)(hi - GELU_STEP_MAGIC);
        while (code(top) != last && top < 0x1p60f) top *= 2.0f;
        if (!walk(-(float)intervals, lowest, -1) || !walk(lowest, top, 1)) return false;
        return lay_out();
    }
    // the code by the pinned sequence
    int code(float x) const { return code_of(gelu(x)); }
    // the code by the table, with the operations of the kernel
    int looked_up(float x) const
    {
        const GeluStep& e = table[entry_of(x)];
        int bits;
        memcpy(&bits, &e.factor, 4);
        return (bits & 0xff) - 128 - (fmaf(x, e.factor, e.addend) < 0.0f ? 1 : 0);
    }
    int entry_of(float x) const
    {
        const float u = std::min(std::max(fmaf(x, index.scale, index.offset), 0.0f), 1.0f), t = fmaf(u, index.span, GELU_STEP_MAGIC);
        int bits;
        memcpy(&bits, &t, 4);
        return (bits & GELU_STEP_MASK) >> 3;
    }

private:
    struct Step { float before, after; int code_before, code_after; };   // neighbouring numbers and their codes
    const float* cubic_ = nullptr;
    int intervals_ = 0;
    float inv_s_ = 0, magic_ = 0, lo_ = 0, hi_ = 0;
    std::vector<Step> steps_;

    float gelu(float x) const
    {
        const float u = std::min(fabsf(x), (float)intervals_ * 0x1.fffffep-1f);
        const int i = (int)u;
        const float d = u - (float)i, *c = cubic_ + 4 * i;
        return std::max(x, 0.0f) - fmaf(fmaf(fmaf(c[3], d, c[2]), d, c[1]), d, c[0]);
    }
    // binary32 numbers in order as integers
    static int64_t order_of(float v)
    {
        int32_t b;
        memcpy(&b, &v, 4);
        return b < 0 ? -(int64_t)(b & 0x7fffffff) : b;
    }
    static float number_at(int64_t o)
    {
        const int32_t b = o < 0 ? (int32_t)(0x80000000u | (uint32_t)-o) : (int32_t)o;
        float v;
        memcpy(&v, &b, 4);
        return v;
    }
    int code_of(float g) const { return (int)(std::min(std::max(fmaf(g, inv_s_, magic_), lo_), hi_) - GELU_STEP_MAGIC); }
    double value_of(float g) const { return (double)g * (double)inv_s_ + ((double)magic_ - (double)GELU_STEP_MAGIC); }   // before rounding
    // The steps of a monotone run from x0 to x1, codes changing by `by` at each.  A step is looked for where the two before it and two secant
    // steps put it, a few numbers off.  (A search that starts over at each step, and a walk that evaluates each neighbour twice, took 52
    // evaluations a step instead of 25: 8 bits on [-0.17, 0.8] 185 -> 120 us.)
    bool walk(float x0, float x1, int by)
    {
        int64_t at = order_of(x0);
        const int64_t end = order_of(x1);
        const int last = code(x1);
        int now = code(x0);
        auto passed = [&](int64_t o) { return (code(number_at(o)) - now) * by > 0; };
        if ((last - now) * by < 0) return false;
        double pitch = 0.0;                                          // from the last step to the one before
        while (now != last) {
            int64_t stride = 1 << 16, far = std::min(at + stride, end);
            if (pitch > 0.0) {
                double x = (double)number_at(at) + pitch;
                for (int k = 0; k < 2; ++k) x += (now + 0.5 * by - value_of(gelu((float)x))) * by * pitch;
                if (x > number_at(at) && x < x1) { far = std::max(order_of((float)x), at + 1); stride = 4; }
            }
            if (passed(far)) {                                       // gallop: `at` has not passed, nor do the numbers before it count
                int64_t low = far - stride;
                while (low > at && passed(low)) { far = low; stride *= 2; low = far - stride; }
                at = std::max(at, low);
            } else {
                while (!passed(far)) { at = far; far = std::min(far + stride, end); stride *= 2; }
            }
            while (far - at > 1) {                                   // then bisect
                const int64_t mid = at + (far - at) / 2;
                if (passed(mid)) far = mid; else at = mid;
            }
            if (code(number_at(far)) != now + by || !clear(at, now, -1) || !clear(far, now + by, 1)) return false;
            pitch = steps_.empty() || steps_.back().code_after - steps_.back().code_before != by ? 0.0 : (double)number_at(far) - steps_.back().after;
            steps_.push_back({number_at(at), number_at(far), now, now + by});
            now += by;
            at = far;
        }
        return true;
    }
    // Whether the numbers from o on in direction `dir` keep the code until their value is out of the reach of the roundings: 2^-21 of the
    // value, some eight units of its last place, against at most four (the three fused multiply-adds, the difference, and the jump of
    // rounded coefficients between two intervals).
    bool clear(int64_t o, int expected, int dir) const
    {
        for (int n = 0; n < 1024; ++n, o += dir) {
            const float g = gelu(number_at(o));
            if (code_of(g) != expected) return false;
            const double v = value_of(g) - (double)expected;         // distance from the code's middle
            if (n > 0 && 0.5 - fabs(v) > 0x1p-21 * fabs((double)g) * (double)inv_s_) return true;
            if (fabs(v) > 0.5 && (expected == (int)(lo_ - GELU_STEP_MAGIC) || expected == (int)(hi_ - GELU_STEP_MAGIC))) return true;                 // saturated: nothing beyond
        }
        return false;
    }
    bool lay_out()
    {
        const int n = (int)steps_.size();
        double gap = 1.0;                                            // no steps, or one
        for (int k = 1; k < n; ++k) gap = k == 1 ? (double)steps_[1].before - steps_[0].after : std::min(gap, (double)steps_[k].before - steps_[k - 1].after);
        const double from = n ? steps_.front().before : 0.0, to = n ? steps_.back().after : 0.0, width = 0.98 * gap;
        if (!(width > 0.0) || !((to - from) / width < GELU_STEP_MAX - 4)) return false;
        const int spans = (int)ceil((to - from) / width) + 3;        // an entry without a step at either end
        const double start = from - 1.5 * width;
        index.scale = (float)(1.0 / (spans * width));
        index.offset = (float)(-start / (spans * width));
        index.span = 8.0f * (float)spans;
        const int entries = spans + 1;
        table.assign((entries + 127) / 128 * 128, GeluStep{0.0f, 0.0f});
        std::vector<char> taken(entries, 0);
        int next = 0, now = code(-(float)intervals_);
        for (const Step& s : steps_) {
            const int first = entry_of(s.before), past = entry_of(s.after);
            if (first < next - 1 || first < 1 || past >= entries - 1) return false;
            for (; next < first; ++next) table[next] = flat(now, next == 0);
            GeluStep e;
            if (!step(s, &e)) return false;
            for (int i = first; i <= past; ++i) {
                if (taken[i]) return false;
                taken[i] = 1;
                table[i] = e;
            }
            next = past + 1;
            now = s.code_after;
        }
        for (; next < entries; ++next) table[next] = flat(now, next == 0);
        return true;
    }
    static float factor_of(int code, int upper, float sign)          // a number from 1 to 2 whose low byte is the code + 128
    {
        return sign * (1.0f + (float)(upper * 256 + code + 128) * 0x1p-23f);
    }
    // never negative, whatever x the entry may see: the first one has no lower end
    static GeluStep flat(int code, bool first) { return {0x1p100f, factor_of(code, 0, first ? -1.0f : 1.0f)}; }
    static bool step(const Step& s, GeluStep* e)
    {
        const bool rising = s.code_after > s.code_before;
        const float low = rising ? s.before : s.after, high = rising ? s.after : s.before;   // neighbours: value < 0 at low, >= 0 at high
        for (int upper = 0; upper < 0x8000; upper += 0x2000) {       // the product may reach the next binade, whose numbers are too far apart
            e->factor = factor_of(std::max(s.code_before, s.code_after), upper, rising ? 1.0f : -1.0f);
            const double at = -(double)e->factor * (double)high;     // exact; the least number that is no less
            e->addend = (float)at;
            if ((double)e->addend < at) e->addend = number_at(order_of(e->addend) + 1);
            if (fmaf(high, e->factor, e->addend) >= 0.0f && fmaf(low, e->factor, e->addend) < 0.0f) return true;
        }
        return false;
    }
};

}  // namespace mixaq

// The plan of a sort by digit passes (radix.hip): which passes run, and through
// which buffers, from what the first count and the sample found.  Plain
// functions, made by one thread on the device; the tests run them on the host.
#pragma once
#include <stdint.h>

namespace hvms {

constexpr int SAMPLE_LEN = 8192;  // elements of a run of the sample

// buffers of a sort; the steps alternate between them
enum { B_IN = 0, B_A = 1, B_B = 2, B_OUT = 3 };
enum { STEP_SKIP = 0, STEP_SCATTER = 1, STEP_COPY = 2, STEP_REVERSE = 3 };

struct Step {
    uint32_t mode, src, dst, first, last;
};

struct Ctl {
    Step step[2][8];  // of the first round and of the second (see radix_finish)
    uint32_t drop;    // low digits the first round left out and radix_finish orders
    uint32_t groups;  // groups listed by radix_finish
    uint32_t again;   // set: these could not order them, the second round sorts
};

// What the first count says about the input's order (flag set = not so).
enum { NOT_ASCENDING = 1, NOT_DESCENDING = 2, VALUES_NOT_ASCENDING = 4 };

// What the first count and the sample found.
struct Found {
    uint32_t flags;
    uint32_t var0, var1;  // bits that differ between two elements: low word, high word
    // smallest difference (xor, minus 1) between an element and the one after it in
    // the input, over those that differ in the low word only, and in the high word
    uint32_t near0, near1;
    // [d < 7]: sampled neighbours that first differ in digit d; [7]: sampled
    // elements equal to the one after next
    const uint32_t *same;
    int runs;             // of the sample; 0: none was taken
    int64_t n;
};

// Whether the plan asks how many low digits can be left out: not for presorted
// input, and not for pairs that skip their value digits (the keys' four are
// too few to leave out two of them at the sizes of a sample).
__host__ __device__ inline bool sample_matters(uint32_t flags, bool keys64)
{
    return (flags & NOT_ASCENDING) && (flags & NOT_DESCENDING) &&
           (keys64 || (flags & VALUES_NOT_ASCENDING));
}

// The steps of one round: modes by pass, and the buffers they go through.
__host__ __device__ inline void set_steps(Step *step, const uint32_t *mode, int passes, bool keys64)
{
    int steps = 0, j = 0;
    for (int p = 0; p < passes; ++p)
        steps += mode[p] != STEP_SKIP;
    uint32_t cur = B_IN;
    for (int p = 0; p < passes; ++p) {
        Step s{mode[p], 0, 0, 0, 0};
        if (mode[p] != STEP_SKIP) {
            s.first = j == 0;
            s.last = j == steps - 1;
            s.src = cur;
            if (s.last)
                s.dst = B_OUT;
            else if (keys64)
                s.dst = (j & 1) ? B_B : B_A;
            else
                s.dst = ((steps - 1 - j) & 1) ? B_A : B_OUT;
            cur = s.dst;
            ++j;
        }
        step[p] = s;
    }
}

// Passes over the digits in `need`.  In place, the first step must not write
// the array it reads: where the count of steps would make it, a pass that is
// not needed copies instead.
__host__ __device__ inline void scatter_modes(uint32_t *mode, uint32_t need, int passes,
                                              bool keys64, bool inplace)
{
    int steps = 0;
    for (int p = 0; p < passes; ++p) {
        mode[p] = (need >> p) & 1 ? STEP_SCATTER : STEP_SKIP;
        steps += (int)((need >> p) & 1);
    }
    if (inplace && (keys64 ? steps == 1 : (steps & 1) != 0))
        for (int p = 0; p < passes; ++p)
            if (mode[p] == STEP_SKIP) {
                mode[p] = STEP_COPY;
                break;
            }
}

// The low digits the first round leaves out, out of those in `need`: the most
// without which the sample leaves an element alike with at most `most` other
// ones on average, half a one up to 2^26 elements, one at 2^27, two from 2^28 on
// (less often another pass, a longer finish).  m elements in groups of g are
// m g / n of that, so one group of more than GROUP_MAX elements is over the line
// up to 1.9e8, and groups that fill the list (longer than half a window) are
// GROUPS_MAX * 33^2 / n of it or more.  Pairs of mixture keys and random values,
// whose one key in 55 is the largest, with all eight passes and with six (about
// 9,000 listed groups at 2^27, 65,000 at 2^28): 10^8 4.20 and 3.67 ms, 2^27 5.62
// and 4.97, 2.4e8 10.6 and 9.3, 2^28 11.8 and 10.4.
//
// The highest digit of `need` stays: where nearly all elements are equal, no
// sampled neighbours differ in it, but a round without a step would never
// write the output.
//
// A sample does not see the few elements that differ from a heavy value by low
// digits only, and one of them sends all the value's equals to the second
// round.  So where one sampled element in 2,048 stands third or later among its
// equals, no digit is left out that tells two neighbours of the input apart,
// which a heavy value and its like are somewhere in an unordered input.
__host__ __device__ inline uint32_t digits_to_drop(const Found &f, uint32_t need)
{
    const double pairs = 0.5 * f.runs * SAMPLE_LEN * SAMPLE_LEN;
    const double part = (double)f.n / 134217728.0;
    const double most = part <= 0.5 ? 0.5 : part <= 2.0 ? part : 2.0;
    uint32_t limit = 7;
    if ((double)f.same[7] * 2048.0 >= (double)f.runs * SAMPLE_LEN)
        limit = f.near0 != ~0u   ? (31 - __builtin_clz(f.near0 + 1)) >> 3
                : f.near1 != ~0u ? 4 + ((31 - __builtin_clz(f.near1 + 1)) >> 3)
                                 : 0;
    uint32_t alike = 0, drop = 0;
    for (uint32_t d = 1; d <= limit && need >> d; ++d) {
        alike += f.same[d - 1];
        if ((double)alike * (double)f.n <= most * pairs)
            drop = d;
    }
    return __builtin_popcount(need & ((1u << drop) - 1)) >= 2 ? drop : 0;
}

// The steps of the sort.
__host__ __device__ inline void plan_sort(const Found &f, int passes, bool two, bool keys64,
                                          bool inplace, Ctl *ctl)
{
    uint32_t mode[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    ctl->drop = 0;
    ctl->groups = 0;
    ctl->again = 0;
    if (!(f.flags & NOT_ASCENDING)) {
        mode[passes - 1] = STEP_COPY;
    } else if (!(f.flags & NOT_DESCENDING)) {
        mode[passes - 1] = STEP_REVERSE;
        if (inplace) {  // through the scratch, since both ends move
            mode[passes - 2] = STEP_REVERSE;
            mode[passes - 1] = STEP_COPY;
        }
    } else {
        uint32_t need = 0;
        for (int p = 0; p < passes; ++p) {
            const uint32_t var = (two && p < 4) ? f.var0 : f.var1;
            if ((var >> (8 * (p & 3))) & 255)
                need |= 1u << p;
        }
        if (two && !keys64 && !(f.flags & VALUES_NOT_ASCENDING))
            need &= 0xf0;
        if (f.runs && sample_matters(f.flags, keys64)) {
            ctl->drop = digits_to_drop(f, need);
            if (ctl->drop) {
                scatter_modes(mode, need, passes, keys64, true);
                set_steps(ctl->step[1], mode, passes, keys64);
                need &= ~((1u << ctl->drop) - 1);
            }
        }
        scatter_modes(mode, need, passes, keys64, inplace);
    }
    set_steps(ctl->step[0], mode, passes, keys64);
}

}  // namespace hvms

// Which kernel a call runs on, by the schedule and width of its rows, what it asks for and its size -- never by what is in
// the tensors or where they lie (but for outputs that lie over inputs: takes_few_backward).  No GPU call and no HIP header: wht_affine.hip takes its launches from here, and
// route_query.cpp, which a host compiler builds, tells the tests which kernel a size reaches.
//
// Sizes are bytes of one [N, d] tensor.  The figures beside the rules are us per call under graph replay, in three settings:
//   again   three sets of inputs and two of outputs in turn, which stay in the Infinity Cache while they are small;
//   inputs  inputs from memory, two sets of outputs in turn: what a program sees whose allocator hands buffers back;
//   memory  inputs and outputs all from memory.
#pragma once
#include <stdint.h>

namespace wht {

enum class Sched { Matrix, Wave, Twelve };

// n: log2 d, or m for rows of 12 * 2^m; bytes: of an element.
struct Rows { Sched sched; int n; int bytes; };
constexpr int row_length(Rows rows) { return rows.sched == Sched::Twelve ? 12 << rows.n : 1 << rows.n; }

// ---- forward -------------------------------------------------------------------------------------------------------------------

// What a forward call returns: y, y with the residual added, that and the norm statistic.
enum class Out { Y, Resid, Stats };

// Few tokens (decoding, short prefills): one token group per workgroup and no token loop (forward_once_kernel), with plain
// stores (Plain), with stores through L2 (Through), and with two token groups per workgroup and stores through L2 (Pair): both
// are requested at once, and alpha and beta, two to four times as many bytes as a thread's part of x, are read half as often.
// Then the persistent kernel (forward_kernel), with y streamed past the caches (Stream) or through L2 (Flow).
// The kernels do the same arithmetic on a token in the same order, so the switches are invisible in y
// (the norm statistic is summed in the order of the launch shape: its last bits may differ).
enum class Way { Plain, Through, Pair, Stream, Flow };

struct Step { double mib; Way way; };       // from this many MiB on
struct Route { Step step[8]; };             // ends with the first step of 0 MiB behind the first one

// The sizes were set by a sweep of every width from 1 to 256 MiB in the three settings: a way is taken where it is faster in them together
// and not slower than the others by more than the runs differ (2 %) in the first.  us per call, again / memory unless more are named:
//   plain against through: 4097 x 1024 4.53 / 5.41 and 4.02 / 5.04, 1024 x 4096 4.68 / 5.66 and 3.74 / 4.75, 16385 x 256 4.36 / 5.46
//     and 3.62 / 5.53; one token of 4096 with the statistic 2.65 and 2.77 (the kernel ends when memory, not L2, has the results); with the
//     statistic 7 MiB of 2048 wide 5.9 / 7.8 and 6.0 / 8.5, 16 MiB 9.0 / 13.6 and 9.1 / 14.7, 30 MiB of float32 2048 15.8 / 21.1 and 16.4 / 22.6, 12 MiB of
//     float32 64 wide 6.7 / 9.0 and 7.0 / 9.0 (so plain there);
//   one group against two, 2048 wide: 1025 tokens 3.05 / 3.86 and 3.03 / 3.76, 4097 6.9 / 9.8 and 6.3 / 8.0; 8 MiB of 1536 wide
//     7.0 / 7.7 and 5.6 / 6.3, of 12288 wide 10.6 / 11.4 and 7.9 / 8.8 (there the persistent kernel took over from 2^22 elements on);
//     below, half the workgroups leave CUs idle: 1 MiB of 2048 wide 2.8 and 3.2; with the statistic 3 MiB of
//     3072 wide 4.7 and 4.9, 13 to 18 MiB of 12288 +6 (one group -7);
//   one pass against persistent: 25 to 48 MiB of 1024 wide 12 to 18 % less again, 13 to 16 less from memory up to 32 MiB, 2 to 3 more beyond; 32 MiB of 256 wide (bfloat16) 11.1 / 14.4
//     and 13.4 / 14.4, of 2048 11.4 / 18.0 and 13.1 / 15.3 (so 24 there), 8 MiB of 16384 6.0 / 8.6 and 9.9 / 10.8, 32 MiB of 1536 14.2 / 15.3 and 11.5 / 13.5; with the
//     residual 25 MiB of 1024 12.5 / 14.6 and 14.6 / 14.7, 29 of 2048 14.8 / 19.1 and 17.5 / 17.5; with the statistic 20 MiB of 1536 +2 / +12 / inputs +9 %, 25 MiB of 12288 +11;
//     without either 14 MiB of 6144 +6, 20 MiB of float32 2048, plain 9.3 / 11.4, through 8.7 / 11.9, persistent 8.0 / 8.9 (inputs 9.9, 10.5 and 9.0), 30 MiB 11.6 /
//     15.0, 10.6 / 16.0 and 12.5 / 13.9 (inputs 12.3, 14.9 and 13.8);
//   y of the persistent kernel through L2, where it is not as in dx_through: 24 to 32 MiB of 4096 wide +1..+8 / +4..+8 / inputs +1, 40 and more -3 / +6 / -5; with
//     the statistic 56 to 134 MiB of 16384 +1..+4 in all three, 60 MiB of float32 8192 +3 / +4 / +2.
// Rows of 12 * 2^m elements have workgroups of one token (two of 768): workgroups of 256 threads, with up to eight tokens,
// leave CUs without any, and from 257 of them on put two on one CU beside others with one (341 x 768 3.33 / 2.34, 1365 x
// 1536 5.60 / 4.80, 683 x 3072 6.01 / 4.83).
// Stream and Flow: see dx_through.  Where a workgroup of the persistent forward kernel has few rounds, each waits for the stores
// of the one before it, and those come back from memory, not L2: forward of 16 MiB of 8192 wide 8.6 / 9.3, of 32 MiB of 16384
// wide 17.0 / 18.0.  Rows of 12 * 2^m whose x is kept (forward_keeps) are streamed: through L2, y and dx would push x out before
// the backward call reads it.
constexpr Route forward_route(Rows rows, Out out) {
    constexpr Way P = Way::Plain, T = Way::Through, R = Way::Pair, S = Way::Stream, F = Way::Flow;
    const bool resid = out != Out::Y, stats = out == Out::Stats;
    const double through = stats ? 2.5 : 1;
    if (rows.sched == Sched::Twelve) {
        const double keep = !resid ? 80 : rows.n <= 8 ? 48 : 56;
        switch (rows.n) {
        case 6:  return {{{0, P}, {through, T}, {resid ? 5.0 : 7.0, R}, {22, S}, {keep, F}, {136, S}}};
        case 7:  return {{{0, P}, {resid ? 3.5 : 2.5, R}, {stats ? 19.0 : resid ? 22.0 : 17.0, S}, {keep, F}, {136, S}}};
        case 8:  return {{{0, P}, {through, T}, {stats ? 4.0 : 2.0, R}, {resid ? 14.0 : 17.0, S}, {keep, F}, {136, S}}};
        case 9:
            if (resid) return {{{0, P}, {3.5, R}, {stats ? 7.0 : 12.0, S}, {keep, F}, {136, S}}};
            return {{{0, P}, {1, T}, {3.5, R}, {13, S}, {15, R}, {18.5, S}, {keep, F}, {136, S}}};
        default:
            if (stats) return {{{0, P}, {4, T}, {7, R}, {13, T}, {19, R}, {25, S}, {keep, F}, {136, S}}};
            return {{{0, P}, {4, T}, {7, R}, {34, S}, {keep, F}, {136, S}}};
        }
    }
    if (rows.sched == Sched::Wave) {
        if (rows.bytes == 2) return {{{0, P}, {through, T}, {resid ? 33.0 : 48.0, F}, {136, S}}};
        if (rows.n <= 10) {
            if (stats) return {{{0, P}, {6, T}, {rows.n <= 6 ? 9.0 : 13.0, P}, {33, F}, {136, S}}};
            return {{{0, P}, {resid ? 6.0 : 1.0, T}, {resid ? 33.0 : 48.0, F}, {136, S}}};
        }
        if (rows.n == 11) {
            if (stats) return {{{0, P}, {through, T}, {25, P}, {33, F}, {136, S}}};
            if (resid) return {{{0, P}, {through, T}, {33, F}, {136, S}}};
            return {{{0, P}, {1, T}, {13, S}, {25, P}, {33, F}, {136, S}}};     // 3072 tokens: 12 to a CU
        }
        if (rows.n == 12) return {{{0, P}, {stats ? 3.5 : through, T}, {17, S}, {24, F}, {136, S}}};
        if (stats) return {{{0, P}, {2.5, T}, {6, P}, {8, T}, {17, S}, {80, F}, {136, S}}};
        return {{{0, P}, {2, T}, {resid ? 17.0 : 9.0, S}, {56, F}, {136, S}}};
    }
    switch (rows.n) {
    case 10:
        if (stats) return {{{0, P}, {2.5, T}, {5.8, P}, {33, F}, {136, S}}};
        if (resid) return {{{0, P}, {1, T}, {33, F}, {136, S}}};
        return {{{0, P}, {1, T}, {2.5, R}, {12, T}, {48, F}, {136, S}}};
    case 11:
        if (stats) return {{{0, P}, {2.5, T}, {6, P}, {33, F}, {136, S}}};
        return {{{0, P}, {1, T}, {resid ? 7.0 : 3.5, R}, {resid ? 33.0 : 24.0, F}, {136, S}}};
    case 12:
        if (stats) return {{{0, P}, {2.5, T}, {7, R}, {8.1, S}, {40, F}, {136, S}}};
        return {{{0, P}, {1, T}, {resid ? 7.0 : 10.0, R}, {17, S}, {resid ? 24.0 : 46.0, F}, {136, S}}};
    case 13:
        if (resid) return {{{0, P}, {through, T}, {stats ? 7.0 : 6.0, P}, {8.1, S}, {56, F}, {136, S}}};
        return {{{0, P}, {1, T}, {13, S}, {56, F}, {136, S}}};
    default:
        if (stats) return {{{0, P}, {4, T}, {24, S}}};
        return {{{0, P}, {4, T}, {24, S}, {56, F}, {136, S}}};
    }
}

constexpr Way forward_way(Rows rows, Out out, int64_t bytes) {
    const Route r = forward_route(rows, out);
    int i = 0;
    while (i < 7 && r.step[i + 1].mib > 0 && (double)bytes >= r.step[i + 1].mib * (1 << 20)) ++i;
    return r.step[i].way;
}
// Whether some size takes this way: the others are not compiled.
constexpr bool forward_reaches(Rows rows, Out out, Way way) {
    const Route r = forward_route(rows, out);
    for (int i = 0; i < 8 && (i == 0 || r.step[i].mib > 0); ++i)
        if (r.step[i].way == way) return true;
    return false;
}

// Rows of 12 * 2^m: x of calls below this is read with the default cache policy, as these rows always have been, and streamed
// from there on.  What has been read with the default policy stays in the Infinity Cache: a backward call that
// follows its forward call finds x there, and a caller that comes back to the same small tensors finds them.
// us per call, kept and streamed y / streamed x and y through L2, again and memory:
//     forward     64 MiB of 768 22.0 / 23.5 and 26.2 / 23.6, 96 36.7 / 32.3 and 36.7 / 32.4, 128 47.6 / 41.5; 96 of 3072 38.4 / 34.1, of 12288 43.0 / 40.5;
//     residual    40 MiB of 768 21.6 / 22.5 and 25.8 / 22.6, 48 26.9 / 25.6 and 29.9 / 25.6, 128 72.3 / 60.2; 48 of 6144 27.8 / 28.8 and 30.6 / 29.4,
//                 64 39.4 / 35.1; 64 of 12288 41.8 / 39.7.
constexpr bool forward_keeps(int m, bool resid, int64_t bytes) {
    return bytes < (int64_t(!resid ? 80 : m <= 8 ? 48 : 56) << 20);
}

// ---- backward ------------------------------------------------------------------------------------------------------------------

// Rows of 12 * 2^m: x and dy of a backward call up to 32 MiB are read with the default cache policy, dy where dx is made alone
// up to 84 (dx_through).  The 32 MiB: backward, default policy / streamed, three sets of buffers in turn and inputs from memory (rows padded to
// 16 * 2^m, before: always default):
//     10923 x 768    16.0 / 17.9   18.1 / 18.4   (16.9, 18.0)        1365 x 6144    18.5 / 22.0   20.3 / 22.3   (19.4, 21.3)
//     21845 x 768    22.6 / 25.5   27.1 / 26.1   (24.9, 27.3)        2731 x 6144    27.0 / 29.4   28.9 / 30.1   (27.9, 29.2)
//     1365 x 3072    14.5 / 15.9   15.6 / 15.9   (15.0, 16.0)        1365 x 12288   37.6 / 40.6   37.5 / 40.9   (49.5, 50.8)
//     2731 x 3072    16.0 / 18.6   19.7 / 18.7   (20.2, 22.1)
//     32768 x 768    36.2 / 33.2   37.1 / 33.2   (38.7, 39.7)        4096 x 6144    41.0 / 36.8   41.3 / 36.8   (43.7, 44.0)
// So the default policy costs up to 5 % from memory at 768 and 3072 and gains more elsewhere; streamed, calls of 6144 and
// 768 would be slower than before.  The power-of-two rows have always been streamed and lose by a change.
constexpr bool backward_keeps(bool grads, int64_t bytes) { return bytes <= (int64_t(grads ? 32 : 84) << 20); }

// Whether dx goes through L2 (and y, in the table above) rather than being streamed past the caches ("nt").  Written through,
// results stay in the Infinity Cache: the next kernel finds them there, and a program that gets the same output buffers back
// overwrites them there.  But a kernel ends when memory has its results, and a workgroup's next round waits for the stores of the
// one before: short calls lose, and rows whose rounds are short.  Through against streamed, again / memory / inputs (a size is written through where
// the three together gain, or lose nothing):
//   backward: 32 to 256 wide rows 1 to 24 MiB +0..+7 % / +1..+7 / -1..+7, 36 to 136 -7..+1 / +0..+3 / -7..+1; float32 512 wide 2 to 8 MiB -6..-4 / -3..+2 / -3..+2, 8 to
//     18 +2..+3 / 0..+1 / +1..+3; other rows below 1 MiB +2 / +6 / +3 (4096 wide and more -2 / +2 / 0), from 1 or 2 MiB on -14..+1 / -6..+2 / -8..+1;
//   dx alone: below 2 MiB -3 / +7 / +4; rows of up to 128 bytes 3 and 4 MiB -8 / +5 / +2, 5 to 7 -10..-5 / +14..+20 / +10..+14, 8 and 9 -34..-20 / +2..+13 / -1..+13, 10 and
//     11 +1 / +4 / 0, 13 on -12..-1 / +1 / -12..-4; 128 to 512 wide bfloat16 3 to 8 MiB -13..-4 / +5 / +2, 9 -20 / +14 / +14, 10
//     and 11 -5..+18 / +8..+16 / +6..+19, float32 (64 to 512 wide) 2 to 8
//     -4 / +6 / +4, 9 and 10 -25 / +1..+10 / +3..+14, 10.6 and 11 +3 / +5 / +11, both 12 to 16 +6..+9 / +7..+9 / +8..+12, 24 on -11..+2 / +0..+4 / -12..-2; 1024 wide
//     bfloat16 2 to 4 MiB -7 / +3 / +1, 5 and 6 -7 / +20 / +13, 7 on -28..-3 / 0..+7 / -13..+5, float32 -8 / +12 / +14 at 9; 2048 to 8192 wide 3 to 10 MiB -13..-3 / +2..+6 / 0..+5,
//     11 to 24 -3..+6 / +1..+8 / -1..+7; bfloat16 4096 and 8192 wide 34 MiB +5..+7 / +7..+9 / +1..+2, 40 on -11..-1 / 0..+6 / -10..-3; float32 2048 and 8192 wide 24 to
//     40 MiB +1..+11 / +3..+11 / 0..+10; 16384 wide -6..+4 / -1..+4 / -2..+2, never together ahead;
//   above 136 MiB 0..+2 / 0..+4 / -8..-18 (dx alone, 150 to 256 MiB), a step of 16384 x 4096 float32 231 / 236 us, backward of 32768 x 8192 276 / 281: streamed.
// Rows of 12 * 2^m: with the sums, where x and dy are kept always; above, up to 136 MiB but for 56 to 80 MiB, where x, y, dy
// and dx of a step just fill the Infinity Cache, and for m = 10: streamed / through, us, backward and a step: 48 MiB of 768 32.6 / 31.4 and
// 48.6 / 48.7 (from memory 50.2 / 49.4), 64 41.6 / 39.4 and 62.9 / 63.5, 128 73.8 / 67.9 and 112.2 / 110.6; 48 of 6144 36.2 / 34.8 and 54.7 / 53.9,
// 128 of 1536 75.0 / 68.5 and 121.6 / 111.3; 48 of 12288 47.1 / 44.1 and 67.5 / 69.6.  dx alone on a dy that is kept: 1 to 46 MiB -7..0 / -3..+11 / -8..+3, above
// +5..+18 / +0..+6 / -9..-3 (75 MiB of 768 24.0 / 28.1 us); on a streamed one, 84 to 128 MiB, against kept and streamed -14..0 / -3..+1 / -14..-5.
constexpr bool dx_through(Rows rows, bool grads, int64_t bytes) {
    constexpr int64_t MiB = 1 << 20;
    const int row = row_length(rows);
    if (bytes > 136 * MiB) return false;
    if (rows.sched == Sched::Twelve) {
        if (grads) return backward_keeps(true, bytes) || (rows.n < 10 && (bytes < 56 * MiB || bytes >= 80 * MiB));
        return bytes < 46 * MiB || !backward_keeps(false, bytes);
    }
    if (grads) {
        if (row <= 256) return bytes >= 36 * MiB;
        if (rows.bytes == 4 && row == 512) return bytes >= 2 * MiB && (bytes < 8 * MiB || bytes >= 18 * MiB);
        return row >= 4096 || bytes >= (rows.bytes == 4 && row == 1024 ? 2 : 1) * MiB;
    }
    const double mib = (double)bytes / MiB;
    if (row == 16384) return false;
    if (row * rows.bytes <= 128) return (mib >= 2.5 && mib < 4.2) || mib >= 7.9;
    if (rows.sched == Sched::Matrix && row == 1024) return (mib >= 2 && mib < 4.2) || mib >= 6.3;
    if (rows.bytes == 4 && row <= 1024) return (row < 1024 && mib >= 8.3 && mib < 10.3) || mib >= 24;
    if (row <= 512) return (mib >= 2.5 && mib < 9.5) || mib >= 24;
    const double again = rows.bytes == 4 ? (row == 2048 ? 56 : row == 4096 ? 24 : 46) : row == 2048 ? 24 : 40;
    const bool wide_f32 = rows.bytes == 4 && row != 4096;
    return (mib >= (wide_f32 ? 4 : 2.5) && mib < (rows.bytes == 4 && row == 4096 ? 12 : 10.4)) || mib >= again;
}

// How the rows of partial sums are written.  Every workgroup writes its row at the end of the kernel, and rows that lie
// dirty in L2 are written back before the next kernel adds them up; written through L2 they are on their way at once and
// wait in the Infinity Cache.  Short rows gain nothing by that, and where dx is streamed beside them they lose; 512 workgroups with rows of
// 32 KiB (float32 4096 wide) are fastest when nothing is kept.  Parameters alone, plain or (2048 to 4096 columns) streamed / through, 1 to 16 MiB:
// 128 columns -1 %, 256 -2..-5, 512 -5..-12, 1024 -4..-12, 1536 -5..-15, 2048 -4..-12, 4096 of bfloat16 0..-12, 6144 -7..-11, 16384 -2..-11; float32
// 4096 0..-6 up to 8 MiB, +2..+3 from 12 on (20 MiB 20.1 / 22.2 us).  With dx, 32 to 128 columns +1..+4 %, 256 +0..+3, 512 and more -1..-9.
enum class Store { Plain, Stream, Through };
constexpr Store sums_store(Rows rows, bool dx) {
    const int row = row_length(rows);
    if (row <= 128 || (dx && row <= 256)) return Store::Plain;
    return rows.bytes == 4 && row == 4096 && !dx ? Store::Stream : Store::Through;
}

// A call of few elements runs on backward_few_kernel: no partial rows and no second launch, which cost the stream 2.5 us and
// the host 3.3, and a workgroup for every 64 columns where a launch of one workgroup has a single one.  Rows must have 8 slices of 64
// columns (float32: 4).  Its workgroups read x, dy and alpha while others write dx, dalpha and dbeta: takes_few_backward.
// us per call under graph replay, before / this kernel, backward: 1 x 512 3.8 / 2.2, 64 x 512 6.1 / 3.4, 64 x 1024 5.7 / 3.9 (91: 5.8 /
// 5.9), 60 x 1536 7.5 / 4.6 (85: 7.6 / 7.1), 16 x 4096 6.3 / 3.1, 32 6.3 / 4.3 (45: 6.4 / 5.5, from memory 6.9 / 7.2), 16 x 8192 6.7 / 4.4 (23: 6.8 / 5.3,
// from memory 7.2 / 6.8), 12 x 16384 12.0 / 9.4 (16: 12.1 / 10.5), 64 x 768 6.5 / 3.9 (121: 6.5 / 6.0), 16 x 12288 12.2 / 5.8; float32
// 64 x 512 6.3 / 3.7 (128: 6.4 / 5.6), 64 x 1024 6.1 / 4.5, 32 x 2048 8.0 / 4.0 (64: 8.0 / 6.1), 12 x 8192 8.9 / 5.1 (16: 9.0 / 6.0).
constexpr bool has_few_backward(Rows rows) { return row_length(rows) % 64 == 0 && row_length(rows) / 64 >= 16 / rows.bytes; }
constexpr int64_t few_backward_elements(Rows rows) {
    const int row = row_length(rows);
    if (!has_few_backward(rows)) return 0;
    if (rows.bytes == 4) return row <= 512 ? 3 << 14 : row == 1024 ? 1 << 16 : 3 << 15;
    return row <= 1024 ? 1 << 16 : row < 2048 ? 3 << 15 : row < 12288 ? 1 << 17 : 3 << 16;
}

// Other calls of up to this many token groups run on one workgroup, which writes dalpha and dbeta itself: no partial rows and no
// second launch.  The groups then run one after the other; up to here that is no slower (us per call, two launches / one: 3 groups
// at d = 256 6.0 / 5.7, at d = 1024 6.1 / 4.9, at float32 d = 1024 6.6 / 6.4; 2 groups at d = 4096 7.6 / 6.5, at d = 8192 6.6 / 5.4; 1 at d =
// 16384 11.0 / 8.1 and at float32 d = 4096 7.7 / 5.2, where 2 already are 11.1 / 12.3 and 7.7 / 8.3; 2 at d = 768 5.8 (3: 6.6 / 7.1), 1 at d =
// 12288 9.1 (2: 11.4 / 12.2)).
constexpr int64_t one_workgroup_groups(Rows rows) {
    const int row = row_length(rows);
    return row >= 12288 ? 1 : row <= 1024 && rows.sched != Sched::Twelve ? 3 : rows.sched != Sched::Wave ? 2 : 1;
}

// Whether a backward call with parameter gradients runs on backward_few_kernel.  With dalpha or dbeta over alpha it cannot.  With dx
// over dy or x, dx is a launch of its own behind the sums, although one workgroup would be faster for the first token groups (us per call,
// one workgroup / sums and dx: 4 x 1024 3.4 / 5.0, 8 x 512 3.8 / 5.2, 2 x 4096 4.3 / 5.8, 4 x 768 4.0 / 5.9; faster from 8 x 4096, 12 x 2048 and 2 x 16384 on):
// dalpha and dbeta are then added in the order of a call on buffers of its own, and in place or not the results are the same bits.
constexpr bool takes_few_backward(Rows rows, int64_t N, bool over_alpha) {
    return !over_alpha && N * row_length(rows) <= few_backward_elements(rows);
}

// Rows of 768: a backward call of up to this many tokens has workgroups of 128 threads (four tokens), so that twice as many share it.
// us per call under graph replay, 256 / 128 threads, inputs that come back: 341 7.00 / 6.63, 512 7.09 / 6.99, 683 7.26 /
// 7.31, 1365 8.22 / 9.87; dx alone 64 3.26 / 2.84, 512 3.33 / 2.95, 1365 3.51 / 3.77.
constexpr int64_t kSmallBackwardTokens = 512;

}  // namespace wht

// Which launches a call takes: where the statistics are put together, and, for the fused step over dense arenas, how the model
// is cut into pieces, once per slot, and what of them a call on a range of layers runs.  Arithmetic on the host only.
#ifndef DDP_PLAN_H
#define DDP_PLAN_H

#include <algorithm>

#include "ddp_internal.h"

namespace ddp {

// Whether the workgroups of a launch put the layers' statistics together themselves: `partials` of them have a pair of partial
// sums, at most `most` in one layer (counted in kFoldGroups groups of kFoldGroup).  That saves a launch (3 us of host time), but each
// of these workgroups waits for its pair and its counter to be where all XCDs see them before it ends.  Up to 5/4 workgroups per CU
// with a share, whatever the launch has besides.  Launch of their own / folded in us, 256 CUs, two layers (four at 396 and 513 pairs):
//                             back to back    waited for    behind other work
//     fused SGD, N = 4  128   8.19 /  7.74   20.9 / 20.3      8.4 /  8.1
//                       198  10.51 / 10.22   23.4 / 22.9     10.7 / 10.4
//                       352  15.19 / 14.22   27.6 / 26.7     15.2 / 14.4
//     average, N = 4    128   6.84 /  5.72   17.9 / 17.8      6.1 /  6.0
//                       256   6.75 /  5.53   17.5 / 17.4      5.9 /  5.9
//     average, N = 12   256   9.27 /  9.11   20.7 / 20.5      9.8 /  9.6
//                       352  11.03 / 11.27   23.1 / 23.1     11.4 / 11.5
//     average, N = 8    396   9.05 /  8.88   21.2 / 21.2      9.5 /  9.3
//                       513  10.98 / 11.41   22.5 / 22.9     11.8 / 12.2
// The line is drawn where the average crosses, and no layer has more than 256 CUs allow in all, whatever the device; the fused step, whose
// workgroups have more to do, still gains at 352 and has a line of its own.
inline bool folds(int cus, int64_t partials, int64_t most) { return 4 * partials <= 5 * (int64_t)cus && most <= 320; }
// Bytes that a thread of the fused step asks for with one vector of all streams.
inline int vector_bytes(int N, bool wire16, bool adamw, bool grad16) { return (wire16 ? 8 : 16) * (N - 1) + (adamw ? 48 : 32) + (grad16 ? 8 : 16); }

// The fused step, whose chunks are half the size (kSmallChunk), up to 5/2 per CU with a pair.  Launch of their own / folded in us:
//     8 layers, one of them scheduled, pairs      257             401             565             626
//         SGD, N = 4                         10.6 /  9.8     15.2 / 13.4     19.7 / 18.1     21.4 / 19.6
//         AdamW, N = 8                       14.8 / 13.7     20.5 / 18.8     28.0 / 26.1     30.6 / 28.8
//     4 layers, one of them scheduled
//         SGD, N = 4                          8.9 /  7.1     10.0 /  9.8     12.5 / 12.6     13.6 / 12.5
//         AdamW, N = 8                       10.4 / 10.5     14.0 / 14.3     18.2 / 18.0     18.8 / 17.1
//         SGD, N = 16                        10.4 / 10.4     13.8 / 14.1     19.6 / 20.2     19.0 / 18.6
// Where every chunk of the call has a pair, and the call asks for 24 MB and more, layers of up to 5/4 as above: the kernel hides the host's time of another
// launch, and a larger layer's counters make its workgroups wait longer.  In smaller calls that launch costs 2 us.  14 to 10 layers, layer by layer (MB a call):
//     all scheduled               14 x 640^2 (400 pairs)           12 x 700^2 (479)                10 x 760^2 (565)
//         SGD, N = 2                  (6.6) 117   /  93.1              (7.8) 102.7 /  85.5             (9.2)  81.7 /  77.5
//         SGD, N = 4                  (9.8) 118.2 /  99.3             (11.8) 104.1 /  92.7            (13.9)  81.8 /  85.3
//         SGD, N = 8                 (16.4) 111.8 / 115.3             (19.6) 113.8 / 109.2            (23.1)  97.3 / 104.1
//         AdamW, N = 8               (17.2) 126.2 / 130.0             (20.6) 120.7 / 125.2            (24.3) 115.3 / 121.4
//         AdamW, N = 16, bf16        (18.0) 145.8 / 150.2             (21.6) 139.1 / 147.0            (25.5) 134.3 / 141.5
//     a quarter or third
//         SGD, N = 4                  (9.8)  65.0 /  56.4             (11.8)  54.7 /  52.2            (13.9)  50.4 /  51.7
//         SGD, N = 8                 (16.4)  65.9 /  61.1             (19.6)  59.2 /  56.3            (23.1)  55.7 /  57.2
//         AdamW, N = 8               (17.2)  72.8 /  73.9             (20.6)  66.6 /  68.1            (24.3)  69.5 /  71.2
//     one
//         SGD, N = 8                 (16.4)  53.9 /  51.0             (19.6)  47.7 /  45.0            (23.1)  43.8 /  43.7
// and small models, all scheduled, AdamW, N = 8: 12 x 200^2 (480 pairs, 40 a layer, 20.2 MB) 9.2 / 7.4, 6 x 300^2 (528, 88) 8.8 / 8.4; 1 x 700^2 (479, 20.6 MB) 8.8 / 7.5.
inline bool folds_fused(int cus, int64_t partials, int64_t most, int64_t chunks, int64_t bytes) {
    const bool waits = 4 * most > 5 * (int64_t)cus && 2 * partials > chunks;
    return 2 * partials <= 5 * (int64_t)cus && !(waits && bytes >= 24'000'000) && most <= kFoldGroup * kFoldGroups;
}

// Where the average of N replicas cuts its chunks of `chunk` elements in two, a workgroup each (0: not).  The kernel for more than
// 16 replicas takes the halves of a chunk one after the other; cut, one workgroup asks while another adds.  Up to 16 replicas both
// halves are in flight together, and cutting spreads the sums of small slots over more CUs.  Not cut / cut in us:
//     fp32, slots of      131 K        262 K        524 K        720 K         2 M         7 M        34 M elements
//     N = 12            6.4 / 6.2    7.0 / 7.1   10.1 / 9.2   11.1 / 11.2             62.5 / 66.1
//     N = 16            6.9 / 6.5    8.4 / 8.3   12.4 / 10.8  13.6 / 13.5             81.6 / 81.5
//     N = 18                                                              31.7 / 33.3   96 / 96     424 / 424
//     N = 24           10.8 / 9.2   17.6 / 14.7  18.6 / 16.1  21.7 / 19.3  40.3 / 40.9  124 / 116   554 / 516
//     N = 32                                     22.3 / 17.1               49.0 / 48.2  155 / 150   729 / 694
//     four calls, bf16 N = 24                                              62.8 / 61.1  179 / 175   804 / 783
//     four calls, bf16 N = 32                                              68.0 / 65.0  197 / 191   894 / 873
// (N = 8: 131 K 5.8 / 5.5, 262 K 6.1 / 6.4; bf16, N = 12, waited for: 524 K 35.0 / 36.1).  A cut chunk has two pairs of partial sums,
// so slots whose pairs would not fit the fixed scratch are not cut, whichever scratch a call has: same bits from both.
inline int mean_cut(int cus, int64_t chunk, int64_t n_chunks, int64_t n_layers, int N, bool wire16) {
    if (N < (wire16 ? kCutReps16 : kCutReps) || N > 32) return 0;
    const bool cut = N <= 16 ? 4 * n_chunks <= 5 * (int64_t)cus
                             : wire16 || N == 32 || 2 * n_chunks <= 3 * (int64_t)cus || n_chunks >= 8 * (int64_t)cus;
    return cut && (2 * n_chunks + n_layers * kStatSlices) * 2 * (int64_t)sizeof(double) <= (int64_t)DDP_STATIC_SCRATCH_BYTES ? (int)(chunk / 2) : 0;
}
// Pairs of partial sums per chunk that a slot's averages may need, whatever the call: two if any is cut.
inline int mean_pairs(int cus, int64_t chunk, int64_t n_chunks, int64_t n_layers) {
    return mean_cut(cus, chunk, n_chunks, n_layers, 32, true) ? 2 : 1;
}

// Whether a model is so small that its update and fused step take chunks of kSmallChunk elements and neither has a cap on the workgroups
// per CU: at two workgroups per CU and 2048 elements each it is one or two rounds of them, the second half empty.
// That shape / this one in us, 8 layers, fused, back to back:
//     chunks of 2048           129          257          513         1026         1409         2050
//     AdamW, N = 8          6.5 / 6.3    8.4 / 7.8   11.1 / 10.4  17.4 / 16.3  22.0 / 22.2  28.7 / 29.0
//     ... separate tensors  6.8 / 6.5    8.5 / 8.1   11.4 / 10.5  17.9 / 16.9  22.4 / 22.0  29.5 / 29.5
//     SGD, N = 4            5.3 / 5.7    5.6 / 6.4    7.6 / 7.3   12.1 / 11.1  14.9 / 14.5  19.1 / 19.0
//     SGD, bf16, N = 12     7.7 / 7.0    8.3 / 7.9   12.4 / 11.2  14.8 / 14.3  17.7 / 17.6  22.4 / 22.7
// Up to 4.5 chunks per CU, then; below 5/4 only with a second moment.  SGD with many bf16 peers gains there too, but replica count and
// wire come with each call, when the tables are long made, and with few replicas SGD loses more than that.  (The smallest models' fused step
// gains with either: SGD, 13 layers of 142^2, N = 16 9.1 / 7.7, 8 of 187^2, N = 32 bf16 11.4 / 8.9; it has these chunks, under a cap that such a
// model does not reach.)
constexpr int64_t kSmallChunk = 1024;
inline bool small_model(int cus, int64_t numel, bool second_moment) {
    const int64_t chunks = (numel + 2047) / 2048;
    return 2 * chunks <= 9 * (int64_t)cus && (second_moment || 4 * chunks > 5 * (int64_t)cus);
}

// Whether a table-free update of numel elements, a few layers of a larger model, takes that shape: with AdamW, up to 7/4 chunks per
// CU.  Layer by layer, 8 layers, us: 600^2 43.7 / 41.3, 724^2 49.6 / 47.0, 886^2 63.9 / 61.8; 1024^2, where two workgroups per CU are
// just one round, 72.3 / 73.2; SGD 886^2 47.1 / 47.0.
inline bool short_update(int cus, int64_t numel, bool adamw) { return adamw && 4 * ((numel + 2047) / 2048) <= 7 * (int64_t)cus; }

// Whether the fused step of N bf16 replicas has two vectors of all streams in flight per thread (fused_body), in a call on `all`
// chunks, `scheduled` of them of the slot's layers: in kernels laid out for 16 and 32 replicas, where a chunk has a second vector for
// each thread, so not in halves of chunks (call_takes_halves) but in whole ones: where the caller gives chunks, in models with a layer of 128 M
// elements, with SGD over separate tensors, and in models of 6 to 10 chunks per CU up to 200 bytes a vector.  That takes up to twice the
// registers and makes every workgroup's ramp longer, which a call of a few rounds of workgroups does not hide.  One vector / two, in chunks of
// 2048 all, us (scheduled of all chunks per CU):
//     8 layers, fused       N = 24, SGD       N = 24, AdamW     N = 32, AdamW
//     543^2  (1.1 of 4.5)   21.3 /  23.5      24.4 /  26.8      27.2 /  30.4
//     640^2  (1.6 of 6.3)   24.0 /  25.4      29.5 /  30.1      31.2 /  33.0
//     724^2  (2 of 8)       31.0 /  30.5      36.4 /  36.3      39.5 /  40.4
//     886^2  (3 of 12)      43.3 /  42.6      52.0 /  51.2      56.7 /  56.3
//     1533^2 (9 of 36)     111.7 / 107.3     138.1 / 134.7     149.6 / 152.3
//     GPT-2 small          674   / 641       836   / 808       879   / 877       (N = 12, AdamW 687 / 677, N = 16 722 / 709)
//     4, layer by layer, all scheduled
//     800^2  (1.2 of 1.2)   71.2 /  86.6      79.0 /  96.0      86.0 / 102.4
//     1448^2 (4 of 4)      148.0 / 152.2     167.8 / 168.8     184.0 / 196.0
//     1773^2 (6 of 6)      212.8 / 206.6     239.1 / 232.1     275.0 / 278.7
// 800^2 at N = 12 and 16, SGD: 47.2 / 51.7, 49.6 / 57.7.  Fewer replicas: GPT-2 small N = 8 634 / 634; fp32 peers are slower so (N = 8 528 /
// 531, N = 2 420 / 427).
inline bool takes_pairs(int cus, int64_t chunk, int64_t all, int64_t scheduled, int N, bool wire16) {
    return wire16 && N > 8 && N <= 32 && chunk >= 2048 && scheduled >= 3 * (int64_t)cus && 2 * all >= 9 * (int64_t)cus;
}

// Whether a model's fused step may have a workgroup for each half (kSmallChunk elements) of a chunk of the update table, if the call asks
// for it (call_takes_halves).  With whole chunks a thread's second vector of all streams waits for what the first one's sum and step leave
// behind.  Not in models with layers of 128 M elements and more, whose long launches run best with the fewest rows in flight.  The line is
// flat: whole / halves and three per CU, us, four layers of 81, 100, 130 and 160 M, one scheduled:
//     AdamW, N = 4       1622 / 1623   2056 / 2044   2628 / 2630   3212 / 3233
//     AdamW, N = 8       1865 / 1854   2376 / 2395   2987 / 3067   3666 / 3683
//     SGD, N = 8         1467 / 1462   1809 / 1789   2401 / 2393   2914 / 2882
// and beyond it: blocks of 4096, 11008 (layers of 202 M and 131 M), AdamW, N = 8 11121 / 11277, layer by layer 11165 / 11362, N = 4 9550 / 9709.
// One such layer decides for the whole model: eight blocks of 20 M beside an embedding of 150 M, N = 8, SGD 1283 / 1283, AdamW
// 1650 / 1650, bf16 peers 1511 / 1502, so nothing is to be had from choosing launch by launch.  Nor over separate tensors with SGD from 16 M elements
// on, where unscheduled layers want whole chunks (GPT-2 small, N = 8 538 / 557, 13 blocks of 1536 1691 / 1746, 12 layers of 1378^2, N = 16 bf16 112 / 117).
// With AdamW over separate tensors the halves, which have nothing to pace (long_launch), gain more than they lose: paced whole chunks and two
// per CU / halves and three, N = 2 and 8, 12 layers of 3000^2 504 / 496, 615 / 598, of 5000^2 1421 / 1375, 1733 / 1714, seven blocks of 44 M 2084 / 2025, 2447 / 2384,
// TinyLlama-1.1B 5257 / 5041, 6450 / 6227, layer by layer 5142 / 5107, 6157 / 6107; but GPT-2 small 581 / 590, 702 / 700, 12 layers of 4096^2 972 / 993, 1184 / 1209.
inline bool takes_halves(int64_t numel, int64_t largest_layer, bool dense, bool second_moment) {
    return largest_layer < (int64_t)1 << 27 && (dense || second_moment || numel < (int64_t)1 << 24);
}

// Whether a call on a slot of such a model, or on a range of its layers, takes halves: one answer for all of a worker's calls, whatever the
// range, so that a slot's statistics have one order of summation.  slot: its elements, layer: the chunks of its largest layer.  Halves have more
// in flight, whole chunks fewer workgroups to start and half the partial sums, which decides in models of a few chunks (2048 elements) per CU
// as long as a vector is small.
// Fused step, whole chunks and two workgroups per CU / halves and three, us, dense arenas, a quarter or a fifth of the layers scheduled:
//         chunks per CU               4.8 (12 x 460^2)   5.4 (5 x 750^2)   7.7 (12 x 580^2)   9.4 (12 x 640^2)  13.2 (12 x 760^2)  18.6 (12 x 900^2)
//     AdamW, N =  4, fp32 (104 bytes)    14.7 / 14.8       15.4 / 15.1       22.5 / 25.0        26.5 / 28.5        38.1 / 39.3        51.9 / 51.8
//     AdamW, N =  8, fp32 (168)          18.3 / 16.6       17.8 / 17.1       26.1 / 28.6        32.0 / 32.2        43.3 / 44.6        58.7 / 58.7
//     AdamW, N =  8, bf16 (112)          15.8 / 15.5       16.4 / 16.1       23.1 / 25.3        27.2 / 29.2        38.8 / 39.3        53.4 / 53.0
//     AdamW, N = 16, bf16 (176)          19.9 / 18.4       20.7 / 19.1       27.1 / 29.1        32.7 / 33.7        45.0 / 44.9        61.7 / 61.7
//     AdamW, N = 16, fp32 (296)          23.4 / 21.3       23.7 / 22.2       32.6 / 34.8        41.9 / 39.3        53.6 / 54.6        76.7 / 73.5
//     SGD,   N =  2, fp32 (64)           10.3 / 10.4       10.8 / 11.1       15.1 / 17.3        18.3 / 19.7        26.2 / 26.1        35.3 / 35.2
//     SGD,   N =  4, fp32 (96)           10.9 / 10.5       11.3 / 11.5       16.3 / 18.2        19.5 / 20.9        28.0 / 28.0        37.9 / 37.8
//     SGD,   N =  8, fp32 (160)          13.8 / 12.5       14.1 / 12.9       19.4 / 21.2        24.2 / 24.3        33.5 / 33.0        44.6 / 44.6
//     SGD,   N = 16, fp32 (288)          18.8 / 17.5       20.0 / 17.8       26.4 / 27.7        34.4 / 31.7        44.6 / 43.6        61.9 / 59.9
// So whole chunks from 6 to 10 chunks per CU, up to 200 bytes a vector, and with SGD below 6 too up to 120 bytes (in models of less than 5/4
// chunks per CU only with a layer of half a chunk per CU: 700^2, N = 2 5.6 / 6.0, separate tensors N = 4 5.7 / 6.4, two of 520^2,
// N = 8 bf16 7.5 / 7.1, 12 layers of 200^2, N = 4 4.9 / 4.9, N = 16 7.3 / 6.4).  Beyond 10 they gain less, and four
// workgroups per CU give most of it (fused_wg_per_cu).  Over dense arenas only for slots of some size: with a small one most of the call are unscheduled
// layers, which are the faster for three workgroups per CU, with a large one the second vector's wait is most of it.  Whole / halves again, by the chunks
// per CU of the slot:
//     12 x 580^2                  0.6           1.3           1.9           3.9         12 x 490^2 (5.5 per CU)    0.5           0.9           1.4           2.7
//         SGD, N = 4          16.9 / 15.8   16.7 / 17.0   16.3 / 17.9   20.1 / 20.7         SGD, N = 4         12.5 / 11.6   12.7 / 11.7   12.2 / 13.2   15.3 / 15.3
//         SGD, N = 8          19.0 / 17.8   20.0 / 19.6   19.6 / 21.4   25.4 / 25.9         N = 4 by layers                                              55.0 / 51.6
//         AdamW, N = 4        23.4 / 23.9   23.0 / 24.6   22.6 / 25.1   26.6 / 26.8         SGD, N = 8 bf16    13.3 / 12.4   13.6 / 12.7   13.3 / 14.3   16.1 / 17.2
//         AdamW, N = 8        25.8 / 25.7   26.6 / 26.8   26.2 / 28.6   32.8 / 32.6
//         AdamW, N = 16 bf16  27.6 / 27.6   28.1 / 28.2   27.2 / 29.7   33.9 / 35.8
// and AdamW, 6 x 880^2, 3.0, N = 2 25.7 / 25.1, N = 8 34.5 / 32.9, by layers 47.8 / 45.2.  Layer by layer AdamW prefers halves throughout (12 x 580^2, 1.9, N = 4
// 57.7 / 57.2, N = 8 62.1 / 60.5), but what the whole-model call gains is more; not with layers of less than half a chunk per CU: 24 x 420^2, 1.4, N = 4
// 23.3 / 24.1 and 90.2 / 87.3, N = 8 27.3 / 26.3 and 97.2 / 89.7, separate tensors, 0.7, N = 8 25.9 / 25.0.
// Over separate tensors, where the unscheduled layers come in halves too, whole chunks whatever the slot (7.7 per CU, slot 0.6, N = 8 SGD 18.9 / 20.0, AdamW
// 25.5 / 26.0), with SGD from 5/4 on: N = 8 5.4 per CU 14.3 / 14.3, 7.2 18.3 / 20.7, 18.6 44.6 / 45.8, bf16 39.6 / 41.2, 27.7 58.2 / 60.8, N = 16
// 24.8 / 27.7 and 88.0 / 89.7, N = 2, 13.2 25.0 / 26.0; but halves for the largest vectors (N = 24, 9.4 per CU 45.2 / 41.9, 14.7 63.1 / 60.5).
inline bool call_takes_halves(int cus, int64_t numel, int64_t slot, int64_t layer, bool dense, int N, bool wire16, bool adamw, bool grad16) {
    const int64_t chunks = (numel + 2047) / 2048, bytes = vector_bytes(N, wire16, adamw, grad16);
    const bool below_6 = chunks < 6 * (int64_t)cus, below_10 = chunks < 10 * (int64_t)cus, large = bytes >= 150, many16 = wire16 && bytes >= 96;
    auto slot_from = [&](int quarters) { return 4 * ((slot + 2047) / 2048) >= quarters * (int64_t)cus; };  // quarters of a chunk per CU
    if (adamw) {
        if (below_6 || !below_10 || bytes >= 200 || 2 * layer < cus) return true;
        return dense && (!slot_from(large ? 6 : 3) || (slot_from(10) && !many16));
    }
    if (bytes >= 300) return true;
    if (4 * chunks <= 5 * (int64_t)cus) return 2 * layer < cus || bytes >= 120 || many16;
    if (!dense) return false;
    return !below_10 || bytes >= (below_6 ? 120 : 200) || !slot_from(large ? 7 : 5) || (below_6 && slot_from(10));
}

// A launch has less than 2^32 threads in x (hipErrorInvalidConfiguration from there on, measured: 2^24 - 1 workgroups of 256 run, 2^24 are
// refused).  The table-driven fused step over all n_update chunks of a model, a workgroup for each half: up to 17 G elements.
inline bool halves_fit(int64_t n_update) { return 2 * n_update < (int64_t)1 << 24; }

// Workgroups per CU that a fused step on `elements` elements asks for where a workgroup takes half a chunk of the update table, kSmallChunk
// elements, one vector of all streams a thread, and the call has `halves` of them.  Halves and three / halves and four, us, 12 layers, a quarter of them scheduled,
// dense arenas:
//                             bytes    1024^2           1536^2           2304^2           3600^2
//     SGD,   N =  2, bf16       56    44.2 /  42.8     94.8 /  92.7    210.4 / 205.1    520.7 /  512.8
//     SGD,   N =  2, fp32       64    44.8 /  44.0     97.5 /  95.4    215.6 / 213.2    527.5 /  523.3
//     SGD,   N =  3, fp32       80    46.0 /  45.4    100.0 /  99.1    220.6 / 219.3    540.3 /  545.3
//     SGD,   N =  6, bf16       88    47.4 /  46.8    102.6 / 102.0    227.5 / 225.4    566.6 /  562.0
//     SGD,   N =  4, fp32       96    47.7 /  47.6    103.6 / 103.8    230.9 / 232.7    563.9 /  574.7
//     SGD,   N =  8, fp32      160    56.7 /  57.2    124.3 / 124.3    275.0 / 279.1    678.3 /  687.2
//     AdamW, N =  2, bf16       64    60.0 /  60.3    129.0 / 130.0    291.5 / 291.5    717.8 /  725.8
//     AdamW, N =  3, bf16       64    62.7 /  62.0    135.5 / 133.9    299.5 / 295.1    734.1 /  728.0
//     AdamW, N =  2, fp32       72    61.2 /  61.9    131.0 / 132.1    293.7 / 294.9    725.4 /  729.1
//     AdamW, N =  4, bf16       72    62.5 /  62.7    133.2 / 134.7    298.8 / 299.8    743.5 /  746.5
//     AdamW, N =  8, fp32      168    74.7 /  75.5    159.5 / 165.0    356.1 / 360.4    878.5 /  887.3
// So four with SGD and less than 96 bytes a vector, with AdamW, a third more bytes to write, for three bf16 replicas; else three.
// Four also in short AdamW calls over dense arenas, of 6 to 16 chunks (2048 elements) per CU, which are too few rounds of workgroups for three, if the slot has 3/2
// and more per CU: 760^2 (13.2), slot 3.3, N = 4 39.3 / 38.9, N = 8 44.6 / 44.1, N = 16, bf16 44.9 / 44.4, slot 2.2, N = 8 41.9 / 40.9, N = 16, bf16 44.7 / 43.2, slot 1.1
// 39.2 / 39.5, 41.0 / 41.5, 5 layers of 1100^2 (11.6), N = 8, bf16 34.4 / 33.6, 24 of 640^2 (18.8), slot 3.1, N = 4 50.8 / 51.1, slot 0.8, N = 16, bf16 51.6 / 52.8,
// separate tensors 760^2, slot 3.3, N = 8 43.7 / 44.6, slot 1.1 38.1 / 39.4.  With less than 96 bytes up to 24 in all cases, 460^2 (4.8), N = 2 13.5 / 12.8
// (N = 8 16.6 / 17.6),
// and where the call is then one round: layer by layer, 1024^2, SGD, N = 8 86.5 / 84.9, bf16, N = 12 90.3 / 87.7, AdamW, N = 8 109.9 / 108.3.
// Two over dense arenas in calls on 64 M elements and more of 16 to 32 fp32 replicas, whose three would have over 200 KB in flight per CU.
// Halves and three / halves and two, 10 layers:
//                    1536^2          3000^2          4096^2
//     N = 16, SGD    150 / 151       585 / 582      1090 / 1033
//     N = 16, AdamW  187 / 197       708 / 702      1297 / 1258
//     N = 24, SGD    192 / 193       748 / 741      1384 / 1318
//     N = 32, AdamW  272 / 280      1063 / 1055     1908 / 1880       (N = 12, AdamW 164 / 180, 1140 / 1157)
// (more replicas, through LDS: 12 of 3600^2, N = 40, SGD 1579 / 1769, N = 64 2953 / 3920; separate tensors, N = 16, AdamW, 12 of 3000^2 775 / 798, 12 of
// 6500^2 3728 / 3819).
inline int fused_wg_per_cu(int cus, bool dense, int N, bool wire16, bool adamw, bool grad16, int64_t elements, int64_t halves, int64_t slot) {
    if (dense && !wire16 && N >= 16 && N <= 32 && elements >= (int64_t)1 << 26) return 2;
    if (halves > 3 * (int64_t)cus && halves <= 4 * (int64_t)cus) return 4;
    const int64_t chunks = (elements + 2047) / 2048;
    const bool little = vector_bytes(N, wire16, adamw, grad16) < 96;
    if (!adamw) return little ? 4 : 3;
    if ((N == 3 && wire16) || (little && chunks < 24 * (int64_t)cus)) return 4;
    return dense && chunks >= 6 * (int64_t)cus && chunks < 16 * (int64_t)cus && 2 * ((slot + 2047) / 2048) >= 3 * (int64_t)cus ? 4 : 3;
}

// Workgroups per CU that the table-driven fused step of a small model asks for, in a call of `chunks` workgroups (0: as many as its registers leave
// room for).  SGD with fp32 gradients on 16 fp32 replicas has room for four: where the call is two rounds of those as well as of three, from 45/8 per CU
// on, three are better.  On 32 bf16 replicas, the update first, it has room for five (the average first, for four): from 7 per CU on four.
// As many as there is room for / three and four, separate tensors, us:
//     N = 16, workgroups per CU   4.7 (18 x 260^2)   5.2 (20 x 260^2)   5.5 (9 x 400^2)   6.1 (10 x 400^2)   6.3 (24 x 260^2)   8.0 (13 x 400^2)
//                                   10.1 / 12.2        10.4 / 12.3        10.5 / 12.3       14.6 / 13.8        15.2 / 13.8        16.5 / 15.1
//     N = 32                      6.1 (10 x 400^2)   6.3 (24 x 260^2)   6.8 (26 x 260^2)  7.9 (30 x 260^2)   8.0 (13 x 400^2)
//                                   14.6 / 17.7        14.1 / 18.0        16.5 / 18.7       22.1 / 19.7        21.5 / 19.6
// and many layers of one to four chunks: N = 16 5.3 (340 x 60^2) 12.6 / 12.0, 5.6 (360 x 60^2) 13.2 / 12.2, 9.0 (230 x 100^2) 17.7 / 16.5.
inline int small_wg_per_cu(int cus, int N, bool wire16, bool adamw, bool grad16, int64_t chunks) {
    if (adamw || grad16) return 0;
    if (N == 16 && !wire16 && 8 * chunks >= 45 * (int64_t)cus) return 3;
    return N == 32 && wire16 && chunks >= 7 * (int64_t)cus ? 4 : 0;
}

// Workgroups of the table-free fused kernel over elements [e0, e1) of the arenas: chunks counted from the multiple of `line`
// (kLine) at or below e0.
inline int64_t dense_workgroups(int64_t e0, int64_t e1, int64_t chunk, int64_t line) { return (e1 - e0 / line * line + chunk - 1) / chunk; }

// Chunks of the widest piece that the kernel's 32-bit indexes allow.
inline int64_t widest_piece(int64_t chunk) { return INT32_MAX / chunk - 1; }

// Elements [begin, end), all of one scheduled layer (flat0 >= 0) or all unscheduled, as pieces of at most `width` chunks behind
// those that p has.
inline void add_pieces(DensePass &p, int64_t begin, int64_t end, int64_t flat0, int64_t pbase, int32_t layer, const LayerSums &of, int64_t width,
                       int64_t chunk, int64_t line) {
    const int64_t base = begin / line * line, wg = dense_workgroups(begin, end, chunk, line);
    for (int64_t b = 0; b < wg; b += width) {
        const int64_t at = b == 0 ? begin : base + b * chunk, to = std::min(end, base + (b + width) * chunk);
        p.pieces[p.n_pieces++] = {at, flat0 < 0 ? -1 : flat0 + (at - begin), (int32_t)(to - at), (int32_t)(pbase + b), of.pos, layer, of.first, of.n};
    }
}

// The launches over the whole model of L layers, layer l being elements [elem0(l), elem0(l + 1)) of the arenas.  A segment is a
// scheduled layer or a run of unscheduled ones.
// Segments of kAlone elements and more get a launch each, the unscheduled ones that of the plain update, whose workgroups start
// sooner; neighbours below that share one, cut into pieces of about the same width, because a launch of its own costs a segment
// some 3 us of ramp.  Shared against own launches, N = 2 / 4 / 8: 20 layers of 10 M 0.94 / 0.95 / 0.92 of the time, of 20 M
// 0.99 / 1.00 / 0.99 (8 of them 0.98 / 0.98 / 0.96, 40 of them 0.99 / 1.02 / 1.02), of 25 M 1.00 / 1.01 / 1.00, of 30 M
// 1.00 / 1.03 / 1.03: the line is where it breaks even.
// A launch takes kMaxSegments; where that makes several and the model is small, the table is the better one (table_first): its
// workgroups start later but all in one launch.  Pieces against the table in us, N = 4: 400 layers of 1000 elements 83 / 8, 21 of
// 64 K 17.0 / 12.5, of 256 K 37.9 / 34.3, of 1 M 117 / 115; N = 2: 21 of 1 M 126 / 129, 40 of 4 M 836 / 868.
// No passes where a launch would need more than kMaxPieces pieces: such a slot always takes the table.
// `plain`: chunks that a workgroup of an unscheduled piece takes.
template <class Elem0>
void plan_dense(FusedPlan &plan, const SlotTables &st, int L, Elem0 &&elem0, int64_t chunk, int64_t line, int64_t plain = 1) {
    constexpr int kMaxSegments = 20;
    struct Segment {
        int64_t begin, end, flat0, pbase, chunk, wg;
        int32_t layer;
        LayerSums of;
    };
    std::vector<Segment> all;
    for (int l = 0; l < L;) {
        const int i = st.layer_pos[(size_t)l];
        int m = l + 1;
        while (i < 0 && m < L && st.layer_pos[(size_t)m] < 0) ++m;
        all.push_back({elem0(l), elem0(m), i < 0 ? -1 : st.layer_begin[(size_t)i], i < 0 ? 0 : plan.update_ranges[2 * (size_t)i],
                       i < 0 ? plain * chunk : chunk, 0, l, {i, 0, 0}});
        all.back().wg = dense_workgroups(elem0(l), elem0(m), all.back().chunk, line);
        if (i >= 0) all.back().of = {i, plan.update_ranges[2 * (size_t)i], plan.update_ranges[2 * (size_t)i + 1] - plan.update_ranges[2 * (size_t)i]};
        l = m;
    }
    std::vector<DensePass> &passes = plan.dense_passes;
    constexpr int64_t kAlone = (int64_t)3 << 23, kPerLaunch = (int64_t)1 << 24;  // 25 M; elements that a launch more is worth
    auto group = [&](size_t k) {  // segments that share the launch of segment k, the first one of it
        size_t n = 1;
        auto large = [&](size_t j) { return all[j].end - all[j].begin >= kAlone; };
        while (!large(k) && n < kMaxSegments && k + n < all.size() && !large(k + n)) ++n;
        return n;
    };
    int64_t shared = 0;
    for (size_t k = 0; k < all.size(); k += group(k)) shared += all[k].end - all[k].begin < kAlone;
    plan.table_first = all.back().end - all[0].begin < (shared - 1) * kPerLaunch;
    const int64_t widest = widest_piece(plain * chunk);
    for (size_t i = 0; i < all.size();) {
        const Segment *seg = &all[i];
        const int n = (int)group(i);
        i += (size_t)n;
        int64_t least = 0;
        for (int k = 0; k < n; ++k) least += (seg[k].wg + widest - 1) / widest;
        if (least > kMaxPieces) {
            passes.clear();
            return;
        }
        passes.emplace_back();
        DensePass &p = passes.back();
        p.width = p.n_pieces = 0;
        p.begin = seg[0].begin;
        p.end = seg[n - 1].end;
        if (n == 1 && seg[0].flat0 < 0) continue;  // a plain update, wherever in a vector it starts
        // the width that leaves the fewest workgroups without work among those that cut some segment evenly
        int64_t width = widest, best = INT64_MAX;
        for (int k = 0; k < n; ++k)
            for (int64_t parts : {1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24}) {
                const int64_t w = (seg[k].wg + parts - 1) / parts;
                if (w > widest) continue;
                int64_t rows = 0;
                for (int j = 0; j < n; ++j) rows += (seg[j].wg + w - 1) / w;
                if (rows <= kMaxPieces && (rows * w < best || (rows * w == best && w > width))) {
                    best = rows * w;
                    width = w;
                }
            }
        p.width = (int)width;
        for (int k = 0; k < n; ++k)
            add_pieces(p, seg[k].begin, seg[k].end, seg[k].flat0, seg[k].pbase, seg[k].layer, seg[k].of, width, seg[k].chunk, line);
    }
}
template <class Elem0>
void plan_dense(SlotTables &st, int L, Elem0 &&elem0, int64_t chunk, int64_t line, int64_t plain = 1) {
    plan_dense(st, st, L, elem0, chunk, line, plain);
}

// The first launch that has elements from e0 on.
inline std::vector<DensePass>::const_iterator first_pass(const FusedPlan &plan, int64_t e0) {
    return std::upper_bound(plan.dense_passes.begin(), plan.dense_passes.end(), e0, [](int64_t e, const DensePass &p) { return e < p.end; });
}

// Whether a call on elements up to e1 whose first launch is `at` runs pieces: where the table is better for the slot, if one
// launch does it.
inline bool takes_pieces(const FusedPlan &plan, std::vector<DensePass>::const_iterator at, int64_t e1) {
    return at != plan.dense_passes.end() && (!plan.table_first || at->end >= e1);
}

// What a call on elements [e0, e1), whole layers, runs of launch p: the pieces inside, runs of unscheduled layers cut at the
// range's ends; a plain update (width 0) where no scheduled layer is inside.  No search and nothing allocated; part is written only as far as its pieces go.
inline void clip_pass(const DensePass &p, int64_t e0, int64_t e1, int64_t chunk, DensePass &part, int64_t line, int64_t plain = 1) {
    part.begin = std::max(p.begin, e0);
    part.end = std::min(p.end, e1);
    part.width = part.n_pieces = 0;
    if (part.begin >= part.end || p.width == 0) return;  // (a plain update as well)
    bool scheduled = false;
    for (int i = 0; i < p.n_pieces; ++i) {
        const Piece &whole = p.pieces[i];
        if (whole.begin >= e1) break;
        const int64_t b = std::max(whole.begin, e0), e = std::min(whole.begin + whole.count, e1);
        if (b >= e) continue;
        Piece &q = part.pieces[part.n_pieces++];
        q = whole;
        q.begin = b;  // (moves in unscheduled pieces only: a scheduled one is part of one layer)
        q.count = (int32_t)(e - b);
        part.width = std::max(part.width, (int)dense_workgroups(b, e, q.flat0 < 0 ? plain * chunk : chunk, line));
        scheduled = scheduled || q.flat0 >= 0;
    }
    // Unscheduled layers alone are a plain update, wherever in a vector they start: its workgroups start sooner, its launch carries 104
    // bytes of arguments, that of the pieces 1.8 KB, and takes 0.3-0.5 us less of the host (8 layers of 509^2, N = 5, layer by layer, us
    // 35.6 / 31.4).
    if (!scheduled) part.width = part.n_pieces = 0;
}

}  // namespace ddp

#endif

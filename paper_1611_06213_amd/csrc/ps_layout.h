// Where the server puts its buffers, and how the apply kernels sweep
// buffers it did not place. Host-only; ps_server.cpp uses it, and it builds
// on its own for host tests.
//
// DRAM serves many concurrent streams fastest when they do not start at one
// offset within 2 MiB (their "phase"), and the distance between them matters
// beyond that: the apply reads 32 or more rows in lockstep, and how their
// addresses spread over HBM channels and banks depends on higher address bits
// too. The server's own large buffers (w, v and the rows of ps_alloc_rows)
// therefore start 1.75 MiB apart beyond their 2 MiB-rounded sizes, so
// consecutive rows step through the eight 256 KiB phases downwards. Buffers
// allocated one by one all start at one phase; for them the kernels sweep
// several fronts instead of one (fronts_log2_for).
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace gadei {

constexpr size_t kRowAlign = size_t(2) << 20;
// Phase granularity: rows under 2 MiB are packed on it, and the front choice
// compares buffer phases at it.
constexpr size_t kPhase = 4096;
// Step between large rows (and from w to v) beyond their 2 MiB-rounded size.
// Measured on the VGG-16 (fp32) and Mixed (bf16) applies from 32 rows, over
// steps of 4 KiB and 64 KiB .. 2 MiB: 64-256 KiB were worst (up to 20%
// slower than 4 KiB), steps near 1 MiB were bad for the bf16 rows, and
// 1.75 MiB was among the best for both. Whole bench steps against 4 KiB:
// VGG-16 7,111-7,119 vs 6,953-6,961 pushes/s, Mixed +2.8%, AlexNet +0.9%.
// The gain is at the default depth: for applies of 16 or fewer gradients
// with momentum, 4 KiB steps measured 1.5-3.7 points of peak faster.
constexpr size_t kRowStagger = size_t(7) << 18;

size_t round_up(size_t x, size_t a);
char *align_up(void *p, size_t a);

// Offset of v from w (w at a 2 MiB boundary): one kRowStagger past w's
// 2 MiB-rounded end.
size_t velocity_offset(size_t w_bytes);

// A set of `count` rows of row_bytes each, from a 2 MiB-aligned base: row i
// at head + i * stride. Rows of 2 MiB or more start two kRowStagger in and
// step by their 2 MiB-rounded size plus kRowStagger, so row i sits at phase
// ((i + 2) * kRowStagger) mod 2 MiB (w, v and the rows of one set cycle
// through the eight 256 KiB phases); smaller rows are packed on kPhase
// boundaries after a head of 2 * kPhase. `span` = bytes from the base to the
// end of the last row.
struct RowLayout {
    size_t head;
    size_t stride;
    size_t span;
};
RowLayout row_layout(size_t row_bytes, int count);

// Fronts (log2) an apply over these streams (gradients, w, v; null entries
// are skipped) should sweep: 2 (four fronts) when there are at least 8
// streams and more than half of them share one phase (compared at kPhase),
// else 0 (one front). Measured on 34 streams of 553 MB: same-phase buffers
// 3.97-4.27 ms with one front, 3.42-3.54 ms with four; staggered buffers
// no better with four.
int fronts_log2_for(const void *const *ptrs, int count);
// Gradients of fewer bytes take one front whatever their offsets: only the
// longest separately allocated buffers are served so much slower by one front
// that four make up for their shorter runs. One front against four, us, torch
// allocations with momentum: fp32 61M, 16 gradients 785 vs 822, 100M 1329 vs
// 1509, 120M (480 MB), 32 gradients 2758 vs 2892; 130M (520 MB) 3556 vs 3172,
// 138M 4300 vs 3502; bf16 200M (400 MB), 32 gradients 2712 vs 2894.
constexpr size_t kFrontsBytes = 500000000;

// Launch shape of an apply of k gradients (fp32, or bf16): how many 256-thread
// blocks one compute unit may hold (0 = as many as fit), and how many gradients
// each lane loads at once (4, 8, 12, 16, 24 or 32; the synchronous step's table
// stops at 16).
// Fewer resident blocks and smaller groups keep fewer DRAM pages and address
// translations live across the k + 2 streams; too few loads in flight starve
// the memory system. Chosen from sweeps at the VGG-16 (fp32) and Mixed (bf16)
// sizes from server rows, % of 8 TB/s: fp32 with momentum, k = 32: one group
// of 32 at one block per CU 82.2, groups of 16 81.7, groups of 4 at two blocks
// 76.2; k = 4: groups of 4 at two blocks 82.9, groups of 16 at three 80.0;
// bf16 with momentum, k = 24: groups of 24 at one block 79.9, of 16 77.9.
struct ApplyShape {
    int blocks_per_cu;
    int group;
};
// n is the vector's length: below kSmallVector coordinates a shallow fp32
// apply without momentum (7..13 gradients) keeps three blocks per CU instead
// of two (Text-CNN-sized vectors, 10M and 17.3M: 77.3-77.7 and 76.2% vs
// 76.2-76.4 and 74.7; from 24M two are best, 80.4 vs 79.2).
constexpr size_t kSmallVector = 20000000;
// Below kMidVector a launch is a few waves of blocks or less and what counts
// is the latency of its first loads, not DRAM pages: more blocks or a larger
// group at once (kernel time, from the table of large vectors to this one; 1M:
// fp32 with momentum k = 4 7.8 -> 6.9 us, 16 16.1 -> 14.9; bf16 with momentum
// k = 32 17.8 -> 15.0; bf16 k = 64 25.9 -> 22.8; 4M: fp32 with momentum k = 16
// 54.8 -> 51.7). At 7M the two are within 5% of each other either way. Below
// kTinyVector one round of blocks holds everything, and all of a lane's loads go
// out together (100k, fp32 k = 64: 10.2 -> 8.4 us).
// `widened`: the launch also writes more than one fp32 replica from bf16
// gradients. Its 8-coordinate lanes write each in two stores 32 bytes apart, and
// more than two blocks a unit then keep more half-written lines than L2 holds (no
// momentum, 1 gradient and 4 replicas: 2M 16.0 us with four, 12.7 with two; 4M 26.1
// vs 23.4).
constexpr size_t kMidVector = 5000000;
constexpr size_t kTinyVector = 500000;
ApplyShape apply_shape(int k, bool momentum, bool bf16, size_t n, bool widened = false);

// The same for a synchronous step over k gradients (one per learner). Below
// kMidVector fp32 steps take shapes of their own, as applies do (packed odd rows,
// where one coordinate per lane took, without momentum: 1M, k = 16 13.0 us against
// 14.4 with the table of large vectors and 11.8 now; 2.5M, k = 20 35.4, 42.5, 37.3;
// with momentum: 4.9M, k = 12 50.5, 58.6, 54.1).
ApplyShape sync_shape(int k, bool momentum, bool bf16, size_t n);

// A launch of several steps of a script (launch_steps), in bytes per
// coordinate: the gradients it reads, the replicas its steps write, and those of
// them that stay (a replica that a later step of the launch writes again is then
// often still in cache).
struct StepsSize {
    int steps = 0;
    size_t grad_bytes = 0;
    size_t pull_bytes = 0;
    size_t final_bytes = 0;
};

// Whether a script's steps are worth joining into this launch. Joining saves a
// read and a write of w (and v) and the fan-out's read of w per step and the
// replicas written again, and mixes the writes of those that stay with the
// gradients' reads. So it must
//   - save an eighth of an average step from kSmallVector coordinates on, a sixth
//     without momentum; between 4M and there, without momentum, the gradients must
//     not dwarf both what is saved and the replicas;
//   - and save, in all, a seventh of what the launch reads and twice what it
//     writes for good (an eleventh below kMidVector), unless those writes fit
//     the memory-side cache (kCacheBytes).
// Measured from server rows, a launch per call against joined, us a step. The
// first condition, each step the same replicas, with momentum: 1M, 1 gradient and
// 1 pull 5.1 vs 1.2; 17M, 32 and 16: 570 vs 545; 61M, 16 and 10: 1162 vs 891;
// 138M, 8 and 8: 1785 vs 1126, 16 and 16: 3125 vs 2361, 32 and 16 (a saving of a
// tenth): 4400-4607 vs 4486-4510; bf16 200M, 32 and 32: 4606 vs 4059 (averaged
// steps 4610 vs 3986), separately allocated 4949 vs 4249. Without: 4M, 4 and 8: 41
// vs 28, 32 and 4: 99 vs 99; 17M, 32 and 4: 414 vs 436, 32 and 32: 721 vs 663.
// The second, every step other replicas, with momentum: 138M, 8 and 8 (saved over
// read and written .16): 1779 vs 1742, 16 and 16 (.08): 3103 vs 3437; 10M, 16 and
// 16: 237 vs 246-257, 32 and 32 (.03): 435 vs 481; bf16 200M, 32 and 32 (.05): 4659
// vs 5360, averaged 4633 vs 4942; bf16 138M, 16 and 16 (.16): 1838 vs 1764, 32 and 8
// (.10): 2261 vs 2305. Half of them again (.37): 61M, 16 and 16: 1362 vs 1201; a
// quarter again (.13): 10M, 32 and 32: 438 vs 454. Without momentum: 10M, 8 steps of
// 8 and 8 (.11): 121 vs 130; bf16 17M, 16 and 16 (.09): 224 vs 253; below kMidVector
// 3.9M, 8 and 8 (.09): 52 vs 46, 16 and 16 (.05): 88 vs 96; 2M, 16 and 16 with
// momentum (.08; 512 MB): 47 vs 51; 1M (256 MB): 24.6 vs 21.6.
bool steps_join(const StepsSize &s, bool momentum, size_t n);
constexpr size_t kCacheBytes = size_t(256) << 20;

// Resident blocks per compute unit of a launch of several steps (launch_steps)
// whose steps write `replicas` replicas each, pull_elem and grad_elem bytes a
// value: two while they write little, one beyond (more waves then keep more
// half-written lines of more replicas in cache than it holds). From server rows
// with momentum, two against one: 60M coordinates, 2 gradients and 4 bf16 replicas
// a step 573 vs 696 us (4 steps), 1 and 1 fp32 479 vs 502 us; 2 and 4 fp32 957 vs
// 936, 8 and 8 fp32 2062 vs 1916; 4M, 2 and 4 fp32 202 vs 207 us (16 steps), 8 and
// 8 fp32 506 vs 455; 1M, 1 and 16 fp32 79.8 vs 71.0 us (8 steps).
// Two also for launches so short that one would only make the same blocks wait
// for a round of their own: up to 512 blocks, and up to 1024 where a step writes 16
// or more (us a step, two against one, a launch per call): 500k fp32, 32 and 32
// 21.5 vs 24.4 (22.3), 32 and 8 13.1 vs 14.2 (15.7); 1M bf16, 32 and 32 22.6 vs 26.4
// (24.6), 8 and 8 4.6 vs 4.6; 1M fp32 (976 blocks), 32 and 32 40.7 vs 44.1 (43.9), 8
// and 8 8.3 vs 7.8 (15.0); 2M bf16, 32 and 32 42.3 vs 47.5 (48.3). From 1,465 on even:
// 1.5M fp32, 32 and 32 62.3 vs 62.7.
int steps_blocks_per_cu(int replicas, size_t pull_elem, size_t grad_elem, size_t n);

// Whether ps_apply_pull writes its r replicas from the apply pass over k
// gradients of an n-coordinate vector (else the apply is followed by the
// tiled fan-out): one replica always; up to 4 when at most 16 gradients are
// folded; up to 6 when at most 8 are folded into a vector of fewer than
// kSmallVector coordinates (10M, k = 8: r = 5 0.100 vs 0.104 ms, r = 6 0.108
// vs 0.110; at 30M and above 5 or 6 are even or slower, 138M r = 6 1.50 vs
// 1.44 ms). For smaller vectors the fan-out's launch weighs more (apply+pull
// with momentum, fused vs separate): below 3M up to 8 when at most 16 are
// folded (2M: k = 1, r = 8 19.1 vs 21.5 us; k = 8, r = 8 28.9 vs 29.4; 4M: k = 8,
// r = 8 54.9 vs 54.3); below 1.5M as long as there are few of one or the
// other (1M: k = 1, r = 16 14.2 vs 16.0; k = 32, r = 4 28.4 vs 30.0, r = 16 36.9
// vs 35.1); below kTinyVector always (100k: k = 1, r = 2 5.5 vs 8.1; k = 32, r =
// 16 30.0 vs 33.5; up to 499k and k = 64, r = 64 at most even but for that one corner, fp32
// 45.0 vs 42.3). Writing replicas from
// the apply adds write streams to its read streams, which costs more than a
// separate fan-out once there are many of either; for few of both it saves
// the fan-out's launch and its second read of w. Measured from server rows
// (apply+pull time, fused vs separate): k = 8, r = 2: 10M coordinates
// 0.079 vs 0.086 ms, 138M 1.07 vs 1.10 ms; k = 16, r = 2: 138M 1.89-1.90 vs
// 1.93-1.94 ms; k = 16, r = 8: 138M 2.47 vs 2.42-2.43 ms; k = 32, r = 2:
// 61M 1.55 vs 1.51 ms.
bool fuse_replicas(int r, int k, size_t n);
// The same by the types too. Beyond what is fused at any size fp32 replicas must
// fit: 64 MiB of them (1M, k = 1, r = 16: 16.2 us apart, 15.1 fused; 1.4M 21.5,
// 23.9; k = 10, r = 12 without momentum 24.0, 27.9), and, `widened` (fp32 replicas of
// bf16 gradients: each lane writes them in two stores 32 bytes apart), what L2
// merges: 30 MB (700k, k = 1, r = 8: 10.2, 9.5, r = 16 13.4, 17.3; 1M, k = 16, r = 6
// 15.4, 14.6, k = 4, r = 8 12.6, 16.2; 1.4M, k = 1, r = 16 21.9, 39.2; 2M, k = 1, r = 8
// 20.3, 30.1). From kMidVector on, widened and without momentum at most 2 replicas
// of more than 4 gradients (k = 8, r = 4: 10M 75 vs 76, 61M 447 vs 431, 138M 1182 vs
// 955 us; r = 2 785 vs 782; k = 16, r = 4 10M 105 vs 101, 138M 1448 vs 1336; k = 4, r
// = 4 814 vs 813; with momentum k = 8, r = 4 1143 vs 1160).
bool fuse_replicas(int r, int k, bool bf16, bool fp32_replicas, bool momentum, size_t n);
constexpr size_t kFusedReplicas = size_t(16) << 20;   // coordinates, all replicas
constexpr size_t kWidenedFused = 7500000;

}  // namespace gadei

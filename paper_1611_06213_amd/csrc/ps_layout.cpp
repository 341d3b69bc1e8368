// Buffer placement and front choice; see ps_layout.h.
#include "ps_layout.h"

namespace gadei {

size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

char *align_up(void *p, size_t a) {
    return reinterpret_cast<char *>(round_up(reinterpret_cast<uintptr_t>(p), a));
}

size_t velocity_offset(size_t w_bytes) { return round_up(w_bytes, kRowAlign) + kRowStagger; }

RowLayout row_layout(size_t row_bytes, int count) {
    RowLayout r;
    if (row_bytes < kRowAlign) {
        // packed on 4 KiB boundaries (their phases differ anyway, and rounding
        // each up to 2 MiB would waste memory)
        r.head = 2 * kPhase;
        r.stride = round_up(row_bytes, kPhase);
    } else {
        r.head = 2 * kRowStagger;
        r.stride = round_up(row_bytes, kRowAlign) + kRowStagger;
    }
    r.span = r.head + (static_cast<size_t>(count) - 1) * r.stride + row_bytes;
    return r;
}

int fronts_log2_for(const void *const *ptrs, int count) {
    constexpr int kMaxStreams = 66;   // PS_MAX_QUEUE_DEPTH gradients + w + v
    uintptr_t ph[kMaxStreams];
    int streams = 0;
    for (int i = 0; i < count && streams < kMaxStreams; ++i) {
        if (ptrs[i] == nullptr) continue;
        ph[streams++] = (reinterpret_cast<uintptr_t>(ptrs[i]) % kRowAlign) / kPhase;
    }
    int most = 0;   // the largest number of streams sharing one phase
    for (int i = 0; i < streams; ++i) {
        int same = 0;
        for (int j = 0; j < streams; ++j) same += ph[j] == ph[i];
        most = same > most ? same : most;
    }
    return (streams >= 8 && 2 * most > streams) ? 2 : 0;
}

namespace {

// apply_shape below kMidVector coordinates. Measured from 100k to 4.9M, from
// server rows, separate allocations and rows of a packed tensor, for the depths 1
// to 64; the figures are the most that a shape lost to the best one in its range.
ApplyShape small_apply_shape(int k, bool momentum, bool bf16, size_t n) {
    const bool tiny = n < kTinyVector;
    if (bf16) {
        if (k <= 11 && !momentum) return {k <= 2 ? 4 : 3, 8};
        if (k <= 31 || tiny) return {2, 16};
        // 32 and 40 gradients: up to 2.9M 5% ({2, 4} 10%), from there 7% (8%)
        if (k <= 47) return n < 3000000 ? ApplyShape{2, 16} : ApplyShape{2, 4};
        if (momentum) return n < 850000 ? ApplyShape{2, 16} : ApplyShape{2, 4};
        return n < 2400000 ? ApplyShape{2, 4} : ApplyShape{1, 24};   // 6% ({2, 4} 8%)
    }
    if (k <= 1 && momentum) return {4, 16};
    if (k <= 9) return {0, 16};
    if (k <= 15) return {4, 16};
    const bool few = n < 1500000;   // six rounds of blocks at one a unit
    if (k <= 31) return few && !tiny ? ApplyShape{4, 16} : ApplyShape{2, 16};
    if (tiny) return {1, 32};
    if (n <= (1u << 19)) return {2, 4};   // one round of two blocks a unit
    if (n <= (1u << 20)) return {4, 4};   // one of four: 5% ({2, 4} 17%)
    // 5% (at 1.1M and 1.2M {2, 4} 9%)
    if (few || (k < 40 && n < 2000000)) return {2, 16};
    return {1, 16};   // 8%, on average 1.4% ({1, 32} 8%, 3%)
}

// sync_shape below kMidVector coordinates, fp32 (the same kind of figures; the
// table of large vectors loses up to 29% there).
ApplyShape small_sync_shape(int k, bool momentum, size_t n) {
    if (k <= 4) return {momentum ? 4 : 0, 4};                    // 4%, 5%
    if (k <= 13) return {4, momentum ? 8 : 4};                   // 6%
    return {momentum && n >= 3000000 ? 3 : 4, 4};                // 6%
}

}  // namespace

ApplyShape apply_shape(int k, bool momentum, bool bf16, size_t n, bool widened) {
    if (n < kMidVector) {
        ApplyShape s = small_apply_shape(k, momentum, bf16, n);
        if (widened && (s.blocks_per_cu == 0 || s.blocks_per_cu > 2)) s.blocks_per_cu = 2;
        return s;
    }
    // Measured at 138,357,544 fp32 / 200,000,000 bf16 parameters for the
    // depths 1, 2, 3, 4, 6, 8, 12, 16, 20, 24, 32, 36, 40, 44, 48 and 64
    // (bf16: from 8); the depths between take a neighbour's shape. A group of
    // 24 or 32 pays only from its own depth on: below it the w/v loads would
    // be waited for before the first (smaller) group.
    if (bf16) {
        if (momentum) {
            if (k <= 11) return {2, 16};
            if (k <= 23) return {1, 16};
            if (k <= 44) return {1, 24};
            return {1, 16};
        }
        if (k <= 11) return {2, 8};
        if (k <= 23) return {1, 16};
        if (k <= 31) return {1, 24};
        if (k <= 47) return {1, 32};
        if (k <= 56) return {1, 16};
        return {1, 8};
    }
    if (momentum) {
        if (k <= 1) return {4, 16};
        if (k == 2) return {3, 4};
        if (k <= 9) return {2, 4};
        if (k <= 13) return {1, 12};
        if (k <= 17) return {1, 16};
        if (k <= 21) return {1, 12};
        if (k <= 31) return {1, 16};
        if (k <= 44) return {1, 32};
        return {1, 8};
    }
    if (k <= 2) return {0, 16};
    if (k <= 6) return {3, 4};
    if (k <= 13) return n < kSmallVector ? ApplyShape{3, 4} : ApplyShape{2, 4};
    if (k <= 17) return {1, 16};
    if (k <= 21) return {2, 4};
    return {1, 8};
}

ApplyShape sync_shape(int k, bool momentum, bool bf16, size_t n) {
    if (!bf16 && n >= kTinyVector && n < kMidVector) {
        if (k <= 27) return small_sync_shape(k, momentum, n);
        if (n < 3000000) return {2, 4};   // 3% (below: 12%)
    }
    // Measured at 138,357,544 fp32 / 200,000,000 bf16 parameters with one
    // gradient per learner, for 4, 8, 12, 16, 20, 24 and 32 learners; the
    // counts between take the next measured one's shape. fp32 steps of one and two
    // learners, and of 17 to 20 without momentum, also from packed odd rows and at 17M
    // and 61M (17M, two with momentum: 66 us with four blocks, 77 with two; 61M, 20
    // without: 823-907, 872-952 with one block and groups of 16).
    if (!bf16 && k <= 2) return momentum || k == 2 ? ApplyShape{4, 16} : ApplyShape{0, 16};
    if (bf16) {
        if (momentum) {
            if (k <= 4) return {3, 16};
            if (k <= 8) return {2, 12};
            if (k <= 12) return {2, 4};
            if (k <= 16) return {1, 16};
            if (k <= 20) return {1, 12};
            if (k <= 24) return {1, 16};
            return {1, 8};
        }
        if (k <= 4) return {3, 4};
        if (k <= 16) return {2, 4};
        return {1, 12};
    }
    if (momentum) {
        if (k <= 4) return {2, 16};
        if (k <= 8) return {2, 4};
        if (k <= 12) return {1, 12};
        if (k <= 16) return {1, 16};
        if (k <= 20) return {1, 12};
        if (k <= 24) return {1, 16};
        return {1, 8};
    }
    if (k <= 4) return {3, 16};
    if (k <= 12) return {2, 4};
    if (k <= 16) return {1, 16};
    if (k <= 20) return {2, 4};
    return {1, 16};
}

bool steps_join(const StepsSize &s, bool momentum, size_t n) {
    if (s.steps < 2) return false;
    const size_t steps = static_cast<size_t>(s.steps);
    const size_t saved = (momentum ? 16 : 8) + 4;
    if (n >= kSmallVector) {
        if (s.grad_bytes + s.pull_bytes + steps * saved > (momentum ? 8 : 6) * steps * saved)
            return false;
    } else if (n >= 4000000 && !momentum) {
        if (s.grad_bytes > 8 * steps * saved && s.pull_bytes < s.grad_bytes) return false;
    }
    if (s.final_bytes * n <= kCacheBytes) return true;
    const size_t all = (steps - 1) * saved + (s.pull_bytes - s.final_bytes);
    return all * (n < kMidVector ? 11 : 7) >= s.grad_bytes + 2 * s.final_bytes;
}

int steps_blocks_per_cu(int replicas, size_t pull_elem, size_t grad_elem, size_t n) {
    const size_t bytes = static_cast<size_t>(replicas) * pull_elem;
    const size_t blocks = n * grad_elem / (16 * 256);   // a lane's chunk: 16 bytes of gradient
    if (blocks <= 512 || (blocks <= 1024 && replicas >= 16)) return 2;
    return bytes <= 8 || (bytes <= 16 && n < 8000000) ? 2 : 1;
}

namespace {
bool fuses_at_any_size(int r, int k, size_t n) {
    return r <= 1 || (r <= 4 && k <= 16) || (r <= 6 && k <= 8 && n < kSmallVector);
}
}  // namespace

bool fuse_replicas(int r, int k, bool bf16, bool fp32_replicas, bool momentum, size_t n) {
    const bool widened = bf16 && fp32_replicas;
    if (fuses_at_any_size(r, k, n))
        return !(widened && !momentum && n >= kMidVector && r > 2 && k > 4);
    if (fp32_replicas && r * n > (widened ? kWidenedFused : kFusedReplicas)) return false;
    return fuse_replicas(r, k, n);
}

bool fuse_replicas(int r, int k, size_t n) {
    if (fuses_at_any_size(r, k, n) || n < kTinyVector) return true;
    if (n < 1500000) return r <= 4 || r * k <= 128;
    return n < 3000000 && r <= 8 && k <= 16;
}

}  // namespace gadei

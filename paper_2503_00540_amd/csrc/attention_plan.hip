// Which kernel takes a bf16 attention launch, and how it splits the keys.  Host code only.
//
// Launches whose 128-row blocks number 512 or more fill the chip (two workgroups per CU) and run on attention_bf16.hip as they
// are.  For the others there are up to four ways, and the one with the least estimated time is taken:
//   wave 1, 2   attention_wave.hip: blocks of 32 or 64 rows, eight or four key runs per workgroup, s splits on top;
//   two groups  attention_bf16.hip, 128-row blocks, two key groups per workgroup, one workgroup per CU, merged by the last arriver;
//   one group   attention_bf16.hip, 128-row blocks of four wavefronts, two workgroups per CU, merged by a second launch.
// The estimates are least-squares fits (no term below zero) to random problems, each timed in every one of the ways and up to nine
// splits, K and V in the caches and from HBM (the mean):
//   more than 32 rows: 2,500 problems with gathered or windowed keys of the heads 14/2/64, 16/8/64, 8/2/128, 28/4/128, 64/8/128,
//     replayed from a graph: live chunks of 1 to 4 frames with windows of 2 to 77, questions of 1 to 32 users over 4 to 64 frames;
//   up to 32 rows: 2,100 decode steps and short questions of those heads and of 1 to 32 KV heads with groups of 1 to 16, 1 to 250
//     users, 64 to 16,000 keys (350 more of up to a million keys count a fifth), replayed and as issued from Python (the mean).
//     A third of the samples are not split: without them the fixed part and the cost of splitting are one column.
// How far from the best measured way the choice is, on 1,100 others of more than 32 rows, nearly half of them of other heads, gathered, in place
// or live: 1.02 on average (95% under 1.14; other heads 1.02 and 1.13), where the estimate that stood here before these, of
// 128-row workgroups of one group against attention_wave.hip alone, was at 1.08 (1.38).  Up to 32 rows, on its own samples: 1.01 and 1.06 to
// 1.07 in each of the three measurements.
// Frames read in place are judged like gathered ones, except at up to 32 rows and where more than 268 MB of them are listed at
// head_dim 64 (see below).
#include "attention_mfma.h"

namespace rekv {
namespace {

constexpr int BM = 128;                   // rows of attention_bf16.hip's blocks
constexpr int WM = 32;                    // and of a row wave
constexpr int WAVES = 8;                  // of attention_wave.hip's workgroups
constexpr int64_t TWO_PER_CU = 512, ONE_PER_CU = 256;

// Microseconds: around everything; per 32-key step of the longest run; per tile of the average run (one at least), more where CUs
// hold two workgroups; where keys are split: once, per split, per size of the partial results; per MB of K and V.  Where only the
// longest run was fitted, it is the average run too.
struct Cost {
    double fixed, step, run, run_of_two, split, per_split, per_size, kv;
};
// [head_dim 64, 128]
constexpr Cost WAVE1_FEW[2] = {{3.635, 0.082, 0.939, 1.360, 2.611, 0.019, 0.110, 0.081}, {4.136, 0.467, 1.614, 0.000, 2.678, 0.000, 0.201, 0.069}};
constexpr Cost ONE_GROUP_FEW[2] = {{4.345, 0.300, 0.000, 0.170, 2.090, 0.018, 0.677, 0.028}, {4.992, 0.430, 0.000, 0.361, 1.698, 0.034, 0.588, 0.041}};
constexpr Cost WAVE1[2] = {{4.282, 0.711, 0.000, 0.683, 1.755, 0.099, 0.081, 0.054}, {5.720, 1.112, 0.000, 0.000, 1.481, 0.089, 0.146, 0.058}};
constexpr Cost WAVE2[2] = {{4.500, 0.721, 0.000, 0.529, 1.152, 0.147, 0.151, 0.030}, {6.328, 1.057, 0.000, 0.000, 0.922, 0.257, 0.140, 0.034}};
constexpr Cost TWO_GROUPS[2] = {{5.500, 0.589, 0.000, 0.000, 1.040, 0.000, 0.485, 0.026}, {8.095, 0.811, 0.000, 0.000, 1.121, 0.000, 0.821, 0.040}};
constexpr Cost ONE_GROUP[2] = {{3.813, 0.479, 0.000, 0.096, 2.045, 0.000, 0.774, 0.035}, {5.761, 0.598, 0.000, 0.158, 1.705, 0.000, 0.544, 0.041}};

double estimate(const Cost& c, int64_t steps, double run, bool two_per_cu, int64_t splits, double size, double kv_mb) {
    double us = c.fixed + (double)steps * c.step + run * (c.run + (two_per_cu ? c.run_of_two : 0.0)) + kv_mb * c.kv;
    if (splits > 1) us += c.split + (double)splits * c.per_split + size * c.per_size;
    return us;
}

constexpr double SPLIT_GAIN = 0.98;
// The most rows of partial results per row block of attention_wave.hip (228 splits of 32 rows, 484 at head_dim 128): more were
// never measured.
constexpr int64_t MOST_SPLIT_ROWS[2] = {7296, 15488};
int64_t up(int64_t n, int64_t d) { return (n + d - 1) / d; }

}  // namespace

AttnPlan attn_bf16_plan(const AttnProblem& p) {
    const int64_t G = p.n_q_heads / p.n_kv_heads, D = p.head_dim, m_rows = p.len_q * G, ik = (int64_t)p.n_items * p.n_kv_heads;
    const int64_t base = ik * up(m_rows, BM);
    const bool few = m_rows <= WM, in_place = p.a_index != nullptr;
    const int d128 = D == 128;
    AttnPlan plan;
    plan.wave = 0;
    plan.n_splits = 1;
    plan.m_tiles = (int32_t)up(m_rows, BM);
    plan.key_groups = 1;
    plan.workspace_bytes = plan.reserve_bytes = 0;
    if (base >= TWO_PER_CU) return plan;

    // The longest tile list of any item; a window counts as far as the stream behind it reaches.
    const int64_t window = p.is_encode ? p.l_l : p.len_a;
    int64_t len_a = window;
    if (p.is_encode) {
        const int64_t past = p.first_token + (int64_t)(p.n_items - 1) * p.len_b;
        if (past < len_a) len_a = past;
    }
    const int64_t tiles_b = up(p.len_b, BN), n_tiles = up(len_a, BN) + tiles_b;
    const int64_t kv_tokens = p.is_encode ? len_a + (int64_t)p.n_items * p.len_b : p.n_items * (len_a + p.len_b);
    const double kv_mb = (double)(kv_tokens * p.n_kv_heads * D) * 4e-6;
    // 128-row blocks: the most splits that still fit one round of resident workgroups (one workgroup more than that costs a
    // whole second round), each of at least 8 tiles, 2 when only one wavefront of four has rows (a decode step).
    const int64_t min_tiles = few ? 2 : 8;
    auto splits_of = [&](int64_t resident, int64_t tiles) {
        const int64_t cap = tiles / min_tiles > 1 ? tiles / min_tiles : 1, s = resident / base;
        return s < cap ? s : cap;
    };
    const size_t block_bytes = (size_t)base * BM * (size_t)(D + 2) * sizeof(float);
    const int64_t reserve = splits_of(TWO_PER_CU, up(window, BN) + tiles_b);
    plan.reserve_bytes = reserve > 1 ? (size_t)reserve * block_bytes : 0;

    struct Way {
        double us;
        int32_t wave, key_groups;
        int64_t splits, row_blocks;
        size_t bytes;
    };
    constexpr double NONE = 1e30;
    // attention_wave.hip.  Beyond what the last-level cache holds a launch is bound by HBM, where the 128-row kernel's three
    // tiles of prefetch count (102 shapes of more than 32 rows above this line took 1.0 to 1.13 times its time on average).  Frames
    // read in place are fewer than their count, questions share them: on 80 such calls of head_dim 64 and more than 32 rows the choice
    // without the line takes 1.005 of the best way's time, with it 1.09 and up to 1.6 (at head_dim 128 the line changes nothing).
    // Resident workgroups: LDS holds one (D = 128) or two per CU.
    const int64_t slots = D == 64 ? TWO_PER_CU : ONE_PER_CU;
    auto wave = [&](int rw) {
        Way best = {NONE, rw, 1, 1, 1, 0};
        const int64_t T = rw * WM, kg = WAVES / rw, row_blocks = up(m_rows, T), blocks = ik * row_blocks, rows = m_rows < T ? m_rows : T;
        if (blocks > slots || ((few || !in_place) && kv_mb > 268.0)) return best;
        const Cost& c = few ? WAVE1_FEW[d128] : rw == 1 ? WAVE1[d128] : WAVE2[d128];
        const size_t split_bytes = (size_t)blocks * T * (size_t)(D + 2) * sizeof(float);
        // K and V that no cache holds, as after a reload, come with little in flight.  372 gathered calls from HBM that the term was not
        // chosen on: 0.952 of the time of the estimate before these with it, 0.962 without (14 of them over 10% longer, 2 with it);
        // with K and V in the caches 0.953 with it and 0.940 without.
        const double cold_us = few || kv_mb <= 8.0 ? 0.0 : (kv_mb - 8.0) * (D == 64 ? 0.06 : 0.15);
        // the fewest splits for every number of steps; more splits have to gain 2%
        for (int64_t s = 1, steps; s <= slots / blocks; s = up(n_tiles, kg * (steps - 1))) {
            steps = up(n_tiles, s * kg);
            if (s > 1 && ((size_t)s * split_bytes > plan.reserve_bytes || s * T > MOST_SPLIT_ROWS[d128])) break;
            const double run = few ? fmax(1.0, (double)n_tiles / (double)(s * kg)) : (double)steps;
            const double us = estimate(c, steps, run, blocks * s > ONE_PER_CU, s, (double)(s * rows * D) * 4e-4, kv_mb) + cold_us;
            if (us < SPLIT_GAIN * best.us) best = Way{us, rw, 1, s, row_blocks, (size_t)s * split_bytes};
            if (steps == 1) break;
        }
        return best;
    };
    const int64_t m_tiles = up(m_rows, BM);
    auto two_groups = [&] {
        if (few || base > ONE_PER_CU) return Way{NONE, 0, 2, 1, m_tiles, 0};
        const int64_t s = splits_of(ONE_PER_CU, n_tiles), steps = up(n_tiles, 2 * s);
        return Way{estimate(TWO_GROUPS[d128], steps, (double)steps, false, s, (double)(s * (m_rows < BM ? m_rows : BM)) / BM, kv_mb),
                   0, 2, s, m_tiles, (size_t)s * block_bytes};
    };
    auto one_group = [&] {
        const int64_t s = splits_of(TWO_PER_CU, n_tiles), steps = up(n_tiles, s);
        return Way{estimate(few ? ONE_GROUP_FEW[d128] : ONE_GROUP[d128], steps, (double)steps, base * s > ONE_PER_CU, s,
                            (double)(ik * s * m_rows * D) * 4e-6, kv_mb),
                   0, 1, s, m_tiles, (size_t)s * block_bytes};
    };
    Way best;
    auto consider = [&](const Way& w, double gain) { if (w.us < gain * best.us) best = w; };
    if (few) {
        // (25 to 32 rows of head_dim 64 over two to six pairs of item and KV head, split either way: from level, 8.0 and 8.2 us for
        // 16/2/64 over 4,000 keys, to a gain of 14%; only more than that counts, so that these stay where their results were)
        const Way w1 = wave(1);
        const bool level = D == 64 && m_rows > 24 && ik > 1 && ik <= 6 && w1.splits > 1;
        // (in place every lane of a 128-row workgroup looks up its frame: 1.09 to 1.10 of the estimate on 1,500 such calls, the split-key
        // kernel 0.99 to 1.04.  With the factor the choice takes 1.004 to 1.008 of the best way's time on them, without 1.011 to 1.021)
        best = one_group();
        consider(w1, (level ? 0.80 : 1.0) * (in_place ? 1.1 : 1.0));
    } else {
        best = two_groups();
        const Way w1 = wave(1), w2 = wave(2);
        // (both split at head_dim 128: 64-row blocks halve the traffic of tiles, and 256 workgroups of either are within 5 to 7%)
        const double gain = D == 128 && w1.splits > 1 && w2.splits > 1 ? 0.90 : 0.97;
        consider(w1.us < gain * w2.us ? w1 : w2, 0.98);
        consider(one_group(), 0.98);
    }
    plan.wave = best.wave;
    plan.n_splits = (int32_t)best.splits;
    plan.m_tiles = (int32_t)best.row_blocks;
    plan.key_groups = best.key_groups;
    plan.workspace_bytes = best.splits > 1 ? best.bytes : 0;
    return plan;
}

}  // namespace rekv

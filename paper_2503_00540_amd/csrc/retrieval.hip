// Internal retrieval: frame vectors (mean key per frame), pooled question vector, Eq. 2
// cosine scores with tau = 1, and exact top-k selection.  All of it is memory-bound: the
// kernels read each input once with 16-byte coalesced accesses and keep reductions in
// registers / wavefront shuffles.
#include <type_traits>

#include "common.h"

namespace rekv {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int I>
using IC = std::integral_constant<int, I>;

// 16-byte load that is not kept in the caches (a table row is read once per pass)
__device__ inline float4 load_stream(const float* p) {
    const f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p));
    return make_float4(v.x, v.y, v.z, v.w);
}

__device__ inline float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ inline float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

__device__ inline float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// ---------------------------------------------------------------------------------------
// Frame vectors: v_f = (1/N_f) sum_j k_{f,j}, heads concatenated.
// A workgroup streams a slab of columns of one frame (a contiguous N_f x D' block): LPR lanes cover the
// slab's row with 16-byte loads (8 bf16 or 4 fp32 each), the 256 / LPR row groups take alternate rows, and their
// partial sums meet in LDS.  A thread's loads leave together, up to eight, and the rows that are left over as one
// batch of just as many (the last row read twice where a row group has one less): each turn of a loop costs a memory round
// trip, and with few frames those are the whole time.  Hence also the slab: 128 bytes wide, 32 row groups, one
// or two batches per thread (mean_rows_launch).  The last frame may be short (n_rows in all; a stream's last block of
// frames).  Many frames are bound by HBM.  Measured with whole rows per workgroup and a loop over the left-over rows, then
// so (us, replayed from a graph; keys in the caches / from HBM): one frame of 196 x 512 4.4 / 6.6 -> 2.4 / 2.4, of 196 x 128 2.7 / 4.3 ->
// 2.2 / 2.6, 64 frames of 196 x 512 7.5 / 8.3 -> 3.4 / 4.7, 256 of them 8.9 / 11.0 -> 7.8 / 10.0 (5.2 TB/s).
// ---------------------------------------------------------------------------------------
// ONE: a frame has no more rows than there are row groups (block vectors, tiny frames): less code to fetch.
template <bool BF16, bool ONE>
__global__ __launch_bounds__(256) void frame_keys_kernel(const void* __restrict__ k, int n_f_all, int64_t n_rows,
                                                         int d_prime, int lpr_log2,
                                                         float* __restrict__ out) {
    constexpr int VEC = BF16 ? 8 : 4;
    constexpr int ES = BF16 ? 2 : 4;
    __shared__ __attribute__((aligned(16))) float red[256 * VEC];    // [row group][column of the slab]
    __shared__ float part[256];
    const int lpr = 1 << lpr_log2, n_rg = 256 >> lpr_log2;
    const int cl = threadIdx.x & (lpr - 1), rg = threadIdx.x >> lpr_log2;
    const int col = (blockIdx.y * lpr + cl) * VEC;
    const int64_t frame = blockIdx.x, row0 = frame * n_f_all;
    const int n_f = n_rows - row0 < n_f_all ? (int)(n_rows - row0) : n_f_all;
    float acc[VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] = 0.f;
    if (col < d_prime) {
        const char* base = static_cast<const char*>(k) + (row0 * (int64_t)d_prime + col) * ES;
        const int64_t pitch = (int64_t)d_prime * ES;
        auto add = [&](const u32x4& w, bool on) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (BF16) {
                    acc[2 * i] += on ? bf16_lo(w[i]) : 0.f;
                    acc[2 * i + 1] += on ? bf16_hi(w[i]) : 0.f;
                } else {
                    acc[i] += on ? __uint_as_float(w[i]) : 0.f;
                }
            }
        };
        // n loads that leave together; where rows may be missing, the last one is read again and its values left out
        auto batch = [&](int j, auto n, auto whole) __attribute__((always_inline)) {
            constexpr int U = decltype(n)::value;
            constexpr bool WHOLE = decltype(whole)::value;
            u32x4 w[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int r = j + n_rg * u;
                w[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(base + (WHOLE || r < n_f ? r : n_f - 1) * pitch));
            }
#pragma unroll
            for (int u = 0; u < U; ++u) add(w[u], WHOLE || j + n_rg * u < n_f);
        };
        if constexpr (ONE) {
            if (rg < n_f) batch(rg, IC<1>(), std::true_type());
        } else {
            int j0 = 0;                              // rows before j0 are in
            for (; j0 + n_rg * 8 <= n_f; j0 += n_rg * 8) batch(j0 + rg, IC<8>(), std::true_type());
            const auto some = std::false_type();
            switch ((n_f - j0 + n_rg - 1) / n_rg) {  // the rows that are left, per row group
                case 8: batch(j0 + rg, IC<8>(), some); break;
                case 7: batch(j0 + rg, IC<7>(), some); break;
                case 6: batch(j0 + rg, IC<6>(), some); break;
                case 5: batch(j0 + rg, IC<5>(), some); break;
                case 4: batch(j0 + rg, IC<4>(), some); break;
                case 3: batch(j0 + rg, IC<3>(), some); break;
                case 2: batch(j0 + rg, IC<2>(), some); break;
                case 1: batch(j0 + rg, IC<1>(), some); break;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < VEC; ++i) red[threadIdx.x * VEC + i] = acc[i];
    __syncthreads();
    const int cols = lpr * VEC;                      // of the slab
    auto write = [&](int c, float sum) {
        const int oc = blockIdx.y * cols + c;
        if (oc < d_prime) out[frame * d_prime + oc] = sum / (float)n_f;
    };
    const int n_used = n_f < n_rg ? n_f : n_rg;      // row groups that had a row
    if (cols >= 256 || n_used <= 16) {
        for (int c = threadIdx.x; c < cols; c += 256) {
            float sum = 0.f;
            for (int g = 0; g < n_used; ++g) sum += red[g * cols + c];
            write(c, sum);
        }
        return;
    }
    // few columns, many row groups: VEC of them per thread, then those sums
    const int c = threadIdx.x & (cols - 1), pt = threadIdx.x / cols;
    float sum = 0.f;
#pragma unroll
    for (int g = 0; g < VEC; ++g) sum += red[(pt * VEC + g) * cols + c];
    part[threadIdx.x] = sum;
    __syncthreads();
    if (threadIdx.x < cols) {
        sum = 0.f;
        for (int g = 0; g < 256 / cols; ++g) sum += part[g * cols + c];
        write(c, sum);
    }
}

// ---------------------------------------------------------------------------------------
// Question vector (the mean of the question's N_q query vectors; the G query heads of a KV
// group averaged so that the vector has D' = Hkv * D entries, like a frame vector).
// One workgroup per (question, KV group, 128 bytes of a head vector): 8 lanes cover those bytes of a
// head, the G heads lie side by side and the threads that are left take further token rows.  A
// thread's loads leave together, up to 16 of them (the rows past the end are masked, not looped
// over one by one: each turn of such a loop costs a memory round trip).  What bounds it is that one
// round trip: 28 questions of 48 tokens 8.9 us with a workgroup per (question, KV group) and a loop over the
// last 8 rows, 4.2 so.  Many questions that the caches hold are slower this way: 64 of 32 tokens at 64/8/128 (33.5 MB) 7.7
// and 10.2 (the retrieval they are part of 29.9 and 28.1 warm, 33.0 and 30.7 from HBM, with its other kernels' changes).
// ---------------------------------------------------------------------------------------
constexpr int POOL_THREADS = 512;
constexpr int POOL_LANES = 8;                  // 16-byte lanes per head

template <bool BF16>
__global__ __launch_bounds__(POOL_THREADS) void pool_question_kernel(const void* __restrict__ q, int n_q_tokens, int hq,
                                                                     int hkv, int d, float* __restrict__ q_vec) {
    constexpr int VEC = BF16 ? 8 : 4;
    constexpr int ES = BF16 ? 2 : 4;
    constexpr int COLS = POOL_LANES * VEC;           // columns of this workgroup
    constexpr int PARTS = POOL_THREADS / COLS;
    __shared__ float red[POOL_THREADS * VEC];        // [thread / 8][column]
    __shared__ float part[PARTS][COLS];
    const int g_sz = hq / hkv;
    const int gw = g_sz < POOL_THREADS / POOL_LANES ? g_sz : POOL_THREADS / POOL_LANES;   // heads side by side
    const int n_rg = POOL_THREADS / (POOL_LANES * gw);                                    // row groups
    const int lane8 = threadIdx.x % POOL_LANES, slot = threadIdx.x / POOL_LANES;
    const int gl = slot % gw, rg = slot / gw;
    const int64_t pitch = (int64_t)hq * d * ES;
    const int col = (blockIdx.z * POOL_LANES + lane8) * VEC;
    float acc[VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] = 0.f;
    if (rg < n_rg && col < d) {
        for (int g = gl; g < g_sz; g += gw) {
            const char* base = static_cast<const char*>(q) + (int64_t)blockIdx.x * n_q_tokens * pitch +
                               ((int64_t)(blockIdx.y * g_sz + g) * d + col) * ES;
            constexpr int U = 16;
            for (int j0 = rg; j0 < n_q_tokens; j0 += n_rg * U) {
                u32x4 w[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    w[u] = u32x4{0u, 0u, 0u, 0u};
                    if (j0 + n_rg * u < n_q_tokens) w[u] = *reinterpret_cast<const u32x4*>(base + (j0 + n_rg * u) * pitch);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if (BF16) {
                            acc[2 * i] += bf16_lo(w[u][i]);
                            acc[2 * i + 1] += bf16_hi(w[u][i]);
                        } else {
                            acc[i] += __uint_as_float(w[u][i]);
                        }
                    }
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < VEC; ++i) red[threadIdx.x * VEC + i] = acc[i];
    __syncthreads();
    const int cc = threadIdx.x % COLS, pt = threadIdx.x / COLS;
    float sum = 0.f;
#pragma unroll
    for (int e = 0; e < POOL_THREADS / POOL_LANES / PARTS; ++e) sum += red[(pt + e * PARTS) * COLS + cc];
    part[pt][cc] = sum;
    __syncthreads();
    const int dd = blockIdx.z * COLS + threadIdx.x;
    if (threadIdx.x < COLS && dd < d) {
        sum = 0.f;
#pragma unroll
        for (int e = 0; e < PARTS; ++e) sum += part[e][threadIdx.x];
        q_vec[((int64_t)blockIdx.x * hkv + blockIdx.y) * d + dd] = sum * (1.f / ((float)g_sz * (float)n_q_tokens));
    }
}

// Sums v[i] over the 64 lanes for all i at once.  Returns, in every lane, the total of the
// value whose index is the lane's top log2(N) bits (lane >> (6 - log2 N)).
template <int N>
__device__ inline float transpose_reduce(float (&v)[N], int lane) {
    int n = N;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        if (n > 1) {
            const int half = n / 2;
            const bool up = (lane & off) != 0;
#pragma unroll
            for (int i = 0; i < half; ++i) {
                const float keep = up ? v[i + half] : v[i];
                const float send = up ? v[i] : v[i + half];
                v[i] = keep + __shfl_xor(send, off);
            }
            n = half;
        } else {
            v[0] += __shfl_xor(v[0], off);
        }
    }
    return v[0];
}

// ---------------------------------------------------------------------------------------
// Exact top-k of one question's scores.  Scores become order-preserving 32-bit keys; a
// 4-pass radix select (8 bits per pass, histogram in LDS) finds the k-th largest key T;
// then one ordered pass over the frames writes, in ascending frame index, every frame with
// key > T and the first (k - count) frames with key == T - the lower index wins ties.
// One block per question.
// ---------------------------------------------------------------------------------------
constexpr int TOPK_THREADS = 256;

__device__ inline uint32_t order_key(float s) {
    uint32_t u = __float_as_uint(s);
    if (u == 0x80000000u) u = 0u;          // -0 and +0 are the same score
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// exclusive scan over the block of two counts per thread, packed into one 64-bit value
// (high word, low word); returns this thread's prefix and the block total through `total`
__device__ inline uint64_t block_excl_scan(uint64_t v, uint64_t* wave_tot, uint64_t& total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint64_t inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint64_t n = __shfl_up(inc, o);
        if (lane >= o) inc += n;
    }
    __syncthreads();                       // wave_tot may still be read from the last call
    if (lane == 63) wave_tot[wave] = inc;
    __syncthreads();
    uint64_t before = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < TOPK_THREADS / 64; ++w) {
        const uint64_t t = wave_tot[w];
        if (w < wave) before += t;
        total += t;
    }
    return before + inc - v;
}

// The whole block works on one question: s its n_frames scores, out its k index slots, n_sel_q
// its count (may be NULL).
__device__ inline void topk_block(const float* s, int n_frames, int k, int32_t* out, int32_t* n_sel_q) {
    // Scores of one question cluster in a few exponent bins, so a single histogram would serialise
    // its LDS atomics on one address: threads spread over NSUB copies, and each thread first adds
    // up runs of equal bins among its own keys.
    // The kernel runs once per question on cold instruction caches, so its loops stay rolled: the
    // code is a few hundred instructions, not thousands.
    constexpr int NSUB = 8;
    constexpr int SPAN = 16;               // consecutive frames a thread owns in the ordered sweep
    __shared__ int hist[NSUB][256];
    __shared__ __attribute__((aligned(16))) uint32_t keys[SPAN * TOPK_THREADS];
    __shared__ uint64_t wave_tot[TOPK_THREADS / 64];
    __shared__ uint32_t sh_prefix;
    __shared__ int sh_need;
    const int tid = threadIdx.x;

    if (k >= n_frames) {                   // everything is selected
        for (int f = tid; f < k; f += TOPK_THREADS) out[f] = f < n_frames ? f : -1;
        if (tid == 0 && n_sel_q) *n_sel_q = n_frames;
        return;
    }

    // Up to 4096 frames the keys live in LDS (frame f at [f % SPAN][f / SPAN], which both the
    // strided and the owner-contiguous access below reach without bank conflicts), so the scores
    // cross the memory system once instead of once per pass.
    const bool resident = n_frames <= TOPK_THREADS * SPAN;
    if (resident) {
#pragma unroll 1
        for (int f = tid; f < n_frames; f += TOPK_THREADS)
            keys[(f % SPAN) * TOPK_THREADS + f / SPAN] = order_key(s[f]);
        __syncthreads();
    }
    auto key_at = [&](int f) -> uint32_t {
        return resident ? keys[(f % SPAN) * TOPK_THREADS + f / SPAN] : order_key(s[f]);
    };

    uint32_t prefix = 0;                   // high bits of T found so far
    int need = k;                          // rank of T among keys matching the prefix
#pragma unroll 1
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
#pragma unroll 1
        for (int sub = 0; sub < NSUB; ++sub) hist[sub][tid] = 0;    // TOPK_THREADS == 256 bins
        __syncthreads();
        const uint32_t hi_mask = pass ? (0xFFFFFFFFu << (shift + 8)) : 0u;
        int* my_hist = hist[tid % NSUB];
        int run_bin = -1, run_len = 0;
#pragma unroll 1
        for (int f = tid; f < n_frames; f += TOPK_THREADS) {
            const uint32_t key = key_at(f);
            if ((key & hi_mask) != prefix) continue;
            const int bin = (int)((key >> shift) & 255u);
            if (bin == run_bin) {
                ++run_len;
            } else {
                if (run_len) atomicAdd(&my_hist[run_bin], run_len);
                run_bin = bin;
                run_len = 1;
            }
        }
        if (run_len) atomicAdd(&my_hist[run_bin], run_len);
        __syncthreads();
        // bin b is chosen iff (#keys in bins above b) < need <= (#keys in bins >= b)
        int mine = 0;
#pragma unroll 1
        for (int sub = 0; sub < NSUB; ++sub) mine += hist[sub][tid];
        uint64_t total;
        const int below = (int)block_excl_scan((uint64_t)mine, wave_tot, total);   // keys in bins < tid
        const int above = (int)total - below - mine;
        if (above < need && need <= above + mine) {
            sh_prefix = prefix | ((uint32_t)tid << shift);
            sh_need = need - above;
        }
        __syncthreads();
        prefix = sh_prefix;
        need = sh_need;
        __syncthreads();
    }
    const uint32_t T = prefix;             // the k-th largest key; `need` of its copies are taken

    // ordered sweep: a thread owns SPAN consecutive frames, so one block scan orders 4096 frames
    int base_gt = 0, base_eq = 0;          // frames above T / equal to T before this sweep
#pragma unroll 1
    for (int f0 = 0; f0 < n_frames; f0 += TOPK_THREADS * SPAN) {
        const int fa = f0 + tid * SPAN;
        uint32_t gt_mask = 0, eq_mask = 0;
#pragma unroll 1
        for (int i = 0; i < SPAN; ++i)
            if (fa + i < n_frames) {
                const uint32_t key = key_at(fa + i);
                gt_mask |= (uint32_t)(key > T) << i;
                eq_mask |= (uint32_t)(key == T) << i;
            }
        uint64_t tot;
        const uint64_t pre = block_excl_scan(((uint64_t)__popc(gt_mask) << 32) | (uint64_t)__popc(eq_mask),
                                             wave_tot, tot);
        int n_gt = base_gt + (int)(pre >> 32), n_eq = base_eq + (int)(pre & 0xFFFFFFFFu);
#pragma unroll 1
        for (int i = 0; i < SPAN; ++i) {
            const bool gt = (gt_mask >> i) & 1, eq = (eq_mask >> i) & 1;
            if (gt || (eq && n_eq < need)) out[n_gt + (n_eq < need ? n_eq : need)] = fa + i;
            n_gt += gt;
            n_eq += eq;
        }
        base_gt += (int)(tot >> 32);
        base_eq += (int)(tot & 0xFFFFFFFFu);
    }
    if (tid == 0 && n_sel_q) *n_sel_q = k;
}

// ---------------------------------------------------------------------------------------
// Top-k for the common sizes (257..4096 frames, k <= 64) without a radix select: few phases,
// each one pass over registers or a short LDS list.
//   1. 1024 threads hold up to 4 keys each; frame f belongs to group f mod 128, so all of a
//      thread's keys are in group (thread mod 128) and every group is non-empty.
//   2. The 128 group maxima are 128 different frames, so the k-th largest of them, T0, is a lower
//      bound of the k-th largest key overall: every frame of the answer has key >= T0.
//      Typically fewer than 2k frames pass that test.
//   3. The survivors are ranked among themselves by (key descending, frame ascending) - all
//      pairs, spread over the 1024 threads - and those of rank < k are the answer, exactly,
//      ties going to the lower frame.  One wavefront puts them in ascending frame order.
// Many equal keys at the cut only make the survivor list longer (all-pairs work grows with
// its square), never wrong.  One workgroup per question.
// ---------------------------------------------------------------------------------------
constexpr int SEL_GROUPS = 128;
constexpr int SEL_MAX_FRAMES = 4096;
constexpr int SEL_MAX_K = 64;
constexpr int SEL_MIN_FRAMES = 257;

template <int SEL_THREADS>      // a multiple of 128 that divides 4096
__global__ __launch_bounds__(SEL_THREADS) void topk_groupmax_kernel(const float* __restrict__ scores,
                                                                   int n_frames, int k,
                                                                   int32_t* __restrict__ idx,
                                                                   int32_t* __restrict__ n_sel) {
    // a candidate is one 64-bit word: key in the high half, ~frame in the low half, so that a
    // larger word means "ranks before" (higher key, or equal key and lower frame)
    __shared__ uint32_t gmax[SEL_GROUPS];
    __shared__ __attribute__((aligned(16))) uint64_t cand[SEL_MAX_FRAMES];
    __shared__ int32_t rank_of[SEL_MAX_FRAMES];
    __shared__ __attribute__((aligned(16))) int32_t sel[SEL_MAX_K];
    __shared__ uint32_t sh_t0;
    __shared__ int32_t n_cand, n_taken;
    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t qi = blockIdx.x;
    const float* s = scores + qi * n_frames;
    int32_t* out = idx + qi * k;

    constexpr int KPT = SEL_MAX_FRAMES / SEL_THREADS;      // keys per thread
    uint32_t key[KPT];
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
        const int f = tid + j * SEL_THREADS;
        key[j] = f < n_frames ? order_key(s[f]) : 0u;        // 0 lies below the key of every number
    }
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
        rank_of[tid + j * SEL_THREADS] = 0;
        cand[tid + j * SEL_THREADS] = 0;                     // ranks before no candidate
    }
    if (tid < SEL_MAX_K) sel[tid] = 0x7FFFFFFF;
    if (tid < SEL_GROUPS) gmax[tid] = 0u;
    if (tid == 0) { n_cand = 0; n_taken = 0; }
    __syncthreads();
    uint32_t mine = key[0];
#pragma unroll
    for (int j = 1; j < KPT; ++j) mine = max(mine, key[j]);
    atomicMax(&gmax[tid & (SEL_GROUPS - 1)], mine);          // tid mod 128 == the group of all its keys
    __syncthreads();
    {                                                        // rank of every group's maximum, a slice of the others per thread
        constexpr int SLICE_G = SEL_GROUPS * SEL_GROUPS / SEL_THREADS;
        const int g = tid & (SEL_GROUPS - 1), j0 = tid / SEL_GROUPS * SLICE_G;
        const uint32_t v = gmax[g];
        int above = 0;
#pragma unroll
        for (int j = j0; j < j0 + SLICE_G; ++j) {
            const uint32_t o = gmax[j];                      // same address in every lane: a broadcast
            above += (o > v) || (o == v && j < g);
        }
        atomicAdd(&rank_of[g], above);
    }
    __syncthreads();
    if (tid < SEL_GROUPS) {
        if (rank_of[tid] == k - 1) sh_t0 = gmax[tid];
        rank_of[tid] = 0;
    }
    __syncthreads();
    const uint32_t t0 = sh_t0;
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
        const int f = tid + j * SEL_THREADS;
        const bool pass = f < n_frames && key[j] >= t0;
        const uint64_t mask = __builtin_amdgcn_ballot_w64(pass);
        if (mask != 0) {                                     // wave-uniform
            int base = 0;
            if (lane == 0) base = atomicAdd(&n_cand, __popcll(mask));
            base = __builtin_amdgcn_readfirstlane(base);
            if (pass) {
                const int slot = base + __popcll(mask & ((1ull << lane) - 1ull));
                cand[slot] = ((uint64_t)key[j] << 32) | (uint32_t)~f;
            }
        }
    }
    __syncthreads();
    const int n = n_cand;                                    // k <= n <= n_frames
    // all pairs: candidate i against the candidates of slice sl; a wavefront's lanes share the slice
    const int n_up = (n + 63) & ~63;
    const int n_slices = n_up < SEL_THREADS ? SEL_THREADS / n_up : 1;
    const int sl = __builtin_amdgcn_readfirstlane(tid / n_up);
    if (sl < n_slices) {
        // slices in whole groups of eight: the last one reads into the zeros behind the list
        const int n8 = (n + 7) >> 3, j0 = n8 * sl / n_slices * 8, j1 = n8 * (sl + 1) / n_slices * 8;
        for (int i = tid - sl * n_up; i < n; i += SEL_THREADS) {
            const uint64_t ci = cand[i];
            int above = 0;
            for (int j = j0; j < j1; j += 8) {
                uint64_t c[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) c[u] = cand[j + u];
#pragma unroll
                for (int u = 0; u < 8; ++u) above += c[u] > ci;
            }
            if (n_slices > 1) atomicAdd(&rank_of[i], above);
            else rank_of[i] = above;
        }
    }
    __syncthreads();
    for (int i = tid; i < n; i += SEL_THREADS)
        if (rank_of[i] < k) sel[atomicAdd(&n_taken, 1)] = (int32_t)~(uint32_t)cand[i];    // exactly k of them
    __syncthreads();
    if (tid < k) {
        const int32_t f = sel[tid];
        // all 64 places (those past k hold no frame): reads that leave together, where a loop over k would wait for each
        const int4* sel4 = reinterpret_cast<const int4*>(sel);
        int before = 0;
#pragma unroll
        for (int j = 0; j < SEL_MAX_K / 4; ++j) {
            const int4 o = sel4[j];
            before += (o.x < f) + (o.y < f) + (o.z < f) + (o.w < f);
        }
        out[before] = f;
    }
    if (tid == 0 && n_sel) n_sel[qi] = k;
}

// ---------------------------------------------------------------------------------------
// Top-k of up to 256 frames: the rank of every frame by (key descending, frame ascending) counted
// against all others, the pairs spread over 1024 threads, and the frames of rank < k written in order.
// One workgroup per question.  Bound by the comparisons' issue slots and the one round trip for the scores:
// 256 frames 4.7 us with one thread per frame, 4.0 us so.
// ---------------------------------------------------------------------------------------
constexpr int RANK_MAX_FRAMES = 256;
constexpr int RANK_THREADS = 1024;

// The whole workgroup works on one question: score(f) its scores, out its k index slots, n_sel_q its count (may be NULL).
template <class Score>
__device__ inline void rank_block(Score score, int n_frames, int k, int32_t* out, int32_t* n_sel_q) {
    __shared__ uint64_t cand[RANK_MAX_FRAMES];               // key in the high half, ~frame in the low half
    __shared__ int32_t rank_of[RANK_MAX_FRAMES];
    __shared__ uint64_t taken[RANK_MAX_FRAMES / 64];
    const int tid = threadIdx.x;
    if (tid < RANK_MAX_FRAMES) {
        cand[tid] = tid < n_frames ? ((uint64_t)order_key(score(tid)) << 32) | (uint32_t)~tid : 0u;
        rank_of[tid] = 0;
    }
    __syncthreads();
    const int n_up = (n_frames + 63) & ~63;                  // threads per slice of the others, whole waves
    const int n_slices = RANK_THREADS / n_up;
    const int sl = __builtin_amdgcn_readfirstlane(tid / n_up), i = tid - sl * n_up;
    if (sl < n_slices) {
        const int n8 = (n_frames + 7) >> 3, j0 = n8 * sl / n_slices * 8, j1 = n8 * (sl + 1) / n_slices * 8;
        const uint64_t ci = cand[i];
        int above = 0;
        for (int j = j0; j < j1; j += 8) {
            uint64_t c[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) c[u] = cand[j + u];
#pragma unroll
            for (int u = 0; u < 8; ++u) above += c[u] > ci;
        }
        atomicAdd(&rank_of[i], above);
    }
    __syncthreads();
    const bool take = tid < n_frames && rank_of[tid & (RANK_MAX_FRAMES - 1)] < k;
    const uint64_t mask = __builtin_amdgcn_ballot_w64(take);
    if (tid < RANK_MAX_FRAMES && (tid & 63) == 0) taken[tid >> 6] = mask;
    __syncthreads();
    if (take) {
        int pos = __popcll(mask & ((1ull << (tid & 63)) - 1ull));
#pragma unroll
        for (int w = 0; w < RANK_MAX_FRAMES / 64; ++w) pos += w < (tid >> 6) ? __popcll(taken[w]) : 0;
        out[pos] = tid;
    }
    if (tid == 0 && n_sel_q) *n_sel_q = k;
}

__global__ __launch_bounds__(RANK_THREADS) void topk_rank_kernel(const float* __restrict__ scores, int n_frames, int k,
                                                                 int32_t* __restrict__ idx, int32_t* __restrict__ n_sel) {
    const int64_t qi = blockIdx.x;
    const float* s = scores + qi * n_frames;
    rank_block([&](int f) { return s[f]; }, n_frames, k, idx + qi * k, n_sel ? n_sel + qi : nullptr);
}

__global__ __launch_bounds__(TOPK_THREADS) void topk_kernel(const float* __restrict__ scores,
                                                            int n_frames, int k,
                                                            int32_t* __restrict__ idx,
                                                            int32_t* __restrict__ n_sel) {
    const int64_t qi = blockIdx.x;
    topk_block(scores + qi * n_frames, n_frames, k, idx + qi * k, n_sel ? n_sel + qi : nullptr);
}


// ---------------------------------------------------------------------------------------
// Eq. 2, one question per pass over a table (a question with its own table, or few questions
// on a shared one): a wavefront takes FR frame rows at a time, the lanes split the D' columns,
// 16-byte loads of the rows and of the question vector are all issued before the first use,
// and a transposing butterfly leaves each row's dot product and squared norm in one lane.
// grid = (frame groups, questions).
// ---------------------------------------------------------------------------------------
constexpr int SCORE_WAVES = 4;
constexpr int SCORE_FR = 8;

// NI > 0: D' <= NI * 256 and the column loop is unrolled NI times, so that all of a row group's
// loads are in flight at once; NI = 0: any D'.
template <int NI>
__global__ __launch_bounds__(SCORE_WAVES * 64) void score_rows_kernel(
    const float* __restrict__ frame_keys, int64_t fk_stride, int n_frames, int d_prime,
    const float* __restrict__ q_vec, float inv_tau, float* __restrict__ scores) {
    constexpr int FR = SCORE_FR;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int qi = blockIdx.y;
    const float* table = frame_keys + (int64_t)qi * fk_stride;
    const float* qv = q_vec + (int64_t)qi * d_prime;
    for (int f0 = (blockIdx.x * SCORE_WAVES + wave) * FR; f0 < n_frames; f0 += gridDim.x * SCORE_WAVES * FR) {
        float acc[FR], vv[FR], qq = 0.f;
#pragma unroll
        for (int i = 0; i < FR; ++i) acc[i] = vv[i] = 0.f;
        const float* vrow[FR];
#pragma unroll
        for (int fr = 0; fr < FR; ++fr) {
            const int f = f0 + fr < n_frames ? f0 + fr : n_frames - 1;   // tail: re-read the last frame
            vrow[fr] = table + (int64_t)f * d_prime;
        }
        auto fold = [&](const float4 (&x)[FR], const float4& y) {
            qq += y.x * y.x + y.y * y.y + y.z * y.z + y.w * y.w;
#pragma unroll
            for (int fr = 0; fr < FR; ++fr) {
                vv[fr] += x[fr].x * x[fr].x + x[fr].y * x[fr].y + x[fr].z * x[fr].z + x[fr].w * x[fr].w;
                acc[fr] += x[fr].x * y.x + x[fr].y * y.y + x[fr].z * y.z + x[fr].w * y.w;
            }
        };
        if (NI > 0) {
            float4 x[NI > 0 ? NI : 1][FR], y[NI > 0 ? NI : 1];
#pragma unroll
            for (int it = 0; it < NI; ++it) {
                const int i = lane * 4 + it * 256;
                const bool on = i < d_prime;
                y[it] = on ? *reinterpret_cast<const float4*>(qv + i) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                for (int fr = 0; fr < FR; ++fr) x[it][fr] = on ? load_stream(vrow[fr] + i) : make_float4(0.f, 0.f, 0.f, 0.f);
            }
#pragma unroll
            for (int it = 0; it < NI; ++it) fold(x[it], y[it]);
        } else {
            for (int i = lane * 4; i < d_prime; i += 256) {
                float4 x[FR];
#pragma unroll
                for (int fr = 0; fr < FR; ++fr) x[fr] = load_stream(vrow[fr] + i);
                fold(x, *reinterpret_cast<const float4*>(qv + i));
            }
        }
        const float dsum = transpose_reduce<FR>(acc, lane);
        const float vsum = transpose_reduce<FR>(vv, lane);
        qq = wave_sum(qq);
        const int fr = lane >> 3;
        if ((lane & 7) == 0 && f0 + fr < n_frames) {
            const float den = sqrtf(vsum) * sqrtf(qq);
            scores[(int64_t)qi * n_frames + f0 + fr] = den > 0.f ? dsum / den * inv_tau : 0.f;
        }
    }
}

// ---------------------------------------------------------------------------------------
// Eq. 2, many questions on one table: a skinny fp32 matrix product, still bound by the table's
// bytes.  A workgroup owns a tile of 32 frames x 32 questions.  Slabs of 128 columns of the
// table rows and of the question vectors are staged in LDS with row-contiguous loads (the next
// slab travels into registers while the current one is used); its 8 wavefronts each take 16
// of the slab's columns and run fp32 MFMAs (v_mfma_f32_32x32x2_f32: full fp32 products, fp32
// sums) on operands read with one 16-byte LDS read per four MFMAs: lane (r, h) holds 4
// consecutive columns of frame r (and of question r), h choosing which 4 of a group of 8.
// Rows are padded by 4 floats, so the 16 lanes of a quarter-wave read 16 different bank
// groups.  The squared norms come from the same registers; the eight partial tiles meet in
// LDS.  The table is read once per 32 questions.  grid = (frame tiles, question tiles).
// ---------------------------------------------------------------------------------------
constexpr int SM_WAVES = 8, SM_TILE = 32, SM_COLS = 128, SM_PITCH = SM_COLS + 4;

typedef float f32x16 __attribute__((ext_vector_type(16)));

__global__ __launch_bounds__(SM_WAVES * 64) void score_shared_mfma_kernel(
    const float* __restrict__ table, int n_frames, int d_prime, const float* __restrict__ q_vec,
    int n_questions, float inv_tau, float* __restrict__ scores) {
    // the staging tiles and the partial results share storage: the partials are written after the last slab
    constexpr int STAGE_FLOATS = 2 * SM_TILE * SM_PITCH, PART_FLOATS = SM_WAVES * 16 * 64;
    __shared__ __attribute__((aligned(16))) float lds[STAGE_FLOATS > PART_FLOATS ? STAGE_FLOATS : PART_FLOATS];
    __shared__ float vpart[SM_WAVES][64], qpart[SM_WAVES][64];
    float* tile_a = lds;
    float* tile_b = lds + SM_TILE * SM_PITCH;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 31, h = lane >> 5;
    const int f0 = blockIdx.x * SM_TILE, q0 = blockIdx.y * SM_TILE;
    // staging: thread t moves float4 number t and t + 512 of each 32 x 32-float4 slab; DEPTH slabs are
    // in flight from memory to registers, because one slab's MFMAs are far shorter than a memory round trip
    constexpr int PER = SM_TILE * (SM_COLS / 4) / (SM_WAVES * 64);       // 2
    constexpr int DEPTH = 4;
    f32x4 xa[DEPTH][PER], xb[DEPTH][PER];
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    // Loads are unconditional (rows and columns past the end are clamped to valid ones, their
    // values replaced by zero or never stored): straight-line code, so the waits for a slab's
    // loads leave the later slabs' loads in flight.
    auto fetch = [&](f32x4 (&ra)[PER], f32x4 (&rb)[PER], int c0) {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int i = threadIdx.x + u * SM_WAVES * 64;
            const int row = i / (SM_COLS / 4);
            int col = c0 + (i % (SM_COLS / 4)) * 4;
            col = col < d_prime ? col : 0;                                  // D' is a multiple of 4
            const int fr = f0 + row < n_frames ? f0 + row : n_frames - 1;
            const int qr = q0 + row < n_questions ? q0 + row : n_questions - 1;
            ra[u] = *reinterpret_cast<const f32x4*>(table + (int64_t)fr * d_prime + col);
            rb[u] = *reinterpret_cast<const f32x4*>(q_vec + (int64_t)qr * d_prime + col);
        }
    };
    f32x16 acc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[i][j] = 0.f;
    float vv = 0.f, qq = 0.f;
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) fetch(xa[d], xb[d], d * SM_COLS);
    // Rounds of DEPTH slabs, no branch inside a round (columns past D' enter the tiles as zeros); the last
    // round fetches nothing and ends with the last slab.
    const int n_rounds = (d_prime + DEPTH * SM_COLS - 1) / (DEPTH * SM_COLS);
    auto slab = [&](int d, int cc, auto more) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int i = threadIdx.x + u * SM_WAVES * 64;
            const int off = (i / (SM_COLS / 4)) * SM_PITCH + (i % (SM_COLS / 4)) * 4;
            const bool on = cc + (i % (SM_COLS / 4)) * 4 < d_prime;
            *reinterpret_cast<f32x4*>(tile_a + off) = on ? xa[d][u] : zero;
            *reinterpret_cast<f32x4*>(tile_b + off) = on ? xb[d][u] : zero;
        }
        __syncthreads();
        if (decltype(more)::value) fetch(xa[d], xb[d], cc + DEPTH * SM_COLS);
#pragma unroll
        for (int g = 0; g < SM_COLS / 8 / SM_WAVES; ++g) {               // this wave's groups of 8 columns
            const int off = r * SM_PITCH + (wave * (SM_COLS / 8 / SM_WAVES) + g) * 8 + 4 * h;
            const f32x4 a = *reinterpret_cast<const f32x4*>(tile_a + off);
            const f32x4 b = *reinterpret_cast<const f32x4*>(tile_b + off);
            vv += a.x * a.x + a.y * a.y + a.z * a.z + a.w * a.w;
            qq += b.x * b.x + b.y * b.y + b.z * b.z + b.w * b.w;
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[j], b[j], acc[j], 0, 0, 0);
        }
        __syncthreads();
    };
    for (int round = 0; round + 1 < n_rounds; ++round) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) slab(d, (round * DEPTH + d) * SM_COLS, std::true_type());
    }
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
        const int cc = ((n_rounds - 1) * DEPTH + d) * SM_COLS;
        if (cc < d_prime) slab(d, cc, std::false_type());
    }
    float* part = lds;                               // [wave][16][64]
#pragma unroll
    for (int j = 0; j < 16; ++j) part[(wave * 16 + j) * 64 + lane] = (acc[0][j] + acc[1][j]) + (acc[2][j] + acc[3][j]);
    vpart[wave][lane] = vv;
    qpart[wave][lane] = qq;
    __syncthreads();
    // element (frame fl, question ql) of the tile sits in lane ql + 32 * ((fl / 4) % 2), register
    // (fl / 8) * 4 + fl % 4 of every wave's accumulator
    for (int e = threadIdx.x; e < SM_TILE * SM_TILE; e += SM_WAVES * 64) {
        const int fl = e & 31, ql = e >> 5;
        if (f0 + fl >= n_frames || q0 + ql >= n_questions) continue;
        const int l = ql + 32 * ((fl >> 2) & 1), j = (fl >> 3) * 4 + (fl & 3);
        float dot = 0.f, v2 = 0.f, q2 = 0.f;
#pragma unroll
        for (int w = 0; w < SM_WAVES; ++w) {
            dot += part[(w * 16 + j) * 64 + l];
            v2 += vpart[w][fl] + vpart[w][fl + 32];
            q2 += qpart[w][ql] + qpart[w][ql + 32];
        }
        const float den = sqrtf(v2) * sqrtf(q2);
        scores[(int64_t)(q0 + ql) * n_frames + f0 + fl] = den > 0.f ? dot / den * inv_tau : 0.f;
    }
}

// ---------------------------------------------------------------------------------------
// Pooling, Eq. 2 and the selection of a short stream (up to 256 frame or block vectors of up to 1,024 entries) in one
// launch.  A workgroup of 16 wavefronts owns 32 rows of the table, two per wavefront, whose loads leave first;
// meanwhile it pools the whole question for itself (redundantly: it comes from the L2) into LDS.  The scores go out with
// device-scope stores, and the workgroup that draws a question's last ticket ranks them (no cache-wide
// fence: the stores have completed before the ticket is drawn, and the reader's loads follow its own draw; the
// ticket words start at zero and are set back by the last arriver).
// What bounds it is a chain of round trips, and as three launches also the host that issues them: replayed from a graph
// a 32-token question on 256 x 512 takes 10.4 us in three launches and 10.3 in one, 5 of 23 tokens on 98 x 128
// 9.1 and 8.3; the calls they are part of, issued one after the other, 32.3 and 29.7, 44.1 and 38.9 us.
// ---------------------------------------------------------------------------------------
constexpr int SHORT_ROWS = 2 * RANK_THREADS / 64;            // table rows per workgroup
constexpr int SHORT_MAX_DIM = 1024;
constexpr int SHORT_MAX_BLOCKS = 64;
static_assert(SHORT_MAX_BLOCKS <= WAVE_TICKETS, "a ticket per question");
constexpr int64_t SHORT_MAX_QUESTION = 256 << 10;

template <bool BF16, int NI>                                 // D' <= NI * 256
__global__ __launch_bounds__(RANK_THREADS) void retrieve_short_kernel(RetrieveArgs a, int d_prime) {
    constexpr int VEC = BF16 ? 8 : 4;
    constexpr int ES = BF16 ? 2 : 4;
    __shared__ __attribute__((aligned(16))) float red[RANK_THREADS * VEC];     // [part][D']
    __shared__ __attribute__((aligned(16))) float qv[NI * 256];
    __shared__ uint32_t sh_last;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t qi = blockIdx.y;
    const int f0 = blockIdx.x * SHORT_ROWS + wave * 2;

    // the rows (past the table: its last row again), in flight while the question is pooled
    const float* table = a.frame_keys + qi * a.frame_keys_stride;
    const float4 zero4 = make_float4(0.f, 0.f, 0.f, 0.f);
    float4 x[2][NI];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int f = f0 + r < a.n_frames ? f0 + r : a.n_frames - 1;
#pragma unroll
        for (int it = 0; it < NI; ++it) {
            const int i = lane * 4 + it * 256;
            x[r][it] = i < d_prime ? load_stream(table + (int64_t)f * d_prime + i) : zero4;
        }
    }

    // ---- the question: a thread owns 16 bytes of D' and every n_parts-th (token, head of the group)
    const int g_sz = a.n_q_heads / a.n_kv_heads, d = a.head_dim;
    const int chunks = d_prime / VEC, n_parts = RANK_THREADS / chunks;
    const int ch = tid % chunks, part = tid / chunks;
    const int kvh = ch * VEC / d, col = ch * VEC - kvh * d;
    const char* base = static_cast<const char*>(a.q_question) +
        (((int64_t)qi * a.n_q_tokens * a.n_q_heads + kvh * g_sz) * d + col) * ES;
    const int n_pairs = a.n_q_tokens * g_sz;
    // from one pair of a thread to its next, without a division per load
    const int head_b = d * ES, step_t = n_parts / g_sz, step_g = n_parts - step_t * g_sz;
    const int step_b = (step_t * a.n_q_heads + step_g) * head_b, wrap_b = (a.n_q_heads - g_sz) * head_b;
    int g = part % g_sz, off = (part / g_sz * a.n_q_heads + g) * head_b;
    float acc[VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] = 0.f;
    if (part < n_parts) {
        constexpr int U = 8;
        for (int e0 = part; e0 < n_pairs; e0 += n_parts * U) {
            u32x4 w[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                w[u] = u32x4{0u, 0u, 0u, 0u};
                if (e0 + u * n_parts < n_pairs) w[u] = *reinterpret_cast<const u32x4*>(base + off);
                g += step_g;
                off += step_b;
                if (g >= g_sz) {
                    g -= g_sz;
                    off += wrap_b;
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (BF16) {
                        acc[2 * i] += bf16_lo(w[u][i]);
                        acc[2 * i + 1] += bf16_hi(w[u][i]);
                    } else {
                        acc[i] += __uint_as_float(w[u][i]);
                    }
                }
        }
#pragma unroll
        for (int i = 0; i < VEC; ++i) red[part * d_prime + ch * VEC + i] = acc[i];
    }
    __syncthreads();
    if (tid < NI * 256) {
        float sum = 0.f;
        if (tid < d_prime) {
#pragma unroll 8
            for (int p = 0; p < n_parts; ++p) sum += red[p * d_prime + tid];
        }
        qv[tid] = sum * (1.f / ((float)g_sz * (float)a.n_q_tokens));
    }
    __syncthreads();

    // ---- two cosines per wavefront
    float dot[2] = {0.f, 0.f}, vv[2] = {0.f, 0.f}, qq = 0.f;
#pragma unroll
    for (int it = 0; it < NI; ++it) {
        const float4 y = *reinterpret_cast<const float4*>(qv + lane * 4 + it * 256);
        qq += y.x * y.x + y.y * y.y + y.z * y.z + y.w * y.w;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const float4 v = x[r][it];
            vv[r] += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
            dot[r] += v.x * y.x + v.y * y.y + v.z * y.z + v.w * y.w;
        }
    }
    const float dsum = transpose_reduce<2>(dot, lane);       // row lane / 32
    const float vsum = transpose_reduce<2>(vv, lane);
    qq = wave_sum(qq);
    float* scores = a.scores + qi * a.n_frames;
    if ((lane & 31) == 0 && f0 + (lane >> 5) < a.n_frames) {
        const float den = sqrtf(vsum) * sqrtf(qq);
        __hip_atomic_store(scores + f0 + (lane >> 5), den > 0.f ? dsum / den * a.inv_tau : 0.f, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }

    // ---- the last workgroup of the question selects
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // this wave's scores are at the point of coherence
    __syncthreads();
    if (tid == 0) {
        const uint32_t n = __hip_atomic_fetch_add(a.tickets + qi, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sh_last = n == gridDim.x - 1u;
        if (sh_last) __hip_atomic_store(a.tickets + qi, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!sh_last) return;
    rank_block([&](int f) { return __hip_atomic_load(scores + f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }, a.n_frames,
               a.k, a.idx + qi * a.k, a.n_sel ? a.n_sel + qi : nullptr);
}

}  // namespace

namespace {

// One vector per `per` rows, n_rows in all.  Lanes per workgroup: a whole row's (up to 256), narrowed to 128 bytes while the
// frames have two rows or more for each row group and the narrow slabs are at most 4,096 workgroups.  Beyond that the chip is
// full either way and whole rows are level or ahead: 1,024 frames of 256 x 512 39.8 us and 41.3 us in slabs (fp32: 450 blocks of 8 x 512 2.8
// and 6.1), 2,048 of 33 x 256 5.3 and 9.0.  The lanes decide the order of a sum, so a frame's vector may differ in its last bits between
// a call with few frames and one with many.
constexpr int MIN_LPR_LOG2 = 3, MAX_SLABS = 4096;
hipError_t mean_rows_launch(const void* k, int64_t n_rows, int per, int d_prime, int dtype, float* out, hipStream_t stream) {
    const int vec = dtype == REKV_BF16 ? 8 : 4;
    const int lanes = (d_prime + vec - 1) / vec;          // 16-byte lanes per key row
    const int64_t frames = (n_rows + per - 1) / per;
    const int64_t most = n_rows < per ? n_rows : per;     // rows of the longest frame (a single short block of frames: 2.1 -> 1.8 us)
    int lpr_log2 = 0;
    while ((1 << lpr_log2) < lanes && lpr_log2 < 8) ++lpr_log2;
    if (frames * ((lanes + (1 << MIN_LPR_LOG2) - 1) >> MIN_LPR_LOG2) <= MAX_SLABS)
        while (lpr_log2 > MIN_LPR_LOG2 && (1024 >> lpr_log2) <= most) --lpr_log2;
    dim3 grid((unsigned)frames, (unsigned)((lanes + (1 << lpr_log2) - 1) >> lpr_log2));
    const bool bf16 = dtype == REKV_BF16, one = most <= 256 >> lpr_log2;
    auto kern = bf16 ? (one ? frame_keys_kernel<true, true> : frame_keys_kernel<true, false>)
                     : (one ? frame_keys_kernel<false, true> : frame_keys_kernel<false, false>);
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, stream, k, per, n_rows, d_prime, lpr_log2, out);
    return hipGetLastError();
}

}  // namespace

hipError_t frame_keys_launch(const void* k, int n_frames, int tokens_per_frame, int d_prime,
                             int dtype, float* frame_keys, hipStream_t stream) {
    return mean_rows_launch(k, (int64_t)n_frames * tokens_per_frame, tokens_per_frame, d_prime, dtype, frame_keys, stream);
}

namespace {

// Frames of the selected blocks, in block order.  One workgroup per question; slot j*b + t of
// the output is frame block[j]*b + t, or -1 past the end of the stream or of the selection.
// Because blocks come in ascending order, only the last selected block can be the stream's
// short one, so the -1 slots are always at the tail.
__global__ __launch_bounds__(256) void expand_blocks_kernel(const int32_t* __restrict__ block_idx,
                                                            int k_blocks, int b, int n_frames,
                                                            int32_t* __restrict__ frame_idx,
                                                            int32_t* __restrict__ n_sel) {
    __shared__ int count;
    const int q = blockIdx.x;
    if (threadIdx.x == 0) count = 0;
    __syncthreads();
    const int n_slots = k_blocks * b;
    int mine = 0;
    for (int s = threadIdx.x; s < n_slots; s += 256) {
        const int blk = block_idx[(int64_t)q * k_blocks + s / b];
        const int64_t f = (int64_t)blk * b + s % b;
        const bool ok = blk >= 0 && f < n_frames;
        frame_idx[(int64_t)q * n_slots + s] = ok ? (int32_t)f : -1;
        mine += ok;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mine += __shfl_xor(mine, off);
    if ((threadIdx.x & 63) == 0 && mine) atomicAdd(&count, mine);
    __syncthreads();
    if (threadIdx.x == 0 && n_sel) n_sel[q] = count;
}

}  // namespace

hipError_t block_keys_launch(const float* frame_keys, int n_frames, int b, int d_prime, float* block_keys,
                             hipStream_t stream) {
    // a block vector is the mean of b rows of the fp32 frame table: the frame-vector kernel with b "tokens" per
    // "frame" (a last block of fewer frames in a launch of its own cost 2 us of kernel time more)
    return mean_rows_launch(frame_keys, n_frames, b, d_prime, REKV_F32, block_keys, stream);
}

hipError_t expand_blocks_launch(const int32_t* block_idx, int n_questions, int k_blocks, int b, int n_frames,
                                int32_t* frame_idx, int32_t* n_sel, hipStream_t stream) {
    hipLaunchKernelGGL(expand_blocks_kernel, dim3((unsigned)n_questions), dim3(256), 0, stream, block_idx,
                       k_blocks, b, n_frames, frame_idx, n_sel);
    return hipGetLastError();
}

hipError_t retrieve_launch(const RetrieveArgs& a, hipStream_t stream) {
    const int d_prime = a.dim > 0 ? a.dim : a.n_kv_heads * a.head_dim;
    const float* q_vec = a.q_vec_given;
    hipError_t e = hipSuccess;
    // Short streams go through one launch while few workgroups pool their whole question at once and that is not
    // long: with questions of 448 KB and 512 KB pooling alone takes the kernel to 11.3 and 13.5 us against 9.3 and 11.5 in
    // three launches, and with 128 and 256 workgroups it is 0.7 and 0.5 us behind (16 questions of 224 KB, 32 of 56 KB).
    const int short_blocks = (a.n_frames + SHORT_ROWS - 1) / SHORT_ROWS;
    const int64_t question_bytes = (int64_t)a.n_q_tokens * a.n_q_heads * a.head_dim * (a.dtype == REKV_BF16 ? 2 : 4);
    if (!q_vec && a.n_frames <= RANK_MAX_FRAMES && a.k < a.n_frames && d_prime <= SHORT_MAX_DIM &&
        (int64_t)short_blocks * a.n_questions <= SHORT_MAX_BLOCKS && question_bytes <= SHORT_MAX_QUESTION) {
        const int ni = (d_prime + 255) / 256;
        const bool bf16 = a.dtype == REKV_BF16;
        auto kern = ni == 1 ? (bf16 ? retrieve_short_kernel<true, 1> : retrieve_short_kernel<false, 1>)
                  : ni == 2 ? (bf16 ? retrieve_short_kernel<true, 2> : retrieve_short_kernel<false, 2>)
                  : ni == 3 ? (bf16 ? retrieve_short_kernel<true, 3> : retrieve_short_kernel<false, 3>)
                            : (bf16 ? retrieve_short_kernel<true, 4> : retrieve_short_kernel<false, 4>);
        hipLaunchKernelGGL(kern, dim3((unsigned)short_blocks, (unsigned)a.n_questions), dim3(RANK_THREADS), 0, stream, a, d_prime);
        return hipGetLastError();
    }
    if (!q_vec) {                      // pooled question vectors: [n_questions, D']
        const int cols = POOL_LANES * (a.dtype == REKV_BF16 ? 8 : 4);
        dim3 grid((unsigned)a.n_questions, (unsigned)a.n_kv_heads, (unsigned)((a.head_dim + cols - 1) / cols));
        if (a.dtype == REKV_BF16)
            hipLaunchKernelGGL(pool_question_kernel<true>, grid, dim3(POOL_THREADS), 0, stream, a.q_question, a.n_q_tokens,
                               a.n_q_heads, a.n_kv_heads, a.head_dim, a.q_vec);
        else
            hipLaunchKernelGGL(pool_question_kernel<false>, grid, dim3(POOL_THREADS), 0, stream, a.q_question, a.n_q_tokens,
                               a.n_q_heads, a.n_kv_heads, a.head_dim, a.q_vec);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        q_vec = a.q_vec;
    }
    // Four or more questions on one table: the matrix-core kernel reads the table once per 32 questions, the other
    // once per question.  Below 56 MB read that way (vectors of up to 1,024 entries, whose loads all leave at once) the
    // caches carry it: 4 to 8 us against 4.4 to 15; at 51 MB 8.0 against 11.7 us
    // (32 questions, 777 x 512) and 10.7 against 12.9 (16, 777 x 1,024), at 66 MB 10.2 against 8.5 (64, 2,000 x 128),
    // 9.8 against 8.8 (16, 2,000 x 512) and 13.4 against 13.0 (8, 2,000 x 1,024).
    const bool per_question = a.n_questions < 4 ||
        (d_prime <= 1024 && (int64_t)a.n_questions * a.n_frames * d_prime * 4 <= 56000000);
    if (a.frame_keys_stride == 0 && !per_question) {
        dim3 grid((unsigned)((a.n_frames + SM_TILE - 1) / SM_TILE), (unsigned)((a.n_questions + SM_TILE - 1) / SM_TILE));
        hipLaunchKernelGGL(score_shared_mfma_kernel, grid, dim3(SM_WAVES * 64), 0, stream, a.frame_keys, a.n_frames,
                           d_prime, q_vec, a.n_questions, a.inv_tau, a.scores);
    } else {
        int fblocks = (a.n_frames + SCORE_WAVES * SCORE_FR - 1) / (SCORE_WAVES * SCORE_FR);
        if (fblocks > 4096) fblocks = 4096;
        dim3 grid((unsigned)fblocks, (unsigned)a.n_questions);
        const int ni = d_prime <= 1024 ? (d_prime + 255) / 256 : 0;
        auto kern = ni == 1 ? score_rows_kernel<1> : ni == 2 ? score_rows_kernel<2> : ni == 3 ? score_rows_kernel<3>
                  : ni == 4 ? score_rows_kernel<4> : score_rows_kernel<0>;
        hipLaunchKernelGGL(kern, grid, dim3(SCORE_WAVES * 64), 0, stream, a.frame_keys,
                           a.frame_keys_stride, a.n_frames, d_prime, q_vec, a.inv_tau, a.scores);
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (a.n_frames >= SEL_MIN_FRAMES && a.n_frames <= SEL_MAX_FRAMES && a.k <= SEL_MAX_K && a.k < a.n_frames)
        hipLaunchKernelGGL(topk_groupmax_kernel<1024>, dim3((unsigned)a.n_questions), dim3(1024), 0, stream,
                           a.scores, a.n_frames, a.k, a.idx, a.n_sel);
    else if (a.n_frames <= RANK_MAX_FRAMES && a.k < a.n_frames)
        hipLaunchKernelGGL(topk_rank_kernel, dim3((unsigned)a.n_questions), dim3(RANK_THREADS), 0, stream,
                           a.scores, a.n_frames, a.k, a.idx, a.n_sel);
    else
        hipLaunchKernelGGL(topk_kernel, dim3((unsigned)a.n_questions), dim3(TOPK_THREADS), 0, stream,
                           a.scores, a.n_frames, a.k, a.idx, a.n_sel);
    return hipGetLastError();
}

}  // namespace rekv

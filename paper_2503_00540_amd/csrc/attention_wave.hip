// bf16 MFMA attention for launches too small to fill the chip with 128-row workgroups: one live
// chunk, a few questions, a decode step.  Same contraction, segments and MFMA layout as
// attention_bf16.hip; the split of the work is the other way round.
//
// Work split.  A workgroup of 8 wavefronts owns a block of only 32 (or 64) query rows of one (item,
// KV head) and its wavefronts divide the KEYS: each (or each pair) walks its own run of 32-key tiles
// through its own LDS stages.  The partial results (running maximum, sum, unnormalised O) meet in
// LDS, so eight (four) key ranges cost no memory traffic and no second launch.  Where that still
// leaves compute units idle (few row blocks), several workgroups split the tile list further;
// each writes its merged partial result past the caches, takes a ticket, and the workgroup that
// draws the last ticket of a row block adds the others up.
//
// Partial results cross the XCDs' L2s without cache-wide fences: they are written and read with
// device-scope accesses (which go to the point of coherence), the writer's loads and stores have
// completed (vmcnt 0) before its workgroup's ticket is drawn, and the reader's accesses follow its
// own draw.  The ticket words start at zero and the last arriver sets its word back to zero.
//
// What bounds it.  These launches are a chain of latencies: about 2 us to the first tile in LDS, 1 us
// for the waves' merge, 1 us for the ticket and about 3 for the last arriver, whose loads leave together; between them a step of 32
// keys per wave takes 1.25 us because eight private K/V tiles (128 KB) come through the CU's 64 B/clk path from L2.
// Measured against splitting 128-row workgroups over the keys with a merge launch (as replayed from a
// graph, us; K and V in the caches, then from HBM): 7B-class live frame, 16-frame window 31.2 -> 21.2, 31.2 -> 24.0; 0.5B-class
// 18.0 -> 11.7, 18.8 -> 12.5; one question over 16 frames 15.8 -> 12.3, 16.7 -> 13.5; a decode step over 64 frames 15.0 ->
// 12.5, 17.5 -> 14.4.  A software-pipelined step (S of the next tile during the softmax, as in
// attention_bf16.hip) measured no faster here and needs 20 to 30 registers more.
#include "attention_mfma.h"

namespace rekv {
namespace {

constexpr int WAVES = 8;
constexpr int THREADS = WAVES * 64;
constexpr int WM = 32;               // query rows per wavefront (one MFMA column block)

// Division by a launch constant: n / d for n * d < 2^32 (the quotient of 32-bit division costs about
// 30 dependent instructions, and a launch this small is mostly its prologue).
struct FastDiv {
    uint32_t d, mul;
};
FastDiv fast_div(uint32_t d) { return FastDiv{d, d > 1 ? (uint32_t)(((1ull << 32) + d - 1) / d) : 0u}; }
__device__ inline int quot(int n, FastDiv f) { return f.d > 1 ? (int)__umulhi((uint32_t)n, f.mul) : n; }

struct WaveArgs {
    AttnProblem p;
    int32_t n_splits, row_blocks;
    FastDiv by_splits, by_row_blocks, by_items, by_group;
    float* part;          // [row block][split] of { O [T][D], (maximum, sum) [T] }, fp32
    uint32_t* tickets;    // [row block]
};
template <int N>
__device__ inline void wait_newest() {           // all vector-memory accesses but the newest N are done
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// A pointer that is the same in all lanes, in scalar registers.
__device__ inline const char* uniform(const char* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<const char*>(((uint64_t)hi << 32) | lo);
}

// RW row waves x KG = 8 / RW key groups.  STREAM: every K/V tile is read by this workgroup only
// (one row block per item).
template <int D, int RW, bool ENCODE, bool INDEXED, bool STREAM>
__global__ __launch_bounds__(THREADS, 2) void attn_wave_kernel(WaveArgs a) {
    static_assert(!(ENCODE && INDEXED), "the encode window is contiguous");
    static_assert(RW == 1 || RW == 2, "the pipelines below");
    constexpr int KG = WAVES / RW;
    constexpr int T = RW * WM;                   // query rows per workgroup
    constexpr int STAGES = RW;                   // LDS stages per key group: 8 K/V tile pairs in all
    constexpr int CH = D / 8;                    // 16-byte chunks per key row
    constexpr int RPI = 64 / CH;                 // key rows one 1 KB wave-wide load covers
    constexpr int N_DMA = BN / RPI / RW;         // such loads per wave, tile and tensor
    constexpr uint32_t TILE_B = BN * D * 2;      // bytes of a K or V tile
    constexpr int CPR = D / 4;                   // 16-byte fp32 chunks per output row
    constexpr uint32_t PART_B = T * (D + 2) * 4; // bytes of one partial result
    __shared__ int32_t frame_of_slot[INDEXED ? MAX_INDEXED_FRAMES : 1];
    // per key group and stage: a K tile, a V tile; at the end per key group: its O [T][D] fp32
    __shared__ __attribute__((aligned(1024))) unsigned char lds[(int64_t)WAVES * 2 * BN * D * 2];
    __shared__ f32x2 ml[KG][T];
    __shared__ f32x2 ml_all[T];
    __shared__ uint32_t sh_last;

    AttnProblem p = a.p;
    p.is_encode = ENCODE;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave / RW, rw = wave % RW;    // key group, row wave
    const int col = lane & 31, hh = lane >> 5;
    const int G = (int)a.by_group.d;

    int L = xcd_remap(blockIdx.x, gridDim.x), q = quot(L, a.by_row_blocks);
    const int rb = L - q * a.row_blocks;
    L = q; q = quot(L, a.by_splits);
    const int split = L - q * a.n_splits;
    const int kvh = quot(q, a.by_items);         // KV head slowest: see attention_bf16.hip
    const int item = q - kvh * p.n_items;

    const ItemSegs seg = item_segments(p, item);
    const int64_t row_stride = (int64_t)p.n_kv_heads * D;
    const uint32_t row_stride_b = (uint32_t)row_stride * 2u;
    const bool k_dense = INDEXED && p.a_k_dense;
    const int64_t ka_off = k_dense ? (int64_t)item * p.len_a : seg.a_off;
    const char* ka = reinterpret_cast<const char*>(static_cast<const bf16_t*>(p.k_a) + ka_off * row_stride + kvh * D);
    const char* va = reinterpret_cast<const char*>(static_cast<const bf16_t*>(p.v_a) + seg.a_off * row_stride + kvh * D);
    const char* kb = reinterpret_cast<const char*>(static_cast<const bf16_t*>(p.k_b) + seg.b_off * row_stride + kvh * D);
    const char* vb = reinterpret_cast<const char*>(static_cast<const bf16_t*>(p.v_b) + seg.b_off * row_stride + kvh * D);

    const int m_rows = p.len_q * G;
    const int row0 = rb * T, lrow = rw * WM + col, row = row0 + lrow;
    const int tok = quot(row, a.by_group);
    const bool row_ok = row < m_rows;
    const bool wave_active = RW == 1 || row0 + rw * WM < m_rows;

    // tiles of this row block: segment A, then the causal tiles of segment B it can see
    const int tiles_a = (seg.len_a + BN - 1) / BN;
    const int q_pos0 = p.len_b - p.len_q;
    int last_tok = quot(row0 + T - 1, a.by_group);
    if (last_tok > p.len_q - 1) last_tok = p.len_q - 1;
    const int n_tiles = tiles_a + (last_tok + q_pos0) / BN + 1;
    const int n_slots = a.n_splits * KG, slot = split * KG + kg;
    const int t_each = n_tiles / n_slots, t_rest = n_tiles - t_each * n_slots;    // the first t_rest runs are one longer
    const int t_begin = t_each * slot + (slot < t_rest ? slot : t_rest);
    const int t_end = t_begin + t_each + (slot < t_rest);
    const int n_steps = t_each + (split * KG < t_rest);                          // of the workgroup's longest run

    // ---- lane-constant addressing (layout of a tile in LDS: attention_bf16.hip)
    const uint32_t lds0 = lds_addr_of(lds) + (uint32_t)(kg * STAGES) * 2u * TILE_B;
    const int dma_row = rw * N_DMA * RPI + lane / CH, dma_p = lane % CH;
    const uint32_t dma_dst = lds0 + (uint32_t)(rw * N_DMA) * 1024u;
    auto coff = [&](int j) { return (uint32_t)(dma_p ^ swz<D>(dma_row + j * RPI)) * 16u; };

    const float inv_n_f = INDEXED ? 1.f / (float)p.n_f : 0.f;
    if (INDEXED) {
        const int n_frames = (seg.len_a + p.n_f - 1) / p.n_f;
        for (int i = tid; i < n_frames; i += THREADS) {
            int f = p.a_index[(int64_t)item * p.a_index_stride + i];
            frame_of_slot[i] = f < 0 ? 0 : (f < p.n_src_frames ? f : p.n_src_frames - 1);
        }
        __syncthreads();
    }
    // Byte offsets of this wave's chunks inside a tile.  The swizzle repeats every 16 rows, so N_OFF lane
    // offsets serve all of its loads; the rest of the address is scalar.
    constexpr int N_OFF = N_DMA < 16 / RPI ? N_DMA : 16 / RPI;
    uint32_t dma_off[N_OFF];
#pragma unroll
    for (int j = 0; j < N_OFF; ++j) dma_off[j] = (uint32_t)(dma_row + j * RPI) * row_stride_b + coff(j);
    // This wave's share of tile t of K or V (dst: stage offset); a segment's ragged last tile
    // re-reads the segment's last key for the rows past its end.
    auto dma_tile = [&](const char* seg_a, const char* seg_b, int t, uint32_t dst, bool through_index) __attribute__((always_inline)) {
        const bool in_b = t >= tiles_a;
        const int key0 = (in_b ? t - tiles_a : t) * BN;
        const int n_valid = (in_b ? p.len_b : seg.len_a) - key0;
        const char* base = uniform((in_b ? seg_b : seg_a) + (int64_t)key0 * row_stride_b);
        if (INDEXED && !in_b && through_index) {
#pragma unroll
            for (int j = 0; j < N_DMA; ++j) {
                int r = dma_row + j * RPI;
                r = (r < n_valid - 1 ? r : n_valid - 1) + key0;
                // rows are below 2^23: the float quotient is off by at most one
                int fs = (int)((float)r * inv_n_f);
                int within = r - fs * p.n_f;
                if (within < 0) { --fs; within += p.n_f; }
                if (within >= p.n_f) { ++fs; within -= p.n_f; }
                const uint32_t src_row = (uint32_t)(frame_of_slot[fs] * p.n_f + within);
                dma16<STREAM>(seg_a, src_row * row_stride_b + coff(j), dma_dst + dst + j * 1024u);
            }
        } else if (n_valid >= BN) {
#pragma unroll
            for (int j = 0; j < N_DMA; ++j)
                dma16<STREAM>(base + (uint32_t)(j / N_OFF * 16) * row_stride_b, dma_off[j % N_OFF], dma_dst + dst + j * 1024u);
        } else {
#pragma unroll 1
            for (int j = 0; j < N_DMA; ++j) {
                int r = dma_row + j * RPI;
                r = r < n_valid - 1 ? r : n_valid - 1;
                dma16<STREAM>(base, (uint32_t)r * row_stride_b + coff(j), dma_dst + dst + j * 1024u);
            }
        }
    };
    auto dma_k = [&](int t, uint32_t stage_b) __attribute__((always_inline)) { dma_tile(ka, kb, t, stage_b, !k_dense); };
    auto dma_v = [&](int t, uint32_t stage_b) __attribute__((always_inline)) { dma_tile(va, vb, t, stage_b + TILE_B, true); };

    // the first tiles' loads leave before anything else is set up
    if (t_begin < t_end) {
        dma_k(t_begin, 0);
        dma_v(t_begin, 0);
    }

    bf16x8 qf[D / 16];
    {
        const bf16_t* qrow = static_cast<const bf16_t*>(p.q) +
            (((int64_t)item * p.len_q + tok) * p.n_q_heads + kvh * G + (row - tok * G)) * D;
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) {
            u32x4 v = {0u, 0u, 0u, 0u};
            if (row_ok) v = *reinterpret_cast<const u32x4*>(qrow + ks * 16 + hh * 8);
            qf[ks] = __builtin_bit_cast(bf16x8, v);
        }
    }
    uint32_t k_addr[D / 16];
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks)
        k_addr[ks] = lds0 + (uint32_t)(col * D + (((ks * 2 + hh) ^ swz<D>(col)) * 8)) * 2u;
    uint32_t v_addr[2][D / 32];
    {
        const int gq = lane >> 4, i16 = lane & 15, qd = i16 & 3, jk = i16 >> 2;
        const int cl = (gq & 1) * 2 + (qd >> 1), half = qd & 1;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int keyl = r * 8 + hh * 4 + jk;
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
                v_addr[r][db] = lds0 + TILE_B + (uint32_t)(keyl * D + (((db * 4 + cl) ^ swz<D>(keyl)) * 8) + half * 4) * 2u;
        }
    }

    f32x16 o[D / 32];
#pragma unroll
    for (int i = 0; i < D / 32; ++i)
#pragma unroll
        for (int j = 0; j < 16; ++j) o[i][j] = 0.f;
    float m_ref = -INFINITY, l_part = 0.f;
    const float sc = p.scale * 1.4426950408889634f;
    // The Q fragments have landed, in a form the compiler's bookkeeping sees (the tile loads are asm and
    // invisible to it): otherwise it would put its own vmcnt(0) in front of the loop's first MFMA.
    wait_vmem();

    auto load_k = [&](uint32_t stage_b, bf16x8 (&kf)[D / 16]) {
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) kf[ks] = *reinterpret_cast<LDS_AS const bf16x8*>(k_addr[ks] + stage_b);
    };
    auto load_v = [&](uint32_t stage_b, bf16x8 (&vf)[2][D / 32]) {
#pragma unroll
        for (int g16 = 0; g16 < 2; ++g16)
#pragma unroll
            for (int db = 0; db < D / 32; ++db) {
                const tr4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
                    reinterpret_cast<LDS_AS tr4_t*>(v_addr[0][db] + stage_b + g16 * 16 * D * 2));
                const tr4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
                    reinterpret_cast<LDS_AS tr4_t*>(v_addr[1][db] + stage_b + g16 * 16 * D * 2));
                vf[g16][db] = __builtin_shufflevector(__builtin_bit_cast(bf16x4, lo), __builtin_bit_cast(bf16x4, hi),
                                                      0, 1, 2, 3, 4, 5, 6, 7);
            }
    };
    auto qk = [&](const bf16x8 (&kf)[D / 16], f32x16& s) {
#pragma unroll
        for (int j = 0; j < 16; ++j) s[j] = 0.f;
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[ks], s, 0, 0, 0);
    };
    // mask, running maximum, probabilities of tile t
    auto softmax = [&](int t, f32x16& s, bf16x8 (&pf)[2]) {
        const bool in_b = t >= tiles_a;
        const int key0 = (in_b ? t - tiles_a : t) * BN;
        if (in_b || key0 + BN > seg.len_a) {     // visible keys of this tile: [0, lim)
            const int lim = (in_b ? (tok + q_pos0 + 1 < p.len_b ? tok + q_pos0 + 1 : p.len_b) : seg.len_a) - key0;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int key = (j >> 2) * 8 + hh * 4 + (j & 3);
                s[j] = key < lim ? s[j] : -INFINITY;
            }
        }
        float mx = s[0];
#pragma unroll
        for (int j = 1; j < 16; ++j) mx = fmaxf(mx, s[j]);
        mx = pair_max(mx);
        const float mt2 = mx * sc;
        if (__builtin_amdgcn_ballot_w64(mt2 > m_ref + RESCALE_GAP) != 0) {
            const float m_new = fmaxf(m_ref, mt2);
            const float alpha = (m_new == -INFINITY) ? 1.f : __builtin_amdgcn_exp2f(m_ref - m_new);
            l_part *= alpha;
#pragma unroll
            for (int i = 0; i < D / 32; ++i)
#pragma unroll
                for (int j = 0; j < 16; ++j) o[i][j] *= alpha;
            m_ref = m_new;
        }
        const float mr = (m_ref == -INFINITY) ? 0.f : m_ref;
#pragma unroll
        for (int g16 = 0; g16 < 2; ++g16) {
            float e[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                e[j] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[g16 * 8 + j], sc, -mr));
                l_part += e[j];
            }
#pragma unroll
            for (int j = 0; j < 8; j += 2) {
                const bf16x2 b2 = __builtin_convertvector((f32x2{e[j], e[j + 1]}), bf16x2);
                pf[g16][j] = b2[0];
                pf[g16][j + 1] = b2[1];
            }
        }
    };
    auto pv = [&](const bf16x8 (&vf)[2][D / 32], const bf16x8 (&pf)[2]) {
#pragma unroll
        for (int g16 = 0; g16 < 2; ++g16)
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
                o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[g16][db], pf[g16], o[db], 0, 0, 0);
    };
    auto lds_reads_done = [] {                   // operands are in registers: their stage may be refilled
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };

    if constexpr (RW == 1) {
        // one wave per key group: no barrier; K(t+1) is fetched as soon as K(t) is in registers, V alike
        for (int t = t_begin; t < t_end; ++t) {
            const bool more = t + 1 < t_end;
            wait_newest<N_DMA>();                // K(t); V(t)'s loads are the only newer ones
            bf16x8 kf[D / 16], vf[2][D / 32], pf[2];
            f32x16 s;
            load_k(0, kf);
            lds_reads_done();
            if (more) dma_k(t + 1, 0);
            qk(kf, s);
            softmax(t, s, pf);
            if (more) wait_newest<N_DMA>();      // V(t); K(t+1)'s loads are newer
            else wait_newest<0>();
            load_v(0, vf);
            lds_reads_done();
            if (more) dma_v(t + 1, 0);
            pv(vf, pf);
        }
    } else {
        // two waves share their key group's tiles and two stages: one barrier per step, after which
        // tile t has landed in both shares and the stage of tile t-1, read by both, takes tile t+1
        auto step = [&](int i, auto st) __attribute__((always_inline)) {
            constexpr uint32_t CUR = decltype(st)::value * 2 * TILE_B;
            constexpr uint32_t NEXT = 2 * TILE_B - CUR;
            const int t = t_begin + i;
            wait_newest<0>();
            asm volatile("s_barrier" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
            if (t + 1 < t_end) {
                dma_k(t + 1, NEXT);
                dma_v(t + 1, NEXT);
            }
            if (t < t_end && wave_active) {
                bf16x8 kf[D / 16], vf[2][D / 32], pf[2];
                f32x16 s;
                load_k(CUR, kf);
                qk(kf, s);
                load_v(CUR, vf);
                softmax(t, s, pf);
                pv(vf, pf);
            }
            lds_reads_done();
        };
        for (int i = 0; i < n_steps; ++i) {
            step(i, IC<0>{});
            if (++i == n_steps) break;
            step(i, IC<1>{});
        }
    }

    // ---- the key groups' results meet in LDS.  A group's O lies in its own stages, 16-byte chunk c of
    // row r at chunk position c ^ r, so that both the writes (a row per lane) and the reads (a row
    // per CPR lanes) touch all banks.  Rows past the last query row are neither written nor read.
    const float l_tot = pair_sum(l_part);
    if (hh == 0) ml[kg][lrow] = f32x2{m_ref, l_tot};
    __syncthreads();
    if (row_ok) {
        float m_all = ml[0][lrow][0];
#pragma unroll
        for (int g = 1; g < KG; ++g) m_all = fmaxf(m_all, ml[g][lrow][0]);
        const float f = (m_ref == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m_ref - m_all);
        f32x4* mine = reinterpret_cast<f32x4*>(lds + (size_t)kg * T * D * 4);
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int j4 = 0; j4 < 4; ++j4) {
                const int c = db * 8 + j4 * 2 + hh;
                mine[lrow * CPR + (c ^ (lrow & (CPR - 1)))] =
                    f32x4{o[db][j4 * 4] * f, o[db][j4 * 4 + 1] * f, o[db][j4 * 4 + 2] * f, o[db][j4 * 4 + 3] * f};
            }
        if (kg == 0 && hh == 0) {
            float l = 0.f;
#pragma unroll
            for (int g = 0; g < KG; ++g) {
                const f32x2 x = ml[g][lrow];
                l += x[0] == -INFINITY ? 0.f : x[1] * __builtin_amdgcn_exp2f(x[0] - m_all);
            }
            ml_all[lrow] = f32x2{m_all, l};
        }
    }
    __syncthreads();
    const int n_rows = m_rows - row0 < T ? m_rows - row0 : T;        // real rows of this block
    const int n_chunks = n_rows * CPR;                               // 16-byte chunks of the block's result
    auto write_out = [&](int e, f32x4 v) {
        const int rr = row0 + e / CPR, tk = quot(rr, a.by_group);
        bf16_t* orow = static_cast<bf16_t*>(p.out) +
            (((int64_t)item * p.len_q + tk) * p.n_q_heads + kvh * G + (rr - tk * G)) * D + (e % CPR) * 4;
        u32x2 w;
        w.x = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{v[0], v[1]}), bf16x2));
        w.y = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{v[2], v[3]}), bf16x2));
        *reinterpret_cast<u32x2*>(orow) = w;
    };
    const int blk = (kvh * p.n_items + item) * a.row_blocks + rb;
    const auto part = part_buffer(a.part, gridDim.x * PART_B);
    const uint32_t part0 = (uint32_t)(blk * a.n_splits) * PART_B;    // byte offset of split 0's result
#pragma unroll
    for (int e0 = 0; e0 < T * CPR; e0 += THREADS) {
        const int e = e0 + tid;
        if (e < n_chunks) {
            const int r = e / CPR, c = e % CPR;
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int g = 0; g < KG; ++g)
                v += *reinterpret_cast<const f32x4*>(lds + (size_t)g * T * D * 4 + (r * CPR + (c ^ (r & (CPR - 1)))) * 16);
            if (a.n_splits == 1)
                write_out(e, v * (1.f / ml_all[r][1]));
            else
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(buf4, v), part, part0 + split * PART_B + e * 16, 0, SC1);
        }
    }
    if (a.n_splits == 1) return;
    if (tid < n_rows)
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(buf2, ml_all[tid]), part,
                                              part0 + split * PART_B + T * D * 4 + tid * 8, 0, SC1);

    wait_newest<0>();                            // this wave's part is at the point of coherence
    __syncthreads();
    if (tid == 0) {
        const uint32_t n = __hip_atomic_fetch_add(a.tickets + blk, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sh_last = n == (uint32_t)a.n_splits - 1u;
        if (sh_last) __hip_atomic_store(a.tickets + blk, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!sh_last) return;

    // ---- last of the row block's workgroups: the splits' results.  Threads form n_grp groups that share
    // the splits; a thread owns P chunks and fetches P * U of them together with their (maximum, sum) pairs, so that up
    // to n_grp * U splits cost one memory round trip and nothing waits for a weight.  The groups meet in LDS.
    f32x4* red = reinterpret_cast<f32x4*>(lds);                      // [group - 1][chunk]
    f32x2* red_ml = reinterpret_cast<f32x2*>(lds + (THREADS - 64) * 16);
    auto merge = [&](auto pc, int n_grp, int per) {
        constexpr int P = decltype(pc)::value, U = 16 / P;
        const int grp = __builtin_amdgcn_readfirstlane(n_grp > 1 ? tid / per : 0);     // (whole waves)
        const int e0 = n_grp > 1 ? tid - grp * per : tid;
        uint32_t off_o[P], off_ml[P];            // past the last chunk: that one again
#pragma unroll
        for (int i = 0; i < P; ++i) {
            const int e = e0 + i * THREADS < n_chunks ? e0 + i * THREADS : n_chunks - 1;
            off_o[i] = part0 + e * 16;
            off_ml[i] = part0 + T * D * 4 + e / CPR * 8;
        }
        f32x4 acc[P];
        float m[P], l[P];
#pragma unroll
        for (int i = 0; i < P; ++i) {
            acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            m[i] = -INFINITY;
            l[i] = 0.f;
        }
        for (int s0 = grp; s0 < a.n_splits && grp < n_grp; s0 += U * n_grp) {
            f32x4 x[P][U];
            f32x2 w[P][U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int s = s0 + u * n_grp;
#pragma unroll
                for (int i = 0; i < P; ++i) {
                    w[i][u] = f32x2{-INFINITY, 0.f};
                    x[i][u] = f32x4{0.f, 0.f, 0.f, 0.f};
                    if (s < a.n_splits) {
                        w[i][u] = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(part, off_ml[i], s * PART_B, SC1));
                        x[i][u] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(part, off_o[i], s * PART_B, SC1));
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < P; ++i) {
                float m_new = m[i];
#pragma unroll
                for (int u = 0; u < U; ++u) m_new = fmaxf(m_new, w[i][u][0]);
                const float f = m[i] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m[i] - m_new);
                l[i] *= f;
                acc[i] *= f;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const float f_u = w[i][u][0] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(w[i][u][0] - m_new);
                    l[i] += w[i][u][1] * f_u;
                    acc[i] += x[i][u] * f_u;
                }
                m[i] = m_new;
            }
        }
        if (n_grp > 1) {
            if (grp > 0 && grp < n_grp) {
                red[(grp - 1) * per + e0] = acc[0];
                red_ml[(grp - 1) * per + e0] = f32x2{m[0], l[0]};
            }
            __syncthreads();
            if (grp > 0) return;
            float m_all = m[0];
            for (int g = 0; g < n_grp - 1; ++g) m_all = fmaxf(m_all, red_ml[g * per + e0][0]);
            const float f = m[0] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m[0] - m_all);
            l[0] *= f;
            acc[0] *= f;
            for (int g = 0; g < n_grp - 1; ++g) {
                const f32x2 x = red_ml[g * per + e0];
                const float f_g = x[0] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(x[0] - m_all);
                l[0] += x[1] * f_g;
                acc[0] += red[g * per + e0] * f_g;
            }
        }
#pragma unroll
        for (int i = 0; i < P; ++i) {
            const int e = e0 + i * THREADS;
            if (e < n_chunks) write_out(e, acc[i] * (1.f / l[i]));
        }
    };
    constexpr int P_MAX = T * CPR / THREADS;
    const int per = (n_chunks + 63) & ~63;                           // threads per group, whole waves
    if (per * 2 <= THREADS) merge(IC<1>{}, THREADS / per, per);
    else if (P_MAX > 1 && n_chunks > THREADS) merge(IC<(P_MAX > 1 ? P_MAX : 1)>{}, 1, THREADS);
    else merge(IC<1>{}, 1, THREADS);
}

template <int D, int RW>
hipError_t launch(const AttnProblem& p, const AttnPlan& plan, void* workspace, uint32_t* tickets, hipStream_t stream) {
    WaveArgs a;
    a.p = p;
    a.n_splits = plan.n_splits;
    a.row_blocks = plan.m_tiles;
    const int64_t blocks = (int64_t)p.n_items * p.n_kv_heads * plan.m_tiles;
    a.by_splits = fast_div((uint32_t)plan.n_splits);
    a.by_row_blocks = fast_div((uint32_t)plan.m_tiles);
    a.by_items = fast_div((uint32_t)p.n_items);
    a.by_group = fast_div((uint32_t)(p.n_q_heads / p.n_kv_heads));
    a.part = static_cast<float*>(workspace);
    a.tickets = tickets;
    const dim3 grid((unsigned)(blocks * plan.n_splits));
    if (p.is_encode)
        hipLaunchKernelGGL((attn_wave_kernel<D, RW, true, false, false>), grid, dim3(THREADS), 0, stream, a);
    else if (p.a_index)
        hipLaunchKernelGGL((attn_wave_kernel<D, RW, false, true, false>), grid, dim3(THREADS), 0, stream, a);
    else if (RW == 1 && plan.m_tiles == 1)       // (never RW = 2: one row block of up to 32 rows)
        hipLaunchKernelGGL((attn_wave_kernel<D, RW, false, false, RW == 1>), grid, dim3(THREADS), 0, stream, a);
    else
        hipLaunchKernelGGL((attn_wave_kernel<D, RW, false, false, false>), grid, dim3(THREADS), 0, stream, a);
    return hipGetLastError();
}

}  // namespace

hipError_t attn_wave_launch(const AttnProblem& p, const AttnPlan& plan, void* workspace, uint32_t* tickets,
                            hipStream_t stream) {
    if (p.head_dim == 128)
        return plan.wave == 1 ? launch<128, 1>(p, plan, workspace, tickets, stream) : launch<128, 2>(p, plan, workspace, tickets, stream);
    if (p.head_dim == 64)
        return plan.wave == 1 ? launch<64, 1>(p, plan, workspace, tickets, stream) : launch<64, 2>(p, plan, workspace, tickets, stream);
    return hipErrorInvalidValue;
}

}  // namespace rekv

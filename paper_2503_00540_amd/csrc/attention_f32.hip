// fp32 attention for Eq. 1 / Eq. 3 when Q/K/V are stored in fp32.  All arithmetic is fp32.
//
// head_dim 64 and 128: attn_f32_mfma_kernel, the contractions on the matrix cores in true fp32
// (v_mfma_f32_16x16x4_f32: fp32 products and sums).  A wavefront owns 16 query rows of one (item, KV
// head) - the G query heads of the head stacked as row = token * G + head - and computes S^T = K Q^T
// and O^T = V^T P^T, so that a query is an MFMA column; the NW wavefronts of a workgroup share the rows
// and take the key steps in turn, and their (maximum, sum, O) meet in LDS.  Operands come straight
// from global memory in 16-byte loads; the contraction indices are assigned to lanes so that no
// value has to change lanes:
//   Q K^T: lane (r = lane % 16, g = lane / 16) holds dims [g D/4, (g+1) D/4) of key (and query) r; MFMA i
//          contracts the dims {g D/4 + i}.
//   P V:   S^T leaves lane (q, g) with keys 4g + j in register j, so MFMA j contracts the keys {4g + j};
//          a 16-byte load of V row 4g + j at dims 4r.. gives the operands of four MFMAs, and block e
//          of O^T holds the dims {4r + e}, which makes the result four consecutive dims per lane.
// Bound: the fp32 matrix rate (two waves per SIMD each issue 64 MFMAs of 32 clocks per 32-key step).  The
// vector kernel below, which serves the other head sizes, scores one key per lane and reads K and V
// again for every query row.  Measured, vector kernel -> this one (us): the 32 chunks of 16 tokens of the
// tiny configuration 26.2 -> 5.9; 32 chunks of 128 tokens at heads 14/2/64, window 512 tokens, 2824 -> 123;
// 8 chunks of 64 at 28/4/128 1170 -> 71; a 47-token question over 528 keys at 14/2/64 146 -> 12.8.
//
// Other head sizes: attn_f32_kernel, on the vector ALU.  One wavefront per query row (token, head):
// for 64 keys at a time each lane scores one key, the wavefront takes the running maximum
// and sum, and the lanes then own the output dimensions for the P.V accumulation.
#include <type_traits>

#include "common.h"

namespace rekv {
namespace {

constexpr int ROWS_PER_BLOCK = 4;   // one wavefront each
constexpr int MAX_D = 256;

__device__ inline float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
}
__device__ inline float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

__global__ __launch_bounds__(ROWS_PER_BLOCK * 64) void attn_f32_kernel(AttnProblem p) {
    __shared__ float q_lds[ROWS_PER_BLOCK][MAX_D];
    __shared__ float p_lds[ROWS_PER_BLOCK][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int D = p.head_dim;
    const int G = p.n_q_heads / p.n_kv_heads;
    const int item = blockIdx.y;
    const int64_t r = (int64_t)blockIdx.x * ROWS_PER_BLOCK + wave;   // over (token, head)
    if (r >= (int64_t)p.len_q * p.n_q_heads) return;                 // whole wavefront leaves
    const int tok = (int)(r / p.n_q_heads), h = (int)(r % p.n_q_heads), kvh = h / G;
    const ItemSegs seg = item_segments(p, item);
    const int64_t row_stride = (int64_t)p.n_kv_heads * D;
    const bool k_dense = p.a_index && p.a_k_dense;      // re-positioned keys in a dense per-item buffer
    const float* ka = static_cast<const float*>(p.k_a) + (k_dense ? (int64_t)item * p.len_a : seg.a_off) * row_stride + kvh * D;
    const float* va = static_cast<const float*>(p.v_a) + seg.a_off * row_stride + kvh * D;
    const float* kb = static_cast<const float*>(p.k_b) + seg.b_off * row_stride + kvh * D;
    const float* vb = static_cast<const float*>(p.v_b) + seg.b_off * row_stride + kvh * D;
    const int64_t qo = (((int64_t)item * p.len_q + tok) * p.n_q_heads + h) * D;
    const float* q = static_cast<const float*>(p.q) + qo;
    for (int d = lane; d < D; d += 64) q_lds[wave][d] = q[d];
    // q_lds[wave] and p_lds[wave] are private to this wavefront: wave-level ordering suffices
    __builtin_amdgcn_wave_barrier();

    float o[MAX_D / 64] = {0.f, 0.f, 0.f, 0.f};
    // row of segment A's token j in k_a / v_a: j itself, or through the frame index list
    auto a_row = [&](int j) -> int64_t {
        if (!p.a_index) return j;
        const int slot = j / p.n_f;
        int f = p.a_index[(int64_t)item * p.a_index_stride + slot];
        f = f < 0 ? 0 : (f < p.n_src_frames ? f : p.n_src_frames - 1);
        return (int64_t)f * p.n_f + (j - slot * p.n_f);
    };
    float m = -INFINITY, l = 0.f;
    const int n_vis_b = tok + (p.len_b - p.len_q) + 1;   // causal part: text tokens up to itself
    const int n_keys = seg.len_a + n_vis_b;
    for (int j0 = 0; j0 < n_keys; j0 += 64) {
        const int j = j0 + lane;
        float s = -INFINITY;
        const float* vrow = nullptr;
        if (j < n_keys) {
            const float* krow = j < seg.len_a ? ka + (k_dense ? (int64_t)j : a_row(j)) * row_stride
                                              : kb + (int64_t)(j - seg.len_a) * row_stride;
            float acc = 0.f;
            for (int d = 0; d < D; d += 4) {
                const float4 kv = *reinterpret_cast<const float4*>(krow + d);
                acc = fmaf(kv.x, q_lds[wave][d], acc);
                acc = fmaf(kv.y, q_lds[wave][d + 1], acc);
                acc = fmaf(kv.z, q_lds[wave][d + 2], acc);
                acc = fmaf(kv.w, q_lds[wave][d + 3], acc);
            }
            s = acc * p.scale;
        }
        const float m_new = fmaxf(m, wave_max(s));      // finite: key j0 is visible
        const float alpha = expf(m - m_new);            // 0 on the first pass (m = -inf)
        const float pj = (j < n_keys) ? expf(s - m_new) : 0.f;
        l = l * alpha + wave_sum(pj);
        m = m_new;
        p_lds[wave][lane] = pj;
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < MAX_D / 64; ++i) o[i] *= alpha;
        const int cnt = n_keys - j0 < 64 ? n_keys - j0 : 64;
        for (int jj = 0; jj < cnt; ++jj) {
            const int jk = j0 + jj;
            vrow = jk < seg.len_a ? va + a_row(jk) * row_stride
                                  : vb + (int64_t)(jk - seg.len_a) * row_stride;
            const float pv = p_lds[wave][jj];
#pragma unroll
            for (int i = 0; i < MAX_D / 64; ++i) {
                const int d = lane + 64 * i;
                if (d < D) o[i] = fmaf(pv, vrow[d], o[i]);
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    float* out = static_cast<float*>(p.out) + qo;
    const float inv = 1.f / l;
#pragma unroll
    for (int i = 0; i < MAX_D / 64; ++i) {
        const int d = lane + 64 * i;
        if (d < D) out[d] = o[i] * inv;
    }
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

// All four lanes (q, q + 16, q + 32, q + 48) of a query combine a value.
template <bool MAX>
__device__ inline float quad_combine(float v) {
    auto op = [](uint32_t a, uint32_t b) {
        const float x = __uint_as_float(a), y = __uint_as_float(b);
        return MAX ? fmaxf(x, y) : x + y;
    };
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = op(r[0], r[1]);
    const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return op(t[0], t[1]);
}

constexpr int FR = 16;                            // query rows per workgroup

// INDEXED: segment A through a frame index list (a branch per key row that the plain layout is spared).
template <int D, int NW, bool INDEXED>
__global__ __launch_bounds__(NW * 64) void attn_f32_mfma_kernel(AttnProblem p, int row_blocks) {
    constexpr int KB = D == 64 ? 2 : 1;           // 16-key blocks per step
    constexpr int KT = 16 * KB;
    constexpr int QD = D / 4;                     // dims per lane of a Q or K row
    constexpr int VB = D / 64;                    // 64-dim blocks of V and O
    __shared__ f32x4 o_lds[NW][VB * 4][64];
    __shared__ float m_lds[NW][FR], l_lds[NW][FR];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int G = p.n_q_heads / p.n_kv_heads;
    const uint32_t ik = blockIdx.x / (uint32_t)row_blocks;
    const int rb = (int)(blockIdx.x - ik * (uint32_t)row_blocks);
    const int kvh = (int)(ik / (uint32_t)p.n_items), item = (int)(ik - (uint32_t)kvh * (uint32_t)p.n_items);
    const ItemSegs seg = item_segments(p, item);
    const int64_t row_stride = (int64_t)p.n_kv_heads * D;
    const bool k_dense = INDEXED && p.a_k_dense;      // re-positioned keys in a dense per-item buffer
    const float* ka = static_cast<const float*>(p.k_a) + (k_dense ? (int64_t)item * p.len_a : seg.a_off) * row_stride + kvh * D;
    const float* va = static_cast<const float*>(p.v_a) + seg.a_off * row_stride + kvh * D;
    const float* kb = static_cast<const float*>(p.k_b) + seg.b_off * row_stride + kvh * D;
    const float* vb = static_cast<const float*>(p.v_b) + seg.b_off * row_stride + kvh * D;

    const int m_rows = p.len_q * G, row = rb * FR + r;
    const int tok = row / G;
    const bool row_ok = row < m_rows;
    const int q_pos0 = p.len_b - p.len_q;
    const int n_vis = seg.len_a + (tok + q_pos0 + 1 < p.len_b ? tok + q_pos0 + 1 : p.len_b);   // keys this lane's query sees
    int last_tok = (rb * FR + FR - 1) / G;
    if (last_tok > p.len_q - 1) last_tok = p.len_q - 1;
    const int n_keys = seg.len_a + last_tok + q_pos0 + 1;             // keys any row of the block sees
    const int n_steps = (n_keys + KT - 1) / KT;
    const int n_all = seg.len_a + rb * FR / G + q_pos0 + 1;           // keys every row of the block sees
    const int64_t qo = (((int64_t)item * p.len_q + tok) * p.n_q_heads + kvh * G + (row - tok * G)) * D;

    // row of segment A's token j in k_a / v_a: j itself, or through the frame index list
    auto a_row = [&](int j, bool dense) -> int64_t {
        if (!INDEXED || dense) return j;
        const int slot = j / p.n_f;
        int f = p.a_index[(int64_t)item * p.a_index_stride + slot];
        f = f < 0 ? 0 : (f < p.n_src_frames ? f : p.n_src_frames - 1);
        return (int64_t)f * p.n_f + (j - slot * p.n_f);
    };
    f32x4 qf[QD / 4];
#pragma unroll
    for (int i = 0; i < QD / 4; ++i)
        qf[i] = row_ok ? *reinterpret_cast<const f32x4*>(static_cast<const float*>(p.q) + qo + g * QD + i * 4) : f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 o[VB][4];
#pragma unroll
    for (int b = 0; b < VB; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[b][e] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f;
    uint64_t dropped = 0;
    f32x4 kf[KB][QD / 4], vf[KB][4][VB];
    auto load_k = [&](int j0) {
#pragma unroll
        for (int kbk = 0; kbk < KB; ++kbk) {
            int j = j0 + kbk * 16 + r;
            j = j < n_keys ? j : n_keys - 1;      // past the end: the last key again, masked below
            const float* krow = j < seg.len_a ? ka + a_row(j, k_dense) * row_stride : kb + (int64_t)(j - seg.len_a) * row_stride;
#pragma unroll
            for (int i = 0; i < QD / 4; ++i) kf[kbk][i] = *reinterpret_cast<const f32x4*>(krow + g * QD + i * 4);
        }
    };
    // a step's K and V leave together, before its first product (fetching K a step ahead measured the same)
    for (int st = wave; st < n_steps; st += NW) {
        const int j0 = st * KT;
        load_k(j0);
#pragma unroll
        for (int kbk = 0; kbk < KB; ++kbk)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                int j = j0 + kbk * 16 + g * 4 + jj;
                j = j < n_keys ? j : n_keys - 1;
                const float* vrow = j < seg.len_a ? va + a_row(j, false) * row_stride : vb + (int64_t)(j - seg.len_a) * row_stride;
#pragma unroll
                for (int b = 0; b < VB; ++b) vf[kbk][jj][b] = *reinterpret_cast<const f32x4*>(vrow + b * 64 + r * 4);
            }
        __builtin_amdgcn_sched_barrier(0);
        f32x4 s[KB];
        float mx = -INFINITY;
#pragma unroll
        for (int kbk = 0; kbk < KB; ++kbk) {
            f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};     // two chains
#pragma unroll
            for (int i = 0; i < QD / 4; ++i)
#pragma unroll
                for (int c = 0; c < 4; c += 2) {
                    s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[kbk][i][c], qf[i][c], s0, 0, 0, 0);
                    s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[kbk][i][c + 1], qf[i][c + 1], s1, 0, 0, 0);
                }
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                const int j = j0 + kbk * 16 + g * 4 + jj;
                s[kbk][jj] = j < n_vis ? (s0[jj] + s1[jj]) * p.scale : -INFINITY;
                mx = fmaxf(mx, s[kbk][jj]);
            }
        }
        mx = quad_combine<true>(mx);
        const float m_new = fmaxf(m, mx);
        const float m_use = m_new == -INFINITY ? 0.f : m_new;
        const float alpha = expf(m - m_use);      // 0 on the first pass (m = -inf)
        m = m_new;
        l *= alpha;
#pragma unroll
        for (int b = 0; b < VB; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) o[b][e] *= alpha;
        // Where not every row sees every key, a probability of 0 keeps a value out only if that value is finite (0 * inf
        // is NaN): a step with others takes none of its non-finite values, which are added after the loop.
        if (j0 + KT > n_all) {
            float nan_or_0 = 0.f;
#pragma unroll
            for (int kbk = 0; kbk < KB; ++kbk)
#pragma unroll
                for (int jj = 0; jj < 4; ++jj)
#pragma unroll
                    for (int b = 0; b < VB; ++b)
#pragma unroll
                        for (int e = 0; e < 4; ++e) nan_or_0 = fmaf(vf[kbk][jj][b][e], 0.f, nan_or_0);
            const uint64_t some = __builtin_amdgcn_ballot_w64(nan_or_0 != 0.f);
            if (some != 0) {
                dropped |= some;
#pragma unroll
                for (int kbk = 0; kbk < KB; ++kbk)
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj)
#pragma unroll
                        for (int b = 0; b < VB; ++b)
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                vf[kbk][jj][b][e] = __builtin_fabsf(vf[kbk][jj][b][e]) < INFINITY ? vf[kbk][jj][b][e] : 0.f;
            }
        }
#pragma unroll
        for (int kbk = 0; kbk < KB; ++kbk)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                const float pj = expf(s[kbk][jj] - m_use);
                l += pj;
#pragma unroll
                for (int b = 0; b < VB; ++b)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        o[b][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[kbk][jj][b][e], pj, o[b][e], 0, 0, 0);
            }
    }
    // lane (q = r, g), register i of block e of o[b]: dim b*64 + 4*(4g + i) + e
    if (dropped != 0) {
        // worked out again, so that the loop above does not carry in registers what only this block needs
        const int lane2 = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        const int g2 = lane2 >> 4, row2 = rb * FR + (lane2 & 15), tok2 = row2 / G;
        const int n_vis2 = row2 < m_rows ? seg.len_a + tok2 + q_pos0 + 1 : 0;
        const float* qrow = static_cast<const float*>(p.q) + (((int64_t)item * p.len_q + tok2) * p.n_q_heads + kvh * G + (row2 - tok2 * G)) * D;
        for (int st = wave; st < n_steps; st += NW) {
            if (st * KT + KT <= n_all) continue;
            for (int j = st * KT; j < st * KT + KT && j < n_vis2; ++j) {
                const float* krow = j < seg.len_a ? ka + a_row(j, k_dense) * row_stride : kb + (int64_t)(j - seg.len_a) * row_stride;
                const float* vrow = j < seg.len_a ? va + a_row(j, false) * row_stride : vb + (int64_t)(j - seg.len_a) * row_stride;
                float s = 0.f;
#pragma unroll 1
                for (int i = 0; i < D; ++i) s = fmaf(krow[i], qrow[i], s);
                const float pj = expf(s * p.scale - (m == -INFINITY ? 0.f : m));
#pragma unroll
                for (int b = 0; b < VB; ++b)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float v = vrow[b * 64 + g2 * 16 + i * 4 + e];
                            if (!(__builtin_fabsf(v) < INFINITY)) o[b][e][i] = fmaf(pj, v, o[b][e][i]);
                        }
            }
        }
    }
    l = quad_combine<false>(l);
    float* out = static_cast<float*>(p.out) + qo;
    if constexpr (NW == 1) {
        if (!row_ok) return;
        const float inv = 1.f / l;
#pragma unroll
        for (int b = 0; b < VB; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *reinterpret_cast<f32x4*>(out + b * 64 + g * 16 + i * 4) =
                    f32x4{o[b][0][i] * inv, o[b][1][i] * inv, o[b][2][i] * inv, o[b][3][i] * inv};
    } else {
#pragma unroll
        for (int b = 0; b < VB; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i) o_lds[wave][b * 4 + i][lane] = f32x4{o[b][0][i], o[b][1][i], o[b][2][i], o[b][3][i]};
        if (g == 0) {
            m_lds[wave][r] = m;
            l_lds[wave][r] = l;
        }
        __syncthreads();
        float m_all = m_lds[0][r], l_all = 0.f, w[NW];
#pragma unroll
        for (int i = 1; i < NW; ++i) m_all = fmaxf(m_all, m_lds[i][r]);
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            w[i] = m_lds[i][r] == -INFINITY ? 0.f : expf(m_lds[i][r] - m_all);
            l_all += l_lds[i][r] * w[i];
        }
        const float inv = 1.f / l_all;
        for (int x = wave; x < VB * 4; x += NW) {         // x: 16-byte chunk (b, i) of the lane's row
            f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < NW; ++i) sum += o_lds[i][x][lane] * w[i];
            if (row_ok) *reinterpret_cast<f32x4*>(out + (x >> 2) * 64 + g * 16 + (x & 3) * 4) = sum * inv;
        }
    }
}

template <int D>
hipError_t launch_mfma(const AttnProblem& p, hipStream_t stream) {
    const int64_t row_blocks = ((int64_t)p.len_q * (p.n_q_heads / p.n_kv_heads) + FR - 1) / FR;
    const int64_t blocks = row_blocks * p.n_items * p.n_kv_heads;
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    // Wavefronts per row block: enough to bring the launch near four per SIMD (4096 in all), but one where the longest item has a
    // single step of keys and four where it has up to four: more of them only lengthen the merge (32 chunks of 16 tokens with a window
    // of 64 at 4/1/64, eight wavefronts and four 5.3 and 5.0 us; 8 chunks of 50 with 60 at 14/2/64 9.0 and 7.4; one step, eight and one 4.8
    // and 4.0).
    constexpr int KT = D == 64 ? 32 : 16;         // keys of a step
    int64_t len_a = p.is_encode ? p.l_l : p.len_a;
    if (p.is_encode) {
        const int64_t past = p.first_token + (int64_t)(p.n_items - 1) * p.len_b;
        if (past < len_a) len_a = past;
    }
    const int64_t steps = (len_a + p.len_b + KT - 1) / KT;
    auto go = [&](auto indexed) {
        constexpr bool IX = decltype(indexed)::value;
        const dim3 grid((unsigned)blocks);
        if (blocks >= 4096 || steps == 1)
            hipLaunchKernelGGL((attn_f32_mfma_kernel<D, 1, IX>), grid, dim3(64), 0, stream, p, (int)row_blocks);
        else if (blocks >= 1024 || steps <= 4)
            hipLaunchKernelGGL((attn_f32_mfma_kernel<D, 4, IX>), grid, dim3(256), 0, stream, p, (int)row_blocks);
        else
            hipLaunchKernelGGL((attn_f32_mfma_kernel<D, 8, IX>), grid, dim3(512), 0, stream, p, (int)row_blocks);
    };
    if (p.a_index) go(std::true_type{});
    else go(std::false_type{});
    return hipGetLastError();
}

}  // namespace

hipError_t attn_f32_launch(const AttnProblem& p, hipStream_t stream) {
    if (p.head_dim == 64) return launch_mfma<64>(p, stream);
    if (p.head_dim == 128) return launch_mfma<128>(p, stream);
    const int64_t rows = (int64_t)p.len_q * p.n_q_heads;
    dim3 grid((unsigned)((rows + ROWS_PER_BLOCK - 1) / ROWS_PER_BLOCK), (unsigned)p.n_items);
    hipLaunchKernelGGL(attn_f32_kernel, grid, dim3(ROWS_PER_BLOCK * 64), 0, stream, p);
    return hipGetLastError();
}

}  // namespace rekv

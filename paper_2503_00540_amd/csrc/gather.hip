// Reload of the retrieved KV: a block copy of whole frames, selected by a device index
// list, from the K and V arenas into one dense buffer per question.  Pure data movement, bound by
// HBM (or by the host link).
//
// A workgroup moves one 4 KB slice, a single 16-byte access per thread, and consecutive workgroups
// move consecutive slices of a frame, so that what is in flight at a time is a few long runs of
// both arrays.  Measured (7B-class frames of 196 KB, 28 x 32 different ones; 72B-class of 288 KB, 64 x 32
// picks from 2,048; read + write): this order 110 us = 6.5 TB/s and 352 us; slices of 16 KB in the same
// order 118 and 374 us; one slice of every frame before the next slice (4 or 16 KB: 132 and 134, 384 us), which
// scatters the writes over strides of a frame; whole frames of all questions' same slot together 116 and 361 us.
// Loads stay cached (questions share frames), stores are non-temporal.
#include "common.h"

namespace rekv {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
constexpr int GATHER_THREADS = 256;
constexpr size_t SLICE = (size_t)GATHER_THREADS * 16;            // bytes per workgroup
constexpr int MAX_GRID_Y = 65535;

// One slice of one frame; frames outside the arena (and the -1 of padded selections) become zeros.
__device__ inline void move_slice(const char* __restrict__ arena, int f, int n_src_frames, size_t frame_bytes,
                                  size_t slice, char* __restrict__ dst) {
    const size_t off = slice * SLICE + (size_t)threadIdx.x * 16;
    if (off >= frame_bytes) return;
    u32x4 v = {0u, 0u, 0u, 0u};
    if (f >= 0 && f < n_src_frames) v = *reinterpret_cast<const u32x4*>(arena + (size_t)f * frame_bytes + off);
    __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(dst + off));
}

// Grid of the device-source copies: slices of a frame fastest, then the blocks (y, and where there are more than a
// grid dimension takes, z), keys before values.
dim3 copy_grid(int n_blocks, size_t frame_bytes, int n_tensors) {
    const int ny = n_blocks < MAX_GRID_Y ? n_blocks : MAX_GRID_Y;
    return dim3((unsigned)((frame_bytes + SLICE - 1) / SLICE), (unsigned)ny, (unsigned)((n_blocks + ny - 1) / ny * n_tensors));
}
// This workgroup's block (over (question, selected slot)) and tensor (0: keys, 1: values).
__device__ inline int64_t copy_block(int n_tensors, int* z) {
    const int chunks = gridDim.z / n_tensors;
    *z = n_tensors > 1 && (int)blockIdx.z >= chunks;
    return (int64_t)(blockIdx.z - *z * chunks) * gridDim.y + blockIdx.y;
}

// values_only: the rope variant turns the keys itself
__global__ __launch_bounds__(GATHER_THREADS) void gather_kernel(
    const char* __restrict__ src_k, const char* __restrict__ src_v, int n_src_frames,
    const int32_t* __restrict__ idx, int n_blocks, size_t frame_bytes, char* __restrict__ dst_k,
    char* __restrict__ dst_v, int values_only) {
    int z;
    const int64_t blk = copy_block(values_only ? 1 : 2, &z);
    if (blk >= n_blocks) return;
    z |= values_only;
    move_slice(z ? src_v : src_k, idx[blk], n_src_frames, frame_bytes, blockIdx.x,
               (z ? dst_v : dst_k) + (size_t)blk * frame_bytes);
}

// The same copy from pinned host memory.  The link is fastest with little in flight: 51 MB again and again take
// 508 us (50.5 GB/s) with a workgroup for every slice of 4 KB, 454 us (56.6 GB/s) with 64 or 96 workgroups walking the slices
// in order, 457 and 459 us with 256 and 512, 525 us with 32.  Host pages the GPU has not read lately need more
// requests in flight to hide their address translation: a question's first pass over new arrays takes 720 us with
// a workgroup per slice or with 512 workgroups, 800 to 900 us with 64 to 256.
constexpr int HOST_WORKGROUPS = 512;
__global__ __launch_bounds__(GATHER_THREADS) void gather_host_kernel(
    const char* __restrict__ src_k, const char* __restrict__ src_v, int n_src_frames,
    const int32_t* __restrict__ idx, int n_blocks, size_t frame_bytes, int n_slices, char* __restrict__ dst_k,
    char* __restrict__ dst_v, int values_only) {
    const int64_t per_tensor = (int64_t)n_blocks * n_slices;
    for (int64_t u = blockIdx.x; u < per_tensor * (values_only ? 1 : 2); u += gridDim.x) {
        const int z = values_only || u >= per_tensor;
        const int64_t w = !values_only && z ? u - per_tensor : u;
        const int64_t blk = w / n_slices;
        move_slice(z ? src_v : src_k, idx[blk], n_src_frames, frame_bytes, (size_t)(w - blk * n_slices),
                   (z ? dst_v : dst_k) + (size_t)blk * frame_bytes);
    }
}

hipError_t copy_launch(const void* src_k, const void* src_v, bool src_on_host, int n_src_frames, const int32_t* idx,
                       int n_blocks, size_t frame_bytes, void* dst_k, void* dst_v, int values_only, hipStream_t stream) {
    const char *sk = static_cast<const char*>(src_k), *sv = static_cast<const char*>(src_v);
    char *dk = static_cast<char*>(dst_k), *dv = static_cast<char*>(dst_v);
    const int n_slices = (int)((frame_bytes + SLICE - 1) / SLICE);
    if (src_on_host)
        hipLaunchKernelGGL(gather_host_kernel, dim3(HOST_WORKGROUPS), dim3(GATHER_THREADS), 0, stream, sk, sv, n_src_frames,
                           idx, n_blocks, frame_bytes, n_slices, dk, dv, values_only);
    else
        hipLaunchKernelGGL(gather_kernel, copy_grid(n_blocks, frame_bytes, values_only ? 1 : 2), dim3(GATHER_THREADS), 0,
                           stream, sk, sv, n_src_frames, idx, n_blocks, frame_bytes, dk, dv, values_only);
    return hipGetLastError();
}

// The same block copy for several layers in one launch (every layer retrieves its own frames from
// its own arenas): the arenas' base pointers travel in the kernel arguments.
struct LayerArenas {
    const char* k[MAX_GATHER_LAYERS];
    const char* v[MAX_GATHER_LAYERS];
};

__global__ __launch_bounds__(GATHER_THREADS) void gather_layers_kernel(
    LayerArenas arenas, int blocks_per_layer, int n_src_frames, const int32_t* __restrict__ idx, int n_blocks,
    size_t frame_bytes, char* __restrict__ dst_k, char* __restrict__ dst_v) {
    int z;
    const int64_t blk = copy_block(2, &z);       // over (layer, question, selected slot)
    if (blk >= n_blocks) return;
    const int layer = (int)blk / blocks_per_layer;
    move_slice(z ? arenas.v[layer] : arenas.k[layer], idx[blk], n_src_frames, frame_bytes, blockIdx.x,
               (z ? dst_v : dst_k) + (size_t)blk * frame_bytes);
}

// Keys of the selected frames, turned to their positions in the question-answering context.
// A unit of work is one (token, KV head, column chunk c): the 16-byte chunk at dims
// [c*EPC, (c+1)*EPC) and its partner at + D/2, which hold both members of EPC rotary pairs
// ("half" layout: element e of the first chunk pairs with element e of the second) or EPC/2
// whole pairs each ("interleaved": neighbours pair up).  The pair frequencies theta_i =
// base^(-2i/D) are set up once per workgroup in double precision; the angle position * theta_i
// is formed and reduced to a fraction of a turn in double precision too, so positions in the
// hundreds of thousands lose nothing, and the hardware sine and cosine take it from there.
// Grid: blocks in x, a block's units interleaved over y, so that what is in flight spreads over many frames.  A run of units per
// workgroup in address order, as the plain copy has it, is slower for keys (keys and values, us): 42 frames of 196 KB 10.3
// against 9.4 so, 41 of 388 KB 15.1 and 14.0, 35 questions x 46 of 392 KB 349 and 293.  From host memory 512
// workgroups and one per frame part take the same (51 MB: 557 us).
template <bool BF16>
__global__ __launch_bounds__(GATHER_THREADS) void gather_rope_kernel(
    const char* __restrict__ src_k, int n_src_frames, const int32_t* __restrict__ idx, int64_t n_blocks, int k_slots,
    int n_f, int n_kv_heads, int d, char* __restrict__ dst_k, RopeArgs ra) {
    constexpr int EPC = BF16 ? 8 : 4;            // elements per 16-byte chunk
    __shared__ double theta[128];                // D / 2 <= 128 pair frequencies
    const int half = d / 2;
    for (int i = threadIdx.x; i < half; i += GATHER_THREADS)
        theta[i] = exp2(-(2.0 * i / d) * ra.log2_base);
    __syncthreads();
    const int cpr = half / EPC;                  // chunk pairs per head row
    const int units = n_f * n_kv_heads * cpr;
    const size_t row_bytes = (size_t)n_kv_heads * d * (BF16 ? 2 : 4);
    for (int64_t blk = blockIdx.x; blk < n_blocks; blk += gridDim.x) {     // over (question, selected slot)
        const int f = idx[blk];
        const bool have = f >= 0 && f < n_src_frames;
        const int slot = (int)(blk % k_slots);
        const char* src = src_k + (size_t)(have ? f : 0) * n_f * row_bytes;
        char* dst = dst_k + (size_t)blk * n_f * row_bytes;
        for (int u = blockIdx.y * GATHER_THREADS + threadIdx.x; u < units; u += gridDim.y * GATHER_THREADS) {
            const int c = u % cpr, th = u / cpr;     // th = token * Hkv + head
            const int tok = th / n_kv_heads;
            const size_t off = ((size_t)th * d + (size_t)c * EPC) * (BF16 ? 2 : 4);
            u32x4 lo = {0u, 0u, 0u, 0u}, hi = {0u, 0u, 0u, 0u};
            if (have) {
                lo = *reinterpret_cast<const u32x4*>(src + off);
                hi = *reinterpret_cast<const u32x4*>(src + off + (size_t)half * (BF16 ? 2 : 4));
                const int64_t new_pos = ra.pos_offset + (ra.is_static ? 0 : (int64_t)slot * n_f + tok);
                const int64_t old_pos = ra.src_rotated ? ra.src_pos_offset + (int64_t)f * n_f + tok : 0;
                const double delta = (double)(new_pos - old_pos);
                float x[2 * EPC];                    // first chunk, then its partner
                if (BF16) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        x[2 * i] = __uint_as_float(lo[i] << 16);
                        x[2 * i + 1] = __uint_as_float(lo[i] & 0xffff0000u);
                        x[EPC + 2 * i] = __uint_as_float(hi[i] << 16);
                        x[EPC + 2 * i + 1] = __uint_as_float(hi[i] & 0xffff0000u);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        x[i] = __uint_as_float(lo[i]);
                        x[EPC + i] = __uint_as_float(hi[i]);
                    }
                }
#pragma unroll
                for (int e = 0; e < EPC; ++e) {
                    // pair e of this unit: its frequency index and its two members in x[]
                    int ti, ia, ib;
                    if (ra.interleaved) {
                        const int in_hi = e >= EPC / 2, m = e - in_hi * (EPC / 2);
                        ti = (in_hi ? half / 2 : 0) + c * (EPC / 2) + m;
                        ia = in_hi * EPC + 2 * m;
                        ib = ia + 1;
                    } else {
                        ti = c * EPC + e;
                        ia = e;
                        ib = EPC + e;
                    }
                    const double turns = delta * theta[ti] * 0.15915494309189535;   // 1 / (2 pi)
                    const float fr = (float)(turns - rint(turns));                    // in [-0.5, 0.5]
                    const float cs = __builtin_amdgcn_cosf(fr), sn = __builtin_amdgcn_sinf(fr);
                    const float a_ = x[ia], b_ = x[ib];
                    x[ia] = a_ * cs - b_ * sn;
                    x[ib] = a_ * sn + b_ * cs;
                }
                if (BF16) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        f32x2 pl = {x[2 * i], x[2 * i + 1]}, ph = {x[EPC + 2 * i], x[EPC + 2 * i + 1]};
                        lo[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pl, bf16x2));
                        hi[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(ph, bf16x2));
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        lo[i] = __float_as_uint(x[i]);
                        hi[i] = __float_as_uint(x[EPC + i]);
                    }
                }
            }
            __builtin_nontemporal_store(lo, reinterpret_cast<u32x4*>(dst + off));
            __builtin_nontemporal_store(hi, reinterpret_cast<u32x4*>(dst + off + (size_t)half * (BF16 ? 2 : 4)));
        }
    }
}

}  // namespace

hipError_t gather_rope_launch(const void* src_k, const void* src_v, bool src_on_host, int n_src_frames,
                              const int32_t* idx, int n_questions, int k_slots, int n_f, int n_kv_heads, int d,
                              int dtype, void* dst_k, void* dst_v, const RopeArgs& ra, hipStream_t stream) {
    const int64_t n_blocks = (int64_t)n_questions * k_slots;
    const size_t es = dtype == REKV_BF16 ? 2 : 4;
    const size_t frame_bytes = (size_t)n_f * n_kv_heads * d * es;
    if (dst_v) {                       // values: the plain block copy (skipped when only keys are wanted)
        hipError_t e = copy_launch(src_k, src_v, src_on_host, n_src_frames, idx, (int)n_blocks, frame_bytes, dst_k, dst_v, 1,
                                   stream);
        if (e != hipSuccess) return e;
    }
    const int units = n_f * n_kv_heads * (d / 2) / (dtype == REKV_BF16 ? 8 : 4);
    int gy = (units + GATHER_THREADS * 4 - 1) / (GATHER_THREADS * 4);      // about 4 units per thread
    if (gy < 1) gy = 1;
    const dim3 kgrid((unsigned)(n_blocks < (1 << 22) ? n_blocks : (1 << 22)), (unsigned)gy);
    if (dtype == REKV_BF16)
        hipLaunchKernelGGL(gather_rope_kernel<true>, kgrid, dim3(GATHER_THREADS), 0, stream,
                           static_cast<const char*>(src_k), n_src_frames, idx, n_blocks, k_slots, n_f, n_kv_heads, d,
                           static_cast<char*>(dst_k), ra);
    else
        hipLaunchKernelGGL(gather_rope_kernel<false>, kgrid, dim3(GATHER_THREADS), 0, stream,
                           static_cast<const char*>(src_k), n_src_frames, idx, n_blocks, k_slots, n_f, n_kv_heads, d,
                           static_cast<char*>(dst_k), ra);
    return hipGetLastError();
}

hipError_t gather_layers_launch(const void* const* src_k, const void* const* src_v, int n_layers, int n_src_frames,
                                const int32_t* idx, int blocks_per_layer, size_t frame_bytes, void* dst_k, void* dst_v,
                                hipStream_t stream) {
    LayerArenas arenas;
    for (int i = 0; i < MAX_GATHER_LAYERS; ++i) {
        arenas.k[i] = static_cast<const char*>(src_k[i < n_layers ? i : 0]);
        arenas.v[i] = static_cast<const char*>(src_v[i < n_layers ? i : 0]);
    }
    const int n_blocks = n_layers * blocks_per_layer;
    hipLaunchKernelGGL(gather_layers_kernel, copy_grid(n_blocks, frame_bytes, 2), dim3(GATHER_THREADS), 0, stream, arenas,
                       blocks_per_layer, n_src_frames, idx, n_blocks, frame_bytes, static_cast<char*>(dst_k),
                       static_cast<char*>(dst_v));
    return hipGetLastError();
}

hipError_t gather_launch(const void* src_k, const void* src_v, bool src_on_host, int n_src_frames, const int32_t* idx,
                         int n_blocks, size_t frame_bytes, void* dst_k, void* dst_v, hipStream_t stream) {
    return copy_launch(src_k, src_v, src_on_host, n_src_frames, idx, n_blocks, frame_bytes, dst_k, dst_v, 0, stream);
}

}  // namespace rekv

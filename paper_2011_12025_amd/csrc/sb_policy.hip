// Heuristic downsampling policy: the per-block detail score and the per-image
// selection of the blocks to process at high resolution (the policy of the
// short paper SegBlocks grew out of, which its ablation on execution
// policies compares with; the paper's reinforcement-learned policy network
// needs trained weights and is out of scope).
//
// Score of block k: for every pixel of the block the Euclidean distance over
// the channels between the pixel and the block's low-resolution version at
// that pixel (the 2x2 average of its cell, computed and rounded as
// BlockSample does, nearest-upsampled), averaged over the bs x bs pixels.
// One workgroup per block; a thread takes 2x2 cells and all their channels
// (the four pixel norms need every channel of the cell), sums in fp32, and
// the workgroup reduces in a fixed tree.
//
// Selection: per image, the k = round(tau * GH * GW) blocks with the highest
// scores are high resolution; equal scores are ranked by block id (lower
// first).  Every block is ranked against all others of its image in LDS: exact
// and independent of timing.
#include "sb_common.h"
#include "sb_kernels.h"

namespace sb {

namespace {

// Element (n, c, Y, X) of a dense map.
template <typename T, int L>
__device__ __forceinline__ T px(const T* __restrict__ x, int n, int C, int H, int W, int Y, int X, int c) {
    if constexpr (L == NHWC) return x[(((size_t)n * H + Y) * W + X) * C + c];
    else                     return x[(((size_t)n * C + c) * H + Y) * W + X];
}

// Squared distances of the four pixels a, b, cc, d of a cell to its average, one channel.
template <typename T>
__device__ __forceinline__ void cell_channel(T a, T b, T cc, T d, float (&d2)[4]) {
    const float m = to_f32(avg4(a, b, cc, d));
    const float e0 = to_f32(a) - m, e1 = to_f32(b) - m, e2 = to_f32(cc) - m, e3 = to_f32(d) - m;
    d2[0] += e0 * e0;
    d2[1] += e1 * e1;
    d2[2] += e2 * e2;
    d2[3] += e3 * e3;
}
__device__ __forceinline__ float cell_norms(const float (&d2)[4]) {
    return (__builtin_sqrtf(d2[0]) + __builtin_sqrtf(d2[1])) + (__builtin_sqrtf(d2[2]) + __builtin_sqrtf(d2[3]));
}

// Two horizontally adjacent pixels of an image of C <= 4 channels, from an
// even column: 2 C elements, loaded together (aligned to two elements).
// Channels-last: they are contiguous; NCHW: two elements of every plane.
template <typename T, int L, int C>
struct PixPair {
    T e[2 * C];  // [channel][pixel] for NCHW, [pixel][channel] for NHWC
    __device__ __forceinline__ void load(const T* __restrict__ x, int n, int H, int W, int Y, int X) {
        if constexpr (L == NHWC) {
            __builtin_memcpy(e, __builtin_assume_aligned(x + (((size_t)n * H + Y) * W + X) * C, 2 * sizeof(T)),
                             sizeof(e));
        } else {
#pragma unroll
            for (int c = 0; c < C; ++c)
                __builtin_memcpy(e + 2 * c,
                                 __builtin_assume_aligned(x + (((size_t)n * C + c) * H + Y) * W + X, 2 * sizeof(T)),
                                 2 * sizeof(T));
        }
    }
    __device__ __forceinline__ T at(int k, int c) const { return L == NHWC ? e[k * C + c] : e[2 * c + k]; }
};

// C = 0: any channel count, element by element.  C = 1..4 (the images the
// policy runs on; W is even and x aligned to two elements): a cell is two
// loads a channel plane or two loads in all, four cells of a thread in flight
// together.  Bound by the latency of those loads: at 1x3x1024x2048 fp16 with
// 128-pixel blocks there are 128 workgroups, so each takes 1024 threads
// (16 waves a CU) instead of 256: 17.4 -> 7.3 us, the selection 4.3 -> 2.5.
// How many blocks the other images of the call add must not show in a score, so
// both sum a block alike: 256 threads with V = 4 keep the four sums of threads
// t, t + 256, ... of the 1024 apart and add them as those would.
template <typename T, int L, int C, int NT, int V>
__global__ __launch_bounds__(NT) void k_policy_score(const T* __restrict__ x, int Cn, int H, int W, int bs, int GH,
                                                     int GW, float* __restrict__ score) {
    const int k = (int)blockIdx.x;
    const int per = GH * GW;
    const int n = k / per, r = k - n * per, gy = r / GW, gx = r - gy * GW;
    const int lb = bs >> 1, cells = lb * lb;
    float acc[V] = {};
    if constexpr (C > 0) {
        constexpr int U = 4;
        static_assert(U % V == 0, "a sum's cells come in order");
        for (int base = (int)threadIdx.x; base < cells; base += U * NT) {
            PixPair<T, L, C> t[U], b[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int cell = min(base + u * NT, cells - 1);  // past the end: a load that is not used
                const int ci = cell / lb, cj = cell - ci * lb;
                const int Y = gy * bs + 2 * ci, X = gx * bs + 2 * cj;
                t[u].load(x, n, H, W, Y, X);
                b[u].load(x, n, H, W, Y + 1, X);
            }
            __builtin_amdgcn_sched_barrier(0);  // (every load before the first use)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float d2[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int c = 0; c < C; ++c) cell_channel(t[u].at(0, c), t[u].at(1, c), b[u].at(0, c), b[u].at(1, c), d2);
                acc[u % V] += base + u * NT < cells ? cell_norms(d2) : 0.0f;
            }
        }
    } else {
        for (int base = (int)threadIdx.x; base < cells; base += V * NT) {
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const int cell = base + v * NT;
                if (cell >= cells) break;
                const int ci = cell / lb, cj = cell - ci * lb;
                const int Y = gy * bs + 2 * ci, X = gx * bs + 2 * cj;
                float d2[4] = {0.f, 0.f, 0.f, 0.f};
                for (int c = 0; c < Cn; ++c)
                    cell_channel(px<T, L>(x, n, Cn, H, W, Y, X, c), px<T, L>(x, n, Cn, H, W, Y, X + 1, c),
                                 px<T, L>(x, n, Cn, H, W, Y + 1, X, c), px<T, L>(x, n, Cn, H, W, Y + 1, X + 1, c), d2);
                acc[v] += cell_norms(d2);
            }
        }
    }
    // fixed-order reduction: lanes of a wave, then the waves (of the NT * V sums)
    constexpr int WAVES = NT * V / 64;
    __shared__ float s_part[WAVES];
    const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
    if constexpr (V == 4) {  // four sums: half of the lanes go on with two of them, then a quarter with each
        const bool up = lane & 32, upper = lane & 16;
        float k[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) k[i] = (up ? acc[2 + i] : acc[i]) + __shfl_xor(up ? acc[i] : acc[2 + i], 32, 64);
        float a = (upper ? k[1] : k[0]) + __shfl_xor(upper ? k[0] : k[1], 16, 64);
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) a += __shfl_xor(a, o, 64);
        if ((lane & 15) == 0) s_part[(lane >> 4) * (NT / 64) + wave] = a;
    } else {
        static_assert(V == 1, "one sum or four");
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) acc[0] += __shfl_xor(acc[0], o, 64);
        if (lane == 0) s_part[wave] = acc[0];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        // in pairs: sixteen sums one after the other round half as much again
        float t[WAVES];
#pragma unroll
        for (int w = 0; w < WAVES; ++w) t[w] = s_part[w];
#pragma unroll
        for (int h = WAVES / 2; h > 0; h >>= 1)
#pragma unroll
            for (int w = 0; w < h; ++w) t[w] += t[w + h];
        score[k] = t[0] / (float)(bs * bs);
    }
}

constexpr int POL_MAXB = 8192;  // blocks per image the LDS score table holds
constexpr int POL_ROWS = 64;    // blocks ranked by one workgroup, four threads each

// Workgroup (image, group of 64 blocks): a block's rank is the number of
// blocks ahead of it; its four threads count a quarter of the scores each
// (neighbouring lanes, so the four reads of a step are one LDS word apart).
__global__ __launch_bounds__(WG) void k_policy_select(const float* __restrict__ score, int per, int groups, int khigh,
                                                      uint8_t* __restrict__ mask) {
    __shared__ float s[POL_MAXB];
    const int n = (int)blockIdx.x / groups, grp = (int)blockIdx.x - n * groups;
    const float* sc = score + (size_t)n * per;
    for (int i = (int)threadIdx.x; i < per; i += WG) s[i] = sc[i];
    __syncthreads();
    const int b = grp * POL_ROWS + ((int)threadIdx.x >> 2), q = (int)threadIdx.x & 3;
    const float v = s[min(b, per - 1)];
    int rank = 0;
#pragma unroll 8
    for (int j = q; j < per; j += 4) {
        const float t = s[j];
        rank += (t > v || (t == v && j < b)) ? 1 : 0;
    }
    rank += __shfl_xor(rank, 1, 64);
    rank += __shfl_xor(rank, 2, 64);
    if (b < per && q == 0) mask[(size_t)n * per + b] = rank < khigh ? 1 : 0;
}

template <typename T, int L, int C>
void score_run(const void* x, int Cn, int H, int W, int bs, int GH, int GW, long long B, float* score, hipStream_t st) {
    // 1024 threads where a block has four cells for each (1024x2048 images with
    // 128-pixel blocks, four at once: 16.5 -> 14.5 us), or one and the blocks
    // alone would leave less than two workgroups of 256 for every CU (512 blocks
    // of 64 pixels an image, three images: 15.1 us with 256 threads, 19.2 with
    // 1024).  A launch holds 2^32 threads.
    auto run = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)B), dim3(threads), 0, st, (const T*)x, Cn, H, W, bs, GH, GW, score);
    };
    const int cells = (bs / 2) * (bs / 2);
    if (cells < 1024) run(k_policy_score<T, L, C, WG, 1>, WG);
    else if ((cells >= 4096 && B < (1LL << 22)) || B < 2LL * device_cus()) run(k_policy_score<T, L, C, 1024, 1>, 1024);
    else run(k_policy_score<T, L, C, WG, 4>, WG);
}

template <typename T, int L>
hipError_t policy_t(const void* x, int N, int C, int H, int W, int bs, float* score, int khigh, uint8_t* mask,
                    hipStream_t st) {
    const int GH = H / bs, GW = W / bs;
    const long long B = (long long)N * GH * GW;
    // (W is even: blocks are)
    const bool pairs = (reinterpret_cast<uintptr_t>(x) & (2 * sizeof(T) - 1)) == 0;
    switch (pairs ? C : 0) {
    case 1: score_run<T, L, 1>(x, C, H, W, bs, GH, GW, B, score, st); break;
    case 2: score_run<T, L, 2>(x, C, H, W, bs, GH, GW, B, score, st); break;
    case 3: score_run<T, L, 3>(x, C, H, W, bs, GH, GW, B, score, st); break;
    case 4: score_run<T, L, 4>(x, C, H, W, bs, GH, GW, B, score, st); break;
    default: score_run<T, L, 0>(x, C, H, W, bs, GH, GW, B, score, st); break;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int groups = (GH * GW + POL_ROWS - 1) / POL_ROWS;
    hipLaunchKernelGGL(k_policy_select, dim3((unsigned)(N * groups)), dim3(WG), 0, st, (const float*)score, GH * GW,
                       groups, khigh, mask);
    return hipGetLastError();
}

}  // namespace

int policy_max_blocks() { return POL_MAXB; }

hipError_t launch_policy(int dtype, int layout, const void* x, int N, int C, int H, int W, int bs, float* score,
                         int khigh, uint8_t* mask, hipStream_t st) {
    switch (dtype) {
    case 0: return layout == NHWC ? policy_t<float, NHWC>(x, N, C, H, W, bs, score, khigh, mask, st)
                                  : policy_t<float, NCHW>(x, N, C, H, W, bs, score, khigh, mask, st);
    case 1: return layout == NHWC ? policy_t<f16, NHWC>(x, N, C, H, W, bs, score, khigh, mask, st)
                                  : policy_t<f16, NCHW>(x, N, C, H, W, bs, score, khigh, mask, st);
    default: return layout == NHWC ? policy_t<bf16, NHWC>(x, N, C, H, W, bs, score, khigh, mask, st)
                                  : policy_t<bf16, NCHW>(x, N, C, H, W, bs, score, khigh, mask, st);
    }
}

}  // namespace sb

// The 7x7/2 stem of an image with at most four channels, with what follows or
// precedes it fused into its epilogue or its tile load (channels-last fp16 /
// bf16):
//
//   k_stem_pool    dense stem, bias, ReLU and 3x3/2 max-pool: the stem's map,
//                  four times the size of the pooled one, never reaches memory.
//   k_stem_blocks  the stem on image blocks: BlockSample and the 3-pixel
//                  BlockPad are done in the tile load, straight from the image,
//                  so neither image stacks nor padded stacks exist; bias and
//                  optional ReLU, packed stacks out.
//   k_pool_blocks  3x3/2 max-pool of packed stacks with the one-pixel BlockPad
//                  fused into the loads.
//
// K is ordered (ky, kx padded to 8, channel padded to 4) as in the dense stem
// kernel: the 8 K values of an MFMA operand lane are two adjacent pixels of
// the LDS tile, one 16-byte read at stride 2.  The pixel of the padding column
// kx = 7 is cleared in the operand, so that an infinity there cannot reach the
// sum through its zero weight.  The weights of a wave's 64 output channels
// stay in registers (7 x 4 operands) for the whole tile: a row of 2 x 16
// pixels then reads 14 operands from LDS for its 56 MFMAs, where reading the
// weights as well would make LDS the bound.
#include "sb_common.h"
#include "sb_kernels.h"
#include "sb_pixel.h"

namespace sb {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

template <typename T> struct SMF;
template <> struct SMF<f16> {
    typedef halfx8 frag;
    static __device__ __forceinline__ floatx4 mma(uint4 a, uint4 b, floatx4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(frag, a), __builtin_bit_cast(frag, b), c, 0, 0, 0);
    }
};
template <> struct SMF<bf16> {
    typedef bf16x8 frag;
    static __device__ __forceinline__ floatx4 mma(uint4 a, uint4 b, floatx4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(frag, a), __builtin_bit_cast(frag, b), c, 0, 0, 0);
    }
};

constexpr int SK = 7;                    // taps per side
constexpr int SWROW = SK * 32 + 8;       // elements of an LDS weight row (padded: no bank conflicts)
constexpr int SW_BYTES = 64 * SWROW * 2;

// output channel of LDS weight row r (within a 32-row group, row 16h + 4kg + i
// holds channel 8kg + 4h + i), so that a lane's two fragments of a group hold
// 8 consecutive channels
__device__ __forceinline__ int sperm(int r) {
    const int l = r & 15;
    return (r & ~31) + (l >> 2) * 8 + ((r >> 4) & 1) * 4 + (l & 3);
}

// The 64 filters from channel co0 on as LDS rows (ky, kx8, ci4), zero where
// there is no tap, channel or filter, and their biases as fp32.  One 16-byte
// chunk (two taps of a row) per item, every load of a thread issued before
// its first LDS write.
template <typename T, int C, int NT>
__device__ __forceinline__ void stage_filters(const T* __restrict__ w, const T* __restrict__ bias, int co0, int C_out,
                                              T* s_w, float* s_bias) {
    constexpr int CH = 64 * SK * 4, U = (CH + NT - 1) / NT;
    const int tid = (int)threadIdx.x;
    Vec<T, 8> v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = tid + u * NT;
        const int r = i / (SK * 4), rem = i - r * (SK * 4), ky = rem >> 2, kq = rem & 3;
        const int co = co0 + sperm(r);
        v[u] = vzero<T, 8>();
        if (i < CH && co < C_out) {
            // (both taps' channels are one run: one load each, at any alignment)
            const T* p = w + (((size_t)co * SK + ky) * SK + 2 * kq) * C;
            T e[2 * C] = {};
            if (kq < 3) __builtin_memcpy(e, p, 2 * C * sizeof(T));
            else __builtin_memcpy(e, p, C * sizeof(T));
#pragma unroll
            for (int ci = 0; ci < C; ++ci) {
                v[u].e[ci] = e[ci];
                v[u].e[4 + ci] = e[C + ci];
            }
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = tid + u * NT;
        const int r = i / (SK * 4), rem = i - r * (SK * 4);
        if (i < CH) *reinterpret_cast<uint4*>(s_w + r * SWROW + rem * 8) = v[u].raw;
    }
    if (tid < 64) s_bias[tid] = (bias && co0 + tid < C_out) ? to_f32(bias[co0 + tid]) : 0.0f;
}

// This lane's weight operands (row l16 of each 16-row fragment).
template <typename T>
__device__ __forceinline__ void load_filters(const T* s_w, uint4 (&wf)[SK][4]) {
    const int lane = lane_id(), l16 = lane & 15, kg = lane >> 4;
#pragma unroll
    for (int ky = 0; ky < SK; ++ky)
#pragma unroll
        for (int ns = 0; ns < 4; ++ns)
            wf[ky][ns] = *reinterpret_cast<const uint4*>(s_w + (ns * 16 + l16) * SWROW + ky * 32 + kg * 8);
}

// One 16-byte pixel operand; the second pixel of lanes kg = 3 is the padding column.
__device__ __forceinline__ uint4 pix_frag(const unsigned char* p, bool last) {
    uint4 v = *reinterpret_cast<const uint4*>(p);
    v.z = last ? 0u : v.z;
    v.w = last ? 0u : v.w;
    return v;
}

// Two adjacent pixels of the image (C dwords from an even column).
template <int C>
struct Pair {
    uint32_t d[C];
};
template <int C>
__device__ __forceinline__ Pair<C> pair_load(const uint32_t* p) {
    Pair<C> r;
#pragma unroll
    for (int i = 0; i < C; ++i) r.d[i] = p[i];
    return r;
}
template <int C>
__device__ __forceinline__ Pair<C> pair_zero() {
    Pair<C> r;
#pragma unroll
    for (int i = 0; i < C; ++i) r.d[i] = 0u;
    return r;
}
// 16-bit element i of a pair (channel i % C of pixel i / C)
template <int C>
__device__ __forceinline__ uint32_t pair_at(const Pair<C>& p, int i) {
    return (i & 1) ? p.d[i >> 1] >> 16 : p.d[i >> 1] & 0xFFFFu;
}
// Pixel k of the pair as four 16-bit channels, missing ones zero.
template <int C>
__device__ __forceinline__ uint2 pair_pixel(const Pair<C>& p, int k) {
    uint32_t e[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) e[c] = c < C ? pair_at<C>(p, k * C + c) : 0u;
    return uint2{e[0] | (e[1] << 16), e[2] | (e[3] << 16)};
}
// The 2x2 average of the cell (top pair, bottom pair), as one pixel.
template <typename T, int C>
__device__ __forceinline__ uint2 pair_avg(const Pair<C>& t, const Pair<C>& b) {
    uint32_t e[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        e[c] = 0u;
        if (c < C) {
            const T r = avg4(__builtin_bit_cast(T, (uint16_t)pair_at<C>(t, c)),
                             __builtin_bit_cast(T, (uint16_t)pair_at<C>(t, C + c)),
                             __builtin_bit_cast(T, (uint16_t)pair_at<C>(b, c)),
                             __builtin_bit_cast(T, (uint16_t)pair_at<C>(b, C + c)));
            e[c] = __builtin_bit_cast(uint16_t, r);
        }
    }
    return uint2{e[0] | (e[1] << 16), e[2] | (e[3] << 16)};
}

// bias (and ReLU) of the two 16-channel fragments of a group, rounded: 8
// consecutive channels of one pixel
template <typename T>
__device__ __forceinline__ uint4 finish8(const floatx4& a, const floatx4& b, const float* bv, bool relu) {
    Vec<T, 8> o;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float f0 = a[i] + bv[i], f1 = b[i] + bv[4 + i];
        o.e[i] = from_f32<T>(relu ? fmaxf(f0, 0.0f) : f0);
        o.e[4 + i] = from_f32<T>(relu ? fmaxf(f1, 0.0f) : f1);
    }
    return o.raw;
}

// ---------------------------------------------------------------------------
// dense stem + max-pool
// ---------------------------------------------------------------------------
// Pooled tile: PH rows (16: eight waves, one workgroup a CU; 8: four waves, two)
// x 32 columns.
constexpr int SP_PW = 32, SP_IW = 4 * SP_PW + 8, SP_PITCH = SP_IW * 8;
constexpr int sp_wg(int ph) { return ph * 32; }
constexpr int sp_rows(int ph) { return 4 * ph + 7; }
constexpr int sp_lds(int ph) { return SW_BYTES + sp_rows(ph) * SP_PITCH + 64 * 4; }

// lane i of a row of 16 lanes takes lane i - 1 (lane 0: `edge`), lane i + 1
// (lane 15: undefined), or lane 15 in lane 0
__device__ __forceinline__ uint32_t row_prev(uint32_t edge, uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)edge, (int)v, 0x111, 0xF, 0xF, false);
}
__device__ __forceinline__ uint32_t row_next(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x101, 0xF, 0xF, true);
}
__device__ __forceinline__ uint32_t row_rot1(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x121, 0xF, 0xF, true);
}
// Values after a ReLU are not negative, so their fp16 / bf16 bit patterns
// order as unsigned integers.
__device__ __forceinline__ uint32_t max2(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}

// One workgroup: PH x 32 pooled pixels, 64 channels.  Wave (rg, ch) makes
// pooled rows 4 rg .. 4 rg + 3, columns 16 ch .. 16 ch + 15, from nine stem
// rows of 32 pixels one after the other: the vertical maxima are taken as the
// rows come, then the horizontal ones across lanes (an operand's 16 pixels are
// one row).  The stem column left of the wave's 32 is one more operand whose
// 16 "pixels" are that column in the wave's nine rows (28 MFMAs beside 504).
// Recomputed at tile borders: one row in nine.
//
// Bound by MFMA issue (K padded from 147 to 224) and, at one image, by the
// single round of workgroups, whose start (image tile and filters from
// memory) nothing overlaps.  1024x2048, 64 channels, tiles of
// 16 / 8 rows: 24.5 / 26.2 us for one image (256 / 512 workgroups, one round
// either way), 86.6 / 79.2 for four (several rounds: one workgroup's start beside
// the other's MFMAs); so 16 rows up to one tile a CU, 8 beyond.  The stem and
// the pool as two kernels take 51 and 199.
template <typename T, int C, int PH>
__global__ __launch_bounds__(sp_wg(PH), PH == 16 ? 1 : 2) void k_stem_pool(const T* __restrict__ x, int H, int W, const T* __restrict__ w,
                                                        const T* __restrict__ bias, int C_out, T* __restrict__ y,
                                                        int Ho, int Wo, int Hp, int Wp, int TY, int TX) {
    constexpr int SP_WG = sp_wg(PH), SP_PH = PH, SP_IH = sp_rows(PH);
    extern __shared__ __align__(16) unsigned char smem[];
    T* s_w = reinterpret_cast<T*>(smem);
    unsigned char* s_in = smem + SW_BYTES;
    float* s_bias = reinterpret_cast<float*>(s_in + SP_IH * SP_PITCH);
    const int tile = (int)blockIdx.x;
    const int n = tile / (TY * TX), tr = tile - n * TY * TX, ty = tr / TX, tx = tr - ty * TX;
    const int pi0 = ty * SP_PH, pj0 = tx * SP_PW, co0 = (int)blockIdx.y * 64;
    const int Y0 = 4 * pi0 - 5, X0 = 4 * pj0 - 5;  // image pixel of LDS pixel (0, 0)
    const int tid = (int)threadIdx.x;

    // Image pairs from even columns X0 - 1 on: LDS pixels 2 p - 1 and 2 p.
    // W is even, so a pair lies inside or outside the image as a whole.
    constexpr int NP = SP_IW / 2 + 1, ITEMS = SP_IH * NP, U = (ITEMS + SP_WG - 1) / SP_WG;
    const T* __restrict__ img = x + (size_t)n * H * W * C;
    {
        Pair<C> v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = tid + u * SP_WG, r = i / NP, p = i - r * NP;
            const int Y = Y0 + r, X = X0 - 1 + 2 * p;
            v[u] = pair_zero<C>();
            if (i < ITEMS && Y >= 0 && Y < H && X >= 0 && X < W)
                v[u] = pair_load<C>(reinterpret_cast<const uint32_t*>(img + ((size_t)Y * W + X) * C));
        }
        stage_filters<T, C, SP_WG>(w, bias, co0, C_out, s_w, s_bias);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = tid + u * SP_WG, r = i / NP, p = i - r * NP;
            if (i < ITEMS) {
                unsigned char* d = s_in + r * SP_PITCH + (2 * p - 1) * 8;
                if (p > 0) *reinterpret_cast<uint2*>(d) = pair_pixel<C>(v[u], 0);
                if (p < NP - 1) *reinterpret_cast<uint2*>(d + 8) = pair_pixel<C>(v[u], 1);
            }
        }
    }
    __syncthreads();

    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l16 = lane & 15, kg = lane >> 4;
    const int ch = wave & 1, lr0 = (wave >> 1) * 8;  // column half; first stem row (local: row 0 is 2 pi0 - 1)
    const int cr0 = 2 * pi0 - 1, oxc0 = 2 * pj0;
    const bool last = kg == 3;
    uint4 wf[SK][4];
    load_filters<T>(s_w, wf);

    // the stem column left of the wave's: lane l16 holds row lr0 + l16 (rows past the ninth repeat it)
    uint4 edge[2];
    {
        floatx4 acc[4];
#pragma unroll
        for (int ns = 0; ns < 4; ++ns) acc[ns] = floatx4{0.f, 0.f, 0.f, 0.f};
        const int r = min(l16, 8);
        const unsigned char* p = s_in + 2 * (lr0 + r) * SP_PITCH + 16 * (32 * ch + kg);
#pragma unroll
        for (int ky = 0; ky < SK; ++ky) {
            const uint4 bf = pix_frag(p + ky * SP_PITCH, last);
#pragma unroll
            for (int ns = 0; ns < 4; ++ns) acc[ns] = SMF<T>::mma(wf[ky][ns], bf, acc[ns]);
        }
        const int cy = cr0 + lr0 + r;
        const bool in = oxc0 + 32 * ch > 0 && oxc0 + 32 * ch - 1 < Wo && cy >= 0 && cy < Ho;
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
            edge[jj] = finish8<T>(acc[2 * jj], acc[2 * jj + 1], s_bias + jj * 32 + kg * 8, true);
            if (!in) edge[jj] = uint4{0u, 0u, 0u, 0u};
        }
    }

    // its maxima over three rows, in the lane of the first
    uint4 edge3[2];
#pragma unroll
    for (int jj = 0; jj < 2; ++jj) {
        uint32_t e[4] = {edge[jj].x, edge[jj].y, edge[jj].z, edge[jj].w};
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const uint32_t n1 = row_next(e[d]);
            e[d] = max2(max2(e[d], n1), row_next(n1));
        }
        edge3[jj] = uint4{e[0], e[1], e[2], e[3]};
    }

    // stem row lr0 + r after bias and ReLU, rounded; zero outside the map
    auto stem_row = [&](int r, uint4 (&h)[2][2]) {
        const int cy = cr0 + lr0 + r;
        if (cy < 0 || cy >= Ho) {  // uniform
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int jj = 0; jj < 2; ++jj) h[t][jj] = uint4{0u, 0u, 0u, 0u};
            return;
        }
        floatx4 acc[2][4];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int ns = 0; ns < 4; ++ns) acc[t][ns] = floatx4{0.f, 0.f, 0.f, 0.f};
        const unsigned char* p = s_in + 2 * (lr0 + r) * SP_PITCH + 16 * (32 * ch + l16 + 1 + kg);
#pragma unroll
        for (int ky = 0; ky < SK; ++ky) {
            uint4 bf[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) bf[t] = pix_frag(p + ky * SP_PITCH + 256 * t, last);
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int ns = 0; ns < 4; ++ns) acc[t][ns] = SMF<T>::mma(wf[ky][ns], bf[t], acc[t][ns]);
        }
#pragma unroll
        for (int jj = 0; jj < 2; ++jj)
#pragma unroll
            for (int t = 0; t < 2; ++t)
                h[t][jj] = finish8<T>(acc[t][2 * jj], acc[t][2 * jj + 1], s_bias + jj * 32 + kg * 8, true);
        if (oxc0 + 64 > Wo) {  // (uniform) the tile passes the map's right edge
#pragma unroll
            for (int t = 0; t < 2; ++t)
                if (oxc0 + 32 * ch + 16 * t + l16 >= Wo) {
#pragma unroll
                    for (int jj = 0; jj < 2; ++jj) h[t][jj] = uint4{0u, 0u, 0u, 0u};
                }
        }
    };
    auto vmax = [](uint4 a, uint4 b) { return uint4{max2(a.x, b.x), max2(a.y, b.y), max2(a.z, b.z), max2(a.w, b.w)}; };

    // three rows to one, then three columns to one (even lanes: pooled column l16 / 2 of fragment t)
    uint4 cur[2][2];
    stem_row(0, cur);
    for (int q = 0; q < 4; ++q) {
        const int pi = pi0 + (lr0 >> 1) + q;
        if (pi >= Hp) return;  // uniform; no barrier follows
        uint4 h[2][2];
        stem_row(2 * q + 1, h);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) cur[t][jj] = vmax(cur[t][jj], h[t][jj]);
        stem_row(2 * q + 2, h);
        T* yrow = y + ((size_t)n * Hp + pi) * Wp * C_out;
        const int src = ((lane & 48) + 2 * q) * 4;
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
            const uint32_t ed[4] = {edge3[jj].x, edge3[jj].y, edge3[jj].z, edge3[jj].w};
            const uint4 c0 = vmax(cur[0][jj], h[0][jj]), c1 = vmax(cur[1][jj], h[1][jj]);
            const uint32_t v0[4] = {c0.x, c0.y, c0.z, c0.w}, v1[4] = {c1.x, c1.y, c1.z, c1.w};
            uint32_t m[2][4];
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const uint32_t e0 = (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)ed[d]);
                m[0][d] = max2(max2(row_prev(e0, v0[d]), v0[d]), row_next(v0[d]));
                m[1][d] = max2(max2(row_prev(row_rot1(v0[d]), v1[d]), v1[d]), row_next(v1[d]));
            }
            const int co = co0 + jj * 32 + kg * 8;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int pj = pj0 + 16 * ch + 8 * t + (l16 >> 1);
                if ((l16 & 1) == 0 && pj < Wp && co < C_out)
                    *reinterpret_cast<uint4*>(yrow + (size_t)pj * C_out + co) = uint4{m[t][0], m[t][1], m[t][2], m[t][3]};
                cur[t][jj] = h[t][jj];
            }
        }
    }
}

// ---------------------------------------------------------------------------
// blockwise stem
// ---------------------------------------------------------------------------
constexpr int SB_WG = 256;               // four waves; two workgroups fit a CU
constexpr int SB_TH = 16, SB_TW = 32;    // output tile of one block: four rows per wave
constexpr int SB_IH = 2 * (SB_TH - 1) + SK, SB_IW = 2 * (SB_TW - 1) + 8, SB_PITCH = SB_IW * 8;
constexpr int SB_LDS = SW_BYTES + SB_IH * SB_PITCH + 64 * 4;

// Neighbour direction of coordinate u in a block of extent e.
__device__ __forceinline__ int side(int u, int e) { return u < 0 ? 0 : (u >= e ? 2 : 1); }

// One workgroup: a 16 x 32 tile of one block's output, 64 channels.  The
// padded input tile comes from the image in 2x2 cells: a cell is four pixels,
// or (in a low block, on either side of a block border) its average.  Bound
// by the latency of that load and by the output's stores.  1024x2048, 8x16
// blocks, half low: 27 us; split, pad and the direct convolution take 3780 us.
template <typename T, int C>
__global__ __launch_bounds__(SB_WG, 2) void k_stem_blocks(Geo g, const uint8_t* __restrict__ mask,
                                                          const T* __restrict__ x, const T* __restrict__ w,
                                                          const T* __restrict__ bias, int C_out, int relu,
                                                          T* __restrict__ ho, T* __restrict__ lo, int hi_cap,
                                                          int lo_cap, int th, int tl) {
    extern __shared__ __align__(16) unsigned char smem[];
    T* s_w = reinterpret_cast<T*>(smem);
    unsigned char* s_in = smem + SW_BYTES;
    float* s_bias = reinterpret_cast<float*>(s_in + SB_IH * SB_PITCH);
    const int bid = (int)blockIdx.x, tid = (int)threadIdx.x, co0 = (int)blockIdx.y * 64;
    const bool high = bid < hi_cap * th;
    const int q = high ? bid : bid - hi_cap * th, per = high ? th : tl;
    const int slot = q / per, tile = q - slot * per;
    WaveMask wm;
    wm.init(mask, (int)g.B);
    const int k = wm.find_nth(slot, high);
    if (k < 0) return;  // uniform over the workgroup
    const int img_blocks = g.GH * g.GW;
    const int n = k / img_blocks, rem = k - n * img_blocks, gy = rem / g.GW, gx = rem - gy * g.GW;
    const Neigh nb = wave_neighbourhood<true>(wm, g.GH, g.GW, n, gy, gx);
    uint32_t have = 0;  // bit d: neighbour d exists and has a place in its stack
#pragma unroll
    for (int d = 0; d < 9; ++d)
        have |= (uint32_t)(((nb.valid >> d) & 1u) && nb.slot[d] < (((nb.high >> d) & 1u) ? hi_cap : lo_cap)) << d;

    const int bs = g.bs, e = high ? bs : bs >> 1, eo = e >> 1;
    const int tx_n = (eo + SB_TW - 1) / SB_TW;
    const int oy0 = (tile / tx_n) * SB_TH, ox0 = (tile - (tile / tx_n) * tx_n) * SB_TW;
    const T* __restrict__ img = x + (size_t)n * g.H * g.W * C;
    const uint32_t rowd = (uint32_t)(g.W * C) >> 1;  // dwords of an image row (W is even)
    stage_filters<T, C, SB_WG>(w, bias, co0, C_out, s_w, s_bias);
    // LDS pixel (0, 0) is block pixel (2 oy0 - 3, 2 ox0 - 3); outputs of the
    // block read up to block pixel e + 1
    if (high) {
        constexpr int CR = (SB_IH + 1) / 2, CC = SB_IW / 2 + 1, ITEMS = CR * CC, U = (ITEMS + SB_WG - 1) / SB_WG;
        Pair<C> t[U], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = tid + u * SB_WG, cy = i / CC, cx = i - cy * CC;
            const int uu = 2 * oy0 - 4 + 2 * cy, vv = 2 * ox0 - 4 + 2 * cx;  // the cell's top-left block pixel
            t[u] = b[u] = pair_zero<C>();
            if (i < ITEMS && uu < e + 2 && vv < e + 2 && ((have >> (side(uu, e) * 3 + side(vv, e))) & 1u)) {
                const uint32_t* p = reinterpret_cast<const uint32_t*>(
                    img + ((size_t)(gy * bs + uu) * g.W + gx * bs + vv) * C);
                t[u] = pair_load<C>(p);
                b[u] = pair_load<C>(p + rowd);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = tid + u * SB_WG, cy = i / CC, cx = i - cy * CC;
            if (i >= ITEMS) continue;
            const int uu = 2 * oy0 - 4 + 2 * cy, vv = 2 * ox0 - 4 + 2 * cx;
            uint2 px[4] = {pair_pixel<C>(t[u], 0), pair_pixel<C>(t[u], 1), pair_pixel<C>(b[u], 0),
                           pair_pixel<C>(b[u], 1)};
            if (!((nb.high >> (side(uu, e) * 3 + side(vv, e))) & 1u))  // a low neighbour, nearest-upsampled
                px[0] = px[1] = px[2] = px[3] = pair_avg<T, C>(t[u], b[u]);
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const int py = 2 * cy - 1 + (a >> 1), pv = 2 * cx - 1 + (a & 1);
                if (py >= 0 && py < SB_IH && pv >= 0 && pv < SB_IW)
                    *reinterpret_cast<uint2*>(s_in + py * SB_PITCH + pv * 8) = px[a];
            }
        }
    } else {
        // a low block sees the cell averages whatever the neighbour's class
        constexpr int ITEMS = SB_IH * SB_IW, U = 4;
        for (int base = tid; base < ITEMS; base += SB_WG * U) {
            Pair<C> t[U], b[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = base + u * SB_WG, py = i / SB_IW, pv = i - py * SB_IW;
                const int uu = 2 * oy0 - 3 + py, vv = 2 * ox0 - 3 + pv;
                t[u] = b[u] = pair_zero<C>();
                if (i < ITEMS && uu < e + 2 && vv < e + 2 && ((have >> (side(uu, e) * 3 + side(vv, e))) & 1u)) {
                    const uint32_t* p = reinterpret_cast<const uint32_t*>(
                        img + ((size_t)(gy * bs + 2 * uu) * g.W + gx * bs + 2 * vv) * C);
                    t[u] = pair_load<C>(p);
                    b[u] = pair_load<C>(p + rowd);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = base + u * SB_WG, py = i / SB_IW, pv = i - py * SB_IW;
                if (i < ITEMS) *reinterpret_cast<uint2*>(s_in + py * SB_PITCH + pv * 8) = pair_avg<T, C>(t[u], b[u]);
            }
        }
    }
    __syncthreads();

    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l16 = lane & 15, kg = lane >> 4;
    const bool last = kg == 3;
    uint4 wf[SK][4];
    load_filters<T>(s_w, wf);
    T* out = (high ? ho : lo) + (size_t)slot * eo * eo * C_out;
    for (int rr = 0; rr < SB_TH / 4; ++rr) {
        const int ol = wave * (SB_TH / 4) + rr, oy = oy0 + ol;
        if (oy >= eo) return;  // uniform over the wave; no barrier follows
        const unsigned char* p = s_in + 2 * ol * SB_PITCH + 16 * (l16 + kg);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if (ox0 + 16 * t >= eo) continue;  // uniform
            floatx4 acc[4];
#pragma unroll
            for (int ns = 0; ns < 4; ++ns) acc[ns] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ky = 0; ky < SK; ++ky) {
                const uint4 bf = pix_frag(p + ky * SB_PITCH + 256 * t, last);
#pragma unroll
                for (int ns = 0; ns < 4; ++ns) acc[ns] = SMF<T>::mma(wf[ky][ns], bf, acc[ns]);
            }
            const int ox = ox0 + 16 * t + l16;
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) {
                const int co = co0 + jj * 32 + kg * 8;
                if (ox < eo && co < C_out)
                    *reinterpret_cast<uint4*>(out + ((size_t)oy * eo + ox) * C_out + co) =
                        finish8<T>(acc[2 * jj], acc[2 * jj + 1], s_bias + jj * 32 + kg * 8, relu != 0);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// max-pool on packed stacks
// ---------------------------------------------------------------------------

// One workgroup: 256 items of one block, an item eight channels of PB_ROWS
// output pixels below one another, whose windows share rows: 27 loads for four
// outputs instead of 36, three rows (nine loads) in flight.  A pixel of the
// halo (the row above or the column left of the block) comes through
// BlockPad's source.  Bound by the input's read from HBM or the Infinity
// Cache.  The stem's output at 1024x2048, half low: 21 us (38 with a
// thread for every output); pad and max-pool as two kernels take 87 us.
constexpr int PB_ROWS = 4;
template <typename T>
__global__ __launch_bounds__(WG) void k_pool_blocks(Geo g, const uint8_t* __restrict__ mask, const T* __restrict__ hi,
                                                    const T* __restrict__ lo, T* __restrict__ ho, T* __restrict__ lo_o,
                                                    int hi_cap, int lo_cap, int th, int tl) {
    const int bid = (int)blockIdx.x;
    const bool high = bid < hi_cap * th;
    const int q = high ? bid : bid - hi_cap * th, per = high ? th : tl;
    const int slot = q / per, piece = q - slot * per;
    WaveMask wm;
    wm.init(mask, (int)g.B);
    const int k = wm.find_nth(slot, high);
    if (k < 0) return;
    const int img_blocks = g.GH * g.GW;
    const int n = k / img_blocks, rem = k - n * img_blocks, gy = rem / g.GW, gx = rem - gy * g.GW;
    const Neigh nb = wave_neighbourhood<true>(wm, g.GH, g.GW, n, gy, gx);
    const int e = high ? g.bs : g.bs >> 1, eo = e >> 1, cv = g.C / 8;
    const int it = piece * WG + (int)threadIdx.x;
    const int strips = (eo + PB_ROWS - 1) / PB_ROWS;
    if (it >= strips * eo * cv) return;
    const int pix = it / cv, c = (it - pix * cv) * 8, strip = pix / eo, j = pix - strip * eo;
    const int i0 = strip * PB_ROWS, rows = min(PB_ROWS, eo - i0);
    const T* own = (high ? hi : lo) + ((size_t)slot * e * e + 2 * j) * g.C + c;
    T* out = (high ? ho : lo_o) + (((size_t)slot * eo + i0) * eo + j) * g.C + c;

    // window row u: its three pixels, requested, then their maximum
    struct Row {
        Vec<T, 8> v[3];
    };
    auto halo = [&](int u, int v) {
        const Src<T> s = packed_src<T, NHWC>(hi, lo, g.C, g.bs, nb, hi_cap, lo_cap, u, v, c);
        if (!s.p) return vzero<T, 8>();
        const Vec<T, 8> a = vload<T, 8>(s.p);
        if (!s.avg) return a;
        return vavg4<T, 8>(a, vload<T, 8>(s.p + s.d1), vload<T, 8>(s.p + s.d2), vload<T, 8>(s.p + s.d2 + s.d1));
    };
    auto load = [&](int u, Row& r) {
        if (u < 0) {
            for (int s = 0; s < 3; ++s) {
                const Vec<T, 8> x = halo(u, 2 * j - 1 + s);
                if (s == 0) r.v[0] = x;
                else if (s == 1) r.v[1] = x;
                else r.v[2] = x;
            }
            return;
        }
        const T* p = own + (size_t)u * e * g.C;
        r.v[1] = vload<T, 8>(p);
        r.v[2] = vload<T, 8>(p + g.C);
        if (j > 0) r.v[0] = vload<T, 8>(p - g.C);
        else r.v[0] = halo(u, -1);
    };
    auto row_max = [](const Row& r, float (&m)[8]) {
#pragma unroll
        for (int b = 0; b < 8; ++b)
            m[b] = fmaxf(fmaxf(to_f32(r.v[0].e[b]), to_f32(r.v[1].e[b])), to_f32(r.v[2].e[b]));
    };
    float prev[8];
    Row a, b;
    {
        Row r;
        load(2 * i0 - 1, r);
        load(2 * i0, a);
        load(2 * i0 + 1, b);
        row_max(r, prev);
    }
    for (int i = 0; i < rows; ++i) {
        Row a2, b2;
        if (i + 1 < rows) {  // the next output's rows, while this one is finished
            load(2 * (i0 + i) + 2, a2);
            load(2 * (i0 + i) + 3, b2);
        }
        float m[8];
        row_max(a, m);
#pragma unroll
        for (int x = 0; x < 8; ++x) m[x] = fmaxf(prev[x], m[x]);
        row_max(b, prev);
        Vec<T, 8> o;
#pragma unroll
        for (int x = 0; x < 8; ++x)  // (a window of nothing but NaN: -inf, as the direct kernel starts from)
            o.e[x] = from_f32<T>(fmaxf(fmaxf(m[x], prev[x]), -INFINITY));
        vstore<T, 8>(out + (size_t)i * eo * g.C, o);
        a = a2;
        b = b2;
    }
}

inline bool al(const void* p, uintptr_t n) { return (reinterpret_cast<uintptr_t>(p) & (n - 1)) == 0; }

template <typename T, int C, int PH>
hipError_t stem_pool_ph(const void* x, int N, int H, int W, const void* w, const void* bias, int C_out, void* y,
                        hipStream_t st) {
    const int Ho = (H - 1) / 2 + 1, Wo = (W - 1) / 2 + 1, Hp = (Ho - 1) / 2 + 1, Wp = (Wo - 1) / 2 + 1;
    const int TY = (Hp + PH - 1) / PH, TX = (Wp + SP_PW - 1) / SP_PW;
    hipError_t e = ensure_dyn_lds((const void*)k_stem_pool<T, C, PH>, sp_lds(PH));
    if (e != hipSuccess) return e;
    const dim3 grid((unsigned)((long long)N * TY * TX), (unsigned)((C_out + 63) / 64));
    hipLaunchKernelGGL((k_stem_pool<T, C, PH>), grid, dim3(sp_wg(PH)), sp_lds(PH), st, (const T*)x, H, W, (const T*)w,
                       (const T*)bias, C_out, (T*)y, Ho, Wo, Hp, Wp, TY, TX);
    return hipGetLastError();
}

template <typename T, int C>
hipError_t stem_pool_c(const void* x, int N, int H, int W, const void* w, const void* bias, int C_out, void* y,
                       hipStream_t st) {
    const long long Hp = (H - 1) / 2 / 2 + 1, Wp = (W - 1) / 2 / 2 + 1;
    const long long tiles16 = N * ((Hp + 15) / 16) * ((Wp + SP_PW - 1) / SP_PW) * ((C_out + 63) / 64);
    if (tiles16 <= device_cus()) return stem_pool_ph<T, C, 16>(x, N, H, W, w, bias, C_out, y, st);
    return stem_pool_ph<T, C, 8>(x, N, H, W, w, bias, C_out, y, st);
}

template <typename T>
hipError_t stem_pool_t(const void* x, int N, int C_in, int H, int W, const void* w, const void* bias, int C_out,
                       void* y, hipStream_t st) {
    switch (C_in) {
    case 1: return stem_pool_c<T, 1>(x, N, H, W, w, bias, C_out, y, st);
    case 2: return stem_pool_c<T, 2>(x, N, H, W, w, bias, C_out, y, st);
    case 3: return stem_pool_c<T, 3>(x, N, H, W, w, bias, C_out, y, st);
    default: return stem_pool_c<T, 4>(x, N, H, W, w, bias, C_out, y, st);
    }
}

template <typename T, int C>
hipError_t stem_blocks_c(const Geo& g, const uint8_t* mask, const void* x, const void* w, const void* bias, int C_out,
                         int relu, void* ho, int hi_cap, void* lo, int lo_cap, hipStream_t st) {
    auto tiles = [](int eo) { return ((eo + SB_TH - 1) / SB_TH) * ((eo + SB_TW - 1) / SB_TW); };
    const int th = tiles(g.bs / 2), tl = tiles(g.bs / 4);
    const long long blocks = (long long)hi_cap * th + (long long)lo_cap * tl;
    if (blocks == 0) return hipSuccess;
    hipError_t e = ensure_dyn_lds((const void*)k_stem_blocks<T, C>, SB_LDS);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_stem_blocks<T, C>), dim3((unsigned)blocks, (unsigned)((C_out + 63) / 64)), dim3(SB_WG), SB_LDS,
                       st, g, mask, (const T*)x, (const T*)w, (const T*)bias, C_out, relu, (T*)ho, (T*)lo, hi_cap,
                       lo_cap, th, tl);
    return hipGetLastError();
}

template <typename T>
hipError_t stem_blocks_t(const Geo& g, const uint8_t* mask, const void* x, const void* w, const void* bias, int C_out,
                         int relu, void* ho, int hi_cap, void* lo, int lo_cap, hipStream_t st) {
    switch (g.C) {
    case 1: return stem_blocks_c<T, 1>(g, mask, x, w, bias, C_out, relu, ho, hi_cap, lo, lo_cap, st);
    case 2: return stem_blocks_c<T, 2>(g, mask, x, w, bias, C_out, relu, ho, hi_cap, lo, lo_cap, st);
    case 3: return stem_blocks_c<T, 3>(g, mask, x, w, bias, C_out, relu, ho, hi_cap, lo, lo_cap, st);
    default: return stem_blocks_c<T, 4>(g, mask, x, w, bias, C_out, relu, ho, hi_cap, lo, lo_cap, st);
    }
}

template <typename T>
hipError_t pool_blocks_t(const Geo& g, const uint8_t* mask, const void* hi, const void* lo, void* ho, void* lo_o,
                         int hi_cap, int lo_cap, hipStream_t st) {
    auto pieces = [&](int eo) {
        return (int)(((long long)((eo + PB_ROWS - 1) / PB_ROWS) * eo * (g.C / 8) + WG - 1) / WG);
    };
    const int th = pieces(g.bs / 2), tl = pieces(g.bs / 4);
    const long long blocks = (long long)hi_cap * th + (long long)lo_cap * tl;
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL((k_pool_blocks<T>), dim3((unsigned)blocks), dim3(WG), 0, st, g, mask, (const T*)hi, (const T*)lo,
                       (T*)ho, (T*)lo_o, hi_cap, lo_cap, th, tl);
    return hipGetLastError();
}

}  // namespace

bool stem_fits(int dtype, int layout, int C_in, int W, int C_out, const void* x, const void* y) {
    return layout == NHWC && (dtype == 1 || dtype == 2) && C_in <= 4 && W % 2 == 0 && C_out % 8 == 0 && al(x, 4) &&
           al(y, 16);
}

hipError_t launch_stem_pool(int dtype, const void* x, int N, int C_in, int H, int W, const void* w, const void* bias,
                            int C_out, void* y, hipStream_t st) {
    if (dtype == 1) return stem_pool_t<f16>(x, N, C_in, H, W, w, bias, C_out, y, st);
    return stem_pool_t<bf16>(x, N, C_in, H, W, w, bias, C_out, y, st);
}

hipError_t launch_stem_blocks(int dtype, const Geo& g, const uint8_t* mask, const void* x, const void* w,
                              const void* bias, int C_out, int relu, void* ho, int hi_cap, void* lo, int lo_cap,
                              hipStream_t st) {
    if (dtype == 1) return stem_blocks_t<f16>(g, mask, x, w, bias, C_out, relu, ho, hi_cap, lo, lo_cap, st);
    return stem_blocks_t<bf16>(g, mask, x, w, bias, C_out, relu, ho, hi_cap, lo, lo_cap, st);
}

hipError_t launch_pool_blocks(int dtype, const Geo& g, const uint8_t* mask, const void* hi, const void* lo, void* ho,
                              void* lo_o, int hi_cap, int lo_cap, hipStream_t st) {
    if (dtype == 1) return pool_blocks_t<f16>(g, mask, hi, lo, ho, lo_o, hi_cap, lo_cap, st);
    return pool_blocks_t<bf16>(g, mask, hi, lo, ho, lo_o, hi_cap, lo_cap, st);
}

}  // namespace sb

// 3x3 block convolution as an MFMA implicit GEMM for gfx950: the general
// kernel, for every type, layout, channel count and block size.
//
// GEMM view per block: output pixels x output channels, K = 9 taps x C_in.
// One workgroup (4 waves) computes a tile of whole rows of one block (about
// 64, 128 or 256 output pixels, chosen per call) x up to 64 output channels.
// K is walked in chunks of 64 bytes of input channels (32 fp16/bf16 or 16
// fp32): the padded input rows of the tile and the chunk's weights are staged
// in LDS with an XOR swizzle of the 16-byte sub-chunks, and every tap reads
// its pixel fragments at a constant offset from the same LDS tile.
//
// MFMA: v_mfma_f32_16x16x32_{f16,bf16} (8 K values per lane) or
// v_mfma_f32_16x16x4_f32, with the weights as the A operand (16 output
// channels) and the pixels as the B operand (16 pixels).  A lane reads 16
// bytes of a row either way: for fp32 its four channels go to four MFMAs (K
// index kg of MFMA i is channel 4 kg + i of the chunk, in both operands).
// A lane's result is 4 consecutive output channels of one pixel, which the
// epilogue stores directly without a trip through LDS.  Each wave owns up to
// four 16-pixel sub-tiles and all 16-channel sub-tiles (64 fp32 accumulators
// per lane); channel sub-tiles past C_out are not computed.
//
// Start-up: chunk 0's weights are requested first (they do not depend on the
// mask), then the block plan gives every pixel of the padded tile a source
// descriptor in LDS (an address, and whether it is a copy or a 2x2 average),
// which every chunk only adds its channel offset to.  While the MFMAs of
// chunk kc run, the weights and the first inputs of chunk kc + 1 are already
// being loaded into registers.  LDS (58.6 KiB for 32-pixel blocks at 256
// pixels a tile) leaves room for two workgroups per CU, so one workgroup's
// loads overlap the other's MFMAs.
//
// Staging follows the memory: channels-last tensors of whole 16-byte vectors
// move those (a thread takes one sub-chunk of one pixel); NCHW tensors are
// read along x (neighbouring lanes take neighbouring pixels of one channel
// plane, a 2x2 cell is two loads of two pixels, the weights of a filter are one
// run of words), other channels-last ones element by element.
//
// Bounds: fp32 by MFMA issue and by the staging beside it (the 256x512,
// 64-channel layer, half low, NCHW: 178 -> 101 us, 39 us of MFMA issue; a 64x64
// layer of 16 channels 31 -> 8 us), small and ragged 16-bit calls by the
// latency of the chain mask -> descriptors -> inputs -> MFMAs (two 96x180 maps,
// 48 -> 72 channels, 12-pixel blocks: 21.5 -> 18.0 us; one 128x256 map of 96
// channels, 16-pixel blocks: 36 -> 22 us).  All-low maps are a few small tiles
// of averages, one wave a SIMD: 96 channels 22.6 -> 19.5 us.  The 16-bit NCHW
// kernels of four sub-tiles a wave are at the 256 registers and spill one or two
// of them (8 to 12 bytes a lane).
//
// The tile loader is where the block modules live:
//   SRC_PADDED : reads padded stacks (plain conv of segblocks_conv3x3)
//   SRC_PACKED : BlockPad fused (neighbour lookup into the packed stacks)
//   SRC_DENSE  : BlockSample + BlockPad fused (reads the dense input map)
// and the store is either a packed stack or BlockCombine into a dense map.
//
// Weights: channels-last calls take OHWI memory ([C_out][3][3][C_in], the
// memory of a channels_last [C_out, C_in, 3, 3] tensor), NCHW calls OIHW.
#include <algorithm>
#include <type_traits>

#include "sb_common.h"
#include "sb_kernels.h"
#include "sb_pixel.h"

namespace sb {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// One 16-byte operand of every lane covers 32 (fp16 / bf16) or 16 (fp32)
// channels: STEPS MFMAs, of which step i takes.  The caller runs a step over
// all of its accumulators before the next: an fp32 MFMA that follows another
// on the same accumulator waits for it (measured: the MFMA phase of a lone
// workgroup took 2.4 times its issue time with the four steps of an
// accumulator back to back).
template <typename T> struct MF;
template <> struct MF<f16> {
    static constexpr int STEPS = 1;
    static __device__ __forceinline__ floatx4 mma(uint4 a, uint4 b, int, floatx4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(halfx8, a), __builtin_bit_cast(halfx8, b), c,
                                                      0, 0, 0);
    }
};
template <> struct MF<bf16> {
    static constexpr int STEPS = 1;
    static __device__ __forceinline__ floatx4 mma(uint4 a, uint4 b, int, floatx4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                       0, 0, 0);
    }
};
template <> struct MF<float> {
    static constexpr int STEPS = 4;
    static __device__ __forceinline__ floatx4 mma(uint4 a, uint4 b, int i, floatx4 c) {
        const floatx4 fa = __builtin_bit_cast(floatx4, a), fb = __builtin_bit_cast(floatx4, b);
        return __builtin_amdgcn_mfma_f32_16x16x4f32(fa[i], fb[i], c, 0, 0, 0);
    }
};

constexpr int NT = 64;     // most output channels per workgroup
constexpr int ROWB = 64;   // LDS bytes per tile pixel / weight row (one K chunk)
constexpr int UI = 4;      // 16-byte input vectors per thread and batch
constexpr int UA = 2;      // of them, averages in flight together
constexpr int UW = 9 * NT * (ROWB / 16) / WG;  // weight vectors per thread per chunk
static_assert(UW * WG == 9 * NT * (ROWB / 16), "weight staging covers the chunk exactly");

// byte offset of 16-byte sub-chunk q of LDS row `row`: sub-chunks are XOR-
// swizzled with bits 1..2 of the row so that 8 consecutive rows read at the
// same sub-chunk hit 8 distinct 16-byte bank groups.
__device__ __forceinline__ int swz(int row, int q) { return row * ROWB + ((q ^ ((row >> 1) & 3)) << 4); }

// Geometry of one workgroup's tile (uniform across the workgroup).
struct Tile {
    int n, gy, gx, slot, high, e, pe, r0, rows, M, in_px;
};

// Source of the tile pixel p (padded-tile coordinates, row-major over
// (rows + 2) x pe), channel 0.
template <typename T, int L, int SRC>
__device__ __forceinline__ Src<T> tile_src(const Geo& g, const ConvArgs& a, const Neigh& nb, const Tile& t, int p) {
    const int pu = p / t.pe, pv = p - pu * t.pe;
    const int u = t.r0 + pu;
    if constexpr (SRC == SRC_PADDED) {
        return src_copy<T>(stack_at<T, L>((const T*)(t.high ? a.in_hi : a.in_lo), t.slot, a.C_in, t.pe, u, pv, 0),
                           !t.high);
    } else if constexpr (SRC == SRC_PACKED) {
        return packed_src<T, L>((const T*)a.in_hi, (const T*)a.in_lo, a.C_in, g.bs, nb, a.hi_cap, a.lo_cap, u - 1,
                                pv - 1, 0, pad_mode(a.flags));
    } else {
        return dense_src<T, L>((const T*)a.in_hi, t.n, a.C_in, g.H, g.W, g.bs, t.gy, t.gx, nb, u - 1, pv - 1, 0,
                               pad_mode(a.flags));
    }
}

// Descriptor of a tile pixel: the byte offset of its source's channel 0 from the
// high stack's (or the map's) base, also where it lies in the low stack, and
// what it is; 0: a zero.  (Offsets from a kernel argument and not addresses,
// nor a choice between two bases: the compiler loses the address space of
// either, loads through the flat path, and the LDS reads of the MFMA loop
// then wait for those loads.)
constexpr unsigned long long SD_AVG = 1ull << 63, SD_LOW = 1ull << 62, SD_SOME = 1ull << 61;
constexpr unsigned long long SD_OFF = SD_SOME - 1;

// What every descriptor of a workgroup shares.
template <typename T>
struct Strides {
    const T* hi;            // the high stack or the map
    long long ch_hi, ch_d;  // elements from a channel to the next (high stack or map); low stack: ch_hi + ch_d
    long long d1, d2;       // to the right and to the lower pixel of an averaged cell
    __device__ __forceinline__ long long ch(unsigned long long d) const { return ch_hi + ((d & SD_LOW) ? ch_d : 0); }
    __device__ __forceinline__ const T* at(unsigned long long d) const {
        return reinterpret_cast<const T*>(reinterpret_cast<const char*>(hi) + ((long long)(d << 3) >> 3));
    }
};
template <typename T, int L, int SRC>
__device__ __forceinline__ Strides<T> make_strides(const Geo& g, const ConvArgs& a, const Tile& t) {
    const long long lb = g.bs >> 1, row = SRC == SRC_DENSE ? g.W : g.bs, px = L == NHWC ? a.C_in : 1;
    Strides<T> s;
    s.hi = (const T*)a.in_hi;
    s.ch_hi = L == NHWC ? 1 : (SRC == SRC_DENSE ? (long long)g.H * g.W
                                                : SRC == SRC_PADDED ? (long long)t.pe * t.pe : (long long)g.bs * g.bs);
    s.ch_d = L == NHWC || SRC == SRC_PADDED ? 0 : lb * lb - s.ch_hi;
    s.d1 = px;
    s.d2 = px * row;
    return s;
}

// The thread index, opaque to the optimiser at each use: the addresses made
// from it are recomputed for every chunk instead of all being kept in
// registers across the MFMAs.
__device__ __forceinline__ int tid_here() {
    int t = (int)threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// ---- channels-last staging in 16-byte vectors: item it is sub-chunk it % 4 of
// pixel it / 4.  issue() requests every item's (first) vector, rest() the
// three others of the averages, finish() writes LDS.
template <typename T>
struct VecIn {
    static constexpr int KC = ROWB / (int)sizeof(T), VQ = 16 / (int)sizeof(T);
    Vec<T, VQ> v[UI];
    bool avg[UI];  // (kept: only an average's descriptor is read again)

    static __device__ __forceinline__ unsigned long long desc(const unsigned long long* s_desc, int C_in, int in_px,
                                                              int it, int kc) {
        return it < in_px * 4 && kc * KC + (it & 3) * VQ < C_in ? s_desc[it >> 2] : 0ull;
    }
    __device__ __forceinline__ void issue(const unsigned long long* s_desc, const Strides<T>& st, int C_in, int in_px,
                                          int base, int kc) {
        const int tid = tid_here();
#pragma unroll
        for (int u = 0; u < UI; ++u) {
            const int it = base + u * WG + tid;
            const unsigned long long d = desc(s_desc, C_in, in_px, it, kc);
            avg[u] = (d & SD_AVG) != 0;
            v[u] = vzero<T, VQ>();
            if (d) v[u] = vload<T, VQ>(st.at(d) + kc * KC + (it & 3) * VQ);
        }
    }
    // the other three vectors of the averages among items u0 .. u0 + UA - 1, and those items to LDS
    struct Rest {
        Vec<T, VQ> r[UA][3];
    };
    __device__ __forceinline__ void rest(Rest& q, int u0, const unsigned long long* s_desc, const Strides<T>& st,
                                         int base, int kc) const {
        const int tid = tid_here();
#pragma unroll
        for (int u = 0; u < UA; ++u) {
            const int it = base + (u0 + u) * WG + tid;
            if (avg[u0 + u]) {
                const T* p = st.at(s_desc[it >> 2]) + kc * KC + (it & 3) * VQ;
                q.r[u][0] = vload<T, VQ>(p + st.d1);
                q.r[u][1] = vload<T, VQ>(p + st.d2);
                q.r[u][2] = vload<T, VQ>(p + st.d2 + st.d1);
            }
        }
    }
    __device__ __forceinline__ void finish(const Rest& q, int u0, int in_px, int base, unsigned char* s_in) {
        const int tid = tid_here();
#pragma unroll
        for (int u = 0; u < UA; ++u) {
            const int it = base + (u0 + u) * WG + tid;
            if (avg[u0 + u]) v[u0 + u] = vavg4<T, VQ>(v[u0 + u], q.r[u][0], q.r[u][1], q.r[u][2]);
            if (it < in_px * 4) *reinterpret_cast<uint4*>(s_in + swz(it >> 2, it & 3)) = v[u0 + u].raw;
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    __device__ __forceinline__ void commit(const unsigned long long* s_desc, const Strides<T>& st, int in_px, int base,
                                           int kc, unsigned char* s_in) {
#pragma unroll
        for (int u = 0; u < UI; u += UA) {
            Rest q;
            rest(q, u, s_desc, st, base, kc);
            finish(q, u, in_px, base, s_in);
        }
    }
};

// The weights of one K chunk as 16-byte vectors of OHWI memory, stored in LDS
// as rows [tap][co] of 64 bytes (the chunk's input channels).
template <typename T>
struct VecW {
    static constexpr int KC = ROWB / (int)sizeof(T), VQ = 16 / (int)sizeof(T);
    Vec<T, VQ> w[UW];

    __device__ __forceinline__ void issue(const ConvArgs& a, int co0, int nt, int kc) {
        const T* __restrict__ wgt = (const T*)a.weight;
        const int tid = tid_here();
#pragma unroll
        for (int u = 0; u < UW; ++u) {
            const int v = u * WG + tid;
            const int col = v / 36, rem = v - col * 36;
            const int tap = rem >> 2, q = rem & 3;
            const int co = co0 + col, ci = kc * KC + q * VQ;
            if (col < nt && co < a.C_out && ci < a.C_in) w[u] = vload<T, VQ>(wgt + ((size_t)co * 9 + tap) * a.C_in + ci);
            else                                         w[u] = vzero<T, VQ>();
        }
    }
    __device__ __forceinline__ void commit(unsigned char* s_w, int nt) const {
        const int tid = tid_here();
#pragma unroll
        for (int u = 0; u < UW; ++u) {
            const int v = u * WG + tid;
            const int col = v / 36, rem = v - col * 36;
            const int tap = rem >> 2, q = rem & 3;
            if (col < nt) *reinterpret_cast<uint4*>(s_w + swz(tap * nt + col, q)) = w[u].raw;
        }
    }
};

// ---- NCHW staging along x: a thread takes whole pixels (every channel of the
// chunk), so neighbouring lanes read neighbouring elements of a plane.  The
// first pixel's copies are requested a chunk ahead.
template <typename T>
struct PlaneIn {
    static constexpr int KC = ROWB / (int)sizeof(T), VQ = 16 / (int)sizeof(T);
    T v[KC];

    static __device__ __forceinline__ unsigned long long desc(const unsigned long long* s_desc, int in_px, int p) {
        return p < in_px ? s_desc[p] : 0ull;
    }
    __device__ __forceinline__ void issue(const unsigned long long* s_desc, const Strides<T>& st, int C_in, int in_px,
                                          int base, int kc) {
        const unsigned long long d = desc(s_desc, in_px, base + (int)threadIdx.x);
        if (C_in - kc * KC < KC) return;  // a partial chunk is staged channel by channel in commit()
#pragma unroll
        for (int c = 0; c < KC; ++c) v[c] = from_f32<T>(0.0f);
        if (d && !(d & SD_AVG)) {
            const long long cs = st.ch(d);
            const T* p = st.at(d) + kc * KC * cs;
#pragma unroll
            for (int c = 0; c < KC; ++c, p += cs) v[c] = *p;
        }
    }
    // to LDS; an average is loaded here, two pixels a load, eight channels in flight
    __device__ __forceinline__ void commit(const unsigned long long* s_desc, const Strides<T>& st, int C_in, int in_px,
                                           int base, int kc, unsigned char* s_in) {
        const int pix = base + (int)threadIdx.x;
        const unsigned long long d = desc(s_desc, in_px, pix);
        if (C_in - kc * KC < KC) {
            if (pix >= in_px) return;
            const long long cs = st.ch(d);
            const T* p = st.at(d) + kc * KC * cs;
#pragma unroll 4
            for (int c = 0; c < KC; ++c, p += cs) {
                T x = from_f32<T>(0.0f);
                if (d && kc * KC + c < C_in) {
                    x = p[0];
                    if (d & SD_AVG) x = avg4(x, p[1], p[st.d2], p[st.d2 + 1]);
                }
                const int byte = c * (int)sizeof(T);
                *reinterpret_cast<T*>(s_in + swz(pix, byte >> 4) + (byte & 15)) = x;
            }
            return;
        }
        if (d & SD_AVG) {
            constexpr int HC = 8;
            const T* p = st.at(d) + kc * KC * st.ch_hi;
#pragma unroll
            for (int h = 0; h < KC / HC; ++h) {
                T top[HC][2], bot[HC][2];
#pragma unroll
                for (int c = 0; c < HC; ++c, p += st.ch_hi) {
                    __builtin_memcpy(top[c], p, 2 * sizeof(T));
                    __builtin_memcpy(bot[c], p + st.d2, 2 * sizeof(T));
                }
#pragma unroll
                for (int c = 0; c < HC; ++c) v[h * HC + c] = avg4(top[c][0], top[c][1], bot[c][0], bot[c][1]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (pix < in_px) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                Vec<T, VQ> o;
#pragma unroll
                for (int e = 0; e < VQ; ++e) o.e[e] = v[q * VQ + e];
                *reinterpret_cast<uint4*>(s_in + swz(pix, q)) = o.raw;
            }
        }
    }
};

// The weights of one K chunk of OIHW memory: thread (co, q) takes the nine taps
// of the VQ channels of sub-chunk q, one run of 144 bytes, and turns them into
// nine 16-byte vectors of one tap each.
template <typename T>
struct PlaneW {
    static constexpr int KC = ROWB / (int)sizeof(T), VQ = 16 / (int)sizeof(T);
    static_assert(NT * 4 == WG, "one filter sub-chunk per thread");
    T w[VQ * 9];

    __device__ __forceinline__ void issue(const ConvArgs& a, int co0, int nt, int kc) {
        const int col = (int)threadIdx.x >> 2, c0 = kc * KC + ((int)threadIdx.x & 3) * VQ;
        const int nc = col < nt && co0 + col < a.C_out ? min(VQ, a.C_in - c0) : 0;  // channels of this thread's run
        const T* p = (const T*)a.weight + ((size_t)(nc > 0 ? co0 + col : 0) * a.C_in + (nc > 0 ? c0 : 0)) * 9;
        if (nc == VQ) {
#pragma unroll
            for (int v = 0; v < 9; ++v) __builtin_memcpy(w + v * VQ, p + v * VQ, 16);
        } else {
#pragma unroll
            for (int e = 0; e < VQ * 9; ++e) {
                w[e] = from_f32<T>(0.0f);
                if (e < nc * 9) w[e] = p[e];
            }
        }
    }
    __device__ __forceinline__ void commit(unsigned char* s_w, int nt) const {
        const int col = (int)threadIdx.x >> 2, q = (int)threadIdx.x & 3;
        if (col >= nt) return;
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
            Vec<T, VQ> o;
#pragma unroll
            for (int e = 0; e < VQ; ++e) o.e[e] = w[e * 9 + tap];
            *reinterpret_cast<uint4*>(s_w + swz(tap * nt + col, q)) = o.raw;
        }
    }
};

// ---- element-wise staging (channels-last tensors that are not whole vectors)
template <typename T>
__device__ __forceinline__ void stage_in_scalar(const unsigned long long* s_desc, const Strides<T>& st, int C_in,
                                                int in_px, int kc, unsigned char* s_in) {
    constexpr int KC = ROWB / (int)sizeof(T), VQ = 16 / (int)sizeof(T);
    for (int it = (int)threadIdx.x; it < in_px * 4; it += WG) {
        const int p = it >> 2, q = it & 3, c0 = kc * KC + q * VQ;
        const unsigned long long d = s_desc[p];
        const long long cs = st.ch(d);
        const T* s = st.at(d) + c0 * cs;
        Vec<T, VQ> val;
#pragma unroll
        for (int e = 0; e < VQ; ++e) {
            T v = from_f32<T>(0.0f);
            if (d && c0 + e < C_in) {
                const T* x = s + e * cs;
                v = (d & SD_AVG) ? avg4(x[0], x[st.d1], x[st.d2], x[st.d2 + st.d1]) : x[0];
            }
            val.e[e] = v;
        }
        *reinterpret_cast<uint4*>(s_in + swz(p, q)) = val.raw;
    }
}
template <typename T>
__device__ __forceinline__ void stage_w_scalar(const ConvArgs& a, int co0, int nt, int kc, unsigned char* s_w) {
    constexpr int KC = ROWB / (int)sizeof(T);
    const T* __restrict__ wgt = (const T*)a.weight;
    for (int it = (int)threadIdx.x; it < nt * KC; it += WG) {
        const int col = it / KC, cil = it - col * KC;
        const int co = co0 + col, ci = kc * KC + cil;
        const bool ok = co < a.C_out && ci < a.C_in;
        const int byte = cil * (int)sizeof(T);
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
            T wv = from_f32<T>(0.0f);
            if (ok) wv = wgt[((size_t)co * 9 + tap) * a.C_in + ci];
            *reinterpret_cast<T*>(s_w + swz(tap * nt + col, byte >> 4) + (byte & 15)) = wv;
        }
    }
}

// How a call's tensors are staged: 16-byte vectors (channels-last), element by
// element (channels-last), along x (NCHW).  What goes through registers a
// chunk ahead: request() asks for chunk kc's weights and first inputs,
// stage() writes them to LDS and stages the other inputs.
enum Stage { ST_VEC = 0, ST_SCALAR = 1, ST_PLANE = 2 };

// (MS: pixel sub-tiles per wave, whose accumulators share the registers.)
template <typename T, int STG, int MS>
struct Stager;
template <typename T, int MS>
struct Stager<T, ST_VEC, MS> {
    VecW<T> w;
    VecIn<T> in;
    // Small tiles have registers left for every vector of their averages, so
    // all of them are in flight across the MFMAs; larger ones request the first
    // of each, and the others after the MFMAs, two items at a time (before the
    // first chunk, when there are no sums yet, all at once as well).
    static constexpr bool AHEAD = MS <= 2;
    typename VecIn<T>::Rest q[UI / UA];
    __device__ __forceinline__ void rests(const unsigned long long* s_desc, const Strides<T>& st, int kc) {
#pragma unroll
        for (int i = 0; i < UI / UA; ++i) in.rest(q[i], i * UA, s_desc, st, 0, kc);
    }
    __device__ __forceinline__ void weights(const ConvArgs& a, int co0, int nt, int kc) { w.issue(a, co0, nt, kc); }
    __device__ __forceinline__ void inputs(const unsigned long long* s_desc, const Strides<T>& st, int C_in, int in_px,
                                           int kc) {
        in.issue(s_desc, st, C_in, in_px, 0, kc);
        if constexpr (AHEAD) rests(s_desc, st, kc);
    }
    template <bool FIRST>
    __device__ __forceinline__ void stage(const ConvArgs& a, int, int nt, int kc, const unsigned long long* s_desc,
                                          const Strides<T>& st, int in_px, unsigned char* s_in, unsigned char* s_w) {
        if constexpr (FIRST && !AHEAD) rests(s_desc, st, kc);
        w.commit(s_w, nt);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (FIRST || AHEAD) {
#pragma unroll
            for (int i = 0; i < UI / UA; ++i) in.finish(q[i], i * UA, in_px, 0, s_in);
        } else {
            in.commit(s_desc, st, in_px, 0, kc, s_in);
        }
        for (int base = WG * UI; base < in_px * 4; base += WG * UI) {
            in.issue(s_desc, st, a.C_in, in_px, base, kc);
            in.commit(s_desc, st, in_px, base, kc, s_in);
        }
    }
};
template <typename T, int MS>
struct Stager<T, ST_PLANE, MS> {
    PlaneW<T> w;
    PlaneIn<T> in;
    __device__ __forceinline__ void weights(const ConvArgs& a, int co0, int nt, int kc) { w.issue(a, co0, nt, kc); }
    __device__ __forceinline__ void inputs(const unsigned long long* s_desc, const Strides<T>& st, int C_in, int in_px,
                                           int kc) {
        in.issue(s_desc, st, C_in, in_px, 0, kc);
    }
    template <bool FIRST>
    __device__ __forceinline__ void stage(const ConvArgs& a, int, int nt, int kc, const unsigned long long* s_desc,
                                          const Strides<T>& st, int in_px, unsigned char* s_in, unsigned char* s_w) {
        w.commit(s_w, nt);
        __builtin_amdgcn_sched_barrier(0);
        in.commit(s_desc, st, a.C_in, in_px, 0, kc, s_in);
        for (int base = WG; base < in_px; base += WG) {
            in.issue(s_desc, st, a.C_in, in_px, base, kc);
            in.commit(s_desc, st, a.C_in, in_px, base, kc, s_in);
        }
    }
};
template <typename T, int MS>
struct Stager<T, ST_SCALAR, MS> {
    __device__ __forceinline__ void weights(const ConvArgs&, int, int, int) {}
    __device__ __forceinline__ void inputs(const unsigned long long*, const Strides<T>&, int, int, int) {}
    template <bool FIRST>
    __device__ __forceinline__ void stage(const ConvArgs& a, int co0, int nt, int kc, const unsigned long long* s_desc,
                                          const Strides<T>& st, int in_px, unsigned char* s_in, unsigned char* s_w) {
        stage_w_scalar<T>(a, co0, nt, kc, s_w);
        stage_in_scalar<T>(s_desc, st, a.C_in, in_px, kc, s_in);
    }
};

// The nine taps of one staged chunk, NS channel sub-tiles by NM pixel sub-tiles.
// (Straight code for every count: a test per sub-tile between the reads and the
// MFMAs of a lone wave cost a quarter of this phase.)  TAPS taps at a time where
// there is one pixel sub-tile: its few MFMAs don't cover the reads of the next.
template <typename T, int NS, int NM, int MS, int TAPS>
__device__ __forceinline__ void chunk_taps(floatx4 (&acc)[MS][4], const unsigned char* wlane, const unsigned char* s_in,
                                           const int (&pbase)[MS], int pe, int kg, int nt) {
#pragma unroll TAPS
    for (int tap = 0; tap < 9; ++tap) {
        const int toff = (tap / 3) * pe + (tap % 3);
        uint4 wf[NS], pf[NM];
#pragma unroll
        for (int ns = 0; ns < NS; ++ns) wf[ns] = *reinterpret_cast<const uint4*>(wlane + (tap * nt + ns * 16) * ROWB);
#pragma unroll
        for (int ms = 0; ms < NM; ++ms) pf[ms] = *reinterpret_cast<const uint4*>(s_in + swz(pbase[ms] + toff, kg));
#pragma unroll
        for (int ms = 0; ms < NM; ++ms)
#pragma unroll
            for (int i = 0; i < MF<T>::STEPS; ++i)
#pragma unroll
                for (int ns = 0; ns < NS; ++ns) acc[ms][ns] = MF<T>::mma(wf[ns], pf[ms], i, acc[ms][ns]);
    }
}
template <typename T, int NS, int MS, int TAPS>
__device__ __forceinline__ void chunk_mfma(floatx4 (&acc)[MS][4], const unsigned char* wlane, const unsigned char* s_in,
                                           const int (&pbase)[MS], int pe, int kg, int nt, int nms) {
    if (nms == 1) return chunk_taps<T, NS, 1, MS, TAPS>(acc, wlane, s_in, pbase, pe, kg, nt);
    if (nms == 2) return chunk_taps<T, NS, 2, MS, 1>(acc, wlane, s_in, pbase, pe, kg, nt);
    if constexpr (MS > 2) {
        if (nms == 3) return chunk_taps<T, NS, 3, MS, 1>(acc, wlane, s_in, pbase, pe, kg, nt);
        if (nms == 4) return chunk_taps<T, NS, 4, MS, 1>(acc, wlane, s_in, pbase, pe, kg, nt);
    }
}

template <typename T, int L, int SRC, int DST, int STG, int MS>
__global__ __launch_bounds__(WG, 2) void k_conv(Geo g, const uint8_t* __restrict__ mask, ConvArgs a, int Rh,
                                                int Rl, int w_off, int d_off, int nt, int vec_out) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int KC = ROWB / (int)sizeof(T);  // channels per K chunk
    constexpr bool NEED_SLOTS = !(SRC == SRC_DENSE && DST == DST_DENSE);
    // (not where it costs registers that the staging needs: fp32 and NCHW tiles
    // of four sub-tiles got 3 to 4 % slower, the others up to 6 % faster)
    constexpr int TAPS = MS <= 2 || (STG == ST_VEC && MF<T>::STEPS == 1) ? 3 : 1;

    unsigned char* s_in = smem;
    unsigned char* s_w = smem + w_off;
    unsigned long long* s_desc = reinterpret_cast<unsigned long long*>(smem + d_off);
    // Tile grp of block k, the blocks fastest, then the channel tiles: the class
    // with fewer tiles fills only the first of a block's places, and workgroups
    // go to the XCDs and their CUs in turn.  With the tiles fastest all-low maps
    // ran on two of the eight XCDs (conv3x3 of 64 channels on 256x512 fp32 NHWC
    // 116 us, now 33), with the channel tiles slowest on half of the CUs (96
    // channels, 16-pixel blocks, fp16: 25.5 us, now 19.5).
    const int B = (int)g.B, ny = (a.C_out + nt - 1) / nt;
    int k = (int)blockIdx.x;
    const int first = k / B, row = first + (int)blockIdx.y, grp = row / ny;  // (one of the two is 0)
    k -= first * B;
    const int co0 = (row - grp * ny) * nt;
    if constexpr (L == NCHW) {
        // runs of four blocks on one XCD: a halo column of a plane is a line of the
        // neighbour's for every row (all-high fp16 256x512 of 64 channels: 37.2 us
        // without, 34.3 with; longer runs would put a map's low region on few XCDs)
        constexpr int RUN = 4;
        const int base = k & ~(8 * RUN - 1), o = k - base;
        if (base + 8 * RUN <= B) k = base + (o & 7) * RUN + (o >> 3);
    }
    const int nsn = (min(nt, a.C_out - co0) + 15) >> 4;  // 16-channel sub-tiles that hold channels
    Tile t;
    {
        const int per = g.GH * g.GW;
        t.n = k / per;
        const int rem = k - t.n * per;
        t.gy = rem / g.GW;
        t.gx = rem - t.gy * g.GW;
    }
    WaveMask wm;
    wm.init(mask, (int)g.B);
    const Neigh nb = wave_neighbourhood<NEED_SLOTS>(wm, g.GH, g.GW, t.n, t.gy, t.gx);
    t.high = (nb.high >> 4) & 1;
    t.slot = nb.slot[4];
    if (NEED_SLOTS && t.slot >= (t.high ? a.hi_cap : a.lo_cap)) return;
    t.e = t.high ? g.bs : (g.bs >> 1);
    const int R = t.high ? Rh : Rl;
    t.r0 = grp * R;
    if (t.r0 >= t.e) return;
    t.rows = min(R, t.e - t.r0);
    t.M = t.rows * t.e;
    t.pe = t.e + 2;
    t.in_px = (t.rows + 2) * t.pe;
    const Strides<T> st = make_strides<T, L, SRC>(g, a, t);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, kg = lane >> 4;

    // -- chunk 0's weights, and the tile's source descriptors
    Stager<T, STG, MS> sg;
    sg.weights(a, co0, nt, 0);
    for (int p = tid; p < t.in_px; p += WG) {
        const Src<T> s = tile_src<T, L, SRC>(g, a, nb, t, p);
        unsigned long long d = 0;
        if (s.p)
            d = ((reinterpret_cast<unsigned long long>(s.p) - reinterpret_cast<unsigned long long>(st.hi)) & SD_OFF) |
                SD_SOME | (s.avg ? SD_AVG : 0ull) | (s.low ? SD_LOW : 0ull);
        s_desc[p] = d;
    }
    __syncthreads();

    const int nst = (t.M + 15) >> 4;  // 16-pixel sub-tiles
    const int nms = __builtin_amdgcn_readfirstlane((nst - wave + 3) >> 2);  // this wave's (wave, wave + 4, ...)
    int pbase[MS];
#pragma unroll
    for (int ms = 0; ms < MS; ++ms) {
        const int m = min((wave + 4 * ms) * 16 + l16, t.M - 1);
        const int i = m / t.e, j = m - i * t.e;
        pbase[ms] = i * t.pe + j;
    }
    const int nchunks = (a.C_in + KC - 1) / KC;

    sg.inputs(s_desc, st, a.C_in, t.in_px, 0);
    sg.template stage<true>(a, co0, nt, 0, s_desc, st, t.in_px, s_in, s_w);
    __syncthreads();

    floatx4 acc[MS][4];
#pragma unroll
    for (int ms = 0; ms < MS; ++ms)
#pragma unroll
        for (int ns = 0; ns < 4; ++ns) acc[ms][ns] = floatx4{0.f, 0.f, 0.f, 0.f};
    const unsigned char* wlane = s_w + swz(l16, kg);  // (nt is a multiple of 16: the swizzle of a row is its l16's)

    for (int kc = 0; kc < nchunks; ++kc) {
        const bool more = kc + 1 < nchunks;
        // -- prefetch the next chunk's weights and first input batch
        if (more) {
            sg.weights(a, co0, nt, kc + 1);
            sg.inputs(s_desc, st, a.C_in, t.in_px, kc + 1);
        }
        // -- MFMA over the 9 taps of this chunk
        switch (nsn) {
        case 1: chunk_mfma<T, 1, MS, TAPS>(acc, wlane, s_in, pbase, t.pe, kg, nt, nms); break;
        case 2: chunk_mfma<T, 2, MS, TAPS>(acc, wlane, s_in, pbase, t.pe, kg, nt, nms); break;
        case 3: chunk_mfma<T, 3, MS, TAPS>(acc, wlane, s_in, pbase, t.pe, kg, nt, nms); break;
        default: chunk_mfma<T, 4, MS, TAPS>(acc, wlane, s_in, pbase, t.pe, kg, nt, nms); break;
        }
        __syncthreads();
        if (more) {
            sg.template stage<false>(a, co0, nt, kc + 1, s_desc, st, t.in_px, s_in, s_w);
            __syncthreads();
        }
    }

    // -- epilogue: lane holds channels co0 + ns*16 + kg*4 + {0..3} of pixel (wave + 4*ms)*16 + l16
    const T* __restrict__ bias = (const T*)a.bias;
    const bool relu = (a.flags & 1) != 0;
    const int co_end = min(co0 + nt, a.C_out);
    float bv[4][4];
#pragma unroll
    for (int ns = 0; ns < 4; ++ns)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int co = co0 + ns * 16 + kg * 4 + r;
            bv[ns][r] = (bias && co < co_end) ? to_f32(bias[co]) : 0.0f;
        }
    const T* res_base = (const T*)(t.high ? a.res_hi : a.res_lo);
    T* out_base = (T*)((DST == DST_DENSE || t.high) ? a.out_hi : a.out_lo);
#pragma unroll
    for (int ms = 0; ms < MS; ++ms) {
        if (wave + 4 * ms >= nst) continue;
        const int m = (wave + 4 * ms) * 16 + l16;
        if (m >= t.M) continue;
        const int i = t.r0 + m / t.e, j = m % t.e;
#pragma unroll
        for (int ns = 0; ns < 4; ++ns) {
            const int co = co0 + ns * 16 + kg * 4;
            if (co >= co_end) continue;
            float f[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) f[r] = acc[ms][ns][r] + bv[ns][r];
            const bool full = vec_out && co + 4 <= co_end;
            if constexpr (DST == DST_PACKED) {
                // packed stack element (slot, co + r, i, j)
                size_t off[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if constexpr (L == NHWC) off[r] = (((size_t)t.slot * t.e + i) * t.e + j) * a.C_out + co + r;
                    else off[r] = (((size_t)t.slot * a.C_out + co + r) * t.e + i) * t.e + j;
                }
                if (res_base) {
                    if (L == NHWC && full) {
                        const Vec<T, 4> rv = vload<T, 4>(res_base + off[0]);
#pragma unroll
                        for (int r = 0; r < 4; ++r) f[r] += to_f32(rv.e[r]);
                    } else {
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (co + r < co_end) f[r] += to_f32(res_base[off[r]]);
                    }
                }
                Vec<T, 4> o;
#pragma unroll
                for (int r = 0; r < 4; ++r) o.e[r] = from_f32<T>(relu ? fmaxf(f[r], 0.0f) : f[r]);
                if (L == NHWC && full) {
                    vstore<T, 4>(out_base + off[0], o);
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (co + r < co_end) out_base[off[r]] = o.e[r];
                }
            } else {
                Vec<T, 4> o;
#pragma unroll
                for (int r = 0; r < 4; ++r) o.e[r] = from_f32<T>(relu ? fmaxf(f[r], 0.0f) : f[r]);
                const int reps = t.high ? 1 : 2;
                for (int dy = 0; dy < reps; ++dy) {
                    const int Y = t.gy * g.bs + (t.high ? i : 2 * i + dy);
                    if constexpr (L == NHWC) {
                        for (int dx = 0; dx < reps; ++dx) {
                            const int X = t.gx * g.bs + (t.high ? j : 2 * j + dx);
                            T* p = out_base + (((size_t)t.n * g.H + Y) * g.W + X) * a.C_out + co;
                            if (full) {
                                vstore<T, 4>(p, o);
                            } else {
#pragma unroll
                                for (int r = 0; r < 4; ++r)
                                    if (co + r < co_end) p[r] = o.e[r];
                            }
                        }
                    } else {
                        const int X = t.gx * g.bs + (t.high ? j : 2 * j);
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            if (co + r >= co_end) continue;
                            T* p = out_base + (((size_t)t.n * a.C_out + co + r) * g.H + Y) * g.W + X;
                            if (t.high) {
                                *p = o.e[r];
                            } else {  // both pixels of the cell's row in one store
                                const T two[2] = {o.e[r], o.e[r]};
                                __builtin_memcpy(p, two, sizeof(two));
                            }
                        }
                    }
                }
            }
        }
    }
}

inline int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }
inline bool aligned(const void* p, int bytes) { return (reinterpret_cast<uintptr_t>(p) & (bytes - 1)) == 0; }

// Rows per tile and output channels per workgroup.  About 256 pixels a tile
// read the fewest halo pixels and weights; 128 or 64 where that many smaller
// tiles still find a place at once (two workgroups a CU), so that more of the
// chip works.  Measured, half low, 256 / 128 / 64 pixels a tile: one 128x256 map
// of 96 channels, 16-pixel blocks, fp16 (256 / 512 / 1024 workgroups) 27.6 /
// 22.2 / 34.4 us; the 256x512 fp32 layer of 64 channels, 32-pixel blocks (512 /
// 1024 / 2048) 98 / 108 / 130 us.  (A fused layer counts every block as high,
// so an all-low map may run with larger tiles than its own count would take:
// that fp32 layer 75 us where 128 pixels a tile give 45.)  The channel tiles of
// a call are equal, so that 72 channels are 48 + 24 and not 64 + 8.
struct ConvPlan {
    int Rh, Rl, G, nt, ny, M;
};
inline ConvPlan conv_plan(const Geo& g, const ConvArgs& a, bool dense) {
    ConvPlan p{};
    const int eh = g.bs, el = g.bs / 2;
    p.ny = (a.C_out + NT - 1) / NT;
    p.nt = ((a.C_out + p.ny - 1) / p.ny + 15) / 16 * 16;
    p.ny = (a.C_out + p.nt - 1) / p.nt;
    // (dense: the class counts are on the device; every block high is the most work)
    const long long nh = dense ? g.B : std::min<long long>(a.hi_cap, g.B);
    const long long nl = dense ? 0 : std::min<long long>(a.lo_cap, g.B);
    for (int mt = 256; mt >= 64; mt /= 2) {
        int Rh = clampi(mt / eh, 1, eh), Rl = clampi(mt / el, 1, el);
        const int Gh = (eh + Rh - 1) / Rh, Gl = (el + Rl - 1) / Rl;
        Rh = (eh + Gh - 1) / Gh;  // equal tiles
        Rl = (el + Gl - 1) / Gl;
        if (mt < 256 && (nh * Gh + nl * Gl) * p.ny > 2LL * device_cus()) break;
        p.Rh = Rh;
        p.Rl = Rl;
        p.G = std::max(nh > 0 ? Gh : 0, dense || nl > 0 ? Gl : 0);
        p.M = std::max(Rh * eh, Rl * el);
    }
    return p;
}

template <typename T, int L, int SRC, int DST, int STG, int MS>
hipError_t run_conv_ms(const Geo& g, const uint8_t* mask, const ConvArgs& a, const ConvPlan& p, hipStream_t st) {
    const int eh = g.bs, el = g.bs / 2;
    const int in_px = std::max((p.Rh + 2) * (eh + 2), (p.Rl + 2) * (el + 2));
    const int w_off = in_px * ROWB, d_off = w_off + 9 * p.nt * ROWB, smem = d_off + in_px * 8;
    const int ob = 4 * (int)sizeof(T);  // one epilogue vector: 4 channels
    const int vec_out = (a.C_out % 4 == 0) && aligned(a.out_hi, ob) && aligned(a.out_lo, ob) &&
                        aligned(a.res_hi, ob) && aligned(a.res_lo, ob);
    hipError_t e = ensure_dyn_lds((const void*)k_conv<T, L, SRC, DST, STG, MS>, smem);
    if (e != hipSuccess || p.G == 0) return e;
    // one row of workgroups per (tile, channel tile), one after the other, or down
    // the grid where a launch's 2^32 threads in x do not hold them
    const bool flat = g.B * p.G * p.ny * WG < (1LL << 32);
    const dim3 grid((unsigned)(flat ? g.B * p.G * p.ny : g.B), (unsigned)(flat ? 1 : p.G * p.ny));
    hipLaunchKernelGGL((k_conv<T, L, SRC, DST, STG, MS>), grid, dim3(WG), smem, st, g, mask, a, p.Rh, p.Rl, w_off,
                       d_off, p.nt, vec_out);
    return hipGetLastError();
}

template <typename T, int L, int SRC, int DST, int STG>
hipError_t run_conv(const Geo& g, const uint8_t* mask, const ConvArgs& a, hipStream_t st) {
    const ConvPlan p = conv_plan(g, a, SRC == SRC_DENSE);
    if (p.M <= 128) return run_conv_ms<T, L, SRC, DST, STG, 2>(g, mask, a, p, st);
    return run_conv_ms<T, L, SRC, DST, STG, 4>(g, mask, a, p, st);
}

template <typename T, int SRC, int DST>
hipError_t conv_l(int layout, const Geo& g, const uint8_t* mask, const ConvArgs& a, hipStream_t st) {
    constexpr int VQ = 16 / (int)sizeof(T);
    if (layout == NHWC) {
        const bool vec = (a.C_in % VQ == 0) && aligned(a.in_hi, 16) && aligned(a.in_lo, 16) &&
                         aligned(a.weight, 16);
        if (vec) return run_conv<T, NHWC, SRC, DST, ST_VEC>(g, mask, a, st);
        return run_conv<T, NHWC, SRC, DST, ST_SCALAR>(g, mask, a, st);
    }
    return run_conv<T, NCHW, SRC, DST, ST_PLANE>(g, mask, a, st);
}

template <typename T>
hipError_t conv_t(int layout, ConvSrc src, ConvDst dst, const Geo& g, const uint8_t* mask, const ConvArgs& a,
                  hipStream_t st) {
    if (src == SRC_PADDED) return conv_l<T, SRC_PADDED, DST_PACKED>(layout, g, mask, a, st);
    if (src == SRC_PACKED) return conv_l<T, SRC_PACKED, DST_PACKED>(layout, g, mask, a, st);
    (void)dst;
    return conv_l<T, SRC_DENSE, DST_DENSE>(layout, g, mask, a, st);
}

}  // namespace

// A fused layer (dense map in and out) with many channels runs on the GEMM:
// with average sampling and blocks that tile the map, as the padded low
// stack (straight from the map) and the GEMM reading the high blocks from
// the map and writing the dense output; otherwise as split, the GEMM's block
// convolution (BlockPad fused) and combine over packed stacks in the
// caller's workspace, with room for every block in either class (the counts
// are only known on the device).  The values equal the one-kernel layer's up
// to the order of the fp32 accumulation.
namespace {

inline size_t round256(size_t b) { return (b + 255) / 256 * 256; }

bool layer_packed_route(int dtype, int layout, const Geo& g, const ConvArgs& a) {
    // Measured on the stage shapes of a 1024x2048 image (8x16 blocks): at 128
    // channels 44-50 -> 38-43 us (all-low 29 -> 38), at 512 105-116 -> 37-62 us
    // with split + GEMM + combine; the dense GEMM route (the padded low stack
    // from the map, high pixels read from it, the output written to it) takes
    // 8-10 us more off (128 channels 34 / 37 -> 24 / 27 us at 0 / 50 % low,
    // 512 channels 41 -> 33 us) and beats the general kernel at 256 channels as
    // well (40 / 43 -> 34 / 35 us on one 64x128 map).  Without the dense route
    // the general kernel stays faster at 129-256 channels on up to 8192 pixels
    // (two maps: 77 / 82 against 56 / 57 us with split + GEMM + combine).
    if (a.C_in <= 64 || layout != NHWC || (dtype != 1 && dtype != 2)) return false;
    if (a.C_in > 128 && a.C_in <= 256 && (long long)g.N * g.H * g.W <= 8192 && !igemm_dense_fits(dtype, layout, g, a))
        return false;
    Geo gi = g, go = g;
    gi.C = a.C_in;
    go.C = a.C_out;
    ConvArgs p = a;
    p.hi_cap = p.lo_cap = (int)g.B;
    return igemm_fits_shape(dtype, layout, g, p) && rows_fit(dtype, layout, gi, {}) && rows_fit(dtype, layout, go, {});
}

// the packed stacks of the route: [hi in][lo in][hi out][lo out][GEMM workspace]
struct PackedLayout {
    size_t hi_in, lo_in, hi_out, lo_out, gemm, total;
};

PackedLayout packed_layout(const Geo& g, const ConvArgs& a) {
    const size_t es = 2, cap = (size_t)g.B, lb = (size_t)g.bs / 2;
    PackedLayout L;
    L.hi_in = round256(cap * g.bs * g.bs * a.C_in * es);
    L.lo_in = round256(cap * lb * lb * a.C_in * es);
    L.hi_out = round256(cap * g.bs * g.bs * a.C_out * es);
    L.lo_out = round256(cap * lb * lb * a.C_out * es);
    ConvArgs p = a;
    p.hi_cap = p.lo_cap = (int)cap;
    L.gemm = igemm_ws_bytes(g, p, 3, 1);
    L.total = L.hi_in + L.lo_in + L.hi_out + L.lo_out + L.gemm;
    return L;
}

hipError_t layer_via_packed(int dtype, const Geo& g, const uint8_t* mask, const ConvArgs& a, Ws ws, hipStream_t st) {
    const PackedLayout L = packed_layout(g, a);
    if (ws.bytes < L.total || !ws.p) return hipErrorInvalidValue;
    const int cap = (int)g.B;
    char* base = (char*)ws.p;
    void *hi = base, *lo = base + L.hi_in, *ho = base + L.hi_in + L.lo_in;
    void* lo_o = base + L.hi_in + L.lo_in + L.hi_out;
    const Ws gws{base + L.hi_in + L.lo_in + L.hi_out + L.lo_out, L.gemm};
    Geo gi = g, go = g;
    gi.C = a.C_in;
    go.C = a.C_out;
    hipError_t e = launch_split_rows(dtype, gi, a.in_hi, mask, hi, cap, lo, cap, st);
    if (e != hipSuccess) return e;
    const ConvArgs p{hi, lo, a.weight, a.bias, nullptr, nullptr, ho, lo_o, a.C_in, a.C_out, a.flags, cap, cap};
    if ((e = launch_igemm(dtype, g, mask, p, 3, 1, gws, st)) != hipSuccess) return e;
    return launch_combine_rows(dtype, go, ho, lo_o, mask, cap, cap, a.out_hi, st);
}

}  // namespace

size_t conv_ws_bytes(int dtype, int layout, ConvSrc src, ConvDst dst, const Geo& g, const ConvArgs& a, bool frugal) {
    if (conv_res_fits_shape(dtype, layout, g, a)) return 0;
    if (src == SRC_PACKED && dst == DST_PACKED && igemm_fits_shape(dtype, layout, g, a))
        return igemm_ws_bytes(g, a, 3, 1, frugal);
    if (src == SRC_DENSE && dst == DST_DENSE && layer_packed_route(dtype, layout, g, a))
        return igemm_dense_fits(dtype, layout, g, a) ? igemm_dense_ws_bytes(g, a) : packed_layout(g, a).total;
    return 0;
}

hipError_t launch_conv(int dtype, int layout, ConvSrc src, ConvDst dst, const Geo& g, const uint8_t* mask,
                       const ConvArgs& a, Ws ws, hipStream_t st) {
    if (conv_res_fits(dtype, layout, g, a)) return launch_conv_res(dtype, src, dst, g, mask, a, st);
    if (src == SRC_PACKED && dst == DST_PACKED && igemm_fits(dtype, layout, g, a))
        return launch_igemm(dtype, g, mask, a, 3, 1, ws, st);
    if (src == SRC_DENSE && dst == DST_DENSE && layer_packed_route(dtype, layout, g, a) &&
        reinterpret_cast<uintptr_t>(a.in_hi) % 16 == 0 && reinterpret_cast<uintptr_t>(a.out_hi) % 16 == 0 &&
        reinterpret_cast<uintptr_t>(a.weight) % 16 == 0) {
        if (igemm_dense_fits(dtype, layout, g, a)) {
            if (ws.bytes < igemm_dense_ws_bytes(g, a)) return hipErrorInvalidValue;
            return launch_igemm_dense(dtype, g, mask, a, ws, st);
        }
        return layer_via_packed(dtype, g, mask, a, ws, st);
    }
    switch (dtype) {
    case 0: return conv_t<float>(layout, src, dst, g, mask, a, st);
    case 1: return conv_t<f16>(layout, src, dst, g, mask, a, st);
    default: return conv_t<bf16>(layout, src, dst, g, mask, a, st);
    }
}

}  // namespace sb

// HIP kernels of the Winograd F(m x m, 3 x 3) convolution on gfx950 other than the
// fused kernel (wino_ws.h, instantiated per blocking by wino_fused_inst.hip): the
// kernel transform, the three-stage pipeline, and the host-side choice and launch
// of the fused kernel's blocking.
#include "wino_split.h"

#include <cstdio>

namespace wino {

// The fused kernel's instantiations live in their own objects.
#define WINO_EXTERN_WS(m, R, kit, tb, fs, csp)                                                              \
    extern template hipError_t launch_ws_t<m, tb, fs, csp>(const Geometry &, const float *, const float *, \
                                                           float *, bool, int, int, const SplitBuffers &,  \
                                                           hipStream_t);
WINO_FUSED_BLOCKINGS(WINO_EXTERN_WS)
#undef WINO_EXTERN_WS
#define WINO_EXTERN_SPLIT(m) \
    extern template hipError_t launch_split_t<m>(const Geometry &, const float *, const float *, float *, int, bool, \
                                                 const SplitBuffers &, hipStream_t);
WINO_SPLIT_M(WINO_EXTERN_SPLIT)
#undef WINO_EXTERN_SPLIT

// ---------------------------------------------------------------------------
// Kernel transform (Sec. 3, step 2: right-hand matrices transformed ahead of
// time).  Thread (kb, cs, lane) transforms kernel (k, c) with k = 16 kb + lane%16,
// c = 4 cs + lane/16 and stores the T^2 values in matrix-core operand order:
// wt[((kb * Cs + cs) * Q + f/4) * 64 + lane][f % 4], Q = ceil(T^2/4).  Channels
// >= C, output channels >= K and frequencies >= T^2 are stored as zeros.
template <int M>
__global__ void __launch_bounds__(256) weight_transform_kernel(const float *__restrict__ w,
                                                               floatx4 *__restrict__ wt, Geometry g,
                                                               unsigned *zero, int nzero) {
    constexpr int T = M + 2, T2 = T * T;
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < nzero; i += blockDim.x) zero[i] = 0u;
    const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long total = (long long)g.Kb_alloc * g.Cs * 64;
    if (gid >= total) return;
    const int lane = (int)(gid & 63);
    const long long grp = gid >> 6;
    const int cs = (int)(grp % g.Cs);
    const int kb = (int)(grp / g.Cs);
    const int c = cs * 4 + (lane >> 4);
    const int k = kb * 16 + (lane & 15);
    float gk[9];
    const bool ok = (c < g.C) && (k < g.K);
    const float *src = w + ((long long)(ok ? k : 0) * g.C + (ok ? c : 0)) * 9;
#pragma unroll
    for (int i = 0; i < 9; ++i) gk[i] = ok ? src[i] : 0.0f;
    constexpr int Q = freq_quads<M>();
    float t[4 * Q];
    kernel_tile_transform<M>(gk, t);
#pragma unroll
    for (int f = T2; f < 4 * Q; ++f) t[f] = 0.0f;
    floatx4 *dst = wt + grp * Q * 64 + lane;
#pragma unroll
    for (int f4 = 0; f4 < Q; ++f4) {
        floatx4 v = {t[4 * f4], t[4 * f4 + 1], t[4 * f4 + 2], t[4 * f4 + 3]};
        dst[f4 * 64] = v;
    }
}

// Kernel transform into split-product operands (launch_weight_transform_split): a
// workgroup transforms 32 output x 16 input channels, one kernel per thread (input
// channel fastest, so that w is read in runs of 16 kernels), splits each value into
// its three bf16 terms and passes FCH frequencies through LDS, from which whole operands
// are stored as 16-byte vectors.  blockIdx.y picks the FCH frequencies a workgroup keeps
// (the transform of the others is dropped by the compiler).  Bound: latency; FCH = 16, but 8
// up to 128 workgroups of 16 and 4 up to 64, so that more compute units have one (whole
// calls with kernels given, us: 4 images of 57 x 61, C = 37, K = 45, F(2) 8 workgroups 15.8 ->
// 14.9 at 4; 64 of 28 x 28, 128 channels, F(4) 96 workgroups 45.5 -> 45.0 at 8, F(6) 128 68.6
// -> 68.1, three-stage C = 64, K = 256, F(7) 192 25.4 -> 25.7).
template <int M, int FCH, int PART>
__device__ __forceinline__ void weight_split_part(const float *gk, unsigned short *st, uintx4 *dst, int tid) {
    constexpr int T2 = (M + 2) * (M + 2), F0 = PART * FCH, FN = T2 - F0 < FCH ? T2 - F0 : FCH;
    float t[T2];
    kernel_tile_transform<M>(gk, t);
    // lane (c % 16) / 8 * 32 + k % 32, element c % 8 of each of the three terms
    const int c = tid & 15, k = tid >> 4, at = ((c >> 3) * 32 + k) * 8 + (c & 7);
#pragma unroll
    for (int f = 0; f < FN; ++f) {
        const float v = t[F0 + f];
        unsigned a, b, e;
        split_pair(v * kSplitScale, 0.0f, a, b, e);
        if (!(__builtin_fabsf(v) < kSplitMax)) {
            a = kSplitRaw;
            b = __builtin_bit_cast(unsigned, v) >> 16;
            e = __builtin_bit_cast(unsigned, v);
        }
        st[f * 1536 + at] = (unsigned short)a;
        st[f * 1536 + 512 + at] = (unsigned short)b;
        st[f * 1536 + 1024 + at] = (unsigned short)e;
    }
    __syncthreads();
    for (int i = tid; i < FN * 192; i += 512) dst[F0 * 192 + i] = reinterpret_cast<const uintx4 *>(st)[i];
}

template <int M, int FCH, int PART = 0>
__device__ __forceinline__ void weight_split_pick(int part, const float *gk, unsigned short *st, uintx4 *dst, int tid) {
    if constexpr (PART * FCH < (M + 2) * (M + 2)) {
        if (part == PART) weight_split_part<M, FCH, PART>(gk, st, dst, tid);
        else weight_split_pick<M, FCH, PART + 1>(part, gk, st, dst, tid);
    }
}

template <int M, int FCH>
__global__ void __launch_bounds__(512) weight_transform_split_kernel(const float *__restrict__ w,
                                                                     uintx4 *__restrict__ wt, Geometry g,
                                                                     unsigned *zero, int nzero) {
    constexpr int T2 = (M + 2) * (M + 2);
    __shared__ __align__(16) unsigned short st[FCH * 1536];
    const int tid = threadIdx.x;
    if (blockIdx.x == 0 && blockIdx.y == 0)
        for (int i = tid; i < nzero; i += blockDim.x) zero[i] = 0u;
    const int cs16 = (g.C + 15) / 16;
    const int kb = blockIdx.x / cs16, cs = blockIdx.x - kb * cs16;
    const int c = cs * 16 + (tid & 15), k = kb * 32 + (tid >> 4);
    const bool ok = c < g.C && k < g.K;
    const float *src = w + ((long long)(ok ? k : 0) * g.C + (ok ? c : 0)) * 9;
    float gk[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) gk[i] = ok ? src[i] : 0.0f;
    weight_split_pick<M, FCH>(blockIdx.y, gk, st, wt + (size_t)blockIdx.x * T2 * 192, tid);
}

// ---------------------------------------------------------------------------
// Three-stage pipeline (Sec. 3): stage 1 writes the transformed input tiles U of
// all tiles to device memory, stage 2 forms M[f][k][tile] = sum_c W'[f][c][k]
// U[f][c][tile] for every frequency f, stage 3 inverse-transforms M into y.
// The intermediates are stored in the matrix-core operand order, four
// consecutive frequencies per 16-byte element, so that every stage moves them
// with one coalesced 1 KB access per wave and instruction:
//   U [F4][TB][Cs][64][4]:    element (f, c, tile) at f4 = f/4, tb = tile/16,
//                             cs = c/4, lane (c%4)*16 + tile%16, slot f%4 (the B
//                             operand of v_mfma_f32_16x16x4f32 for 4 frequencies);
//   M [F4][TB][Kb][4][64][4]: element (f, k, tile) at f4, tb, kb = k/16, v = k%4,
//                             lane ((k%16)/4)*16 + tile%16, slot f%4 (the
//                             accumulator layout: lane l holds D[4(l/16)+v][l%16]).
// TB = tiles_p / 16, Cs = ceil(C/4), Kb = Kb_alloc; channels, output channels and
// tiles past the problem hold zeros.

// Workgroup b of a 1-D grid of n runs on XCD b % 8; the index returned numbers the
// workgroups so that each XCD takes one contiguous range of them.
__device__ __forceinline__ int xcd_contiguous_block(int b, int n) {
    const int xcd = b % 8, per = n / 8, extra = n % 8;
    return xcd * per + (xcd < extra ? xcd : extra) + b / 8;
}

// Input tile of F(7x7,3x3) (T = 9, too wide for the row-vector loader's halo
// exchange within 16 lanes): per row the lane's own 7 columns as 4-byte-aligned
// vector loads (4 + 2 + 1 floats) and its two halo columns as single loads; rows
// and halo columns outside the image read as zero through the buffer range check,
// own columns past W (the last tile of a row) are cleared.
template <int M>
struct WideRowTile {
    static constexpr int T = M + 2;
    static_assert(M == 7, "loader of the 9 x 9 input tiles");
    unsigned roff[T];
    unsigned own, left, right, ownok;

    __device__ __forceinline__ void init(const Geometry &g, const TileIdx &t, int lane_c) {
        const unsigned base = (unsigned)(((long long)t.n * g.C + lane_c) * g.H * g.W) * 4u;
#pragma unroll
        for (int a = 0; a < T; ++a) {
            const int h = t.ty * M - 1 + a;
            roff[a] = (t.ok && h >= 0 && h < g.H) ? base + (unsigned)(h * g.W) * 4u : kOutside;
        }
        own = (unsigned)(t.tx * M) * 4u;
        left = t.tx > 0 ? own - 4u : kOutside;
        right = t.tx * M + M < g.W ? own + 4u * M : kOutside;
        ownok = 0u;
#pragma unroll
        for (int j = 0; j < M; ++j)
            if (t.tx * M + j < g.W) ownok |= 1u << j;
    }

    __device__ __forceinline__ void load(int32x4 r, float *d) const {
#pragma unroll
        for (int a = 0; a < T; ++a) {
            const unsigned ro = roff[a];
            const floatx4 q4 = buffer_load_f32x4(r, __builtin_elementwise_add_sat(ro, own), 0, 0);
            const floatx2 q2 = buffer_load_f32x2(r, __builtin_elementwise_add_sat(ro, own + 16u), 0, 0);
            const float q1 = buffer_load_f32(r, __builtin_elementwise_add_sat(ro, own + 24u), 0, 0);
            d[a * T] = buffer_load_f32(r, __builtin_elementwise_add_sat(ro, left), 0, 0);
            d[a * T + T - 1] = buffer_load_f32(r, __builtin_elementwise_add_sat(ro, right), 0, 0);
#pragma unroll
            for (int j = 0; j < 4; ++j) d[a * T + 1 + j] = q4[j];
            d[a * T + 5] = q2[0];
            d[a * T + 6] = q2[1];
            d[a * T + 7] = q1;
        }
        if (ownok != (1u << M) - 1u) {
#pragma unroll
            for (int a = 0; a < T; ++a)
#pragma unroll
                for (int j = 0; j < M; ++j)
                    if (!((ownok >> j) & 1u)) d[a * T + 1 + j] = 0.0f;
        }
    }
};

// Stage 1: the workgroup's 256 threads are 16 tiles x 16 channels (the producer
// mapping of the fused kernel: lane%16 = tile, so the row-vector loader's DPP halo
// exchange applies); each transforms its tile and stores one float4 per four
// frequencies.  Workgroups are numbered tile block fastest within a channel group
// and XCD-contiguously, so the input rows shared by vertically adjacent tiles
// (the two overlap rows of the windows) are read from HBM once and then from L2.
template <int M, bool VX>
__global__ void __launch_bounds__(256) input_transform_kernel(const float *__restrict__ x,
                                                              floatx4 *__restrict__ U, Geometry g) {
    constexpr int T2 = (M + 2) * (M + 2);
    const int tid = threadIdx.x, lane = tid & 63;
    const int tr = tid & 15, cl = tid >> 4;
    const int TB = g.tiles_p / 16;
    const int lb = xcd_contiguous_block(blockIdx.x, gridDim.x);
    const int tb = lb % TB, c = (lb / TB) * 16 + cl;
    if (c >= g.Cs * 4) return;  // past the last 4-channel step
    const TileIdx ti = decode_tile(g, tb * 16 + tr);
    const long long HW = (long long)g.H * g.W;
    const int32x4 rs = make_rsrc(x, (unsigned)((long long)g.N * g.C * HW * 4));
    float d[T2];
    if constexpr (VX && M == 7) {
        WideRowTile<M> ld;
        ld.init(g, ti, c);
        ld.load(rs, d);
    } else if constexpr (VX) {
        RowTile<M> ld;
        TileIdx rf, rl;
        row_edges<1>(g, tb * 16, tr, rf, rl);
        ld.init(g, ti, rf, rl, c, tr);
        ld.issue(rs, d);
        RowTile<M>::finish(d, ld.flags(), (g.W % M) != 0);
    } else {
        BufTile<M, (M <= 2)> ld;
        ld.init(g, ti, c);
        ld.load(rs, d);
    }
    if (c >= g.C) {  // channel padding (its loads read another channel's plane)
#pragma unroll
        for (int f = 0; f < T2; ++f) d[f] = 0.0f;
    }
    floatx4 *dst = U + ((long long)tb * g.Cs + (c >> 2)) * 64 + lane;
    const long long fstride = (long long)TB * g.Cs * 64;
    input_tile_transform_emit<M>(d, [&](int f4, float a, float b, float cc, float e) {
        dst[f4 * fstride] = floatx4{a, b, cc, e};
    });
}

// Buffer-unit copy from memory straight into LDS (gfx950: `buffer_load_dwordx4 ...
// lds`): lane l's `size` bytes at voffset + soffset of the resource land at byte
// size * l of the wave-uniform LDS address lds.  No registers hold the data; its
// completion is counted by vmcnt like any load.
typedef __attribute__((address_space(3))) void *lds_void_ptr;
__device__ void buffer_load_lds(int32x4 rsrc, lds_void_ptr lds, int size, unsigned voffset, unsigned soffset,
                                int offset, int aux) __asm("llvm.amdgcn.raw.buffer.load.lds");
template <class P>
__device__ __forceinline__ lds_void_ptr lds_ptr(P *p) {
    return (lds_void_ptr)(p);
}
// Waits until at most N vector-memory accesses of this wave are outstanding (other
// counters untouched).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}
// Workgroup barrier with no memory wait of its own (the caller has waited for what
// it needs); also a compiler barrier, so no LDS access moves across it.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_barrier" ::: "memory"); }

// v at the scale of the split products, in a register of its own, so that loads into v's
// can be issued and a loop needs no copies (and waits for them) at its end.
__device__ __forceinline__ float taken_scaled(float v) {
    float r;
    asm volatile("v_mul_f32 %0, %1, %2" : "=v"(r) : "s"(kSplitScale), "v"(v));
    return r;
}

// LDS ring depth of the three-stage product kernel, in channel steps of 8 KB
// (measured: 3 steps is 1-6 % faster than 4-6 on the deep layers, equal on the
// others).
constexpr int kGemmSteps = 3;

// Stage 2: per workgroup four frequencies (one float4 of operands) x 4 tile blocks
// x 4 output blocks (64 tiles x 64 output channels); each of the 4 waves
// multiplies 2 tile blocks by 2 output blocks for the 4 frequencies (16 matrix
// products per 4-channel step).  A channel step's operands -- 4 KB of W' and 4 KB
// of U, each 1 KB block already in matrix-core lane order -- are copied straight
// from memory into an LDS ring of NS steps by the buffer unit (no registers), one
// W' block and one U block per wave, NS - 1 steps ahead of the products; each
// wave then reads its 2 + 2 blocks from LDS, so every operand crosses L2 once per
// workgroup.  Workgroups are numbered so that the output groups of one tile group
// are consecutive on one XCD (workgroup b runs on XCD b % 8), so the tile group's
// U is read from HBM once and then from that XCD's L2.
template <int M>
__global__ void __launch_bounds__(256) frequency_gemm_kernel(const floatx4 *__restrict__ U,
                                                             const floatx4 *__restrict__ wt,
                                                             floatx4 *__restrict__ Mout, Geometry g) {
    constexpr int Q = freq_quads<M>();
    constexpr int NS = kGemmSteps;
    __shared__ floatx4 ring[NS][8][64];  // per step: W' blocks 0..3, then U blocks 0..3
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int TB = g.tiles_p / 16, TG = TB / 4, KG = g.Kb_alloc / 4;
    const int lb = xcd_contiguous_block(blockIdx.x, gridDim.x);
    const int kg = lb % KG, rest = lb / KG;
    const int tg = rest % TG, f4 = rest / TG;
    const int Cs = g.Cs;
    // The blocks this wave copies: output block 4 kg + wave of W', tile block
    // 4 tg + wave of U; step cs at byte offset cs * Q KB (W') or cs KB (U).
    const floatx4 *abase = wt + ((long long)(kg * 4 + wave) * Cs * Q + f4) * 64;
    const floatx4 *bbase = U + (((long long)f4 * TB + tg * 4 + wave) * Cs) * 64;
    const int32x4 ar = make_rsrc_uniform(reinterpret_cast<const float *>(abase),
                                         (unsigned)(Cs - 1) * Q * 1024u + 1024u);
    const int32x4 br = make_rsrc_uniform(reinterpret_cast<const float *>(bbase), (unsigned)Cs * 1024u);
    const unsigned vo = (unsigned)lane * 16u;
    // Steps past the last are clamped to it (the copies stay in bounds and every
    // iteration issues the same number, which the vmcnt wait below relies on).
    auto issue = [&](int st) {
        const unsigned c = (unsigned)(st < Cs ? st : Cs - 1);
        floatx4 *slot = ring[st % NS][0];
        buffer_load_lds(ar, lds_ptr(slot + wave * 64), 16, vo, c * Q * 1024u, 0, 0);
        buffer_load_lds(br, lds_ptr(slot + (4 + wave) * 64), 16, vo, c * 1024u, 0, 0);
    };
    floatx4 acc[2][2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[i][j][q] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int st = 0; st < NS - 1; ++st) issue(st);
    const int ai = (wave & 1) * 2, bj = 4 + (wave >> 1) * 2;
    for (int cs = 0; cs < Cs; ++cs) {
        // This wave's copies of step cs are complete once at most the 2 (NS - 2)
        // copies issued after them are outstanding; the barrier then makes every
        // wave's copies of step cs visible, and tells that every wave has read
        // step cs - 1, whose slot the next copies overwrite.
        wait_vmcnt<2 * (NS - 2)>();
        lds_barrier();
        issue(cs + NS - 1);
        const floatx4(*sl)[64] = ring[cs % NS];
        floatx4 a[2], b[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) a[i] = sl[ai + i][lane];
#pragma unroll
        for (int j = 0; j < 2; ++j) b[j] = sl[bj + j][lane];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][q], b[j][q], acc[i][j][q], 0, 0, 0);
    }
    // The copies issued past the last step (clamped repeats of it) must land
    // before the workgroup ends and its LDS can be given to another workgroup.
    wait_vmcnt<0>();
    // M: one float4 (4 frequencies) per lane and (tile block, output block, v)
    const int kb0 = kg * 4 + (wave & 1) * 2, tb0 = tg * 4 + (wave >> 1) * 2;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                Mout[((((long long)f4 * TB + tb0 + j) * g.Kb_alloc + kb0 + i) * 4 + v) * 64 + lane] =
                    floatx4{acc[i][j][0][v], acc[i][j][1][v], acc[i][j][2][v], acc[i][j][3][v]};
}

// Stage 2 with split products (wino_split.h; kernels transformed by
// weight_transform_split_kernel): per workgroup the same 64 tiles x 64 output channels
// of four frequencies, in steps of 16 channels.  Each of the 4 waves takes 32 tiles and
// 2 of the frequencies for all 64 output channels, so that it splits each of its
// transformed inputs once (56 vector instructions a step beside 24 matrix products of
// 32 cycles).  The kernels of a step, 24 KB, are copied into one of two LDS buffers
// by the buffer unit while the other is multiplied, each 1 KB already one operand
// term in lane order; the transformed inputs go to registers, one step ahead.  Bound:
// the 56 vector-memory instructions a workgroup and step (16 cycles each) about
// balance its 768 cycles of products per SIMD.  Measured on the 14x14 C = K = 512
// layer at F(7): 80 us (fp32 products 105), 64 us without its loads and 66 with a sixth
// of its products; three LDS buffers and two workgroups per compute unit 86 us.
template <int M>
__global__ void __launch_bounds__(256, 3) frequency_gemm_split_kernel(const float *__restrict__ U,
                                                                      const unsigned char *__restrict__ wt,
                                                                      float *__restrict__ Mout, Geometry g) {
    constexpr int T2 = (M + 2) * (M + 2);
    __shared__ uintx4 ring[2][24][64];  // per buffer: [output block][frequency][term]
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int TB = g.tiles_p / 16, TG = TB / 4, KG = g.Kb_alloc / 4;
    const int lb = xcd_contiguous_block(blockIdx.x, gridDim.x);
    const int kg = lb % KG, rest = lb / KG;
    const int tg = rest % TG, f4 = rest / TG;
    const int Cs = g.Cs, steps = (g.C + 15) / 16;
    const int th = wave & 1, fp = wave >> 1;
    const unsigned stepb = (unsigned)T2 * kSplitOperandBytes;
    // kernels: chunk 6 wave + j of a step is block kb, frequency fi, term t (the last
    // group's frequencies past T^2 repeat the last one: their inputs are zero)
    const int kb = wave >> 1;
    const int32x4 ar = make_rsrc_uniform(
        reinterpret_cast<const float *>(wt + (size_t)(kg * 2 + kb) * (size_t)steps * stepb), (unsigned)steps * stepb);
    const unsigned vo = (unsigned)lane * 16u;
    auto copy = [&](int st, int slot) {
#pragma unroll
        for (int j = 0; j < 6; ++j) {
            const int fi = (wave & 1) * 2 + j / 3, t = j % 3;
            const int f = 4 * f4 + fi < T2 ? 4 * f4 + fi : T2 - 1;
            buffer_load_lds(ar, lds_ptr(&ring[slot][kb * 12 + fi * 3 + t][0]), 16, vo,
                            (unsigned)st * stepb + (unsigned)f * kSplitOperandBytes + t * 1024u, 0, 0);
        }
    };
    // inputs: lane = tile 32 th + lane % 32, channels 8 (lane / 32) .. + 7 of a step
    const int32x4 br = make_rsrc_uniform(U + ((long long)f4 * TB + tg * 4) * Cs * 256, 4u * (unsigned)Cs * 1024u);
    const unsigned bo = ((unsigned)(2 * th + ((lane >> 4) & 1)) * (unsigned)Cs + 2u * (lane >> 5)) * 1024u +
                        (unsigned)(lane & 15) * 16u + (unsigned)fp * 8u;
    auto fetch = [&](int st, floatx2 (&raw)[8]) WS_INLINE {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            // channel steps past the last read as zero
            const bool in = 4 * st + 2 * (lane >> 5) + q < Cs;
            const unsigned o = in ? bo + (unsigned)(4 * st + q) * 1024u : kOutside;
#pragma unroll
            for (int j = 0; j < 4; ++j) raw[4 * q + j] = buffer_load_f32x2(br, o + 256u * j, 0, 0);
        }
    };
    floatx16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int k = 0; k < 2; ++k) acc[i][k] = floatx16{};
    floatx2 raw[8];
    copy(0, 0);
    fetch(0, raw);
    for (int st = 0; st < steps; ++st) {
        // this step's kernels and inputs have arrived; behind the barrier every wave's,
        // and every wave has multiplied the step before, whose buffer the next copies use
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        floatx4 r[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                r[i][q] = floatx4{taken_scaled(raw[4 * q][i]), taken_scaled(raw[4 * q + 1][i]), taken_scaled(raw[4 * q + 2][i]),
                                  taken_scaled(raw[4 * q + 3][i])};
            }
        // past the end the last step's copies and loads again: nobody reads them
        const int nx = st + 1 < steps ? st + 1 : st;
        copy(nx, (st + 1) & 1);
        fetch(nx, raw);
        __builtin_amdgcn_sched_barrier(0);
        const uintx4(*sl)[64] = ring[st & 1];
        SplitOperand b[2], a[2];
        auto operand = [&](int u) WS_INLINE {  // unit u: frequency 2 fp + u / 2, output block u % 2
#pragma unroll
            for (int t = 0; t < 3; ++t) a[u & 1].t[t] = sl[(u & 1) * 12 + (2 * fp + u / 2) * 3 + t][lane];
        };
        operand(0);
#pragma unroll
        for (int s = 0; s < 5; ++s) split_step(s, r[0], b[0]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (u + 1 < 4) operand(u + 1);
#pragma unroll
            for (int n = 0; n < 6; ++n) {
                const int at = n == 0 ? 2 : n < 3 ? 1 : 0, bt = n == 1 ? 1 : n == 3 ? 2 : n == 4 ? 1 : 0;
                acc[u / 2][u % 2] = mfma_bf16(a[u & 1].t[at], b[u / 2].t[bt], acc[u / 2][u % 2]);
                if (u < 2 && n < 5 && (n & 1) == u % 2) split_step(u == 0 ? n / 2 : 3 + n / 2, r[1], b[1]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    // the copies issued with the last step must land before the workgroup ends and its
    // LDS can be given to another workgroup
    wait_vmcnt<0>();
    const int tb = tg * 4 + 2 * th + ((lane >> 4) & 1);
    // M of the lane's element v of output block k
    auto out = [&](int k, int v) {
        const int kb16 = kg * 4 + 2 * k + v / 8, l16 = (2 * ((v / 4) & 1) + (lane >> 5)) * 16 + (lane & 15);
        return Mout + (((((long long)f4 * TB + tb) * g.Kb_alloc + kb16) * 4 + v % 4) * 64 + l16) * 4 + 2 * fp;
    };
    // a frequency past T^2 (the wave's second one only) is zero, whatever the kernels repeated for it hold
    const int f0 = 4 * f4 + 2 * fp, nf = T2 % 4 == 0 || T2 - f0 >= 2 ? 2 : T2 - f0 < 0 ? 0 : T2 - f0;
    float sum[4] = {};  // of the results: not finite if one of them is not
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            floatx2 r;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                r[i] = i < nf ? acc[i][k][v] * kSplitUnscale : 0.0f;
                sum[v % 4] += acc[i][k][v];
            }
            *reinterpret_cast<floatx2 *>(out(k, v)) = r;
        }
    // Sums beyond the scaled range (or of infinities) again, as fp32 products: the lane's
    // element of each of its tiles' frequencies straight from U and the kernels.
    if (__builtin_amdgcn_ballot_w64(!finite((sum[0] + sum[1]) + (sum[2] + sum[3]))) == 0) return;
    unsigned again[2] = {0u, 0u};  // bit 16 k + v
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int n = 0; n < 32; ++n) again[i] |= (i < nf && !finite(acc[i][n / 16][n % 16])) ? 1u << n : 0u;
    const float *ub = U + (((long long)f4 * TB + tb) * Cs * 64 + (lane & 15)) * 4 + 2 * fp;
    for (int i = 0; i < 2; ++i)
        for (int n = 0; n < 32; ++n) {
            if (!((again[i] >> n) & 1u)) continue;
            const int k = kg * 64 + (n / 16) * 32 + ((n % 16) / 8) * 16 + (2 * ((n / 4) & 1) + (lane >> 5)) * 4 + n % 4;
            float m = 0.0f;
            for (int cs = 0; cs < Cs * 4; cs += 16) {  // 16 channels on their own, as the matrix products add them
                float part = 0.0f;
                for (int c = cs; c < Cs * 4 && c < cs + 16; ++c)
                    part = __builtin_fmaf(split_kernel_value<M>(wt, steps, k, c, f0 + i),
                                          ub[((c >> 2) * 64 + (c & 3) * 16) * 4 + i], part);
                m += part;
            }
            out(n / 16, n % 16)[i] = m;
        }
}

// Stage 3: the workgroup's 4 waves are the four v of one (tile block, output
// block): lane = 16 * q + tile%16 with output channel k = 16 kb + 4 q + v, so a
// wave reads one 1 KB float4 row of M per four frequencies.
template <int M>
__global__ void __launch_bounds__(256) output_transform_kernel(const floatx4 *__restrict__ Min,
                                                               float *__restrict__ y, Geometry g) {
    constexpr int T2 = (M + 2) * (M + 2), Q = freq_quads<M>();
    const int lane = threadIdx.x & 63, v = threadIdx.x >> 6;
    const int tb = blockIdx.x, kb = blockIdx.y;
    const int TB = g.tiles_p / 16;
    const int tile = tb * 16 + (lane & 15), k = kb * 16 + (lane >> 4) * 4 + v;
    const floatx4 *src = Min + (((long long)tb * g.Kb_alloc + kb) * 4 + v) * 64 + lane;
    const long long fstride = (long long)TB * g.Kb_alloc * 4 * 64;
    float mm[4 * Q];
#pragma unroll
    for (int f4 = 0; f4 < Q; ++f4) {
        const floatx4 q4 = src[f4 * fstride];
#pragma unroll
        for (int e = 0; e < 4; ++e) mm[4 * f4 + e] = q4[e];
    }
    if (tile >= g.ntiles || k >= g.K) return;
    const TileIdx ti = decode_tile(g, tile);
    float yy[M * M];
    output_tile_transform<M>(mm, yy);
    (void)T2;
    if constexpr (M % 2 == 1) {
        // odd m: rows of tiles whose m columns lie inside the image are stored as
        // 4-byte-aligned vector pieces (y is below 2^31 bytes), rows below the
        // image skipped, the rows of tiles cut by the right edge element by element
        const int h0 = ti.ty * M, w0 = ti.tx * M;
        const bool fullw = w0 + M <= g.W;
        const int32x4 yrs = make_rsrc(y, (unsigned)((long long)g.N * g.K * g.H * g.W * 4));
        const unsigned vb = (unsigned)(((((long long)ti.n * g.K + k) * g.H + h0) * g.W + w0) * 4);
        float *yp = y + ((long long)ti.n * g.K + k) * g.H * g.W;
#pragma unroll
        for (int i = 0; i < M; ++i) {
            if (h0 + i >= g.H) break;
            if (fullw) {
                store_row_buf<M, false>(yrs, vb, (unsigned)i * (unsigned)g.W * 4u, yy + i * M);
            } else {
#pragma unroll
                for (int jj = 0; jj < M; ++jj)
                    if (w0 + jj < g.W) yp[(long long)(h0 + i) * g.W + w0 + jj] = yy[i * M + jj];
            }
        }
        return;
    }
    const bool vec = (M == 4) ? (g.W % 4 == 0 && (reinterpret_cast<uintptr_t>(y) & 15) == 0)
                              : (g.W % 2 == 0 && (reinterpret_cast<uintptr_t>(y) & 7) == 0);
    store_tile<M>(y + ((long long)ti.n * g.K + k) * g.H * g.W, yy, ti.ty * M, ti.tx * M, g, vec);
}

// ---------------------------------------------------------------------------
// Launchers.

// Tile sizes of the kernel transform and the three-stage kernels: the fused
// kernel's and F(7x7,3x3) (T = 9: its 21 float4s of frequencies per tile and
// channel exceed the fused kernel's LDS stage ring).
#define WINO_DISPATCH_M(m, CALL)          \
    switch (m) {                          \
        case 2: { constexpr int MM = 2; CALL; } break; \
        case 4: { constexpr int MM = 4; CALL; } break; \
        case 5: { constexpr int MM = 5; CALL; } break; \
        case 6: { constexpr int MM = 6; CALL; } break; \
        case 7: { constexpr int MM = 7; CALL; } break; \
        default: return hipErrorInvalidValue; \
    }

hipError_t launch_weight_transform(const Geometry &g, const float *w, float *wt, hipStream_t s,
                                   unsigned *zero, int nzero) {
    const long long total = (long long)g.Kb_alloc * g.Cs * 64;
    dim3 block(256), grid((unsigned)((total + 255) / 256));
    WINO_DISPATCH_M(g.m, hipLaunchKernelGGL(weight_transform_kernel<MM>, grid, block, 0, s, w,
                                            reinterpret_cast<floatx4 *>(wt), g, zero, nzero));
    return hipGetLastError();
}

hipError_t launch_weight_transform_split(const Geometry &g, const float *w, float *wt, hipStream_t s,
                                         unsigned *zero, int nzero) {
    const unsigned nx = (unsigned)(g.Kb_alloc / 2 * ((g.C + 15) / 16));
    auto go = [&](auto kern, int fch) {
        hipLaunchKernelGGL(kern, dim3(nx, (unsigned)((g.T2 + fch - 1) / fch)), dim3(512), 0, s, w,
                           reinterpret_cast<uintx4 *>(wt), g, zero, nzero);
    };
    if (nx * (unsigned)((g.T2 + 15) / 16) <= 64u) {
        WINO_DISPATCH_M(g.m, go(weight_transform_split_kernel<MM, 4>, 4));
    } else if (nx * (unsigned)((g.T2 + 15) / 16) <= 128u) {
        WINO_DISPATCH_M(g.m, go(weight_transform_split_kernel<MM, 8>, 8));
    } else {
        WINO_DISPATCH_M(g.m, go(weight_transform_split_kernel<MM, 16>, 16));
    }
    return hipGetLastError();
}

void unsplit_weights(const Geometry &g, const unsigned short *split, float *out, size_t count) {
    const int cs16 = (g.C + 15) / 16, Q = (g.T2 + 3) / 4;
    for (size_t i = 0; i < count; ++i) {
        const int f4 = (int)(i & 3), lane = (int)(i >> 2 & 63);
        const size_t grp = i >> 8;
        const int f = (int)(grp % Q) * 4 + f4, cs = (int)(grp / Q % g.Cs), kb = (int)(grp / Q / g.Cs);
        const int c = cs * 4 + (lane >> 4), k = kb * 16 + (lane & 15);
        if (f >= g.T2) {
            out[i] = 0.0f;
            continue;
        }
        const unsigned short *p = split + (((size_t)(k / 32) * cs16 + c / 16) * g.T2 + f) * 1536 +
                                  ((c % 16 / 8) * 32 + k % 32) * 8 + c % 8;
        out[i] = split_value(p[0], p[512], p[1024]);
    }
}

bool fused_blocking_built(int m, int R, int kit) {
    for (const FusedBlocking &b : kFusedBlockings)
        if (b.m == m && b.R == R && b.kit == kit) return true;
    return false;
}

// Whether a layer runs on the split-product kernel (wino_split.h).  Its tasks are two
// to four times the fp32 kernel's, so a layer needs enough of them.  Measured against
// the fp32 kernel (us per call, C = K):
//  * F(4) to F(6) from 80 tasks (5/16 of the compute units): F(4) 40 images of 14 x
//    14, 256 channels, 80 tasks 80.4 -> 45.6, 32 of 224 x 224, 64 channels 373 -> 313;
//    F(5) 32 of 28 x 28, 256 channels, 288 tasks 148 -> 127; F(6) 32 of 112 x 112, 128
//    channels, 1444 tasks 405 -> 374.  At 50 tasks of 4 or 8 stages 0.64-0.94 times as
//    fast, as the fp32 kernel's smaller tasks then fit one round.
//  * Tasks cut into pieces from more than 64 (1/4) at 6 stages: F(5) 16 images of 28 x
//    28, 128 channels, 72 tasks 48.1 -> 36.0, F(6) 4 of 75 x 53, C = 96, K = 160, 75
//    tasks 67.8 -> 38.0; and from 32 (1/8) at 16 stages: 64 images of 7 x 7, 512
//    channels, F(4) 64 tasks 114 -> 58; 16 of 14 x 14, 256 channels, F(4) 32 tasks
//    39.5 -> 35.8; F(6) 40 tasks 53.4 -> 44.4.  Below, 8 to 28 tasks: 0.86-1.08 times.
//  * F(2) from 48 (3/16): 3 images of 56 x 56, 64 channels, 74 tasks 14.5 -> 12.9, at 49 12.4
//    against 12.8 (12.3 before it added stages on their own, below), at 25 0.73 times.
// Output channels that pad a task count as no work (K = 32, 98 half-empty tasks at F(4):
// 0.79 times), F(5), whose gain is the smallest, takes at most a quarter of them (19
// images of 56 x 56, C = 33, K = 65: 39.4 us against 42.0), and one stage of channels,
// C <= 16, is left to the fp32 kernel, whose task has the shorter epilogue (32 images of
// 112 x 112, C = 3, K = 64: 37.6 us against 41.7).  The transformed kernels take up to 2.4 times the fp32 kernel's (6 bytes a
// value, channels padded to 16); those of one task are addressed with 32-bit byte
// offsets, which 64 output channels at F(4) exceed from 310,000 input channels on.
template <int M>
static bool split_enough(const Geometry &g, int num_cus) {
    using S = SplitShape<M>;
    const SplitInfo si = split_kernel_info<M>(g, num_cus);
    if (M == 5 && 4 * g.K < 3 * si.n_kgroups * S::KIT) return false;
    const double items = (double)si.n_items * g.K / (si.n_kgroups * S::KIT);
    if (16.0 * items >= (M == 2 ? 3.0 : 5.0) * num_cus) return true;
    if (M == 2 || si.n_tail == 0) return false;
    return (si.stages >= 6 && 4.0 * items > num_cus) || (si.stages >= 16 && 8.0 * items >= num_cus);
}
// Whether the fp32 kernel at its own blocking is the faster one although split_enough says
// yes: it runs tasks of half the size, so that a layer may fill its rounds and leave half
// of this kernel's units idle.  Times are estimated as rounds x (channel slope x channels +
// output transform) + launch, in us, fitted to 74 layers of 32 to 512 channels that fill one
// to four rounds of the fp32 kernel exactly (64 to 256 images of 32 x 32 at F(4), 32 to 128 of
// 40 x 40 at F(5) and of 48 x 48 at F(6)); the estimates lie within 8%.  Rows that end inside
// a tile cost the fp32 kernel its wide stores: 64 images of 32 x 30 at F(4) take 26.8 us for
// 19.2, 32 of 40 x 37 at F(5) 23.3 for 20.4, of 48 x 46 and 48 x 45 at F(6) 27.6 and 34.4 for
// 25.0; rows that are missing at the bottom cost it nothing.  Measured, one full round: F(4)
// 64 channels 19.3 us against 24.1, F(5) 20.4 against 29.0, F(6) 25.0 against 36.2, 192
// channels F(4) 44.0 -> 43.2, F(5) 41.9 against 46.5, F(6) 50.0 against 57.2; two: F(4) 64
// channels 33.7 -> 28.2, F(5) 33.4 -> 31.0, F(6) 41.5 -> 39.6; three: F(4) 32 channels 27.6 against
// 31.3, F(5) 64 46.5 against 51.7, F(6) 57.4 against 66.7; many: 32 channels, 512 of 48 x 48
// F(6) 159 against 168, 17 channels, 1 of 2040 x 2040 F(4) 1040 against 1108.  F(2): one
// full round of tasks smaller than this kernel's, 8 images of 32 x 32, 64 channels 8.9
// against 12.6, 160 channels 15.7 against 16.4, 192 17.3 -> 16.8.  F(5) and F(6) outputs of
// 128 MiB and more in whole tiles whose rows are no multiple of 32 and 64 bytes cost this
// kernel, which has more stores in flight, a further 3 and 5 a round: C = K = 64, 304 images of
// 45 x 45 F(5) 179 against 194, 60 of 102 x 102 F(6) 171 against 186, 22 of 168 x 168 155
// against 176; aligned 24 of 160 x 160 F(5) 161 -> 141, 67 of 96 x 96 F(6) 149 -> 148.
static bool fp32_rounds_better(const Geometry &g, int num_cus) {
    const FusedCfg f = fused_cfg_default(g, num_cus, FusedKernel::kFp32);
    const SplitInfo si = fused_split_info(g, FusedCfg{0, 0, num_cus, 0, true, false});
    const int items = fused_split_info(g, f).n_items;
    if (g.m == 2) return items == num_cus && f.R * f.kit < 32 * 64 && si.stages <= 11;
    if (f.kit != (g.m == 4 ? 64 : 32)) return false;
    struct Cost {
        double slope, round, launch, piece, part;  // part: share of a round that a last one of whole items takes
    };
    const Cost cf = g.m == 4   ? Cost{0.196, 1.9, 4.8, 0, 1}
                    : g.m == 5 ? Cost{0.183, 1.5, 7.0, 0, 1}
                               : Cost{0.203, 3.1, 8.7, 0, 1};
    const Cost cs = g.m == 4   ? Cost{0.240, 9.5, 3.0, 7.7, 0.8}
                    : g.m == 5 ? Cost{0.288, 5.9, 6.5, 6.4, 0.85}
                               : Cost{0.333, 10.0, 8.0, 7.0, 0.85};
    const double C = 16.0 * si.stages, rounds = (items + num_cus - 1) / num_cus;
    const double ragged = g.W % g.m == 0 ? 0 : g.m == 4 ? 7.0 : g.m == 5 ? 2.9 : g.W % 2 == 0 ? 2.6 : 10.0;
    const double tf = cf.launch + rounds * (cf.slope * C + cf.round + ragged);
    const bool large = (long long)g.N * g.K * g.H * g.W * 4 >= kStreamOutputBytes && g.W % g.m == 0;
    const double round = cs.round + (!large ? 0 : g.m == 5 && g.W % 8 != 0 ? 3.0 : g.m == 6 && g.W % 16 != 0 ? 5.0 : 0);
    const int tail = si.n_items % num_cus;
    double ts = cs.launch + si.nfull * (cs.slope * C + round);
    if (si.n_tail > 0) ts += cs.slope * 16.0 * si.piece + round + cs.piece;
    else if (tail > 0) ts += (2 * tail <= num_cus ? cs.part : 1.0) * (cs.slope * C + round);
    return tf < 0.96 * ts;
}
static bool split_fits(const Geometry &g, int num_cus) {
    if (!split_possible(g) || fp32_rounds_better(g, num_cus)) return false;
#define WINO_SPLIT_ENOUGH(m_) \
    if (g.m == m_) return split_enough<m_>(g, num_cus);
    WINO_SPLIT_M(WINO_SPLIT_ENOUGH)
#undef WINO_SPLIT_ENOUGH
    return false;
}
bool split_possible(const Geometry &g) {
#define WINO_SPLIT_POSSIBLE(m_)                                                                                \
    if (g.m == m_) {                                                                                           \
        using S = SplitShape<m_>;                                                                              \
        const unsigned long long stages = (g.C + S::CC - 1) / S::CC;                                           \
        return stages > 1 && (S::KB * stages * S::T2 * kSplitOperandBytes >> 32) == 0;                         \
    }
    WINO_SPLIT_M(WINO_SPLIT_POSSIBLE)
#undef WINO_SPLIT_POSSIBLE
    return false;
}
// The split-product kernel's configuration (R = 0), or of the fp32 kernel (R > 0).
// Precision: where the fp32 kernel would run at a blocking that adds two halves of the
// channels (layers too small for its larger tasks), its error is 4 to 12% below that of this
// kernel's single sums from three stages on.  There F(2) and F(4) add stages on their own
// (SplitShape; error 0.72-0.85 of the fp32 kernel's; F(2) 4 images of 56 x 56, 64 channels
// 12.4 -> 13.0 us, fp32 kernel 14.7; F(4) 20 of 46 x 46 22.9 -> 24.5, fp32 34.1), F(5) and F(6)
// cut their items into two and more pieces (0.72-0.86; F(6) 34.1 -> 33.5, fp32 40.9; F(5)
// 29.8 -> 29.9, fp32 31.8), and F(5) of three stages, which that makes slower than the fp32
// kernel (29.3 against 27.2), is left to it.
static bool split_cfg(const Geometry &g, int num_cus, FusedKernel kernel, FusedCfg *cfg) {
    if (kernel == FusedKernel::kFp32 || !split_possible(g)) return false;
    if (kernel == FusedKernel::kByRule && !split_fits(g, num_cus)) return false;
    *cfg = FusedCfg{0, 0, num_cus, 0, true, false};
    const SplitInfo si = fused_split_info(g, *cfg);
    if (si.stages < 3 || si.n_tail > 0) return true;
    const FusedCfg f = fused_cfg_default(g, num_cus, FusedKernel::kFp32);
    bool halves = false;
    for (const FusedBlocking &b : kFusedBlockings)
        if (b.m == g.m && b.R == f.R && b.kit == f.kit) halves = b.csp == 2;
    if (halves && g.m > 4) return false;
    cfg->own = halves;
    return true;
}

// Default blocking of a layer, from the capacity bounds of Sec. 4.1 and the
// number of work items.
//  * Capacity: a task's result matrices (R tiles x Kit output channels x T^2
//    frequencies) live in the consumer waves' registers, at most 144 per lane of
//    four waves: R * Kit * T^2 <= 36864.  F(2), F(4): Kit <= 64 (R = 32 only for
//    F(2)); F(5), F(6): R = 16, Kit <= 32.
//  * Reuse: every transformed input tile is multiplied by the Kit output
//    channels' kernels (the input-transform work per product falls as 1 / Kit)
//    and every transformed-kernel operand read from L2 by the R tiles (the
//    paper's task arithmetic intensity against the shared cache, R / 2).  So the
//    largest task that fits is taken: Kit at its maximum; R = 32 for F(2) when C
//    <= 64 (measured: with more channels the 16-channel stages of R = 16 run
//    faster), else 16 ...
//  * ... as long as the layer has at least one task per compute unit.  A layer
//    with fewer takes the blocking with the most tasks instead (smaller Kit,
//    then smaller R): on the N=1, 56x56, C=K=64 layer at F(2) 196 tasks of 16 x
//    16 run in 8.4 us against 14.8 us for 25 tasks of 32 x 64.
// Measured on every layer (steady state, one MI355X): splitting a task's output
// channels among its consumer waves costs more than the transform reuse it gives
// up whenever the larger tasks already fill the compute units.
FusedCfg fused_cfg_default(const Geometry &g, int num_cus, FusedKernel kernel, int want_R, int want_kit) {
    FusedCfg best{};
    if (split_cfg(g, num_cus, kernel, &best)) return best;
    best = FusedCfg{};
    int best_items = -1;
    bool best_fills = false;
    const int pref_R = (g.m == 2 && g.C <= 64) ? 32 : 16;
    for (const FusedBlocking &b : kFusedBlockings) {
        if (b.m != g.m || (want_R && b.R != want_R) || (want_kit && b.kit != want_kit)) continue;
        const FusedCfg c{b.R, b.kit, num_cus, 0, false, false};
        const int items = fused_split_info(g, c).n_items;
        const bool fills = items >= num_cus;
        bool take;
        if (best.R == 0) take = true;
        else if (fills != best_fills) take = fills;
        else if (fills) {
            // both fill the units: the largest task, R = pref_R first
            const bool bp = best.R == pref_R, cp = b.R == pref_R;
            take = b.kit > best.kit || (b.kit == best.kit && cp && !bp);
        } else {
            // neither fills the units: the most tasks
            take = items > best_items;
        }
        if (take) {
            best = c;
            best_items = items;
            best_fills = fills;
        }
    }
    return best;
}

SplitInfo fused_split_info(const Geometry &g, const FusedCfg &cfg) {
    if (cfg.split) {
#define WINO_INFO_SPLIT(m_) \
    if (g.m == m_) return split_kernel_info<m_>(g, cfg.num_cus);
        WINO_SPLIT_M(WINO_INFO_SPLIT)
#undef WINO_INFO_SPLIT
    }
#define WINO_SPLIT_WS(m_, R_, kit_, tb, fs, csp) \
    if (g.m == m_ && cfg.R == R_ && cfg.kit == kit_) return ws_split_info<m_, tb, fs, csp>(g, cfg.num_cus, cfg.csplit);
    WINO_FUSED_BLOCKINGS(WINO_SPLIT_WS)
#undef WINO_SPLIT_WS
    return SplitInfo{};
}

void describe_fused(const Geometry &g, const FusedCfg &cfg, char *buf, size_t len) {
    const SplitInfo si = fused_split_info(g, cfg);
    if (cfg.split) {
        snprintf(buf, len,
                 "fused_ws_kernel<M=%d,split products> R=%d tiles x Kit=%d output channels per item, 16 input channels per "
                 "stage, %d items (%d tile groups x %d channel groups), %d stages per item, grid %d, split items %d "
                 "x %d pieces%s",
                 g.m, 32, g.m <= 4 ? 64 : 32, si.n_items, si.n_items / si.n_kgroups, si.n_kgroups,
                 si.stages, si.grid, si.n_tail, si.maxc, cfg.own ? ", stages added on their own" : "");
        return;
    }
    int tb = 0, fs = 0, csp = 0;
    for (const FusedBlocking &b : kFusedBlockings)
        if (b.m == g.m && b.R == cfg.R && b.kit == cfg.kit) {
            tb = b.tb;
            fs = b.fs;
            csp = b.csp;
        }
    snprintf(buf, len,
             "fused_ws_kernel<M=%d,TB=%d,FS=%d,CSP=%d,VX,SPLIT=%d> R=%d tiles x Kit=%d output channels per "
             "item, %d input channels per stage, %d items (%d tile groups x %d channel groups), %d stages per "
             "item, grid %d, split items %d x %d pieces",
             g.m, tb, fs, csp, si.n_tail > 0 ? 1 : 0, cfg.R, cfg.kit, 256 / cfg.R, si.n_items,
             si.n_kgroups > 0 ? si.n_items / si.n_kgroups : 0, si.n_kgroups, si.stages, si.grid, si.n_tail, si.maxc);
}

hipError_t launch_fused(const Geometry &g, const FusedCfg &cfg, const float *x, const float *wt,
                        float *y, const SplitBuffers &sb, hipStream_t s) {
    if (cfg.split) {
#define WINO_LAUNCH_SPLIT(m_) \
    if (g.m == m_) return launch_split_t<m_>(g, x, wt, y, cfg.num_cus, cfg.own, sb, s);
        WINO_SPLIT_M(WINO_LAUNCH_SPLIT)
#undef WINO_LAUNCH_SPLIT
        return hipErrorInvalidValue;
    }
    if (!fused_blocking_built(g.m, cfg.R, cfg.kit)) return hipErrorInvalidValue;
    const uintptr_t ya = reinterpret_cast<uintptr_t>(y);
    // rows of whole tiles stored as vectors: 16-byte aligned for m = 4, 8-byte for m =
    // 2, 6; m = 5 uses buffer stores that need only 4-byte alignment
    const bool vec = (g.m == 5) ? true
                     : (g.m == 4) ? (g.W % 4 == 0 && ya % 16 == 0) : (g.W % 2 == 0 && ya % 8 == 0);
#define WINO_LAUNCH_WS(m_, R_, kit_, tb, fs, csp)                                                         \
    if (g.m == m_ && cfg.R == R_ && cfg.kit == kit_)                                                        \
        return launch_ws_t<m_, tb, fs, csp>(g, x, wt, y, vec, cfg.num_cus, cfg.csplit, sb, s);
    WINO_FUSED_BLOCKINGS(WINO_LAUNCH_WS)
#undef WINO_LAUNCH_WS
    return hipErrorInvalidValue;
}

void describe_three_stage(const Geometry &g, bool split, char *buf, size_t len) {
    snprintf(buf, len, "input_transform_kernel<M=%d>, frequency_gemm%s_kernel<M=%d>, output_transform_kernel<M=%d>: "
             "%d tiles, U and M of %d frequencies in device memory", g.m, split ? "_split" : "", g.m, g.m, g.ntiles, g.T2);
}

hipError_t launch_input_transform(const Geometry &g, const float *x, float *U, hipStream_t s) {
    dim3 block(256), grid((unsigned)((long long)(g.tiles_p / 16) * ((g.Cs * 4 + 15) / 16)));
    // row-vector input loads need every row start aligned to the vector width
    // (m = 5, 7: 4-byte-aligned vector loads)
    const unsigned vw = (g.m == 4) ? 16u : (g.m == 5 || g.m == 7) ? 4u : 8u;
    const bool vx = (reinterpret_cast<uintptr_t>(x) % vw == 0) && ((unsigned)g.W * 4u) % vw == 0;
    floatx4 *u4 = reinterpret_cast<floatx4 *>(U);
    if (vx) {
        WINO_DISPATCH_M(g.m, hipLaunchKernelGGL((input_transform_kernel<MM, true>), grid, block, 0, s, x, u4, g));
    } else {
        WINO_DISPATCH_M(g.m, hipLaunchKernelGGL((input_transform_kernel<MM, false>), grid, block, 0, s, x, u4, g));
    }
    return hipGetLastError();
}

hipError_t launch_frequency_gemm(const Geometry &g, const float *U, const float *wt, float *Mout,
                                 hipStream_t s) {
    const long long nblk = (long long)(g.tiles_p / 64) * (g.Kb_alloc / 4) * ((g.T2 + 3) / 4);
    dim3 block(256), grid((unsigned)nblk);
    WINO_DISPATCH_M(g.m, hipLaunchKernelGGL(frequency_gemm_kernel<MM>, grid, block, 0, s,
                                            reinterpret_cast<const floatx4 *>(U),
                                            reinterpret_cast<const floatx4 *>(wt),
                                            reinterpret_cast<floatx4 *>(Mout), g));
    return hipGetLastError();
}

hipError_t launch_frequency_gemm_split(const Geometry &g, const float *U, const float *wt, float *Mout,
                                       hipStream_t s) {
    const long long nblk = (long long)(g.tiles_p / 64) * (g.Kb_alloc / 4) * ((g.T2 + 3) / 4);
    dim3 block(256), grid((unsigned)nblk);
    WINO_DISPATCH_M(g.m, hipLaunchKernelGGL(frequency_gemm_split_kernel<MM>, grid, block, 0, s, U,
                                            reinterpret_cast<const unsigned char *>(wt), Mout, g));
    return hipGetLastError();
}

// With few channels the pipeline is bound by U and M in memory, a step of 16 channels is
// partly padding and M is written in 8-byte halves: measured against the fp32 products
// 0.84-0.98 times as fast at C <= 32, 1.00-1.52 times from 80 channels on (whole pipelines,
// F(2) to F(7), 1 to 64 images, kernels ahead of time: the 14x14 C = K = 512 layer at F(7)
// 152 -> 121 us, 7x7 C = K = 512 N = 64 at F(4) 94.2 -> 61.9, 56x56 C = 80, K = 256 N = 16 F(6)
// 83.2 -> 78.1).  Between, 64 to 79 channels gain 0 to 8%, except where
//  * U and M leave the caches and few output channels reuse them: 56x56 C = K = 64 N = 32,
//    115 MB at F(4), 55.3 against 58 us, 115 at F(5) 57.0 against 57.5, 105 at F(6) 57.0
//    against 58.8 (N = 16 F(4) 33.3 -> 32.0; K = 256 N = 32 F(4) 193.9 -> 190.1);
//  * kernels are given at every call and are many for their products, as their transform
//    takes longer (6 bytes a value): C = 64, K = 256 14x14 N = 2 F(7) 24.4 against 25.3, C = 70,
//    K = 200 30x30 N = 8 F(6) 30.5 against 31.6, C = 72, K = 256 28x28 N = 8 F(4), 2.6e8
//    products, 30.2 against 31.3 (C = 64, K = 512 F(6), 4.2e8, 44.9 -> 41.2, 40x40 N = 16 F(4),
//    1.9e9, 81.1 -> 78.2; C = 64, K = 128 28x28 N = 8 F(6) 26.4 -> 26.0).
// F(7) layers of more than 256 x 256 channels keep the fp32 products up to 128 tiles, where
// the transform of the largest kernels weighs most: with kernels given 14x14 C = K = 512 N = 1
// measured 78.2 against 94.7 us, and 77.3 against 75.6 with the transform as it is now, C =
// 256, K = 512 52.8 against 54.0; kernels ahead of time would gain there (59.1 -> 47.4).
bool three_stage_split(const Geometry &g) {
    if (g.C < 64 || (g.m == 7 && g.tiles_p <= 128 && (long long)g.C * g.K > 256 * 256)) return false;
    if (g.C >= 80) return true;
    if (g.K > 2 * g.C) return (double)g.T2 * g.tiles_p * g.C * g.K >= 3e8;
    return (double)g.T2 * g.tiles_p * (g.C + g.K) * sizeof(float) <= 96e6;
}

hipError_t launch_output_transform(const Geometry &g, const float *Min, float *y, hipStream_t s) {
    dim3 block(256), grid((unsigned)(g.tiles_p / 16), (unsigned)g.Kb);
    WINO_DISPATCH_M(g.m, hipLaunchKernelGGL(output_transform_kernel<MM>, grid, block, 0, s,
                                            reinterpret_cast<const floatx4 *>(Min), y, g));
    return hipGetLastError();
}

}  // namespace wino

// FFT-tile fused 3x3 convolution for gfx950 (the FFT transform of Sec. 2.1 and
// Sec. 4 with the fusion of Sec. 3): 16x16 input tiles overlapping by 2 give
// 14x14 output tiles; a tile's spectrum is conjugate symmetric, so only the
// 16 x 9 frequencies with column index q <= 8 are kept (Sec. 2.1).
//
// Per frequency f = p*9 + q the contraction over input channels is complex:
//     Z[f][k][t] = sum_c D[f][c][t] * conj(Wp[f][k][c])
// (the convolution theorem for the cross-correlation of Eq. 1; circular on the
// 16x16 tile, equal to the linear one on the 14x14 output tile).  With
// D = Dr + i Di and Wp = Wr + i Wi:
//     Re Z = sum Wr Dr + Wi Di,   Im Z = sum Wr Di + (-Wi) Dr,
// four real products per complex one, on v_mfma_f32_16x16x4_f32 with the
// output channels as rows (operand A, from the transformed kernels) and tiles as
// columns (operand B, from LDS).
//
// Work item = 16 tiles x 16 output channels, one workgroup of 8 waves each: the
// item's 16 x 16 x 144 complex sums (1.18 MB for 64 output channels) do not fit
// a compute unit, so an item holds one 16-channel block; wave w accumulates
// frequencies 18w .. 18w + 17 (36 accumulator tiles = 144 registers).  Per
// stage of 4 input channels: the 64 input tiles are loaded into LDS, transformed
// (16-point FFTs along rows, then along the 9 kept columns), and each wave runs
// its 72 products.  After the last stage the sums go back through LDS a quarter
// of the output channels at a time for the inverse transforms.
//
// Bound by the phases of a stage one after the other (LDS fill, row and column
// transforms, 4608 cycles of products per SIMD), as one workgroup fills a compute unit.
// The two real columns (0 and 8) share one complex transform, so the column pass is one
// transform for each of the 512 threads where the ninth column took a second round of
// one wave; input addresses are formed once per item instead of per element and stage;
// input loads go out behind the kernel operands they would otherwise hold up: 64 images
// of 28 x 28, C = K = 128 236 -> 197 us.
#include "wino_internal.h"

#include <hip/hip_runtime.h>

namespace wino {

typedef float fft_floatx4 __attribute__((ext_vector_type(4)));
typedef int fft_int32x4 __attribute__((ext_vector_type(4)));

// Raw buffer loads: an offset at or past the resource's size reads 0, which
// gives the zero padding of input windows without branches.  (Declared outside
// the anonymous namespace below: they name LLVM intrinsics, which have external
// linkage.)
__device__ float fft_buffer_load_f32(fft_int32x4 rsrc, unsigned voffset, unsigned soffset, int aux)
    __asm("llvm.amdgcn.raw.buffer.load.f32");
__device__ fft_floatx4 fft_buffer_load_f32x4(fft_int32x4 rsrc, unsigned voffset, unsigned soffset, int aux)
    __asm("llvm.amdgcn.raw.buffer.load.v4f32");
__device__ void fft_raw_buffer_store_f32x4(fft_floatx4 v, fft_int32x4 rsrc, unsigned voffset, unsigned soffset, int aux)
    __asm("llvm.amdgcn.raw.buffer.store.v4f32");
// The next instruction must not overwrite the data registers of a store of more than 64
// bits; the compiler does not see to it where the scalar offset is in a register.
__device__ __forceinline__ void fft_buffer_store_f32x4(fft_floatx4 v, fft_int32x4 rsrc, unsigned voffset, unsigned soffset,
                                                       int aux) {
    fft_raw_buffer_store_f32x4(v, rsrc, voffset, soffset, aux);
    asm volatile("s_nop 0" ::"v"(v));
}
__device__ void fft_buffer_store_f32(float v, fft_int32x4 rsrc, unsigned voffset, unsigned soffset, int aux)
    __asm("llvm.amdgcn.raw.buffer.store.f32");

namespace {

typedef fft_floatx4 floatx4;
typedef fft_int32x4 int32x4;
__device__ __forceinline__ int32x4 fft_rsrc(const float *base, unsigned bytes) {
    const unsigned long long p = reinterpret_cast<unsigned long long>(base);
    int32x4 r;
    r[0] = (int)(unsigned)(p & 0xffffffffull);
    r[1] = (int)(unsigned)((p >> 32) & 0xffffull);  // stride 0
    r[2] = (int)bytes;                                 // range-checked size
    r[3] = 0x00020000;                                 // 32-bit data format
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = __builtin_amdgcn_readfirstlane(r[i]);
    return r;
}
constexpr int kFDeviceCoherent = 1 << 4;        // cache policy: coherent across the device
constexpr unsigned kFOutside = 0x80000000u;  // past every buffer (each is below 2^31 bytes)

constexpr int kFT = 16;             // tile edge
constexpr int kFM = 14;             // output tile edge
constexpr int kFQ = kFT / 2 + 1;    // kept spectrum columns
constexpr int kFF = kFT * kFQ;      // kept frequencies per tile (144)
constexpr int kFWaves = 8;
constexpr int kFPerWave = kFF / kFWaves;  // 18 frequencies per wave
static_assert(kFF % kFWaves == 0, "frequencies split evenly over the waves");

// cos(2 pi j / 16) and sin(2 pi j / 16): the 16th roots of unity, written out
// (cos(pi/8) = sqrt(2 + sqrt 2) / 2, cos(pi/4) = sqrt(2) / 2, cos(3 pi/8) =
// sqrt(2 - sqrt 2) / 2, rounded to float).
__host__ __device__ constexpr float cos16(int j) {
    switch (j & 15) {
        case 0: return 1.0f;
        case 1: case 15: return 0.923879532511286756f;
        case 2: case 14: return 0.707106781186547524f;
        case 3: case 13: return 0.382683432365089772f;
        case 4: case 12: return 0.0f;
        case 5: case 11: return -0.382683432365089772f;
        case 6: case 10: return -0.707106781186547524f;
        case 7: case 9: return -0.923879532511286756f;
        default: return -1.0f;
    }
}
__host__ __device__ constexpr float sin16(int j) { return cos16(j + 12); }  // sin x = cos(x - pi/2)

__host__ __device__ constexpr int bitrev4(int k) {
    return ((k & 1) << 3) | ((k & 2) << 1) | ((k & 4) >> 1) | ((k & 8) >> 3);
}

// In-place 16-point DFT X[a] = sum_b x[b] exp(S * 2 pi i a b / 16), S = -1
// (forward) or +1 (inverse, unscaled): radix-2 decimation in time.  The loops
// unroll completely, so every twiddle is a constant; the trivial ones (1 and
// +-i) are taken without multiplications.
template <int S>
__device__ __forceinline__ void dft16(float (&re)[16], float (&im)[16]) {
    float r[16], i[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        r[k] = re[bitrev4(k)];
        i[k] = im[bitrev4(k)];
    }
#pragma unroll
    for (int len = 2; len <= 16; len <<= 1) {
        const int half = len / 2;
#pragma unroll
        for (int s = 0; s < 16; s += len) {
#pragma unroll
            for (int j = 0; j < half; ++j) {
                const int tw = j * (16 / len);  // exp(S 2 pi i tw / 16)
                const int a = s + j, b = s + j + half;
                float xr, xi;
                if (tw == 0) {
                    xr = r[b];
                    xi = i[b];
                } else if (tw == 4) {  // multiply by S i
                    xr = -S * i[b];
                    xi = S * r[b];
                } else {
                    const float c = cos16(tw), sn = S * sin16(tw);
                    xr = r[b] * c - i[b] * sn;
                    xi = r[b] * sn + i[b] * c;
                }
                r[b] = r[a] - xr;
                i[b] = i[a] - xi;
                r[a] = r[a] + xr;
                i[a] = i[a] + xi;
            }
        }
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        re[k] = r[k];
        im[k] = i[k];
    }
}

// Tile t of the layer: image n and tile row / column, as for the Winograd path
// with m = 14.
struct FTile {
    int n, ty, tx;
    bool ok;
};
__device__ __forceinline__ FTile fft_tile(const Geometry &g, int t) {
    FTile r;
    r.ok = t < g.ntiles;
    const int tt = r.ok ? t : 0;
    const int per = g.TH * g.TW;
    r.n = tt / per;
    const int rem = tt - r.n * per;
    r.ty = rem / g.TW;
    r.tx = rem - r.ty * g.TW;
    return r;
}

// Transformed kernels: wt[((cs * Kb + kb) * 144 + f) * 64 + lane] = {Re Wp,
// Im Wp, -Im Wp, 0} of output channel kb*16 + lane % 16 and input channel
// cs*4 + lane / 16 (the MFMA A-operand order), zero for padding channels.  One
// thread per (c, k), the spectrum summed from its definition (9 taps).
__global__ void __launch_bounds__(256) fft_weight_transform_kernel(const float *__restrict__ w,
                                                                    floatx4 *__restrict__ wt, Geometry g) {
    const int KP = g.Kb * 16;
    const long long total = (long long)g.Cs * 4 * KP;
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= total) return;
    const int c = (int)(idx / KP), k = (int)(idx - (long long)c * KP);
    float tap[9];
    const bool ok = c < g.C && k < g.K;
#pragma unroll
    for (int e = 0; e < 9; ++e) tap[e] = ok ? w[((long long)k * g.C + c) * 9 + e] : 0.0f;
    const int lane = (c & 3) * 16 + (k & 15);
    floatx4 *dst = wt + ((long long)((c >> 2) * g.Kb + (k >> 4)) * kFF) * 64 + lane;
#pragma unroll
    for (int p = 0; p < kFT; ++p) {
#pragma unroll
        for (int q = 0; q < kFQ; ++q) {
            // Wp[p][q] = sum_{u,v} w[u][v] exp(-2 pi i (p u + q v) / 16)
            float re = 0.0f, im = 0.0f;
#pragma unroll
            for (int u = 0; u < 3; ++u)
#pragma unroll
                for (int v = 0; v < 3; ++v) {
                    const int a = p * u + q * v;
                    re += tap[u * 3 + v] * cos16(a);
                    im -= tap[u * 3 + v] * sin16(a);
                }
            dst[(p * kFQ + q) * 64] = floatx4{re, im, -im, 0.0f};
        }
    }
}

// Row transforms of two real rows at once: z = a + i b has spectrum Z, and
// A[q] = (Z[q] + conj Z[-q]) / 2, B[q] = (Z[q] - conj Z[-q]) / 2i.
__device__ __forceinline__ void unpack_real_pair(const float (&zr)[16], const float (&zi)[16], int q,
                                                 float &ar, float &ai, float &br, float &bi) {
    const int qc = (16 - q) & 15;
    ar = 0.5f * (zr[q] + zr[qc]);
    ai = 0.5f * (zi[q] - zi[qc]);
    br = 0.5f * (zi[q] + zi[qc]);
    bi = 0.5f * (zr[qc] - zr[q]);
}

// Threads that hold output rows in the epilogue, two rows each, and the floats of an
// item's partial outputs: four rounds of 28 per thread.
constexpr int kFRowThreads = 64 * (kFM / 2);
constexpr int kFPartFloats = 4 * 2 * kFM * kFRowThreads;

// PC: items are cut into P pieces of L channel stages (launch_fft_fused), workgroup
// piece * items + item.  The inverse transforms are linear, so each piece writes its
// own outputs to part, device-coherently, [round][float4][thread], and the last of an
// item's pieces to arrive (cnt, back at zero afterwards) adds them in piece order.
template <bool PC>
__global__ void __launch_bounds__(512) fft_fused_kernel(const float *__restrict__ x,
                                                         const floatx4 *__restrict__ wt,
                                                         float *__restrict__ y, Geometry g, int n_items, int P, int L,
                                                         float *part, unsigned *cnt) {
    // xin: the stage's 64 input tiles, element (tc, i, j) at tc * kXT + i * kXR + j,
    //      tc = channel-in-stage * 16 + tile (rows padded to 17 floats and tiles
    //      to 273, so that 64 lanes reading the same element of 64 tiles, or 16
    //      rows of one tile, fall in distinct banks)
    // spec: spectra [(f * 2 + part) * 64 + tc] (part 0 real, 1 imaginary), reused
    //       for the sums [(f * 2 + part) * 64 + lane] in the epilogue
    constexpr int kXR = 17, kXT = 273;
    __shared__ float xin[64 * kXT];
    __shared__ float spec[kFF * 2 * 64];
    // per tile of the item: x offset of its window's first element in channel 0
    // (may be negative: the window starts one row and column before the tile),
    // the rows (bits 0-15) and columns (bits 16-31) of the window inside the
    // image (0: no tile), the image, and the first output row and column
    __shared__ int tbase[16], tmask[16], tn[16], toy[16], tox[16];

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int piece = PC ? blockIdx.x / n_items : 0, item = blockIdx.x - piece * n_items;
    const int sb = PC ? piece * L : 0, se = PC && sb + L < g.Cs ? sb + L : g.Cs;
    const int tg = item / g.Kb, kb = item - tg * g.Kb;
    const long long HW = (long long)g.H * g.W;
    if (tid < 16) {
        const FTile ft = fft_tile(g, tg * 16 + tid);
        const int oy = ft.ty * kFM, ox = ft.tx * kFM;
        unsigned rows = 0, cols = 0;
        for (int e = 0; e < kFT; ++e) {
            if (oy - 1 + e >= 0 && oy - 1 + e < g.H) rows |= 1u << e;
            if (ox - 1 + e >= 0 && ox - 1 + e < g.W) cols |= 1u << e;
        }
        tbase[tid] = (int)((long long)ft.n * g.C * HW + (long long)(oy - 1) * g.W + (ox - 1));
        tmask[tid] = ft.ok ? (int)(rows | (cols << 16)) : 0;
        tn[tid] = ft.ok ? ft.n : -1;
        toy[tid] = oy;
        tox[tid] = ox;
    }

    floatx4 acc_re[kFPerWave], acc_im[kFPerWave];
#pragma unroll
    for (int j = 0; j < kFPerWave; ++j) {
        acc_re[j] = floatx4{0.f, 0.f, 0.f, 0.f};
        acc_im[j] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    const floatx4 *wk = wt + (long long)kb * kFF * 64 + lane;  // + cs * Kb * 144 * 64
    __syncthreads();

    // Input element s (0..31) of this thread in a stage: tile-channel tc =
    // (tid >> 8) + 2 s (channel s >> 3, tile (tid >> 8) + 2 (s & 7)), window row
    // ei = (tid >> 4) & 15, column ej = tid & 15; 16 consecutive threads read one
    // window row.
    const int eh = tid >> 8, ei = (tid >> 4) & 15, ej = tid & 15;
    const int erel = ei * g.W + ej;
    const int32x4 xrs = fft_rsrc(x, (unsigned)((long long)g.N * g.C * HW * 4));
    const int32x4 yrs = fft_rsrc(y, (unsigned)((long long)g.N * g.K * HW * 4));
    // byte offsets of the elements in channel 0 (they do not depend on the stage),
    // past the buffer outside the window's valid part, without a branch around the load
    unsigned xo[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const unsigned msk = (unsigned)tmask[eh + 2 * s];
        const bool in = (msk >> ei) & (msk >> (16 + ej)) & 1u;
        xo[s] = in ? ((unsigned)tbase[eh + 2 * s] + (unsigned)erel) * 4u : kFOutside;
    }
    float xr[32];
    auto load_part = [&](int cs, int s0, int s1) {
#pragma unroll
        for (int s = s0; s < s1; ++s) {
            const int ch = cs * 4 + (s >> 3);
            const bool in = ch < g.C;
            xr[s] = fft_buffer_load_f32(xrs, in ? xo[s & 7] : kFOutside, in ? (unsigned)ch * (unsigned)HW * 4u : 0u, 0);
        }
    };
    load_part(sb, 0, 32);

    for (int cs = sb; cs < se; ++cs) {
        // 1. the stage's input tiles (loaded during the previous stage's products)
#pragma unroll
        for (int s = 0; s < 32; ++s) xin[(eh + 2 * s) * kXT + ei * kXR + ej] = xr[s];
        __syncthreads();
        // kernel operands of the first frequencies, in flight during the transforms
        const floatx4 *ws = wk + (long long)cs * g.Kb * kFF * 64 + wave * kFPerWave * 64;
        constexpr int kCh = 3;  // frequencies per operand chunk
        floatx4 a0[kCh];
#pragma unroll
        for (int j = 0; j < kCh; ++j) a0[j] = ws[j * 64];
        // 2. along rows: rows i and i + 8 of tile-channel tc (= tid & 63, i = tid >> 6)
        //    as one complex transform; row i's 9 kept values go to spec at
        //    frequency i * 9 + q for now
        {
            const int tc = tid & 63, i = tid >> 6;
            float re[16], im[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                re[j] = xin[tc * kXT + i * kXR + j];
                im[j] = xin[tc * kXT + (i + 8) * kXR + j];
            }
            dft16<-1>(re, im);
#pragma unroll
            for (int q = 0; q < kFQ; ++q) {
                float ar, ai, br, bi;
                unpack_real_pair(re, im, q, ar, ai, br, bi);
                spec[((i * kFQ + q) * 2 + 0) * 64 + tc] = ar;
                spec[(((i + 8) * kFQ + q) * 2 + 0) * 64 + tc] = br;
                if (q == 0 || q == 8) continue;  // real
                spec[((i * kFQ + q) * 2 + 1) * 64 + tc] = ai;
                spec[(((i + 8) * kFQ + q) * 2 + 1) * 64 + tc] = bi;
            }
        }
        __syncthreads();
        // 3. along columns, in place over their 16 rows: wave q transforms column q of
        //    the 64 tile-channels, wave 0 the real columns 0 and 8 as one complex transform
        {
            const int im_at = wave == 0 ? 2 * 8 : 1;
            float re[16], im[16];
#pragma unroll
            for (int p = 0; p < 16; ++p) {
                re[p] = spec[(p * kFQ + wave) * 2 * 64 + lane];
                im[p] = spec[((p * kFQ + wave) * 2 + im_at) * 64 + lane];
            }
            dft16<-1>(re, im);
            if (wave == 0) {
#pragma unroll
                for (int p = 0; p < 16; ++p) {
                    float ar, ai, br, bi;
                    unpack_real_pair(re, im, p, ar, ai, br, bi);
                    spec[(p * kFQ * 2 + 0) * 64 + lane] = ar;
                    spec[(p * kFQ * 2 + 1) * 64 + lane] = ai;
                    spec[((p * kFQ + 8) * 2 + 0) * 64 + lane] = br;
                    spec[((p * kFQ + 8) * 2 + 1) * 64 + lane] = bi;
                }
            } else {
#pragma unroll
                for (int p = 0; p < 16; ++p) {
                    spec[((p * kFQ + wave) * 2 + 0) * 64 + lane] = re[p];
                    spec[((p * kFQ + wave) * 2 + 1) * 64 + lane] = im[p];
                }
            }
        }
        __syncthreads();
        // 4. products of the wave's frequencies: lane = channel-in-stage * 16 +
        //    tile reads operand B; its kernel operands {Wr, Wi, -Wi} come as one
        //    float4, the next chunk's loaded while one is multiplied
        floatx4 a1[kCh];
#pragma unroll
        for (int j0 = 0; j0 < kFPerWave; j0 += kCh) {
            if (j0 + kCh < kFPerWave) {
#pragma unroll
                for (int j = 0; j < kCh; ++j) a1[j] = ws[(j0 + kCh + j) * 64];
            }
            // the next stage's input tiles, in flight during the products: a sixth with
            // each chunk and behind its operands, whose waits then do not include them
            // (past the last stage loads nobody uses, of channels in range or zeros)
            load_part(cs + 1, j0 / kCh * 32 / (kFPerWave / kCh), (j0 / kCh + 1) * 32 / (kFPerWave / kCh));
#pragma unroll
            for (int j = 0; j < kCh; ++j) {
                const int f = wave * kFPerWave + j0 + j;
                const float br = spec[(f * 2 + 0) * 64 + lane], bi = spec[(f * 2 + 1) * 64 + lane];
                acc_re[j0 + j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[j].x, br, acc_re[j0 + j], 0, 0, 0);
                acc_re[j0 + j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[j].y, bi, acc_re[j0 + j], 0, 0, 0);
                acc_im[j0 + j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[j].x, bi, acc_im[j0 + j], 0, 0, 0);
                acc_im[j0 + j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[j].z, br, acc_im[j0 + j], 0, 0, 0);
            }
#pragma unroll
            for (int j = 0; j < kCh; ++j) a0[j] = a1[j];
        }
        __syncthreads();  // xin and spec are rewritten by the next stage
    }

    // Epilogue, in four rounds v = 0..3: the sums of output channels
    // kb*16 + 4h + v (h = lane >> 4, accumulator element v) for tile lane & 15,
    // i.e. one sum per lane ("pair" = lane), pass through spec.
    constexpr float kScale = 1.0f / (kFT * kFT);
    // Output rows i and i + 7 of pair pr (tid < 64 * 7) in round v.  Stores outside the
    // image (or of a missing tile or output channel) get an offset past the buffer and
    // are dropped.
    auto store_rows = [&](int v, const float *re, const float *im) {
        const int pr = tid & 63, i = tid >> 6;
        const int t = pr & 15, k = kb * 16 + 4 * (pr >> 4) + v;
        const int n = tn[t], ox0 = tox[t];
        const bool ok = n >= 0 && k < g.K;
        // (unsigned arithmetic: offsets that are not used may wrap)
        const unsigned kbase = ((unsigned)(ok ? n : 0) * (unsigned)g.K + (unsigned)k) * (unsigned)HW;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int oy = toy[t] + i + 7 * half;
            const bool rok = ok && oy < g.H;
            const unsigned rowoff = (kbase + (unsigned)(oy * g.W + ox0)) * 4u;
#pragma unroll
            for (int j = 0; j < kFM; ++j) {
                const unsigned off = (rok && ox0 + j < g.W) ? rowoff + 4u * j : kFOutside;
                fft_buffer_store_f32((half ? im[j] : re[j]) * kScale, yrs, off, 0, 0);
            }
        }
    };
    float *const mine = PC ? part + ((long long)item * P + piece) * kFPartFloats : nullptr;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
#pragma unroll
        for (int j = 0; j < kFPerWave; ++j) {
            const int f = wave * kFPerWave + j;
            spec[(f * 2 + 0) * 64 + lane] = acc_re[j][v];
            spec[(f * 2 + 1) * 64 + lane] = acc_im[j][v];
        }
        __syncthreads();
        // inverse along columns (pair lane, column wave), in place; row p of the result
        // is output row p of the circular correlation.  Columns 0 and 8 of a real tile
        // are real then: wave 0 takes column 0 plus i times column 8.
        {
            const int im_at = wave == 0 ? 2 * 8 : 1;
            float re[16], im[16];
#pragma unroll
            for (int p = 0; p < 16; ++p) {
                re[p] = spec[((p * kFQ + wave) * 2 + 0) * 64 + lane];
                im[p] = spec[((p * kFQ + wave) * 2 + 1) * 64 + lane];
                if (wave == 0) {
                    re[p] -= spec[((p * kFQ + 8) * 2 + 1) * 64 + lane];
                    im[p] += spec[((p * kFQ + 8) * 2 + 0) * 64 + lane];
                }
            }
            dft16<1>(re, im);
#pragma unroll
            for (int p = 0; p < 16; ++p) {
                spec[(p * kFQ + wave) * 2 * 64 + lane] = re[p];
                spec[((p * kFQ + wave) * 2 + im_at) * 64 + lane] = im[p];
            }
        }
        __syncthreads();
        // inverse along rows for output rows i and i + 7 (i < 7) of pair pr as one
        // complex transform: row i's spectrum (completed by conjugate symmetry,
        // imaginary parts at q = 0 and 8 dropped as for a real row) plus i times
        // row i + 7's gives row i in the real part, row i + 7 in the imaginary part
        if (tid < 64 * 7) {
            const int pr = tid & 63, i = tid >> 6;
            float re[16], im[16];
#pragma unroll
            for (int q = 0; q < kFQ; ++q) {
                const float ar = spec[((i * kFQ + q) * 2 + 0) * 64 + pr];
                const float ai = (q == 0 || q == 8) ? 0.0f : spec[((i * kFQ + q) * 2 + 1) * 64 + pr];
                const float br = spec[(((i + 7) * kFQ + q) * 2 + 0) * 64 + pr];
                const float bi = (q == 0 || q == 8) ? 0.0f : spec[(((i + 7) * kFQ + q) * 2 + 1) * 64 + pr];
                re[q] = ar - bi;
                im[q] = ai + br;
                if (q > 0 && q < 8) {  // column 16 - q: conj(A) + i conj(B)
                    re[16 - q] = ar + bi;
                    im[16 - q] = br - ai;
                }
            }
            dft16<1>(re, im);
            if constexpr (PC) {
                const int32x4 prs = fft_rsrc(mine, kFPartFloats * 4u);
                auto val = [&](int e) { return e < kFM ? re[e] : im[e - kFM]; };
#pragma unroll
                for (int e = 0; e < 2 * kFM / 4; ++e)
                    fft_buffer_store_f32x4(floatx4{val(4 * e), val(4 * e + 1), val(4 * e + 2), val(4 * e + 3)}, prs,
                                           (unsigned)tid * 16u, (unsigned)(v * 7 + e) * (kFRowThreads * 16u),
                                           kFDeviceCoherent);
            } else {
                store_rows(v, re, im);
            }
        }
        __syncthreads();  // spec is rewritten by the next round
    }
    if constexpr (PC) {
        __shared__ unsigned last;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's partial outputs are stored
        __syncthreads();
        if (tid == 0) {
            const unsigned old = __hip_atomic_fetch_add(cnt + item, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            last = old + 1 == (unsigned)P ? 1u : 0u;
            if (last) __hip_atomic_store(cnt + item, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        if (last == 0 || tid >= kFRowThreads) return;
        const int32x4 all = fft_rsrc(part + (long long)item * P * kFPartFloats, (unsigned)P * kFPartFloats * 4u);
#pragma unroll 1
        for (int v = 0; v < 4; ++v) {
            float sum[2 * kFM] = {};
#pragma unroll 1
            for (int j0 = 0; j0 < P; j0 += 4) {
                floatx4 pv[4][2 * kFM / 4];  // pieces loaded before any is added
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int j = j0 + c < P ? j0 + c : P - 1;
#pragma unroll
                    for (int e = 0; e < 2 * kFM / 4; ++e)
                        pv[c][e] = fft_buffer_load_f32x4(all, (unsigned)tid * 16u,
                                                         (unsigned)j * (kFPartFloats * 4u) +
                                                             (unsigned)(v * 7 + e) * (kFRowThreads * 16u),
                                                         kFDeviceCoherent);
                }
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (j0 + c < P) {
#pragma unroll
                        for (int e = 0; e < 2 * kFM; ++e) sum[e] += pv[c][e / 4][e % 4];
                    }
            }
            store_rows(v, sum, sum + kFM);
        }
    }
}

}  // namespace

hipError_t launch_fft_weight_transform(const Geometry &g, const float *w, float *wt, hipStream_t s) {
    const long long total = (long long)g.Cs * 4 * g.Kb * 16;
    const unsigned blocks = (unsigned)((total + 255) / 256);
    hipLaunchKernelGGL(fft_weight_transform_kernel, dim3(blocks), dim3(256), 0, s, w,
                       reinterpret_cast<floatx4 *>(wt), g);
    return hipGetLastError();
}

static long long fft_items(const Geometry &g) { return (long long)((g.ntiles + 15) / 16) * g.Kb; }

// Pieces of channel stages an item is cut into: those with the fewest stage times over
// the rounds of workgroups, one per compute unit, counting a piece's inverse transforms
// and partial outputs as kEnd stages; 1 unless a fifth is saved.
int fft_pieces(const Geometry &g, int num_cus) {
    constexpr int kMaxPieces = 8, kEnd = 4;
    const long long items = fft_items(g), cus = num_cus < 1 ? 1 : num_cus;
    auto cost = [&](int p) { return (items * p + cus - 1) / cus * ((g.Cs + p - 1) / p + (p > 1 ? kEnd : 0)); };
    int best = 1;
    for (int p = 2; p <= kMaxPieces && items * p <= 2 * cus; ++p) {
        const int l = (g.Cs + p - 1) / p;
        if ((long long)l * (p - 1) < g.Cs && cost(p) < cost(best)) best = p;  // no piece without stages
    }
    return 5 * cost(best) <= 4 * cost(1) ? best : 1;
}
size_t fft_part_bytes(const Geometry &g, int pieces) {
    return pieces > 1 ? (size_t)fft_items(g) * pieces * kFPartFloats * sizeof(float) : 0;
}
size_t fft_cnt_bytes(const Geometry &g, int pieces) { return pieces > 1 ? (size_t)fft_items(g) * sizeof(unsigned) : 0; }

hipError_t launch_fft_fused(const Geometry &g, const float *x, const float *wt, float *y, int pieces,
                            const SplitBuffers &sb, hipStream_t s) {
    const int items = (int)fft_items(g), L = (g.Cs + pieces - 1) / pieces;
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3((unsigned)(items * pieces)), dim3(512), 0, s, x,
                           reinterpret_cast<const floatx4 *>(wt), y, g, items, pieces, L, sb.part, sb.cnt);
    };
    if (pieces > 1) go(fft_fused_kernel<true>);
    else go(fft_fused_kernel<false>);
    return hipGetLastError();
}

}  // namespace wino

// Filter gradient, split-K over output pixels, on the bf16 matrix cores with
// fp32 operands held as three bf16 parts.
//
//   dw[n,u,v,d] = sum_b sum_{i<HO, j<WO} dy[b,i,j,n] * x[b,i+u,j+v,d]
//
// GEMM view: rows = filters n, columns = taps q = (u, v, d), contraction over
// output pixels.  Every fp32 value is exactly the sum of three bf16 values
// (each the rounded remainder of the ones before); a product of two values is
// six bf16 products, hh into one accumulator and the five small ones into
// another.  See the register-streamed correlation kernel for the reasons and
// the error; here too fp32 matrix instructions set the pace before (the
// contraction has one 16x16x32 instruction per 32 pixels and part pair, 16
// cycles, against eight 32-cycle fp32 instructions for the same 32 pixels).
//
// What bounds it.  A 16x16x32 instruction takes eight consecutive
// contraction values per lane, here eight pixels of one filter or tap, while
// memory has the filters and taps contiguous.  ds_read_b64_tr_b16 transposes
// on the way out of LDS: 16 lanes name four rows (pixels) of 16 values and
// each gets one column's four pixels.  So both operands are staged as they
// are in memory.  For x this works for any tap: the (v, d) run of a pixel
// starts D values further on for the next pixel, and a lane names four
// consecutive values of the run of its pixel.  These are 8-byte reads, so
// where D is not a multiple of 4 the rows are staged in COPIES copies, copy
// c shifted by c values, and a lane takes the copy that makes its run
// aligned (the pixel's index mod 4 is the lane's, whatever the step).
//
// Work split.  A workgroup owns RT*16 filters and a range of the 16-tap
// column tiles, dealt to its NW waves as evenly as they go (CTM or CTM - 1
// each: 49 tiles over 16 waves give 15 waves 3 tiles and one 4).  It walks
// down a strip of RW output columns, RH output rows at a time: every step
// stages the next RH rows of dy and of x (in a ring of RING rows, so each x
// row is read once per strip, not once per filter row) while the products of
// the current step run, with one barrier per step.  Of the two waves that
// share a SIMD one stages first and the other computes first, so that the
// conversions of one run beside the products of the other.  A segment is
// RSEG rows of a strip of an image; workgroup column g takes segments g,
// g + NP, ... and writes its sums to part[g][n][q]; a separate kernel adds
// the NP partials in a fixed order, so results do not depend on timing.
//
// Range of the parts: x and dy are scaled by 2^XSH while staged (undone at
// the end, both exact), so that every last bit, of subnormal numbers too, is
// at least 2^-126 and no product is lost that fp32 would hold.  Sums of the
// PIXW pixels of a workgroup stay below 2^127 for magnitudes below 2^XHI.  A
// workgroup that staged a larger one, an infinity or a NaN computes its sums
// again with fp32 matrix instructions straight from memory.
//
// Measured against the kernel of fp32 instructions: 32 images 128x128x16, 64
// 7x7 filters, 451 and 237 us; 24 problems of 1 to 100 channels 1.0 to 3.6
// times as fast.
//
// Compile-time constants (FB_<name>):
//   problem  BATCH FH FW D N H W HO WO
//   tiling   RT (16-filter tiles per workgroup) NW (waves) NCB (workgroups
//            that share the columns) RH RW (output rows and columns per
//            step; RW a multiple of 16, RH*RW of 32) RSEG (output rows per
//            segment) NP (partials)
#ifndef __HIPCC_RTC__
#include <hip/hip_runtime.h>
#endif

#ifdef FB_INJECT_ERROR
#error "injected code-generation failure (test hook)"
#endif

typedef float ds_f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int ds_u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int ds_u32x4 __attribute__((ext_vector_type(4)));
typedef short ds_i16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 ds_bf16x8 __attribute__((ext_vector_type(8)));

#define BATCH FB_BATCH
#define FH FB_FH
#define FW FB_FW
#define D FB_D
#define N FB_N
#define H FB_H
#define W FB_W
#define HO FB_HO
#define WO FB_WO
#define RT FB_RT
#define NW FB_NW
#define NCB FB_NCB
#define RH FB_RH
#define RW FB_RW
#define RSEG FB_RSEG
#define NP FB_NP

#define NTHREADS (NW * 64)
#define QTOT (FH * FW * D)
#define FWD (FW * D)
#define R4 ((FWD + 3) / 4 * 4)           // a filter row's taps, in whole groups of 4
#define QP (FH * R4)
#define T16 ((QP + 15) / 16)             // column tiles
#define TWAVES (NCB * NW)                // waves that share them
#define CTM ((T16 + TWAVES - 1) / TWAVES)
#define RB (RT * 16)                     // filters per workgroup
#define NRB ((N + RB - 1) / RB)
#define PXS (RH * RW)                    // pixels per step
#define NKS (PXS / 32)
#define COPIES (D % 4 == 0 ? 1 : D % 2 == 0 ? 2 : 4)
#define NSTR ((WO + RW - 1) / RW)
#define NRS ((HO + RSEG - 1) / RSEG)
#define NSEG (BATCH * NSTR * NRS)

// First column tile of wave gw (of all TWAVES).
constexpr int first_tile(int gw) { return (int)((long)gw * T16 / TWAVES); }
// Most filter rows that one workgroup's columns touch.
constexpr int max_rows() {
    int m = 1;
    for (int cb = 0; cb < NCB; ++cb) {
        const int lo = first_tile(cb * NW) * 16 / R4;
        const int last = first_tile((cb + 1) * NW) * 16 - 1;
        const int hi = last / R4 < FH - 1 ? last / R4 : FH - 1;
        m = hi - lo + 1 > m ? hi - lo + 1 : m;
    }
    return m;
}
#define XRM max_rows()
#define RING (XRM + 2 * RH - 1)
#define XRE (((RW - 1) * D + R4 + 3) / 4 * 4)     // values of a staged x row
#define RSB (2 * XRE)                             // its bytes
#define COPYB (RING * RSB)
#define XPB (COPIES * COPYB)                      // bytes per part
#define DPB (2 * PXS * RB)
#define LDS_BYTES (3 * XPB + 2 * 3 * DPB)
#define GITEMS (PXS * RB / 4)                     // groups of 4 dy values per step
#define GPER ((GITEMS + NTHREADS - 1) / NTHREADS)
#define XROWI (COPIES * XRE / 4)                  // groups of 4 x values per row
#define XITEMS (RH * XROWI)
#define XPER ((XITEMS + NTHREADS - 1) / NTHREADS)
#define XSH 24
// most pixels that one workgroup sums, and the magnitude's limit
#define PIXW ((long)((NSEG + NP - 1) / NP) * RSEG * RW)
#define XHI ((127 - 2 * XSH - log2_up(PIXW)) / 2)
// the A fragments of the next 32 pixels are read ahead while they fit
#define AHEAD (RT * CTM * 8 + RT * 24 + 24 <= 152)

static_assert(RW % 16 == 0 && PXS % 32 == 0, "whole instructions per step");

constexpr int log2_up(long n) {
    int b = 0;
    while ((1L << b) < n) ++b;
    return b;
}

// Largest magnitude of the values staged by a thread, as a bit pattern
// (infinities and NaNs above every finite value).
struct DsRange {
    unsigned hi = 0u;
    __device__ __forceinline__ void see(const float v) {
        const unsigned a = __builtin_bit_cast(unsigned, v) & 0x7fffffffu;
        hi = hi > a ? hi : a;
    }
    // some magnitude of 2^XHI or more
    __device__ __forceinline__ bool outside() const { return hi >= (127u + XHI) << 23; }
};

__device__ __forceinline__ unsigned ds_pair(const float a, const float b) {
    const unsigned lo = __builtin_bit_cast(unsigned short, (__bf16)a);       // nearest even
    const unsigned hi = __builtin_bit_cast(unsigned short, (__bf16)b);
    return lo | (hi << 16);
}

// Four values, scaled, as their three parts, PB bytes apart.
__device__ __forceinline__ void ds_put(unsigned char* dst, const int pb, const float* v, DsRange& range) {
    ds_u32x2 h, m, l;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        range.see(v[2 * i]);
        range.see(v[2 * i + 1]);
        const float a = v[2 * i] * (float)(1 << XSH), b = v[2 * i + 1] * (float)(1 << XSH);
        h[i] = ds_pair(a, b);
        const float ra = a - __builtin_bit_cast(float, h[i] << 16);
        const float rb = b - __builtin_bit_cast(float, h[i] & 0xffff0000u);
        m[i] = ds_pair(ra, rb);
        l[i] = ds_pair(ra - __builtin_bit_cast(float, m[i] << 16), rb - __builtin_bit_cast(float, m[i] & 0xffff0000u));
    }
    *(ds_u32x2*)dst = h;
    *(ds_u32x2*)(dst + pb) = m;
    *(ds_u32x2*)(dst + 2 * pb) = l;
}

// One fragment: two transposed reads, pixels 0..15 and 16..31 of a step.
__device__ __forceinline__ ds_bf16x8 ds_frag(const unsigned char* p0, const unsigned char* p1) {
    typedef __attribute__((address_space(3))) ds_i16x4* lds_ptr;
    const ds_i16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)p0);
    const ds_i16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)p1);
    return __builtin_bit_cast(ds_bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

template <int V> struct DsInt { static constexpr int value = V; };

extern "C" __global__ void __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(2)))
fbcorr_dw_split(const float* __restrict__ x, const float* __restrict__ dy, float* __restrict__ part)
{
    __shared__ __attribute__((aligned(16))) unsigned char lds[LDS_BYTES];
    unsigned char* const xl = lds;
    unsigned char* const gl = lds + 3 * XPB;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, li = lane & 15, lj = li >> 2, lc = li & 3;
    const int cb = blockIdx.y % NCB, n0 = blockIdx.y / NCB * RB;

    // this workgroup's filter rows, this wave's column tiles
    const int blo = first_tile(cb * NW) * 16 / R4;
    const int blast = first_tile((cb + 1) * NW) * 16 - 1;
    const int xrn = (blast / R4 < FH - 1 ? blast / R4 : FH - 1) - blo + 1;
    const int t0 = first_tile(cb * NW + wave);
    const int nct = first_tile(cb * NW + wave + 1) - t0;

    // Lane offsets.  A: pixel 4g + lj, the 16-filter units of a row exchanged
    // by pixel (fsw) so that the eight pixels that are read together lie in
    // different banks.  B: the run of pixel 4g + lj at this lane's four taps.
    const int fsw = RT == 4 ? (lj >> 1) | ((g & 1) << 1) : RT == 2 ? (g & 1) : 0;
    int la[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) la[rt] = 2 * ((4 * g + lj) * RB + (rt ^ fsw) * 16 + lc * 4);
    int lb[CTM], slot[CTM];
    const int copy = (lj * D) % 4;
    const int copyi = COPIES == 4 ? copy : copy / 2;
#pragma unroll
    for (int ct = 0; ct < CTM; ++ct) {
        const int q = (t0 + ct) * 16 + lc * 4;
        const bool in = ct < nct && q < QP;
        const int u = in ? q / R4 : blo, r0 = in ? q % R4 : 0;
        lb[ct] = 2 * ((4 * g + lj) * D + r0 - copy) + copyi * COPYB;
        slot[ct] = u - blo;
    }

    ds_f32x4 acc[RT][CTM][2];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int ct = 0; ct < CTM; ++ct)
#pragma unroll
            for (int k = 0; k < 2; ++k) acc[rt][ct][k] = (ds_f32x4){0.f, 0.f, 0.f, 0.f};

    DsRange range;
    float greg[GPER][4], xreg[XPER][4];
    int b = 0, i0 = 0, j0 = 0, rows = 0;           // the segment

    // Group e of a row of x: input row ii, values of copy c from 4*q on.
    auto load_x = [&](const int ii, const int e, float* v) {
        const int c = e / (XRE / 4), q = e % (XRE / 4);
        const int pos = j0 * D + 4 * q + (COPIES == 2 ? 2 * c : c);       // in the image row
        const float* src = x + ((long)b * H + ii) * W * D + pos;
#if D % 4 == 0
        ds_f32x4 x4 = {0.f, 0.f, 0.f, 0.f};
        if (ii < H && pos < W * D) x4 = *(const ds_f32x4*)src;
        v[0] = x4[0]; v[1] = x4[1]; v[2] = x4[2]; v[3] = x4[3];
#else
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = ii < H && pos + k < W * D ? src[k] : 0.f;
#endif
    };
    auto store_x = [&](const int sl, const int e, const float* v) {
        const int c = e / (XRE / 4), q = e % (XRE / 4);
        ds_put(xl + c * COPYB + sl * RSB + 8 * q, XPB, v, range);
    };
    // Group e of a step's dy.
    auto load_g = [&](const int t, const int e, float* v) {
        const int p = e / (RB / 4), n = n0 + e % (RB / 4) * 4;
        const int r = t * RH + p / RW, j = j0 + p % RW;
        const float* src = dy + (((long)b * HO + i0 + r) * WO + j) * N + n;
        const bool in = r < rows && j < WO;
#if N % 4 == 0
        ds_f32x4 x4 = {0.f, 0.f, 0.f, 0.f};
        if (in && n < N) x4 = *(const ds_f32x4*)src;
        v[0] = x4[0]; v[1] = x4[1]; v[2] = x4[2]; v[3] = x4[3];
#else
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = in && n + k < N ? src[k] : 0.f;
#endif
    };
    auto store_g = [&](const int buf, const int e, const float* v) {
        const int p = e / (RB / 4), c4 = e % (RB / 4);
        const int f = RT == 4 ? (p >> 1) & 3 : RT == 2 ? (p >> 2) & 1 : 0;
        ds_put(gl + buf * 3 * DPB + 2 * (p * RB + ((c4 >> 2) ^ f) * 16 + (c4 & 3) * 4), DPB, v, range);
    };
    // The rows of step t that are not staged yet: RH of dy, RH of x.
    auto fetch = [&](const int t) {
#pragma unroll
        for (int k = 0; k < GPER; ++k) {
            const int e = tid + k * NTHREADS;
            if (GITEMS % NTHREADS == 0 || e < GITEMS) load_g(t, e, greg[k]);
        }
#pragma unroll
        for (int k = 0; k < XPER; ++k) {
            const int e = tid + k * NTHREADS;
            if (XITEMS % NTHREADS == 0 || e < XITEMS)
                load_x(i0 + blo + t * RH + xrn - 1 + e / XROWI, e % XROWI, xreg[k]);
        }
    };
    auto store = [&](const int t) {
#pragma unroll
        for (int k = 0; k < GPER; ++k) {
            const int e = tid + k * NTHREADS;
            if (GITEMS % NTHREADS == 0 || e < GITEMS) store_g(t & 1, e, greg[k]);
        }
#pragma unroll
        for (int k = 0; k < XPER; ++k) {
            const int e = tid + k * NTHREADS;
            if (XITEMS % NTHREADS == 0 || e < XITEMS)
                store_x((t * RH + xrn - 1 + e / XROWI) % RING, e % XROWI, xreg[k]);
        }
    };

    // The products of one step: NKS x 32 pixels, NCT column tiles.
    auto compute = [&](const int buf, const bool full) {
        constexpr int NCT = CTM;
        const unsigned char* const ga = gl + buf * 3 * DPB;
        // 16-pixel unit k of the step: its row, its first column
        auto urow = [](int k) { return k / (RW / 16); };
        auto ucol = [](int k) { return k % (RW / 16) * 16; };
        const unsigned char* xb[NCT][RH];
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
            for (int r = 0; r < RH; ++r) {
                const int s = slot[ct] + r;
                xb[ct][r] = xl + lb[ct] + (s < RING ? s : s - RING) * RSB;
            }
        ds_bf16x8 a[AHEAD ? 2 : 1][RT][3], bf[2][3];
        auto read_a = [&](const int ks, ds_bf16x8 (&dst)[RT][3]) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int p = 0; p < 3; ++p)
                    dst[rt][p] = ds_frag(ga + la[rt] + p * DPB + 2 * ks * 32 * RB,
                                         ga + la[rt] + p * DPB + 2 * (ks * 32 + 16) * RB);
        };
        auto read_b = [&](const int ks, const int ct, ds_bf16x8 (&dst)[3]) {
#pragma unroll
            for (int p = 0; p < 3; ++p)
                dst[p] = ds_frag(xb[ct][urow(2 * ks)] + p * XPB + 2 * ucol(2 * ks) * D,
                                 xb[ct][urow(2 * ks + 1)] + p * XPB + 2 * ucol(2 * ks + 1) * D);
        };
        read_a(0, a[0]);
        read_b(0, 0, bf[0]);
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) {
                const int it = ks * NCT + ct, ab = AHEAD ? ks & 1 : 0;
                const bool last = it + 1 == NKS * NCT;
                if (!last) read_b((it + 1) / NCT, (it + 1) % NCT, bf[(it + 1) & 1]);
                if (AHEAD && ct == 0 && ks + 1 < NKS) read_a(ks + 1, a[ab ^ 1]);
                constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
                // (the same in every lane of the wave)
                if (ct < NCT - 1 || full)
#pragma unroll
                for (int q = 0; q < 6; ++q)
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
                        acc[rt][ct][q < 5] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            a[ab][rt][PA[q]], bf[it & 1][PB[q]], acc[rt][ct][q < 5], 0, 0, 0);
                if (!AHEAD && ct == NCT - 1 && ks + 1 < NKS) read_a(ks + 1, a[0]);
                // (the reads above stay ahead of these products)
                __builtin_amdgcn_sched_barrier(0);
            }
    };

    const bool early = wave < NW / 2;
#pragma unroll 1
    for (int seg = blockIdx.x; seg < NSEG; seg += NP) {
        b = seg / (NSTR * NRS);
        j0 = seg / NRS % NSTR * RW;
        i0 = seg % NRS * RSEG;
        rows = HO - i0 < RSEG ? HO - i0 : RSEG;
        const int steps = (rows + RH - 1) / RH;
        // the first step's rows of x and dy (every wave is past the last
        // segment's products)
#pragma unroll 1
        for (int e0 = 0; e0 < (xrn + RH - 1) * XROWI; e0 += 4 * NTHREADS) {
            float v[4][4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int e = e0 + k * NTHREADS + tid;
                if (e < (xrn + RH - 1) * XROWI) load_x(i0 + blo + e / XROWI, e % XROWI, v[k]);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int e = e0 + k * NTHREADS + tid;
                if (e < (xrn + RH - 1) * XROWI) store_x(e / XROWI, e % XROWI, v[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < GPER; ++k) {
            const int e = tid + k * NTHREADS;
            if (GITEMS % NTHREADS == 0 || e < GITEMS) {
                load_g(0, e, greg[k]);
                store_g(0, e, greg[k]);
            }
        }
        if (steps > 1) fetch(1);
#pragma unroll
        for (int ct = 0; ct < CTM; ++ct) {
            const int q = (t0 + ct) * 16 + lc * 4;
            slot[ct] = (ct < nct && q < QP ? q / R4 : blo) - blo;
        }
        __syncthreads();
#pragma unroll 1
        for (int t = 0; t < steps; ++t) {
            auto stage = [&]() {
                if (t + 1 < steps) {
                    store(t + 1);
                    if (t + 2 < steps) fetch(t + 2);
                }
            };
            if (early) stage();
            compute(t & 1, nct == CTM);
            if (!early) stage();
#pragma unroll
            for (int ct = 0; ct < CTM; ++ct) {
                slot[ct] += RH;
                slot[ct] = slot[ct] < RING ? slot[ct] : slot[ct] - RING;
            }
            __syncthreads();
        }
    }

    // Partial sums: part[g][n][q] (zeros from workgroups without segments).
    float* const out = part + (long)blockIdx.x * N * QTOT;
    float os = 1.0f / (float)(1L << 2 * XSH);
    if (__builtin_amdgcn_readfirstlane(__syncthreads_or(range.outside()))) {
        // Values that the parts cannot hold: 16x16x4 fp32 products, four
        // pixels of an output row at a time, lane group g its pixel g, each
        // operand loaded where it is used (2 images 60x70x8, 64 7x7 filters,
        // two such values: 24 us, with one sum per thread 185; without any 12,
        // the kernel of fp32 instructions 18).
        os = 1.f;
        int to[CTM];
#pragma unroll
        for (int ct = 0; ct < CTM; ++ct) {
            const int q = (t0 + ct) * 16 + li, u = q / R4, r = q % R4;
            to[ct] = ct < nct && q < QP && r < FWD ? u * (W * D) + r : -1;
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int k = 0; k < 2; ++k) acc[rt][ct][k] = (ds_f32x4){0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll 1
        for (int seg = blockIdx.x; seg < NSEG; seg += NP) {
            const int sb = seg / (NSTR * NRS), sj = seg / NRS % NSTR * RW, si = seg % NRS * RSEG;
            const int cols = WO - sj < RW ? WO - sj : RW;
#pragma unroll 1
            for (int i = si; i < si + RSEG && i < HO; ++i) {
                const float* const gr = dy + (((long)sb * HO + i) * WO + sj) * N + n0 + li;
                const float* const xr = x + (((long)sb * H + i) * W + sj) * D;
#pragma unroll 2
                for (int j = 0; j < cols; j += 4) {
                    const int p = j + g;
                    float a[RT], bv[CTM];
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
                        a[rt] = p < cols && n0 + rt * 16 + li < N ? gr[(long)p * N + rt * 16] : 0.f;
#pragma unroll
                    for (int ct = 0; ct < CTM; ++ct) bv[ct] = p < cols && to[ct] >= 0 ? xr[p * D + to[ct]] : 0.f;
#pragma unroll
                    for (int ct = 0; ct < CTM; ++ct)
#pragma unroll
                        for (int rt = 0; rt < RT; ++rt)
                            acc[rt][ct][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[rt], bv[ct], acc[rt][ct][0], 0, 0, 0);
                }
            }
        }
    }
#pragma unroll
    for (int ct = 0; ct < CTM; ++ct) {
        const int q = (t0 + ct) * 16 + li, u = q / R4, r = q % R4;
        if (ct >= nct || q >= QP || r >= FWD) continue;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int n = n0 + rt * 16 + 4 * g + k;
                if (n < N) out[(long)n * QTOT + u * FWD + r] = (acc[rt][ct][0][k] + acc[rt][ct][1][k]) * os;
            }
    }
}

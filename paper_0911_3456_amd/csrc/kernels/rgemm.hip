// Implicit-GEMM valid correlation on the matrix cores with the filter
// operand streamed straight into registers.
//
//   O[b,i,j,c] = sum_{u<FH, v<FW, k<CIN} Ipad[b, i+u, j+v, k] * Wt[c, u, v, k]
//
// (Ipad: the input I[b][HI][WI][CIN] with PADH/PADW rows/columns of virtual
// zeros on every side.)  Same GEMM view as the LDS-staged kernel: rows =
// output pixels, columns = output channels (filters), contraction over
// (u, v, k).  What differs is where the operands come from.
//
// * The filter bank is first rewritten by fbcorr_pack_frag (below) in the
//   exact order in which the matrix-core instructions consume it: for an
//   MF-filter column tile j, a channel chunk, a filter row u and a step t,
//   the 64 lanes' 16-byte fragments are one contiguous kilobyte.  Each wave
//   loads its own column tiles' fragments from L2 with one 16-byte load per
//   lane per tile and step, PF steps ahead, into a ring of registers.  The
//   filters never pass through LDS, so there is no per-filter-row staging
//   and no barrier inside a channel chunk: a chunk is one uninterrupted run
//   of FH * NSTEP steps of products.
// * The input tile of a channel chunk (with its FH-1 / FW-1 halo) is staged
//   once in LDS as 16-byte cells of PE consecutive channels, NPL = KC/PE
//   planes of cells.  The 16 lanes that read together take 16 consecutive
//   pixel columns of one plane: 256 contiguous bytes.  (gfx950 also pairs
//   lanes l and l+16 of each half-wave: their two 256-byte runs cost no
//   extra cycle only when they start at the same offset modulo 256 bytes,
//   i.e. when the row stride TCP is a multiple of 16 cells for MC = 16;
//   XPADC sets the stride.)
//
// Contraction order.  Within a filter row u and chunk, the run of (v, k)
// pairs (tap-major, FW*KC values) is cut into cells of PE values, zero-padded
// to CPR whole cells; the rows' cells follow one another, and a step takes
// NKG = 64/MF of them, one per lane group of an instruction.  A step may
// therefore straddle two filter rows, so the padding is less than a cell per
// row and less than a step per chunk (a 9-tap row of 8 channels costs 9
// cells, not 10 or 12).  For 16-bit operands one step is one
// v_mfma_f32_{32x32x16,16x16x32} (8 values per lane); for fp32 it is four
// v_mfma_f32_{32x32x2,16x16x4}_f32 (value q of the lane's cell in product
// q).  A and B use the same order, so every padding value multiplies a zero
// weight; it is zeroed itself first (mask_a), so that an infinity there does
// not make a NaN.
//
// LDS layout of the input tile.  KC a power-of-two number of cells: planes
// of 16-byte cells as above.  Any other KC (16-bit operands): the rows as
// they are, KC values per pixel; a cell is then any 8-byte aligned run of 8
// values, which may straddle pixels (4 channels: two taps per cell).  The
// lanes of a tile are S*KC values apart, so S*KC is a multiple of 4: a
// single-channel image takes S = 4, which costs little where a row of taps
// is padded to whole cells anyway (11 taps + 3 shifts: 14 of 16 values).
//
// fp32 as three bf16 parts (DT 3).  fp32 matrix instructions run at 1/16 of
// the bf16 rate.  Every fp32 value is exactly the sum of three bf16 values
// h + m + l (each the rounded remainder of the ones before), and the product
// of two such sums needs six bf16 products (hh, hm, mh, mm, hl, lh; what is
// left out is below 2^-24 of |x||w|), so a step is six instructions on
// operands staged as three parts instead of 8 * 2 of the fp32 kind: 290
// against 133-150 TFLOP/s of fp32 work with the operands in registers.  hh
// goes to one accumulator and the five small products to another, added at
// the end: the sum is then rounded once per 16 products instead of once per
// product, and the error against fp64 is a third of the fp32 instructions'
// (rms 7e-9 against 2.4e-8 of sum |x||w|, contractions of 144 to 16384; all
// terms positive: 1.5e-7 against 4.2e-7 at 784).
//
// Range of the parts.  A part is exact while the value's last bit is at least
// 2^-126, and a product of parts must not be lost below 2^-126 where fp32
// would hold it, so both operands are scaled up by powers of two (exact, and
// undone in UNSCALE): input values by 2^XSH, a filter so that its largest
// magnitude lies in [2^WSH, 2^(WSH+1)).  With 24 and 32:
//   input values: every last bit is at least 2^(24-149).
//   filters below 2^10: likewise, whatever the range inside a filter.
//   products: what falls below 2^-126 was below 2^(-182+e) before the
//   scaling, for a filter of magnitude 2^e: no more than fp32 loses below
//   2^-149 as long as e <= 24.
//   sums: K values below 2^XHI stay below 2^127, XHI = 70 - log2 K.
// Filters outside (2^25 and more; 2^10 and more beside magnitudes below
// 2^-135 of the largest; non-finite values) are marked by the pack with an
// UNSCALE of 0.  A workgroup that meets one of those, or whose tile holds a
// magnitude from 2^XHI up, an infinity or a NaN, computes its outputs with
// plain fp32 fused multiply-adds instead (slow_tile); small tails, down to
// subnormal numbers, stay on the matrix units.
// Measured, forward calls with fp32 instructions before and with three parts
// now: 1024x1024x8 with 16 5x5 filters 73.2 and 44.6 us, 480x640x3 with 32
// 7x7 42.4 and 24.3 us.
//
// Column shift S (narrow outputs).  A workgroup's NCOLW = WN*NT*MF matrix
// columns are S shifts x CB = NCOLW/S output channels: column (s, c)
// computes output column S*j + s of base pixel column j, with filter
// B[(u, v', k), (s, c)] = Wt[c, u, v'-s, k] (zero outside 0 <= v'-s < FW)
// over NTAPF = FW+S-1 taps per filter row; the pack writes each shifted
// copy, and a lane's A run starts at pixel column S*j.  A run then holds
// values that are outside some columns' windows: 16-bit tiles with infinities
// or NaNs go to slow_tile (which costs ordinary tiles of narrow banks up to
// 4 %: 65x424x16 with 9 7x7 filters 14.0 and 14.6 us).
//
// Compile-time constants (FB_<name>):
//   problem  BATCH FH FW CIN COUT HI WI HO WO PADH PADW
//   DT       0 fp32 operands, 1 bf16, 2 fp16, 3 fp32 operands as three bf16
//            parts (1-3: B pre-scaled and rounded by the pack; UNSCALE[c]
//            multiplies each output, and for 3 is 0 for a filter that the
//            parts cannot hold)
//   XMOFF    fp16 only: UNSCALE[XMOFF .. XMOFF+255] hold partial maxima of |x|
//            (fbcorr_absmax); when the input reaches 2^15 it is scaled by
//            2^-k while staged (max |x| * 2^-k < 2^15, inside the fp16
//            range) and the outputs by 2^k -- both exact powers of two
//   tiling   MF (32 or 16: MFMA tile), KC (channels per chunk: PE times a
//            power of two, or for 16-bit operands any multiple of 4, or CIN
//            where S*CIN is one), S (column shift, above), MR (rows of an
//            MF-pixel tile), MT NT (tiles per
//            wave), WM WN (waves), PF (filter-fragment ring depth in steps),
//            XPADC (LDS row padding in cells), WPE (waves per SIMD the
//            register budget is sized for), UNR (1: unroll the step loop
//            completely), XCDMAP (XCD-aware workgroup order), NTS (1:
//            non-temporal output stores), STE (1: tiles store through LDS as
//            16-byte vectors, pixels past the image edge and channels past
//            COUT skipped)
//   naming   KNAME   EPILOGUE(v, c) as in the LDS-staged kernel
#ifndef __HIPCC_RTC__
#include <hip/hip_runtime.h>
#endif

#ifdef FB_INJECT_ERROR
#error "injected code-generation failure (test hook)"
#endif

#ifndef FBC_RGEMM_COMMON
#define FBC_RGEMM_COMMON
typedef float rg_f32x4 __attribute__((ext_vector_type(4)));
typedef float rg_f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int rg_u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int rg_u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 rg_bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 rg_f16x8 __attribute__((ext_vector_type(8)));
#endif

// The batched kernel pastes what stands between the BODY markers
// once per variant, each in a namespace of its own, with the pack beside the
// correlation and the image extents left run-time; its bodies are functions
// that one kernel calls.
#ifdef FB_BATCHED
#define RG_PACK_ATTR __attribute__((noinline))
#define RG_GLOBAL __attribute__((address_space(1)))
#define RG_LDS __attribute__((address_space(3)))
#else
#define RG_PACK_ATTR __forceinline__
#define RG_GLOBAL
#define RG_LDS
#endif

//@@BODY-BEGIN
#define FH FB_FH
#define FW FB_FW
#define CIN FB_CIN
#define COUT FB_COUT
#define DT FB_DT
#define KC FB_KC
#ifdef FB_MF
#define MF FB_MF
#else
#define MF 32
#endif

#if DT == 0
#define PE 4                      // channels per 16-byte cell
#else
#define PE 8
#endif
#if DT == 3
#define NSP 3                     // bf16 parts of a value
#define NACC 2                    // accumulators per tile: hh, the small products
#define XSH 24                    // powers of two of the scales (range of the parts, above)
#define WSH 32
#else
#define NSP 1
#define NACC 1
#endif
#ifdef FB_S
#define S FB_S
#else
#define S 1
#endif
// Tiles that hold what must not meet a zero weight are computed by slow_tile:
// values outside the parts' range, and infinities and NaNs where a shifted
// column's window is narrower than the run of taps that its lanes read.
#if DT == 3 || (DT != 0 && S > 1)
#define GUARD 1
#else
#define GUARD 0
#endif
#define NKG (64 / MF)             // lane groups of one instruction
#define NPL (KC / PE)             // cell planes per channel chunk
#if KC % PE == 0 && (NPL & (NPL - 1)) == 0
#define LIN 0                     // planes of cells
#else
#define LIN 1                     // rows as they are
#endif
#define NTAPF (FW + S - 1)        // taps of one filter row with the column shifts
#define CPR ((NTAPF * KC + PE - 1) / PE)   // cells per filter row
#define NTAPS ((CPR * PE + KC - 1) / KC)   // taps covered, padding included
#define NCHUNK ((CIN + KC - 1) / KC)
#define NCELL (FH * CPR)                   // cells per chunk
#define KSTEPS ((NCELL + NKG - 1) / NKG)   // steps per chunk
#ifdef FB_PF
#define KSTEPS2 (KSTEPS + FB_PF)        // packed steps per chunk: PF zero steps after the real ones
#endif

static_assert(MF == 32 || MF == 16, "MFMA tiles are 32x32 or 16x16");
static_assert(!LIN || (DT != 0 && S * KC % 4 == 0), "KC must be PE times a power of two, or S*KC a multiple of 4 (16-bit)");
static_assert(KC % 4 == 0 || KC == CIN, "a channel count that is not a multiple of 4 cannot be cut into chunks");

// The three bf16 parts of eight fp32 values: h rounds x to nearest even, m
// the remainder x - h, l what is left (exact: 3 x 8 significant bits).
__device__ __forceinline__ void rg_split(const float* v, rg_u32x4& ch, rg_u32x4& cm, rg_u32x4& cl) {
    rg_bf16x8 h, m, l;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        h[i] = (__bf16)v[i];
        const float r = v[i] - (float)h[i];
        m[i] = (__bf16)r;
        l[i] = (__bf16)(r - (float)m[i]);
    }
    ch = __builtin_bit_cast(rg_u32x4, h);
    cm = __builtin_bit_cast(rg_u32x4, m);
    cl = __builtin_bit_cast(rg_u32x4, l);
}

// ------------------------------------------------------------------ pack
#if defined(FB_PACK_FRAG) || defined(FB_BATCHED)
// One workgroup per column pc of the packed bank: whole column blocks of
// the correlation kernel, NCOLW columns each, column (s, c) of a block
// holding filter c shifted by s taps (columns of filters at or past COUT
// are zero).  Layout: 16-byte cell (((j*NCHUNK + chunk)*KSTEPS2 + t)*NSP +
// part)*64 + lane for column tile j = pc / MF, step t = cell / NKG, lane =
// MF*(cell % NKG) + pc%MF.  16-bit operands and parts: e_c = floor(log2
// max|w[c]|), values scaled by 2^-e_c (exact) and rounded to nearest even,
// unscale[pc] = 2^e_c (an all-zero filter gets e_c = 0).  Parts: scaled by
// 2^s, s = WSH - e_c but at most 126 - XSH (filters below 2^-70 have bits to
// spare), unscale[pc] = 2^-(s+XSH), or 0 for a filter that the parts cannot
// hold.  FB_FLIP: the
// filters are those of the input-gradient correlation, read from the
// forward bank w[CIN][FH][FW][COUT] flipped in (u, v) with the channel axes
// exchanged.
// red: 4 floats of LDS.
static __device__ RG_PACK_ATTR void rg_pack(RG_GLOBAL const float* __restrict__ w_,
                                            RG_GLOBAL rg_u32x4* __restrict__ bp_,
                                            RG_GLOBAL float* __restrict__ unscale_, const int pc, RG_LDS float* red)
{
    const float* const w = (const float*)w_;
    rg_u32x4* const bp = (rg_u32x4*)bp_;
    float* const unscale = (float*)unscale_;
    // items: the cells (chunk, filter row, cell of the row), cell fastest; a
    // thread takes items tid, tid + 256, ...  When they fit (HELD), every
    // item's values are loaded once, all loads in flight together, and kept
    // for both the maximum and the packing; otherwise they are read twice.
    constexpr int ITEMS = NCHUNK * NCELL;
    constexpr int PER = (ITEMS + 255) / 256;
    constexpr bool HELD = PER * PE <= 64;
    const int j = pc / MF, col = pc % MF;
#ifdef FB_NCOLW
    // column (s, c) of its block
    const int sh = (pc % FB_NCOLW) / (FB_NCOLW / S);
    const int c = (pc / FB_NCOLW) * (FB_NCOLW / S) + (pc % FB_NCOLW) % (FB_NCOLW / S);
#else
    const int sh = 0, c = pc;
#endif
    const bool real = c < COUT;
    auto load_item = [&](int e, float* vals) {
        const int kci = e / NCELL, u = (e % NCELL) / CPR, cc = e % CPR;
#if KC % 4 != 0
#pragma unroll
        for (int i = 0; i < PE; ++i) {
            const int vf = (cc * PE + i) / KC - sh, ch = (cc * PE + i) % KC;      // one chunk
            const bool ok = e < ITEMS && real && vf >= 0 && vf < FW;
#ifdef FB_FLIP
            vals[i] = ok ? w[(((long)ch * FH + (FH - 1 - u)) * FW + (FW - 1 - vf)) * COUT + c] : 0.f;
#else
            vals[i] = ok ? w[(((long)c * FH + u) * FW + vf) * CIN + ch] : 0.f;
#endif
        }
        (void)kci;
#else
        // groups of 4 values stay within one tap
#pragma unroll
        for (int q = 0; q < PE; q += 4) {
            const int pos = cc * PE + q;
            const int vf = pos / KC - sh;             // filter tap of this (shifted) column
            const int ch0 = kci * KC + pos % KC;
            const bool ok = e < ITEMS && real && vf >= 0 && vf < FW;
#if !defined(FB_FLIP) && CIN % 4 == 0
            // consecutive channels of one tap: contiguous in w[c][u][v][:]
            rg_f32x4 x4 = {0.f, 0.f, 0.f, 0.f};
            if (ok && ch0 < CIN) x4 = *(const rg_f32x4*)(w + (((long)c * FH + u) * FW + vf) * CIN + ch0);
            vals[q] = x4[0]; vals[q + 1] = x4[1]; vals[q + 2] = x4[2]; vals[q + 3] = x4[3];
#else
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int ch = ch0 + i;
#ifdef FB_FLIP
                vals[q + i] = (ok && ch < CIN)
                                  ? w[(((long)ch * FH + (FH - 1 - u)) * FW + (FW - 1 - vf)) * COUT + c] : 0.f;
#else
                vals[q + i] = (ok && ch < CIN) ? w[(((long)c * FH + u) * FW + vf) * CIN + ch] : 0.f;
#endif
            }
#endif
        }
#endif
    };
    auto store_item = [&](int e, const float* vals, float sc) {
        if (e >= ITEMS) return;
        const int kci = e / NCELL, cell = e % NCELL;
        const int t = cell / NKG, g = cell % NKG;
        rg_u32x4* const dst = bp + (((long)j * NCHUNK + kci) * KSTEPS2 + t) * NSP * 64 + g * MF + col;
#if DT == 0
        (void)sc;
        dst[0] = __builtin_bit_cast(rg_u32x4, (rg_f32x4){vals[0], vals[1], vals[2], vals[3]});
#elif DT == 3
        float sv[PE];
#pragma unroll
        for (int i = 0; i < PE; ++i) sv[i] = vals[i] * sc;       // exact: power of two
        rg_u32x4 ch, cm, cl;
        rg_split(sv, ch, cm, cl);
        dst[0] = ch; dst[64] = cm; dst[128] = cl;
#else
        rg_u32x4 cell4;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float lo_v = vals[2 * i] * sc, hi_v = vals[2 * i + 1] * sc;   // exact: power of two
#if DT == 1
            const unsigned lo = __builtin_bit_cast(unsigned short, (__bf16)lo_v);
            const unsigned hi = __builtin_bit_cast(unsigned short, (__bf16)hi_v);
#else
            const unsigned lo = __builtin_bit_cast(unsigned short, (_Float16)lo_v);
            const unsigned hi = __builtin_bit_cast(unsigned short, (_Float16)hi_v);
#endif
            cell4[i] = lo | (hi << 16);
        }
        dst[0] = cell4;
#endif
    };

    float held[HELD ? PER : 1][PE];
    float m = 0.f;
    bool fin = true;                  // every value finite
    float lo = 3.402823466e38f;       // smallest non-zero magnitude of this thread
    auto scan = [&](const float* vals) {
#pragma unroll
        for (int q = 0; q < PE; ++q) {
            m = fmaxf(m, fabsf(vals[q]));
#if DT == 3
            fin = fin && fabsf(vals[q]) <= 3.402823466e38f;      // false for infinities and NaNs
            lo = vals[q] != 0.f ? fminf(lo, fabsf(vals[q])) : lo;
#endif
        }
    };
    if (HELD) {
#pragma unroll
        for (int i = 0; i < (HELD ? PER : 1); ++i) load_item(threadIdx.x + i * 256, held[i]);
#pragma unroll
        for (int i = 0; i < (HELD ? PER : 1); ++i) scan(held[i]);
    } else {
        for (int e = threadIdx.x; e < ITEMS; e += 256) {
            float vals[PE];
            load_item(e, vals);
            scan(vals);
        }
    }
    float sc = 1.0f;
#if DT != 0
    // e_c = floor(log2 max|w[c]|) over the filter's values (the padding
    // zeros change nothing)
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    fin = !__syncthreads_or(!fin);
    m = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    int ex = 0;
    if (fin && m > 0.f) {
        (void)frexpf(m, &ex);     // m = f * 2^ex, f in [0.5, 1)
        ex -= 1;                  // floor(log2 m)
    }
#if DT == 3
    const int se = WSH - ex < 126 - XSH ? WSH - ex : 126 - XSH;
    sc = ldexpf(1.0f, se);
    bool exact = fin && ex <= 24;
    // last bits below 2^-126 (the same branch in every thread)
    if (exact && se < 23) exact = !__syncthreads_or(lo * sc < 0x1p-103f);
    if (threadIdx.x == 0) unscale[pc] = exact ? ldexpf(1.0f, -(se + XSH)) : 0.f;
#else
    sc = ldexpf(1.0f, -ex);
    if (threadIdx.x == 0) unscale[pc] = real ? ldexpf(1.0f, ex) : 0.f;
#endif
#else
    (void)unscale;
    (void)m;
    (void)fin;
    (void)red;
#endif
    (void)lo;
    if (HELD) {
#pragma unroll
        for (int i = 0; i < (HELD ? PER : 1); ++i) store_item(threadIdx.x + i * 256, held[i], sc);
    } else {
        for (int e = threadIdx.x; e < ITEMS; e += 256) {
            float vals[PE];
            load_item(e, vals);
            store_item(e, vals, sc);
        }
    }
    // the zero cells after each chunk: the rest of its last step, and the
    // steps read by the ring's last refills
    constexpr int ZC = KSTEPS2 * NKG - NCELL;
    for (int e = threadIdx.x; e < NCHUNK * ZC * NSP; e += 256) {
        const int cell = NCELL + e % ZC, sp = (e / ZC) % NSP, kci = e / (ZC * NSP);
        const rg_u32x4 z = {0u, 0u, 0u, 0u};
        bp[((((long)j * NCHUNK + kci) * KSTEPS2 + cell / NKG) * NSP + sp) * 64 + (cell % NKG) * MF + col] = z;
    }
}
#endif  // pack

// ---------------------------------------------------------------- correlation
#ifndef FB_PACK_FRAG
#ifdef FB_HI
#define HI FB_HI
#define WI FB_WI
#define HO FB_HO
#define WO FB_WO
#else
#define HI hi_
#define WI wi_
#define HO ho_
#define WO wo_
#endif
#define PADH FB_PADH
#define PADW FB_PADW
#define MR FB_MR
#define MT FB_MT
#define NT FB_NT
#define WM FB_WM
#define WN FB_WN
#define PF FB_PF
#define XPADC FB_XPADC
#ifdef FB_WPE
#define WPE FB_WPE
#else
#define WPE 2
#endif

#define NREG (MF * MF / 64)           // accumulator registers per tile
#define MC (MF / MR)                  // pixel columns of a tile
#define TH (WM * MT * MR)             // output rows per workgroup
#define TWO (S * MC)                  // output columns per workgroup
#define NCOLW (WN * NT * MF)          // matrix columns per workgroup
#define CB (NCOLW / S)                // filters per workgroup
#define TR (TH + FH - 1)              // tile rows
#define TC (S * (MC - 1) + NTAPS)     // tile columns any lane reads
#define NTHREADS (WM * WN * 64)
// The tile in LDS, in units of UB bytes: planes of 16-byte cells, one cell
// per pixel (LIN 0), or rows of KC values per pixel in 8-byte units (LIN 1).
// In planes, a row holds the columns of each shift phase (column mod S)
// together: the lanes of a tile, S columns apart, then read neighbouring
// cells (without it a shift of 2 reads with a 32-byte stride, two bank
// conflicts per read).
#if LIN
#define UB 8
#define LSTEP (S * KC / 4)            // units from a lane's pixel to the next lane's
#define ITEM 4                        // values staged per item
#define ROWU ((TC * KC + 3) / 4)      // units of a tile row
#define RSU (ROWU + XPADC)            // tile row stride
#define SPU ((TR * RSU + 1) / 2 * 2)  // units per part (whole cells)
#define SITEMS (TR * ROWU)            // staging items
typedef rg_u32x2 rg_unit;
#else
#define UB 16
#define LSTEP 1
#define ITEM PE
#define PHASE ((TC + S - 1) / S)      // columns of a phase
#define COLPOS(cc) ((cc) % S * PHASE + (cc) / S)
#define RSU (S * PHASE + XPADC)
#define PLANE (TR * RSU)              // units per plane
#define SPU (NPL * PLANE)
#define SITEMS (NPL * TR * TC)
typedef rg_u32x4 rg_unit;
#endif
#define TILE_CELLS (NSP * SPU * UB / 16)
#if defined(FB_STE) && FB_STE
// Stores through LDS: per wave, one pixel tile's worth of its columns as
// rows of NT*MF floats (+8: the two lane groups' rows land on different
// banks), read back as 16-byte vectors
#define STE 1
#define SROW (NT * MF + 8)
#define SWAVE (MF * SROW)
#define STE_CELLS ((WM * WN * SWAVE + 3) / 4)
#define LDS_CELLS (TILE_CELLS > STE_CELLS ? TILE_CELLS : STE_CELLS)
#else
#define STE 0
#define LDS_CELLS TILE_CELLS
#endif
// items staged per thread and batch (all of them when they are few)
#define SMAX (64 / ITEM)
#define SCELLS ((SITEMS + NTHREADS - 1) / NTHREADS)
#define SB (SCELLS < SMAX ? SCELLS : SMAX)
// Lane group g of step t reads cell NKG*t + g.  When a row is a whole number
// of steps (SEP) the groups' offsets differ by a constant.
#define SEP (CPR % NKG == 0 && (LIN || NPL % NKG == 0 || (S == 1 && NKG % NPL == 0)))
// Steps after which the pattern of cell offsets repeats, PROWS filter rows
// further down; the step loop is unrolled over whole periods and over whole
// turns of the fragment ring (PF) and of the two A buffers.
#define PROWS (SEP ? 1 : NKG)
#define PSTEPS (PROWS * CPR / NKG)

static_assert(MF % MR == 0, "MR must divide MF");
static_assert(NCOLW % S == 0, "the columns must split evenly into shifts");
static_assert(!STE || S == 1, "stores through LDS need unshifted columns");
static_assert(PF >= 1, "ring depth");
static_assert(LIN || CIN % PE == 0 || KC == PE, "partial cells need KC == PE");

template <bool V> struct RgBool { static constexpr bool value = V; };

#if DT == 3
constexpr int rg_log2(long n) {            // rounded up
    int b = 0;
    while ((1L << b) < n) ++b;
    return b;
}
#define XHI (127 - XSH - (WSH + 1) - rg_log2((long)FH * FW * CIN))
#else
#define XHI 128                   // infinities and NaNs
#endif

#ifdef FB_BATCHED
template <typename T> __device__ __forceinline__ RG_GLOBAL T* rg_uniform(RG_GLOBAL T* p) {
    const unsigned long long a = (unsigned long long)p;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
    return (RG_GLOBAL T*)((unsigned long long)hi << 32 | lo);
}
#endif

#if MF == 32
typedef rg_f32x16 rg_acc;
#else
typedef rg_f32x4 rg_acc;
#endif

// fp16 input scale exponent k >= 0 from the 256 partial maxima of |x| (four
// per lane of the wave, combined by shuffles; the same in every lane).
__device__ __forceinline__ int rg_input_scale_exp(const float* __restrict__ UNSCALE) {
#if DT == 2 && defined(FB_XMOFF)
    const float* pm = UNSCALE + FB_XMOFF + 4 * (threadIdx.x & 63);
    float m = fmaxf(fmaxf(pm[0], pm[1]), fmaxf(pm[2], pm[3]));
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    int e = 0;
    if (m >= 32768.f) (void)frexpf(m, &e);    // m < 2^e
    return e > 15 ? e - 15 : 0;
#else
    (void)UNSCALE;
    return 0;
#endif
}

// Largest magnitude of the values staged by a thread, as a bit pattern (in
// the order of the magnitudes; infinities and NaNs above every finite value).
struct RgRange {
    unsigned hi = 0u;
    __device__ __forceinline__ void see(const float v) {
        const unsigned a = __builtin_bit_cast(unsigned, v) & 0x7fffffffu;
        hi = hi > a ? hi : a;
    }
    // some magnitude of 2^XHI or more
    __device__ __forceinline__ bool outside() const { return hi >= (127u + XHI) << 23; }
};

// Two values (fp16: scaled by xs, exact) rounded to nearest even, packed.
__device__ __forceinline__ unsigned rg_pair(const float a, const float b, const float xs) {
#if DT == 2
    const unsigned lo = __builtin_bit_cast(unsigned short, (_Float16)(a * xs));
    const unsigned hi = __builtin_bit_cast(unsigned short, (_Float16)(b * xs));
#else
    (void)xs;
    const unsigned lo = __builtin_bit_cast(unsigned short, (__bf16)a);
    const unsigned hi = __builtin_bit_cast(unsigned short, (__bf16)b);
#endif
    return lo | (hi << 16);
}

// One staged item (ITEM values) into the tile, every part of it.
__device__ __forceinline__ void rg_put(rg_unit* __restrict__ dst, const float* v, const float xs, RgRange& range) {
#if DT == 0
    (void)xs; (void)range;
    dst[0] = __builtin_bit_cast(rg_u32x4, (rg_f32x4){v[0], v[1], v[2], v[3]});
#elif DT == 3
    rg_unit h, m, l;
#pragma unroll
    for (int i = 0; i < ITEM / 2; ++i) {
        range.see(v[2 * i]);
        range.see(v[2 * i + 1]);
        const float a = v[2 * i] * xs, b = v[2 * i + 1] * xs;
        h[i] = rg_pair(a, b, xs);
        const float ra = a - __builtin_bit_cast(float, h[i] << 16);
        const float rb = b - __builtin_bit_cast(float, h[i] & 0xffff0000u);
        m[i] = rg_pair(ra, rb, xs);
        l[i] = rg_pair(ra - __builtin_bit_cast(float, m[i] << 16), rb - __builtin_bit_cast(float, m[i] & 0xffff0000u), xs);
    }
    dst[0] = h; dst[SPU] = m; dst[2 * SPU] = l;
#else
    rg_unit c;
#pragma unroll
    for (int i = 0; i < ITEM / 2; ++i) {
        if (GUARD) {
            range.see(v[2 * i]);
            range.see(v[2 * i + 1]);
        }
        c[i] = rg_pair(v[2 * i], v[2 * i + 1], xs);
    }
    dst[0] = c;
#endif
}

// The cell at unit offset o.
__device__ __forceinline__ rg_u32x4 rg_read(const rg_unit* __restrict__ tile, const int o) {
#if LIN && (LSTEP % 2 != 0 || RSU % 2 != 0)
    const rg_u32x2 p0 = tile[o], p1 = tile[o + 1];           // 8-byte aligned
    return (rg_u32x4){p0[0], p0[1], p1[0], p1[1]};
#elif LIN
    return *(const rg_u32x4*)(tile + o);
#else
    return tile[o];
#endif
}

// acc += A * B for one step of one (pixel tile, column tile) pair.
__device__ __forceinline__ void rg_mma(rg_acc& acc, const rg_u32x4 a, const rg_u32x4 b) {
#if DT == 0
    const rg_f32x4 af = __builtin_bit_cast(rg_f32x4, a);
    const rg_f32x4 bf = __builtin_bit_cast(rg_f32x4, b);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#if MF == 32
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af[q], bf[q], acc, 0, 0, 0);
#else
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(af[q], bf[q], acc, 0, 0, 0);
#endif
    }
#elif (DT == 1 || DT == 3) && MF == 32
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(rg_bf16x8, a), __builtin_bit_cast(rg_bf16x8, b),
                                                  acc, 0, 0, 0);
#elif DT == 1 || DT == 3
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(rg_bf16x8, a), __builtin_bit_cast(rg_bf16x8, b),
                                                  acc, 0, 0, 0);
#elif MF == 32
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(rg_f16x8, a), __builtin_bit_cast(rg_f16x8, b),
                                                 acc, 0, 0, 0);
#else
    acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(rg_f16x8, a), __builtin_bit_cast(rg_f16x8, b),
                                                 acc, 0, 0, 0);
#endif
}


// Orders the LDS accesses of a wave's lanes, and keeps control flow that
// some lanes skip from being moved across.
__device__ __forceinline__ void rg_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

constexpr int rg_lcm(int a, int b) {
    int m = a;
    while (m % b) m += a;
    return m;
}

#if GUARD
// The tile's outputs by plain fp32 fused multiply-adds from the filters as
// they are (16-bit operands: rounded as for the matrix units): for the rare
// tile whose values the bf16 parts cannot hold (16-bit: not finite).  A lane has one pixel and a wave SQ filters, the same in every lane: an input
// value that is loaded serves SQ products, and pixels outside the image take
// no part (their zeros would turn an infinite weight into a NaN).  With 8
// filters, 96x110x16 and 64 7x7 filters with a huge value in every tile 82
// us, fp32 instructions throughout 31 us, one filter at a time 1076 us.  The
// batched kernel's bodies are functions: past 30 scalar registers they save
// their return address, two scratch accesses per lane and tile (32 images of
// ordinary values: 2 % slower with 8 filters).
#ifdef FB_BATCHED
#define SQ 2
#define SKU 1
#else
#define SQ 8
#define SKU 2
#endif
// A value as the products hold it: itself (three parts), or scaled by s and
// rounded to nearest even.
__device__ __forceinline__ float rg_rounded(const float v, const float s) {
#if DT == 1
    return (float)(__bf16)(v * s);
#elif DT == 2
    return (float)(_Float16)(v * s);
#else
    (void)s;
    return v;
#endif
}
__device__ __forceinline__ void slow_tile(const float* __restrict__ Ib, const float* __restrict__ Wr,
                                          const float* __restrict__ us, float* __restrict__ Ob, const int hi_,
                                          const int wi_, const int ho_, const int wo_, const int oi0, const int oj0,
                                          const int c0, const float xs) {
    (void)us; (void)xs;
    (void)hi_; (void)wi_; (void)ho_; (void)wo_;
    constexpr int PGS = (TH * TWO + 63) / 64, QGS = (CB + SQ - 1) / SQ;
    constexpr int KV = CIN % 4 == 0 ? 4 : 1;                  // input values per load
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll 1
    for (int item = wave; item < PGS * QGS; item += NTHREADS / 64) {
        const int e = item % PGS * 64 + lane, cq = c0 + item / PGS * SQ;
        if (cq >= COUT) break;
        const int oi = oi0 + e / TWO, oj = oj0 + e % TWO;
        const bool real = e < TH * TWO && oi < HO && oj < WO;
        float acc[SQ], sc[SQ];
#pragma unroll
        for (int q = 0; q < SQ; ++q) {
            acc[q] = 0.f;
            sc[q] = DT == 3 ? 1.f : 1.f / us[cq + q < COUT ? cq - c0 + q : COUT - 1 - c0];
        }
#pragma unroll 1
        for (int u = 0; u < FH; ++u)
#pragma unroll 1
            for (int v = 0; v < FW; ++v) {
                const int ii = oi + u - PADH, jj = oj + v - PADW;
                if (real && ii >= 0 && ii < HI && jj >= 0 && jj < WI) {
                    const float* const px = Ib + ((long)ii * WI + jj) * CIN;
#pragma unroll SKU
                    for (int k = 0; k < CIN; k += KV) {
                        float xv[KV], wv[KV][SQ];
#pragma unroll
                        for (int i = 0; i < KV; ++i) xv[i] = rg_rounded(px[k + i], xs);
#pragma unroll
                        for (int q = 0; q < SQ; ++q) {
                            const int c = cq + q < COUT ? cq + q : COUT - 1;
#pragma unroll
                            for (int i = 0; i < KV; ++i)
#ifdef FB_FLIP
                                wv[i][q] = Wr[(((long)(k + i) * FH + (FH - 1 - u)) * FW + (FW - 1 - v)) * COUT + c];
#else
                                wv[i][q] = rg_rounded(Wr[(((long)c * FH + u) * FW + v) * CIN + k + i], sc[q]);
#endif
                        }
#pragma unroll
                        for (int i = 0; i < KV; ++i)
#pragma unroll
                            for (int q = 0; q < SQ; ++q) acc[q] = fmaf(xv[i], wv[i][q], acc[q]);
                    }
                }
            }
        if (real)
#pragma unroll
            for (int q = 0; q < SQ; ++q)
                if (cq + q < COUT && item / PGS * SQ + q < CB) {
                    float val = DT == 3 ? acc[q] : acc[q] / (sc[q] * xs);      // exact: powers of two
                    const int c = cq + q;
                    (void)c;
#ifdef FB_EPILOGUE
                    val = FB_EPILOGUE(val, c);
#endif
                    Ob[((long)oi * WO + oj) * COUT + c] = val;
                }
    }
}
#endif

// One output tile: rows oi0.., columns oj0.., column block cblk.  I and O
// point at the image's input and output, Bp at its packed bank, UNSCALE at
// the bank's column scales, Wr at the filters themselves.
__device__ __forceinline__ void rgemm_tile(
    const float* __restrict__ Ib, const rg_u32x4* __restrict__ Bp, const float* __restrict__ UNSCALE,
    const float* __restrict__ Wr, float* __restrict__ Ob, const int hi_, const int wi_, const int ho_, const int wo_,
    const int oi0, const int oj0, const int cblk, rg_u32x4* __restrict__ lds)
{
    (void)hi_; (void)wi_; (void)ho_; (void)wo_;
    const int c0 = cblk * CB;
    rg_unit* const tile = (rg_unit*)lds;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM;
    const int lr = lane % MF, g = lane / MF;       // tile row (pixel) / lane group
    const int ti = lr / MC, tj = lr % MC;
    // Unit offset of cell c of the chunk from a pixel's first cell.
    auto cell_off = [](const int c) -> int {
        const int u = c / CPR, cc = c % CPR;
#if LIN
        return u * RSU + cc * 2;
#else
        return u * RSU + (cc % NPL) * PLANE + COLPOS(cc / NPL);
#endif
    };
    // this lane's first pixel (pixel tile 0), and its group's share of an
    // offset when the groups differ by a constant
    const int lp = (wm * MT * MR + ti) * RSU + tj * LSTEP;
    const int lb = SEP ? lp + (g == 0 ? 0 : g == 1 ? cell_off(1) : g == 2 ? cell_off(2) : cell_off(3)) : lp;
    // offset of this lane's cell of step t; cells from lim on (the padding of
    // the last step) read cell lim - 1 instead
    auto step_off = [&](const int t, const int lim) -> int {
        const int o = cell_off(NKG * t);
        if (SEP) return o;
        auto off = [&](const int k) { return cell_off(NKG * t + k < lim ? NKG * t + k : lim - 1) - o; };
        return o + (g == 0 ? 0 : g == 1 ? off(1) : g == 2 ? off(2) : off(3));
    };
    // this wave's first column tile of the packed bank (which has whole
    // column blocks, so every tile a wave names exists)
    const int j0 = cblk * (NCOLW / MF) + wn * NT;
    const long jst = (long)NCHUNK * KSTEPS2 * NSP * 64;     // cells per column tile
    const rg_u32x4* bw = Bp + j0 * jst;                     // the same in every lane
    const unsigned boff = lane * 16;
    auto load_b = [&](const rg_u32x4* p) { return *(const rg_u32x4*)((const char*)p + boff); };

    rg_acc acc[MT][NT][NACC];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int k = 0; k < NACC; ++k)
#pragma unroll
                for (int r = 0; r < NREG; ++r) acc[mt][nt][k][r] = 0.f;

    // fp16: per-tensor input scale 2^-kx (1 unless the input reaches 2^15)
#if DT == 2
    const int kx = rg_input_scale_exp(UNSCALE);
    const float xs = ldexpf(1.f, -kx), ys = ldexpf(1.f, kx);
#elif DT == 3
    const float xs = (float)(1 << XSH), ys = 1.f;       // (undone in UNSCALE)
#else
    const float xs = 1.f, ys = 1.f;
#endif
    (void)ys; (void)Wr;
#if GUARD
    // a staged value (below), or with parts a filter of this block, that
    // slow_tile has to take
    bool odd = false;
#endif
#if DT == 3
    for (int i = tid; i < NCOLW; i += NTHREADS) odd = odd || UNSCALE[cblk * NCOLW + i] == 0.f;
#endif

#pragma unroll 1
    for (int kci = 0; kci < NCHUNK; ++kci) {
        const rg_u32x4* bc = bw + (long)kci * KSTEPS2 * NSP * 64;
        rg_u32x4 bq[PF][NT][NSP];
        // the first PF steps' fragments are in flight while the tile is staged
#pragma unroll
        for (int r = 0; r < PF; ++r)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int p = 0; p < NSP; ++p) bq[r][nt][p] = load_b(bc + nt * jst + (r * NSP + p) * 64);
        if (kci > 0) __syncthreads();        // every wave is done with the previous chunk
        // Stage the chunk's input tile: ITEM channels of input pixel
        // (oi0+r-PADH, oj0+cc-PADW) per item; zero outside the image and
        // past CIN.  In batches of SB items per thread, every load of a
        // batch issued before the first conversion (one memory latency per
        // batch, not per item).
        RgRange range;
#pragma unroll 1
        for (int e0 = 0; e0 < SITEMS; e0 += SB * NTHREADS) {
            float v[SB][ITEM];
            // item e: tile row r, column cc, channels kci*KC + q0..; its unit
            auto item = [&](const int e, int& r, int& cc, int& q0) -> int {
#if LIN
                const int q = e % ROWU;
                r = e / ROWU; cc = q * 4 / KC; q0 = q * 4 % KC;
                return r * RSU + q;
#else
                const int rc = e / NPL, p = e % NPL;
                cc = rc % TC; r = rc / TC; q0 = p * PE;
                return (p * TR + r) * RSU + COLPOS(cc);
#endif
            };
#pragma unroll
            for (int i = 0; i < SB; ++i) {
                const int e = e0 + i * NTHREADS + tid;
                int r, cc, q0;
                item(e, r, cc, q0);
                const int ii = oi0 + r - PADH, jj = oj0 + cc - PADW;
                const int ch = kci * KC + q0;
                const bool in = e < SITEMS && ii >= 0 && ii < HI && jj >= 0 && jj < WI;
                const float* src = Ib + ((long)ii * WI + jj) * CIN + ch;
#if KC % 4 != 0
                // an item may straddle pixels (of whole image rows in memory)
#pragma unroll
                for (int q = 0; q < ITEM; ++q) {
                    const int j2 = jj + (q0 + q) / KC;
                    v[i][q] = (e < SITEMS && ii >= 0 && ii < HI && j2 >= 0 && j2 < WI) ? src[q] : 0.f;
                }
                (void)in;
#elif CIN % 4 == 0
#pragma unroll
                for (int q = 0; q < ITEM; q += 4) {
                    rg_f32x4 x4 = {0.f, 0.f, 0.f, 0.f};
                    if (in && ch + q < CIN) x4 = *(const rg_f32x4*)(src + q);
                    v[i][q] = x4[0]; v[i][q + 1] = x4[1]; v[i][q + 2] = x4[2]; v[i][q + 3] = x4[3];
                }
#else
#pragma unroll
                for (int q = 0; q < ITEM; ++q) v[i][q] = (in && ch + q < CIN) ? src[q] : 0.f;
#endif
            }
#pragma unroll
            for (int i = 0; i < SB; ++i) {
                const int e = e0 + i * NTHREADS + tid;
                int r, cc, q0;
                const int dst = item(e, r, cc, q0);
                if (e < SITEMS) rg_put(tile + dst, v[i], xs, range);
            }
        }
#if GUARD
        odd = odd || range.outside();
#endif
        __syncthreads();

        // A fragments one step ahead of the products that use them
        rg_u32x4 a[2][MT][NSP];
        auto read_a = [&](const int base, const int t, const int lim, rg_u32x4 (&dst)[MT][NSP]) {
            const int o = lb + base + step_off(t, lim);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int p = 0; p < NSP; ++p) dst[mt][p] = rg_read(tile, o + mt * MR * RSU + p * SPU);
        };
        // What meets zero weights -- the values past a row's taps, and (end:
        // the chunk's last steps) the cells past the last -- is zeroed before
        // its products: an infinity there would make them NaNs.
        auto mask_a = [&](const int t, const int lim, rg_u32x4 (&src)[MT][NSP], auto end) {
            constexpr int KEEP = PE - (CPR * PE - NTAPF * KC), PER = PE / 4;
#pragma unroll
            for (int k = 0; k < NKG; ++k) {
                const int c = NKG * t + k;
                const bool past = decltype(end)::value && c >= lim;
                if (past || (KEEP < PE && c % CPR == CPR - 1)) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const unsigned m = past || i * PER >= KEEP ? 0u : (i + 1) * PER > KEEP ? 0xffffu : ~0u;
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt) src[mt][0][i] &= g == k ? m : ~0u;
                    }
                }
            }
        };
        read_a(0, 0, NCELL, a[0]);

        // One step, t past unit offset base: read the next step's A fragments
        // (step tn, lim cells left there), the products of this one, then refill this ring slot
        // with the fragments PF steps ahead (the packed bank has PF zero
        // steps after each chunk, so the refill needs no bounds test).
        auto step = [&](const int base, const int t, const int tn, const int lim, const rg_u32x4* brow, const int r,
                        const int ab, auto end) {
            if (!GUARD) mask_a(t, lim, a[ab], end);
            read_a(base, tn, lim, a[ab ^ 1]);
#if DT == 3
            // the small products first; neighbouring instructions on
            // different tiles
            constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
            for (int q = 0; q < 6; ++q)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
                        rg_mma(acc[mt][nt][q < 5], a[ab][mt][PA[q]], bq[r][nt][PB[q]]);
#else
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) rg_mma(acc[mt][nt][0], a[ab][mt][0], bq[r][nt][0]);
#endif
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int p = 0; p < NSP; ++p) bq[r][nt][p] = load_b(brow + nt * jst + (PF * NSP + p) * 64);
            // Keep this order (LDS reads, products, refill loads) and keep
            // each step's instructions within the step: left free, the
            // scheduler sinks the refills next to their use, which leaves
            // the ring one step deep.
            __builtin_amdgcn_sched_group_barrier(0x100, MT * NSP, 0);                         // LDS reads
            __builtin_amdgcn_sched_group_barrier(0x008, MT * NT * (DT == 0 ? 4 : DT == 3 ? 6 : 1), 0);   // products
            __builtin_amdgcn_sched_group_barrier(0x020, NT * NSP, 0);                         // global loads
            __builtin_amdgcn_sched_barrier(0);
        };
        // whole groups of G steps (the ring slot, the A buffer and the
        // pattern of offsets repeat with that period), then the rest,
        // unrolled; the last step of all has no next one, and the one before
        // it reads the padded step
        constexpr int GL = rg_lcm(PSTEPS, rg_lcm(PF, 2));
        // (a long period is cut to whole ring turns, its offsets computed)
        constexpr bool PERIODIC = GL <= 64;
        constexpr int G = PERIODIC ? GL : rg_lcm(PF, 2);
        constexpr int NG = (KSTEPS - (NCELL % NKG ? 2 : 1)) / G;
        int base = 0;
#if defined(FB_UNR) && FB_UNR
#pragma unroll
#else
#pragma unroll 1
#endif
        for (int gi = 0; gi < NG; ++gi) {
            const rg_u32x4* bg = bc + (long)gi * G * NSP * 64;
            const int t0 = PERIODIC ? 0 : gi * G;
#pragma unroll
            for (int r2 = 0; r2 < G; ++r2) step(base, t0 + r2, t0 + r2 + 1, NCELL, bg + r2 * NSP * 64, r2 % PF, r2 & 1, RgBool<false>{});
            if (PERIODIC) base += G / PSTEPS * PROWS * RSU;
        }
        constexpr int REST = KSTEPS - NG * G;
        const rg_u32x4* br = bc + (long)NG * G * NSP * 64;
        const int tr0 = PERIODIC ? 0 : NG * G, lim = PERIODIC ? NCELL - NG * G * NKG : NCELL;
#pragma unroll
        for (int r2 = 0; r2 < REST; ++r2)
            step(base, tr0 + r2, tr0 + (r2 + 1 < REST ? r2 + 1 : r2), lim, br + r2 * NSP * 64, r2 % PF, r2 & 1,
                 RgBool<true>{});
    }
#if GUARD
    // (the same decision in every wave of the workgroup)
    if (__builtin_amdgcn_readfirstlane(__syncthreads_or(odd))) {
        slow_tile(Ib, Wr, UNSCALE + cblk * NCOLW, Ob, hi_, wi_, ho_, wo_, oi0, oj0, c0, xs);
        return;
    }
#endif
#if DT == 3
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int r = 0; r < NREG; ++r) acc[mt][nt][0][r] += acc[mt][nt][1][r];
#endif

    // Epilogue.  Accumulator layouts: 32x32 -- lane l, register r holds tile
    // row 8*(r/4) + 4*(l/32) + r%4 and column l%32; 16x16 -- row 4*(l/16) + r
    // and column l%16.  Workgroups whose tile lies inside the output store
    // without per-element bounds tests.
    const bool interior = oi0 + TH <= HO && oj0 + TWO <= WO && c0 + CB <= COUT;
#if !STE
    auto store_all = [&](auto checked) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int col = (wn * NT + nt) * MF + lr;       // matrix column: (shift, filter)
            const int sh = col / CB, cc = c0 + col % CB;
#if DT != 0
            const float us = (!decltype(checked)::value || cc < COUT) ? UNSCALE[cblk * NCOLW + col] * ys : 0.f;   // exact: powers of two
#endif
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
                for (int r = 0; r < NREG; ++r) {
#if MF == 32
                    const int m = 8 * (r >> 2) + 4 * g + (r & 3);
#else
                    const int m = 4 * g + r;
#endif
                    const int oi = oi0 + (wm * MT + mt) * MR + m / MC;
                    const int oj = oj0 + S * (m % MC) + sh;
                    if (!decltype(checked)::value || (oi < HO && oj < WO && cc < COUT)) {
#if DT == 0
                        float val = acc[mt][nt][0][r];
#else
                        float val = acc[mt][nt][0][r] * us;
#endif
#ifdef FB_EPILOGUE
                        val = FB_EPILOGUE(val, cc);
#endif
                        // unsigned 32-bit offset from the image's base: a
                        // scalar base plus a vector offset per store
                        float* const dst = Ob + (unsigned)((oi * WO + oj) * COUT + cc);
#if defined(FB_NTS) && FB_NTS
                        // streaming store: the output is not read again here,
                        // and leaving L2 to the filter fragments and input
                        // tiles that every workgroup re-reads
                        __builtin_nontemporal_store(val, dst);
#else
                        *dst = val;
#endif
                    }
                }
            }
        }
    };
    if (interior) store_all(RgBool<false>{});
    else store_all(RgBool<true>{});
#else
    // Stores through LDS: each pixel tile of the wave's columns goes to
    // the wave's own LDS rows (the input tile is dead once every wave is
    // past its last step) and back out as 16-byte vectors, so that one
    // store instruction writes whole runs of a pixel's channels.  A vector
    // exists as a whole (COUT is a multiple of 4); those of pixels past
    // the image edge and of channels past COUT are skipped.
    __syncthreads();
    float* const sbuf = (float*)lds + wave * SWAVE;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int col = (wn * NT + nt) * MF + lr;
#if DT != 0
            const float us = UNSCALE[cblk * NCOLW + col] * ys;      // exact: powers of two
#endif
#pragma unroll
            for (int r = 0; r < NREG; ++r) {
#if MF == 32
                const int m = 8 * (r >> 2) + 4 * g + (r & 3);
#else
                const int m = 4 * g + r;
#endif
#if DT == 0
                float val = acc[mt][nt][0][r];
#else
                float val = acc[mt][nt][0][r] * us;
#endif
#ifdef FB_EPILOGUE
                const int ch = c0 + col;      // (the macro's argument is used as it is)
                val = FB_EPILOGUE(val, ch);
#endif
                sbuf[m * SROW + nt * MF + lr] = val;
            }
        }
        // (the rows are exchanged between the lanes of the wave: every
        // lane's writes come before any lane's reads, and those before
        // the next tile's writes)
        rg_wave_sync();
        // MF rows of NT*MF/4 vectors, 64 per instruction
#pragma unroll
        for (int it = lane; it < MF * NT * MF / 4; it += 64) {
            const int m = it / (NT * MF / 4), c4 = it % (NT * MF / 4);
            const rg_f32x4 v = *(const rg_f32x4*)(sbuf + m * SROW + c4 * 4);
            const int oi = oi0 + (wm * MT + mt) * MR + m / MC;
            const int oj = oj0 + m % MC;
            rg_f32x4* const dst =
                (rg_f32x4*)(Ob + (unsigned)((oi * WO + oj) * COUT + c0 + wn * NT * MF + c4 * 4));
            if (interior || (oi < HO && oj < WO && c0 + wn * NT * MF + c4 * 4 < COUT)) {
#if defined(FB_NTS) && FB_NTS
                __builtin_nontemporal_store(v, dst);
#else
                *dst = v;
#endif
            }
        }
        rg_wave_sync();
    }
#endif
}

#ifdef FB_BATCHED
// Tile t of an image (tile column fastest, then tile row, then column block);
// the wave ends here, so that nothing waits for the tile's stores.  The
// arguments arrive in vector registers: the same in every lane, they are put
// back in scalar ones.  Pointers keep their address space (through generic
// ones the fragment loads become flat loads, which every LDS wait includes).
// A local function that is never tail-called keeps no register for its
// caller: without that attribute a tile first stored about 100 registers per
// lane, more bytes than its outputs (387x506x3, 64 5x5: 73 us).
static __device__ __attribute__((noinline)) __attribute__((not_tail_called)) void rgemm_body(
    RG_GLOBAL const float* I, RG_GLOBAL const rg_u32x4* Bp, RG_GLOBAL const float* UNSCALE, RG_GLOBAL const float* Wr,
    RG_GLOBAL float* O, int hi_, int wi_, int ho_, int wo_, int t, RG_LDS rg_u32x4* lds)
{
    hi_ = __builtin_amdgcn_readfirstlane(hi_); wi_ = __builtin_amdgcn_readfirstlane(wi_);
    ho_ = __builtin_amdgcn_readfirstlane(ho_); wo_ = __builtin_amdgcn_readfirstlane(wo_);
    t = __builtin_amdgcn_readfirstlane(t);
    const int ntx = (WO + TWO - 1) / TWO, nty = (HO + TH - 1) / TH;
    const int tx = t % ntx, ty = t / ntx % nty, cblk = t / (ntx * nty);
    rgemm_tile((const float*)rg_uniform(I), (const rg_u32x4*)rg_uniform(Bp), (const float*)rg_uniform(UNSCALE),
               (const float*)rg_uniform(Wr), (float*)rg_uniform(O), hi_, wi_, ho_, wo_, ty * TH, tx * TWO, cblk,
               (rg_u32x4*)lds);
    __builtin_amdgcn_endpgm();
    __builtin_unreachable();
}
#endif
#endif  // !FB_PACK_FRAG
//@@BODY-END

#if defined(FB_PACK_FRAG)
extern "C" __global__ void __launch_bounds__(256)
fbcorr_pack_frag(const float* __restrict__ w, rg_u32x4* __restrict__ bp, float* __restrict__ unscale)
{
    __shared__ float red[4];
    rg_pack(w, bp, unscale, blockIdx.x, red);
}
#elif !defined(FB_BATCHED)
#define BATCH FB_BATCH
extern "C" __global__ void __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(WPE, WPE)))
FB_KNAME(const float* __restrict__ I, const rg_u32x4* __restrict__ Bp, const float* __restrict__ UNSCALE,
         float* __restrict__ O, const float* __restrict__ Wr)
{
    __shared__ rg_u32x4 lds[LDS_CELLS];
    // Workgroup -> (image, column block, tile row, tile column); with XCDMAP
    // each XCD gets a contiguous range (shared halos stay in its L2).
    const int ntx = (WO + TWO - 1) / TWO;
    const int nty = (HO + TH - 1) / TH;
    const int ncb = (COUT + CB - 1) / CB;
    const int total = ntx * nty * ncb * BATCH;
    int lin = blockIdx.x;
#if FB_XCDMAP
    {
        const int q = total / 8, r = total % 8, x = lin % 8;
        lin = x * q + (x < r ? x : r) + lin / 8;
    }
#endif
    const int tx = lin % ntx;
    const int ty = (lin / ntx) % nty;
    const int cblk = (lin / (ntx * nty)) % ncb;
    const int b = lin / (ntx * nty * ncb);
    rgemm_tile(I + (long)b * HI * WI * CIN, Bp, UNSCALE, Wr, O + (long)b * HO * WO * COUT,
               HI, WI, HO, WO, ty * TH, tx * TWO, cblk, lds);
}
#endif

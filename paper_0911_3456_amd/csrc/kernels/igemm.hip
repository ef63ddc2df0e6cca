// Implicit-GEMM valid correlation on the CDNA matrix cores (MFMA).
//
//   O[b,i,j,c] = sum_{u<FH, v<FW, k<CIN} Ipad[b, i+u, j+v, k] * Wt[c, u, v, k]
//
// where Ipad is the input I[b][HI][WI][CIN] with PADH/PADW rows/columns of
// virtual zeros on every side.  With I = x, Wt = w and no padding this is the
// forward filter-bank correlation of Sec. 6.2; with I = dy, Wt = w flipped in
// (u, v) and transposed n <-> d, and padding (FH-1, FW-1), it is the input
// gradient.  GEMM view: rows = output pixels, columns = output channels,
// contraction over (u, v, k).  A (the im2col matrix) is never materialised:
// for a fixed filter row u the (v, k) pairs of one output pixel are one
// contiguous run of FW*KC values in the LDS input tile, so each lane reads
// its A fragment straight from the staged tile.
//
// Tiles.  An MF-row MFMA tile (MF = 32 or 16) is MF "base pixels" laid out
// as MR rows x MC columns (MC = MF/MR).  Column-shift packing: when COUT is
// smaller than the MF MFMA columns, a column is a pair (c, s), s < S, computing output column
// S*tj + s for base pixel column tj; the contraction then runs over FW+S-1
// taps per filter row with B[(u, v', k), (c, s)] = Wt[c, u, v'-s, k] (zero
// outside 0 <= v'-s < FW).  A wave holds MT x NT tiles; WM x WN waves cover
// the workgroup's output tile; KS groups of such waves split the contraction
// (each group owns its own LDS buffers and a contiguous range of (channel
// chunk, filter-row stage) units) and add their accumulators in a fixed
// order at the end.  Filter slices are double-buffered in LDS and the next
// slice is fetched into registers while the current one is consumed
// (pre-fetching and software pipelining, Sec. 6.2).
//
// Compile-time constants (Sec. 4.2 "hardcoding", Sec. 5.3 keyword
// substitution), passed as FB_<name>:
//   problem  BATCH FH FW CIN COUT HI WI HO WO PADH PADW
//   tiling   MF (MFMA tile: 32 -> 32x32, 16 -> 16x16; default 32)
//            KC (channels per chunk)  S (column shift)  MR (tile rows)
//            MT NT (tiles per wave)  WM WN (waves)  KS (contraction split)
//            USTAGE (filter rows per stage)  XPAD WPAD (LDS row padding)
//            XCDMAP (XCD-aware workgroup order)
//            SWZ (1: 16-bit tiles in 16-channel chunks with the channel halves
//            of every other group of eight pixels exchanged, see SWZ_E)
//            UUNR (1: unroll the loop over the filter rows of a stage, so
//            the loads of one row are scheduled under the products of the
//            previous one)
//   naming   KNAME (kernel symbol)  TAG (suffix of this variant's device
//            functions)
//   EPILOGUE(v, c)  optional elementwise function of an output value v and
//            its channel c, applied before the store (a fused nonlinearity)
//
// Everything between the BODY markers is one variant's device code.  The
// batched kernel is generated by pasting this section once per
// distinct problem key, with TAG set and the image extents left run-time,
// followed by the kernel that calls them (FB_BATCHED then omits the kernel below).
//   type     DT: 0 = fp32 operands (v_mfma 32x32x2 f32), 1 = bf16, 2 = fp16
//            (32x32x16 with 8 operands per lane; Wt is then pre-scaled and
//            pre-rounded 16-bit and UNSCALE[c] multiplies each output)
//   XMOFF    fp16 only: UNSCALE[XMOFF .. XMOFF+255] hold partial maxima of |x|
//            (fbcorr_absmax); when the input reaches 2^15 it is scaled by
//            2^-k while staged (max |x| * 2^-k < 2^15, inside the fp16
//            range) and the outputs by 2^k -- both exact powers of two
#ifndef __HIPCC_RTC__
#include <hip/hip_runtime.h>
#endif

#ifdef FB_INJECT_ERROR
#error "injected code-generation failure (test hook)"
#endif
#ifndef FBC_IGEMM_COMMON
#define FBC_IGEMM_COMMON
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));
#endif

#ifndef FB_TAG
#define FB_TAG single
#endif

// In the batched kernel each variant's body is its own function:
// inlined into one kernel, dozens of bodies defeat the register
// allocator (hundreds of spills even though no single body needs them).
#ifndef FB_BODY_ATTR
#ifdef FB_BATCHED
#define FB_BODY_ATTR __attribute__((noinline))
#else
#define FB_BODY_ATTR __forceinline__
#endif
#endif

//@@BODY-BEGIN
// Specialisation constants arrive as FB_<name> (see the host generator).
// The image extents may instead be run-time values (the batched
// kernel): then the body reads its hi_/wi_/ho_/wo_ arguments.
#define FH FB_FH
#define FW FB_FW
#define CIN FB_CIN
#define COUT FB_COUT
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
#define KC FB_KC
#define S FB_S
#define MR FB_MR
#define MT FB_MT
#define NT FB_NT
#define WM FB_WM
#define WN FB_WN
#define KS FB_KS
#define DT FB_DT
#define XPAD FB_XPAD
#define WPAD FB_WPAD
#define USTAGE FB_USTAGE
#ifdef FB_MF
#define MF FB_MF
#else
#define MF 32
#endif
#ifdef FB_SWZ
#define SWZ FB_SWZ
#else
#define SWZ 0
#endif
// per-variant names: IGN(x) pastes the variant tag onto x
#define IGN_PASTE_(a, b) a##_##b
#define IGN_PASTE(a, b) IGN_PASTE_(a, b)
#define IGN(a) IGN_PASTE(a, FB_TAG)

// MFMA tile: MF x MF outputs (32 or 16); NKG lane groups split the
// contraction of one instruction; NREG accumulator registers per lane.
#define NKG (64 / MF)
#define NREG (MF * MF / 64)
#define MC (MF / MR)              // base-pixel columns of one MFMA tile
#define GWAVES (WM * WN)          // waves per contraction group
#define NTHREADS (GWAVES * KS * 64)
#define GTHREADS (GWAVES * 64)
#define TH (WM * MT * MR)         // output rows per workgroup
#define TWO (S * MC)              // output columns per workgroup
#define NCOL (WN * NT * MF)       // MFMA columns per workgroup
#define CB (NCOL / S)             // output channels per workgroup
#define TR (TH + FH - 1)          // input tile rows
#define KRRAW ((FW + S - 1) * KC) // contraction run per filter row and chunk
#if DT == 0
#define RUNIT (NKG * 4)
#else
#define RUNIT (NKG * 8)
#endif
#define KR (((KRRAW + RUNIT - 1) / RUNIT) * RUNIT)
#define HALF (KR / NKG)                 // contraction run of one lane group
#define ROWE ((MC - 1) * S * KC + KR)   // tile row elements any lane may read
#define ROWS (ROWE + XPAD)              // tile row stride
// Filter slice: one row per output channel of the block holding the FW*KC
// filter values of a filter row and channel chunk between (S-1)*KC zeros on
// the left and KR-FW*KC zeros on the right.  A lane of shift s reads the row
// starting s*KC to the left, which realises B[(u,v',k),(c,s)] = Wt[c,u,v'-s,k]
// (zero outside the filter) without staging S shifted copies.
#define RAWW ((S - 1) * KC)
#define WREAL (FW * KC)
#define WRS (RAWW + KR + WPAD)          // filter-slice row stride
#define TILE_ELEMS (((TR * ROWS) + 7) / 8 * 8)
#define WSL_ELEMS (USTAGE * CB * WRS)
#define NCHUNK ((CIN + KC - 1) / KC)
#define NUS ((FH + USTAGE - 1) / USTAGE)      // filter-row stages per chunk
#define NUNITS (NCHUNK * NUS)                 // contraction units
#define UPG ((NUNITS + KS - 1) / KS)          // units per group
#define GROUP_ELEMS (((TILE_ELEMS + 2 * WSL_ELEMS) + 7) / 8 * 8)
// filter-slice staging: groups of 4 consecutive kr (same tap, 4 channels)
#define WVEC ((KC % 4 == 0 && CIN % 4 == 0) ? 4 : 1)
#ifdef FB_FLIPW
// Input gradient with the flip fused into the staging: Wt points at the
// forward bank w[CIN][FH][FW][COUT] and the filters used are
// w[k][FH-1-u][FW-1-v][c].  An item is FVEC consecutive output channels of
// one (u, v, k): one load along the channels of w, scattered to FVEC rows.
#define FLIPW 1
#define FVEC ((COUT % 4 == 0 && CB % 4 == 0) ? 4 : 1)
#define WITEMS (USTAGE * FW * KC * (CB / FVEC))
#else
#define FLIPW 0
#define WITEMS (USTAGE * CB * (WREAL / WVEC))
#endif
#define ZW (RAWW + KR - WREAL)          // zero entries per filter-slice row
#define WPER ((WITEMS + GTHREADS - 1) / GTHREADS)

#if DT == 0
#define ELEM_T float
#define WVEC_T f32x4                // 4 fp32 filter values
#define ESZ 4
#else
#define ELEM_T unsigned short       // raw 16-bit patterns
#define WVEC_T u16x4                // 4 16-bit filter values
#define ESZ 2
#endif
// the split-K reduction reuses the LDS of groups 1..KS-1 (fp32 accumulators)
#define RED_FLOATS ((KS - 1) * GWAVES * MT * NT * NREG * 64)
#define LDS_ELEMS_LOOP (KS * GROUP_ELEMS)
#define LDS_BYTES_LOOP (LDS_ELEMS_LOOP * ESZ)
#define LDS_BYTES ((LDS_BYTES_LOOP > RED_FLOATS * 4) ? LDS_BYTES_LOOP : RED_FLOATS * 4)

// A-read vector width (elements) from the lane-to-lane stride S*KC.
#if DT == 0
#define AV (((S * KC) % 4 == 0) ? 4 : (((S * KC) % 2 == 0) ? 2 : 1))
#else
#define AV (((S * KC) % 8 == 0) ? 8 : (((S * KC) % 4 == 0) ? 4 : (((S * KC) % 2 == 0) ? 2 : 1)))
#endif

static_assert(MF == 32 || MF == 16, "MFMA tiles are 32x32 or 16x16");
// Tile swizzle (16-bit operands, 16-channel chunks): a pixel's 32 bytes are
// two 16-byte halves, and in every other group of eight pixel columns the
// halves are exchanged.  Sixteen lanes reading the same half of sixteen
// consecutive pixels (a 32-byte stride, two-way bank conflicts) then hit
// sixteen distinct 16-byte bank groups.  Element index e within a tile row.
#if SWZ
static_assert(DT != 0 && KC == 16 && AV == 8, "the tile swizzle is for 16-bit operands in 16-channel chunks");
#define SWZ_E(e) ((e) ^ ((((e) >> 7) & 1) << 3))
#else
#define SWZ_E(e) (e)
#endif
static_assert(MF % MR == 0, "MR must divide the tile rows");
static_assert(NCOL % S == 0, "columns must split evenly into shifts");
static_assert(ROWS % AV == 0, "tile rows must keep the A reads aligned");
// B-read vector width (elements): the shift offset (S-1-s)*KC must keep it aligned.
#if DT == 0
#define BV ((S == 1 || KC % 4 == 0) ? 4 : ((KC % 2 == 0) ? 2 : 1))
#else
#define BV ((S == 1 || KC % 8 == 0) ? 8 : ((KC % 4 == 0) ? 4 : ((KC % 2 == 0) ? 2 : 1)))
#endif
static_assert(WRS % BV == 0, "filter rows must keep the B reads aligned");

// fp16 input scale exponent k >= 0 from the 256 partial maxima of |x| (four
// per lane of the wave, combined by shuffles; the same in every lane).
__device__ __forceinline__ int IGN(input_scale_exp)(const float* __restrict__ UNSCALE) {
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

__device__ __forceinline__ ELEM_T IGN(to_elem)(float v) {
#if DT == 0
    return v;
#elif DT == 1
    __bf16 h = (__bf16)v;                 // round to nearest even
    return __builtin_bit_cast(unsigned short, h);
#else
    _Float16 h = (_Float16)v;             // round to nearest even
    return __builtin_bit_cast(unsigned short, h);
#endif
}


// One staged filter slice item: 4 (or 1) consecutive (v, k) values of one
// output channel.
__device__ __forceinline__ void IGN(w_item)(int e, int kc0, int u0, int c0, int& dst, bool& ok, long& src) {
    const int per_c = WREAL / WVEC;
    const int uu = e / (CB * per_c);
    const int rem = e % (CB * per_c);
    const int c = rem / per_c;
    const int kr = (rem % per_c) * WVEC;
    const int v = kr / KC, k = kr % KC;
    const int u = u0 + uu, cc = c0 + c, ch = kc0 + k;
    ok = (u < FH && cc < COUT && ch < CIN);
    src = ((((long)cc * FH + u) * FW + v) * CIN + ch);
    dst = (uu * CB + c) * WRS + RAWW + kr;
}

#if FLIPW
static_assert(DT == 0, "the fused flip is fp32 only");
// One item of the fused-flip staging: channels c0+cq*FVEC.. of tap (u, v),
// input channel k; dst0 is the LDS position of the first channel's row.
__device__ __forceinline__ void IGN(wf_item)(int e, int kc0, int u0, int c0, int& dst0, bool& ok, long& src) {
    const int cq = e % (CB / FVEC);
    int r = e / (CB / FVEC);
    const int k = r % KC;
    r /= KC;
    const int v = r % FW, uu = r / FW;
    const int u = u0 + uu, cc = c0 + cq * FVEC, ch = kc0 + k;
    ok = (u < FH && cc < COUT && ch < CIN);
    src = (((long)ch * FH + (FH - 1 - u)) * FW + (FW - 1 - v)) * COUT + cc;
    dst0 = (uu * CB + cq * FVEC) * WRS + RAWW + v * KC + k;
}
#endif

// The (chunk, stage) of unit q.
__device__ __forceinline__ void IGN(unit_of)(int q, int& kci, int& us) {
    kci = q / NUS;
    us = q % NUS;
}

// One output tile of this variant: rows oi0.., columns oj0.., channels c0..
// I and O point at the image's input and output.
__device__ FB_BODY_ATTR void IGN(igemm_body)(
    const float* __restrict__ I, const ELEM_T* __restrict__ Wt, const float* __restrict__ UNSCALE,
    float* __restrict__ O, const int hi_, const int wi_, const int ho_, const int wo_,
    const int oi0, const int oj0, const int c0, unsigned char* __restrict__ lds_raw)
{
    (void)hi_; (void)wi_; (void)ho_; (void)wo_;

    ELEM_T* const lds = (ELEM_T*)lds_raw;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int kg = wave / GWAVES;             // contraction group
    const int gw = wave % GWAVES;             // wave within the group
    const int gtid = tid % GTHREADS;          // thread within the group
    const int wm = gw % WM;
    const int wn = gw / WM;
    const int l32 = lane % MF;                // tile row (A) / column (B) of this lane
    const int h = lane / MF;                  // contraction group of this lane
    const int ti = l32 / MC, tj = l32 % MC;   // this lane's base pixel in a tile

    ELEM_T* const tile = lds + kg * GROUP_ELEMS;
    ELEM_T* const wsl0 = tile + TILE_ELEMS;
#if SWZ
    // swizzled element offsets of this lane's A run, one per 8-element step
    // (the run start depends on the lane only)
    int aoff[HALF / 8];
#pragma unroll
    for (int i = 0; i < HALF / 8; ++i) aoff[i] = SWZ_E(S * tj * KC + h * HALF + 8 * i);
#endif

    // fp16: per-tensor input scale 2^-kx (1 unless the input reaches 2^15)
#if DT == 2
    const int kx = IGN(input_scale_exp)(UNSCALE);
    const float xs = ldexpf(1.f, -kx), ys = ldexpf(1.f, kx);
#else
    constexpr float xs = 1.f, ys = 1.f;
#endif
    (void)xs; (void)ys;

    // every item starts after the previous item is done with the LDS
    __syncthreads();

#if MF == 32
    f32x16 acc[MT][NT];
#else
    f32x4 acc[MT][NT];
#endif
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int r = 0; r < NREG; ++r) acc[mt][nt][r] = 0.0f;

    // Stage the group's input tile for a channel chunk (virtual zero padding,
    // zero fill past the data).
    auto load_tile = [&](int kc0) {
#if (KC % 4 == 0) && (CIN % 4 == 0)
        for (int e = gtid * 4; e < TR * ROWE; e += GTHREADS * 4) {
            const int r = e / ROWE, q = e % ROWE;
            const int tc = q / KC, k = q % KC;
            const int ii = oi0 + r - PADH, jj = oj0 + tc - PADW, ch = kc0 + k;
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
            if (ii >= 0 && ii < HI && jj >= 0 && jj < WI && ch < CIN)
                v = *(const f32x4*)(I + ((long)ii * WI + jj) * CIN + ch);
            ELEM_T* dst = tile + r * ROWS + SWZ_E(q);
#if DT == 0
            dst[0] = v[0]; dst[1] = v[1]; dst[2] = v[2]; dst[3] = v[3];
#else
            // one 8-byte store of the four converted values (ROWS and q are
            // multiples of four): 2-byte stores from neighbouring lanes would
            // share LDS banks
            static_assert(ROWS % 4 == 0, "8-byte tile stores need rows in whole groups of four");
            const u16x4 h = {IGN(to_elem)(v[0] * xs), IGN(to_elem)(v[1] * xs), IGN(to_elem)(v[2] * xs),
                             IGN(to_elem)(v[3] * xs)};
            *(u16x4*)dst = h;
#endif
        }
#else
        for (int e = gtid; e < TR * ROWE; e += GTHREADS) {
            const int r = e / ROWE, q = e % ROWE;
            const int tc = q / KC, k = q % KC;
            const int ii = oi0 + r - PADH, jj = oj0 + tc - PADW, ch = kc0 + k;
            float v = 0.f;
            if (ii >= 0 && ii < HI && jj >= 0 && jj < WI && ch < CIN)
                v = I[((long)ii * WI + jj) * CIN + ch];
            tile[r * ROWS + SWZ_E(q)] = IGN(to_elem)(v * xs);
        }
#endif
    };

    // Filter-slice prefetch registers.
    WVEC_T wreg[WPER];
    auto fetch_w = [&](int q) {
        int kci, us;
        IGN(unit_of)(q, kci, us);
#pragma unroll
        for (int i = 0; i < WPER; ++i) {
            const int e = gtid + i * GTHREADS;
            WVEC_T v = {};
            if (e < WITEMS) {
                int dst; bool ok; long src;
#if FLIPW
                IGN(wf_item)(e, kci * KC, us * USTAGE, c0, dst, ok, src);
                if (ok) {
#if FVEC == 4
                    v = *(const WVEC_T*)(Wt + src);
#else
                    v[0] = Wt[src];
#endif
                }
#else
                IGN(w_item)(e, kci * KC, us * USTAGE, c0, dst, ok, src);
                if (ok) {
#if WVEC == 4
                    v = *(const WVEC_T*)(Wt + src);
#else
                    v[0] = Wt[src];
#endif
                }
#endif
            }
            wreg[i] = v;
        }
    };
    auto store_w = [&](int q, ELEM_T* wsl) {
        int kci, us;
        IGN(unit_of)(q, kci, us);
#pragma unroll
        for (int i = 0; i < WPER; ++i) {
            const int e = gtid + i * GTHREADS;
            if (e < WITEMS) {
                int dst; bool ok; long src;
#if FLIPW
                IGN(wf_item)(e, kci * KC, us * USTAGE, c0, dst, ok, src);
#pragma unroll
                for (int j = 0; j < FVEC; ++j) wsl[dst + j * WRS] = wreg[i][j];
#else
                IGN(w_item)(e, kci * KC, us * USTAGE, c0, dst, ok, src);
#if WVEC == 4
                *(WVEC_T*)(wsl + dst) = wreg[i];
#else
                wsl[dst] = wreg[i][0];
#endif
#endif
            }
        }
    };

    // Units [q0, q1) of this group, processed in lock-step rounds with the
    // other groups (every group runs UPG rounds; units past the end idle).
    const int q0 = kg * UPG;
    const int q1 = (q0 + UPG < NUNITS) ? q0 + UPG : NUNITS;
    // the zero margins of both filter buffers (never overwritten below)
#if ZW > 0
    for (int e = gtid; e < 2 * USTAGE * CB * ZW; e += GTHREADS) {
        const int row = e / ZW, z = e % ZW;
        wsl0[row * WRS + (z < RAWW ? z : WREAL + z)] = (ELEM_T)0;
    }
#endif
    int cur_chunk = -1;
    if (q0 < q1) {
        // filter and tile loads of the first unit are in flight together
        fetch_w(q0);
        int kci, us;
        IGN(unit_of)(q0, kci, us);
        load_tile(kci * KC);
        cur_chunk = kci;
        store_w(q0, wsl0);
    }
    __syncthreads();

#pragma unroll 1
    for (int rnd = 0; rnd < UPG; ++rnd) {
        const int q = q0 + rnd;
        const bool active = q < q1;
        const bool more = q + 1 < q1;
        if (more) fetch_w(q + 1);
        ELEM_T* const wsl = wsl0 + (rnd & 1) * WSL_ELEMS;
        if (active) {
            int kci, us;
            IGN(unit_of)(q, kci, us);
#if defined(FB_UUNR) && FB_UUNR
#pragma unroll
#else
#pragma unroll 1
#endif
            for (int uu = 0; uu < USTAGE; ++uu) {
                const int u = us * USTAGE + uu;
                if (u >= FH) break;
                const ELEM_T* arow[MT];
#if SWZ
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    arow[mt] = tile + ((wm * MT + mt) * MR + ti + u) * ROWS;
#else
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    arow[mt] = tile + ((wm * MT + mt) * MR + ti + u) * ROWS + S * tj * KC + h * HALF;
#endif
                const ELEM_T* brow[NT];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    const int col = (wn * NT + nt) * MF + l32;
                    const int sh = col / CB, c = col % CB;
                    brow[nt] = wsl + (uu * CB + c) * WRS + RAWW - sh * KC + h * HALF;
                }
#if DT == 0
#pragma unroll
                for (int t = 0; t < HALF; t += 4) {
                    f32x4 av[MT], bv[NT];
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
#if AV == 4
                        av[mt] = *(const f32x4*)(arow[mt] + t);
#elif AV == 2
                        const float2 p0 = *(const float2*)(arow[mt] + t);
                        const float2 p1 = *(const float2*)(arow[mt] + t + 2);
                        av[mt][0] = p0.x; av[mt][1] = p0.y; av[mt][2] = p1.x; av[mt][3] = p1.y;
#else
                        av[mt][0] = arow[mt][t]; av[mt][1] = arow[mt][t + 1];
                        av[mt][2] = arow[mt][t + 2]; av[mt][3] = arow[mt][t + 3];
#endif
                    }
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
#if BV == 4
                        bv[nt] = *(const f32x4*)(brow[nt] + t);
#elif BV == 2
                        const float2 p0 = *(const float2*)(brow[nt] + t);
                        const float2 p1 = *(const float2*)(brow[nt] + t + 2);
                        bv[nt][0] = p0.x; bv[nt][1] = p0.y; bv[nt][2] = p1.x; bv[nt][3] = p1.y;
#else
                        bv[nt][0] = brow[nt][t]; bv[nt][1] = brow[nt][t + 1];
                        bv[nt][2] = brow[nt][t + 2]; bv[nt][3] = brow[nt][t + 3];
#endif
                    }
#pragma unroll
                    for (int qq = 0; qq < 4; ++qq)
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                            for (int nt = 0; nt < NT; ++nt)
#if MF == 32
                                acc[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(
                                    av[mt][qq], bv[nt][qq], acc[mt][nt], 0, 0, 0);
#else
                                acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                                    av[mt][qq], bv[nt][qq], acc[mt][nt], 0, 0, 0);
#endif
                }
#else
#pragma unroll
                for (int t = 0; t < HALF; t += 8) {
                    u16x8 av[MT], bv[NT];
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
#if SWZ
                        av[mt] = *(const u16x8*)(arow[mt] + aoff[t / 8]);
#elif AV == 8
                        av[mt] = *(const u16x8*)(arow[mt] + t);
#elif AV == 4
                        const u16x4 p0 = *(const u16x4*)(arow[mt] + t);
                        const u16x4 p1 = *(const u16x4*)(arow[mt] + t + 4);
#pragma unroll
                        for (int qq = 0; qq < 4; ++qq) { av[mt][qq] = p0[qq]; av[mt][qq + 4] = p1[qq]; }
#else
#pragma unroll
                        for (int qq = 0; qq < 8; ++qq) av[mt][qq] = arow[mt][t + qq];
#endif
                    }
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
#if BV == 8
                        bv[nt] = *(const u16x8*)(brow[nt] + t);
#elif BV == 4
                        const u16x4 p0 = *(const u16x4*)(brow[nt] + t);
                        const u16x4 p1 = *(const u16x4*)(brow[nt] + t + 4);
#pragma unroll
                        for (int qq = 0; qq < 4; ++qq) { bv[nt][qq] = p0[qq]; bv[nt][qq + 4] = p1[qq]; }
#else
#pragma unroll
                        for (int qq = 0; qq < 8; ++qq) bv[nt][qq] = brow[nt][t + qq];
#endif
                    }
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) {
#if DT == 1 && MF == 32
                            acc[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                __builtin_bit_cast(bf16x8, av[mt]), __builtin_bit_cast(bf16x8, bv[nt]),
                                acc[mt][nt], 0, 0, 0);
#elif DT == 1
                            acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                __builtin_bit_cast(bf16x8, av[mt]), __builtin_bit_cast(bf16x8, bv[nt]),
                                acc[mt][nt], 0, 0, 0);
#elif MF == 32
                            acc[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                                __builtin_bit_cast(f16x8, av[mt]), __builtin_bit_cast(f16x8, bv[nt]),
                                acc[mt][nt], 0, 0, 0);
#else
                            acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                                __builtin_bit_cast(f16x8, av[mt]), __builtin_bit_cast(f16x8, bv[nt]),
                                acc[mt][nt], 0, 0, 0);
#endif
                        }
                }
#endif
            }
        }
        if (rnd + 1 < UPG) {
            // The other filter buffer was last read in the previous round,
            // which ended with a barrier: fill it now.
            if (more) store_w(q + 1, wsl0 + ((rnd + 1) & 1) * WSL_ELEMS);
            // A new channel chunk needs a new input tile: wait until every
            // wave is done with the current one first.
            int nk = -1, nus = 0;
            if (more) IGN(unit_of)(q + 1, nk, nus);
            const bool new_tile = more && nk != cur_chunk;
            if (__syncthreads_or(new_tile)) {
                if (new_tile) {
                    load_tile(nk * KC);
                    cur_chunk = nk;
                }
                __syncthreads();
            }
        }
    }

#if KS > 1
    // Fixed-order reduction of the KS groups' accumulators through LDS.
    __syncthreads();
    float* const red = (float*)lds_raw;
    if (kg > 0) {
        float* dst = red + (((kg - 1) * GWAVES + gw) * MT * NT * NREG) * 64 + lane;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int r = 0; r < NREG; ++r) dst[((mt * NT + nt) * NREG + r) * 64] = acc[mt][nt][r];
    }
    __syncthreads();
    if (kg == 0) {
#pragma unroll 1
        for (int g = 1; g < KS; ++g) {
            const float* src = red + (((g - 1) * GWAVES + gw) * MT * NT * NREG) * 64 + lane;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int r = 0; r < NREG; ++r) acc[mt][nt][r] += src[((mt * NT + nt) * NREG + r) * 64];
        }
    }
    if (kg != 0) return;
#endif

    // Epilogue.  Accumulator layouts: 32x32 -- lane l, register r holds row
    // 8*(r/4) + 4*(l/32) + r%4 (base pixel) and column l%32; 16x16 -- row
    // 4*(l/16) + r and column l%16.
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int col = (wn * NT + nt) * MF + l32;
        const int s = col / CB, cc = c0 + col % CB;
#if DT != 0
        const float us = (cc < COUT) ? UNSCALE[cc] * ys : 0.f;      // exact: powers of two
#endif
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
            for (int r = 0; r < NREG; ++r) {
#if MF == 32
                const int m = 8 * (r >> 2) + 4 * h + (r & 3);
#else
                const int m = 4 * h + r;
#endif
                const int oi = oi0 + (wm * MT + mt) * MR + m / MC;
                const int oj = oj0 + S * (m % MC) + s;
                if (oi < HO && oj < WO && cc < COUT) {
#if DT == 0
                    float val = acc[mt][nt][r];
#else
                    float val = acc[mt][nt][r] * us;
#endif
#ifdef FB_EPILOGUE
                    val = FB_EPILOGUE(val, cc);     // fused elementwise epilogue
#endif
                    O[((long)oi * WO + oj) * COUT + cc] = val;
                }
            }
        }
    }
}
//@@BODY-END

#ifndef FB_BATCHED
// The symbol name is chosen by the generator (forward and input-gradient
// instances get distinct names, so profiles tell them apart).
#ifndef FB_KNAME
#define FB_KNAME fbcorr_igemm
#endif
extern "C" __global__ void __launch_bounds__(NTHREADS)
FB_KNAME(const float* __restrict__ I, const ELEM_T* __restrict__ Wt,
         const float* __restrict__ UNSCALE, float* __restrict__ O)
{
    __shared__ __attribute__((aligned(16))) unsigned char lds_raw[LDS_BYTES];
    // Workgroup -> tile.  With XCDMAP the dispatcher's round-robin over the
    // eight XCDs is undone so that each XCD works on a contiguous range of
    // tiles (shared halos and filter slices stay in that XCD's L2).
    const int ntx = (WO + TWO - 1) / TWO;
    const int nty = (HO + TH - 1) / TH;
    const int ncb = (COUT + CB - 1) / CB;
    const int total = ntx * nty * ncb * FB_BATCH;   // == gridDim.x
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
    const int oi0 = ty * TH;
    const int oj0 = tx * TWO;
    const int c0 = cblk * CB;

    IGN(igemm_body)(I + (long)b * HI * WI * CIN, Wt, UNSCALE, O + (long)b * HO * WO * COUT,
                    HI, WI, HO, WO, oi0, oj0, c0, lds_raw);
}
#endif

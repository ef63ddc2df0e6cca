// Kernel configurations: defaults, validation, geometry and source generation.
//
// A configuration is the set of code-variant knobs the paper's vision
// application tunes over (Sec. 6.2: loop unrolling depth, block/grid
// dimensions, thread work size, shared-memory padding), extended by the
// matrix-core tiling.  Each knob becomes a -D constant of the kernel source
// (Sec. 5.3, keyword substitution), so every variant is compiled for exactly
// one problem (Sec. 4.2).
#include "geometry.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <sstream>

namespace fbc {

int Config::get(const char* k) const {
    auto it = v.find(k);
    return it == v.end() ? 0 : it->second;
}

std::string Config::str() const {
    std::string s = "algo=" + algo;
    for (auto& kv : v) s += " " + kv.first + "=" + std::to_string(kv.second);
    return s;
}

bool parse_config(const std::string& text, Config& base, std::string& err) {
    std::istringstream is(text);
    std::string tok;
    Config c = base;
    while (is >> tok) {
        auto eq = tok.find('=');
        if (eq == std::string::npos || eq == 0) { err = "bad token '" + tok + "'"; return false; }
        std::string k = tok.substr(0, eq), val = tok.substr(eq + 1);
        if (k == "algo") {
            if (val != "igemm" && val != "direct" && val != "dw" && val != "nn" && val != "rgemm" && val != "dws") {
                err = "unknown algo '" + val + "'";
                return false;
            }
            if (val != c.algo) {
                c.algo = val;
                c.v.clear();          // keys of another algorithm do not carry over
            }
            continue;
        }
        char* end = nullptr;
        long x = strtol(val.c_str(), &end, 10);
        if (!end || *end || val.empty()) { err = "bad value in '" + tok + "'"; return false; }
        c.v[k] = (int)x;
    }
    base = c;
    return true;
}

static int round_up(int a, int m) { return (a + m - 1) / m * m; }
static int cdiv(int a, int b) { return (a + b - 1) / b; }
static int cdivl(long a, long b) { return (int)((a + b - 1) / b); }

// ------------------------------------------------------------ defaults

static int pick_kc(int cin, bool lowp) {
    if (lowp) {
        if (cin % 16 == 0) return 16;
        if (cin % 8 == 0) return 8;
        return cin <= 16 ? cin : 8;
    }
    if (cin <= 16) return cin;
    if (cin % 16 == 0) return 16;
    if (cin % 8 == 0) return 8;
    return 8;
}

static int pick_shift(int cout) {
    if (cout >= 32) return 1;
    if (cout >= 16) return 2;
    if (cout >= 8) return 4;
    return 8;
}

Config default_igemm(int cin, int cout, bool lowp) {
    Config c;
    c.algo = "igemm";
    const int s = pick_shift(cout);
    const int cols = cout * s;
    const int nt = cols >= 64 ? 2 : 1;
    const int kc = pick_kc(cin, lowp);
    const int nchunk = (cin + kc - 1) / kc;
    c.v = {{"mf", 32}, {"kc", kc}, {"s", s}, {"mr", s >= 2 ? 4 : 1}, {"mt", 1}, {"nt", nt}, {"wm", s >= 2 ? 1 : 4},
           {"wn", 1}, {"ks", s >= 2 ? std::min(4, nchunk) : 1}, {"xpad", lowp ? 8 : 4},
           {"wpad", lowp ? 8 : 4}, {"ustage", 1}, {"xcd", 1}};
    return c;
}

// Filter fragments streamed into registers (rgemm.hip): 2 x 2 waves of
// 4 x 2 tiles (256 pixels x 128 filters per workgroup), whole channel
// chunks of up to 16 (fp32) or 32 (16-bit) channels, three steps in flight;
// for at most 16 output channels four waves of eight 16x16 tiles.
Config default_rgemm(int cin, int cout, bool lowp) {
    Config c;
    c.algo = "rgemm";
    const int pe = lowp ? 8 : 4;
    int kc = pe;
    for (int k : {4 * pe, 2 * pe})
        if (cin % k == 0 || cin > k) { kc = k; break; }
    if (cin % pe) kc = pe;
    if (cout <= 16) {
        // 16x16 tiles: a 32-wide tile would leave half its columns empty
        c.v = {{"mf", 16}, {"kc", kc}, {"mr", 1}, {"mt", 8}, {"nt", 1}, {"wm", 4}, {"wn", 1}, {"pf", 3},
               {"xpadc", 0}, {"wpe", 2}, {"xcd", 1}};
        return c;
    }
    const int nt = cout > 32 ? 2 : 1;
    const int wn = cout > 64 ? 2 : 1;
    c.v = {{"mf", 32}, {"kc", kc}, {"mr", 2}, {"mt", 4}, {"nt", nt}, {"wm", 2}, {"wn", wn}, {"pf", 3},
           {"xpadc", 0}, {"wpe", 2}, {"xcd", 1}};
    return c;
}

// The register-streamed kernel's tiling for a problem, by a cost model.
//
// Every tiling of a grid (tile size, column shift, tile rows, per-wave tiles,
// waves, chunk width) is priced as a sum of the times a compute unit needs
// for the parts of its work, and the cheapest is taken.  The prices are a
// non-negative least-squares fit to 2300 timings of random tilings on MI355X
// over 31 problems (21 forward, 10 input gradients; 1 to 100 channels, 4 to
// 128 filters of 1x1 to 13x13, 0.01 to 50 GFLOP); the fit's error is 11 %,
// and its choice was on average 9 % behind the fastest of about 75 tilings
// timed per problem.  (One fixed tiling per kernel was 1.3 to 13 times slower
// than that on the same problems.)
struct CorrProblem {
    int batch, hi, wi, cin, cout, fh, fw, padh, padw;
};
struct TilePrices {
    // microseconds per: MFMA cycle of a SIMD; the same for 32x32 tiles;
    // the same short of two waves; LDS cycle of the A reads; the same for
    // rows without planes; L1 cycle of the B loads; the same, once per
    // workgroup; staged value of a lane, tiles of more than two rows, and
    // divided by the workgroups that overlap it; stored value of a lane, and
    // not through LDS, and not streaming; channel chunk and step one after
    // another; MFMA cycle of one wave; call
    double mfma, mfma32, mfma1, lds, ldslin, b, bwg, stage, stage_rows, stage_alone, store, store_plain, store_cached,
        chunk, step, chain, call;
};
static const TilePrices kSplitPrices = {3.293e-4, 1.535e-4, 5.901e-5, 2.977e-5, 7.707e-5, 2.093e-4,
                                        7.344e-5, 4.956e-3, 9.328e-4, 5.676e-3, 2.983e-3, 3.991e-3,
                                        1.534e-3, 0.8924,   1.758e-2, 1.088e-4, 8.234};
// 16-bit operands: 1230 timings over 14 problems, error 14 %, choice 10 %
// behind the fastest of about 85 tilings.
static const TilePrices kLowpPrices = {4.676e-4, 1.435e-4, 3.716e-5, 8.939e-5, 1.729e-4, 1.736e-4,
                                       2.166e-5, 5.877e-3, 5.469e-4, 0.0,      8.826e-4, 9.000e-3,
                                       7.279e-4, 0.9402,   0.0,      0.0,      8.339};

struct Tiling {
    int mf, kc, s, mr, mt, nt, wm, wn, pf, nts, ste;
};

// nsp: bf16 parts per fp32 value (3), or 1 for 16-bit operands.
// shared: tiles of the batched kernel, two workgroups of four
// waves per CU whatever the variant.
static double price_tiling(const Tiling& c, const CorrProblem& p, int nsp, const TilePrices& pr, bool shared) {
    const int npl = c.kc / 8, nkg = 64 / c.mf, w = c.wm * c.wn, nm = nsp == 3 ? 6 : 1;
    const bool planes = c.kc % 8 == 0 && !(npl & (npl - 1));
    const int regs =
        c.mt * c.nt * (c.mf * c.mf / 64) * (nsp == 3 ? 2 : 1) + c.pf * c.nt * 4 * nsp + 2 * c.mt * 4 * nsp + 24;
    if (regs > 256) return 1e30;
    const int ho = p.hi + 2 * p.padh - p.fh + 1, wo = p.wi + 2 * p.padw - p.fw + 1;
    const int cpr = cdiv((p.fw + c.s - 1) * c.kc, 8), nch = cdiv(p.cin, c.kc), ks = cdiv(p.fh * cpr, nkg);
    // More than 64 stored values per lane after few steps, or in plain stores:
    // a wave's stores have nothing to run beside (3 x 3 windows: 4 x 2 tiles
    // of 32 in plain stores 25 us, 2 x 2 tiles 18; with 4 channels, through
    // LDS, 20.0 us, 2 x 1 tiles 17.0).
    if ((!c.ste || ks * nch < 8) && c.mt * c.nt * (c.mf * c.mf / 64) > 64) return 1e30;
    const int mc = c.mf / c.mr, th = c.wm * c.mt * c.mr, two = c.s * mc, cb = c.wn * c.nt * c.mf / c.s;
    const int tr = th + p.fh - 1, tc = c.s * (mc - 1) + cdiv(cpr * 8, c.kc);
    long lds = nsp * (planes ? (long)npl * tr * cdiv(tc, c.s) * c.s * 16
                             : ((long)tr * cdiv(tc * c.kc, 4) + 1) / 2 * 16);
    if (c.ste) lds = std::max(lds, (long)w * c.mf * (c.nt * c.mf + 8) * 4);
    if (lds > (shared ? kBatchedLds : 160 * 1024)) return 1e30;
    const int wps = std::min(8, 512 / ((regs + 7) / 8 * 8));
    const int occ = shared ? 2 : std::min({(int)(160 * 1024 / std::max(lds, 1L)), wps * 4 / w, 8});
    if (occ < 1) return 1e30;
    // the busiest CU runs q workgroups, cc at a time; later rounds even out
    const double n = (double)cdiv(wo, two) * cdiv(ho, th) * cdiv(p.cout, cb) * p.batch;
    const double q = std::ceil(n / 256.0), cc = std::min((double)occ, q);
    const double qe = q > cc ? 0.5 * (n / 256.0 + q) : q;
    const double seq = std::ceil(q / cc);
    const double steps = (double)ks * nch;
    const double mfma = steps * c.mt * c.nt * nm * c.mf;                       // cycles of a wave
    const double per_simd = cc * w / 4.0;
    const double tm = qe * mfma * w / 4.0 * std::max(1.0, std::ceil(per_simd) / per_simd);
    const double tl = qe * steps * c.mt * nsp * 8 * w, tb = qe * steps * c.nt * nsp * 16 * w;
    const double st = (double)tr * tc * c.kc * nch / 64.0, te = qe * th * two * cb * 4 / 256.0;
    double t = pr.call + tm * (pr.mfma + (c.mf == 32 ? pr.mfma32 : 0.0) + pr.mfma1 * std::max(0.0, 2.0 - per_simd));
    t += tl * (pr.lds + (planes ? 0.0 : pr.ldslin)) + tb * (pr.b + pr.bwg * c.wn / w);
    t += qe * st * (pr.stage + (c.mr > 2 ? pr.stage_rows : 0.0) + pr.stage_alone / cc);
    // plain stores: a row of 32 columns is a whole line, one of 16 half of one
    t += te * (pr.store + (c.ste ? 0.0 : pr.store_plain * (c.mf == 32 ? 0.75 : 1.0)) +
               (c.nts ? 0.0 : pr.store_cached));
    return t + seq * (nch * pr.chunk + steps * pr.step + mfma * pr.chain);
}

static Config cheapest_rgemm(const CorrProblem& p, int nsp, bool shared = false) {
    const TilePrices& pr = nsp == 3 ? kSplitPrices : kLowpPrices;
    const int cin = p.cin, cout = p.cout;
    const long ho = p.hi + 2 * p.padh - p.fh + 1, wo = p.wi + 2 * p.padw - p.fw + 1;
    std::vector<int> kcs;
    auto kc_add = [&](int k) { if (std::find(kcs.begin(), kcs.end(), k) == kcs.end()) kcs.push_back(k); };
    if (cin % 4 == 0 && cin <= 32) kc_add(cin);
    if (cin > 4) kc_add(8);
    for (int k : {16, 24, 32})
        if (cin % k == 0) kc_add(k);
    if (cin % 4 && cin < 32) { kc_add(round_up(cin, 4)); kc_add(cin); }
    Tiling c, best{};
    // a step of 16-bit operands has a sixth of the products: the fragment
    // ring has to reach further ahead (4 steps 5-15 % faster than 2 or 3)
    c.pf = nsp == 3 ? 2 : 4;
    // Streaming stores leave L2 to the operands; an output that L2 can hold
    // (8 x 4 MB) is stored through it, for the kernel that reads it next.
    // Only whole 64-byte pieces stream: others need L2 to come together (100
    // filters up to 1.8 times the time; 48, 80 and 96 filters 0.8 to 1.2
    // times the speed of plain stores, 1.03 on average).
    const bool past_l2 = (double)p.batch * ho * wo * cout * 4 > 32.0 * (1 << 20);
    double best_t = 1e30;
    for (int kc : kcs)
        for (int mf : {16, 32})
            for (int s : {1, 2, 4, 8}) {
                const int npl = kc / 8;
                const bool planes = kc % 8 == 0 && !(npl & (npl - 1));
                if (planes && cin % 8 && kc != 8) continue;
                if (!planes && (s * kc) % 4) continue;
                // shifts fill a tile from a narrow bank (or align a narrow input)
                if (s > 1 && cout * s > 64 && kc % 4 == 0) continue;
                if (s == 8 && cout > 8) continue;
                c.kc = kc; c.mf = mf; c.s = s;
                c.ste = s == 1 && cout % 4 == 0 ? 1 : 0;
                c.nts = past_l2 && c.ste && cout % 16 == 0;
                const int need = cdiv(cout * s, mf) * mf / s;        // filters that can be used
                for (c.wn = 1; c.wn <= 4; ++c.wn)
                    for (c.nt = 1; c.nt <= 4; ++c.nt) {
                        const int ncol = c.wn * c.nt * mf;
                        if (ncol % s || (ncol / s > need && ncol != mf)) continue;
                        for (c.wm = 1; c.wm * c.wn <= 8; c.wm *= 2) {
                            const int w = c.wm * c.wn;
                            if (shared ? w != 4 : w < 2 || (w == 2 && cdiv(cin, kc) > 2)) continue;
                            for (c.mr = 1; c.mr <= 8; c.mr *= 2)
                                for (c.mt = 1; c.mt <= (nsp == 3 ? 4 : 8); c.mt *= 2) {
                                    const double t = price_tiling(c, p, nsp, pr, shared);
                                    if (t < best_t) { best_t = t; best = c; }
                                }
                        }
                    }
            }
    Config out;
    if (best_t >= 1e30) return out;          // nothing fits
    out.algo = "rgemm";
    out.v = {{"mf", best.mf}, {"kc", best.kc}, {"s", best.s}, {"mr", best.mr}, {"mt", best.mt}, {"nt", best.nt},
             {"wm", best.wm}, {"wn", best.wn}, {"pf", best.pf}, {"xpadc", 0}, {"wpe", 2}, {"xcd", 1},
             {"nts", best.nts}, {"ste", best.ste}};
    if (nsp == 3) out.v["sp"] = 1;
    return out;
}

// Variants of a default that use fewer resources, tried in order until one
// fits the device.
static std::vector<Config> shrink_sequence(const Config& base) {
    std::vector<Config> out{base};
    Config c = base;
    for (int step = 0; step < 16; ++step) {
        if (c.algo == "igemm") {
            if (c.v["ks"] > 1) c.v["ks"] /= 2;
            else if (c.v["kc"] > 4 && c.v["kc"] % 2 == 0) c.v["kc"] /= 2;
            else if (c.v["nt"] > 1) c.v["nt"] /= 2;
            else if (c.v["wm"] > 1) c.v["wm"] /= 2;
            else if (c.v["mr"] > 1) c.v["mr"] /= 2;
            else if (c.v["kc"] > 1) c.v["kc"] = (c.v["kc"] + 1) / 2;
            else break;
        } else if (c.algo == "direct") {
            if (c.v["th"] > 1) c.v["th"] /= 2;
            else break;
        } else {
            if (c.v["pf"]) c.v["pf"] = 0;
            else if (c.v["rh"] > 1) c.v["rh"] /= 2;
            else if (c.v["rw"] > 8) c.v["rw"] /= 2;
            else if (c.v["nw"] < 16) c.v["nw"] *= 2;
            else break;
        }
        out.push_back(c);
    }
    return out;
}

Config default_direct(const fbcorr_desc& d) {
    Config c;
    c.algo = "direct";
    int q = 16;
    while (q > 4 && q > round_up(d.N, 4)) q /= 2;
    int nb = std::min(64, round_up(d.N, q));
    c.v = {{"th", 8}, {"tw", 32}, {"p", 4}, {"q", q}, {"nb", nb}, {"ds", 1}, {"layout", 1},
           {"xpad", 1}, {"wpad", 4}, {"ud", 1}, {"xcd", 1}};
    // keep the workgroup within 1024 threads
    while ((c.v["th"] * (c.v["tw"] / c.v["p"]) * (nb / q)) > 1024 && c.v["th"] > 1) c.v["th"] /= 2;
    return c;
}

static int dw_tiles(const fbcorr_desc& d) {
    return cdiv(d.N, 32) * cdiv(d.fh * d.fw * d.D, 32);
}

Config default_dw(const fbcorr_desc& d, int cus) {
    Config c;
    c.algo = "dw";
    const int tiles = dw_tiles(d);
    const int tpb = cdiv(tiles, 2);
    const int ho = d.H - d.fh + 1, wo = d.W - d.fw + 1;
    const long nchunks = (long)d.batch * cdiv(ho, 2) * cdiv(wo, 32);
    const int np = (int)std::max<long>(1, std::min<long>(nchunks, std::max(1, cus) / 2));
    c.v = {{"rh", 2}, {"rw", 32}, {"nw", 8}, {"tpb", tpb}, {"np", np}, {"gpad", 0}, {"xpad", 0}, {"pf", 1},
           {"bal", 0}, {"unr", 4}};
    return c;
}

// Resources of a three-part filter-gradient tiling (dws.hip).
struct DwsGeom {
    int t16 = 0, ctm = 0, xrm = 0, xre = 0, copies = 0, regs = 0;
    long lds = 0;
};
static DwsGeom dws_geom(const fbcorr_desc& d, int rt, int nw, int ncb, int rh, int rw) {
    DwsGeom g;
    const int r4 = round_up(d.fw * d.D, 4), waves = ncb * nw, threads = nw * 64;
    g.t16 = cdiv(d.fh * r4, 16);
    g.ctm = cdiv(g.t16, waves);
    g.copies = d.D % 4 == 0 ? 1 : (d.D % 2 == 0 ? 2 : 4);
    g.xre = round_up((rw - 1) * d.D + r4, 4);
    // registers per lane: accumulators, A fragments (two sets while they
    // fit), offsets, staging; weights fitted to 144 compiled kernels (17
    // registers off on average)
    const int a_sets = rt * g.ctm * 8 + rt * 24 + 24 <= 152 ? 2 : 1;
    g.regs = (int)(12 + 0.87 * rt * g.ctm * 8 + 12.6 * rt * a_sets + 5.9 * rt + (5.8 + 1.6 * (rh - 1)) * g.ctm +
                   13.0 * cdiv(rh * rw * rt * 4, threads) +
                   (15.3 + (d.D % 4 ? 2.3 : 0.0)) * cdiv(rh * g.copies * g.xre / 4, threads) + 5.8 * (rh * rw / 32));
    auto first = [&](int gw) { return (int)((long)gw * g.t16 / waves); };
    g.xrm = 1;
    for (int cb = 0; cb < ncb; ++cb) {
        const int lo = first(cb * nw) * 16 / r4, last = first((cb + 1) * nw) * 16 - 1;
        g.xrm = std::max(g.xrm, std::min(last / r4, d.fh - 1) - lo + 1);
    }
    g.lds = 3L * g.copies * (g.xrm + 2 * rh - 1) * 2 * g.xre + 6L * 2 * rh * rw * rt * 16;
    return g;
}

// The filter gradient's tiling by a cost model of the same kind: 1210
// timings over 18 problems, error 13 %, choice 9 % behind the fastest of
// about 65 tilings.  Workgroups are counted out to one, two or three per
// CU, segments to one or two per workgroup.
std::vector<Config> dws_tilings(const fbcorr_desc& d, int cus, int count) {
    const int ho = d.H - d.fh + 1, wo = d.W - d.fw + 1;
    const double L = (double)d.N * d.fh * d.fw * d.D;
    struct Priced { double t; int rt, nw, ncb, rh, rw, rseg, np; };
    std::vector<Priced> all;
    for (int rt = 1; rt <= 4; ++rt) {
        if (rt > 1 && rt * 16 >= d.N + 16) break;
        const int nrb = cdiv(d.N, rt * 16);
        for (int nw : {2, 4, 6, 8})
            for (int ncb = 1; ncb <= 4; ++ncb)
                for (int rh : {1, 2})
                    for (int rw : {16, 32, 48, 64, 80, 96, 128}) {
                        if ((rh * rw) % 32) continue;
                        const int nstr = cdiv(wo, rw);
                        if (rw > 32 && cdiv(wo, nstr) <= rw - 16) continue;      // a narrower strip does
                        const DwsGeom g = dws_geom(d, rt, nw, ncb, rh, rw);
                        if ((ncb - 1) * nw >= g.t16 || g.regs > 300 || g.lds > 160 * 1024) continue;
                        const int occ = std::min((int)(160 * 1024 / g.lds), 8 / nw);
                        const int nks = rh * rw / 32;
                        const double tiles = (double)g.t16 / (ncb * nw), el = rh * rw * rt * 16 + rh * g.copies * g.xre;
                        for (int per_cu = 1; per_cu <= 3; ++per_cu)
                            for (int k = 1; k <= 2; ++k) {
                                const int npt = std::max(1, per_cu * cus / (nrb * ncb));
                                const int segs = std::max(1, cdivl((long)npt * k, (long)d.batch * nstr));
                                const int rseg = round_up(std::max(rh, cdiv(ho, segs)), rh);
                                const long nseg = (long)d.batch * nstr * cdiv(ho, rseg);
                                const long per = nseg > npt ? std::max(1L, (nseg + npt / 2) / npt) : 1;
                                const int np = cdivl(nseg, per);
                                const double wgs = (double)np * nrb * ncb;
                                const double spw = cdivl(nseg, np), steps = spw * cdiv(std::min(rseg, ho), rh);
                                const double q = std::ceil(wgs / cus), cc = std::min((double)occ, q);
                                const double seq = std::ceil(q / cc), simd = std::ceil(cc * nw / 4.0);
                                // microseconds per: MFMA cycle of a SIMD; LDS cycle; staged value of a
                                // lane, of a row in shifted copies, of a thread step by step; value of
                                // the first rows; step; byte of partials; MFMA cycle of one wave; call
                                double t = 9.598 + 3.674e-7 * np * L * 4.0;
                                t += 3.954e-4 * seq * std::max(cc * steps * nks * tiles * nw * rt * 24.0,
                                                               simd * steps * nks * tiles * rt * 96.0);
                                t += 1.222e-4 * seq * cc * steps * nw * nks * 24.0 * (rt + tiles);
                                t += (1.386e-3 + (d.D % 4 ? 2.377e-3 : 0.0)) * seq * cc * steps * el / 64.0;
                                t += 3.777e-2 * seq * steps * el / (nw * 64);
                                t += 1.375e-2 * seq * cc * spw * (g.xrm + rh - 1) * g.copies * g.xre / 64.0;
                                t += 0.1182 * seq * steps + 2.439e-4 * seq * steps * nks * g.ctm * rt * 96.0;
                                // registers that spill (25 of them: 253 against 224 us)
                                t *= 1.0 + 0.005 * std::max(0, g.regs - 256);
                                all.push_back({t, rt, nw, ncb, rh, rw, rseg, np});
                            }
                    }
    }
    std::vector<Config> out;
    const size_t n = std::min(all.size(), (size_t)count);
    std::partial_sort(all.begin(), all.begin() + n, all.end(),
                      [](const Priced& a, const Priced& b) { return a.t < b.t; });
    for (size_t i = 0; i < n; ++i) {
        const Priced& a = all[i];
        Config c;
        c.algo = "dws";
        c.v = {{"rt", a.rt}, {"nw", a.nw}, {"ncb", a.ncb}, {"rh", a.rh}, {"rw", a.rw}, {"rseg", a.rseg}, {"np", a.np}};
        out.push_back(c);
    }
    return out;
}

// The kernels that need no repacked filters, any size.
static Config plain_config(const fbcorr_desc& d, int role, int cus) {
    const bool lowp = d.precision != FBCORR_FP32;
    switch (role) {
    case FBCORR_ROLE_FORWARD:
        if (d.algo == FBCORR_ALGO_DIRECT && !lowp) return default_direct(d);
        return default_igemm(d.D, d.N, lowp);
    case FBCORR_ROLE_BACKWARD_X:
        return default_igemm(d.N, d.D, false);
    default:
        return default_dw(d, cus);
    }
}

bool three_parts_window(const fbcorr_desc& d) {
    return d.fh * d.fw * d.D > (d.D == 1 ? 64 : 16);
}

// Where the kernels that stage slices of the filters in LDS stay ahead: few
// products per value staged or stored.  630 short-window problems, each kernel
// timed: 4-byte stores (16 channels to 38, 1x1, in bf16: 31 us register-
// streamed, 19 us), channel counts that are staged value by value (51 to 32,
// 1x1: 29 and 20 us), windows without reuse of the staged tile (fp32, 51 to
// 32, 1x1: 22 and 16 us), few channels to contract for many stored (input
// gradient, 4 to 51, 3x1: 41 and 27 us).  Outside these lines the register-
// streamed kernel is 1.4 to 1.75 times as fast on average there.
static bool staged_slices_pay(int role, bool lowp, int cin, int cout, int fh, int fw) {
    const int win = fh * fw;
    const double per_value = 0.5 * win * cin * cout / (cin + cout);      // operations per byte
    if (role == FBCORR_ROLE_BACKWARD_X) return cout > 16 && (win == 1 || (cin <= 8 && win <= 5));
    if (!lowp) return win == 1 || win * cin < 36;
    return (cout % 4 && per_value < 12) || (win == 1 && cin % 4 && cin > 16);
}

static Config heuristic_config(const fbcorr_desc& d, int role, int cus) {
    const bool lowp = d.precision != FBCORR_FP32;
    const int ho = d.H - d.fh + 1, wo = d.W - d.fw + 1;
    const double flops = 2.0 * d.batch * ho * wo * d.N * d.fh * d.fw * d.D;
    // The forward pass in fp32: three bf16 parts pay for the extra launch
    // that repacks the filters from about 0.2 GFLOP on (fp32 instructions,
    // one launch, against this: 8.5 and 11.4 us at 0.1 GFLOP, 23 and 14 us
    // at 1.3), and not where the windows are too short to be anything but
    // memory traffic (a single channel, 5x5: 20 and 28 us).  The other
    // kernels here need a launch for the filters anyway.
    Config c;
    const bool dx = role == FBCORR_ROLE_BACKWARD_X;
    if (role != FBCORR_ROLE_BACKWARD_W && staged_slices_pay(role, lowp, dx ? d.N : d.D, dx ? d.D : d.N, d.fh, d.fw))
        return plain_config(d, role, cus);
    if (role == FBCORR_ROLE_FORWARD && lowp)
        c = cheapest_rgemm({d.batch, d.H, d.W, d.D, d.N, d.fh, d.fw, 0, 0}, 1);
    else if (role == FBCORR_ROLE_FORWARD && d.algo != FBCORR_ALGO_DIRECT && flops >= 2.0e8 &&
             three_parts_window(d))
        c = cheapest_rgemm({d.batch, d.H, d.W, d.D, d.N, d.fh, d.fw, 0, 0}, 3);
    else if (role == FBCORR_ROLE_BACKWARD_X)
        c = cheapest_rgemm({d.batch, ho, wo, d.N, d.D, d.fh, d.fw, d.fh - 1, d.fw - 1}, 3);
    else if (role == FBCORR_ROLE_BACKWARD_W) {
        // three bf16 parts throughout (the smallest problem timed: 13.1 us
        // with fp32 instructions, 10.9 us; the others 1.1 to 4.7 times)
        const std::vector<Config> cs = dws_tilings(d, cus, 1);
        if (!cs.empty()) c = cs[0];
    }
    return c.algo.empty() ? plain_config(d, role, cus) : c;
}

bool batched_form(const Config& c) {
    if (c.algo == "rgemm") return c.get("sp") == 1 && c.get("wpe") == 2 && c.get("wm") * c.get("wn") == 4;
    return c.algo == "igemm" && c.get("wm") * c.get("wn") * c.get("ks") == 4;
}

Config batched_parts(const fbcorr_desc& d) {
    // many images share the launch: priced on a chip full of this one
    return cheapest_rgemm({64, d.H, d.W, d.D, d.N, d.fh, d.fw, 0, 0}, 3, true);
}

// ---------------------------------------------------------- geometry

static void opt(std::vector<std::string>& o, const char* k, long v) {
    // Every constant is passed as FB_<name>: hiprtc's implicit runtime header
    // sees -D macros too, and short names such as N would collide with it.
    o.push_back(std::string("-DFB_") + k + "=" + std::to_string(v));
}

// igemm: valid correlation over a virtually padded input (see igemm.hip).
static bool geom_igemm(const char* kname, const Config& c, int batch, int hi, int wi, int cin, int cout,
                       int fh, int fw, int padh, int padw, int dt, const DeviceInfo& di, LaunchGeom& g,
                       KernelSource& ks, std::string& err) {
    const int kc = c.get("kc"), s = c.get("s"), mt = c.get("mt"), nt = c.get("nt");
    const int wm = c.get("wm"), wn = c.get("wn"), xpad = c.get("xpad"), wpad = c.get("wpad");
    const int ustage = std::min(c.get("ustage"), fh), xcd = c.get("xcd");
    const int mr = c.get("mr"), ksp = c.get("ks");
    const int mf = c.v.count("mf") ? c.get("mf") : 32;
    if (kc < 1 || s < 1 || mt < 1 || nt < 1 || wm < 1 || wn < 1 || xpad < 0 || wpad < 0 || ustage < 1 ||
        mr < 1 || ksp < 1) {
        err = "igemm: every knob must be positive"; return false;
    }
    if (mf != 32 && mf != 16) { err = "igemm: mf must be 32 or 16"; return false; }
    if (s != 1 && s != 2 && s != 4 && s != 8) { err = "igemm: s must be 1, 2, 4 or 8"; return false; }
    if (mf % mr) { err = "igemm: mr must divide mf"; return false; }
    const int threads = wm * wn * ksp * 64;
    if (threads > std::min(1024, di.max_threads)) { err = "igemm: too many threads"; return false; }
    const int nreg = mf * mf / 64;
    // accumulators live in the AGPR half of the register file: at most 256
    if (mt * nt * nreg > 256) { err = "igemm: more than 256 accumulator registers per lane"; return false; }
    const int ncol = wn * nt * mf;
    if (ncol % s) { err = "igemm: columns must split evenly into shifts"; return false; }
    const int cb = ncol / s;
    const int mc = mf / mr;
    const int ho = hi + 2 * padh - fh + 1, wo = wi + 2 * padw - fw + 1;
    const int esz = dt == 0 ? 4 : 2;
    const int runit = (64 / mf) * (dt == 0 ? 4 : 8);
    const int krraw = (fw + s - 1) * kc;
    const int kr = round_up(krraw, runit);
    const int rowe = (mc - 1) * s * kc + kr;
    const int rows = rowe + xpad;
    const int wrs = (s - 1) * kc + kr + wpad;
    int av, bv;
    if (dt == 0) {
        av = ((s * kc) % 4 == 0) ? 4 : (((s * kc) % 2 == 0) ? 2 : 1);
        bv = (s == 1 || kc % 4 == 0) ? 4 : ((kc % 2 == 0) ? 2 : 1);
    } else {
        av = ((s * kc) % 8 == 0) ? 8 : (((s * kc) % 4 == 0) ? 4 : (((s * kc) % 2 == 0) ? 2 : 1));
        bv = (s == 1 || kc % 8 == 0) ? 8 : ((kc % 4 == 0) ? 4 : ((kc % 2 == 0) ? 2 : 1));
    }
    if (rows % av) { err = "igemm: xpad breaks A-read alignment"; return false; }
    if (wrs % bv) { err = "igemm: wpad breaks B-read alignment"; return false; }
    const int th = wm * mt * mr;
    const int tr = th + fh - 1;
    const long tile = round_up(tr * rows, 8);
    const long wsl = (long)ustage * cb * wrs;
    const long group = (tile + 2 * wsl + 7) / 8 * 8;
    const long red = (long)(ksp - 1) * wm * wn * mt * nt * nreg * 64 * 4;
    const long lds = std::max(ksp * group * esz, red);
    if (lds > di.lds_per_block) { err = "igemm: LDS " + std::to_string(lds) + " B exceeds the device limit"; return false; }
    const long grid = (long)cdiv(wo, s * mc) * cdiv(ho, th) * cdiv(cout, cb) * batch;
    if (grid <= 0 || grid > 0x7fffffffL) { err = "igemm: grid out of range"; return false; }
    g.grid_x = (int)grid;
    g.grid_y = 1;
    g.threads = threads;
    g.lds = (int)lds;
    ks.name = kname;
    ks.file = "igemm";
    ks.source = template_source("igemm");
    ks.options.clear();
    ks.options.push_back(std::string("-DFB_KNAME=") + kname);
    opt(ks.options, "BATCH", batch); opt(ks.options, "FH", fh); opt(ks.options, "FW", fw);
    opt(ks.options, "CIN", cin); opt(ks.options, "COUT", cout);
    opt(ks.options, "HI", hi); opt(ks.options, "WI", wi); opt(ks.options, "HO", ho); opt(ks.options, "WO", wo);
    opt(ks.options, "PADH", padh); opt(ks.options, "PADW", padw);
    opt(ks.options, "MF", mf); opt(ks.options, "KC", kc); opt(ks.options, "S", s); opt(ks.options, "MR", mr);
    opt(ks.options, "MT", mt); opt(ks.options, "NT", nt);
    opt(ks.options, "WM", wm); opt(ks.options, "WN", wn); opt(ks.options, "KS", ksp); opt(ks.options, "DT", dt);
    opt(ks.options, "XPAD", xpad); opt(ks.options, "WPAD", wpad);
    opt(ks.options, "USTAGE", ustage); opt(ks.options, "XCDMAP", xcd ? 1 : 0);
    if (c.get("uunr")) opt(ks.options, "UUNR", 1);
    if (c.get("swz")) {
        if (dt == 0 || kc != 16) { err = "igemm: swz needs 16-bit operands and kc=16"; return false; }
        opt(ks.options, "SWZ", 1);
    }
    return true;
}

// rgemm: implicit GEMM with the filter fragments streamed into registers
// (see rgemm.hip).  Returns the packed bank's size in bytes in bank_bytes.
static bool geom_rgemm(const char* kname, const Config& c, int batch, int hi, int wi, int cin, int cout,
                       int fh, int fw, int padh, int padw, int dt, const DeviceInfo& di, LaunchGeom& g,
                       KernelSource& ks, KernelSource& pack, LaunchGeom& pack_geom, size_t& bank_bytes,
                       std::string& err) {
    const int kc = c.get("kc"), mr = c.get("mr"), mt = c.get("mt"), nt = c.get("nt");
    const int wm = c.get("wm"), wn = c.get("wn"), pf = c.get("pf"), xpadc = c.get("xpadc");
    const int wpe = c.v.count("wpe") ? c.get("wpe") : 2, xcd = c.get("xcd"), unr = c.get("unr");
    const int mf = c.v.count("mf") ? c.get("mf") : 32;
    const int sh = c.v.count("s") ? c.get("s") : 1;
    if (kc < 1 || mr < 1 || mt < 1 || nt < 1 || wm < 1 || wn < 1 || pf < 1 || xpadc < 0) {
        err = "rgemm: every knob must be positive"; return false;
    }
    if (sh != 1 && sh != 2 && sh != 4 && sh != 8) { err = "rgemm: s must be 1, 2, 4 or 8"; return false; }
    if ((wn * nt * mf) % sh) { err = "rgemm: the columns must split evenly into shifts"; return false; }
    if (mf != 32 && mf != 16) { err = "rgemm: mf must be 32 or 16"; return false; }
    if (pf > 8) { err = "rgemm: pf is at most 8"; return false; }
    if (wpe < 1 || wpe > 8) { err = "rgemm: wpe must be 1..8"; return false; }
    if (mf % mr) { err = "rgemm: mr must divide mf"; return false; }
    // fp32 operands as three bf16 parts: 16-bit cells, two accumulators
    const int sp = c.get("sp");
    if (sp != 0 && sp != 1) { err = "rgemm: sp is 0 or 1"; return false; }
    if (sp && dt != 0) { err = "rgemm: sp applies to fp32 operands"; return false; }
    if (sp) dt = 3;
    const int nsp = sp ? 3 : 1, nacc = sp ? 2 : 1;
    const int pe = dt == 0 ? 4 : 8, nkg = 64 / mf;
    const int npl = kc / pe;
    const bool planes = kc % pe == 0 && !(npl & (npl - 1));
    if (dt == 0 && !planes) {
        err = "rgemm: kc must be " + std::to_string(pe) + " times a power of two"; return false;
    }
    if (!planes && (sh * kc) % 4) { err = "rgemm: s*kc must be a multiple of 4"; return false; }
    if (!planes && kc < cin && cin % kc) {
        err = "rgemm: kc must be " + std::to_string(pe) + " times a power of two or cut the channels evenly"; return false;
    }
    if (kc % 4 && kc != cin) { err = "rgemm: a kc that is not a multiple of 4 must be the channel count"; return false; }
    if (kc > 64) { err = "rgemm: kc is at most 64"; return false; }
    if (planes && cin % pe && kc != pe) { err = "rgemm: channels not a multiple of the cell width need kc=" + std::to_string(pe); return false; }
    const int threads = wm * wn * 64;
    if (threads > std::min(1024, di.max_threads)) { err = "rgemm: too many threads"; return false; }
    // accumulators, the fragment ring and two sets of A fragments must fit
    // the per-lane register budget of wpe waves per SIMD (512 / wpe)
    const int regs = mt * nt * (mf * mf / 64) * nacc + pf * nt * 4 * nsp + 2 * mt * 4 * nsp + 24;
    if (regs > 512 / wpe) {
        err = "rgemm: needs about " + std::to_string(regs) + " registers per lane, more than wpe allows"; return false;
    }
    const int cpr = cdiv((fw + sh - 1) * kc, pe);      // cells per filter row
    const int ntaps = cdiv(cpr * pe, kc);
    const int nchunk = (cin + kc - 1) / kc;
    const int ksteps2 = cdiv(fh * cpr, nkg) + pf;
    const int mc = mf / mr;
    const int ncolw = wn * nt * mf, cb = ncolw / sh;
    const int th = wm * mt * mr, two = sh * mc;
    const int tr = th + fh - 1, tc = sh * (mc - 1) + ntaps;
    const int ste = c.get("ste");
    if (ste && (sh != 1 || cout % 4)) { err = "rgemm: ste needs s=1 and a multiple of 4 output channels"; return false; }
    long lds = nsp * (planes ? (long)npl * tr * (cdiv(tc, sh) * sh + xpadc) * 16
                             : ((long)tr * (cdiv(tc * kc, 4) + xpadc) + 1) / 2 * 16);
    if (ste) lds = std::max(lds, (long)wm * wn * mf * (nt * mf + 8) * 4);
    if (lds > di.lds_per_block) { err = "rgemm: LDS " + std::to_string(lds) + " B exceeds the device limit"; return false; }
    const int ho = hi + 2 * padh - fh + 1, wo = wi + 2 * padw - fw + 1;
    const long grid = (long)cdiv(wo, two) * cdiv(ho, th) * cdiv(cout, cb) * batch;
    if (grid <= 0 || grid > 0x7fffffffL) { err = "rgemm: grid out of range"; return false; }
    // the packed bank covers whole column blocks of the correlation kernel
    // (NCOLW columns of shifted filters each): one kilobyte per column tile,
    // chunk and step
    const int ncols = cdiv(cout, cb) * ncolw;
    bank_bytes = (size_t)(ncols / mf) * nchunk * ksteps2 * nsp * 1024;
    g.grid_x = (int)grid;
    g.grid_y = 1;
    g.threads = threads;
    g.lds = (int)lds;
    ks.name = kname;
    ks.file = "rgemm";
    ks.source = template_source("rgemm");
    ks.options.clear();
    ks.options.push_back(std::string("-DFB_KNAME=") + kname);
    opt(ks.options, "BATCH", batch); opt(ks.options, "FH", fh); opt(ks.options, "FW", fw);
    opt(ks.options, "CIN", cin); opt(ks.options, "COUT", cout);
    opt(ks.options, "HI", hi); opt(ks.options, "WI", wi); opt(ks.options, "HO", ho); opt(ks.options, "WO", wo);
    opt(ks.options, "PADH", padh); opt(ks.options, "PADW", padw); opt(ks.options, "DT", dt);
    opt(ks.options, "MF", mf); opt(ks.options, "KC", kc); opt(ks.options, "MR", mr);
    opt(ks.options, "MT", mt); opt(ks.options, "NT", nt); opt(ks.options, "S", sh);
    opt(ks.options, "WM", wm); opt(ks.options, "WN", wn); opt(ks.options, "PF", pf);
    opt(ks.options, "XPADC", xpadc); opt(ks.options, "WPE", wpe); opt(ks.options, "XCDMAP", xcd ? 1 : 0);
    if (unr) opt(ks.options, "UNR", 1);
    if (c.get("nts")) opt(ks.options, "NTS", 1);
    if (ste) opt(ks.options, "STE", 1);
    pack = KernelSource();
    pack.name = "fbcorr_pack_frag";
    pack.file = "rgemm";
    pack.source = template_source("rgemm");
    pack.options.push_back("-DFB_PACK_FRAG");
    opt(pack.options, "FH", fh); opt(pack.options, "FW", fw); opt(pack.options, "CIN", cin);
    opt(pack.options, "COUT", cout); opt(pack.options, "DT", dt); opt(pack.options, "MF", mf);
    opt(pack.options, "KC", kc); opt(pack.options, "PF", pf); opt(pack.options, "S", sh);
    opt(pack.options, "NCOLW", ncolw);
    pack_geom = LaunchGeom{ncols, 1, 256, 0};
    return true;
}

static bool geom_direct(const Config& c, const fbcorr_desc& d, const DeviceInfo& di, LaunchGeom& g,
                        KernelSource& ks, std::string& err) {
    const int th = c.get("th"), tw = c.get("tw"), p = c.get("p"), q = c.get("q"), nb = c.get("nb");
    const int ds = c.get("ds"), layout = c.get("layout"), xpad = c.get("xpad"), wpad = c.get("wpad");
    const int ud = c.get("ud"), xcd = c.get("xcd"), fsrc = c.get("fsrc"), sb = c.get("sb");
    if (th < 1 || tw < 1 || p < 1 || q < 1 || nb < 1 || ds < 1 || xpad < 0 || wpad < 0 || ud < 1) {
        err = "direct: every knob must be positive"; return false;
    }
    if (fsrc != 0 && fsrc != 1) { err = "direct: fsrc is 0 or 1"; return false; }
    if (sb != 0 && sb != 1) { err = "direct: sb is 0 or 1"; return false; }
    if (fsrc && (ds != 1 || (th * (tw / p)) % 64 != 0)) {
        err = "direct: scalar weights (fsrc=1) need ds=1 and th*tw/p a multiple of 64"; return false;
    }
    if (tw % p) { err = "direct: p must divide tw"; return false; }
    if (nb % q) { err = "direct: q must divide nb"; return false; }
    if (q % 4) { err = "direct: q must be a multiple of 4"; return false; }
    if ((ds & (ds - 1)) || ds > 64 || d.D % ds) { err = "direct: ds must be a power of two dividing D"; return false; }
    if ((nb + wpad) % 4) { err = "direct: nb + wpad must be a multiple of 4"; return false; }
    if (layout != 0 && layout != 1) { err = "direct: layout is 0 or 1"; return false; }
    const int threads = th * (tw / p) * (nb / q) * ds;
    if (threads > std::min(1024, di.max_threads) || threads < 64 || threads % 64) {
        err = "direct: workgroup must be 64..1024 threads in whole waves"; return false;
    }
    const int ho = d.H - d.fh + 1, wo = d.W - d.fw + 1;
    const int trr = th + d.fh - 1, tcc = tw + d.fw - 1;
    const long tile = layout == 0 ? (long)trr * (tcc * d.D + xpad) : (long)d.D * trr * (tcc + xpad);
    const long lds = (tile + (fsrc ? 0L : (long)d.fw * d.D * (nb + wpad))) * 4;
    if (lds > di.lds_per_block) { err = "direct: LDS " + std::to_string(lds) + " B exceeds the device limit"; return false; }
    const long grid = (long)cdiv(wo, tw) * cdiv(ho, th) * cdiv(d.N, nb) * d.batch;
    if (grid <= 0 || grid > 0x7fffffffL) { err = "direct: grid out of range"; return false; }
    g.grid_x = (int)grid;
    g.grid_y = 1;
    g.threads = threads;
    g.lds = (int)lds;
    ks.name = "fbcorr_direct";
    ks.file = "direct";
    ks.source = template_source("direct");
    ks.options.clear();
    opt(ks.options, "BATCH", d.batch); opt(ks.options, "FH", d.fh); opt(ks.options, "FW", d.fw);
    opt(ks.options, "D", d.D); opt(ks.options, "N", d.N); opt(ks.options, "H", d.H); opt(ks.options, "W", d.W);
    opt(ks.options, "HO", ho); opt(ks.options, "WO", wo);
    opt(ks.options, "TH", th); opt(ks.options, "TW", tw); opt(ks.options, "P", p); opt(ks.options, "Q", q);
    opt(ks.options, "NB", nb); opt(ks.options, "DS", ds); opt(ks.options, "LAYOUT", layout);
    opt(ks.options, "XPAD", xpad); opt(ks.options, "WPAD", wpad); opt(ks.options, "UD", ud);
    opt(ks.options, "XCDMAP", xcd ? 1 : 0);
    if (sb) opt(ks.options, "SB", 1);
    if (fsrc) {
        opt(ks.options, "FSRC", 1);
        opt(ks.options, "NPAD", cdiv(d.N, nb) * nb);
    }
    return true;
}

static bool geom_dw(const Config& c, const fbcorr_desc& d, const DeviceInfo& di, LaunchGeom& g,
                    KernelSource& ks, int& np_out, std::string& err) {
    const int rh = c.get("rh"), rw = c.get("rw"), nw = c.get("nw"), tpb = c.get("tpb");
    const int gpad = c.get("gpad"), xpad = c.get("xpad"), pf = c.get("pf"), bal = c.get("bal");
    const int unr = c.v.count("unr") ? c.get("unr") : 4;
    int np = c.get("np");
    if (rh < 1 || rw < 1 || nw < 1 || tpb < 1 || gpad < 0 || xpad < 0 || np < 1) {
        err = "dw: every knob must be positive"; return false;
    }
    if ((rh * rw) % 2) { err = "dw: rh*rw must be even"; return false; }
    const int tiles = dw_tiles(d);
    const int tpb_eff = std::min(tpb, tiles);
    if (bal < 0 || bal > 1) { err = "dw: bal must be 0 or 1"; return false; }
    if (unr < 0 || unr > 64) { err = "dw: unr must be 0 (complete) or 1..64"; return false; }
    // accumulator slots per wave: round-robin tiles, or full rounds + two
    // slots for the left-over tiles split by pixels
    const int slots = bal ? tpb_eff / nw + 2 : cdiv(tpb_eff, nw);
    if (slots > 8) { err = "dw: more than 8 accumulator tiles per wave"; return false; }
    const int threads = nw * 64;
    if (threads > std::min(1024, di.max_threads)) { err = "dw: too many threads"; return false; }
    const int ho = d.H - d.fh + 1, wo = d.W - d.fw + 1;
    const int npad = cdiv(d.N, 32) * 32;
    const int pc = rh * rw;
    if (pf < 0 || pf > 2) { err = "dw: pf must be 0, 1 or 2"; return false; }
    const long stage = (pf == 2 ? 2 : 1) *
                       ((long)pc * (npad + gpad) + (long)(rh + d.fh - 1) * ((rw + d.fw - 1) * d.D + xpad)) * 4;
    // with bal the staging memory is reused for the left-over slots (two
    // 32x32 fp32 tiles per wave)
    const long lds = std::max(stage, bal ? (long)nw * 2 * 1024 * 4 : 0L);
    if (lds > di.lds_per_block) { err = "dw: LDS " + std::to_string(lds) + " B exceeds the device limit"; return false; }
    const long prefetch_regs = pf ? (cdivl((long)pc * npad, threads) + cdivl((long)(rh + d.fh - 1) * (rw + d.fw - 1) * d.D, threads)) : 0;
    if (prefetch_regs > 96) { err = "dw: prefetch needs too many registers"; return false; }
    const long nchunks = (long)d.batch * cdiv(ho, rh) * cdiv(wo, rw);
    if (np > nchunks) np = (int)nchunks;
    if (np > 65535) { err = "dw: partial count out of range"; return false; }
    g.grid_x = np;
    g.grid_y = cdiv(tiles, tpb_eff);
    g.threads = threads;
    g.lds = (int)lds;
    np_out = np;
    ks.name = "fbcorr_dw_partial";
    ks.file = "dw";
    ks.source = template_source("dw");
    ks.options.clear();
    opt(ks.options, "BATCH", d.batch); opt(ks.options, "FH", d.fh); opt(ks.options, "FW", d.fw);
    opt(ks.options, "D", d.D); opt(ks.options, "N", d.N); opt(ks.options, "H", d.H); opt(ks.options, "W", d.W);
    opt(ks.options, "HO", ho); opt(ks.options, "WO", wo);
    opt(ks.options, "RH", rh); opt(ks.options, "RW", rw); opt(ks.options, "NW", nw); opt(ks.options, "TPB", tpb_eff);
    opt(ks.options, "NP", np); opt(ks.options, "GPAD", gpad); opt(ks.options, "XPAD", xpad);
    opt(ks.options, "PF", pf);
    if (bal) opt(ks.options, "BAL", bal);
    if (c.get("skipe")) opt(ks.options, "SKIPE", 1);
    opt(ks.options, "UNR", unr);
    return true;
}

// dws: fp32 operands as three bf16 parts, a strip of output columns walked
// row by row (see dws.hip).
static bool geom_dws(const Config& c, const fbcorr_desc& d, const DeviceInfo& di, LaunchGeom& g,
                     KernelSource& ks, int& np_out, std::string& err) {
    const int rt = c.get("rt"), nw = c.get("nw"), ncb = c.get("ncb"), rh = c.get("rh"), rw = c.get("rw");
    const int rseg = c.get("rseg");
    int np = c.get("np");
    if (rt < 1 || nw < 1 || ncb < 1 || rh < 1 || rw < 1 || rseg < 1 || np < 1) {
        err = "dws: every knob must be positive"; return false;
    }
    if (rt > 4) { err = "dws: rt is at most 4"; return false; }
    if (rw % 16 || (rh * rw) % 32) { err = "dws: rw must be a multiple of 16 and rh*rw of 32"; return false; }
    const int threads = nw * 64;
    if (threads > std::min(1024, di.max_threads)) { err = "dws: too many threads"; return false; }
    const int ho = d.H - d.fh + 1, wo = d.W - d.fw + 1;
    const DwsGeom q = dws_geom(d, rt, nw, ncb, rh, rw);
    if (q.regs > 300) { err = "dws: needs about " + std::to_string(q.regs) + " registers per lane"; return false; }
    const long lds = q.lds;
    if (lds > di.lds_per_block) { err = "dws: LDS " + std::to_string(lds) + " B exceeds the device limit"; return false; }
    const long nseg = (long)d.batch * cdiv(wo, rw) * cdiv(ho, rseg);
    if (nseg > 0x7fffffffL) { err = "dws: too many segments"; return false; }
    if (np > nseg) np = (int)nseg;
    const long gy = (long)cdiv(d.N, rt * 16) * ncb;
    if (np > 65535 || gy > 65535) { err = "dws: grid out of range"; return false; }
    g.grid_x = np;
    g.grid_y = (int)gy;
    g.threads = threads;
    g.lds = (int)lds;
    np_out = np;
    ks.name = "fbcorr_dw_split";
    ks.file = "dws";
    ks.source = template_source("dws");
    ks.options.clear();
    opt(ks.options, "BATCH", d.batch); opt(ks.options, "FH", d.fh); opt(ks.options, "FW", d.fw);
    opt(ks.options, "D", d.D); opt(ks.options, "N", d.N); opt(ks.options, "H", d.H); opt(ks.options, "W", d.W);
    opt(ks.options, "HO", ho); opt(ks.options, "WO", wo);
    opt(ks.options, "RT", rt); opt(ks.options, "NW", nw); opt(ks.options, "NCB", ncb); opt(ks.options, "RH", rh);
    opt(ks.options, "RW", rw); opt(ks.options, "RSEG", rseg); opt(ks.options, "NP", np);
    return true;
}

static KernelSource util_source(const char* name, const char* define) {
    KernelSource ks;
    ks.name = name;
    ks.file = "util";
    ks.source = template_source("util");
    ks.options.push_back(std::string("-DFB_") + define);
    return ks;
}

static size_t align256(size_t x) { return (x + 255) / 256 * 256; }

// fp16 forward: the per-tensor input scale (reading c-10).  256 partial
// maxima of |x| from fbcorr_absmax, written after `ucount` unscale floats,
// are combined by the correlation kernel (option FB_XMOFF).  Returns the
// bytes of the unscale + partials region.
static const int kInputMaxParts = 256;
static size_t add_input_scale(const fbcorr_desc& d, int dt, size_t ucount, RoleBuild& rb) {
    if (dt != 2) return align256(ucount * 4);
    const size_t xmoff = (ucount + 63) / 64 * 64;
    rb.main.options.push_back("-DFB_XMOFF=" + std::to_string(xmoff));
    KernelSource ks = util_source("fbcorr_absmax", "ABSMAX");
    rb.aux.push_back(ks);
    rb.aux_geom.push_back(LaunchGeom{kInputMaxParts, 1, 256, 0});
    rb.ws_xmax = rb.ws_unscale + xmoff * 4;
    rb.nxp = kInputMaxParts;
    (void)d;
    return align256((xmoff + kInputMaxParts) * 4);
}

static bool build_role_impl(const fbcorr_desc& d, int role, const Config& c, const DeviceInfo& di,
                            RoleBuild& rb, std::string& err);

bool build_role(const fbcorr_desc& d, int role, const Config& c, const DeviceInfo& di,
                RoleBuild& rb, std::string& err) {
    if (!build_role_impl(d, role, c, di, rb, err)) return false;
    // Test hook: "inject_error=1" makes the generated source fail to compile.
    if (c.get("inject_error")) rb.main.options.push_back("-DFB_INJECT_ERROR");
    return true;
}

static bool known_keys(const Config& c, std::string& err) {
    static const std::map<std::string, std::vector<std::string>> keys = {
        {"igemm", {"mf", "kc", "s", "mr", "mt", "nt", "wm", "wn", "ks", "xpad", "wpad", "ustage", "xcd", "flip",
                   "uunr", "swz"}},
        {"direct", {"th", "tw", "p", "q", "nb", "ds", "layout", "xpad", "wpad", "ud", "xcd", "fsrc", "sb"}},
        {"dw", {"rh", "rw", "nw", "tpb", "np", "gpad", "xpad", "pf", "bal", "unr", "skipe"}},
        {"dws", {"rt", "nw", "ncb", "rh", "rw", "rseg", "np"}},
        {"rgemm", {"mf", "kc", "s", "mr", "mt", "nt", "wm", "wn", "pf", "xpadc", "wpe", "unr", "xcd", "flip", "nts",
                   "ste", "sp"}},
    };
    auto it = keys.find(c.algo);
    if (it == keys.end()) { err = "unknown algorithm '" + c.algo + "'"; return false; }
    for (auto& kv : c.v) {
        if (kv.first == "inject_error") continue;
        if (std::find(it->second.begin(), it->second.end(), kv.first) == it->second.end()) {
            err = "unknown key '" + kv.first + "' for algo=" + c.algo;
            return false;
        }
    }
    return true;
}

static bool build_role_impl(const fbcorr_desc& d, int role, const Config& c, const DeviceInfo& di,
                            RoleBuild& rb, std::string& err) {
    rb = RoleBuild();
    rb.cfg = c;
    if (!known_keys(c, err)) return false;
    const int ho = d.H - d.fh + 1, wo = d.W - d.fw + 1;
    const long K = (long)d.fh * d.fw * d.D;
    if (role == FBCORR_ROLE_FORWARD) {
        const int dt = d.precision == FBCORR_BF16 ? 1 : (d.precision == FBCORR_FP16 ? 2 : 0);
        if (c.algo == "direct") {
            if (dt != 0) { err = "the direct kernel is fp32 only"; return false; }
            if (!geom_direct(c, d, di, rb.main_geom, rb.main, err)) return false;
            if (c.get("fsrc")) {
                // tap-major copy of the filters for the scalar loads
                const int npad = cdiv(d.N, c.get("nb")) * c.get("nb");
                KernelSource ks = util_source("fbcorr_transpose_filters", "TRANSPOSE_FILTERS");
                opt(ks.options, "N", d.N); opt(ks.options, "FH", d.fh); opt(ks.options, "FW", d.fw);
                opt(ks.options, "D", d.D); opt(ks.options, "NPAD", npad);
                rb.aux.push_back(ks);
                rb.aux_geom.push_back(LaunchGeom{cdivl(K * npad, 256), 1, 256, 0});
                rb.ws_lowp_w = 0;
                rb.ws_bytes = align256((size_t)K * npad * 4);
            }
        } else if (c.algo == "igemm") {
            if (c.get("flip")) { err = "flip applies to the input-gradient role only"; return false; }
            if (!geom_igemm("fbcorr_fwd_igemm", c, d.batch, d.H, d.W, d.D, d.N, d.fh, d.fw, 0, 0, dt, di,
                            rb.main_geom, rb.main, err))
                return false;
        } else if (c.algo == "rgemm") {
            if (c.get("flip")) { err = "flip applies to the input-gradient role only"; return false; }
            // the filters are always repacked (fragment order; scaled and
            // rounded for 16-bit operands)
            KernelSource pk;
            LaunchGeom pg;
            size_t bank = 0;
            if (!geom_rgemm("fbcorr_fwd_rgemm", c, d.batch, d.H, d.W, d.D, d.N, d.fh, d.fw, 0, 0, dt, di,
                            rb.main_geom, rb.main, pk, pg, bank, err))
                return false;
            rb.aux.push_back(pk);
            rb.aux_geom.push_back(pg);
            rb.ws_lowp_w = 0;
            rb.ws_unscale = align256(bank);
            rb.ws_bytes = rb.ws_unscale + add_input_scale(d, dt, (size_t)pg.grid_x, rb);
            return true;
        } else {
            err = "forward role needs algo=igemm, algo=rgemm or algo=direct";
            return false;
        }
        if (dt != 0) {
            KernelSource ks = util_source("fbcorr_pack_lowp", "PACK_LOWP");
            opt(ks.options, "N", d.N); opt(ks.options, "FH", d.fh); opt(ks.options, "FW", d.fw);
            opt(ks.options, "D", d.D); opt(ks.options, "LOWP", dt);
            rb.aux.push_back(ks);
            rb.aux_geom.push_back(LaunchGeom{d.N, 1, 256, 0});
            rb.ws_lowp_w = 0;
            rb.ws_unscale = align256((size_t)d.N * K * 2);
            rb.ws_bytes = rb.ws_unscale + add_input_scale(d, dt, (size_t)d.N, rb);
        }
        return true;
    }
    if (role == FBCORR_ROLE_BACKWARD_X && c.algo == "rgemm") {
        // dx = valid correlation of dy (padded by fh-1, fw-1) with the
        // flipped, transposed filters, which the pack reads straight from
        // the forward bank (the flip is part of the repacking)
        KernelSource pk;
        LaunchGeom pg;
        size_t bank = 0;
        if (!geom_rgemm("fbcorr_dx_rgemm", c, d.batch, ho, wo, d.N, d.D, d.fh, d.fw, d.fh - 1, d.fw - 1, 0, di,
                        rb.main_geom, rb.main, pk, pg, bank, err))
            return false;
        pk.options.push_back("-DFB_FLIP");
        rb.main.options.push_back("-DFB_FLIP");
        rb.aux.push_back(pk);
        rb.aux_geom.push_back(pg);
        rb.ws_unscale = align256(bank);
        rb.ws_bytes = rb.ws_unscale + align256((size_t)pg.grid_x * 4);
        return true;
    }
    if (role == FBCORR_ROLE_BACKWARD_X) {
        if (c.algo != "igemm") { err = "input-gradient role needs algo=igemm or algo=rgemm"; return false; }
        // dx = valid correlation of dy (padded by fh-1, fw-1) with flipped,
        // transposed filters: CIN = N, COUT = D, input extent Ho x Wo.
        if (!geom_igemm("fbcorr_dx_igemm", c, d.batch, ho, wo, d.N, d.D, d.fh, d.fw, d.fh - 1, d.fw - 1, 0, di,
                        rb.main_geom, rb.main, err))
            return false;
        if (c.get("flip")) {
            // the flip happens while staging: the kernel reads the forward bank
            rb.main.options.push_back("-DFB_FLIPW");
            return true;
        }
        KernelSource ks = util_source("fbcorr_flip_filters", "FLIP_FILTERS");
        opt(ks.options, "N", d.N); opt(ks.options, "FH", d.fh); opt(ks.options, "FW", d.fw); opt(ks.options, "D", d.D);
        rb.aux.push_back(ks);
        rb.aux_geom.push_back(LaunchGeom{cdivl((long)d.N * K, 256), 1, 256, 0});
        rb.ws_bytes = align256((size_t)d.N * K * 4);
        return true;
    }
    if (role == FBCORR_ROLE_BACKWARD_W) {
        int np = 0;
        if (c.algo == "dw") {
            if (!geom_dw(c, d, di, rb.main_geom, rb.main, np, err)) return false;
        } else if (c.algo == "dws") {
            if (!geom_dws(c, d, di, rb.main_geom, rb.main, np, err)) return false;
        } else {
            err = "filter-gradient role needs algo=dw or algo=dws";
            return false;
        }
        rb.np = np;
        const long L = (long)d.N * K;
        // 16 slices x 16 lanes per workgroup: several hundred workgroups for
        // a few hundred kilobytes of output, each thread with NP/16 loads
        const int rs = 16, lanes = 16;
        const int sv = (L % 4 == 0) ? 4 : 1;    // outputs per thread (16-byte loads when possible)
        KernelSource ks = util_source("fbcorr_sum_partials", "SUM_PARTIALS");
        opt(ks.options, "L", L); opt(ks.options, "NP", np); opt(ks.options, "RS", rs);
        opt(ks.options, "LANES", lanes);
        rb.aux.push_back(ks);
        rb.aux_geom.push_back(LaunchGeom{cdivl(L / sv, lanes), 1, lanes * rs, 0});
        rb.ws_bytes = align256((size_t)np * L * 4);
        return true;
    }
    err = "unknown role";
    return false;
}

// The tuning database's entry for this hardware and problem, if it builds.
// form: the entry of one kernel form ("igemm", "rgemm"), kept beside the
// problem's own where another form is faster.
static bool database_config(const fbcorr_desc& d, int role, const DeviceInfo& di, Config& out,
                            const std::string& form = "") {
    std::string text, err;
    if (!tuning_db_lookup(di.arch, role, d, text, form)) return false;
    Config probe;
    probe.algo = plain_config(d, role, di.cus).algo;
    if (!parse_config(text, probe, err)) return false;
    // start from the named algorithm's hand-written defaults
    const int cin = role == FBCORR_ROLE_BACKWARD_X ? d.N : d.D;
    const int cout = role == FBCORR_ROLE_BACKWARD_X ? d.D : d.N;
    const bool lp = d.precision != FBCORR_FP32 && role == FBCORR_ROLE_FORWARD;
    Config base = plain_config(d, role, di.cus);
    if (probe.algo != base.algo)
        base = probe.algo == "direct" ? default_direct(d)
               : probe.algo == "rgemm" ? default_rgemm(cin, cout, lp)
               : probe.algo == "dws"   ? probe
                                       : default_igemm(cin, cout, d.precision != FBCORR_FP32);
    RoleBuild rb;
    if (!parse_config(text, base, err) || !build_role(d, role, base, di, rb, err)) return false;
    out = base;
    return true;
}

// The kernels of plain_config, shrunk until they fit the device.
static Config plain_default(const fbcorr_desc& d, int role, const DeviceInfo& di) {
    const Config h = plain_config(d, role, di.cus);
    RoleBuild rb;
    std::string err;
    for (const Config& c : shrink_sequence(h))
        if (build_role(d, role, c, di, rb, err)) return c;
    return h;   // nothing fits: the caller reports the heuristic's error
}

Config heuristic_default(const fbcorr_desc& d, int role, const DeviceInfo& di) {
    const Config h = heuristic_config(d, role, di.cus);
    RoleBuild rb;
    std::string err;
    const Config plain = plain_default(d, role, di);
    if (h.algo == plain.algo || !build_role(d, role, h, di, rb, err)) return plain;
    // A forward pass whose packed bank would outgrow the static scratch keeps
    // fp32 instructions (parts are 6 bytes a weight; not timed at that size).
    RoleBuild pb;
    // Which filter gradients a plan takes does not hang on the choice of
    // kernel: one that algo=dw refuses for its size is refused here too.
    if (role == FBCORR_ROLE_BACKWARD_W && !build_role(d, role, plain, di, pb, err)) return plain;
    if (role == FBCORR_ROLE_FORWARD && rb.ws_bytes > kNoAllocScratchBytes &&
        build_role(d, role, plain, di, pb, err) && pb.ws_bytes <= kNoAllocScratchBytes)
        return plain;
    return h;
}

Config default_config(const fbcorr_desc& d, int role, const DeviceInfo& di) {
    Config c;
    return database_config(d, role, di, c) ? c : heuristic_default(d, role, di);
}

bool scratchless_forward(const fbcorr_desc& d, const DeviceInfo& di, const Config& current, Config& out) {
    const int role = FBCORR_ROLE_FORWARD;
    std::string text, err;
    if (d.precision != FBCORR_FP32 || current.algo != "rgemm" || !current.get("sp")) return false;
    Config c;
    // (a problem whose fp32 instructions are an rgemm entry packs its bank too)
    if (database_config(d, role, di, c) || tuning_db_lookup(di.arch, role, d, text, "rgemm")) return false;
    if (heuristic_default(d, role, di).str() != current.str()) return false;
    if (!database_config(d, role, di, c, "igemm")) c = plain_default(d, role, di);
    RoleBuild rb;
    if (!build_role(d, role, c, di, rb, err) || rb.ws_bytes) return false;
    out = c;
    return true;
}

bool config_from_text(const fbcorr_desc& d, int role, const DeviceInfo& di, const std::string& text,
                      bool reset_named, Config& out, std::string& err) {
    // A text that names an algorithm starts from that algorithm's
    // hand-written defaults ("algo=direct" alone is a complete
    // configuration), "algo=dws" from the tilings' cheapest, one that names
    // none from those of the kernels that fit any size; where the database
    // has an entry (for a text without an algorithm: also one of a form that
    // is not the problem's default), unnamed knobs are the entry's instead
    // (but not on the forward role with reset_named, if the text names an
    // algorithm).
    Config named;
    std::istringstream is(text);
    std::string tok;
    while (is >> tok)
        if (tok.compare(0, 5, "algo=") == 0) named.algo = tok.substr(5);
    Config c;
    bool entry = database_config(d, role, di, c);
    for (const char* form : {"igemm", "rgemm", "dw"})
        if (!entry && (named.algo.empty() || named.algo == form)) entry = database_config(d, role, di, c, form);
    if (!entry) c = plain_default(d, role, di);
    const int cin = role == FBCORR_ROLE_BACKWARD_X ? d.N : d.D;
    const int cout = role == FBCORR_ROLE_BACKWARD_X ? d.D : d.N;
    const bool lp = d.precision != FBCORR_FP32 && role == FBCORR_ROLE_FORWARD;
    const bool other = named.algo != c.algo, reset = other || (reset_named && role == FBCORR_ROLE_FORWARD);
    if (named.algo == "direct" && role == FBCORR_ROLE_FORWARD) c = default_direct(d);
    else if (named.algo == "igemm" && role != FBCORR_ROLE_BACKWARD_W && reset) c = default_igemm(cin, cout, lp);
    else if (named.algo == "rgemm" && role != FBCORR_ROLE_BACKWARD_W && reset) c = default_rgemm(cin, cout, lp);
    else if (named.algo == "dw" && role == FBCORR_ROLE_BACKWARD_W && other) c = plain_default(d, role, di);
    else if (named.algo == "dws" && role == FBCORR_ROLE_BACKWARD_W && other) {
        // (where none fits, the text has to name every knob)
        const std::vector<Config> cs = dws_tilings(d, di.cus, 1);
        if (!cs.empty()) c = cs[0];
    }
    if (!parse_config(text, c, err)) return false;
    out = c;
    return true;
}

}  // namespace fbc

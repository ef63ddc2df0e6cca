// Many uneven images in one launch.
//
// Every distinct problem key (fh, fw, D, N) of the batch gets one tile
// configuration, and the generator emits one kernel holding exactly those
// variants (Sec. 4.2: generate code for exactly one purpose): the body
// section of the key's kernel -- fp32 operands as three bf16 parts (rgemm),
// or fp32 instructions (igemm) -- is pasted once per key with that key's
// constants substituted and the image extents left run-time.  Each body stays
// a function of its own, so registers are allocated per variant.  At plan
// time the host builds a work table of (variant, image, tile) items sorted by
// cost, largest first; each workgroup runs one.  Before it, one launch packs
// the banks of the images whose variant is an rgemm, one workgroup per
// column.  Both launches can be captured once into a HIP graph per stream and
// replayed.
//
// One workgroup per item, not workgroups that loop over a counter: a wave
// that ends does not wait for its stores, one that takes another tile waits
// for them at its next load, and two workgroups per CU do not hide that (32
// images of 96 to 512 pixels a side, 365 GFLOP, three-part variants: 2115 us
// looping, 1590 us so; with fp32 instructions 3553 and 3390 us).
#include "plan.h"

#include <algorithm>
#include <cstring>
#include <numeric>
#include <set>
#include <sstream>

namespace fbc {

struct BVariant {
    int fh, fw, D, N;
    Config cfg;
    int th, two, cb;       // tile geometry: output rows, columns, channels
    int lds;
    int ncols = 0;         // rgemm: columns of a packed bank, and its bytes
    size_t bank = 0;
    bool parts() const { return cfg.algo == "rgemm"; }
    // the -DFB_<name>[=<value>] options build_role generated for this key's
    // standalone kernel (clamped and completed exactly as that kernel was)
    std::vector<std::string> opts;
};

struct BatchedState {
    std::vector<fbcorr_desc> descs;
    std::vector<BVariant> vars;
    std::vector<int> img_var;
    std::vector<int32_t> items;     // 4 ints per item: variant, image, tile, 0
    // 8 ints per image: H, W, Ho, Wo, then (rgemm) where its packed bank and
    // its column scales start in the workspace, in units of 256 bytes
    std::vector<int32_t> imgs;
    std::vector<int32_t> cols;      // 4 ints per packed column: variant, image, column, 0
    Kernel kernel, pack;
    int grid = 0, threads = 256, per_cu = 1;
    size_t off_items = 0, off_imgs = 0, off_cols = 0, ws_bytes = 0;
    int64_t nitems = 0;
    double flops = 0;
    std::string source_desc;
    // uploads and graphs
    std::set<void*> uploaded;
    struct GraphKey {
        hipStream_t s;
        void* ws;
        const void *xs, *wts, *ys;
        bool operator<(const GraphKey& o) const {
            return std::tie(s, ws, xs, wts, ys) < std::tie(o.s, o.ws, o.xs, o.wts, o.ys);
        }
    };
    std::map<GraphKey, std::pair<hipGraph_t, hipGraphExec_t>> graphs;
    std::mutex mu;           // uploads and graphs are shared by calling threads
};

static int cdiv(int a, int b) { return (a + b - 1) / b; }
static size_t align256(size_t x) { return (x + 255) / 256 * 256; }

// fp32 instructions; four waves per workgroup for every variant (one block
// size for the launch).
static Config batched_variant_config(int D, int N) {
    Config c = default_igemm(D, N, false);
    const int s = c.get("s");
    const int tiles = std::min(4, std::max(1, cdiv(N * s, 32)));
    int nt = 1, wn = 1;
    if (tiles >= 4) { nt = 2; wn = 2; }
    else if (tiles >= 2) { nt = 2; wn = 1; }
    const int wm = 4 / wn;
    c.v["nt"] = nt;
    c.v["wn"] = wn;
    c.v["wm"] = wm;
    c.v["ks"] = 1;
    c.v["mt"] = 1;
    c.v["mr"] = 2;
    c.v["ustage"] = 1;
    c.v["kc"] = D <= 16 ? D : 16;
    c.v["mf"] = 32;
    return c;
}

static std::vector<std::string> body_macros(const std::string& body) {
    std::vector<std::string> names;
    std::istringstream is(body);
    std::string line;
    while (std::getline(is, line)) {
        size_t p = line.find_first_not_of(" \t");
        if (p == std::string::npos || line.compare(p, 7, "#define") != 0) continue;
        std::istringstream ls(line.substr(p + 7));
        std::string name;
        ls >> name;
        auto paren = name.find('(');
        if (paren != std::string::npos) name = name.substr(0, paren);
        if (!name.empty()) names.push_back(name);
    }
    return names;
}

// The part of a kernel template between its BODY markers, and what precedes it.
struct Body {
    std::string header, text;
    std::vector<std::string> macros;
};

static bool template_body(const std::string& file, Body& out, std::string& err) {
    const std::string& tpl = template_source(file);
    const auto b0 = tpl.find("//@@BODY-BEGIN"), b1 = tpl.find("//@@BODY-END");
    if (b0 == std::string::npos || b1 == std::string::npos) { err = file + " template lacks body markers"; return false; }
    out.header = tpl.substr(0, b0);
    // without comments: the text is repeated per key, and every plan hashes it
    bool comment = false;
    for (size_t i = b0; i < b1; ++i) {
        if (tpl[i] == '\n') comment = false;
        else if (tpl[i] == '/' && tpl[i + 1] == '/') comment = true;
        if (!comment) out.text += tpl[i];
    }
    out.macros = body_macros(out.text);
    return true;
}

static bool generate(BatchedState& st, KernelSource& ks, std::string& err) {
    Body igemm, rgemm;
    if (!template_body("igemm", igemm, err) || !template_body("rgemm", rgemm, err)) return false;
    std::ostringstream src;
    src << "// Generated batched filter-bank correlation: " << st.vars.size() << " variant(s).\n";
    src << "#define FB_BATCHED 1\n" << igemm.header << rgemm.header;
    int maxlds = 16;
    // Options of the standalone kernel that do not apply inside the
    // batched kernel: its name, the batch, the image extents (run-time
    // arguments here) and the workgroup order (the work table).
    static const std::set<std::string> skip = {"FB_KNAME", "FB_BATCH", "FB_HI", "FB_WI", "FB_HO", "FB_WO",
                                               "FB_XCDMAP"};
    for (size_t v = 0; v < st.vars.size(); ++v) {
        const BVariant& bv = st.vars[v];
        const Body& body = bv.parts() ? rgemm : igemm;
        src << "\n// ---- variant " << v << ": fh=" << bv.fh << " fw=" << bv.fw << " D=" << bv.D << " N=" << bv.N
            << "  [" << bv.cfg.str() << "]\n";
        src << "#undef FB_TAG\n#define FB_TAG v" << v << "\n";
        // The variant's constants are exactly those its standalone kernel
        // was built (and tuned) with: clamped values, unrolling switches and
        // all.
        std::vector<std::string> defined;
        for (const std::string& o : bv.opts) {
            if (o.compare(0, 2, "-D") != 0) continue;
            const auto eq = o.find('=');
            const std::string name = o.substr(2, eq == std::string::npos ? std::string::npos : eq - 2);
            if (skip.count(name) || name.find('(') != std::string::npos) continue;
            src << "#define " << name << " " << (eq == std::string::npos ? std::string("1") : o.substr(eq + 1))
                << "\n";
            defined.push_back(name);
        }
        if (bv.parts()) {
            src << "#define FB_NCOLW (FB_WN * FB_NT * FB_MF)\n";       // as the pack is given it
            defined.push_back("FB_NCOLW");
            src << "namespace v" << v << " {\n" << body.text << "\n}\n";
        } else {
            src << body.text << "\n";
        }
        for (auto& m : body.macros) src << "#undef " << m << "\n";
        for (auto& d : defined) src << "#undef " << d << "\n";
        maxlds = std::max(maxlds, bv.lds);
    }
    src << "\n#define MAXLDS " << ((maxlds + 15) / 16 * 16) << "\n";
    src << R"KSRC(
// One workgroup per item (variant, image, tile) of the table.  Two waves per
// SIMD (registers within 256; every variant's LDS within half a CU): two
// workgroups per CU.
extern "C" __global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
fbcorr_batched(const int4* __restrict__ items, const int4* __restrict__ imgs,
               const float* const* __restrict__ xs, const float* const* __restrict__ wts,
               float* const* __restrict__ ys, const char* __restrict__ ws, const int first)
{
    __shared__ __attribute__((aligned(16))) unsigned char lds_raw[MAXLDS];
    const int4 w = items[first + blockIdx.x];
    const int4 im = imgs[2 * w.y], at = imgs[2 * w.y + 1];
    const float* x = xs[w.y];
    const float* wt = wts[w.y];
    float* y = ys[w.y];
    RG_GLOBAL const rg_u32x4* bank = (RG_GLOBAL const rg_u32x4*)(ws + (size_t)(unsigned)at.x * 256);
    RG_GLOBAL const float* unscale = (RG_GLOBAL const float*)(ws + (size_t)(unsigned)at.y * 256);
    (void)bank; (void)unscale;
    switch (w.x) {
)KSRC";
    for (size_t v = 0; v < st.vars.size(); ++v) {
        const BVariant& bv = st.vars[v];
        src << "    case " << v << ":";
        if (bv.parts())
            src << " v" << v << "::rgemm_body((RG_GLOBAL const float*)x, bank, unscale, (RG_GLOBAL const float*)wt, "
                << "(RG_GLOBAL float*)y, im.x, im.y, im.z, im.w, w.z, (RG_LDS rg_u32x4*)lds_raw);\n";
        else
            src << " {\n"
                << "        const int ntx = (im.w + " << bv.two - 1 << ") / " << bv.two << ";\n"
                << "        const int nty = (im.z + " << bv.th - 1 << ") / " << bv.th << ";\n"
                << "        const int tx = w.z % ntx, ty = (w.z / ntx) % nty, cb = w.z / (ntx * nty);\n"
                << "        igemm_body_v" << v << "(x, wt, nullptr, y, im.x, im.y, im.z, im.w, ty * " << bv.th
                << ", tx * " << bv.two << ", cb * " << bv.cb << ", lds_raw);\n"
                << "    } break;\n";
    }
    src << R"KSRC(    default: break;
    }
}

// Before it: the packed banks, one workgroup per column of the table.
extern "C" __global__ void __launch_bounds__(256)
fbcorr_batched_pack(const int4* __restrict__ cols, const int4* __restrict__ imgs,
                    const float* const* __restrict__ wts, char* __restrict__ ws)
{
    __shared__ float red[4];
    const int4 w = cols[blockIdx.x];
    const int4 at = imgs[2 * w.y + 1];
    const float* wt = wts[w.y];
    RG_GLOBAL rg_u32x4* bank = (RG_GLOBAL rg_u32x4*)(ws + (size_t)(unsigned)at.x * 256);
    RG_GLOBAL float* unscale = (RG_GLOBAL float*)(ws + (size_t)(unsigned)at.y * 256);
    (void)wt; (void)bank; (void)unscale;
    switch (w.x) {
)KSRC";
    for (size_t v = 0; v < st.vars.size(); ++v)
        if (st.vars[v].parts())
            src << "    case " << v << ": v" << v << "::rg_pack((RG_GLOBAL const float*)wt, bank, unscale, w.z, (RG_LDS float*)red); break;\n";
    src << R"KSRC(    default: break;
    }
}
)KSRC";
    ks.name = "fbcorr_batched";
    ks.file = "batched";
    ks.source = src.str();
    ks.options.clear();
    return true;
}

void destroy_batched(Plan* p) {
    if (!p->bstate) return;
    for (auto& g : p->bstate->graphs) {
        hipGraphExecDestroy(g.second.second);
        hipGraphDestroy(g.second.first);
    }
    delete p->bstate;
    p->bstate = nullptr;
}

std::string batched_describe(const Plan* p) {
    if (!p->bstate) return "batched";
    std::ostringstream os;
    os << "batched images=" << p->bstate->descs.size() << " variants=" << p->bstate->vars.size()
       << " items=" << p->bstate->nitems << " grid=" << p->bstate->grid << " per_cu=" << p->bstate->per_cu;
    for (size_t v = 0; v < p->bstate->vars.size(); ++v) {
        const BVariant& b = p->bstate->vars[v];
        os << " | v" << v << " fh=" << b.fh << " fw=" << b.fw << " D=" << b.D << " N=" << b.N << " " << b.cfg.str();
    }
    return os.str();
}

// Plan-time work shared by the device and the offline paths: variants, the
// work table, the workspace layout and the generated source.
using KeyT = std::tuple<int, int, int, int>;

// The tuning-database key of a batched variant: role "batched", extents 0.
static fbcorr_desc variant_key_desc(int fh, int fw, int D, int N) {
    fbcorr_desc k{};
    k.batch = 1; k.H = 0; k.W = 0; k.D = D; k.N = N; k.fh = fh; k.fw = fw;
    k.precision = FBCORR_FP32; k.algo = FBCORR_ALGO_AUTO; k.flags = 0;
    return k;
}
static const int kRoleBatched = 3;

// Which keys gain from three-part products.  Packing reads and writes every
// weight of every image (6 ps a weight, many banks), whatever the number of
// output pixels; it pays where that is less than what the products save, 0.6
// of the time on fp32 instructions (the rest is what three parts take).  That
// time: a workgroup's staging and products one after another (63 ns per
// contraction value; 95 where rows have fewer than 16 channels), 350
// workgroups at a time, or the filters it reads (3 TB/s; 1.2 TB/s when all
// banks together are past the last-level cache); for the whole batch at
// least one workgroup's, shared by the keys as their parts are.  Measured,
// us on fp32 instructions and with parts: 256 images of 64 channels with 256
// 3x3 filters, 16 output pixels each 63 and 280, 256 pixels 219 and 397, 529
// pixels 645 and 495; 48 of 32 channels with 512 9x9 filters, 16 pixels 289
// and 454, 256 pixels 946 and 513; 32 of 32 with 128 11x11, 16 pixels 227
// and 104.
static std::set<KeyT> parts_that_pay(int32_t count, const fbcorr_desc* descs) {
    struct Work { double weights = 0, wgs = 0, chain = 0, bytes = 0; };
    std::map<KeyT, Work> keys;
    double banks = 0;
    for (int32_t i = 0; i < count; ++i) {
        const fbcorr_desc& d = descs[i];
        Config c = batched_variant_config(d.D, d.N);
        const int s = c.get("s"), th = c.get("wm") * c.get("mt") * c.get("mr"), two = s * c.get("mf") / c.get("mr");
        const int cb = c.get("wn") * c.get("nt") * c.get("mf") / s;
        const double k = (double)d.fh * d.fw * d.D;
        const double wgs = (double)cdiv(d.H - d.fh + 1, th) * cdiv(d.W - d.fw + 1, two) * cdiv(d.N, cb);
        Work& w = keys[std::make_tuple(d.fh, d.fw, d.D, d.N)];
        w.weights += k * d.N;
        w.wgs += wgs;
        w.chain = k * (d.D >= 16 ? 0.063 : 0.095);
        w.bytes += wgs * std::min(cb, d.N) * k * 4;
        banks += k * d.N * 4;
    }
    const double rate = banks > 192e6 ? 1.2e6 : 3e6;          // bytes per microsecond
    auto plain = [&](const Work& w) { return std::max(w.chain * w.wgs / 350, w.bytes / rate); };
    double sum = 0, chain = 0;
    for (auto& kv : keys) {
        sum += plain(kv.second);
        chain = std::max(chain, kv.second.chain);
    }
    std::set<KeyT> out;
    for (auto& kv : keys)
        if (6e-6 * kv.second.weights < 0.6 * plain(kv.second) * std::max(1.0, chain / sum)) out.insert(kv.first);
    return out;
}

static fbcorr_status prepare_batched(const DeviceInfo& dev, int32_t count, const fbcorr_desc* descs,
                                     BatchedState* st, KernelSource& ks,
                                     const std::map<KeyT, Config>* overrides = nullptr) {
    for (int32_t i = 0; i < count; ++i) {
        fbcorr_status s0 = validate_desc(&descs[i]);
        if (s0 != FBCORR_OK) return s0;
        FBC_RETURN_IF(descs[i].batch != 1, FBCORR_ERR_INVALID_ARGUMENT, "batched descriptors must have batch = 1");
        FBC_RETURN_IF(descs[i].precision != FBCORR_FP32, FBCORR_ERR_UNSUPPORTED, "batched plans compute in fp32");
    }
    std::map<KeyT, int> keyidx;
    std::map<KeyT, fbcorr_desc> largest;          // of each key, by input pixels
    for (int32_t i = 0; i < count; ++i) {
        const fbcorr_desc& d = descs[i];
        auto l = largest.emplace(std::make_tuple(d.fh, d.fw, d.D, d.N), d).first;
        if ((double)d.H * d.W > (double)l->second.H * l->second.W) l->second = d;
    }
    const std::set<KeyT> pays = parts_that_pay(count, descs);
    for (int32_t i = 0; i < count; ++i) {
        const fbcorr_desc d = descs[i];
        st->descs.push_back(d);
        auto key = std::make_tuple(d.fh, d.fw, d.D, d.N);
        auto it = keyidx.find(key);
        if (it == keyidx.end()) {
            BVariant bv{d.fh, d.fw, d.D, d.N, batched_variant_config(d.D, d.N), 0, 0, 0, 0};
            RoleBuild rb;
            std::string err;
            bool ok = false;
            // a tuned configuration for this key: from the caller, else the database
            Config tuned;
            bool have = false;
            if (overrides) {
                auto o = overrides->find(key);
                if (o != overrides->end()) { tuned = o->second; have = true; }
            }
            std::string text;
            if (!have && tuning_db_lookup(dev.arch, kRoleBatched, variant_key_desc(d.fh, d.fw, d.D, d.N), text)) {
                tuned = bv.cfg;
                have = parse_config(text, tuned, err);
            }
            auto fits = [&](const Config& c) {
                return build_role(d, FBCORR_ROLE_FORWARD, c, dev, rb, err) && rb.main_geom.lds <= kBatchedLds;
            };
            if (have && batched_form(tuned) && fits(tuned)) {
                bv.cfg = tuned;
                ok = true;
            }
            // three bf16 parts, but for windows too short to be anything but
            // memory traffic, 1x1 windows of many channels, staged chunk by
            // chunk for one use (16 images of 64 channels with 200 filters
            // 355 us on fp32 instructions, 525 with parts; 32 of 33 with 60,
            // 156 and 196), and banks that take longer to pack than their
            // products save
            if (!ok && three_parts_window(d) && (d.fh * d.fw > 1 || d.D <= 32) && pays.count(key)) {
                const Config parts = batched_parts(largest[key]);
                if (batched_form(parts) && fits(parts)) {
                    bv.cfg = parts;
                    ok = true;
                }
            }
            // otherwise fp32 instructions, shrunk until they fit half a CU's LDS
            // (the launch's occupancy is set by its largest variant: two
            // workgroups per CU need every variant within half)
            for (int attempt = 0; attempt < 8 && !ok; ++attempt) {
                ok = fits(bv.cfg);
                if (!ok) {
                    if (bv.cfg.v["kc"] > 4) bv.cfg.v["kc"] /= 2;
                    else if (bv.cfg.v["mr"] > 1) bv.cfg.v["mr"] /= 2;
                    else if (bv.cfg.v["nt"] > 1) bv.cfg.v["nt"] /= 2;
                    else break;
                }
            }
            // the smallest configuration if even that does not fit half
            if (!ok) ok = build_role(d, FBCORR_ROLE_FORWARD, bv.cfg, dev, rb, err);
            FBC_RETURN_IF(!ok, FBCORR_ERR_UNSUPPORTED, "no batched variant fits for key: " + err);
            const int s = bv.cfg.get("s");
            bv.th = bv.cfg.get("wm") * bv.cfg.get("mt") * bv.cfg.get("mr");
            const int mf = bv.cfg.get("mf");
            bv.two = s * (mf / bv.cfg.get("mr"));
            bv.cb = bv.cfg.get("wn") * bv.cfg.get("nt") * mf / s;
            bv.lds = rb.main_geom.lds;
            bv.opts = rb.main.options;
            if (bv.parts()) {
                bv.ncols = rb.aux_geom[0].grid_x;
                bv.bank = rb.ws_unscale;
            }
            it = keyidx.emplace(key, (int)st->vars.size()).first;
            st->vars.push_back(bv);
        }
        st->img_var.push_back(it->second);
    }
    // Work table, images with the costliest tiles first (stable).  Workgroups
    // go to the eight XCDs in turn: each XCD takes a contiguous part of an
    // image's tiles (shared halos stay in its L2), the longest part left once
    // its own is used up.  An image of at most 16 tiles goes to one XCD as a
    // whole, so that its bank is read into one L2 (128 images of two tiles
    // with 128 11x11x32 filters: 325 us, 539 with the tiles side by side).
    for (int32_t i = 0; i < count; ++i) {
        const fbcorr_desc& d = st->descs[i];
        const BVariant& bv = st->vars[st->img_var[i]];
        const int ho = d.H - d.fh + 1, wo = d.W - d.fw + 1;
        st->imgs.insert(st->imgs.end(), {d.H, d.W, ho, wo, 0, 0, 0, 0});
        for (int c = 0; c < bv.ncols; ++c) st->cols.insert(st->cols.end(), {st->img_var[i], i, c, 0});
        st->flops += 2.0 * ho * wo * d.N * d.fh * d.fw * d.D;
    }
    std::vector<int32_t> order(count);
    std::iota(order.begin(), order.end(), 0);
    auto tile_cost = [&](int32_t i) {
        const BVariant& bv = st->vars[st->img_var[i]];
        // (an operation of the fp32 instructions takes twice as long)
        return (double)bv.th * bv.two * bv.cb * bv.fh * bv.fw * bv.D * (bv.parts() ? 1 : 2);
    };
    std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return tile_cost(a) > tile_cost(b); });
    std::vector<std::pair<int32_t, int32_t>> queue[8];
    double load[8] = {};
    size_t total = 0;
    for (int32_t i : order) {
        const fbcorr_desc& d = st->descs[i];
        const BVariant& bv = st->vars[st->img_var[i]];
        const long nt = (long)cdiv(d.W - d.fw + 1, bv.two) * cdiv(d.H - d.fh + 1, bv.th) * cdiv(d.N, bv.cb);
        total += nt;
        FBC_RETURN_IF(total > 0x7fffffff, FBCORR_ERR_UNSUPPORTED, "too many tiles");
        // few tiles: all on one XCD, the one with the least work
        const int one = nt <= 16 ? (int)(std::min_element(load, load + 8) - load) : -1;
        for (long k = 0; k < nt; ++k) {
            const int x = one >= 0 ? one : (int)(k * 8 / nt);
            queue[x].push_back({i, (int32_t)k});
            load[x] += tile_cost(i);
        }
    }
    // workgroups go to the XCDs in turn
    size_t at[8] = {}, left = 0;
    for (auto& q : queue) left += q.size();
    for (int x = 0; left > 0; --left, x = (x + 1) % 8) {
        int z = x;
        if (at[x] == queue[x].size())
            for (int k = 0; k < 8; ++k)
                if (queue[k].size() - at[k] > queue[z].size() - at[z]) z = k;
        const auto& t = queue[z][at[z]++];
        st->items.insert(st->items.end(), {st->img_var[t.first], t.first, t.second, 0});
    }
    st->nitems = (int64_t)(st->items.size() / 4);
    // workspace: items | image table | column table | packed banks and their
    // scales
    st->off_items = 0;
    st->off_imgs = st->off_items + align256(st->items.size() * 4);
    st->off_cols = st->off_imgs + align256(st->imgs.size() * 4);
    st->ws_bytes = st->off_cols + align256(st->cols.size() * 4);
    for (int32_t i = 0; i < count; ++i) {
        const BVariant& bv = st->vars[st->img_var[i]];
        if (!bv.parts()) continue;
        st->imgs[8 * i + 4] = (int32_t)(uint32_t)(st->ws_bytes / 256);
        st->ws_bytes += align256(bv.bank);
        st->imgs[8 * i + 5] = (int32_t)(uint32_t)(st->ws_bytes / 256);
        st->ws_bytes += align256((size_t)bv.ncols * 4);
    }
    FBC_RETURN_IF(st->ws_bytes / 256 > 0xffffffffull, FBCORR_ERR_UNSUPPORTED, "packed banks too large");
    std::string err;
    FBC_RETURN_IF(!generate(*st, ks, err), FBCORR_ERR_INTERNAL, err);
    return FBCORR_OK;
}

static fbcorr_status build_batched(Plan* p, int32_t count, const fbcorr_desc* descs) {
    std::unique_ptr<BatchedState> st(new BatchedState());
    KernelSource ks;
    fbcorr_status s = prepare_batched(p->dev, count, descs, st.get(), ks);
    if (s != FBCORR_OK) return s;
    s = load_kernel(ks, p->device, st->kernel);
    if (s != FBCORR_OK) return s;
    KernelSource rs = ks;
    rs.name = "fbcorr_batched_pack";
    s = load_kernel(rs, p->device, st->pack);
    if (s != FBCORR_OK) return s;
    int per_cu = 0;
    hipError_t e = hipModuleOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, st->kernel.fn, 256, 0);
    if (e != hipSuccess || per_cu < 1) per_cu = 1;
    st->per_cu = per_cu;
    st->grid = (int)st->nitems;
    p->batch_ws = st->ws_bytes;
    p->bstate = st.release();
    return FBCORR_OK;
}

static fbcorr_status launch_batched(Plan* p, const float* const* xs, const float* const* wts, float* const* ys,
                                    void* ws, hipStream_t s) {
    BatchedState* st = p->bstate;
    char* base = (char*)ws;
    const void* items = base + st->off_items;
    const void* imgs = base + st->off_imgs;
    const void* cols = base + st->off_cols;
    fbcorr_status r = FBCORR_OK;
    hipEvent_t ev;
    timing_begin(p, FBCORR_ROLE_FORWARD, s, ev);
    if (!st->cols.empty()) {
        void* a0[] = {(void*)&cols, (void*)&imgs, (void*)&wts, &base};
        r = launch(st->pack, LaunchGeom{(int)(st->cols.size() / 4), 1, 256, 0}, s, a0);
    }
    int first = 0;
    void* a1[] = {(void*)&items, (void*)&imgs, (void*)&xs, (void*)&wts, (void*)&ys, &base, &first};
    // (a launch has less than 2^32 threads)
    constexpr int kMostGroups = 0xffffffffu / 256;
    for (; r == FBCORR_OK && first < st->grid; first += std::min(kMostGroups, st->grid - first))
        r = launch(st->kernel, LaunchGeom{std::min(kMostGroups, st->grid - first), 1, 256, 0}, s, a1);
    timing_end(p, FBCORR_ROLE_FORWARD, s, ev);
    return r;
}

// Representative problem of a variant: its largest image.
static fbcorr_desc variant_rep(const BatchedState* st, size_t v) {
    const BVariant& bv = st->vars[v];
    fbcorr_desc best{};
    double bf = -1;
    for (size_t i = 0; i < st->descs.size(); ++i) {
        if (st->img_var[i] != (int)v) continue;
        const fbcorr_desc& d = st->descs[i];
        const double f = (double)(d.H - d.fh + 1) * (d.W - d.fw + 1);
        if (f > bf) { bf = f; best = d; }
    }
    (void)bv;
    return best;
}

size_t batched_tune_workspace(const Plan* p) {
    size_t need = 0;
    if (!p->bstate) return 0;
    for (size_t v = 0; v < p->bstate->vars.size(); ++v) {
        Plan tmp;
        tmp.desc = variant_rep(p->bstate, v);
        tmp.device = p->device;
        tmp.dev = p->dev;
        need = std::max(need, tune_workspace(&tmp));
    }
    return need;
}

// Per-key tuning of a batched plan (Sec. 6.2: the best variant differs per
// input): each variant is tuned on its largest image among the candidates
// that the batched kernel can hold, then the batched kernel is regenerated.
fbcorr_status tune_batched(Plan* p, void* workspace, size_t workspace_bytes, hipStream_t s,
                           const fbcorr_tune_opts* opts, fbcorr_tune_report* report) {
    BatchedState* st = p->bstate;
    FBC_RETURN_IF(!st, FBCORR_ERR_INVALID_ARGUMENT, "not a batched plan");
    fbcorr_tune_opts o{};
    if (opts) o = *opts;
    o.role = FBCORR_ROLE_FORWARD;
    o.flags &= ~(1u | 4u);      // no direct variants in the batched kernel
    const bool record = opts && (opts->flags & 2u);
    fbcorr_tune_report total;
    memset(&total, 0, sizeof total);
    std::map<KeyT, Config> chosen;
    for (size_t v = 0; v < st->vars.size(); ++v) {
        const BVariant& bv = st->vars[v];
        Plan tmp;
        tmp.desc = variant_rep(st, v);
        tmp.device = p->device;
        tmp.dev = p->dev;
        fbcorr_tune_report r;
        Config best;
        fbcorr_status e = tune_plan(&tmp, nullptr, nullptr, nullptr, workspace, workspace_bytes, s, &o, true, false,
                                    &r, &best);
        if (e != FBCORR_OK) return e;
        total.n_tried += r.n_tried;
        total.n_compiled += r.n_compiled;
        total.n_rejected_resources += r.n_rejected_resources;
        total.n_rejected_parity += r.n_rejected_parity;
        total.n_failed += r.n_failed;
        total.best_ms += r.best_ms;
        total.default_ms += r.default_ms;
        const KeyT key = std::make_tuple(bv.fh, bv.fw, bv.D, bv.N);
        if (batched_form(best)) {
            chosen[key] = best;
            if (record) {
                std::string err;
                FBC_RETURN_IF(!tuning_db_record(p->dev.arch, kRoleBatched, variant_key_desc(bv.fh, bv.fw, bv.D, bv.N),
                                                best.str(), err),
                              FBCORR_ERR_INTERNAL, err);
            }
        }
    }
    // regenerate the batched kernel with the chosen variants
    std::unique_ptr<BatchedState> ns(new BatchedState());
    KernelSource ks;
    fbcorr_status e = prepare_batched(p->dev, (int32_t)st->descs.size(), st->descs.data(), ns.get(), ks, &chosen);
    if (e != FBCORR_OK) return e;
    e = load_kernel(ks, p->device, ns->kernel);
    if (e != FBCORR_OK) return e;
    KernelSource rs = ks;
    rs.name = "fbcorr_batched_pack";
    e = load_kernel(rs, p->device, ns->pack);
    if (e != FBCORR_OK) return e;
    int per_cu = 0;
    if (hipModuleOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, ns->kernel.fn, 256, 0) != hipSuccess || per_cu < 1)
        per_cu = 1;
    ns->per_cu = per_cu;
    ns->grid = (int)ns->nitems;
    destroy_batched(p);
    p->batch_ws = ns->ws_bytes;
    p->bstate = ns.release();
    snprintf(total.best_cfg, sizeof total.best_cfg, "%zu variants tuned", chosen.size());
    snprintf(total.default_cfg, sizeof total.default_cfg, "per-key heuristics");
    if (report) *report = total;
    return FBCORR_OK;
}

}  // namespace fbc

using namespace fbc;

extern "C" fbcorr_status fbcorr_plan_batched(int32_t count, const fbcorr_desc* descs, int device, fbcorr_plan_t* out) {
    try {
        clear_error();
        FBC_RETURN_IF(!out || !descs, FBCORR_ERR_INVALID_ARGUMENT, "NULL argument");
        FBC_RETURN_IF(count <= 0, FBCORR_ERR_INVALID_ARGUMENT, "count must be >= 1");
        std::unique_ptr<Plan> p(new Plan());
        p->desc = descs[0];
        p->device = device;
        p->batched = true;
        fbcorr_status st = device_info(device, p->dev);
        if (st != FBCORR_OK) return st;
        DeviceGuard g(device);
        st = build_batched(p.get(), count, descs);
        if (st != FBCORR_OK) return st;
        *out = reinterpret_cast<fbcorr_plan_t>(p.release());
        return FBCORR_OK;
    } catch (const std::exception& e) {
        set_error(FBCORR_ERR_INTERNAL, std::string("exception: ") + e.what());
        return FBCORR_ERR_INTERNAL;
    }
}

extern "C" fbcorr_status fbcorr_forward_batched(fbcorr_plan_t plan, const float* const* xs, const float* const* ws_,
                                                float* const* ys, void* workspace, size_t workspace_bytes,
                                                void* stream, int use_graph) {
    try {
        clear_error();
        Plan* p = reinterpret_cast<Plan*>(plan);
        FBC_RETURN_IF(!p || !p->batched || !p->bstate, FBCORR_ERR_INVALID_ARGUMENT, "not a batched plan");
        FBC_RETURN_IF(!xs || !ws_ || !ys, FBCORR_ERR_INVALID_ARGUMENT, "pointer arrays must not be NULL");
        BatchedState* st = p->bstate;
        fbcorr_status r = check_ws(workspace, workspace_bytes, st->ws_bytes);
        if (r != FBCORR_OK) return r;
        DeviceGuard g(p->device);
        hipStream_t s = (hipStream_t)stream;
        std::lock_guard<std::mutex> lock(st->mu);
        if (!st->uploaded.count(workspace)) {
            // the work table and image table live in the caller's workspace
            char* base = (char*)workspace;
            hipError_t e = hipMemcpyAsync(base + st->off_items, st->items.data(), st->items.size() * 4,
                                          hipMemcpyHostToDevice, s);
            if (e == hipSuccess)
                e = hipMemcpyAsync(base + st->off_imgs, st->imgs.data(), st->imgs.size() * 4,
                                   hipMemcpyHostToDevice, s);
            if (e == hipSuccess && !st->cols.empty())
                e = hipMemcpyAsync(base + st->off_cols, st->cols.data(), st->cols.size() * 4, hipMemcpyHostToDevice,
                                   s);
            if (e == hipSuccess) e = hipStreamSynchronize(s);
            FBC_RETURN_IF(e != hipSuccess, FBCORR_ERR_LAUNCH, std::string("table upload: ") + hipGetErrorString(e));
            st->uploaded.insert(workspace);
        }
        if (!use_graph) return launch_batched(p, xs, ws_, ys, workspace, s);
        FBC_RETURN_IF(s == nullptr, FBCORR_ERR_INVALID_ARGUMENT,
                      "graph capture needs a created stream, not the null stream");
        BatchedState::GraphKey key{s, workspace, xs, ws_, ys};
        auto it = st->graphs.find(key);
        if (it == st->graphs.end()) {
            hipGraph_t graph = nullptr;
            hipGraphExec_t exec = nullptr;
            hipError_t e = hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal);
            FBC_RETURN_IF(e != hipSuccess, FBCORR_ERR_LAUNCH, std::string("begin capture: ") + hipGetErrorString(e));
            const bool was = p->timing;
            p->timing = false;             // no event records inside the graph
            r = launch_batched(p, xs, ws_, ys, workspace, s);
            p->timing = was;
            e = hipStreamEndCapture(s, &graph);
            FBC_RETURN_IF(r != FBCORR_OK, r, fbcorr_last_error());
            FBC_RETURN_IF(e != hipSuccess, FBCORR_ERR_LAUNCH, std::string("end capture: ") + hipGetErrorString(e));
            e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
            if (e != hipSuccess) {
                hipGraphDestroy(graph);
                set_error(FBCORR_ERR_LAUNCH, std::string("graph instantiate: ") + hipGetErrorString(e));
                return FBCORR_ERR_LAUNCH;
            }
            it = st->graphs.emplace(key, std::make_pair(graph, exec)).first;
        }
        hipEvent_t ev;
        timing_begin(p, FBCORR_ROLE_FORWARD, s, ev);
        hipError_t e = hipGraphLaunch(it->second.second, s);
        timing_end(p, FBCORR_ROLE_FORWARD, s, ev);
        FBC_RETURN_IF(e != hipSuccess, FBCORR_ERR_LAUNCH, std::string("graph launch: ") + hipGetErrorString(e));
        return FBCORR_OK;
    } catch (const std::exception& e) {
        set_error(FBCORR_ERR_INTERNAL, std::string("exception: ") + e.what());
        return FBCORR_ERR_INTERNAL;
    }
}

extern "C" fbcorr_status fbcorr_compile_check_batched(int32_t count, const fbcorr_desc* descs, const char* arch,
                                                     size_t* code_bytes) {
    try {
        clear_error();
        FBC_RETURN_IF(!descs || count <= 0, FBCORR_ERR_INVALID_ARGUMENT, "need at least one descriptor");
        DeviceInfo di;
        di.arch = arch ? arch : "gfx950";
        di.cus = 256;
        di.lds_per_block = 160 * 1024;
        di.max_threads = 1024;
        BatchedState st;
        KernelSource ks;
        fbcorr_status s = prepare_batched(di, count, descs, &st, ks);
        if (s != FBCORR_OK) return s;
        std::shared_ptr<const std::vector<char>> code;
        s = compile_cached(ks, di.arch, code);
        if (s != FBCORR_OK) return s;
        if (code_bytes) *code_bytes = code->size();
        return FBCORR_OK;
    } catch (const std::exception& e) {
        set_error(FBCORR_ERR_INTERNAL, std::string("exception: ") + e.what());
        return FBCORR_ERR_INTERNAL;
    }
}

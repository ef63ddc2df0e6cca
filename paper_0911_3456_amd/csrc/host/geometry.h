// Launch geometry and per-role build descriptions.
#pragma once

#include "internal.h"

namespace fbc {

struct LaunchGeom {
    int grid_x = 0, grid_y = 1;
    int threads = 0;
    int lds = 0;
};

// Everything needed to run one role: the main kernel, helper kernels (run
// before the main kernel for the forward/input-gradient roles, after it for
// the filter-gradient role), their launch shapes, and workspace use.
struct RoleBuild {
    Config cfg;
    KernelSource main;
    LaunchGeom main_geom;
    std::vector<KernelSource> aux;
    std::vector<LaunchGeom> aux_geom;
    size_t ws_bytes = 0;
    size_t ws_lowp_w = 0, ws_unscale = 0;   // forward low-precision layout
    size_t ws_xmax = 0;                     // fp16: partial maxima of |x| (aux[1])
    int nxp = 0;                            //   their count (0: no input scale)
    int np = 0;                             // filter-gradient partial count
};

// The static device scratch of fbcorr_forward_noalloc (noalloc.hip): room
// for the packed bank of any filter bank up to a few million weights.
constexpr size_t kNoAllocScratchBytes = 16u << 20;

// LDS of a variant of the batched kernel: two workgroups per CU.
constexpr int kBatchedLds = 80 * 1024 - 256;

// Default configuration of a role: the tuning database's entry for this
// hardware and problem if there is one, else the hand-written heuristic
// (shrunk until it fits the device).
Config default_config(const fbcorr_desc& d, int role, const DeviceInfo& di);
Config heuristic_default(const fbcorr_desc& d, int role, const DeviceInfo& di);

// Whether `current`, the forward configuration of a plan, is the default that
// three bf16 parts gave it; then the configuration that the pass has without
// them, which needs no scratch.
bool scratchless_forward(const fbcorr_desc& d, const DeviceInfo& di, const Config& current, Config& out);

// tuning_db.cpp
std::string tuning_db_path();
bool tuning_db_lookup(const std::string& arch, int role, const fbcorr_desc& d, std::string& cfg,
                      const std::string& form = "");
bool tuning_db_record(const std::string& arch, int role, const fbcorr_desc& d, const std::string& cfg,
                      std::string& err);
void tuning_db_reload();
bool tuning_db_lookup_key(const std::string& key, std::string& cfg);
bool tuning_db_record_key(const std::string& key, const std::string& cfg, std::string& err);
Config default_igemm(int cin, int cout, bool lowp);
Config default_rgemm(int cin, int cout, bool lowp);
Config default_direct(const fbcorr_desc& d);
Config default_dw(const fbcorr_desc& d, int cus);
// The cheapest three-part tiling of four waves for the batched kernel (no
// algorithm if none fits).
Config batched_parts(const fbcorr_desc& d);
// Whether the batched kernel can hold the configuration: four waves, and
// (rgemm) three-part operands at two waves per SIMD.
bool batched_form(const Config& c);
// Windows long enough for three bf16 parts to pay.
bool three_parts_window(const fbcorr_desc& d);
// The cheapest `count` three-part filter-gradient tilings, cheapest first.
std::vector<Config> dws_tilings(const fbcorr_desc& d, int cus, int count);
// The configuration a text such as "algo=rgemm mt=2" describes for a role:
// unnamed knobs come from the role's default, or from the named algorithm's
// hand-written defaults when it differs from the default's (always, on the
// forward role, with reset_named).
bool config_from_text(const fbcorr_desc& d, int role, const DeviceInfo& di, const std::string& text,
                      bool reset_named, Config& out, std::string& err);
bool build_role(const fbcorr_desc& d, int role, const Config& c, const DeviceInfo& di,
                RoleBuild& rb, std::string& err);

// Tuning grids (tune.cpp).
std::vector<Config> tune_candidates(const fbcorr_desc& d, int role, bool with_direct, bool direct_only);

}  // namespace fbc

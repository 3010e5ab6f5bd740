// host_keys.hip -- the tuner key of a set and the plan index of a hop, as host
// functions, for the CPU tests of what they tell apart.  Test infrastructure only;
// linked with libwilson.so.
#include <cstring>

#include "../paper_2001_05706_amd/csrc/wl_host.h"

using namespace wl;

// The key of the FP32 recon-12 hop of a set of n systems of extents L[4 i ..] with
// nrhs[i] right-hand sides (no device call: the set is never initialised)
extern "C" int hop_key_of(int n, const int32_t *L, const int32_t *nrhs, char *out, int size)
{
    std::vector<std::unique_ptr<wl_gauge_s>> g;
    std::vector<SysEntry> sys;
    for (int i = 0; i < n; ++i) {
        g.emplace_back(new wl_gauge_s());
        SysDesc &d = g.back()->geom;
        d = SysDesc{};
        d.Vh = 1;
        for (int m = 0; m < 4; ++m) {
            d.L[m] = L[4 * i + m];
            d.Vh *= d.L[m];
        }
        d.Vh /= 2;
        d.Lxh = d.L[0] / 2;
        d.stride = padded(d.Vh);
        sys.push_back(SysEntry{g.back().get(), nrhs[i], 0.1});
    }
    ExecSet S(sys);
    S.nvec = 0;
    S.total_sites = 0;
    for (auto &e : sys) {
        S.nvec += e.nrhs;
        S.total_sites += (size_t)e.nrhs * e.g->geom.stride;
    }
    const std::string k = hop_key(S, P_F32, 12, false);
    if ((int)k.size() >= size) return 1;
    strcpy(out, k.c_str());
    return 0;
}

// The plan index of the D-slash call's hop (twin: of both parities) that reads the
// canonical input itself (direct) or a packed one
extern "C" int plan_id_of(int prec, int nx, int twin, int direct)
{
    double canon[1] = {0};
    Epi e;
    e.nx = nx;
    e.canon = canon;
    e.canon_in = direct ? canon : nullptr;
    return plan_id(prec, 12, false, false, e, false, twin != 0);
}

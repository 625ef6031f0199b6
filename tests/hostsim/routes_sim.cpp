// Stand-in launchers of kernels_sim.cpp with what the route tests add: they
// note launches whose kernel cannot serve the entries that it is given. Test
// infrastructure only.
#include "../../paper_2009_09103_amd/csrc/kernels.h"

#define launch_select placeholder_select
#include "kernels_sim.cpp"
#undef launch_select

namespace hipsim_hooks {
std::atomic<int64_t> misrouted{0};  // unbiased draws given to the kernel that draws by weight alone
}  // namespace hipsim_hooks

namespace csaw {

// Checked when the launch runs, so that a replayed launch is checked against
// the tables of the call that it serves.
void launch_select(const SampleLayer& p, int grid, hipStream_t s, LaunchEvents ev) {
    hipsim::enqueue(s, [p] {
        for (int64_t e = 0; p.wave_only && e < p.ctl->fcount[p.layer]; ++e) {
            const int32_t P = p.fpos[e] & ~kWideList;
            if (p.bias[p.fi[e]] == kUniform && p.cnt[e] > 0 && p.cnt[e] < P) ++hipsim_hooks::misrouted;
        }
    });
    placeholder_select(p, grid, s, ev);
}

}  // namespace csaw

// Host-only build of the library (test infrastructure): the engine launcher
// the host builder calls.  Without a stub device it fails; with one it keeps
// what would have been launched, for tests of the engine choice.
#include <hip/hip_runtime.h>

#include <string>

#include "../../include/simgpu.h"
#include "../../paper_2606_10440_amd/csrc/sim_internal.h"

namespace {
simgpu::DevNet last;
unsigned char scratch[SIM_NOALLOC_SCRATCH_BYTES];
}  // namespace

namespace simgpu {
int launch_engine(const DevNet &d, void *) {
    if (!stub_device()) return hipErrorNoDevice;
    last = d;
    return hipGetLastError();  // as the launchers do
}
sim_status run_on_scratch(sim_ctx *c, void *stream, uint32_t *d_completion, uint64_t *d_tx_lines,
                          uint64_t *d_busy_cycles, uint32_t *d_makespan, uint64_t max_cycles, void *scratch,
                          size_t scratch_bytes);
}  // namespace simgpu

// A number of the last launch, by name (-1: unknown name).
extern "C" int64_t stub_last(const char *name) {
    const std::string n(name);
    if (n == "engine") return last.engine;
    if (n == "lds_bytes") return last.lds_bytes;
    if (n == "wv_lineup") return last.wv_lineup;
    if (n == "wv_chain") return last.wv_chain;
    if (n == "wv_W") return last.wv_W;
    if (n == "wv_G") return last.wv_G;
    if (n == "wv_nblk") return last.wv_nblk;
    if (n == "wv_wpb") return last.wv_wpb;
    if (n == "gd_wave") return last.gd_wave;
    if (n == "gd_window") return last.gd_window;
    if (n == "gd_nb") return last.gd_nb;
    if (n == "gd_one") return last.gd_one;
    return -1;
}

// Wave of each slot (wv_nblk * wv_wpb) and scenario of each wave slot (wv_W * wv_G).
extern "C" const int32_t *stub_blk_wave() { return last.blk_wave; }
extern "C" const int32_t *stub_wv_sc() { return last.wv_sc; }

// The allocation-free run needs the device array of its own source file.
extern "C" sim_status sim_run_noalloc(sim_ctx *c, void *stream, uint32_t *d_completion, uint64_t *d_tx_lines,
                                      uint64_t *d_busy_cycles, uint32_t *d_makespan, uint64_t max_cycles) {
    if (!stub_device()) return SIM_ERR_DEVICE;
    return simgpu::run_on_scratch(c, stream, d_completion, d_tx_lines, d_busy_cycles, d_makespan, max_cycles, scratch,
                                  sizeof scratch);
}

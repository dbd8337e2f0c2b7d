// The wave engine's general round-robin loops at up to eight lines per cycle,
// in a translation unit of their own because they are scheduled differently.
#define SIMGPU_WAVE_RR8
#include "engine_wave.hip"

// Storage for the emulated HIP built-ins (see hip_emu.h).
#include "hip_emu.h"
thread_local uint3_ threadIdx;
thread_local uint3_ blockIdx;
thread_local dim3 blockDim, gridDim;
thread_local emu::Block* emu::g_block = nullptr;
thread_local emu::CoopRun* emu::g_coop = nullptr;
thread_local emu_graph* emu_capture = nullptr;
int emu_coop_blocks = 1, emu_spin_limit = 1000000, emu_stream_waits = 0, emu_event_waits = 0, emu_launches = 0, emu_trig = 0;

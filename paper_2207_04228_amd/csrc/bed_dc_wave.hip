// Instantiations of the divide-and-conquer kernels for 10 < n <= 32.
#include "bed_dc_wave_kernel.hpp"

namespace bed {
hipError_t launch_dc_wave(const KernelArgs& args, int stage, bool want_v, hipStream_t stream) {
    const int n = args.n;
    if (n <= 12) return launch_dc_n<12>(args, stage, want_v, stream);
    if (n <= 16) return launch_dc_n<16>(args, stage, want_v, stream);
    if (n <= 20) return launch_dc_n<20>(args, stage, want_v, stream);
    if (n <= 24) return launch_dc_n<24>(args, stage, want_v, stream);
    if (n <= 28) return launch_dc_n<28>(args, stage, want_v, stream);
    return launch_dc_n<32>(args, stage, want_v, stream);
}
}  // namespace bed

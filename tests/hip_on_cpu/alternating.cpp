// The alternating quantizer's kernels on the CPU.
#include <dlfcn.h>

#include "../../paper_2210_03858_amd/csrc/bcq_alternating.hip"

thread_local bool bcq::tl_dry_run = false;
namespace bcq {
alignas(16) unsigned char alt_smem[160 * 1024];  // the workgroup's shared memory
}
unsigned char* const emu::shared = bcq::alt_smem;
const size_t emu::shared_bytes = sizeof bcq::alt_smem;

extern "C" int quantize_alternating(const float* W, int64_t V, int64_t n, int q, int iters, float* alpha, uint32_t* packed, int* status,
                                    int backwards, int64_t* operations) {
    emu::backwards = backwards != 0;
    emu::operations = 0;
    const hipError_t e = bcq::launch_quantize_alternating(W, V, n, q, iters, alpha, packed, nullptr, status, nullptr);
    *operations = emu::operations;
    return e;
}

extern "C" const char* last_kernel() {  // its mangled name
    Dl_info info;
    return dladdr(emu::kernel, &info) && info.dli_sname ? info.dli_sname : "";
}

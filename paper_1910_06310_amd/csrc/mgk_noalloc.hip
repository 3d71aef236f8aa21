// Storage for mgk_pairs_noalloc: fixed arrays in device memory that exist once per GPU for the life of the
// process, so that the entry point needs no device allocation.  Compiled once for the job list and once for the packets
// of the separable product on chip: a module of its own each, loaded when its address is first asked for.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mgk_internal.h"
#include "mgk_launch.h"

#if defined(MGK_NOALLOC_JOBS)
#define MGK_BYTES ((size_t)MGK_NOALLOC_MAX_PAIRS * sizeof(MgkJob))   // 16 bytes a job, 1 MiB
#elif defined(MGK_NOALLOC_PACKETS)
#define MGK_BYTES ((size_t)MGK_ONCHIP_PACKET_BYTES)                  // as much as any call may use
#else
#error "compile with -DMGK_NOALLOC_JOBS or -DMGK_NOALLOC_PACKETS"
#endif

namespace {

// The job list, or the packets, of one call.  Every call on a GPU uses this one array and overwrites it from the start; it
// keeps what the previous call left until then, and nothing in it has to be cleared.
static __device__ __align__(256) unsigned char scratch[MGK_BYTES];

constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices] = {};   // device address of `scratch` on each GPU, 0 = not looked up yet

// Device address of the array on `device` (each GPU holds its own copy at its own
// address), looked up once per device with that device current.  In host code the array's
// name stands for the symbol, not for an address a kernel could use: only the pointer
// returned here is ever passed on.
hipError_t address_of_scratch(int device, void** out) {
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidValue;
    if (g_scratch_ptr[device] == nullptr) {
        int current = -1;
        hipError_t e = hipGetDevice(&current);
        if (e != hipSuccess) return e;
        if (current != device) {
            e = hipSetDevice(device);
            if (e != hipSuccess) return e;
        }
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (current != device && current >= 0) (void)hipSetDevice(current);
        if (e != hipSuccess) return e;
        if (ptr == nullptr) return hipErrorInvalidSymbol;
        g_scratch_ptr[device] = ptr;
    }
    *out = g_scratch_ptr[device];
    return hipSuccess;
}

}  // namespace

#ifdef MGK_NOALLOC_JOBS
hipError_t mgk_noalloc_job_storage(int device, MgkJob** jobs, int64_t* capacity) {
    if (!jobs || !capacity) return hipErrorInvalidValue;
    void* p = nullptr;
    hipError_t e = address_of_scratch(device, &p);
    if (e != hipSuccess) return e;
    *jobs = static_cast<MgkJob*>(p);
    *capacity = MGK_NOALLOC_MAX_PAIRS;
    return hipSuccess;
}
#else
hipError_t mgk_noalloc_packet_storage(int device, float** packets) {
    if (!packets) return hipErrorInvalidValue;
    void* p = nullptr;
    hipError_t e = address_of_scratch(device, &p);
    if (e == hipSuccess) *packets = static_cast<float*>(p);
    return e;
}
#endif

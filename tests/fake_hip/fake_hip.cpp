// Stands in for the HIP runtime calls that deft_plan_upload and the calls make, on a machine without a GPU: loaded with
// RTLD_GLOBAL before libdeft.so, its functions are the ones the library finds.  Kernels are counted and not run, copies are done
// at once.  What the calls answer is set by the test (tests/test_upload_errors.py, tests/test_recut.py).
#include <cstdint>
#include <cstdlib>
#include <cstring>

#include <hip/hip_runtime_api.h>

extern "C" {
struct {
    int32_t device, stream_device, pointer_device, pointer_type, capturing, event_error;  // answers
    int32_t launches, copies, events_recorded;                                            // calls made
    int32_t grid[16];         // workgroups of the launches, the last 16 of them,
    const void *kernel[16];   // and their kernels
} fake = {0, 0, 0, hipMemoryTypeDevice, hipStreamCaptureStatusNone, hipSuccess, 0, 0, 0, {}, {}};
static dim3 pushed;

hipError_t hipGetDevice(int *d) { *d = fake.device; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "fake"; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = aligned_alloc(4096, (n + 4095) / 4096 * 4096); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void **d, void *p, unsigned) { *d = p; return hipSuccess; }
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = (hipEvent_t)calloc(1, 8); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { ++fake.events_recorded; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return (hipError_t)fake.event_error; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *to, const void *from, size_t n, hipMemcpyKind, hipStream_t) {
    ++fake.copies;
    memcpy(to, from, n);
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *) {
    a->type = (hipMemoryType)fake.pointer_type;
    a->device = fake.pointer_device;
    return hipSuccess;
}
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t *d) { *d = fake.stream_device; return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) { *s = (hipStreamCaptureStatus)fake.capturing; return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3 grid, dim3, size_t, hipStream_t) { pushed = grid; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *, size_t *, hipStream_t *) { *grid = pushed; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipLaunchKernel(const void *kernel, dim3 grid, dim3, void **, size_t, hipStream_t) {
    fake.grid[fake.launches % 16] = (int32_t)grid.x;
    fake.kernel[fake.launches++ % 16] = kernel;
    return hipSuccess;
}
hipError_t hipExtLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t, hipEvent_t, hipEvent_t, int) {
    ++fake.launches;
    return hipSuccess;
}
}

// Results on their way to the host: words of the workspace into pinned host memory, by a kernel's own stores.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tessel_common.h"

namespace tessel {

// Words are written through to host memory one by one (system scope), the last one when all others have arrived.  One wave.
__device__ __forceinline__ void mail_word(uint32_t *to, uint32_t v) { __hip_atomic_store(to, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM); }

__global__ __launch_bounds__(kWave) void tell_kernel(const uint32_t *__restrict__ from, int words, DevMail *mail, uint32_t told)
{
    for (int w = threadIdx.x; w < words; w += kWave) mail_word(mail->words + w, from[w]);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // (all lanes' words have arrived)
    if (threadIdx.x == 0) mail_word(&mail->told, told);
}

// The launch's own status is returned.  (hipGetLastError() would also report a call that failed before on this thread, and the
// caller would take back the mail of a kernel that is on its way.)
int launch_tell(void *ws, size_t offset, size_t bytes, DevMail *mail, uint32_t told, void *stream)
{
    const uint32_t *from = (const uint32_t *)((char *)ws + offset);
    int words = (int)(bytes / 4);
    void *args[] = {&from, &words, &mail, &told};
    const hipError_t e = hipLaunchKernel((const void *)tell_kernel, dim3(1), dim3(kWave), args, 0, (hipStream_t)stream);
    if (e != hipSuccess) (void)hipGetLastError();
    return (int)e;
}

}  // namespace tessel

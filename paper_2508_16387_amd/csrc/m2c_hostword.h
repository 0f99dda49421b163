// m2c_hostword.h -- the calling thread's host-pinned words for the results
// of a call that waits for its stream before it returns.
//
// A word that a kernel stores there is visible to the host after the wait
// and costs nothing more than the wait (11 us on an MI355X, kernel included;
// a copy of one word from device memory into pageable memory and the wait
// take 22 us, into pinned memory 14 us, and the device word had to be
// allocated and cleared).  One block per host thread, allocated by its first
// call and freed when the thread ends: calls of several threads, and of one
// thread on several streams or GPUs, never share a block in flight, because
// each call has waited for its kernels when it returns.  Kernels write it
// with plain stores (an atomic on host memory would need the bus's support).
#ifndef M2C_HOSTWORD_H
#define M2C_HOSTWORD_H

#include <hip/hip_runtime.h>

namespace m2c {

constexpr size_t HOST_WORDS = 128;     // 8-byte words per thread

struct HostWords {
    unsigned long long* p = nullptr;
    HostWords() = default;
    HostWords(const HostWords&) = delete;
    HostWords& operator=(const HostWords&) = delete;
    ~HostWords()
    {
        if (p) (void)hipHostFree(p);
    }
};

// nullptr: no memory
inline unsigned long long* host_words()
{
    static thread_local HostWords w;
    if (!w.p && hipHostMalloc((void**)&w.p, HOST_WORDS * sizeof(*w.p), hipHostMallocPortable | hipHostMallocMapped) !=
                    hipSuccess)
        w.p = nullptr;
    return w.p;
}

}  // namespace m2c

#endif

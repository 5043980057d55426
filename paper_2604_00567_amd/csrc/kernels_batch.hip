// Instantiations of the uneven-batch persistent kernel for both precisions.
#include "batch_launch.hpp"
#include "fft_batch.hpp"

namespace dsfft {

template <class E>
static size_t batch_lds_bytes_t() {
    return batch_prefix_bytes<E>() + (size_t)batch_lds_elems() * sizeof(E);
}

static_assert(batch_prefix_bytes<uint32_t>() + (size_t)batch_lds_elems() * sizeof(uint32_t) <= kLdsBytes &&
                  batch_prefix_bytes<f2_t>() + (size_t)batch_lds_elems() * sizeof(f2_t) <= kLdsBytes,
              "the persistent kernel fits a workgroup's LDS");

size_t batch_lds_bytes(int dtype) {
    return dtype == 0 ? batch_lds_bytes_t<uint32_t>() : batch_lds_bytes_t<f2_t>();
}

const void* batch_kernel_func(int dtype, bool quarter) {
    if (dtype == 0)
        return quarter ? (const void*)&fft_batch_kernel<uint32_t, ENC_QUARTER>
                       : (const void*)&fft_batch_kernel<uint32_t, ENC_TABLE>;
    return quarter ? (const void*)&fft_batch_kernel<f2_t, ENC_QUARTER>
                   : (const void*)&fft_batch_kernel<f2_t, ENC_TABLE>;
}

// The binary16 list kernels, 1024 threads each: 2^16 points with 64 elements
// per lane (radix 2^6, 2^5, 2^5; each exchange in two rounds of half the rows)
// and 2^15 points with 32 (radix 2^5 passes); the middle pass reads table
// entries [L0, L0 R) from the LDS prefix (2048 and 1024 entries).
template <int ENC> static constexpr auto kList16 = &fft_list_kernel<uint32_t, 16, 6, 6, 5, 5, 2048, ENC>;
template <int ENC> static constexpr auto kList15 = &fft_list_kernel<uint32_t, 15, 5, 5, 5, 5, 1024, ENC>;
static_assert(kListLog[0] == 16 && kListLog[1] == 15 && kListThreads == (1 << (16 - 6)) &&
                  kListThreads == (1 << (15 - 5)),
              "list kernel geometry");

size_t batch_list_lds_bytes(int list) {
    return list == 0 ? 2048 * sizeof(TwH) +
                           unit_lds_elems<uint32_t, 6, MODE_SMALL, 1, PassPlan<16, 6, 5, 5, 0>>() * sizeof(uint32_t)
                     : 1024 * sizeof(TwH) +
                           unit_lds_elems<uint32_t, 5, MODE_SMALL, 1, PassPlan<15, 5, 5, 5, 0>>() * sizeof(uint32_t);
}
static_assert(2048 * sizeof(TwH) + unit_lds_elems<uint32_t, 6, MODE_SMALL, 1, PassPlan<16, 6, 5, 5, 0>>() *
                                       sizeof(uint32_t) <= kLdsBytes &&
                  1024 * sizeof(TwH) + unit_lds_elems<uint32_t, 5, MODE_SMALL, 1, PassPlan<15, 5, 5, 5, 0>>() *
                                           sizeof(uint32_t) <= kLdsBytes,
              "list kernels fit a workgroup's LDS");

const void* batch_list_func(int list, bool quarter) {
    if (list == 0) return (const void*)(quarter ? kList16<ENC_QUARTER> : kList16<ENC_TABLE>);
    return (const void*)(quarter ? kList15<ENC_QUARTER> : kList15<ENC_TABLE>);
}

hipError_t launch_batch_list(int list, bool quarter, const void* in, void* out, const void* lt,
                             const int64_t* offs, int64_t count, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    if (count > 0x7fffffffLL || list < 0 || list >= kNumLists) return hipErrorInvalidValue;
    void* args[] = {&in, &out, &lt, &offs, &count};
    return hipLaunchKernel(batch_list_func(list, quarter), dim3((unsigned)count), dim3(kListThreads), args,
                           batch_list_lds_bytes(list), s);
}

// A serving step's work list (48 bytes an item: 75 KiB for a step of 12 requests with
// 49 split transforms), read once over the host link: bound by that link's latency,
// so every 16 bytes have a lane of their own and no load waits for another.  2 to
// 4 us in the stream's order; an asynchronous copy of more than 16 KiB goes to a copy
// engine, and the handover there and back left the compute units idle: that step
// took 104.5 us with it, 89.9 with the kernel.
__global__ __launch_bounds__(256) void stage_copy_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst,
                                                         unsigned chunks) {
    const unsigned i = blockIdx.x * 256 + threadIdx.x;
    if (i < chunks) dst[i] = src[i];
}

hipError_t launch_stage_copy(const void* src, void* dst, size_t bytes, hipStream_t s) {
    const size_t chunks = (bytes + 15) / 16, blocks = (chunks + 255) / 256;
    if (chunks == 0) return hipSuccess;
    if (blocks > 0xffffffu) return hipErrorInvalidValue;
    unsigned n = (unsigned)chunks;
    void* args[] = {&src, &dst, &n};
    return hipLaunchKernel((const void*)&stage_copy_kernel, dim3((unsigned)blocks), dim3(256), args, 0, s);
}

hipError_t launch_batch(int dtype, bool quarter, const void* in, void* out, void* ws, const void* lt,
                        const void* items, const int64_t* offs, int first, int nitems,
                        unsigned* q, int grid, hipStream_t s) {
    void* args[] = {&in, &out, &ws, &lt, &items, &offs, &first, &nitems, &q};
    return hipLaunchKernel(batch_kernel_func(dtype, quarter), dim3(grid), dim3(kBatchThreads), args,
                           batch_lds_bytes(dtype), s);
}

hipError_t launch_batch_phases(int dtype, bool quarter, const void* in, void* out, void* ws, const void* lt,
                               const void* items, const int64_t* offs, int phase0, int nitems,
                               unsigned* ctl, int grid0, int grid1, hipStream_t s) {
    hipError_t e = hipSuccess;
    if (phase0 > 0)
        e = launch_batch(dtype, quarter, in, out, ws, lt, items, offs, 0, phase0, ctl, grid0, s);
    if (e == hipSuccess && nitems > phase0)
        e = launch_batch(dtype, quarter, in, out, ws, lt, items, offs, phase0, nitems - phase0, ctl + 2,
                         grid1, s);
    return e;
}

}  // namespace dsfft

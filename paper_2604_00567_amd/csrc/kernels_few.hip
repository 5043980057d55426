// Kernels for calls of few transforms of the larger whole-transform sizes
// (binary16 2^14 .. 2^16, binary32 2^13 .. 2^15): the two-pass split with its
// intermediate in the output, in workgroups of 8, 16 or 32 units.
#include "fft_device.hpp"
#include "kernels.hpp"
#include "tables.hpp"

namespace dsfft {

template <class E, int LOG_NU, int LOG_E, int UPW, int MODE, int LR0, int LR1, int LR2, int ENC>
static hipError_t launch_few(const void* in, void* out, const void* lt, int64_t units, int log_m,
                             hipStream_t stream) {
    constexpr int NT = UPW << (LOG_NU - LOG_E);
    constexpr size_t LDS = unit_lds_bytes<E, LOG_NU, LOG_E, MODE, UPW, 0, 0, PassPlan<LOG_NU, LR0, LR1, LR2, 0>>();
    static_assert(LDS <= kLdsBytes / 2, "several workgroups per compute unit");
    // units: 2^log_m a transform, a multiple of UPW
    if (units <= 0 || (units & (UPW - 1)) || (1 << log_m) < UPW || units / UPW > 0x7fffffffLL)
        return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((fft_few_kernel<E, LOG_NU, LOG_E, UPW, MODE, LR0, LR1, LR2, ENC>),
                       dim3((unsigned)(units / UPW)), dim3(NT), LDS, stream, (const E*)in, (E*)out,
                       (const typename TwOf<E>::type*)lt, units, log_m);
    return hipGetLastError();
}

// The same over the transforms at element offsets offs[0 .. count) of in and out.
template <int ENC>
struct FewListGeo : GridGeoT<false, ENC, 0, true> {
    const int64_t* offs;
    __device__ __forceinline__ int64_t transform_in(int) const { return offs[this->ublk >> this->log_m]; }
    __device__ __forceinline__ int64_t transform_out(int) const { return offs[this->ublk >> this->log_m]; }
};
template <class E, int LOG_NU, int LOG_E, int UPW, int MODE, int LR0, int LR1, int LR2, int ENC>
__global__ void __launch_bounds__(UPW << (LOG_NU - LOG_E))
fft_few_list_kernel(const E* in, E* out, const typename TwOf<E>::type* __restrict__ lt, int64_t units, int log_m,
                    const int64_t* __restrict__ offs) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    E* lds = reinterpret_cast<E*>(lds_raw);
    E v[1 << LOG_E];
    const FewListGeo<ENC> gp{{(int64_t)blockIdx.x * UPW, units, log_m, (int)threadIdx.x}, offs};
    unit_pass<E, LOG_NU, LOG_E, UPW, 1, MODE, LR0, LR1, LR2, 0, 0, 0, 0>(v, lds, lt, in, out, gp);
}
template <class E, int LOG_NU, int LOG_E, int UPW, int MODE, int LR0, int LR1, int LR2, int ENC>
static hipError_t launch_few_list(const void* in, void* out, const void* lt, int64_t units, int log_m,
                                  const int64_t* offs, hipStream_t stream) {
    constexpr int NT = UPW << (LOG_NU - LOG_E);
    constexpr size_t LDS = unit_lds_bytes<E, LOG_NU, LOG_E, MODE, UPW, 0, 0, PassPlan<LOG_NU, LR0, LR1, LR2, 0>>();
    if (units <= 0 || (units & (UPW - 1)) || (1 << log_m) < UPW || units / UPW > 0x7fffffffLL)
        return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((fft_few_list_kernel<E, LOG_NU, LOG_E, UPW, MODE, LR0, LR1, LR2, ENC>),
                       dim3((unsigned)(units / UPW)), dim3(NT), LDS, stream, (const E*)in, (E*)out,
                       (const typename TwOf<E>::type*)lt, units, log_m, offs);
    return hipGetLastError();
}

// binary16 only: the batches' lists hold its 2^15- and 2^16-point transforms
template <class E, int LOG_NU, int LOG_E, int UPW, int MODE, int LR0, int LR1, int LR2, int ENC>
static constexpr FewListFn list_launch() {
    if constexpr (std::is_same_v<E, uint32_t> && LOG_NU >= 7)
        return &launch_few_list<E, LOG_NU, LOG_E, UPW, MODE, LR0, LR1, LR2, ENC>;
    else
        return nullptr;
}

#define FEW1(E, DT, MODE, LOG_NU, LOG_E, UPW, LR0, LR1, LR2)                                 \
    {DT, MODE, LOG_NU, UPW,                                                                  \
     &launch_few<E, LOG_NU, LOG_E, UPW, MODE, LR0, LR1, LR2, ENC_TABLE>,                     \
     &launch_few<E, LOG_NU, LOG_E, UPW, MODE, LR0, LR1, LR2, ENC_QUARTER>,                   \
     &launch_few<E, LOG_NU, LOG_E, UPW, MODE, LR0, LR1, LR2, ENC_QUARTER_INV>,               \
     list_launch<E, LOG_NU, LOG_E, UPW, MODE, LR0, LR1, LR2, ENC_TABLE>(),                   \
     list_launch<E, LOG_NU, LOG_E, UPW, MODE, LR0, LR1, LR2, ENC_QUARTER>()},
#define FEW(MODE, LOG_NU, LOG_E, UPW, LR0, LR1, LR2)                                         \
    FEW1(uint32_t, DT_F16, MODE, LOG_NU, LOG_E, UPW, LR0, LR1, LR2)                          \
    FEW1(f2_t, DT_F32, MODE, LOG_NU, LOG_E, UPW, LR0, LR1, LR2)

// narrowest first within a (mode, log_nu)
static const FewCfg kFew[] = {
    FEW(MODE_COLS, 7, 3, 8, 3, 2, 2)
    FEW(MODE_COLS, 7, 4, 16, 4, 3, 0)
    FEW(MODE_COLS, 7, 4, 32, 4, 3, 0)
    FEW(MODE_COLS, 8, 3, 8, 3, 3, 2)
    FEW(MODE_COLS, 8, 4, 16, 4, 4, 0)
    FEW(MODE_COLS, 8, 4, 32, 4, 4, 0)
    FEW(MODE_ROWS, 6, 3, 8, 3, 3, 0)
    FEW(MODE_ROWS, 6, 3, 16, 3, 3, 0)
    FEW(MODE_ROWS, 6, 3, 32, 3, 3, 0)
    FEW(MODE_ROWS, 7, 3, 8, 3, 2, 2)
    FEW(MODE_ROWS, 7, 4, 16, 4, 3, 0)
    FEW(MODE_ROWS, 7, 4, 32, 4, 3, 0)
    FEW(MODE_ROWS, 8, 3, 8, 3, 3, 2)
    FEW(MODE_ROWS, 8, 4, 16, 4, 4, 0)
    FEW(MODE_ROWS, 8, 4, 32, 4, 4, 0)
};
#undef FEW
#undef FEW1

const FewCfg* few_table(int* count) {
    *count = (int)(sizeof(kFew) / sizeof(kFew[0]));
    return kFew;
}

}  // namespace dsfft

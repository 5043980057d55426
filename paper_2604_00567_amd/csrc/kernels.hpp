// Registry of compiled kernel configurations (one entry per template
// instantiation of fft_unit_kernel).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace dsfft {

typedef hipError_t (*LaunchFn)(const void* in, void* out, const void* lt, int64_t units,
                               int log_m, hipStream_t stream);

struct KernelCfg {
    int dtype;      // DT_F16 / DT_F32 / DT_F16F32
    int mode;       // MODE_SMALL / MODE_COLS / MODE_ROWS
    int log_nu;     // unit size (log2)
    int log_e;      // elements per lane and unit (log2)
    int upw;        // units per workgroup
    int upl;        // units per lane (a lane's groups of one position in UPL units)
    int lr[3];      // register-pass radices (log2; 0 = absent)
    int staged;     // 1: block copied through LDS with 16-byte accesses
    int lane_tail;  // 1: the last two stages run across lanes (permlane swaps)
    int pipelined;  // 1: persistent workgroups prefetch the next block into registers;
                    // 2: each pass loads the next pass's twiddles
    int encoding;   // path encoding of the butterfly (ENC_*)
    int threads;    // workgroup size
    size_t lds_bytes;
    LaunchFn launch;
    // the same results from about half of the twiddle loads, for tables with
    // quarter symmetry: forward and inverse (null where not compiled)
    LaunchFn launch_quarter, launch_quarter_inverse;
    size_t lds_quarter;     // LDS bytes of those forms, whose twiddle copies are shorter
    const void* func;
};

// One half of the two-pass schedule through the output (kernels_few.hip);
// units: columns or rows of the launch, log_m: log2 of those in a transform.
typedef hipError_t (*FewListFn)(const void* in, void* out, const void* lt, int64_t units, int log_m,
                                const int64_t* offs, hipStream_t stream);
struct FewCfg {
    int dtype, mode, log_nu, upw;
    LaunchFn launch, launch_quarter, launch_quarter_inverse;
    // over the transforms at a list of offsets (null where batches have none)
    FewListFn list, list_quarter;
};
const FewCfg* few_table(int* count);
// The one for a launch over `units`: the narrowest whose workgroups number at
// most one per compute unit, else the widest; null if there is none.
const FewCfg* few_half(int dtype, int mode, int log_nu, int64_t units, int cus);
// Up to how many transforms the split beats the whole transform, in sixteenths
// of the compute units.
int split_limit(int dtype, int log_n);

// The compiled parts of a dtype's configurations: each part's table has every
// configuration, with mode -1 where another part compiles it (or none does).
constexpr int kParts = 3;
constexpr int kernel_part(int mode, int log_nu) { return mode != 0 ? 2 : (log_nu > 11 ? 1 : 0); }
template <int PART> const KernelCfg* kernel_table_f16(int* count);
template <int PART> const KernelCfg* kernel_table_f32(int* count);
template <int PART> const KernelCfg* kernel_table_f16f32(int* count);
template <> const KernelCfg* kernel_table_f16<0>(int* count);
template <> const KernelCfg* kernel_table_f16<1>(int* count);
template <> const KernelCfg* kernel_table_f16<2>(int* count);
template <> const KernelCfg* kernel_table_f32<0>(int* count);
template <> const KernelCfg* kernel_table_f32<1>(int* count);
template <> const KernelCfg* kernel_table_f32<2>(int* count);
template <> const KernelCfg* kernel_table_f16f32<0>(int* count);
template <> const KernelCfg* kernel_table_f16f32<1>(int* count);
template <> const KernelCfg* kernel_table_f16f32<2>(int* count);

}  // namespace dsfft

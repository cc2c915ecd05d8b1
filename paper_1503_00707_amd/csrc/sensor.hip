// sensor.hip -- launchers of the sensor, training and hybrid-step kernels
// (sensor_impl.h), both storage precisions.
#include <hip/hip_runtime.h>

#include <mutex>

#include "sensor_impl.h"

namespace dvm {

// Static scratch of dvm_mlp_gradient_noalloc: the blocks' gradient sums and
// loss partials (train_blocks is at most kTrainBlocks whatever the batch).
// Each GPU holds its own copy until the process ends; every call on a GPU
// shares it.
namespace {
constexpr size_t kScratchGrad = (size_t(kTrainBlocks) * kMlpWeights * sizeof(double) + 255) & ~size_t(255);
constexpr size_t kScratchLoss = (size_t(kTrainBlocks) * sizeof(double) + 255) & ~size_t(255);
constexpr int kMaxDevices = 64;
// Up to these sizes the sensor runs with 16 lanes per cell, above with a
// thread per cell: the first is bound by the latency of one tile, the second
// by the tiles' number.  Network, 16 lanes / a thread per cell: 16,384 cells
// 11.9 / 27.3 us, 32,768: 19.0 / 27.8, 65,536: 32.4 / 29.0, 1e6: 407 / 196.
// Gradient length: 16,384 cells 8.8 / 8.9, 32,768: 10.9 / 9.2, 1e6: 253 / 100.
constexpr int64_t kSensorSmallNet = 49152, kSensorSmallKn = 16384;
}  // namespace
static __device__ __align__(256) char scratch[kScratchGrad + kScratchLoss];

// Device address of this GPU's scratch (the host-side name of the array is
// not a device address): looked up once per device, with it current.
static hipError_t scratch_on_device(char **out) {
    static std::mutex mu;
    static char *ptr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        ptr[dev] = static_cast<char *>(p);
    }
    *out = ptr[dev];
    return hipSuccess;
}

static_assert(sizeof(SensorArgsPub) == sizeof(impl::FeatArgs), "argument layout");
static_assert(sizeof(HybArgsPub) == sizeof(impl::HybArgs), "argument layout");
static_assert(kMlpParams == impl::kParams && kMlpWeights == impl::kWeights, "parameter block");
static_assert(kFluxRecord == impl::kFluxRec, "flux records");
static_assert(kFaceRecord == 6 * 5, "face flux records");

static impl::FeatArgs feat(const SensorArgsPub &a) {
    impl::FeatArgs f;
    __builtin_memcpy(&f, &a, sizeof f);
    return f;
}

hipError_t launch_features(const SensorArgsPub &a, float *x, hipStream_t st) {
    hipLaunchKernelGGL(impl::k_features, dim3(unsigned((a.n + 255) / 256)), dim3(256), 0, st, feat(a), x);
    return hipGetLastError();
}

hipError_t launch_labels(bool fp64, const void *f, float *r, int64_t n, const VelGrid &g, hipStream_t st) {
    return fp64 ? impl::labels_dispatch<double>(f, r, n, g, st) : impl::labels_dispatch<float>(f, r, n, g, st);
}

hipError_t launch_mlp_forward(const float *params, const float *x, int64_t n, int mode, float *z, hipStream_t st) {
    if (mode == 0)
        hipLaunchKernelGGL(impl::k_mlp_fwd32, dim3(unsigned((n + 255) / 256)), dim3(256), 0, st, params, x, n, z);
    else
        hipLaunchKernelGGL(impl::k_mlp_fwd_mfma, dim3(unsigned(n < 16 * 2048 ? (n + 15) / 16 : 2048)), dim3(256), 0, st, params, x, n, z);
    return hipGetLastError();
}

hipError_t launch_sensor(const SensorArgsPub &a, const float *params, double kappa, uint8_t *mask, float *score,
                         hipStream_t st) {
    if (a.n <= (params ? kSensorSmallNet : kSensorSmallKn))
        hipLaunchKernelGGL(impl::k_sensor<16>, dim3(unsigned((a.n + 15) / 16)), dim3(256), 0, st, feat(a), params,
                           kappa, mask, score);
    else
        hipLaunchKernelGGL(impl::k_sensor<256>, dim3(unsigned((a.n + 255) / 256)), dim3(256), 0, st, feat(a), params,
                           kappa, mask, score);
    return hipGetLastError();
}

static hipError_t train(const float *params, const float *x, const float *y, int64_t n, float pos_weight,
                        double *part, double *loss_part, float *grad, double *loss, const impl::AdamArgs &adam,
                        hipStream_t st) {
    const int nb = train_blocks(n);
    hipLaunchKernelGGL(impl::k_train_tiles, dim3(unsigned(nb)), dim3(256), 0, st, params, x, y, n, pos_weight, part,
                       loss_part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(impl::k_train_reduce, dim3(unsigned((impl::kWeights + 63) / 64)), dim3(256), 0, st, part,
                       loss_part, nb, n, grad, loss, adam);
    return hipGetLastError();
}

hipError_t launch_train(const float *params, const float *x, const float *y, int64_t n, float pos_weight,
                        double *part, double *loss_part, float *grad, double *loss, hipStream_t st) {
    return train(params, x, y, n, pos_weight, part, loss_part, grad, loss, impl::AdamArgs{}, st);
}

hipError_t launch_train_adam(float *params, const float *x, const float *y, int64_t n, float pos_weight,
                             double *part, double *loss_part, float *grad, double *loss, float *m, float *v, float lr,
                             float c1, float c2, hipStream_t st) {
    return train(params, x, y, n, pos_weight, part, loss_part, grad, loss, impl::AdamArgs{params, m, v, lr, c1, c2},
                 st);
}

hipError_t launch_train_noalloc(const float *params, const float *x, const float *y, int64_t n, float pos_weight,
                                float *grad, double *loss, hipStream_t st) {
    if (n < 1 || n > kNoAllocMaxBatch) return hipErrorInvalidValue;
    char *base = nullptr;
    hipError_t e = scratch_on_device(&base);
    if (e != hipSuccess) return e;
    // every sum and partial the reduction reads is written first by the tiles'
    // kernel of the same call: nothing to clear
    return launch_train(params, x, y, n, pos_weight, reinterpret_cast<double *>(base),
                        reinterpret_cast<double *>(base + kScratchGrad), grad, loss, st);
}

hipError_t launch_adam(float *params, float *m, float *v, const float *grad, float lr, float c1, float c2,
                       hipStream_t st) {
    hipLaunchKernelGGL(impl::k_adam, dim3(unsigned((impl::kWeights + 255) / 256)), dim3(256), 0, st,
                       impl::AdamArgs{params, m, v, lr, c1, c2}, grad);
    return hipGetLastError();
}

hipError_t launch_norm_stats(const float *x, int64_t n, float *params, hipStream_t st) {
    hipLaunchKernelGGL(impl::k_norm_stats, dim3(impl::kIn), dim3(256), 0, st, x, n, params);
    return hipGetLastError();
}

hipError_t launch_mask_eff(const uint8_t *in, uint8_t *out, const DevCell *cells, int64_t n, hipStream_t st) {
    hipLaunchKernelGGL(impl::k_mask_eff, dim3(unsigned((n + 63) / 64)), dim3(64), 0, st, in, out, cells, n);
    return hipGetLastError();
}

hipError_t launch_fluid_moments(const uint8_t *mask, const double *mom, double *out, int64_t n, hipStream_t st) {
    hipLaunchKernelGGL(impl::k_fluid_moments, dim3(unsigned((n + 255) / 256)), dim3(256), 0, st, mask, mom, out, n);
    return hipGetLastError();
}

hipError_t launch_hybrid(bool fp64, const StepArgs &a, const HybArgsPub &h, hipStream_t st) {
    impl::HybArgs hh;
    __builtin_memcpy(&hh, &h, sizeof hh);
    return fp64 ? impl::hybrid_dispatch<double>(a, hh, st) : impl::hybrid_dispatch<float>(a, hh, st);
}

}  // namespace dvm

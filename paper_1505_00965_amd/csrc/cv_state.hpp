// The control-variate network's host state and what its two translation
// units share: parameters, estimation samplers and tables (cv.hip), training
// (cv_train.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "context.hpp"
#include "cv.hpp"

// Samples a training chunk holds at least (cv_train.hip).
constexpr uint64_t kTrainChunk = 32768;

struct mlmc_cv {
    mlmc_ctx* ctx = nullptr;
    int D = 2;                    // network inputs
    int np = 0;                   // parameter count
    float* d_params = nullptr;    // fp32 master
    float* d_m1 = nullptr;        // Adam moments
    float* d_m2 = nullptr;
    mlmc::cvnet::bf16x8* d_afwd = nullptr;   // bf16 W2 operands (forward), 8 x 64 entries
    mlmc::cvnet::bf16x8* d_abwd = nullptr;   // bf16 W2 operands (backward: W2^T)
    float* d_phi0 = nullptr;      // [0] phi(0, S0), [1] its tabulated value: see cv_ensure_phi0
    int adam_t = 0;
    uint64_t version = 0;         // bumped by every parameter change
    uint64_t phi0_version[2] = {~0ull, ~0ull};
    mlmc_model phi0_model[2]{};
    hipStream_t phi0_stream[2] = {nullptr, nullptr};
    // tabulated network (estimation launches only; training evaluates it)
    int tabulated = 0;
    float* d_table = nullptr;
    size_t table_cap = 0;         // floats allocated
    uint64_t table_version = ~0ull;
    mlmc_model table_model{};
    hipStream_t table_stream = nullptr;
    // training scratch: one allocation, cut up by each step (cv_train.hip)
    char* d_train = nullptr;
    size_t train_cap = 0;         // bytes allocated
    uint64_t train_least = kTrainChunk;   // halved while the device refuses the memory
    double* d_loss = nullptr;     // loss and per-level variances
};

namespace mlmc {

struct CvKernelArgs {
    const float* params;
    const cvnet::bf16x8* afwd;
    cvnet::NetConsts nc;
    int D;
};

// Network input and output scales of a model (cv.hip).
cvnet::NetConsts net_consts(const mlmc_model& m);

}  // namespace mlmc

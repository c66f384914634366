// me_unweight.hip -- two-stage unweighting driven by the surrogate network
// (Danziger, Janssen, Schumann, Siegert, SciPost Phys. 12 (2022) 164): the
// network's weight decides a first accept/reject, the exact float64 matrix
// element of the survivors a second one, and the output weights
// max(1, s/s_max) max(1, (w/s)/r_max) keep every point's expected
// contribution proportional to its exact weight w.
#include <hip/hip_runtime.h>

#include <cmath>

#include "../../include/mlp.h"
#include "me_internal.h"

#define HCHK(expr)                                                                                   \
    do {                                                                                             \
        hipError_t _e = (expr);                                                                      \
        if (_e != hipSuccess) return me_fail(ME_EDEVICE, std::string(#expr ": ") + hipGetErrorString(_e)); \
    } while (0)

// Append of the block's `take` threads to list[*count]: returns the slot.  One
// atomic per block of UW_BLOCK threads: with one per wave its 16,384 additions
// to one address took 62 us for 2^20 points, about five times the data's time.
#define UW_BLOCK 1024
__device__ __forceinline__ int append_slot(bool take, int* count) {
    __shared__ int at[UW_BLOCK / 64];
    const unsigned long long ballot = __ballot(take);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) at[wave] = __popcll(ballot);
    __syncthreads();
    if (threadIdx.x == 0) {
        int sum = 0;
        for (int w = 0; w < UW_BLOCK / 64; ++w) {
            const int c = at[w];
            at[w] = sum;
            sum += c;
        }
        const int base = sum ? atomicAdd(count, sum) : 0;
        for (int w = 0; w < UW_BLOCK / 64; ++w) at[w] += base;
    }
    __syncthreads();
    return take ? at[wave] + __popcll(ballot & ((1ull << lane) - 1ull)) : -1;
}

__global__ void k_uw_zero(int* count) {
    if (threadIdx.x < 2 && blockIdx.x == 0) count[threadIdx.x] = 0;
}

// stage 1: s = exp(sigma y + mu) w_ps; survivors appended to idx1 (count[0])
__global__ void k_uw_stage1(const float* __restrict__ y, const double* __restrict__ w_ps,
                            const double* __restrict__ u, int64_t n, double mu, double sigma, double s_max,
                            double* __restrict__ s_out, int* __restrict__ idx1, int* __restrict__ count) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    bool take = false;
    if (i < n) {
        const double s = exp(sigma * (double)y[i] + mu) * w_ps[i];
        s_out[i] = s;
        take = u[2 * i] < fmin(1.0, s / s_max);
    }
    const int slot = append_slot(take, &count[0]);
    if (take) idx1[slot] = (int)i;
}

// stage 2 over the survivors: exact weight from the float64 matrix element
__global__ void k_uw_stage2(const int* __restrict__ idx1, const double* __restrict__ me2,
                            const double* __restrict__ w_ps, const double* __restrict__ s_in,
                            const double* __restrict__ u, double s_max, double r_max, int* __restrict__ count,
                            int32_t* __restrict__ out_idx, double* __restrict__ out_w) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x, kept = count[0];
    if ((int)(blockIdx.x * blockDim.x) >= kept) return;
    bool take = false;
    int i = 0;
    double wt = 0.0;
    if (j < kept) {
        i = idx1[j];
        const double s = s_in[i];
        const double r = me2[i] * w_ps[i] / s;
        take = u[2 * (int64_t)i + 1] < fmin(1.0, r / r_max);
        wt = fmax(1.0, s / s_max) * fmax(1.0, r / r_max);
    }
    const int slot = append_slot(take, &count[1]);
    if (take) {
        out_idx[slot] = i;
        out_w[slot] = wt;
    }
}

static int ensure_uw(me_ctx* c, int64_t n) {
    if (n <= c->uw_cap) return ME_OK;
    HCHK(hipDeviceSynchronize());
    const size_t k = (size_t)n;
    const hipError_t e = me_regrow(n, c->uw_cap,
                                   {{(void**)&c->uw_y, k * sizeof(float)}, {(void**)&c->uw_s, k * sizeof(double)},
                                    {(void**)&c->uw_me2, k * sizeof(double)}, {(void**)&c->uw_idx1, k * sizeof(int)}},
                                   [](void** p, size_t bytes) { return hipMalloc(p, bytes); }, hipFree);
    if (e != hipSuccess) {
        (void)hipGetLastError();  // not the error of a later call
        return me_fail(ME_EDEVICE, std::string("unweight_two_stage: scratch: ") + hipGetErrorString(e));
    }
    return ME_OK;
}

extern "C" int unweight_two_stage(me_ctx* c, me_mlp* mlp, const double* momenta, const double* w_ps, int64_t n,
                                  const double* uniforms, double y_mu, double y_sigma, double s_max, double r_max,
                                  int32_t* out_idx, double* out_w, int32_t* out_count, void* stream) {
    if (!c || !mlp || n < 0) return me_fail(ME_EINVAL, "unweight_two_stage: null argument or negative n");
    if (!(s_max > 0) || !(r_max > 0)) return me_fail(ME_EINVAL, "unweight_two_stage: s_max, r_max must be positive");
    if (!out_count) return me_fail(ME_EINVAL, "unweight_two_stage: null out_count");
    if (n > 0x7fffffffLL) return me_fail(ME_EINVAL, "unweight_two_stage: n above 2^31 - 1");
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(k_uw_zero, dim3(1), dim3(64), 0, s, out_count);
    if (n == 0) {
        HCHK(hipGetLastError());
        return ME_OK;
    }
    if (!momenta || !w_ps || !uniforms || !out_idx || !out_w) return me_fail(ME_EINVAL, "unweight_two_stage: null buffer");
    const int npart = c->proc->npart;
    if (mlp_n_in(mlp) != 4 * npart) return me_fail(ME_EINVAL, "unweight_two_stage: network inputs != 4 npart");
    int rc = ensure_uw(c, n);
    if (rc != ME_OK) return rc;
    rc = mlp_forward_momenta(mlp, momenta, n, c->uw_y, s);
    if (rc != ME_OK) return rc;
    const dim3 grid((unsigned)((n + UW_BLOCK - 1) / UW_BLOCK));
    hipLaunchKernelGGL(k_uw_stage1, grid, dim3(UW_BLOCK), 0, s, c->uw_y, w_ps, uniforms, n, y_mu, y_sigma, s_max, c->uw_s,
                       c->uw_idx1, out_count);
    // exact float64 matrix element of the stage-1 survivors only
    HCHK(me_launch_idx(c, momenta, n, c->uw_me2, c->uw_idx1, out_count, s));
    hipLaunchKernelGGL(k_uw_stage2, grid, dim3(UW_BLOCK), 0, s, c->uw_idx1, c->uw_me2, w_ps, c->uw_s, uniforms, s_max,
                       r_max, out_count, out_idx, out_w);
    HCHK(hipGetLastError());
    return ME_OK;
}

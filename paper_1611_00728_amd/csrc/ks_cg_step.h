// The end of a CG step on the device, shared by the direction kernel and by the hopping term that
// forms the direction as it gathers it.
#pragma once

#include "ks_blas.h"
#include "ks_device.h"

namespace ks {

// Every block reduces the previous kernel's partial sums itself: thread t adds partials t,
// t + NT, ... then the fixed block order, so all blocks hold the same value bit for bit.
// fused_load gives a thread's share, fused_total the block's total in every thread (it passes
// one block barrier).
template <int NT>
__device__ __forceinline__ double fused_load(const double* __restrict__ in, int n)
{
    double t = 0.0;
    for (int k = threadIdx.x; k < n; k += NT) t += in[k];
    return t;
}

template <int NT>
__device__ __forceinline__ double fused_total(double t)
{
    __shared__ double part[NT / 64];
    t = wave_sum(t);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = t;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < NT / 64; ++k) s += part[k];
    return s;
}

// Keeps a vector's loads ahead of what follows: they are in flight together with the partial
// sums' and the state's, so a step's kernel waits for memory once and not once for each of them
// (8^4 FP64 with the register sums of wave_sum: update 5.3 -> 3.1 us, direction 4.0 -> 2.9 us a
// launch).
template <class R>
__device__ __forceinline__ void pin(cx<R> v[3])
{
#pragma unroll
    for (int k = 0; k < 3; ++k) asm volatile("" : "+v"(v[k].r), "+v"(v[k].i));
}

// What a block decides the step's end from: the copies the update kernel took (s_*) and fields no
// block writes meanwhile (stop2, delta, max_iter), so every block takes the same branch.
struct StepEnd {
    double s_rho, maxr, stop2, delta;
    int stop, iter, max_iter;
    __device__ __forceinline__ explicit StepEnd(const CGState* st)
        : s_rho(st->s_rho), maxr(st->s_maxr), stop2(st->stop2), delta(st->delta), stop(st->s_gate),
          iter(st->s_iter + 1), max_iter(st->max_iter)
    {
    }
    // With the total |r|^2: whether the step goes on to a new direction, and its beta.  The lead
    // thread of the grid alone writes the live state.
    __device__ __forceinline__ bool decide(CGState* st, double rho_new, bool lead, double* coef,
                                           int coef_cap, double& beta) const
    {
        if (lead) {
            st->iter = iter;
            st->rho_new = rho_new;
        }
        if (!isfinite(rho_new)) {
            if (lead) {
                st->status = KS_ERR_NONFINITE;
                st->gate = 1;
            }
            return false;
        }
        const double rn = sqrt(rho_new);
        if (rho_new <= stop2 || rn < delta * maxr) {
            // FP64 recomputation of r = b - A x decides (reliable update or final check); the
            // step's beta is then not a CG coefficient
            if (lead) {
                st->ru_pending = 1;
                st->gate = 1;
                if (iter - 1 < coef_cap) coef[2 * (iter - 1) + 1] = __builtin_nan("");
            }
            return false;
        }
        beta = rho_new / s_rho;
        const bool last = iter >= max_iter;
        if (lead) {
            if (iter - 1 < coef_cap) coef[2 * (iter - 1) + 1] = beta;
            st->beta = beta;
            st->rho = rho_new;
            st->maxr = fmax(maxr, rn);
            if (last) st->gate = 1;
        }
        return !last;
    }
};

}  // namespace ks

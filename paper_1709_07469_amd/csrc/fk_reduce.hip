// fk_reduce.hip -- the per-walk samples u_p = g(x_e) - 2 pi G (dt/2) S from the
// walks' exit records (Dirichlet data read at the exit point, FP64), and the
// per-station statistics of the samples (the sample mean of arXiv:1709.07469
// eq. 11, with the unbiased variance and standard error), with the paired
// central difference of eq. 6 for g_z.
//
// Deterministic two-level reduction (fk_stats.hpp): one block per (station,
// chunk) pair turns the pair's samples into a (count, mean, M2) partial in a
// fixed order; a second kernel merges a station's partials in chunk order.
// A bounded workspace runs the first kernel once per slice of pairs, as soon
// as the slice's walks are done, and the second once at the end.  Stations of
// one chunk need no second kernel: the block of their pair writes their result.
#include <hip/hip_runtime.h>

#include "fk_stats.hpp"

namespace fk {

namespace {

// Bound by the evaluation of the Dirichlet data (24 corner terms a prism, FP64
// vector arithmetic).  One block per pair leaves most of the chip idle where
// pairs are few (sample_parts in fk_api.cpp): two passes then, the first with
// several blocks per pair.
template <int PASS>
__global__ void __launch_bounds__(kReduceBlock) chunk_kernel(const ReduceArgs R)
{
    const int64_t q = R.q0 + blockIdx.x;
    const int64_t s = q / R.n_chunks;
    const int64_t c = q - s * R.n_chunks;
    const int64_t i0 = c * R.chunk;
    const int64_t i1 = (i0 + R.chunk < R.N) ? i0 + R.chunk : R.N;

    DataTables tb{nullptr, nullptr};
    if (PASS != kFromSamples && R.bc.kind == FK_BC_PRISMS) tb = fill_data_tables();   // uniform: every thread takes it

    const PairSpan P{R.exits, R.steps, R.values, s * R.N * R.npair - R.task0, i0, i1, R.npair, R.two_h};
    auto data = [&](const ExitRecord& r) {
        if (PASS == kFromSamples) return r.S;
        const double e[3] = {r.x, r.y, r.z};
        return boundary_value(R.bc, R.lo, R.hi, R.G, e, tb) - R.w * r.S;
    };
    if constexpr (PASS == kSamples) sample_pair(P, data, blockIdx.y, gridDim.y);
    else reduce_pair(P, data, R.partials + q, R.status, R.n_chunks == 1 ? R.out + s : nullptr, R.N);
}

__global__ void __launch_bounds__(64) station_kernel(const ReduceArgs R)
{
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= R.n_stations) return;
    R.out[s] = finish_station(R.partials + s * R.n_chunks, R.n_chunks, R.N);
}

}  // namespace

hipError_t launch_reduce(const ReduceArgs& a, int64_t n_pairs, int parts, bool finish, hipStream_t stream)
{
    if (n_pairs > 0) {
        if (parts > 1) {
            hipLaunchKernelGGL(chunk_kernel<kSamples>, dim3((unsigned)n_pairs, (unsigned)parts), dim3(kReduceBlock), 0,
                               stream, a);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL(chunk_kernel<kFromSamples>, dim3((unsigned)n_pairs), dim3(kReduceBlock), 0, stream, a);
        } else {
            hipLaunchKernelGGL(chunk_kernel<kOnePass>, dim3((unsigned)n_pairs), dim3(kReduceBlock), 0, stream, a);
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (!finish || a.n_chunks == 1) return hipSuccess;
    hipLaunchKernelGGL(station_kernel, dim3((unsigned)((a.n_stations + 63) / 64)), dim3(64), 0, stream, a);
    return hipGetLastError();
}

}  // namespace fk

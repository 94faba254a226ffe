// Server side of a round (paper Algorithm 1, server lines "Aggregate all update estimators" and
// "Updates the model"): decode M sparse payloads into the M estimator copies, then one dense pass
//     x <- x - gamma * sum_m w_m u_hat_m.
// The decode touches a few percent of the estimators; the model step reads M + 1 dense vectors and
// writes one: it is the other HBM-bound kernel of the method, 4 (M + 2) bytes per element.
#pragma once
#include <hip/hip_fp16.h>
#include "common.h"

namespace kimad {

constexpr uint32_t MAX_WORKERS = 16;         // must equal KIMAD_MAX_WORKERS of the public header

// The estimators and weights of the model step.  The arrays are indexed with compile-time
// constants only (unrolled loops): a run-time index into a by-value kernel argument makes the
// compiler copy the whole table to scratch memory in every thread.
struct ServerArgs {
    const float* u_hat[MAX_WORKERS];
    double w[MAX_WORKERS];
    uint32_t M;
    uint64_t d;
};
// The payloads of the decode, likewise.
struct DecodeArgs {
    const uint32_t* idx[MAX_WORKERS];
    const float* val[MAX_WORKERS];
    const uint64_t* off[MAX_WORKERS];
    uint64_t capacity_pairs[MAX_WORKERS];
    float* u_hat[MAX_WORKERS];
    uint32_t f16;                            // bit m: worker m's values are binary16
};

// The workers' payloads into their estimators, worker first + blockIdx.y by a row of workgroups: one thread per pair.
// The pair's layer is found by bisection in the worker's offsets; indices inside a payload are distinct, so
// the additions need no atomics.  The payload is what a worker sent, not something this library produced: every
// workgroup first checks the offsets (non-decreasing, starting at 0, the total within the buffers'
// capacity, the layer starts non-decreasing up to d) and leaves without a write if they are not; a
// pair whose index lies outside its layer is skipped.  Either way the status word gets err_payload.
// Bound by the 128-byte lines that the 4-byte updates touch.  One launch for all workers (they write disjoint
// estimators; the caller sends them one by one where they do not), the offsets bisected in LDS.  Calls without a model,
// against a launch per worker: sixteen payloads of 58 K pairs 103 -> 57 us, four of 622 K 129 -> 103, one of 622 K 32 and
// one of 58 K 16 either way.  (Four pairs per thread with their loads together: 59, 110, 33 and 18 us.)
constexpr uint32_t DECODE_LDS_L = 1023;      // layers whose offsets and starts are kept in LDS
__global__ __launch_bounds__(256) void k_server_decode(DecodeArgs a, uint32_t first, const uint64_t* __restrict__ layer_start,
                                                       uint32_t L, uint64_t d, int32_t* status_out, int32_t err_payload) {
    __shared__ uint64_t s_off[DECODE_LDS_L + 1], s_start[DECODE_LDS_L + 1];
    __shared__ int bad;
    const uint32_t m = first + blockIdx.y;
    const uint32_t* idx = nullptr;
    const float* val = nullptr;
    const uint64_t* off = nullptr;
    uint64_t capacity_pairs = 0;
    float* u_hat = nullptr;
#pragma unroll
    for (uint32_t k = 0; k < MAX_WORKERS; ++k)
        if (k == m) { idx = a.idx[k]; val = a.val[k]; off = a.off[k]; capacity_pairs = a.capacity_pairs[k]; u_hat = a.u_hat[k]; }
    const bool f16 = (a.f16 >> m) & 1u;
    const bool in_lds = L <= DECODE_LDS_L;
    if (threadIdx.x == 0) bad = 0;
    __syncthreads();
    int mine = 0;
    for (uint32_t i = threadIdx.x; i <= L; i += 256u) {
        const uint64_t o = off[i], ls = layer_start[i];
        if (in_lds) { s_off[i] = o; s_start[i] = ls; }
        if (i == 0 && o != 0) mine = 1;
        if (i < L && (off[i + 1] < o || layer_start[i + 1] < ls)) mine = 1;
        if (i == L && (o > capacity_pairs || ls != d)) mine = 1;
    }
    if (mine) bad = 1;
    __syncthreads();
    if (bad) {
        if (blockIdx.x == 0 && threadIdx.x == 0) atomicMin(status_out + m, err_payload);
        return;
    }
    const uint64_t total = off[L];
    const uint64_t stride = (uint64_t)gridDim.x * 256u;
    for (uint64_t p = (uint64_t)blockIdx.x * 256u + threadIdx.x; p < total; p += stride) {
        const uint32_t t = idx[p];
        // half-precision payloads carry binary16 bit patterns: the worker added the decoded value, so does the server
        const float v = f16 ? __half2float(__ushort_as_half(reinterpret_cast<const uint16_t*>(val)[p])) : val[p];
        uint32_t lo = 0, hi = L;                 // largest layer i with off[i] <= p
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if ((in_lds ? s_off[mid] : off[mid]) <= p) lo = mid; else hi = mid;
        }
        const uint64_t start = in_lds ? s_start[lo] : layer_start[lo];
        const uint64_t n = (in_lds ? s_start[lo + 1u] : layer_start[lo + 1u]) - start;
        if ((uint64_t)t >= n) { atomicMin(status_out + m, err_payload); continue; }
        float* u = u_hat + start + t;
        gstore(u, gload(u) + v);
    }
}

// The model step, four elements per thread and trip; the tail and unaligned buffers take the
// scalar loop.  fp64 arithmetic per element, workers in order: every result is reproducible and
// equal to a plain sequential evaluation.  HBM-bound.
// (Four estimators of 124 M elements: 468 us, 6.4 TB/s.  All of a thread's loads asked for together, the worker count fixed at
// compile time, 557; two or four quads a thread and runs of blocks per XCD were slower as well.)
//
// Nontemporal stores keep the model's lines from displacing the estimators' in passing, but then the next round
// cannot find the model in the 256 MB cache either.  Ten rounds back to back with small payloads, us a round with ordinary
// and with nontemporal stores:
//     model (MiB)  1 worker    2 workers   3 workers   4 workers
//       48          36  33      45  43      55  53      63  62
//       80          51  50      67  68      84  83      99  97
//       96          59  58      78  79      95  98     111 113
//      128          74  75      98 105     120 126     145 150
//      192         105 112     140 149     175 190     212 217
//      256         134 144     190 196     239 239     298 284
//      288         151 161     216 220     296 269     370 319
//      320         170 179     273 244     353 298     425 363
//      448         247 255     398 350     509 414     611 503
//      576         307 320     528 445     643 537     774 635
//      720         420 401     647 550     788 664     951 783
//     1000         586 555     851 755    1069 914    1307 1087
// (Six to sixteen workers: equal up to 192 MiB, nontemporal 7 to 20 % faster from 256 on.  After a gigabyte of other memory
// was written in between, nontemporal stores are as fast or faster at every size.)  So ordinary stores for models of
// 96 MiB and more as long as model and estimators together are at most three and a half times the cache, with one worker
// five times.
inline bool model_stores_stream(uint32_t M, uint64_t d) {
    const uint64_t mib = 4 * d >> 20;
    return mib < 96 || (M + 1) * mib > (M == 1 ? 1280 : 896);
}
// (A template: a branch between the two stores is merged into one ordinary store by the compiler.)
template <bool STREAM_STORES>
__global__ __launch_bounds__(256) void k_server_step(ServerArgs a, float* x, double gamma, uint32_t vec_ok) {
    const uint64_t gid = (uint64_t)blockIdx.x * 256u + threadIdx.x, stride = (uint64_t)gridDim.x * 256u;
    const uint64_t n4 = vec_ok ? a.d / 4 : 0;
    for (uint64_t q = gid; q < n4; q += stride) {
        const float4 xv = gload4_stream(x + 4 * q);
        double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
#pragma unroll
        for (uint32_t m = 0; m < MAX_WORKERS; ++m) {
            if (m < a.M) {
                const float4 u = gload4_stream(a.u_hat[m] + 4 * q);   // read once per step
                const double w = a.w[m];
                s0 = s0 + w * (double)u.x; s1 = s1 + w * (double)u.y;
                s2 = s2 + w * (double)u.z; s3 = s3 + w * (double)u.w;
            }
        }
        float4 r;
        r.x = (float)((double)xv.x - gamma * s0); r.y = (float)((double)xv.y - gamma * s1);
        r.z = (float)((double)xv.z - gamma * s2); r.w = (float)((double)xv.w - gamma * s3);
        if (STREAM_STORES) gstore4_stream(x + 4 * q, r);
        else gstore4(x + 4 * q, r);
    }
    for (uint64_t t = 4 * n4 + gid; t < a.d; t += stride) {
        double acc = 0.0;
#pragma unroll
        for (uint32_t m = 0; m < MAX_WORKERS; ++m)
            if (m < a.M) acc = acc + a.w[m] * (double)gload(a.u_hat[m] + t);
        gstore(x + t, (float)((double)gload(x + t) - gamma * acc));
    }
}

}  // namespace kimad

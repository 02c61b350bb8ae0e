// A chunk of kChunk entries of a sparse layout, as the kernels that multiply with it take it apart.
#pragma once

#include "device_util.h"

namespace tron {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef double v2d __attribute__((ext_vector_type(2)));
typedef unsigned int v2u __attribute__((ext_vector_type(2)));

constexpr int kQuarter = kChunk / 4;

// x[c] through a 32-bit byte offset (tron_dataset_create_csr accepts n, d < 2^29 only)
__device__ __forceinline__ double load_elem(const double *__restrict__ x, int c)
{
    return *reinterpret_cast<const double *>(reinterpret_cast<const char *>(x) + (size_t)((uint32_t)c << 3));
}

// ------------------------------------------------------------------ segment sums of a chunk
// The entries of a chunk are in segment order (a segment = the entries of one row inside the chunk) and a flag bit
// marks the last entry of every segment.  Thread t owns entries 8t .. 8t+7: it sums its own runs in registers, the open run
// at its end is carried to the following threads by a segmented scan over the wavefront (DPP) and across the four
// wavefronts through LDS.  No loop depends on how long the segments are.  (With the entries stored in order the products were
// passed through LDS, from load order to thread order: a barrier more and, 500,000 x 750,000 with values, 52.6 instead of 47.6 us
// in the tiles, 45.7 / 43.8 in the head partition, 45.1 / 42.9 and 41.7 / 40.3 in the ranges.)
constexpr int kOutOffset = 16;                  // segment sums are parked at prod[kOutOffset ...] (behind the wavefront totals)
constexpr int kSegPasses = kChunk / kBlock;     // a chunk holds at most kChunk segments: 8 passes of 256
constexpr int kProdDoubles = kOutOffset + kChunk;

// tid = the thread among the kBlock that share the chunk, f = its 8 flag bits.  p[e] in: the product of entry 8 * tid + e.  On return p[e] = sum of the thread's entries from the start of the run
// containing e up to e, cin = what the entries before the thread add to its first run, idx0 = number of flags in the
// threads before it.  Uses prod[0..7] for the wavefront totals; contains one barrier.
__device__ __forceinline__ void runs_from_regs(double *prod, const int tid, const unsigned f, double (&p)[8], double &cin, int &idx0)
{
    const int lane = tid & (kWave - 1), wv = tid / kWave;
    double run = 0.0;
    const unsigned nf = ~f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        run += p[e];
        p[e] = run;
        const int keep = (int)(nf << (31 - e)) >> 31;   // all ones unless entry e ends a segment
        run = __hiloint2double(__double2hiint(run) & keep, __double2loint(run) & keep);
    }
    const int cnt = __popc(f);
    double t = run;
    int h = (f != 0u);
    wave_seg_scan(t, h);
    const int ci = wave_scan_add(cnt);
    const double ext = lane_before(t);
    const int exh = lane_before(h);
    if (lane == kWave - 1) {
        prod[2 * wv] = t;
        *reinterpret_cast<int2 *>(prod + 2 * wv + 1) = make_int2(h, ci);
    }
    __syncthreads();
    double ct = 0.0;
    int cb = 0;
#pragma unroll
    for (int w = 0; w < kWavesPerBlock - 1; ++w) {
        if (w < wv) {
            const double wt = prod[2 * w];
            const int2 hc = *reinterpret_cast<const int2 *>(prod + 2 * w + 1);
            ct = hc.x ? wt : ct + wt;
            cb += hc.y;
        }
    }
    cin = exh ? ext : ct + ext;
    idx0 = cb + ci - cnt;
}

}  // namespace tron

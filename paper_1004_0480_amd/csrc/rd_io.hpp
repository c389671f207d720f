// rd_io.hpp -- the kernels around the stepping: FP64 reductions, conversion
// between dense and padded fields, and the copy probe.  Included by the engine
// alone (non-template kernels have one definition).
#pragma once

#include "rd_device.hpp"
#include "rd_io_cfg.hpp"

namespace rdk {

// Fields are walked as rows (padded rows start every `pitch` cells, dense ones
// every nx) of units of four cells, the last of a row holding what is left.
// A workgroup owns a run of whole rows (or a part of a long one) and its threads
// take the run's units in turn, several at a time (DEPTH) so that several loads
// of a thread are in flight, or one where a thread has no more than one anyway:
// one 32-bit division per unit finds its row, where a division in 64 bits per
// cell would cost more than the cell's bytes.  Bound by memory: 403x301x300 FP32
// (146 MB a field, fastest traced, cell by cell before against this) write
// 89 -> 57 us, read 84 -> 53, reduction 105 -> 30, where the bytes at the rate of
// a streaming copy take 44, 44 and 22.
struct IoUnit { long long row; int x, n; };       // n cells (0: none) from cell x of a row

__device__ __forceinline__ IoUnit io_unit(unsigned u, unsigned units, int nx4, int nx, long long row0) {
    const unsigned r = u / unsigned(nx4);
    const int x = int(u - r * unsigned(nx4)) * 4;
    return IoUnit{row0 + r, x, u < units ? min(4, nx - x) : 0};
}

// The four cells from `at` on of `end` readable ones, moved back where they
// would pass the end (io_cells puts that right), so that the loads of a turn
// are one straight run (a branch around each, for the units at the ends of rows:
// reduction 41 us, read 57).  The address need only be aligned to a cell
// (dense rows start anywhere).
template <class T>
__device__ __forceinline__ Vec<T, 4> io_load(const void* base, long long at, long long end) {
    Vec<T, 4> v{};
    if (end >= 4) __builtin_memcpy(&v, gload_ptr<T>(base) + min(at, end - 4), 4 * sizeof(T));
    return v;
}
// A unit's cells, those past n 0; at the end of the field they are loaded one
// by one.
template <class T>
__device__ __forceinline__ void io_cells(const void* base, long long at, long long end, int n, Vec<T, 4>& v) {
    if (at + 4 > end && n > 0) {
        const RD_GLOBAL T* p = gload_ptr<T>(base) + at;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i < n) v.v[i] = p[i];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) v.v[i] = i < n ? v.v[i] : T(0);
}
// (non-temporal: what is written here passes through once; read 57 -> 53 us,
// and a reduction after a write 42 -> 36)
template <class T>
__device__ __forceinline__ void io_store(void* base, long long at, int n, const Vec<T, 4>& v) {
    RD_GLOBAL T* p = gstore_ptr<T>(base) + at;
    if (n == 4) {
        typedef T vt __attribute__((ext_vector_type(4), aligned(sizeof(T))));
        vt w;
        __builtin_memcpy(&w, &v, sizeof(w));
        __builtin_nontemporal_store(w, (RD_GLOBAL vt*)p);
    } else {
#pragma unroll
        for (int i = 0; i < 3; ++i)
            if (i < n) p[i] = v.v[i];
    }
}

// ------------------------------------------------------------- reductions

// Sums over a workgroup of 256 threads, in a fixed order; the result is in
// thread 0.
__device__ __forceinline__ void block_sum2(double& s, double& q) {
    __shared__ double ss[4], sq[4];
#pragma unroll
    for (int k = 32; k > 0; k >>= 1) {
        s += __shfl_down(s, k, 64);
        q += __shfl_down(q, k, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        ss[threadIdx.x >> 6] = s;
        sq[threadIdx.x >> 6] = q;
    }
    __syncthreads();
    s = (ss[0] + ss[1]) + (ss[2] + ss[3]);
    q = (sq[0] + sq[1]) + (sq[2] + sq[3]);
}

// Workgroup b sums rows [b, b+1) * rows / gridDim.x: the same cells in the same
// order whatever the pitch.
template <class S>
__global__ __launch_bounds__(256) void reduce_partial(const void* f, int nx, long long rows, int pitch,
                                                      double* part) {
    const long long row0 = rows * blockIdx.x / gridDim.x, row1 = rows * (blockIdx.x + 1) / gridDim.x;
    const int nx4 = (nx + 3) / 4;
    const unsigned units = unsigned(row1 - row0) * unsigned(nx4);
    const long long end = (rows - 1) * pitch + (pitch & 3 ? nx : pitch);   // (padded rows are whole units)
    double s[4] = {}, q[4] = {};
    for (unsigned u = threadIdx.x; u < units; u += 256 * IO_DEPTH) {
        Vec<typename S::T, 4> v[IO_DEPTH];
        IoUnit t[IO_DEPTH];
#pragma unroll
        for (int k = 0; k < IO_DEPTH; ++k) {
            t[k] = io_unit(u + 256 * k, units, nx4, nx, row0);
            v[k] = io_load<typename S::T>(f, t[k].row * pitch + t[k].x, end);
        }
#pragma unroll
        for (int k = 0; k < IO_DEPTH; ++k) {
            io_cells(f, t[k].row * pitch + t[k].x, end, t[k].n, v[k]);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const double c = S::up(v[k].v[i]);
                s[i] += c;
                q[i] = __fma_rn(c, c, q[i]);
            }
        }
    }
    double ts = (s[0] + s[1]) + (s[2] + s[3]), tq = (q[0] + q[1]) + (q[2] + q[3]);
    block_sum2(ts, tq);
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = ts;
        part[2 * blockIdx.x + 1] = tq;
    }
}

// at most 1024 partial pairs
__global__ __launch_bounds__(256) void reduce_final(const double* part, int n, double h3, double* out) {
    double s = 0.0, q = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int i = threadIdx.x + 256 * k;
        if (i < n) {
            s += part[2 * i];
            q += part[2 * i + 1];
        }
    }
    block_sum2(s, q);
    if (threadIdx.x == 0) {
        out[0] = s * h3;
        out[1] = q * h3;
    }
}

// ------------------------------------------------------ layout conversion

// A workgroup converts `run` rows of `in` cells apart, or one of the `parts` of
// a row, to rows `out` cells apart, cell by cell through `up` and `down` (FP32
// between).
template <int DEPTH, class In, class Out, class Up, class Down>
__device__ __forceinline__ void convert_rows(const void* src, void* dst, int nx, long long rows, int run, int parts,
                                             int in, int out, Up up, Down down) {
    const int nx4 = (nx + 3) / 4;
    long long row0 = (long long)blockIdx.x * run;
    unsigned first = 0, units = unsigned(nx4);
    if (parts == 1) {
        units *= unsigned(min((long long)run, rows - row0));
    } else {                                     // (run is 1)
        const unsigned each = (units + unsigned(parts) - 1) / unsigned(parts);
        row0 = blockIdx.x / unsigned(parts);
        first = (blockIdx.x - unsigned(row0) * unsigned(parts)) * each;
        units = min(first + each, units);
    }
    const long long end = (rows - 1) * in + (in & 3 ? nx : in);
    for (unsigned u = first + threadIdx.x; u < units; u += 256 * DEPTH) {
        Vec<In, 4> v[DEPTH];
        IoUnit t[DEPTH];
#pragma unroll
        for (int k = 0; k < DEPTH; ++k) {
            t[k] = io_unit(u + 256 * k, units, nx4, nx, row0);
            v[k] = io_load<In>(src, t[k].row * in + t[k].x, end);
        }
#pragma unroll
        for (int k = 0; k < DEPTH; ++k) {
            Vec<Out, 4> w;
            io_cells(src, t[k].row * in + t[k].x, end, t[k].n, v[k]);
#pragma unroll
            for (int i = 0; i < 4; ++i) w.v[i] = down(up(v[k].v[i]));
            // (padded rows take whole units: zeros past the row's end)
            io_store<Out>(dst, t[k].row * out + t[k].x, t[k].n > 0 && !(out & 3) ? 4 : t[k].n, w);
        }
    }
}

// dense [nz][ny][nx] of transfer type Src -> padded storage S
template <class S, class Src, int DEPTH>
__global__ __launch_bounds__(256) void pack_kernel(const void* src, void* dst, int nx, long long rows, int run,
                                                   int parts, int pitch) {
    convert_rows<DEPTH, typename Src::T, typename S::T>(
        src, dst, nx, rows, run, parts, nx, pitch, [](typename Src::T v) { return Src::up(v); },
        [](float v) { return S::down(v); });
}

template <class S, typename DstT, int DEPTH>
__global__ __launch_bounds__(256) void unpack_kernel(const void* src, DstT* dst, int nx, long long rows, int run,
                                                     int parts, int pitch) {
    convert_rows<DEPTH, typename S::T, DstT>(
        src, dst, nx, rows, run, parts, pitch, nx, [](typename S::T v) { return S::up(v); },
        [](float v) { return DstT(v); });
}

// ----------------------------------------------------------- copy ceiling

// One 16-byte element per thread, streamed with non-temporal load/store:
// the read+write bandwidth ceiling a kernel can reach.
__global__ __launch_bounds__(256) void copy_kernel(const float4* __restrict__ src,
                                                   float4* __restrict__ dst, long long n4) {
    typedef float v4f __attribute__((ext_vector_type(4)));
    const long long i = blockIdx.x * 256LL + threadIdx.x;
    if (i < n4) {
        const v4f v = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(src) + i);
        __builtin_nontemporal_store(v, reinterpret_cast<v4f*>(dst) + i);
    }
}

}  // namespace rdk

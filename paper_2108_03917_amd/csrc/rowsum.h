// Column sums of row-major fp32 matrices of partial results, in a fixed
// order (so that the sums do not depend on scheduling): out[j] = sum over
// r < rows of part[r * n + j], for up to kRsJobs matrices in one launch.
//
// A workgroup takes up to 16 columns of one matrix (fewer when the matrix is
// narrower) and up to kRsChunk rows of them: thread (g, c) adds rows g,
// g + G, g + 2G, .. of column c in fp64, eight loads in flight, and the G
// threads of a column are added in a fixed tree, rounded to fp32 once.  The
// callers' matrices have at most a few thousand rows (one per wavefront or
// per chunk of points), which one workgroup walks in 64 loads a thread; a
// taller one is added chunk by chunk and the chunk sums by the next level.
// What bounds it is the launch, not the bytes: two levels of 64-row chunks,
// one matrix at a time, took eight launches of 5 us for the four sums of a
// DeformSlice backward; one launch of all four takes 5-6 us.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

// Each source file that includes this gets its own copy of the kernel.
namespace rowsum {

struct Job {
    const float *part;
    float *out;
    int64_t rows, n;
};

namespace {

constexpr int kRsJobs = 4;
constexpr int64_t kRsChunk = 8192;
constexpr int kRsBlock = 1024;

struct Jobs {
    Job j[kRsJobs];
    int64_t first[kRsJobs + 1];  // first column block of each matrix
};

__global__ __launch_bounds__(kRsBlock) void k_rowsum(Jobs jobs, int count) {
    __shared__ double red[kRsBlock];
    int k = 0;
    while (k + 1 < count && (int64_t)blockIdx.x >= jobs.first[k + 1]) ++k;
    const Job job = jobs.j[k];
    const int64_t n = job.n;
    int cols = 16;
    while (cols > 1 && cols / 2 >= n) cols /= 2;
    const int G = kRsBlock / cols;
    const int c = threadIdx.x & (cols - 1), g = threadIdx.x / cols;
    const int64_t j = ((int64_t)blockIdx.x - jobs.first[k]) * cols + c;
    const int64_t r0 = (int64_t)blockIdx.y * kRsChunk;
    if (r0 > 0 && r0 >= job.rows) return;  // a shorter matrix than the launch's tallest
    const int64_t r1 = r0 + kRsChunk < job.rows ? r0 + kRsChunk : job.rows;
    double s = 0.0;
    if (j < n) {
        int64_t r = r0 + g;
        for (; r + 7 * G < r1; r += 8 * G) {
            float x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = job.part[(r + u * G) * n + j];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += (double)x[u];
        }
        for (; r < r1; r += G) s += (double)job.part[r * n + j];
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int h = G / 2; h > 0; h /= 2) {
        if (g < h) red[threadIdx.x] += red[threadIdx.x + h * cols];
        __syncthreads();
    }
    if (g == 0 && j < n) job.out[(int64_t)blockIdx.y * n + j] = (float)red[threadIdx.x];
}

inline int64_t column_blocks(int64_t n) {
    int cols = 16;
    while (cols > 1 && cols / 2 >= n) cols /= 2;
    return (n + cols - 1) / cols;
}

// Floats of scratch that sum() needs for `rows` rows of n columns.
inline int64_t scratch_floats(int64_t rows, int64_t n) {
    int64_t total = 0;
    for (int64_t r = rows; r > kRsChunk;) {
        r = (r + kRsChunk - 1) / kRsChunk;
        total += r * n;
    }
    return total;
}

// Matrices of at most kRsChunk rows each, in one launch; rows = 0 writes zeros.
inline hipError_t launch_level(hipStream_t stream, const Job *job, int count, int64_t chunks) {
    Jobs jobs = {};
    int64_t at = 0;
    int used = 0;
    for (int i = 0; i < count; ++i) {
        if (job[i].n <= 0 || !job[i].out) continue;
        jobs.j[used] = job[i];
        jobs.first[used++] = at;
        at += column_blocks(job[i].n);
    }
    jobs.first[used] = at;
    if (used == 0) return hipSuccess;
    hipLaunchKernelGGL(k_rowsum, dim3((unsigned)at, (unsigned)chunks), dim3(kRsBlock), 0, stream, jobs, used);
    return hipGetLastError();
}

// out[0..n) = column sums of part [rows][n]; `tmp` holds scratch_floats(rows,
// n) floats (the levels' chunk sums).  rows = 0 writes zeros.
inline hipError_t sum(hipStream_t stream, const float *part, int64_t rows, int64_t n, float *tmp, float *out) {
    if (n <= 0) return hipSuccess;
    while (rows > kRsChunk) {
        const int64_t chunks = (rows + kRsChunk - 1) / kRsChunk;
        const Job job = {part, tmp, rows, n};
        const hipError_t e = launch_level(stream, &job, 1, chunks);
        if (e != hipSuccess) return e;
        part = tmp;
        tmp += chunks * n;
        rows = chunks;
    }
    const Job job = {part, out, rows, n};
    return launch_level(stream, &job, 1, 1);
}

// Up to kRsJobs such sums (jobs without an output are passed over): the
// matrices that one workgroup can walk go together in one launch.
inline hipError_t sum_all(hipStream_t stream, const Job *job, int count, float *tmp) {
    Job one[kRsJobs];
    int used = 0;
    for (int i = 0; i < count; ++i) {
        if (!job[i].out) continue;
        if (job[i].rows <= kRsChunk) {
            one[used++] = job[i];
            continue;
        }
        const hipError_t e = sum(stream, job[i].part, job[i].rows, job[i].n, tmp, job[i].out);
        if (e != hipSuccess) return e;
    }
    return launch_level(stream, one, used, 1);
}

}  // namespace
}  // namespace rowsum

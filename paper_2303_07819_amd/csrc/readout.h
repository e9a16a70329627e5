// Read-outs to host memory: one kernel gathers every part of a read-out into a
// buffer of pinned host memory that its object keeps, one wait, one host copy.
//
// A copy to pageable memory costs 15 to 70 us apart from its bytes (the runtime
// pins or stages each by itself and waits for it), and a small read-out is
// several: statistics rows, an error word, seven floe arrays.  Here a read-out
// costs a launch and a wait.  4 x 4 cells of 32 floes, 20 steps and all three
// read-outs: 379 -> 242 us; 64 x 64 cells, 32 steps, statistics and continuum:
// 739 -> 680 us; loss gradient of 300 rows, 158 KB: 61 -> 37 us.  Pinning takes
// 0.35 us per KB, so objects reserve for their usual read-out when they are made.
// Read-outs beyond kStagingMax go to the caller's memory directly: there the
// bytes cost (0.06 us per KB, against 0.035 here), and the pinned memory an
// object holds stays bounded.
#pragma once

namespace spdem {

constexpr size_t kStagingStep = 64 * 1024, kStagingMax = 4 * 1024 * 1024;
constexpr int kReadParts = 10;

// n elements of 4 (or, wide, 8) bytes: element i is src[(i / len) * row + (i % len) * col].
struct ReadPart {
    const void* src;
    uint32_t n, len, row, col, dst;   // dst: byte offset in the staging buffer
    int32_t wide;
};

struct ReadParts {
    ReadPart p[kReadParts];
};

__global__ __launch_bounds__(256) void readout_kernel(ReadParts a, unsigned char* out)
{
    const ReadPart p = a.p[blockIdx.y];
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < p.n; i += gridDim.x * 256) {
        const uint32_t r = i / p.len;
        const size_t at = (size_t)r * p.row + (size_t)(i - r * p.len) * p.col;
        if (p.wide)
            reinterpret_cast<double*>(out + p.dst)[i] = static_cast<const double*>(p.src)[at];
        else
            reinterpret_cast<uint32_t*>(out + p.dst)[i] = static_cast<const uint32_t*>(p.src)[at];
    }
}

}  // namespace spdem

namespace {

// The pinned buffer of one object (a simulation, a network, a global DEM).  A
// read-out holds `mu` from reserving the buffer to its last copy out of it:
// threads that read the same object out take turns.
struct Staging {
    std::mutex mu;
    unsigned char* host = nullptr;
    size_t cap = 0;

    void release()
    {
        if (host) (void)hipHostFree(host);
        host = nullptr;
        cap = 0;
    }
    // At least `bytes`, or false (nothing may still be reading or writing it).
    bool reserve(size_t bytes)
    {
        if (bytes <= cap) return true;
        if (bytes > spdem::kStagingMax) return false;
        const size_t want = (bytes + spdem::kStagingStep - 1) / spdem::kStagingStep * spdem::kStagingStep;
        release();
        void* p = nullptr;
        if (hipHostMalloc(&p, want, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            return false;
        }
        host = static_cast<unsigned char*>(p);
        cap = want;
        return true;
    }
};

// One read-out: add() its parts (at most kReadParts), then run() once, which
// waits for the stream and fills the parts' outputs.  Parts that do not fit the
// staging buffer are copied one by one; run() returns false, with nothing done,
// only if one of those is strided (len != 1).
class Readout {
public:
    void add(void* out, const void* src, size_t n, bool wide, uint32_t len = 1, uint32_t row = 1, uint32_t col = 1)
    {
        if (n == 0) return;
        const size_t at = (bytes_ + 15) & ~(size_t)15;
        bytes_ = at + n * (wide ? 8 : 4);
        a_.p[parts_] = spdem::ReadPart{src, (uint32_t)n, len, row, col, (uint32_t)at, wide ? 1 : 0};
        to_[parts_] = out;
        size_[parts_++] = n * (wide ? 8 : 4);
        strided_ = strided_ || len != 1;
        most_ = std::max(most_, n);
    }

    bool run(Staging& s, hipStream_t stream, hipError_t& err)
    {
        err = hipSuccess;
        std::lock_guard<std::mutex> lock(s.mu);
        const bool staged = parts_ > 0 && s.reserve(bytes_);
        if (staged) {
            const unsigned blocks = (unsigned)std::min<size_t>((most_ + 1023) / 1024, 256);
            hipLaunchKernelGGL(spdem::readout_kernel, dim3(blocks, (unsigned)parts_), dim3(256), 0, stream, a_, s.host);
            err = hipGetLastError();
        } else {
            if (strided_) return false;
            for (int i = 0; i < parts_ && err == hipSuccess; ++i)
                err = hipMemcpyAsync(to_[i], a_.p[i].src, size_[i], hipMemcpyDeviceToHost, stream);
        }
        if (err == hipSuccess) err = hipStreamSynchronize(stream);
        if (err == hipSuccess && staged)
            for (int i = 0; i < parts_; ++i) memcpy(to_[i], s.host + a_.p[i].dst, size_[i]);
        return true;
    }

private:
    spdem::ReadParts a_;
    void* to_[spdem::kReadParts];
    size_t size_[spdem::kReadParts];
    size_t bytes_ = 0, most_ = 0;
    int parts_ = 0;
    bool strided_ = false;
};

}  // namespace

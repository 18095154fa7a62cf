// HostFetch (paper_2511_09165_amd/csrc/dmas_fetch.hpp) on the CPU: the HIP
// calls it makes are defined here over host memory and counted. Destinations
// that HIP knows take one hipMemcpy, pageable ones the chunks; where the
// buffers, streams or threads cannot be had every copy is one hipMemcpy and no
// error is left behind. Prints "ok <checks>".
#include "../paper_2511_09165_amd/csrc/dmas_fetch.hpp"

#include <cstdio>
#include <cstdlib>

static std::atomic<int> n_memcpy{0}, n_async{0}, n_streams{0}, n_hosts{0};
static hipError_t last_error = hipSuccess;
static const void *known = nullptr;          // memory that HIP knows
static hipMemoryType known_type = hipMemoryTypeHost;
static bool unknown_is_error = false;
static int streams_left = 1 << 30;

extern "C" {
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = std::malloc(n); ++n_hosts; return hipSuccess; }
hipError_t hipHostFree(void *p) { std::free(p); --n_hosts; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned)
{
    if (streams_left-- <= 0) return last_error = hipErrorOutOfMemory;
    *s = reinterpret_cast<hipStream_t>(std::malloc(1));
    ++n_streams;
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { std::free((void *)s); --n_streams; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError(void) { const hipError_t e = last_error; last_error = hipSuccess; return e; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { ++n_memcpy; std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    ++n_async;
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p)
{
    if (p == known) {
        a->type = known_type;
        return hipSuccess;
    }
    if (unknown_is_error) return last_error = hipErrorInvalidValue;
    a->type = hipMemoryTypeUnregistered;
    return hipSuccess;
}
}

static long checks = 0;
#define CHECK(cond)                                                    \
    do {                                                               \
        ++checks;                                                      \
        if (!(cond)) {                                                 \
            std::fprintf(stderr, "line %d: %s\n", __LINE__, #cond);    \
            std::exit(1);                                              \
        }                                                              \
    } while (0)

static void fetch(dmas::HostFetch &f, size_t bytes, bool direct)
{
    std::vector<unsigned char> src(bytes), dst(bytes);
    for (size_t i = 0; i < bytes; ++i) src[i] = (unsigned char)(i * 2654435761u >> 24);
    if (direct) known = dst.data();
    n_memcpy = n_async = 0;
    CHECK(f.copy(dst.data(), src.data(), bytes) == hipSuccess);
    known = nullptr;
    CHECK(src == dst);
    CHECK(last_error == hipSuccess);
}

int main()
{
    const size_t C = dmas::HostFetch::kChunk;
    {
        dmas::HostFetch f;
        CHECK(f.start(0) == hipSuccess);
        for (bool as_error : {false, true}) {
            unknown_is_error = as_error;
            for (size_t bytes : {(size_t)4, 2 * C - 1}) {      // small: one copy wherever it goes
                fetch(f, bytes, false);
                CHECK(n_memcpy == 1 && n_async == 0);
            }
            for (size_t bytes : {2 * C, 5 * C + 12345, 16 * C}) {
                fetch(f, bytes, false);
                CHECK(n_memcpy == 0 && n_async == (int)((bytes + C - 1) / C));
                for (hipMemoryType t : {hipMemoryTypeHost, hipMemoryTypeManaged, hipMemoryTypeDevice}) {
                    known_type = t;
                    fetch(f, bytes, true);
                    CHECK(n_memcpy == 1 && n_async == 0);
                }
            }
        }
    }
    CHECK(n_streams == 0 && n_hosts == 0);
    {
        dmas::HostFetch f;                                     // no second stream
        streams_left = 1;
        CHECK(f.start(0) == hipErrorOutOfMemory);
        CHECK(last_error == hipSuccess);
        CHECK(n_streams == 0 && n_hosts == 0);
        fetch(f, 4 * C, false);
        CHECK(n_memcpy == 1 && n_async == 0);
    }
    std::printf("ok %ld\n", checks);
    return 0;
}

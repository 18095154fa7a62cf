// Host checks of how a plan sizes its launches, on the CPU: the RF segments
// (choose_rf_segments) and the root pass's grid (root_grid) over sizes up to
// the limits of the entry points, and the blocks of launches without a root
// plane (direct_block_of) against the tables', and the padding and
// memory of root planes (plane_pads, allocate_plane). Prints "ok <checks>".
#include "../paper_2511_09165_amd/csrc/dmas_plan.hpp"

#include <cstdio>
#include <cstdlib>

static hipError_t g_error = hipSuccess;
extern "C" hipError_t hipGetLastError(void)
{
    const hipError_t e = g_error;
    g_error = hipSuccess;
    return e;
}

static long checks = 0;
#define CHECK(cond, ...)                              \
    do {                                              \
        ++checks;                                     \
        if (!(cond)) {                                \
            std::fprintf(stderr, "%s: ", #cond);      \
            std::fprintf(stderr, __VA_ARGS__);        \
            std::fprintf(stderr, "\n");               \
            std::exit(1);                             \
        }                                             \
    } while (0)

constexpr int64_t kThreads32 = (int64_t)1 << 32;   // a launch holds fewer in each dimension

static void rf_segments()
{
    const int wg = dmas::kDirsPerTile * dmas::kWaveSize;
    for (int64_t tiles : {1, 7, 523, 4096, 65537, 1 << 20, 4194304, 8388607}) {
        for (int64_t T : {1, 256, 257, 769, 4096, 65536, 1 << 20, 1073739000}) {
            for (int64_t slots : {256, 768, 1024, 2048}) {
                int seg = 0, nseg = 0;
                dmas::choose_rf_segments((int)T, (int)tiles, slots, 0, &seg, &nseg);
                CHECK(seg > 0 && seg % 32 == 0, "tiles %ld T %ld seg %d", (long)tiles, (long)T, seg);
                CHECK((int64_t)seg * nseg >= T && (int64_t)seg * (nseg - 1) < T, "tiles %ld T %ld", (long)tiles, (long)T);
                CHECK(tiles * nseg * wg < kThreads32, "tiles %ld T %ld nseg %d", (long)tiles, (long)T, nseg);
                // three chunks at most where the launch holds them
                const int64_t three = (T + 3 * dmas::kChunk - 1) / (3 * dmas::kChunk);
                if (tiles * three * wg < kThreads32) CHECK(seg <= 3 * dmas::kChunk, "tiles %ld T %ld", (long)tiles, (long)T);
            }
        }
    }
    int seg = 0, nseg = 0;
    dmas::choose_rf_segments(1000, 5, 768, 100, &seg, &nseg);
    CHECK(seg == 128 && nseg == 8, "fixed segments %d x %d", seg, nseg);
}

static void root_pass()
{
    for (int64_t M : {1, 8, 1024, 65535, 65536, 70000, 16777216, 1 << 30}) {
        for (int64_t stride : {1, 1023, 1024, 1025, 16384, 1 << 24, 1700000000}) {
            unsigned gx = 0, gy = 0;
            dmas::root_grid((int)M, (int)stride, &gx, &gy);
            CHECK((int64_t)gx * dmas::kRootThreads < kThreads32 && gy >= 1 && gy <= 65535, "M %ld stride %ld", (long)M, (long)stride);
            CHECK((int64_t)gx * dmas::kRootBlock >= stride && ((int64_t)gx - 1) * dmas::kRootBlock < stride,
                  "M %ld stride %ld", (long)M, (long)stride);
        }
    }
}

// A plane-free launch walks blocks of b microphones over tables built for
// blocks of mb: with the row the kernel keeps (zero at the first block, b more
// at each, zero again at mb), microphone i's row is that of the tables.
static void direct_blocks()
{
    for (int M = 1; M <= 80; ++M) {
        for (int mb = 1; mb <= M; ++mb) {
            for (int cap : {4, 16}) {
                const int b = dmas::direct_block_of(mb, M, cap);
                CHECK(b >= 1 && b <= cap && b <= mb, "M %d mb %d cap %d", M, mb, cap);
                int trow = 0;
                for (int m0 = 0; m0 < M; m0 += b) {
                    for (int i = m0; i < m0 + b && i < M; ++i)
                        CHECK(i % mb - trow == i - m0, "M %d mb %d b %d microphone %d", M, mb, b, i);
                    trow += b;
                    if (trow >= mb) trow = 0;
                }
            }
        }
    }
}

// Padded rows hold every window of a plan: a chunk starts in [0, T), a window
// at its microphone's smallest delay in the tile (tables) or at the reference
// delay less the halo, and is `row` pairs long.
static void plane_padding()
{
    int padded = 0, plain = 0;
    for (bool tables : {true, false}) {
        for (double delay : {0.0, 0.4, 13.7, 105.5, 105.49951, 700.0, 5000.0, 9.9e7}) {
            for (int halo : {0, 1, 29, 62, 400}) {
                for (int range : {halo, halo + halo / 4, 2 * halo}) {
                    for (int T : {1, 255, 300, 2048, 8192, 100000, 1073739000}) {
                        for (int M : {1, 64, 1024, 20000000}) {
                            dmas_plan_s p;
                            p.tables = tables;
                            p.roots = true;
                            p.halo = halo;
                            p.range = range;
                            p.M = M;
                            p.T = T;
                            p.row = (dmas::kChunk + (tables ? range : 2 * halo) + 3) & ~3;
                            dmas::plane_pads(&p, delay);
                            const size_t extra = dmas::padded_plane_bytes(&p) - dmas::plane_bytes(&p);
                            CHECK(p.pad0 >= 0 && p.pad1 >= 0 && p.pad0 % 4 == 0 && p.pad1 % 4 == 0, "T %d", T);
                            CHECK((int64_t)p.pad0 + T + p.pad1 <= INT32_MAX && p.pad0 + p.pad1 <= T + 1024, "T %d", T);
                            CHECK(extra <= (size_t)256 << 20, "M %d T %d: %zu bytes of padding", M, T, extra);
                            if (!p.pad1) {
                                ++plain;
                                continue;
                            }
                            ++padded;
                            const int d = (int)std::ceil(delay) + 1;        // delays lie in [-d, d]
                            const int first = 0 - d - (tables ? 0 : halo);
                            const int last = T - 1 + d - (tables ? 0 : halo) + p.row;
                            CHECK(first >= -p.pad0 && last <= T + p.pad1, "delay %g halo %d range %d T %d: [%d, T%+d) in [%d, T%+d)",
                                  delay, halo, range, T, first, last - T, -p.pad0, p.pad1);
                        }
                    }
                }
            }
        }
    }
    CHECK(padded > 100 && plain > 100, "%d padded, %d plain", padded, plain);
}

// Where the device has no room for the padding the plane goes without it.
static void plane_memory()
{
    dmas_plan_s p;
    p.roots = true;
    p.M = 8;
    p.T = 1000;
    p.pad0 = 40;
    p.pad1 = 300;
    const size_t plain = 8 * 1000 * 8, full = 8 * 1340 * 8;
    float2 *plane = nullptr;
    bool padded = false;
    for (size_t room : {full, full - 1, plain, plain - 1}) {
        int calls = 0;
        auto alloc = [&](void **mem, size_t bytes) {
            ++calls;
            if (bytes > room) {
                g_error = hipErrorOutOfMemory;
                return hipErrorOutOfMemory;
            }
            *mem = &p;
            return hipSuccess;
        };
        g_error = hipSuccess;
        const hipError_t e = dmas::allocate_plane(&p, alloc, &plane, &padded);
        CHECK((e == hipSuccess) == (room >= plain), "room %zu", room);
        CHECK((plane != nullptr) == (e == hipSuccess), "room %zu", room);
        if (e == hipSuccess) CHECK(padded == (room >= full) && g_error == hipSuccess, "room %zu", room);
        CHECK(calls == (room >= full ? 1 : 2), "room %zu: %d calls", room, calls);
    }
    int calls = 0;                                  // other errors are reported as they are
    auto broken = [&](void **, size_t) { ++calls; return hipErrorInvalidValue; };
    CHECK(dmas::allocate_plane(&p, broken, &plane, &padded) == hipErrorInvalidValue && calls == 1, "%d calls", calls);
}

int main()
{
    plane_padding();
    plane_memory();
    rf_segments();
    direct_blocks();
    root_pass();
    std::printf("ok %ld\n", checks);
    return 0;
}

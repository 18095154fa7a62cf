// Envelope filter as a pass of its own over an RF image that is already in
// the output buffer: env[t] = sum_k h[k] |y[t + H - k]|, y = 0 outside [0, T),
// row by row and in place.
//
// The same 16 x 16 Toeplitz products in FP32 on the matrix cores, in the same
// K order, as the beamformer's fused epilogue (dmas_kernel.hpp): an output's
// products depend on its time index modulo 16 only, so both forms give the
// same bits. That includes samples that are not finite. The products of a
// block of 16 outputs run over 2H + 16 samples, for odd H over 2H + 18, and so
// multiply samples outside an output's taps by zero, which a NaN or infinity
// turns into NaN: up to 17 outputs before and 15 after those whose taps hold it.
// Where the fused kernel has a zero in place of such a sample (past the end of
// its chunk), this one takes a zero too (products_again).
//
// Bound: HBM (each sample read and written once) and the matrix cores, whose
// FP32 products do not run beside one another's loads well: 4186 x 16384
// samples take 134 us (4.1 TB/s), 90 us with the products left out (6.1 TB/s;
// a large copy reaches 5.1-5.4) and 80 us for the products alone. Loads one
// step ahead and barriers that wait for LDS only brought it there from 190 us;
// a block's operand reads ahead of its products took another 2 us off small
// images (361 x 4096: 10.8 -> 8.9 us).
#include "dmas_barrier.hpp"
#include "dmas_internal.hpp"

namespace dmas {

namespace {

constexpr int kRowThreads = 256;
constexpr int kRowWaves = kRowThreads / kWaveSize;
constexpr int kRowBlock = 2048;   // outputs of one walk step
static_assert(kRowBlock % (kChunk * kRowWaves) == 0, "each wave takes whole output blocks");

// LDS window of a walk step: |y| of indices [0, kRowBlock + 2H + kPast), which
// are all that the FIR's K steps use (kPast: those past the last output's
// taps), and zeros up to the last index that is read. Index i lies in plane i % 4
// at i / 4: a lane's operand of K steps 4q .. 4q + 3 is then 16 consecutive
// bytes (one ds_read_b128 instead of four 4-byte reads), and the planes lie
// 16 banks apart, so that both those reads and the element-wise fill, 64
// consecutive indices a wave, fall on distinct banks.
constexpr int kPast = 2;
__host__ __device__ constexpr int row_logical(int H) { return kRowBlock + 2 * H + 24; }
__host__ __device__ constexpr int row_plane(int H) { return ((row_logical(H) / 4 + 1 + 63) & ~63) + 16; }
__host__ __device__ constexpr int row_floats(int H) { return 4 * row_plane(H); }
// Output staging of a wave whose rows are not 16-byte aligned.
constexpr int kRowStage = kChunk;

// A workgroup walks whole rows, blockIdx.x and every gridDim.x-th after it, in
// steps of kRowBlock outputs, and loads the next step's samples while it works
// on this one's. The step at o0 holds |y| of [o0 - H, o0 + kRowBlock + H +
// kPast) (its first 2H + kPast values kept from the step before) and stores
// [o0, o0 + kRowBlock); the samples loaded ahead start at o0 + kRowBlock + H +
// kPast or in another row, so no output is stored over a sample that is still
// to be loaded. seg_len: the fused kernel's outputs per segment (a multiple of
// 32), seg_inv = floor((2^32 - 1) / (seg_len / 32)).
// KS: the K steps, with a lane's taps in registers (0: any number, taps read
// per block).
template <int KS>
__global__ void __launch_bounds__(kRowThreads, 8)
envelope_rows_kernel(float *__restrict__ img, const float *__restrict__ taps, int D, int T, int L, int seg_len,
                     uint32_t seg_inv)
{
    typedef float v4f __attribute__((ext_vector_type(4)));
    extern __shared__ float smem[];
    const int H = (L - 1) / 2;
    const int plane = row_plane(H);
    float *win = smem;
    float *stage = smem + row_floats(H);
    float *tap_lds = stage + kRowWaves * kRowStage;
    const int tid = threadIdx.x;
    const int lane = tid & (kWaveSize - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWaveSize);
    const int g = lane >> 4, c = lane & 15;
    const int ks = env_ksteps(H);
    auto at = [&](int i) { return (i & 3) * plane + (i >> 2); };

    const int keep_len = 2 * H + kPast;   // <= kRowThreads

    // new samples of a step: t = o0 + H + kPast + j * kRowThreads + tid; the first
    // step of a row also has samples 0 .. H + kPast - 1
    constexpr int kLoads = kRowBlock / kRowThreads;
    float v[kLoads], head = 0.0f;
    auto fetch = [&](int d, int o0) {
        const float *src = img + (size_t)d * (size_t)T;
#pragma unroll
        for (int j = 0; j < kLoads; ++j) {
            const int t = o0 + H + kPast + j * kRowThreads + tid;
            v[j] = t < T ? src[t] : 0.0f;
        }
        if (o0 == 0) head = tid >= H && tid < keep_len && tid - H < T ? src[tid - H] : 0.0f;
    };
    int d = blockIdx.x, o0 = 0;
    if (d < D) fetch(d, 0);

    for (int j = tid; j < env_taps_len(H); j += kRowThreads) {
        const int k = j - kTapLead;   // reversed: entry kTapLead + k holds h[2H - k]
        tap_lds[j] = (k >= 0 && k <= 2 * H) ? taps[2 * H - k] : 0.0f;
    }
    for (int i = kRowBlock + keep_len + tid; i < row_logical(H); i += kRowThreads) win[at(i)] = 0.0f;
    lds_barrier();
    const float *ha = tap_lds + kTapLead + g - c;   // hr[m - i] of K step kk at ha[4 kk]
    float a[KS > 0 ? KS : 1];
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) a[kk] = ha[4 * kk];

    // Outputs that are not finite are formed again, a K step at a time: products of
    // the wave's block of 256 outputs at t0 with the window operands at rq. Where
    // the fused kernel has a zero in place of the sample that K row 3 of the last
    // step holds, the first one past the chunk that yields the 16 outputs, it is a
    // zero here too. A segment at g0 walks chunks from max(g0 - lead, 0); a chunk's
    // last outputs reach past it only if H + 1 is a multiple of 32 (= lead). That
    // sample's tap is zero, so it matters only where it is not finite, and then all
    // 16 outputs are not. (Choosing the operand ahead of the products cost
    // registers, 0.5-2.5 % of a call, and with taps read per block 6 %.)
    const bool reaches = ((H + 1) & 31) == 0;
    auto products_again = [&](const float *rq, int t0) {
        int me = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        asm volatile("" : "+v"(me));   // lane values formed here: kept from above they cost registers
        const int g = me >> 4, c = me & 15;
        const float *ha = tap_lds + kTapLead + g - c;
        v4f e0 = {0.0f, 0.0f, 0.0f, 0.0f}, e1 = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
        for (int kk = 0; kk < ks; ++kk) {
            float r = rq[kk];
            if (kk == ks - 1) {
                const int tb = t0 + 16 * c, lead = env_lead(H);
                const uint32_t n = (uint32_t)tb >> 5, len = (uint32_t)seg_len >> 5;
                uint32_t seg = __umulhi(n, seg_inv);   // n / len or one less
                if (n - seg * len >= len) ++seg;
                const int start = max((int)seg * seg_len - lead, 0);
                if (g == 3 && ((tb + lead + 16 - start) & (kChunk - 1)) == 0) r = 0.0f;
            }
            const v4f e = __builtin_amdgcn_mfma_f32_16x16x4f32(ha[4 * kk], r, kk & 1 ? e1 : e0, 0, 0, 0);
            if (kk & 1) e1 = e;
            else e0 = e;
        }
        return e0 + e1;
    };

    while (d < D) {
        // window index i holds |y[o0 - H + i]|
        float keep = __builtin_fabsf(head);            // indices 0 .. keep_len - 1
        if (o0 > 0) {
            if (tid < keep_len) keep = win[at(kRowBlock + tid)];
            lds_barrier();
        }
        if (tid < keep_len) win[at(tid)] = keep;
#pragma unroll
        for (int j = 0; j < kLoads; ++j) win[at(keep_len + j * kRowThreads + tid)] = __builtin_fabsf(v[j]);
        lds_barrier();
        float *row = img + (size_t)d * (size_t)T;
        const int o = o0;
        o0 += kRowBlock;
        if (o0 >= T) {
            o0 = 0;
            d += gridDim.x;
        }
        if (d < D) fetch(d, o0);

        for (int b = wave * kChunk; b < min(kRowBlock, T - o); b += kRowWaves * kChunk) {
            // outputs o + b + q, q = 16j + i: F[i][j] = sum_m hr[m - i] r[16j + m], r = window
            // from b; lane l supplies r[16c + 4kk + g] and receives the outputs 16c + 4g ..+3
            const v4f *rq = reinterpret_cast<const v4f *>(win + g * plane + (b >> 2) + 4 * c);
            v4f e0 = {0.0f, 0.0f, 0.0f, 0.0f}, e1 = {0.0f, 0.0f, 0.0f, 0.0f};
            if constexpr (KS > 0) {
                v4f r[(KS + 3) / 4];   // all reads first
#pragma unroll
                for (int q = 0; q < (KS + 3) / 4; ++q) r[q] = rq[q];
#pragma unroll
                for (int kk = 0; kk < KS; ++kk) {
                    if (kk & 1) e1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[kk], r[kk >> 2][kk & 3], e1, 0, 0, 0);
                    else e0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[kk], r[kk >> 2][kk & 3], e0, 0, 0, 0);
                }
            } else {
                for (int q = 0; 4 * q < ks; ++q) {
                    const v4f r = rq[q];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        if (4 * q + u >= ks) break;
                        if (u & 1) e1 = __builtin_amdgcn_mfma_f32_16x16x4f32(ha[16 * q + 4 * u], r[u], e1, 0, 0, 0);
                        else e0 = __builtin_amdgcn_mfma_f32_16x16x4f32(ha[16 * q + 4 * u], r[u], e0, 0, 0, 0);
                    }
                }
            }
            v4f e = e0 + e1;
            if (reaches && __builtin_amdgcn_ballot_w64(!(__builtin_fabsf(e[0]) <= __FLT_MAX__)) != 0)   // wave-uniform
                e = products_again(reinterpret_cast<const float *>(rq), o + b);
            const int t0 = o + b;
            const int t = t0 + 16 * c + 4 * g;
            if ((reinterpret_cast<uintptr_t>(row) & 15) == 0) {   // wave-uniform
                float *dst = row + t;
                if (t + 3 < T) {
                    __builtin_nontemporal_store(e, reinterpret_cast<v4f *>(dst));
                } else {
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (t + u < T) __builtin_nontemporal_store(e[u], dst + u);
                }
            } else {
                // rows off the 16-byte grid: through LDS, so that a wave stores 256
                // consecutive bytes at a time instead of 4-byte pieces 16 apart
                float *st = stage + wave * kRowStage;
                *reinterpret_cast<v4f *>(st + 16 * c + 4 * g) = e;
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int q = lane + kWaveSize * u;
                    if (t0 + q < T) __builtin_nontemporal_store(st[q], row + t0 + q);
                }
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
        }
        lds_barrier();   // the window is read before the next step fills it
    }
}

}  // namespace

hipError_t launch_envelope_rows(float *img, const float *taps, int D, int T, int L, int seg_len, int cus,
                                hipStream_t stream)
{
    const int H = (L - 1) / 2;
    const size_t lds = sizeof(float) * (size_t)(row_floats(H) + kRowWaves * kRowStage + env_taps_len(H));
    // workgroups for eight a CU (their LDS and registers allow eight)
    const unsigned grid = (unsigned)(D < 8 * cus ? D : 8 * cus);
    // 20 K steps: 63 (the default) and 65 taps
    auto kern = env_ksteps(H) == 20 ? envelope_rows_kernel<20> : envelope_rows_kernel<0>;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kRowThreads), lds, stream, img, taps, D, T, L, seg_len,
                       0xffffffffu / ((uint32_t)seg_len >> 5));
    return hipGetLastError();
}

}  // namespace dmas

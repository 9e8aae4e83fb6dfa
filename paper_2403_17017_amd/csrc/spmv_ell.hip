// Stand-alone kernels and launchers of ELL,TM: the conversion from CSR (its preprocessing)
// and the product; device code and layout are described in spmv_bodies.hiph.
#include "spmv_bodies.hiph"

namespace seer {

__global__ __launch_bounds__(kWG) void ell_convert_kernel(
    int rows, uint32_t rows_pad, uint32_t width, const int *__restrict__ rp, const int *__restrict__ ci,
    const float *__restrict__ va, int *__restrict__ ec, float *__restrict__ ev, int *__restrict__ shift,
    uint32_t *__restrict__ sampled)
{
    ell_convert_body(rows, rows_pad, width, rp, ci, va, ec, ev, shift, sampled);
}

template <bool NT, bool OFFSETS>
__global__ __launch_bounds__(kWG) void spmv_ell_kernel(
    int rows, uint32_t rows_pad, uint32_t width, const int *__restrict__ ec, const float *__restrict__ ev,
    const float *__restrict__ x, float *__restrict__ y, uint32_t n_tiles, int remap, const int *__restrict__ shift)
{
    const uint32_t tile = tile_of_block(blockIdx.x, n_tiles, remap);
    if (tile >= n_tiles) return;
    ell_body<NT, OFFSETS>(rows, rows_pad, width, ec, ev, x, y, tile, shift);
}

uint32_t ell_rows_pad(int rows) { return ((uint32_t)rows + kEllRowMultiple - 1) / kEllRowMultiple * kEllRowMultiple; }

// columns then values, each rows_pad * width words; 0 if the arrays cannot be indexed
size_t ell_plan_bytes(int rows, int width)
{
    if (rows <= 0 || width < 0) return 0;
    const uint64_t words = (uint64_t)ell_rows_pad(rows) * (uint64_t)width;
    if (words >= (1ull << 31)) return 0;
    const size_t one = ((size_t)words * 4 + 255) & ~(size_t)255;
    return one ? 2 * one : 256;
}

// behind the arrays, where there is room: a word per slot and 64 rows, then the sample
size_t ell_shift_bytes(int rows, int width)
{
    return (((size_t)(ell_rows_pad(rows) / kEllRowMultiple) * (size_t)width * 4 + 255) & ~(size_t)255) + 256;
}
static uint32_t *ell_sampled(void *plan_mem, int rows, int width)
{
    static_assert(kEllSamples * 4 == 256, "the sample's place");
    return reinterpret_cast<uint32_t *>(static_cast<char *>(plan_mem) + ell_plan_bytes(rows, width) +
                                        ell_shift_bytes(rows, width) - kEllSamples * 4);
}

// Whether three quarters of the slots sampled have one distance, into pinned host memory (max_len).  One wave, a
// sample per lane.
__global__ __launch_bounds__(kWave) void ell_judge_kernel(
    uint32_t rows_pad, uint32_t width, const uint32_t *__restrict__ sampled, FeatureRaw *__restrict__ mailbox, uint64_t seq)
{
    static_assert(kEllSamples == kWave, "a sample per lane");
    const bool is = threadIdx.x * ell_sample_stride(rows_pad) < rows_pad / kEllRowMultiple;
    const auto add = [](uint32_t a, uint32_t b) { return a + b; };   // (64 rows of `width` slots are fewer than 2^31)
    const uint32_t one = wave_fold(is ? sampled[threadIdx.x] : 0u, add), all = wave_fold(is ? width : 0u, add);
    if (threadIdx.x != 0) return;
    mailbox->max_len = 4ull * one >= 3ull * all ? 1 : 0;
    __threadfence_system();
    *reinterpret_cast<volatile uint64_t *>(&mailbox->seq) = seq;
}

void launch_ell_judge(int rows, int width, void *plan_mem, FeatureRaw *mailbox_dev, uint64_t seq, hipStream_t st)
{
    hipLaunchKernelGGL(ell_judge_kernel, dim3(1), dim3(kWave), 0, st, ell_rows_pad(rows), (uint32_t)width,
                       static_cast<const uint32_t *>(ell_sampled(plan_mem, rows, width)), mailbox_dev, seq);
}

static float *ell_values(void *plan_mem, int rows, int width)
{
    return reinterpret_cast<float *>(static_cast<char *>(plan_mem) + ell_plan_bytes(rows, width) / 2);
}

void launch_ell_convert(int rows, int width, const int *rp, const int *ci, const float *va, void *plan_mem,
                        bool with_shift, hipStream_t st)
{
    if (rows <= 0 || width <= 0) return;
    const uint32_t rows_pad = ell_rows_pad(rows);
    hipLaunchKernelGGL(ell_convert_kernel, dim3((rows_pad + kWG - 1) / kWG), dim3(kWG), 0, st, rows, rows_pad,
                       (uint32_t)width, rp, ci, va, static_cast<int *>(plan_mem), ell_values(plan_mem, rows, width),
                       with_shift ? reinterpret_cast<int *>(static_cast<char *>(plan_mem) + ell_plan_bytes(rows, width)) : nullptr,
                       with_shift ? ell_sampled(plan_mem, rows, width) : nullptr);
}

void launch_ell(const SpmvArgs &a, int width, bool with_shift, const void *plan_mem, hipStream_t st)
{
    if (a.rows <= 0) return;
    const uint32_t rows_pad = ell_rows_pad(a.rows), n_tiles = ((uint32_t)a.rows + kWG - 1) / kWG;
    const int *ec = static_cast<const int *>(plan_mem);
    const float *ev = ell_values(const_cast<void *>(plan_mem), a.rows, width);
    const dim3 grid(a.remap ? tiles_per_xcd(n_tiles) * kXCD : n_tiles);
    const int *shift = reinterpret_cast<const int *>(static_cast<const char *>(plan_mem) + ell_plan_bytes(a.rows, width));
#define SEER_ELL_LAUNCH(...)                                                                                    \
    hipLaunchKernelGGL((spmv_ell_kernel<__VA_ARGS__>), grid, dim3(kWG), 0, st, a.rows, rows_pad, (uint32_t)width, ec, ev, \
                       a.x, a.y, n_tiles, a.remap, shift)
    if (with_shift) {
        if (a.nt) SEER_ELL_LAUNCH(true, true); else SEER_ELL_LAUNCH(false, true);
    } else {
        if (a.nt) SEER_ELL_LAUNCH(true, false); else SEER_ELL_LAUNCH(false, false);
    }
#undef SEER_ELL_LAUNCH
}

} // namespace seer

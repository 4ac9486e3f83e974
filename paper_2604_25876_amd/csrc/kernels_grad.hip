// The gradient / observables kernels and the printed-form kernels of both precisions, and the
// choice between the precisions' kernels.
#include "formp.hpp"
#include "kernels.hpp"

namespace skyr {

// Their one output is written once and read by no sweep after them: streamed whatever its size.
template <typename T, class G> static const void* grad_of(int ext, int& threads)
{
    threads = G::THREADS;
    if (ext == EXT_SEXTIC) return (const void*)sweep_kernel<T, G, MODE_GRAD, EXT_SEXTIC, STREAM_ALL>;
    if (ext == EXT_POT) return (const void*)sweep_kernel<T, G, MODE_GRAD, EXT_POT, STREAM_ALL>;
    return (const void*)sweep_kernel<T, G, MODE_GRAD, EXT_NONE, STREAM_ALL>;
}

const void* grad_kernel(skyr_precision prec, int variant, int ext, int& threads)
{
    if (prec == SKYR_F64) {
        int v = 0;
#define SKYR_CASE(a, b, c, d, ...) \
    if (variant == v) return grad_of<double, Geo<a, b, c, d>>(ext, threads); \
    ++v;
        SKYR_SHAPES_F64(SKYR_CASE)
#undef SKYR_CASE
    } else {
        int v = 0;
#define SKYR_CASE(a, b, c, d, ...) \
    if (variant == v) return grad_of<float, Geo<a, b, c, d>>(ext, threads); \
    ++v;
        SKYR_SHAPES_F32(SKYR_CASE)
#undef SKYR_CASE
    }
    threads = 0;
    return nullptr;
}

const void* step_kernel(skyr_precision prec, int variant, int ext, int stream, int& threads)
{
    return prec == SKYR_F64 ? step_kernel_of<double>(variant, ext, stream, threads)
                            : step_kernel_of<float>(variant, ext, stream, threads);
}

const void* batch_kernel(skyr_precision prec, int variant, int ext, int stream, int& threads)
{
    return prec == SKYR_F64 ? batch_kernel_of<double>(variant, ext, stream, threads)
                            : batch_kernel_of<float>(variant, ext, stream, threads);
}

template <typename T, int MODE, bool EXT, bool GROUPS> static const void* printed_of(int stream)
{
    if constexpr (MODE == MODE_STEP) {
        if (stream == STREAM_NONE) return (const void*)formp_kernel<T, MODE, EXT, STREAM_NONE, GROUPS>;
        if (stream == STREAM_STORES) return (const void*)formp_kernel<T, MODE, EXT, STREAM_STORES, GROUPS>;
    }
    return (const void*)formp_kernel<T, MODE, EXT, STREAM_ALL, GROUPS>;
}
template <typename T> static const void* printed_of(int mode, bool ext, int stream, bool groups)
{
    if (mode != MODE_STEP)
        return ext ? printed_of<T, MODE_GRAD, true, false>(stream) : printed_of<T, MODE_GRAD, false, false>(stream);
    if constexpr (sizeof(T) == 4)
        if (groups) return ext ? printed_of<T, MODE_STEP, true, true>(stream) : printed_of<T, MODE_STEP, false, true>(stream);
    return ext ? printed_of<T, MODE_STEP, true, false>(stream) : printed_of<T, MODE_STEP, false, false>(stream);
}

const void* printed_kernel(skyr_precision prec, int mode, bool ext, int stream, bool groups, int& threads)
{
    threads = prec == SKYR_F64 ? FpGeoF64::THREADS : FpGeoF32::THREADS;
    return prec == SKYR_F64 ? printed_of<double>(mode, ext, stream, groups) : printed_of<float>(mode, ext, stream, groups);
}

}  // namespace skyr

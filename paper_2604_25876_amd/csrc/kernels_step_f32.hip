// The step-sweep kernels of one field, float.
#include "sweep.hpp"
#include "kernels.hpp"

namespace skyr {

template <typename T, class G, int EXT> static const void* of_stream(int stream)
{
    if (stream == STREAM_NONE) return (const void*)sweep_kernel<T, G, MODE_STEP, EXT, STREAM_NONE>;
    if (stream == STREAM_STORES) return (const void*)sweep_kernel<T, G, MODE_STEP, EXT, STREAM_STORES>;
    return (const void*)sweep_kernel<T, G, MODE_STEP, EXT, STREAM_ALL>;
}

template <typename T, class G> static const void* of_ext(int ext, int stream, int& threads)
{
    threads = G::THREADS;
    if (ext == EXT_SEXTIC) return of_stream<T, G, EXT_SEXTIC>(stream);
    if (ext == EXT_POT) return of_stream<T, G, EXT_POT>(stream);
    return of_stream<T, G, EXT_NONE>(stream);
}

template <> const void* step_kernel_of<float>(int variant, int ext, int stream, int& threads)
{
    int v = 0;
#define SKYR_CASE(a, b, c, d, ...) \
    if (variant == v) return of_ext<float, Geo<a, b, c, d>>(ext, stream, threads); \
    ++v;
    SKYR_SHAPES_F32(SKYR_CASE)
#undef SKYR_CASE
    threads = 0;
    return nullptr;
}

}  // namespace skyr

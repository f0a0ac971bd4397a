// Shared by the translation units of the C ABI: the lookup-table handle and the argument checks that several
// entry points repeat.  Declarations and the contract of every entry point are in include/fb4.h.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <cstdlib>

#include "../../include/fb4.h"
#include "fb4_tables.hpp"

struct fb4_luts {
    uint8_t host_blob[fb4::kBlobBytes];
    uint8_t* dev_blob;   // the table blob, then the two GeLU tables
    int n_dialects;
    int device;
    int n_cu;
};

namespace fb4 {

inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

// Kernel launches.  The runtime keeps up to 112 bytes of kernel arguments with the launch itself and allocates for more, and the
// launch syntax stores the configuration aside and fetches it back: an empty kernel, one launch behind the other from the host, takes
// 3.42 us with 224 bytes in that syntax, 3.25 in one call, 2.64 with 16 to 112 bytes in one call (116 bytes: 3.25; 2.25 to 2.8 from machine
// to machine and process to process).  So no kernel here
// takes more, and a kernel that needs its grid's or workgroup's size, 256 bytes of implicit arguments, gets it passed.  fb4_quantize of
// 300 x 1152, 40 calls in a row: 3.35 us of the host per call with 192 bytes and the syntax, 2.83 so (over thousands of calls the
// kernels' own 3.4 us one behind the other are the longer part: 3.65 to 3.55).
constexpr size_t kMaxArgumentBytes = 112;

template <typename... P>
constexpr size_t argument_bytes()
{
    size_t n = 0;
    ((n = (n + alignof(P) - 1) / alignof(P) * alignof(P) + sizeof(P)), ...);
    return n;
}
template <typename T> struct same_type { typedef T type; };   // (arguments convert to the kernel's types)

// (an error stays for hipGetLastError)
template <typename... P>
inline void launch(void (*kernel)(P...), dim3 grid, dim3 block, size_t lds_bytes, hipStream_t stream, typename same_type<P>::type... values)
{
    static_assert(argument_bytes<P...>() <= kMaxArgumentBytes, "more arguments than a launch carries by itself");
    void* arguments[] = {const_cast<void*>(static_cast<const void*>(&values))...};
    (void)hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, arguments, lds_bytes, stream);
}

// The tables live on the device the handle was built on: launching from another current device would hand
// the kernels a foreign pointer.
inline int check_device(const fb4_luts* l)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return FB4_ERR_HIP;
    }
    return dev == l->device ? FB4_OK : FB4_ERR_INVALID_ARG;
}

inline int check_opts(const fb4_opts* o)
{
    if (!o) return FB4_ERR_INVALID_ARG;
    if (o->selector != FB4_SEL_SSE && o->selector != FB4_SEL_LUT) return FB4_ERR_INVALID_ARG;
    if (o->flags & ~FB4_FLAG_TWO_STAGE) return FB4_ERR_INVALID_ARG;
    if (o->block != 32 && o->block != 16) return FB4_ERR_INVALID_ARG;
    if (o->selector == FB4_SEL_LUT &&
        ((o->num_groups != 8 && o->num_groups != 16 && o->num_groups != 32) || o->num_groups > o->block))
        return FB4_ERR_INVALID_ARG;
    return FB4_OK;
}

// Shared validation of the tensor arguments of the quantizing calls.
inline int check_tensor(const fb4_luts* l, const fb4_opts* o, const void* x, int64_t rows, int64_t cols,
                        int64_t row_stride, const void* codes, const void* meta)
{
    if (!l) return FB4_ERR_INVALID_ARG;
    int rc = check_opts(o);
    if (rc != FB4_OK) return rc;
    if (rows < 0 || cols < 0 || row_stride < cols) return FB4_ERR_INVALID_ARG;
    if (cols % o->block) return FB4_ERR_UNSUPPORTED;
    if (rows == 0 || cols == 0) return FB4_OK;
    if (!x || !codes || !meta) return FB4_ERR_INVALID_ARG;
    if (!aligned(x, 16) || (row_stride % 8) || !aligned(codes, 4) || !aligned(meta, 2)) return FB4_ERR_UNSUPPORTED;
    return FB4_OK;
}

}  // namespace fb4

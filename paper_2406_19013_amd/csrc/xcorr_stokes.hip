// Full-Stokes visibilities of dual-polarisation feeds from the input
// visibilities (paper Section 1: full-Stokes output of 96 dual-polarisation
// feeds; Section 3.3: X north-south, Y east-west).  Input 2 f + pol is feed
// f's polarisation pol (0 = X, 1 = Y); for feeds a >= b
//   XX = V(2a, 2b), YY = V(2a+1, 2b+1), XY = V(2a, 2b+1), YX = V(2a+1, 2b)
// (for a = b, XY = conj V(2a+1, 2a), the stored entry), and
//   I = XX + YY, Q = XX - YY, U = XY + YX, V = -i (XY - YX)
// in exact int64 arithmetic.  Four lanes per (channel, feed pair), one for
// each Stokes parameter: a lane reads the two int32 (re, im) products its
// parameter combines and writes 16 bytes, so that a wave's loads and its store
// are contiguous (256, 256 and 1024 bytes).  HBM-bound: 192 inputs x 1024
// channels read 152 MB and write 305 MB; one lane per pair with four 16-byte
// stores 64 bytes apart took 125 us (3.7 TB/s), this takes 78.5 (5.8 TB/s).
#include "xcorr.h"
#include "xcorr_internal.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>

namespace xc {
namespace {

constexpr int kStokesChans = 4;   // channels per thread (the pair's indices are formed once)
// A launch counts the threads of each grid dimension in 32 bits and drops the
// rest without an error: a row of the grid is at most this many work-groups,
// and further ones go along z.
constexpr int64_t kStokesRow = 1 << 22;

__global__ __launch_bounds__(256) void xc_stokes_kernel(const int2 *__restrict__ vis, int F, int64_t P, int64_t Pf,
                                                        longlong2 *__restrict__ out)
{
    const int64_t e = ((int64_t)blockIdx.z * gridDim.x + blockIdx.x) * 256 + threadIdx.x;   // (feed pair, parameter)
    const int64_t q = e >> 2;
    const int s = (int)(e & 3);
    if (q >= Pf)
        return;
    // feed pair q = a (a + 1) / 2 + b, b <= a
    int64_t a = (int64_t)((sqrtf(8.0f * (float)q + 1.0f) - 1.0f) * 0.5f);
    while (a * (a + 1) / 2 > q)
        --a;
    while ((a + 1) * (a + 2) / 2 <= q)
        ++a;
    const int64_t b = q - a * (a + 1) / 2;
    const int64_t r0 = (2 * a) * (2 * a + 1) / 2 + 2 * b, r1 = (2 * a + 1) * (2 * a + 2) / 2 + 2 * b;   // rows 2a, 2a + 1
    // I, Q: x = XX, y = YY; U, V: x = XY (for a = b the conjugate of the stored
    // YX), y = YX
    const bool cross = s >= 2, conj = cross && a == b;
    const int64_t px = !cross ? r0 : conj ? r1 : r0 + 1, py = cross ? r1 : r1 + 1;
    const int64_t sx = conj ? -1 : 1;              // sign of x's imaginary part
    const int64_t sy = s == 0 || s == 2 ? 1 : -1;  // sign of y
#pragma unroll
    for (int k = 0; k < kStokesChans; ++k) {
        const int64_t f = (int64_t)blockIdx.y * kStokesChans + k;
        if (f >= F)
            break;
        const int2 x = vis[f * P + px], y = vis[f * P + py];
        const long long re = x.x + sy * y.x, im = sx * x.y + sy * y.y;
        // V = -i (XY - YX)
        out[(f * Pf + q) * 4 + s] = s == 3 ? make_longlong2(im, -re) : make_longlong2(re, im);
    }
}

}  // namespace
}  // namespace xc

extern "C" int xcorr_stokes(const void *d_vis, int32_t n_inputs, int32_t n_chans, void *d_out, void *stream)
{
    using namespace xc;
    if (!d_vis || !d_out || n_inputs < 2 || n_inputs % 2 || n_chans < 1 || n_chans > 65535 ||
        (uintptr_t)d_vis % 8 || (uintptr_t)d_out % 16)
        return XCORR_E_INVAL;
    const int nf = n_inputs / 2;
    const int64_t P = (int64_t)n_inputs * (n_inputs + 1) / 2, Pf = (int64_t)nf * (nf + 1) / 2;
    const int64_t blocks = (4 * Pf + 255) / 256, row = std::min(blocks, kStokesRow), rows = (blocks + row - 1) / row;
    if (rows > 65535)
        return XCORR_E_INVAL;
    hipLaunchKernelGGL(xc_stokes_kernel,
                       dim3((unsigned)row, (unsigned)((n_chans + kStokesChans - 1) / kStokesChans), (unsigned)rows), dim3(256), 0,
                       reinterpret_cast<hipStream_t>(stream), (const int2 *)d_vis, n_chans, P, Pf, (longlong2 *)d_out);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? XCORR_OK : api_error(XCORR_E_HIP, std::string("stokes launch: ") + hipGetErrorString(e));
}

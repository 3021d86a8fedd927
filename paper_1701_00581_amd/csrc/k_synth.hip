// Inverse transform of modulus and phase, and the mosaic (Section 3.2).
//
// k_synth: one workgroup per patch builds the Hermitian spectrum
// filter(w) |O(w)| e(w) on W in LDS and inverts it with the forward FFT:
// Re IFFT(X) = Re FFT(conj X) / N^2.  The mean level removed at ingest is
// put back under the taper.
// k_mosaic: each thread gathers, for its pixels of one image, the subimages
// covering them, out = sum r_k / sum taper_k (0 where < 1e-3).
#include "device_common.hpp"
#include "kernels.hpp"

namespace nvsm {

namespace {

constexpr int NT = 256;
// The tile (133 KB at N = 128) allows one k_synth workgroup per CU there, so
// it runs 16 waves to hide the latency of its LDS passes: 205 us for 1287
// patches with 4 waves, 127 with 8, 101 with 16 (the values do not depend
// on the thread count).
template <int N> constexpr int synth_threads() { return N == 128 ? 1024 : 256; }

template <int N>
__global__ __launch_bounds__(synth_threads<N>()) void k_synth(int nW, const int *__restrict__ Wxy,
                                              const double *__restrict__ amp,
                                              const double2 *__restrict__ phasor,
                                              const float *__restrict__ filt, const float *__restrict__ mu,
                                              int window, const float *__restrict__ hann,
                                              const float2 *__restrict__ twiddle,
                                              float *__restrict__ patches) {
    constexpr int P = LdsPitch<N>::v, ST = synth_threads<N>();
    __shared__ float2 z[N * P];
    __shared__ float2 tw[N];
    __shared__ float hw[N];
    const int patch = blockIdx.x, tid = threadIdx.x;
    for (int i = tid; i < N; i += ST) {
        tw[i] = twiddle[i];
        hw[i] = window ? hann[i] : 1.0f;
    }
    for (int j = tid; j < N * P; j += ST) z[j] = make_float2(0.f, 0.f);
    __syncthreads();
    for (int i = tid; i < nW; i += ST) {
        const int wx = Wxy[2 * i], wy = Wxy[2 * i + 1];
        const float a = (float)amp[(size_t)patch * nW + i] * (filt ? filt[i] : 1.0f);
        const double2 e = phasor[(size_t)patch * nW + i];
        const float2 v = make_float2(a * (float)e.x, a * (float)e.y);
        z[(wy & (N - 1)) * P + (wx & (N - 1))] = conjf2(v);
        z[((-wy) & (N - 1)) * P + ((-wx) & (N - 1))] = v;
    }
    __syncthreads();
    fft2d_lds_inline<N, ST>(z, tw);
    const float m = mu[patch];
    constexpr float inv = 1.0f / (float)(N * N);
    float *out = patches + (size_t)patch * N * N;
    for (int j = tid; j < N * N; j += ST) {
        const int y = j / N, x = j % N;
        out[j] = z[fft_pos<N>(y) * P + fft_pos<N>(x)].x * inv + m * (hw[y] * hw[x]);
    }
}

// PX pixels per thread, x .. x + PX - 1 of one image row, the threads of an
// image in row order over workgroups of its own (BurstDesc::mosaic0), so that
// images of any width, alone and beside others, leave no lanes idle.  PX = 4
// needs tile origins and sizes in x that are multiples of 4: the four pixels
// then lie in the same subimages and are loaded as one vector, and the row and
// tile arithmetic is done once for four (2560 x 2160: 58 us with one pixel and a
// 64-bit division per thread, 26 now.  A workgroup per row of the launch's
// widest image took 26 as well there, but 4.6 ms instead of 0.07 for fifteen
// images 64 pixels wide beside one of 16384).
template <int PX>
__global__ __launch_bounds__(NT) void k_mosaic(const BurstTable bt, const float *__restrict__ all_patches, int N,
                                               int stride, int window, const float *__restrict__ hann) {
    const BurstDesc &bd = bt.b[burst_of(bt, blockIdx.x, [](const BurstDesc &d) { return (int64_t)d.mosaic0; })];
    const int H = bd.H, W = bd.W, ny = bd.ny, nx = bd.nx;
    const unsigned t = (blockIdx.x - bd.mosaic0) * NT + threadIdx.x, row = (unsigned)W / PX;   // (t < H W + NT < 2^32)
    const int y = (int)(t / row), x = (int)(t % row) * PX;
    if (y >= H) return;
    const float *patches = all_patches + (size_t)bd.patch0 * N * N;
    float num[PX], dx[PX], dy = 0.f;
#pragma unroll
    for (int i = 0; i < PX; ++i) num[i] = dx[i] = 0.f;
    const int ky0 = y >= N ? (y - N) / stride : 0;
    const int kx0 = x >= N ? (x - N) / stride : 0;
    for (int kx = kx0; kx < nx; ++kx) {
        const int ox = min(kx * stride, W - N);
        if (ox > x) break;
        if (x < ox + N) {
#pragma unroll
            for (int i = 0; i < PX; ++i) dx[i] += window ? hann[x - ox + i] : 1.0f;
        }
    }
    for (int ky = ky0; ky < ny; ++ky) {
        const int oy = min(ky * stride, H - N);
        if (oy > y) break;
        if (y >= oy + N) continue;
        dy += window ? hann[y - oy] : 1.0f;
        for (int kx = kx0; kx < nx; ++kx) {
            const int ox = min(kx * stride, W - N);
            if (ox > x) break;
            if (x >= ox + N) continue;
            const float *r = patches + ((size_t)(ky * nx + kx) * N + (y - oy)) * N + (x - ox);
            if constexpr (PX == 4) {
                const float4 v = *(const float4 *)r;
                num[0] += v.x; num[1] += v.y; num[2] += v.z; num[3] += v.w;
            } else {
                num[0] += *r;
            }
        }
    }
    float *out = bd.out + (size_t)y * W + x;
#pragma unroll
    for (int i = 0; i < PX; ++i) {
        const float den = dy * dx[i];
        num[i] = den >= 1e-3f ? num[i] / den : 0.f;
        out[i] = num[i];
    }
}

template <int N>
hipError_t launch_synth_t(const SynthArgs &a, hipStream_t st) {
    hipLaunchKernelGGL(k_synth<N>, dim3(a.bt.patches), dim3(synth_threads<N>()), 0, st, a.nW, a.Wxy, a.amp, a.phasor, a.filt,
                       a.mu, a.window, a.hann, a.twiddle, a.patch_buf);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !a.mosaic) return e;
    // four pixels per thread where every tile starts and every image ends at a
    // multiple of 4 (and the subimages are aligned for it)
    BurstTable bt = a.bt;
    bool quad = a.stride % 4 == 0 && (uintptr_t)a.patch_buf % 16 == 0;
    for (int i = 0; i < bt.nb; ++i) quad = quad && bt.b[i].W % 4 == 0;
    int wgs = 0;
    for (int i = 0; i < bt.nb; ++i) {
        bt.b[i].mosaic0 = wgs;
        wgs += (int)(((int64_t)bt.b[i].H * bt.b[i].W / (quad ? 4 : 1) + NT - 1) / NT);
    }
    const dim3 grid(wgs);
    if (quad)
        hipLaunchKernelGGL(k_mosaic<4>, grid, dim3(NT), 0, st, bt, a.patch_buf, N, a.stride, a.window, a.hann);
    else
        hipLaunchKernelGGL(k_mosaic<1>, grid, dim3(NT), 0, st, bt, a.patch_buf, N, a.stride, a.window, a.hann);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_synth(const SynthArgs &a, hipStream_t st) {
    if (a.bt.patches == 0) return hipSuccess;
    return a.N == 128 ? launch_synth_t<128>(a, st) : launch_synth_t<64>(a, st);
}

}  // namespace nvsm

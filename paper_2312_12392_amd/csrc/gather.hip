// Screen-space variant of recursive camera painting.
//
// With the eye fixed (Section 3's colour mapping has V_e = 0), the rendered
// image already holds most directions a displaced camera would see, so a
// pass reduces to fetching each pixel's new colour from a position displaced
// by its own red and green (Section 6).  Positions outside the image follow
// an edge rule: clamp, wrap or mirror (Section 6.1).
//
// An image is 12 B per pixel, written once per pass and read at least once by
// the next; what a pass can do without is the rest:
//  - A launch runs up to three passes.  Pass k's colour of a pixel is pass
//    k - 1's colour of another, I_k(p) = I_{k-1}(s(I_{k-1}(p))), so a thread
//    computes its pixels' next images from the launch's input alone: 1, 2, 4
//    fetches of it for the first, second and third image.  They lie within a
//    few displacements of the pixel and hit the caches.  The images in between
//    are not read again, so they are stored past the caches, which then still
//    hold the last one for the next launch.
//  - Each XCD takes one contiguous band of the image (workgroups go to the
//    XCDs round robin), so that a row is read into one L2, not into all eight.
//  - The fetches are dependent loads; a thread has several pixels' in flight.
// 3840 x 2160, 5 passes, 6 px, mirror: 268 us with one pass per launch in row
// order, 222 in bands, 181 with two passes per launch (0.64 of what a copy of
// the 597 MB would reach); stored through the caches 236.  Three per launch
// were slower from 10 px on (247 against 228 us for 6 passes).
#include "rcp_internal.hpp"

namespace rcp {
namespace {

constexpr int kB = 256;
constexpr int kTileW = 64, kTileH = kB / kTileW;   // pixels of a workgroup: a wave is part of one row
constexpr int kXcds = 8;

struct GatherArgs {
    const float* in;     // the image the first pass reads
    float* out;          // the first pass's image; the next ones follow
    int W, H;
    uint32_t tiles_x, n_tiles;   // tiles_x 0: workgroups take the pixels in a row, whatever the image's width
    uint32_t band;       // workgroups of an XCD's band; 0: workgroups in row order
    float smudge;
    int edge, centred;
};

__device__ inline int edge_index(int i, int n, int edge) {
    if ((uint32_t)i < (uint32_t)n) return i;
    if (edge == RCP_EDGE_CLAMP) return i < 0 ? 0 : n - 1;
    if (edge == RCP_EDGE_WRAP) {
        const int m = i % n;
        return m < 0 ? m + n : m;
    }
    // mirror about the border, the border pixel repeated: -1 -> 0, n -> n - 1
    const int p = 2 * n;
    int m = i % p;
    if (m < 0) m += p;
    return m < n ? m : p - 1 - m;
}

struct Colour {
    float r, g, b;
};

// The pixels that pixels (x, y) of colours c take their next colours from.
template <int N>
__device__ inline void source(const GatherArgs& a, const Colour (&c)[N], const int (&x)[N], const int (&y)[N], int (&sx)[N],
                              int (&sy)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
        // red moves the sample right, green up (towards row 0)
        const float mr = a.centred ? 2.0f * c[i].r - 1.0f : c[i].r;
        const float mg = a.centred ? 2.0f * c[i].g - 1.0f : c[i].g;
        const float px = ((float)x[i] + 0.5f) + mr * a.smudge;
        const float py = ((float)y[i] + 0.5f) - mg * a.smudge;
        sx[i] = edge_index((int)floorf(px), a.W, a.edge);
        sy[i] = edge_index((int)floorf(py), a.H, a.edge);
    }
}

// Image L passes after the launch's input, at pixels (x, y).
template <int L, int N>
__device__ inline void image(const GatherArgs& a, const int (&x)[N], const int (&y)[N], Colour (&c)[N]) {
    if constexpr (L == 0) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const float* p = a.in + 3 * ((size_t)y[i] * (size_t)a.W + (size_t)x[i]);
            c[i] = Colour{p[0], p[1], p[2]};
        }
    } else {
        int sx[N], sy[N];
        image<L - 1, N>(a, x, y, c);
        source<N>(a, c, x, y, sx, sy);
        image<L - 1, N>(a, sx, sy, c);
    }
}

// Images L, L + 1 .. F of the first `live` of pixels (x, y), from their images
// L - 1.  STREAM: those before F bypass the caches.
template <int L, int F, int N, bool STREAM>
__device__ inline void passes(const GatherArgs& a, Colour (&c)[N], const int (&x)[N], const int (&y)[N], int live) {
    int sx[N], sy[N];
    source<N>(a, c, x, y, sx, sy);
    image<L - 1, N>(a, sx, sy, c);
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (i < live) {
            float* q = a.out + 3 * ((size_t)(L - 1) * (size_t)a.H * (size_t)a.W + (size_t)y[i] * (size_t)a.W + (size_t)x[i]);
            if constexpr (L < F && STREAM) {
                __builtin_nontemporal_store(c[i].r, q);
                __builtin_nontemporal_store(c[i].g, q + 1);
                __builtin_nontemporal_store(c[i].b, q + 2);
            } else {
                q[0] = c[i].r;
                q[1] = c[i].g;
                q[2] = c[i].b;
            }
        }
    if constexpr (L < F) passes<L + 1, F, N, STREAM>(a, c, x, y, live);
}

template <int F, int N, bool STREAM>
__global__ __launch_bounds__(kB) void k_gather(GatherArgs a) {
    const uint32_t tile = a.band ? (blockIdx.x % kXcds) * a.band + blockIdx.x / kXcds : blockIdx.x;
    if (tile >= a.n_tiles) return;
    int x[N], y[N], live = 0;
    if (a.tiles_x != 0u) {
        const int x0 = (int)(tile % a.tiles_x) * kTileW + (int)(threadIdx.x % kTileW);
        const int y0 = (int)(tile / a.tiles_x) * kTileH * N + (int)(threadIdx.x / kTileW);
        if (x0 >= a.W || y0 >= a.H) return;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            x[i] = x0;
            y[i] = min(y0 + i * kTileH, a.H - 1);
            live += y0 + i * kTileH < a.H ? 1 : 0;
        }
    } else {
        const uint32_t P = (uint32_t)a.W * (uint32_t)a.H, p0 = tile * (uint32_t)(kB * N) + threadIdx.x;
        if (p0 >= P) return;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const uint32_t p = min(p0 + (uint32_t)(i * kB), P - 1u);
            y[i] = (int)(p / (uint32_t)a.W);
            x[i] = (int)(p - (uint32_t)y[i] * (uint32_t)a.W);
            live += p0 + (uint32_t)(i * kB) < P ? 1 : 0;
        }
    }
    Colour c[N];
    image<0, N>(a, x, y, c);
    passes<1, F, N, STREAM>(a, c, x, y, live);
}

}  // namespace

namespace {

template <int F, int N, bool STREAM>
rcp_status launch(GatherArgs a, bool bands, hipStream_t stream) {
    // Tiles 64 pixels wide, a wave per row, but not where an eighth of their lanes
    // or more would lie beyond the image's side: such narrow images are taken
    // pixel by pixel (5 passes, 6 px, us, tiles / in a row: 65 x 200,000 540 / 336, 1
    // x 4M 2163 / 65, 9 x 4M 2481 / 783).
    a.tiles_x = (uint32_t)((a.W + kTileW - 1) / kTileW);
    a.n_tiles = a.tiles_x * (uint32_t)((a.H + kTileH * N - 1) / (kTileH * N));
    if (8 * ((int)a.tiles_x * kTileW - a.W) >= a.W) {
        a.tiles_x = 0u;
        a.n_tiles = ((uint32_t)a.W * (uint32_t)a.H + (uint32_t)(kB * N) - 1u) / (uint32_t)(kB * N);
    }
    a.band = bands ? (a.n_tiles + kXcds - 1) / kXcds : 0u;
    hipLaunchKernelGGL((k_gather<F, N, STREAM>), dim3(bands ? a.band * kXcds : a.n_tiles), dim3(kB), 0, stream, a);
    RCP_CHECK_LAUNCH();
    return RCP_OK;
}

}  // namespace

rcp_status gather_passes(const float* in, int W, int H, int n, float smudge, int edge, int centred, float* out,
                         hipStream_t stream) {
    const size_t P = (size_t)W * (size_t)H;
    GatherArgs a{};
    a.W = W;
    a.H = H;
    a.smudge = smudge;
    a.edge = edge;
    a.centred = centred;
    // The rows a pixel's sources lie in.  Two passes per launch while they
    // stay well inside an XCD's 4 MB L2 (3840 wide: 18 px 255 against 299 us
    // for one pass per launch, 64 px 431 against 362); bands per XCD while
    // they are not far beyond it (64 px 366 against 391 in row order, 1920
    // wide 200 px 96 against 113; 3840 wide 400 px 550 against 480).  Images
    // that fit the L2s are bound by their launches: three passes each
    // (481 x 271, 8 passes: 16 against 26 us).
    const double window = (2.0 * (double)smudge + 1.0) * (double)W * 12.0;
    const bool small = P <= 400000, two = window <= 2e6, bands = window <= 16e6 || small;
    for (int k = 0; k < n;) {
        a.in = k == 0 ? in : out + (size_t)(k - 1) * P * 3;
        a.out = out + (size_t)k * P * 3;
        const int left = n - k;
        rcp_status st;
        int f = 1;
        if (small) {
            f = left < 3 ? left : 3;
            st = f == 3 ? launch<3, 1, false>(a, bands, stream)
                        : (f == 2 ? launch<2, 1, false>(a, bands, stream) : launch<1, 1, false>(a, bands, stream));
        } else if (two && left >= 2) {
            f = 2;
            st = launch<2, 4, true>(a, bands, stream);
        } else {
            st = bands ? launch<1, 2, false>(a, true, stream) : launch<1, 1, false>(a, false, stream);
        }
        if (st != RCP_OK) return st;
        k += f;
    }
    return RCP_OK;
}

}  // namespace rcp

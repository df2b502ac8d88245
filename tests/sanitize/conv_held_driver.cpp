// Plans of conv_held_kernel (choose_held), walked on the host: the kernel's LDS entries, shifts, rows and strips in its own steps, without its arithmetic.
// For every stored output pixel the entries its nine taps read hold the pixels they should, or zeros, no read leaves the LDS, copies and
// kept sums fit their parts of it, and every output pixel is stored once.  Built from the library's host code with empty tables of
// tile kernels, under the host sanitizers.  Exit code 0 = pass.
#include "ucl_api.hip"

#include <algorithm>
#include <set>

using namespace ucl;

static int fails = 0;
#define EXPECT(c, ...) do { if (!(c) && ++fails < 20) { std::fprintf(stderr, "line %d: %s: ", __LINE__, #c); std::fprintf(stderr, __VA_ARGS__); std::fprintf(stderr, "\n"); } } while (0)

struct Geom { int mode, stride, n, H, W, C, N; };
constexpr int64_t kUnset = -2, kZero = -1;

static int kernel_divide(int x, float rcp) { return (int)(((float)x + 0.5f) * rcp); }

// (bands: how many of the first, middle and last bands are walked; all of them: every output is counted)
static bool walk(const Geom &g, int most_bands, bool may_stay = false) {
    const int P = (g.H - 1) / g.stride + 1, Q = (g.W - 1) / g.stride + 1;
    Launch L;
    L.mode = g.mode; L.dt = 0; L.dtD = UCL_BF16; L.N = g.N; L.M = (int64_t)g.n * P * Q; L.K = 9ll * g.C;
    held_launch(L, g.n, g.H, g.W, P, Q, g.C, 3, 3, 1, 1, g.stride, g.stride, 1, 1);
    EXPECT(may_stay || L.held_stride == g.stride, "%dx%dx%dx%d->%d", g.n, g.H, g.W, g.C, g.N);
    if (!L.held_stride) return false;
    EXPECT(L.gathered < (1ll << 31) && L.M * L.N * 2 < (1ll << 31), "offsets of 32 bits");
    for (int residual = 0; residual < 2; ++residual) {
        const HeldPlan h = choose_held(L, residual != 0);
        char what[160];
        std::snprintf(what, sizeof what, "mode %d stride %d %dx%dx%dx%d -> %d: kg %d ng %d R %d split %d passes %d", g.mode, g.stride, g.n, g.H, g.W, g.C, g.N, h.kg, h.ng, h.R, h.strip_split, h.passes);
        if (h.R == 0) continue;
        // ---- what launch_conv_held_mode is built for
        static const std::set<int> built = {12, 10, 20, 18, 17, 34, 33};
        EXPECT(h.passes == 1 ? built.count(h.kg * 8 + h.ng) : g.mode == 3 && h.kg == 4 && h.ng <= 2, "%s", what);
        const int MG = 8 / (h.kg * h.ng), ST = g.stride, pitch = h.pitch, line = ST * pitch, Pp = P + 1;
        const bool multi = h.passes > 1;
        EXPECT(h.strip_split <= MG && (h.strip_split & (h.strip_split - 1)) == 0 && pitch % 16 == 0 && pitch > Q && h.passes * 64 * h.kg >= g.C, "%s", what);
        EXPECT((int64_t)h.bands * h.R >= h.rows && (int64_t)(h.bands - 1) * h.R < h.rows && h.tiles_n * 32 * h.ng >= g.N, "%s", what);
        const int64_t plane = held_plane_bytes(ST, h.R, pitch);
        EXPECT(plane * h.kg + h.keep_bytes <= held_patch_capacity(h.kg, h.ng) && plane % 1024 == 0, "%s: %lld + %d", what, (long long)plane * h.kg, h.keep_bytes);
        const int sgroups = h.strip_split, rgroups = MG / sgroups, per = held_rows_of_wave(h.R, rgroups, h.kg, multi), strip_rounds = (h.strips + sgroups - 1) / sgroups;
        EXPECT(h.keep_bytes == (multi ? (per * strip_rounds + 2) * 512 * (8 / h.kg) * 4 : 0), "%s", what);
        // ---- workgroup numbers and row numbers by their reciprocals
        for (int d : {h.bands, h.tiles_n}) {
            const float rcp = 1.f / (float)d;
            const int grid = h.bands * h.tiles_n;
            for (int t = 0; t < grid; t += grid / 997 + 1) EXPECT(kernel_divide(t, rcp) == t / d, "%s: %d / %d", what, t, d);
            EXPECT(kernel_divide(grid - 1, rcp) == (grid - 1) / d, "%s", what);
        }
        const bool all = h.bands <= most_bands;
        std::vector<char> stored(all ? (size_t)L.M : 0);
        std::vector<int64_t> lds;
        for (int b = 0; b < (all ? h.bands : most_bands); ++b) {
            const int band = all || b < most_bands / 3 ? b : b < 2 * (most_bands / 3) ? h.bands / 2 + b : h.bands - (most_bands - b);
            if (band >= h.bands) continue;
            const int row0 = band * h.R;
            // ---- copies, one plane (the others differ in their channels only)
            lds.assign((size_t)(plane / 128), kUnset);
            const int img_first = kernel_divide(row0, 1.f / (float)Pp);
            EXPECT(img_first == row0 / Pp, "%s", what);
            const int rows_in = ST * h.R + 3 - ST;
            for (int i = 0; i < rows_in; ++i) {
                const int at_row = ST * (row0 % Pp) + i, im0 = row0 / Pp + at_row / (ST * Pp), hh = at_row % (ST * Pp) - 1;
                for (int even = 0; even < ST; ++even)
                    for (int col = 0; col < pitch; ++col) {
                        int e = col, im = im0 * h.pair;
                        if (h.pair == 2) {
                            const bool second = ST == 1 ? col > 8 : col >= 8;
                            im += second;
                            e = second ? col - 8 : col;
                        }
                        const int w = ST == 1 ? e - 1 : 2 * e - 1 + even;
                        const bool in = hh >= 0 && hh < g.H && w >= 0 && w < g.W && im < g.n;
                        lds[(size_t)(i * line + even * pitch + col)] = in ? ((int64_t)im * g.H + hh) * g.W + w : kZero;
                    }
            }
            if (ST == 1)
                for (int e = 0; e < 8; ++e) lds[(size_t)((h.R + 2) * pitch + e)] = kZero;
            // ---- the waves of one tile of filters
            const int64_t lds_entries = (kLdsBytesPerCU - (h.kg - 1) * plane) / 128;
            for (int mg = 0; mg < MG; ++mg) {
                const int ms = mg & (sgroups - 1), mr = mg / sgroups, first = mr * per;
                if (h.kg == 1 && first >= h.R) continue;
                const int own = h.R - first < per ? h.R - first : per;
                const int left = own < h.rows - row0 - first ? own : h.rows - row0 - first;
                const int img0 = kernel_divide(row0 + first, 1.f / (float)Pp), p0 = row0 + first - img0 * Pp;
                int64_t at = (int64_t)(first < h.R ? first : 0) * ST * line + ms * 16, now = at;     // entries: to be fetched next, in registers
                for (int sr = 0; sr < strip_rounds; ++sr) {
                    int img = img0, p = p0;
                    for (int o = 0; o < per; o += 2) {
                        const bool one = h.kg > 1 && !multi && o + 1 >= own;
                        const int ROWS = one ? 3 : ST + 3;
                        const int back = o + 2 < per ? (one ? 2 * ST - 2 : ST - 2) * line : sr + 1 < strip_rounds ? sgroups * 16 - (ST * (one ? o : per - 1) + 2) * line : 0;
                        int64_t row_at[5];
                        for (int j = 0; j < ROWS; ++j) {
                            row_at[j] = now;
                            at += j == ROWS - 1 ? back : line;
                            // (the farthest entry of a fragment: 15 + two columns, or the plane of even columns)
                            EXPECT(at >= 0 && at + (ST == 1 ? 17 : pitch + 15) < lds_entries && at + 16 < lds_entries, "%s: reads entry %lld", what, (long long)at);
                            now = at;
                        }
                        for (int k = 0, ik = img, pk = p; k < 2; ++k) {
                            // (a store out of range has its row in a scalar register all the same, behind a lane's offset of 2^31)
                            EXPECT(((int64_t)ik * h.pair * P + pk) * Q * g.N * 2 < (1ll << 31), "%s: row %d of image %d", what, pk, ik);
                            if (++pk == Pp) { pk = 0; ++ik; }
                        }
                        for (int k = 0; k < (one ? 1 : 2); ++k) {
                            const int ik = img + (p + k >= Pp), pk = p + k >= Pp ? 0 : p + k;
                            for (int l = 0; l < 16; ++l) {
                                int q = (sr * sgroups + ms) * 16 + l, im = ik * h.pair;
                                if (h.pair == 2) { q = l & 7; im += l >= 8; }
                                const int e_last = h.pair == 2 && l >= 8 ? g.n / 2 : g.n;
                                if (!(pk < P && o + k < left && ik < e_last && q < Q)) continue;
                                EXPECT(im < g.n, "%s: stores image %d", what, im);
                                if (all && im < g.n) EXPECT(!stored[((size_t)im * P + pk) * Q + q]++, "%s: stores %d %d %d twice", what, im, pk, q);
                                for (int tap = 0; tap < 9; ++tap) {
                                    const int r = tap / 3, s = tap % 3, y = pk * ST - 1 + r, x = q * ST - 1 + s;
                                    const int64_t want = y < 0 || y >= g.H || x < 0 || x >= g.W ? kZero : ((int64_t)im * g.H + y) * g.W + x;
                                    const int64_t e = row_at[ST * k + r] + l + (ST == 1 ? s : (s >> 1) + (s == 1 ? pitch : 0));
                                    EXPECT(e < (int64_t)lds.size() && lds[(size_t)e] == want, "%s: band %d, %d %d %d tap %d", what, band, im, pk, q, tap);
                                }
                            }
                        }
                        for (int k = 0; k < 2; ++k)
                            if (++p == Pp) { p = 0; ++img; }
                    }
                }
            }
        }
        if (all) EXPECT(std::count(stored.begin(), stored.end(), 1) == (std::ptrdiff_t)stored.size(), "%s: outputs are missing", what);
    }
    return true;
}

int main() {
    uint32_t x = 12345;
    auto upto = [&](int most) { x = x * 1664525u + 1013904223u; return 1 + (int)((x >> 8) % (uint32_t)most); };
    for (int i = 0; i < 600; ++i) {
        const int mode = 2 + (i % 3 == 0), stride = mode == 2 && i % 2 ? 2 : 1, side = i % 5 ? 40 : 9;
        walk({mode, stride, upto(i % 4 ? 6 : 60), upto(side), upto(side), 8 * upto(mode == 3 ? 130 : 32), 8 * upto(40)}, 1 << 30);
    }
    // wide rows: several strips per wave, one row per workgroup, up to the widest that is served; narrow and tall ones
    for (int w : {63, 64, 65, 80, 97, 112, 113, 128, 160, 200, 224, 225, 320, 511, 640, 1000, 1024})
        for (int c : {40, 64, 128, 256})
            for (int stride : {1, 2}) {
                walk({2, stride, 2, 1 + w / 4, w, c, 72}, 9);
                walk({2, stride, 37, 19, w, c, 136}, 9);
                if (stride == 1) walk({3, 1, 2, 1 + w / 4, w, 4 * c, 200}, 9);
            }
    for (int h : {1000, 100003, (1 << 20) - 2}) {
        walk({2, 1, 1, h, 3, 16, 32}, 30);
        walk({3, 1, 1, h, 9, 16, 8}, 30);
        walk({2, 2, 1, h, 7, 24, 32}, 30);
    }
    // outputs of nearly 2 GiB, whose last bands name rows behind them
    int served = 0;
    for (int p : {1, 2, 3, 5, 9, 17, 40, 100, 333})
        for (int q : {5, 7, 8, 30, 63, 100, 200})
            for (int n_out : {128, 512, 1000, 4096, 65536})
                for (int c : {8, 72, 136, 520}) {
                    const int64_t row = (int64_t)p * q * n_out, n = ((1ll << 30) - 1) / row;
                    for (int fewer : {0, 130 / p + 1})
                        if (n > fewer) served += walk({c > 256 ? 3 : 2, 1, (int)(n - fewer), p, q, c, n_out}, 6, true);
                }
    EXPECT(served > 100, "%d", served);
    if (fails) return 1;
    std::printf("held plans: ok\n");
    return 0;
}

// The quantised cell scan on the CPU: cell_scan.h compiled for the host, every read checked against the
// arrays it may touch, and what it visits against all pairs.  Prints the first fault and exits with 1.
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <random>
#include <vector>

#define __device__
#define __host__
#define __forceinline__ inline
#define __restrict__
using std::max;
using std::min;
struct float4 { float x, y, z, w; };
struct double4 { double x, y, z, w; };
struct uint2 { uint32_t x, y; };
struct int4 { int x, y, z, w; };
struct uint4 { uint32_t x, y, z, w; };
typedef void *hipStream_t, *hipEvent_t, *hipGraph_t, *hipGraphExec_t;
static uint2 make_uint2(uint32_t x, uint32_t y) { return {x, y}; }
static uint4 make_uint4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) { return {x, y, z, w}; }
static long long __double_as_longlong(double d) { long long v; memcpy(&v, &d, 8); return v; }
static float __int_as_float(int i) { float v; memcpy(&v, &i, 4); return v; }
static int __float_as_int(float f) { int v; memcpy(&v, &f, 4); return v; }
template <class V>
static int host_dot2(V a, V b, int c, bool) { return (int)((uint32_t)(a[0] * b[0]) + (uint32_t)(a[1] * b[1]) + (uint32_t)c); }
#define __builtin_amdgcn_sdot2 host_dot2
#define __builtin_amdgcn_ballot_w64(x) ((uint64_t)(x))
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_sqrtf sqrtf
#define __builtin_amdgcn_logf log2f
#define __builtin_amdgcn_cosf cosf

// the arrays the scan may read, and the copies it makes from them
static const char *span[2][2];
static void checked_copy(void* to, const void* from, size_t bytes) {
    const char* p = (const char*)from;
    for (auto& s : span)
        if (p >= s[0] && p + bytes <= s[1]) {
            memcpy(to, from, bytes);
            return;
        }
    printf("a read of %zu bytes lies %td bytes into the copy of %td bytes\n", bytes, p - span[1][0], span[1][1] - span[1][0]);
    exit(1);
}
#define __builtin_memcpy checked_copy
#include "cell_scan.h"

using namespace db;

template <int PARTS>
static void check(const Box& X, const std::vector<int>& start, const std::vector<uint2>& xq,
                  const std::vector<double4>& at, double reach) {
    const int n = (int)at.size();
    const uint32_t cut = quantised_cut(X, reach);
    if (!cut) {
        printf("the scan does not serve edge %g reach %g\n", X.L, reach);
        exit(1);
    }
    for (int i = 0; i < n; ++i) {
        std::vector<int> seen(n, 0), kept(n, 0);
        for (int part = 0; part < PARTS; ++part)
            scan_cells_quantised<PARTS>(X, start.data(), xq.data(), at[i], reach, part,
                                        [&](int p, int rem, const uint32_t (&r2)[4], const uint32_t (&)[4]) {
                for (int q = 0; q < 4 && q < rem; ++q) {
                    ++seen[p + q];
                    kept[p + q] += r2[q] < cut;
                }
            });
        for (int j = 0; j < n; ++j) {
            double d2 = 0.0;
            for (int c = 0; c < 3; ++c) {
                double d = (&at[j].x)[c] - (&at[i].x)[c];
                d -= X.L * std::round(d / X.L);
                d2 += d * d;
            }
            // kept: all within reach, none beyond it by more than the widening and the quanta's own error
            const double far = reach + 4.0 * X.L / 65536.0;
            if (seen[j] > 1 || (d2 < reach * reach && kept[j] != 1) || (d2 > far * far && kept[j])) {
                printf("parts %d, bead %d of %d, entry %d at %g (reach %g): visited %d times, kept %d\n", PARTS, i, n, j,
                       std::sqrt(d2), reach, seen[j], kept[j]);
                exit(1);
            }
        }
    }
}

// words of a position that a step has just left not finite or outside its box: read before the host stops, they may
// be anything but must not come from a conversion out of range (the build traps on one)
static void odd_positions() {
    Box X{};
    for (double L : {2.0, 125.99, 65536.0}) {
        X.L = L;
        for (float v : {NAN, INFINITY, -INFINITY, -1e30f, 1e30f, -0.25f, (float)L, (float)(2.0 * L)}) quantise(X, v, v, v, 3);
        const uint2 top = quantise(X, (float)L, 0.0f, (float)(0.5 * L), 0);
        if (top.x || (top.y & 0xFFFFu) != 32768u) {
            printf("the edge of a box of %g is not its origin: %x %x\n", L, top.x, top.y);
            exit(1);
        }
    }
}

int main() {
    odd_positions();
    std::mt19937_64 gen(5);
    auto uniform = [&](double a) { return a * (double)(gen() >> 11) * 0x1p-53; };
    for (int nc : {3, 4, 5, 9})
        for (int n : {1, 2, 3, 5, 17, 40, 300})
            for (int form = 0; form < 4; ++form) {
                Box X{};
                const double reach = 1.1;
                X.L = nc * reach * (1.0 + 0.2 * form / nc);
                X.hL = 0.5 * X.L;
                X.invL = 1.0 / X.L;
                X.nc = nc;
                X.cell_scale = nc / X.L;
                X.noff = 3;
                X.off[0] = -1;
                X.off[2] = 1;
                std::vector<double4> x(n);
                for (auto& b : x) {
                    b = {uniform(X.L), uniform(X.L), uniform(X.L), 0.0};
                    if (form == 1)   // all in the last cell: runs at the end of the list
                        b = {X.L - uniform(0.9), X.L - uniform(0.9), X.L - uniform(0.9), 0.0};
                    if (form == 2) b = {std::fmod(X.L - 0.5 + uniform(1.0), X.L), std::fmod(X.L - 0.5 + uniform(1.0), X.L), uniform(X.L), 0.0};
                }
                auto cell = [&](const double4& b) {
                    return (cell_coord(b.z, X.cell_scale, nc) * nc + cell_coord(b.y, X.cell_scale, nc)) * nc +
                           cell_coord(b.x, X.cell_scale, nc);
                };
                std::stable_sort(x.begin(), x.end(), [&](auto& a, auto& b) { return cell(a) < cell(b); });
                std::vector<int> start(nc * nc * nc + 1, 0);
                for (auto& b : x) ++start[cell(b) + 1];
                for (size_t k = 1; k < start.size(); ++k) start[k] += start[k - 1];
                std::vector<uint2> xq(n + DB_XS_PAD, uint2{0u, 0u});
                for (int k = 0; k < n; ++k) xq[k] = quantise(X, (float)x[k].x, (float)x[k].y, (float)x[k].z, 0);
                span[0][0] = (const char*)start.data();
                span[0][1] = (const char*)(start.data() + start.size());
                span[1][0] = (const char*)xq.data();
                span[1][1] = (const char*)(xq.data() + n + DB_XS_PAD);
                check<1>(X, start, xq, x, reach);
                check<4>(X, start, xq, x, reach);
            }
    printf("ok\n");
    return 0;
}

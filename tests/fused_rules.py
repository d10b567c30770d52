"""A small C++ program that asks the built library's host code how steps are launched (not
collected: no test_ prefix)."""
import os
import subprocess

import paper_2108_13241_amd as pkg

HERE = os.path.dirname(os.path.abspath(pkg.__file__))
CSRC = os.path.join(HERE, "csrc")

DRIVER = r"""
#include <cstdio>
#include <cstring>
#include "lbm3d_launch.h"
#include "lbm_launch.h"
#include "lbm.h"
using namespace lbm;
static char mem[2][64];
static float drag[1];
static DevState state(int nx, int ny, int dtype, int layout, int force, int alpha, int open,
                      int coll, double fluid)
{
    DevState s;
    s.nx = nx; s.ny = ny; s.pitch = (nx + 63) / 64 * 64; s.dtype = dtype; s.layout = layout;
    s.f[0] = mem[0]; s.f[1] = mem[1];
    s.gx = force ? 1e-6 : 0.0;
    s.alpha = alpha ? drag : nullptr;
    s.open = open; s.trt = coll == 1; s.mrt = coll == 2;
    s.fluid_frac = fluid; s.interior_frac = fluid;
    return s;
}
int main(int argc, char **argv)
{
    // lines of "nx ny dtype layout force drag open collision fluid left": the steps a launch
    // takes, and those of the next one of a call with `left` steps to go
    // "3": nx ny nz dtype aa force fluid, whether pairs of D3Q19 steps are taken
    if (argc > 1 && !strcmp(argv[1], "3")) {
        int v[6];
        double fluid;
        while (scanf("%d%d%d%d%d%d%lf", v, v + 1, v + 2, v + 3, v + 4, v + 5, &fluid) == 7) {
            lbm3::State3 s;
            s.nx = v[0]; s.ny = v[1]; s.nz = v[2]; s.pitch = (v[0] + 63) / 64 * 64;
            s.dtype = v[3]; s.aa = v[4]; s.gy = v[5] ? 1e-6 : 0.0;
            s.f[0] = mem[0]; s.f[1] = mem[1];
            s.fluid_frac = fluid; s.interior_frac = fluid == 1.0;
            printf("%d\n", lbm3::pair_supported3(s) ? 1 : 0);
        }
        return 0;
    }
    // "adjoint": nx ny dtype fluid, the reverse steps a launch takes
    if (argc > 1 && !strcmp(argv[1], "adjoint")) {
        int v[3];
        double fluid;
        while (scanf("%d%d%d%lf", v, v + 1, v + 2, &fluid) == 4)
            printf("%d\n", adjoint_square_steps(state(v[0], v[1], v[2], 0, 1, 1, 0, 0, fluid)));
        return 0;
    }
    if (argc > 1) {
        int v[8], left;
        double fluid;
        while (scanf("%d%d%d%d%d%d%d%d%lf%d", v, v + 1, v + 2, v + 3, v + 4, v + 5, v + 6, v + 7,
                     &fluid, &left) == 10) {
            DevState s = state(v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], fluid);
            printf("%d %d\n", max_fused_steps(s), next_steps(s, left));
        }
        return 0;
    }
    int bad = 0, seen = 0, fused = 0;
    auto check = [&](bool ok, const DevState &s, const char *what) {
        if (!ok && bad++ < 20)
            printf("%s: %dx%d dtype %d layout %d force %d drag %d open %d trt %d mrt %d fluid %g: %d\n",
                   what, s.nx, s.ny, s.dtype, s.layout, s.gx != 0, s.alpha != nullptr, s.open, s.trt,
                   s.mrt, s.fluid_frac, max_fused_steps(s));
    };
    const int sizes[][2] = {{1, 1}, {300, 200}, {540, 541}, {929, 931}, {1216, 912}, {2048, 2048},
                            {4096, 4096}, {40011, 9}, {7, 60000}};
    const double fluids[] = {0.05, 0.2, 0.35, 0.5, 0.7, 0.86, 0.97, 1.0};
    for (auto &n : sizes)
    for (int dtype = 0; dtype < 4; ++dtype)
    for (int layout = 0; layout < 4; ++layout)
    for (int v = 0; v < 24; ++v)
    for (double fluid : fluids) {
        DevState s = state(n[0], n[1], dtype, layout, v & 1, v & 2, (v >> 2) & 1, v >> 3, fluid);
        const bool sparse = layout == kTiled16 || layout == kIndirect;
        int square = 0;
        const int k = square_steps(s.nx, s.ny, dtype, square), most = max_fused_steps(s);
        const int limit = square ? k : strip_steps(dtype == kF64, dtype > kF32, sparse,
                                                   (v & 1) && !(v & 2), v & 2, (v >> 2) & 1,
                                                   s.trt, s.mrt);
        ++seen;
        fused += most > 1;
        for (int left = 1; left < 70; left += 1 + left / 12) {
            // every launch of a call is one the kernel takes, and they add up
            int n = left, launches = 0;
            for (; n > 0 && launches <= left; ++launches) {
                const int steps = next_steps(s, n);
                check(steps == 1 || (steps >= 2 && steps <= most && steps <= n), s, "next steps");
                n -= steps;
            }
            check(n == 0, s, "steps left");
            ThereAndBack p = there_and_back(s, left & ~1);
            const int64_t m = p.steps;
            check(p.launches % 2 == 0 && m % 2 == 0 && m <= left, s, "there and back");
            check(p.launches > 0 || most < 2 || left < 4 * most, s, "nothing borrowed");
            int64_t sum = 0;
            while (p.launches > 0 && sum <= left) {
                const int steps = p.next();
                check(steps >= 2 && steps % 2 == 0 && steps <= most, s, "even launch");
                sum += steps;
            }
            check(sum == m && p.steps == 0, s, "even steps");
        }
        check(most == 1 || (most >= 2 && most <= limit), s, "steps beyond the kernel's");
        // one more than the kernel takes, and any number where there is none
        check(launch_steps(s, 0, (layout == kDenseAA ? limit + 2 - limit % 2 : limit + 1)) ==
                  hipErrorInvalidValue, s, "accepted too many steps");
        check(launch_steps(s, 0, 1) == hipErrorInvalidValue, s, "accepted one step");
        if (limit == 0)
            check(launch_steps(s, 0, 2) == hipErrorInvalidValue, s, "accepted a missing variant");
        if (!square) {  // strips do not store every step
            s.every = 64;
            check(launch_steps(s, 0, 2) == hipErrorInvalidValue, s, "dropped the steps between");
        }
    }
    // D3Q19 pairs: force and walls that no kernel is compiled for
    int bad3 = 0;
    for (int n : {16, 64, 256})
    for (int dtype = 0; dtype < 4; ++dtype)
    for (int v = 0; v < 12; ++v)
    for (double interior : {0.0, 0.5, 1.0}) {
        lbm3::State3 s;
        s.nx = s.ny = s.nz = n; s.pitch = (n + 63) / 64 * 64; s.dtype = dtype;
        s.f[0] = mem[0]; s.f[1] = mem[1];
        s.gy = v & 1 ? 1e-6 : 0.0; s.aa = (v >> 1) & 1; s.trt = v >> 2 == 1; s.mrt = v >> 2 == 2;
        s.interior_frac = interior;
        const bool lost = dtype >= 2 ? ((v & 1) || interior != 1.0) : dtype == 1 && s.mrt && (v & 1);
        if (lbm3::pair_compiled3(s) == lost || (lbm3::pair_supported3(s) && lost) ||
            (lost && lbm3::launch_pair3(s, 0) != hipErrorInvalidValue))
            ++bad3;
    }
    printf("%d %d %d %d\n", seen, fused, bad, bad3);
    return bad || bad3;
}
"""


def build(directory):
    """The program, compiled against the built library: its path."""
    src = directory / "drv.cpp"
    src.write_text(DRIVER)
    exe = directory / "drv"
    pkg.load()
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(HERE, "..", "include"), "-I", CSRC, str(src), "-o", str(exe),
                    "-L", HERE, "-l:liblbm_hip.so", f"-Wl,-rpath,{HERE}",
                    "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib"], check=True)
    return str(exe)


def ask(exe, cases, what="ask"):
    """The program's answers, a list of numbers for each case (formats: in the program)."""
    text = "\n".join(" ".join(map(str, c)) for c in cases)
    r = subprocess.run([exe, what], input=text, capture_output=True, text=True, check=True)
    return [list(map(int, line.split())) for line in r.stdout.split("\n") if line]

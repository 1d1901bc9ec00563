// Functions of the kernels' own headers, run on the host: built with hipcc as
// HIP source; no device is used (test_host_kernels.py).
//   odd: doubles on stdin, to_f32_odd of each as float bits on stdout
//   alpha: nodes of 41 f_q and 41 f_eq,q - f_q (floats) on stdin, the entropic
//          path length of each in FP32 arithmetic on stdout, for 32-bit and for
//          16-bit storage
//   map: records of four 64-bit integers (remap, bytes of a q-block, of its
//        stride, of both buffers) on stdin, xcd_map of each on stdout (32-bit)
#include <cstdio>
#include <cstring>

#include "../paper_1909_08406_amd/csrc/kernels_io.hpp"

static int run_odd()
{
    double v;
    while (fread(&v, sizeof(v), 1, stdin) == 1) {
        const float t = lbm::to_f32_odd(v);
        fwrite(&t, sizeof(t), 1, stdout);
    }
    return 0;
}

static int run_alpha()
{
    float n[2 * lbm::Q];
    auto fd = [&](auto qc, float& f, float& d) {
        constexpr int q = decltype(qc)::value;
        f = n[q];
        d = n[lbm::Q + q];
    };
    while (fread(n, sizeof(n), 1, stdin) == 1) {
        const float a[2] = {lbm::path_length<float, false>(fd, fd, [] {}, [](auto) {}),
                            lbm::path_length<float, true>(fd, fd, [] {}, [](auto) {})};
        fwrite(a, sizeof(a), 1, stdout);
    }
    return 0;
}

static int run_map()
{
    uint64_t r[4];
    while (fread(r, sizeof(r), 1, stdin) == 1) {
        const uint32_t m = lbm::xcd_map(uint32_t(r[0]), r[1], r[2], r[3]);
        fwrite(&m, sizeof(m), 1, stdout);
    }
    return 0;
}

int main(int argc, char** argv)
{
    if (argc == 2 && !strcmp(argv[1], "odd")) return run_odd();
    if (argc == 2 && !strcmp(argv[1], "alpha")) return run_alpha();
    if (argc == 2 && !strcmp(argv[1], "map")) return run_map();
    return 2;
}

// Functions of the kernels' own headers, run on the host: built with hipcc as
// HIP source; no device is used (test_host_kernels.py).
//   odd: doubles on stdin, to_f32_odd of each as float bits on stdout
//   alpha: nodes of 41 f_q and 41 f_eq,q - f_q (floats) on stdin, the entropic
//          path length of each in FP32 arithmetic on stdout, for 32-bit and for
//          16-bit storage
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

int main(int argc, char** argv)
{
    if (argc == 2 && !strcmp(argv[1], "odd")) return run_odd();
    if (argc == 2 && !strcmp(argv[1], "alpha")) return run_alpha();
    return 2;
}

// Functions of the kernels' own headers, run on the host: built with hipcc as
// HIP source; no device is used (test_host_kernels.py).
//   odd: doubles on stdin, to_f32_odd of each as float bits on stdout
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

int main(int argc, char** argv)
{
    if (argc == 2 && !strcmp(argv[1], "odd")) return run_odd();
    return 2;
}

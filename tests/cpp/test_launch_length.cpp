// CPU unit test of pso_launch_length.hpp: runs whose iterations take what was
// measured are cut into launches near the time meant for them.  Prints "ok".
#include <cstdio>

#include "../../paper_2205_01313_amd/csrc/pso_launch_length.hpp"

#define CHECK(c)                                                                                          \
    do {                                                                                                  \
        if (!(c)) {                                                                                       \
            std::printf("FAIL line %d: %s (N=%.0f D=%d us=%.2f)\n", __LINE__, #c, m.N, m.D, m.us);        \
            return 1;                                                                                     \
        }                                                                                                 \
    } while (0)

struct Measured {
    double N;
    int D;
    bool held, wide;
    uint32_t parts;
    double us; // per iteration
};

int main()
{
    const Measured all[] = {
        {1024, 2, false, false, 4, 2.0},      {1000, 30, false, false, 16, 4.5},     {1000, 128, false, false, 63, 7.1},
        {4000, 30, false, false, 63, 4.3},    {32768, 7, false, false, 128, 4.3},    {32768, 128, false, false, 256, 11.6},
        {65536, 128, false, false, 256, 17.4}, {262144, 30, false, false, 256, 14.0}, {131072, 2, false, false, 256, 0.5},
        {1 << 20, 4, true, false, 256, 28.0}, {1 << 20, 32, true, false, 256, 94.0}, {1500000, 32, true, false, 256, 172.0},
        {200, 30, false, true, 13, 5.5},      {1000, 128, false, true, 63, 10.5},    {4000, 30, false, true, 63, 6.5},
        {32768, 128, false, true, 256, 26.0}, {262144, 30, true, true, 256, 44.0},   {1 << 20, 32, true, true, 256, 238.0},
        {4000000, 512, true, true, 256, 20000.0}};
    for (const Measured &m : all) {
        const double want = pso::launch_us(m.parts);
        for (double queued : {0.0, 80000.0}) { // work the stream held before the run
            pso::LaunchLength length{want, pso::gang_iteration_us(m.N, m.D, m.held, m.wide)};
            long long left = 300000, launches = 0;
            const double whole = left * m.us;
            while (left > 0) {
                const long long T = length.next(left);
                CHECK(T >= 1 && T <= left && T <= (long long)pso::GANG_MAX_T);
                CHECK(T * m.us <= 1.75 * want || T == 1);
                length.took(T, T * m.us + 30.0 + (launches == 0 ? queued : 0.0));
                left -= T;
                ++launches;
            }
            CHECK(launches <= 8 + 1.4 * whole / std::min(want, whole) || m.us > want);
        }
        // the shortest runs are one launch
        pso::LaunchLength length{want, pso::gang_iteration_us(m.N, m.D, m.held, m.wide)};
        CHECK(length.next(1) == 1);
    }
    std::printf("ok\n");
    return 0;
}

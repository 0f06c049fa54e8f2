// block_driver.cpp -- runs the block kernel's body (fft_block.hpp) on CPU
// threads, one block after the other, with exactly the launch's LDS.
//
//   block_driver <dtype 0|1> <A> <B> <C> <naxes> <threads> <blocks> <backward>
//                <case c> <case b> <case a>
//
// transforms in[i] = sin(0.37 i + 0.1) + i cos(0.91 i) and prints the output;
// backward conjugates on both sides and scales by 1/(A B C).  Built by
// tests/test_block_kernel_host.py with g++ -fsanitize=address,undefined; the
// cases are in block_cases_emu.inc.
#include "hip_emu.h"

#include <cmath>
#include <cstdlib>
#include <thread>
#include <vector>

#include "fft_block.hpp"
#include "block_cases_emu.inc"

thread_local EmuDim threadIdx;
EmuDim blockIdx, blockDim, gridDim;
EmuBarrier g_emu_barrier;
thread_local long g_emu_barrier_count = 0;

using namespace offt;

template <typename V> static int run(char** v) {
    using S = decltype(V{}.x);
    const int A = atoi(v[0]), B = atoi(v[1]), C = atoi(v[2]), naxes = atoi(v[3]), T = atoi(v[4]), blocks = atoi(v[5]),
              bwd = atoi(v[6]);
    const int n = A * B * C;
    std::vector<V> in((size_t)n * blocks), out((size_t)n * blocks);
    for (size_t i = 0; i < in.size(); ++i) {
        in[i].x = (S)std::sin(0.37 * (double)i + 0.1);
        in[i].y = (S)std::cos(0.91 * (double)i);
    }
    BlockArgs a{};
    a.in = in.data();
    a.out = out.data();
    a.A = A;
    a.B = B;
    a.C = C;
    a.naxes = naxes;
    a.pitch = block_pitch(C);
    a.rcp_C = block_rcp(C);
    a.conj_in = a.conj_out = bwd;
    a.scale = bwd ? 1.0 / n : 1.0;
    std::vector<V> tw[3];
    const int len[3] = {C, B, A};
    for (int x = 0; x < naxes; ++x) {
        a.kid[x] = atoi(v[7 + x]);
        tw[x].resize(len[x]);
        for (int m = 0; m < len[x]; ++m) {
            const long double th = -2.0L * acosl(-1.0L) * m / len[x];
            tw[x][m].x = (S)cosl(th);
            tw[x][m].y = (S)sinl(th);
        }
        a.tw[x] = tw[x].data();
    }
    blockDim.x = T;
    gridDim.x = blocks;
    for (int b = 0; b < blocks; ++b) {
        std::vector<V> lds((size_t)block_lds_elems(A, B, C));
        g_emu_barrier.reset(T);
        std::vector<std::thread> th;
        std::vector<long> barriers(T);
        for (int t = 0; t < T; ++t)
            th.emplace_back([&, t] {
                threadIdx.x = t;
                g_emu_barrier_count = 0;
                block_body<V>(a, lds.data(), b, EmuPass<V>{});
                barriers[t] = g_emu_barrier_count;
            });
        for (auto& x : th) x.join();
        for (int t = 0; t < T; ++t)
            if (g_emu_barrier.broken || barriers[t] != barriers[0]) {
                std::fprintf(stderr, "barrier mismatch\n");
                return 2;
            }
    }
    std::printf("OK\n");
    for (const V& x : out) std::printf("%.17g %.17g\n", (double)x.x, (double)x.y);
    return 0;
}

int main(int argc, char** argv) {
    if (argc < 11) return 1;
    return atoi(argv[1]) == 0 ? run<double2>(argv + 2) : run<float2>(argv + 2);
}

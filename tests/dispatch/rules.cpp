// Asks the library's own dispatch rules, on the CPU: the whole host side is compiled in, without its kernels, and no call here
// reaches the device.  tests/test_dispatch_rules.py names the questions and checks the answers.
#include "../../paper_2203_13085_amd/csrc/lasgd.hip"

#include <cstdlib>

static lasgd_ctx context(int K, uint64_t n, bool bf16)
{
    lasgd_ctx c;
    c.K = K;
    c.n_tensors = 1;
    c.all = K == 64 ? ~0ull : (1ull << K) - 1ull;
    c.storage = bf16 ? LASGD_BF16 : LASGD_F32;
    c.main = (hipStream_t)1;                 // two streams that are not the same; never used
    c.side = (hipStream_t)2;
    c.packed = round_up(n, kArenaAlign);
    c.npad = padded(c.packed);
    c.tune = default_tuning(c);
    return c;
}

int main(int argc, char **argv)
{
    if (argc < 5) return 2;
    const std::string what = argv[1];
    const int K = atoi(argv[2]);
    lasgd_ctx c = context(K, strtoull(argv[3], nullptr, 10), !strcmp(argv[4], "bf16"));
    if (what == "mean_on_main") printf("%d %d\n", (int)mean_on_main((uint32_t)K, c.packed), c.tune.avg_split);
    else return 2;
    return 0;
}

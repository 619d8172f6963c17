// Host driver of the rule which products read row patterns.  argv: bytes per
// value (8 or 4), block width, rows, mean run of rows with one pattern, 1 for
// the plain product or 2 for the two-block omega pass; prints 1 when it does.
#include <cstdio>
#include <cstdlib>

#include "internal.h"
#include "ops.h"

namespace {
template <typename T>
struct Rule {
    int32_t n, run;
    bool omega;
    template <int M>
    bool operator()() const
    {
        return omega ? mrhs::pattern_pays<T, M, mrhs::OpSpmv2<T, M>>(n, run)
                     : mrhs::pattern_pays<T, M, mrhs::OpStore<T, M>>(n, run);
    }
};
} // namespace

int main(int argc, char **argv)
{
    if (argc != 6)
        return 2;
    const int m = std::atoi(argv[2]);
    const int32_t n = static_cast<int32_t>(std::atoll(argv[3]));
    const int32_t run = std::atoi(argv[4]);
    const bool omega = argv[5][0] == '2';
    const bool on = argv[1][0] == '8' ? mrhs::dispatch_m(m, Rule<double>{n, run, omega})
                                      : mrhs::dispatch_m(m, Rule<float>{n, run, omega});
    std::printf("%d\n", on ? 1 : 0);
    return 0;
}

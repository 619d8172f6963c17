// Host driver of the rule which plain products read row patterns.  argv: bytes
// per value (8 or 4), block width, rows; prints 1 when they do, else 0.
#include <cstdio>
#include <cstdlib>

#include "internal.h"
#include "ops.h"

namespace {
template <typename T>
struct Rule {
    int32_t n;
    template <int M>
    bool operator()() const
    {
        return mrhs::pattern_pays<T, M, mrhs::OpStore<T, M>>(n);
    }
};
} // namespace

int main(int argc, char **argv)
{
    if (argc != 4)
        return 2;
    const int m = std::atoi(argv[2]);
    const int32_t n = static_cast<int32_t>(std::atoll(argv[3]));
    const bool on = argv[1][0] == '8' ? mrhs::dispatch_m(m, Rule<double>{n}) : mrhs::dispatch_m(m, Rule<float>{n});
    std::printf("%d\n", on ? 1 : 0);
    return 0;
}

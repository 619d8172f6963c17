// Host driver of the row range of the row-pattern form.  argv[1]: rows of a
// matrix; prints 1 when such a matrix may have patterns, else 0.
#include <cstdio>
#include <cstdlib>

#include "core.h"

int main(int argc, char **argv)
{
    if (argc != 2)
        return 2;
    std::printf("%d\n", mrhs::pattern_rows(static_cast<int32_t>(std::atoll(argv[1]))) ? 1 : 0);
    return 0;
}

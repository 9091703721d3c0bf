// Host-only: the far field's size rule (field_wanted, mppi_field.hpp).  Reads
// "model K T J P shape_kind cost_mode" lines and prints 1 or 0 for each.
#include <cstdio>

#include "mppi_field.hpp"

int main()
{
    int model, K, T, J, P, kind, mode;
    while (std::scanf("%d %d %d %d %d %d %d", &model, &K, &T, &J, &P, &kind, &mode) == 7)
        std::printf("%d\n", dbas::field_wanted(model, K, T, J, P, kind, mode) ? 1 : 0);
    return 0;
}

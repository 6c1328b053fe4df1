// Prints march_step_pays (march_rule.h) for each "nx ny nz box elem products
// stored_ap" line of stdin.
#include <cstdio>

#include "march_rule.h"

int main()
{
    long long nx, ny, nz;
    int box, elem, products, ap;
    while (std::scanf("%lld %lld %lld %d %d %d %d", &nx, &ny, &nz, &box, &elem, &products, &ap) == 7)
        std::printf("%d\n", int(sstep::march_step_pays(nx, ny, nz, box != 0, elem, products != 0, ap != 0)));
    return 0;
}

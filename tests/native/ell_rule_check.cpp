// Prints ell_keep_pays (ell_rule.h) for each "values span elem" line of stdin.
#include <cstdio>

#include "ell_rule.h"

int main()
{
    long long values, span;
    int elem;
    while (std::scanf("%lld %lld %d", &values, &span, &elem) == 3)
        std::printf("%d\n", int(sstep::ell_keep_pays(values, span, elem)));
    return 0;
}

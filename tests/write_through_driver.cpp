// Which configured launches write their outputs through, for tests/test_write_through.py.  Host code only.
// One launch per line: op (0: add+RMSNorm, 1: silu_and_mul, 2: merge_attn_states) dtype M N and the cfg's eight numbers; 0 or 1
// per line of output.
#include <stdio.h>

#include "addrms_internal.h"

int main()
{
    int op, dtype, v[8];
    long long M, N;
    while (scanf("%d %d %lld %lld", &op, &dtype, &M, &N) == 4 &&
           scanf("%d,%d,%d,%d,%d,%d,%d,%d", v, v + 1, v + 2, v + 3, v + 4, v + 5, v + 6, v + 7) == 8) {
        const addrms_cfg c{v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7]};
        printf("%d\n", addrms_host::launch_write_through(c, M, N, dtype, op) ? 1 : 0);
    }
    return 0;
}

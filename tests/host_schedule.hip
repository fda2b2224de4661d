// Stages of the cooling schedule as the chain kernels step through them, on the
// CPU: lines "n_steps n_stages first last" on standard input; for each the first
// step in first..last whose stage is not floor(step n_stages / n_steps), or -1.
#include <cstdio>

#include "sat_chain.hpp"

int main()
{
    long long n_steps, n_stages, first, last;
    while (std::scanf("%lld %lld %lld %lld", &n_steps, &n_stages, &first, &last) == 4) {
        pila::Schedule s;
        s.start(first, n_steps, (int32_t)n_stages, 1.0, 0.5, PILA_SCHED_LINEAR);
        long long bad = -1;
        for (long long t = first; t <= last && bad < 0; ++t) {
            s.at(t);
            if (s.stage != (int64_t)((__int128)t * n_stages / n_steps)) bad = t;
            if (s.next <= t || s.next > n_steps) bad = t;
        }
        std::printf("%lld\n", bad);
    }
    return 0;
}

// The copy function of csrc/afun.hpp, compiled for the host for test_afun_host.py.
#include "afun.hpp"

static smc::AFun make(long long n, unsigned long long S, unsigned long long U)
{
    smc::AFun f;
    f.n = n;
    f.set_systematic(S, U);
    return f;
}

extern "C" {
double afun_slack() { return smc::kSlack; }

double afun_estimate(long long n, unsigned long long S, unsigned long long U,
                     unsigned long long sj)
{
    const smc::AFun f = make(n, S, U);
    return fma(smc::u64_to_f64(sj), f.nS, f.uS);
}

unsigned afun_copies(long long n, unsigned long long S, unsigned long long U,
                     unsigned long long sj)
{
    return make(n, S, U).A_of(0, sj);
}

int afun_before(long long n, unsigned long long S, unsigned long long U, unsigned long long sj,
                long long j, long long k)
{
    return make(n, S, U).pred_at(j, sj, k);
}
}

// Prints how prefill_cut (csrc/fbq_internal.h) cuts layers into blocks, as "<rows>/<K split>" or "<rows>+<rows of the second
// launch>" with " single" behind it where low tiles have one K group: one line for each "M N K r" on stdin, then - without the
// number of splits - every kind that a million calls of ordinary sizes meet, with its count.  With an argument: for each "M N K r" the token
// tiles and K slices of the down-projection and how many of the slices are dealt out to the XCDs whole.
#include <cstdio>
#include <map>
#include <random>
#include <string>

#include "fbq_internal.h"

using namespace fbq;

static std::string kind(int M, int N, int K, int r, bool with_split)
{
    const PrefillCut c = prefill_cut(M, N, K, r);
    std::string s = std::to_string(32 * c.tm);
    if (c.tail_tm) s += "+" + std::to_string(32 * c.tail_tm);
    else if (c.ksplit > 1) s += with_split ? "/" + std::to_string(c.ksplit) : "/split";
    return c.single ? s + " single" : s;
}

int main(int argc, char **)
{
    int M, N, K, r;
    while (argc > 1 && scanf("%d %d %d %d", &M, &N, &K, &r) == 4)
        printf("%d %d %d\n", ceil_div(M, 32), down_slices(M, K), down_slices_by_xcd(M, N, K, r));
    if (argc > 1) return 0;
    while (scanf("%d %d %d %d", &M, &N, &K, &r) == 4) printf("%s\n", kind(M, N, K, r, true).c_str());
    std::mt19937_64 gen(1);
    auto log_uniform = [&](double lo, double hi) { return (int)std::lround(lo * std::pow(hi / lo, (double)(gen() >> 11) * 0x1p-53)); };
    std::map<std::string, long> kinds;
    for (int i = 0; i < 1000000; ++i) {
        M = log_uniform(65, 2048);
        N = log_uniform(500, 33000);
        K = kGroup * log_uniform(1, 224);
        ++kinds[kind(M, N, K, i % 2 * 64, false)];
    }
    printf("kinds\n");
    for (const auto &k : kinds) printf("%ld %s\n", k.second, k.first.c_str());
    return 0;
}

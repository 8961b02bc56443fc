// Host run of the plan table (launch.h): how often plans are made for a network's worth of problems called in turn.
#include "../../paper_2104_04731_amd/csrc/launch.h"

#include <stdio.h>
#include <stdlib.h>

struct Key {
    int v[12];
};
struct Val {
    int id, pad[30];
};
static c2i8::PlanTable<Key, Val, 64> table;

static Key key_of(int i)   // layers that differ in a few of their integers
{
    Key k{};
    const int c[] = {16, 32, 64, 128, 256, 512};
    k.v[0] = 1 + i % 3, k.v[1] = c[i % 6], k.v[2] = 7 << (i % 4), k.v[3] = c[i / 6 % 6], k.v[4] = i, k.v[11] = i & 1;
    return k;
}

// Plans made while `n` problems are called `passes` times in turn; -1 if a wrong plan came back.
static int made(int first, int n, int passes)
{
    int count = 0;
    for (int p = 0; p < passes; ++p)
        for (int i = first; i < first + n; ++i) {
            const Val *v = table.get(key_of(i), [&](Val *o) { return o->id = i, ++count, true; });
            if (!v || v->id != i) return -1;
        }
    return count;
}

int main()
{
    if (table.get(key_of(1000), [](Val *) { return false; })) return 1;   // nothing to keep: asked again the next time
    if (made(0, 20, 5) != 20) return puts("20 problems"), 1;
    if (made(0, 64, 5) != 44) return puts("64 problems"), 1;               // the first twenty are there
    if (table.get(key_of(1000), [](Val *) { return false; })) return 1;   // ... and a refusal displaces none
    if (made(0, 64, 1) != 0) return puts("after a refusal"), 1;
    if (made(100, 1, 3) != 1 || made(0, 64, 1) > 2) return puts("one more than the table holds"), 1;
    const int cycling = made(0, 96, 4);
    if (cycling < 0) return puts("96 problems"), 1;
    puts("ok");
    return 0;
}

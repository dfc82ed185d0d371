// Host check of the bounded store of past calls (test program).  Exit status 0
// when every statement holds.
#include <cstdio>

#include "../../paper_0710_3747_amd/csrc/kept.hpp"

using namespace spinqp;

static int bad = 0;
#define HOLDS(x)                          \
    do {                                  \
        if (!(x)) {                       \
            std::printf("not: %s\n", #x); \
            ++bad;                        \
        }                                 \
    } while (0)

int main() {
    static int alive = 0;
    struct Thing {
        Thing() { ++alive; }
        ~Thing() { --alive; }
    };
    auto key = [](int n) { return std::vector<double>{double(n)}; };
    {
        // by number: the one unused for longest goes, one in use or pinned does not
        Kept<Thing> k(4, 1000);
        for (int n = 0; n < 4; ++n) HOLDS(k.insert(key(n), std::make_shared<Thing>(), 10).empty());
        HOLDS(k.find(key(0)) && k.find(key(1), true));
        for (int n = 4; n < 100; ++n) HOLDS(k.insert(key(n), std::make_shared<Thing>(), 10).size() == 1);
        HOLDS(k.size() == 4 && k.bytes() == 40 && alive == 4);
        HOLDS(k.find(key(1)) && k.find(key(99)) && !k.find(key(0)) && !k.find(key(96)) && k.find(key(97)));
        std::shared_ptr<Thing> held = k.find(key(99));
        for (int n = 100; n < 110; ++n) k.insert(key(n), std::make_shared<Thing>(), 10);
        HOLDS(!k.find(key(99)) && alive == 5);
        held.reset();
        HOLDS(alive == 4);
        HOLDS(k.clear().size() == 4);
        HOLDS(k.size() == 0 && k.bytes() == 0 && alive == 0);
    }
    {
        // by bytes; replaced entries are counted once; a large one stays by itself
        Kept<Thing> k(100, 1000);
        for (int n = 0; n < 50; ++n) k.insert(key(n), std::make_shared<Thing>(), 100);
        HOLDS(k.size() == 10 && k.bytes() == 1000 && alive == 10);
        for (int n = 0; n < 5; ++n) HOLDS(k.insert(key(49), std::make_shared<Thing>(), 100).size() == 1);
        HOLDS(k.size() == 10 && k.bytes() == 1000 && alive == 10);
        HOLDS(k.insert(key(60), std::make_shared<Thing>(), 5000).size() == 10);
        HOLDS(k.size() == 1 && k.find(key(60)) && alive == 1);
        k.insert(key(61), std::make_shared<Thing>(), 1);
        HOLDS(k.size() == 1 && k.find(key(61)) && !k.find(key(60)));
    }
    HOLDS(alive == 0);
    return bad ? 1 : 0;
}

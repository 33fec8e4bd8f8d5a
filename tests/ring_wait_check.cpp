// Host check of ring_wait_count: the order in which a wave issues its copies and weight loads is played
// through for both loops, and at every wait the operations issued after the copies of the stage that is
// read next must be at least the count that the kernel lets stay in flight.
#include <cstdio>
#include <vector>
#include "ring.h"
using namespace dvi;

struct Wave {
    int PX, ops = 0;
    std::vector<int> end;  // operations issued up to and with the copies of each stage
    void copy(int stage) {
        if ((int)end.size() <= stage) end.resize(stage + 1, -1);
        ops += PX;
        end[stage] = ops;
    }
    int younger(int stage) const { return ops - end[stage]; }
};

int main() {
    int checked = 0;
    for (int CPS = 1; CPS <= 4; ++CPS)
        for (int NS = 2; NS <= 8; ++NS)
            for (int WD = CPS; WD <= 16; WD += CPS)
                for (int RT = 1; RT <= 4; ++RT)
                    for (int PX = 1; PX <= 4; ++PX)
                        for (int piped = 0; piped <= 1; ++piped) {
                            const int count = ring_wait_count(CPS, NS, WD, RT, PX, piped);
                            int least = 1 << 30;
                            Wave w{PX};
                            for (int s = 0; s < NS - 1; ++s) w.copy(s);
                            w.ops += WD * RT;
                            auto wait = [&](int stage) { least = w.younger(stage) < least ? w.younger(stage) : least; };
                            if (piped) {
                                wait(0);
                                w.copy(NS - 1);
                            }
                            for (int s = 0; s < 4 * NS; ++s) {
                                if (!piped) {
                                    wait(s);
                                    w.copy(s + NS - 1);
                                    w.ops += CPS * RT;
                                } else {
                                    w.ops += (CPS - 1) * RT;
                                    wait(s + 1);
                                    w.copy(s + NS);
                                    w.ops += RT;
                                }
                            }
                            if (count > least || (count < least && count < 63)) {
                                printf("CPS %d NS %d WD %d RT %d PX %d piped %d: count %d, certainly younger %d\n", CPS, NS, WD,
                                       RT, PX, piped, count, least);
                                return 1;
                            }
                            ++checked;
                        }
    printf("ok %d\n", checked);
    return 0;
}

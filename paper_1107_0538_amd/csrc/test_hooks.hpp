// What the tests of the on-chip solver set for the calls of their own thread:
// conditions that the hardware brings about only rarely.
#pragma once

#include "resident.hpp"

namespace jpcg {

struct TestHooks {
    long long wait_limit = -1;  // device ticks that a workgroup waits; < 0: as ever
    int absent = -1;            // this member of every team leaves at once, as if it had not come
    int quit = -1;              // this member of every team gives up at the end of the solve
    bool no_memory = false;     // there is no memory for on-chip solvers

    void apply(RsRun& run) const
    {
        if (wait_limit >= 0) run.limit_first = run.limit = wait_limit;
        run.absent = absent;
        run.quit = quit;
    }
};

TestHooks& test_hooks();

}  // namespace jpcg

extern "C" {
// For the calling thread, until the next call.
void jpcg_test_on_chip(long long wait_limit, int absent, int quit);
void jpcg_test_no_memory(int on);
// Whether the last solve's result came from the chip (-1: not solved yet).
int jpcg_test_solved_on_chip(const cg_ctx* c);
int jpcg_test_batch_solved_on_chip(const cg_batch* b);
}

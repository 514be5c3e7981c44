// What the tests of the on-chip solver set for the calls of their own thread:
// conditions that the hardware brings about only rarely.
#pragma once

#include "resident.hpp"

namespace jpcg {

struct TestHooks {
    long long wait_limit = -1;  // device ticks that a workgroup waits; < 0: as ever
    int absent = 0;             // members of every group that a solve is launched without
    bool given_up = false;      // a workgroup gave up as the others finished
    bool no_memory = false;     // there is no memory for on-chip solvers
};

TestHooks& test_hooks();

}  // namespace jpcg

extern "C" {
// For the calling thread, until the next call.
void jpcg_test_on_chip(long long wait_limit, int absent, int given_up);
void jpcg_test_no_memory(int on);
// Whether the last solve's result came from the chip (-1: not solved yet).
int jpcg_test_solved_on_chip(const cg_ctx* c);
int jpcg_test_batch_solved_on_chip(const cg_batch* b);
}

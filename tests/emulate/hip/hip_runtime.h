// Stands in for HIP's header when a kernel source is compiled for the CPU by
// tests/emulate: every GPU thread is a fiber on one OS thread, so a workgroup
// runs deterministically, and the order in which its waves get on between two
// points where they wait is chosen by the test (see lanes.hpp).
#pragma once
#include "../lanes.hpp"

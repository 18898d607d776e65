// What the host-side plans know about the chip (gfx950).
#pragma once

namespace rl {

constexpr int kComputeUnits = 256;
constexpr int kDies = 8;  // blocks go to them in turn, each has an L2 of its own

}  // namespace rl

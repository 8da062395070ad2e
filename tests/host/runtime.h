// A HIP runtime and the library's kernel launches as host code, so that the
// host sources (program.cpp, dl_api.cpp, serve.cpp) run on the CPU: device
// memory is host memory with a limit, events and streams are always complete,
// and launches only record what the tests ask about.
#pragma once
#include <cstddef>
#include <cstdint>
#include <string>
#include <vector>

namespace fake {
extern size_t limit;  // bytes of device memory
extern size_t live;   // allocated now
struct Emit {
  int Np, n;
  int64_t ld;
};
extern std::vector<Emit> emits;               // copies of models to the caller
extern std::vector<std::string> launches;     // names of the launches, in order
}  // namespace fake

// score_once_pair.hip -- two calls of score_once.hpp in one launch: a target call (one layer, one
// column tile over one, two or four KV heads), then a draft call, as a verification step scores them.
#include "score_once.hpp"

namespace dustin {

namespace {

template <int NU, int TW>
struct LaunchPair {
  const ChunkArgs& a;
  hipStream_t stream;
  template <class S>
  hipError_t operator()(S) const { return launch_once<ChunkShape<128, NU, 0, TW>, S>(a, stream); }
};

template <int NU>
hipError_t launch_pair(const ChunkArgs& a, hipStream_t stream) {
  const ChunkCall& draft = a.call[1];
  return draft.tw == 8 ? draft_shape<8>(draft, LaunchPair<NU, 8>{a, stream})
                       : draft_shape<4>(draft, LaunchPair<NU, 4>{a, stream});
}

}  // namespace

bool score_once_pair_supported(const ChunkCall& c0, const ChunkCall& c1) {
  return c0.tw == c1.tw && c0.head_dim == 128 && c0.nt == 0 && c0.n_layers == 1 &&
         (c0.nu == 1 || c0.nu == 2 || c0.nu == 4) && c1.head_dim == 64 && c1.nu == 2 && !c1.per_layer &&
         (c1.nt == 0 || (c1.nt == 1 && c1.n_layers == 3));
}

hipError_t launch_score_once_pair(const ChunkArgs& a, hipStream_t stream) {
  switch (a.call[0].nu) {
    case 1: return launch_pair<1>(a, stream);
    case 2: return launch_pair<2>(a, stream);
    case 4: return launch_pair<4>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace dustin

// score_once.hip -- the calls of score_once.hpp that are a launch of their own.
#include "score_once.hpp"

namespace dustin {

namespace {

// one layer, pairs of all KV heads in one column tile
template <int D, int NU>
hipError_t launch_shared(const ChunkArgs& a, hipStream_t stream) {
  return a.call[0].tw == 8 ? launch_once<ChunkShape<D, NU, 0, 8>, NoShape>(a, stream)
                           : launch_once<ChunkShape<D, NU, 0, 4>, NoShape>(a, stream);
}

template <int D>
hipError_t launch_nu(const ChunkArgs& a, hipStream_t stream) {
  switch (a.call[0].nu) {
    case 1: return launch_shared<D, 1>(a, stream);
    case 2: return launch_shared<D, 2>(a, stream);
    case 3: return launch_shared<D, 3>(a, stream);
    case 4: return launch_shared<D, 4>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

// a draft's layers
struct LaunchAlone {
  const ChunkArgs& a;
  hipStream_t stream;
  template <class S>
  hipError_t operator()(S) const { return launch_once<S, NoShape>(a, stream); }
};

}  // namespace

// One layer per output, or a draft's summed layers (over two KV heads of 64-element rows); pairs in one
// column tile, or (such a draft, of one layer or three) one or two for each KV head.
bool score_once_supported(const ChunkCall& c) {
  const bool draft = c.head_dim == 64 && c.nu == 2;
  if (c.nt > 0 && !draft) return false;
  if (c.n_layers == 1 || c.per_layer) return true;
  return draft && (c.nt == 0 || (c.nt == 1 && c.n_layers == 3));
}

hipError_t launch_score_once(const ChunkArgs& a, int n_calls, hipStream_t stream) {
  if (n_calls == 2) return launch_score_once_pair(a, stream);
  const ChunkCall& c = a.call[0];
  if (c.n_layers > 1 && !c.per_layer)
    return c.tw == 8 ? draft_shape<8>(c, LaunchAlone{a, stream}) : draft_shape<4>(c, LaunchAlone{a, stream});
  if (c.nt == 0) return c.head_dim == 128 ? launch_nu<128>(a, stream) : launch_nu<64>(a, stream);
  return c.nt == 1 ? launch_once<ChunkShape<64, 2, 1, 4>, NoShape>(a, stream)
                   : launch_once<ChunkShape<64, 2, 2, 4>, NoShape>(a, stream);
}

}  // namespace dustin

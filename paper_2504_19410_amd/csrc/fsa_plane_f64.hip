// passes B, C, D of small planes in one launch, FP64
#include "fsa_plane_launch.hpp"
template struct fsa::PlaneV<double>;

// size_passes.hip -- the specialised passes of one size and type of ns_size_plans.hpp:
// the build compiles this file once for each, with NS_SIZE_N and NS_SIZE_T defined.
#include "ns_size_eval.hpp"

template const nsh::SizePasses<NS_SIZE_T>* nsh::size_passes<NS_SIZE_T, NS_SIZE_N>();

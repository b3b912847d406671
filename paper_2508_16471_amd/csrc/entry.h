// Exceptions end at the C entry points: host allocations in them throw, nothing
// is thrown across the ABI.  An entry point that allocates is a function-try-
// block, `extern "C" int f(...) try { ... } VIE_CATCH`.
#pragma once

#include <new>
#include <stdexcept>

#include "../../include/vie.h"

#define VIE_CATCH                                        \
  catch (const std::bad_alloc&) { return VIE_ENOMEM; }   \
  catch (const std::length_error&) { return VIE_ENOMEM; } \
  catch (...) { return VIE_EDEVICE; }

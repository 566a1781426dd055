// Definitions behind step_table.hpp; included only by the per-storage
// translation units that instantiate them.
#pragma once

#define LBM_STEP_TU
#include "step_table.hpp"

namespace lbm {

template <typename S, bool RED, bool NT>
const void* step_pair_fn(int collision, int wall_tmpl) {
  if constexpr (sizeof(S) == 2) {
    switch (collision * 2 + wall_tmpl) {
      case 0: return (const void*)step_pair_kernel<S, kSRT, kSBB, RED, NT>;
      case 1: return (const void*)step_pair_kernel<S, kSRT, kCLI, RED, NT>;
      case 2: return (const void*)step_pair_kernel<S, kTRT, kSBB, RED, NT>;
      case 3: return (const void*)step_pair_kernel<S, kTRT, kCLI, RED, NT>;
      case 4: return (const void*)step_pair_kernel<S, kMRT, kSBB, RED, NT>;
      default: return (const void*)step_pair_kernel<S, kMRT, kCLI, RED, NT>;
    }
  }
  return nullptr;
}

template <typename S, bool RED, int MEM>
const void* step_fn(int collision, int wall_tmpl) {
  if constexpr (kUnscaledStorage<S>) {
    if (wall_tmpl == kGEN) {  // (one form within and beyond the cache)
      constexpr int M = MEM == kBeyondCache ? kCached : MEM;
      switch (collision) {
        case 0: return (const void*)step_kernel<S, kSRT, kGEN, RED, M>;
        case 1: return (const void*)step_kernel<S, kTRT, kGEN, RED, M>;
        default: return (const void*)step_kernel<S, kMRT, kGEN, RED, M>;
      }
    }
  }
  switch (collision * 2 + wall_tmpl) {
    case 0: return (const void*)step_kernel<S, kSRT, kSBB, RED, MEM>;
    case 1: return (const void*)step_kernel<S, kSRT, kCLI, RED, MEM>;
    case 2: return (const void*)step_kernel<S, kTRT, kSBB, RED, MEM>;
    case 3: return (const void*)step_kernel<S, kTRT, kCLI, RED, MEM>;
    case 4: return (const void*)step_kernel<S, kMRT, kSBB, RED, MEM>;
    default: return (const void*)step_kernel<S, kMRT, kCLI, RED, MEM>;
  }
}

template <typename S, bool RED>
const void* step_mem(int mem, bool pairs, int collision, int wall_tmpl) {
  if (pairs)
    return mem == kStreaming ? step_pair_fn<S, RED, true>(collision, wall_tmpl)
                             : step_pair_fn<S, RED, false>(collision, wall_tmpl);
  if (mem == kStreaming) return step_fn<S, RED, kStreaming>(collision, wall_tmpl);
  if constexpr (kUnscaledStorage<S>) {  // (16-bit values: one form)
    if (mem == kBeyondCache) return step_fn<S, RED, kBeyondCache>(collision, wall_tmpl);
  }
  return step_fn<S, RED, kCached>(collision, wall_tmpl);
}

template <typename S>
const void* step_kernel_entry(bool red, int mem, bool pairs, int collision, int wall_tmpl) {
  return red ? step_mem<S, true>(mem, pairs, collision, wall_tmpl)
             : step_mem<S, false>(mem, pairs, collision, wall_tmpl);
}

template <typename S, bool RED, int MEM>
const void* batch_fn(int collision, int wall_tmpl) {
  if (wall_tmpl == kGEN) {
    switch (collision) {
      case 0: return (const void*)batch_step_kernel<S, kSRT, kGEN, RED, MEM>;
      case 1: return (const void*)batch_step_kernel<S, kTRT, kGEN, RED, MEM>;
      default: return (const void*)batch_step_kernel<S, kMRT, kGEN, RED, MEM>;
    }
  }
  switch (collision * 2 + wall_tmpl) {
    case 0: return (const void*)batch_step_kernel<S, kSRT, kSBB, RED, MEM>;
    case 1: return (const void*)batch_step_kernel<S, kSRT, kCLI, RED, MEM>;
    case 2: return (const void*)batch_step_kernel<S, kTRT, kSBB, RED, MEM>;
    case 3: return (const void*)batch_step_kernel<S, kTRT, kCLI, RED, MEM>;
    case 4: return (const void*)batch_step_kernel<S, kMRT, kSBB, RED, MEM>;
    default: return (const void*)batch_step_kernel<S, kMRT, kCLI, RED, MEM>;
  }
}

template <typename S, bool RED>
const void* batch_mem(int mem, int collision, int wall_tmpl) {
  if (mem == kStreaming) return batch_fn<S, RED, kStreaming>(collision, wall_tmpl);
  if (mem == kBeyondCache) return batch_fn<S, RED, kBeyondCache>(collision, wall_tmpl);
  return batch_fn<S, RED, kCached>(collision, wall_tmpl);
}

template <typename S>
const void* batch_kernel_entry(bool red, int mem, int collision, int wall_tmpl) {
  return red ? batch_mem<S, true>(mem, collision, wall_tmpl)
             : batch_mem<S, false>(mem, collision, wall_tmpl);
}

}  // namespace lbm

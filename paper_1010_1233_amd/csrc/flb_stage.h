// flb_stage.h -- transfers between a handle's device data and the caller's
// (pageable) host memory.
//
// A transfer is cut into chunks.  Each chunk goes through a slot of pinned
// host memory that a kernel writes (or reads) directly over PCIe, already
// in the caller's layout and type; a worker thread per slot copies between
// the slot and the caller's memory, so that the first touch of the caller's
// pages, which a single thread does at about 10 GB/s, is spread over cores
// and runs beside the next chunks' kernels.  No device memory is needed.
#pragma once

#include <stddef.h>

#include <functional>

#include "flb_internal.h"

namespace flbdev {

constexpr int kStageSlots = 8;                      // worker threads at most
constexpr size_t kStageSlotDoubles = (size_t)1 << 19;  // 4 MiB a slot

// Every open handle holds a reference; the slots (32 MiB, shared by all
// handles, one transfer at a time) are allocated by the first transfer and
// freed with the last reference.
void stage_retain();
void stage_release();

// Enqueues the kernel for `n` doubles of the transfer, from its double
// `first` on, on stream s; `slot` is their place in the pinned memory.
using StageKernel = std::function<hipError_t(double *slot, size_t first, size_t n, hipStream_t s)>;

// Fills out[0 .. n-1] through kernels on stream s (behind the work already
// there); returns when out is complete.
hipError_t stage_out(int device, hipStream_t s, double *out, size_t n, const StageKernel &kernel);
// Hands in[0 .. n-1] to kernels on stream s; returns when they have run.
hipError_t stage_in(int device, hipStream_t s, const double *in, size_t n,
                    const StageKernel &kernel);

}  // namespace flbdev

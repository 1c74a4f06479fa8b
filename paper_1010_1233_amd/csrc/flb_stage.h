// flb_stage.h -- transfers between a handle's device data and the caller's
// (pageable) host memory.
//
// A transfer is cut into chunks.  Each chunk goes through a slot of pinned
// host memory that a kernel writes (or reads) directly over PCIe, already
// in the caller's layout and type; the calling thread and helper threads
// copy between the slots and the caller's memory, each taking the next chunk
// when it is free, so that the first touch of the caller's pages, which a
// single thread does at about 10 GB/s, is spread over cores and runs beside
// the next chunks' kernels, and a helper that finds no free core holds
// nothing up.  No device memory is needed.
#pragma once

#include <stddef.h>

#include <functional>

#include "flb_internal.h"

namespace flbdev {

constexpr int kStageWorkers = 8;  // threads of a transfer, the caller's among them
constexpr size_t kStageSlotDoubles = (size_t)1 << 18;  // 2 MiB a slot, two per thread
// Transfers of up to this many values go through a place of 512 KiB of their
// own: a program that only reads small lattices pins no slots.
constexpr size_t kStageSmallDoubles = (size_t)1 << 16;

// Every open handle holds a reference; the slots (up to 32 MiB, shared by all
// handles, one transfer at a time) and the helper threads are made by the
// first transfer that needs so many and given back with the last reference.
// A transfer that finds them taken goes through a place or two slots of its
// own (kept likewise, for at most kStageExtra at a time): their holder may be waiting
// for steps that its stream has still to run.  Opening and closing a handle
// waits for no transfer.
constexpr int kStageExtra = 7;
void stage_retain();
void stage_release();

// (StageDone: flb_internal.h)
constexpr int kStageFlags = 64;  // blocks at most
// Blocks of 256 values each that a kernel gets for n values.
constexpr size_t kStageBlock = 256;

// Enqueues the kernel for `n` doubles of the transfer, from its double
// `first` on, on stream s, in ceil(n / kStageBlock) blocks; `slot` is their
// place in the pinned memory.
using StageKernel =
    std::function<hipError_t(double *slot, size_t first, size_t n, StageDone done, hipStream_t s)>;

// Fills out[0 .. n-1] through kernels on stream s (behind the work already
// there); returns when out is complete.
hipError_t stage_out(int device, hipStream_t s, double *out, size_t n, const StageKernel &kernel);
// Hands in[0 .. n-1] to kernels on stream s; returns when they have run.
hipError_t stage_in(int device, hipStream_t s, const double *in, size_t n,
                    const StageKernel &kernel);

}  // namespace flbdev

// Resident workgroups of kernel shapes, kept per device and LDS size (host
// code only, no HIP): a query costs the runtime an attribute call and an
// occupancy computation, so each is made once in a process, whatever the
// number of layers and epilogues it runs.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <atomic>

#include "sl_internal.h"

namespace sl {

// One slot a possible LDS size: sizes are multiples of kStep, at most MaxLds.
template <int Devices, int Shapes, size_t MaxLds>
class ResidentTable {
public:
    static constexpr size_t kStep = 256;

    // *out = what query(out) gives for (device, shape, lds), from the table
    // after the first time. Threads that meet an empty slot together fill it
    // with equal values; a failed query is not kept.
    template <class F>
    sl_status get(int device, int shape, size_t lds, int *out, F &&query)
    {
        const bool kept = device >= 0 && device < Devices && shape >= 0 && shape < Shapes && lds <= MaxLds &&
                          lds % kStep == 0;
        if (kept) {
            const int v = slot_[device][shape][lds / kStep].load(std::memory_order_relaxed);
            if (v > 0) {
                *out = v - 1;
                return SL_OK;
            }
        }
        const sl_status st = query(out);
        if (st == SL_OK && kept && *out >= 0 && *out < INT16_MAX)
            slot_[device][shape][lds / kStep].store((int16_t)(*out + 1), std::memory_order_relaxed);
        return st;
    }

private:
    std::atomic<int16_t> slot_[Devices][Shapes][MaxLds / kStep + 1] = {};  // 0: not known, else the value plus 1
};

}  // namespace sl

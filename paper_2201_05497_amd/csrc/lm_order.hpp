// Event lists in spatial order (lm_order.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lm_device.hpp"
#include "lm_host.hpp"

namespace lmk {

// A caller's event, padded to whole words.
struct __align__(4) OrderedEvent {
  int16_t ev[6];
};

// Device arrays of an order: the events in order, a value for each, the place
// in the order of every event of the list, and temporaries (22 bytes per
// event in all).
struct EventOrder {
  OrderedEvent *rec = nullptr;
  float *val = nullptr;
  unsigned *place = nullptr;
  uint16_t *bins = nullptr;
  unsigned *total = nullptr, *base = nullptr;
};

// Scanners whose crystal positions fit the binning kernel's LDS.
bool order_possible(const GeomDev &g);
void add_order(lmh::Slab &arrays, long long n, EventOrder &o);
// Orders the n < 2^31 events of ev.
int launch_order(const GeomDev &g, const int16_t *ev, long long n, const EventOrder &o, hipStream_t st);
// Values in order (val) -> out in list order.
int launch_order_back(const EventOrder &o, long long n, float *out, hipStream_t st);

}  // namespace lmk

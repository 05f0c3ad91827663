// Memory pass of the 32-bit path with a candidate's gap table in LDS (peaks.hip).
#pragma once

#include "ss_internal.h"

// Counters the pass takes its candidates from, a 64-byte line each; zero at launch.
constexpr int kPeakTickets = 16, kTicketPitch = 16, kTicketWords = kPeakTickets * kTicketPitch;

// How the pass runs for one GMG; ok is false when its table does not fit a
// workgroup's LDS (or, with ports, its graph is not one of the packed form).
struct PeaksShape {
  bool ok = false;
  bool csr = false;       // general graphs: successors from the CSR
  int threads = 64;       // per workgroup (candidate)
  int lds_nodes = 0;      // hard-gap events held in LDS
  size_t lds = 0;         // dynamic LDS of a workgroup
  int64_t blocks = 0;     // workgroups the device holds at once
  int64_t node_cap = 0;   // most hard-gap events of a candidate
};
PeaksShape ss_peaks_shape(const ss_gmg *g, bool ports, int cus, int64_t lds_block, int64_t lds_cu);
// Scratch of one workgroup: its event list, gap table, list of ops and (unless the ranks are given) rank table.
size_t ss_peaks_slot_bytes(const ss_gmg *g, const PeaksShape &s, bool given_ranks);
// Peaks and verdicts of nb candidates (placement rows P, finish rows of pitch
// fpitch; arr: rows of arrivals per predecessor edge, or null; given: ranks in
// dispatch order in candidate rows, or null for index order).  slots holds
// n_slots workgroups' scratch; ticket points to kTicketWords zeroed words.
int ss_launch_peaks(const ss_gmg *g, const PeaksShape &s, const uint8_t *P, const uint32_t *fin, int64_t fpitch,
                    const uint32_t *arr, uint16_t *given, void *slots, int64_t n_slots, int64_t nb, uint32_t *ticket,
                    int64_t *peak, uint8_t *violation, hipStream_t stream);

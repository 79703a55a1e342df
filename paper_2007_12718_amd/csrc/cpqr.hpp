// Device state of one CPQR row ID, shared by its launches (one per pivot).
// Host and device code; no other header needed.
#pragma once

#ifdef __HIPCC__
#define LSH_HOST_DEVICE __host__ __device__
#else
#define LSH_HOST_DEVICE
#endif

namespace lsh {

struct CpqrState {
  int k;        // the rank: min(rows, columns) until step j stops the loop, then j
  int done;     // (the host's read-back between batches of launches)
  double thr2;  // squared stopping threshold

  // Launch j's test at its entry.  Workgroup 0 of the launch that stops calls
  // stop(j) while other workgroups, and the wavefronts of one of them, may not
  // have made the test yet: it has to give them all the same answer.  k is the
  // full rank (above j) or j in launch j, so none leaves there, and below j in
  // every later launch, so all leave.  done would change under them: some
  // wavefronts of a workgroup would leave and the others reduce over LDS that
  // those never wrote.
  LSH_HOST_DEVICE bool over(int j) const { return k < j; }
  LSH_HOST_DEVICE void stop(int j) {
    k = j;
    done = 1;
  }
};

}  // namespace lsh

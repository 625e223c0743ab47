// Set-up of the file-scope scratch array behind helios_dedup_noalloc (noalloc.hip).
#pragma once

namespace helios {

// Looks up the address of the calling thread's current device's copy of the scratch array and keeps
// it for that device, filled and ready for the first call; helios_create calls it with the context's
// device current.  Waits for the stream the first time.  Returns a helios_status.
int noalloc_init(int device, hipStream_t stream);

}  // namespace helios

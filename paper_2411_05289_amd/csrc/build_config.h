// Which build of the kernels a translation unit holds.  The device code is written for a
// workgroup of MDSD_WG threads (kWaves = MDSD_WG / 64 wavefronts sharing one node) and lives in
// namespace MDSD_NS.  The library's main build is 512 threads in namespace mdsd; the files
// wave_verify.hip, pair_*.hip and quad_*.hip build the generic kernels again for 64, 128 and 256
// threads in namespaces of their own: fewer wavefronts per node, for rows that would leave most of a
// 512-thread workgroup without a part of them.
#pragma once

#ifndef MDSD_WG
#define MDSD_WG 512
#endif
#ifndef MDSD_NS
#define MDSD_NS mdsd
#endif
// slab sums a node keeps in LDS: bounds the vocabulary (64 chunks of 16 bytes per slab)
#ifndef MDSD_MAX_SLABS
#define MDSD_MAX_SLABS 2048
#endif

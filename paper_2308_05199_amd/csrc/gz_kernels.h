// gz_kernels.h -- launchers exported by gz_kernels.hip to the host runtime.
#pragma once
#include <hip/hip_runtime.h>

#include "gz_common.h"

namespace gzk {

// op: 0 compress, 1 decompress, 2 fused step, 3 decode-and-accumulate (2, 3:
// fp32 only)
hipError_t launch_single(uint32_t op, const Job& J, const Ctl& C, uint32_t tpb, uint32_t grid,
                         hipStream_t st);
// LDS one workgroup of tpb threads uses (wide: fp64 strips)
size_t lds_bytes(uint32_t wide, uint32_t tpb);
// op: as launch_single.  wide: the batch holds fp64 jobs (larger LDS staging).  d_strip_job: total
// (job, strip) pairs in ticket order, unused when njobs > 0 (njobs jobs of
// equal strip counts, interleaved round-robin).
hipError_t launch_batch(uint32_t op, const Job* d_jobs, const uint32_t* d_strip_job,
                        uint32_t njobs, uint32_t total, const Ctl& C, uint32_t tpb,
                        uint32_t grid, bool wide, hipStream_t st);
// Per-wave decoding of one fp32 stream (mode 0): every wave decodes whole
// superblocks, assigned statically; grid = min(CUs, superblocks per wave).
hipError_t launch_decompress_wave(const Job& J, const Ctl& C, uint32_t cus, hipStream_t st);
size_t wave_decode_lds();  // its workgroup's LDS bytes
size_t unit_decode_lds();
// Per-wave decode-and-accumulate of one fp32 stream (as launch_decompress_wave).
hipError_t launch_accum_wave(const Job& J, const Ctl& C, uint32_t cus, hipStream_t st);
// Batched decoding of fp32 1D jobs by shares: d_map holds jw (job, first
// superblock, stride) triples, one per wave's share of a job (its whole
// superblocks decoded as a pipeline).
hipError_t launch_decode_shares(const Job* d_jobs, const uint32_t* d_map, uint32_t jw,
                                uint32_t cus, const Ctl& C, hipStream_t st);
// Per-wave batched decode-and-accumulate (fp32): total superblocks, superblock
// i = (d_map[2i], d_map[2i+1]) as (job, superblock), or without a map (jobs of
// equal superblock counts) superblock i / njobs of job i % njobs.
hipError_t launch_accum_wave_batch(const Job* d_jobs, const uint32_t* d_map, uint32_t njobs,
                                   uint32_t total, uint32_t cus, const Ctl& C, hipStream_t st);
// Per-wave fused step of njobs fp32 jobs of the same superblock count and
// block length: every wave codes whole superblocks, a workgroup's waves the 8
// of a round (one look-back word); total = njobs * wave_rounds(NS), round
// ticket t = round t / njobs of job t % njobs.
hipError_t launch_fused_wave(const Job* d_jobs, uint32_t njobs, uint32_t total, uint32_t log2L,
                             const Ctl& C, uint32_t cus, hipStream_t st);
// The same of one stream: wave_rounds(J.NS) look-back words.
hipError_t launch_fused_wave_single(const Job& J, const Ctl& C, uint32_t cus, hipStream_t st);
constexpr uint64_t WAVE_ROUND = 8;  // superblocks per round
size_t wave_fused_lds();            // its workgroup's LDS bytes
inline uint64_t wave_rounds(uint64_t NS) { return (NS + WAVE_ROUND - 1) / WAVE_ROUND; }
// Unit encoding (op 0 compression of either type or of 8x8 tiles, op 2 the fp32
// fused step): every working wave codes units of 2048 elements, the `workers` of a
// workgroup (which has one wave more, the scheduler) a round of that many
// units (one look-back word).  J.nstrips = total rounds (unit_rounds).
hipError_t launch_unit(uint32_t op, const Job& J, const Ctl& C, uint32_t workers, uint32_t cus,
                       hipStream_t st);
// total rounds of njobs jobs of equal round counts (njobs > 0: round t is
// round t / njobs of job t % njobs) or of the (job, round) pairs of d_map;
// longest: rounds of the longest chain.
hipError_t launch_batch_unit(uint32_t op, const Job* d_jobs, const uint32_t* d_map,
                             uint32_t njobs, uint32_t total, bool wide, const Ctl& C,
                             uint32_t workers, uint32_t longest, uint32_t cus, hipStream_t st);
constexpr uint32_t UNIT_WORKERS = 15;        // most workers of a workgroup: compression
constexpr uint32_t UNIT_WORKERS_FUSED = 11;  // the fused step
constexpr uint64_t UNIT_ELEMS = 2048;
size_t unit_lds(bool fused, uint32_t workers);  // its workgroup's LDS bytes
// Workgroups a CU holds (16 waves, the fused step's 12).
inline uint32_t unit_per_cu(bool fused, uint32_t workers) {
  return ((fused ? UNIT_WORKERS_FUSED : UNIT_WORKERS) + 1) / (workers + 1);
}
inline uint64_t unit_rounds(uint64_t n, uint32_t workers) {  // an empty stream is one unit
  const uint64_t units = n ? (n + UNIT_ELEMS - 1) / UNIT_ELEMS : 1;
  return (units + workers - 1) / workers;
}
// Unit decoding of one stream (mode 0, either type, or 8x8 tiles), a wave per
// 2048 elements.
hipError_t launch_unit_decode(const Job& J, const Ctl& C, uint32_t cus, hipStream_t st);
// Unit decoding of a batch (mode 0, either type) of total superblocks, d_map
// and njobs as launch_accum_wave_batch.
hipError_t launch_batch_unit_decode(const Job* d_jobs, const uint32_t* d_map, uint32_t njobs,
                                    uint32_t total, uint32_t cus, const Ctl& C, hipStream_t st);
constexpr uint64_t DEC_WAVES_F32 = 8;  // waves per workgroup of the fp32 per-wave decoders
hipError_t launch_quantize(const void* x, uint64_t n, const Job& J, int32_t* q, uint8_t* fail,
                           hipStream_t st);
// mode 1 (8x8 tiles, fp32): op 0 compress, 1 decompress
hipError_t launch_tiles(uint32_t op, const Job& J, const Ctl& C, uint32_t tpb, uint32_t grid,
                        hipStream_t st);
hipError_t launch_tile_trial(const Job& J, int8_t* feat, uint32_t* sizes, uint8_t* label,
                             hipStream_t st);
hipError_t launch_reset(const Ctl& C, hipStream_t st);
// writes the sticky device status (a gz_status code) to *status, if given,
// and clears it
hipError_t launch_finish(const Ctl& C, uint32_t* status, hipStream_t st);
// Kernels of occupancy_blocks: ops 0-2 as launch_single, OCC_BATCH + k = batched
// op k (dtype 1: a batch with fp64), tile compress/decompress, single-stream
// decode-and-accumulate.
enum : uint32_t { OCC_BATCH = 3, OCC_TILE_C = 7, OCC_TILE_D = 8, OCC_ACCUM = 9 };
// resident workgroups per CU of a kernel
int occupancy_blocks(uint32_t op, uint32_t dtype, uint32_t log2L, uint32_t tpb);

}  // namespace gzk
